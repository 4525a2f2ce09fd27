// The reports of a pseudo-time loop in mapped host memory: what the device writes
// and when the host may take it. Plain C++, so that the host's side can be checked
// without a GPU.
//
// Device writes to different lines of host memory can become visible out of order
// (a fence between them does not prevent it: a separate stop flag was read stale
// once in about 10^4 loops, which ended the loop there). So a report is one line
// that carries its own proof of being complete, and whatever the host reads beside
// it is named in the report.
#pragma once

#include <stdint.h>
#include <string.h>

#if defined(__HIPCC__)
#define DTSPH_BOTH __host__ __device__
#else
#define DTSPH_BOTH
#endif

namespace dtsph {

// Build flag words
enum Flag { F_NBR_OVERFLOW = 0, F_NBR_NEEDED = 1, F_CELL_OVERFLOW = 2, F_OUTSIDE = 3, F_SKIN = 4, F_COUNT = 5 };

struct alignas(64) MirrorRep {
    double rp_mean, rv_mean, rp_max, rv_max, disp;
    long long pairs;
    int iters;
    uint32_t state;   // bits 0..7 stop reason, 8 stopped, 16.. build flags moved to host memory (move_build_flags)
    uint32_t seq;     // the sim's count of published reports
    uint32_t check;   // report_check of the 15 words before it
};
static_assert(sizeof(MirrorRep) == 64, "one line");

DTSPH_BOTH inline uint32_t report_check(const uint32_t w[16])
{
    uint32_t h = 0x2545f491u;
    for (int k = 0; k < 15; ++k) h = (h ^ w[k]) * 0x9e3779b1u + (h >> 15);
    return h;
}

// Moves the build flags that are set to host memory. Returns the bits of all flags
// moved since the host last cleared them (kept in *moved): the host may take a later
// report than the one they came with, which then names them too.
DTSPH_BOTH inline uint32_t move_build_flags(int *flags, int *h_flags, uint32_t *moved)
{
    uint32_t m = *moved;
    int f[F_COUNT], any = 0;  // all loads at once: the report waits for them
    for (int k = 0; k < F_COUNT; ++k) any |= f[k] = flags[k];
    if (!any) return m;
    for (int k = 0; k < F_COUNT; ++k)
        if (f[k]) {
            h_flags[k] = f[k];
            flags[k] = 0;
            m |= 1u << k;
        }
    *moved = m;
    return m;
}

// Takes the report in `line` into r if it is complete, is that of the publishing
// launch with sequence number `want` or a later one, and the build flags that it
// names have arrived.
inline bool accept_report(const volatile uint32_t *line, const volatile int *flags, int want, MirrorRep &r)
{
    if ((int)(line[14] - (uint32_t)want) < 0) return false;
    uint32_t w[16];
    for (int k = 0; k < 16; ++k) w[k] = line[k];
    if (w[15] != report_check(w) || (int)(w[14] - (uint32_t)want) < 0) return false;
    memcpy(&r, w, sizeof r);
    for (int k = 0; k < F_COUNT; ++k)
        if (((r.state >> (16 + k)) & 1u) && !flags[k]) return false;
    return true;
}

// The largest particle shift of a step: a line of its own, with the number of its
// launch.
struct alignas(16) ShiftRep {
    double most;
    uint32_t seq, check;
};

DTSPH_BOTH inline void shift_words(uint32_t w[4], double most, uint32_t seq)
{
    uint64_t b;
    memcpy(&b, &most, 8);
    w[0] = (uint32_t)b;
    w[1] = (uint32_t)(b >> 32);
    w[2] = seq;
    w[3] = ((w[0] * 0x9e3779b1u ^ w[1]) * 0x85ebca77u ^ seq) * 0xc2b2ae3du + 0x2545f491u;
}

// Takes the largest shift in `line` if it is complete and that of launch `want` or a
// later one.
inline bool accept_shift(const volatile uint32_t *line, int want, double &most)
{
    uint32_t w[4], full[4];
    for (int k = 0; k < 4; ++k) w[k] = line[k];
    double m;
    memcpy(&m, w, 8);
    shift_words(full, m, w[2]);
    if (w[3] != full[3] || (int)(w[2] - (uint32_t)want) < 0) return false;
    most = m;
    return true;
}

}  // namespace dtsph
