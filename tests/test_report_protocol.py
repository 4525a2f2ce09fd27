"""When the host may take a report from mapped memory (csrc/dtsph_report.h): a C++
driver plays the device, whose writes to different lines arrive in any order. A
report is taken only when it is whole and not older than the one waited for, and
an error flag moved with an earlier report of the same loop is waited for also
when only a later report is seen. The largest shift of a step has the same proof."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1904_00861_amd", "csrc")

DRIVER = r"""
#include "dtsph_report.h"
#include <stdio.h>
using namespace dtsph;

static int fails = 0;
#define EXPECT(e) do { if (!(e)) { printf("line %d: %s\n", __LINE__, #e); ++fails; } } while (0)

// The device: flags, and what it has written (in flight until delivered).
struct Device {
    int flags[F_COUNT] = {};
    uint32_t moved = 0, seq = 0;
    int out_flags[F_COUNT] = {};
    uint32_t out_line[16] = {};
    void publish(int iters, bool done)
    {
        MirrorRep r{};
        r.iters = iters;
        r.pairs = 1234567890123ll + iters;
        r.rp_mean = 0.5 / iters;
        r.state = 1u | (done ? 256u : 0u) | (move_build_flags(flags, out_flags, &moved) << 16);
        r.seq = ++seq;
        memcpy(out_line, &r, 64);
        out_line[15] = report_check(out_line);
    }
};
// The host's memory.
struct Host {
    int flags[F_COUNT] = {};
    uint32_t line[16] = {};
    void line_arrives(const Device &d, int from = 0, int to = 16)
    {
        for (int k = from; k < to; ++k) line[k] = d.out_line[k];
    }
    void flag_arrives(const Device &d, int k) { flags[k] = d.out_flags[k]; }
    bool take(int want, MirrorRep &r) { return accept_report(line, flags, want, r); }
};

int main()
{
    MirrorRep r;
    {   // nothing there, then a report in two halves in either order, then a newer one
        Device d;
        Host h;
        EXPECT(!h.take(1, r));
        d.publish(2, false);
        h.line_arrives(d, 8, 16);
        EXPECT(!h.take(1, r));
        h.line_arrives(d, 0, 8);
        EXPECT(h.take(1, r) && r.iters == 2 && r.pairs == 1234567890125ll && !(r.state & 256u));
        EXPECT(!h.take(2, r));
        d.publish(4, true);
        h.line_arrives(d, 0, 8);
        EXPECT(!h.take(1, r) && !h.take(2, r));  // torn: neither the old nor the new one
        h.line_arrives(d);
        EXPECT(h.take(1, r) && h.take(2, r) && r.iters == 4 && (r.state & 256u));
    }
    for (int f = 0; f < F_COUNT; ++f) {
        // two groups in flight: the flag moves with the first report, the host sees the
        // second report's line before the flag
        Device d;
        Host h;
        d.flags[f] = 17;
        d.publish(2, false);
        d.publish(4, false);
        h.line_arrives(d);
        EXPECT(!h.take(1, r) && !h.take(2, r));
        h.flag_arrives(d, f);
        EXPECT(h.take(1, r) && ((r.state >> 16) & (1u << f)) && h.flags[f] == 17);
        // a second flag, moved with a report of its own, is named beside the first
        const int g = (f + 1) % F_COUNT;
        d.flags[g] = 5;
        d.publish(6, true);
        d.publish(8, true);
        h.line_arrives(d);
        EXPECT(!h.take(3, r));
        h.flag_arrives(d, g);
        EXPECT(h.take(3, r) && (r.state >> 16) == ((1u << f) | (1u << g)));
        // the host has taken and cleared everything (k_publish forgets what was moved)
        for (int k = 0; k < F_COUNT; ++k) h.flags[k] = 0;
        d.moved = 0;
        d.publish(1, false);
        h.line_arrives(d);
        EXPECT(h.take(5, r) && (r.state >> 16) == 0);
    }
    // the count of reports wraps
    {
        Device d;
        Host h;
        d.seq = 0x7fffffffu;
        d.publish(1, false);
        h.line_arrives(d);
        EXPECT(h.take((int)0x80000000u, r) && h.take(0x7fffffff, r) && !h.take((int)0x80000001u, r));
    }
    {   // the largest shift: whole, and not an earlier launch's
        uint32_t line[4] = {}, w[4];
        double m = -1;
        EXPECT(!accept_shift(line, 1, m));
        shift_words(w, 0.0, 1);
        for (int k = 0; k < 4; ++k) line[k] = w[k];
        EXPECT(accept_shift(line, 1, m) && m == 0.0 && !accept_shift(line, 2, m));
        shift_words(w, 0.75, 2);
        for (int half = 0; half < 2; ++half) {
            uint32_t torn[4] = {line[0], line[1], line[2], line[3]};
            for (int k = 0; k < 2; ++k) torn[2 * half + k] = w[2 * half + k];
            EXPECT(!accept_shift(torn, 1, m) && !accept_shift(torn, 2, m));
        }
        EXPECT(accept_shift(w, 2, m) && m == 0.75 && accept_shift(w, 1, m));
    }
    printf(fails ? "%d checks failed\n" : "all checks passed\n", fails);
    return fails != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_reports_are_taken_whole_with_their_flags(tmp_path):
    src, exe = tmp_path / "reports.cpp", tmp_path / "reports"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stdout
