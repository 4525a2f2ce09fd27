// Launches of the pair pass (device code: dtsph_pass_dev.h) for one pass type and
// dimension. The kernel has many variants (walls, artificial viscosity,
// regularisers, lanes per particle, advective sums, coefficient cache), so the
// build compiles this file once per (DTSPH_PAIR_T, DTSPH_PAIR_DIM), in parallel.
#include <hip/hip_ext.h>

#include "dtsph_pass_dev.h"

#if !defined(DTSPH_PAIR_T) || !defined(DTSPH_PAIR_DIM)
#error "compile with -DDTSPH_PAIR_T=float|double -DDTSPH_PAIR_DIM=2|3"
#endif

namespace dtsph {

namespace {

// A timed pair pass goes through hipExtLaunchKernelGGL, whose events take the
// kernel's own start and end timestamps (no queue gaps in the interval).
// Pseudo-iterations of a context with steady sims take the variant with the
// convective sum (zero coefficient for the time-accurate sims).
template <typename T, int DIM, bool WALLS, bool AV, bool SEPDEN, int LPP, bool CONV, int CACHE, bool MOVE = false>
void launch_pseudo(Ctx &c, const PassArgs<T> &a, dim3 grid)
{
    if (c.ext_start)
        hipExtLaunchKernelGGL((k_pass<T, DIM, WALLS, AV, SEPDEN, MODE_PSEUDO, LPP, CONV, CACHE, MOVE>), grid,
                              dim3(c.block), 0, c.stream, c.ext_start, c.ext_stop, 0, a);
    else
        DTSPH_LAUNCH(c, (k_pass<T, DIM, WALLS, AV, SEPDEN, MODE_PSEUDO, LPP, CONV, CACHE, MOVE>), grid,
                     dim3(c.block), 0, c.stream, a);
}

// Cached pair coefficients hold one regulariser: contexts with separate EDAC
// or artificial-viscosity regularisers always recompute.
template <typename T, int DIM, bool WALLS, bool AV, bool SEPDEN, int LPP, bool CONV>
void dispatch_pseudo(Ctx &c, const PassArgs<T> &a, dim3 grid)
{
    if (SEPDEN || c.cache_phase == 0) launch_pseudo<T, DIM, WALLS, AV, SEPDEN, LPP, CONV, 0>(c, a, grid);
    else if (c.cache_phase == 1) launch_pseudo<T, DIM, WALLS, AV, false, LPP, CONV, 1>(c, a, grid);
    else launch_pseudo<T, DIM, WALLS, AV, false, LPP, CONV, 2>(c, a, grid);
}

template <typename T, int DIM, bool WALLS, bool AV, bool SEPDEN, int LPP>
void dispatch_mode(Ctx &c, int mode, const PassArgs<T> &a, dim3 grid)
{
    if (mode == MODE_PRE)
        DTSPH_LAUNCH(c, (k_pass<T, DIM, WALLS, AV, SEPDEN, MODE_PRE, LPP, false>), grid, dim3(c.block), 0, c.stream,
                     a);
    else if (c.any_move)  // moving particles: advective sums, no coefficient cache
        launch_pseudo<T, DIM, WALLS, AV, SEPDEN, LPP, true, 0, true>(c, a, grid);
    else if (c.any_steady)
        dispatch_pseudo<T, DIM, WALLS, AV, SEPDEN, LPP, true>(c, a, grid);
    else
        dispatch_pseudo<T, DIM, WALLS, AV, SEPDEN, LPP, false>(c, a, grid);
}

template <typename T, int DIM, bool WALLS, bool AV, bool SEPDEN>
void dispatch_lpp(Ctx &c, int mode, const PassArgs<T> &a, dim3 grid)
{
    switch (c.lpp) {
    case 1: dispatch_mode<T, DIM, WALLS, AV, SEPDEN, 1>(c, mode, a, grid); break;
    case 2: dispatch_mode<T, DIM, WALLS, AV, SEPDEN, 2>(c, mode, a, grid); break;
    case 4: dispatch_mode<T, DIM, WALLS, AV, SEPDEN, 4>(c, mode, a, grid); break;
    default: dispatch_mode<T, DIM, WALLS, AV, SEPDEN, 8>(c, mode, a, grid); break;
    }
}

template <typename T, int DIM, bool WALLS, bool AV>
void dispatch_sep(Ctx &c, int mode, const PassArgs<T> &a, dim3 grid)
{
    if (c.sep_den) dispatch_lpp<T, DIM, WALLS, AV, true>(c, mode, a, grid);
    else dispatch_lpp<T, DIM, WALLS, AV, false>(c, mode, a, grid);
}

template <typename T, int DIM, bool WALLS>
void dispatch_av(Ctx &c, int mode, const PassArgs<T> &a, dim3 grid)
{
    if (c.any_av) dispatch_sep<T, DIM, WALLS, true>(c, mode, a, grid);
    else dispatch_sep<T, DIM, WALLS, false>(c, mode, a, grid);
}

template <typename T, int DIM>
void dispatch_walls(Ctx &c, int mode, const PassArgs<T> &a, dim3 grid)
{
    if (c.any_walls) dispatch_av<T, DIM, true>(c, mode, a, grid);
    else dispatch_av<T, DIM, false>(c, mode, a, grid);
}

}  // namespace

template <>
void launch_pass_dim<DTSPH_PAIR_T, DTSPH_PAIR_DIM>(Ctx &c, int mode, bool cand_lists)
{
    using T = DTSPH_PAIR_T;
    PassArgs<T> a = pass_args<T>(c, mode, cand_lists);
    if (a.n_tiles == 0) return;
    const int grid = c.xcd_remap ? 8 * ((a.n_tiles + 7) / 8) : a.n_tiles;
    const int t0 = mode == MODE_PSEUDO ? timer_slot(c, 0) : -1;
    if (t0 >= 0) {
        c.ext_start = c.ev_pool[t0];
        c.ext_stop = c.ev_pool[t0 + 1];
    }
    dispatch_walls<T, DTSPH_PAIR_DIM>(c, mode, a, dim3(grid));
    c.ext_start = c.ext_stop = nullptr;
    DTSPH_HIP_CHECK(hipGetLastError());
    timer_book(c, t0, 0);
}

}  // namespace dtsph
