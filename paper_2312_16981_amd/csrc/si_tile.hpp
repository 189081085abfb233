// The 1-D source iteration in tiles (si_tile.hip): rounds of several sweeps
// per launch.  Shared with the commit (kernels.hip), which reads the iterate
// the iteration converged to.
//
// A launch ("round") takes up to K.tile_S sweeps.  A block holds a tile of
// consecutive cells: K.tile_H cells on either side of its interior are
// computed along (fewer each sweep), so that no block waits for another.  The
// number of sweeps is known only once the whole instance's residuals are, so
// every sweep of a round keeps its output; the sweep at which the step before
// converged writes where the step's result belongs (rho_new, phi0n, T_new), so
// that the commit has nothing to copy when this step takes as many.
#pragma once
#include <hip/hip_runtime.h>
#include "common.hpp"
#include "device_common.hpp"

namespace ugk {

// The rounds of a step whose predecessor took `prev` sweeps (0: none yet): sweeps of
// round 0 and of round 1 (a batch's ends where its instance's iteration ended before, a
// single instance's rounds are planned so by the host), S after; and the sweep whose
// output is written in place.
struct TilePlan {
    int s0, s1, fin;
};
__device__ inline TilePlan tile_plan(const Consts& K, int prev)
{
    TilePlan p;
    p.s0 = min(prev > 0 ? min(prev + K.tile_extra, K.tile_S) : K.tile_S, K.si_max);
    p.s1 = K.n_inst > 1 && prev > p.s0 ? min(prev - p.s0, K.tile_S) : K.tile_S;
    p.fin = (prev > 0 ? prev : p.s0) - 1;
    return p;
}

// First sweep and number of sweeps of a round, within the iteration's limit.
struct TileRound {
    int k0, ns;
};
__device__ inline TileRound tile_round(const Consts& K, const TilePlan& p, int round)
{
    TileRound r;
    r.k0 = round == 0 ? 0 : p.s0 + (round == 1 ? 0 : p.s1 + (round - 2) * K.tile_S);
    const int most = round == 0 ? p.s0 : (round == 1 ? p.s1 : K.tile_S);
    r.ns = max(0, min(most, K.si_max - r.k0));
    return r;
}

// Where the output of the iteration's sweep k lies: `final` (rho_new, phi0n,
// T_new, uend) or plane `at` of the sweep arrays.
struct TileOut {
    bool final;
    int at;
};
__device__ inline TileOut tile_out(const Consts& K, const TilePlan& p, int k)
{
    TileOut o;
    o.final = k == p.fin;
    if (k < p.s0) o.at = k;
    else if (k < p.s0 + p.s1) o.at = K.tile_cap + k - p.s0;
    else {
        const int q = k - p.s0 - p.s1, round = 2 + q / K.tile_S;
        o.at = (round & 1) * K.tile_cap + q % K.tile_S;
    }
    return o;
}

// Boundary wave inflow of a sweep whose wave flux follows the iterate, by plane (the
// last one: the sweep whose output lies in place): the low cell's groups, then the high cell's.
__device__ inline double* tile_inflow(const Dev& D, const Consts& K, int inst, int at)
{
    return D.winflow + ((int64_t)at * K.n_inst + inst) * 2 * MAX_G;
}

// Residual entries of a round, one per sweep and block: no atomics, nothing to clear.
__device__ inline Resid* tile_res(const Dev& D, const Consts& K, int round, int m)
{
    return D.tile_res + ((int64_t)(round & 1) * K.tile_cap + m) * K.tile_blocks;
}

// The maxima of a sweep's entries b, b + step, .. below b1, for one thread.
__device__ inline Resid tile_most(const Dev& D, const Consts& K, int round, int m, int b, int b1, int step)
{
    const Resid* res = tile_res(D, K, round, m);
    Resid x = {0ull, 0ull, 0ull, 0ull};
    for (; b < b1; b += 4 * step) {
        Resid y[4];            // four entries in flight
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            y[q] = Resid{0ull, 0ull, 0ull, 0ull};
            if (b + q * step < b1) y[q] = res[b + q * step];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            x.drho = max(x.drho, y[q].drho);
            x.rho = max(x.rho, y[q].rho);
            x.dT = max(x.dT, y[q].dT);
            x.T = max(x.T, y[q].T);
        }
    }
    return x;
}

// The maxima over a wavefront's lanes.
__device__ inline Resid tile_wave_most(const Resid& x)
{
    return {wave_max_bits(bitsd(x.drho)), wave_max_bits(bitsd(x.rho)), wave_max_bits(bitsd(x.dT)), wave_max_bits(bitsd(x.T))};
}

// The stopping test of a sweep from its maxima: 1 converged, 0 not, -1 a temperature was
// non-positive or not finite.
__device__ inline int tile_verdict(const Consts& K, const Resid& x)
{
    const double drho = bitsd(x.drho), mrho = bitsd(x.rho), dT = bitsd(x.dT), mT = bitsd(x.T);
    if (mT != mT) return -1;
    return drho <= K.si_tol * mrho && dT <= K.si_tol * mT ? 1 : 0;
}

// The test by a wavefront, from its blocks' entries b0 .. b1-1.
__device__ inline int tile_test(const Dev& D, const Consts& K, int round, int m, int b0, int b1, int lane)
{
    return tile_verdict(K, tile_wave_most(tile_most(D, K, round, m, b0 + lane, b1, WAVE)));
}

// The outcome after a round for the only instance of a context, taken by every
// thread of a block alike (for many tiles, K.tile_fold = 0, read only), in two parts: tile_gather tests every plane of the round
// (a wavefront per plane; without waiting for the number of sweeps it took, so that
// its loads go out with the kernel's first) and reads the recorded state once per
// block (block 0 of the launch may record it meanwhile); after a barrier tile_outcome
// gives the sweeps the iteration took when it converged, -1 when a temperature
// failed first, 0 to go on.  sh: TILE_S_MAX + 1 words.
__device__ inline void tile_gather(const Dev& D, const Consts& K, int round, int* sh)
{
    if (threadIdx.x == 0) sh[TILE_S_MAX] = D.ist[0].conv_sweeps;
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
    for (int m = wid; m < K.tile_fold; m += nw) {
        const int v = tile_test(D, K, round, m, 0, K.tile_blocks, lane);
        if (lane == 0) sh[m] = v;
    }
}

__device__ inline int tile_outcome(const Consts& K, int round, const TilePlan& p, const int* sh)
{
    int out = sh[TILE_S_MAX];
    if (out != 0) return out;          // recorded by an earlier launch or just now
    const TileRound q = tile_round(K, p, round);
    for (int m = min(q.ns, K.tile_fold) - 1; m >= 0; --m) {
        const int v = sh[m];
        if (v != 0) out = v > 0 ? q.k0 + m + 1 : -1;
    }
    return out;
}

// Record the outcome of the iteration (block 0 of a single instance's launch, or
// a decide kernel): the sweep count, or the failed temperature.
__device__ inline void tile_record(const Dev& D, int inst, int out)
{
    D.ist[inst].conv_sweeps = out;
    if (out > 0) atomicAdd((unsigned long long*)(D.counters + CNT_CONV), 1ull);
    else atomicOr((unsigned long long*)(D.counters + CNT_ERR), ERR_TEMP);
}

}  // namespace ugk
