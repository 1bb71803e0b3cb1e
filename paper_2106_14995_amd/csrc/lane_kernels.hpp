// lane_kernels.hpp -- the lane-per-instance solve kernel (n <= 8): one instance per lane of
// 64- or 256-lane workgroups, the solver state in registers (lane_tron.hpp).
#pragma once

#include "lane_tron.hpp"
#include "tron_internal.hpp"

// The largest workgroup a plan selects (64 is the default). The launch bound caps the size
// the kernel accepts; with one wave per SIMD either way, the register budget is the same.
constexpr int kLaneBlock = 256;

// Solve instance b in the calling lane; own: store its results (else the lane repeats another's).
template <class F, int N>
__device__ __forceinline__ void lane_solve(const LaneArgs &a, int64_t b, bool own)
{
    const int n = a.nper ? a.nper[b] : a.n_uniform;
    const int64_t po = a.poff ? a.poff[b] : b * (int64_t)a.psize;
    const int64_t vo = a.voff ? a.voff[b] : b * (int64_t)n;
    const int64_t t0 = a.ts ? (int64_t)wall_clock64() : 0;
    mt::LaneTron<F, N> s;
    s.fam.load(a.params + po, n);
    const double *lo = a.lo + vo, *hi = a.hi + vo, *x0 = a.x0 + vo;
    MT_UNROLL for (int i = 0; i < N; i++) {
        const bool in = i < n;
        const int k = in ? i : 0;
        s.lo[i] = in ? lo[k] : F::pad;
        s.hi[i] = in ? hi[k] : F::pad;
        s.x[i] = in ? x0[k] : F::pad;
    }
    const double din = a.opt.warm ? a.state[b] : 0.0;
    const double ain = a.opt.warm ? a.state[a.batch + b] : 0.0;
    const int32_t st = s.solve(a.opt, din, ain);
    if (!own) return;
    double *xo = a.x + vo;
    MT_UNROLL for (int i = 0; i < N; i++)
        if (i < n) xo[i] = s.x[i];
    a.f[b] = s.f;
    a.status[b] = st;
    a.iters[b] = s.iters;
    a.state[b] = s.delta;
    a.state[a.batch + b] = s.alphac;
    if (a.ts) {
        a.ts[2 * b] = t0;
        a.ts[2 * b + 1] = (int64_t)wall_clock64();
    }
}

template <class F, int N>
__global__ __launch_bounds__(kLaneBlock) void lane_kernel(LaneArgs a)
{
    bool own;
    const int64_t t = mt_wave_item((int)threadIdx.x & 63, a.share, a.count, own);
    if (t < 0) return;
    lane_solve<F, N>(a, a.index ? (int64_t)a.index[t] : t, own);
}

template <class F, int N>
static void launch_lane(const LaneArgs &a, hipStream_t st)
{
    const int blk = a.lane_block == 64 ? 64 : kLaneBlock;
    LaneArgs s = a;
    // The branch solve is short (3.5 iterations) and its first pass over the code and the
    // parameters' loads are much of it, so it goes on one wave per CU rather than per SIMD, and
    // not apart at all once a quarter of the lanes of those would have an own instance. Measured,
    // packed / a wave per CU / per SIMD: 1,500 instances 48.8 / 47.3 / 49.0 us; 4,096 50.6 / 49.3 /
    // 51.2; 9,000 50.6 / 51.8 / 52.8.
    const int waves = F::kSpread ? kSimds : a.count <= 16 * (kSimds / 4) ? kSimds / 4 : 1;
    s.share = mt_wave_share(a.count, 64, waves);
    const int64_t per = (int64_t)s.share.per * (blk / 64);
    const unsigned grid = (unsigned)((a.count + per - 1) / per);
    const size_t lds = sizeof(double) * (size_t)F::kLdsDoubles * (size_t)blk;
    if (grid) hipLaunchKernelGGL((lane_kernel<F, N>), dim3(grid), dim3(blk), lds, st, s);
}
