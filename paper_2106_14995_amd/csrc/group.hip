// group.hip -- kernels of the group solver (group_tron.hpp): one instance per group of G
// consecutive lanes, up to 64 / G instances per wavefront.
#include <hip/hip_runtime.h>

#include "group_tron.hpp"
#include "tron_internal.hpp"

template <class Fam, int N, int G, bool kTwin = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void group_kernel(LaneArgs a)
{
    using S = mt::GroupTron<Fam, N, G, kTwin>;
    bool own;  // the same in all lanes of a group
    const int64_t t = mt_wave_item((int)(threadIdx.x & 63) / S::X::kLanes, a.share, a.count, own);
    if (t < 0) return;
    const int64_t b = a.index ? (int64_t)a.index[t] : t;
    const int n = a.nper ? a.nper[b] : a.n_uniform;
    const int64_t po = a.poff ? a.poff[b] : b * (int64_t)a.psize;
    const int64_t vo = a.voff ? a.voff[b] : b * (int64_t)n;
    const int64_t t0 = a.ts ? (int64_t)wall_clock64() : 0;
    S s;
    s.n = n;
    s.set_lane((int)(threadIdx.x & (G - 1)));
    s.fam.load(s, a.params + po, n);
    const double *lo = a.lo + vo, *hi = a.hi + vo, *x0 = a.x0 + vo;
    MT_UNROLL for (int r = 0; r < S::R; r++) {
        const int i = s.row(r);
        const bool in = i < n;
        const int k = in ? i : 0;
        s.lo[r] = in ? lo[k] : Fam::pad;
        s.hi[r] = in ? hi[k] : Fam::pad;
        s.x[r] = in ? x0[k] : Fam::pad;
    }
    const double din = a.opt.warm ? a.state[b] : 0.0;
    const double ain = a.opt.warm ? a.state[a.batch + b] : 0.0;
    const int32_t st = s.solve(a.opt, din, ain);
    if (!own) return;
    double *xo = a.x + vo;
    MT_UNROLL for (int r = 0; r < S::R; r++)
        if (s.row(r) < n) xo[s.row(r)] = s.x[r];
    if (s.k == 0) {
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
}

template <class Fam, int N, int G>
static void launch_group(const LaneArgs &a, hipStream_t st)
{
    const int blk = a.lane_block == 64 ? 64 : 256;
    LaneArgs s = a;
    // The builds for n <= 16 spill, and every wavefront more brings its scratch traffic along: these
    // are spread over fewer. Quartics of n = 16, groups of 8, packed (before) / on up to 128 wavefronts / on
    // up to 1,024, rows of 16: 256 instances 541 / 419 / 494 us, 1,000 531 / 499 / 879; groups of
    // 16, packed / up to 256 / up to 1,024: 256 instances 270 / 214 / 215 us, 1,000 266 / 253 / 421.
    s.share = mt_wave_share(a.count, 64 / G, N <= 8 ? kSimds : G == 16 ? kSimds / 4 : kSimds / 8);
    const int64_t per = (int64_t)s.share.per * (blk / 64);
    const unsigned grid = (unsigned)((a.count + per - 1) / per);
    if (!grid) return;
    if constexpr (G == 8 && N <= 8) {
        // Up to four instances per wavefront (4,096 of them) groups of 8 leave half the lanes
        // without an instance: each group then takes a row of 16, where a broadcast is one
        // instruction (and rides on the products for N = 8). Measured, groups of 8 lanes against
        // rows of 16: 256 quartics of n = 8 36.8 / 31.6 us, of n = 5 35.5 / 30.5, HS45M of n = 8
        // 71.2 / 63.5, branches 25.6 / 23.7; 4,096: 47.0 / 40.0, 41.8 / 36.3, 100 / 86, 34.0 / 31.1.
        // With more instances it would take twice the wavefronts.
        if (s.share.per <= 4) {
            hipLaunchKernelGGL((group_kernel<Fam, N, 8, true>), dim3(grid), dim3(blk), 0, st, s);
            return;
        }
    }
    hipLaunchKernelGGL((group_kernel<Fam, N, G>), dim3(grid), dim3(blk), 0, st, s);
}

lane_launch_fn mt_group_launcher(tron_family fam, int N, int G)
{
    using namespace mt;
    if (fam == TRON_FAMILY_BR6 && N == 6) {
        if (G == 2) return launch_group<GBR6<2>, 6, 2>;
        if (G == 4) return launch_group<GBR6<4>, 6, 4>;
        if (G == 8) return launch_group<GBR6<8>, 6, 8>;
    }
    if (fam == TRON_FAMILY_QP4) {
        if (N == 8 && G == 2) return launch_group<GQP4<8, 2>, 8, 2>;
        if (N == 8 && G == 4) return launch_group<GQP4<8, 4>, 8, 4>;
        if (N == 8 && G == 8) return launch_group<GQP4<8, 8>, 8, 8>;
        if (N == 16 && G == 4) return launch_group<GQP4<16, 4>, 16, 4>;
        if (N == 16 && G == 8) return launch_group<GQP4<16, 8>, 16, 8>;
        if (N == 16 && G == 16) return launch_group<GQP4<16, 16>, 16, 16>;
    }
    if (fam == TRON_FAMILY_HS45M) {
        if (N == 8 && G == 2) return launch_group<GHS45M<8, 2>, 8, 2>;
        if (N == 8 && G == 4) return launch_group<GHS45M<8, 4>, 8, 4>;
        if (N == 8 && G == 8) return launch_group<GHS45M<8, 8>, 8, 8>;
        if (N == 16 && G == 8) return launch_group<GHS45M<16, 8>, 16, 8>;
        if (N == 16 && G == 16) return launch_group<GHS45M<16, 16>, 16, 16>;
    }
    return nullptr;
}
