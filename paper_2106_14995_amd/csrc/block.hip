// block.hip -- the workgroup-per-instance solve kernels (block_tron.hpp) of the quartic family.
#include "block_tron.hpp"
#include "tron_internal.hpp"

namespace {

template <int R, int W, bool kGlobal>
__global__ __launch_bounds__(64 * W) void block_kernel(LaneArgs a, int64_t first)
{
    extern __shared__ double block_smem[];
    const int64_t t = first + blockIdx.x;
    if (t >= a.count) return;
    const int64_t b = a.index ? (int64_t)a.index[t] : t;
    const int n = a.nper ? a.nper[b] : a.n_uniform;
    const int64_t po = a.poff ? a.poff[b] : b * (int64_t)a.psize;
    const int64_t vo = a.voff ? a.voff[b] : b * (int64_t)n;
    const int64_t t0 = a.ts ? (int64_t)wall_clock64() : 0;
    using Solver = mt::BlockTron<R, W, kGlobal>;
    Solver s;
    s.n = n;
    s.lane = threadIdx.x & 63;
    s.k.ld = (n + 1) | 1;
    // the workspace form reads whole 128-byte lines where the slot has room for rows of an odd
    // number of them (odd, so that a column walk changes memory channels)
    if (kGlobal && (int64_t)n * mt_block_ld(n) <= a.ws_stride) s.k.ld = mt_block_ld(n);
    s.k.w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    s.k.L0 = (mt::lds_double *)block_smem;
    if constexpr (kGlobal) s.k.M = (mt::glb_double *)(a.ws + t * a.ws_stride);
    else s.k.M = s.k.L0 + Solver::oU;
    s.load(a.params + po, a.lo + vo, a.hi + vo, a.x0 + vo);
    const double din = a.opt.warm ? a.state[b] : 0.0;
    const double ain = a.opt.warm ? a.state[a.batch + b] : 0.0;
    const int32_t st = s.solve(a.opt, din, ain);
    __syncthreads();  // every wave has read its inputs: x0 and x may be one buffer
    if (s.k.w != 0) return;
    double *xo = a.x + vo;
    MT_UNROLL for (int r = 0; r < R; r++)
        if (s.valid(r)) xo[s.row(r)] = s.x[r];
    if (s.lane == 0) {
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

// a launch may not have 2^32 threads
constexpr int64_t kMostGroups = 1 << 22;

template <int R, int W, bool kGlobal>
void launch(const LaneArgs &a, int nmax, hipStream_t st)
{
    const size_t lds = mt::BlockTron<R, W, kGlobal>::lds_bytes(nmax);
    for (int64_t first = 0; first < a.count; first += kMostGroups) {
        const int64_t left = a.count - first, groups = left < kMostGroups ? left : kMostGroups;
        hipLaunchKernelGGL((block_kernel<R, W, kGlobal>), dim3((unsigned)groups), dim3(64 * W), lds, st, a, first);
    }
}

template <int R, int W, bool kGlobal>
void prepare()
{
    (void)hipFuncSetAttribute((const void *)block_kernel<R, W, kGlobal>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)mt::BlockTron<R, W, kGlobal>::lds_bytes(64 * R));
}

}  // namespace

void mt_launch_block(const LaneArgs &a, int nmax, hipStream_t st)
{
    if (a.count <= 0) return;
    if (nmax <= kLdsMaxN) launch<2, 8, false>(a, nmax, st);
    else if (nmax <= 256) launch<4, 8, true>(a, nmax, st);
    else launch<8, 8, true>(a, nmax, st);
}

size_t mt_block_lds_bytes(int nmax)
{
    if (nmax <= kLdsMaxN) return mt::BlockTron<2, 8, false>::lds_bytes(nmax);
    return nmax <= 256 ? mt::BlockTron<4, 8, true>::lds_bytes(nmax) : mt::BlockTron<8, 8, true>::lds_bytes(nmax);
}

void mt_prepare_block_kernels()
{
    prepare<2, 8, false>();
    prepare<4, 8, true>();
    prepare<8, 8, true>();
}
