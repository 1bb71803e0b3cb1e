// tron_internal.hpp -- declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lane_tron.hpp"
#include "tron.h"

// instances per wavefront, and ceil(2^16 / per)
struct WaveShare {
    int32_t per, inv;
};

// Arguments of the solve kernels.
struct LaneArgs {
    const double *params, *lo, *hi, *x0;
    double *x, *f;
    int32_t *status, *iters;
    double *state;           // radius [batch], Cauchy step [batch]
    const int32_t *index;    // instance list of this bucket, or null (all, in order)
    const int32_t *nper;     // per-instance n, or null (n_uniform)
    const int64_t *poff, *voff;
    int64_t *ts;             // optional: per-instance start / end device clock (2 per instance)
    int64_t count, batch;
    int32_t n_uniform, psize;
    int32_t lane_block;      // workgroup size of the lane kernels (64 or 256; 0 means 256)
    WaveShare share;         // lane and group kernels: instances per wavefront (mt_wave_share)
    mt::Options opt;
    double *ws;              // n > 128: per-instance matrix workspace in global memory (or null)
    int64_t ws_stride;       // doubles per instance in ws (bucket slot t uses ws + t stride)
};

// Largest n of any family with a wave kernel; n in (kLdsMaxN, kMaxN] keeps its matrices in a
// global-memory workspace instead of LDS.
constexpr int kLdsMaxN = 128;
constexpr int kMaxN = 512;
// doubles of one instance's matrix array for bucket size nmax (n rows, odd stride > n)
__host__ __device__ inline int64_t mt_wave_matrix_doubles(int nmax) { return (int64_t)nmax * (int64_t)((nmax + 1) | 1); }

// Row stride of the workspace form: an odd number of 16-double lines.
__host__ __device__ inline int mt_block_ld(int n) { return 16 * (((n + 15) / 16) | 1); }
// doubles of a workspace slot that holds it; a slot of mt_wave_matrix_doubles works as well, with
// the stride (n + 1) | 1
__host__ __device__ inline int64_t mt_block_slot_doubles(int nmax) { return (int64_t)nmax * mt_block_ld(nmax); }

// Instances per wavefront of the kernels that hold several (at most `most`: 64 lanes or 64 / G
// groups): as many as leave every SIMD of the card one wavefront (or `waves` in all), so that a batch too small to
// fill the card is spread instead of packed. A wavefront runs every branch that any of its
// instances takes and lasts as long as its slowest one, so fewer instances end sooner; more
// than one wavefront per SIMD does not pay (the branch solves of 16,384 instances: 54 us at one,
// 80 at two; of 8,192 quartics of n = 6: 63 and 94).
// The lanes that this leaves without an instance repeat one (mt_wave_item): a CU whose
// wavefronts execute with 32 or fewer active lanes together issues about one wavefront's
// instructions at a time, whatever the instruction (a chain of multiply-adds on 256 x 4
// wavefronts: 42 us with 9 or more lanes active in each, 147 with 8; on 256 x 1: 42 with 33,
// 54 with 32), and the repetition keeps all 64 active. Measured, packed -> spread with idle
// lanes -> spread with repeating ones: 256 quartics of n = 8 in groups of 8 lanes
// 60 -> 59 -> 52 us; 1,000 of n = 6 65 -> 89 -> 58; 512 multiplier loops 832 -> 676 -> 533,
// 16,384 1,340 -> 1,500 -> 1,210; 25 ADMM iterations on 3,000 branches 834 -> 1,400 -> 790.
constexpr int kSimds = 1024;
inline WaveShare mt_wave_share(int64_t count, int most, int waves = kSimds)
{
    int64_t per = (count + waves - 1) / waves;
    per = per < 1 ? 1 : per < most ? per : most;
    return {(int32_t)per, (int32_t)((65535 + per) / per)};
}
// The instance (of `count`) that lane or group l of the calling wavefront solves; own: it is the
// one that stores the results; without an own instance it repeats one of its wavefront's. -1: the
// wavefront has none (the last workgroup's).
__device__ __forceinline__ int64_t mt_wave_item(int l, WaveShare s, int64_t count, bool &own)
{
    const int64_t first = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * s.per;
    const int64_t t = first + (l - s.per * ((l * s.inv) >> 16));  // l mod per, exact for l < 64
    own = l < s.per && t < count;
    return t < count ? t : first < count ? first : -1;
}

typedef void (*lane_launch_fn)(const LaneArgs &, hipStream_t);

// Launch the BR6 lane kernel (n = 6) over a.count instances.
void mt_launch_br6(const LaneArgs &a, hipStream_t st);
// Let the BR6 lane kernel take the LDS of its largest workgroup (once per process and device).
void mt_prepare_br6();
// The lane kernel for (family, N <= 8), or null when unsupported.
lane_launch_fn mt_lane_launcher(tron_family fam, int N);
// The wavefront-per-instance kernel of the family (QP4 or HS45M) for instances with
// n <= nmax (nmax <= kLdsMaxN: LDS sized for nmax; larger nmax: a.ws must hold a.count
// slots of a.ws_stride >= mt_wave_matrix_doubles(nmax) doubles).
void mt_launch_wave(tron_family fam, const LaneArgs &a, int nmax, hipStream_t st);
// The workgroup-per-instance kernel of the quartic family for n <= nmax (nmax <= kLdsMaxN: LDS
// sized for nmax; larger nmax: a.ws as above), and the LDS bytes of one instance.
void mt_launch_block(const LaneArgs &a, int nmax, hipStream_t st);
size_t mt_block_lds_bytes(int nmax);
void mt_prepare_block_kernels();
// LDS bytes of one instance of a bucket of `count` instances with n <= nmax (nmax <= kLdsMaxN), on
// whichever kernel mt_launch_wave gives the bucket.
size_t mt_wave_lds_bytes(tron_family fam, int nmax, int64_t count);
// Make the wave kernels and the BR6 lane kernel accept their largest LDS request (once per
// process and device).
void mt_prepare_wave_kernels();

// Record an error message for tron_last_error() and return `code`.
tron_err mt_fail(tron_err code, const char *fmt, ...);

#define HIP_TRY(expr)                                                                         \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return mt_fail(TRON_ERR_DEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));   \
    } while (0)

// The group-solver kernel for (family, N, G): one instance per G lanes, n <= N; null when
// that build does not exist (group.hip).
lane_launch_fn mt_group_launcher(tron_family fam, int N, int G);
