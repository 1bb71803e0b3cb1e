// block_tron.hpp -- one trust-region Newton solve per workgroup of W wavefronts (quartic
// family, n > 64).
//
// Every wave holds every vector (lane l the rows l + 64 r, as in wave_tron.hpp) and runs the
// vector-level steps of TronSteps on the same values, so all waves take the same decisions
// without talking to each other. Only the O(n^2) and O(n^3) steps are divided: products by
// rows and accumulators, the factorisation by 16 x 16 blocks and rows, the substitutions by
// blocks of 64 rows. Their parts meet in LDS. Every sum keeps the order of the one-wave form
// (four accumulators by column index mod 4 in products, two by panel chunk in the matrix-core
// updates, even and odd columns inside a panel), so results do not depend on W.
//
// What bounds it: up to n = 256 the trips to L2 and the serial steps (pivots of a panel's
// diagonal block, the substitutions' 16-row blocks) at one workgroup per CU, since 256
// registers per lane leave two waves per SIMD; at n = 512 the traffic past L2 (49 GB in 13.7 ms
// for 256 instances, 3.6 TB/s; matrix cores busy 15 %). Scratch is part of it: every wave keeps
// vectors of the solve there across the matrix steps (1.7 KB per lane for n > 256, 0.5 KB up to
// 256). Against one wave per instance: 512 x n = 200 16.4 -> 3.7 ms, 512 x n = 512 157 -> 24.0 ms.
//
// Where the matrices live:
//   kGlobal false  H (upper triangle with diagonal) and L (strict lower triangle) share one
//                  LDS array of n rows, odd stride ld > n, as in wave_tron.hpp; pivots and
//                  their reciprocals are vectors of their own.
//   kGlobal true   H's off-diagonal is the caller's packed parameter block (read in place,
//                  each element once per product: 64 x 64 tiles go through LDS and serve the
//                  rows of both of their sides); the workspace holds L by rows below the
//                  diagonal and by columns above it, so that every step reads it with
//                  consecutive lanes on consecutive addresses.
#pragma once

#include "wave_tron.hpp"

namespace mt {

// The matrix steps are functions of their own: inlined at every use they overflow the
// instruction cache and the register file. Arguments go by value, in registers, and pointers
// carry their address space, so that no argument passes through scratch or a generic address.
#define MT_STEP __device__ __attribute__((noinline))

typedef __attribute__((address_space(1))) double glb_double;
typedef __attribute__((address_space(1))) char glb_char;
template <bool kGlobal> struct MatrixPtr { typedef lds_double *type; };
template <> struct MatrixPtr<true> { typedef glb_double *type; };

MT_INLINE int uni_i(int v) { return __builtin_amdgcn_readfirstlane(v); }
MT_INLINE uint64_t uni64(uint64_t v)
{
    return ((uint64_t)(uint32_t)uni_i((int)(uint32_t)(v >> 32)) << 32) | (uint32_t)uni_i((int)(uint32_t)v);
}
MT_INLINE lds_double *uni_p(lds_double *q) { return (lds_double *)(uintptr_t)(uint32_t)uni_i((int)(uint32_t)(uintptr_t)q); }
MT_INLINE glb_double *uni_p(glb_double *q) { return (glb_double *)uni64((uint64_t)q); }

template <int R_, int W_, bool kGlobal>
struct BlockTron : TronSteps<BlockTron<R_, W_, kGlobal>, R_, LdsVec> {
    static constexpr int R = R_, W = W_, kRows = 64 * R;
    static constexpr bool kTight = false;
    using Steps = TronSteps<BlockTron<R_, W_, kGlobal>, R_, LdsVec>;
    using Steps::n;
    using Steps::lane;
    using Steps::hd;
    using Steps::lo;
    using Steps::hi;
    using Steps::x;
    using Steps::g;
    using Steps::has_l;
    using Steps::row;
    using Steps::valid;
    using Steps::dot;
    using Steps::own_free;
    typedef double d4 __attribute__((ext_vector_type(4)));
    typedef typename MatrixPtr<kGlobal>::type MPtr;

    // LDS, in doubles from the start of the workgroup's dynamic allocation
    static constexpr int oA = 0;                                  // partial sums: four, two products
    static constexpr int oD = oA + 2 * 4 * kRows;                 // reciprocal pivots
    static constexpr int oPV = oD + kRows;                        // pivots
    static constexpr int oY = oPV + kRows;                        // substitution results
    static constexpr int oHD = oY + kRows;                        // H's diagonal
    static constexpr int oQD = oHD + kRows;                       // Q's diagonal
    static constexpr int oVec = oQD + kRows;                      // lo, hi, x, g, c
    static constexpr int oV = oVec + 5 * kRows;                   // a product's operands
    static constexpr int oMk = oV + 2 * kRows;                    // free set, R words
    static constexpr int oP = oMk + (R + 1) / 2 * 2;              // a panel's diagonal block of L
    static constexpr int oF = oP + 16 * 17;                       // failed-pivot flag
    static constexpr int oU = oF + 2;                             // tiles / panel / matrix array
    static constexpr int kTile = 64 * 65;
    static constexpr int kU = 2 * kTile > kRows * 17 ? 2 * kTile : kRows * 17;  // kGlobal
    // (a last panel's steps read 16 entries of a row where fewer are left: up to 15 doubles past
    // the matrix array, which no result depends on)
    static constexpr size_t lds_bytes(int nmax)
    {
        return sizeof(double) * (size_t)(oU + (kGlobal ? kU : nmax * ((nmax + 1) | 1) + 16));
    }

    // what the matrix steps need
    struct Ctx {
        lds_double *L0;   // the LDS
        MPtr M;           // matrix array (LDS or workspace)
        glb_double *p;    // packed parameters
        int n, ld, w, lane;
        // a function's arguments arrive as per-lane values: back to scalars
        MT_INLINE Ctx scalar() const { return Ctx{uni_p(L0), uni_p(M), uni_p(p), uni_i(n), uni_i(ld), uni_i(w), lane}; }
        MT_INLINE int row(int r) const { return lane + 64 * r; }
    };
    // word q (uniform) of the free set, 0 past the last
    static MT_INLINE uint64_t word(const Ctx &k, int q)
    {
        const uint64_t v = uni64((uint64_t)__double_as_longlong(k.L0[oMk + (q < R ? q : 0)]));
        return q < R ? v : 0ull;
    }

    Ctx k;
    LdsVec qd, c;
    double kap;

    MT_INLINE void sync() const { __syncthreads(); }
    MT_INLINE void before_accept() const { __syncthreads(); }

    // ordering between a wave's own LDS writes and reads
    static MT_INLINE void wave_order()
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // slot s (uniform) of a row-distributed vector
    static MT_INLINE double slot(const double (&v)[R], int s)
    {
        double t = v[0];
        MT_UNROLL for (int r = 1; r < R; r++) t = s == r ? v[r] : t;
        return t;
    }

    MT_INLINE void load(const double *pp, const double *lop, const double *hip_, const double *x0p)
    {
        k.p = (glb_double *)pp;
        k.n = n;
        k.lane = lane;
        hd.v = k.L0 + oHD + lane;
        qd.v = k.L0 + oQD + lane;
        lo.v = k.L0 + oVec + lane;
        hi.v = lo.v + kRows;
        x.v = lo.v + 2 * kRows;
        g.v = lo.v + 3 * kRows;
        c.v = lo.v + 4 * kRows;
        const double *cp = pp + n * (n + 1) / 2;
        kap = cp[n];
        MT_UNROLL for (int r = 0; r < R; r++) {
            const int i = row(r);
            const bool in = i < n;
            const int j = in ? i : 0;
            lo[r] = in ? lop[j] : 0.0;
            hi[r] = in ? hip_[j] : 0.0;
            x[r] = in ? x0p[j] : 0.0;
            qd[r] = in ? pp[j * (j + 1) / 2 + j] : 0.0;
            c[r] = in ? cp[j] : 0.0;
        }
        if constexpr (!kGlobal) {
            // strict upper part of Q: row j of the packed lower triangle is column j
            for (int j = k.w; j < n; j += W) {
                MT_UNROLL for (int r = 0; r < R; r++) {
                    const int i = row(r);
                    if (i < j) k.M[i * k.ld + j] = pp[j * (j + 1) / 2 + i];
                }
            }
        }
    }

    MT_INLINE void hess()
    {
        MT_UNROLL for (int r = 0; r < R; r++) hd[r] = fma(12.0 * kap * x[r], x[r], qd[r]);
    }

    // ---------------------------------------------------------------------------------
    // y = A v, A = H's off-diagonal part with the diagonal at LDS offset o0 (and y1 = A1 v1
    // when NV = 2); rows >= n give 0. The operands come in LDS (operand()), the four partial
    // sums of each row are left there (sums()).
    // ---------------------------------------------------------------------------------
    MT_INLINE void operand(int q, const double (&v)[R])
    {
        if (k.w < R) k.L0[oV + q * kRows + 64 * k.w + lane] = slot(v, k.w);
    }
    MT_INLINE void sums(int o, double (&y)[R]) const
    {
        const lds_double *A = k.L0 + o;
        MT_UNROLL for (int r = 0; r < R; r++) {
            const int i = row(r);
            const double s = (A[i] + A[kRows + i]) + (A[2 * kRows + i] + A[3 * kRows + i]);
            y[r] = valid(r) ? s : 0.0;
        }
    }

    // Accumulator u over the columns of one block of 64: entries h(jj) for jj = u, u + 4, ...
    // times v's entries, which lane t of each 16-lane row holds for jj = u + 4 t; below the last
    // multiple of 4 of jend, and what is left over for u = 0 (v there from vt, lane jj).
    template <int NV, class H>
    static MT_INLINE void columns(int u, int jend, H h, const double (&vb)[NV], const lds_double *(&vt)[NV], double (&a)[NV])
    {
        if (jend == 64) {
            double e[NV][16];
            MT_UNROLL for (int t = 0; t < 16; t++) {
                const int jj = u + 4 * t;
                MT_UNROLL for (int q = 0; q < NV; q++) e[q][t] = h(jj, q);
            }
            MT_UNROLL for (int q = 0; q < NV; q++) {
                fma_row4<0>(a[q], vb[q], e[q][0], e[q][1], e[q][2], e[q][3]);
                fma_row4<4>(a[q], vb[q], e[q][4], e[q][5], e[q][6], e[q][7]);
                fma_row4<8>(a[q], vb[q], e[q][8], e[q][9], e[q][10], e[q][11]);
                fma_row4<12>(a[q], vb[q], e[q][12], e[q][13], e[q][14], e[q][15]);
            }
        } else {
            const int jfull = jend > 0 ? jend & ~3 : 0;
#pragma unroll 1
            for (int jj = u; jj < jfull; jj += 4)
                MT_UNROLL for (int q = 0; q < NV; q++) a[q] = fma(h(jj, q), vt[q][jj], a[q]);
            if (u == 0) {
#pragma unroll 1
                for (int jj = jfull; jj < jend; jj++)
                    MT_UNROLL for (int q = 0; q < NV; q++) a[q] = fma(h(jj, q), vt[q][jj], a[q]);
            }
        }
    }

    template <int NV>
    static MT_INLINE void product_body(const Ctx &ka, int o0, int o1)
    {
        const Ctx k = ka.scalar();
        const int n = k.n, lane = k.lane;
        lds_double *V = k.L0 + oV;
        if constexpr (!kGlobal) {
            // wave: one slot of rows, one of the four accumulators
            static_assert(W == 4 * R, "one wave per row slot and accumulator");
            lds_double *A = k.L0 + oA;
            const int sl = k.w % R, u = k.w / R;
            const int i = lane + 64 * sl, ii = i < n ? i : 0;
            double d[NV], a[NV];
            d[0] = k.L0[o0 + i];
            if constexpr (NV > 1) d[1] = k.L0[o1 + i];
            MT_UNROLL for (int q = 0; q < NV; q++) a[q] = 0.0;
            __syncthreads();
            MT_UNROLL for (int rr = 0; rr < R; rr++) {
                const int jend = n - 64 * rr < 64 ? n - 64 * rr : 64;
                double vb[NV];
                const lds_double *vt[NV];
                MT_UNROLL for (int q = 0; q < NV; q++) {
                    vt[q] = V + q * kRows + 64 * rr;
                    vb[q] = vt[q][u + 4 * (lane & 15)];
                }
                columns<NV>(u, jend, [&](int jj, int q) -> double {
                    const int j = 64 * rr + jj;
                    const int mn = j < ii ? j : ii;
                    const double m = k.M[(int)__umul24((unsigned)mn, (unsigned)(k.ld - 1)) + j + ii];
                    return j == ii ? d[q] : m;
                }, vb, vt, a);
            }
            MT_UNROLL for (int q = 0; q < NV; q++) A[(4 * q + u) * kRows + i] = a[q];
        } else {
            // 64 x 64 tiles (I, J), I <= J, in the order J = 0.., I = 0..J: the rows of block I
            // then meet column blocks in ascending order, and so do the rows of block J. Waves
            // 0..3 take the rows of block I, 4..7 those of block J, one accumulator each. A tile
            // of the diagonal is stored with both of its triangles.
            static_assert(W == 8, "two sides of a tile, four accumulators");
            const int nb = (n + 63) >> 6, nt = nb * (nb + 1) / 2;
            const int u = k.w & 3, side = k.w >> 2;
            lds_double *A = k.L0 + oA, *T = k.L0 + oU;
            double f0[8], f1[8];  // tiles on their way, every other one
            int I = 0, J = 0;     // tile in hand
            int FI = 0, FJ = 0;   // tile being fetched
            // Rows 8 w .. 8 w + 7 of a tile. Rows past n repeat row n - 1; entries right of the
            // diagonal (at most 63, inside the block's c) are read and not used.
            auto fetch = [&](double (&fb)[8]) {
                const uint32_t at = (uint32_t)(64 * FI + lane) * 8u;
                int j = 64 * FJ + 8 * k.w;
                MT_UNROLL for (int q = 0; q < 8; q++, j++) {
                    const int jc = j < n ? j : n - 1;
                    const glb_char *pj =
                        (const glb_char *)(k.p + (uint32_t)(jc * (jc + 1)) / 2u);
                    fb[q] = *(const glb_double *)(pj + at);
                }
                if (++FI > FJ) { FI = 0; FJ++; }
            };
            auto tile = [&](lds_double *tb, double (&fb)[8], bool more) {
                const bool diag = I == J;
                if (!diag) {
                    MT_UNROLL for (int q = 0; q < 8; q++) tb[(8 * k.w + q) * 65 + lane] = fb[q];
                } else {
                    const double e = k.L0[o0 + 64 * J + lane];
                    MT_UNROLL for (int q = 0; q < 8; q++) {
                        const int jj = 8 * k.w + q;
                        if (lane <= jj) {
                            const double v = lane == jj ? e : fb[q];
                            tb[jj * 65 + lane] = v;
                            tb[lane * 65 + jj] = v;
                        }
                    }
                }
                if (more) fetch(fb);
                __syncthreads();
                if (side == 0 || !diag) {
                    // own: block of the rows, oth: block of the columns
                    const int own = side == 0 ? I : J, oth = side == 0 ? J : I;
                    const int at = u * kRows + 64 * own + lane;
                    const bool fresh = side == 0 ? J == 0 : I == 0;
                    double a[NV], vb[NV];
                    const lds_double *vt[NV];
                    MT_UNROLL for (int q = 0; q < NV; q++) {
                        const double a0 = A[4 * q * kRows + at];
                        a[q] = fresh ? 0.0 : a0;
                        vt[q] = V + q * kRows + 64 * oth;
                        vb[q] = vt[q][u + 4 * (lane & 15)];
                    }
                    const int jend = n - 64 * oth < 64 ? n - 64 * oth : 64;
                    // side 0 walks a column of the tile's array, side 1 a row
                    const lds_double *tl = tb + (side == 0 ? lane : 65 * lane);
                    const int st = side == 0 ? 65 : 1;
                    if (NV > 1 && diag) {
                        const double e1 = k.L0[o1 + 64 * J + lane];
                        columns<NV>(u, jend, [&](int jj, int q) -> double {
                            const double h = tl[jj * st];
                            return q == 1 && jj == lane ? e1 : h;
                        }, vb, vt, a);
                    } else {
                        columns<NV>(u, jend, [&](int jj, int) -> double { return tl[jj * st]; }, vb, vt, a);
                    }
                    MT_UNROLL for (int q = 0; q < NV; q++) A[4 * q * kRows + at] = a[q];
                }
                if (++I > J) { I = 0; J++; }
            };
            fetch(f0);
            if (nt > 1) fetch(f1);
#pragma unroll 1
            for (int t = 0; t < nt; t += 2) {
                tile(T, f0, t + 2 < nt);
                if (t + 1 < nt) tile(T + kTile, f1, t + 3 < nt);
            }
        }
        __syncthreads();
    }
    static MT_STEP void product1(Ctx k, int o0) { product_body<1>(k, o0, o0); }
    static MT_STEP void product2(Ctx k, int o0, int o1) { product_body<2>(k, o0, o1); }

    MT_INLINE void hmul(const double (&v)[R], double (&y)[R])
    {
        operand(0, v);
        product1(k, oHD);
        sums(oA, y);
    }

    MT_INLINE double f_of(const double (&v)[R], const double (&y)[R], double (&gr)[R]) const
    {
        double acc = 0.0;
        MT_UNROLL for (int r = 0; r < R; r++) {
            const double x2 = v[r] * v[r];
            gr[r] = valid(r) ? fma(4.0 * kap * x2, v[r], y[r] + c[r]) : 0.0;
            acc = fma(v[r], fma(0.5, y[r], c[r]), acc);
            acc = fma(kap * x2, x2, acc);
        }
        return uni(wave_sum(acc));
    }

    MT_INLINE double fg(const double (&v)[R], double (&gr)[R])
    {
        double y[R];
        operand(0, v);
        product1(k, oQD);
        sums(oA, y);
        return f_of(v, y, gr);
    }

    // the model's product and the trial evaluation read the matrix once for both
    MT_INLINE bool model(const double (&s)[R], double (&hs)[R], const double (&v)[R], double (&gt)[R], double &ft)
    {
        double y[R];
        operand(0, s);
        operand(1, v);
        product2(k, oHD, oQD);
        sums(oA, hs);
        sums(oA + 4 * kRows, y);
        ft = f_of(v, y, gt);
        return true;
    }

    // ---------------------------------------------------------------------------------
    // Cholesky factorisation of H_FF + alpha I with the identity outside F, in panels of 16
    // columns: (1) the matrix cores form the panel S = A - L L^T from the columns before it,
    // 16 x 16 blocks dealt to the waves; (2) one wave factors the panel's 16 x 16 diagonal
    // block, its rows in the lanes of a 16-lane row, values passed by row broadcasts; (3) the
    // rows below take their entries by a triangular solve against that block, one row per lane.
    // ---------------------------------------------------------------------------------

    // Blocks of a wave: rows j0 + 16 (w + W t), t < kMost. Panels are taken in pairs: the
    // products of both read the earlier columns of L once.
    static constexpr int kMost = (4 * R + W - 1) / W;
    struct Sum { d4 v[2]; };                    // two sums per block
    static constexpr int kStage = 256;          // kGlobal: columns of the panels' own rows in LDS at a time

    // S's starting values: A = H_FF + alpha I with the identity outside F at the 16 x 16 block of
    // row k0, column j0 (lane: row lq + 4 v, column lr). Rows past n repeat row n - 1 and entries
    // right of the diagonal (at most 31, inside the parameter block) are read; none is kept.
    static MT_INLINE Sum block_start(const Ctx &k, int k0, int j0, uint64_t fk, uint64_t fw, double hj, double alpha)
    {
        const int lr = k.lane & 15, lq = k.lane >> 4, jb = j0 + lr;
        const bool fj = (fw >> (jb & 63)) & 1ull;
        double h[4];
        MT_UNROLL for (int v = 0; v < 4; v++) {
            const int i0 = k0 + lq + 4 * v, i = i0 < k.n ? i0 : k.n - 1;
            if constexpr (kGlobal) h[v] = *(const glb_double *)((const glb_char *)k.p + (uint32_t)((i * (i + 1) / 2 + jb) * 8));
            else h[v] = k.M[(jb < k.n ? jb : k.n - 1) * k.ld + i];
        }
        Sum s;
        MT_UNROLL for (int v = 0; v < 4; v++) {
            const int i = k0 + lq + 4 * v;
            s.v[0][v] = i == jb ? (fj ? hj + alpha : 1.0) : ((fj && ((fk >> (i & 63)) & 1ull)) ? h[v] : 0.0);
            s.v[1][v] = 0.0;
        }
        return s;
    }

    // a, b: the two panels' blocks of this wave (CNT or one fewer) less their products with the
    // columns before j0. The panels' own rows are read by every wave: in the workspace form they
    // go through LDS, panel by panel, 16 rows of a column side by side (two columns span the
    // banks once); a wave's A operands come straight from the workspace, 16 columns' worth in
    // flight while another 16 are used. Rows past n read row n - 1; their results are not kept.
    template <int CNT>
    static MT_INLINE void panel_products(const Ctx &k, int j0, int cnt, Sum (&a)[kMost], Sum (&b)[kMost])
    {
        const bool all = cnt == CNT;  // this wave has CNT blocks, else one fewer
        const int n = k.n, ld = k.ld, lane = k.lane, lr = lane & 15, lq = lane >> 4;
        lds_double *Bs = k.L0 + oU;
        uint32_t oa[CNT];
        MT_UNROLL for (int t = 0; t < CNT; t++) {
            const int i0 = j0 + 16 * (k.w + W * t) + lr, i = i0 < n ? i0 : n - 1;
            oa[t] = kGlobal ? (uint32_t)(lq * ld + i) * 8u : (uint32_t)(i * ld + lq);
        }
        struct Ops { double a[CNT][4]; };
        auto fetch = [&](int q, Ops &o) {
            MT_UNROLL for (int v = 0; v < 4; v++)
                MT_UNROLL for (int t = 0; t < CNT; t++) {
                    if constexpr (kGlobal)
                        o.a[t][v] = *(const glb_double *)((const glb_char *)(k.M + (uint32_t)((q + 4 * v) * ld)) + oa[t]);
                    else o.a[t][v] = k.M[oa[t] + (uint32_t)(q + 4 * v)];
                }
        };
        // the products of 16 columns; p1, p2: this lane's entries of the panels' rows
        auto use = [&](const Ops &o, const lds_double *p1, const lds_double *p2, int step) {
            double b1[4], b2[4];
            MT_UNROLL for (int v = 0; v < 4; v++) {
                b1[v] = p1[v * step];
                b2[v] = p2[v * step];
            }
            MT_UNROLL for (int t = 0; t < CNT; t++) {
                if (t == CNT - 1 && !all) continue;
                MT_UNROLL for (int v = 0; v < 4; v++) {
                    const double m = -o.a[t][v];
                    a[t].v[v & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(m, b1[v], a[t].v[v & 1], 0, 0, 0);
                    b[t].v[v & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(m, b2[v], b[t].v[v & 1], 0, 0, 0);
                }
            }
        };
        if constexpr (kGlobal) {
#pragma unroll 1
            for (int qb = 0; qb < j0; qb += kStage) {
                const int qn = j0 - qb < kStage ? j0 - qb : kStage;  // a multiple of 32
                if (qb > 0) __syncthreads();
                {
                    const int r0 = j0 + (lane & 31), r = r0 < n ? r0 : n - 1;
                    lds_double *to = Bs + ((lane >> 4) & 1) * (16 * kStage) + lr + 16 * (lane >> 5);
                    const glb_double *from = k.M + (uint32_t)(qb * ld);
                    const uint32_t at = (uint32_t)((lane >> 5) * ld + r) * 8u;
                    // (an even number per wave; eight loads on their way at a time)
#pragma unroll 1
                    for (int c = 2 * k.w; c < qn; c += 16 * W) {
                        double st[8];
                        MT_UNROLL for (int e = 0; e < 8; e += 2)
                            if (c + 2 * W * e < qn) {
                                st[e] = *(const glb_double *)((const glb_char *)(from + (uint32_t)((c + 2 * W * e) * ld)) + at);
                                st[e + 1] = *(const glb_double *)((const glb_char *)(from + (uint32_t)((c + 2 * W * (e + 1)) * ld)) + at);
                            }
                        MT_UNROLL for (int e = 0; e < 8; e += 2)
                            if (c + 2 * W * e < qn) {
                                to[16 * (c + 2 * W * e)] = st[e];
                                to[16 * (c + 2 * W * (e + 1))] = st[e + 1];
                            }
                    }
                }
                Ops x, y;
                fetch(qb, x);
                fetch(qb + 16, y);
                __syncthreads();
                const lds_double *p1 = Bs + lane, *p2 = p1 + 16 * kStage;  // column lq of four, row lr
                if (CNT > 1 || all) {
#pragma unroll 1
                    for (int q = 0; q < qn; q += 32) {
                        use(x, p1 + 16 * q, p2 + 16 * q, 64);
                        if (q + 32 < qn) fetch(qb + q + 32, x);
                        use(y, p1 + 16 * (q + 16), p2 + 16 * (q + 16), 64);
                        if (q + 32 < qn) fetch(qb + q + 48, y);
                    }
                }
            }
            if (j0 > 0) __syncthreads();  // the panels go where their rows were
        } else {
            const int jb1 = j0 + lr < n ? j0 + lr : n - 1, jb2 = j0 + 16 + lr < n ? j0 + 16 + lr : n - 1;
            const lds_double *p1 = k.M + jb1 * ld + lq, *p2 = k.M + jb2 * ld + lq;
#pragma unroll 1
            for (int q = 0; q < j0; q += 16) {
                Ops x;
                fetch(q, x);
                use(x, p1 + q, p2 + q, 4);
            }
        }
    }

    // the second panel's products with the first panel's columns (in LDS since rows_below)
    static MT_INLINE void panel_link(const Ctx &k, int j0, int k0, Sum &b)
    {
        const int n = k.n, lr = k.lane & 15, lq = k.lane >> 4;
        const int jb = j0 + 16 + lr < n ? j0 + 16 + lr : j0, i = k0 + lr < n ? k0 + lr : j0;
        const lds_double *L = k.L0 + oU + lq;
        const lds_double *pb = kGlobal ? L + (jb - j0) * 17 : L + jb * k.ld + j0;
        const lds_double *pa = kGlobal ? L + (i - j0) * 17 : L + i * k.ld + j0;
        MT_UNROLL for (int v = 0; v < 4; v++)
            b.v[v & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-pa[4 * v], pb[4 * v], b.v[v & 1], 0, 0, 0);
    }

    // a block of the panel at j0 to its slots
    static MT_INLINE void block_store(const Ctx &k, int k0, int j0, const Sum &a)
    {
        const int n = k.n, lr = k.lane & 15, lq = k.lane >> 4, jb = j0 + lr;
        MT_UNROLL for (int v = 0; v < 4; v++) {
            const int i = k0 + lq + 4 * v;
            const double s = a.v[0][v] + a.v[1][v];
            if (i < n && jb < n && i >= jb) {
                if constexpr (kGlobal) k.L0[oU + (i - j0) * 17 + lr] = s;
                else k.M[(int)__umul24((unsigned)i, (unsigned)k.ld) + (i == jb ? n : jb)] = s;
            }
        }
    }

    // Column C of the diagonal block (lane il of each 16-lane row holds row il): its entry of
    // the pivot row, the pivot, the scale, then its products off the columns after it, the sum
    // over even columns in sv and over odd ones in s1; the newest column comes last. Rows and
    // columns outside F need no masks: S is the identity there, so their entries stay 0 and
    // their pivots 1. The reciprocal pivot goes straight to the block's column 16.
    template <int C>
    static MT_INLINE void diag_column(double (&sv)[16], double (&s1)[16], int cols, bool &bad, lds_double *P)
    {
        if constexpr (C < 16) {
            double s = sv[C] + s1[C], own = s;
            if constexpr (C > 0) own = fma(-sv[C - 1], sv[C - 1], s);  // in lane C, the pivot's own update
            const double d = row_bcast<C>(own);
            const double rinv = rsqrt_pos(d);
            if constexpr (C > 0) {
                fnma_row<C>(s, sv[C - 1], sv[C - 1]);
                diag_tail<C - 1, C + 1>(sv, s1);
            }
            bad = bad || (C < cols && !(d > 0.0));
            P[C * 17 + 16] = rinv;
            sv[C] = s * rinv;
            diag_column<C + 1>(sv, s1, cols, bad, P);
        }
    }
    template <int C, int C2>
    static MT_INLINE void diag_tail(double (&sv)[16], double (&s1)[16])
    {
        if constexpr (C2 + 3 < 16) {
            double(&d)[16] = (C & 1) ? s1 : sv;
            fnma_row4<C2>(d[C2], d[C2 + 1], d[C2 + 2], d[C2 + 3], sv[C], sv[C]);
            diag_tail<C, C2 + 4>(sv, s1);
        } else if constexpr (C2 < 16) {
            double(&d)[16] = (C & 1) ? s1 : sv;
            fnma_row<C2>(d[C2], sv[C], sv[C]);
            diag_tail<C, C2 + 1>(sv, s1);
        }
    }

    static MT_INLINE void diag_block(const Ctx &k, int j0)
    {
        const int il = k.lane & 15, i = j0 + il, n = k.n;
        lds_double *P = k.L0 + oP;
        double sv[16], s1[16];
        // Entries right of the diagonal and rows past n hold whatever was there: they only meet
        // their own lane's entries further right, which nothing reads.
        const lds_double *src = kGlobal ? k.L0 + oU + il * 17 : k.L0 + oU + (i < n ? i : j0) * k.ld + j0;
        const double own = kGlobal ? 0.0 : src[n - j0];  // the LDS form keeps the diagonal in column n
        MT_UNROLL for (int cc = 0; cc < 16; cc++) {
            const double v = src[cc];
            sv[cc] = !kGlobal && cc == il ? own : v;
            s1[cc] = 0.0;
        }
        const bool ownf = (word(k, j0 >> 6) >> (i & 63)) & 1ull;
        bool bad = false;
        diag_column<0>(sv, s1, n - j0, bad, P);
        if (k.lane < 16) {
            MT_UNROLL for (int cc = 0; cc < 16; cc++) P[il * 17 + cc] = sv[cc];
            wave_order();
            if (i < n) {
                k.L0[oD + i] = ownf ? P[il * 17 + 16] : 1.0;
                k.L0[oPV + i] = ownf ? P[il * 17 + il] : 1.0;  // d / sqrt(d)
            }
            if (il == 0) k.L0[oF] = bad ? 1.0 : 0.0;
        }
    }

    // Rows below the panel's diagonal block, t the lane's entries: columns in turn, each with
    // the products of the columns before it (even ones in one sum, odd ones in the other, row
    // cc of the block broadcast from lane cc's q). kLate: the newest column goes with its even or
    // odd fellows (rows past the panel's own 64 in the workspace form); otherwise it comes last.
    template <bool kLate, int C>
    static MT_INLINE void row_column(double (&t)[16], const double (&q)[16], double qr)
    {
        if constexpr (C < 16) {
            double p0 = t[C], p1 = 0.0;
            row_sums<C, 0, kLate ? C : C - 1>(t, q, p0, p1);
            double v = p0 + p1;
            if constexpr (!kLate && C > 0) fnma_row<C>(v, q[C - 1], t[C - 1]);
            t[C] = v * row_bcast<C>(qr);
            row_column<kLate, C + 1>(t, q, qr);
        }
    }
    // wave w: the rows of block (j0 / 64) + w that are below the panel
    static MT_INLINE void rows_below(const Ctx &k, int j0)
    {
        const int n = k.n, ld = k.ld, lane = k.lane;
        const lds_double *P = k.L0 + oP;
        lds_double *S = k.L0 + oU;
        // the diagonal block's entries go to their places (the last wave: it has the fewest rows)
        if (k.w == W - 1) {
            MT_UNROLL for (int it = 0; it < 4; it++) {
                const int a = 4 * it + (lane >> 4), b = lane & 15;
                if (b < a && j0 + a < n) k.M[(j0 + a) * ld + j0 + b] = P[a * 17 + b];
                if constexpr (kGlobal)
                    if (a < b && j0 + b < n) k.M[(j0 + a) * ld + j0 + b] = P[b * 17 + a];
            }
        }
        const int sl = (j0 >> 6) + k.w;
        if (j0 + 16 >= n || 64 * sl >= n || 64 * sl + 63 < j0 + 16) return;
        const int i = 64 * sl + lane;
        const bool in = i >= j0 + 16 && i < n;
        double t[16], q[16];
        lds_double *src;
        if constexpr (kGlobal) src = S + (in ? i - j0 : 16) * 17;
        else src = k.M + (in ? i : j0) * ld + j0;
        MT_UNROLL for (int cc = 0; cc < 16; cc++) {
            t[cc] = src[cc];
            q[cc] = P[(lane & 15) * 17 + cc];
        }
        const double qr = P[(lane & 15) * 17 + 16];
        if (kGlobal && k.w > 0) row_column<true, 0>(t, q, qr);
        else row_column<false, 0>(t, q, qr);
        if (in) MT_UNROLL for (int cc = 0; cc < 16; cc++) src[cc] = t[cc];
        if constexpr (kGlobal) {
            if (in) MT_UNROLL for (int cc = 0; cc < 16; cc++) k.M[(j0 + cc) * ld + i] = t[cc];
            wave_order();
            // by rows: sixteen lanes write the panel's 16 entries of one row
            MT_UNROLL for (int it = 0; it < 16; it++) {
                const int a = 64 * sl + 4 * it + (lane >> 4), b = lane & 15;
                if (a >= j0 + 16 && a < n) k.M[a * ld + j0 + b] = S[(a - j0) * 17 + b];
            }
        }
    }

    // one panel, S in its slots: false when a free pivot is not positive
    static MT_INLINE bool panel_finish(const Ctx &k, int j0)
    {
        __syncthreads();
        if (k.w == 0) diag_block(k, j0);
        __syncthreads();
        if (k.L0[oF] != 0.0) return false;
        rows_below(k, j0);
        __syncthreads();
        return true;
    }

    static MT_STEP int chol(Ctx ka, double alpha)
    {
        const Ctx k = ka.scalar();
        Sum b[kMost];
#pragma unroll 1
        for (int j0 = 0; j0 < k.n; j0 += 32) {
            Sum a[kMost];
            const int blocks = ((k.n - j0 + 15) >> 4) - k.w;  // from this wave's first on, every W-th its own
            {
                const int lr = k.lane & 15;
                const uint64_t fw = word(k, j0 >> 6);
                const double h1 = k.L0[oHD + j0 + lr], h2 = k.L0[oHD + (j0 + 16 < kRows ? j0 + 16 : j0) + lr];
                MT_UNROLL for (int t = 0; t < kMost; t++) {
                    const int k0 = j0 + 16 * (k.w + W * t);
                    const uint64_t fk = word(k, k0 >> 6);
                    a[t] = block_start(k, k0, j0, fk, fw, h1, alpha);
                    b[t] = block_start(k, k0, j0 + 16, fk, fw, h2, alpha);
                }
            }
            // The form is the one the first wave needs, in all waves: its barriers must not stand in
            // a branch that waves take differently.
            const int most = ((k.n - j0 + 15) >> 4) + W - 1, cnt = (blocks + W - 1) / W;
            if (kMost >= 4 && most >= 4 * W) panel_products<kMost >= 4 ? 4 : 1>(k, j0, cnt, a, b);
            else if (kMost >= 3 && most >= 3 * W) panel_products<kMost >= 3 ? 3 : 1>(k, j0, cnt, a, b);
            else if (kMost >= 2 && most >= 2 * W) panel_products<kMost >= 2 ? 2 : 1>(k, j0, cnt, a, b);
            else panel_products<1>(k, j0, cnt, a, b);
            MT_UNROLL for (int t = 0; t < kMost; t++)
                if (blocks > W * t) block_store(k, j0 + 16 * (k.w + W * t), j0, a[t]);
#pragma unroll 1
            for (int j1 = j0;;) {
                if (!panel_finish(k, j1)) return 0;
                if (j1 > j0 || j0 + 16 >= k.n) break;
                j1 = j0 + 16;
                MT_UNROLL for (int t = 0; t < kMost; t++) {
                    const int k0 = j0 + 16 * (k.w + W * t);
                    if (k0 < k.n) panel_link(k, j0, k0, b[t]);
                }
                if constexpr (kGlobal) __syncthreads();
                MT_UNROLL for (int t = 0; t < kMost; t++) {
                    const int k0 = j0 + 16 * (k.w + W * t);
                    if (k0 < k.n) block_store(k, k0, j1, b[t]);
                }
            }
        }
        return 1;
    }

    // Returns the shift that succeeded, or -1 when the diagonal fallback was used.
    MT_INLINE double precond(const uint64_t (&fm)[R])
    {
        double mn = __builtin_inf(), mx = 0.0;
        MT_UNROLL for (int r = 0; r < R; r++) {
            if (valid(r) && own_free(fm, r)) {
                mn = hd[r] < mn ? hd[r] : mn;
                mx = fabs(hd[r]) > mx ? fabs(hd[r]) : mx;
            }
        }
        mn = -uni(wave_max(-mn));
        mx = uni(wave_max(mx));
        const double beta = 1e-3 * (mx > 1.0 ? mx : 1.0);
        double alpha = mn > 0.0 ? 0.0 : beta - mn;
        // every wave writes the same words, the last readers being behind a barrier
        MT_UNROLL for (int r = 0; r < R; r++) k.L0[oMk + r] = __longlong_as_double((long long)fm[r]);
        for (int t = 0; t < kShiftTries; t++) {
            if (uni_i(chol(k, alpha))) return alpha;
            alpha = 2.0 * alpha > beta ? 2.0 * alpha : beta;
        }
        sync();
        for (int j = k.w; j < n; j += W) {
            MT_UNROLL for (int r = 0; r < R; r++) {
                const int i = row(r);
                if (i < n && i > j) {
                    k.M[i * k.ld + j] = 0.0;
                    if constexpr (kGlobal) k.M[j * k.ld + i] = 0.0;
                }
            }
        }
        MT_UNROLL for (int r = 0; r < R; r++) {
            const int i = row(r);
            if (i < n && k.w == r) {
                const double v = fabs(hd[r]);
                const double piv = own_free(fm, r) ? sqrt(v > beta ? v : beta) : 1.0;
                k.L0[oPV + i] = piv;
                k.L0[oD + i] = 1.0 / piv;
            }
        }
        sync();
        return -1.0;
    }

    // ---------------------------------------------------------------------------------
    // Substitutions, 16 rows at a time: the wave that holds them (wave w the rows 64 w + lane,
    // residuals kept unscaled as in wave_tron.hpp) solves the 16 x 16 block with row broadcasts,
    // its results go to LDS, and after one barrier every row still to come subtracts their 16
    // columns. The entries for the next 16 columns are loaded meanwhile.
    // ---------------------------------------------------------------------------------
    // kUp false: L y = b; true: L^T y = b, blocks and rows in descending order. bb: this wave's
    // rows of b; the results are left in LDS.
    template <bool kUp>
    static MT_INLINE void substitute(const Ctx &ka, double bb)
    {
        const Ctx k = ka.scalar();
        const int n = k.n, ld = k.ld, lane = k.lane, il = lane & 15;
        const int nb = (n + 15) >> 4;
        const int i = lane + 64 * k.w;
        const bool mine = 64 * k.w < n && k.w < R;  // the wave holds rows
        const bool in = mine && i < n;
        const int ik = in ? i : 0;
        const double dv = in ? k.L0[oD + ik] : 1.0;
        lds_double *Y = k.L0 + oY;
        // L(i, j0 + t) (kUp: L(j0 + t, i)), by columns where the workspace holds them
        auto entry = [&](int j) -> double {
            const int jc = j < n ? j : n - 1;
            if constexpr (kGlobal)
                return *(const glb_double *)((const glb_char *)(k.M + (uint32_t)(jc * ld)) + (uint32_t)ik * 8u);
            else if constexpr (kUp) return k.M[jc * ld + ik];
            else return k.M[ik * ld + jc];
        };
        auto fetch = [&](int q, double (&l)[16]) {
            const int blk = kUp ? nb - 1 - q : q;
            MT_UNROLL for (int t = 0; t < 16; t++) l[t] = entry(16 * blk + t);
        };
        double dl[16], l0[16], l1[16];
        if (mine) {
            MT_UNROLL for (int t = 0; t < 16; t++) {
                const int j = i - il + t, jc = j < n ? j : n - 1;
                double v;
                if constexpr (kUp || kGlobal) v = k.M[jc * ld + ik];
                else v = k.M[ik * ld + jc];
                dl[t] = v;
            }
            fetch(0, l0);
            if (nb > 1) fetch(1, l1);
            MT_UNROLL for (int t = 0; t < 16; t++) {
                const bool ok = in && (kUp ? t > il && i - il + t < n : t < il);
                dl[t] = ok ? dl[t] : 0.0;
            }
        }
        __syncthreads();  // the last results' readers are done
        auto step = [&](int q, double (&l)[16]) {
            const int blk = kUp ? nb - 1 - q : q;
            if (k.w == blk >> 2) {
                // every 16-lane row runs the steps; only the block's own row keeps them
                double t = bb;
                block_solve<kUp>(t, dv, dl, n - 16 * blk);
                const bool own = (lane >> 4) == (blk & 3);
                bb = own ? t : bb;
                const double y = bb * dv;
                if (own && in) Y[i] = y;
            }
            __syncthreads();
            if (mine && (kUp ? k.w <= blk >> 2 : k.w >= blk >> 2)) {
                const double y0 = Y[16 * blk + il];
                const double y = 16 * blk + il < n ? y0 : 0.0;
                double t = bb;
                block_update<kUp>(t, y, l);
                const bool left = in && (kUp ? i < 16 * blk : i >= 16 * blk + 16);
                bb = left ? t : bb;
                if (q + 2 < nb) fetch(q + 2, l);
            }
        };
#pragma unroll 1
        for (int q = 0; q < nb; q += 2) {
            step(q, l0);
            if (q + 1 < nb) step(q + 1, l1);
        }
    }
    static MT_STEP void solve_l(Ctx k, double bb) { substitute<false>(k, bb); }
    static MT_STEP void solve_lt(Ctx k, double bb) { substitute<true>(k, bb); }

    MT_INLINE void solved(double (&b)[R]) const
    {
        MT_UNROLL for (int r = 0; r < R; r++) {
            const double y = k.L0[oY + row(r)];
            b[r] = valid(r) ? y : b[r];
        }
    }
    MT_INLINE void fwd(double (&b)[R])
    {
        solve_l(k, slot(b, k.w));
        solved(b);
    }
    MT_INLINE void bwd(double (&b)[R])
    {
        solve_lt(k, slot(b, k.w));
        solved(b);
    }

    // L^T s in four partial sums by k mod 4 (see wave_tron.hpp); W / R waves share the sums of
    // one slot of rows
    static MT_STEP void lt_product(Ctx ka)
    {
        constexpr int kGroups = W / R, kOwn = 4 / kGroups;
        static_assert(kGroups * R == W && kOwn * kGroups == 4, "waves per row slot");
        const Ctx k = ka.scalar();
        const int n = k.n, ld = k.ld;
        lds_double *A = k.L0 + oA;
        const int sl = k.w % R, ug = k.w / R;
        const int i = k.lane + 64 * sl;
        double acc[kOwn];
        MT_UNROLL for (int a = 0; a < kOwn; a++) acc[a] = 0.0;
        const int nfull = n & ~3;
        // entry (j, i) of L, rows j from the block's first; 0 above the diagonal
        auto entry = [&](int j) -> double {
            const int jc = j < n ? j : n - 1;
            double v;
            if constexpr (kGlobal)
                v = *(const glb_double *)((const glb_char *)(k.M + (uint32_t)(jc * ld)) + (uint32_t)(i < n ? i : 0) * 8u);
            else v = k.M[jc * ld + (i < n ? i : 0)];
            return v;
        };
        __syncthreads();
        const lds_double *V = k.L0 + oV;
        int j0 = 64 * sl;
        // 16 / kGroups of them at a time, 64 / kGroups rows ahead
        constexpr int kQ = 16 / kGroups * (kGroups > 1 ? 2 : 1), kRowsStep = kQ * kGroups;
        double l[kQ];
        auto fetch = [&](int j) {
            MT_UNROLL for (int q = 0; q < kQ; q++) l[q] = entry(j + 4 * (q / kOwn) + kOwn * ug + q % kOwn);
        };
        if (j0 < nfull) fetch(j0);
#pragma unroll 1
        for (; j0 < nfull; j0 += kRowsStep) {
            double cur[kQ];
            MT_UNROLL for (int q = 0; q < kQ; q++) cur[q] = l[q];
            if (j0 + kRowsStep < nfull) fetch(j0 + kRowsStep);
            MT_UNROLL for (int q = 0; q < kQ; q++) {
                const int j = j0 + 4 * (q / kOwn) + kOwn * ug + q % kOwn;
                const double sj = V[j < nfull ? j : 0];
                const bool ok = i < j && j < nfull;
                acc[q % kOwn] = fma(ok ? cur[q] : 0.0, sj, acc[q % kOwn]);
            }
        }
        if (ug == 0) {
#pragma unroll 1
            for (int j = nfull > 64 * sl ? nfull : 64 * sl; j < n; j++) {
                const double v = entry(j);
                acc[0] = fma(i < j ? v : 0.0, V[j], acc[0]);
            }
        }
        MT_UNROLL for (int a = 0; a < kOwn; a++) A[(kOwn * ug + a) * kRows + i] = acc[a];
        __syncthreads();
    }

    MT_INLINE double step_norm(const double (&s)[R])
    {
        if (!has_l) return sqrt(dot(s, s));
        operand(0, s);
        lt_product(k);
        double y[R], t[R];
        sums(oA, y);
        MT_UNROLL for (int r = 0; r < R; r++) t[r] = valid(r) ? fma(k.L0[oPV + row(r)], s[r], y[r]) : 0.0;
        return sqrt(dot(t, t));
    }
};

}  // namespace mt
