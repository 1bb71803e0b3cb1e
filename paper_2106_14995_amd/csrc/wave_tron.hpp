// wave_tron.hpp -- one trust-region Newton solve per wavefront, for 8 < n <= 128.
//
// Lane l of the wave owns rows i = l + 64 r, r < R, of every vector (R = 1 up to n = 64, 2 up
// to 128). The n x n Hessian and its Cholesky factor share one array (LDS, or global memory when
// the plan asks for it) of n rows and odd
// row stride ld >= n + 1 (odd, so that both row and column walks touch distinct banks): the
// Hessian's upper triangle with its diagonal, the factor's strict lower triangle below it,
// and the factor's pivots in the spare column n. A Hessian-vector product then reads every
// H_kj from one address, min(j,k) ld + max(j,k) = min(j,k) (ld - 1) + j + k, with no
// special case on the diagonal.
// Every decision of the method is taken on wave-reduced, wave-uniform values (the free set
// is a 64-bit ballot), so the 64 lanes never diverge.
// Sums use a butterfly of lane swaps (every lane ends with the same bits). What one row passes to
// the others (an operand of a product, a row of a panel, a substitution's results) rides on the
// multiply-add that uses it, as a row broadcast: sixteen values lie in the sixteen lanes of every
// 16-lane row, and a multiply-add takes one of them for its whole row. That is one instruction
// where a pair of readlanes and the multiply-add were three, and its chain is shorter. The
// Cholesky factorisation is blocked in panels of 16 columns: FP64 matrix-core products form each
// panel from the columns before it, and the panel is factored in registers (chol_lds); the
// substitutions run in blocks of 16 rows. Per batch, against the form that broadcast by readlane
// and solved row by row: 2,048 x n = 64 0.85 -> 0.59 ms, 4,096 x n = 48 0.64 -> 0.45 ms, 10,000 x
// n = 24 0.55 -> 0.45 ms, 1,024 x n = 100 2.32 -> 1.56 ms, bitwise the same results.
//
// The steps and readings are those of lane_tron.hpp (Algorithm 1 with the TRON ratio test,
// the step measured in the trust region's norm, and the trapezoid reduction near rounding
// level); only the data layout differs.
#pragma once

#include "lane_tron.hpp"

namespace mt {

// DPP lane permutation within 16-lane rows (VALU only, no LDS traffic)
template <int CTRL>
MT_INLINE double dpp_mov(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
constexpr int kDppSwap1 = 0xB1;      // quad_perm [1,0,3,2]
constexpr int kDppSwap2 = 0x4E;      // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <- 7 - i within 8 lanes
constexpr int kDppMirror = 0x140;     // lane i <- 15 - i within 16 lanes

MT_INLINE double bcast(double v, int src);

// Sum over the 64 lanes; every lane returns the same bits: within each 16-lane row the
// partners of every step are combined commutatively, and the four row sums are read back
// and added in one fixed order.
MT_INLINE double wave_sum(double v)
{
    v += dpp_mov<kDppSwap1>(v);
    v += dpp_mov<kDppSwap2>(v);
    v += dpp_mov<kDppHalfMirror>(v);
    v += dpp_mov<kDppMirror>(v);
    return (bcast(v, 0) + bcast(v, 16)) + (bcast(v, 32) + bcast(v, 48));
}

// make a value the compiler treats as per-lane into a scalar (all lanes hold the same bits)
MT_INLINE double uni(double v)
{
    const int lo = __builtin_amdgcn_readfirstlane(__double2loint(v));
    const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
    return __hiloint2double(hi, lo);
}

MT_INLINE double bcast(double v, int src)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}

MT_INLINE double max_nan(double a, double b) { return (b > a || b != b) ? b : a; }  // NaN propagates

MT_INLINE double wave_max(double v)
{
    v = max_nan(v, dpp_mov<kDppSwap1>(v));
    v = max_nan(v, dpp_mov<kDppSwap2>(v));
    v = max_nan(v, dpp_mov<kDppHalfMirror>(v));
    v = max_nan(v, dpp_mov<kDppMirror>(v));
    return max_nan(max_nan(bcast(v, 0), bcast(v, 16)), max_nan(bcast(v, 32), bcast(v, 48)));
}

// Row broadcasts read lanes that must be switched on: none of these stands in a condition that
// differs between lanes. A source written just before takes two wait states.

// value of lane S of each 16-lane row in every lane of the row
template <int S>
MT_INLINE double row_bcast(double v)
{
    double d;
    asm volatile("s_nop 1\n\t"
        "v_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
        : "=v"(d) : "v"(v), "n"(S));
    return d;
}
// d -= (value of q in lane S of the lane's 16-lane row) * m, in one instruction. The broadcast
// rides on the multiply-add (its source register may have been written just before, which
// takes two wait states), so a row of a panel's update costs one instruction, not three.
template <int S>
MT_INLINE void fnma_row(double &d, double q, double m)
{
    asm volatile("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
        : "+&v"(d) : "v"(q), "v"(m), "n"(S));
}
// d0..d3 -= (q in lanes S, S + 1, S + 2, S + 3) * m
template <int S>
MT_INLINE void fnma_row4(double &d0, double &d1, double &d2, double &d3, double q, double m)
{
    asm volatile("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, -%5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %4, -%5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %4, -%5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %4, -%5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+&v"(d0), "+&v"(d1), "+&v"(d2), "+&v"(d3)
        : "v"(q), "v"(m), "n"(S), "n"(S + 1), "n"(S + 2), "n"(S + 3));
}
// d += (q in lane S) m0 + (q in lane S + 1) m1 + ..., one after the other
template <int S>
MT_INLINE void fma_row4(double &d, double q, double m0, double m1, double m2, double m3)
{
    asm volatile("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+&v"(d)
        : "v"(q), "v"(m0), "v"(m1), "v"(m2), "v"(m3), "n"(S), "n"(S + 1), "n"(S + 2), "n"(S + 3));
}
// d -= (q in lane S) m0, then lane S + D, S + 2 D, S + 3 D
template <int S, int D>
MT_INLINE void fnma_row4x(double &d, double q, double m0, double m1, double m2, double m3)
{
    asm volatile("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, -%2 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, -%3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, -%4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, -%5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+&v"(d)
        : "v"(q), "v"(m0), "v"(m1), "v"(m2), "v"(m3), "n"(S), "n"(S + D), "n"(S + 2 * D), "n"(S + 3 * D));
}
// d -= (q0 in lane S) m0, then (q1 in lane S) m1: a column pair of a triangular solve, its even
// column into e and its odd one into o
template <int S>
MT_INLINE void fnma_pair(double &e, double &o, double q0, double m0, double q1, double m1)
{
    asm volatile("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, -%3 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %4, -%5 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
        : "+&v"(e), "+&v"(o) : "v"(q0), "v"(m0), "v"(q1), "v"(m1), "n"(S));
}
// d0..d3 += (q in lanes S, S + 1, S + 2, S + 3) * (m0..m3)
template <int S>
MT_INLINE void fma_row4a(double &d0, double &d1, double &d2, double &d3, double q, double m0, double m1, double m2, double m3)
{
    asm volatile("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %4, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %4, %7 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %4, %8 row_newbcast:%12 row_mask:0xf bank_mask:0xf"
        : "+&v"(d0), "+&v"(d1), "+&v"(d2), "+&v"(d3)
        : "v"(q), "v"(m0), "v"(m1), "v"(m2), "v"(m3), "n"(S), "n"(S + 1), "n"(S + 2), "n"(S + 3));
}

// Sums of a column C of a triangular solve by columns: p0 and p1 less the products of columns C1
// .. E - 1 (even ones from p0, odd ones from p1) of the lane's entries t with the pivot row's,
// which lane C of each 16-lane row holds in q.
template <int C, int C1, int E>
MT_INLINE void row_sums(const double (&t)[16], const double (&q)[16], double &p0, double &p1)
{
    if constexpr (C1 + 1 < E) {
        fnma_pair<C>(p0, p1, q[C1], t[C1], q[C1 + 1], t[C1 + 1]);
        row_sums<C, C1 + 2, E>(t, q, p0, p1);
    } else if constexpr (C1 < E) {
        fnma_row<C>(p0, q[C1], t[C1]);  // C1 is even
    }
}

// One 16 x 16 diagonal block of a substitution, a row per lane of each 16-lane row: step by step
// the row's result b dv goes to the others (l: the lane's entries in the block, 0 where it is not
// to be changed). kUp: from the last row to the first. Four steps at a time, those past the
// block's `rows` rows left out.
template <int S, bool kUp>
MT_INLINE void block_steps(double &b, double dv, const double (&l)[16])
{
    constexpr int D = kUp ? -1 : 1, F = kUp ? S + 3 : S;
    fnma_row<F>(b, b * dv, l[F]);
    fnma_row<F + D>(b, b * dv, l[F + D]);
    fnma_row<F + 2 * D>(b, b * dv, l[F + 2 * D]);
    fnma_row<F + 3 * D>(b, b * dv, l[F + 3 * D]);
}
template <bool kUp>
MT_INLINE void block_solve(double &b, double dv, const double (&l)[16], int rows)
{
    if constexpr (kUp) {
        if (rows > 12) block_steps<12, true>(b, dv, l);
        if (rows > 8) block_steps<8, true>(b, dv, l);
        if (rows > 4) block_steps<4, true>(b, dv, l);
        block_steps<0, true>(b, dv, l);
    } else {
        block_steps<0, false>(b, dv, l);
        if (rows <= 4) return;
        block_steps<4, false>(b, dv, l);
        if (rows <= 8) return;
        block_steps<8, false>(b, dv, l);
        if (rows <= 12) return;
        block_steps<12, false>(b, dv, l);
    }
}
// b less the products of 16 results (lane t of each 16-lane row holds result t in y) with l
template <bool kUp>
MT_INLINE void block_update(double &b, double y, const double (&l)[16])
{
    constexpr int D = kUp ? -1 : 1, F = kUp ? 15 : 0;
    fnma_row4x<F, D>(b, y, l[F], l[F + D], l[F + 2 * D], l[F + 3 * D]);
    fnma_row4x<F + 4 * D, D>(b, y, l[F + 4 * D], l[F + 5 * D], l[F + 6 * D], l[F + 7 * D]);
    fnma_row4x<F + 8 * D, D>(b, y, l[F + 8 * D], l[F + 9 * D], l[F + 10 * D], l[F + 11 * D]);
    fnma_row4x<F + 12 * D, D>(b, y, l[F + 12 * D], l[F + 13 * D], l[F + 14 * D], l[F + 15 * D]);
}

// Objective families of the wave kernel. Each holds its own per-lane data and supplies
//   load(s, p)     read the instance's parameters (after the solver has read l, u, x0);
//   fg(s, v, g)    f(v) and its gradient on the lane's rows (0 on rows >= n);
//   hess(s)        the Hessian at s.x: its diagonal into s.hd, its strict upper triangle
//                  into the LDS array s.M when it depends on x.
// QP4: f = x'Qx/2 + c'x + kappa sum x_i^4 (Q packed lower by rows, then c, then kappa); the
// strict upper triangle of H is Q's and is written once at load.
template <int R_>
struct WaveFamQP4 {
    static constexpr int R = R_;
    double qd[R], c[R];  // Q's diagonal and c on the lane's rows
    double kap;

    template <class S>
    MT_INLINE void load(S &s, const double *__restrict__ p)
    {
        const int n = s.n;
        const double *cp = p + n * (n + 1) / 2;
        kap = cp[n];
        MT_UNROLL for (int r = 0; r < R; r++) {
            const int i = s.row(r);
            const bool in = i < n;
            const int k = in ? i : 0;
            qd[r] = in ? p[k * (k + 1) / 2 + k] : 0.0;
            c[r] = in ? cp[k] : 0.0;
        }
        // strict upper part of Q (row i, column j > i = packed lower entry (j, i)); at each j
        // the lanes i < j read consecutive addresses
        for (int j = 1; j < n; j++) {
            MT_UNROLL for (int r = 0; r < R; r++) {
                const int i = s.row(r);
                if (i < j) s.M[i * s.ld + j] = p[j * (j + 1) / 2 + i];
            }
        }
    }

    template <class S>
    MT_INLINE double fg(const S &s, const double (&v)[R], double (&gr)[R]) const
    {
        double y[R];
        s.amul(v, qd, y);
        double acc = 0.0;
        MT_UNROLL for (int r = 0; r < R; r++) {
            const double x2 = v[r] * v[r];
            gr[r] = s.valid(r) ? fma(4.0 * kap * x2, v[r], y[r] + c[r]) : 0.0;
            acc = fma(v[r], fma(0.5, y[r], c[r]), acc);
            acc = fma(kap * x2, x2, acc);
        }
        return uni(wave_sum(acc));
    }

    template <class S>
    MT_INLINE void hess(S &s) const
    {
        MT_UNROLL for (int r = 0; r < R; r++) {
            s.hd[r] = fma(12.0 * kap * s.x[r], s.x[r], qd[r]);
            if (s.valid(r)) s.M[s.row(r) * (s.ld + 1)] = s.hd[r];
        }
        s.sync();
    }
};

// HS45M: f = 120 - prod_k x_k (no parameters). Products run over k in ascending order with
// the excluded factors replaced by 1 (exact), so f and every gradient component carry the
// rounding of the plain left-to-right product.
template <int R_>
struct WaveFamHS45M {
    static constexpr int R = R_;

    template <class S>
    MT_INLINE void load(S &, const double *__restrict__) {}

    // step(0), step(1), ... step(n - 1), four to a turn of the loop. The solve takes an iteration or
    // two, so these loops and hess()'s backward sweep are much of it: a column at a time against
    // four, 12,000 instances of n = 24 54.5 / 51.4 us, of n = 40 83.6 / 76.1, 1,000 of n = 128
    // 219 / 184.
    template <class F>
    static MT_INLINE void in_fours(int n, F step)
    {
        int k = 0;
        for (; k + 4 <= n; k += 4) MT_UNROLL for (int u = 0; u < 4; u++) step(k + u);
        for (; k < n; k++) step(k);
    }

    template <class S>
    MT_INLINE double fg(const S &s, const double (&v)[R], double (&gr)[R]) const
    {
        double pr = 1.0, q[R];
        MT_UNROLL for (int r = 0; r < R; r++) q[r] = 1.0;
        in_fours(s.n, [&](int k) {
            const double xk = s.comp(v, k);
            pr *= xk;
            MT_UNROLL for (int r = 0; r < R; r++) q[r] *= s.row(r) == k ? 1.0 : xk;
        });
        MT_UNROLL for (int r = 0; r < R; r++) gr[r] = s.valid(r) ? -q[r] : 0.0;
        return 120.0 - pr;
    }

    // H_ij = -prod_{k != i, j} x_k, H_ii = 0. Row i is the product of prefix and suffix
    // products of y = x with y_i = 1: H_ij = -(prod_{k < j} y_k)(prod_{k > j} y_k). The prefix
    // is stored in the strict upper row, then scaled by the suffix in a backward sweep.
    template <class S>
    MT_INLINE void hess(S &s) const
    {
        const int n = s.n, ld = s.ld;
        double pre[R];
        MT_UNROLL for (int r = 0; r < R; r++) pre[r] = 1.0;
        in_fours(n, [&](int j) {
            const double xj = s.comp(s.x.v, j);
            MT_UNROLL for (int r = 0; r < R; r++) {
                const int i = s.row(r);
                if (i < j) s.M[i * ld + j] = pre[r];
                pre[r] *= i == j ? 1.0 : xj;
            }
        });
        // four columns at a time, their reads under way together
        double suf[R];
        MT_UNROLL for (int r = 0; r < R; r++) suf[r] = 1.0;
        auto back = [&](int j, const double (&m)[R]) {
            const double xj = s.comp(s.x.v, j);
            MT_UNROLL for (int r = 0; r < R; r++) {
                const int i = s.row(r);
                if (i < j) s.M[i * ld + j] = -(m[r] * suf[r]);
                suf[r] *= i == j ? 1.0 : xj;
            }
        };
        int j = n - 1;
        for (; j >= 3; j -= 4) {
            double m[4][R];
            MT_UNROLL for (int u = 0; u < 4; u++)
                MT_UNROLL for (int r = 0; r < R; r++) m[u][r] = s.M[(s.valid(r) ? s.row(r) : 0) * ld + j - u];
            MT_UNROLL for (int u = 0; u < 4; u++) back(j - u, m[u]);
        }
        for (; j >= 0; j--) {
            double m[R];
            MT_UNROLL for (int r = 0; r < R; r++) m[r] = s.M[(s.valid(r) ? s.row(r) : 0) * ld + j];
            back(j, m);
        }
        MT_UNROLL for (int r = 0; r < R; r++) {
            s.hd[r] = 0.0;
            if (s.valid(r)) s.M[s.row(r) * (ld + 1)] = 0.0;
        }
        s.sync();
    }
};

// The vector-level steps of one solve on a wavefront, shared by the solvers that differ in
// where the matrices live and who works on them (WaveTron here, BlockTron in block_tron.hpp).
// Lane l holds rows l + 64 r, r < R, of every vector. Derived supplies the matrix steps:
//   hmul(v, y)              y = H v
//   fg(v, g)                f(v) and its gradient
//   model(s, hs, v, gt, ft) hs = H s and, when it is cheaper together, f and gradient at v
//                           (returns whether it evaluated them)
//   hess()                  the Hessian at x
//   precond(fm), fwd, bwd, step_norm, sync() after the start point is projected, and
//   before_accept() when the last readers of x and g may still be on their way.
// Vec holds the vectors that live through the whole solve: in registers (RegVec) or, where R
// rows per lane of each would not fit, in LDS (LdsVec).
template <int R>
struct RegVec {
    double v[R];
    MT_INLINE double &operator[](int r) { return v[r]; }
    MT_INLINE double operator[](int r) const { return v[r]; }
};
// the lane's rows 64 r of an array in LDS; every wave of a workgroup stores the same values
typedef __attribute__((address_space(3))) double lds_double;
struct LdsVec {
    lds_double *v;
    MT_INLINE lds_double &operator[](int r) { return v[64 * r]; }
    MT_INLINE const lds_double &operator[](int r) const { return v[64 * r]; }
};

template <class Derived, int R_, class Vec = RegVec<R_>>
struct TronSteps {
    static constexpr int R = R_;
    int n;
    mutable int lane;          // (see renew)
    Vec hd;                    // H diagonal (own rows)
    Vec lo, hi, x, g;
    double xs[R];
    double hc[R];              // H (xs - x) while hc_ok: the accepted Cauchy trial's product
    bool hc_ok;
    bool has_l;
    double f, delta, alphac;
    int32_t iters;

    MT_INLINE Derived &self() { return static_cast<Derived &>(*this); }
    MT_INLINE const Derived &self() const { return static_cast<const Derived &>(*this); }
    MT_INLINE int row(int r) const { return lane + 64 * r; }
    MT_INLINE bool valid(int r) const { return row(r) < n; }

    // Called where a matrix step starts. With Derived::kTight the compiler takes the lane number for
    // a new one, so that the addresses the step derives from it live in the step; it would else
    // compute them all before the solve's first iteration, which costs registers throughout.
    MT_INLINE void renew() const
    {
        if constexpr (Derived::kTight) asm volatile("" : "+v"(lane));
    }

    template <class A, class B>
    MT_INLINE double dot(const A &a, const B &b) const
    {
        double s = 0.0;
        MT_UNROLL for (int r = 0; r < R; r++) s = fma(a[r], b[r], s);
        return uni(wave_sum(s));
    }

    // component k (< n) of a row-distributed vector, the same in every lane
    MT_INLINE double comp(const double (&v)[R], int k) const
    {
        double t = v[0];
        MT_UNROLL for (int r = 1; r < R; r++) t = (k >> 6) == r ? v[r] : t;
        return bcast(t, k & 63);
    }

    MT_INLINE double pg_inf() const
    {
        double m = 0.0;
        MT_UNROLL for (int r = 0; r < R; r++) m = fmax(m, valid(r) ? fabs(pg_comp(x[r], lo[r], hi[r], g[r])) : 0.0);
        return uni(wave_max(m));
    }

    MT_INLINE double pg_nrm2() const
    {
        double s = 0.0;
        MT_UNROLL for (int r = 0; r < R; r++) {
            const double v = valid(r) ? pg_comp(x[r], lo[r], hi[r], g[r]) : 0.0;
            s = fma(v, v, s);
        }
        return sqrt(uni(wave_sum(s)));
    }

    // bit j of a row-distributed mask; a select chain rather than a runtime index, so the
    // mask stays in registers for every R
    MT_INLINE bool is_free(const uint64_t (&fm)[R], int j) const
    {
        uint64_t w = fm[0];
        MT_UNROLL for (int r = 1; r < R; r++) w = (j >> 6) == r ? fm[r] : w;
        return (w >> (j & 63)) & 1ull;
    }
    MT_INLINE bool own_free(const uint64_t (&fm)[R], int r) const { return (fm[r] >> lane) & 1ull; }

    MT_INLINE double trqsol(const double (&v)[R], const double (&p)[R]) const
    {
        const double ptx = dot(p, v), ptp = dot(p, p), xtx = dot(v, v);
        const double dsq = delta * delta;
        double disc = fma(ptx, ptx, ptp * (dsq - xtx));
        disc = disc < 0.0 ? 0.0 : disc;
        const double rad = sqrt(disc);
        const double sig = ptx >= 0.0 ? (dsq - xtx) / (ptx + rad) : (rad - ptx) / ptp;
        return sig > 0.0 ? sig : 0.0;
    }

    // have: the norm test let the product hs = H (xt - x) be formed
    MT_INLINE bool cauchy_trial(double a, double (&xt)[R], double (&hs)[R], bool &have)
    {
        double st[R];
        MT_UNROLL for (int r = 0; r < R; r++) {
            xt[r] = clampf(fma(-a, g[r], x[r]), lo[r], hi[r]);
            st[r] = xt[r] - x[r];
        }
        have = dot(st, st) <= delta * delta;
        if (!have) return false;
        self().hmul(st, hs);
        double ss[R];
        MT_UNROLL for (int r = 0; r < R; r++) ss[r] = fma(0.5, hs[r], g[r]);
        const double gts = dot(g, st);
        const double q = dot(st, ss);  // g's + s'Hs/2
        return q <= kMu0 * gts;
    }

    MT_INLINE bool below_last_breakpoint(double a) const
    {
        bool any = false, below = false;
        MT_UNROLL for (int r = 0; r < R; r++) {
            const double d = -g[r];
            const bool up = valid(r) && d > 0.0 && isfinite(hi[r]);
            const bool dn = valid(r) && d < 0.0 && isfinite(lo[r]);
            any = any || up || dn;
            below = below || (up && a * d < hi[r] - x[r]) || (dn && a * d > lo[r] - x[r]);
        }
        const bool wany = __ballot(any) != 0ull, wbelow = __ballot(below) != 0ull;
        return !wany || wbelow;
    }

    // From the stored step length: extrapolate by 10 while acceptable and below the largest
    // breakpoint, keeping the last acceptable point, else interpolate by 0.1 until acceptable.
    MT_INLINE void cauchy()
    {
        double a = alphac, at = a;
        int t = 0;
        bool up = false;  // extrapolating: xs holds an acceptable point
        for (;;) {
            double xt[R], ht[R];
            bool have;
            const bool ok = cauchy_trial(at, xt, ht, have);
            if (up && !ok) break;
            a = at;
            hc_ok = have;
            MT_UNROLL for (int r = 0; r < R; r++) {
                xs[r] = xt[r];
                hc[r] = ht[r];
            }
            if (ok) {
                up = up || t == 0;
                if (!up || t == kCauchyMax || !below_last_breakpoint(a)) break;
                at = 10.0 * a;
            } else {
                if (t == kCauchyMax) break;
                at = 0.1 * a;
            }
            t++;
        }
        alphac = a;
    }

    MT_INLINE void free_mask(const double (&v)[R], uint64_t (&fm)[R]) const
    {
        MT_UNROLL for (int r = 0; r < R; r++) fm[r] = __ballot(valid(r) && lo[r] < v[r] && v[r] < hi[r]);
    }

    // exact: no shift was needed, so the preconditioned matrix is the identity and the first
    // CG step, s_hat = r_hat cut at the radius, is the whole solve (see lane_tron.hpp)
    MT_INLINE int pcg(const uint64_t (&fm)[R], int m, const double (&rv)[R], double (&sh)[R],
                      double cg_rtol, bool exact)
    {
        double rh[R], p[R];
        MT_UNROLL for (int r = 0; r < R; r++) {
            rh[r] = own_free(fm, r) ? -rv[r] : 0.0;
            sh[r] = 0.0;
        }
        self().fwd(rh);
        MT_UNROLL for (int r = 0; r < R; r++) p[r] = rh[r];
        double rr = dot(rh, rh);
        if (rr == 0.0) return kCgConv;
        if (exact) {
            if (rr >= delta * delta) {
                const double sig = trqsol(sh, p);
                MT_UNROLL for (int r = 0; r < R; r++) sh[r] = sig * p[r];
                return kCgBnd;
            }
            MT_UNROLL for (int r = 0; r < R; r++) sh[r] = p[r];
            return kCgConv;
        }
        const double tol2 = cg_rtol * cg_rtol * rr;
        for (int j = 0; j < m; j++) {
            double z[R], q[R];
            MT_UNROLL for (int r = 0; r < R; r++) z[r] = p[r];
            self().bwd(z);
            self().hmul(z, q);
            MT_UNROLL for (int r = 0; r < R; r++) q[r] = own_free(fm, r) ? q[r] : 0.0;
            self().fwd(q);
            const double kap_ = dot(p, q);
            if (!(kap_ > 0.0)) {
                const double sig = trqsol(sh, p);
                MT_UNROLL for (int r = 0; r < R; r++) sh[r] = fma(sig, p[r], sh[r]);
                return kCgNeg;
            }
            const double a = rr / kap_;
            double tv[R];
            MT_UNROLL for (int r = 0; r < R; r++) tv[r] = fma(a, p[r], sh[r]);
            if (dot(tv, tv) >= delta * delta) {
                const double sig = trqsol(sh, p);
                MT_UNROLL for (int r = 0; r < R; r++) sh[r] = fma(sig, p[r], sh[r]);
                return kCgBnd;
            }
            MT_UNROLL for (int r = 0; r < R; r++) {
                sh[r] = tv[r];
                rh[r] = fma(-a, q[r], rh[r]);
            }
            const double rrn = dot(rh, rh);
            if (rrn <= tol2) return kCgConv;
            const double b = rrn / rr;
            MT_UNROLL for (int r = 0; r < R; r++) p[r] = fma(b, p[r], rh[r]);
            rr = rrn;
        }
        return kCgMaxit;
    }

    MT_INLINE void subspace(double cg_rtol)
    {
        has_l = false;
        for (int pass = 0; pass < n; pass++) {
            uint64_t fm[R];
            free_mask(xs, fm);
            int m = 0;
            MT_UNROLL for (int r = 0; r < R; r++) m += __builtin_popcountll(fm[r]);
            if (m == 0) break;
            // the first pass starts from the Cauchy point, whose trial has formed this product
            double s[R], rv[R];
            if (!hc_ok) {
                MT_UNROLL for (int r = 0; r < R; r++) s[r] = xs[r] - x[r];
                self().hmul(s, hc);
            }
            hc_ok = false;
            MT_UNROLL for (int r = 0; r < R; r++) rv[r] = hc[r] + g[r];
            const double shift = self().precond(fm);
            has_l = true;
            double w[R];
            const int ex = pcg(fm, m, rv, w, cg_rtol, shift == 0.0);
            self().bwd(w);
            double beta = 1.0;
            bool acc = false;
            double xt[R];
            for (int t = 0; t <= kSearchHalvings; t++) {
                double d[R], hdv[R];
                MT_UNROLL for (int r = 0; r < R; r++) {
                    xt[r] = clampf(fma(beta, w[r], xs[r]), lo[r], hi[r]);
                    d[r] = xt[r] - xs[r];
                }
                self().hmul(d, hdv);
                double hh[R];
                MT_UNROLL for (int r = 0; r < R; r++) hh[r] = fma(0.5, hdv[r], rv[r]);
                const double rd = dot(rv, d);
                const double dq = dot(d, hh);  // r'd + d'Hd/2
                if (dq <= kMu0 * rd) { acc = true; break; }
                beta *= 0.5;
            }
            if (acc) MT_UNROLL for (int r = 0; r < R; r++) xs[r] = xt[r];
            uint64_t fm2[R];
            free_mask(xs, fm2);
            bool newly = false;
            MT_UNROLL for (int r = 0; r < R; r++) newly = newly || (fm[r] & ~fm2[r]) != 0ull;
            if (!((ex == kCgConv || ex == kCgMaxit) && newly)) break;
        }
    }

    MT_INLINE double radius_update(double rho, double ared, double gts, double snorm, bool fin) const
    {
        double astar;
        if (!fin) {
            astar = kSig1;
            rho = -__builtin_inf();
        } else {
            const double gam = -ared - gts;
            if (gam <= 0.0) astar = kSig3;
            else {
                astar = -0.5 * gts / gam;
                if (astar < kSig1) astar = kSig1;
            }
        }
        if (rho <= kEta0) return dmin((astar > kSig1 ? astar : kSig1) * snorm, kSig2 * delta);
        if (rho <= kEta1) return dmax(kSig1 * delta, dmin(astar * snorm, kSig2 * delta));
        if (rho < kEta2) return dmax(kSig1 * delta, dmin(astar * snorm, kSig3 * delta));
        return dmax(delta, dmin(astar * snorm, kSig3 * delta));
    }

    MT_INLINE int32_t solve(const Options &o, double delta_in, double alphac_in)
    {
        iters = 0;
        delta = 0.0;
        alphac = 1.0;
        f = __builtin_nan("");
        bool bad = false;
        MT_UNROLL for (int r = 0; r < R; r++) bad = bad || (valid(r) && !(lo[r] <= hi[r]));
        if (__ballot(bad) != 0ull) return kBadBounds;
        MT_UNROLL for (int r = 0; r < R; r++) x[r] = clampb(x[r], lo[r], hi[r]);
        self().sync();
        {
            double x1[R], g1[R];
            MT_UNROLL for (int r = 0; r < R; r++) x1[r] = x[r];
            f = self().fg(x1, g1);
            MT_UNROLL for (int r = 0; r < R; r++) g[r] = g1[r];
        }
        bool fin = true;
        MT_UNROLL for (int r = 0; r < R; r++) fin = fin && isfinite(g[r]);
        fin = isfinite(f) && __ballot(!fin) == 0ull;
        if (!fin) return kNonfinite;
        if (pg_inf() <= o.gtol) return kConverged;
        if (o.warm && delta_in > 0.0) delta = delta_in;
        else if (o.delta0 > 0.0) delta = o.delta0;
        else {
            delta = pg_nrm2();
            if (delta == 0.0) delta = 1.0;
        }
        if (o.warm && alphac_in > 0.0) alphac = alphac_in;
        self().hess();
        int32_t status;
        for (;;) {
            cauchy();
            subspace(o.cg_rtol);
            double s[R], hs[R];
            MT_UNROLL for (int r = 0; r < R; r++) s[r] = xs[r] - x[r];
            const double snorm = self().step_norm(s);
            double gt[R], ft = 0.0;
            const bool have_ft = self().model(s, hs, xs, gt, ft);
            double hh[R];
            MT_UNROLL for (int r = 0; r < R; r++) hh[r] = fma(0.5, hs[r], g[r]);
            const double gts = dot(g, s);
            const double pred = -dot(s, hh);
            iters++;
            if (!(pred > 0.0)) { status = kStalled; break; }
            if (!have_ft) ft = self().fg(xs, gt);
            const bool tfin = isfinite(ft);
            double ared = f - ft;
            if (tfin && pred <= kAredSwitch * (fabs(f) > 1.0 ? fabs(f) : 1.0)) {
                double sg[R];
                MT_UNROLL for (int r = 0; r < R; r++) sg[r] = g[r] + gt[r];
                ared = -0.5 * dot(sg, s);
            }
            const double rho = tfin ? ared / pred : -__builtin_inf();
            delta = radius_update(rho, ared, gts, snorm, tfin);
            const bool accept = rho > kEta0;
            if (accept) {
                self().before_accept();
                MT_UNROLL for (int r = 0; r < R; r++) { x[r] = xs[r]; g[r] = gt[r]; }
                f = ft;
            }
            bool ok = true;
            MT_UNROLL for (int r = 0; r < R; r++) ok = ok && isfinite(g[r]);
            ok = isfinite(f) && __ballot(!ok) == 0ull;
            if (!ok) { status = kNonfinite; break; }
            if (pg_inf() <= o.gtol) { status = kConverged; break; }
            if (iters >= o.max_iter) { status = kMaxIter; break; }
            const double tiny = kStallRel * (fabs(f) > 1.0 ? fabs(f) : 1.0);
            if (tfin && fabs(ared) <= tiny && pred <= tiny) { status = kStalled; break; }
            if (accept) self().hess();
        }
        return status;
    }
};

// One trust-region Newton solve per wave for the family Fam, Fam::R rows per lane
// (n <= 64 R).
// kGlobal: the matrix array M lives in global memory (a device workspace, when the plan asks for
// it) instead of LDS; only the scope of the ordering between the lanes' writes and reads changes.
// kTight: the build has fewer registers than the solve's addresses want (see renew).
template <class Fam, bool kGlobal = false, bool kTight_ = false>
struct WaveTron : TronSteps<WaveTron<Fam, kGlobal, kTight_>, Fam::R> {
    static constexpr int R = Fam::R;
    static constexpr bool kTight = kTight_;
    using Steps = TronSteps<WaveTron<Fam, kGlobal, kTight_>, Fam::R>;
    using Steps::n;
    using Steps::lane;
    using Steps::hd;
    using Steps::lo;
    using Steps::hi;
    using Steps::x;
    using Steps::has_l;
    using Steps::row;
    using Steps::renew;
    using Steps::valid;
    using Steps::dot;
    using Steps::comp;
    using Steps::is_free;
    using Steps::own_free;

    // order LDS writes before other lanes' LDS reads (the wave's LDS operations run in order)
    MT_INLINE void lds_sync() const
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // make every lane's writes to M visible to every lane of the wave
    MT_INLINE void sync() const
    {
        if (kGlobal) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
    Fam fam;
    int ld;
    double *M;                 // LDS: H upper with diagonal, L strict lower, pivots in column n
    double *P;                 // with M in global memory: LDS copy of a panel's 16 x 16 block
                               // of L (row stride 17), so that its columns meet at wave scope
    double *Q;                 // with M in global memory: kStage steps of each lane's entries of
                               // L, parked in LDS by the substitutions (slot (t R + r) 64 + lane)
    static constexpr int kStage = 8;
    double dinv[R], pv[R];     // the factor's reciprocal pivots and pivots (own rows)

    // H_kj (upper triangle, diagonal included) sits at min(j,k) ld + max(j,k) = min(j,k)
    // (ld - 1) + j + k: with blk = M + k + j0 for a block of columns j = j0 + u (u a
    // constant after unrolling), the j0 + k part is the block's base, u an immediate offset,
    // and the rest one 24-bit multiply-add into a byte offset (indices stay far below 2^24);
    // ldb = 8 (ld - 1)
    MT_INLINE double hrd(const double *blk, unsigned ldb, int k, int j, int u) const
    {
        if constexpr (kGlobal) {
            // in global memory a 32-bit element index off the wave's uniform base keeps the
            // loads in their scalar-base form (a per-lane 64-bit base costs more than it saves)
            const int a = j < k ? j : k, b = j < k ? k : j;
            return M[(int)__umul24((unsigned)a, (unsigned)ld) + b];
        } else {
            const unsigned m = (unsigned)(j < k ? j : k);
            return *(const double *)((const char *)blk + __umul24(m, ldb) + 8 * u);
        }
    }

    // A copy of v in column n (rows < n), from which every lane reads back the 16 entries its
    // 16-lane row broadcasts in turn.
    MT_INLINE void spread(const double (&v)[R]) const
    {
        MT_UNROLL for (int r = 0; r < R; r++)
            if (valid(r)) M[(int)__umul24((unsigned)row(r), (unsigned)ld) + n] = v[r];
        lds_sync();
    }
    MT_INLINE double chunk(int k) const
    {
        const int i = 16 * k + (lane & 15);
        return M[(int)__umul24((unsigned)(i < n ? i : 0), (unsigned)ld) + n];
    }

    // acc[r][u] = sum over j = u mod 4 of entry(r, j0, u) v_j (j = j0 + u, u a constant), the
    // columns past the last multiple of 4 in acc[r][0]. A product is one instruction: v_j rides on
    // it by a row broadcast, 16 columns (what is left of them: 4 at a time) from one copy of v's
    // entries; with n < 16 the one 16-lane row that has rows holds v itself.
    template <class E>
    MT_INLINE void products(const double (&v)[R], E entry, double (&acc)[R][4]) const
    {
        MT_UNROLL for (int r = 0; r < R; r++) acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0;
        const int n4 = n & ~3;
        int j0 = 0;
        double q = v[0];
        if (n >= 16) {
            spread(v);
            q = chunk(0);
#pragma unroll 1
            for (; j0 + 16 <= n; j0 += 16) {
                const double vq = q;
                if (j0 + 16 < n4) q = chunk((j0 >> 4) + 1);
                MT_UNROLL for (int r = 0; r < R; r++) {
                    double e[16];
                    MT_UNROLL for (int u = 0; u < 16; u++) e[u] = entry(r, j0, u);
                    fma_row4a<0>(acc[r][0], acc[r][1], acc[r][2], acc[r][3], vq, e[0], e[1], e[2], e[3]);
                    fma_row4a<4>(acc[r][0], acc[r][1], acc[r][2], acc[r][3], vq, e[4], e[5], e[6], e[7]);
                    fma_row4a<8>(acc[r][0], acc[r][1], acc[r][2], acc[r][3], vq, e[8], e[9], e[10], e[11]);
                    fma_row4a<12>(acc[r][0], acc[r][1], acc[r][2], acc[r][3], vq, e[12], e[13], e[14], e[15]);
                }
            }
        }
        if (j0 < n4) {
            MT_UNROLL for (int r = 0; r < R; r++) {
                double e[12];
                MT_UNROLL for (int u = 0; u < 4; u++) e[u] = entry(r, j0, u);
                if (j0 + 4 < n4) MT_UNROLL for (int u = 4; u < 8; u++) e[u] = entry(r, j0, u);
                if (j0 + 8 < n4) MT_UNROLL for (int u = 8; u < 12; u++) e[u] = entry(r, j0, u);
                fma_row4a<0>(acc[r][0], acc[r][1], acc[r][2], acc[r][3], q, e[0], e[1], e[2], e[3]);
                if (j0 + 4 < n4) fma_row4a<4>(acc[r][0], acc[r][1], acc[r][2], acc[r][3], q, e[4], e[5], e[6], e[7]);
                if (j0 + 8 < n4) fma_row4a<8>(acc[r][0], acc[r][1], acc[r][2], acc[r][3], q, e[8], e[9], e[10], e[11]);
            }
        }
#pragma unroll 1
        for (j0 = n4; j0 < n; j0++) {
            const double vj = this->comp(v, j0);
            MT_UNROLL for (int r = 0; r < R; r++) acc[r][0] = fma(entry(r, j0, 0), vj, acc[r][0]);
        }
    }

    // y = H v over the first n rows (H's diagonal read from LDS, as hess() stored it); rows
    // >= n give 0. Four independent accumulators per row; no lane-dependent branches.
    MT_INLINE void hmul(const double (&v)[R], double (&y)[R]) const
    {
        if constexpr (kGlobal) {
            hmul_global(v, y);
            return;
        }
        renew();
        double acc[R][4];
        int kk[R];
        MT_UNROLL for (int r = 0; r < R; r++) kk[r] = row(r) < n ? row(r) : 0;
        const unsigned ldb = 8u * (unsigned)(ld - 1);
        products(v, [&](int r, int j0, int u) { return hrd(M + kk[r] + j0, ldb, kk[r], j0 + u, u); }, acc);
        MT_UNROLL for (int r = 0; r < R; r++)
            y[r] = valid(r) ? (acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3]) : 0.0;
    }

    // y = A v over the first n rows, A = H's off-diagonal part with diagonal diag (QP4's f
    // and gradient use Q's diagonal); rows >= n give 0. H's diagonal makes way for the product.
    template <class D>
    MT_INLINE void diagonal(const D &d) const
    {
        MT_UNROLL for (int r = 0; r < R; r++)
            if (valid(r)) M[(int)__umul24((unsigned)row(r), (unsigned)(ld + 1))] = d[r];
    }
    MT_INLINE void amul(const double (&v)[R], const double (&diag)[R], double (&y)[R]) const
    {
        if constexpr (kGlobal) {
            amul_global(v, diag, y);
            return;
        }
        diagonal(diag);
        hmul(v, y);
        diagonal(hd);
        lds_sync();
    }

    // the same with M in global memory: a 32-bit index off the wave's uniform base, components
    // of v by readlane
    MT_INLINE void hmul_global(const double (&v)[R], double (&y)[R]) const
    {
        double acc[R][4];
        int kk[R];
        MT_UNROLL for (int r = 0; r < R; r++) {
            acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0;
            kk[r] = row(r) < n ? row(r) : 0;
        }
        const unsigned ldb = 8u * (unsigned)(ld - 1);
        MT_UNROLL for (int rr = 0; rr < R; rr++) {
            const int jend = n - 64 * rr < 64 ? n - 64 * rr : 64;
            int jj = 0;
            for (; jj + 4 <= jend; jj += 4) {
                double vj[4];
                MT_UNROLL for (int u = 0; u < 4; u++) vj[u] = bcast(v[rr], jj + u);
                MT_UNROLL for (int r = 0; r < R; r++) {
                    const double *blk = M + kk[r] + 64 * rr + jj;
                    MT_UNROLL for (int u = 0; u < 4; u++)
                        acc[r][u] = fma(hrd(blk, ldb, kk[r], 64 * rr + jj + u, u), vj[u], acc[r][u]);
                }
            }
            for (; jj < jend; jj++) {
                const double vj = bcast(v[rr], jj);
                MT_UNROLL for (int r = 0; r < R; r++)
                    acc[r][0] = fma(hrd(M + kk[r] + 64 * rr + jj, ldb, kk[r], 64 * rr + jj, 0), vj, acc[r][0]);
            }
        }
        MT_UNROLL for (int r = 0; r < R; r++)
            y[r] = valid(r) ? (acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3]) : 0.0;
    }


    MT_INLINE void amul_global(const double (&v)[R], const double (&diag)[R], double (&y)[R]) const
    {
        double acc[R][4];
        int kk[R];
        MT_UNROLL for (int r = 0; r < R; r++) {
            acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0;
            kk[r] = row(r) < n ? row(r) : 0;
        }
        const unsigned ldb = 8u * (unsigned)(ld - 1);
        MT_UNROLL for (int rr = 0; rr < R; rr++) {
            const int jend = n - 64 * rr < 64 ? n - 64 * rr : 64;
            int jj = 0;
            for (; jj + 4 <= jend; jj += 4) {
                double vj[4];
                MT_UNROLL for (int u = 0; u < 4; u++) vj[u] = bcast(v[rr], jj + u);
                MT_UNROLL for (int r = 0; r < R; r++) {
                    const double *blk = M + kk[r] + 64 * rr + jj;
                    MT_UNROLL for (int u = 0; u < 4; u++) {
                        const int j = 64 * rr + jj + u;
                        const double h = hrd(blk, ldb, kk[r], j, u);
                        acc[r][u] = fma(j == kk[r] ? diag[r] : h, vj[u], acc[r][u]);
                    }
                }
            }
            for (; jj < jend; jj++) {
                const double vj = bcast(v[rr], jj);
                MT_UNROLL for (int r = 0; r < R; r++) {
                    const int j = 64 * rr + jj;
                    const double h = hrd(M + kk[r] + j, ldb, kk[r], j, 0);
                    acc[r][0] = fma(j == kk[r] ? diag[r] : h, vj, acc[r][0]);
                }
            }
        }
        MT_UNROLL for (int r = 0; r < R; r++)
            y[r] = valid(r) ? (acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3]) : 0.0;
    }

    MT_INLINE void load(const double *__restrict__ p, const double *__restrict__ lop,
                        const double *__restrict__ hip_, const double *__restrict__ x0p)
    {
        MT_UNROLL for (int r = 0; r < R; r++) {
            const int i = row(r);
            const bool in = i < n;
            const int k = in ? i : 0;
            lo[r] = in ? lop[k] : 0.0;
            hi[r] = in ? hip_[k] : 0.0;
            x[r] = in ? x0p[k] : 0.0;
        }
        fam.load(*this, p);
    }

    MT_INLINE double fg(const double (&v)[R], double (&gr)[R]) const { return fam.fg(*this, v, gr); }

    MT_INLINE void hess() { fam.hess(*this); }

    MT_INLINE void before_accept() const {}

    MT_INLINE bool model(const double (&s)[R], double (&hs)[R], const double (&)[R], double (&)[R], double &) const
    {
        hmul(s, hs);
        return false;
    }

    // Cholesky factor of H_FF + alpha I with the identity outside F: the factor's strict lower
    // triangle into M's lower part, its pivots into column n, their reciprocals into dinv.
    // False when a pivot of a free column is not positive (the caller then raises alpha).
    MT_INLINE bool chol(const uint64_t (&fm)[R], double alpha)
    {
        if constexpr (kGlobal) return chol_panels(fm, alpha);
        else return chol_lds(fm, alpha);
    }

    // Entry (k, j), k >= j, of H_FF + alpha I with the identity outside F, and 0 above the
    // diagonal and outside the first n rows and columns. k and j may differ between lanes.
    MT_INLINE double shifted(const uint64_t (&fm)[R], int k, int j, double alpha) const
    {
        const bool in = k < n && j < n && k >= j;
        // H_jk from the upper triangle; the address is clamped rather than branched on
        const double h = M[in ? (int)__umul24((unsigned)j, (unsigned)ld) + k : 0];
        const bool fj = is_free(fm, j);
        const double e = k == j ? (fj ? h + alpha : 1.0) : ((fj && is_free(fm, k)) ? h : 0.0);
        return in ? e : 0.0;
    }

    // Factor the 16 columns j0 .. j0 + 15 of S (left in the factor's slots, its diagonal in
    // column n), left-looking, a column at a time. Every 16-lane row holds the panel's own 16 rows
    // (sv; what stands right of their diagonal is whatever was there and meets only itself), so
    // that the entries of a pivot row reach every lane by row broadcasts; each lane also holds
    // its own rows below the panel (t, kBelow). The serial chain per column is the pivot's last
    // update, its broadcast, the reciprocal square root and the scale; the sums of the next
    // column up to its last but one term fill the waits. Entries of rows and columns outside F
    // need no masks: S is the identity there, so they stay exact zeros beside pivots of 1. The
    // pivots before their square roots go to column n.
    template <int C, bool kBelow>
    MT_INLINE void panel_column(double (&sv)[16], double (&t)[R][16], double (&e)[2], double s0, const double (&w0)[R],
                                double dg, int j0, const int (&irow)[R], double *const (&dst)[R], bool &bad)
    {
        if constexpr (C < 16) {
            if (!kBelow && j0 + C >= n) return;
            double own = dg;
            if constexpr (C > 0) own = fma(-sv[C - 1], sv[C - 1], e[0] + e[1]);
            const double d = row_bcast<C>(own);
            const double rinv = rsqrt_pos(d);
            double s = s0, w[R];
            MT_UNROLL for (int r = 0; r < R; r++) w[r] = w0[r];
            if constexpr (C > 0) {
                fnma_row<C>(s, sv[C - 1], sv[C - 1]);
                if constexpr (kBelow) MT_UNROLL for (int r = 0; r < R; r++) fnma_row<C>(w[r], sv[C - 1], t[r][C - 1]);
            }
            double sn = 0.0, wn[R];
            if constexpr (C + 1 < 16) {
                double p1 = 0.0;
                sn = sv[C + 1];
                row_sums<C + 1, 0, C>(sv, sv, sn, p1);
                sn = sn + p1;
                MT_UNROLL for (int r = 0; r < R; r++) {
                    wn[r] = 0.0;
                    if constexpr (kBelow) {
                        double q1 = 0.0;
                        wn[r] = t[r][C + 1];
                        row_sums<C + 1, 0, C>(t[r], sv, wn[r], q1);
                        wn[r] = wn[r] + q1;
                    }
                }
            }
            if constexpr (C > 0) e[(C - 1) & 1] = fma(-sv[C - 1], sv[C - 1], e[(C - 1) & 1]);
            const int j = j0 + C;
            bad = bad || !(d > 0.0);
            M[(int)__umul24((unsigned)j, (unsigned)ld) + n] = d;
            sv[C] = s * rinv;
            MT_UNROLL for (int r = 0; r < R; r++) {
                if constexpr (kBelow) t[r][C] = w[r] * rinv;
                if (irow[r] > j) dst[r][C] = kBelow ? t[r][C] : sv[C];
            }
            panel_column<C + 1, kBelow>(sv, t, e, sn, wn, dg, j0, irow, dst, bad);
        }
    }

    // 16 consecutive entries of a row of M, those past column n - 1 replaced by others (columns
    // of a partial panel that are not there)
    MT_INLINE void row16(const double *p, int cols, double (&v)[16]) const
    {
        if (cols >= 16) MT_UNROLL for (int c = 0; c < 16; c++) v[c] = p[c];
        else MT_UNROLL for (int c = 0; c < 16; c++) v[c] = p[c < cols ? c : 0];
    }

    template <bool kBelow>
    MT_INLINE bool panel_factor(int j0)
    {
        renew();
        const int il = lane & 15, cols = n - j0;
        const int ip = il < cols ? j0 + il : j0;
        const double *pr = M + (int)__umul24((unsigned)ip, (unsigned)ld);
        double sv[16], t[R][16], e[2], w0[R];
        const double dg = pr[n];
        if constexpr (kBelow) MT_UNROLL for (int c = 0; c < 16; c++) sv[c] = pr[j0 + c];
        else row16(pr + j0, cols, sv);
        int irow[R];
        double *dst[R];
        MT_UNROLL for (int r = 0; r < R; r++) {
            // the lane's row to store: its own where the panel's rows hold for all lanes, or
            // where that is one of the panel's rows
            const int i = row(r);
            const bool in = i < n && (kBelow || (i >= j0));
            irow[r] = in ? i : -1;
            dst[r] = M + (int)__umul24((unsigned)(in ? i : 0), (unsigned)ld) + j0;
            if constexpr (kBelow) MT_UNROLL for (int c = 0; c < 16; c++) t[r][c] = dst[r][c];
            w0[r] = kBelow ? t[r][0] : 0.0;
        }
        e[0] = dg;
        e[1] = 0.0;
        bool bad = false;
        panel_column<0, kBelow>(sv, t, e, sv[0], w0, dg, j0, irow, dst, bad);
        lds_sync();
        return __builtin_amdgcn_readfirstlane((int)bad) == 0;
    }

    // S's starting values at the 16 x 16 block of row k0, column j0 (lane: row lq + 4 v, column
    // lr): A = H_FF + alpha I with the identity outside F. Entries outside the lower part of the
    // first n rows are not kept.
    MT_INLINE void block_start(const uint64_t (&fm)[R], int k0, int j0, double alpha, double (&e)[4]) const
    {
        const int lr = lane & 15, lq = lane >> 4;
        const int jb = j0 + lr, jbk = jb < n ? jb : n - 1;
        const uint32_t fj = (uint32_t)(mask_word(fm, j0 >> 6) >> (j0 & 63)) >> lr;
        const uint32_t fk = (fj & 1u) ? (uint32_t)(mask_word(fm, k0 >> 6) >> (k0 & 63)) >> lq : 0u;
        const double *p = M + (int)__umul24((unsigned)jbk, (unsigned)ld);
        MT_UNROLL for (int v = 0; v < 4; v++) {
            const int i0 = k0 + lq + 4 * v, i = i0 < n ? i0 : n - 1;
            const double h = p[i];
            e[v] = ((fk >> (4 * v)) & 1u) ? h : 0.0;
            if (k0 == j0) e[v] = lq + 4 * v == lr ? ((fj & 1u) ? h + alpha : 1.0) : e[v];
        }
    }
    MT_INLINE uint64_t mask_word(const uint64_t (&fm)[R], int q) const
    {
        uint64_t t = fm[0];
        MT_UNROLL for (int r = 1; r < R; r++) t = q == r ? fm[r] : t;
        return t;
    }

    // Blocked left-looking factorisation in panels of 16 columns. For the panel starting at
    // column j0, the matrix cores form S = A[j0:n, panel] - L[j0:n, 0:j0] L[panel, 0:j0]^T,
    // 16 x 16 blocks by 16 x 16 x 4 FP64 products (operands read from LDS once, no
    // broadcasts); then panel_factor.
    // Lane layout of the 16 x 16 x 4 FP64 product: A(i, k) in lane i + 16 k, B(k, j) in lane
    // j + 16 k, C(i, j) in lane j + 16 (i mod 4), element i / 4 of the lane's four. Rows and
    // columns past n read row n - 1; their results are not kept.
    MT_INLINE bool chol_lds(const uint64_t (&fm)[R], double alpha)
    {
        renew();
        typedef double d4 __attribute__((ext_vector_type(4)));
        const int lr = lane & 15, lq = lane >> 4;
#pragma unroll 1
        for (int j0 = 0; j0 < n; j0 += 16) {
            const int jb = j0 + lr, jbk = jb < n ? jb : n - 1;
            const double *rb = M + (int)__umul24((unsigned)jbk, (unsigned)ld) + lq;
#pragma unroll 1
            for (int k0 = j0; k0 < n; k0 += 16) {
                const int kak = k0 + lr < n ? k0 + lr : n - 1;
                const double *ra = M + (int)__umul24((unsigned)kak, (unsigned)ld) + lq;
                double e[4];
                block_start(fm, k0, j0, alpha, e);
                d4 acc0, acc1 = {0.0, 0.0, 0.0, 0.0};
                MT_UNROLL for (int v = 0; v < 4; v++) acc0[v] = e[v];
#pragma unroll 1
                for (int q0 = 0; q0 < j0; q0 += 16) {
                    double a[4], b[4];
                    MT_UNROLL for (int v = 0; v < 4; v++) {
                        a[v] = -ra[q0 + 4 * v];
                        b[v] = rb[q0 + 4 * v];
                    }
                    acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], b[0], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1], b[1], acc1, 0, 0, 0);
                    acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2], b[2], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[3], b[3], acc1, 0, 0, 0);
                }
                MT_UNROLL for (int v = 0; v < 4; v++) {
                    const int k = k0 + lq + 4 * v;
                    // S below the diagonal into the factor's slots, its diagonal into column n
                    if (k < n && jb < n && k >= jb)
                        M[(int)__umul24((unsigned)k, (unsigned)ld) + (k == jb ? n : jb)] = acc0[v] + acc1[v];
                }
            }
            lds_sync();
            if (!(j0 + 16 < n ? panel_factor<true>(j0) : panel_factor<false>(j0))) return false;
        }
        MT_UNROLL for (int r = 0; r < R; r++) {
            const double d = M[(int)__umul24((unsigned)(valid(r) ? row(r) : 0), (unsigned)ld) + n];
            const double rinv = rsqrt_pos(d);
            const bool fr = valid(r) && own_free(fm, r);
            dinv[r] = fr ? rinv : 1.0;
            pv[r] = fr ? d * rinv : 1.0;
        }
        return true;
    }

    // The same panel step with M in global memory, in two passes that
    // keep 16 values per lane live instead of 16 per row slot. First the register slot that
    // holds the panel's rows, pipelined as above, with the panel's 16 x 16 block of L and its
    // pivot reciprocals mirrored in LDS (P, row stride 17, reciprocal in column 16) so that
    // its columns meet at wave scope; then every later slot by a triangular solve against
    // that block, its entries read from LDS at one address in every lane.
    MT_INLINE bool panel_factor_split(const uint64_t (&fm)[R], int j0)
    {
        const int rp = j0 >> 6;
        const int i = lane + 64 * rp;
        const bool ownf = i < n && is_free(fm, i);
        double sv[16], pv = 1.0, dv = 1.0;
        MT_UNROLL for (int c = 0; c < 16; c++) {
            const int j = j0 + c;
            const bool in = i < n && i >= j;
            const double v = M[in ? (int)__umul24((unsigned)i, (unsigned)ld) + (i == j ? n : j) : 0];
            sv[c] = in ? v : 0.0;
        }
        bool bad = false;
        MT_UNROLL for (int c = 0; c < 16; c++) {
            const int j = j0 + c;
            if (j >= n) break;
            double pre[16];
            if (c + 1 < 16) MT_UNROLL for (int c1 = 0; c1 < c; c1++) pre[c1] = P[(c + 1) * 17 + c1];
            double own = sv[c];
            if (c > 0) own = fma(-sv[c - 1], sv[c - 1], own);
            const double d = uni(bcast(own, j & 63));
            if (c > 0) {
                const double l = bcast(sv[c - 1], j & 63);
                sv[c] = fma(-sv[c - 1], l, sv[c]);
            }
            const bool fj = is_free(fm, j);
            bad = bad || (fj && !(d > 0.0));
            const double rinv = fj ? rsqrt_pos(fj ? d : 1.0) : 1.0;
            const double piv = fj ? d * rinv : 1.0;
            sv[c] = (fj && ownf) ? sv[c] * rinv : 0.0;
            pv = i == j ? piv : pv;
            dv = i == j ? rinv : dv;
            if (i < n && i > j) M[__umul24((unsigned)i, (unsigned)ld) + j] = sv[c];
            if (i > j && i < j0 + 16) P[(i - j0) * 17 + c] = sv[c];
            if (lane == 0) P[c * 17 + 16] = rinv;
            if (c + 1 < 16) {
                double p0 = sv[c + 1], p1 = 0.0;
                MT_UNROLL for (int c1 = 0; c1 < c; c1++) {
                    if (c1 & 1) p1 = fma(-sv[c1], pre[c1], p1);
                    else p0 = fma(-sv[c1], pre[c1], p0);
                }
                sv[c + 1] = p0 + p1;
            }
            lds_sync();
        }
        const bool inp = i >= j0 && i < j0 + 16 && i < n;
        if (inp) M[__umul24((unsigned)i, (unsigned)ld) + n] = pv;
        MT_UNROLL for (int r = 0; r < R; r++) dinv[r] = (r == rp && inp) ? dv : dinv[r];
        // rows of the later slots: L(i, j0 + c) = (S(i, j0 + c) - sum_{c1 < c} L(i, j0 + c1)
        // L(j0 + c, j0 + c1)) / L(j0 + c, j0 + c)
        for (int r2 = rp + 1; r2 < R && 64 * r2 < n; r2++) {
            const int i2 = lane + 64 * r2;
            const bool in2 = i2 < n;
            const bool f2 = in2 && is_free(fm, i2);
            const int base = (int)__umul24((unsigned)(in2 ? i2 : 0), (unsigned)ld) + j0;
            double t[16];
            MT_UNROLL for (int c = 0; c < 16; c++) {
                const double v = M[base + c];
                t[c] = in2 ? v : 0.0;
            }
            MT_UNROLL for (int c = 0; c < 16; c++) {
                if (j0 + c >= n) break;
                double p0 = t[c], p1 = 0.0;
                MT_UNROLL for (int c1 = 0; c1 < c; c1++) {
                    const double l = P[c * 17 + c1];
                    if (c1 & 1) p1 = fma(-t[c1], l, p1);
                    else p0 = fma(-t[c1], l, p0);
                }
                t[c] = (is_free(fm, j0 + c) && f2) ? (p0 + p1) * P[c * 17 + 16] : 0.0;
                if (in2) M[base + c] = t[c];
            }
        }
        sync();
        return !bad;
    }

    // The same with M in global memory, the operands of eight chunks loaded per trip to L2.
    MT_INLINE bool chol_panels(const uint64_t (&fm)[R], double alpha)
    {
        typedef double d4 __attribute__((ext_vector_type(4)));
        const int lr = lane & 15, lq = lane >> 4;
        for (int j0 = 0; j0 < n; j0 += 16) {
            const int jb = j0 + lr;  // this lane's panel column (B row, C column)
            const int jbk = jb < n ? jb : 0;
            for (int k0 = j0; k0 < n; k0 += 16) {
                const int ka = k0 + lr;  // this lane's A row
                const int kak = ka < n ? ka : 0;
                d4 acc0, acc1 = {0.0, 0.0, 0.0, 0.0};
                MT_UNROLL for (int v = 0; v < 4; v++) acc0[v] = shifted(fm, k0 + lq + 4 * v, jb, alpha);
                const double *ra = M + __umul24((unsigned)kak, (unsigned)ld) + lq;
                const double *rb = M + __umul24((unsigned)jbk, (unsigned)ld) + lq;
                // rows past n read row 0 (always present) and use 0
                const bool ain = ka < n, bin = jb < n;
                int q0 = 0;
                for (; q0 + 32 <= j0; q0 += 32) {
                    double av[8], bv[8];
                    MT_UNROLL for (int u = 0; u < 8; u++) {
                        av[u] = ra[q0 + 4 * u];
                        bv[u] = rb[q0 + 4 * u];
                    }
                    MT_UNROLL for (int u = 0; u < 8; u += 2) {
                        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(ain ? -av[u] : 0.0, bin ? bv[u] : 0.0, acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(ain ? -av[u + 1] : 0.0, bin ? bv[u + 1] : 0.0, acc1, 0, 0, 0);
                    }
                }
                for (; q0 + 8 <= j0; q0 += 8) {
                    const double a0 = ra[q0], b0 = rb[q0], a1 = ra[q0 + 4], b1 = rb[q0 + 4];
                    acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(ain ? -a0 : 0.0, bin ? b0 : 0.0, acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(ain ? -a1 : 0.0, bin ? b1 : 0.0, acc1, 0, 0, 0);
                }
                if (q0 < j0) {
                    const double a0 = ra[q0], b0 = rb[q0];
                    acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(ain ? -a0 : 0.0, bin ? b0 : 0.0, acc0, 0, 0, 0);
                }
                MT_UNROLL for (int v = 0; v < 4; v++) {
                    const int k = k0 + lq + 4 * v;
                    // S below the diagonal into the factor's slots, its diagonal into column n
                    if (k < n && jb < n && k >= jb)
                        M[__umul24((unsigned)k, (unsigned)ld) + (k == jb ? n : jb)] = acc0[v] + acc1[v];
                }
            }
            sync();
            if (!panel_factor_split(fm, j0)) return false;
        }
        return true;
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
        for (int t = 0; t < kShiftTries; t++) {
            if (chol(fm, alpha)) return alpha;
            alpha = 2.0 * alpha > beta ? 2.0 * alpha : beta;
        }
        for (int j = 0; j < n; j++) {
            MT_UNROLL for (int r = 0; r < R; r++) {
                const int i = row(r);
                if (i < n && i > j) M[__umul24((unsigned)i, (unsigned)ld) + j] = 0.0;
            }
        }
        MT_UNROLL for (int r = 0; r < R; r++) {
            const int i = row(r);
            if (i < n) {
                const double v = fabs(hd[r]);
                const double piv = own_free(fm, r) ? sqrt(v > beta ? v : beta) : 1.0;
                if constexpr (kGlobal) M[__umul24((unsigned)i, (unsigned)ld) + n] = piv;
                pv[r] = piv;
                dinv[r] = 1.0 / piv;
            }
        }
        sync();
        return -1.0;
    }

    // component j of b * dinv, taken from its owner lane (wave-uniform result)
    MT_INLINE double owner_scaled(const double (&b)[R], int j) const
    {
        double v = b[0] * dinv[0];
        MT_UNROLL for (int r = 1; r < R; r++) v = (j >> 6) == r ? b[r] * dinv[r] : v;
        return bcast(v, j & 63);
    }

    // The steps of a substitution in blocks of 16 rows, kUp false: L y = b, true: L^T y = b (then
    // from the last block to the first). The block's 16-lane row runs its 16 steps by row
    // broadcasts, its results go to column n, and every row still to come subtracts their 16
    // columns. b keeps unscaled residuals.
    template <bool kUp>
    MT_INLINE void substitute(double (&b)[R]) const
    {
        renew();
        const int il = lane & 15, nb = (n + 15) >> 4;
        double dl[16];
#pragma unroll 1
        for (int q = 0; q < nb; q++) {
            const int blk = kUp ? nb - 1 - q : q, sl = blk >> 2, j0 = 16 * blk;
            if (q == 0 || (blk & 3) == (kUp ? 3 : 0)) {
                // the lane's entries in the diagonal block of its own row in this slot
                // (rows past n, whose residuals are 0, stay 0 and pass 0 on)
                const int i = lane + 64 * sl, ik = i < n ? i : n - 1, i0 = i - il;
                const int from = i < n ? il : kUp ? 16 : 0;
                // byte offsets along the row (or down the column), kept inside the array
                const unsigned step = kUp ? 8u * (unsigned)ld : 8u;
                const unsigned at = 8u * (kUp ? __umul24((unsigned)i0, (unsigned)ld) + (unsigned)ik : __umul24((unsigned)ik, (unsigned)ld) + (unsigned)i0);
                const unsigned last = at + (unsigned)(n - 1 - i0) * step;
                MT_UNROLL for (int t = 0; t < 16; t++) {
                    const unsigned o = at + (unsigned)t * step;
                    const double v = *(const double *)((const char *)M + (o < last ? o : last));
                    dl[t] = (kUp ? t > from : t < from) ? v : 0.0;
                }
            }
            double tb = b[0], dv = dinv[0];
            MT_UNROLL for (int r = 1; r < R; r++) {
                tb = sl == r ? b[r] : tb;
                dv = sl == r ? dinv[r] : dv;
            }
            const int own = lane + 64 * sl;
            dv = own < n ? dv : 1.0;
            const bool more = q + 1 < nb;
            // entries of the rows still to come, loaded ahead of the block's steps
            double l[R][16];
            if (more) {
                MT_UNROLL for (int r = 0; r < R; r++) {
                    if (R > 1 && (kUp ? r > sl : r < sl)) continue;
                    const int ik = valid(r) ? row(r) : 0;
                    MT_UNROLL for (int t = 0; t < 16; t++) {
                        if (kUp) l[r][t] = M[(int)__umul24((unsigned)(j0 + t < n ? j0 + t : n - 1), (unsigned)ld) + ik];
                        else l[r][t] = M[(int)__umul24((unsigned)ik, (unsigned)ld) + j0 + t];
                    }
                }
            }
            double t = tb;
            block_solve<kUp>(t, dv, dl, n - j0);
            const bool mine = (lane >> 4) == (blk & 3);
            tb = mine ? t : tb;
            MT_UNROLL for (int r = 0; r < R; r++) b[r] = sl == r ? tb : b[r];
            if (!more) break;
            const double y = tb * dv;
            if (mine && own < n) M[(int)__umul24((unsigned)own, (unsigned)ld) + n] = y;
            lds_sync();
            const int iy = j0 + il;
            const double y0 = M[(int)__umul24((unsigned)(iy < n ? iy : 0), (unsigned)ld) + n];
            const double yq = iy < n ? y0 : 0.0;
            MT_UNROLL for (int r = 0; r < R; r++) {
                if (R > 1 && (kUp ? r > sl : r < sl)) continue;
                double u = b[r];
                block_update<kUp>(u, yq, l[r]);
                const bool left = valid(r) && (kUp ? row(r) < j0 : row(r) >= j0 + 16);
                b[r] = left ? u : b[r];
            }
        }
    }

    // L y = b in place (b zero outside the factored set stays zero). Each row keeps its
    // residual unscaled while the substitution runs and is scaled by its reciprocal pivot once
    // at the end (the value its own step would have taken): the step's chain is then the
    // owner's scaling, the broadcast and one FMA, with no select on it. Rows not below the
    // step subtract an exact zero.
    MT_INLINE void fwd(double (&b)[R]) const
    {
        if constexpr (kGlobal) {
            // M in global memory: the lane's entries of L for kStage steps are loaded together
            // (one trip to L2 per kStage steps instead of one per step) and parked in the lane's
            // own LDS slots, which only it reads back
            for (int j0 = 0; j0 < n; j0 += kStage) {
                MT_UNROLL for (int t = 0; t < kStage; t++) {
                    MT_UNROLL for (int r = 0; r < R; r++) {
                        const int i = row(r);
                        const bool below = i > j0 + t && i < n && j0 + t < n;
                        const double v = M[below ? (int)__umul24((unsigned)i, (unsigned)ld) + j0 + t : 0];
                        Q[(t * R + r) * 64 + lane] = below ? v : 0.0;
                    }
                }
                MT_UNROLL for (int t = 0; t < kStage; t++) {
                    if (j0 + t >= n) break;
                    const double yj = owner_scaled(b, j0 + t);
                    MT_UNROLL for (int r = 0; r < R; r++) b[r] = fma(-Q[(t * R + r) * 64 + lane], yj, b[r]);
                }
            }
        } else {
            substitute<false>(b);
        }
        MT_UNROLL for (int r = 0; r < R; r++) b[r] = valid(r) ? b[r] * dinv[r] : b[r];
    }

    // L^T y = b in place, the same way
    MT_INLINE void bwd(double (&b)[R]) const
    {
        if constexpr (kGlobal) {
            for (int j0 = ((n - 1) / kStage) * kStage; j0 >= 0; j0 -= kStage) {
                MT_UNROLL for (int t = 0; t < kStage; t++) {
                    MT_UNROLL for (int r = 0; r < R; r++) {
                        const int i = row(r);
                        const bool above = i < j0 + t && j0 + t < n;
                        const double v = M[above ? (int)__umul24((unsigned)(j0 + t), (unsigned)ld) + i : 0];
                        Q[(t * R + r) * 64 + lane] = above ? v : 0.0;
                    }
                }
                MT_UNROLL for (int t = kStage - 1; t >= 0; t--) {
                    if (j0 + t >= n) continue;
                    const double yj = owner_scaled(b, j0 + t);
                    MT_UNROLL for (int r = 0; r < R; r++) b[r] = fma(-Q[(t * R + r) * 64 + lane], yj, b[r]);
                }
            }
        } else {
            substitute<true>(b);
        }
        MT_UNROLL for (int r = 0; r < R; r++) b[r] = valid(r) ? b[r] * dinv[r] : b[r];
    }

    MT_INLINE double step_norm(const double (&s)[R]) const
    {
        if (!has_l) return sqrt(dot(s, s));
        // t = L^T s: t_i = L_ii s_i + sum_{k > i} L_ki s_k, in four partial sums by k mod 4
        // (entries of rows not below i count as exact zeros)
        if constexpr (!kGlobal) {
            double acc[R][4], t[R];
            int kk[R];
            MT_UNROLL for (int r = 0; r < R; r++) kk[r] = valid(r) ? row(r) : n;
            products(s, [&](int r, int k0, int u) {
                const bool in = kk[r] < k0 + u;
                const double l = M[(int)__umul24((unsigned)(k0 + u), (unsigned)ld) + (in ? kk[r] : 0)];
                return in ? l : 0.0;
            }, acc);
            MT_UNROLL for (int r = 0; r < R; r++)
                t[r] = valid(r) ? fma(pv[r], s[r], (acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3])) : 0.0;
            return sqrt(dot(t, t));
        }
        // t = L^T s: t_i = L_ii s_i + sum_{k > i} L_ki s_k (the pivot L_ii sits in column n), in
        // four independent partial sums, four broadcasts and loads at a time (entries of rows
        // not below i are read as exact zeros, no selects)
        double acc[R][4];
        MT_UNROLL for (int r = 0; r < R; r++) acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0;
        int k = 0;
        for (; k + 4 <= n; k += 4) {
            double sk[4];
            MT_UNROLL for (int u = 0; u < 4; u++) sk[u] = comp(s, k + u);
            MT_UNROLL for (int r = 0; r < R; r++) {
                const int i = row(r);
                MT_UNROLL for (int u = 0; u < 4; u++) {
                    const bool in = i < k + u;
                    const double l = M[in ? (int)__umul24((unsigned)(k + u), (unsigned)ld) + i : 0];
                    acc[r][u] = fma(in ? l : 0.0, sk[u], acc[r][u]);
                }
            }
        }
        for (; k < n; k++) {
            const double sk = comp(s, k);
            MT_UNROLL for (int r = 0; r < R; r++) {
                const int i = row(r);
                const bool in = i < k;
                const double l = M[in ? (int)__umul24((unsigned)k, (unsigned)ld) + i : 0];
                acc[r][0] = fma(in ? l : 0.0, sk, acc[r][0]);
            }
        }
        double t[R];
        MT_UNROLL for (int r = 0; r < R; r++) {
            const int i = row(r);
            const double piv = M[valid(r) ? (int)__umul24((unsigned)i, (unsigned)ld) + n : 0];
            t[r] = valid(r) ? fma(piv, s[r], (acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3])) : 0.0;
        }
        return sqrt(dot(t, t));
    }

};

}  // namespace mt
