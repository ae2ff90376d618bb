// Strip kernels: the batched render, the fused forward + adjoint and the per-visit
// background, all walking vertical strips of L pixels.
//
// Along a column the exponent of a Gaussian is a quadratic in the row offset, so the
// value at the next row is the current one times a ratio that itself shrinks by the
// constant factor exp(-P_yy) per row.  A lane therefore pays two exps per Gaussian per
// strip (value and first ratio at the strip's top row) and two multiplies per further
// row, instead of one exp per Gaussian per pixel; the result equals the direct
// evaluation up to a few ulps per row.  In the adjoint the per-row derivative terms are
// polynomials of degree <= 2 in the row offset, so each Gaussian contributes through
// three moments sum_k g_k, sum_k g_k k, sum_k g_k k^2 of its weighted values.
// Where the PSFs are wide enough the value and the ratio at the strip's centre and row factors
// shared by all lanes take the recurrence's place (stage_rows).
// Where they are so narrow that the value at a strip's top row could underflow above rows that
// count, the plan cuts lower strips (highest_strip in api.cpp).
//
// Work item = a run of up to `chunk` strips of one box (strip s of a box of width w:
// column s mod w, rows L (s / w) ... L (s / w) + L - 1 clipped to the box).  Lane j of a
// wave takes strips start + j, start + j + 64, ...; consecutive lanes hold consecutive
// columns, so pixel loads of one row are contiguous.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "internal.h"
#include "model.h"

namespace cel {

__device__ __forceinline__ double clamp_arg(double v) { return v < 700.0 ? v : 700.0; }
__device__ __forceinline__ dual clamp_arg(dual v) { return v.v < 700.0 ? v : mkd(700.0, 0.0); }

__device__ __forceinline__ void strip_geometry(const PairDev& p, int s, int L, int& c, int& r0, int& nrow) {
    const int rb = s / p.w;
    c = p.c0 + (s - rb * p.w);
    r0 = p.r0 + rb * L;
    nrow = min(L, p.h - rb * L);
}

// Value and first row ratio of component e at column px, top row py0.
template <class T>
__device__ __forceinline__ void strip_seed(const T* e, double px, double py0, T& n, T& rt, T& pdx0, T& pdy0,
                                           const double* __restrict__ t2) {
    const T dx = px - e[F_CX], dy = py0 - e[F_CY];
    pdx0 = e[F_PXX] * dx + e[F_PXY] * dy;
    pdy0 = e[F_PXY] * dx + e[F_PYY] * dy;
    n = fexp(e[F_LOGW] - 0.5 * (dx * pdx0 + dy * pdy0), t2);
    rt = fexp(clamp_arg(-(pdy0 + 0.5 * e[F_PYY])), t2);
}

// Pass A: star and galaxy profile values down the strip.
// SGN: also fgd[k] = sum of the de Vaucouleurs minus the exponential components (d fg /
// d frac_dev).
// live (with CULL): the components to evaluate (item_live); the others are skipped.
template <class T, int L, bool SGN = false, bool CULL = false>
__device__ __forceinline__ void strip_values(const T* __restrict__ tab, double px, double py0, T* fs, T* fg,
                                             const double* __restrict__ t2, T* fgd = nullptr,
                                             uint64_t live = ~0ull) {
    const T zero = scalar_traits<T>::make(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < L; ++k) fs[k] = fg[k] = zero;
    if constexpr (SGN) {
#pragma unroll
        for (int k = 0; k < L; ++k) fgd[k] = zero;
    }
#pragma unroll
    for (int c = 0; c < NPSF; ++c) {
        if (CULL && !((live >> c) & 1)) continue;
        const T* e = tab + c * CST;
        T n, rt, pdx0, pdy0;
        strip_seed(e, px, py0, n, rt, pdx0, pdy0, t2);
        const T rdy = e[F_RDY];
#pragma unroll
        for (int k = 0; k < L; ++k) {
            fs[k] += n;
            if (k + 1 < L) {
                n = n * rt;
                rt = rt * rdy;
            }
        }
    }
#pragma unroll scalar_traits<T>::gal_unroll
    for (int c = NPSF; c < NCOMP; ++c) {
        if (CULL && !((live >> c) & 1)) continue;
        const T* e = tab + c * CST;
        T n, rt, pdx0, pdy0;
        strip_seed(e, px, py0, n, rt, pdx0, pdy0, t2);
        const T rdy = e[F_RDY], wt = e[F_WT];
#pragma unroll
        for (int k = 0; k < L; ++k) {
            fg[k] += n * wt;
            if constexpr (SGN) fgd[k] += n * e[F_SGN];
            if (k + 1 < L) {
                n = n * rt;
                rt = rt * rdy;
            }
        }
    }
}

// Pass B: d/d(position, frac_dev, shape covariance) accumulated with per-row weights
// Gs (star) and Gg (galaxy).
template <class T, int L, bool CULL = false>
__device__ __forceinline__ void strip_adjoint(const T* __restrict__ tab, double px, double py0, const T* Gs,
                                              const T* Gg, T* acc, const double* __restrict__ t2,
                                              uint64_t live = ~0ull) {
    // Row moments by repeated running sums: with t_k = G_k value_k and u = L - k,
    //   A = sum t,  B = sum_k (sum_{i<=k} t_i) = sum t u,  C = sum_k (B after row k) = sum t u(u+1)/2,
    // so about the strip centre KC = (L-1)/2 (h = KC + 1 = (L+1)/2):
    //   m0 = sum t = A,  m1 = sum t (k-KC) = h A - B,  m2 = sum t (k-KC)^2 = h^2 A - (2h+1) B + 2C.
    // One fused multiply-add and two adds per row instead of a product and three accumulations.
    constexpr double KC = 0.5 * (L - 1);
    constexpr double H = KC + 1.0;
    const T zero = scalar_traits<T>::make(0.0, 0.0);
#pragma unroll
    for (int c = 0; c < NPSF; ++c) {
        if (CULL && !((live >> c) & 1)) continue;
        const T* e = tab + c * CST;
        T n, rt, pdx0, pdy0;
        strip_seed(e, px, py0, n, rt, pdx0, pdy0, t2);
        const T rdy = e[F_RDY];
        T A = zero, B = zero;
#pragma unroll
        for (int k = 0; k < L; ++k) {
            A += Gs[k] * n;
            B += A;
            if (k + 1 < L) {
                n = n * rt;
                rt = rt * rdy;
            }
        }
        const T m0 = A, m1 = H * A - B;
        const T pdxc = pdx0 + e[F_PXY] * KC, pdyc = pdy0 + e[F_PYY] * KC;
        acc[A_UX] += pdxc * m0 + e[F_PXY] * m1;
        acc[A_UY] += pdyc * m0 + e[F_PYY] * m1;
    }
#pragma unroll scalar_traits<T>::gal_unroll
    for (int c = NPSF; c < NCOMP; ++c) {
        if (CULL && !((live >> c) & 1)) continue;
        const T* e = tab + c * CST;
        T n, rt, pdx0, pdy0;
        strip_seed(e, px, py0, n, rt, pdx0, pdy0, t2);
        const T rdy = e[F_RDY];
        T A = zero, B = zero, C = zero;
#pragma unroll
        for (int k = 0; k < L; ++k) {
            A += Gg[k] * n;
            B += A;
            C += B;
            if (k + 1 < L) {
                n = n * rt;
                rt = rt * rdy;
            }
        }
        const T m0 = A, m1 = H * A - B, m2 = (H * H) * A - (2.0 * H + 1.0) * B + 2.0 * C;
        const T a = e[F_PXX], b = e[F_PXY], d = e[F_PYY];
        const T pdxc = pdx0 + b * KC, pdyc = pdy0 + d * KC;
        const T wt = e[F_WT], wnu = e[F_WNU];
        acc[A_FDEV] += e[F_SGN] * m0;
        acc[A_UX] += wt * (pdxc * m0 + b * m1);
        acc[A_UY] += wt * (pdyc * m0 + d * m1);
        acc[A_SXX] += wnu * ((pdxc * pdxc - a) * m0 + 2.0 * (pdxc * b) * m1 + (b * b) * m2);
        acc[A_SXY] += wnu * ((pdxc * pdyc - b) * m0 + (pdxc * d + pdyc * b) * m1 + (b * d) * m2);
        acc[A_SYY] += wnu * ((pdyc * pdyc - d) * m0 + 2.0 * (pdyc * d) * m1 + (d * d) * m2);
    }
}

// Pass B of the value-gradient adjoint from a box table staged in LDS.
// The star component and the 14 galaxy components of one PSF component share their centre
// (the source position plus that PSF component's offset), so the offsets dx = px - cx,
// dy = py0 - cy and their products are formed once per group and strip.  With
// P = [[a, b], [b, d]] and j = py0 + k - cy the row offset from the centre, a component's
// exponent is LW - (a dx^2 + 2 b dx dy + d dy^2) / 2 and its first row ratio
// exp(-(b dx + d dy) - d / 2), and every intermediate's contribution is a combination of
// the raw row moments M_i = sum_k t_k j^i (t_k = row weight x value).  With
// U = a dx M0 + b M1, U' = b dx M0 + d M1 (the sums of t (P (m - mu))_x and _y),
// W = a dx M1 + b M2 and W' = b dx M1 + d M2:
//   position:  wt U, wt U';    frac_dev: sgn M0;
//   shape xx:  wnu (a (dx U - M0) + b W),   xy: wnu (b (dx U - M0) + d W),
//   shape yy:  wnu (b dx U' + d (W' - M0)),
// (the sums of t ((P (m - mu))_x^2 - a), t ((P (m - mu))_x (P (m - mu))_y - b) and
// t ((P (m - mu))_y^2 - d)).  The moments come from the running sums A, B, C of the strip
// recurrence through the row-moment identity about a centre c with L - c = e = L + dy:
// M0 = A, M1 = e A - B, M2 = e^2 A - (2e + 1) B + 2C.  Per galaxy component this takes 29
// operations after the rows, against about 38 for the same fold about the strip centre with
// per-lane products of the precision, and the seed 6 instead of 12.
// Staged table: field-major, [NDF][NCP] (lane c writes component c's fields at stride NCP,
// no bank conflicts; every lane then reads the same words); stars at slots 0..2, galaxy
// group g at 4 + 14 g, so that the pairs of the unrolled galaxy loop are 16-byte aligned.
constexpr int NCP = 46;
enum DerivedField { D_CX = 0, D_CY, D_LW, D_RDY, D_A, D_B, D_D, D_WT, D_WNU, D_SGN, NDF };

__device__ __forceinline__ int staged_slot(int c) { return c < NPSF ? c : c + 1; }

// One wave writes the staged table of a box into its LDS slot (lane c: component c).  Lane
// NCOMP fills the spare slot NPSF with a component that is zero everywhere (log weight -1000,
// flat, every weight 0): the loops over the live components below pair an odd one with it.
__device__ __forceinline__ void stage_derived(const double* __restrict__ tab, double* my, int lane) {
    if (lane < NCOMP) {
        const double* e = tab + lane * CST;
        double* o = my + staged_slot(lane);
        o[D_CX * NCP] = e[F_CX];
        o[D_CY * NCP] = e[F_CY];
        o[D_LW * NCP] = e[F_LOGW];
        o[D_RDY * NCP] = e[F_RDY];
        o[D_A * NCP] = e[F_PXX];
        o[D_B * NCP] = e[F_PXY];
        o[D_D * NCP] = e[F_PYY];
        o[D_WT * NCP] = e[F_WT];
        o[D_WNU * NCP] = e[F_WNU];
        o[D_SGN * NCP] = e[F_SGN];
    } else if (lane == NCOMP) {
        double* o = my + NPSF;
        o[D_CX * NCP] = 0.0;
        o[D_CY * NCP] = 0.0;
        o[D_LW * NCP] = -1000.0;   // exp underflows to exactly 0
        o[D_RDY * NCP] = 1.0;
        o[D_A * NCP] = 0.0;
        o[D_B * NCP] = 0.0;
        o[D_D * NCP] = 0.0;
        o[D_WT * NCP] = 0.0;
        o[D_WNU * NCP] = 0.0;
        o[D_SGN * NCP] = 0.0;
    }
}

// Row factors.  About the strip's centre row (KC = (L - 1) / 2), a component's value in row k is
// n_k = N0 r^k q_|k - KC| with r = exp(-(b dx + d dy_c)) the lane's row ratio at the centre,
// N0 = n_c r^-KC and q_j+1/2 = exp(-d (j + 1/2)^2 / 2) the same for every lane: with the q in
// LDS (q_1/2 .. q_15/2 per component, staged with the table) a row of the value pass takes two
// operations per component (p *= r, f += q p) instead of the recurrence's three, and a row of
// the adjoint four instead of five (strip_adjoint_q).  It needs r^(L-1) and N0 within range:
// for P_yy = d <= 1.5, (b dx + d dy_c)^2 <= d (quadratic form at the centre), so where
// log r > 40 the exponent of N0 is below -40^2 / (2 d) - 40 KC: -833 at 16 rows (N0 is exactly
// 0), -673 at 8, -593 at 4.  With r clamped to e^40 there, N0 r^(L-1) stays below e^-393 of the
// component's scale, as do the rows' true values, so that the clamp cannot be seen; r^(L-1)
// stays below e^600 and N0 below e^42.  A component whose value in
// some row exceeds exp(-50) of its peak has log r < 24, so the terms are formed as exactly as
// with the recurrence from the top row.  Every component covariance holds its PSF
// component's, so d <= 1.5 everywhere when the PSF covariances' eigenvalues are at least
// 2/3 px^2 (sigma >= 0.82 px): the plan tests that (Geometry::smooth), and plans with a
// sharper PSF take the recurrence.
constexpr double LOG_R_MAX = 40.0;
constexpr int NQ = 8;   // row factors per component (L / 2 of them are used)

// One wave writes the row factors of a box's components into its LDS slot [NCP][NQ] (0 for the
// zero component): q_j+1 = q_j rho^(j+1), rho = exp(-d).
template <class T>
__device__ __forceinline__ void stage_rows(const T* __restrict__ tab, double* myq, int lane,
                                           const double* __restrict__ t2) {
    if (lane > NCOMP) return;
    double q[NQ];
    if (lane < NCOMP) {
        const T* e = tab + lane * CST;
        const double rho = value_of(e[F_RDY]);
        double pw = rho;
        q[0] = fexp(-0.125 * value_of(e[F_PYY]), t2);
#pragma unroll
        for (int j = 1; j < NQ; ++j) {
            q[j] = q[j - 1] * pw;
            pw *= rho;
        }
    } else {
#pragma unroll
        for (int j = 0; j < NQ; ++j) q[j] = 0.0;
    }
    double* o = myq + (lane < NCOMP ? staged_slot(lane) : NPSF) * NQ;
#pragma unroll
    for (int j = 0; j < NQ; j += 2) *reinterpret_cast<double2*>(o + j) = make_double2(q[j], q[j + 1]);
}

// Components that are negligible on every pixel of a work item are left out of its strips.
// The item's strips cover at most three rectangles of its box: the rest of its first band,
// whole bands, the start of its last band.  For P = [[a, b], [b, d]] positive definite,
// minimising the quadratic form over one coordinate gives
// (x, y) P (x, y)^T >= x^2 det P / d  and  >= y^2 det P / a,
// so a component whose form exceeds CULL_Q on each rectangle by one of these bounds stays
// below exp(-CULL_Q / 2) (< 2e-22) of its own peak on the whole item: far below the
// rounding of any pixel's expected count, which holds the sky.  Returns the live
// components as a wave-uniform bit set (bit c: table component c); lane c tests component c.
constexpr double CULL_Q = 100.0;

template <class T>
__device__ __forceinline__ uint64_t item_live(const T* __restrict__ tab, const PairDev& p, const Item& it, int L,
                                              int lane) {
    bool cull = false;
    if (lane < NCOMP) {
        const T* e = tab + lane * CST;
        const double cx = value_of(e[F_CX]), cy = value_of(e[F_CY]), a = value_of(e[F_PXX]),
                     b = value_of(e[F_PXY]), d = value_of(e[F_PYY]);
        const double det = fma(a, d, -(b * b));
        const double qa = CULL_Q * a, qd = CULL_Q * d;
        // > 0 if the form exceeds CULL_Q on columns ca..cb, rows ra..rb of the box
        auto far = [&](int ca, int cb, int ra, int rb) {
            const double x0 = (double)(p.c0 + ca) - cx, x1 = (double)(p.c0 + cb) - cx;
            const double y0 = (double)(p.r0 + ra) - cy, y1 = (double)(p.r0 + rb) - cy;
            const double ux = fmax(fmax(x0, -x1), 0.0), uy = fmax(fmax(y0, -y1), 0.0);
            return fmax(fma(ux * ux, det, -qd), fma(uy * uy, det, -qa));
        };
        const int s0 = it.start, s1 = it.start + it.count - 1;
        const int rb0 = s0 / p.w, rb1 = s1 / p.w;
        double m = far(s0 - rb0 * p.w, rb1 > rb0 ? p.w - 1 : s1 - rb0 * p.w, rb0 * L, min(rb0 * L + L, p.h) - 1);
        if (rb1 > rb0) {
            m = fmin(m, far(0, s1 - rb1 * p.w, rb1 * L, min(rb1 * L + L, p.h) - 1));
            if (rb1 > rb0 + 1) m = fmin(m, far(0, p.w - 1, (rb0 + 1) * L, rb1 * L - 1));
        }
        cull = a > 0.0 && det > 0.0 && m > 0.0 && cx - cx == 0.0 && cy - cy == 0.0;
    }
    return ~__builtin_amdgcn_ballot_w64(cull) & ((1ull << NCOMP) - 1);
}

// Staged slots of the live galaxy components of PSF group grp, two at a time (an odd last
// one paired with the zero component in slot NPSF).
template <class F>
__device__ __forceinline__ void for_live_pairs(uint64_t live, int grp, F&& f) {
    uint32_t gm = (uint32_t)(live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1);
    const int base = NPSF + 1 + grp * NGAL_PER_PSF;
    while (gm) {
        const int s0 = base + __builtin_ctz(gm);
        gm &= gm - 1;
        int s1 = NPSF;
        if (gm) {
            s1 = base + __builtin_ctz(gm);
            gm &= gm - 1;
        }
        f(s0, s1);
    }
}

// Values n[0..1] and first row ratios rt[0..1] of two components (staged table entries e0, e1;
// the fields of both staged layouts up to D_D coincide) in their PSF group's frame: both
// entries' fields read together, then the four exponentials together.
__device__ __forceinline__ void seed_pair(const double* __restrict__ e0, const double* __restrict__ e1, double h2x,
                                          double mxy, double h2y, double mdx, double mdyh, double* n, double* rt,
                                          const double* __restrict__ t2) {
    const double a0 = e0[D_A * NCP], b0 = e0[D_B * NCP], d0 = e0[D_D * NCP], l0 = e0[D_LW * NCP];
    const double a1 = e1[D_A * NCP], b1 = e1[D_B * NCP], d1 = e1[D_D * NCP], l1 = e1[D_LW * NCP];
    __builtin_amdgcn_sched_barrier(0);
    const double x[4] = {fma(a0, h2x, fma(b0, mxy, fma(d0, h2y, l0))), fma(a1, h2x, fma(b1, mxy, fma(d1, h2y, l1))),
                         clamp_arg(fma(b0, mdx, d0 * mdyh)), clamp_arg(fma(b1, mdx, d1 * mdyh))};
    double e[4];
    fexps<4>(x, e, t2);
    n[0] = e[0];
    n[1] = e[1];
    rt[0] = e[2];
    rt[1] = e[3];
}

// One galaxy component's rows and fold (strip_adjoint_staged) from its value n and row ratio
// rt at the strip's top row, in its PSF group's frame.
template <int L>
__device__ __forceinline__ void gal_adjoint_staged(const double* __restrict__ e, const double* Gg, double n, double rt,
                                                   double dx, double ev, double ev2, double e21, double* acc) {
    const double a = e[D_A * NCP], b = e[D_B * NCP], d = e[D_D * NCP];
    const double rdy = e[D_RDY * NCP];
    double A = 0.0, B = 0.0, C = 0.0;
#pragma unroll
    for (int k = 0; k < L; ++k) {
        A = fma(Gg[k], n, A);
        B += A;
        C += B;
        if (k + 1 < L) {
            n = n * rt;
            rt = rt * rdy;
        }
    }
    const double M1 = fma(ev, A, -B), M2 = fma(ev2, A, fma(-e21, B, C + C));
    const double X1 = dx * A, Y1 = dx * M1;
    const double U = fma(a, X1, b * M1), Up = fma(b, X1, d * M1);
    const double W = fma(a, Y1, b * M2), Wp = fma(b, Y1, d * M2);
    const double dU = fma(dx, U, -A), dUp = dx * Up, Wm = Wp - A;
    const double wt = e[D_WT * NCP], wnu = e[D_WNU * NCP];
    const double wna = wnu * a, wnb = wnu * b, wnd = wnu * d;
    acc[A_FDEV] = fma(e[D_SGN * NCP], A, acc[A_FDEV]);
    acc[A_UX] = fma(wt, U, acc[A_UX]);
    acc[A_UY] = fma(wt, Up, acc[A_UY]);
    acc[A_SXX] = fma(wna, dU, fma(wnb, W, acc[A_SXX]));
    acc[A_SXY] = fma(wnb, dU, fma(wnd, W, acc[A_SXY]));
    acc[A_SYY] = fma(wnb, dUp, fma(wnd, Wm, acc[A_SYY]));
}

// live: the components to evaluate (item_live); the others are skipped.
template <int L>
__device__ __forceinline__ void strip_adjoint_staged(const double* __restrict__ lt, double px, double py0,
                                                     const double* Gs, const double* Gg, double* acc,
                                                     const double* __restrict__ t2, uint64_t live) {
#pragma unroll 1
    for (int grp = 0; grp < NPSF; ++grp) {
        const bool star = (live >> grp) & 1;
        if (!star && !((live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1))) continue;
        const double* es = lt + grp;
        const double dx = px - es[D_CX * NCP], dy = py0 - es[D_CY * NCP];
        const double h2x = -0.5 * (dx * dx), mxy = -(dx * dy), h2y = -0.5 * (dy * dy);
        const double mdx = -dx, mdyh = -(dy + 0.5);
        const double ev = (double)L + dy;
        const double ev2 = ev * ev, e21 = 2.0 * ev + 1.0;
        if (star) {
            const double a = es[D_A * NCP], b = es[D_B * NCP], d = es[D_D * NCP];
            double n = fexp(fma(a, h2x, fma(b, mxy, fma(d, h2y, es[D_LW * NCP]))), t2);
            double rt = fexp(clamp_arg(fma(b, mdx, d * mdyh)), t2);
            const double rdy = es[D_RDY * NCP];
            double A = 0.0, B = 0.0;
#pragma unroll
            for (int k = 0; k < L; ++k) {
                A = fma(Gs[k], n, A);
                B += A;
                if (k + 1 < L) {
                    n = n * rt;
                    rt = rt * rdy;
                }
            }
            const double M1 = fma(ev, A, -B), X1 = dx * A;
            acc[A_UX] = fma(a, X1, fma(b, M1, acc[A_UX]));
            acc[A_UY] = fma(b, X1, fma(d, M1, acc[A_UY]));
        }
        for_live_pairs(live, grp, [&](int s0, int s1) {
            double n[2], rt[2];
            seed_pair(lt + s0, lt + s1, h2x, mxy, h2y, mdx, mdyh, n, rt, t2);
            gal_adjoint_staged<L>(lt + s0, Gg, n[0], rt[0], dx, ev, ev2, e21, acc);
            gal_adjoint_staged<L>(lt + s1, Gg, n[1], rt[1], dx, ev, ev2, e21, acc);
        });
    }
}

// Pass A of the render's strip pass from the box table staged in LDS (strip_adjoint_staged's
// layout): star and galaxy profile values down the strip, the offsets from each PSF group's
// shared centre formed once per group.
// SGN: also fgd[k] = sum of the de Vaucouleurs minus the exponential components (d fg /
// d frac_dev).
template <int L, bool SGN>
__device__ __forceinline__ void gal_values_staged(const double* __restrict__ e, double n, double rt, double* fg,
                                                  double* fgd) {
    const double rdy = e[D_RDY * NCP], wt = e[D_WT * NCP];
    const double sgn = SGN ? e[D_SGN * NCP] : 0.0;
#pragma unroll
    for (int k = 0; k < L; ++k) {
        fg[k] = fma(n, wt, fg[k]);
        if constexpr (SGN) fgd[k] = fma(n, sgn, fgd[k]);
        if (k + 1 < L) {
            n = n * rt;
            rt = rt * rdy;
        }
    }
}

template <int L, bool SGN = false>
__device__ __forceinline__ void strip_values_staged(const double* __restrict__ lt, double px, double py0,
                                                    double* fs, double* fg, const double* __restrict__ t2,
                                                    uint64_t live, double* fgd = nullptr) {
#pragma unroll
    for (int k = 0; k < L; ++k) fs[k] = fg[k] = 0.0;
    if constexpr (SGN) {
#pragma unroll
        for (int k = 0; k < L; ++k) fgd[k] = 0.0;
    }
#pragma unroll 1
    for (int grp = 0; grp < NPSF; ++grp) {
        const bool star = (live >> grp) & 1;
        if (!star && !((live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1))) continue;
        const double* es = lt + grp;
        const double dx = px - es[D_CX * NCP], dy = py0 - es[D_CY * NCP];
        const double h2x = -0.5 * (dx * dx), mxy = -(dx * dy), h2y = -0.5 * (dy * dy);
        const double mdx = -dx, mdyh = -(dy + 0.5);
        if (star) {
            const double a = es[D_A * NCP], b = es[D_B * NCP], d = es[D_D * NCP];
            double n = fexp(fma(a, h2x, fma(b, mxy, fma(d, h2y, es[D_LW * NCP]))), t2);
            double rt = fexp(clamp_arg(fma(b, mdx, d * mdyh)), t2);
            const double rdy = es[D_RDY * NCP];
#pragma unroll
            for (int k = 0; k < L; ++k) {
                fs[k] += n;
                if (k + 1 < L) {
                    n = n * rt;
                    rt = rt * rdy;
                }
            }
        }
        for_live_pairs(live, grp, [&](int s0, int s1) {
            double n[2], rt[2];
            seed_pair(lt + s0, lt + s1, h2x, mxy, h2y, mdx, mdyh, n, rt, t2);
            gal_values_staged<L, SGN>(lt + s0, n[0], rt[0], fg, fgd);
            gal_values_staged<L, SGN>(lt + s1, n[1], rt[1], fg, fgd);
        });
    }
}

// Row factors of a component from LDS.
template <int L>
__device__ __forceinline__ void load_rows(const double* __restrict__ qs, double* q) {
#pragma unroll
    for (int j = 0; j < L / 2; j += 2) {
        const double2 v = *reinterpret_cast<const double2*>(qs + j);
        q[j] = v.x;
        q[j + 1] = v.y;
    }
}
// Index of the factor of row k of L: rows k and L - 1 - k share one.
template <int L>
__device__ __forceinline__ constexpr int row_q(int k) {
    return k < L / 2 ? L / 2 - 1 - k : k - L / 2;
}

// N0 and r of two components (the form of strip_values_q): the offsets are those of the centre row.
template <int L>
__device__ __forceinline__ void seed_pair_q(const double* __restrict__ e0, const double* __restrict__ e1, double h2x,
                                            double mxy, double h2y, double mdx, double mdy, double* n, double* r,
                                            const double* __restrict__ t2) {
    constexpr double KC = 0.5 * (L - 1);
    const double a0 = e0[D_A * NCP], b0 = e0[D_B * NCP], d0 = e0[D_D * NCP], l0 = e0[D_LW * NCP];
    const double a1 = e1[D_A * NCP], b1 = e1[D_B * NCP], d1 = e1[D_D * NCP], l1 = e1[D_LW * NCP];
    __builtin_amdgcn_sched_barrier(0);
    const double g0 = fma(b0, mdx, d0 * mdy), g1 = fma(b1, mdx, d1 * mdy);   // log r
    const double x[4] = {fma(-KC, g0, fma(a0, h2x, fma(b0, mxy, fma(d0, h2y, l0)))),
                         fma(-KC, g1, fma(a1, h2x, fma(b1, mxy, fma(d1, h2y, l1)))), fmin(g0, LOG_R_MAX),
                         fmin(g1, LOG_R_MAX)};
    double e[4];
    fexps<4>(x, e, t2);
    n[0] = e[0];
    n[1] = e[1];
    r[0] = e[2];
    r[1] = e[3];
}
template <int L>
__device__ __forceinline__ void seed_one_q(const double* __restrict__ e, double h2x, double mxy, double h2y, double mdx,
                                           double mdy, double& n, double& r, const double* __restrict__ t2) {
    constexpr double KC = 0.5 * (L - 1);
    const double a = e[D_A * NCP], b = e[D_B * NCP], d = e[D_D * NCP];
    const double g = fma(b, mdx, d * mdy);
    const double x[2] = {fma(-KC, g, fma(a, h2x, fma(b, mxy, fma(d, h2y, e[D_LW * NCP])))), fmin(g, LOG_R_MAX)};
    double o[2];
    fexps<2>(x, o, t2);
    n = o[0];
    r = o[1];
}

// strip_values_staged through the row factors (lq: the wave's [NCP][NQ]): the weight (de
// Vaucouleurs / exponential share) goes into N0.  SGN: fg and fgd receive the sums of the de
// Vaucouleurs and of the exponential components, of which the caller forms both profiles.
template <int L, bool SGN = false>
__device__ __forceinline__ void strip_values_q(const double* __restrict__ lt, const double* __restrict__ lq, double px,
                                               double py0, double* fs, double* fg, const double* __restrict__ t2,
                                               uint64_t live, double* fgd = nullptr) {
    constexpr double KC = 0.5 * (L - 1);
#pragma unroll
    for (int k = 0; k < L; ++k) fs[k] = fg[k] = 0.0;
    if constexpr (SGN) {
#pragma unroll
        for (int k = 0; k < L; ++k) fgd[k] = 0.0;
    }
    auto rows = [&](int slot, double p, double r, double* f) {
        double q[NQ];
        load_rows<L>(lq + slot * NQ, q);
#pragma unroll
        for (int k = 0; k < L; ++k) {
            f[k] = fma(q[row_q<L>(k)], p, f[k]);
            if (k + 1 < L) p *= r;
        }
    };
#pragma unroll 1
    for (int grp = 0; grp < NPSF; ++grp) {
        const bool star = (live >> grp) & 1;
        if (!star && !((live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1))) continue;
        const double* es = lt + grp;
        const double dx = px - es[D_CX * NCP], dy = py0 + KC - es[D_CY * NCP];
        const double h2x = -0.5 * (dx * dx), mxy = -(dx * dy), h2y = -0.5 * (dy * dy);
        if (star) {
            double n, r;
            seed_one_q<L>(es, h2x, mxy, h2y, -dx, -dy, n, r, t2);
            rows(grp, n, r, fs);
        }
        auto pair = [&](int s0, int s1, double* f) {
            double n[2], r[2];
            seed_pair_q<L>(lt + s0, lt + s1, h2x, mxy, h2y, -dx, -dy, n, r, t2);
            rows(s0, SGN ? n[0] : n[0] * lt[s0 + D_WT * NCP], r[0], f);
            rows(s1, SGN ? n[1] : n[1] * lt[s1 + D_WT * NCP], r[1], f);
        };
        if constexpr (SGN) {
            constexpr uint64_t dev = ((1ull << NDEV) - 1) << NPSF;
            for_live_pairs(live & (dev << (grp * NGAL_PER_PSF)), grp, [&](int s0, int s1) { pair(s0, s1, fg); });
            for_live_pairs(live & ~(dev << (grp * NGAL_PER_PSF)), grp, [&](int s0, int s1) { pair(s0, s1, fgd); });
        } else {
            for_live_pairs(live, grp, [&](int s0, int s1) { pair(s0, s1, fg); });
        }
    }
}

// strip_adjoint_staged through the row factors: with c_k = G_k q_k the moments of t_k = G_k n_k
// are those of the polynomial P(r) = sum c_k r^k, sum t_k = N0 P, sum t_k k = N0 r P',
// sum t_k k (k - 1) = N0 r^2 P'', P and its derivatives by Horner's rule (one product and three
// multiply-adds a row, two for a star, which needs P and P' only).
template <int L>
__device__ __forceinline__ void strip_adjoint_q(const double* __restrict__ lt, const double* __restrict__ lq, double px,
                                                double py0, const double* Gs, const double* Gg, double* acc,
                                                const double* __restrict__ t2, uint64_t live) {
    constexpr double KC = 0.5 * (L - 1);
#pragma unroll 1
    for (int grp = 0; grp < NPSF; ++grp) {
        const bool star = (live >> grp) & 1;
        if (!star && !((live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1))) continue;
        const double* es = lt + grp;
        const double dx = px - es[D_CX * NCP], dy = py0 - es[D_CY * NCP], dyc = dy + KC;
        const double h2x = -0.5 * (dx * dx), mxy = -(dx * dyc), h2y = -0.5 * (dyc * dyc);
        const double dy2 = dy * dy, dy21 = 2.0 * dy + 1.0;
        if (star) {
            double n, r, q[NQ];
            seed_one_q<L>(es, h2x, mxy, h2y, -dx, -dyc, n, r, t2);
            load_rows<L>(lq + grp * NQ, q);
            double h1 = Gs[L - 1] * q[row_q<L>(L - 1)];
            double h0 = fma(h1, r, Gs[L - 2] * q[row_q<L>(L - 2)]);
#pragma unroll
            for (int k = L - 3; k >= 0; --k) {
                h1 = fma(h1, r, h0);
                h0 = fma(h0, r, Gs[k] * q[row_q<L>(k)]);
            }
            const double a = es[D_A * NCP], b = es[D_B * NCP], d = es[D_D * NCP];
            const double M0 = n * h0, M1 = fma(dy, M0, (n * r) * h1), X1 = dx * M0;
            acc[A_UX] = fma(a, X1, fma(b, M1, acc[A_UX]));
            acc[A_UY] = fma(b, X1, fma(d, M1, acc[A_UY]));
        }
        auto gal = [&](int slot, double n, double r) {
            const double* e = lt + slot;
            double q[NQ];
            load_rows<L>(lq + slot * NQ, q);
            double h2 = Gg[L - 1] * q[row_q<L>(L - 1)];
            double h1 = fma(h2, r, Gg[L - 2] * q[row_q<L>(L - 2)]);   // h0 of the second step
            double h0 = fma(h1, r, Gg[L - 3] * q[row_q<L>(L - 3)]);
            h1 = fma(h2, r, h1);
#pragma unroll
            for (int k = L - 4; k >= 0; --k) {
                h2 = fma(h2, r, h1);
                h1 = fma(h1, r, h0);
                h0 = fma(h0, r, Gg[k] * q[row_q<L>(k)]);
            }
            const double a = e[D_A * NCP], b = e[D_B * NCP], d = e[D_D * NCP];
            const double nr = n * r, A = n * h0, m1 = nr * h1, m2 = (nr * r) * (h2 + h2);
            const double M1 = fma(dy, A, m1), M2 = fma(dy2, A, fma(dy21, m1, m2));
            const double X1 = dx * A, Y1 = dx * M1;
            const double U = fma(a, X1, b * M1), Up = fma(b, X1, d * M1);
            const double W = fma(a, Y1, b * M2), Wp = fma(b, Y1, d * M2);
            const double dU = fma(dx, U, -A), dUp = dx * Up, Wm = Wp - A;
            const double wt = e[D_WT * NCP], wnu = e[D_WNU * NCP];
            const double wna = wnu * a, wnb = wnu * b, wnd = wnu * d;
            acc[A_FDEV] = fma(e[D_SGN * NCP], A, acc[A_FDEV]);
            acc[A_UX] = fma(wt, U, acc[A_UX]);
            acc[A_UY] = fma(wt, Up, acc[A_UY]);
            acc[A_SXX] = fma(wna, dU, fma(wnb, W, acc[A_SXX]));
            acc[A_SXY] = fma(wnb, dU, fma(wnd, W, acc[A_SXY]));
            acc[A_SYY] = fma(wnb, dUp, fma(wnd, Wm, acc[A_SYY]));
        };
        for_live_pairs(live, grp, [&](int s0, int s1) {
            // one seed after the other: a pair's do not fit beside the row weights
            double n, r;
            seed_one_q<L>(lt + s0, h2x, mxy, h2y, -dx, -dyc, n, r, t2);
            gal(s0, n, r);
            seed_one_q<L>(lt + s1, h2x, mxy, h2y, -dx, -dyc, n, r, t2);
            gal(s1, n, r);
        });
    }
}

// Pixel term of one row: accumulates the value and d/dk1..k4 and returns the row
// weights d l / d f_star and d l / d f_gal.
// (The -log(x!) constant is not added here: each box's sum of it is precomputed once.)
// VALUE: the value too.
template <class T, bool DERIV, bool VALUE = true>
__device__ __forceinline__ void strip_pixel(double x, T E, T V, T fs, T fg, const T* k, T* acc, T& Gs, T& Gg,
                                            const double2* __restrict__ tl) {
    const T Es = k[C_K1] * fs + k[C_K2] * fg;
    const T inv = frcp(E);
    const T r = V * inv * inv;
    if (VALUE) acc[A_VAL] += x * (flog(E, tl) - 0.5 * r) - E;
    if (DERIV) {
        const T lE = x * inv * (1.0 + r) - 1.0;
        const T lV = -0.5 * x * (inv * inv);
        const T A = lE - 2.0 * Es * lV;
        acc[A_K1] += A * fs;
        acc[A_K2] += A * fg;
        acc[A_K3] += lV * (fs * fs);
        acc[A_K4] += lV * (fg * fg);
        Gs = A * k[C_K1] + 2.0 * lV * (k[C_K3] * fs);
        Gg = A * k[C_K2] + 2.0 * lV * (k[C_K4] * fg);
    }
}

// Second derivatives of one pixel term in the box's brightness factors k1..k4, added into
// h[NKK]: with l_EE = -x/E^2 - 3xV/E^4, l_EV = x/E^3, l_V = -x/(2E^2) (l_VV = 0), dE/dk =
// (fs, fg, 0, 0) and dV/dk = (-2 Es fs, -2 Es fg, fs^2, fg^2), d2V/dk1dk1 = -2 fs^2,
// d2V/dk1dk2 = -2 fs fg, d2V/dk2dk2 = -2 fg^2:
// h_ij = l_EE E_i E_j + l_EV (E_i V_j + V_i E_j) + l_V V_ij.
// frac_dev f enters only through the galaxy profile, fg = f fgd_dev + (1 - f) fg_exp, so
// dfg/df = fgd (the dev minus the exp profile) and, with E_f = k2 fgd,
// V_f = 2 fgd (k4 fg - Es k2), V_ff = 2 fgd^2 (k4 - k2^2), V_f1 = -2 fs k2 fgd,
// V_f2 = -2 (fg k2 + Es) fgd, V_f4 = 2 fg fgd, E_f2 = fgd:
// h_fi = l_EE E_f E_i + l_EV (E_f V_i + V_f E_i) + l_V V_fi + l_E E_fi.
__device__ __forceinline__ void pixel_kk(double x, double E, double V, double fs, double fg, double fgd,
                                         const double* k, double* h) {
    const double inv = frcp(E);
    const double inv2 = inv * inv;
    const double r = V * inv2;
    const double lE = x * inv * (1.0 + r) - 1.0;
    const double lEE = -x * inv2 * (1.0 + 3.0 * r);
    const double lEV = x * inv2 * inv;
    const double lV = -0.5 * x * inv2;
    const double Es = k[C_K1] * fs + k[C_K2] * fg;
    const double Q = lEE - 4.0 * lEV * Es - 2.0 * lV;
    const double a = lEV * fs, b = lEV * fg;
    h[KK_11] += Q * (fs * fs);
    h[KK_12] += Q * (fs * fg);
    h[KK_22] += Q * (fg * fg);
    h[KK_13] += a * (fs * fs);
    h[KK_14] += a * (fg * fg);
    h[KK_23] += b * (fs * fs);
    h[KK_24] += b * (fg * fg);
    const double Ef = k[C_K2] * fgd;
    const double Vf = 2.0 * fgd * (k[C_K4] * fg - Es * k[C_K2]);
    h[KK_F1] += lEE * (Ef * fs) + lEV * (Ef * (-2.0 * Es * fs) + Vf * fs) + lV * (-2.0 * fs * k[C_K2] * fgd);
    h[KK_F2] += lEE * (Ef * fg) + lEV * (Ef * (-2.0 * Es * fg) + Vf * fg) +
                lV * (-2.0 * (fg * k[C_K2] + Es) * fgd) + lE * fgd;
    h[KK_F3] += lEV * Ef * (fs * fs);
    h[KK_F4] += lEV * Ef * (fg * fg) + lV * (2.0 * fg * fgd);
    h[KK_FF] += lEE * (Ef * Ef) + 2.0 * lEV * (Ef * Vf) + lV * (2.0 * fgd * fgd * (k[C_K4] - k[C_K2] * k[C_K2]));
}

// Sky plus the light of every other box of the image that covers each row of the strip.
template <int L>
__device__ __forceinline__ void strip_background(const PairDev& p, const PairDev* __restrict__ pairs,
                                                 const int32_t* __restrict__ nbr, const double* __restrict__ tabv,
                                                 const double* __restrict__ coefv, const celeste_image& im, int c,
                                                 int r0, double* Eb, double* Vb, const double* __restrict__ t2) {
#pragma unroll
    for (int k = 0; k < L; ++k) {
        Eb[k] = r0 + k < im.H ? sky_at(im, r0 + k, c) : im.sky;
        Vb[k] = 0.0;
    }
    for (int q = p.nbr_begin; q < p.nbr_end; ++q) {
        const int pi = __builtin_amdgcn_readfirstlane(nbr[q]);
        const PairDev o = pairs[pi];
        if (c < o.c0 || c >= o.c0 + o.w || r0 + L <= o.r0 || r0 >= o.r0 + o.h) continue;
        double fs[L], fg[L];
        strip_values<double, L>(tabv + (size_t)pi * NCOMP * CST, (double)c, (double)r0, fs, fg, t2);
        const double* kk = coefv + (size_t)pi * NCOEF;
        const double k1 = kk[C_K1], k2 = kk[C_K2], k3 = kk[C_K3], k4 = kk[C_K4];
#pragma unroll
        for (int k = 0; k < L; ++k) {
            const int r = r0 + k;
            if (r < o.r0 || r >= o.r0 + o.h) continue;
            const double Et = k1 * fs[k] + k2 * fg[k];
            Eb[k] += Et;
            Vb[k] += k3 * fs[k] * fs[k] + k4 * fg[k] * fg[k] - Et * Et;
        }
    }
}

// Sky plus the light of every other box of the image covering each row of the strip, from
// the boxes' stored own profile values (ascending box order).
template <int L>
__device__ __forceinline__ void strip_background_fg(const PairDev& p, const PairDev* __restrict__ pairs,
                                                    const int32_t* __restrict__ nbr,
                                                    const double* __restrict__ coefv,
                                                    const double* __restrict__ fgm, const celeste_image& im, int c, int r0,
                                                    double* Eb, double* Vb) {
#pragma unroll
    for (int k = 0; k < L; ++k) {
        Eb[k] = r0 + k < im.H ? sky_at(im, r0 + k, c) : im.sky;
        Vb[k] = 0.0;
    }
    for (int q = p.nbr_begin; q < p.nbr_end; ++q) {
        const int pi = __builtin_amdgcn_readfirstlane(nbr[q]);
        const PairDev o = pairs[pi];
        if (c < o.c0 || c >= o.c0 + o.w || r0 + L <= o.r0 || r0 >= o.r0 + o.h) continue;
        const double* kk = coefv + (size_t)pi * NCOEF;
        const double k1 = kk[C_K1], k2 = kk[C_K2], k3 = kk[C_K3], k4 = kk[C_K4];
#pragma unroll
        for (int k = 0; k < L; ++k) {
            const int r = r0 + k;
            if (r < o.r0 || r >= o.r0 + o.h) continue;
            const size_t vi = (size_t)o.visit_off + (size_t)(r - o.r0) * o.w + (c - o.c0);
            const double fs = fgm[2 * vi], fg = fgm[2 * vi + 1];
            const double Et = k1 * fs + k2 * fg;
            Eb[k] += Et;
            Vb[k] += k3 * fs * fs + k4 * fg * fg - Et * Et;
        }
    }
}

// The next item of the dynamic queue for the whole wave (called with every lane active, so
// the first active lane is lane 0); wave-uniform, so the item loop stays scalar.
__device__ inline int next_item_s(int* counter, int lane) {
    int v = 0;
    if (lane == 0) v = atomicAdd(counter, 1);
    return __builtin_amdgcn_readfirstlane(v);
}

// ----------------------------------------------------------------------- planes
__global__ void __launch_bounds__(256) k_fill_planes(const celeste_image* __restrict__ images,
                                                     double* __restrict__ E, double* __restrict__ V,
                                                     const int* status) {
    if (*status) return;
    const celeste_image& im = images[blockIdx.y];
    const int64_t npix = (int64_t)im.H * im.W;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < npix; i += (int64_t)gridDim.x * blockDim.x) {
        E[im.pix_offset + i] = im.sky_map ? im.sky_map[i] : im.sky;
        V[im.pix_offset + i] = 0.0;
    }
}

// Adds the light of the boxes of one conflict-free class to the planes (no two boxes of a
// class share a pixel, so the read-modify-write needs no atomics; classes run in order).
template <int L>
__global__ void __launch_bounds__(256) k_render_strips(Sel sel, const Item* __restrict__ items,
                                                       const PairDev* __restrict__ pairs,
                                                       const celeste_image* __restrict__ images,
                                                       const double* __restrict__ tab,
                                                       const double* __restrict__ coef, double* __restrict__ E,
                                                       double* __restrict__ V, const int* status) {
    if (*status) return;
    __shared__ double t2[EXP_TAB];
    load_tables(t2, nullptr);
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    for (int j = blockIdx.x * wpb + (threadIdx.x >> 6); j < sel.n; j += nw) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(sel, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        const celeste_image& im = images[p.img];
        const double* tb = tab + (size_t)it.pair * NCOMP * CST;
        const double* kp = coef + (size_t)it.pair * NCOEF;
        const double k1 = kp[C_K1], k2 = kp[C_K2], k3 = kp[C_K3], k4 = kp[C_K4];
        for (int q = lane; q < it.count; q += 64) {
            int c, r0, nrow;
            strip_geometry(p, it.start + q, L, c, r0, nrow);
            double fs[L], fg[L];
            strip_values<double, L>(tb, (double)c, (double)r0, fs, fg, t2);
#pragma unroll
            for (int k = 0; k < L; ++k) {
                if (k >= nrow) break;
                const size_t gi = (size_t)im.pix_offset + (size_t)(r0 + k) * im.W + c;
                const double Et = k1 * fs[k] + k2 * fg[k];
                E[gi] += Et;
                V[gi] += k3 * fs[k] * fs[k] + k4 * fg[k] * fg[k] - Et * Et;
            }
        }
    }
}

// ----------------------------------------------------------------------- adjoint
// Doubles of LDS per wave: the staged table [NDF][NCP] and the row factors [NCP][NQ].
constexpr int STAGED = NCP * NDF + NCP * NQ;

// The value-gradient pass over stored own profile values (the hot path): one wave per work
// item; per strip the pixel terms row by row (their row weights stay in registers), then the
// adjoint of every live Gaussian.  What bounds it is a wave's own latency as much as its
// instructions: without any Gaussian the pass still took 233 of 557 us on the 2000-source
// field, the rows' loads (40 B a visit) being waited for one row after another and three waves
// a SIMD not covering it.  So the rows are loaded RB at a time, the next RB while these are
// worked off, the first two lots before the box's table is staged; the tables of the
// elementary functions are read instead of computed; the eleven sums leave by the swap
// exchanges of wave_sums_dealt.  Row weights, two lots of rows and the sums take more than the 168
// registers that three waves a SIMD allow: 21 spill at 16 rows (0.2 GB of writes a launch on the
// 2000-source field; none at 8 and 4).  2000-source field: 557 -> 535 us (four rows a lot
// spill 32 registers: 549), one source 27.0 -> 25.5 us.
template <int BASE, int L, bool ROWQ>
__global__ void __launch_bounds__(256, 3) k_adjoint_stored(AdjArgs a, const Item* __restrict__ items,
                                                           const PairDev* __restrict__ pairs,
                                                           const celeste_image* __restrict__ images,
                                                           const int32_t* __restrict__ nbr,
                                                           const double* __restrict__ xs,
                                                           const double* __restrict__ Ep,
                                                           const double* __restrict__ Vp,
                                                           const double* __restrict__ tabp,
                                                           const double* __restrict__ coefp,
                                                           const uint8_t* __restrict__ active,
                                                           const double* __restrict__ fgm,
                                                           double* __restrict__ partials) {
    if (*a.status) return;
    __shared__ double t2[EXP_TAB];
    __shared__ double2 tl[128];
    extern __shared__ double ltab[];   // [waves per block][STAGED], sized at launch
    load_tables(t2, tl);
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    double* my = ltab + (threadIdx.x >> 6) * STAGED;
    constexpr int RB = 2, NB = L / RB;   // rows per lot, lots
    int j = a.dynamic ? next_item_s(a.counter, lane) : blockIdx.x * wpb + (threadIdx.x >> 6);
    while (j < a.items.n) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(a.items, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        if (!active || active[p.src]) {
            const celeste_image& im = images[p.img];
            const double* tab = tabp + (size_t)it.pair * NCOMP * CST;
            // Row addresses as 32-bit byte offsets from wave-uniform bases (the image's planes,
            // the box's stored values; plan creation bounds images below 2^29 pixels and boxes
            // below 2^28 visits): one add and one select per row.
            const char* xb = reinterpret_cast<const char*>(xs + im.pix_offset);
            const char* eb = reinterpret_cast<const char*>(Ep + im.pix_offset);
            const char* vb = reinterpret_cast<const char*>(Vp + im.pix_offset);
            const char* fb = reinterpret_cast<const char*>(fgm + 2 * p.visit_off);
            const uint32_t W8 = (uint32_t)im.W * 8u, w16 = (uint32_t)p.w * 16u;
            int c = 0, r0 = 0, nrow = 0;
            uint32_t go = 0, vo = 0;
            double x_[2][RB], e_[2][RB], v_[2][RB], s_[2][RB], g_[2][RB];
            // lot b of the current strip's rows (a row past the box: the strip's top row)
            auto load = [&](int b) {
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    const int rr = b * RB + i, u = b & 1;
                    const bool in = rr < nrow;
                    const uint32_t gr = go + (in ? (uint32_t)rr * W8 : 0u);
                    const uint32_t vr = vo + (in ? (uint32_t)rr * w16 : 0u);
                    x_[u][i] = *reinterpret_cast<const double*>(xb + gr);
                    if constexpr (BASE == BASE_PLANES) {
                        e_[u][i] = *reinterpret_cast<const double*>(eb + gr);
                        v_[u][i] = *reinterpret_cast<const double*>(vb + gr);
                    }
                    const double2 sg = *reinterpret_cast<const double2*>(fb + vr);
                    s_[u][i] = sg.x;
                    g_[u][i] = sg.y;
                }
            };
            const double* kp = coefp + (size_t)it.pair * NCOEF;
            const double k[NCOEF] = {kp[0], kp[1], kp[2], kp[3]};
            double acc[NACC];
#pragma unroll
            for (int f = 0; f < NACC; ++f) acc[f] = 0.0;
            uint64_t live = 0;
            for (int q0 = 0; q0 < it.count; q0 += 64) {
                // lanes without a strip take the last one's with every row masked
                strip_geometry(p, it.start + min(q0 + lane, it.count - 1), L, c, r0, nrow);
                if (q0 + lane >= it.count) nrow = 0;
                go = (uint32_t)(r0 * im.W + c) * 8u;
                vo = (uint32_t)((r0 - p.r0) * p.w + (c - p.c0)) * 16u;
                load(0);
                if (q0 == 0) {
                    // the wave's previous item has finished reading its copy (in-order LDS)
                    __builtin_amdgcn_wave_barrier();
                    stage_derived(tab, my, lane);
                    if constexpr (ROWQ) stage_rows(tab, my + NCP * NDF, lane, t2);
                    live = item_live(tab, p, it, L, lane);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
                if constexpr (NB > 1) load(1);
                double Eb[L], Vb[L];
                if constexpr (BASE == BASE_FG) strip_background_fg<L>(p, pairs, nbr, coefp, fgm, im, c, r0, Eb, Vb);
                double Gs[L], Gg[L];
#pragma unroll
                for (int b = 0; b < NB; ++b) {
#pragma unroll
                    for (int i = 0; i < RB; ++i) {
                        const int kk = b * RB + i, u = b & 1;
                        double gs = 0.0, gg = 0.0;
                        if (kk < nrow && x_[u][i] == x_[u][i]) {
                            double E, V;
                            if constexpr (BASE == BASE_PLANES) {
                                E = e_[u][i];
                                V = v_[u][i];
                            } else {
                                const double Es = k[C_K1] * s_[u][i] + k[C_K2] * g_[u][i];
                                E = Eb[kk] + Es;
                                V = Vb[kk] + (k[C_K3] * (s_[u][i] * s_[u][i]) + k[C_K4] * (g_[u][i] * g_[u][i]) -
                                              Es * Es);
                            }
                            strip_pixel<double, true>(x_[u][i], E, V, s_[u][i], g_[u][i], k, acc, gs, gg, tl);
                        }
                        Gs[kk] = gs;
                        Gg[kk] = gg;
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (b + 2 < NB) load(b + 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
                const double px = (double)c, py0 = (double)r0;
                if constexpr (ROWQ) strip_adjoint_q<L>(my, my + NCP * NDF, px, py0, Gs, Gg, acc, t2, live);
                else strip_adjoint_staged<L>(my, px, py0, Gs, Gg, acc, t2, live);
            }
            int f;
            const double s = wave_sums_dealt<NACC>(acc, lane, f);
            if (f >= 0) partials[(size_t)ii * NACC + f] = s;
        }
        j = a.dynamic ? next_item_s(a.counter, lane) : j + nw;
    }
}

// ------------------------------------------------------------- tangent over stored values
// Gradient and tangent of a box's pixel sum along the direction in the tangent table, over
// stored own profile values (Hessian-vector products).  A component's tangent is its value
// times that of its logarithm, which down a strip is a quadratic in the row offset kappa from
// the centre row: n'_k = n_k (C0 + kappa (C1 + kappa C2)).  So the rows need the values only,
// by the row factors: the own profiles' tangents take 4.5 operations a row and component
// (their values are the stored ones), the adjoint 11: with w = G' + G lambda the tangents of the
// moments are the moments of w n, so two Horner schemes run side by side (strip_adjoint_q).
// In dual numbers the row recurrences took 11 and 15, with the values evaluated again, and the
// table came through the scalar cache: 1250 us on 1024 sources (1.6e7 visits), this 980 (the
// row weights and their tangents take 128 registers of 16-row strips, two waves a SIMD; a pair
// of seeds at a time spills, and takes as long).
// Staged table [NTF][NCP] of (value, tangent), then the row factors [NCP][NQ].
enum TangentField { T_CX = 0, T_CY, T_LW, T_A, T_B, T_D, T_WT, T_WNU, T_SGN, NTF };
constexpr int STAGED_T = 2 * NCP * NTF + NCP * NQ;   // doubles of LDS per wave

__device__ __forceinline__ dual dmul(dual a, dual b) { return mkd(a.v * b.v, fma(a.t, b.v, a.v * b.t)); }
__device__ __forceinline__ dual dfma(dual a, dual b, dual c) {
    return mkd(fma(a.v, b.v, c.v), fma(a.t, b.v, fma(a.v, b.t, c.t)));
}

__device__ __forceinline__ void stage_tangent(const dual* __restrict__ tab, dual* my, int lane) {
    constexpr int from[NTF] = {F_CX, F_CY, F_LOGW, F_PXX, F_PXY, F_PYY, F_WT, F_WNU, F_SGN};
    if (lane > NCOMP) return;
    dual* o = my + (lane < NCOMP ? staged_slot(lane) : NPSF);
#pragma unroll
    for (int f = 0; f < NTF; ++f)
        o[f * NCP] = lane < NCOMP ? tab[lane * CST + from[f]] : mkd(f == T_LW ? -1000.0 : 0.0);
}

// A strip in its PSF group's frame: the offsets of its column and centre row from the group's
// centre, with their tangents (the same in every lane).
struct TFrame {
    double dx, dy, dxt, dyt;
};
template <int L>
__device__ __forceinline__ TFrame tangent_frame(const dual* __restrict__ es, double px, double py0) {
    const dual cx = es[T_CX * NCP], cy = es[T_CY * NCP];
    TFrame f;
    f.dx = px - cx.v;
    f.dy = py0 + 0.5 * (L - 1) - cy.v;
    f.dxt = -lane_bcast(cx.t, 0);
    f.dyt = -lane_bcast(cy.t, 0);
    return f;
}

// N0 and r of N components (the form of strip_values_q) and the quadratics of their
// logarithms' tangents.
template <int L, int N>
__device__ __forceinline__ void seed_t(const dual* const* e, const TFrame& f, double* n, double* r, double (*c)[3],
                                       const double* __restrict__ t2) {
    constexpr double KC = 0.5 * (L - 1);
    double x[2 * N], o[2 * N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const dual a = e[i][T_A * NCP], b = e[i][T_B * NCP], d = e[i][T_D * NCP], lw = e[i][T_LW * NCP];
        const double zx = fma(a.v, f.dx, b.v * f.dy), zy = fma(b.v, f.dx, d.v * f.dy);
        const double tx = fma(a.t, f.dx, b.t * f.dy), ty = fma(b.t, f.dx, d.t * f.dy);
        x[i] = fma(KC, zy, fma(-0.5, fma(f.dx, zx, f.dy * zy), lw.v));
        x[N + i] = fmin(-zy, LOG_R_MAX);
        c[i][0] = fma(-0.5, fma(f.dx, tx, f.dy * ty), lw.t) - fma(zx, f.dxt, zy * f.dyt);
        c[i][1] = -ty - fma(b.v, f.dxt, d.v * f.dyt);
        c[i][2] = -0.5 * d.t;
    }
    fexps<2 * N>(x, o, t2);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        n[i] = o[i];
        r[i] = o[N + i];
    }
}

// Tangents of the own profile values down the strip.
template <int L>
__device__ __forceinline__ void strip_tangents_q(const dual* __restrict__ lt, const double* __restrict__ lq, double px,
                                                 double py0, double* fst, double* fgt, const double* __restrict__ t2,
                                                 uint64_t live) {
    constexpr double KC = 0.5 * (L - 1);
#pragma unroll
    for (int k = 0; k < L; ++k) fst[k] = fgt[k] = 0.0;
    auto rows = [&](int slot, double p, double r, double c0, double c1, double c2, double* f) {
        double q[NQ], ev[L / 2];
        load_rows<L>(lq + slot * NQ, q);
#pragma unroll
        for (int j = 0; j < L / 2; ++j) ev[j] = fma((j + 0.5) * (j + 0.5), c2, c0);
#pragma unroll
        for (int k = 0; k < L; ++k) {
            f[k] = fma(q[row_q<L>(k)] * p, fma(k - KC, c1, ev[row_q<L>(k)]), f[k]);
            if (k + 1 < L) p *= r;
        }
    };
#pragma unroll 1
    for (int grp = 0; grp < NPSF; ++grp) {
        const bool star = (live >> grp) & 1;
        if (!star && !((live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1))) continue;
        const TFrame f = tangent_frame<L>(lt + grp, px, py0);
        if (star) {
            const dual* e[1] = {lt + grp};
            double n, r, c[1][3];
            seed_t<L, 1>(e, f, &n, &r, c, t2);
            rows(grp, n, r, c[0][0], c[0][1], c[0][2], fst);
        }
        for_live_pairs(live, grp, [&](int s0, int s1) {
            const dual* e[2] = {lt + s0, lt + s1};
            double n[2], r[2], c[2][3];
            seed_t<L, 2>(e, f, n, r, c, t2);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                // the weight (de Vaucouleurs / exponential share) and its tangent
                const dual w = e[i][T_WT * NCP];
                rows(i ? s1 : s0, n[i], r[i], fma(w.v, c[i][0], w.t), w.v * c[i][1], w.v * c[i][2], fgt);
            }
        });
    }
}

// strip_adjoint_q with tangents: row weights Gs, Gg with their tangents Gst, Ggt.
template <int L>
__device__ __forceinline__ void strip_adjoint_t(const dual* __restrict__ lt, const double* __restrict__ lq, double px,
                                                double py0, const double* Gs, const double* Gst, const double* Gg,
                                                const double* Ggt, dual* acc, const double* __restrict__ t2,
                                                uint64_t live) {
    constexpr double KC = 0.5 * (L - 1);
#pragma unroll 1
    for (int grp = 0; grp < NPSF; ++grp) {
        const bool star = (live >> grp) & 1;
        if (!star && !((live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1))) continue;
        const TFrame f = tangent_frame<L>(lt + grp, px, py0);
        const dual dx = mkd(f.dx, f.dxt), dy = mkd(f.dy - KC, f.dyt);   // the top row's
        if (star) {
            const dual* e = lt + grp;
            double n, r, c[1][3], q[NQ];
            seed_t<L, 1>(&e, f, &n, &r, c, t2);
            load_rows<L>(lq + grp * NQ, q);
            double h1 = 0.0, h0 = 0.0, g1 = 0.0, g0 = 0.0;
#pragma unroll
            for (int k = L - 1; k >= 0; --k) {
                const double lam = fma(k - KC, fma(k - KC, c[0][2], c[0][1]), c[0][0]), qk = q[row_q<L>(k)];
                h1 = fma(h1, r, h0);
                h0 = fma(h0, r, Gs[k] * qk);
                g1 = fma(g1, r, g0);
                g0 = fma(g0, r, fma(Gs[k], lam, Gst[k]) * qk);
            }
            const dual a = e[T_A * NCP], b = e[T_B * NCP], d = e[T_D * NCP];
            const double nr = n * r;
            const dual M0 = mkd(n * h0, n * g0), M1 = dfma(dy, M0, mkd(nr * h1, nr * g1)), X1 = dmul(dx, M0);
            acc[A_UX] = dfma(a, X1, dfma(b, M1, acc[A_UX]));
            acc[A_UY] = dfma(b, X1, dfma(d, M1, acc[A_UY]));
        }
        uint32_t gm = (uint32_t)(live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1);
        while (gm) {
            const int slot = NPSF + 1 + grp * NGAL_PER_PSF + __builtin_ctz(gm);
            gm &= gm - 1;
            const dual* e = lt + slot;
            double n, r, c[1][3], q[NQ];
            seed_t<L, 1>(&e, f, &n, &r, c, t2);
            load_rows<L>(lq + slot * NQ, q);
            double h2 = 0.0, h1 = 0.0, h0 = 0.0, g2 = 0.0, g1 = 0.0, g0 = 0.0;
#pragma unroll
            for (int k = L - 1; k >= 0; --k) {
                const double lam = fma(k - KC, fma(k - KC, c[0][2], c[0][1]), c[0][0]), qk = q[row_q<L>(k)];
                h2 = fma(h2, r, h1);
                h1 = fma(h1, r, h0);
                h0 = fma(h0, r, Gg[k] * qk);
                g2 = fma(g2, r, g1);
                g1 = fma(g1, r, g0);
                g0 = fma(g0, r, fma(Gg[k], lam, Ggt[k]) * qk);
            }
            const dual a = e[T_A * NCP], b = e[T_B * NCP], d = e[T_D * NCP];
            const double nr = n * r, nr2 = 2.0 * (nr * r);
            const dual A = mkd(n * h0, n * g0), m1 = mkd(nr * h1, nr * g1), m2 = mkd(nr2 * h2, nr2 * g2);
            const dual M1 = dfma(dy, A, m1), M2 = dfma(dy, M1 + m1, m1 + m2);
            const dual X1 = dmul(dx, A), Y1 = dmul(dx, M1);
            const dual U = dfma(a, X1, dmul(b, M1)), Up = dfma(b, X1, dmul(d, M1));
            const dual W = dfma(a, Y1, dmul(b, M2)), Wp = dfma(b, Y1, dmul(d, M2));
            const dual dU = dfma(dx, U, -A), dUp = dmul(dx, Up), Wm = Wp - A;
            const dual wt = e[T_WT * NCP], wnu = e[T_WNU * NCP];
            const dual wna = dmul(wnu, a), wnb = dmul(wnu, b), wnd = dmul(wnu, d);
            const double sgn = e[T_SGN * NCP].v;
            acc[A_FDEV] = mkd(fma(sgn, A.v, acc[A_FDEV].v), fma(sgn, A.t, acc[A_FDEV].t));
            acc[A_UX] = dfma(wt, U, acc[A_UX]);
            acc[A_UY] = dfma(wt, Up, acc[A_UY]);
            acc[A_SXX] = dfma(wna, dU, dfma(wnb, W, acc[A_SXX]));
            acc[A_SXY] = dfma(wnb, dU, dfma(wnd, W, acc[A_SXY]));
            acc[A_SYY] = dfma(wnb, dUp, dfma(wnd, Wm, acc[A_SYY]));
        }
    }
}

// The pass itself, one wave per work item, rows loaded as in k_adjoint_stored.  (No value: the
// tangent passes' callers do not read it.)
template <int L>
__global__ void __launch_bounds__(256, 2) k_tangent_stored(AdjArgs a, const Item* __restrict__ items,
                                                           const PairDev* __restrict__ pairs,
                                                           const celeste_image* __restrict__ images,
                                                           const double* __restrict__ xs,
                                                           const double* __restrict__ Ep,
                                                           const double* __restrict__ Vp,
                                                           const dual* __restrict__ tabp,
                                                           const dual* __restrict__ coefp,
                                                           const uint8_t* __restrict__ active,
                                                           const double* __restrict__ fgm,
                                                           dual* __restrict__ partials) {
    if (*a.status) return;
    __shared__ double t2[EXP_TAB];
    extern __shared__ double ltab[];   // [waves per block][STAGED_T], sized at launch
    load_tables(t2, nullptr);
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    dual* my = reinterpret_cast<dual*>(ltab + (threadIdx.x >> 6) * STAGED_T);
    double* myq = reinterpret_cast<double*>(my + NCP * NTF);
    constexpr int RB = 2, NB = L / RB;   // rows per lot, lots
    int j = a.dynamic ? next_item_s(a.counter, lane) : blockIdx.x * wpb + (threadIdx.x >> 6);
    while (j < a.items.n) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(a.items, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        if (!active || active[p.src]) {
            const celeste_image& im = images[p.img];
            const dual* tab = tabp + (size_t)it.pair * NCOMP * CST;
            // the wave's previous item has finished reading its copy (in-order LDS)
            __builtin_amdgcn_wave_barrier();
            stage_tangent(tab, my, lane);
            stage_rows(tab, myq, lane, t2);
            const uint64_t live = item_live(tab, p, it, L, lane);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const char* xb = reinterpret_cast<const char*>(xs + im.pix_offset);
            const char* eb = reinterpret_cast<const char*>(Ep + im.pix_offset);
            const char* vb = reinterpret_cast<const char*>(Vp + im.pix_offset);
            const char* fb = reinterpret_cast<const char*>(fgm + 2 * p.visit_off);
            const uint32_t W8 = (uint32_t)im.W * 8u, w16 = (uint32_t)p.w * 16u;
            const dual* kp = coefp + (size_t)it.pair * NCOEF;
            const dual k[NCOEF] = {kp[0], kp[1], kp[2], kp[3]};
            dual acc[NACC];
#pragma unroll
            for (int f = 0; f < NACC; ++f) acc[f] = mkd(0.0);
            for (int q0 = 0; q0 < it.count; q0 += 64) {
                // lanes without a strip take the last one's with every row masked
                int c, r0, nrow;
                strip_geometry(p, it.start + min(q0 + lane, it.count - 1), L, c, r0, nrow);
                if (q0 + lane >= it.count) nrow = 0;
                const uint32_t go = (uint32_t)(r0 * im.W + c) * 8u;
                const uint32_t vo = (uint32_t)((r0 - p.r0) * p.w + (c - p.c0)) * 16u;
                double x_[2][RB], e_[2][RB], v_[2][RB], s_[2][RB], g_[2][RB];
                // lot b of the strip's rows (a row past the box: the strip's top row)
                auto load = [&](int b) {
#pragma unroll
                    for (int i = 0; i < RB; ++i) {
                        const int rr = b * RB + i, u = b & 1;
                        const bool in = rr < nrow;
                        const uint32_t gr = go + (in ? (uint32_t)rr * W8 : 0u);
                        const uint32_t vr = vo + (in ? (uint32_t)rr * w16 : 0u);
                        x_[u][i] = *reinterpret_cast<const double*>(xb + gr);
                        e_[u][i] = *reinterpret_cast<const double*>(eb + gr);
                        v_[u][i] = *reinterpret_cast<const double*>(vb + gr);
                        const double2 sg = *reinterpret_cast<const double2*>(fb + vr);
                        s_[u][i] = sg.x;
                        g_[u][i] = sg.y;
                    }
                };
                load(0);
                if constexpr (NB > 1) load(1);
                const double px = (double)c, py0 = (double)r0;
                double Gs[L], Gst[L], Gg[L], Ggt[L];   // tangents of the own values first
                strip_tangents_q<L>(my, myq, px, py0, Gst, Ggt, t2, live);
#pragma unroll
                for (int b = 0; b < NB; ++b) {
#pragma unroll
                    for (int i = 0; i < RB; ++i) {
                        const int kk = b * RB + i, u = b & 1;
                        dual gs = mkd(0.0), gg = mkd(0.0);
                        if (kk < nrow && x_[u][i] == x_[u][i]) {
                            const dual fs = mkd(s_[u][i], Gst[kk]), fg = mkd(g_[u][i], Ggt[kk]);
                            const dual Es = k[C_K1] * fs + k[C_K2] * fg;
                            const dual Vs = k[C_K3] * (fs * fs) + k[C_K4] * (fg * fg) - Es * Es;
                            strip_pixel<dual, true, false>(x_[u][i], value_with_tangent(e_[u][i], Es),
                                                           value_with_tangent(v_[u][i], Vs), fs, fg, k, acc, gs, gg,
                                                           nullptr);
                        }
                        Gs[kk] = gs.v;
                        Gst[kk] = gs.t;
                        Gg[kk] = gg.v;
                        Ggt[kk] = gg.t;
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (b + 2 < NB) load(b + 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
                strip_adjoint_t<L>(my, myq, px, py0, Gs, Gst, Gg, Ggt, acc, t2, live);
            }
            double v[2 * NACC];
#pragma unroll
            for (int f = 0; f < NACC; ++f) {
                v[2 * f] = acc[f].v;
                v[2 * f + 1] = acc[f].t;
            }
            int f;
            const double s = wave_sums_dealt<2 * NACC>(v, lane, f);
            if (f >= 0) reinterpret_cast<double*>(partials)[(size_t)ii * 2 * NACC + f] = s;
        }
        j = a.dynamic ? next_item_s(a.counter, lane) : j + nw;
    }
}

// KK (double passes over stored backgrounds only): also the brightness-factor and frac_dev
// block of each box's intermediate Hessian, per item into a.kk, and the own profile values
// into a.fg_out.  KK_FULL is the whole gradient pass; KK_PIXEL leaves pass B out (the
// position, frac_dev and shape sums of the gradient come from the row moments that
// k_hess_second takes anyway), so it holds no row weights and needs no second evaluation of
// the Gaussians: on 1024 sources (1.6e7 visits) 618 -> 376 us a pass (bounded to three waves
// per SIMD it spills 71 VGPRs and takes as long), k_hess_second 560 -> 600 us; with the row
// factors and the dealt sums the pass takes 311 us, k_hess_second since then 415.
enum KKMode { KK_NONE = 0, KK_FULL = 1, KK_PIXEL = 2 };

// Whether a pass reads each box's table from LDS: the double passes that evaluate Gaussians
// and take the background from planes, stored backgrounds or stored values.
template <class T, int BASE, bool DERIV, bool FGM>
constexpr bool lds_table() {
    if (!std::is_same<T, double>::value || FGM) return false;
    return BASE == BASE_BG || (DERIV && BASE == BASE_PLANES);
}

// The passes that k_adjoint_stored and k_tangent_stored do not take.
// At least two waves per SIMD: the dual-number variants would otherwise take 256 VGPRs
// plus accumulation registers and run one wave per SIMD; with the bound they spill a few
// hundred bytes per lane and run 17% faster (the value variants fit without spilling).
template <class T, int BASE, bool DERIV, int L, bool FGM, int KK, bool ROWQ>
__global__ void __launch_bounds__(256, 2) k_adjoint_strips(AdjArgs a, const Item* __restrict__ items,
                                                        const PairDev* __restrict__ pairs,
                                                        const celeste_image* __restrict__ images,
                                                        const int32_t* __restrict__ nbr,
                                                        const double* __restrict__ xs, const double* __restrict__ Ep,
                                                        const double* __restrict__ Vp, const double* __restrict__ bg,
                                                        const double* __restrict__ tabp,
                                                        const double* __restrict__ coefp,
                                                        const double* __restrict__ tabv,
                                                        const double* __restrict__ coefv,
                                                        const uint8_t* __restrict__ active,
                                                        const double* __restrict__ fgm,
                                                        double* __restrict__ partials) {
    if (*a.status) return;
    __shared__ double t2[EXP_TAB];
    __shared__ double2 tl[128];
    // The double passes read each box's table from LDS, staged by the wave at the start of each
    // item in the derived form of strip_adjoint_staged: the per-component loads of the galaxy
    // loop then wait on LDS instead of missing the scalar cache (38% of the scalar loads missed
    // with the table read from global memory), and the table leaves the scalar registers.
    constexpr bool LDS_TAB = lds_table<T, BASE, DERIV, FGM>();
    extern __shared__ double ltab[];   // LDS_TAB: [waves per block][STAGED], sized at launch
    load_tables(t2, tl);
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    const T zero = scalar_traits<T>::make(0.0, 0.0);
    int j = a.dynamic ? next_item_s(a.counter, lane) : blockIdx.x * wpb + (threadIdx.x >> 6);
    while (j < a.items.n) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(a.items, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        if (!active || active[p.src]) {
            const celeste_image& im = images[p.img];
            const T* tab = reinterpret_cast<const T*>(tabp) + (size_t)it.pair * NCOMP * CST;
            // dual passes (HVP, Hessian tangents) read the table directly; they cull too
            constexpr bool CULL_T = !LDS_TAB && std::is_same<T, dual>::value;
            uint64_t live = 0;
            const double* lt = ltab + (threadIdx.x >> 6) * STAGED;
            const double* lq = lt + NCP * NDF;
            if constexpr (CULL_T) live = item_live(tab, p, it, L, lane);
            if constexpr (LDS_TAB) {
                // the wave's previous item has finished reading its copy (in-order LDS)
                double* my = ltab + (threadIdx.x >> 6) * STAGED;
                __builtin_amdgcn_wave_barrier();
                stage_derived(reinterpret_cast<const double*>(tab), my, lane);
                if constexpr (ROWQ) stage_rows(reinterpret_cast<const double*>(tab), my + NCP * NDF, lane, t2);
                live = item_live(reinterpret_cast<const double*>(tab), p, it, L, lane);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            const T* kp = reinterpret_cast<const T*>(coefp) + (size_t)it.pair * NCOEF;
            const T k[NCOEF] = {kp[0], kp[1], kp[2], kp[3]};
            T acc[NACC];
#pragma unroll
            for (int f = 0; f < NACC; ++f) acc[f] = zero;
            double kh[NKK_USED];
#pragma unroll
            for (int f = 0; f < NKK_USED; ++f) kh[f] = 0.0;
            for (int q = lane; q < it.count; q += 64) {
                int c, r0, nrow;
                strip_geometry(p, it.start + q, L, c, r0, nrow);
                const double px = (double)c, py0 = (double)r0;
                if constexpr (!FGM && (DERIV ? (BASE == BASE_PLANES || BASE == BASE_BG) : (LDS_TAB && BASE == BASE_BG))) {
                    // Own values from pass A, then the pixel terms row by row, the next row's
                    // loads in flight.
                    T fs[L], fg[L], fgd[KK != KK_NONE ? L : 1];
                    if constexpr (LDS_TAB) {
                        if constexpr (ROWQ) {
                            strip_values_q<L, KK != KK_NONE>(lt, lq, px, py0, fs, fg, t2, live, fgd);
                            if constexpr (KK != KK_NONE) {
                                const double fdev = lt[NPSF + 1 + D_WT * NCP];   // a de Vaucouleurs component's weight
#pragma unroll
                                for (int kk = 0; kk < L; ++kk) {
                                    const double dv = fg[kk], ex = fgd[kk];
                                    fg[kk] = fma(fdev, dv, (1.0 - fdev) * ex);
                                    fgd[kk] = dv - ex;
                                }
                            }
                        } else {
                            strip_values_staged<L, KK != KK_NONE>(lt, px, py0, fs, fg, t2, live, fgd);
                        }
                    } else
                        strip_values<T, L, KK != KK_NONE, CULL_T>(tab, px, py0, fs, fg, t2, fgd, live);
                    const double* xs_i = xs + im.pix_offset;
                    auto row_load = [&](int rr, double& x_, double& e_, double& v_) {
                        const size_t gi = (size_t)(r0 + rr) * im.W + c;
                        x_ = xs_i[gi];
                        if constexpr (BASE == BASE_PLANES) {
                            e_ = Ep[im.pix_offset + gi];
                            v_ = Vp[im.pix_offset + gi];
                        } else {
                            const size_t vi = (size_t)p.visit_off + (size_t)(r0 + rr - p.r0) * p.w + (c - p.c0);
                            e_ = bg[2 * vi];
                            v_ = bg[2 * vi + 1];
                        }
                    };
                    double cx_, ce_, cv_;
                    row_load(0, cx_, ce_, cv_);
#pragma unroll
                    for (int kk = 0; kk < L; ++kk) {
                        double nx_ = 0.0, ne_ = 0.0, nv_ = 0.0;
                        if (kk + 1 < L) row_load(kk + 1 < nrow ? kk + 1 : 0, nx_, ne_, nv_);
                        T gs = zero, gg = zero;
                        if constexpr (KK != KK_NONE) {
                            // own values for the closed-form Hessian pass that follows
                            if (a.fg_out && kk < nrow) {
                                const size_t vi = (size_t)p.visit_off + (size_t)(r0 + kk - p.r0) * p.w + (c - p.c0);
                                a.fg_out[2 * vi] = fs[kk];
                                a.fg_out[2 * vi + 1] = fg[kk];
                            }
                        }
                        if (kk < nrow && cx_ == cx_) {
                            const T Es = k[C_K1] * fs[kk] + k[C_K2] * fg[kk];
                            const T Vs = k[C_K3] * (fs[kk] * fs[kk]) + k[C_K4] * (fg[kk] * fg[kk]) - Es * Es;
                            T E, V;
                            if constexpr (BASE == BASE_PLANES) {
                                E = value_with_tangent(ce_, Es);
                                V = value_with_tangent(cv_, Vs);
                            } else {
                                E = ce_ + Es;
                                V = cv_ + Vs;
                            }
                            strip_pixel<T, DERIV>(cx_, E, V, fs[kk], fg[kk], k, acc, gs, gg, tl);
                            if constexpr (KK != KK_NONE) pixel_kk(cx_, E, V, fs[kk], fg[kk], fgd[kk], k, kh);
                        }
                        if constexpr (DERIV && KK != KK_PIXEL) {
                            fs[kk] = gs;
                            fg[kk] = gg;
                        }
                        cx_ = nx_;
                        ce_ = ne_;
                        cv_ = nv_;
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (DERIV && KK != KK_PIXEL) {
                        if constexpr (LDS_TAB) {
                            if constexpr (ROWQ) strip_adjoint_q<L>(lt, lq, px, py0, fs, fg, acc, t2, live);
                            else strip_adjoint_staged<L>(lt, px, py0, fs, fg, acc, t2, live);
                        } else
                            strip_adjoint<T, L, CULL_T>(tab, px, py0, fs, fg, acc, t2, live);
                    }
                    continue;
                }
                double x[L], Eb[L], Vb[L];
                if (BASE == BASE_NBR) {
                    strip_background<L>(p, pairs, nbr, tabv, coefv, im, c, r0, Eb, Vb, t2);
                } else if (BASE == BASE_FG) {
                    strip_background_fg<L>(p, pairs, nbr, coefv, fgm, im, c, r0, Eb, Vb);
                }
#pragma unroll
                for (int kk = 0; kk < L; ++kk) {
                    const int rr = kk < nrow ? kk : 0;   // rows past the box reuse row 0 (masked below)
                    const size_t gi = (size_t)im.pix_offset + (size_t)(r0 + rr) * im.W + c;
                    x[kk] = kk < nrow ? xs[gi] : __builtin_nan("");
                    if (BASE == BASE_PLANES) {
                        Eb[kk] = Ep[gi];
                        Vb[kk] = Vp[gi];
                    } else if (BASE == BASE_BG) {
                        const size_t vi = (size_t)p.visit_off + (size_t)(r0 + rr - p.r0) * p.w + (c - p.c0);
                        Eb[kk] = bg[2 * vi];
                        Vb[kk] = bg[2 * vi + 1];
                    }
                }
                if (BASE == BASE_PLANES && !DERIV) {
                    // value only: the planes already hold the totals
#pragma unroll
                    for (int kk = 0; kk < L; ++kk) {
                        if (!(x[kk] == x[kk])) continue;
                        T gs, gg;
                        strip_pixel<T, false>(x[kk], scalar_traits<T>::make(Eb[kk], 0.0),
                                              scalar_traits<T>::make(Vb[kk], 0.0), zero, zero, k, acc, gs, gg, tl);
                    }
                    continue;
                }
                T fs[L], fg[L];
                if (FGM) {
                    // own profile values stored by the render's strip pass
#pragma unroll
                    for (int kk = 0; kk < L; ++kk) {
                        const int rr = kk < nrow ? kk : 0;
                        const size_t vi = (size_t)p.visit_off + (size_t)(r0 + rr - p.r0) * p.w + (c - p.c0);
                        fs[kk] = scalar_traits<T>::make(fgm[2 * vi], 0.0);
                        fg[kk] = scalar_traits<T>::make(fgm[2 * vi + 1], 0.0);
                    }
                } else {
                    strip_values<T, L>(tab, px, py0, fs, fg, t2);
                }
                // fs, fg become the row weights of pass B
#pragma unroll
                for (int kk = 0; kk < L; ++kk) {
                    T gs = zero, gg = zero;
                    if (x[kk] == x[kk]) {
                        const T Es = k[C_K1] * fs[kk] + k[C_K2] * fg[kk];
                        const T Vs = k[C_K3] * (fs[kk] * fs[kk]) + k[C_K4] * (fg[kk] * fg[kk]) - Es * Es;
                        T E, V;
                        if (BASE == BASE_PLANES) {
                            E = value_with_tangent(Eb[kk], Es);
                            V = value_with_tangent(Vb[kk], Vs);
                        } else {
                            E = Eb[kk] + Es;
                            V = Vb[kk] + Vs;
                        }
                        strip_pixel<T, DERIV>(x[kk], E, V, fs[kk], fg[kk], k, acc, gs, gg, tl);
                    }
                    fs[kk] = gs;
                    fg[kk] = gg;
                    // one row at a time: interleaving the rows' log/division chains would
                    // multiply the live registers without adding useful parallelism
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (DERIV) strip_adjoint<T, L>(tab, px, py0, fs, fg, acc, t2);
            }
            T* out = reinterpret_cast<T*>(partials) + (size_t)ii * NACC;
            constexpr int NOUT = !DERIV ? A_VAL + 1 : KK == KK_PIXEL ? A_K4 + 1 : NACC;   // the sums this pass forms
            if constexpr (std::is_same<T, double>::value) {
                constexpr int NV = NOUT + (KK != KK_NONE ? NKK_USED : 0);
                double v[NV];
#pragma unroll
                for (int f = 0; f < NV; ++f) v[f] = f < NOUT ? acc[f] : kh[f - NOUT];
                int f;
                const double s = wave_sums_dealt<NV>(v, lane, f);
                if (f >= 0) {
                    if (f < NOUT) out[f] = s;
                    else a.kk[(size_t)ii * NKK + f - NOUT] = s;
                }
            } else {
#pragma unroll
                for (int f = 0; f < NOUT; ++f) {
                    const T s = wave_sum(acc[f]);
                    if (lane == 0) out[f] = s;
                }
            }
        }
        j = a.dynamic ? next_item_s(a.counter, lane) : j + nw;
    }
}

// ------------------------------------------------- closed-form geometric Hessian block
// Second derivatives of a box's pixel sum in its position, frac_dev and shape intermediates
// (the exact Hessians of Section IV-D), evaluated pixel by pixel in closed form.  For a
// component n = w N(m; mu, C) with z = P (m - mu), P = C^-1 = [[a, b], [b, d]] and
// D_ij = z_i z_j - P_ij, and with the operators d/du_i (position) and s_ij = c_ij d/dS_ij
// (c = 2 on the diagonal: the accumulator scaling of the gradient pass) on a galaxy
// component of covariance C = nu S + PSF:
//   d n/du_i = n z_i,                 d2 n/du_i du_j = n D_ij,
//   s_ij n = nu n D_ij,               d/du_i s_kl n = nu n (z_i D_kl - P_ki z_l - P_li z_k),
//   s_ij s_kl n = nu^2 n (D_ij D_kl - T_ij,kl),
// where, from s_ij z = -nu P E_ij z and s_ij P = -nu P E_ij P (E_xx = 2 e_x e_x^T,
// E_xy = e_x e_y^T + e_y e_x^T, E_yy = 2 e_y e_y^T), T_ij,kl is y_k z_l + z_k y_l - Q_kl with
// y = P E_ij z and Q = P E_ij P, linear in D:
//   T_xx,xx = 4a Dxx + 2a^2,  T_xx,xy = 2a Dxy + 2b Dxx + 2ab,  T_xx,yy = 4b Dxy + 2b^2,
//   T_xy,xy = a Dyy + 2b Dxy + d Dxx + ad + b^2,  T_xy,yy = 2b Dyy + 2d Dxy + 2bd,
//   T_yy,yy = 4d Dyy + 2d^2.
// frac_dev enters the galaxy profile linearly (weight +1 de Vaucouleurs, -1 exponential).
// With the pixel term l(E, V), E = Eb + k1 fs + k2 fg, V = Vb + k3 fs^2 + k4 fg^2 - Es^2
// (Es = k1 fs + k2 fg), l_VV = 0 and the row weights Gs, Gg of the gradient pass, the entry
// between geometric intermediates g, h is
//   (l_EE - 2 l_V) E_g E_h + l_EV (E_g V_h + V_g E_h) + 2 l_V (k3 fs_g fs_h + k4 fg_g fg_h)
//   + Gs fs_gh + Gg fg_gh,
// and the entry between g and k_i follows from dE/dk = (fs, fg, 0, 0) and
// dV/dk = (-2 Es fs, -2 Es fg, fs^2, fg^2).  Entry layout: see HGField.
// The terms Gs fs_gh + Gg fg_gh are summed per strip from row moments (k_hess_second);
// k_hess_geom adds the products of first derivatives and the k-block entries.

// ---------------------------------------------- closed-form Hessian: second-derivative terms
// The second-derivative terms of the geometric block (each pixel's row weight Gs or Gg times a
// profile's second derivatives in position, frac_dev and shape) are, per Gaussian, the
// weighted pixel sum of n times a polynomial of degree <= 4 in z = P (m - mu).  Down a strip
// z is affine in the row: z_k = z_c + (b, d) s_k with z_c its value at the strip centre and
// s_k = k - (L - 1)/2, so with the strip recurrence for n and the exact centred row moments
// U_m = sum_k t_k s_k^m (t_k = row weight x value, m <= 4; s_k^m are compile-time constants)
// the sums N_pq = sum_k t_k zx_k^p zy_k^q follow by two kinds of map: V_q = N_0q = (Y^q U)_0 with
// (Y U)_m = zy_c U_m + d U_(m+1), and, zx = g + beta zy along the strip (beta = b / d,
// g = (a - beta b) dx), N_pq = (X^p V)_q with (X V)_q = g V_q + beta V_(q+1): ten steps of each.
// With the moments about the strip centre, every term of these expansions is bounded by the
// strip's own values of |z|^4 (beta zy by the bound of zx: b^2 < a d), so no cancellation
// beyond a small factor arises.  The entries
// (galaxy component, weights wt, sgn, wnu = wt nu):
//   XX, XY, YY: wt (N20 - a N00, N11 - b N00, N02 - d N00);   XF, YF: sgn N10, sgn N01;
//   F_Sxx, F_Sxy, F_Syy: sgn nu times the same three as XX, XY, YY;
//   X_Sxx: wnu (N30 - 3a N10);   X_Sxy = Y_Sxx: wnu (N21 - 2b N10 - a N01);
//   X_Syy = Y_Sxy: wnu (N12 - d N10 - 2b N01);   Y_Syy: wnu (N03 - 3d N01);
//   Sxx_Sxx: wnu nu (N40 - 6a N20 + 3a^2 N00);   Sxx_Sxy: wnu nu (N31 - 3b N20 - 3a N11 + 3ab N00);
//   Sxx_Syy = Sxy_Sxy: wnu nu (N22 - d N20 - a N02 - 4b N11 + (ad + 2b^2) N00);
//   Sxy_Syy: wnu nu (N13 - 3d N11 - 3b N02 + 3bd N00);   Syy_Syy: wnu nu (N04 - 6d N02 + 3d^2 N00)
// (the expansions of the per-pixel formulas), and for a star (weight Gs):
// XX, XY, YY: N20 - a N00, N11 - b N00, N02 - d N00.  The same moments give the gradient's
// position, frac_dev and shape sums (acc, A_UX .. A_SYY): wt (N10, N01), sgn N00 and wnu
// (N20 - a N00, N11 - b N00, N02 - d N00); N10, N01 for a star.  One pass over the components per strip
// (two exps per component), against one exp and about 55 operations per pixel and component
// for the same terms pixel by pixel.
enum HessStagedField { H_CX = 0, H_CY, H_LW, H_RDY, H_A, H_B, H_D, H_WT, H_WNU, H_SGN, H_NU, H_BE, NDH };

// One wave writes the staged table of a box (field-major [NDH][NCP], slots as in
// stage_derived) into its LDS slot; nu[g]: nu of galaxy component g.
__device__ __forceinline__ void stage_hess(const double* __restrict__ tab, const double* __restrict__ nu,
                                           double* my, int lane) {
    if (lane < NCOMP) {
        const double* e = tab + lane * CST;
        double* o = my + staged_slot(lane);
        o[H_CX * NCP] = e[F_CX];
        o[H_CY * NCP] = e[F_CY];
        o[H_LW * NCP] = e[F_LOGW];
        o[H_RDY * NCP] = e[F_RDY];
        o[H_A * NCP] = e[F_PXX];
        o[H_B * NCP] = e[F_PXY];
        o[H_D * NCP] = e[F_PYY];
        o[H_WT * NCP] = e[F_WT];
        o[H_WNU * NCP] = e[F_WNU];
        o[H_SGN * NCP] = e[F_SGN];
        o[H_NU * NCP] = lane < NPSF ? 0.0 : nu[lane - NPSF];
        o[H_BE * NCP] = e[F_PXY] / e[F_PYY];
    } else if (lane == NCOMP) {   // the zero component (stage_derived)
        double* o = my + NPSF;
#pragma unroll
        for (int f = 0; f < NDH; ++f) o[f * NCP] = 0.0;
        o[H_LW * NCP] = -1000.0;
        o[H_RDY * NCP] = 1.0;
    }
}

template <int L>
__device__ __forceinline__ void hess_second_strip(const double* __restrict__ lt, double px, double py0,
                                                  const double* Gs, const double* Gg, double* H, double* acc,
                                                  const double* __restrict__ t2, uint64_t live) {
    constexpr double KC = 0.5 * (L - 1);
#pragma unroll 1
    for (int grp = 0; grp < NPSF; ++grp) {
        const bool star = (live >> grp) & 1;
        if (!star && !((live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1))) continue;
        const double* es = lt + grp;
        const double dx = px - es[H_CX * NCP], dy = py0 - es[H_CY * NCP];
        const double h2x = -0.5 * (dx * dx), mxy = -(dx * dy), h2y = -0.5 * (dy * dy);
        const double mdx = -dx, mdyh = -(dy + 0.5), dyc = dy + KC;
        if (star) {
            const double a = es[H_A * NCP], b = es[H_B * NCP], d = es[H_D * NCP];
            double n = fexp(fma(a, h2x, fma(b, mxy, fma(d, h2y, es[H_LW * NCP]))), t2);
            double rt = fexp(clamp_arg(fma(b, mdx, d * mdyh)), t2);
            const double rdy = es[H_RDY * NCP];
            double U0 = 0.0, U1 = 0.0, U2 = 0.0;
#pragma unroll
            for (int k = 0; k < L; ++k) {
                const double sk = (double)k - KC;
                const double t = Gs[k] * n;
                U0 += t;
                U1 = fma(sk, t, U1);
                U2 = fma(sk * sk, t, U2);
                if (k + 1 < L) {
                    n = n * rt;
                    rt = rt * rdy;
                }
            }
            const double zx = fma(a, dx, b * dyc), zy = fma(b, dx, d * dyc);
            const double X10 = fma(zx, U0, b * U1), X11 = fma(zx, U1, b * U2);
            const double Y10 = fma(zy, U0, d * U1), Y11 = fma(zy, U1, d * U2);
            const double N20 = fma(zx, X10, b * X11), N11 = fma(zy, X10, d * X11), N02 = fma(zy, Y10, d * Y11);
            H[HG_XX] += fma(-a, U0, N20);
            H[HG_XY] += fma(-b, U0, N11);
            H[HG_YY] += fma(-d, U0, N02);
            acc[A_UX - A_UX] += X10;
            acc[A_UY - A_UX] += Y10;
        }
        auto gal = [&](const double* __restrict__ e, double n, double rt) {
            const double a = e[H_A * NCP], b = e[H_B * NCP], d = e[H_D * NCP];
            const double rdy = e[H_RDY * NCP];
            double U[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < L; ++k) {
                const double sk = (double)k - KC;
                const double t = Gg[k] * n;
                U[0] += t;
                U[1] = fma(sk, t, U[1]);
                U[2] = fma(sk * sk, t, U[2]);
                U[3] = fma(sk * sk * sk, t, U[3]);
                U[4] = fma(sk * sk * sk * sk, t, U[4]);
                if (k + 1 < L) {
                    n = n * rt;
                    rt = rt * rdy;
                }
            }
            // the maps of the head comment
            const double zy = fma(b, dx, d * dyc), be = e[H_BE * NCP], g = fma(-be, b, a) * dx;
            double Y1[4], Y2[3], Y3[2];
#pragma unroll
            for (int m = 0; m < 4; ++m) Y1[m] = fma(zy, U[m], d * U[m + 1]);
#pragma unroll
            for (int m = 0; m < 3; ++m) Y2[m] = fma(zy, Y1[m], d * Y1[m + 1]);
#pragma unroll
            for (int m = 0; m < 2; ++m) Y3[m] = fma(zy, Y2[m], d * Y2[m + 1]);
            const double N00 = U[0], N01 = Y1[0], N02 = Y2[0], N03 = Y3[0], N04 = fma(zy, Y3[0], d * Y3[1]);
            const double N10 = fma(g, N00, be * N01), N11 = fma(g, N01, be * N02), N12 = fma(g, N02, be * N03),
                         N13 = fma(g, N03, be * N04);
            const double N20 = fma(g, N10, be * N11), N21 = fma(g, N11, be * N12), N22 = fma(g, N12, be * N13);
            const double N30 = fma(g, N20, be * N21), N31 = fma(g, N21, be * N22);
            const double N40 = fma(g, N30, be * N31);
            const double wt = e[H_WT * NCP], sg = e[H_SGN * NCP], wnu = e[H_WNU * NCP], nu = e[H_NU * NCP];
            const double snu = sg * nu, vnu = wnu * nu;
            const double e20 = fma(-a, N00, N20), e11 = fma(-b, N00, N11), e02 = fma(-d, N00, N02);
            H[HG_XX] = fma(wt, e20, H[HG_XX]);
            H[HG_XY] = fma(wt, e11, H[HG_XY]);
            H[HG_YY] = fma(wt, e02, H[HG_YY]);
            H[HG_XF] = fma(sg, N10, H[HG_XF]);
            H[HG_YF] = fma(sg, N01, H[HG_YF]);
            H[HG_F_SXX] = fma(snu, e20, H[HG_F_SXX]);
            H[HG_F_SXY] = fma(snu, e11, H[HG_F_SXY]);
            H[HG_F_SYY] = fma(snu, e02, H[HG_F_SYY]);
            acc[A_UX - A_UX] = fma(wt, N10, acc[A_UX - A_UX]);
            acc[A_UY - A_UX] = fma(wt, N01, acc[A_UY - A_UX]);
            acc[A_FDEV - A_UX] = fma(sg, N00, acc[A_FDEV - A_UX]);
            acc[A_SXX - A_UX] = fma(wnu, e20, acc[A_SXX - A_UX]);
            acc[A_SXY - A_UX] = fma(wnu, e11, acc[A_SXY - A_UX]);
            acc[A_SYY - A_UX] = fma(wnu, e02, acc[A_SYY - A_UX]);
            const double x1 = fma(-3.0 * a, N10, N30);
            const double x2 = fma(-2.0 * b, N10, fma(-a, N01, N21));
            const double x3 = fma(-d, N10, fma(-2.0 * b, N01, N12));
            const double x4 = fma(-3.0 * d, N01, N03);
            H[HG_X_SXX] = fma(wnu, x1, H[HG_X_SXX]);
            H[HG_X_SXY] = fma(wnu, x2, H[HG_X_SXY]);
            H[HG_X_SYY] = fma(wnu, x3, H[HG_X_SYY]);
            H[HG_Y_SYY] = fma(wnu, x4, H[HG_Y_SYY]);
            const double s1 = fma(-6.0 * a, N20, fma(3.0 * (a * a), N00, N40));
            const double s2 = fma(-3.0 * b, N20, fma(-3.0 * a, N11, fma(3.0 * (a * b), N00, N31)));
            const double s3 = fma(-d, N20, fma(-a, N02, fma(-4.0 * b, N11, fma(fma(a, d, 2.0 * (b * b)), N00, N22))));
            const double s4 = fma(-3.0 * d, N11, fma(-3.0 * b, N02, fma(3.0 * (b * d), N00, N13)));
            const double s5 = fma(-6.0 * d, N02, fma(3.0 * (d * d), N00, N04));
            H[HG_SXX_SXX] = fma(vnu, s1, H[HG_SXX_SXX]);
            H[HG_SXX_SXY] = fma(vnu, s2, H[HG_SXX_SXY]);
            H[HG_SXX_SYY] = fma(vnu, s3, H[HG_SXX_SYY]);
            H[HG_SXY_SYY] = fma(vnu, s4, H[HG_SXY_SYY]);
            H[HG_SYY_SYY] = fma(vnu, s5, H[HG_SYY_SYY]);
        };
        for_live_pairs(live, grp, [&](int s0, int s1) {
            double n[2], rt[2];
            seed_pair(lt + s0, lt + s1, h2x, mxy, h2y, mdx, mdyh, n, rt, t2);
            gal(lt + s0, n[0], rt[0]);
            gal(lt + s1, n[1], rt[1]);
        });
    }
}

// Second-derivative terms of the geometric block, one lane per strip: the row weights Gs, Gg
// from the stored background and own profile values of each row, then hess_second_strip.
// Writes hg[item] (geometric entries; the k-block entries zero), to which k_hess_geom then
// adds the first-derivative products, and the position, frac_dev and shape entries of
// a.partials[item].  Items of sources outside a.active get zeros.
// The rows come four at a time, loaded whether masked or not and the next four while these are
// worked off: loaded each behind its pixel's mask, row after row, they were what a third wave
// per SIMD was worth spilling 69 registers for.  Two waves unspilled have room for the seeds of
// two components at a time.  1024 sources (1.6e7 visits): 532 us with masked loads and three
// waves, 427 with lots of two rows, 415 with lots of four and paired seeds.
template <int L>
__global__ void __launch_bounds__(256, 2) k_hess_second(AdjArgs a, const Item* __restrict__ items,
                                                     const PairDev* __restrict__ pairs,
                                                     const celeste_image* __restrict__ images,
                                                     const double* __restrict__ xs, const double* __restrict__ bg,
                                                     const double* __restrict__ tabp,
                                                     const double* __restrict__ coefp,
                                                     const double* __restrict__ own, const double* __restrict__ nu,
                                                     double* __restrict__ hg) {
    if (*a.status) return;
    __shared__ double t2[EXP_TAB];
    extern __shared__ double ltab[];   // [waves per block][NDH][NCP], sized at launch
    load_tables(t2, nullptr);
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    double* my = ltab + (threadIdx.x >> 6) * (NCP * NDH);
    int j = a.dynamic ? next_item_s(a.counter, lane) : blockIdx.x * wpb + (threadIdx.x >> 6);
    while (j < a.items.n) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(a.items, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        double* out = hg + (size_t)ii * NHG;
        if (a.active && !a.active[p.src]) {
            if (lane < NHG) out[lane] = 0.0;
            j = a.dynamic ? next_item_s(a.counter, lane) : j + nw;
            continue;
        }
        const celeste_image& im = images[p.img];
        const double* kp = coefp + (size_t)it.pair * NCOEF;
        const double k1 = kp[C_K1], k2 = kp[C_K2], k3 = kp[C_K3], k4 = kp[C_K4];
        __builtin_amdgcn_wave_barrier();
        stage_hess(tabp + (size_t)it.pair * NCOMP * CST, nu, my, lane);
        const uint64_t live = item_live(tabp + (size_t)it.pair * NCOMP * CST, p, it, L, lane);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        double H[NHG_GEO], acc[NACC - A_UX];
#pragma unroll
        for (int f = 0; f < NHG_GEO; ++f) H[f] = 0.0;
#pragma unroll
        for (int f = 0; f < NACC - A_UX; ++f) acc[f] = 0.0;
        const double* xi = xs + im.pix_offset;
        const double2* oi = reinterpret_cast<const double2*>(own) + p.visit_off;
        const double2* bi = reinterpret_cast<const double2*>(bg) + p.visit_off;
        constexpr int RB = L < 4 ? L : 4, NB = L / RB;   // rows per lot, lots
        for (int q = lane; q < it.count; q += 64) {
            int c, r0, nrow;
            strip_geometry(p, it.start + q, L, c, r0, nrow);
            const uint32_t go = (uint32_t)(r0 * im.W + c), vo = (uint32_t)((r0 - p.r0) * p.w + (c - p.c0));
            double x_[2][RB];
            double2 o_[2][RB], b_[2][RB];
            auto load = [&](int b) {
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    const int rr = b * RB + i < nrow ? b * RB + i : 0;   // rows past the box reuse row 0 (weight 0)
                    x_[b & 1][i] = xi[go + (uint32_t)(rr * im.W)];
                    o_[b & 1][i] = oi[vo + (uint32_t)(rr * p.w)];
                    b_[b & 1][i] = bi[vo + (uint32_t)(rr * p.w)];
                }
            };
            load(0);
            if constexpr (NB > 1) load(1);
            double Gs[L], Gg[L];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    const int kk = b * RB + i;
                    const double x = x_[b & 1][i];
                    double gs = 0.0, gg = 0.0;
                    if (kk < nrow && x == x) {
                        const double fs = o_[b & 1][i].x, fgv = o_[b & 1][i].y;
                        const double Es = k1 * fs + k2 * fgv;
                        const double E = b_[b & 1][i].x + Es;
                        const double V = b_[b & 1][i].y + k3 * (fs * fs) + k4 * (fgv * fgv) - Es * Es;
                        const double inv = frcp(E);
                        const double inv2 = inv * inv;
                        const double lE = x * inv * (1.0 + V * inv2) - 1.0;
                        const double lV = -0.5 * x * inv2;
                        const double A = lE - 2.0 * Es * lV;
                        gs = A * k1 + 2.0 * lV * (k3 * fs);
                        gg = A * k2 + 2.0 * lV * (k4 * fgv);
                    }
                    Gs[kk] = gs;
                    Gg[kk] = gg;
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (b + 2 < NB) load(b + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            hess_second_strip<L>(my, (double)c, (double)r0, Gs, Gg, H, acc, t2, live);
        }
        H[HG_Y_SXX] = H[HG_X_SXY];   // the same sums
        H[HG_Y_SXY] = H[HG_X_SYY];
        H[HG_SXY_SXY] = H[HG_SXX_SYY];
        double v[NHG_GEO + NACC - A_UX];
#pragma unroll
        for (int f = 0; f < NHG_GEO; ++f) v[f] = H[f];
#pragma unroll
        for (int f = 0; f < NACC - A_UX; ++f) v[NHG_GEO + f] = acc[f];
        int f;
        const double sum = wave_sums_dealt<NHG_GEO + NACC - A_UX>(v, lane, f);
        if (f >= 0) {
            if (f < NHG_GEO) out[f] = sum;
            else a.partials[(size_t)ii * NACC + A_UX + f - NHG_GEO] = sum;
        }
        if (lane >= NHG_GEO && lane < NHG) out[lane] = 0.0;
        j = a.dynamic ? next_item_s(a.counter, lane) : j + nw;
    }
}

// One wave per work item.  The item's pixels (stored backgrounds and own profile values of
// the listed boxes) are cut into runs of R rows of one strip; the runs, taken by row index and
// then by strip, are dealt round-robin to the wave's 32 pairs of lanes, so that an item of
// fewer than 64 strips still fills the wave.  The wave adds its NHG sums onto hg[item], which
// k_hess_second has filled with the second-derivative terms; the items of sources outside
// a.active (when given) get zeros.
// Each component costs its two exponentials once per run, so long runs pay, and a lane holds
// six sums per row beside the 40 of the Hessian: four rows a lane is what fits two waves a
// SIMD.  So a pair of lanes shares a run of twice as many rows: each takes every other
// component for all R rows, the even lane downwards and the odd lane upwards, then they
// exchange the farther halves of their rows' sums and each forms the products of its nearer
// R / 2.  Runs of four rows on one lane took 748 us on 1024 sources (1.6e7 visits), this 670
// (640 in blocks of one wave).
// A run may start up to R - 1 rows outside its box, where a narrow component must not have
// underflowed: eight rows with smooth PSFs (the exponent falls by less than 40 in seven rows
// at the centre), four otherwise (by 450 at the narrowest PSF there may be, sigma = 0.1 px).
constexpr int HESS_RUN = 8, HESS_RUN_SHARP = 4;   // rows per run of k_hess_geom

// v of the other lane of the pair (lanes 2 i, 2 i + 1).
__device__ __forceinline__ double pair_swap(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0xB1, 0xf, 0xf, true);   // quad_perm [1, 0, 3, 2]
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0xB1, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <int L, int R>
__global__ void __launch_bounds__(256, 2) k_hess_geom(AdjArgs a, const Item* __restrict__ items,
                                                   const PairDev* __restrict__ pairs,
                                                   const celeste_image* __restrict__ images,
                                                   const double* __restrict__ xs, const double* __restrict__ bg,
                                                   const double* __restrict__ tabp,
                                                   const double* __restrict__ coefp,
                                                   const double* __restrict__ own, const double* __restrict__ nu,
                                                   double* __restrict__ hg) {
    if (*a.status) return;
    __shared__ double t2[EXP_TAB];
    extern __shared__ double ltab[];   // [waves per block][NDH][NCP], sized at launch
    load_tables(t2, nullptr);
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    double* my = ltab + (threadIdx.x >> 6) * (NCP * NDH);
    int j = a.dynamic ? next_item_s(a.counter, lane) : blockIdx.x * wpb + (threadIdx.x >> 6);
    while (j < a.items.n) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(a.items, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        if (a.active && !a.active[p.src]) {
            if (lane < NHG) hg[(size_t)ii * NHG + lane] = 0.0;
            j = a.dynamic ? next_item_s(a.counter, lane) : j + nw;
            continue;
        }
        const celeste_image& im = images[p.img];
        const double* kp = coefp + (size_t)it.pair * NCOEF;
        const double k[NCOEF] = {kp[0], kp[1], kp[2], kp[3]};
        __builtin_amdgcn_wave_barrier();
        stage_hess(tabp + (size_t)it.pair * NCOMP * CST, nu, my, lane);
        const uint64_t live = item_live(tabp + (size_t)it.pair * NCOMP * CST, p, it, L, lane);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        double H[NHG];
#pragma unroll
        for (int f = 0; f < NHG; ++f) H[f] = 0.0;
        // runs of R rows per strip: those of the item's first strip, the longest
        const int nk = (min(L, p.h - (it.start / p.w) * L) + R - 1) / R;
        constexpr int HR = R / 2;
        const bool up = lane & 1;               // this lane walks its run upwards
        const double sg_row = up ? -1.0 : 1.0;
        for (int g = lane >> 1; g < it.count * nk; g += 32) {
            const int kr = g / it.count, q = g - kr * it.count;
            int c, r0, nrow;
            strip_geometry(p, it.start + q, L, c, r0, nrow);
            const int kk = kr * R;
            if (kk >= nrow) continue;   // both lanes of the pair
            const double px = (double)c, py0 = (double)(r0 + kk + (up ? R - 1 : 0));
            // first derivatives of the galaxy profile along the run (row i of the lane is row
            // kk + i of the strip, or kk + R - 1 - i upwards), summed over every other live
            // component: each component's value by the strip recurrence, z affine in the row
            double F[R][6];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int f = 0; f < 6; ++f) F[r][f] = 0.0;
#pragma unroll 1
            for (int grp = 0; grp < NPSF; ++grp) {
                if (!((live >> (NPSF + grp * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1))) continue;
                const double* es = my + grp;
                const double dx = px - es[H_CX * NCP], dy = py0 - es[H_CY * NCP];
                const double h2x = -0.5 * (dx * dx), mxy = -(dx * dy), h2y = -0.5 * (dy * dy);
                const double mdx = -sg_row * dx, mdyh = -fma(sg_row, dy, 0.5);
                for_live_pairs(live, grp, [&](int s0, int s1) {
                    const double* e = my + (up ? s1 : s0);
                    const double a = e[H_A * NCP], b = e[H_B * NCP], d = e[H_D * NCP];
                    const double xs2[2] = {fma(a, h2x, fma(b, mxy, fma(d, h2y, e[H_LW * NCP]))),
                                           clamp_arg(fma(b, mdx, d * mdyh))};
                    double ex[2];
                    fexps<2>(xs2, ex, t2);
                    double n = ex[0], rt = ex[1];
                    const double rdy = e[H_RDY * NCP];
                    const double wt = e[H_WT * NCP], sg = e[H_SGN * NCP], wnu = e[H_WNU * NCP];
                    const double zx0 = fma(a, dx, b * dy), zy0 = fma(b, dx, d * dy);
                    const double bs = b * sg_row, ds = d * sg_row;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double zx = fma(bs, (double)r, zx0), zy = fma(ds, (double)r, zy0);
                        const double wn = wt * n, vn = wnu * n;
                        F[r][0] = fma(wn, zx, F[r][0]);
                        F[r][1] = fma(wn, zy, F[r][1]);
                        F[r][2] = fma(sg, n, F[r][2]);
                        F[r][3] = fma(vn, fma(zx, zx, -a), F[r][3]);
                        F[r][4] = fma(vn, fma(zx, zy, -b), F[r][4]);
                        F[r][5] = fma(vn, fma(zy, zy, -d), F[r][5]);
                        if (r + 1 < R) {
                            n = n * rt;
                            rt = rt * rdy;
                        }
                    }
                });
            }
            // the lane's nearer rows, with the other lane's share of them
#pragma unroll
            for (int r = 0; r < HR; ++r)
#pragma unroll
                for (int f = 0; f < 6; ++f) F[r][f] += pair_swap(F[R - 1 - r][f]);
            // the star profile's, for those rows
            double S[HR][2];
#pragma unroll
            for (int r = 0; r < HR; ++r) S[r][0] = S[r][1] = 0.0;
#pragma unroll 1
            for (int grp = 0; grp < NPSF; ++grp) {
                if (!((live >> grp) & 1)) continue;
                const double* es = my + grp;
                const double dx = px - es[H_CX * NCP], dy = py0 - es[H_CY * NCP];
                const double a = es[H_A * NCP], b = es[H_B * NCP], d = es[H_D * NCP];
                const double zx0 = fma(a, dx, b * dy), zy0 = fma(b, dx, d * dy);
                const double xs2[2] = {fma(-0.5, fma(dx, zx0, dy * zy0), es[H_LW * NCP]),
                                       clamp_arg(-fma(sg_row, zy0, 0.5 * d))};
                double ex[2];
                fexps<2>(xs2, ex, t2);
                double n = ex[0], rt = ex[1];
                const double rdy = es[H_RDY * NCP];
                const double bs = b * sg_row, ds = d * sg_row;
#pragma unroll
                for (int r = 0; r < HR; ++r) {
                    S[r][0] = fma(n, fma(bs, (double)r, zx0), S[r][0]);
                    S[r][1] = fma(n, fma(ds, (double)r, zy0), S[r][1]);
                    if (r + 1 < HR) {
                        n = n * rt;
                        rt = rt * rdy;
                    }
                }
            }
            // products of first derivatives and the k-block entries, row by row (the pixel
            // scalars from the row's stored background and own values)
#pragma unroll
            for (int r = 0; r < HR; ++r) {
                const int at = up ? kk + R - 1 - r : kk + r;
                const int row = at < nrow ? at : kk;   // rows past the strip reuse row kk
                const size_t gi = (size_t)im.pix_offset + (size_t)(r0 + row) * im.W + c;
                const double x = xs[gi];
                if (!(at < nrow && x == x)) continue;
                const size_t vi = (size_t)p.visit_off + (size_t)(r0 + row - p.r0) * p.w + (c - p.c0);
                const double fs = own[2 * vi], fg = own[2 * vi + 1];
                const double Es = k[C_K1] * fs + k[C_K2] * fg;
                const double E = bg[2 * vi] + Es;
                const double V = bg[2 * vi + 1] + k[C_K3] * (fs * fs) + k[C_K4] * (fg * fg) - Es * Es;
                const double inv = frcp(E);
                const double inv2 = inv * inv;
                const double rr = V * inv2;
                const double lE = x * inv * (1.0 + rr) - 1.0;
                const double lV = -0.5 * x * inv2;
                const double lEE = -x * inv2 * (1.0 + 3.0 * rr);
                const double lEV = x * inv2 * inv;
                const double A = lE - 2.0 * Es * lV;
                // E_g = k1 S_g + k2 F_g and V_g = vS S_g + vF F_g (S_g = 0 but for the position),
                // so every entry is a combination of products of S and F with the scalars below
                const double k1 = k[C_K1], k2 = k[C_K2];
                const double vS = 2.0 * (k[C_K3] * fs - Es * k1), vF = 2.0 * (k[C_K4] * fg - Es * k2);
                const double lV2 = 2.0 * lV, lEE2 = lEE - lV2;
                const double cSS = fma(k1, fma(lEE2, k1, 2.0 * (lEV * vS)), lV2 * k[C_K3]);
                const double cFF = fma(k2, fma(lEE2, k2, 2.0 * (lEV * vF)), lV2 * k[C_K4]);
                const double cSF = fma(lEE2 * k1, k2, lEV * fma(k1, vF, k2 * vS));
                const double S0 = S[r][0], S1 = S[r][1];
                const double Q0 = fma(cSS, S0, cSF * F[r][0]), Q1 = fma(cSS, S1, cSF * F[r][1]);
                const double R0 = fma(cSF, S0, cFF * F[r][0]), R1 = fma(cSF, S1, cFF * F[r][1]);
                H[HG_XX] = fma(Q0, S0, fma(R0, F[r][0], H[HG_XX]));
                H[HG_XY] = fma(Q0, S1, fma(R0, F[r][1], H[HG_XY]));
                H[HG_YY] = fma(Q1, S1, fma(R1, F[r][1], H[HG_YY]));
#pragma unroll
                for (int qq = HG_YY + 1; qq < NHG_GEO; ++qq) {
                    const int g1 = hg_row(qq), h1 = hg_col(qq);
                    H[qq] = fma(g1 == 0 ? R0 : g1 == 1 ? R1 : cFF * F[r][g1], F[r][h1], H[qq]);
                }
                const double Rc = fma(-2.0 * lEV, Es, lEE2);
                const double rS = fma(Rc, k1, lEV * vS), rF = fma(Rc, k2, lEV * vF);
                const double ls = lEV * (fs * fs), lg = lEV * (fg * fg);
                const double cF[4] = {fs * rF, fma(fg, rF, A), ls * k2, fma(lg, k2, lV2 * fg)};
                const double cS[4] = {fma(fs, rS, A), fg * rS, fma(ls, k1, lV2 * fs), lg * k1};
#pragma unroll
                for (int qq = 0; qq < 5; ++qq) {
                    const int g1 = qq < 2 ? qq : qq + 1;
                    double* o = H + NHG_GEO + 4 * qq;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (g1 < 2) o[i] = fma(cS[i], S[r][g1], o[i]);
                        o[i] = fma(cF[i], F[r][g1], o[i]);
                    }
                }
            }
        }
        // added onto the second-derivative terms of k_hess_second
        int f;
        const double hv = wave_sums_dealt<NHG>(H, lane, f);
        if (f >= 0) hg[(size_t)ii * NHG + f] += hv;
        j = a.dynamic ? next_item_s(a.counter, lane) : j + nw;
    }
}

template <int L>
__global__ void __launch_bounds__(256) k_background_strips(BgArgs a, const Item* __restrict__ items,
                                                           const PairDev* __restrict__ pairs,
                                                           const celeste_image* __restrict__ images,
                                                           const int32_t* __restrict__ nbr,
                                                           const double* __restrict__ tabv,
                                                           const double* __restrict__ coefv,
                                                           double* __restrict__ bg) {
    if (*a.status) return;
    __shared__ double t2[EXP_TAB];
    load_tables(t2, nullptr);
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    for (int j = blockIdx.x * wpb + (threadIdx.x >> 6); j < a.items.n; j += nw) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(a.items, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        const celeste_image& im = images[p.img];
        for (int q = lane; q < it.count; q += 64) {
            int c, r0, nrow;
            strip_geometry(p, it.start + q, L, c, r0, nrow);
            double Eb[L], Vb[L];
            strip_background<L>(p, pairs, nbr, tabv, coefv, im, c, r0, Eb, Vb, t2);
#pragma unroll
            for (int k = 0; k < L; ++k) {
                if (k >= nrow) break;
                const size_t vi = (size_t)p.visit_off + (size_t)(r0 + k - p.r0) * p.w + (c - p.c0);
                bg[2 * vi] = Eb[k];
                bg[2 * vi + 1] = Vb[k];
            }
        }
    }
}

// Background of the listed visits from the other boxes' stored own profile values (sweeps:
// the stored values are kept current box by box), no Gaussian evaluated: strip_background_fg
// with the waits taken together.  Lane i reads the box and coefficients of neighbour i (64 at a
// time) and tests it against the item's rectangle; the wave then walks the neighbours that
// meet it, in order, their fields broadcast from that lane, and loads a lot of RB rows before
// adding it, rows outside the neighbour as its nearest row.  One neighbour after the other,
// each waiting for its index, its box, its coefficients and every row in turn, took 228 us for
// 1024 sources (1.6e7 visits) and 30 for 24 of 257 sources; this takes 147 and 14.
template <int L>
__global__ void __launch_bounds__(256) k_background_fg(BgArgs a, const Item* __restrict__ items,
                                                       const PairDev* __restrict__ pairs,
                                                       const celeste_image* __restrict__ images,
                                                       const int32_t* __restrict__ nbr,
                                                       const double* __restrict__ coefv,
                                                       const double* __restrict__ fgm, double* __restrict__ bg) {
    if (*a.status) return;
    constexpr int RB = L < 8 ? L : 8;
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    for (int j = blockIdx.x * wpb + (threadIdx.x >> 6); j < a.items.n; j += nw) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(a.items, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        const celeste_image& im = images[p.img];
        // rows and columns of the item's strips
        const int b0 = it.start / p.w, b1 = (it.start + it.count - 1) / p.w;
        const int ra = p.r0 + b0 * L, rb = p.r0 + min((b1 + 1) * L, p.h) - 1;
        const int ca = p.c0 + (b0 == b1 ? it.start - b0 * p.w : 0);
        const int cb = p.c0 + (b0 == b1 ? it.start + it.count - 1 - b0 * p.w : p.w - 1);
        for (int q0 = 0; q0 < it.count; q0 += 64) {
            int c, r0, nrow;
            strip_geometry(p, it.start + min(q0 + lane, it.count - 1), L, c, r0, nrow);
            if (q0 + lane >= it.count) nrow = 0;
            double Eb[L], Vb[L];
#pragma unroll
            for (int k = 0; k < L; ++k) {
                Eb[k] = r0 + k < im.H ? sky_at(im, r0 + k, c) : im.sky;
                Vb[k] = 0.0;
            }
            for (int n0 = p.nbr_begin; n0 < p.nbr_end; n0 += 64) {
                const int pi = nbr[min(n0 + lane, p.nbr_end - 1)];
                const PairDev* o = pairs + pi;
                const int or0 = o->r0, oc0 = o->c0, oh = o->h, ow = o->w;
                const long long off = o->visit_off;
                const double* kk = coefv + (size_t)pi * NCOEF;
                const double kn[NCOEF] = {kk[0], kk[1], kk[2], kk[3]};
                uint64_t meet = __builtin_amdgcn_ballot_w64(n0 + lane < p.nbr_end && or0 <= rb && or0 + oh > ra &&
                                                            oc0 <= cb && oc0 + ow > ca);
                while (meet) {
                    const int l = __builtin_ctzll(meet);
                    meet &= meet - 1;
                    const int nr0 = __builtin_amdgcn_readlane(or0, l), nc0 = __builtin_amdgcn_readlane(oc0, l);
                    const int nh = __builtin_amdgcn_readlane(oh, l), nww = __builtin_amdgcn_readlane(ow, l);
                    const uint64_t no = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(off >> 32), l) << 32 |
                                        (uint32_t)__builtin_amdgcn_readlane((int)off, l);
                    const double k1 = lane_bcast(kn[C_K1], l), k2 = lane_bcast(kn[C_K2], l),
                                 k3 = lane_bcast(kn[C_K3], l), k4 = lane_bcast(kn[C_K4], l);
                    if (c < nc0 || c >= nc0 + nww || r0 + L <= nr0 || r0 >= nr0 + nh) continue;
                    const double2* ob = reinterpret_cast<const double2*>(fgm) + no;
#pragma unroll
                    for (int b = 0; b < L; b += RB) {
                        double2 f[RB];
#pragma unroll
                        for (int i = 0; i < RB; ++i)
                            f[i] = ob[(uint32_t)(min(max(r0 + b + i - nr0, 0), nh - 1) * nww + (c - nc0))];
#pragma unroll
                        for (int i = 0; i < RB; ++i) {
                            const int r = r0 + b + i;
                            if (r < nr0 || r >= nr0 + nh) continue;
                            const double fs = f[i].x, fg = f[i].y;
                            const double Et = k1 * fs + k2 * fg;
                            Eb[b + i] += Et;
                            Vb[b + i] += k3 * fs * fs + k4 * fg * fg - Et * Et;
                        }
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < L; ++k) {
                if (k < nrow) {
                    const size_t vi = (size_t)p.visit_off + (size_t)(r0 + k - p.r0) * p.w + (c - p.c0);
                    reinterpret_cast<double2*>(bg)[vi] = make_double2(Eb[k], Vb[k]);
                }
            }
        }
    }
}

// Sum over each box of log(x!) (masked pixels excluded): a constant of the pixel terms,
// computed once per plan, one wave per box, fixed-order reduction.
__global__ void __launch_bounds__(256) k_pair_lgamma(const PairDev* __restrict__ pairs, int n_pairs,
                                                     const celeste_image* __restrict__ images,
                                                     const double* __restrict__ xs, double* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int w = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (w >= n_pairs) return;
    const PairDev p = pairs[w];
    const celeste_image& im = images[p.img];
    double acc = 0.0;
    for (int i = lane; i < p.h * p.w; i += 64) {
        const int rr = i / p.w;
        const double x = xs[(size_t)im.pix_offset + (size_t)(p.r0 + rr) * im.W + p.c0 + (i - rr * p.w)];
        if (x == x) acc += lgamma(x + 1.0);
    }
    acc = wave_sum(acc);
    if (lane == 0) out[w] = acc;
}

// Own star and galaxy profile values of every visit of the selected items, stored as
// [visit][2] (render pass 1; the fused adjoint reads them back instead of recomputing).
// Like the fused adjoint, the wave stages each item's box table into LDS and takes the seeds
// in the PSF groups' centre frames: the table read through scalar loads had the waves
// waiting on the scalar cache (render 0.488 -> 0.460 ms on the 2000-source field).
template <int L, bool ROWQ>
__global__ void __launch_bounds__(256) k_strip_fg(Sel sel, const Item* __restrict__ items,
                                                  const PairDev* __restrict__ pairs, const double* __restrict__ tab,
                                                  double* __restrict__ fgm, const int* status) {
    if (*status) return;
    __shared__ double t2[EXP_TAB];
    extern __shared__ double ltab[];   // [waves per block][STAGED], sized at launch
    load_tables(t2, nullptr);
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    double* my = ltab + (threadIdx.x >> 6) * STAGED;
    for (int j = blockIdx.x * wpb + (threadIdx.x >> 6); j < sel.n; j += nw) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(sel, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        const double* tb = tab + (size_t)it.pair * NCOMP * CST;
        __builtin_amdgcn_wave_barrier();
        stage_derived(tb, my, lane);
        if constexpr (ROWQ) stage_rows(tb, my + NCP * NDF, lane, t2);
        const uint64_t live = item_live(tb, p, it, L, lane);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int q = lane; q < it.count; q += 64) {
            int c, r0, nrow;
            strip_geometry(p, it.start + q, L, c, r0, nrow);
            double fs[L], fg[L];
            if constexpr (ROWQ) strip_values_q<L>(my, my + NCP * NDF, (double)c, (double)r0, fs, fg, t2, live);
            else strip_values_staged<L>(my, (double)c, (double)r0, fs, fg, t2, live);
#pragma unroll
            for (int k = 0; k < L; ++k) {
                if (k >= nrow) break;
                const size_t vi = (size_t)p.visit_off + (size_t)(r0 + k - p.r0) * p.w + (c - p.c0);
                fgm[2 * vi] = fs[k];
                fgm[2 * vi + 1] = fg[k];
            }
        }
    }
}

// Work of the strip passes under the component culling, for the FLOP count of a launch:
// one wave per item, each lane testing its component as the strip kernels do (item_live).
// out[0] strips, [1] visits, [2] PSF groups evaluated x strips, [3] live stars x strips,
// [4] live galaxy components x strips, [5] zero-component pads x strips, [6] live stars x
// visits, [7] live galaxy components x visits, [8] pads x visits (all summed over items).
__global__ void __launch_bounds__(64) k_live_counts(Sel sel, const Item* __restrict__ items,
                                                    const PairDev* __restrict__ pairs,
                                                    const double* __restrict__ tab, int L,
                                                    unsigned long long* __restrict__ out, const int* status) {
    if (*status) return;
    const int lane = threadIdx.x;
    unsigned long long sum[NLIVE_COUNTS] = {};   // this wave's items (lane 0)
    for (int j = blockIdx.x; j < sel.n; j += gridDim.x) {
        const int ii = __builtin_amdgcn_readfirstlane(sel_at(sel, j));
        const Item it = items[ii];
        const PairDev p = pairs[it.pair];
        const uint64_t live = item_live(tab + (size_t)it.pair * NCOMP * CST, p, it, L, lane);
        long long v = 0;   // visits of the item's strips
        for (int q = lane; q < it.count; q += 64) v += min(L, p.h - ((it.start + q) / p.w) * L);
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        unsigned long long groups = 0, stars = 0, gal = 0, pads = 0;
        for (int g = 0; g < NPSF; ++g) {
            const uint32_t gm = (uint32_t)(live >> (NPSF + g * NGAL_PER_PSF)) & ((1u << NGAL_PER_PSF) - 1);
            const int st = (int)((live >> g) & 1), ng = __builtin_popcount(gm);
            groups += (st || ng) ? 1 : 0;
            stars += st;
            gal += ng;
            pads += ng & 1;
        }
        const unsigned long long n = (unsigned long long)it.count, vv = (unsigned long long)v;
        sum[0] += n;
        sum[1] += vv;
        sum[2] += n * groups;
        sum[3] += n * stars;
        sum[4] += n * gal;
        sum[5] += n * pads;
        sum[6] += vv * stars;
        sum[7] += vv * gal;
        sum[8] += vv * pads;
    }
    if (lane == 0)
        for (int f = 0; f < NLIVE_COUNTS; ++f) atomicAdd(out + f, sum[f]);
}

// Render pass 2: E and V of every pixel of a tile, summing the stored own values of the
// tile's boxes in ascending box order (deterministic, no atomics).  Tile = (64 / tile_w * RP)
// rows x tile_w columns; lane l owns rows l / tile_w + k (64 / tile_w), k < RP.
// SUMS: the pixel terms of covered pixels summed per tile instead of the planes, which the
// total ELBO alone does not read.  The kernel runs at the rate of its loads and stores; on
// the 2000-source field the sums took 234 us with the planes written as well and a division
// per pixel, without them and with the reciprocal's Newton steps 194 (the table log instead
// of the library's: 192, not worth its block's table load).
template <int RP, bool SUMS>
__global__ void __launch_bounds__(256) k_gather_planes(RenderArgs a, const TileDev* __restrict__ tiles,
                                                       const int32_t* __restrict__ tile_list,
                                                       const PairDev* __restrict__ pairs,
                                                       const celeste_image* __restrict__ images,
                                                       const double* __restrict__ coef,
                                                       const double* __restrict__ fgm, double* __restrict__ Eout,
                                                       double* __restrict__ Vout, const double* __restrict__ xs,
                                                       double* __restrict__ tile_sums) {
    if (*a.status) return;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (t >= a.n_tiles) return;
    const TileDev td = tiles[t];
    const celeste_image& im = images[td.img];
    const int rows_per_pass = 64 / a.tile_w;
    const int c = td.c0 + lane % a.tile_w;
    int r[RP];
    double E[RP], V[RP];
    bool covered[RP];
#pragma unroll
    for (int k = 0; k < RP; ++k) {
        r[k] = td.r0 + lane / a.tile_w + k * rows_per_pass;
        E[k] = (r[k] < im.H && c < im.W) ? sky_at(im, r[k], c) : im.sky;
        V[k] = 0.0;
        covered[k] = false;
    }
    // boxes in list order (the sums are fixed-order); GU boxes' loads are issued before any
    // of them is added, so that their latencies overlap (2000-source field, 16 x 16 tiles: 0.533 ->
    // 0.499 ms for the render; four or eight boxes at a time cost occupancy and are slower)
    constexpr int GU = RP == 4 ? 2 : 4;   // two at 4 rows per lane keeps 7 waves per SIMD
    int j = td.list_begin;
    for (; j + GU <= td.list_end; j += GU) {
        double2 v[GU][RP];
        bool in[GU][RP];
        double kk[GU][NCOEF];
#pragma unroll
        for (int u = 0; u < GU; ++u) {
            const int pi = __builtin_amdgcn_readfirstlane(tile_list[j + u]);
            const PairDev o = pairs[pi];
            const double* kp = coef + (size_t)pi * NCOEF;
#pragma unroll
            for (int q = 0; q < NCOEF; ++q) kk[u][q] = kp[q];
#pragma unroll
            for (int k = 0; k < RP; ++k) {
                in[u][k] = !(r[k] < o.r0 || r[k] >= o.r0 + o.h || c < o.c0 || c >= o.c0 + o.w);
                const size_t vi = (size_t)o.visit_off + (size_t)(r[k] - o.r0) * o.w + (c - o.c0);
                v[u][k] = in[u][k] ? reinterpret_cast<const double2*>(fgm)[vi] : make_double2(0.0, 0.0);
            }
        }
#pragma unroll
        for (int u = 0; u < GU; ++u)
#pragma unroll
            for (int k = 0; k < RP; ++k) {
                if (!in[u][k]) continue;
                const double fs = v[u][k].x, fg = v[u][k].y;
                const double Et = kk[u][C_K1] * fs + kk[u][C_K2] * fg;
                E[k] += Et;
                V[k] += kk[u][C_K3] * fs * fs + kk[u][C_K4] * fg * fg - Et * Et;
                if constexpr (SUMS) covered[k] = true;
            }
    }
    for (; j < td.list_end; ++j) {
        const int pi = __builtin_amdgcn_readfirstlane(tile_list[j]);
        const PairDev o = pairs[pi];
        const double* kp = coef + (size_t)pi * NCOEF;
        const double k1 = kp[C_K1], k2 = kp[C_K2], k3 = kp[C_K3], k4 = kp[C_K4];
#pragma unroll
        for (int k = 0; k < RP; ++k) {
            if (r[k] < o.r0 || r[k] >= o.r0 + o.h || c < o.c0 || c >= o.c0 + o.w) continue;
            const size_t vi = (size_t)o.visit_off + (size_t)(r[k] - o.r0) * o.w + (c - o.c0);
            const double fs = fgm[2 * vi], fg = fgm[2 * vi + 1];
            const double Et = k1 * fs + k2 * fg;
            E[k] += Et;
            V[k] += k3 * fs * fs + k4 * fg * fg - Et * Et;
            if constexpr (SUMS) covered[k] = true;
        }
    }
    double l = 0.0;
#pragma unroll
    for (int k = 0; k < RP; ++k) {
        if (r[k] >= im.H || c >= im.W) continue;
        const size_t gi = (size_t)im.pix_offset + (size_t)r[k] * im.W + c;
        if constexpr (!SUMS) {
            Eout[gi] = E[k];
            Vout[gi] = V[k];
        } else {
            // pixel term of a pixel some box covers (the total ELBO counts each such pixel once)
            const double x = xs[gi];
            if (covered[k] && x == x) {
                const double inv = frcp(E[k]);
                double lk = x * (log(E[k]) - 0.5 * (V[k] * inv * inv)) - E[k];
                if (a.g.consts.flags & CELESTE_INCLUDE_LGAMMA) lk -= lgamma(x + 1.0);
                l += lk;
            }
        }
    }
    if constexpr (SUMS) {
        l = wave_sum(l);
        if (lane == 0) tile_sums[t] = l;
    }
}

// Elementwise table-driven exp (fn 0), table-driven log (fn 1) and Newton reciprocal (fn 2),
// for testing them against the host's libm.
__global__ void __launch_bounds__(256) k_debug_math(int fn, const double* __restrict__ x, double* __restrict__ y,
                                                    int n) {
    __shared__ double t2[EXP_TAB];
    __shared__ double2 tl[128];
    load_tables(t2, tl);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    y[i] = fn == 0 ? fexp(x[i], t2) : fn == 1 ? flog(x[i], tl) : frcp(x[i]);
}

// ----------------------------------------------------------------------- launchers
hipError_t launch_debug_math(int fn, const double* x, double* y, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_debug_math, dim3((n + 255) / 256), dim3(256), 0, st, fn, x, y, n);
    return hipGetLastError();
}

hipError_t launch_pair_lgamma(const Geometry& g, int n_pairs, double* out, hipStream_t st) {
    if (n_pairs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pair_lgamma, dim3((n_pairs + 3) / 4), dim3(256), 0, st, g.pairs, n_pairs, g.images, g.x, out);
    return hipGetLastError();
}

hipError_t launch_fill_planes(const celeste_image* images, int n_img, int max_pix, double* E, double* V,
                              const int* status, hipStream_t st) {
    if (n_img <= 0) return hipSuccess;
    int bx = (max_pix + 255) / 256;
    if (bx > 4096) bx = 4096;
    hipLaunchKernelGGL(k_fill_planes, dim3(bx, n_img), dim3(256), 0, st, images, E, V, status);
    return hipGetLastError();
}

hipError_t launch_strip_fg(const Sel& sel, const Geometry& g, const double* tab, double* fg, int L, int grid, int wpb,
                           const int* status, hipStream_t st) {
    if (sel.n <= 0) return hipSuccess;
    const int need = (sel.n + wpb - 1) / wpb;
    if (grid > need) grid = need;
    if (grid < 1) grid = 1;
#define CEL_FG(LL, RQ)                                                                                          \
    hipLaunchKernelGGL((k_strip_fg<LL, RQ>), dim3(grid), dim3(64 * wpb), (size_t)wpb * STAGED * sizeof(double), st, \
                       sel, g.items, g.pairs, tab, fg, status)
    if (L == 8) {
        if (g.smooth) CEL_FG(8, true);
        else CEL_FG(8, false);
    } else if (L == 4) {
        if (g.smooth) CEL_FG(4, true);
        else CEL_FG(4, false);
    } else if (L == 16) {
        if (g.smooth) CEL_FG(16, true);
        else CEL_FG(16, false);
    } else {
        return hipErrorInvalidValue;
    }
#undef CEL_FG
    return hipGetLastError();
}

hipError_t launch_live_counts(const Sel& sel, const Geometry& g, const double* tab, int L,
                              unsigned long long* out, const int* status, hipStream_t st) {
    hipError_t e = hipMemsetAsync(out, 0, NLIVE_COUNTS * sizeof(unsigned long long), st);
    if (e != hipSuccess || sel.n <= 0) return e;
    const int grid = sel.n < 1024 ? sel.n : 1024;
    hipLaunchKernelGGL(k_live_counts, dim3(grid), dim3(64), 0, st, sel, g.items, g.pairs, tab, L, out, status);
    return hipGetLastError();
}

hipError_t launch_gather_planes(const RenderArgs& a, const double* fg, int wpb, hipStream_t st) {
    if (a.n_tiles <= 0) return hipSuccess;
    const dim3 grid((a.n_tiles + wpb - 1) / wpb);
    const int rp = a.tile_h * a.tile_w / 64;
    const Geometry& g = a.g;
#define GATHER_ARGS a, a.tiles, a.tile_list, g.pairs, g.images, a.coef, fg, a.E, a.V, g.x, a.tile_sums
    if (a.tile_sums) {
        if (rp == 1) hipLaunchKernelGGL((k_gather_planes<1, true>), grid, dim3(64 * wpb), 0, st, GATHER_ARGS);
        else if (rp == 2) hipLaunchKernelGGL((k_gather_planes<2, true>), grid, dim3(64 * wpb), 0, st, GATHER_ARGS);
        else if (rp == 4) hipLaunchKernelGGL((k_gather_planes<4, true>), grid, dim3(64 * wpb), 0, st, GATHER_ARGS);
        else return hipErrorInvalidValue;
    } else {
        if (rp == 1) hipLaunchKernelGGL((k_gather_planes<1, false>), grid, dim3(64 * wpb), 0, st, GATHER_ARGS);
        else if (rp == 2) hipLaunchKernelGGL((k_gather_planes<2, false>), grid, dim3(64 * wpb), 0, st, GATHER_ARGS);
        else if (rp == 4) hipLaunchKernelGGL((k_gather_planes<4, false>), grid, dim3(64 * wpb), 0, st, GATHER_ARGS);
        else return hipErrorInvalidValue;
    }
#undef GATHER_ARGS
    return hipGetLastError();
}

hipError_t launch_render_strips(const Sel& sel, const Geometry& g, const double* tab, const double* coef, double* E,
                                double* V, int L, int grid, int wpb, const int* status, hipStream_t st) {
    if (sel.n <= 0) return hipSuccess;
    const int need = (sel.n + wpb - 1) / wpb;
    if (grid > need) grid = need;
    if (grid < 1) grid = 1;
    if (L == 8)
        hipLaunchKernelGGL(k_render_strips<8>, dim3(grid), dim3(64 * wpb), 0, st, sel, g.items, g.pairs, g.images, tab,
                           coef, E, V, status);
    else if (L == 4)
        hipLaunchKernelGGL(k_render_strips<4>, dim3(grid), dim3(64 * wpb), 0, st, sel, g.items, g.pairs, g.images, tab,
                           coef, E, V, status);
    else if (L == 16)
        hipLaunchKernelGGL(k_render_strips<16>, dim3(grid), dim3(64 * wpb), 0, st, sel, g.items, g.pairs, g.images,
                           tab, coef, E, V, status);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <class T, int BASE, bool DERIV, int L, bool FGM, int KK, bool ROWQ = false>
static void adjk(const AdjArgs& a, int grid, int wpb, hipStream_t st) {
    const Geometry& g = a.g;
    // row factors where the pass reads the staged table and the plan's PSFs allow them
    if constexpr (!ROWQ && lds_table<T, BASE, DERIV, FGM>()) {
        if (g.smooth) {
            adjk<T, BASE, DERIV, L, FGM, KK, true>(a, grid, wpb, st);
            return;
        }
    }
    const size_t lds = lds_table<T, BASE, DERIV, FGM>() ? (size_t)wpb * STAGED * sizeof(double) : 0;
    hipLaunchKernelGGL((k_adjoint_strips<T, BASE, DERIV, L, FGM, KK, ROWQ>), dim3(grid), dim3(64 * wpb), lds, st, a,
                       g.items, g.pairs, g.images, g.nbr, g.x, a.E, a.V, a.bg, a.tab, a.coef, a.tab_val, a.coef_val,
                       a.active, a.fg, a.partials);
}

template <class T, int BASE, bool DERIV, int L>
static hipError_t adjs(const AdjArgs& a, int grid, int wpb, hipStream_t st) {
    constexpr bool is_double = std::is_same<T, double>::value;
    // own profile values from the render's stored values: double passes over planes or stored values
    constexpr bool own_fg = is_double && (BASE == BASE_PLANES || BASE == BASE_FG);
    // the pixel-level rows of the intermediate Hessian: double gradient passes over stored
    // backgrounds (own values from pass A, which also gives d fg / d frac_dev)
    constexpr bool can_kk = is_double && DERIV && BASE == BASE_BG;
    if (a.kk && !can_kk) return hipErrorInvalidValue;
    if constexpr (can_kk) {
        if (a.kk) {
            if (a.kk_pixel) adjk<T, BASE, DERIV, L, false, KK_PIXEL>(a, grid, wpb, st);
            else adjk<T, BASE, DERIV, L, false, KK_FULL>(a, grid, wpb, st);
            return hipSuccess;
        }
    }
    if constexpr (own_fg) {
        if (a.fg) {
            if constexpr (DERIV) {
                const Geometry& g = a.g;
                const size_t lds = (size_t)wpb * STAGED * sizeof(double);
#define CEL_ADJ(RQ)                                                                                                    \
    hipLaunchKernelGGL((k_adjoint_stored<BASE, L, RQ>), dim3(grid), dim3(64 * wpb), lds, st, a, g.items, g.pairs,      \
                       g.images, g.nbr, g.x, a.E, a.V, a.tab, a.coef, a.active, a.fg, a.partials)
                if (g.smooth) CEL_ADJ(true);
                else CEL_ADJ(false);
#undef CEL_ADJ
            } else {
                adjk<T, BASE, DERIV, L, true, KK_NONE>(a, grid, wpb, st);
            }
            return hipSuccess;
        }
    }
    if constexpr (!is_double && DERIV && BASE == BASE_PLANES) {
        // tangents over the render's stored values, where the row factors may be taken
        const Geometry& g = a.g;
        if (a.fg && g.smooth) {
            hipLaunchKernelGGL((k_tangent_stored<L>), dim3(grid), dim3(64 * wpb), (size_t)wpb * STAGED_T * sizeof(double),
                               st, a, g.items, g.pairs, g.images, g.x, a.E, a.V, reinterpret_cast<const dual*>(a.tab),
                               reinterpret_cast<const dual*>(a.coef), a.active, a.fg, reinterpret_cast<dual*>(a.partials));
            return hipSuccess;
        }
    }
    adjk<T, BASE, DERIV, L, false, KK_NONE>(a, grid, wpb, st);
    return hipSuccess;
}

template <class T, int BASE, bool DERIV>
static hipError_t adjs_L(const AdjArgs& a, int grid, int wpb, int L, hipStream_t st) {
    if (L == 8) return adjs<T, BASE, DERIV, 8>(a, grid, wpb, st);
    if (L == 4) return adjs<T, BASE, DERIV, 4>(a, grid, wpb, st);
    if (L == 16) return adjs<T, BASE, DERIV, 16>(a, grid, wpb, st);
    return hipErrorInvalidValue;
}

template <class T, int BASE>
static hipError_t adjs_D(const AdjArgs& a, bool deriv, int grid, int wpb, int L, hipStream_t st) {
    return deriv ? adjs_L<T, BASE, true>(a, grid, wpb, L, st) : adjs_L<T, BASE, false>(a, grid, wpb, L, st);
}

template <class T>
static hipError_t adjs_B(const AdjArgs& a, int base, bool deriv, int grid, int wpb, int L, hipStream_t st) {
    switch (base) {
        case BASE_PLANES: return adjs_D<T, BASE_PLANES>(a, deriv, grid, wpb, L, st);
        case BASE_BG: return adjs_D<T, BASE_BG>(a, deriv, grid, wpb, L, st);
        case BASE_NBR: return adjs_D<T, BASE_NBR>(a, deriv, grid, wpb, L, st);
        case BASE_FG: return a.fg ? adjs_D<T, BASE_FG>(a, deriv, grid, wpb, L, st) : hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_adjoint(const AdjArgs& a, bool tangent, int base, bool deriv, int grid, int wpb, int L,
                          hipStream_t st) {
    if (a.items.n <= 0) return hipSuccess;
    if (a.dynamic) {
        hipError_t e = launch_fill_int(a.counter, 0, 1, st);
        if (e != hipSuccess) return e;
    }
    const int need = (a.items.n + wpb - 1) / wpb;   // never more waves than items
    if (grid > need) grid = need;
    if (grid < 1) grid = 1;
    const hipError_t e = tangent ? adjs_B<dual>(a, base, deriv, grid, wpb, L, st)
                                 : adjs_B<double>(a, base, deriv, grid, wpb, L, st);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}


hipError_t launch_hess_geom(const AdjArgs& a, const double* nu, double* hg, int grid, int wpb, int L,
                            hipStream_t st) {
    if (a.items.n <= 0) return hipSuccess;
    if (L != 16 && L != 8 && L != 4) return hipErrorInvalidValue;
    const int need = (a.items.n + wpb - 1) / wpb;   // never more waves than items
    if (grid > need) grid = need;
    if (grid < 1) grid = 1;
    const Geometry& g = a.g;
    const size_t lds = (size_t)wpb * NCP * NDH * sizeof(double);
    // second-derivative terms first (they write hg), then the first-derivative products (added
    // onto hg); each kernel takes the items from a fresh queue when the queue is dynamic
    for (int pass = 0; pass < 2; ++pass) {
        if (a.dynamic) {
            hipError_t e = launch_fill_int(a.counter, 0, 1, st);
            if (e != hipSuccess) return e;
        }
#define CEL_GEOM(LL, RR)                                                                                           \
    hipLaunchKernelGGL((k_hess_geom<LL, RR>), dim3(grid), dim3(64 * wpb), lds, st, a, g.items, g.pairs, g.images,  \
                       g.x, a.bg, a.tab, a.coef, a.fg, nu, hg)
#define CEL_HG(LL)                                                                                                 \
    if (pass == 0)                                                                                                 \
        hipLaunchKernelGGL((k_hess_second<LL>), dim3(grid), dim3(64 * wpb), lds, st, a, g.items, g.pairs, g.images, \
                           g.x, a.bg, a.tab, a.coef, a.fg, nu, hg);                                                \
    else if (g.smooth)                                                                                             \
        CEL_GEOM(LL, (HESS_RUN < LL ? HESS_RUN : LL));                                                             \
    else                                                                                                           \
        CEL_GEOM(LL, HESS_RUN_SHARP)
        if (L == 16)
            CEL_HG(16);
        else if (L == 8)
            CEL_HG(8);
        else
            CEL_HG(4);
#undef CEL_HG
#undef CEL_GEOM
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_background(const BgArgs& a, int grid, int wpb, int L, hipStream_t st) {
    if (a.items.n <= 0) return hipSuccess;
    const int need = (a.items.n + wpb - 1) / wpb;
    if (grid > need) grid = need;
    if (grid < 1) grid = 1;
    const Geometry& g = a.g;
    if (a.fg) {
        if (L == 8)
            hipLaunchKernelGGL(k_background_fg<8>, dim3(grid), dim3(64 * wpb), 0, st, a, g.items, g.pairs, g.images,
                               g.nbr, a.coef_val, a.fg, a.bg);
        else if (L == 4)
            hipLaunchKernelGGL(k_background_fg<4>, dim3(grid), dim3(64 * wpb), 0, st, a, g.items, g.pairs, g.images,
                               g.nbr, a.coef_val, a.fg, a.bg);
        else if (L == 16)
            hipLaunchKernelGGL(k_background_fg<16>, dim3(grid), dim3(64 * wpb), 0, st, a, g.items, g.pairs, g.images,
                               g.nbr, a.coef_val, a.fg, a.bg);
        else
            return hipErrorInvalidValue;
        return hipGetLastError();
    }
    if (L == 8)
        hipLaunchKernelGGL(k_background_strips<8>, dim3(grid), dim3(64 * wpb), 0, st, a, g.items, g.pairs, g.images,
                           g.nbr, a.tab_val, a.coef_val, a.bg);
    else if (L == 4)
        hipLaunchKernelGGL(k_background_strips<4>, dim3(grid), dim3(64 * wpb), 0, st, a, g.items, g.pairs, g.images,
                           g.nbr, a.tab_val, a.coef_val, a.bg);
    else if (L == 16)
        hipLaunchKernelGGL(k_background_strips<16>, dim3(grid), dim3(64 * wpb), 0, st, a, g.items, g.pairs, g.images,
                           g.nbr, a.tab_val, a.coef_val, a.bg);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace cel
