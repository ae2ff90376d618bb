// Batched Newton trust-region step (Section IV-D of Regier et al. 2018: Newton's method
// with exact Hessians and a trust region; the paper solves the trust-region subproblem
// through an eigendecomposition, Section VI-B).  One wave per source:
//  1. map gradient and Hessian to unconstrained coordinates (logit of q, frac_dev and
//     axis ratio; log of radius and of every variance; identity otherwise; with the
//     colour-prior mixture, each type's 8 responsibilities through a softmax whose last
//     logit is fixed at 0, so 27 + 2 x 7 = 41 coordinates: B = J^T (-H) J - sum_i g_i
//     d2 theta_i / d eta^2 with the Jacobian J of theta(eta));
//  2. Householder reduction of the model Hessian (27 x 27, or 41 x 41) to tridiagonal
//     form T = Q^T B Q, lane t holding row t in registers; Q is kept as its reflectors (Q p is
//     applied reflector by reflector), never formed;
//  3. exact subproblem  min g'p + p'Bp/2, |p| <= radius  on T (More and Sorensen's
//     method; Nocedal & Wright, Alg. 4.3): 64 values of mu at a time, one a lane, each with
//     its own O(n) factorisation and solve, narrow the bracket of the least mu for which
//     T + mu I is positive definite and |p(mu)| <= radius (mu = 0: the interior Newton step);
//  4. near the hard case (gradient nearly orthogonal to the lowest eigenvector), the full
//     eigendecomposition instead: implicit QL with Wilkinson's shift on T (Golub and Van
//     Loan, Matrix Computations, Sec. 8.3; Bowdler, Martin, Reinsch and Wilkinson, Numer.
//     Math. 11, 1968) and the subproblem in the eigenbasis, the hard case along the
//     eigenvector of the smallest eigenvalue;
//  5. trial point and predicted increase.
// k_tr_update compares the actual and predicted increase and updates point and radius; where
// the trial point was accepted its gradient and Hessian are then formed in place of the
// current ones.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "model.h"

namespace cel {

constexpr int NEM = NP + 2 * (NMIX - 1);   // unconstrained coordinates with the mixture: 41
constexpr int QL_MAX_ITER = 60;   // QL iterations per eigenvalue before giving up
constexpr double EPS_D = 2.220446049250313e-16;   // 2^-52

// Wave-wide minimum and maximum (every lane receives the result).
__device__ inline double wave_min(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ inline double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ inline int param_kind(int i) {
    // 1: logit, 2: log, 0: identity
    if (i == 2 || i == 3 || i == 6) return 1;
    if (i == 5) return 2;
    if (i >= 7) {
        const int o = (i - 7) % 10;
        if (o == 1 || o >= 6) return 2;
    }
    return 0;
}

// theta -> eta and the first two derivatives of theta(eta).
__device__ inline void to_unconstrained(int i, double th, double& eta, double& d1, double& d2) {
    const int k = param_kind(i);
    if (k == 1) {
        eta = log(th) - log1p(-th);
        d1 = th * (1.0 - th);
        d2 = d1 * (1.0 - 2.0 * th);
    } else if (k == 2) {
        eta = log(th);
        d1 = th;
        d2 = th;
    } else {
        eta = th;
        d1 = 1.0;
        d2 = 0.0;
    }
}

__device__ inline double from_unconstrained(int i, double eta) {
    const int k = param_kind(i);
    if (k == 1) return 1.0 / (1.0 + exp(-eta));
    if (k == 2) return exp(eta);
    return eta;
}

// Trial row theta(eta + p) from the unconstrained coordinates and the step (LDS), one lane per
// entry of the row: the 27 model parameters through their own maps; with the mixture, each
// type's responsibilities through the softmax of its 7 coordinates and a fixed 0 (shifted by
// their maximum so that no exponential overflows); zero padding.
template <int M>
__device__ inline void write_trial(int t, const double* eta, const double* p, double* trial) {
    if (t < NP) {
        trial[t] = from_unconstrained(t, eta[t] + p[t]);
    } else if (M != NP && t < NPK) {
        const int ty = (t - NP) / NMIX, d = (t - NP) % NMIX;
        const int c0 = NP + (NMIX - 1) * ty;
        double mx = 0.0;
        for (int e = 0; e < NMIX - 1; ++e) mx = fmax(mx, eta[c0 + e] + p[c0 + e]);
        double z = exp(-mx);
        for (int e = 0; e < NMIX - 1; ++e) z += exp(eta[c0 + e] + p[c0 + e] - mx);
        const double num = d < NMIX - 1 ? exp(eta[c0 + d] + p[c0 + d] - mx) : exp(-mx);
        trial[t] = num / z;
    } else if (t < ROW) {
        trial[t] = 0.0;
    }
}

// Sum over the wave (every lane receives it) by data-parallel-primitive moves: rows of 16
// lanes by shifts, then across the rows.  No LDS round trips: six shuffles cost several times
// as much, and the reflections below wait on two sums each.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wsum(double v) {
    v = dpp_add<0x111, 0xf>(v);   // row_shr:1, 2, 4, 8: lane 15 of a row holds its sum
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return lane_bcast(v, 63);
}

// Householder steps k = k0 .. k1 - 1 of the reduction B = Q T Q^T (T tridiagonal: diagonal
// dv, ev of lane i coupling rows i and i + 1; Q = H_0 H_1 ..., H_k = I - bh_k v_k v_k^T).  Lane
// t holds row t in registers, b[c] being column k + c at step k: each update moves the row
// one column to the left, so that all register indices are constants while k is a loop
// counter (unrolled over k the code would run out of the instruction cache).  The entries of
// v and w = beta B v - ... that every row needs come by v_readlane.  SZ >= M - k0: columns
// carried.  g becomes H_k g; v_k goes to row k of Q.
template <int M, int SZ, int LD>
__device__ __forceinline__ void reflect(int k0, int k1, int t, double (&b)[M], double& dv, double& ev, double& bhv,
                                        double& g, double (*Q)[LD]) {
    for (int k = k0; k < k1; ++k) {
        const double x = b[0];
        const double dk = lane_bcast(x, k), x0 = lane_bcast(x, k + 1);
        const double ci = (t >= k + 2 && t < M) ? x : 0.0;
        const double sigma = wsum(ci * ci);
        double vi = 0.0, alpha = x0, beta = 0.0;   // sigma = 0: already tridiagonal in this column, H_k = I
        if (sigma != 0.0) {
            const double mu = sqrt(x0 * x0 + sigma);
            alpha = x0 > 0.0 ? -mu : mu;
            const double v0 = x0 - alpha;
            beta = 2.0 / (v0 * v0 + sigma);
            vi = (t == k + 1) ? v0 : ci;
        }
        dv = t == k ? dk : dv;
        ev = t == k ? alpha : ev;
        bhv = t == k ? beta : bhv;
        if (t < M) Q[k][t] = vi;
        double p0 = 0.0, p1 = 0.0;
#pragma unroll
        for (int c = 1; c < SZ; ++c) {
            const double vc = lane_bcast(vi, k + c);
            if (c & 1) p0 = fma(b[c], vc, p0);
            else p1 = fma(b[c], vc, p1);
        }
        const double pi = (t > k && t < M) ? beta * (p0 + p1) : 0.0;
        const double vp = wsum(vi * pi), vg = wsum(vi * g);
        g = fma(-(beta * vg), vi, g);
        const double wi = fma(-(0.5 * beta * vp), vi, pi);
#pragma unroll
        for (int c = 1; c < SZ; ++c)
            b[c - 1] = fma(-wi, lane_bcast(vi, k + c), fma(-vi, lane_bcast(wi, k + c), b[c]));
    }
}

// y = -(T + mu I)^-1 g for this lane's own mu, T and g (in LDS as (d_i, e_i) and g_i) being
// those of the wave's source: eliminated from both ends at once (the twisted factorisation:
// two independent chains of pivots half as long as one), meeting in row M / 2.  Returns
// whether every pivot is positive (T + mu I positive definite: the pivots have its inertia);
// n2 = |y|^2.
template <int M>
__device__ __forceinline__ bool shifted_solve(const double2* __restrict__ de, const double* __restrict__ g, double mu,
                                              double (&y)[M], double& n2) {
    constexpr int H = M / 2;
    double c[M];
    bool pos = true;
    double ct = 0.0, at = 0.0, et = 0.0;   // top chain: c and a of the row above, its coupling
    double cb = 0.0, ab = 0.0;             // bottom chain
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const double2 u = de[i];
        const double den = fma(-et, ct, u.x + mu);
        pos = pos && den > 0.0;
        const double inv = frcp(den);
        at = fma(-et, at, -g[i]) * inv;
        ct = u.y * inv;
        et = u.y;
        y[i] = at;
        c[i] = ct;
        const int q = M - 1 - i;
        if (q > H) {
            const double2 w = de[q];
            const double eq = q < M - 1 ? w.y : 0.0, ep = de[q - 1].y;
            const double dnb = fma(-eq, cb, w.x + mu);
            pos = pos && dnb > 0.0;
            const double ivb = frcp(dnb);
            ab = fma(-eq, ab, -g[q]) * ivb;
            cb = ep * ivb;
            y[q] = ab;
            c[q] = cb;
        }
    }
    {
        const double2 u = de[H];
        const double den = fma(-et, ct, fma(-u.y, cb, u.x + mu));
        pos = pos && den > 0.0;
        y[H] = fma(-et, at, fma(-u.y, ab, -g[H])) * frcp(den);
    }
#pragma unroll
    for (int i = 1; i <= H; ++i) {
        if (H - i >= 0) y[H - i] = fma(-c[H - i], y[H - i + 1], y[H - i]);
        if (H + i < M) y[H + i] = fma(-c[H + i], y[H + i - 1], y[H + i]);
    }
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int i = 0; i < M; ++i) {
        if (i & 1) s1 = fma(y[i], y[i], s1);
        else s0 = fma(y[i], y[i], s0);
    }
    n2 = s0 + s1;
    return pos;
}

// M = NP (27 parameters) or NEM (43 parameters with the colour-prior mixture, 41
// unconstrained coordinates); NT parameters in theta, gradient and Hessian.
//
// One wave per source, so a launch lasts as long as one source's chain of dependent
// operations (and no longer for 1024 sources than for one).  Held against the form that kept
// the matrix in LDS, formed the smallest eigenvalue by Sturm counts and walked the secular
// equation one mu at a time: 27 parameters 123 -> 43 us (batches of a 400-source sweep), 172
// -> 50 us (1024 sources); 41 coordinates 235 -> 83 us (16 sources).
template <int M>
__global__ void __launch_bounds__(64) k_tr_solve(TrArgs a) {
    constexpr int NT = M == NP ? NP : NPK;
    constexpr int NJ = M == NP ? 28 : 44;   // rows of the LDS matrices (NT, padded)
    constexpr int LD = M == NP ? 29 : 45;   // padded LDS row (odd: rows and columns free of bank conflicts)
    if (*a.status) return;
    const int j = blockIdx.x;
    const int s = sel_at(a.srcs, j);
    const int t = threadIdx.x;
    __shared__ double B[NJ][LD];   // the Hessian, the model Hessian; later the eigenvectors Z of T (QL path)
    __shared__ double Q[NJ][LD];   // row k: the k-th Householder reflector v_k
    __shared__ double2 de[NJ];     // T: (d_i, e_i), e_i coupling rows i and i + 1
    __shared__ double vs[NJ], dd[NJ], gt[NJ], eta[NJ], d1[NJ], ph[NJ], pv[NJ];
    const double* th = a.theta + (size_t)s * ROW;
    const double* gr = a.grad + (size_t)s * ROW;
    const double* H = a.hess + (size_t)j * NT * NT;
    for (int idx = t; idx < NT * NT; idx += 64) B[idx / NT][idx % NT] = H[idx];
    double gmv = 0.0, lamv = 0.0;   // lane i: gradient in coordinate i; its diagonal curvature term
    if (t < NP) {
        double e, p1, p2;
        to_unconstrained(t, th[t], e, p1, p2);
        eta[t] = e;
        d1[t] = p1;
        // minimise f = -ELBO
        gmv = -p1 * gr[t];
        lamv = p2 * gr[t];   // diagonal curvature term of the ELBO
    }
    double b[M];   // lane t: row t of the model Hessian
    __syncthreads();
    if constexpr (M == NP) {
        const double dt = t < M ? -0.5 * d1[t] : 0.0;
        const int r = t < M ? t : 0;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            b[c] = dt * (B[r][c] + B[c][r]) * d1[c];
            if (t == c) b[c] -= lamv;
        }
    } else {
        // softmax coordinates of the responsibilities: kappa_d = e^{eta_d} / (1 + sum_e e^{eta_e})
        // (d < 7), kappa_7 = 1 / (1 + ...); J_de = kappa_d (delta_de - kappa_e), so for a vector x
        // over the responsibilities (J^T x)_e = kappa_e (x_e - sum_d kappa_d x_d);
        // sum_d g_d d2 kappa_d / d eta_e d eta_f = delta_ef (gk_e - S kappa_e) - gk_e kappa_f
        // - kappa_e gk_f + 2 S kappa_e kappa_f with gk_e = g_e kappa_e, S = sum_d g_d kappa_d
        __shared__ double kap[2][NMIX], gkp[2][NMIX], sk[2];
        double (*G)[LD] = Q;            // symmetric H times J (where Q is kept later)
        __shared__ double SG[2][LD];    // sum_d kappa_d G[d][c] of each type
        if (t < 2 * NMIX) {
            kap[t / NMIX][t % NMIX] = th[NP + t];
            gkp[t / NMIX][t % NMIX] = th[NP + t] * gr[NP + t];
        }
        __syncthreads();
        const int ty = t >= NP ? (t - NP) / (NMIX - 1) : 0, e = t >= NP ? (t - NP) % (NMIX - 1) : 0;
        if (t < 2) {
            double S = 0.0;
            for (int d = 0; d < NMIX; ++d) S += gkp[t][d];
            sk[t] = S;
        }
        __syncthreads();
        if (t >= NP && t < M) {
            eta[t] = log(kap[ty][e]) - log(kap[ty][NMIX - 1]);
            gmv = -(gkp[ty][e] - kap[ty][e] * sk[ty]);
        }
        // G = Hs J, lane k owning row k
        if (t < NT) {
            for (int c = 0; c < NP; ++c) G[t][c] = 0.5 * (B[t][c] + B[c][t]) * d1[c];
            for (int y = 0; y < 2; ++y) {
                double h[NMIX], S = 0.0;
#pragma unroll
                for (int d = 0; d < NMIX; ++d) {
                    const int k = NP + NMIX * y + d;
                    h[d] = 0.5 * (B[t][k] + B[k][t]);
                    S = fma(h[d], kap[y][d], S);
                }
#pragma unroll
                for (int d = 0; d < NMIX - 1; ++d) G[t][NP + (NMIX - 1) * y + d] = kap[y][d] * (h[d] - S);
            }
        }
        __syncthreads();
        if (t < M)
            for (int y = 0; y < 2; ++y) {
                double S = 0.0;
                for (int d = 0; d < NMIX; ++d) S = fma(kap[y][d], G[NP + NMIX * y + d][t], S);
                SG[y][t] = S;
            }
        __syncthreads();
        // -J^T G - curvature, lane r owning row r
        if (t < M)
            for (int c = 0; c < M; ++c) {
                double v;
                if (t < NP) {
                    v = -d1[t] * G[t][c];
                    if (c == t) v -= lamv;
                } else {
                    v = -kap[ty][e] * (G[NP + NMIX * ty + e][c] - SG[ty][c]);
                    if (c >= NP && (c - NP) / (NMIX - 1) == ty) {
                        const int f = (c - NP) % (NMIX - 1);
                        const double ke = kap[ty][e], kf = kap[ty][f], S = sk[ty];
                        double curv = -gkp[ty][e] * kf - ke * gkp[ty][f] + 2.0 * S * ke * kf;
                        if (e == f) curv += gkp[ty][e] - S * ke;
                        v -= curv;
                    }
                }
                B[t][c] = v;
            }
        __syncthreads();
        // symmetrised (the two halves differ by rounding only)
        const int r = t < M ? t : 0;
#pragma unroll
        for (int c = 0; c < M; ++c) b[c] = t < M ? 0.5 * (B[r][c] + B[c][r]) : 0.0;
    }
    // stop test on the unconstrained gradient
    const double gmax = wave_max((t < M) ? fabs(gmv) : 0.0);
    const bool stop = a.done[s] || !(gmax >= a.gtol);
    if (t == 0) a.live[s] = stop ? 0 : 1;
    double* trial = a.theta_trial + (size_t)s * ROW;
    if (stop) {
        if (t < ROW) trial[t] = (t < NT) ? th[t] : 0.0;
        if (t == 0) {
            a.pred[2 * s] = 0.0;
            a.pred[2 * s + 1] = 0.0;
            a.done[s] = 1;
        }
        return;
    }
    // ---- reduction to tridiagonal form; lane i ends with d_i, e_i, (Q^T g)_i and bh_i
    double dv = 0.0, ev = 0.0, bhv = 0.0, gtv = gmv;
    {
        constexpr int K1 = M / 3, K2 = 2 * M / 3;
        reflect<M, M, LD>(0, K1, t, b, dv, ev, bhv, gtv, Q);
        reflect<M, M - K1, LD>(K1, K2, t, b, dv, ev, bhv, gtv, Q);
        reflect<M, M - K2, LD>(K2, M - 2, t, b, dv, ev, bhv, gtv, Q);
        const double d2 = lane_bcast(b[0], M - 2), e2 = lane_bcast(b[0], M - 1), dl = lane_bcast(b[1], M - 1);
        dv = t == M - 2 ? d2 : t == M - 1 ? dl : dv;
        ev = t == M - 2 ? e2 : ev;
    }
    if (t < M) {
        de[t] = make_double2(dv, ev);
        gt[t] = gtv;
    }
    __syncthreads();
    // x <- Q x for the vector whose entry i lane i holds: the reflectors one by one (every lane
    // takes part in the wave sums)
    auto apply_q = [&](double x) {
        double vk = (t < M) ? Q[M - 3][t] : 0.0;
        for (int k = M - 3; k >= 0; --k) {
            const double vn = (t < M && k > 0) ? Q[k - 1][t] : 0.0;
            x -= lane_bcast(bhv, k) * wsum(vk * x) * vk;
            vk = vn;
        }
        return x;
    };
    // ---- subproblem on T (More and Sorensen's method; Nocedal & Wright, Alg. 4.3): the least
    // mu >= 0 with T + mu I positive definite and |p(mu)| <= R, p(mu) = -(T + mu I)^-1 Q^T g.
    // That predicate is false below the answer and true above it, so each round tries 64
    // values of mu, one a lane: first mu = 0 (the interior step) and a geometric ladder up to
    // a bound where it holds; then the bracket between the last false and the first true one,
    // around its secant point on 1 / |p(mu)| (nearly linear in mu) when T + mu I is positive
    // definite at the left end, evenly otherwise.  A bracket that shrinks onto the pole at the
    // smallest eigenvalue with |p| < R above it is the hard case (the gradient nearly
    // orthogonal to the lowest eigenvector), left to the eigenbasis below.
    const double R = a.radius[s];
    const double gn = sqrt(wsum((t < M) ? gtv * gtv : 0.0));
    double glo, scale;
    {
        const double em1 = __shfl(ev, t > 0 ? t - 1 : 0, 64);
        const double ep = t < M - 1 ? fabs(ev) : 0.0, em = t > 0 ? fabs(em1) : 0.0;
        glo = wave_min((t < M) ? dv - em - ep : INFINITY);
        scale = wave_max((t < M) ? fabs(dv) + em + ep : 0.0);
    }
    double lo = 0.0, hi = fmax(0.0, -glo) + gn / R + 1e-300;
    hi += 4.0 * EPS_D * hi;
    double fl = 0.0, fr = 0.0;   // 1 / |p| at the ends
    bool left_pd = false, hard = false;
    int pick = -1;   // the lane whose mu is taken
    double y[M], n2 = 0.0, nrm = 0.0;
    for (int round = 0; round < 64 && pick < 0 && !hard; ++round) {
        double mu;
        if (round == 0) {
            mu = t == 0 ? 0.0 : hi * exp2(-0.5 * (double)(63 - t));
        } else if (left_pd) {
            const double f = 1.0 / R;
            double ms = lo + (hi - lo) * ((f - fl) / (fr - fl));
            if (!(ms > lo && ms < hi)) ms = 0.5 * (lo + hi);
            mu = t < 31 ? ms - (ms - lo) * exp2(-1.5 * (double)(t + 1))
                 : t == 31 ? ms : t < 63 ? ms + (hi - ms) * exp2(-1.5 * (double)(63 - t)) : hi;
        } else {
            mu = t < 63 ? lo + (hi - lo) * ((double)(t + 1) / 64.0) : hi;
        }
        const bool pos = shifted_solve<M>(de, gt, mu, y, n2) && n2 < INFINITY;
        nrm = sqrt(n2);
        const unsigned long long ok = __ballot(pos && nrm <= R);
        // (at the upper bound the predicate holds up to rounding: taken as true)
        const int first = ok ? __ffsll((long long)ok) - 1 : 63;
        if (round == 0 && first == 0) {
            pick = 0;   // the interior step
            break;
        }
        const double dist = pos ? fabs(nrm - R) : INFINITY;
        const double best = wave_min(dist);
        if (best <= 1e-13 * R) {
            pick = __ffsll((long long)__ballot(dist == best)) - 1;
            break;
        }
        const unsigned long long pdm = __ballot(pos);
        const double finv = 1.0 / nrm;
        const double nhi = lane_bcast(mu, first);
        const double nfr = lane_bcast(finv, first);
        if (first > 0) {
            const double nlo = lane_bcast(mu, first - 1);
            if (nlo > lo || round == 0) {
                lo = nlo;
                left_pd = (pdm >> (first - 1)) & 1;
                fl = lane_bcast(finv, first - 1);
            }
        }
        const bool shrunk = nhi < hi || first > 0;
        hi = nhi;
        fr = nfr;
        // the bracket is as narrow as it gets (or, onto the pole, as the hard case is told by)
        if (!left_pd && hi - lo <= 1e-12 * scale) hard = true;
        else if (!shrunk || hi - lo <= 2.0 * EPS_D * hi) pick = first;
    }
    if (!hard) {
        if (pick < 0) pick = 63;   // not met: the last round's upper end
        if (t == pick) {
#pragma unroll
            for (int i = 0; i < M; ++i) vs[i] = y[i];
        }
        __syncthreads();
        const double yv = t < M ? vs[t] : 0.0;
        // predicted increase -(g.p + p.B.p/2) with p = Q y: g.p = gt.y, p.B.p = y.T.y
        const double yn = t < M - 1 ? vs[t + 1] : 0.0;
        const double tyy = (t < M) ? dv * yv * yv + (t < M - 1 ? 2.0 * ev * yv * yn : 0.0) : 0.0;
        const double pr = -(wsum((t < M) ? gtv * yv : 0.0) + 0.5 * wsum(tyy));
        if (t == 0) {
            a.pred[2 * s] = pr;
            a.pred[2 * s + 1] = lane_bcast(nrm, pick);
        }
        const double pq = apply_q(yv);   // p = Q y
        if (t < M) pv[t] = pq;
        __syncthreads();
        write_trial<M>(t, eta, pv, trial);
        return;
    }
    // ---- otherwise the full eigendecomposition: implicit QL on T.  Lane i keeps d_i and e_i in registers;
    // the scalar recurrence runs in every lane alike on values read across lanes with a
    // wave-uniform index, and lane i applies the rotations to row i of the eigenvector
    // matrix Z of T (in LDS, where B was; the eigenvectors of the model Hessian are Q Z).
    for (int idx = t; idx < NJ * NJ; idx += 64) {
        const int r = idx / NJ, c = idx - r * NJ;
        B[r][c] = (c == r) ? 1.0 : 0.0;
    }
    if (t < NJ) vs[t] = gtv;
    __syncthreads();
    bool converged = true;
    for (int l = 0; l < M && converged; ++l) {
        for (int iter = 0;; ++iter) {
            // m: the first index from l on whose e_m is negligible against its neighbours
            // (M - 1 if none), every lane testing its own e at once
            const double dn = __shfl(dv, t < 63 ? t + 1 : t, 64);
            const bool small = t < M - 1 && fabs(ev) <= EPS_D * (fabs(dv) + fabs(dn));
            const unsigned long long sm = __ballot(small) & (~0ull << l);
            const int m = sm ? __ffsll((long long)sm) - 1 : M - 1;
            if (m == l) break;
            if (iter == QL_MAX_ITER) {
                converged = false;
                break;
            }
            const double el = lane_bcast(ev, l), dl = lane_bcast(dv, l);
            double g = (lane_bcast(dv, l + 1) - dl) / (2.0 * el);
            double r = hypot(g, 1.0);
            g = lane_bcast(dv, m) - dl + el / (g + copysign(r, g));
            double sn = 1.0, cs = 1.0, p = 0.0;
            bool deflated = false;
            // row t of Z: entry zpos, rotated but not yet stored, is carried in zc
            int zpos = m;
            double zc = (t < M) ? B[t][m] : 0.0;
            for (int i = m - 1; i >= l; --i) {
                const double ei = lane_bcast(ev, i);
                const double f = sn * ei, b = cs * ei;
                // r = hypot(f, g) and 1 / r: the reciprocal square root of f^2 + g^2 (hardware
                // estimate, two Newton steps) where the squares stay far from overflow and
                // underflow; hypot and a division elsewhere
                const double q2 = fma(f, f, g * g);
                double rinv = 0.0;
                if (q2 > 0x1p-1000 && q2 < 0x1p+1000) {
                    double y = __builtin_amdgcn_rsq(q2);
                    y = fma(y, 0.5 * fma(-q2 * y, y, 1.0), y);
                    y = fma(y, 0.5 * fma(-q2 * y, y, 1.0), y);
                    rinv = y;
                    r = q2 * y;
                } else {
                    r = hypot(f, g);
                    if (r != 0.0) rinv = 1.0 / r;
                }
                ev = t == i + 1 ? r : ev;
                if (r == 0.0) {   // underflow: the matrix splits here
                    dv = t == i + 1 ? dv - p : dv;
                    ev = t == m ? 0.0 : ev;
                    deflated = true;
                    break;
                }
                sn = f * rinv;
                cs = g * rinv;
                g = lane_bcast(dv, i + 1) - p;
                r = (lane_bcast(dv, i) - g) * sn + 2.0 * cs * b;
                p = sn * r;
                dv = t == i + 1 ? g + p : dv;
                g = cs * r - b;
                if (t < M) {
                    const double zi = B[t][i];
                    B[t][i + 1] = sn * zi + cs * zc;
                    zc = cs * zi - sn * zc;
                }
                zpos = i;
            }
            if (t < M) B[t][zpos] = zc;
            if (deflated) continue;
            dv = t == l ? dv - p : dv;
            ev = t == l ? g : (t == m ? 0.0 : ev);
        }
    }
    if (t < NJ) dd[t] = dv;
    __syncthreads();
    if (!converged) {   // no step this iteration: the source stops (not met in practice)
        if (t < ROW) trial[t] = (t < NT) ? th[t] : 0.0;
        if (t == 0) {
            a.pred[2 * s] = 0.0;
            a.pred[2 * s + 1] = 0.0;
            a.done[s] = 1;
            a.live[s] = 0;
        }
        return;
    }
    // ---- subproblem in the eigenbasis: lane i holds lambda_i and entry i of (Q Z)^T g; the
    // sums over the eigenvalues are wave sums (equal in every lane, so every lane takes the
    // same branches)
    const double ev_t = (t < M) ? dv : 0.0;   // eigenvalue t
    double ghv = 0.0;   // (Q Z)^T g = Z^T (Q^T g)
    if (t < M)
        for (int k = 0; k < M; ++k) ghv += B[k][t] * vs[k];
    const double lmin = wave_min((t < M) ? ev_t : INFINITY);
    const double lmax = wave_max((t < M) ? fabs(ev_t) : 0.0);
    const int imin = __ffsll((long long)__ballot(t < M && ev_t == lmin)) - 1;   // its first lane
    const double gn2 = wave_sum(ghv * ghv);
    double phv = 0.0;
    bool solved = false;
    if (lmin > 0.0) {
        const double q = (t < M) ? ghv / ev_t : 0.0;
        if (wave_sum(q * q) <= R * R) {
            phv = -q;
            solved = true;
        }
    }
    if (!solved) {
        const double lo0 = fmax(0.0, -lmin);
        const double tol = 1e-12 * fmax(lmax, 1e-300);
        // hard case: gradient (numerically) orthogonal to the lowest eigenspace
        const bool low = t < M && ev_t <= lmin + tol;
        const double vr = (t < M && !low) ? ghv / (ev_t + lo0) : 0.0;
        const double gmin2 = wave_sum(low ? ghv * ghv : 0.0), prest2 = wave_sum(vr * vr);
        if (lo0 > 0.0 && gmin2 <= 1e-28 * fmax(gn2, 1e-300) && prest2 <= R * R) {
            phv = (t == imin) ? sqrt(fmax(R * R - prest2, 0.0)) : -vr;
        } else {
            double lo = lo0, hi = lo0 + sqrt(gn2) / R + 1e-300;
            double mu = hi;
            for (int itn = 0; itn < 200; ++itn) {
                const double den = ev_t + mu;
                const double v = (t < M) ? ghv / den : 0.0;
                const double n2 = wave_sum(v * v), d3 = wave_sum((t < M) ? v * v / den : 0.0);
                const double nrm = sqrt(n2);
                if (fabs(nrm - R) <= 1e-13 * R) break;
                if (nrm > R) lo = mu;
                else hi = mu;
                // Newton step on 1/R - 1/|p(mu)|
                double nmu = mu + (nrm - R) / R * (n2 / d3);
                if (!(nmu > lo && nmu < hi)) nmu = 0.5 * (lo + hi);
                if (nmu == mu) break;
                mu = nmu;
            }
            phv = (t < M) ? -ghv / (ev_t + mu) : 0.0;
        }
    }
    {
        const double pr = -wave_sum(ghv * phv + 0.5 * ev_t * phv * phv);
        const double pn = wave_sum(phv * phv);
        if (t == 0) {
            a.pred[2 * s] = pr;
            a.pred[2 * s + 1] = sqrt(pn);
        }
    }
    if (t < M) ph[t] = phv;
    __syncthreads();
    double zp = 0.0;   // Z ph, then p = Q (Z ph)
    if (t < M)
        for (int i = 0; i < M; ++i) zp += B[t][i] * ph[i];
    const double pq = apply_q(zp);
    if (t < M) pv[t] = pq;
    __syncthreads();
    write_trial<M>(t, eta, pv, trial);
}

__global__ void __launch_bounds__(128) k_tr_update(TrArgs a) {
    if (*a.status) return;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= a.srcs.n) return;
    const int s = sel_at(a.srcs, j);
    a.accepted[s] = 0;
    if (a.done[s]) return;
    const double f0 = a.elbo_cur[s], f1 = a.elbo_trial[s];
    const double pr = a.pred[2 * s], pn = a.pred[2 * s + 1];
    double R = a.radius[s];
    double rho = -1.0;
    const bool finite = (f1 == f1) && fabs(f1) < INFINITY;
    if (finite && pr > 0.0) rho = (f1 - f0) / pr;
    if (!finite || rho < 0.25) R = 0.25 * R;
    else if (rho > 0.75 && pn >= 0.99 * a.radius[s]) R = fmin(2.0 * R, a.radius_max);
    if (finite && rho > a.eta_accept) {
        double* th = a.theta + (size_t)s * ROW;
        const double* tr = a.theta_trial + (size_t)s * ROW;
        for (int i = 0; i < a.npar; ++i) th[i] = tr[i];
        a.elbo_cur[s] = f1;
        a.accepted[s] = 1;
    }
    // no further progress possible at working precision
    if (!(pr > 1e-15 * fabs(f0)) || R < 1e-12) a.done[s] = 1;
    a.radius[s] = R;
}

hipError_t launch_tr_solve(const TrArgs& a, hipStream_t st) {
    if (a.srcs.n <= 0) return hipSuccess;
    if (a.npar == NPK)
        hipLaunchKernelGGL(k_tr_solve<NEM>, dim3(a.srcs.n), dim3(64), 0, st, a);
    else if (a.npar == NP)
        hipLaunchKernelGGL(k_tr_solve<NP>, dim3(a.srcs.n), dim3(64), 0, st, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_tr_update(const TrArgs& a, hipStream_t st) {
    if (a.srcs.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tr_update, dim3((a.srcs.n + 127) / 128), dim3(128), 0, st, a);
    return hipGetLastError();
}

}  // namespace cel
