// HIP kernels of the FP64 ELBO path for gfx950 (CDNA4, wave64).
//
// Work decomposition:
//  * k_prep:      one wave per (source, image) box, one lane per table entry, builds the
//                 box's 45-Gaussian table (staged in LDS, written out contiguously) and
//                 brightness factors (value, or value + tangent).
//  * k_render:    one wave per render tile sums E[F] and Var[F] of every box that
//                 covers each pixel, in box order (deterministic, no atomics), and
//                 optionally the pixel terms of covered pixels (total ELBO).
//  * the fused adjoint and the strip render live in strips.hip.
//  * k_finalize:  one wave per source: 16 lanes sum a box's items in order, one lane per box
//                 applies the chain rule to the 27 parameters, lane i sums entry i over the
//                 boxes, and the KL term is added, its prior terms dealt to the lanes.
// Table entries are addressed with wave-uniform indices so the compiler serves them
// through scalar loads; pixel data is read coalesced along box rows.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "internal.h"
#include "model.h"

namespace cel {

// ----------------------------------------------------------------------- validation
// Domain of a source row: finite; q in (0,1); frac_dev in [0,1]; axis ratio in (0,1];
// radius > 0; variances > 0; with the colour-prior mixture (npar = NPK) every
// responsibility positive and each type's eight summing to 1 within 1e-9.  Branch-free so
// that the row's loads issue together.
__device__ inline bool row_ok(const double* __restrict__ p, int npar) {
    double v[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) v[i] = p[i];
    bool ok = true;
#pragma unroll
    for (int i = 0; i < NP; ++i) ok &= (bool)isfinite(v[i]);
    if (npar == NPK) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            double sum = 0.0;
#pragma unroll
            for (int d = 0; d < NMIX; ++d) {
                const double k = p[NP + NMIX * t + d];
                ok &= k > 0.0 && k <= 1.0;
                sum += k;
            }
            ok &= fabs(sum - 1.0) <= 1e-9;
        }
    }
    ok &= v[6] > 0.0 && v[6] < 1.0;
    ok &= v[2] >= 0.0 && v[2] <= 1.0;
    ok &= v[3] > 0.0 && v[3] <= 1.0;
    ok &= v[5] > 0.0;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int base = 7 + 10 * t;
        ok &= v[base + 1] > 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) ok &= v[base + 6 + k] > 0.0;
    }
    return ok;
}

__device__ inline bool listed_row_bad(const double* __restrict__ theta, const uint8_t* active, const int32_t* list,
                                      int j, int S, int npar) {
    const int s = list ? list[j] : j;
    if (s < 0 || s >= S) return true;
    if (active && !active[s]) return false;
    return !row_ok(theta + (size_t)s * ROW, npar);
}

// One thread per listed source; the status word was cleared by the launcher's fill.
__global__ void __launch_bounds__(256) k_validate(const double* __restrict__ theta, const uint8_t* active,
                                                  const int32_t* list, int n, int S, int npar, int* status) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n && listed_row_bad(theta, active, list, j, S, npar)) atomicOr(status, CELESTE_EDOMAIN);
}

// A few sources in one block: it alone writes the status word, so no launch has to clear the
// word first (one source's gradient 51.1 -> 50.3 us, 16 sources 61.1 -> 59.6).  A block reads
// all its rows through one compute unit: of 1024 sources it takes 10 us, the two launches 8.
constexpr int VALIDATE_BLOCK = 256;
__global__ void __launch_bounds__(VALIDATE_BLOCK) k_validate_block(const double* __restrict__ theta,
                                                                   const uint8_t* active, const int32_t* list, int n,
                                                                   int S, int npar, int* status) {
    const int j = threadIdx.x;
    const int bad = __syncthreads_or(j < n && listed_row_bad(theta, active, list, j, S, npar));
    if (j == 0) *status = bad ? CELESTE_EDOMAIN : 0;
}

// ----------------------------------------------------------------------- prep
// One wave per box, four boxes per block.  The boxes' intermediates (brightness factors,
// shape, PSF terms) are computed first by lanes 0..3 of the first wave, one box per lane,
// and passed through LDS (one wave pass for the block's four boxes instead of four);
// then lane c of each wave writes table entry c of its box and lane NCOMP the four
// brightness coefficients.
template <class T>
__global__ void __launch_bounds__(256) k_prep(PrepArgs a) {
    if (*a.status) return;
    // the box's table is staged in LDS and written out contiguously by the whole wave
    constexpr int TW = NCOMP * CST * scalar_traits<T>::width;   // doubles per table
    __shared__ double stage[4][TW];
    __shared__ T wsh[4][NW];
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    if (threadIdx.x < wpb) {   // box of wave threadIdx.x
        const int jb = blockIdx.x * wpb + threadIdx.x;
        if (jb < a.pairs.n) {
            const PairDev pd = a.g.pairs[sel_at(a.pairs, jb)];
            const celeste_image& im = a.g.images[pd.img];
            T* w = wsh[threadIdx.x];
            if (a.dir_mode == DIR_W) {
                // tangent along one of the box's intermediates
                double p[NP], wd[NW];
                for (int i = 0; i < NP; ++i) p[i] = a.theta[(size_t)pd.src * ROW + i];
                pair_w<double>(p, im, wd);
                for (int i = 0; i < NW; ++i) w[i] = scalar_traits<T>::make(wd[i], i == a.dir_unit ? 1.0 : 0.0);
            } else {
                T p[NP];
                for (int i = 0; i < NP; ++i) p[i] = seed<T>(a.theta, a.dir, a.dir_mode, a.dir_unit, pd.src, i);
                pair_w<T>(p, im, w);
            }
        }
    }
    __syncthreads();
    const int j = blockIdx.x * wpb + wave;
    const bool valid = j < a.pairs.n;
    const int pi = valid ? sel_at(a.pairs, j) : 0;
    if (valid) {
        const PairDev pd = a.g.pairs[pi];
        const celeste_image& im = a.g.images[pd.img];
        T* coef = reinterpret_cast<T*>(a.coef) + (size_t)pi * NCOEF;
        T w[NW];
        for (int i = 0; i < NW; ++i) w[i] = wsh[wave][i];
        if (lane < NCOMP) {
            build_comp_from_w<T>(w, im, a.g.consts, lane, reinterpret_cast<T*>(stage[wave]) + lane * CST);
        } else if (lane == NCOMP) {
            coef[C_K1] = w[W_K1];
            coef[C_K2] = w[W_K2];
            coef[C_K3] = w[W_K3];
            coef[C_K4] = w[W_K4];
        }
    }
    __syncthreads();
    if (valid) {
        double* out = reinterpret_cast<double*>(a.tab) + (size_t)pi * TW;
        for (int i = lane; i < TW; i += 64) out[i] = stage[wave][i];
    }
}

// ----------------------------------------------------------------------- render
// Tile = (64 / tile_w * RP) rows x tile_w cols; lane l owns rows (l / tile_w) + k * (64 / tile_w),
// k < RP, of column l % tile_w.
template <int RP>
__global__ void __launch_bounds__(256) k_render(RenderArgs a, const TileDev* __restrict__ tiles,
                                                const int32_t* __restrict__ tile_list,
                                                const PairDev* __restrict__ pairs,
                                                const celeste_image* __restrict__ images,
                                                const double* __restrict__ tab, const double* __restrict__ coef,
                                                const double* __restrict__ xs, double* __restrict__ Eout,
                                                double* __restrict__ Vout, double* __restrict__ tile_sums) {
    if (*a.status) return;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (t >= a.n_tiles) return;
    const TileDev td = tiles[t];
    const celeste_image& im = images[td.img];
    const int rows_per_pass = 64 / a.tile_w;
    const int c = td.c0 + lane % a.tile_w;
    int r[RP];
    bool inside[RP], covered[RP];
    double E[RP], V[RP], px[RP], py[RP];
#pragma unroll
    for (int k = 0; k < RP; ++k) {
        r[k] = td.r0 + lane / a.tile_w + k * rows_per_pass;
        inside[k] = r[k] < im.H && c < im.W;
        covered[k] = false;
        E[k] = inside[k] ? sky_at(im, r[k], c) : im.sky;
        V[k] = 0.0;
        px[k] = (double)c;
        py[k] = (double)r[k];
    }
    for (int j = td.list_begin; j < td.list_end; ++j) {
        const int pi = __builtin_amdgcn_readfirstlane(tile_list[j]);
        const PairDev o = pairs[pi];
        bool in[RP];
        bool any = false;
#pragma unroll
        for (int k = 0; k < RP; ++k) {
            in[k] = inside[k] && r[k] >= o.r0 && r[k] < o.r0 + o.h && c >= o.c0 && c < o.c0 + o.w;
            any |= in[k];
        }
        if (!any) continue;
        double fs[RP], fg[RP];
        eval_value<RP>(tab + (size_t)pi * NCOMP * CST, px, py, fs, fg);
        const double* k4 = coef + (size_t)pi * NCOEF;
        const double k1 = k4[C_K1], k2 = k4[C_K2], k3 = k4[C_K3], kk4 = k4[C_K4];
#pragma unroll
        for (int k = 0; k < RP; ++k) {
            if (!in[k]) continue;
            covered[k] = true;
            const double Et = k1 * fs[k] + k2 * fg[k];
            E[k] += Et;
            V[k] += k3 * fs[k] * fs[k] + kk4 * fg[k] * fg[k] - Et * Et;
        }
    }
    double l = 0.0;
#pragma unroll
    for (int k = 0; k < RP; ++k) {
        if (!inside[k]) continue;
        const size_t gi = (size_t)im.pix_offset + (size_t)r[k] * im.W + c;
        Eout[gi] = E[k];
        Vout[gi] = V[k];
        if (tile_sums && covered[k]) {
            const double x = xs[gi];
            if (x == x) {
                double lk = x * (log(E[k]) - 0.5 * V[k] / (E[k] * E[k])) - E[k];
                if (a.g.consts.flags & CELESTE_INCLUDE_LGAMMA) lk -= lgamma(x + 1.0);
                l += lk;
            }
        }
    }
    if (tile_sums) {
        l = wave_sum(l);
        if (lane == 0) tile_sums[t] = l;
    }
}

// ----------------------------------------------------------------------- finalize
// One wave per source.  The work of a source is short chains of transcendental functions
// and dependent loads, so a launch takes the latency of one source: everything that can go
// side by side is dealt to lanes (each box's item sums by 16 lanes, one per accumulator; the
// chain rule one box per lane; the KL one prior term per lane), against eight lanes a source
// looping over items, boxes and prior terms before.
// Time of the gradient form: one source 11.6 -> 7.0 us, 2000 sources 19 -> 15 us (dual
// numbers, 1024 sources: 37 -> 15 us).  Far more sources than that are bound by issue, which idle
// lanes cost: 20000 took 31 us with eight lanes a source, 55 so, and 48 with the registers held
// to four waves a SIMD (131 would take three; few sources take the same time).
constexpr int FIN_BOXES = 16;   // boxes per pass of a wave (a source has a handful)

// KL(q || prior) of the source whose row p[NPK] is in LDS, by one wave (every lane takes
// part).  With the mixture (K.mix set), a type's colour term is KL(Cat(kappa) || Cat(w)) +
// sum_d kappa_d KL(N(c_mu, diag c_var) || N(mu_d, S_d)), where the Gaussian KL is
// (sum_k P_kk v_k + delta^T P delta - 4 + log det S - sum_k log v_k) / 2, delta = c_mu - mu_d,
// P = S_d^-1; its derivatives: in kappa_d, log(kappa_d / w_d) + 1 + KL_d; in c_mu,
// sum_d kappa_d P_d delta_d; in c_var_k, sum_d kappa_d (P_d,kk - 1 / v_k) / 2.  Lanes 5 t + j, j = 0..4: the brightness (j = 0) and colour
// Gaussians of type t; lanes 16 + 8 t + d: mixture component d of type t; lanes 32, 33: the
// logarithms of the type's own term.  Returns the KL in every lane; with `grad`, gk[NPK]
// (LDS) receives minus its gradient.  sc: LDS scratch.
template <class T>
struct KlScratch {
    T lv[2][4];                 // log of the colour variances
    T part[2 * NMIX][9];        // kappa_d, kappa_d P_d delta_d, kappa_d diag P_d
};

template <class T>
__device__ inline T kl_wave(const T* p, const Consts& K, int lane, bool grad, T* gk, KlScratch<T>& sc) {
    const T zero = scalar_traits<T>::make(0.0, 0.0);
    const double phi = K.prior_phi;
    const T q = p[6], nq = 1.0 - q;
    const bool norm = lane < 10, comp = K.mix && lane >= 16 && lane < 16 + 2 * NMIX;
    const int t = norm ? lane / 5 : lane >= 16 + NMIX ? 1 : 0;
    const int j = norm ? lane - 5 * t : 0, d = comp ? lane - 16 - NMIX * t : 0;
    const int base = 7 + 10 * t;
    const int im = j == 0 ? base : base + 1 + j, iv = j == 0 ? base + 1 : base + 5 + j;
    const double m0 = j == 0 ? K.prior_r[t][0] : K.prior_c[t][0][j - 1];
    const double v0 = j == 0 ? K.prior_r[t][1] : K.prior_c[t][1][j - 1];
    // one logarithm a lane
    T arg = scalar_traits<T>::make(1.0, 0.0);
    if (norm) arg = p[iv];
    else if (comp) arg = p[NP + NMIX * t + d];
    else if (lane == 32) arg = q / phi;
    else if (lane == 33) arg = nq / (1.0 - phi);
    const T lg = log(arg);
    T c = zero;   // this lane's part of its type's KL
    const T w = t == 0 ? q : nq;
    const bool single = norm && (j == 0 || !K.mix);
    if (single) {
        const T dm = p[im] - m0;
        c = 0.5 * (log(v0) - lg + (p[iv] + dm * dm) / v0 - 1.0);
        if (grad) {
            gk[im] = zero - w * (dm / v0);
            gk[iv] = zero - w * (0.5 * (1.0 / v0 - 1.0 / p[iv]));
        }
    }
    if (K.mix) {
        if (norm && j > 0) sc.lv[t][j - 1] = lg;
        __syncthreads();
        if (comp) {
            const double* m = K.mix + (size_t)(t * NMIX + d) * MIXF;
            const T logv = sc.lv[t][0] + sc.lv[t][1] + sc.lv[t][2] + sc.lv[t][3];
            T dl[4], quad = zero, tr = zero;
#pragma unroll
            for (int k = 0; k < 4; ++k) dl[k] = p[base + 2 + k] - m[MX_MEAN + k];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                T r = zero;
#pragma unroll
                for (int l = 0; l < 4; ++l) r += m[MX_P + 4 * k + l] * dl[l];
                quad += dl[k] * r;
                tr += m[MX_P + 5 * k] * p[base + 6 + k];
                sc.part[lane - 16][1 + k] = arg * r;
                sc.part[lane - 16][5 + k] = arg * m[MX_P + 5 * k];
            }
            sc.part[lane - 16][0] = arg;
            const T kln = 0.5 * (tr + quad + (m[MX_LOGDET] - 4.0) - logv);
            const T lk = lg - m[MX_LOGW];
            c = arg * (lk + kln);
            if (grad) gk[NP + NMIX * t + d] = zero - w * (lk + 1.0 + kln);
        }
        __syncthreads();
        if (grad && norm && j > 0) {
            T gm = zero, gv = zero, ksum = zero;
#pragma unroll
            for (int e = 0; e < NMIX; ++e) {
                const T* pe = sc.part[NMIX * t + e];
                ksum += pe[0];
                gm += pe[j];
                gv += pe[4 + j];
            }
            gk[im] = zero - w * gm;
            gk[iv] = zero - w * (0.5 * (gv - ksum / p[iv]));
        }
    } else if (grad && lane >= 16 && lane < 16 + 2 * NMIX) {
        gk[NP + lane - 16] = zero;
    }
    const T k0 = wave_sum(t == 0 ? c : zero), k1 = wave_sum(t == 1 ? c : zero);
    const T lq = lane_bcast(lg, 32), lnq = lane_bcast(lg, 33);
    if (grad && lane < 6) gk[lane] = zero;
    if (grad && lane == 6) gk[6] = zero - (lq - lnq + k0 - k1);
    return q * lq + nq * lnq + q * k0 + nq * k1;
}

// Sum of the pixel terms of source s (every item of its boxes, which are consecutive), less
// the boxes' log(x!) sums: lanes over the items, a fixed butterfly.
template <class T>
__device__ inline T source_value(const FinArgs& a, int s, int lane) {
    const T* part = reinterpret_cast<const T*>(a.partials);
    const int pb = a.patch_ptr[s], pe = a.patch_ptr[s + 1];
    T v = scalar_traits<T>::make(0.0, 0.0);
    if (pb < pe) {
        const int i1 = a.g.pairs[pe - 1].item_end;
        for (int it = a.g.pairs[pb].item_begin + lane; it < i1; it += 64) v += part[(size_t)it * NACC + A_VAL];
        if (a.pair_lgamma)
            for (int pi = pb + lane; pi < pe; pi += 64) v = v - a.pair_lgamma[pi];
    }
    return wave_sum(v);
}

template <class T>
__global__ void __launch_bounds__(64, sizeof(T) == sizeof(double) ? 4 : 2) k_finalize(FinArgs a) {
    if (*a.status) return;
    const int lane = threadIdx.x;
    const int j = blockIdx.x;
    const int s = sel_at(a.srcs, j);
    if (a.active && !a.active[s]) return;
    __shared__ T p[NPK], gk[NPK];
    __shared__ KlScratch<T> sc;
    __shared__ T z[FIN_BOXES][NACC];
    __shared__ T g[FIN_BOXES][NP];
    const T zero = scalar_traits<T>::make(0.0, 0.0);
    if (lane < NPK) p[lane] = seed<T>(a.theta, a.dir, a.dir_mode, a.dir_unit, s, lane);
    __syncthreads();
    T val = zero, gs = zero;   // lane i: entry i of the gradient
    if (!a.deriv) {
        val = source_value<T>(a, s, lane);
    } else {
        const T* part = reinterpret_cast<const T*>(a.partials);
        const int pe = a.patch_ptr[s + 1];
        for (int b0 = a.patch_ptr[s]; b0 < pe; b0 += FIN_BOXES) {
            const int nb = min(FIN_BOXES, pe - b0);
            const int f = lane & 15;
            for (int q = lane >> 4; q < nb; q += 4) {
                if (f >= NACC) continue;
                T v = zero;
                const int i1 = a.g.pairs[b0 + q].item_end;
#pragma unroll 4
                for (int it = a.g.pairs[b0 + q].item_begin; it < i1; ++it) v += part[(size_t)it * NACC + f];
                if (f == A_VAL && a.pair_lgamma) v = v - a.pair_lgamma[b0 + q];
                z[q][f] = v;
            }
            __syncthreads();
            if (lane < nb) {
                T pr[NP], zr[NACC], gr[NP];
                for (int i = 0; i < NP; ++i) pr[i] = p[i];
                for (int i = 0; i < NP; ++i) gr[i] = zero;
                for (int i = 0; i < NACC; ++i) zr[i] = z[lane][i];
                chain_pair<T>(pr, a.g.images[a.g.pairs[b0 + lane].img], zr, gr);
                for (int i = 0; i < NP; ++i) g[lane][i] = gr[i];
            }
            __syncthreads();
            for (int q = 0; q < nb; ++q) {
                val += z[q][A_VAL];
                if (lane < NP) gs += g[q][lane];
            }
            __syncthreads();
        }
    }
    if (a.g.consts.flags & CELESTE_INCLUDE_KL) {
        val -= kl_wave<T>(p, a.g.consts, lane, a.deriv != 0, gk, sc);
        __syncthreads();
        if (a.deriv && lane < NPK) gs += gk[lane];
    }
    if (a.elbo && lane == 0) a.elbo[s] = value_of(val);
    if (!a.deriv || lane >= ROW) return;
    if (a.grad) a.grad[(size_t)s * ROW + lane] = lane < NPK ? value_of(gs) : 0.0;
    if (a.tangent && (lane < NPK || a.tangent_pad))
        a.tangent[(size_t)(a.tangent_by_list ? j : s) * a.tangent_stride + lane] = lane < NPK ? tangent_of(gs) : 0.0;
}

// Per-box sums of the item sums and each box's Hessian in its ten intermediates: one wave
// per box, lane f summing field f of the box's items in order (the 11 gradient sums, with
// `kk` the NKK_USED pixel-level and with `hg` the NHG closed-form Hessian sums: 63 fields),
// then the entries of hw[box] dealt to the lanes.  gw[box] receives the gradient sums.  One
// lane per box looping over items and fields took 20 + 36 us on 1024 sources, this 9.5 us.
// hw[dir][f] is the entry between dir and f over c_dir, the sums being in the accumulator
// scaling c_dir c_f d2L / dw_dir dw_f (c = 2 for Sxx, Syy).
// tangent: the tangent parts of accumulators 1..10 into hw[box][dir] instead (a tangent pass
// along intermediate dir).
__global__ void __launch_bounds__(256) k_pair_block(Sel sel, const PairDev* __restrict__ pairs,
                                                    const double* __restrict__ partials,
                                                    const double* __restrict__ kk, const double* __restrict__ hg,
                                                    int tangent, int dir, double* __restrict__ gw,
                                                    double* __restrict__ hw, const uint8_t* __restrict__ active,
                                                    const int* status) {
    if (*status) return;
    __shared__ double sums[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = blockIdx.x * 4 + wave;
    const int pi = sel_at(sel, min(j, sel.n - 1));
    const PairDev pd = pairs[pi];
    const bool on = j < sel.n && !(active && !active[pd.src]);
    const double* src = nullptr;
    int stride = 0;
    if (tangent) {
        if (lane < NW) {
            src = partials + 2 * (lane + 1) + 1;
            stride = 2 * NACC;
        }
    } else if (lane < NACC) {
        src = partials + lane;
        stride = NACC;
    } else if (lane < NACC + NKK_USED) {
        src = kk ? kk + (lane - NACC) : nullptr;
        stride = NKK;
    } else if (lane < NACC + NKK_USED + NHG) {
        src = hg ? hg + (lane - NACC - NKK_USED) : nullptr;
        stride = NHG;
    }
    double v = 0.0;
    if (on && src) {
#pragma unroll 4
        for (int it = pd.item_begin; it < pd.item_end; ++it) v += src[(size_t)it * stride];
    }
    if (tangent) {
        if (on && lane < NW) hw[((size_t)pi * NW + dir) * NW + lane] = v;
        return;
    }
    if (on && lane < NACC) gw[(size_t)pi * NACC + lane] = v;
    sums[wave][lane] = v;
    __syncthreads();
    if (!on) return;
    const double* K = sums[wave] + NACC;
    const double* H = K + NKK_USED;
    // kind of each intermediate: pixel-level index (k1..k4, frac_dev) and geometric index
    // (ux, uy, frac_dev, Sxx, Sxy, Syy)
    constexpr int pix[NW] = {0, 1, 2, 3, -1, -1, 4, -1, -1, -1};
    constexpr int geo[NW] = {-1, -1, -1, -1, 0, 1, 2, 3, 4, 5};
    constexpr int blk[5][5] = {{KK_11, KK_12, KK_13, KK_14, KK_F1},
                               {KK_12, KK_22, KK_23, KK_24, KK_F2},
                               {KK_13, KK_23, -1, -1, KK_F3},
                               {KK_14, KK_24, -1, -1, KK_F4},
                               {KK_F1, KK_F2, KK_F3, KK_F4, KK_FF}};
    for (int e = lane; e < NW * NW; e += 64) {
        const int r = e / NW, f = e - r * NW;
        if (pix[r] >= 0) {
            if (kk && pix[f] >= 0) {
                const int b = blk[pix[r]][pix[f]];
                hw[(size_t)pi * NW * NW + e] = b < 0 ? 0.0 : K[b];
            }
        } else if (hg) {
            const double inv_c = (r == W_SXX || r == W_SYY) ? 0.5 : 1.0;
            double h;
            if (f < 4) {
                h = H[NHG_GEO + 4 * (geo[r] < 2 ? geo[r] : geo[r] - 1) + f];
            } else {
                const int lo = min(geo[r], geo[f]), hi = max(geo[r], geo[f]);
                int k = 0;
                while (k < NHG_GEO && !(hg_row(k) == lo && hg_col(k) == hi)) ++k;
                h = H[k];
            }
            hw[(size_t)pi * NW * NW + e] = h * inv_c;
        }
    }
}

// Dense Hessian of ELBO_s (and, with `grad`, its gradient row) of the listed sources, one
// block each.  A box's ten intermediates depend on the parameters through 11 coordinates
// y = (u_x, u_y, frac_dev, ratio, angle, radius, q, m_s, v_s, m_g, v_g): m and v of a type are
// the mean and variance of its log flux in the box's band, sums of the type's brightness and
// (signed) colour entries.  Per box: J = dw/dy (10 x 11), H_y = J^T H_w J + sum_a (dL/dw_a)
// d2 w_a / dy2 in LDS; then entry (i, k) of the source's Hessian is the sum over its boxes of
// the signs times the entry of H_y that i and k map to, less the KL's second derivative.  The
// boxes' brightness factors are those of the tables at theta.  One thread per direction
// carrying dual numbers through every box's chain rule took 42 us on 1024 sources of 5 boxes
// and 67 us with up to 20 boxes a source (the transcendental functions and the 10 x 10
// products once per direction); this 30 and 27 us.
constexpr int NY = 11;           // coordinates of a box's intermediates
constexpr int ASM_BOXES = 10;     // boxes per pass of a block

// Coordinate of parameter i (< NP), and its coefficient in band `band`.
__device__ inline int y_of_param(int i) {
    if (i < 7) return i;
    const int t = (i - 7) / 10, o = (i - 7) - 10 * t;
    return 7 + 2 * t + (o == 1 || o >= 6 ? 1 : 0);
}
__device__ inline double y_coefficient(int i, int band) {
    const int o = i < 7 ? 0 : (i - 7) % 10;
    if (o < 2) return 1.0;
    const int k = o < 6 ? o - 2 : o - 6;   // colour; its sign in the band is BSIGN[band][k]
    const double sg = k < 2 ? (band <= k ? -1.0 : 0.0) : (band > k ? 1.0 : 0.0);
    return o < 6 ? sg : sg * sg;
}

// Shape covariance (xx, xy, yy) of the world frame and its first and second derivatives in
// (ratio, angle, radius): d[0..2], dd[rr, ra, re, aa, ae, ee].
__device__ inline void shape_derivatives(const double* p, double d[3][3], double dd[6][3]) {
    const double c = cos(p[4]), s = sin(p[4]), re = p[5], rho = p[3];
    const double c2 = c * c, s2 = s * s, cs = c * s, df = c2 - s2, q2 = rho * rho, om = 1.0 - q2, r2 = re * re;
    const double b[3] = {c2 + q2 * s2, cs * om, s2 + q2 * c2};   // covariance / radius^2
    const double e[3] = {s2, -cs, c2};                           // its derivative in ratio / (2 ratio)
    const double h[3] = {-2.0 * cs, df, 2.0 * cs};               // its derivative in angle / (1 - ratio^2)
    const double hh[3] = {-2.0 * df, -4.0 * cs, 2.0 * df};
    for (int k = 0; k < 3; ++k) {
        d[0][k] = 2.0 * r2 * rho * e[k];
        d[1][k] = r2 * om * h[k];
        d[2][k] = 2.0 * re * b[k];
        dd[0][k] = 2.0 * r2 * e[k];
        dd[1][k] = -2.0 * r2 * rho * h[k];
        dd[2][k] = 4.0 * re * rho * e[k];
        dd[3][k] = r2 * om * hh[k];
        dd[4][k] = 2.0 * re * om * h[k];
        dd[5][k] = 2.0 * b[k];
    }
}

// Entry (i, k) of the second derivative of -KL at row p (LDS), with gk and sc as kl_wave left
// them.
__device__ inline double kl_second(int i, int k, const double* p, const Consts& K, const double* gk,
                                   const KlScratch<double>& sc) {
    if (i > k) {
        const int t = i;
        i = k;
        k = t;
    }
    if (i < 6 || k < 6) return 0.0;
    const double q = p[6];
    if (k == 6) return -(1.0 / q + 1.0 / (1.0 - q));
    const int t = k >= NP ? (k - NP) / NMIX : (k - 7) / 10;
    const double w = t == 0 ? q : 1.0 - q;
    if (i == 6) return (t == 0 ? gk[k] : -gk[k]) / w;
    if ((i >= NP ? (i - NP) / NMIX : (i - 7) / 10) != t) return 0.0;
    const int base = 7 + 10 * t, oi = i - base, ok = k - base;
    if (k >= NP) {   // responsibility kappa_d
        const int d = k - NP - NMIX * t;
        const double* m = K.mix + (size_t)(t * NMIX + d) * MIXF;
        if (i >= NP) return i == k ? -w / p[k] : 0.0;
        if (oi < 2) return 0.0;
        if (oi < 6) return -w * (sc.part[t * NMIX + d][oi - 1] / p[k]);
        return -w * (0.5 * (m[MX_P + 5 * (oi - 6)] - 1.0 / p[i]));
    }
    const bool var = oi == 1 || oi >= 6;
    if (K.mix && oi >= 2) {
        double v = 0.0;
        if (!var && ok < 6) {
            for (int d = 0; d < NMIX; ++d)
                v += sc.part[t * NMIX + d][0] * K.mix[(size_t)(t * NMIX + d) * MIXF + MX_P + 4 * (oi - 2) + (ok - 2)];
            return -w * v;
        }
        if (i != k) return 0.0;
        for (int d = 0; d < NMIX; ++d) v += sc.part[t * NMIX + d][0];
        return -w * (0.5 * v / (p[i] * p[i]));
    }
    if (i != k) return 0.0;
    if (var) return -w * (0.5 / (p[i] * p[i]));
    return -w / (oi == 0 ? K.prior_r[t][1] : K.prior_c[t][1][oi - 2]);
}

template <int NPAR>
__global__ void __launch_bounds__(256) k_assemble_hessian(Sel srcs, Geometry g, const int32_t* __restrict__ patch_ptr,
                                                          const double* __restrict__ theta,
                                                          const double* __restrict__ coef,
                                                          const double* __restrict__ gw,
                                                          const double* __restrict__ hw,
                                                          double* __restrict__ hess, double* __restrict__ grad,
                                                          const uint8_t* __restrict__ active, const int* status) {
    if (*status) return;
    const int s = sel_at(srcs, blockIdx.x);
    if (active && !active[s]) return;
    const int tid = threadIdx.x;
    __shared__ double p[NPK], gk[NPK];
    __shared__ KlScratch<double> sc;
    __shared__ double sd[3][3], sdd[6][3];
    __shared__ double Hw[ASM_BOXES][NW * NW], J[ASM_BOXES][NW * NY], M[ASM_BOXES][NW * NY], Hy[ASM_BOXES][NY * NY];
    __shared__ double gx[ASM_BOXES][NW], gy[ASM_BOXES][NY];
    __shared__ double cf[ASM_BOXES][NP];   // coefficient of each parameter in its coordinate
    constexpr int NE = (NPAR * NPAR + 255) / 256;
    double out[NE], og = 0.0;
#pragma unroll
    for (int e = 0; e < NE; ++e) out[e] = 0.0;
    if (tid < NPK) p[tid] = theta[(size_t)s * ROW + tid];
    __syncthreads();
    if (tid == 64) shape_derivatives(p, sd, sdd);
    const bool kl = g.consts.flags & CELESTE_INCLUDE_KL;
    // the first wave forms the KL's gradient while the others wait at its barriers
    if (kl) (void)kl_wave<double>(p, g.consts, tid, true, gk, sc);
    const int pe = patch_ptr[s + 1];
    for (int b0 = patch_ptr[s]; b0 < pe; b0 += ASM_BOXES) {
        const int nb = min(ASM_BOXES, pe - b0);
        __syncthreads();
        // dL/dw (the sums hold twice the derivative in Sxx and Syy) and the symmetric d2L/dw2
        for (int e = tid; e < nb * NW; e += 256) {
            const int q = e / NW, a = e - q * NW;
            gx[q][a] = gw[(size_t)(b0 + q) * NACC + a + 1] * (a == W_SXX || a == W_SYY ? 0.5 : 1.0);
        }
        for (int e = tid; e < nb * NW * NW; e += 256) {
            const int q = e / (NW * NW), r = (e - q * NW * NW) / NW, c = e % NW;
            const bool pix_r = r < 4 || r == W_FDEV, pix_c = c < 4 || c == W_FDEV;
            const double* h = hw + (size_t)(b0 + q) * NW * NW;
            // pixel-level rows hold only their own block: the rest by symmetry
            Hw[q][r * NW + c] = (pix_r && !pix_c) ? h[c * NW + r]
                                                  : h[r * NW + c] * (c == W_SXX || c == W_SYY ? 0.5 : 1.0);
        }
        for (int e = tid; e < nb * NP; e += 256) {
            const int q = e / NP, i = e - q * NP;
            cf[q][i] = y_coefficient(i, g.images[g.pairs[b0 + q].img].band);
        }
        for (int e = tid; e < nb * NY; e += 256) {   // one column of J
            const int q = e / NY, y = e - q * NY;
            const celeste_image& im = g.images[g.pairs[b0 + q].img];
            const double* k = coef + (size_t)(b0 + q) * NCOEF;
            double* o = J[q] + y;
            for (int a = 0; a < NW; ++a) o[a * NY] = 0.0;
            const double a00 = im.wcs[0][0], a01 = im.wcs[0][1], a10 = im.wcs[1][0], a11 = im.wcs[1][1];
            if (y < 2) {
                o[W_UX * NY] = im.wcs[0][y];
                o[W_UY * NY] = im.wcs[1][y];
            } else if (y == 2) {
                o[W_FDEV * NY] = 1.0;
            } else if (y < 6) {
                const double xx = sd[y - 3][0], xy = sd[y - 3][1], yy = sd[y - 3][2];
                o[W_SXX * NY] = a00 * a00 * xx + 2.0 * a00 * a01 * xy + a01 * a01 * yy;
                o[W_SXY * NY] = a00 * a10 * xx + (a00 * a11 + a01 * a10) * xy + a01 * a11 * yy;
                o[W_SYY * NY] = a10 * a10 * xx + 2.0 * a10 * a11 * xy + a11 * a11 * yy;
            } else if (y == 6) {
                o[W_K1 * NY] = k[C_K1] / p[6];
                o[W_K2 * NY] = -k[C_K2] / (1.0 - p[6]);
                o[W_K3 * NY] = k[C_K3] / p[6];
                o[W_K4 * NY] = -k[C_K4] / (1.0 - p[6]);
            } else {
                const int t = (y - 7) / 2;
                o[(W_K1 + t) * NY] = ((y - 7) & 1 ? 0.5 : 1.0) * k[C_K1 + t];
                o[(W_K3 + t) * NY] = 2.0 * k[C_K3 + t];
            }
        }
        __syncthreads();
        for (int e = tid; e < nb * NW * NY; e += 256) {
            const int q = e / (NW * NY), a = (e - q * NW * NY) / NY, y = e % NY;
            double v = 0.0;
#pragma unroll
            for (int b = 0; b < NW; ++b) v = fma(Hw[q][a * NW + b], J[q][b * NY + y], v);
            M[q][a * NY + y] = v;
        }
        for (int e = tid; e < nb * NY; e += 256) {
            const int q = e / NY, y = e - q * NY;
            double v = 0.0;
#pragma unroll
            for (int a = 0; a < NW; ++a) v = fma(gx[q][a], J[q][a * NY + y], v);
            gy[q][y] = v;
        }
        __syncthreads();
        for (int e = tid; e < nb * NY * NY; e += 256) {
            const int q = e / (NY * NY), y = (e - q * NY * NY) / NY, x = e % NY;
            double v = 0.0;
#pragma unroll
            for (int a = 0; a < NW; ++a) v = fma(J[q][a * NY + y], M[q][a * NY + x], v);
            const int lo = min(y, x), hi = max(y, x);
            const double* G = gx[q];
            const double* k = coef + (size_t)(b0 + q) * NCOEF;
            if (lo >= 3 && hi < 6) {
                const celeste_image& im = g.images[g.pairs[b0 + q].img];
                const double a00 = im.wcs[0][0], a01 = im.wcs[0][1], a10 = im.wcs[1][0], a11 = im.wcs[1][1];
                const int r = lo - 3, c = hi - 3;
                const double* S = sdd[r == 0 ? c : r == 1 ? 2 + c : 5];
                v += G[W_SXX] * (a00 * a00 * S[0] + 2.0 * a00 * a01 * S[1] + a01 * a01 * S[2]) +
                     G[W_SXY] * (a00 * a10 * S[0] + (a00 * a11 + a01 * a10) * S[1] + a01 * a11 * S[2]) +
                     G[W_SYY] * (a10 * a10 * S[0] + 2.0 * a10 * a11 * S[1] + a11 * a11 * S[2]);
            } else if (hi >= 7) {
                const int t = (hi - 7) / 2;
                const double f1 = G[W_K1 + t] * k[C_K1 + t], f2 = G[W_K3 + t] * k[C_K3 + t];
                const bool hv = (hi - 7) & 1;   // variance coordinate
                if (lo == 6) {
                    v += ((hv ? 0.5 : 1.0) * f1 + 2.0 * f2) / (t == 0 ? p[6] : p[6] - 1.0);
                } else if (lo >= 7 && (lo - 7) / 2 == t) {
                    v += (hv ? 0.5 : 1.0) * ((lo - 7) & 1 ? 0.5 : 1.0) * f1 + 4.0 * f2;
                }
            }
            Hy[q][y * NY + x] = v;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int idx = tid + 256 * e, i = idx / NPAR, k = idx - i * NPAR;
            if (i >= NP || k >= NP) continue;
            const int at = y_of_param(i) * NY + y_of_param(k);
            for (int q = 0; q < nb; ++q) out[e] = fma(cf[q][i] * cf[q][k], Hy[q][at], out[e]);
        }
        if (tid < NP)
            for (int q = 0; q < nb; ++q) og = fma(cf[q][tid], gy[q][y_of_param(tid)], og);
    }
    __syncthreads();
    double* o = hess + (size_t)blockIdx.x * NPAR * NPAR;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int idx = tid + 256 * e, i = idx / NPAR, k = idx - i * NPAR;
        if (idx < NPAR * NPAR) o[idx] = out[e] + (kl ? kl_second(i, k, p, g.consts, gk, sc) : 0.0);
    }
    if (grad && tid < ROW)
        grad[(size_t)s * ROW + tid] = tid < NPAR ? og + (kl ? gk[tid] : 0.0) : 0.0;
}

// Total ELBO: a fixed-order two-level sum.  Block b of k_total_partial sums its contiguous
// slices of the per-tile pixel sums and of the sources' KL terms (a fixed tree per block) into
// part[b]; k_total_final sums the TT_BLOCKS partials in block order.  Deterministic, and
// spread over the chip instead of one work-group.
constexpr int TT_THREADS = 256;
constexpr int TT_BLOCKS = 1024;

__device__ inline double block_sum_256(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = TT_THREADS / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    return red[0];
}

__global__ void __launch_bounds__(TT_THREADS) k_total_partial(const double* __restrict__ tile_sums, int n_tiles,
                                                              const double* __restrict__ theta, Consts K, int S,
                                                              double* __restrict__ part, const int* status) {
    if (*status) return;
    __shared__ double red[TT_THREADS];
    const int b = blockIdx.x;
    const int t0 = (int)((int64_t)n_tiles * b / TT_BLOCKS), t1 = (int)((int64_t)n_tiles * (b + 1) / TT_BLOCKS);
    double acc = 0.0;
    for (int t = t0 + threadIdx.x; t < t1; t += TT_THREADS) acc += tile_sums[t];
    if (K.flags & CELESTE_INCLUDE_KL) {
        // the block's sources dealt to its waves (one after another they took 8 us more of a total
        // over 20000 sources than one a thread had, 38 more over 60000; dealt, 15 and 32 less)
        constexpr int NWV = TT_THREADS / 64;
        __shared__ double p[NWV][NPK];
        __shared__ KlScratch<double> sc[NWV];
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int s0 = (int)((int64_t)S * b / TT_BLOCKS), s1 = (int)((int64_t)S * (b + 1) / TT_BLOCKS);
        for (int sb = s0; sb < s1; sb += NWV) {   // every wave takes part in the barriers
            const int s = min(sb + wave, s1 - 1);
            if (lane < NPK) p[wave][lane] = theta[(size_t)s * ROW + lane];
            __syncthreads();
            const double kl = kl_wave<double>(p[wave], K, lane, false, nullptr, sc[wave]);
            if (lane == 0 && sb + wave < s1) acc -= kl;
            __syncthreads();
        }
    }
    const double v = block_sum_256(acc, red);
    if (threadIdx.x == 0) part[b] = v;
}

__global__ void __launch_bounds__(TT_THREADS) k_total_final(const double* __restrict__ part, double* out,
                                                            const int* status) {
    if (*status) return;
    __shared__ double red[TT_THREADS];
    double acc = 0.0;
    for (int b = threadIdx.x; b < TT_BLOCKS; b += TT_THREADS) acc += part[b];
    const double v = block_sum_256(acc, red);
    if (threadIdx.x == 0) out[0] = v;
}

__global__ void k_fill_int(int* p, int v, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_u8_sel(uint8_t* p, Sel s, uint8_t v) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < s.n) p[sel_at(s, j)] = v;
}

__global__ void k_fill_f64_sel(double* p, Sel s, double v) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < s.n) p[sel_at(s, j)] = v;
}

__global__ void k_copy_f64_sel(double* __restrict__ out, const double* __restrict__ in, Sel s, const int* status) {
    if (*status) return;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < s.n) out[sel_at(s, j)] = in[sel_at(s, j)];
}

// ----------------------------------------------------------------------- launchers
hipError_t launch_validate(const double* theta, const uint8_t* active, const int32_t* list, int n,
                           int S, int npar, int* status, hipStream_t st) {
    if (n > 0 && n <= VALIDATE_BLOCK) {
        hipLaunchKernelGGL(k_validate_block, dim3(1), dim3((n + 63) / 64 * 64), 0, st, theta, active, list, n, S, npar,
                           status);
        return hipGetLastError();
    }
    const hipError_t e = launch_fill_int(status, 0, 1, st);
    if (e != hipSuccess || n <= 0) return e;
    hipLaunchKernelGGL(k_validate, dim3((n + 255) / 256), dim3(256), 0, st, theta, active, list, n, S, npar,
                       status);
    return hipGetLastError();
}

hipError_t launch_prep(const PrepArgs& a, bool tangent, hipStream_t st) {
    if (a.pairs.n <= 0) return hipSuccess;
    const dim3 grid((a.pairs.n + 3) / 4);
    if (tangent) hipLaunchKernelGGL(k_prep<dual>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(k_prep<double>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_render(const RenderArgs& a, int wpb, hipStream_t st) {
    if (a.n_tiles <= 0) return hipSuccess;
    const dim3 grid((a.n_tiles + wpb - 1) / wpb);
    const int rp = a.tile_h * a.tile_w / 64;
    const Geometry& g = a.g;
#define RENDER_ARGS a, a.tiles, a.tile_list, g.pairs, g.images, a.tab, a.coef, g.x, a.E, a.V, a.tile_sums
    if (rp == 1) hipLaunchKernelGGL(k_render<1>, grid, dim3(64 * wpb), 0, st, RENDER_ARGS);
    else if (rp == 2) hipLaunchKernelGGL(k_render<2>, grid, dim3(64 * wpb), 0, st, RENDER_ARGS);
    else if (rp == 4) hipLaunchKernelGGL(k_render<4>, grid, dim3(64 * wpb), 0, st, RENDER_ARGS);
    else return hipErrorInvalidValue;
#undef RENDER_ARGS
    return hipGetLastError();
}

hipError_t launch_finalize(const FinArgs& a, bool tangent, hipStream_t st) {
    if (a.srcs.n <= 0) return hipSuccess;
    const dim3 grid(a.srcs.n);
    if (tangent) hipLaunchKernelGGL(k_finalize<dual>, grid, dim3(64), 0, st, a);
    else hipLaunchKernelGGL(k_finalize<double>, grid, dim3(64), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_tile_total(const double* tile_sums, int n_tiles, const double* theta, const Consts& c,
                             int S, double* part, double* out, const int* status, hipStream_t st) {
    hipLaunchKernelGGL(k_total_partial, dim3(TT_BLOCKS), dim3(TT_THREADS), 0, st, tile_sums, n_tiles, theta, c, S,
                       part, status);
    hipLaunchKernelGGL(k_total_final, dim3(1), dim3(TT_THREADS), 0, st, part, out, status);
    return hipGetLastError();
}

hipError_t launch_fill_u8_sel(uint8_t* p, const Sel& s, uint8_t v, hipStream_t st) {
    if (s.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u8_sel, dim3((s.n + 255) / 256), dim3(256), 0, st, p, s, v);
    return hipGetLastError();
}

hipError_t launch_fill_f64_sel(double* p, const Sel& s, double v, hipStream_t st) {
    if (s.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f64_sel, dim3((s.n + 255) / 256), dim3(256), 0, st, p, s, v);
    return hipGetLastError();
}

hipError_t launch_copy_f64_sel(double* out, const double* in, const Sel& s, const int* status, hipStream_t st) {
    if (s.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy_f64_sel, dim3((s.n + 255) / 256), dim3(256), 0, st, out, in, s, status);
    return hipGetLastError();
}

hipError_t launch_pair_block(const Sel& sel, const PairDev* dpairs, const double* partials, const double* kk,
                             const double* hg, bool tangent, int dir, double* gw, double* hw, const uint8_t* active,
                             const int* status, hipStream_t st) {
    if (sel.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pair_block, dim3((sel.n + 3) / 4), dim3(256), 0, st, sel, dpairs, partials, kk, hg,
                       tangent ? 1 : 0, dir, gw, hw, active, status);
    return hipGetLastError();
}

hipError_t launch_assemble_hessian(const Sel& srcs, const Geometry& g, const int32_t* patch_ptr, const double* theta,
                                   const double* coef, const double* gw, const double* hw, double* hess,
                                   double* grad, const uint8_t* active, const int* status, hipStream_t st) {
    if (srcs.n <= 0) return hipSuccess;
    if (g.consts.npar == NPK)
        hipLaunchKernelGGL(k_assemble_hessian<NPK>, dim3(srcs.n), dim3(256), 0, st, srcs, g, patch_ptr, theta, coef,
                           gw, hw, hess, grad, active, status);
    else
        hipLaunchKernelGGL(k_assemble_hessian<NP>, dim3(srcs.n), dim3(256), 0, st, srcs, g, patch_ptr, theta, coef,
                           gw, hw, hess, grad, active, status);
    return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int v, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_int, dim3((n + 255) / 256), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

}  // namespace cel
