// The VJP for split templates (see tfsc_vjp_common.hpp and split_shape).
//
// Which products the compiler fuses follows from small things (code beside the track tangents, a field in the argument
// block), and the FP32 results carry it: a change here is compared with the results before it.
#include "tfsc_vjp_common.hpp"

#include <type_traits>

namespace tfsc {

// ------------------------------------------------------------------ bin sums
// S1_c = sum conj(D_ck) H_k, U_c,p = sum conj(D_ck) dH_k/dp, S2 = sum |H_k|^2, V_p = sum conj(H_k) dH_k/dp (without w_m).
template <int C, class R>
struct VjpSums {
    R S1r[C], S1i[C], Ur[C][2], Ui[C][2], Vr[2], Vi[2], S2;
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int c = 0; c < C; ++c) S1r[c] = S1i[c] = Ur[c][0] = Ur[c][1] = Ui[c][0] = Ui[c][1] = (R)0;
        Vr[0] = Vr[1] = Vi[0] = Vi[1] = S2 = (R)0;
    }
    // a bin's weighted value with its tangents
    __device__ __forceinline__ void add(const CDn<2, R> &H, const cx<R> (&D)[C]) {
        const R hr = H.re.v, hi = H.im.v;
        S2 += hr * hr + hi * hi;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            Vr[p] += hr * H.re.d[p] + hi * H.im.d[p];
            Vi[p] += hr * H.im.d[p] - hi * H.re.d[p];
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const R dr = D[c].re, di = D[c].im;
            // conj(D) x
            S1r[c] += dr * hr + di * hi;
            S1i[c] += dr * hi - di * hr;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                Ur[c][p] += dr * H.re.d[p] + di * H.im.d[p];
                Ui[c][p] += dr * H.im.d[p] - di * H.re.d[p];
            }
        }
    }
};

template <class R>
__device__ __forceinline__ void cfma(cx<R> &acc, cx<R> a, cx<R> b) {  // acc += a b
    acc.re += a.re * b.re;
    acc.re -= a.im * b.im;
    acc.im += a.re * b.im;
    acc.im += a.im * b.re;
}
template <class R>
__device__ __forceinline__ void cfma(cx<R> &acc, cx<R> a, R b) {
    acc.re += a.re * b;
    acc.im += a.im * b;
}

// Asymptotic bins.  With a = 1/(x - j), b = 1/(x - j + beta) and the weight u, H = e0 u a b + dl u b (e0 = i Q beta E0,
// dl = i Q (E0 - E1), as in BinSums), and its tangents add u b^2, u a^2 b and u a b^2.  A bin therefore adds only real
// multiples f_q conj(D_c) of its pixels, f = (u a b, u b, u b^2, u a^2 b, u a b^2), and seven of the products f_q f_r (two
// more coincide with them); the tranche's constants and their tangents are applied once, in finish: 38 vector
// instructions a bin instead of about 85 with the tangents carried through every bin.  FP64 arithmetic only: it changes
// the rounding, by 3e-15 in FP64 but by 3e-7 in FP32, whose results are kept.
template <int C, class R>
struct VjpMoments {
    cx<R> M[C][5];
    R G00, G01, G11, G02, G12, G03, G04;

    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int q = 0; q < 5; ++q) M[c][q] = {(R)0, (R)0};
        G00 = G01 = G11 = G02 = G12 = G03 = G04 = (R)0;
    }

    __device__ __forceinline__ void add(R xj, R beta, R u, const cx<R> (&D)[C]) {
        const R xj1 = xj + beta;
        const R t = vrcp(xj * xj1), a = xj1 * t, b = xj * t;
        const R f1 = u * b, f0 = f1 * a, f2 = f1 * b, f3 = f0 * a, f4 = f0 * b;
        G00 += f0 * f0;
        G01 += f0 * f1;
        G11 += f1 * f1;
        G02 += f0 * f2;
        G12 += f1 * f2;
        G03 += f0 * f3;
        G04 += f0 * f4;
        const R f[5] = {f0, f1, f2, f3, f4};
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                M[c][q].re += f[q] * D[c].re;
                M[c][q].im -= f[q] * D[c].im;
            }
    }

    __device__ __forceinline__ void finish(const SpecD<R> &S, VjpSums<C, R> &s) const {
        // e0 = i Q beta E0, dl = i Q (E0 - E1) with their tangents
        const CDn<2, R> q0 = cdscale(S.E0, S.Q * S.beta), q1 = cdscale(cdsub(S.E0, S.E1), S.Q);
        const cx<R> e0 = {-q0.im.v, q0.re.v}, dl = {-q1.im.v, q1.re.v};
#pragma unroll
        for (int c = 0; c < C; ++c) {
            cx<R> v = cmul(e0, M[c][0]);
            cfma(v, dl, M[c][1]);
            s.S1r[c] = v.re;
            s.S1i[c] = v.im;
        }
        s.S2 = (e0.re * e0.re + e0.im * e0.im) * G00 + (dl.re * dl.re + dl.im * dl.im) * G11 +
               (R)2 * (e0.re * dl.re + e0.im * dl.im) * G01;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const R dx = S.x.d[p], dx1 = dx + S.beta.d[p];
            const cx<R> de = {-q0.im.d[p], q0.re.d[p]}, dd = {-q1.im.d[p], q1.re.d[p]};
            const cx<R> c2 = cscale(dl, -dx1), c3 = cscale(e0, -dx), c4 = cscale(e0, -dx1);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                cx<R> u = cmul(de, M[c][0]);
                cfma(u, dd, M[c][1]);
                cfma(u, c2, M[c][2]);
                cfma(u, c3, M[c][3]);
                cfma(u, c4, M[c][4]);
                s.Ur[c][p] = u.re;
                s.Ui[c][p] = u.im;
            }
            // sum f_0 dH and sum f_1 dH (f_1 f_3 = f_0 f_0, f_1 f_4 = f_0 f_2)
            cx<R> h0 = cscale(de, G00), h1 = cscale(de, G01);
            cfma(h0, dd, G01);
            cfma(h0, c2, G02);
            cfma(h0, c3, G03);
            cfma(h0, c4, G04);
            cfma(h1, dd, G11);
            cfma(h1, c2, G12);
            cfma(h1, c3, G00);
            cfma(h1, c4, G02);
            cx<R> v = cmul(cx<R>{e0.re, -e0.im}, h0);
            cfma(v, cx<R>{dl.re, -dl.im}, h1);
            s.Vr[p] = v.re;
            s.Vi[p] = v.im;
        }
    }
};

// A pixel between its load and its use, a bin later: the word of a 16-bit store, converted where it is used (held as two
// floats, the conversion waits for the load at once: 20,000 templates of the two-year grid, I16 19.6 ms, so 17.3).
template <class PixT, bool W = PixTraits<PixT>::scaled>
struct PixHeld {
    using type = cx<typename PixTraits<PixT>::R>;
    __device__ static __forceinline__ type load(const void *p, size_t idx) { return PixTraits<PixT>::load(p, idx); }
    __device__ static __forceinline__ type value(type v) { return v; }
};
template <class PixT>
struct PixHeld<PixT, true> {
    using type = uint32_t;
    __device__ static __forceinline__ type load(const void *p, size_t idx) {
        return reinterpret_cast<const uint32_t *>(p)[idx];
    }
    __device__ static __forceinline__ cx<float> value(type v) { return PixTraits<PixT>::load(&v, 0); }
};

// R = double: the FP64 form; R = float: FP32 spectra, response, pixel sums and tangents (the
// track, its tangents, the phases and every integer decision stay FP64, as in the FP32 forward).
// The FP32 form holds half the registers and runs two waves per SIMD.
//
// k_vjp_units: split templates, one unit per wave, in runs per XCD (run_item, in the bank's own order); k_vjp_finish adds
// the units.
//
// Bound: FP64, latency of dependent FP64 chains at one wave per SIMD; FP32, vector-ALU issue at two.  Two-year grid, A+E:
// 320 templates FP64 2282 us with a wave per template and the tangents carried through every bin, 1058 in units with the
// moments, 913 with each lane's own band instead of the wave's, 590 with the units dealt out to all XCDs, 527 with sincospi
// and reciprocals for sincos, pow and divisions; 65,536 templates FP32 40 -> 33.7 ms from units in runs
// per XCD, a pixel's address in one multiply-add for every layout, and the next bin's loads ahead.
template <int C, class PixT, class R>
__global__ __launch_bounds__(256, sizeof(R) == 4 ? 2 : 1) void k_vjp_units(VjpArgs a) {
    using Held = PixHeld<PixT>;
    using HT = typename Held::type;
    extern __shared__ unsigned char smem_raw[];
    const int KP = a.K + 2 * kHalfBins;
    R *u_pad = reinterpret_cast<R *>(smem_raw);
    const double u_mul = a.u_scale[0];
    const int kmax = a.M / 2 - 1;
    for (int q = threadIdx.x; q < KP; q += blockDim.x) {
        const int k = q - kHalfBins;
        u_pad[q] = (R)((k >= 1 && k <= kmax) ? a.inv_asd[k] * u_mul : 0.0);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    int unit;
    const int64_t i = run_item(a.n, unit);
    if (i >= a.n || unit >= a.units) return;
    {
        double gr[5] = {0, 0, 0, 0, 0};
        const double mci = a.mc[i];
        const bool ok = params_valid(mci, a.eta[i], a.f0[i], a.ct[i], a.ci[i]);
        if (ok) {
            const int ns = a.nseg[i];
            const int64_t off = a.seg_offset[i];
            const double gs = a.g_stat ? a.g_stat[i] : 0.0;
            Track T;
            load_track(a.rec + i * kRecDoubles, lane, T);
            TrackTan TT = track_tangents(T, a.f0[i]);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                TT.mu[p] = wave_uniform(TT.mu[p]);
                TT.dtc[p] = wave_uniform(TT.dtc[p]);
            }
            SkyD<R> S;
            sky_dual(S, a.ct[i], a.phi[i], a.psi[i], a.ci[i]);
            const int m_beg = unit * a.chunks * 64;
            int m_end = min(a.Nt, m_beg + a.chunks * 64);
            // FP32 form (two waves per SIMD): each chunk's track is evaluated during the previous chunk, beside
            // that chunk's response tangents, so the dependent FP64 chain overlaps the FP32 work.  The FP64 form
            // (one wave per SIMD, at its register limit) evaluates it at the top of its chunk, which measured faster.
            constexpr bool kAhead = sizeof(R) == 4;
            double Phi = 0.0, f = 0.0, fdot = 0.0, s_th = 1.0;
            int code = 0;
            if constexpr (kAhead) {
                const int mf = m_beg + lane;
                code = track_step_lanes(T, (double)(mf < a.Nt ? mf : a.Nt - 1) * a.dT, a.dT, a.df, a.fnyq, Phi, f, fdot,
                                        &s_th);
                code = mf < a.Nt ? code : 0;
            }
            for (int m0 = m_beg; m0 < m_end; m0 += 64) {
                const int m = m0 + lane;
                const bool inr = m < a.Nt;
                if constexpr (!kAhead) {
                    code = track_step_lanes(T, (double)(inr ? m : a.Nt - 1) * a.dT, a.dT, a.df, a.fnyq, Phi, f, fdot,
                                            &s_th);
                    code = inr ? code : 0;
                }
                const uint64_t viol = __ballot(code != 0);
                int lim = a.Nt;
                if (viol) {
                    lim = m0 + __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)viol) - 1);
                    m_end = lim;
                }
                const bool active = inr && m < lim;
                const double wm = active ? a.tranche_w[m] : 0.0;
                // adjoint coefficients of this tranche's segment
                double ar = 0.0, ai = 0.0, b = 0.0;
                int sn = 0;
                if (active && wm != 0.0) {
                    sn = (int)(((int64_t)m * ns) / a.Nt);
                    const int64_t o = off + sn;
                    const double zr = a.seg_zn[3 * o], zi = a.seg_zn[3 * o + 1], Nn = a.seg_zn[3 * o + 2];
                    const double g = gs + (a.g_seg ? a.g_seg[o] : 0.0);
                    if (Nn > 0.0 && g != 0.0) {
                        const double iN = 1.0 / Nn;
                        ar = 4.0 * g * zr * iN;
                        ai = -4.0 * g * zi * iN;
                        b = 4.0 * g * (zr * zr + zi * zi) * iN * iN;
                    }
                }
                const bool work = ar != 0.0 || ai != 0.0 || b != 0.0;
                // pixel and spectrum sums of the working lanes.  FP64: each lane's asymptotic bins through their moments,
                // then its other bins one by one.  FP32: every bin by itself.
                R S1r[C], S1i[C], Ur[C][2], Ui[C][2];
                R S2 = (R)0, Vr[2] = {(R)0, (R)0}, Vi[2] = {(R)0, (R)0};
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    S1r[c] = S1i[c] = (R)0;
                    Ur[c][0] = Ur[c][1] = Ui[c][0] = Ui[c][1] = (R)0;
                }
                R dfr[2] = {(R)0, (R)0};
                {
                    if (work) {
                        const int m_ref = (int)(((int64_t)sn * a.Nt + ns - 1) / ns);
                        double dref[2];
                        dphi_at(T, TT, (double)m_ref * a.dT, dref);
                        const TrackDual TD = track_dual<R>(T, TT, (double)m * a.dT, f, s_th);
                        dfr[0] = (R)TD.df[0];
                        dfr[1] = (R)TD.df[1];
                        SpecD<R> sp;
                        const int kc = spec_dual(sp, Phi, f, fdot, TD, dref, a.dT);
                        const char *pix = reinterpret_cast<const char *>(a.pix) + (size_t)m * a.col * (2 * sizeof(PixT));
                        const uint32_t row = a.row * (uint32_t)(2 * sizeof(PixT));
                        // weight and pixels of bin kc + j; outside 1 .. M/2 - 1 the weight is 0 and a row inside is read
                        auto bin = [&](int j, R &u, HT (&Dl)[C]) {
                            const int k = min(max(kc + j, 1), kmax);
                            const char *p = pix + (uint64_t)(uint32_t)k * row;
#pragma unroll
                            for (int c = 0; c < C; ++c) Dl[c] = Held::load(p, (size_t)c * a.chan);
                            u = u_pad[kc + j + kHalfBins];
                            if (a.rho) u *= (R)a.rho[(size_t)k * a.Nt + m];
                        };
                        auto to_arith = [&](int j, const HT (&Dl)[C], cx<R> (&D)[C]) {
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                const auto v = Held::value(Dl[c]);
                                D[c] = {(R)v.re, (R)v.im};
                                if constexpr (PixTraits<PixT>::scaled) {
                                    const R sc = (R)a.layer_scale[c * a.K + min(max(kc + j, 1), kmax)];
                                    D[c].re *= sc;
                                    D[c].im *= sc;
                                }
                            }
                        };
                        if constexpr (sizeof(R) == 8) {
                            VjpMoments<C, R> mom;
                            mom.zero();
                            // three bins' loads are issued before the first is used
#pragma unroll 1
                            for (int j0 = -kHalfBins; j0 <= kHalfBins; j0 += 3) {
                                R u[3];
                                HT Dl[3][C];
#pragma unroll
                                for (int q = 0; q < 3; ++q) bin(j0 + q, u[q], Dl[q]);
#pragma unroll
                                for (int q = 0; q < 3; ++q) {
                                    const int j = j0 + q;
                                    cx<R> D[C];
                                    to_arith(j, Dl[q], D);
                                    if (j < sp.j0lo || j > sp.j1hi) mom.add(sp.x.v - (R)j, sp.beta.v, u[q], D);
                                }
                            }
                            VjpSums<C, R> sum;
                            mom.finish(sp, sum);
                            for (int j = max(sp.j0lo, -kHalfBins); j <= min(sp.j1hi, kHalfBins); ++j) {
                                R u;
                                HT Dl[C];
                                bin(j, u, Dl);
                                cx<R> D[C];
                                to_arith(j, Dl, D);
                                sum.add(cdscale(bin_dual(sp, j), u), D);
                            }
                            S2 = sum.S2;
#pragma unroll
                            for (int p = 0; p < 2; ++p) {
                                Vr[p] = sum.Vr[p];
                                Vi[p] = sum.Vi[p];
                            }
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                S1r[c] = sum.S1r[c];
                                S1i[c] = sum.S1i[c];
#pragma unroll
                                for (int p = 0; p < 2; ++p) {
                                    Ur[c][p] = sum.Ur[c][p];
                                    Ui[c][p] = sum.Ui[c][p];
                                }
                            }
                        } else {
                            // Each bin's loads are issued before the bin ahead of it is evaluated, the first bin's in a
                            // turn of their own: beside the FP64 track tangents above they would change which of those
                            // products are fused.
                            R un = (R)0;
                            HT Dn[C] = {};
#pragma unroll 1
                            for (int j = -kHalfBins - 1; j <= kHalfBins; ++j) {
                                const R u = un;
                                HT Dl[C];
#pragma unroll
                                for (int c = 0; c < C; ++c) Dl[c] = Dn[c];
                                if (j < kHalfBins) bin(j + 1, un, Dn);
                                if (j < -kHalfBins) continue;
                                CDn<2, R> H = bin_dual(sp, j);
                                H = cdscale(H, u);
                                const R hr = H.re.v, hi = H.im.v;
                                S2 += hr * hr + hi * hi;
#pragma unroll
                                for (int p = 0; p < 2; ++p) {
                                    Vr[p] += hr * H.re.d[p] + hi * H.im.d[p];
                                    Vi[p] += hr * H.im.d[p] - hi * H.re.d[p];
                                }
#pragma unroll
                                for (int c = 0; c < C; ++c) {
                                    const auto dv = Held::value(Dl[c]);
                                    R dr = (R)dv.re, di = (R)dv.im;
                                    if constexpr (PixTraits<PixT>::scaled) {
                                        const R sc = (R)a.layer_scale[c * a.K + min(max(kc + j, 1), kmax)];
                                        dr *= sc;
                                        di *= sc;
                                    }
                                    // conj(D) x.  Of an I16 store k_vjp_wave's text rounds the first product and fuses the
                                    // second, here it would be the other way round: written out, for the same results.
                                    if constexpr (std::is_same<PixT, int16_t>::value)
                                        S1r[c] += fma(di, hi, dr * hr);
                                    else
                                        S1r[c] += dr * hr + di * hi;
                                    S1i[c] += dr * hi - di * hr;
#pragma unroll
                                    for (int p = 0; p < 2; ++p) {
                                        Ur[c][p] += dr * H.re.d[p] + di * H.im.d[p];
                                        Ui[c][p] += dr * H.im.d[p] - di * H.re.d[p];
                                    }
                                }
                            }
                        }
                    }
                }
                // this chunk's response tangents and the next chunk's track, for every lane (values of lanes
                // without work are not used; the geometry row is clamped into the table)
                CDn<4, R> Tc[3];
                {
                    double gm[kGeoRows];
                    load_geo(a.geo, inr ? m : a.Nt - 1, a.Nt, gm);
                    transfer_ae_dual<(C == 3)>(S, gm, f, Tc[0], Tc[1], Tc[2]);
                    if constexpr (kAhead) {
                        const int mn = m + 64;
                        int cn = track_step_lanes(T, (double)(mn < a.Nt ? mn : a.Nt - 1) * a.dT, a.dT, a.df, a.fnyq, Phi,
                                                  f, fdot, &s_th);
                        code = mn < a.Nt ? cn : 0;
                    }
                }
                if (work) {
                    {
                        // tranche weight: H carries w_m
                        const R wr = (R)wm, w2 = wr * wr;
                        S2 *= w2;
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            Vr[p] *= w2;
                            Vi[p] *= w2;
                        }
                        const R arr = (R)ar, air = (R)ai, br = (R)b;
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const R tr = Tc[c].re.v, ti = Tc[c].im.v;
                            // G_c = a S1_c - b conj(T_c) S2
                            const R s1r = S1r[c] * wr, s1i = S1i[c] * wr;
                            const R Gr = (arr * s1r - air * s1i) - br * tr * S2;
                            const R Gi = (arr * s1i + air * s1r) + br * ti * S2;
                            // Re(dT/dq G) for the response slots
                            R rg[4];
#pragma unroll
                            for (int q = 0; q < 4; ++q) rg[q] = Tc[c].re.d[q] * Gr - Tc[c].im.d[q] * Gi;
#pragma unroll
                            for (int p = 0; p < 2; ++p) {
                                const R ur = Ur[c][p] * wr, ui = Ui[c][p] * wr;
                                // J = a U - b conj(T) V
                                const R Jr = (arr * ur - air * ui) - br * (tr * Vr[p] + ti * Vi[p]);
                                const R Ji = (arr * ui + air * ur) - br * (tr * Vi[p] - ti * Vr[p]);
                                gr[p] += (double)(rg[0] * dfr[p] + (tr * Jr - ti * Ji));
                            }
                            gr[2] += (double)rg[1];
                            gr[3] += (double)rg[2];
                            gr[4] += (double)rg[3];
                        }
                    }
                }
                if (viol) break;
            }
        }
#pragma unroll
        for (int p = 0; p < 5; ++p) gr[p] = dpp_sum_f64(gr[p]);
        if (lane == 0) {
            // ln Mc, f0, cos theta, phi, psi
            double *o = a.part + 5 * (i * a.units + unit);
#pragma unroll
            for (int p = 0; p < 5; ++p) o[p] = gr[p];
        }
    }
}

// Sum of a template's units, in order; one thread per component.
__global__ __launch_bounds__(256) void k_vjp_finish(int64_t n, int units, const double *__restrict__ part,
                                                    double *__restrict__ g_params) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= 5 * n) return;
    const double *p = part + (e / 5) * 5 * units + e % 5;
    double s = 0.0;
    for (int u = 0; u < units; ++u) s += p[5 * u];
    g_params[e] = s;
}

template <int C, class PixT, class R>
static hipError_t launch_vjp_t(const VjpArgs &a, int block_waves, hipStream_t st) {
    const size_t shmem = sizeof(R) * ((size_t)a.K + 2 * kHalfBins);
    hipLaunchKernelGGL((k_vjp_units<C, PixT, R>), dim3(run_groups(a.n, block_waves, a.units)), dim3(64 * block_waves),
                       shmem, st, a);
    hipLaunchKernelGGL(k_vjp_finish, dim3((unsigned)((5 * a.n + 255) / 256)), dim3(256), 0, st, a.n, a.units, a.part,
                       a.g_params);
    return hipGetLastError();
}

template <int C, class R>
static hipError_t dispatch_vjp(const VjpArgs &a, int dtype, int block_waves, hipStream_t st) {
    switch (dtype) {
        case 0: return launch_vjp_t<C, double, R>(a, block_waves, st);
        case 1: return launch_vjp_t<C, float, R>(a, block_waves, st);
        case 2: return launch_vjp_t<C, __hip_bfloat16, R>(a, block_waves, st);
        case 3: return launch_vjp_t<C, __half, R>(a, block_waves, st);
        case 4: return launch_vjp_t<C, int16_t, R>(a, block_waves, st);
    }
    return hipErrorInvalidValue;
}

template <class R>
static hipError_t dispatch_vjp_c(const VjpArgs &a, int C, int dtype, int block_waves, hipStream_t st) {
    if (C == 3) return dispatch_vjp<3, R>(a, dtype, block_waves, st);
    return C == 1 ? dispatch_vjp<1, R>(a, dtype, block_waves, st) : dispatch_vjp<2, R>(a, dtype, block_waves, st);
}

hipError_t launch_vjp_units(const VjpArgs &a, int precision, int C, int dtype, int block_waves, hipStream_t st) {
    return precision == 1 ? dispatch_vjp_c<float>(a, C, dtype, block_waves, st)
                          : dispatch_vjp_c<double>(a, C, dtype, block_waves, st);
}

}  // namespace tfsc
