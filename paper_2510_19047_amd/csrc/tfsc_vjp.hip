// The VJP for whole templates, and its entry point; the kernel for split templates is in tfsc_vjp_units.hip.
#include "tfsc_vjp_common.hpp"

namespace tfsc {

// Whole templates, for banks too large to split (over forty a wave) and workspaces without room for it: each wave takes its
// next template from the work counter, which evens out banks in any order.  The bins one by one in both arithmetics.
// A text of its own beside the units' kernel: with the units' fetch inside this loop the compiler hoists other products out
// of the bin loop, which changes the FP32 results (by 1e-7 of the largest).
template <int C, class PixT, class R>
__global__ __launch_bounds__(256, sizeof(R) == 4 ? 2 : 1) void k_vjp_wave(VjpArgs a, int layout, uint32_t *counter) {
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
    for (;;) {
        // dynamic work fetch, as in the statistic kernel: one atomic per wave on a uniform address
        const uint32_t mine = atomicAdd(counter, lane == 0 ? 1u : 0u);
        const int64_t i = (int64_t)__builtin_amdgcn_readfirstlane(mine);
        if (i >= a.n) break;
        double gr[5] = {0, 0, 0, 0, 0};
        const double mci = a.mc[i];
        const bool ok = params_valid(mci, a.eta[i], a.f0[i], a.ct[i], a.ci[i]);
        if (ok) {
            const int ns = a.nseg[i];
            const int64_t off = a.seg_offset[i];
            const double gs = a.g_stat ? a.g_stat[i] : 0.0;
            Track T;
            track_init(T, mci, a.eta[i], a.f0[i]);
            wave_uniform(T);
            TrackTan TT = track_tangents(T, a.f0[i]);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                TT.mu[p] = wave_uniform(TT.mu[p]);
                TT.dtc[p] = wave_uniform(TT.dtc[p]);
            }
            SkyD<R> S;
            sky_dual(S, a.ct[i], a.phi[i], a.psi[i], a.ci[i]);
            int m_end = a.Nt;
            // FP32 form (two waves per SIMD): each chunk's track is evaluated during the previous chunk, beside
            // that chunk's response tangents, so the dependent FP64 chain overlaps the FP32 work.  The FP64 form
            // (one wave per SIMD, at its register limit) evaluates it at the top of its chunk, which measured faster.
            constexpr bool kAhead = sizeof(R) == 4;
            double Phi = 0.0, f = 0.0, fdot = 0.0, s_th = 1.0;
            int code = 0;
            if constexpr (kAhead) {
                code = track_step_lanes(T, (double)(lane < a.Nt ? lane : a.Nt - 1) * a.dT, a.dT, a.df, a.fnyq, Phi, f,
                                        fdot, &s_th);
                code = lane < a.Nt ? code : 0;
            }
            for (int m0 = 0; m0 < m_end; m0 += 64) {
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
                // pixel and spectrum sums of the working lanes
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
                        for (int j = -kHalfBins; j <= kHalfBins; ++j) {
                            const int k = kc + j;
                            if (k < 1 || k > kmax) continue;
                            R u = u_pad[k + kHalfBins];
                            if (a.rho) u *= (R)a.rho[(size_t)k * a.Nt + m];
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
                                // one expression for every layout, or of a 16-bit store one per layout (two-year grid, A+E,
                                // one against the other, ms: 90,000 templates FP32 57.7 / 62.5; 40,000 I16 33.4 / 32.6)
                                size_t idx = (size_t)c * a.chan + (size_t)k * a.row + m * a.col;
                                if constexpr (PixTraits<PixT>::scaled)
                                    idx = layout == 0 ? ((size_t)c * a.K + k) * a.Nt + m
                                          : (layout == 1 ? ((size_t)c * a.Nt + m) * a.K + k
                                                         : ((size_t)k * a.Nt + m) * C + c);
                                cx<typename PixTraits<PixT>::R> dv = PixTraits<PixT>::load(a.pix, idx);
                                R dr = (R)dv.re, di = (R)dv.im;
                                if constexpr (PixTraits<PixT>::scaled) {
                                    const R sc = (R)a.layer_scale[c * a.K + k];
                                    dr *= sc;
                                    di *= sc;
                                }
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
#pragma unroll
            for (int p = 0; p < 5; ++p) a.g_params[5 * i + p] = gr[p];
        }
    }
}

template <int C, class PixT, class R>
static hipError_t launch_vjp_t(const VjpArgs &a, int layout, uint32_t *counter, int n_groups, int block_waves, hipStream_t st) {
    const size_t shmem = sizeof(R) * ((size_t)a.K + 2 * kHalfBins);
    const int64_t groups = (a.n + block_waves - 1) / block_waves;
    hipLaunchKernelGGL((k_vjp_wave<C, PixT, R>), dim3((unsigned)(groups < n_groups ? groups : n_groups)),
                       dim3(64 * block_waves), shmem, st, a, layout, counter);
    return hipGetLastError();
}

template <int C, class R>
static hipError_t dispatch_vjp(const VjpArgs &a, int layout, uint32_t *counter, int dtype, int n_groups, int block_waves, hipStream_t st) {
    switch (dtype) {
        case 0: return launch_vjp_t<C, double, R>(a, layout, counter, n_groups, block_waves, st);
        case 1: return launch_vjp_t<C, float, R>(a, layout, counter, n_groups, block_waves, st);
        case 2: return launch_vjp_t<C, __hip_bfloat16, R>(a, layout, counter, n_groups, block_waves, st);
        case 3: return launch_vjp_t<C, __half, R>(a, layout, counter, n_groups, block_waves, st);
        case 4: return launch_vjp_t<C, int16_t, R>(a, layout, counter, n_groups, block_waves, st);
    }
    return hipErrorInvalidValue;
}

template <class R>
static hipError_t dispatch_vjp_c(const VjpArgs &a, int layout, uint32_t *counter, int C, int dtype, int n_groups, int block_waves, hipStream_t st) {
    if (C == 3) return dispatch_vjp<3, R>(a, layout, counter, dtype, n_groups, block_waves, st);
    return C == 1 ? dispatch_vjp<1, R>(a, layout, counter, dtype, n_groups, block_waves, st)
                  : dispatch_vjp<2, R>(a, layout, counter, dtype, n_groups, block_waves, st);
}

hipError_t launch_vjp(const VjpLaunch &V, hipStream_t st) {
    const StatLaunch &L = V.s;
    if (L.n == 0) return hipSuccess;
    VjpArgs a;
    a.M = L.M;
    a.K = L.M / 2 + 1;
    a.Nt = L.Nt;
    a.C = L.C;
    a.dT = (double)L.M * L.dt;
    a.df = 1.0 / a.dT;
    a.fnyq = 0.5 / L.dt;
    a.pix = L.pix;
    // [C][K][Nt], [C][Nt][K] or [K][Nt][C]
    a.chan = L.layout == 2 ? 1 : (size_t)a.K * a.Nt;
    a.col = L.layout == 0 ? 1 : (L.layout == 1 ? (size_t)a.K : (size_t)a.C);
    a.row = L.layout == 0 ? (uint32_t)a.Nt : (L.layout == 1 ? 1u : (uint32_t)a.Nt * (uint32_t)a.C);
    a.layer_scale = L.layer_scale;
    a.inv_asd = L.inv_asd;
    a.tranche_w = L.tranche_w;
    a.geo = L.geo;
    a.u_scale = L.u_scale;
    a.rho = L.rho;
    a.n = L.n;
    a.mc = L.mc;
    a.eta = L.eta;
    a.f0 = L.f0;
    a.ct = L.ct;
    a.phi = L.phi;
    a.psi = L.psi;
    a.ci = L.ci;
    a.nseg = L.nseg;
    a.seg_offset = L.seg_offset;
    a.seg_zn = V.seg_zn;
    a.g_stat = V.g_stat;
    a.g_seg = V.g_seg;
    a.g_params = V.g_params;
    a.units = L.split.units;
    a.chunks = L.split.chunks;
    a.rec = L.split.rec;
    a.part = reinterpret_cast<double *>(L.split.head);
    if (a.units) return launch_vjp_units(a, L.precision, L.C, L.pix_dtype, kRunWaves, st);
    return L.precision == 1 ? dispatch_vjp_c<float>(a, L.layout, L.counter, L.C, L.pix_dtype, L.n_groups, L.block_waves, st)
                            : dispatch_vjp_c<double>(a, L.layout, L.counter, L.C, L.pix_dtype, L.n_groups, L.block_waves, st);
}

}  // namespace tfsc
