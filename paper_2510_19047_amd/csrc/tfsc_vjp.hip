// Vector-Jacobian product of the statistic with respect to (ln Mc, f0, cos theta, phi, psi).
//
// For L = sum_n g_n Upsilon_n with Upsilon_n = 2 |z_n|^2 / N_n (Eq. (Upsilon-seg)),
//   dL = sum_n sum_{pixels of n} Re[(a_n conj(D) - b_n conj(Y)) dY],
//   a_n = 4 g_n conj(z_n) / N_n,  b_n = 4 g_n |z_n|^2 / N_n^2,
// with (z_n, N_n) taken from the forward pass.  Nothing per pixel is stored: each
// wave recomputes its template's track, tranche spectra and response with
// forward-mode tangents (FP64 dual numbers) and contracts them with the adjoint
// on the fly, one lane per tranche as in the forward WAVE schedule.
//
// Per tranche, with H_k = h_k u_k w_m (channel independent) and Y_ck = T_c H_k:
//   G_c    = sum_k adj_ck H_k        = a S1_c - b conj(T_c) S2
//   J_c,p  = sum_k adj_ck dH_k/dp    = a U_c,p - b conj(T_c) V_p
//   dL/dp += Re(dT_c/dp G_c) + Re(T_c J_c,p),
// S1_c = sum conj(D_ck) H_k, S2 = sum |H_k|^2, U_c,p = sum conj(D_ck) dH_k/dp,
// V_p = sum conj(H_k) dH_k/dp.
//
// A phase shift common to all pixels of a segment leaves Upsilon_n unchanged, so
// the phase tangent of tranche m is taken relative to the segment's first tranche
// (dPhi_m - dPhi_ref).  This is exact in real arithmetic and removes the large
// common part of dPhi/d ln Mc (phase counted from coalescence) before it meets
// rounding in the adjoint.
#include "tfsc_device.hpp"
#include "tfsc_kernels.hpp"
#include "tfsc_stat_common.hpp"  // wave_uniform, dpp_sum_f64

// The tangent arithmetic below contracts multiply-adds into FMAs.  The FP64 track that fixes
// the integer structure (track_step, from tfsc_device.hpp, included above) is not affected.
#pragma clang fp contract(fast)

namespace tfsc {

// ------------------------------------------------------------------ dual numbers
// Dn<N, R>: a value and N tangents in arithmetic R (double, or float for the FP32 form).  Scalars
// mixed with a dual number take its type (nd_t keeps them out of template deduction).
template <class T>
struct nodeduce {
    using type = T;
};
template <class T>
using nd_t = typename nodeduce<T>::type;

template <int N, class R = double>
struct Dn {
    R v;
    R d[N];
};

template <int N, class R>
__device__ __forceinline__ Dn<N, R> dconst(nd_t<R> v) {
    Dn<N, R> r;
    r.v = v;
#pragma unroll
    for (int i = 0; i < N; ++i) r.d[i] = (R)0;
    return r;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator+(Dn<N, R> a, Dn<N, R> b) {
    Dn<N, R> r;
    r.v = a.v + b.v;
#pragma unroll
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] + b.d[i];
    return r;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator-(Dn<N, R> a, Dn<N, R> b) {
    Dn<N, R> r;
    r.v = a.v - b.v;
#pragma unroll
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] - b.d[i];
    return r;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator-(Dn<N, R> a) {
    Dn<N, R> r;
    r.v = -a.v;
#pragma unroll
    for (int i = 0; i < N; ++i) r.d[i] = -a.d[i];
    return r;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator*(Dn<N, R> a, Dn<N, R> b) {
    Dn<N, R> r;
    r.v = a.v * b.v;
#pragma unroll
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] * b.v + a.v * b.d[i];
    return r;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator*(Dn<N, R> a, nd_t<R> s) {
    Dn<N, R> r;
    r.v = a.v * s;
#pragma unroll
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] * s;
    return r;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator*(nd_t<R> s, Dn<N, R> a) {
    return a * s;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator+(Dn<N, R> a, nd_t<R> s) {
    a.v += s;
    return a;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator+(nd_t<R> s, Dn<N, R> a) {
    a.v += s;
    return a;
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> operator-(nd_t<R> s, Dn<N, R> a) {
    return (-a) + s;
}
// 1/x.  The FP64 operands here are normal and far from the range limits (see rcp_rn: the division's bits for 7 of its 11
// instructions).
__device__ __forceinline__ double vrcp(double x) { return rcp_rn(x); }
__device__ __forceinline__ float vrcp(float x) { return rcp(x); }
template <int N, class R>
__device__ __forceinline__ Dn<N, R> drcp(Dn<N, R> a) {
    const R r = vrcp(a.v), r2 = -r * r;
    Dn<N, R> o;
    o.v = r;
#pragma unroll
    for (int i = 0; i < N; ++i) o.d[i] = a.d[i] * r2;
    return o;
}
__device__ __forceinline__ double vsqrt(double x) { return sqrt(x); }
__device__ __forceinline__ float vsqrt(float x) { return sqrtf(x); }
__device__ __forceinline__ double half_rcp(double s) { return 0.5 * rcp_rn(s); }
__device__ __forceinline__ float half_rcp(float s) { return 0.5f * rcp(s); }
template <int N, class R>
__device__ __forceinline__ Dn<N, R> dsqrt(Dn<N, R> a) {
    const R s = vsqrt(a.v), h = half_rcp(s);
    Dn<N, R> o;
    o.v = s;
#pragma unroll
    for (int i = 0; i < N; ++i) o.d[i] = a.d[i] * h;
    return o;
}
// sine and cosine of 2 pi r for r in revolutions (|r| <= 1/2)
__device__ __forceinline__ void sincos_rev(double r, double &s, double &c) { sincospi(2.0 * r, &s, &c); }
__device__ __forceinline__ void sincos_rev(float r, float &s, float &c) {
    s = __builtin_amdgcn_sinf(r);
    c = __builtin_amdgcn_cosf(r);
}
// sin(2 pi r) with its tangent; in FP32 the value is taken of the argument folded into
// [-1/4, 1/4] (exact in FP32) so that it keeps its relative precision near the zeros r = +-1/2
template <int N, class R>
__device__ __forceinline__ Dn<N, R> dsin_rev(Dn<N, R> r) {
    R s, c;
    sincos_rev(r.v, s, c);
    if constexpr (sizeof(R) == 4) {
        const float rf = r.v > 0.25f ? 0.5f - r.v : (r.v < -0.25f ? -0.5f - r.v : r.v);
        s = sin_rev_accurate(rf);
    }
    Dn<N, R> o;
    o.v = s;
#pragma unroll
    for (int i = 0; i < N; ++i) o.d[i] = (R)kTwoPi * c * r.d[i];
    return o;
}
// sin(x)/x and its derivative (cos x - sin x / x) / x, for x >= 0
__device__ __forceinline__ void sinc_d(double x, double &v, double &dv) {
    if (fabs(x) < 1e-4) {
        v = 1.0 - x * x * (1.0 / 6.0);
        dv = -x * (1.0 / 3.0);
    } else {
        // in half turns: no reduction of large arguments (pi f L (1 -+ k.n) is below a few turns)
        double s, c;
        sincospi(x * (1.0 / kPi), &s, &c);
        const double ir = rcp_rn(x);
        v = s * ir;
        dv = (c - v) * ir;
    }
}
__device__ __forceinline__ void sinc_d(float x, float &v, float &dv) {
    if (x < 0.5f) {
        // Taylor series of sin x / x through x^8 and of its derivative through x^7 (first omitted
        // terms below 6e-10 and 1.3e-10 at x = 1/2), free of the cancellation in (cos x - v) / x
        const float x2 = x * x;
        v = 1.0f - x2 * (1.0f / 6.0f - x2 * (1.0f / 120.0f - x2 * (1.0f / 5040.0f - x2 * (1.0f / 362880.0f))));
        dv = -x * (1.0f / 3.0f - x2 * (1.0f / 30.0f - x2 * (1.0f / 840.0f - x2 * (1.0f / 45360.0f))));
    } else {
        const float r = x * (float)(1.0 / kTwoPi), ir = rcp(x);
        v = __builtin_amdgcn_sinf(r) * ir;
        dv = (__builtin_amdgcn_cosf(r) - v) * ir;
    }
}
template <int N, class R>
__device__ __forceinline__ Dn<N, R> dsinc(Dn<N, R> x) {
    R v, dv;
    sinc_d(x.v, v, dv);
    Dn<N, R> o;
    o.v = v;
#pragma unroll
    for (int i = 0; i < N; ++i) o.d[i] = dv * x.d[i];
    return o;
}

template <int N, class R = double>
struct CDn {
    Dn<N, R> re, im;
};
template <int N, class R>
__device__ __forceinline__ CDn<N, R> cdmul(CDn<N, R> a, CDn<N, R> b) {
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <int N, class R>
__device__ __forceinline__ CDn<N, R> cdadd(CDn<N, R> a, CDn<N, R> b) {
    return {a.re + b.re, a.im + b.im};
}
template <int N, class R>
__device__ __forceinline__ CDn<N, R> cdsub(CDn<N, R> a, CDn<N, R> b) {
    return {a.re - b.re, a.im - b.im};
}
template <int N, class R>
__device__ __forceinline__ CDn<N, R> cdscale(CDn<N, R> a, Dn<N, R> s) {
    return {a.re * s, a.im * s};
}
template <int N, class R>
__device__ __forceinline__ CDn<N, R> cdscale(CDn<N, R> a, nd_t<R> s) {
    return {a.re * s, a.im * s};
}
// e^{2 pi i r} for r in revolutions (|r| <= 1/2)
template <int N, class R>
__device__ __forceinline__ CDn<N, R> dexpi_rev(Dn<N, R> r) {
    R s, c;
    sincos_rev(r.v, s, c);
    CDn<N, R> o;
    o.re.v = c;
    o.im.v = s;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        o.re.d[i] = -(R)kTwoPi * s * r.d[i];
        o.im.d[i] = (R)kTwoPi * c * r.d[i];
    }
    return o;
}
template <class R, int N>
__device__ __forceinline__ Dn<N, R> to_r(const Dn<N, double> &a) {
    Dn<N, R> o;
    o.v = (R)a.v;
#pragma unroll
    for (int i = 0; i < N; ++i) o.d[i] = (R)a.d[i];
    return o;
}

// ------------------------------------------------------------------ track tangents
// Tangent slots: 0 = ln Mc, 1 = f0 (eta is held fixed).  M scales with Mc, so
// dM/M = (1, 0); theta0 follows from theta0^3 P(theta0) = 8 pi M f0 by implicit
// differentiation; t_c = 5 M theta0^-8 / eta.
struct TrackTan {
    double mu[2];   // dM/M
    double dtc[2];  // dt_c
};

__device__ inline TrackTan track_tangents(const Track &T, double f0) {
    TrackTan G;
    const double th = T.th0, th2 = th * th, th3 = th2 * th, th4 = th2 * th2;
    const double dP = ((3.0 + (5.0 * T.a2) * th2) + (6.0 * T.a3) * th3) + (7.0 * T.a4) * th4;
    const double z = T.c8 * f0;
    const double dz[2] = {z, T.c8};
    G.mu[0] = 1.0;
    G.mu[1] = 0.0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const double dth0 = dz[p] / (th2 * dP);
        G.dtc[p] = T.tc * (G.mu[p] - 8.0 * dth0 / th);
    }
    return G;
}

// Phase, frequency and chirp tangents at t < t_c.  s = 1/theta comes from the forward's track_at (its theta is
// rcp_rn(s)); the per-template divisors enter through their reciprocals and theta^-6 as s^6, since the
// tangents need no correctly rounded quotients.
struct TrackDual {
    double dPhi[2], df[2], dfdot[2];
};

template <class R>
__device__ inline TrackDual track_dual(const Track &T, const TrackTan &G, double t, double f, double s) {
    const double tau = T.tc - t;
    const double itau = rcp_rn(tau);
    const double th = rcp_rn(s);
    const double th2 = th * th, th3 = th2 * th, th4 = th2 * th2, th5 = th4 * th, th9 = th5 * th4;
    const double s2 = s * s, s6 = (s2 * s2) * s2;  // theta^-6
    const double dPf = ((3.0 + (5.0 * T.a2) * th2) + (6.0 * T.a3) * th3) + (7.0 * T.a4) * th4;
    const double ddPf = ((10.0 * T.a2) * th + (18.0 * T.a3) * th2) + (28.0 * T.a4) * th3;
    const double dfdth = (th2 * T.rc8) * dPf;
    const double dthdt = (T.eta * th9) * T.r40M;
    const double Pp = ((1.0 + T.b2 * th2) + T.b3 * th3) + T.b4 * th4;
    const double dPp = ((2.0 * T.b2) * th + (3.0 * T.b3) * th2) + (4.0 * T.b4) * th3;
    const double dPhidth = (2.0 * T.reta) * (5.0 * Pp - th * dPp) * s6;
    TrackDual D;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const double mu = G.mu[p];
        const double dth = -0.125 * th * (G.dtc[p] * itau - mu);
        D.df[p] = dfdth * dth - f * mu;
        const double d_dfdth = ((2.0 * th * dPf + th2 * ddPf) * T.rc8) * dth - dfdth * mu;
        // FP32 form: the quotient, whose rounding its results carry; FP64 form: s = 1/theta
        double dlnth;
        if constexpr (sizeof(R) == 4)
            dlnth = 9.0 * dth / th;
        else
            dlnth = 9.0 * dth * s;
        const double d_dthdt = dthdt * (dlnth - mu);
        D.dfdot[p] = d_dfdth * dthdt + dfdth * d_dthdt;
        D.dPhi[p] = dPhidth * dth;
    }
    return D;
}

__device__ inline void dphi_at(const Track &T, const TrackTan &G, double t, double out[2]) {
    const double tau = T.tc - t;
    const double itau = rcp_rn(tau);
    const double s = sqrt_pos(sqrt_pos(sqrt_pos((T.eta * tau) * T.r5M)));
    const double th = rcp_rn(s);
    const double th2 = th * th, th3 = th2 * th, th4 = th2 * th2;
    const double s2 = s * s, s6 = (s2 * s2) * s2;  // theta^-6
    const double Pp = ((1.0 + T.b2 * th2) + T.b3 * th3) + T.b4 * th4;
    const double dPp = ((2.0 * T.b2) * th + (3.0 * T.b3) * th2) + (4.0 * T.b4) * th3;
    const double dPhidth = (2.0 * T.reta) * (5.0 * Pp - th * dPp) * s6;
#pragma unroll
    for (int p = 0; p < 2; ++p) out[p] = dPhidth * (-0.125 * th * (G.dtc[p] * itau - G.mu[p]));
}

// ------------------------------------------------------------------ response tangents
// Tangent slots: 0 = f, 1 = cos theta, 2 = phi, 3 = psi.  Same formulas as transfer_ae.  The
// sky constants are formed in FP64 and rounded to R; kv keeps the FP64 propagation direction,
// from which the light-travel phases are formed in FP64 in both arithmetics.
template <class R>
struct SkyD {
    Dn<4, R> k[3], u[3], v[3], c2, s2;
    R ap, ci;
    double kv[3];
};

template <class R>
__device__ inline void sky_dual(SkyD<R> &S, double ct, double phi, double psi, double ci) {
    Dn<4> c = dconst<4, double>(ct);
    c.d[1] = 1.0;
    double sp, cp, s2, c2;
    sincos(phi, &sp, &cp);
    sincos(2.0 * psi, &s2, &c2);
    Dn<4> Sp = dconst<4, double>(sp), Cp = dconst<4, double>(cp);
    Sp.d[2] = cp;
    Cp.d[2] = -sp;
    Dn<4> st = dsqrt(1.0 - c * c);
    const Dn<4> k[3] = {-(st * Cp), -(st * Sp), -c};
    const Dn<4> u[3] = {c * Cp, c * Sp, -st};
    const Dn<4> v[3] = {Sp, -Cp, dconst<4, double>(0.0)};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        S.k[i] = to_r<R>(k[i]);
        S.u[i] = to_r<R>(u[i]);
        S.v[i] = to_r<R>(v[i]);
        S.kv[i] = k[i].v;
    }
    S.c2 = dconst<4, R>((R)c2);
    S.s2 = dconst<4, R>((R)s2);
    S.c2.d[3] = (R)(-2.0 * s2);
    S.s2.d[3] = (R)(2.0 * c2);
    S.ap = (R)((1.0 + ci * ci) / 2.0);
    S.ci = (R)ci;
}

template <bool WITH_T, class R>
__device__ inline void transfer_ae_dual(const SkyD<R> &S, const double (&g)[kGeoRows], double f, CDn<4, R> &TA,
                                        CDn<4, R> &TE, CDn<4, R> &TT) {
    const double L = kArmM / kClight;
    Dn<4, R> F = dconst<4, R>((R)f);
    F.d[0] = (R)1;
    Dn<4, R> kp[3];
    double kpv[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        kp[i] = S.k[0] * (R)g[3 * i] + S.k[1] * (R)g[3 * i + 1] + S.k[2] * (R)g[3 * i + 2];
        kpv[i] = S.kv[0] * g[3 * i] + S.kv[1] * g[3 * i + 1] + S.kv[2] * g[3 * i + 2];
    }
    const Dn<4, R> pfL = F * (R)(kPi * L);
    CDn<4, R> Gd[3], Gr[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int s = a, r = (a + 1) % 3;
        const R n0 = (R)g[9 + 3 * a + 0];
        const R n1 = (R)g[9 + 3 * a + 1];
        const R n2 = (R)g[9 + 3 * a + 2];
        Dn<4, R> kn = S.k[0] * n0 + S.k[1] * n1 + S.k[2] * n2;
        Dn<4, R> nu = S.u[0] * n0 + S.u[1] * n1 + S.u[2] * n2;
        Dn<4, R> nv = S.v[0] * n0 + S.v[1] * n1 + S.v[2] * n2;
        Dn<4, R> xp0 = nu * nu - nv * nv, xx0 = 2.0 * (nu * nv);
        Dn<4, R> xp = S.c2 * xp0 + S.s2 * xx0;
        Dn<4, R> xx = S.s2 * (-xp0) + S.c2 * xx0;
        CDn<4, R> amp = {xp * S.ap, xx * (-S.ci)};
        // -pi f (L + k.(p_s + p_r)) in revolutions: value reduced in FP64, tangents in R
        const double ksv = (kpv[s] + kpv[r]) + L;
        const double fh = f * (-0.5);
        Dn<4, R> rev;
        rev.v = (R)frac_rev(fh * ksv);
#pragma unroll
        for (int q = 0; q < 4; ++q) rev.d[q] = (R)fh * (kp[s].d[q] + kp[r].d[q]);
        rev.d[0] += (R)(-0.5 * ksv);
        CDn<4, R> Ea = cdmul(dexpi_rev(rev), amp);
        CDn<4, R> B = {pfL * Ea.im, -(pfL * Ea.re)};
        Gd[a] = cdscale(B, dsinc(pfL * (1.0 - kn)));
        Gr[a] = cdscale(B, dsinc(pfL * (1.0 + kn)));
    }
    const CDn<4, R> G01 = Gd[0], G10 = Gr[0], G12 = Gd[1], G21 = Gr[1], G20 = Gd[2], G02 = Gr[2];
    // 1 - D^2 = 2 i sin(2 pi f L) D, D = e^{-2 pi i f L}
    Dn<4, R> rl = dconst<4, R>((R)frac_rev(f * L));
    rl.d[0] = (R)L;
    const CDn<4, R> D = dexpi_rev(-rl);
    const Dn<4, R> s2 = dsin_rev(rl);
    const CDn<4, R> om = {(-2.0) * (s2 * D.im), 2.0 * (s2 * D.re)};
    const CDn<4, R> TX = cdmul(om, cdsub(cdadd(G20, cdmul(D, G02)), cdadd(G10, cdmul(D, G01))));
    const CDn<4, R> TY = cdmul(om, cdsub(cdadd(G01, cdmul(D, G10)), cdadd(G21, cdmul(D, G12))));
    const CDn<4, R> TZ = cdmul(om, cdsub(cdadd(G12, cdmul(D, G21)), cdadd(G02, cdmul(D, G20))));
    const double is2 = 0.70710678118654752440, is6 = 0.40824829046386301637;
    TA = cdscale(cdsub(TZ, TX), is2);
    TE = cdscale(cdadd(cdsub(TX, cdscale(TY, 2.0)), TZ), is6);
    if constexpr (WITH_T) TT = cdscale(cdadd(cdadd(TX, TY), TZ), 0.57735026918962576451);  // (X + Y + Z) / sqrt3
}

// ------------------------------------------------------------------ spectrum tangents
// Tangent slots: 0 = ln Mc, 1 = f0.  Bin-relative Fresnel form as in tranche_spectrum_bin; the
// bin index, offset, phases and the Fresnel branch ranges come from FP64 as in tranche_setup,
// so the integer structure is the forward's.
template <class R>
struct SpecD {
    Dn<2, R> x, beta, s, P, Q, hib;
    CDn<2, R> E0, E1;
    double rev0;
    R drev0[2];
    int j0lo, j0hi, j1lo, j1hi;
};

template <class R>
__device__ inline int spec_dual(SpecD<R> &S, double Phi, double f, double fdot, const TrackDual &D,
                                const double dref[2], double dT) {
    const double fT = f * dT;
    const double kc = ceil(fT);
    const double x = fT - kc, beta = (fdot * dT) * dT;
    S.x = dconst<2, R>((R)x);
    S.beta = dconst<2, R>((R)beta);
    Dn<2, R> A, Fd = dconst<2, R>((R)fdot);
    if constexpr (sizeof(R) == 8) {
        const double c = cbrt(f);
        A.v = c * c;
    } else
        A.v = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf((float)f) * (2.0f / 3.0f));
    const R dlnA = (R)(2.0 / 3.0) * (A.v / (R)f);
    const double rev0 = phase_to_rev(Phi);
    Dn<2, R> r0 = dconst<2, R>((R)rev0);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        S.x.d[p] = (R)(dT * D.df[p]);
        S.beta.d[p] = (R)((dT * dT) * D.dfdot[p]);
        A.d[p] = dlnA * (R)D.df[p];
        Fd.d[p] = (R)D.dfdot[p];
        r0.d[p] = (R)((D.dPhi[p] - dref[p]) * (1.0 / kTwoPi));
    }
    S.s = dsqrt(2.0 * drcp(S.beta));
    S.P = A * drcp(dsqrt(2.0 * Fd));
    S.Q = A * (dT / kTwoPi);
    S.hib = 0.5 * drcp(S.beta);
    {
        const double r6 = sqrt(18.0 * beta);  // 6 / s: |v| <= 6 takes the paper's rational forms
        S.j0lo = (int)ceil(x - r6);
        S.j0hi = (int)floor(x + r6);
        S.j1lo = (int)ceil((x + beta) - r6);
        S.j1hi = (int)floor((x + beta) + r6);
    }
    Dn<2, R> r1 = r0 + S.x + 0.5 * S.beta;
    r1.v = (R)frac_rev(rev0 + x + 0.5 * beta);
    S.E0 = dexpi_rev(r0);
    S.E1 = dexpi_rev(r1);
    S.rev0 = rev0;
    S.drev0[0] = r0.d[0];
    S.drev0[1] = r0.d[1];
    return (int)kc;
}

template <class R>
__device__ __forceinline__ void fresnel_fg_dual(Dn<2, R> av, bool rational, Dn<2, R> &f, Dn<2, R> &g) {
    if (!rational) {
        f = drcp(kPi * av);
        g = dconst<2, R>((R)0);
    } else {
        Dn<2, R> a2 = av * av;
        f = (1.0 + 0.926 * av) * drcp((2.0 + 1.792 * av) + 3.104 * a2);
        g = drcp(((2.0 + 4.142 * av) + 3.492 * a2) + 6.670 * (a2 * av));
    }
}

template <class R>
__device__ inline CDn<2, R> bin_dual(const SpecD<R> &S, int j) {
    const Dn<2, R> xj = S.x + (R)(-j);
    const Dn<2, R> xj1 = xj + S.beta;
    if (j < S.j0lo || j > S.j1hi) {
        // asymptotic Fresnel on both edges, no crossing: h = i Q (E0 / xj - E1 / xj1)
        const Dn<2, R> a = drcp(xj), b = drcp(xj1);
        const Dn<2, R> re = S.E0.re * a - S.E1.re * b;
        const Dn<2, R> im = S.E0.im * a - S.E1.im * b;
        return {-(S.Q * im), S.Q * re};
    }
    const Dn<2, R> v0 = S.s * xj, v1 = S.s * xj1;
    const R sg0 = v0.v > (R)0 ? (R)1 : (v0.v < (R)0 ? (R)-1 : (R)0);
    const R sg1 = v1.v > (R)0 ? (R)1 : (v1.v < (R)0 ? (R)-1 : (R)0);
    Dn<2, R> f0, g0, f1, g1;
    fresnel_fg_dual(v0 * (sg0 < (R)0 ? (R)-1 : (R)1), j >= S.j0lo && j <= S.j0hi, f0, g0);
    fresnel_fg_dual(v1 * (sg1 < (R)0 ? (R)-1 : (R)1), j >= S.j1lo && j <= S.j1hi, f1, g1);
    const CDn<2, R> t0 = cdmul(CDn<2, R>{g0 * sg0, f0 * sg0}, S.E0);
    const CDn<2, R> t1 = cdmul(CDn<2, R>{g1 * sg1, f1 * sg1}, S.E1);
    CDn<2, R> h = cdsub(t0, t1);
    const R ds = sg1 - sg0;
    if (ds != (R)0) {
        // stationary-phase term e^{2 pi i (rev0 - xj^2 / (2 beta))}
        const Dn<2, R> q = (xj * xj) * S.hib;
        Dn<2, R> rv;
        rv.v = (R)frac_rev(S.rev0 - (double)q.v);
        rv.d[0] = S.drev0[0] - q.d[0];
        rv.d[1] = S.drev0[1] - q.d[1];
        const CDn<2, R> e = dexpi_rev(rv);
        const R hh = (R)0.5 * ds;
        h.re = h.re + hh * (e.re - e.im);
        h.im = h.im + hh * (e.re + e.im);
    }
    return cdscale(h, S.P);
}

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

// ------------------------------------------------------------------ kernel
struct VjpArgs {
    int M, K, Nt, C;
    double dT, df, fnyq;
    const void *pix;
    // pixel (channel c, bin k, tranche m) is element c * chan + k * row + m * col of the store, whatever its layout
    size_t chan, col;
    uint32_t row;
    const float *layer_scale;
    const double *inv_asd, *tranche_w, *geo, *u_scale;
    const float *rho;  // [K][Nt] per-pixel weight factor (general per-tranche PSD), else NULL
    int64_t n;
    const double *mc, *eta, *f0, *ct, *phi, *psi, *ci;
    const int32_t *nseg;
    const int64_t *seg_offset;
    const double *seg_zn, *g_stat, *g_seg;
    double *g_params;
    // each wave takes one unit of `chunks` chunks of a template (units per template: 1 = whole templates)
    int units, chunks;
    const double *rec;  // template records (k_prepare), or NULL
    double *part;       // [n][units][5] gradients of the units, if units > 1
};

// R = double: the FP64 form; R = float: FP32 spectra, response, pixel sums and tangents (the
// track, its tangents, the phases and every integer decision stay FP64, as in the FP32 forward).
// The FP32 form holds half the registers and runs two waves per SIMD.
//
// One unit per wave, in runs per XCD (run_item, in the bank's own order); k_vjp_finish adds the units.
//
// Bound: FP64, latency of dependent FP64 chains at one wave per SIMD; FP32, vector-ALU issue at two.  Two-year grid, A+E:
// 320 templates FP64 2282 us with a wave per template and the tangents carried through every bin, 1058 in units with the
// moments, 913 with each lane's own band instead of the wave's, 590 with the units dealt out to all XCDs, 527 with sincospi
// and reciprocals for sincos, pow and divisions; 65,536 templates FP32 40 -> 33.7 ms from units in runs
// per XCD, a pixel's address in one multiply-add for every layout, and the next bin's loads ahead.
template <int C, class PixT, class R>
__global__ __launch_bounds__(256, sizeof(R) == 4 ? 2 : 1) void k_vjp_wave(VjpArgs a) {
    using PR = typename PixTraits<PixT>::R;
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
            if (a.rec) {
                load_track(a.rec + i * kRecDoubles, lane, T);
            } else {
                track_init(T, mci, a.eta[i], a.f0[i]);
                wave_uniform(T);
            }
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
                        auto bin = [&](int j, R &u, cx<PR> (&Dl)[C]) {
                            const int k = min(max(kc + j, 1), kmax);
                            const char *p = pix + (uint64_t)(uint32_t)k * row;
#pragma unroll
                            for (int c = 0; c < C; ++c) Dl[c] = PixTraits<PixT>::load(p, (size_t)c * a.chan);
                            u = u_pad[kc + j + kHalfBins];
                            if (a.rho) u *= (R)a.rho[(size_t)k * a.Nt + m];
                        };
                        auto to_arith = [&](int j, const cx<PR> (&Dl)[C], cx<R> (&D)[C]) {
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                D[c] = {(R)Dl[c].re, (R)Dl[c].im};
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
                                cx<PR> Dl[3][C];
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
                                cx<PR> Dl[C];
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
                            cx<PR> Dn[C] = {};
#pragma unroll 1
                            for (int j = -kHalfBins - 1; j <= kHalfBins; ++j) {
                                const R u = un;
                                cx<PR> Dl[C];
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
                                    R dr = (R)Dl[c].re, di = (R)Dl[c].im;
                                    if constexpr (PixTraits<PixT>::scaled) {
                                        const R sc = (R)a.layer_scale[c * a.K + min(max(kc + j, 1), kmax)];
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
            double *o = a.units > 1 ? a.part + 5 * (i * a.units + unit) : a.g_params + 5 * i;
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

// Whole templates go one to a block, so that a long one holds up no others.
template <int C, class PixT, class R>
static hipError_t launch_vjp_t(const VjpArgs &a, int block_waves, hipStream_t st) {
    const size_t shmem = sizeof(R) * ((size_t)a.K + 2 * kHalfBins);
    const int bw = a.units > 1 ? block_waves : 1;
    hipLaunchKernelGGL((k_vjp_wave<C, PixT, R>), dim3(run_groups(a.n, bw, a.units)), dim3(64 * bw), shmem, st, a);
    if (a.units > 1)
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
    a.units = L.split.units ? L.split.units : 1;
    a.chunks = L.split.units ? L.split.chunks : (L.Nt + 63) / 64;
    a.rec = L.split.units ? L.split.rec : nullptr;
    a.part = reinterpret_cast<double *>(L.split.head);
    return L.precision == 1 ? dispatch_vjp_c<float>(a, L.C, L.pix_dtype, L.block_waves, st)
                            : dispatch_vjp_c<double>(a, L.C, L.pix_dtype, L.block_waves, st);
}

}  // namespace tfsc
