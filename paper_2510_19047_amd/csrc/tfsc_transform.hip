// Data -> whitened TF pixels (paper Sec. "Implementation details": every
// tranche is Tukey-windowed and Fourier transformed once; per-tranche PSD;
// tranches overlapping gaps are excluded).
//
// Consecutive tranches of a channel go in pairs as the real and imaginary parts of one complex
// sequence through a radix-2 Stockham FFT (natural order in and out, twiddles from a per-block LDS
// table), are split into the two tranches' spectra, whitened and stored in the layout asked for.
// 16-bit stores go through an FP32 staging buffer and a second pass that applies a per-layer scale.
#include "tfsc_device.hpp"
#include "tfsc_kernels.hpp"

namespace tfsc {

__device__ __forceinline__ bool psd_ok(double S) { return S > 0.0 && S < __builtin_huge_val(); }

// Window value n of the Tukey window with tapers of `width` + 1 samples (width = floor(alpha (M - 1) / 2), -1: none).
template <class R>
__device__ __forceinline__ R tukey_w(int n, int M, double alpha, int width) {
    const int nn = min(n, M - 1 - n);
    if (nn > width) return (R)1;
    return (R)(0.5 * (1.0 + cospi(-1.0 + 2.0 * nn / (alpha * (M - 1)))));
}

template <class R>
__device__ __forceinline__ cx<R> twiddle(double frac);  // exp(-2 pi i frac)
template <>
__device__ __forceinline__ cx<double> twiddle<double>(double frac) {
    double s, c;
    sincospi(-2.0 * frac, &s, &c);
    return {c, s};
}
template <>
__device__ __forceinline__ cx<float> twiddle<float>(double frac) {
    float s, c;
    sincospif((float)(-2.0 * frac), &s, &c);
    return {c, s};
}

// Windowed FFT and whitening.  A thread holds 8 of the M points of a pair's complex sequence (points t + i M/8) and
// runs three radix-2 Stockham stages on them in registers between two exchanges through LDS, so an M-point transform
// makes ceil(log2(M) / 3) exchanges instead of log2(M); M/8 threads share a transform and a block of 256 (512 for
// M = 4096) runs 2048 / M of them side by side on consecutive tranches.  The butterflies, their twiddles and their
// order are those of the plain radix-2 algorithm, so the results are the same bits.
//
// The first stages take their points from the series itself; the last exchange puts Z in natural order for the split
// of the two tranches.  A thread keeps the whitened values of NIT transforms (a pair of tranches of each of the CC
// channels of a cell, or NIT pairs of one channel) and writes a run of 16 or 32 bytes per frequency layer.  Consecutive
// tiles go to one XCD, whose L2 joins the runs of neighbouring tiles.  Each group's largest values of a 16-bit store's
// layers meet in LDS before the global atomics: with one atomic per layer and group they queued up at the few addresses of
// a small M (A+E, M = 128, 60,000 tranches, 16 bits: 2528 us a call, now 100).
//
// Bound: latency, at three to four waves per SIMD (53 KB of LDS at M = 2048 allow three blocks a CU).  Two years of A+E,
// FP32 (100.7 MB in, 100.8 MB out): 80 us, 2.5 TB/s, against 520 us with one exchange per stage, a branch (and a wait)
// around every load and 8-byte stores.  With a loop over two such runs in a block the transforms' registers passed 150 and
// a few spilled: 87 us, and short sets waited for twice the work (A+E, M = 1024, 33 tranches: 21 us a call against 14).
// Holding the runs of four tranches or the window in registers across the transforms spilled and took 139-168 us; forming
// the whitening factors (a division and a square root per bin and tranche) for each channel anew, 10 us more.
//
// -i w: the twiddle a quarter turn on.  For a twiddle below exp(-i pi / 4) it has the table's bits; from there on the
// table's own entry is read (its sine and cosine of pi / 4 differ in the last place).
template <class R>
__device__ __forceinline__ cx<R> mul_neg_i(cx<R> w) { return {w.im, -w.re}; }

// (a, b) -> (a + w b, a - w b).  The product's roundings are written out (b.im w.im and b.re w.im are rounded, the rest is
// fused): left to the compiler they would depend on whether w comes from the table or from mul_neg_i.
template <class R>
__device__ __forceinline__ void butterfly(cx<R> &a, cx<R> &b, cx<R> w) {
    const R p = b.im * w.im, q = b.re * w.im;
    const cx<R> bw = {fma(b.re, w.re, -p), fma(b.im, w.re, q)};
    b = csub(a, bw);
    a = cadd(a, bw);
}

// A complex value in LDS, moved with one 16-byte (FP64) or 8-byte (FP32) access.
template <class R>
struct alignas(2 * sizeof(R)) lds_cx {
    R re, im;
    __device__ __forceinline__ operator cx<R>() const { return {re, im}; }
};

// Padding: one element in 8 (the stage outputs lie 8 apart), one in 64 for the twiddles.  The lanes' positions are
// base + constant, so that every offset is an immediate of the access.
__host__ __device__ constexpr int lds_pos(int i) { return i + (i >> 3); }
__host__ __device__ constexpr int tw_pos(int i) { return i + (i >> 6); }

// Three radix-2 stages on the thread's points v[i] = src[t + i M/8], at sub-transform length NS, kk = t mod NS.
template <int M, int NS, class R>
__device__ __forceinline__ void stages3(cx<R> (&v)[8], const lds_cx<R> *tw, int kk) {
    const cx<R> w1 = tw[tw_pos(kk * (M / (2 * NS)))];
#pragma unroll
    for (int i = 0; i < 4; ++i) butterfly(v[i], v[i + 4], w1);  // v[i] = (i, b0 = 0), v[i + 4] = (i, b0 = 1)
    const cx<R> w2 = tw[tw_pos(kk * (M / (4 * NS)))], w2i = tw[tw_pos((kk + NS) * (M / (4 * NS)))];
    butterfly(v[0], v[2], w2);
    butterfly(v[1], v[3], w2);
    butterfly(v[4], v[6], w2i);
    butterfly(v[5], v[7], w2i);
    constexpr int Q = M / (8 * NS);
    const cx<R> w3 = tw[tw_pos(kk * Q)], w3b = tw[tw_pos((kk + NS) * Q)], w3d = tw[tw_pos((kk + 3 * NS) * Q)];
    butterfly(v[0], v[1], w3);             // b0 = 0, b1 = 0: outputs 0 and 4
    butterfly(v[4], v[5], w3b);            // b0 = 1, b1 = 0: outputs 1 and 5
    butterfly(v[2], v[3], mul_neg_i(w3));  // b0 = 0, b1 = 1: outputs 2 and 6
    butterfly(v[6], v[7], w3d);            // b0 = 1, b1 = 1: outputs 3 and 7
}

// Output q of stages3 belongs at 8 (t - kk) + kk + q NS.
template <int NS, class R>
__device__ __forceinline__ void store8(const cx<R> (&v)[8], lds_cx<R> *buf, int t, int kk) {
    constexpr int from[8] = {0, 4, 2, 6, 1, 5, 3, 7};
    lds_cx<R> *p = buf + lds_pos(8 * (t - kk) + kk);
#pragma unroll
    for (int q = 0; q < 8; ++q)
        p[NS == 1 ? q : lds_pos(q * NS)] = {v[from[q]].re, v[from[q]].im};
}

template <int T8, class R>
__device__ __forceinline__ void load8(cx<R> (&v)[8], const lds_cx<R> *buf, int t) {
    const lds_cx<R> *p = buf + lds_pos(t);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[lds_pos(i * T8)];
}

// One block's transforms: CC channels (1, or all of a channel-interleaved cell) of TB tranches per group of M/8
// threads.  Tranches are transformed in pairs, z = x_m + i x_{m+1}: X_m[k] = (Z[k] + conj Z[M-k]) / 2 and
// X_{m+1}[k] = (Z[k] - conj Z[M-k]) / (2i).
template <class R, class XT, class OutT, int M, int CC, int NIT>
__global__ __launch_bounds__(M == 4096 ? 512 : 256, CC == 3 ? 2 : 3) void k_transform(
    TransformLaunch L, double w2, int width, uint32_t *__restrict__ layer_max, int n_tiles) {
    constexpr int TB = 2 * NIT / CC;  // tranches per group
    constexpr int K = M / 2 + 1, T8 = M / 8, NT = M == 4096 ? 512 : 256, NG = NT / T8;
    __shared__ lds_cx<R> tw[tw_pos(M / 2)];        // exp(-2 pi i k / M)
    __shared__ lds_cx<R> bufs[NG * lds_pos(M)];
    const int Nt = L.Nt;
    const int t0 = threadIdx.x & (T8 - 1), grp = threadIdx.x / T8;
    lds_cx<R> *buf = bufs + grp * lds_pos(M);
    uint32_t *top = reinterpret_cast<uint32_t *>(bufs);  // [NG][CC][K] after the transforms: the groups' layer maxima
    for (int k = threadIdx.x; k < M / 2; k += NT) {
        const cx<R> w = twiddle<R>((double)k / M);
        tw[tw_pos(k)] = {w.re, w.im};
    }
    // tiles of consecutive tranches on one XCD (workgroups go round the 8 XCDs)
    const int per_xcd = (n_tiles + 7) / 8;
    const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || tile >= n_tiles) return;
    const int c0 = blockIdx.y * CC;
    // whitening factor for the PSD value S of a tranche with its keep mark; a bin whose PSD is not positive and finite
    // (DC or Nyquist may carry 0 or inf) gets pixel 0 rather than inf or NaN; its template weight is 0 as well.  No
    // branches here nor in the loads: the latencies of a thread's values then overlap.
    auto scale = [&](double S, bool kept) -> R {
        const bool ok = kept && psd_ok(S);
        const double v = sqrt(2.0 * L.dt / ((double)M * w2 * (ok ? S : 1.0)));
        return (R)(ok ? v : 0.0);
    };
    auto psd = [&](int k, int mj, double mu) -> double {  // mj < Nt
        return L.psd_tf ? L.psd_tf[(size_t)k * Nt + mj] : L.psd0[k] * mu;
    };
    const int m0 = (tile * NG + grp) * TB;
    // held[it][i][tr]: bin k = t + i M/8 of tranche m + tr; DC and Nyquist are real, so bin 0 holds (DC, Nyquist)
    cx<OutT> held[NIT][4][2] = {};
    R sc[4][2], scn[2];
    // a cell's channels one after the other without a loop, so that the pair's whitening factors and the values
    // held live only as long as they must; of one channel the loop stays (unrolled it would spill)
    constexpr int kUnroll = CC == 1 ? 1 : NIT;
#pragma unroll kUnroll
    for (int it = 0; it < NIT; ++it) {
        const int c = c0 + it % CC, m = m0 + 2 * (it / CC);
        // the thread's index anew for each transform: the addresses, window and PSD values that depend on it are then
        // formed where they are used instead of being held in registers (and spilled) across the transforms
        int t = t0;
        asm volatile("" : "+v"(t));
        cx<R> v[8];
        {
            // tranches past the end read the last one and count as zero
            const int ma = min(m, Nt - 1), mb = min(m + 1, Nt - 1);
            const XT *xa = reinterpret_cast<const XT *>(L.x) + ((size_t)c * Nt + ma) * M + t;
            const XT *xb = reinterpret_cast<const XT *>(L.x) + ((size_t)c * Nt + mb) * M + t;
            XT a[8], b[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                a[i] = xa[i * T8];
                b[i] = xb[i * T8];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const R win = tukey_w<R>(t + i * T8, M, L.alpha, width);
                v[i].re = m < Nt ? (R)a[i] * win : (R)0;
                v[i].im = m + 1 < Nt ? (R)b[i] * win : (R)0;
            }
        }
        __syncthreads();  // the twiddles are there, and the last transform's split has read its points
        stages3<M, 1>(v, tw, 0);
        store8<1>(v, buf, t, 0);
        __syncthreads();
        load8<T8>(v, buf, t);
        stages3<M, 8>(v, tw, t & 7);
        __syncthreads();
        store8<8>(v, buf, t, t & 7);
        __syncthreads();
        if constexpr (M >= 512) {
            load8<T8>(v, buf, t);
            stages3<M, 64>(v, tw, t & 63);
            __syncthreads();
            store8<64>(v, buf, t, t & 63);
            __syncthreads();
        }
        if constexpr (M >= 4096) {
            load8<T8>(v, buf, t);
            stages3<M, 512>(v, tw, t & 511);
            __syncthreads();
            store8<512>(v, buf, t, t & 511);
            __syncthreads();
        }
        constexpr int LEFT = M >= 512 ? (M >= 4096 ? M / 4096 : M / 512) : M / 64;  // stages left: 1, 2 or 4 points
        if constexpr (LEFT == 2) {
            constexpr int NS = M / 2;
            load8<T8>(v, buf, t);
            __syncthreads();
            lds_cx<R> *p = buf + lds_pos(t);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                butterfly(v[i], v[i + 4], (cx<R>)tw[tw_pos(t + i * T8)]);
                p[lds_pos(i * T8)] = {v[i].re, v[i].im};
                p[lds_pos(i * T8 + NS)] = {v[i + 4].re, v[i + 4].im};
            }
            __syncthreads();
        } else if constexpr (LEFT == 4) {
            constexpr int NS = M / 4;
            load8<T8>(v, buf, t);
            __syncthreads();
            lds_cx<R> *p = buf + lds_pos(t);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int kk = t + i * T8;  // < NS
                const cx<R> wa = tw[tw_pos(2 * kk)], wb = tw[tw_pos(kk)], wbi = tw[tw_pos(kk + NS)];
                butterfly(v[i], v[i + 4], wa);
                butterfly(v[i + 2], v[i + 6], wa);
                butterfly(v[i], v[i + 2], wb);        // b0 = 0: outputs 0 and 2
                butterfly(v[i + 4], v[i + 6], wbi);   // b0 = 1: outputs 1 and 3
                p[lds_pos(i * T8)] = {v[i].re, v[i].im};
                p[lds_pos(i * T8 + NS)] = {v[i + 4].re, v[i + 4].im};
                p[lds_pos(i * T8 + 2 * NS)] = {v[i + 2].re, v[i + 2].im};
                p[lds_pos(i * T8 + 3 * NS)] = {v[i + 6].re, v[i + 6].im};
            }
            __syncthreads();
        }
        // the whitening factors of the pair, where the transform's registers are free
        const int ma = min(m, Nt - 1), mb = min(m + 1, Nt - 1);
        const double mua = L.psd_tf ? 1.0 : L.mu[ma], mub = L.psd_tf ? 1.0 : L.mu[mb];
        const bool ka = L.keep[ma] != 0, kb = L.keep[mb] != 0;
        if (it % CC == 0) {
            double sa[4], sb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sa[i] = psd(t + i * T8, ma, mua);
                sb[i] = psd(t + i * T8, mb, mub);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sc[i][0] = scale(sa[i], ka);
                sc[i][1] = scale(sb[i], kb);
            }
            if (t == 0) {
                scn[0] = scale(psd(M / 2, ma, mua), ka);
                scn[1] = scale(psd(M / 2, mb, mub), kb);
            }
        }
        // the oldest transform's values stand first after the last turn
#pragma unroll
        for (int q = 0; q + 1 < NIT; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                held[q][i][0] = held[q + 1][i][0];
                held[q][i][1] = held[q + 1][i][1];
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = t + i * T8;
            const cx<R> zk = buf[lds_pos(t) + lds_pos(i * T8)], zn = buf[lds_pos((M - k) & (M - 1))];
            cx<R> X[2] = {{(R)0.5 * (zk.re + zn.re), (R)0.5 * (zk.im - zn.im)},
                          {(R)0.5 * (zk.im + zn.im), (R)0.5 * (zn.re - zk.re)}};
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                cx<R> o = cscale(X[j], sc[i][j]);
                if (i == 0 && t == 0) {
                    const cx<R> zq = buf[lds_pos(M / 2)];
                    o.im = (j == 0 ? zq.re : zq.im) * scn[j];
                }
                held[NIT - 1][i][j] = {(OutT)o.re, (OutT)o.im};
            }
        }
    }

    OutT *pix = reinterpret_cast<OutT *>(L.pix);
    auto put = [&](int k, int q, int j, cx<OutT> o) {  // the pixel of transform q, tranche j of its pair
        const int c = c0 + q % CC, m = m0 + 2 * (q / CC) + j;
        if (m >= Nt) return;
        const size_t idx = L.out_layout == 0   ? ((size_t)c * K + k) * Nt + m
                           : L.out_layout == 1 ? ((size_t)c * Nt + m) * K + k
                                               : ((size_t)k * Nt + m) * L.C + c;
        reinterpret_cast<cx<OutT> *>(pix)[idx] = o;
    };
    // one 16-byte store per FP32 A+E cell
    auto put_cells = [&](int k, const cx<OutT> (&a)[2], const cx<OutT> (&b)[2], int q) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int m = m0 + 2 * (q / CC) + j;
            if (m >= Nt) continue;
            reinterpret_cast<float4 *>(pix)[(size_t)k * Nt + m] =
                float4{(float)a[j].re, (float)a[j].im, (float)b[j].re, (float)b[j].im};
        }
    };
    auto put_row = [&](int k, const cx<OutT> (&row)[NIT][2]) {
        if constexpr (CC == 2 && sizeof(OutT) == 4) {
#pragma unroll
            for (int q = 0; q < NIT; q += 2) put_cells(k, row[q], row[q + 1], q);
        } else {
#pragma unroll
            for (int q = 0; q < NIT; ++q)
#pragma unroll
                for (int j = 0; j < 2; ++j) put(k, q, j, row[q][j]);
        }
        if constexpr (sizeof(OutT) == 4)
            if (layer_max) {
#pragma unroll
                for (int cc = 0; cc < CC; ++cc) {
                    float mx = 0.0f;
#pragma unroll
                    for (int q = cc; q < NIT; q += CC)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            if (m0 + 2 * (q / CC) + j < Nt)
                                mx = fmaxf(fmaxf(mx, fabsf((float)row[q][j].re)), fabsf((float)row[q][j].im));
                    if constexpr (NG == 1)
                        atomicMax(layer_max + (size_t)(c0 + cc) * K + k, __float_as_uint(mx));
                    else
                        top[(grp * CC + cc) * K + k] = __float_as_uint(mx);
                }
            }
    };
    if (NG > 1 && layer_max) __syncthreads();  // the last transform's split has read its points
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = t0 + i * T8;
        cx<OutT> row[NIT][2];
#pragma unroll
        for (int q = 0; q < NIT; ++q)
#pragma unroll
            for (int j = 0; j < 2; ++j) row[q][j] = held[q][i][j];
        if (i == 0 && t0 == 0) {
            cx<OutT> nyq[NIT][2];
#pragma unroll
            for (int q = 0; q < NIT; ++q)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const cx<OutT> o = row[q][j];
                    nyq[q][j] = {o.im, o.im - o.im};
                    row[q][j] = {o.re, o.re - o.re};
                }
            put_row(M / 2, nyq);
        }
        put_row(k, row);
    }
    if (NG > 1 && layer_max) {
        // the groups' maxima of a layer go out as one
        __syncthreads();
        for (int q = threadIdx.x; q < CC * K; q += NT) {
            uint32_t mx = top[q];
            for (int g = 1; g < NG; ++g) mx = max(mx, top[g * CC * K + q]);
            atomicMax(layer_max + (size_t)c0 * K + q, mx);
        }
    }
}

template <class Q>
__device__ __forceinline__ Q to_q(float v);
template <>
__device__ __forceinline__ __half to_q<__half>(float v) { return __float2half_rn(v); }
template <>
__device__ __forceinline__ __hip_bfloat16 to_q<__hip_bfloat16>(float v) { return __float2bfloat16(v); }
template <>
__device__ __forceinline__ int16_t to_q<int16_t>(float v) {
    // v = value / layer_scale lies in [-32767, 32767] up to rounding of the scale; nearest integer
    return (int16_t)fminf(fmaxf(rintf(v), -32767.0f), 32767.0f);
}
// Largest stored magnitude of each type: the floating types hold value / (layer max) in [-1, 1],
// the fixed-point type value / (layer max / 32767) on the integer grid.
template <class Q>
constexpr float q_full = 1.0f;
template <>
constexpr float q_full<int16_t> = 32767.0f;

// Scale and round the FP32 staging store, which has the final layout, to 16 bits: one streaming pass over the rows of the
// layout: a layer (layout 0), a tranche of a channel (1) or the cells of a bin (2).  A block takes `per` rows of up to 256
// elements each, or a part of a longer row; the blocks go over the groups of rows in gridDim.x (a tranche-major store has
// C Nt rows, which no other grid dimension holds).
template <class Q, int LAYOUT>
__global__ __launch_bounds__(256) void k_quantize(int C, int K, int Nt, int rows, int len, int per, int parts,
                                                  const float2 *__restrict__ st, const uint32_t *__restrict__ mx,
                                                  float *__restrict__ layer_scale, Q *__restrict__ out) {
    const int in_group = per > 1 ? (int)threadIdx.x / len : 0;
    const int e0 = per > 1 ? (int)threadIdx.x - in_group * len : (int)(blockIdx.x % parts) * 256 + (int)threadIdx.x;
    const int step = (int)(gridDim.x / parts) * per;
    if (in_group >= per) return;
    for (int row = (int)(blockIdx.x / parts) * per + in_group; row < rows; row += step) {
        for (int e = e0; e < len; e += parts * 256) {
            const int layer = LAYOUT == 0 ? row : (LAYOUT == 1 ? row / Nt * K + e : e % C * K + row);
            const float m = __uint_as_float(mx[layer]);
            const float inv = m > 0.0f ? q_full<Q> / m : 1.0f;
            // one writer per layer: the first element of its row (its first tranche)
            if (LAYOUT == 0 ? e == 0 : (LAYOUT == 1 ? row % Nt == 0 : e < C))
                layer_scale[layer] = m > 0.0f ? m / q_full<Q> : 1.0f;
            const size_t at = (size_t)row * len + e;
            const float2 v = st[at];
            struct alignas(4) Pair {
                Q re, im;
            };
            reinterpret_cast<Pair *>(out)[at] = Pair{to_q<Q>(v.x * inv), to_q<Q>(v.y * inv)};
        }
    }
}

__global__ void k_weights(int K, int Nt, const double *__restrict__ psd0, const double *__restrict__ mu,
                          const uint8_t *__restrict__ keep, double *__restrict__ inv_asd, double *__restrict__ tw,
                          uint32_t *__restrict__ layer_max, int n_layers) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (layer_max && i < n_layers) layer_max[i] = 0u;
    if (i < K) inv_asd[i] = psd_ok(psd0[i]) ? 1.0 / sqrt(psd0[i]) : 0.0;
    if (i < Nt) tw[i] = keep[i] && psd_ok(mu[i]) ? 1.0 / sqrt(mu[i]) : 0.0;
}

// Template weights for a per-pixel PSD S_m(f_k) (psd[K][Nt]): one block per bin k forms
// S0_k = mean over the tranches of S_m(f_k) (fixed-order partial sums, then a fixed tree),
// u_k = 1/sqrt(S0_k) and rho_mk = sqrt(S0_k / S_m(f_k)); block 0 also writes w_m = keep_m.
__global__ __launch_bounds__(256) void k_weights_tf(int K, int Nt, const double *__restrict__ psd,
                                                   const uint8_t *__restrict__ keep, double *__restrict__ inv_asd,
                                                   double *__restrict__ tw, float *__restrict__ rho,
                                                   uint32_t *__restrict__ layer_max, int C) {
    if (layer_max && (int)threadIdx.x < C) layer_max[threadIdx.x * K + blockIdx.x] = 0u;
    __shared__ double part[256];
    const int k = blockIdx.x;
    const double *row = psd + (size_t)k * Nt;
    double s = 0.0;
    for (int m = threadIdx.x; m < Nt; m += blockDim.x) s += row[m];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
        __syncthreads();
    }
    const double S0 = part[0] / (double)Nt;
    // a layer whose mean PSD is not positive and finite (DC or Nyquist may carry 0 or inf), or a
    // pixel whose own PSD is not, gets weight 0 (u_k or rho_mk), as its pixel is 0
    const bool ok0 = psd_ok(S0);
    if (threadIdx.x == 0) inv_asd[k] = ok0 ? 1.0 / sqrt(S0) : 0.0;
    for (int m = threadIdx.x; m < Nt; m += blockDim.x)
        rho[(size_t)k * Nt + m] = ok0 && psd_ok(row[m]) ? (float)sqrt(S0 / row[m]) : 0.0f;
    if (k == 0)
        for (int m = threadIdx.x; m < Nt; m += blockDim.x) tw[m] = keep[m] ? 1.0 : 0.0;
}

static double window_w2(int M, double alpha) {
    // mean of w^2 of the symmetric Tukey window (host side, FP64)
    if (alpha <= 0.0) return 1.0;
    double width = floor(alpha * (M - 1) / 2.0), s = 0.0;
    for (int n = 0; n < M; ++n) {
        int nn = n < M - 1 - n ? n : M - 1 - n;
        double w = 1.0;
        if ((double)nn <= width) w = 0.5 * (1.0 + cos(kPi * (-1.0 + 2.0 * nn / (alpha * (M - 1)))));
        s += w * w;
    }
    return s / M;
}

template <class R, class XT, class OutT, int M, int CC, int NIT>
static hipError_t run_fft_m(const TransformLaunch &L, double w2, uint32_t *layer_max, hipStream_t st) {
    const int threads = M == 4096 ? 512 : 256, n_grp = threads / (M / 8);
    const int per_block = n_grp * (2 * NIT / CC), n_tiles = (L.Nt + per_block - 1) / per_block;
    const dim3 grid((unsigned)((n_tiles + 7) / 8 * 8), (unsigned)(L.C / CC));
    const int width = L.alpha > 0.0 ? (int)floor(L.alpha * (M - 1) / 2.0) : -1;
    hipLaunchKernelGGL((k_transform<R, XT, OutT, M, CC, NIT>), grid, dim3(threads), 0, st, L, w2, width, layer_max, n_tiles);
    return hipGetLastError();
}

// FP64 arithmetic up to M = 2048, FP32 for M = 4096.
template <class R, class XT, class OutT, int CC, int NIT>
static hipError_t run_fft_t(const TransformLaunch &L, double w2, uint32_t *layer_max, hipStream_t st) {
    if constexpr (sizeof(R) == 4) {
        if (L.M == 4096) return run_fft_m<R, XT, OutT, 4096, CC, NIT>(L, w2, layer_max, st);
    } else {
        switch (L.M) {
            case 64: return run_fft_m<R, XT, OutT, 64, CC, NIT>(L, w2, layer_max, st);
            case 128: return run_fft_m<R, XT, OutT, 128, CC, NIT>(L, w2, layer_max, st);
            case 256: return run_fft_m<R, XT, OutT, 256, CC, NIT>(L, w2, layer_max, st);
            case 512: return run_fft_m<R, XT, OutT, 512, CC, NIT>(L, w2, layer_max, st);
            case 1024: return run_fft_m<R, XT, OutT, 1024, CC, NIT>(L, w2, layer_max, st);
            case 2048: return run_fft_m<R, XT, OutT, 2048, CC, NIT>(L, w2, layer_max, st);
        }
    }
    return hipErrorInvalidValue;
}

// Which transforms a block runs one after the other, NIT of them, until its store.  Blocks of one transform (1, 1) fill the
// chip where a set is short: it is done when its longest block is.  Above that the cells of two channels take both in one
// block, for whole cells per store (M = 512, FP64 store, 500 tranches: 13.2 us a call with one transform a block, 15.0
// with a cell's two; M = 2048, FP32, 3,083: 54.8 against 45.4).  One channel, and the layouts that keep channels apart,
// stay with one transform (one channel, M = 2048, 3,083 tranches, FP32: 32 us against 43 with two pairs), as do FP32 cells
// of three channels (M = 1024, 500: 15 against 20; M = 2048, 3,083: 80 against 77).  From more than 1024 blocks on (768
// run at once) three channels' FP64 cells and 16-bit stores take a cell's channels, or two pairs of a channel: the writes
// of a cell join, and a block sends half the maxima (M = 2048, C = 3, FP64: 500 tranches, 750 blocks, 24 us against 26;
// 3,083: 137 against 124; 16 bits of one channel, 1,500: 37 against 38; 6,144: 96 against 87).  Not for M = 4096, whose
// blocks of 512 threads come one or two to a CU (16 bits of one channel, 3,083 tranches: 85 against 97).
// The 16-byte stores of FP32 A+E cells need a store aligned to them; another one takes the one-channel form, which writes
// any layout 8 or 16 bytes at a time.
template <class R, class XT, class OutT>
static hipError_t run_fft(const TransformLaunch &L, double w2, uint32_t *layer_max, hipStream_t st) {
    const bool cells = L.out_layout == 2 && L.C > 1 && reinterpret_cast<uintptr_t>(L.pix) % 16 == 0;
    const int per = 2 * (sizeof(R) == 8 ? 2048 / L.M : 1);  // tranches of a block of one transform per group
    const int64_t blocks = (int64_t)L.C * ((L.Nt + per - 1) / per);
    if (cells && L.C == 2 && blocks > (sizeof(R) == 8 ? 512 : 256)) return run_fft_t<R, XT, OutT, 2, 2>(L, w2, layer_max, st);
    if constexpr (sizeof(R) == 8) {
        const bool many = blocks > 1024;
        if (many && cells && L.C == 3 && (layer_max || sizeof(OutT) == 8))
            return run_fft_t<R, XT, OutT, 3, 3>(L, w2, layer_max, st);
        if constexpr (sizeof(OutT) == 4)
            if (many && layer_max) return run_fft_t<R, XT, OutT, 1, 2>(L, w2, layer_max, st);
    }
    return run_fft_t<R, XT, OutT, 1, 1>(L, w2, layer_max, st);
}

template <class Q>
static hipError_t run_quantize(const TransformLaunch &L, const uint32_t *mx, hipStream_t st) {
    const int K = L.M / 2 + 1;
    const int rows = L.out_layout == 0 ? L.C * K : (L.out_layout == 1 ? L.C * L.Nt : K);
    const int len = L.out_layout == 0 ? L.Nt : (L.out_layout == 1 ? K : L.Nt * L.C);
    const int per = len < 256 ? 256 / len : 1, parts = (len + 255) / 256 > 8 ? 8 : (len + 255) / 256;
    const int groups = (rows + per - 1) / per, most = 1 << 20;  // blocks of 256 threads: below 2^32 in all
    const dim3 g((unsigned)((groups < most ? groups : most) * parts));
    const float2 *src = reinterpret_cast<const float2 *>(L.ws);
    Q *out = reinterpret_cast<Q *>(L.pix);
    if (L.out_layout == 0)
        hipLaunchKernelGGL((k_quantize<Q, 0>), g, dim3(256), 0, st, L.C, K, L.Nt, rows, len, per, parts, src, mx,
                           L.layer_scale, out);
    else if (L.out_layout == 1)
        hipLaunchKernelGGL((k_quantize<Q, 1>), g, dim3(256), 0, st, L.C, K, L.Nt, rows, len, per, parts, src, mx,
                           L.layer_scale, out);
    else
        hipLaunchKernelGGL((k_quantize<Q, 2>), g, dim3(256), 0, st, L.C, K, L.Nt, rows, len, per, parts, src, mx,
                           L.layer_scale, out);
    return hipGetLastError();
}

hipError_t launch_transform(const TransformLaunch &L, hipStream_t st) {
    const int K = L.M / 2 + 1;
    const double w2 = window_w2(L.M, L.alpha);
    const bool q16 = L.out_dtype == 2 || L.out_dtype == 3 || L.out_dtype == 4;
    uint32_t *mx = nullptr;  // 16-bit stores: the layers' largest |component|, after the staging store in the workspace
    if (q16) {
        size_t st_bytes = sizeof(float) * 2 * (size_t)L.C * K * L.Nt;
        st_bytes = (st_bytes + 255) / 256 * 256;
        mx = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(L.ws) + st_bytes);
    }
    int nw = K > L.Nt ? K : L.Nt;
    if (q16 && L.C * K > nw) nw = L.C * K;
    if (L.psd_tf)
        hipLaunchKernelGGL(k_weights_tf, dim3(K), dim3(256), 0, st, K, L.Nt, L.psd_tf, L.keep, L.inv_asd,
                           L.tranche_w, L.rho, mx, L.C);
    else
        hipLaunchKernelGGL(k_weights, dim3((nw + 255) / 256), dim3(256), 0, st, K, L.Nt, L.psd0, L.mu, L.keep,
                           L.inv_asd, L.tranche_w, mx, L.C * K);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // The FFT runs in FP64 for M <= 2048: whitening divides by sqrt(S0), which near the TDI nulls is ~1e5 smaller
    // than at low frequency, so FP32 FFT rounding (set by the red low-frequency power) would be amplified there.
    const bool big = L.M > 2048;
    if (q16) {
        // FP32 staging in the store's layout with the layers' maxima, then per-layer scale and quantisation
        TransformLaunch Lw = L;
        Lw.pix = L.ws;
        if (L.x_dtype == 0)
            e = big ? run_fft<float, double, float>(Lw, w2, mx, st) : run_fft<double, double, float>(Lw, w2, mx, st);
        else
            e = big ? run_fft<float, float, float>(Lw, w2, mx, st) : run_fft<double, float, float>(Lw, w2, mx, st);
        if (e != hipSuccess) return e;
        if (L.out_dtype == 4) return run_quantize<int16_t>(L, mx, st);
        return L.out_dtype == 3 ? run_quantize<__half>(L, mx, st) : run_quantize<__hip_bfloat16>(L, mx, st);
    }
    if (L.out_dtype == 0) return big ? hipErrorInvalidValue : run_fft<double, double, double>(L, w2, nullptr, st);
    if (L.x_dtype == 0)
        return big ? run_fft<float, double, float>(L, w2, nullptr, st) : run_fft<double, double, float>(L, w2, nullptr, st);
    return big ? run_fft<float, float, float>(L, w2, nullptr, st) : run_fft<double, float, float>(L, w2, nullptr, st);
}

}  // namespace tfsc
