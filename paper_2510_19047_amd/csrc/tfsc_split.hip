// The WAVE schedule with one item per wave and no work counter.
//
// k_stat_runs: a whole template, in runs of the processing order per XCD (run_item).  Bound by vector-ALU issue like
// k_stat_wave; what it saves is reads behind L2 (1,000,020 templates, A+E: 134.8 -> 130.4 ms).  A bank without a
// processing order keeps the counter, which evens out templates of any length.
//
// k_stat_split: a unit of a template's chunks, for a few thousand templates and fewer.  Every chunk is evaluated as in
// k_stat_wave.  A unit closes the segments that lie inside it; of a segment across units the first keeps its running
// sums (SplitUnit) and the later ones each chunk's (head), and k_stat_finish adds them in the order of k_stat_wave: the
// results are the same bits.
//
// Bound: latency for few templates (20 of 96 chunks: 36 us a call with its three launches, whole templates 547), vector-
// ALU issue from a few thousand on.  The rule and its figures: split_shape.
#include "tfsc_stat_common.hpp"

namespace tfsc {

template <int C, class R, class PixT, int LAYOUT, bool RHO>
__global__ __launch_bounds__(256, 4) void k_stat_split(StatArgs a) {
    stat_wave_body<C, R, PixT, LAYOUT, RHO, kFresnelPaper, false, kUnits>(a);
}

// One chunk per wave: two waves per SIMD, whose registers hold all the pixels of a chunk, so that they cost one latency
// instead of seven (the rows lie a page or more apart).
template <int C, class R, class PixT, int LAYOUT, bool RHO>
__global__ __launch_bounds__(256, 2) void k_stat_chunk(StatArgs a) {
    stat_wave_body<C, R, PixT, LAYOUT, RHO, kFresnelPaper, false, kChunk>(a);
}

// Whole templates of a bank with a processing order.
template <int C, class R, class PixT, int LAYOUT, bool RHO>
__global__ __launch_bounds__(256, 4) void k_stat_runs(StatArgs a) {
    stat_wave_body<C, R, PixT, LAYOUT, RHO, kFresnelPaper, false, kRuns>(a);
}

// Join the units of a template: one wave per template, a lane per segment.
template <class R>
__global__ __launch_bounds__(256) void k_stat_finish(StatArgs a) {
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= a.n) return;
    const int64_t i = a.order ? (int64_t)a.order[t] : t;
    if (i < 0 || i >= a.n) return;  // malformed processing order: skip rather than fault
    const int ns = a.nseg[i], units = a.split.units, unit_len = a.split.chunks * 64;
    const int64_t off = a.seg_offset[i];
    const bool valid = a.split.rec[i * kRecDoubles + kRecValid] != 0.0;
    const SplitUnit *un = a.split.unit + i * units;
    // the unit in which the track ends (units: in none), its flag and tranche; units after it do not count
    int ue = units, code = 0, m_end = valid ? a.Nt : 0, n_act = 0, any = 0;
    for (int u0 = 0; valid && u0 < units && ue == units; u0 += 64) {
        const int u = u0 + lane, ul = min(u, units - 1);
        const int uc = un[ul].code, um = un[ul].m_end, ua = un[ul].n_act, us = un[ul].any;
        const uint64_t ends = __ballot(u < units && uc != 0);
        if (ends) {
            const int l = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)ends) - 1);
            ue = u0 + l;
            code = __builtin_amdgcn_readlane(uc, l);
            m_end = __builtin_amdgcn_readlane(um, l);
        }
        const bool counts = u < units && u <= ue;
        n_act += counts ? ua : 0;
        any |= counts ? us : 0;
    }
    for (int o = 32; o > 0; o >>= 1) n_act += __shfl_xor(n_act, o, 64);
    const int last_chunk = m_end >> 6;  // a track that ends at a chunk's first tranche adds nothing there
    double total = 0.0;
    for (int s0 = 0; s0 < ns; s0 += 64) {
        const int s = s0 + lane;
        double v = 0.0;
        if (s < ns) {
            const int lo = (int)(((int64_t)s * a.Nt + ns - 1) / ns), hi = (int)(((int64_t)(s + 1) * a.Nt + ns - 1) / ns);
            const int ua = lo / unit_len, ub = hi > lo ? (hi - 1) / unit_len : ua;
            const bool counts = valid && hi > lo && ua <= ue && ua < units;
            if (counts && ua == ub) {
                v = a.seg_terms[off + s];
            } else {
                double zr = 0.0, zi = 0.0, N = 0.0;
                if (counts) {
                    zr = un[ua].zr;
                    zi = un[ua].zi;
                    N = un[ua].N;
                    const int c1 = min((hi - 1) >> 6, m_end & 63 ? last_chunk : last_chunk - 1);
                    const R *head = reinterpret_cast<const R *>(a.split.head) + i * a.split.n_chunks * 3;
                    // eight chunks' loads are in flight together; the sums keep their order
                    for (int c = (ua + 1) * a.split.chunks; c <= c1; c += 8) {
                        R h[8][3];
#pragma unroll
                        for (int q = 0; q < 8; ++q)
#pragma unroll
                            for (int e = 0; e < 3; ++e) h[q][e] = head[3 * min(c + q, c1) + e];
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            if (c + q <= c1) {
                                zr += (double)h[q][0];
                                zi += (double)h[q][1];
                                N += (double)h[q][2];
                            }
                    }
                }
                v = N > 0.0 ? 2.0 * (zr * zr + zi * zi) / N : 0.0;
                any |= N > 0.0;
                a.seg_terms[off + s] = v;
                if (a.seg_zn) {
                    a.seg_zn[3 * (off + s) + 0] = zr;
                    a.seg_zn[3 * (off + s) + 1] = zi;
                    a.seg_zn[3 * (off + s) + 2] = N;
                }
            }
        }
        const int cnt = min(64, ns - s0);
        for (int l = 0; l < cnt; ++l) total += lane_double(v, l);
    }
    const bool some = __ballot(any != 0) != 0;
    if (lane == 0) {
        int flag = valid ? code : kFlagInvalid;
        if (valid && m_end == 0) flag |= kFlagEmpty;
        if (valid && !some && m_end > 0) flag |= kFlagAllExcluded;
        a.stat[i] = total;
        a.flags[i] = flag;
        if (a.n_active) a.n_active[i] = n_act;
    }
}

template <int C, class R, class PixT, int LAYOUT, bool RHO>
static hipError_t launch_split_l(const StatArgs &a, int block_waves, hipStream_t st) {
    const size_t KP = (size_t)a.K + 2 * kHalfBins;
    const size_t shmem = sizeof(R) * KP + (PixTraits<PixT>::scaled ? sizeof(float) * C * KP : 0);
    const dim3 block(64 * block_waves);
    if (a.split.units) {
        const dim3 grid(run_groups(a.n, block_waves, a.split.units));
        // Up to 8192 chunks (two rounds of four waves per SIMD) latency counts: 257 templates of 20 chunks 28.7 us a call
        // against 30.5 with k_stat_split, 20 of 96 in FP64 45 against 61; from 10,000 chunks on both take the same.
        if (a.split.chunks == 1 && a.n * a.split.units <= 8192)
            hipLaunchKernelGGL((k_stat_chunk<C, R, PixT, LAYOUT, RHO>), grid, block, shmem, st, a);
        else
            hipLaunchKernelGGL((k_stat_split<C, R, PixT, LAYOUT, RHO>), grid, block, shmem, st, a);
        hipLaunchKernelGGL(k_stat_finish<R>, dim3((unsigned)((a.n + 3) / 4)), dim3(256), 0, st, a);
    } else {
        hipLaunchKernelGGL((k_stat_runs<C, R, PixT, LAYOUT, RHO>), dim3(run_groups(a.n, block_waves, 1)), block, shmem, st, a);
    }
    return hipGetLastError();
}

template <int C, class R, class PixT>
static hipError_t launch_split_t(const StatLaunch &L, const StatArgs &a, hipStream_t st) {
    const int w = kRunWaves;
    if constexpr (!PixTraits<PixT>::scaled) {
        if (a.rho)
            return L.layout == 2 ? launch_split_l<C, R, PixT, 2, true>(a, w, st)
                                 : launch_split_l<C, R, PixT, 0, true>(a, w, st);
    } else {
        if (a.rho) return hipErrorInvalidValue;
    }
    return L.layout == 2 ? launch_split_l<C, R, PixT, 2, false>(a, w, st)
                         : launch_split_l<C, R, PixT, 0, false>(a, w, st);
}

template <int C>
static hipError_t launch_split_c(const StatLaunch &L, const StatArgs &a, hipStream_t st) {
    if (L.precision == 0) {
        if (L.pix_dtype == 0) return launch_split_t<C, double, double>(L, a, st);
        return L.pix_dtype == 1 ? launch_split_t<C, double, float>(L, a, st) : hipErrorInvalidValue;
    }
    switch (L.pix_dtype) {
        case 1: return launch_split_t<C, float, float>(L, a, st);
        case 2: return launch_split_t<C, float, __hip_bfloat16>(L, a, st);
        case 3: return launch_split_t<C, float, __half>(L, a, st);
        case 4: return launch_split_t<C, float, int16_t>(L, a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_statistic_split(const StatLaunch &L, hipStream_t st) {
    const StatArgs a = make_args(L);
    if (L.C == 1) return launch_split_c<1>(L, a, st);
    return L.C == 3 ? launch_split_c<3>(L, a, st) : launch_split_c<2>(L, a, st);
}

}  // namespace tfsc
