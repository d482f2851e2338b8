// Internal launch descriptors shared by the C ABI layer and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tfsc {

// Layout of the statistic workspace's tail: the WAVE schedule's uint32 work counter at
// +0, the FP64 weight scale at +kTailScale.
constexpr int kTailScale = 64;

// Geometry tables in the statistic workspace: 18 FP64 rows of Nt values, then (256-byte
// aligned) the FP32 copy of the 9 arm-vector rows.
inline size_t geo64_bytes(int Nt) { return (sizeof(double) * 18 * (size_t)Nt + 255) / 256 * 256; }
inline size_t geo32_bytes(int Nt) { return (sizeof(float) * 9 * (size_t)Nt + 255) / 256 * 256; }
inline float *geo32_of(const double *geo, int Nt) {
    return reinterpret_cast<float *>(reinterpret_cast<char *>(const_cast<double *>(geo)) + geo64_bytes(Nt));
}

struct LayoutLaunch {
    int64_t n;
    const double *mc, *eta, *f0, *ct, *ci;
    const double *ln_mc;  // the bank given in ln Mc (mc unused), else NULL
    int nseg_fixed;
    int32_t *nseg;
    int64_t *seg_offset;
    int64_t *block_sums;  // workspace, ceil(n / 256) entries
};

// Few templates: each template's chunks of 64 tranches are shared out in units of `chunks` of them, one unit per
// wave (k_stat_split, k_stat_chunk, k_vjp_units), and a finishing kernel joins the units.  units = 0: not split.
constexpr int kSplitRun = 64;    // consecutive templates on one XCD (see run_item)
constexpr int kRecDoubles = 32;  // doubles of a template record
// Most whole templates in runs, one wave each: a grid holds fewer than 2^32 threads, 67 million waves.  Larger banks in a
// processing order take the persistent grid and its work counter.
constexpr int64_t kRunsMost = 1 << 25;
// Waves per block of these kernels, whatever block_waves says: a block stages the weight table for its waves' templates
// only, not for all that a persistent wave goes through (1M templates, two years: 2 waves 131.8 ms, 4 waves 127.1).
constexpr int kRunWaves = 4;
// Runs are for FP32 and FP64 stores.  A 16-bit store's blocks would stage its layer scales as well, and its rows are half
// as wide: 1M templates, two years, counter against runs: FP32 136.0 / 130.5 ms, but FP16 142.3 / 146.7, BF16 140.0 /
// 143.7, I16 144.3 / 147.6; 4M templates x 16 realisations in pairs: FP32 5.49 / 5.18 s, I16 5.81 / 6.12.
inline bool in_runs(int64_t n, int pix_dtype) { return n <= kRunsMost && pix_dtype <= 1; }
struct SplitUnit {
    double zr, zi, N;  // sums of the segment that goes on into the next unit
    int code, m_end;   // flag and tranche of the track's end, if it ends in the unit (m_end: else the unit's end)
    int n_act, any;    // tranches with work; whether a segment closed in the unit has N > 0
};
struct SplitWs {
    int n_chunks, chunks, units;  // chunks per template, per unit; units per template
    double *rec;                  // [n][kRecDoubles]
    void *head;                   // [n][n_chunks][3] of R: chunk sums of a segment that began in an earlier unit
    SplitUnit *unit;              // [n][units]
};

// Chunks per unit and units per template for n templates of Nt tranches on n_waves waves, if there are at most `most`
// templates a wave (units = 0: whole templates).
// Few templates leave waves idle, and up to some twenty a wave the units of a window, run together, also save reads behind
// L2 (65,536 templates: 2.9 GB instead of 21.9).  Two-year grid, A+E, FP32, whole (one counter / runs) against split, us:
// 1024: 645 / 537 / 270; 4099: 963 / 939 / 821; 16,000: 2831 / 2893 / 2572; 65,536: 10,035 / 9680 / 9290 (A+E+T 14,276 /
// 12,594 / 11,067); 262,144: 36,703 / 34,960 / 34,740, where the records and sums would take 430 MB.  A wave gets up to
// eight units, at least one chunk and at most 16 each: at 16,000 templates 12 chunks took 2572, 24 2592, 48 2767 us.
inline void split_shape(int64_t n, int Nt, int64_t n_waves, SplitWs &s, int most = 20) {
    s.n_chunks = (Nt + 63) / 64;
    s.chunks = s.units = 0;
    if (n < 1 || n > most * n_waves || s.n_chunks < 2) return;
    const int64_t per = n * s.n_chunks / (8 * n_waves);
    s.chunks = (int)(per < 1 ? 1 : (per > 16 ? 16 : per));
    s.units = (s.n_chunks + s.chunks - 1) / s.chunks;
    if (s.units < 2) s.units = 0;
}

struct StatLaunch {
    int M, Nt, C;
    double dt;
    int pix_dtype;  // tfsc_dtype
    int layout;     // tfsc_layout
    int precision;  // 0 FP64, 1 FP32
    int schedule;   // 0 THREAD, 1 WAVE
    int n_groups, block_waves;
    const void *pix;
    const float *layer_scale;
    const double *inv_asd, *tranche_w, *geo;
    const float *rho;       // [K][Nt] per-pixel weight factor, NULL for a separable PSD
    const double *links;    // [6][Nt] link light times (unequal arms), NULL for equal arms
    int tdi2;               // with links: second-generation TDI combinations
    const double *u_scale;  // device scalar written by launch_prepare
    int64_t n;
    const double *mc, *eta, *f0, *ct, *phi, *psi, *ci;
    const double *ln_mc;  // the bank given in ln Mc: the entry point fills mc (a workspace table) from it
    const int32_t *nseg;
    const int64_t *seg_offset;
    const int32_t *order;
    double *seg_terms, *stat, *seg_zn;
    int32_t *flags;
    int32_t *n_active;
    uint32_t *counter;
    // several realisations (launch_statistic_multi only)
    int n_real;
    int64_t real_stride;  // bytes between realisation stores
    int64_t seg_stride;   // elements between realisation planes of seg_terms
    int multi_group;      // realisations sharing one pass over the bank: 1, 2, 4 or 8
    SplitWs split;
    bool from_counter;  // whole templates from the work counter also with a processing order
};

constexpr int kMultiGroupDefault = 8;
constexpr int kMaxRealisations = 64;

struct VjpLaunch {
    StatLaunch s;  // seg_terms / stat / flags unused
    const double *seg_zn;
    const double *g_stat, *g_seg;
    double *g_params;
};

// Processing order: templates grouped by the frequency bin of f0, then by ln Mc in kOrderMcClasses classes
// over [kOrderLnMcLo, kOrderLnMcHi) (clamped at the ends).
constexpr int kOrderMcClasses = 256;
constexpr double kOrderLnMcLo = -0.6931471805599453;  // ln 0.5
constexpr double kOrderLnMcHi = 6.214608098422191;    // ln 500

struct OrderLaunch {
    int M;
    double dt;
    int64_t n;
    const double *mc, *eta, *f0, *ct, *ci;
    const double *ln_mc;
    int32_t *order;
    uint32_t *ws;  // 2 nb + ceil(nb / 1024) counters, nb = (M/2 + 1) kOrderMcClasses + 1
};

struct FollowLaunch {
    int Nt;
    double dT;
    int64_t n;
    double *mc, *f0, *ct, *phi, *psi;  // updated in place
    double *ln_mc;                     // updated in place instead of mc when the bank is given in ln Mc
    const double *eta, *ci;
    const int32_t *nseg;
    const double *stat, *g_params;
    double *state;  // [n][16]
    double lr_scale;
    int step;
};

struct TransformLaunch {
    int M, Nt, C;
    double dt, alpha;
    const void *x;
    int x_dtype;
    const double *psd0, *mu;
    const double *psd_tf;  // [K][Nt] S_m(f_k) for a general per-pixel PSD (then psd0, mu unused), else NULL
    const uint8_t *keep;
    int out_dtype, out_layout;
    void *pix;
    float *layer_scale;
    double *inv_asd, *tranche_w;
    float *rho;  // written when psd_tf is set
    void *ws;  // FP32 staging for 16-bit outputs
};

hipError_t launch_layout(const LayoutLaunch &L, hipStream_t st);
// What the statistic and VJP kernels read besides the caller's arrays, in one launch: the geometry tables (of the
// analytic orbit or the caller's), the weight scale, the zeroed work counter, the chirp masses of a bank given in
// ln Mc and, for split templates, their records (precision: that of the sky vectors).
hipError_t launch_prepare(const StatLaunch &L, const double *orbit, hipStream_t st);
hipError_t launch_orbit_positions(int Nt, double dT, double *out, hipStream_t st);
hipError_t launch_link_lengths(int Nt, double dT, const double *orbit, double *out, hipStream_t st);
hipError_t launch_statistic_interleaved(const StatLaunch &L, hipStream_t st);
hipError_t launch_interleave(int64_t cells, int C, int K, int NR, int r, int elem_bytes, const void *src,
                             const float *src_scale, void *dst, float *dst_scale, hipStream_t st);
hipError_t launch_statistic(const StatLaunch &L, hipStream_t st);
hipError_t launch_statistic_split(const StatLaunch &L, hipStream_t st);
hipError_t launch_statistic_accurate(const StatLaunch &L, hipStream_t st);
hipError_t launch_statistic_links(const StatLaunch &L, hipStream_t st);
constexpr int kMaxHarmonics = 4;
hipError_t launch_statistic_harmonics(const StatLaunch &L, int n_harm, const int *harm, const double *amp,
                                      hipStream_t st);
hipError_t launch_statistic_multi(const StatLaunch &L, hipStream_t st);
hipError_t launch_vjp(const VjpLaunch &L, hipStream_t st);
hipError_t launch_transform(const TransformLaunch &L, hipStream_t st);
hipError_t launch_follow_step(const FollowLaunch &L, hipStream_t st);
hipError_t launch_order(const OrderLaunch &L, hipStream_t st);
hipError_t launch_tile_max(const double *stat, const int32_t *tile, int64_t n, int32_t n_tiles, double *tile_max,
                           int64_t *tile_arg, hipStream_t st);
hipError_t launch_track(int64_t n, int M, int Nt, double dt, const double *mc, const double *ln_mc, const double *eta,
                        const double *f0, const double *ct, const double *ci, double *out, hipStream_t st);

}  // namespace tfsc
