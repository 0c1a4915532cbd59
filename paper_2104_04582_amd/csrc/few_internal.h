// Internal declarations shared by the host runtime (few_api.cpp,
// host_core.cpp) and the gfx950 kernels (kernels.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace few {

constexpr int kMaxKnots = 1024;       // phase-solve LDS: eight binary64 arrays of this length (64 KiB)
constexpr int kMaxL = 30;             // Wigner-d sum stays well conditioned in binary64
constexpr int kMaxAbsN = 1000;
constexpr int kMaxAbsK = 30;          // polar index of generic-Kerr modes
constexpr int kWave = 64;
constexpr int kMaxGap = 4;            // zero terms filled inside one segment
#ifndef FEW_SEG_UNROLL
#define FEW_SEG_UNROLL 2
#endif
#ifndef FEW_CHUNK_TERMS
#define FEW_CHUNK_TERMS 1024
#endif
// Amplitude series per fit workgroup (lane = series; the four waves take a
// quarter of the rows each, or wave 0 all of them on larger grids).
constexpr int kFitSeriesPerBlock = 64;
// Grids of at most this many knots keep each lane's knot values in registers
// (a quarter of the rows per wave) and factor the grid with one wave's scan;
// larger grids stream knot values with one lane per series (45 us at 137 knots,
// where the wave form takes 25).
constexpr int kFitStageKnots = 192;
constexpr int kChunkTerms = FEW_CHUNK_TERMS;   // terms staged in LDS at once (binary32: 32 B each)

// Samples per lane in one wave tile of the summation kernel.
#ifndef FEW_SL_F32
#define FEW_SL_F32 4
#endif
#ifndef FEW_SL_F64
#define FEW_SL_F64 2
#endif
constexpr int kSamplesPerLaneF32 = FEW_SL_F32;
constexpr int kSamplesPerLaneF64 = FEW_SL_F64;

// Samples per tile: a workgroup of 4 waves (binary32) or one wave (binary64).
inline int tile_samples(bool fp32) {
    return fp32 ? 4 * kWave * kSamplesPerLaneF32 : kWave * kSamplesPerLaneF64;
}

// Binary32: the last samples of a single-request launch are cut into short
// tiles (half the samples per lane) so the end of the launch drains evenly.
// The short-tile region holds FEW_SHORT_QUARTERS / 4 of one round of long tiles
// over the resident workgroups.  (Binary64 tiles read their coefficients with
// scalar loads, which short tiles amortise poorly: long tiles only.)
#ifndef FEW_SL_SHORT
#define FEW_SL_SHORT 2
#endif
#ifndef FEW_SHORT_QUARTERS
#define FEW_SHORT_QUARTERS 2
#endif
constexpr int kSamplesPerLaneShort = FEW_SL_SHORT;
inline int short_tile_samples(bool fp32) {
    return fp32 ? 4 * kWave * kSamplesPerLaneShort : kWave * kSamplesPerLaneF64;
}

// Binary32 sums run over four term groups (consecutive segments with about a
// quarter of the terms each): every sample's compensated sum restarts, and its
// harmonic seed is recomputed, at each group's first segment, and the four
// group values are added in group order.  A term-split tile uses that: its four
// waves take the same 64 x kSamplesPerLaneF32 samples, one group each, staging
// their group kSplitTerms terms at a time in their own quarter of the LDS
// buffer.  Requests whose segments all fit a quarter cut their short tiles this
// way (the end of a launch then drains in pieces a quarter as long); others
// keep the 2-sample short tiles.  Either way a sample gets the same rounded
// operations.
constexpr int kTermGroups = 4;
constexpr int kSplitTerms = FEW_CHUNK_TERMS / kTermGroups;
// Requests with fewer folded terms form one group (reseeding at group starts
// costs a few sincos per sample and tile, which short sums do not repay) and
// keep the 2-sample short tiles.
constexpr int kGroupMinTerms = 1024;
inline int split_tile_samples() { return kWave * kSamplesPerLaneF32; }

// Matrix-core summation (binary32 output).  Per knot interval the folded sum
// is a contraction: with rows = the distinct signed m values (a complex row
// each, as a real re/im pair) and columns n,
//   h = sum_m e^{-i m Phi_phi} sum_p u^p sum_n C^p_{m,n} f^n,
// f = e^{-i Phi_r}.  For each p the sum over n is the product of the
// coefficient matrix [rows x (n, re/im)] with the matrix of powers f^n over
// the samples, run on v_mfma_f32_16x16x32_f16 with both operands split into
// fp16 hi + lo parts (hi*hi + hi*lo + lo*hi, about 22 significant bits) and
// fp32 accumulation; the sum over p is a Horner recurrence in u on the
// accumulators.  Only the powers f^a, a = |n| >= 0, are formed: a column of
// n < 0 multiplies conj(f^|n|), and the conjugation lives in the coefficient
// matrix, so the terms n and -n meet the same operand fragment and their
// coefficient rows are added into one (the product is linear in them).
// Fixed shape: kMfMT tiles of 16 matrix rows (8 signed m each), kMfT steps of
// 32 columns (16 values of |n| each; |n| < 16 kMfT), kMfNT tiles of 16
// samples (one sample per lane) per wave and round, kMfWaves waves per
// workgroup, one workgroup per compute unit: two waves per SIMD, so that a
// wave can keep a block's operands (72 registers) and its sums in the 256
// registers it then has (with 12 waves and 168 registers the block operands
// spill: 426 against 388 us on 12.6 million samples).  A request takes this
// path when its term layout fits the shape and is long enough to repay it.
#ifndef FEW_MF_NT
#define FEW_MF_NT 4
#endif
#ifndef FEW_MF_WAVES
#define FEW_MF_WAVES 8
#endif
constexpr int kMfMT = 3;
constexpr int kMfT = 2;
constexpr int kMfNT = FEW_MF_NT;
constexpr int kMfWaves = FEW_MF_WAVES;
constexpr int kMfRows = 8 * kMfMT;          // signed m values per request
constexpr int kMfA = 16 * kMfT;             // |n| < kMfA
constexpr int kMfRound = kMfWaves * kMfNT * 16;   // samples per workgroup round (static tables)
// operand values of one interval, binary32: [mt][p 4][t][lane 64][8]
constexpr size_t kMfIntervalFloats = (size_t)kMfMT * 4 * kMfT * 64 * 8;
// What the summation needs to know of an interval's values: the scale of each
// pair of signed m rows, and an upper bound of the largest |scaled value| of
// every fragment (the leading 16 bits of a binary32 value, rounded up).
struct MfInfo {
    float scale[kMfRows / 2];
    unsigned short top[kMfMT * 4 * kMfT];   // [mt][p][t]
};
static_assert(sizeof(MfInfo) == 96, "4-byte granularity, no padding");
// From this many folded terms on a binary32 list is folded straight into the
// operand table, whatever its length; shorter lists go through the fold table, and
// mf_terms_path decides.
constexpr int kMfMinTerms = 480;

// ---------------------------------------------------------------------------
// Device-side job descriptors.  Pointers are device addresses in the plan
// arena (or caller memory for inputs/outputs).
// ---------------------------------------------------------------------------

// Spline stage for one request.
struct FitJob {
    const double *t;        // [K] knot times
    const double *phi_phi;  // [K]
    const double *phi_r;    // [K]
    const double *phi_theta;  // [K] (generic Kerr) or null
    const double *amp;      // [K][M][2]
    double *pcoef;          // [K-1][n_ph][4][2] double-double phase cubics
    double *acoef;          // amplitude cubics: [K-1][M][4][2], or [K-1][4][2M] if pmajor
    int acoef_pmajor;       // 1: coefficient p of series q = 2k + re/im at [i][p][q]
                            // (matrix-core requests: read by fold_pack), 0: mode-major
    int K, M;
    int n_ph;               // phases: Phi_phi, Phi_r (, Phi_theta)
    int amp_blocks;         // blocks covering the 2M amplitude series (after n_ph phase blocks)
    // Upload carried by this launch (single-request fits): up_bytes bytes
    // from the pinned, host-coherent staging slot up_src to the request's
    // arena block up_dst, copied by the amplitude workgroups' waves that do
    // not sweep; t then points at the knots in the staging slot.  0: none.
    const uint4 *up_src;
    uint4 *up_dst;
    long long up_bytes;
};

constexpr int kMaxPhases = 3;

// Knot times of a single-request fit of at most kFitStageKnots knots, passed
// by value as a launch argument.
template <int R>
struct FitKnots {
    double t[R > 0 ? R * kWave : 1];
};

// Fold + interval bookkeeping for one request.
struct PrepJob {
    const double *t;
    const double *acoef;
    const int *term_ptr;    // [n_terms + 1]
    const int2 *term_src;   // [n_src]: (mode, l | m << 8 | mirror << 16)
    double2 *ybuf;          // [n_src] harmonic weight of each contributor
    void *table;            // [K-1][n_terms][8] binary32 or binary64, terms in reverse order
    long long *starts;      // [K]
    int *tile_pref;         // [parts][K]: tiles before each interval, per part
    double theta, phi, scale, t_start, dt;
    double scale_im;        // imaginary part of a complex overall factor (0: real scale)
    long long n;
    long long short_len;    // samples at the end of each part cut into short tiles
    int parts;              // contiguous sample parts (one per XCD) or 1
    int K, M, n_terms, n_src;
    int tile;               // samples per tile
    int short_tile;         // samples per short tile
    int fold_terms;         // consecutive terms folded by one workgroup
    int fold_blocks;        // term groups of the fold
    // matrix-core path: the fold writes the operand table and its scales
    const int4 *segs;       // [n_segs]
    const int2 *mrows;      // [n_mrows + 1]: (m, first segment) per row, sentinel (0, n_segs)
    float *mtab;            // [K-1][kMfIntervalFloats]: values of a row pair times 2^-E
    MfInfo *minfo;          // [K-1]
    int n_mrows, n_min, n_segs;
    int l_max;              // largest listed l
};

// Split of the matrix-core summation between the eight XCDs: the XCDs of
// one device run at different clocks under load, so a store launch may give
// XCD x a share of the samples proportional to a weight w[x], and each of its
// workgroups then reports its time (with the launch's tag) in pinned host
// memory, from which the host forms the weights of later launches.  Only
// performance depends on it: any weights give a split that covers every
// sample once.
constexpr int kMfBalanceWG = 256;       // workgroups a report array holds
constexpr int kMfTagShift = 40;         // report word: tag << 40 | s_memrealtime ticks

// Summation stage for one request.
struct SumJob {
    const double *t;
    const double *pcoef;    // [K-1][n_ph][4][2]
    const void *table;
    const int4 *segs;       // [n_segs]: (m + 256 k, n_lo, length, first term)
    const int *chunks;      // [n_chunks + 1]: first segment of each LDS chunk
    const long long *starts;
    const int *tile_pref;
    void *out;              // [n] complex output (store launches)
    const void *data;       // [n] complex data d (inner-product launches)
    double2 *partial;       // per tile slot: (sum Re(conj(d) h), sum |h|^2)
    double t_start, dt;
    long long n;
    long long short_len;    // samples at the end of each part cut into short tiles
    int parts;              // contiguous sample parts (one per XCD) or 1
    int K, n_terms, n_segs, n_chunks;
    int n_ph;               // phases in pcoef (3: generic Kerr, Phi_theta last)
    int wave_base;          // first global tile slot of this job (batched launch)
    int grp[kTermGroups - 1];   // first segment of term groups 1..3 (binary32)
    int split;              // short tiles are term-split tiles
    // matrix-core path: rows of consecutive signed m (mtab); sums from the
    // fold table, 10 row tiles + steps needed (0: not); their lowest signed m
    signed char mf_consec, mf_terms, mf_m0;
    signed char mf_ns;      // steps of two |n| (binary64)
    const float *mtab;      // [K-1][kMfIntervalFloats] operand values
    const MfInfo *minfo;    // [K-1]
    const int2 *mrows;      // [n_mrows + 1]
    int n_mrows, n_min;
    long long sample_base;  // first sample of this job in a batched launch's range
    // matrix-core store launches: XCD split weights (all 0: equal split), and
    // where each workgroup reports (tag << kMfTagShift | its time), or nullptr
    float bw[8];
    unsigned long long *btime;
    unsigned btag;
    signed char mf_k0;      // sums from the fold table: polar indices k0 ..
    unsigned char mf_nk;    // .. k0 + nk - 1
    signed char mf_f64;     // the fold table is binary64
};

// Launchers (kernels.hip).  All enqueue on `stream` and return the HIP status.
// Binary32 summation workgroups resident at once on the current device, for
// the two-phase (Schwarzschild) or three-phase (generic Kerr) kernel.
int sum_resident_workgroups(int n_ph);
hipError_t launch_upload(const void *src, void *dst, size_t bytes, hipStream_t stream);
// acoef [K-1][4][2M] -> dst [K-1][M][4][2] (the few_spline_coefs layout)
hipError_t launch_acoef_export(const double *src, double *dst, int K, int M,
                               hipStream_t stream);
// t_host: the K knot times in host memory (copied into the launch's arguments
// when K <= kFitStageKnots).
hipError_t launch_fit(const FitJob &job, const double *t_host, hipStream_t stream);
hipError_t launch_fit_batch(const FitJob *jobs_dev, int n_jobs, int max_blocks, int max_K,
                            hipStream_t stream);
hipError_t launch_prepare(const PrepJob &job, bool fp32, hipStream_t stream);
hipError_t launch_prepare_batch(const PrepJob *jobs_dev, int n_jobs, int max_fold_blocks,
                                bool fp32, hipStream_t stream);
hipError_t launch_sum(const SumJob &job, int slots, bool fp32, hipStream_t stream);
// Inner-product variant of launch_sum: instead of storing h, every tile slot
// writes its partial sums to job.partial (inner_slots(...) entries), then one
// workgroup adds them in a fixed order into out2 = 2 dt (<d|h> sum, <h|h> sum).
hipError_t launch_sum_inner(const SumJob &job, int slots, bool fp32, double two_dt,
                            double *out2, hipStream_t stream);
long long inner_slots(int parts, int slots, bool fp32);
// Allocation-free inner product: partial sums go to a static device array of
// kNoAllocSlots entries (2 MiB, one copy per GPU).  noalloc_scratch() returns
// its device address on `device`, which must be the current device; it looks
// the address up (hipGetSymbolAddress) on the first call per device.
constexpr long long kNoAllocSlots = 131072;
constexpr int kMaxDevices = 64;
hipError_t noalloc_scratch(int device, double2 **out);
hipError_t launch_sum_batch(const SumJob *jobs_dev, int n_jobs, int total_wave_slots,
                            bool fp32, bool persistent, unsigned *counter_dev,
                            hipStream_t stream);
hipError_t launch_zero_u32(unsigned *p, int n, hipStream_t stream);
// Matrix-core path: the prepare step (interval starts, fold and the
// operand table, one request or n_jobs of them with max_K knots at most), and
// the summation (every workgroup takes an equal contiguous share of the
// samples; n_wg workgroups; with INNER each writes its partial sums to
// job.partial[b] and one more launch adds them into out2 = two_dt * sums).
hipError_t launch_fold_pack(const PrepJob &job, hipStream_t stream);
hipError_t launch_fold_pack_batch(const PrepJob *jobs_dev, int n_jobs, int max_K,
                                  hipStream_t stream);
int mfma_workgroups();
hipError_t launch_sum_mfma(const SumJob &job, int n_wg, hipStream_t stream);
hipError_t launch_sum_mfma_inner(const SumJob &job, int n_wg, double two_dt, double *out2,
                                 hipStream_t stream);
hipError_t launch_sum_mfma_batch(const SumJob *jobs_dev, int n_jobs, long long total,
                                 bool consec, int n_wg, hipStream_t stream);
hipError_t launch_sum_mfma_terms_batch(const SumJob *jobs_dev, int n_jobs, long long total,
                                       bool f64, int n_wg, hipStream_t stream);
hipError_t launch_select(const double *amp, int K, int M, double eps, bool sorted, int *keep,
                         hipStream_t stream);
constexpr int kMaxSelectModes = 4096;   // LDS: (binary64 key + int index) per padded mode

// ---------------------------------------------------------------------------
// Host core (host_core.cpp): no device work.
// ---------------------------------------------------------------------------
struct TermLayout {
    int n_segs = 0, n_terms = 0, n_src = 0, n_chunks = 0;
    int *segs = nullptr;       // 4 * n_segs
    int *term_ptr = nullptr;   // n_terms + 1
    int *term_src = nullptr;   // 2 * n_src
    int *chunks = nullptr;     // n_chunks + 1: first segment of each chunk of <= kChunkTerms terms
    int grp[kTermGroups - 1] = {0, 0, 0};   // first segment of term groups 1..3
    int max_seg_terms = 0;     // longest segment
    // matrix-core path: distinct signed m values (rows) and the n range
    int n_mrows = 0, n_min = 0, n_max = 0, l_max = 0;
    int *mrows = nullptr;      // 2 * (n_mrows + 1): (m, first segment), sentinel (0, n_segs)
    bool consec = false;       // those m are consecutive
    bool mfma = false;         // layout fits the matrix-core shape (Schwarzschild terms)
    // matrix-core sum from the fold table (mf_terms_path): 10 row tiles +
    // steps needed, 0: outside its shapes
    int mf_terms = 0;
    int m_min = 0, k_min = 0, k_max = 0;
};

// Whether a sum over n samples on K knots of this layout (mf_terms != 0, not mfma)
// runs on the matrix cores.  Their cost per sample depends on the shape alone
// (rows, |n|), the vector kernel's on the terms, and each workgroup first forms
// its operands (with one round of samples 6 us for 16 rows and |n| < 16 to 12 us for
// 24 rows and |n| < 32 in binary32, 11 to 38 us in binary64; per interval and polar
// index), which only many samples repay; short generic-Kerr sums are split over the terms
// by the vector kernel.  Measured as sums of a kept spline, fold included (10 s
// cadence, log-spaced knots; vector / matrix-core on smooth amplitudes / on
// amplitudes with 10 % noise at every knot, us):
//   3.16 million samples, 60 knots: 7 rows, |n| <= 5, 77 terms 90 / 57 / 66; 11 rows,
//     |n| <= 3, 77 terms 96 / 67 / 85; 17 rows, |n| <= 4, 153 terms 156 / 106 / 135;
//     on 1000 knots 122 / 94 / 103, 129 / 106 / 126, 198 / 163 / 192
//   1 million samples, 60 knots: 39 / 30 / 33, 40 / 34 / 41, 17 rows, |n| <= 8, 289
//     terms 93 / 51 / 59; on 1000 knots 70 / 69 / 70, 73 / 76 / 82, 145 / 112 / 114
//   262144 samples, 60 knots: 7 rows, |n| <= 8, 119 terms 23 / 20 / 20; 11 rows, |n| <= 6,
//     143 terms 26 / 22 / 22; 7 rows, |n| <= 17, 245 terms 36 / 24 / 25; 17 rows,
//     |n| <= 8 44 / 31 / 32; on 1000 knots 65 / 58 / 59, 73 / 65 / 67, 93 / 71 / 73, 110 / 89 / 92
//   Kerr, 8640 samples, 60 knots, terms per polar index: 3 x 147 45 / 24 / 25, 5 x 187
//     87 / 39 / 39, 5 x 1281 210 / 72 / 75; 1000 samples on 900 knots 78 / 98 / 98,
//     124 / 154 / 159, 628 / 447 / 462
// (The lines for short Kerr sums are cautious: sums that would gain lie below them,
// 8640 samples, 5 x 341 terms 67 / 40, 5 x 425 85 / 62.)
// Binary64: both kernels are bound by the binary64 unit, the vector one with
// its terms, the matrix one with the cells (row, n) that its products cover,
// empty ones too, and with the powers of the cubic that take binary64 products:
// two on smooth amplitudes, three or four on noise, which the rule cannot know.
// Vector / matrix-core smooth / 10 % noise, us, terms of cells:
//   100 knots: 3.16 million samples 1281 of 1536 1539 / 916 / 1183, 1037 of 1536 1258 / 919 /
//     1178, 671 of 1024 824 / 668 / 856, 217 of 256 314 / 273 / 316; 0.8 million 496 / 277 /
//     397, 430 / 277 / 417, 268 / 204 / 282, 106 / 95 / 109; 262144 277 / 167 / 188, 226 /
//     165 / 186, 148 / 122 / 133, 62 / 53 / 57
//   1000 knots: 0.8 million samples 617 / 442 / 627, 497 / 433 / 610, 348 / 322 / 438,
//     142 / 159 / 182; 262144 327 / 319 / 353, 268 / 312 / 345, 186 / 233 / 252, 87 / 110 / 118
//   so the line rises with the knots; on smooth amplitudes nothing beyond it is slower
//   than the vector kernel (up to 2 % at 1000 knots), on 10 % noise up to 1.2 times
//   (0.66 of the cells filled, 150 knots, 3.16 million samples 842 / 688 / 1002).
//   Kerr, 0.4 million samples, 60 knots, five polar indices: 341 of 512 460 / 402 /
//     499, 425 of 672 592 / 547 / 601, 1281 of 1536 1603 / 911 / 1151
// Below one round per SIMD the vector kernel's serial walk over the terms is
// what a call waits for: 8640 samples, 60 knots, Kerr, 5 x 119 terms 134 / 56, 5 x 341
// 340 / 94; 30000 samples 135 / 74 and 341 / 132; 8640 samples on 400 knots 152 / 114 and
// 376 / 194.
// Schwarzschild requests below 262144 samples stay on the vector kernel: alone
// they would gain (1281 terms over one day, binary64, 265 / 111), but batches of
// them share its persistent launch, and a second launch of few workgroups at
// work each costs more than it saves (6 of up to 10 days, binary32, 111 / 127
// us; 6 of up to 30 days, binary64, 430 / 465).
// Binary32, accuracy: the matrix kernel forms f^n as a power of the sample's
// rounded f, an error that grows with |n|; the vector kernel seeds a segment with its
// exact phase and then walks it, an error that grows with the segment's length
// (and with the rows whose seeds are chained).  Lists that lie far from n = 0
// stay on the vector kernel: 21 rows, n in [a, b], 3 million samples, largest
// error of matrix-core / vector (mean of 10 draws; modes of one size and
// decaying ones): [20, 31] 1.3e-6 / 7.1e-7 and 9.5e-7 / 4.7e-7, [12, 31] 9.9e-7 / 1.0e-6
// and 7.6e-7 / 6.6e-7, [2, 12] 7.3e-7 / 7.0e-7 and 5.4e-7 / 4.4e-7; on the other side of
// the line [5, 31] 1.0e-6 / 1.5e-6 and 6.7e-7 / 7.4e-7, [0, 20] 7.8e-7 / 9.9e-7 and
// 5.4e-7 / 7.1e-7, [-3, 3] 6.8e-7 / 1.1e-6 and 5.3e-7 / 7.7e-7.
// (The fold table, its size and its launches are the same either way.)
inline bool mf_terms_path(const TermLayout &L, long long n, int K, bool fp32) {
    if (L.mf_terms == 0) return false;
    const int mt = L.mf_terms / 10, t = L.mf_terms % 10;
    const int shape = mt == 1 && t == 1 ? 0 : mt <= 2 && t == 1 ? 1 : mt <= 2 ? 2 : 3;
    const int nk = L.k_max - L.k_min + 1;
    if (nk == 1 && n < 262144) return false;
    if (fp32 && 10 * (L.max_seg_terms - 1) < 7 * std::max(-L.n_min, L.n_max) + 39) return false;
    if (!fp32) {
        const int steps = (L.n_max > -L.n_min ? L.n_max : -L.n_min) / 2 + 1;
        const int cells = 8 * (shape == 0 ? 1 : shape == 3 ? 3 : 2) * 4 * steps;
        long long least = n < 262144 ? 150 + cells * 11 / 20
                                     : 74 + cells * (nk > 1 ? 6 : 5) / 10 + (long long)cells * K / 4000;
        const long long brief = n >= 16384 ? 120 : 72;
        if (n < 65536 && least > brief) least = brief;
        return L.n_terms >= least * nk;
    }
    static const int kShortKerr[4] = {136, 160, 450, 660};
    static const int kShort[4] = {124, 140, 216, 300};
    // many samples: terms that cost the shape's rate, plus the staging shared out
    // over the samples (terms x 10^6 samples)
    static const int kRate[4] = {37, 44, 92, 94}, kStage[4] = {24, 31, 50, 60};
    // (196608 samples: 1.5 rounds of every wave of 256 workgroups)
    const int brief = nk > 1 && n < 196608 ? kShortKerr[shape] + K / 30 : kShort[shape];
    long long least = brief;
    if (n >= 196608)
        least = std::min<long long>(brief, kRate[shape] + K / 60 + (nk > 1 ? 16 : 0) +
                                               kStage[shape] * 1000000ll / n);
    return L.n_terms >= least * nk;
}

// Relative time of a sample of such a sum (shape 10 row tiles + steps; ns steps of
// two |n| in binary64): the shares of a batched launch are cut in these units.
__host__ __device__ inline int mf_terms_cost(int shape, int ns, bool f64) {
    const int mt = shape / 10, t = shape % 10;
    const int tiles = mt == 1 && t == 1 ? 1 : mt <= 2 ? 2 : 3;
    return f64 ? 8 + tiles * ns : tiles == 1 ? 5 : tiles == 3 ? 10 : t == 1 ? 6 : 8;
}

// The gap of an interval in a matrix-core sum's split between workgroups: the
// samples that its operands (formed, or staged from the operand table, and the
// round that its last samples leave part empty) are worth, at most two shares'
// samples.  Without it a workgroup at the dense end of a grid visits several
// intervals while others sum, and a short request's shares run across interval
// starts, two visits in place of one: binary64, 1281 terms, 262144 samples on 1000
// knots 642 -> 321 us, 5 x 171 Kerr terms, 8640 samples on 60 knots 131 -> 73 us, binary32
// from the fold table, 5 x 187, 100000 samples on 900 knots 326 -> 171 us, from operand
// tables, 1281 terms, 8640 samples 25.7 -> 20.9 us and 400000 on 1000 knots 109 -> 104 us.
// Twice these gaps gave the same or less (1000 knots, binary64, 400000 samples:
// 0.89 of the time without gaps against 0.79), half of them less.
constexpr int kMfGapTerms = 1024, kMfGap = 512;     // binary32 from the fold table, others
__host__ __device__ inline long long mf_gap(long long n, int most) {
    const long long two = n / 128;
    return two < most ? two : most;
}

// Build the folded term layout; returns 0 or a few_status error code.
int build_term_layout(int M, const int32_t *modes, int width, int max_gap, TermLayout *out);
void free_term_layout(TermLayout *t);

// Detector frame (see few_host_frame): source viewing angles and the complex
// factor -e^{-2 i psi}; returns 0 or FEW_E_ARG.
int detector_frame(double theta_s, double phi_s, double theta_k, double phi_k,
                   double *theta_src, double *phi_src, double *rot_re, double *rot_im);

// starts[i] for i in [0, K): see few_host_interval_starts.
void interval_starts(int K, const double *t, double t_start, double dt, long long n,
                     long long *starts);

// Upper bound of the wave tiles a request needs.
inline long long tile_upper_bound(long long n, int K, int tile) {
    return (n + tile - 1) / tile + (K - 1);
}

// Single-request launches split the samples into kParts contiguous parts,
// [floor(p n / kParts), floor((p + 1) n / kParts)), one per XCD, so each XCD
// reads the coefficient tables of its own intervals only.
constexpr int kParts = 8;

__host__ __device__ inline long long part_begin(long long n, int parts, int p) {
    return n * p / parts;
}

// Tiles of one part (at most ceil(n / parts) samples) whose last short_len
// samples use short tiles: each interval adds at most one partial tile of
// each kind.
inline long long part_tile_bound(long long n, int parts, long long short_len, int K, int tile,
                                 int short_tile) {
    const long long len = (n + parts - 1) / parts;
    if (short_len <= 0) return tile_upper_bound(len, K, tile);
    const long long s = short_len < len ? short_len : len;
    return (len + tile - 1) / tile + (s + short_tile - 1) / short_tile + 2LL * (K - 1);
}

// Arena layout of one request's resident state.
struct ReqLayout {
    size_t off_t, off_segs, off_term_ptr, off_term_src, off_chunks, off_mrows,
        upload_end;   // host-staged
    size_t off_pcoef, off_acoef, off_ybuf, off_table, off_starts, off_tile_pref, off_mtab,
        off_minfo, total;
    size_t dev_begin;       // first device-produced offset (== off_pcoef)
};
// mfma: binary32 request on the matrix-core path (binary32 operand table in
// place of the fold table; n_mrows rows)
ReqLayout request_layout(bool fp32, int K, int M, int n_segs, int n_terms, int n_src,
                         int n_chunks, int n_ph, bool mfma = false, int n_mrows = 0);

// Binary64 sample time exactly as written: t_start + j * dt, no contraction.
double sample_time(double t_start, double dt, long long j);

}  // namespace few
