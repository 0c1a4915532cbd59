// gfx950 kernels of libfew: the interpolated harmonic-mode summation of
// arXiv:2104.04582, Sec. III C (spline stage, then summation stage) for the
// Schwarzschild sum of Eq. (10) with the mirror modes of Eq. (9), and the
// generic-Kerr sum of Sec. VII (a third phase).
//
//  upload_kernel   copies a batch's host tables (knots, term layouts, job
//                  descriptors) from pinned host memory, ordered on the
//                  compute queue (a single-request fit carries its own copy).
//  fit_kernel      not-a-knot cubic splines of every series on the shared knot
//                  grid.  Amplitude series: binary64, one lane per real series,
//                  rows split over the workgroup's four waves and joined by
//                  the multipliers' products; the grid's tridiagonal factor by
//                  one wave's scan.  Phase series: double-double (one
//                  refinement step, scan solves).
//  fold_pack_kernel  long Schwarzschild lists with a binary32 result: interval
//                  starts; per interval and row tile, -2Y_lm, the fold of the
//                  l-sum, the row scales and the operand values of the products.
//  prepare_kernel  all other requests: interval starts and tile prefixes;
//                  -2Y_lm and the fold of the l-sum into one complex cubic per
//                  signed (m, [k,] n) term.
//  sum_mfma_kernel binary32 result on the matrix cores: per interval the
//                  product of the coefficient matrix (signed m rows) with the
//                  harmonics f^|n| of the samples, v_mfma_f32_16x16x32_f16 on
//                  fp16 hi/lo parts with fp32 accumulation; the cubic in time
//                  about the centre of blocks of samples (one Horner step) or
//                  of the interval (three); rows combined with e^{-i m Phi_phi}.
//  sum_mfma_terms_kernel  the same from prepare_kernel's terms (middle lists,
//                  generic Kerr), operands formed by each workgroup.
//  sum_mfma_f64_kernel  the same in binary64 (v_mfma_f64_16x16x4_f64; small
//                  curvature from fp16 hi/lo parts with fp32 accumulation).
//  sum_wg_kernel   binary32 on the vector units (few terms, or few samples):
//                  one workgroup of 4 waves = one
//                  tile of consecutive samples inside one knot interval; the
//                  term coefficients are staged in LDS and broadcast to VGPR
//                  operands.  Per sample: phases in binary64 reduced mod 2 pi,
//                  one sincos each; then for every segment of terms a Horner
//                  recurrence in e^{-i Phi_r} over n, seeded by
//                  e^{-i(m Phi_phi + n_lo Phi_r)} (chained across consecutive
//                  m or k), Kahan-compensated within four term groups whose
//                  values are added in order; the end of a launch uses
//                  term-split tiles (the four waves take one group each).
//  sum_kernel      binary64 on the vector units (sparse lists, short sums): one wave = one
//                  tile; phases in double-double; coefficients read by scalar
//                  loads into SGPR operands.
//  select_kernel   the mode selector of Sec. III D: per knot a radix select
//                  with error-bounded sums, the sorted sequential sums when a
//                  comparison falls inside the bound.
#include "dd.h"
#include "few_internal.h"
#include "swsh.h"

#include <climits>
#include <cstring>
#include <mutex>
#include <type_traits>

namespace few {

#define FEW_AS4 __attribute__((address_space(4)))

// Minimum waves per SIMD (a register cap) of the single-request binary32
// summation kernel: 4, i.e. at most 128 registers, which keeps the three-phase
// (generic-Kerr) instantiation at four workgroups per CU as well.
#ifndef FEW_SUM_WAVES
#define FEW_SUM_WAVES 4
#endif
#define FEW_SUM_ATTR __attribute__((amdgpu_waves_per_eu(FEW_SUM_WAVES)))
// Binary64: the five-FMA chains per component need more waves in flight than
// the register count alone allows (4 per SIMD); 5 costs one spill outside the
// term loop.
#ifndef FEW_F64_WAVES
#define FEW_F64_WAVES 5
#endif
#define FEW_F64_ATTR __attribute__((amdgpu_waves_per_eu(FEW_F64_WAVES)))

// Wave-uniform read-only data: the constant address space makes the compiler
// use scalar loads (SGPR destinations) for uniform addresses.
template <typename T>
__device__ __forceinline__ const FEW_AS4 T *cptr(const T *p) {
    return (const FEW_AS4 T *)(p);
}

// Copy a trivially copyable object from a wave-uniform address as 32-bit
// scalar loads.
template <typename T>
__device__ __forceinline__ T load_uniform(const T *p) {
    static_assert(sizeof(T) % 4 == 0, "4-byte granularity");
    T v;
    const FEW_AS4 uint32_t *s = (const FEW_AS4 uint32_t *)(p);
    uint32_t *d = reinterpret_cast<uint32_t *>(&v);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) d[i] = s[i];
    return v;
}

__device__ __forceinline__ float fmar(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmar(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Binary64 sample time exactly as written: t_start + j * dt.
__device__ __forceinline__ double dev_sample_time(double t_start, double dt, long long j) {
    return __dadd_rn(t_start, __dmul_rn((double)j, dt));
}

// ===========================================================================
// Spline stage (Sec. III C: not-a-knot spline, all series on one knot grid).
//
// Slope form: on [t_i, t_{i+1}], x = t - t_i, h_i = t_{i+1} - t_i,
// delta_i = (y_{i+1} - y_i) / h_i and end slopes s_i, s_{i+1}:
//   y = y_i + s_i x + c_i x^2 + d_i x^3,
//   c_i = (3 delta_i - 2 s_i - s_{i+1}) / h_i,  d_i = (s_i + s_{i+1} - 2 delta_i) / h_i^2.
// Tridiagonal system for the slopes (rows: sub, diag, super | rhs):
//   row 0      : -, h_1, h_0 + h_1 | ((h_0 + 2(h_0 + h_1)) h_1 delta_0 + h_0^2 delta_1) / (h_0 + h_1)
//   row 1..K-2 : h_i, 2 (h_{i-1} + h_i), h_{i-1} | 3 (h_i delta_{i-1} + h_{i-1} delta_i)
//   row K-1    : h_{K-2} + h_{K-3}, h_{K-3}, - |
//                (h_{K-2}^2 delta_{K-3} + (2 (h_{K-3} + h_{K-2}) + h_{K-2}) h_{K-3} delta_{K-2})
//                / (h_{K-3} + h_{K-2})
// (interior rows: continuous second derivative; end rows: the not-a-knot
// conditions d_0 = d_1 and d_{K-3} = d_{K-2} with s_2 / s_{K-3} eliminated).
// Solved by forward elimination and back substitution without pivoting.
// ===========================================================================

// LU factor of the slope system on the shared grid: inverse pivots invd[r] and
// multipliers w[r] = c_r invd[r] of the forward sweep (c_r the super-diagonal),
// with pivots den_r = a_r - b_r w_{r-1} (a_r diagonal, b_r sub-diagonal).
// The pivot recurrence is a continued fraction; with w_r = p_r / q_r it is the
// division-free pair
//   q_r = a_r q_{r-1} - b_r p_{r-1},   p_r = c_r q_{r-1},   den_r = q_r / q_{r-1},
// rescaled at every row by a power of two (exact, ratios unchanged) so it
// cannot overflow.  One lane runs it (fit_factor_serial: a multiply, an FMA and
// the rescale per row, knot spacings fetched 16 at a time), storing q_{r-1}
// and q_r per row in invd / wv; then every lane forms the ratios
// (fit_factor_finish).  A division per row on the serial chain was its
// latency bound.
__device__ __forceinline__ void fit_factor_serial(const double *h, int K, double *num,
                                                  double *den) {
    constexpr int C = 16;
    double q = h[1], p = h[0] + h[1];               // row 0: diag h_1, super h_0 + h_1
    num[0] = 1.0;
    den[0] = q;
    double hp = h[0];                               // h_{r-1}
    auto row = [&](int r, double hr) {              // interior row r: b = h_r, a = 2(h_{r-1} + h_r), c = h_{r-1}
        const double Q = (2.0 * (hp + hr)) * q - hr * p;
        num[r] = q;
        den[r] = Q;
        int e;
        const double m = frexp(Q, &e);
        p = ldexp(hp * q, -e);
        q = m;
        hp = hr;
    };
    int r0 = 1;
    for (; r0 + C <= K - 1; r0 += C) {
        double hv[C];
#pragma unroll
        for (int c = 0; c < C; ++c) hv[c] = h[r0 + c];
#pragma unroll
        for (int c = 0; c < C; ++c) row(r0 + c, hv[c]);
    }
    for (; r0 <= K - 2; ++r0) row(r0, h[r0]);
    // row K-1: sub h_{K-2} + h_{K-3}, diag h_{K-3}
    num[K - 1] = q;
    den[K - 1] = h[K - 3] * q - (h[K - 2] + h[K - 3]) * p;
}

// Ratios of the factor: inverse pivots invd[r], back-sweep multipliers
// wv[r] = c_r invd[r] and forward-sweep multipliers bv[r] = b_r invd[r] (b_r
// the sub-diagonal), so each forward step is one fused multiply-add on the
// serial chain: g_r = rhs_r invd_r - bv_r g_{r-1}.
__device__ __forceinline__ void fit_factor_finish(const double *h, int K, double *invd,
                                                  double *wv, double *bv) {
    for (int r = threadIdx.x; r < K; r += blockDim.x) {
        const double id = invd[r] / wv[r];
        const double c = r == 0 ? h[0] + h[1] : (r < K - 1 ? h[r - 1] : 0.0);
        const double b = r == 0 ? 0.0 : (r < K - 1 ? h[r] : h[K - 2] + h[K - 3]);
        invd[r] = id;
        wv[r] = c * id;
        bv[r] = b * id;
    }
}

// LDS writes of one wave made visible to its other lanes (the wave's LDS
// accesses complete in order; this keeps the compiler from moving them).
__device__ __forceinline__ void lds_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Row r of the slope system: sub-diagonal b, diagonal a, super-diagonal c
// (the table above).
__device__ __forceinline__ void slope_row(const double *h, int K, int r, double *b, double *a,
                                          double *c) {
    if (r == 0) {
        *b = 0.0;
        *a = h[1];
        *c = h[0] + h[1];
    } else if (r < K - 1) {
        *b = h[r];
        *a = 2.0 * (h[r - 1] + h[r]);
        *c = h[r - 1];
    } else {
        *b = h[K - 2] + h[K - 3];
        *a = h[K - 3];
        *c = 0.0;
    }
}

// The same factor (invd, wv, bv as fit_factor_finish leaves them) on one wave
// for K <= R kWave.  With every continuant divided by the diagonals,
// qt_r = q_r / (a_0 ... a_r), the recurrence becomes
//   qt_r = qt_{r-1} - g_r qt_{r-2},  g_r = b_r c_{r-1} / (a_r a_{r-1}),
// qt_{-1} = qt_0 = 1, and den_r = a_r qt_r / qt_{r-1}.  For this system
// 0 <= g_r <= 1/4 on interior rows and g_r = 1/2 on rows 1 and K - 1, so
// qt_r / qt_{r-1} lies in [1/2, 1] on rows 1 .. K - 2 (by induction) and in
// (0, 1) on row K - 1: the qt stay positive and above 2^-K times the last
// ratio, with no rescaling.  In matrix form (qt_r, qt_{r-1}) =
// T_r (qt_{r-1}, qt_{r-2}), T_r = [[1, -g_r], [1, 0]]; lane l takes rows
// R l + 1 .. R l + R, and the lanes' products are composed by a log-step scan
// (later rows on the left).
template <int R>
__device__ void fit_factor_wave(const double *h, int K, double *invd, double *wv, double *bv) {
    const int lane = threadIdx.x & (kWave - 1);
    const int r0 = R * lane + 1;
    double bb[R], aa[R], cc[R], gg[R];
    // this lane's product T_{r0+R-1} .. T_{r0} (identity rows past the end)
    double m00 = 1.0, m01 = 0.0, m10 = 0.0, m11 = 1.0;
    {
        double ap = 1.0, cp = 0.0;
        if (r0 < K) {
            double bp;
            slope_row(h, K, r0 - 1, &bp, &ap, &cp);
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            bb[j] = cc[j] = gg[j] = 0.0;
            aa[j] = 1.0;
            if (r0 + j < K) {
                slope_row(h, K, r0 + j, &bb[j], &aa[j], &cc[j]);
                gg[j] = bb[j] * cp / (aa[j] * ap);
                ap = aa[j];
                cp = cc[j];
                const double n00 = fma(-gg[j], m10, m00), n01 = fma(-gg[j], m11, m01);
                m10 = m00;
                m11 = m01;
                m00 = n00;
                m01 = n01;
            }
        }
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const double o00 = __shfl_up(m00, d), o01 = __shfl_up(m01, d);
        const double o10 = __shfl_up(m10, d), o11 = __shfl_up(m11, d);
        if (lane >= d) {
            const double n00 = fma(m00, o00, m01 * o10), n01 = fma(m00, o01, m01 * o11);
            const double n10 = fma(m10, o00, m11 * o10), n11 = fma(m10, o01, m11 * o11);
            m00 = n00; m01 = n01; m10 = n10; m11 = n11;
        }
    }
    // (qt_{r0-1}, qt_{r0-2}) = (rows before this lane's) applied to (1, 1)
    double p00 = __shfl_up(m00, 1), p01 = __shfl_up(m01, 1);
    double p10 = __shfl_up(m10, 1), p11 = __shfl_up(m11, 1);
    if (lane == 0) { p00 = 1.0; p01 = 0.0; p10 = 0.0; p11 = 1.0; }
    double qa = p00 + p01, qb = p10 + p11;          // qt_{r-1}, qt_{r-2}
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (r0 + j < K) {
            const double q = fma(-gg[j], qb, qa);
            const double id = qa / (aa[j] * q);
            invd[r0 + j] = id;
            wv[r0 + j] = cc[j] * id;
            bv[r0 + j] = bb[j] * id;
            qb = qa;
            qa = q;
        }
    }
    if (lane == 0) {                                 // row 0: den_0 = a_0
        const double id = 1.0 / h[1];
        invd[0] = id;
        wv[0] = (h[0] + h[1]) * id;
        bv[0] = 0.0;
    }
}

// y_r = a(r) + m(r) y_{r-1} for r < n <= R kWave, y_{-1} = 0, on one wave:
// lane l takes rows R l .. R l + R - 1, and the lanes' affine maps y -> A + M y
// are composed by a log-step scan (later rows on the left).  y: this lane's
// values; rows past n are identities.
template <int R, typename FA, typename FM>
__device__ __forceinline__ void wave_affine(int n, FA a, FM m, double (&y)[R]) {
    const int lane = threadIdx.x & (kWave - 1);
    double av[R], mv[R], A = 0.0, M = 1.0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int r = R * lane + j;
        av[j] = 0.0;
        mv[j] = 1.0;
        if (r < n) { av[j] = a(r); mv[j] = m(r); }
        A = j == 0 ? av[0] : fma(mv[j], A, av[j]);
        M = j == 0 ? mv[0] : mv[j] * M;
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const double Ao = __shfl_up(A, d), Mo = __shfl_up(M, d);
        if (lane >= d) {
            A = fma(M, Ao, A);
            M = M * Mo;
        }
    }
    double v = __shfl_up(A, 1);
    if (lane == 0) v = 0.0;
#pragma unroll
    for (int j = 0; j < R; ++j) y[j] = v = fma(mv[j], v, av[j]);
}

// Phase series ph (workgroup ph), to double-double accuracy by one step of
// iterative refinement: solve the slope system in binary64 (Thomas), form
// the residual with the exact double-double matrix and right-hand side, solve
// again for the correction and add it.  After one step the error is of order
// (eps cond)^2, far below double-double rounding, and only the two binary64
// sweeps are serial.  pcoef[((i * 2 + ph) * 4 + p) * 2 + {0, 1}] = (hi, lo) of
// coefficient p on interval i; p = 0 holds y_i reduced mod 2 pi.
// LDS (binary64 arrays of length K): h hi/lo, delta hi/lo, w, inverse pivot,
// first solution s0, right-hand side / residual / correction.
// K <= R kWave: the sweeps run on one wave (R = 0: longer grids, one lane).
template <int R>
__device__ void fit_phase_dd(const FitJob &jb, const double *t, int ph, double *lds) {
    const double *y = ph == 0 ? jb.phi_phi : (ph == 1 ? jb.phi_r : jb.phi_theta);
    const int K = jb.K;
    const int tid = threadIdx.x, bs = blockDim.x;
    double *Hh = lds, *Hl = lds + K, *Dh = lds + 2 * K, *Dl = lds + 3 * K;
    double *wv = lds + 4 * K, *invd = lds + 5 * K, *s0 = lds + 6 * K, *rr = lds + 7 * K;
    double *bv = lds + 8 * K;
    auto H = [&](int i) { return dd_make(Hh[i], Hl[i]); };
    auto D = [&](int i) { return dd_make(Dh[i], Dl[i]); };
    // row r of the slope system: sub, diag, super (double-double)
    auto row = [&](int r, dd *sub, dd *diag, dd *sup) {
        if (r == 0) {
            *sub = dd_make(0.0);
            *diag = H(1);
            *sup = dd_add(H(0), H(1));
        } else if (r < K - 1) {
            *sub = H(r);
            *diag = dd_mul_d(dd_add(H(r - 1), H(r)), 2.0);
            *sup = H(r - 1);
        } else {
            *sub = dd_add(H(K - 2), H(K - 3));
            *diag = H(K - 3);
            *sup = dd_make(0.0);
        }
    };
    auto rhs = [&](int r) {
        if (r == 0) {
            const dd h0 = H(0), h1 = H(1), sup = dd_add(h0, h1);
            return dd_div(dd_add(dd_mul(dd_mul(dd_add(h0, dd_mul_d(sup, 2.0)), h1), D(0)),
                                 dd_mul(dd_mul(h0, h0), D(1))),
                          sup);
        }
        if (r < K - 1)
            return dd_mul_d(dd_add(dd_mul(H(r), D(r - 1)), dd_mul(H(r - 1), D(r))), 3.0);
        const dd ha = H(K - 3), hb = H(K - 2), sum = dd_add(ha, hb);
        return dd_div(dd_add(dd_mul(dd_mul(hb, hb), D(K - 3)),
                             dd_mul(dd_mul(dd_add(dd_mul_d(sum, 2.0), hb), ha), D(K - 2))),
                      sum);
    };
    // binary64 Thomas sweeps with the factor in invd / wv / bv (of the rounded
    // matrix; the refinement step uses the exact rows): x <- A^-1 x in place.
    // R > 0: wave 0 takes each sweep as one affine scan (wave_affine; the back
    // sweep in reversed row order).  Otherwise one lane
    // carries the recurrence in registers: the LDS operands of C rows are
    // loaded together, the rows eliminated (one fused multiply-add each on
    // the serial chain), and the C results stored after the batch.
    constexpr bool wave_solve = R > 0;
    auto solve_wave = [&](double *x) {
        constexpr int RR = R > 0 ? R : 1;
        const int r0 = RR * tid;
        double g[RR];
        wave_affine<RR>(
            K, [&](int r) { return x[r] * invd[r]; }, [&](int r) { return -bv[r]; }, g);
#pragma unroll
        for (int j = 0; j < RR; ++j)
            if (r0 + j < K) x[r0 + j] = g[j];
        lds_wave_sync();
        wave_affine<RR>(
            K, [&](int r) { return x[K - 1 - r]; }, [&](int r) { return -wv[K - 1 - r]; }, g);
        lds_wave_sync();
#pragma unroll
        for (int j = 0; j < RR; ++j)
            if (r0 + j < K) x[K - 1 - r0 - j] = g[j];
    };
    auto solve = [&](double *x) {
        constexpr int C = 16;
        double g = x[0] * invd[0];
        x[0] = g;
        int r0 = 1;
        for (; r0 + C <= K; r0 += C) {
            double xv[C], bb[C], iv[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                xv[c] = x[r0 + c];
                bb[c] = bv[r0 + c];
                iv[c] = invd[r0 + c];
            }
#pragma unroll
            for (int c = 0; c < C; ++c) xv[c] = xv[c] * iv[c];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                g = fma(-bb[c], g, xv[c]);
                xv[c] = g;
            }
#pragma unroll
            for (int c = 0; c < C; ++c) x[r0 + c] = xv[c];
        }
        for (; r0 < K; ++r0) {
            g = fma(-bv[r0], g, x[r0] * invd[r0]);
            x[r0] = g;
        }
        double nx = x[K - 1];
        r0 = K - 2;
        for (; r0 - C + 1 >= 0; r0 -= C) {
            double xv[C], wr[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                xv[c] = x[r0 - c];
                wr[c] = wv[r0 - c];
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                xv[c] = fma(-wr[c], nx, xv[c]);
                nx = xv[c];
            }
#pragma unroll
            for (int c = 0; c < C; ++c) x[r0 - c] = xv[c];
        }
        for (; r0 >= 0; --r0) {
            x[r0] = fma(-wv[r0], nx, x[r0]);
            nx = x[r0];
        }
    };

    for (int i = tid; i < K - 1; i += bs) {
        const dd h = two_sum(t[i + 1], -t[i]);
        const dd d = dd_div(two_sum(y[i + 1], -y[i]), h);
        Hh[i] = h.hi; Hl[i] = h.lo;
        Dh[i] = d.hi; Dl[i] = d.lo;
    }
    __syncthreads();
    // binary64 factor of the rounded matrix (wave 0, or one lane of it) while
    // the other waves form the right-hand side, then the first solve
    if (wave_solve) {
        if (tid < kWave) fit_factor_wave<(R > 0 ? R : 1)>(Hh, K, invd, wv, bv);
    } else if (tid == 0) {
        fit_factor_serial(Hh, K, invd, wv);
    }
    if (tid >= kWave)
        for (int r = tid - kWave; r < K; r += bs - kWave) s0[r] = rhs(r).hi;
    __syncthreads();
    if (!wave_solve) {
        fit_factor_finish(Hh, K, invd, wv, bv);
        __syncthreads();
    }
    if (wave_solve ? tid < kWave : tid == 0) {
        if (wave_solve) solve_wave(s0); else solve(s0);
    }
    __syncthreads();
    // residual of the exact (double-double) system at s0
    for (int r = tid; r < K; r += bs) {
        dd sub, diag, sup;
        row(r, &sub, &diag, &sup);
        dd ax = dd_mul_d(diag, s0[r]);
        if (r > 0) ax = dd_add(ax, dd_mul_d(sub, s0[r - 1]));
        if (r < K - 1) ax = dd_add(ax, dd_mul_d(sup, s0[r + 1]));
        rr[r] = dd_sub(rhs(r), ax).hi;
    }
    __syncthreads();
    if (wave_solve ? tid < kWave : tid == 0) {
        if (wave_solve) solve_wave(rr); else solve(rr);
    }
    __syncthreads();
    double *pc = jb.pcoef;
    for (int r = tid; r < K - 1; r += bs) {
        const dd sa = two_sum(s0[r], rr[r]), sb = two_sum(s0[r + 1], rr[r + 1]);
        const dd h = H(r), d = D(r);
        const dd c = dd_div(dd_sub(dd_sub(dd_mul_d(d, 3.0), dd_mul_d(sa, 2.0)), sb), h);
        const dd e = dd_div(dd_sub(dd_add(sa, sb), dd_mul_d(d, 2.0)), dd_mul(h, h));
        const dd a = dd_reduce_2pi(dd_make(y[r]));
        double *o = pc + ((size_t)r * jb.n_ph + ph) * 8;
        o[0] = a.hi; o[1] = a.lo;
        o[2] = sa.hi; o[3] = sa.lo;
        o[4] = c.hi; o[5] = c.lo;
        o[6] = e.hi; o[7] = e.lo;
    }
}

// The two sweeps of one real amplitude series q (lane tid of wave 0) for
// grids of more than kFitStageKnots knots: knot values stream from global
// memory, the forward results go through the coefficient array, and each
// row's coefficients are stored as its slope is found.
__device__ __forceinline__ void fit_sweeps(const FitJob &jb, int tid, int q, int K, int M,
                                           const double *hs, const double *invd,
                                           const double *wv, const double *ih,
                                           const double *bv) {
    constexpr int C = 16;
    const size_t ys_stride = 2 * (size_t)M;
    // coefficient p of series q on interval r at o[r * cs + p * ps]
    // ([K-1][4][2M] or [K-1][M][4][2])
    const bool pm = jb.acoef_pmajor != 0;
    const size_t ps = pm ? 2 * (size_t)M : 2, cs = 8 * (size_t)M;
    const int k = q >> 1, comp = q & 1;
    const double *__restrict__ y = jb.amp + 2 * (size_t)k + comp;
    double *__restrict__ o = jb.acoef + (pm ? (size_t)q : 8 * (size_t)k + comp);
    // knot value idx (clamped to the grid: in bounds, unused past it)
    auto ldy = [&](int idx) {
        const int i = min(max(idx, 0), K - 1);
        return y[(size_t)i * ys_stride];
    };
    auto stg = [&](int r, double gv) { o[(size_t)r * cs + ps] = gv; };
    auto ldg = [&](int r) { return o[(size_t)max(r, 0) * cs + ps]; };

    // Forward elimination.  Knot idx gives delta_{idx-1}; rows 0 and 1 close
    // at knot 2, row idx - 1 at every later knot, row K - 1 after the last.
    double yprev = ldy(0);
    double dm1, d0, g;
    {
        const double y1 = ldy(1), y2 = ldy(2);
        const double h0 = hs[0], h1 = hs[1];
        dm1 = (y1 - yprev) * ih[0];
        d0 = (y2 - y1) * ih[1];
        yprev = y2;
        g = ((h0 + 2.0 * (h0 + h1)) * h1 * dm1 + h0 * h0 * d0) / (h0 + h1) * invd[0];
        stg(0, g);
        const double rhs = 3.0 * (h1 * dm1 + h0 * d0);
        g = fma(-bv[1], g, rhs * invd[1]);
        stg(1, g);
    }
    // one row: r = idx - 1 closes at knot idx
    auto fwd = [&](int idx, double yi) {
        const int r = idx - 1;
        dm1 = d0;
        d0 = (yi - yprev) * ih[r];
        yprev = yi;
        g = fma(-bv[r], g, (3.0 * (hs[r] * dm1 + hs[r - 1] * d0)) * invd[r]);
        stg(r, g);
    };
    // C rows: operands first, then the chain, then the stores
    auto fwd_batch = [&](int i0, const double *ya) {
        double hr[C], hm[C], iv[C], bb[C], rv[C];
        const int rb = i0 - 1;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            hr[c] = hs[rb + c];
            hm[c] = hs[rb + c - 1];
            rv[c] = ih[rb + c];
            iv[c] = invd[rb + c];
            bb[c] = bv[rb + c];
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            dm1 = d0;
            d0 = (ya[c] - yprev) * rv[c];
            yprev = ya[c];
            rv[c] = (3.0 * (hr[c] * dm1 + hm[c] * d0)) * iv[c];
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            g = fma(-bb[c], g, rv[c]);
            rv[c] = g;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) stg(rb + c, rv[c]);
    };
    double ya[C];
#pragma unroll
    for (int c = 0; c < C; ++c) ya[c] = ldy(3 + c);
    int i0 = 3;
    for (; i0 + C <= K; i0 += C) {
        double yb[C];
#pragma unroll
        for (int c = 0; c < C; ++c) yb[c] = ldy(i0 + C + c);
        fwd_batch(i0, ya);
#pragma unroll
        for (int c = 0; c < C; ++c) ya[c] = yb[c];
    }
    for (int c = 0; i0 + c < K; ++c) fwd(i0 + c, ya[c]);
    {
        const double ha = hs[K - 3], hb = hs[K - 2];
        const double rhs = (hb * hb * dm1 + (2.0 * (ha + hb) + hb) * ha * d0) / (ha + hb);
        g = fma(-bv[K - 1], g, rhs * invd[K - 1]);
    }
    // Back substitution and coefficients, interval K-2 down to 0, in batches
    // of C rows r0, r0 - 1, ...: operands first (the batch's forward results
    // and knot values, and the next batch's in flight), then the chain.
    double s_next = g;
    double yr1 = yprev;                              // y_{K-1}
    double ga[C], yv[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        ga[c] = ldg(K - 2 - c);
        yv[c] = ldy(K - 2 - c);
    }
    auto back = [&](int r, double gr, double yv0) {
        const double ir = ih[r];
        const double dr = (yr1 - yv0) * ir;
        const double sv = fma(-wv[r], s_next, gr);
        double *orow = o + (size_t)r * cs;
        orow[0] = yv0;
        orow[ps] = sv;
        orow[2 * ps] = (3.0 * dr - 2.0 * sv - s_next) * ir;
        orow[3 * ps] = (sv + s_next - 2.0 * dr) * (ir * ir);
        s_next = sv;
        yr1 = yv0;
    };
    int r0 = K - 2;
    for (; r0 - C + 1 >= 0; r0 -= C) {
        double gb[C], yw[C], irv[C], wrv[C], sv[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            gb[c] = ldg(r0 - C - c);
            yw[c] = ldy(r0 - C - c);
            irv[c] = ih[r0 - c];
            wrv[c] = wv[r0 - c];
        }
        double sn = s_next;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            sn = fma(-wrv[c], sn, ga[c]);
            sv[c] = sn;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int r = r0 - c;
            const double sh = c == 0 ? s_next : sv[c - 1];    // slope at knot r + 1
            const double yh = c == 0 ? yr1 : yv[c - 1];       // value at knot r + 1
            const double ir = irv[c];
            const double dr = (yh - yv[c]) * ir;
            double *orow = o + (size_t)r * cs;
            orow[0] = yv[c];
            orow[ps] = sv[c];
            orow[2 * ps] = (3.0 * dr - 2.0 * sv[c] - sh) * ir;
            orow[3 * ps] = (sv[c] + sh - 2.0 * dr) * (ir * ir);
        }
        s_next = sn;
        yr1 = yv[C - 1];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            ga[c] = gb[c];
            yv[c] = yw[c];
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (r0 - c >= 0) back(r0 - c, ga[c], yv[c]);
}

// The upload carried by a single-request fit launch: amplitude workgroup blk
// copies its share of the 16-byte words (the tail word may run into the
// block's alignment padding; the staging slot is at least 1 MiB), on the
// lanes of waves 1-3, which do not take part in the sweeps.
__device__ __forceinline__ void fit_copy_upload(const FitJob &jb, int blk) {
    if (jb.up_bytes <= 0) return;
    const long long words = (jb.up_bytes + 15) / 16;
    const long long per = (words + jb.amp_blocks - 1) / jb.amp_blocks;
    const long long w0 = (long long)blk * per, w1 = min(words, w0 + per);
    const int lanes = (int)blockDim.x - kWave;
    for (long long x = w0 + ((int)threadIdx.x - kWave); x < w1; x += lanes)
        jb.up_dst[x] = jb.up_src[x];
}

// Binary64 solve of the amplitude series handled by this workgroup for grids
// of more than kFitStageKnots knots, one lane of wave 0 per real series.  LDS:
// h[K], inverse pivots invd[K], multipliers wv[K] and bv[K] and 1 / h[K] of
// the shared grid (the sweeps multiply by 1 / h_i instead of dividing: a
// division is a long dependent sequence on this hardware, and the sweeps are
// latency bound).  Wave 0 forms the grid and one of its lanes the factor;
// each lane streams its knot values from global memory, both sweeps working in
// batches of C rows (operands first, the serial chain in registers, the
// results stored after it).
__device__ void fit_amplitudes_stream(const FitJob &jb, const double *t, int blk, double *lds) {
    const int K = jb.K, M = jb.M;
    const int tid = threadIdx.x;
    double *hs = lds, *invd = lds + K, *wv = lds + 2 * K, *ih = lds + 3 * K, *bv = lds + 4 * K;
    const int q0 = blk * kFitSeriesPerBlock;
    if (tid < kWave) {
        for (int i = tid; i < K - 1; i += kWave) {
            const double h = t[i + 1] - t[i];
            hs[i] = h;
            ih[i] = 1.0 / h;
        }
        __builtin_amdgcn_wave_barrier();
        if (tid == 0) fit_factor_serial(hs, K, invd, wv);
    }
    __syncthreads();
    fit_factor_finish(hs, K, invd, wv, bv);
    __syncthreads();
    const int q = q0 + tid;
    if (tid < kFitSeriesPerBlock && q < 2 * M) fit_sweeps(jb, tid, q, K, M, hs, invd, wv, ih, bv);
    if (tid >= kWave) fit_copy_upload(jb, blk);
}

// Row l of a wave-uniform value held by lane l (both halves by readlane).
__device__ __forceinline__ double lane_value(double v, int l) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Binary64 solve of the amplitude series of workgroup blk (64 real series,
// lane = series) for K <= R kWave.  The rows are split over the four
// waves: wave w takes rows [R_w, R_{w+1}) and keeps its lanes' knot values
// y_{R_w - 1} .. y_{R_{w+1}} and its forward results and slopes in
// registers; row-wise constants are formed lane-parallel (lane c for row
// R_w + c) and broadcast with readlane.  Wave 0 forms the factor
// (fit_factor_wave) while every wave's knot values are in flight.  Row r's
// forward input rhs_r invd_r is
//   al_r (y_{a+1} - y_a) + be_r (y_{a+2} - y_{a+1}),  a = clamp(r - 1, 0, K - 3)
// (its two divided differences).  Each wave runs its rows from a zero start
// and the chunks are joined afterwards, since a first-order recurrence at row
// r is its zero-start value plus the product of the multipliers since the
// chunk start times the value entering the chunk:
//   forward g_r = rhs_r invd_r - bv_r g_{r-1}:  g_r = gl_r + F_r G,
//           F_r = prod_{j = R_w .. r} (-bv_j), G = g_{R_w - 1};
//   back    s_r = g_r - wv_r s_{r+1}:          s_r = sl_r + B_r S,
//           B_r = prod_{j = r .. R_{w+1} - 1} (-wv_j), S = s_{R_{w+1}}.
// The values entering the chunks follow from the chunk ends (exchanged in
// LDS) in at most three steps.  Each wave then writes the coefficients of its
// intervals.
template <int R>
__device__ void fit_amplitudes_staged(const FitJob &jb, const double *t, int blk, double *lds) {
    constexpr int NW = 4;                            // waves (launched with 256 lanes)
    constexpr int LC = R * kWave / NW;               // most rows of a chunk
    const int K = jb.K, M = jb.M;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    double *hs = lds, *invd = lds + K, *wv = lds + 2 * K, *bv = lds + 3 * K;
    double *cf = lds + 4 * K;                        // [NW][64] forward values at chunk ends
    double *cb = cf + NW * kWave;                    // [NW][64] back values at chunk starts
    double *fe = cb + NW * kWave;                    // [NW] F at chunk ends
    double *bs0 = fe + NW;                           // [NW] B at chunk starts
    const int q = blk * kFitSeriesPerBlock + lane;
    const bool live = q < 2 * M;
    const int L = (K + NW - 1) / NW;
    const int r_lo = min(K, w * L), n = min(K, r_lo + L) - r_lo;
    // The knot times of the spacings h_i = t_{i+1} - t_i that wave 0 forms for
    // the factor (i = lane, lane + 64, ..., clamped), requested first: a wave's
    // loads complete in order, so the factor waits only for these and starts
    // while the knot values and the upload requested below are in flight.
    double ta[R], tb[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int i = min(lane + j * kWave, K - 2);
        ta[j] = t[i];
        tb[j] = t[i + 1];
    }
    // the workgroup's share of the upload: each lane's first word requested
    // now (host memory is far) and stored at the end
    long long up_x = -1, up_end = 0;
    uint4 up_w = make_uint4(0u, 0u, 0u, 0u);
    if (jb.up_bytes > 0) {
        const long long words = (jb.up_bytes + 15) / 16;
        const long long per = (words + jb.amp_blocks - 1) / jb.amp_blocks;
        up_end = min(words, (long long)blk * per + per);
        up_x = (long long)blk * per + tid;
        if (up_x < up_end) up_w = jb.up_src[up_x];
    }
    // knot values y_{r_lo - 2 + j} (clamped to the grid), all in flight
    double yv[LC + 4];
    {
        const double *y = jb.amp + q;
        const size_t stride = 2 * (size_t)M;
#pragma unroll
        for (int j = 0; j < LC + 4; ++j) {
            const int i = min(max(r_lo - 2 + j, 0), K - 1);
            yv[j] = live ? y[(size_t)i * stride] : 0.0;
        }
    }
    // the knot times are taken here, after the loads above were issued (this
    // keeps the compiler from moving their loads into the branch below)
#pragma unroll
    for (int j = 0; j < R; ++j) asm volatile("" : "+v"(ta[j]), "+v"(tb[j]));
    if (w == 0) {
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (lane + j * kWave < K - 1) hs[lane + j * kWave] = tb[j] - ta[j];
        lds_wave_sync();
        fit_factor_wave<R>(hs, K, invd, wv, bv);
    }
    __syncthreads();
    // row-wise constants of row r_lo + c in lane c
    double c_al = 0.0, c_be = 0.0, c_bv = 0.0, c_wv = 0.0, c_ih = 0.0;
    if (lane < n) {
        const int r = r_lo + lane;
        double P, Q;
        int a;
        if (r == 0) {
            const double h0 = hs[0], h1 = hs[1];
            P = (h0 + 2.0 * (h0 + h1)) * h1 / (h0 + h1);
            Q = h0 * h0 / (h0 + h1);
            a = 0;
        } else if (r < K - 1) {
            P = 3.0 * hs[r];
            Q = 3.0 * hs[r - 1];
            a = r - 1;
        } else {
            const double ha = hs[K - 3], hb = hs[K - 2];
            P = hb * hb / (ha + hb);
            Q = (2.0 * (ha + hb) + hb) * ha / (ha + hb);
            a = K - 3;
        }
        const double id = invd[r];
        c_al = id * P / hs[a];
        c_be = id * Q / hs[a + 1];
        c_bv = bv[r];
        c_wv = wv[r];
        c_ih = r < K - 1 ? 1.0 / hs[r] : 0.0;
    }
    // chunk products: F in lane c over rows r_lo .. r_lo + c, B over
    // r_lo + c .. r_lo + n - 1 (log-step scans; identities past the chunk)
    double c_F = lane < n ? -c_bv : 1.0, c_B = lane < n ? -c_wv : 1.0;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const double fo = __shfl_up(c_F, d), bo = __shfl_down(c_B, d);
        if (lane >= d) c_F *= fo;
        if (lane + d < kWave) c_B *= bo;
    }
    // forward chain of the chunk from a zero start
    double gv[LC];
    double g = 0.0;
#pragma unroll
    for (int c = 0; c < LC; ++c) {
        if (c < n) {
            const int r = r_lo + c;
            // y_a, y_{a+1}, y_{a+2}: yv[c+1 ..] on interior rows (a = r - 1),
            // one further on row 0 (a = 0) and one back on row K - 1 (a = K - 3)
            const int sh = r == 0 ? 1 : (r == K - 1 ? -1 : 0);
            const double y0 = sh > 0 ? yv[c + 2] : (sh < 0 ? yv[c] : yv[c + 1]);
            const double y1 = sh > 0 ? yv[c + 3] : (sh < 0 ? yv[c + 1] : yv[c + 2]);
            const double y2 = sh > 0 ? yv[c + 4] : (sh < 0 ? yv[c + 2] : yv[c + 3]);
            const double v = fma(lane_value(c_al, c), y1 - y0, lane_value(c_be, c) * (y2 - y1));
            g = fma(-lane_value(c_bv, c), g, v);
            gv[c] = g;
        }
    }
    cf[w * kWave + lane] = g;
    if (lane == max(n, 1) - 1) fe[w] = n > 0 ? c_F : 1.0;
    __syncthreads();
    {
        // forward value entering the chunk, then the back chain of the chunk
        // on the joined forward values
        double G = 0.0;
        for (int cc = 0; cc < w; ++cc) G = fma(fe[cc], G, cf[cc * kWave + lane]);
        double sl = 0.0;
#pragma unroll
        for (int c = LC - 1; c >= 0; --c) {
            if (c < n) {
                const double gj = fma(lane_value(c_F, c), G, gv[c]);
                sl = fma(-lane_value(c_wv, c), sl, gj);
                gv[c] = sl;
            }
        }
        cb[w * kWave + lane] = sl;
        if (lane == 0) bs0[w] = n > 0 ? c_B : 1.0;
    }
    __syncthreads();
    // slope entering the chunk from above, s_{r_lo + n}
    double Sx = 0.0;
    for (int cc = NW - 1; cc > w; --cc) Sx = fma(bs0[cc], Sx, cb[cc * kWave + lane]);
#pragma unroll
    for (int c = 0; c < LC; ++c)
        if (c < n) gv[c] = fma(lane_value(c_B, c), Sx, gv[c]);
    // coefficients of the chunk's intervals r = r_lo + c <= K - 2: stored
    // directly in the [K-1][4][2M] layout (each store 512 contiguous bytes);
    // in the [K-1][M][4][2] layout through the wave's 2 KB LDS slot, so that
    // the wave stores each interval's run of 32 modes as two 1 KB pieces
    const bool pm = jb.acoef_pmajor != 0;
    const int k0 = blk * (kFitSeriesPerBlock / 2);
    const int ns = min(kFitSeriesPerBlock, 2 * M - blk * kFitSeriesPerBlock);
    double *slot = bs0 + NW + (size_t)w * 4 * kWave;
#pragma unroll
    for (int c = 0; c < LC; ++c) {
        const int r = r_lo + c;
        if (c < n && r <= K - 2) {
            const double y0 = yv[c + 2], y1 = yv[c + 3];
            // s_{r+1}: past the chunk's last row, the next chunk's first
            const double s1 = (c + 1 < LC && c + 1 < n) ? gv[c + 1 < LC ? c + 1 : c] : Sx;
            const double s0 = gv[c];
            const double ir = lane_value(c_ih, c);
            const double dr = (y1 - y0) * ir;
            const double c2 = (3.0 * dr - 2.0 * s0 - s1) * ir, c3 = (s0 + s1 - 2.0 * dr) * (ir * ir);
            if (pm) {
                if (live) {
                    double *orow = jb.acoef + (size_t)r * 8 * M + q;
                    const size_t ps = 2 * (size_t)M;
                    orow[0] = y0;
                    orow[ps] = s0;
                    orow[2 * ps] = c2;
                    orow[3 * ps] = c3;
                }
            } else {
                double *d = slot + 8 * (lane >> 1) + (lane & 1);
                d[0] = y0;
                d[2] = s0;
                d[4] = c2;
                d[6] = c3;
                lds_wave_sync();
                const double2 *rd = (const double2 *)slot;
                double2 *dst = (double2 *)(jb.acoef + ((size_t)r * M + k0) * 8);
                const double2 v0 = rd[lane], v1 = rd[kWave + lane];
                if (lane < 2 * ns) dst[lane] = v0;               // run of 4 ns doubles
                if (kWave + lane < 2 * ns) dst[kWave + lane] = v1;
                lds_wave_sync();
            }
        }
    }
    if (up_x >= 0) {
        if (up_x < up_end) jb.up_dst[up_x] = up_w;
        for (long long x = up_x + (long long)blockDim.x; x < up_end; x += blockDim.x)
            jb.up_dst[x] = jb.up_src[x];
    }
}

// Workgroups 0 .. n_ph-1 fit the phases, the rest the amplitude series; t:
// the knot times.
template <int R>
__device__ __forceinline__ void fit_body(const FitJob &jb, const double *t, double *lds) {
    if ((int)blockIdx.x < jb.n_ph) {
        fit_phase_dd<R>(jb, t, blockIdx.x, lds);
        return;
    }
    const int blk = (int)blockIdx.x - jb.n_ph;
    if (blk >= jb.amp_blocks) return;
    if constexpr (R > 0)
        fit_amplitudes_staged<R>(jb, t, blk, lds);
    else
        fit_amplitudes_stream(jb, t, blk, lds);
}

// Single-request fit.  Grids of at most R kWave knots also arrive in the
// launch's arguments (kt), so no workgroup waits on the host-memory staging
// slot for them.  R = 2 up to 128 knots, 3 up to 192 (whose chunks of 48 rows take
// half as many registers again): 137 knots, 611 modes 45 -> 25 us.
template <int R>
__global__ __launch_bounds__(256) void fit_kernel(FitJob jb, FitKnots<R> kt) {
    extern __shared__ double lds_fit[];
    fit_body<R>(jb, R > 0 ? kt.t : jb.t, lds_fit);
}

// R: the longest grids of the batch (its other grids take their own form).
template <int R>
__global__ __launch_bounds__(256) void fit_batch_kernel(const FitJob *jobs) {
    extern __shared__ double lds_fit[];
    const FitJob jb = jobs[blockIdx.y];
    if (jb.K <= 2 * kWave)
        fit_body<2>(jb, jb.t, lds_fit);
    else if (R == 3 || (R == 0 && jb.K <= kFitStageKnots))
        fit_body<3>(jb, jb.t, lds_fit);
    else if constexpr (R == 0)
        fit_body<0>(jb, jb.t, lds_fit);
}

// ===========================================================================
// Prepare stage.
// ===========================================================================

// starts[i] = min{ j in [0, n] : t_start + j dt >= t_i } (binary64 times).
__device__ long long dev_interval_start(double ti, double t_start, double dt, long long n) {
    double est = ceil((ti - t_start) / dt);
    long long j;
    if (!(est > 0.0)) j = 0;
    else if (est >= (double)n) j = n;
    else j = (long long)est;
    while (j > 0 && dev_sample_time(t_start, dt, j - 1) >= ti) --j;
    while (j < n && dev_sample_time(t_start, dt, j) < ti) ++j;
    return j;
}

// Samples of part p that lie in interval i, [lo, hi), and where its short
// tiles start (every tile lies inside one interval and one part).
struct PieceRange {
    long long lo, hi, split;
};

__device__ __forceinline__ PieceRange piece_range(long long a, long long e, long long n,
                                                  int parts, int p, long long short_len) {
    const long long b0 = part_begin(n, parts, p), b1 = part_begin(n, parts, p + 1);
    PieceRange r;
    r.lo = max(a, b0);
    r.hi = max(r.lo, min(e, b1));
    const long long s0 = b1 - min(b1 - b0, short_len);
    r.split = min(r.hi, max(r.lo, s0));
    return r;
}

// ceil(a / b) for 0 <= a < 2^53 and b > 0, exactly: a binary64 estimate (off
// by at most one) corrected with integer products, instead of the long
// instruction sequence of a 64-bit integer division.
__device__ __forceinline__ long long ceil_div_pos(long long a, int b) {
    long long q = (long long)((double)a / (double)b);
    if (q * b < a) ++q;
    if (q > 0 && (q - 1) * b >= a) --q;
    return q;
}

__device__ int piece_tiles(const PrepJob &jb, int p, int i) {
    const PieceRange r = piece_range(jb.starts[i], jb.starts[i + 1], jb.n, jb.parts, p,
                                     jb.short_len);
    return (int)(ceil_div_pos(r.split - r.lo, jb.tile) +
                 ceil_div_pos(r.hi - r.split, jb.short_tile));
}

__device__ void prep_intervals(const PrepJob &jb) {
    const int tid = threadIdx.x;
    const int K = jb.K;
    for (int i = tid; i < K; i += blockDim.x) {
        long long s;
        if (i == 0) s = 0;
        else if (i == K - 1) s = jb.n;
        else s = dev_interval_start(jb.t[i], jb.t_start, jb.dt, jb.n);
        jb.starts[i] = s;
    }
    __syncthreads();
    // per part (one wave each): tiles per interval and their exclusive prefix,
    // 64 intervals at a time by a shuffle scan
    const int P = K - 1;
    const int lane = tid & (kWave - 1), waves = blockDim.x / kWave;
    for (int pt = tid / kWave; pt < jb.parts; pt += waves) {
        int *tp = jb.tile_pref + (size_t)pt * K;
        int run = 0;
        for (int c0 = 0; c0 < P; c0 += kWave) {
            const int i = c0 + lane;
            const int cnt = (i < P) ? piece_tiles(jb, pt, i) : 0;
            int incl = cnt;
            for (int off = 1; off < kWave; off <<= 1) {
                const int v = __shfl_up(incl, off);
                if (lane >= off) incl += v;
            }
            if (i < P) tp[i] = run + incl - cnt;
            run += __shfl(incl, kWave - 1);
        }
        if (lane == 0) tp[P] = run;
    }
}

// Harmonic weight of one contributor: -2Y_lm for a listed mode and
// (-1)^{l+k} -2Y_{l,-m} for its mirror (Eq. (9); k = 0 in Schwarzschild).
__device__ void prep_harmonic(const PrepJob &jb, int e) {
    if (e >= jb.n_src) return;
    const int2 s = jb.term_src[e];
    const int l = s.y & 255, m = (s.y >> 8) & 255, mir = (s.y >> 16) & 1;
    const int kp = ((s.y >> 17) & 127) - 64;
    double yr, yi;
    if (!mir) {
        few_swsh_m2(l, m, jb.theta, jb.phi, &yr, &yi);
    } else {
        few_swsh_m2(l, -m, jb.theta, jb.phi, &yr, &yi);
        if ((l + kp) & 1) {
            yr = -yr;
            yi = -yi;
        }
    }
    jb.ybuf[e] = make_double2(yr, yi);
}

// Fold the l-sum for one (interval, term) pair:
//   C_term = scale * sum_e Y_e * (A_k or conj(A_k)),
// rescaled to u = x / h_i (coefficient p times h_i^p).
template <typename Real>
__device__ void fold_pair(const PrepJob &jb, int i, int term) {
    double acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = 0.0;
    auto add = [&](double2 w, int2 src, const double *a) {
        const double sgn = ((src.y >> 16) & 1) ? -1.0 : 1.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double ar = a[2 * q], ai = sgn * a[2 * q + 1];
            acc[2 * q] += w.x * ar - w.y * ai;
            acc[2 * q + 1] += w.x * ai + w.y * ar;
        }
    };
    // acoef [K-1][M][4][2] (vector-path requests): the 8 values of mode k on
    // interval i are contiguous, one 64-byte segment per contributor
    const double *arow = jb.acoef + (size_t)i * 8 * jb.M;
    auto load8 = [&](int k, double *a) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double2 v = *(const double2 *)(arow + 8 * (size_t)k + 2 * p);
            a[2 * p] = v.x;
            a[2 * p + 1] = v.y;
        }
    };
    const int ea = jb.term_ptr[term], eb = jb.term_ptr[term + 1];
    int e = ea;
    // four contributors at a time: their weights, indices and coefficient rows
    // are all loaded before any is added (in contributor order, as one by one)
    for (; e + 4 <= eb; e += 4) {
        double2 w[4];
        int2 src[4];
        double av[4][8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w[j] = jb.ybuf[e + j];
            src[j] = jb.term_src[e + j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) load8(src[j].x, av[j]);
#pragma unroll
        for (int j = 0; j < 4; ++j) add(w[j], src[j], av[j]);
    }
    for (; e < eb; ++e) {
        double a[8];
        load8(jb.term_src[e].x, a);
        add(jb.ybuf[e], jb.term_src[e], a);
    }
    const double h = jb.t[i + 1] - jb.t[i];
    double f = jb.scale;
    // terms are stored in reverse order (position n_terms - 1 - term), so the
    // summation walks each segment from its highest n upwards in memory
    Real *dst = (Real *)jb.table + ((size_t)i * jb.n_terms + (jb.n_terms - 1 - term)) * 8;
    if (jb.scale_im == 0.0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            dst[2 * q] = (Real)(acc[2 * q] * f);
            dst[2 * q + 1] = (Real)(acc[2 * q + 1] * f);
            f *= h;
        }
    } else {
        // complex overall factor (scale, scale_im) (the detector-frame rotation)
        double g = jb.scale_im;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            dst[2 * q] = (Real)(acc[2 * q] * f - acc[2 * q + 1] * g);
            dst[2 * q + 1] = (Real)(acc[2 * q] * g + acc[2 * q + 1] * f);
            f *= h;
            g *= h;
        }
    }
}

// Prepare and fold in one launch.  Workgroup 0 computes the interval starts
// and the per-part tile prefixes; workgroup 1 + g folds the group of
// fold_terms consecutive terms starting at g fold_terms over every interval
// (fold_terms is chosen so that a group is about one (interval, term) pair per
// lane).
// The group first forms the harmonic weight of each of its contributors (each
// contributor belongs to one term, so each weight is formed once, by the one
// workgroup that reads it), then folds.  Consecutive lanes take consecutive
// terms of one interval, so table stores are contiguous.
template <typename Real>
__device__ void prepare_body(const PrepJob &jb, int b) {
    if (b == 0) {
        prep_intervals(jb);
        return;
    }
    const int t0 = (b - 1) * jb.fold_terms;
    if (t0 >= jb.n_terms) return;                   // uniform per workgroup
    const int nt = min(jb.fold_terms, jb.n_terms - t0);
    const int e0 = jb.term_ptr[t0], e1 = jb.term_ptr[t0 + nt];
    for (int e = e0 + (int)threadIdx.x; e < e1; e += blockDim.x) prep_harmonic(jb, e);
    __syncthreads();                                // weights visible to the workgroup
    const int pairs = (jb.K - 1) * nt;
    for (int q = threadIdx.x; q < pairs; q += blockDim.x)
        fold_pair<Real>(jb, q / nt, t0 + q % nt);
}

template <typename Real>
__global__ __launch_bounds__(256) void prepare_kernel(PrepJob jb) {
    prepare_body<Real>(jb, blockIdx.x);
}

template <typename Real>
__global__ __launch_bounds__(256) void prepare_batch_kernel(const PrepJob *jobs) {
    const PrepJob jb = jobs[blockIdx.y];
    prepare_body<Real>(jb, blockIdx.x);
}

// ===========================================================================
// Summation stage.  No contraction: every sample goes through the same rounded
// operations whatever the tile shape, so results do not depend on tiling.
// ===========================================================================
#pragma clang fp contract(off)

// One reduced phase at one sample (in [-pi, pi]).  c: the interval's [4][2]
// double-double cubic of that phase.
template <bool DD>
__device__ __forceinline__ double phase_eval(const FEW_AS4 double *c, dd x) {
    if (DD) {
        dd v = dd_make(c[6], c[7]);
        v = dd_add(dd_mul(v, x), dd_make(c[4], c[5]));
        v = dd_add(dd_mul(v, x), dd_make(c[2], c[3]));
        v = dd_mul(v, x);
        v = dd_add(v, dd_make(c[0], c[1]));
        return dd_reduce_2pi(v).hi;
    }
    const double xx = x.hi;
    const double v = fma(fma(fma(c[6], xx, c[4]), xx, c[2]), xx, c[0]);
    return d_reduce_2pi(v);
}

// One phase at one sample, not reduced: the interval's binary64 cubic (the
// leading parts of the double-double coefficients) at offset x.
__device__ __forceinline__ double phase_raw(const FEW_AS4 double *c, double x) {
    return fma(fma(fma(c[6], x, c[4]), x, c[2]), x, c[0]);
}

// e^{-i a} for a reduced phase a in [-pi, pi] (binary64): the binary32 path
// rounds a to binary32 and takes the binary32 sincos (harmonics are binary32
// there), the binary64 path the binary64 one.
template <typename Real>
__device__ __forceinline__ void unit_phasor(double a, Real *re, Real *im) {
    if constexpr (sizeof(Real) == 4) {
        float sn, cs;
        sincosf((float)a, &sn, &cs);
        *re = cs;
        *im = -sn;
    } else {
        double sn, cs;
        sincos(a, &sn, &cs);
        *re = cs;
        *im = -sn;
    }
}

// Per-lane state of SL samples of one tile.  NP = 3 (generic Kerr) adds the
// polar phase and e^{-i Phi_theta}.
template <typename Real, int SL, int NP>
struct LaneState {
    static constexpr int ST = NP == 3 ? SL : 1;
    Real u[SL], fr[SL], fi[SL], er[SL], ei[SL], tr[ST], ti[ST];
    double pf[SL], pr[SL], pt[ST];
    long long jj[SL];
    Real hr[SL], hq[SL], cr[SL], cq[SL], zr[SL], zi[SL];
    Real gr[SL], gi[SL];    // binary32: sum of the closed term groups
    int pm, pk, pn;
};

// Segment record x = m + 256 k (k = 0 in Schwarzschild).
__device__ __forceinline__ int seg_k(int x) { return (x + 128) >> 8; }

// Knot interval of tile `local` (tp: tiles before each interval of one part).
__device__ __forceinline__ int tile_interval(const FEW_AS4 int *tp, int K, int local) {
    int lo = 0, hi = K - 2;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tp[mid] <= local) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Per-sample setup: samples j0 + s * 64 + lane (s < SL), valid below j1.
template <typename Real, int SL, bool DD, int NP>
__device__ __forceinline__ void lane_setup(LaneState<Real, SL, NP> &L, const SumJob &jb, int iv,
                                           long long j0, long long j1) {
    const int lane = threadIdx.x & (kWave - 1);
    const FEW_AS4 double *tk = cptr(jb.t);
    const double ti = tk[iv];
    const double inv_h = 1.0 / (tk[iv + 1] - ti);
    const FEW_AS4 double *pc = cptr(jb.pcoef) + (size_t)iv * 8 * NP;   // Phi_phi, Phi_r (, Phi_theta)
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        long long j = j0 + s * kWave + lane;
        L.jj[s] = j;
        if (j >= j1) j = j1 - 1;
        const double tj = dev_sample_time(jb.t_start, jb.dt, j);
        const dd x = two_sum(tj, -ti);
        L.pf[s] = phase_eval<DD>(pc, x);
        L.pr[s] = phase_eval<DD>(pc + 8, x);
        L.u[s] = (Real)(x.hi * inv_h);
        unit_phasor<Real>(L.pf[s], &L.er[s], &L.ei[s]);
        unit_phasor<Real>(L.pr[s], &L.fr[s], &L.fi[s]);
        if constexpr (NP == 3) {
            L.pt[s] = phase_eval<DD>(pc + 16, x);
            unit_phasor<Real>(L.pt[s], &L.tr[s], &L.ti[s]);
        }
        L.hr[s] = L.hq[s] = L.cr[s] = L.cq[s] = (Real)0;
        L.zr[s] = L.zi[s] = (Real)0;
        L.gr[s] = L.gi[s] = (Real)0;
    }
    L.pm = INT_MIN / 2;
    L.pk = INT_MIN / 2;
    L.pn = INT_MIN / 2;
}

// The 8 coefficients of one term: scalar loads from the constant address space,
// or two 16-byte LDS reads (every lane of a wave reads the same address, so the
// LDS broadcasts).
template <typename Real>
__device__ __forceinline__ void load_term(const FEW_AS4 Real *cp, Real *c) {
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = cp[i];
}

__device__ __forceinline__ void load_term(const float *cp, float *c) {
    const float4 a = *(const float4 *)cp;
    const float4 b = *(const float4 *)(cp + 4);
    c[0] = a.x; c[1] = a.y; c[2] = a.z; c[3] = a.w;
    c[4] = b.x; c[5] = b.y; c[6] = b.z; c[7] = b.w;
}

// One Horner step over n for every sample of the lane: S <- S f + C_n(u),
// with C_n's eight coefficients (c0r, c0i, ..., c3i) in c.  Binary32
// (coefficients in VGPRs) evaluates C_n(u) by Horner in u apart from the
// recurrence, leaving two dependent FMAs per term on it; binary64
// (coefficients in SGPRs, one scalar operand per instruction) chains all five
// FMAs of each component into the recurrence.
template <typename Real, int SL, int NP>
__device__ __forceinline__ void term_step(const LaneState<Real, SL, NP> &L, Real *sr, Real *si,
                                          const Real *c) {
    const Real c0r = c[0], c0i = c[1], c1r = c[2], c1i = c[3];
    const Real c2r = c[4], c2i = c[5], c3r = c[6], c3i = c[7];
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const Real u = L.u[s];
        Real nr, ni;
        if constexpr (sizeof(Real) == 4) {
            // coefficients in VGPRs: cubic first, two FMAs on the recurrence
            const Real pr = fmar(fmar(fmar(c3r, u, c2r), u, c1r), u, c0r);
            const Real pi = fmar(fmar(fmar(c3i, u, c2i), u, c1i), u, c0i);
            nr = fmar(sr[s], L.fr[s], fmar(-si[s], L.fi[s], pr));
            ni = fmar(sr[s], L.fi[s], fmar(si[s], L.fr[s], pi));
        } else {
            // coefficients in SGPRs: one scalar operand per FMA
            const Real u2 = u * u, u3 = u2 * u;
            nr = fmar(sr[s], L.fr[s], c0r);
            nr = fmar(-si[s], L.fi[s], nr);
            nr = fmar(u, c1r, nr);
            nr = fmar(u2, c2r, nr);
            nr = fmar(u3, c3r, nr);
            ni = fmar(sr[s], L.fi[s], c0i);
            ni = fmar(si[s], L.fr[s], ni);
            ni = fmar(u, c1i, ni);
            ni = fmar(u2, c2i, ni);
            ni = fmar(u3, c3i, ni);
        }
        sr[s] = nr;
        si[s] = ni;
    }
}

// One segment: seed e^{-i(m Phi_phi + k Phi_theta + n_lo Phi_r)} (chained
// from the previous segment's by e^{-i Phi_phi} when only m steps by one, or by
// e^{-i Phi_theta} when only k does, at the same n_lo; else one sincos),
// Horner over its terms in f = e^{-i Phi_r} from the highest n down,
//   S <- S f + C_n(u),  C_n(u) = c0 + c1 u + c2 u^2 + c3 u^3,
// then h += seed * S (Kahan-compensated when COMP).  `last` points at the 8
// values (c0r, c0i, ..., c3i) of the segment's highest-n term; the lower-n
// terms follow it at a stride of 8 (the table stores terms in reverse order,
// so the walk runs upward in memory and the loads of two unrolled terms share
// one base register with immediate offsets).
template <typename Real, int SL, bool COMP, int NP, typename Ptr>
__device__ __forceinline__ void seg_step(LaneState<Real, SL, NP> &L, const int4 S, Ptr last) {
    const int k = NP == 3 ? seg_k(S.x) : 0;
    const int m = S.x - 256 * k;
    const bool step_m = m == L.pm + 1 && k == L.pk && S.y == L.pn;
    const bool step_k = NP == 3 && m == L.pm && k == L.pk + 1 && S.y == L.pn;
    if (step_m || step_k) {
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            Real gr, gi;
            if constexpr (NP == 3) {
                gr = step_k ? L.tr[s] : L.er[s];
                gi = step_k ? L.ti[s] : L.ei[s];
            } else {
                gr = L.er[s];
                gi = L.ei[s];
            }
            const Real a = L.zr[s] * gr - L.zi[s] * gi;
            const Real b = L.zr[s] * gi + L.zi[s] * gr;
            L.zr[s] = a;
            L.zi[s] = b;
        }
    } else {
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            double ph = (double)m * L.pf[s] + (double)S.y * L.pr[s];
            if constexpr (NP == 3) ph = ph + (double)k * L.pt[s];
            unit_phasor<Real>(d_reduce_2pi(ph), &L.zr[s], &L.zi[s]);
        }
    }
    L.pm = m;
    L.pk = k;
    L.pn = S.y;
    Real sr[SL], si[SL];
#pragma unroll
    for (int s = 0; s < SL; ++s) sr[s] = si[s] = (Real)0;
    const int len = S.z;
    if constexpr (sizeof(Real) == 4) {
        // LDS operands: each pair of unrolled terms is read by four 16-byte
        // loads at immediate offsets from one base, waited on at once; the
        // other waves of the SIMD cover the latency.
#pragma unroll FEW_SEG_UNROLL
        for (int q = 0; q < len; ++q) {
            Real c[8];
            load_term(last + 8 * q, c);
            term_step<Real, SL, NP>(L, sr, si, c);
        }
    } else {
        // scalar-load operands: the next term is loaded into a second register
        // set while the current one is used, so each load has a term's FMAs
        // to return in (scalar loads may return out of order, so every wait is
        // for all of them); the last prefetch re-reads the last term, so it
        // stays in bounds.
        Ptr cp = last;
        Real c[8];
        load_term(cp, c);
#pragma unroll FEW_SEG_UNROLL
        for (int q = 0; q < len; ++q) {
            const Ptr np = (q + 1 < len) ? cp + 8 : cp;
            Real cn[8];
            load_term(np, cn);
            term_step<Real, SL, NP>(L, sr, si, c);
#pragma unroll
            for (int i = 0; i < 8; ++i) c[i] = cn[i];
            cp = np;
        }
    }
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const Real vr = L.zr[s] * sr[s] - L.zi[s] * si[s];
        const Real vi = L.zr[s] * si[s] + L.zi[s] * sr[s];
        if (COMP) {
            const Real yr = vr - L.cr[s];
            const Real tr = L.hr[s] + yr;
            L.cr[s] = (tr - L.hr[s]) - yr;
            L.hr[s] = tr;
            const Real yi = vi - L.cq[s];
            const Real ti2 = L.hq[s] + yi;
            L.cq[s] = (ti2 - L.hq[s]) - yi;
            L.hq[s] = ti2;
        } else {
            L.hr[s] += vr;
            L.hq[s] += vi;
        }
    }
}

// Value of the current (compensated) sum of sample s.
template <typename Real, int SL, bool COMP, int NP>
__device__ __forceinline__ void acc_value(const LaneState<Real, SL, NP> &L, int s, Real *re,
                                          Real *im) {
    *re = COMP ? L.hr[s] - L.cr[s] : L.hr[s];
    *im = COMP ? L.hq[s] - L.cq[s] : L.hq[s];
}

// Close a term group (binary32): add its value to the group total, restart
// the compensated sum, and make the next segment seed by sincos.
template <typename Real, int SL, bool COMP, int NP>
__device__ __forceinline__ void group_close(LaneState<Real, SL, NP> &L) {
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        Real vr, vi;
        acc_value<Real, SL, COMP, NP>(L, s, &vr, &vi);
        L.gr[s] = L.gr[s] + vr;
        L.gi[s] = L.gi[s] + vi;
        L.hr[s] = L.hq[s] = L.cr[s] = L.cq[s] = (Real)0;
    }
    L.pm = INT_MIN / 2;
    L.pk = INT_MIN / 2;
    L.pn = INT_MIN / 2;
}

// Final value of sample s: the group total (binary32, after the last group is
// closed) or the running sum (binary64).
template <typename Real, int SL, bool COMP, int NP>
__device__ __forceinline__ void lane_value(const LaneState<Real, SL, NP> &L, int s, Real *re,
                                           Real *im) {
    if constexpr (sizeof(Real) == 4) {
        *re = L.gr[s];
        *im = L.gi[s];
    } else {
        acc_value<Real, SL, COMP, NP>(L, s, re, im);
    }
}

template <typename Real, int SL, bool COMP, int NP>
__device__ __forceinline__ void lane_store(const LaneState<Real, SL, NP> &L, const SumJob &jb,
                                           long long j1) {
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        if (L.jj[s] < j1) {
            Real *o = (Real *)jb.out + 2 * L.jj[s];
            lane_value<Real, SL, COMP, NP>(L, s, &o[0], &o[1]);
        }
    }
}

// Inner-product epilogue: this lane's sums of Re(conj(d_j) h_j) and |h_j|^2
// over its valid samples, in binary64, with h_j exactly the value a store
// launch would write.
template <typename Real, int SL, bool COMP, int NP>
__device__ __forceinline__ double2 lane_inner(const LaneState<Real, SL, NP> &L,
                                              const SumJob &jb, long long j1) {
    double dh = 0.0, hh = 0.0;
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        if (L.jj[s] < j1) {
            Real re, im;
            lane_value<Real, SL, COMP, NP>(L, s, &re, &im);
            const Real *d = (const Real *)jb.data + 2 * L.jj[s];
            const double hr = re, hi = im, dr = d[0], di = d[1];
            dh = dh + (dr * hr + di * hi);
            hh = hh + (hr * hr + hi * hi);
        }
    }
    return make_double2(dh, hh);
}

// Sum over the 64 lanes of a wave by a fixed butterfly (every lane ends with
// the same bits: each step adds the same two values in either lane).
__device__ __forceinline__ double2 wave_sum(double2 v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        v.x = v.x + __shfl_xor(v.x, off);
        v.y = v.y + __shfl_xor(v.y, off);
    }
    return v;
}

// Wave tile (binary64 path): 64 x SL consecutive samples [j0, j1) of interval
// iv, coefficients read by scalar loads straight into SGPR operands.
template <typename Real, int SL, bool COMP, bool DD, int NP, bool INNER>
__device__ __forceinline__ double2 sum_wave_run(const SumJob &jb, int iv, long long j0,
                                                long long j1) {
    static_assert(sizeof(Real) == 8, "binary32 terms are read from LDS only");
    LaneState<Real, SL, NP> L;
    lane_setup<Real, SL, DD, NP>(L, jb, iv, j0, j1);
    const FEW_AS4 Real *tab = cptr((const Real *)jb.table) + (size_t)iv * jb.n_terms * 8;
    for (int g = 0; g < jb.n_segs; ++g) {
        const int4 S = load_uniform(jb.segs + g);
        seg_step<Real, SL, COMP, NP>(L, S, tab + (size_t)(jb.n_terms - S.w - S.z) * 8);
    }
    if constexpr (INNER) {
        return lane_inner<Real, SL, COMP, NP>(L, jb, j1);
    } else {
        lane_store<Real, SL, COMP, NP>(L, jb, j1);
        return make_double2(0.0, 0.0);
    }
}

// Wave tile `local` of part `pt` of a request (binary64 launches use long
// tiles only).
template <typename Real, bool COMP, bool DD, int NP, bool INNER>
__device__ __forceinline__ double2 sum_tile(const SumJob &jb, int pt, int local) {
    const FEW_AS4 int *tp = cptr(jb.tile_pref) + (size_t)pt * jb.K;
    if (local >= tp[jb.K - 1]) return make_double2(0.0, 0.0);
    const int iv = tile_interval(tp, jb.K, local);
    const FEW_AS4 long long *st = cptr(jb.starts);
    const PieceRange pr = piece_range(st[iv], st[iv + 1], jb.n, jb.parts, pt, 0);
    constexpr int LT = kWave * kSamplesPerLaneF64;
    const long long j0 = pr.lo + (long long)(local - tp[iv]) * LT;
    return sum_wave_run<Real, kSamplesPerLaneF64, COMP, DD, NP, INNER>(jb, iv, j0,
                                                                       min(j0 + LT, pr.hi));
}

// Workgroup tile (binary32 path): 4 waves x 64 x SL consecutive samples
// [base, j1) of interval iv.  The workgroup stages the interval's coefficients
// in LDS, one chunk of whole segments (at most kChunkTerms terms) at a time, and
// every wave reads each term with broadcast LDS loads into VGPRs: FMAs without
// scalar operands issue at twice the rate on gfx950.  Every lane of the
// workgroup reaches every barrier.
template <typename Real, int SL, bool COMP, bool DD, int NP, bool INNER>
__device__ __forceinline__ double2 sum_wg_run(const SumJob &jb, int iv, long long base,
                                              long long j1, Real *buf) {
    static_assert(sizeof(Real) == 4, "binary64 terms are read by scalar loads");
    constexpr int WT = kWave * SL;                  // samples per wave
    const int wave = threadIdx.x / kWave;
    // a wave past the end of a partial tile only helps stage coefficients
    const bool busy = base + (long long)wave * WT < j1;
    LaneState<Real, SL, NP> L;
    if (busy) lane_setup<Real, SL, DD, NP>(L, jb, iv, base + (long long)wave * WT, j1);
    const Real *tab = (const Real *)jb.table + (size_t)iv * jb.n_terms * 8;
    const FEW_AS4 int *ch = cptr(jb.chunks);
    for (int c = 0; c < jb.n_chunks; ++c) {
        const int g0 = ch[c], g1 = ch[c + 1];
        const int t0 = load_uniform(jb.segs + g0).w;
        const int4 Sl = load_uniform(jb.segs + g1 - 1);
        const int t1 = Sl.w + Sl.z;                 // terms [t0, t1), stored reversed
        const int nv = (t1 - t0) * 8 * (int)sizeof(Real) / 16;
        __syncthreads();                            // previous chunk fully consumed
        const float4 *src = (const float4 *)(tab + (size_t)(jb.n_terms - t1) * 8);
        float4 *dst = (float4 *)buf;
        for (int v = threadIdx.x; v < nv; v += blockDim.x) dst[v] = src[v];
        __syncthreads();
        if (busy) {
            for (int g = g0; g < g1; ++g) {
#pragma unroll
                for (int q = 0; q < kTermGroups - 1; ++q)
                    if (g == jb.grp[q]) group_close<Real, SL, COMP, NP>(L);
                const int4 S = load_uniform(jb.segs + g);
                seg_step<Real, SL, COMP, NP>(L, S, buf + (t1 - S.w - S.z) * 8);
            }
        }
    }
    if (!busy) return make_double2(0.0, 0.0);
    // close the last group, then any empty groups after it (each adds zero,
    // as in a term-split tile)
    group_close<Real, SL, COMP, NP>(L);
#pragma unroll
    for (int q = 0; q < kTermGroups - 1; ++q)
        if (jb.grp[q] == jb.n_segs) group_close<Real, SL, COMP, NP>(L);
    if constexpr (INNER) {
        return lane_inner<Real, SL, COMP, NP>(L, jb, j1);
    } else {
        lane_store<Real, SL, COMP, NP>(L, jb, j1);
        return make_double2(0.0, 0.0);
    }
}

// Term-split tile (binary32): 64 x SL samples [base, j1) of interval iv, taken
// by all four waves; wave w sums term group w (segments [grp[w-1], grp[w])),
// staging it kSplitTerms terms (whole segments) at a time in its own quarter
// of the LDS buffer, so the waves need no barrier until they combine.  Each
// wave leaves its group value in its quarter; wave 0 adds the four in group
// order, starting from zero, exactly as a long tile closes its groups.  Needs
// every segment to fit a quarter (checked on the host).
template <typename Real, int SL, bool COMP, bool DD, int NP, bool INNER>
__device__ __forceinline__ double2 sum_wg_split(const SumJob &jb, int iv, long long base,
                                                long long j1, Real *buf) {
    static_assert(sizeof(Real) == 4, "term-split tiles are binary32 tiles");
    const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    LaneState<Real, SL, NP> L;
    lane_setup<Real, SL, DD, NP>(L, jb, iv, base, j1);
    const int gb = wave == 0 ? 0 : jb.grp[wave - 1];
    const int ge = wave == kTermGroups - 1 ? jb.n_segs : jb.grp[wave];
    Real *wb = buf + (size_t)wave * kSplitTerms * 8;
    const Real *tab = (const Real *)jb.table + (size_t)iv * jb.n_terms * 8;
    for (int g = gb; g < ge;) {
        // whole segments [g, h) with at most kSplitTerms terms
        const int t0 = load_uniform(jb.segs + g).w;
        int h = g, t1 = t0;
        while (h < ge) {
            const int4 S = load_uniform(jb.segs + h);
            if (S.w + S.z - t0 > kSplitTerms) break;
            t1 = S.w + S.z;
            ++h;
        }
        // terms [t0, t1) are stored reversed: one contiguous run
        const int nv = (t1 - t0) * 8 * (int)sizeof(Real) / 16;
        const float4 *src = (const float4 *)(tab + (size_t)(jb.n_terms - t1) * 8);
        float4 *dst = (float4 *)wb;
        for (int v = lane; v < nv; v += kWave) dst[v] = src[v];
        __builtin_amdgcn_wave_barrier();
        for (; g < h; ++g) {
            const int4 S = load_uniform(jb.segs + g);
            seg_step<Real, SL, COMP, NP>(L, S, wb + (t1 - S.w - S.z) * 8);
        }
        __builtin_amdgcn_wave_barrier();
    }
    // this wave's group value, next to its staging area
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        Real vr, vi;
        acc_value<Real, SL, COMP, NP>(L, s, &vr, &vi);
        wb[(s * kWave + lane) * 2] = vr;
        wb[(s * kWave + lane) * 2 + 1] = vi;
    }
    __syncthreads();
    if (wave != 0) return make_double2(0.0, 0.0);
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        Real gr = (Real)0, gi = (Real)0;
#pragma unroll
        for (int w = 0; w < kTermGroups; ++w) {
            const Real *v = buf + (size_t)w * kSplitTerms * 8 + (s * kWave + lane) * 2;
            gr = gr + v[0];
            gi = gi + v[1];
        }
        L.gr[s] = gr;
        L.gi[s] = gi;
    }
    if constexpr (INNER) {
        return lane_inner<Real, SL, COMP, NP>(L, jb, j1);
    } else {
        lane_store<Real, SL, COMP, NP>(L, jb, j1);
        return make_double2(0.0, 0.0);
    }
}

// Tile `local` of part `pt` of a request: the part's samples in its interval,
// [lo, hi), are covered by long tiles up to `split` and short tiles after it.
// The branch is uniform per workgroup.
template <typename Real, bool COMP, bool DD, int NP, bool INNER, bool SPLIT>
__device__ __forceinline__ double2 sum_wg_tile(const SumJob &jb, int pt, int local, Real *buf) {
    const FEW_AS4 int *tp = cptr(jb.tile_pref) + (size_t)pt * jb.K;
    if (local >= tp[jb.K - 1]) return make_double2(0.0, 0.0);
    const int iv = tile_interval(tp, jb.K, local);
    const FEW_AS4 long long *st = cptr(jb.starts);
    const PieceRange pr = piece_range(st[iv], st[iv + 1], jb.n, jb.parts, pt, jb.short_len);
    constexpr int LT = 4 * kWave * kSamplesPerLaneF32;
    constexpr int ST = 4 * kWave * kSamplesPerLaneShort;
    constexpr int XT = kWave * kSamplesPerLaneF32;   // term-split tile
    const int n_long = (int)((pr.split - pr.lo + LT - 1) / LT);
    const int r = local - tp[iv];
    if (r < n_long) {
        const long long base = pr.lo + (long long)r * LT;
        return sum_wg_run<Real, kSamplesPerLaneF32, COMP, DD, NP, INNER>(
            jb, iv, base, min(base + LT, pr.split), buf);
    } else if (SPLIT && jb.split) {
        const long long base = pr.split + (long long)(r - n_long) * XT;
        return sum_wg_split<Real, kSamplesPerLaneF32, COMP, DD, NP, INNER>(
            jb, iv, base, min(base + XT, pr.hi), buf);
    } else {
        const long long base = pr.split + (long long)(r - n_long) * ST;
        return sum_wg_run<Real, kSamplesPerLaneShort, COMP, DD, NP, INNER>(
            jb, iv, base, min(base + ST, pr.hi), buf);
    }
}

// Workgroups are numbered so that each of the 8 XCDs (which receive workgroups
// round-robin) works on one contiguous eighth of the range, i.e. on a few knot
// intervals whose coefficient tables stay in its own L2.
__device__ __forceinline__ int xcd_block_id() {
    const int nb = gridDim.x;                       // multiple of 8
    const int b = blockIdx.x;
    return (b & 7) * (nb >> 3) + (b >> 3);
}

__device__ __forceinline__ int xcd_wave_id() {
    return xcd_block_id() * (blockDim.x / kWave) + (threadIdx.x / kWave);
}

// Batched launch: job j owns slots [wave_base_j, wave_base_{j+1}).
__device__ __forceinline__ int find_job(const SumJob *jobs, int n_jobs, int w) {
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        const int base = *cptr(&jobs[mid].wave_base);
        if (base <= w) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ---- binary64: one wave per tile -------------------------------------------
// One request: workgroup b runs on XCD b mod 8 (workgroups are dealt to the
// XCDs in turn), so part b mod parts is that XCD's; its waves take the part's
// tiles in dispatch order.  `slots`: wave tiles per part.
// INNER: every wave writes its tile's partial sums (zero without a tile) to
// partial[b * 4 + wave].
template <typename Real, bool COMP, bool DD, int NP, bool INNER>
__global__ __launch_bounds__(256) FEW_F64_ATTR void sum_kernel(SumJob jb, int slots) {
    const int b = blockIdx.x;
    const int pt = b % jb.parts;
    const int w = __builtin_amdgcn_readfirstlane(
        (int)((b / jb.parts) * (blockDim.x / kWave) + threadIdx.x / kWave));
    double2 v = make_double2(0.0, 0.0);
    if (w < slots) v = sum_tile<Real, COMP, DD, NP, INNER>(jb, pt, w);
    if constexpr (INNER) {
        v = wave_sum(v);
        if ((threadIdx.x & (kWave - 1)) == 0)
            jb.partial[(size_t)b * (blockDim.x / kWave) + threadIdx.x / kWave] = v;
    }
}

template <typename Real, bool COMP, bool DD>
__device__ __forceinline__ void sum_slot(const SumJob *jobs, int n_jobs, int w) {
    const int jx = __builtin_amdgcn_readfirstlane(find_job(jobs, n_jobs, w));
    const SumJob jb = load_uniform(jobs + jx);
    sum_tile<Real, COMP, DD, 2, false>(jb, 0, w - jb.wave_base);
}

template <typename Real, bool COMP, bool DD>
__global__ __launch_bounds__(256) FEW_F64_ATTR void sum_batch_kernel(const SumJob *jobs, int n_jobs,
                                                        int slots) {
    const int w = __builtin_amdgcn_readfirstlane(xcd_wave_id());
    if (w >= slots) return;
    sum_slot<Real, COMP, DD>(jobs, n_jobs, w);
}

// Persistent variant: a fixed grid of waves pulls wave slots from one atomic
// counter until all `slots` are handed out; every wave then exits.
template <typename Real, bool COMP, bool DD>
__global__ __launch_bounds__(256) FEW_F64_ATTR void sum_persistent_kernel(const SumJob *jobs, int n_jobs,
                                                             int slots, unsigned *counter) {
    const int lane = threadIdx.x & (kWave - 1);
    for (;;) {
        unsigned v = 0;
        if (lane == 0) v = atomicAdd(counter, 1u);
        const int w = __builtin_amdgcn_readfirstlane((int)v);
        if (w >= slots) break;
        sum_slot<Real, COMP, DD>(jobs, n_jobs, w);
    }
}

// ---- binary32: one workgroup per tile ---------------------------------------
// One request: workgroup b runs on XCD b mod 8, takes part b mod parts and
// that part's tiles in dispatch order, so each XCD reads the coefficients of its
// own intervals and ends on its short tiles while its last long tiles finish.
// `slots`: tiles per part.
// INNER: every workgroup writes its tile's partial sums (zero without a tile)
// to partial[b], adding its four waves in order.
template <typename Real, bool COMP, bool DD, int NP, bool INNER>
__global__ __launch_bounds__(256) FEW_SUM_ATTR void sum_wg_kernel(SumJob jb, int slots) {
    extern __shared__ float4 sum_lds[];
    const int b = blockIdx.x;
    const int local = b / jb.parts;     // < slots: the grid is parts x slots
    double2 v = sum_wg_tile<Real, COMP, DD, NP, INNER, true>(jb, b % jb.parts, local,
                                                       (Real *)sum_lds);
    if constexpr (INNER) {
        __shared__ double2 red[4];
        v = wave_sum(v);
        if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            double2 t = red[0];
            for (int w = 1; w < (int)(blockDim.x / kWave); ++w) {
                t.x = t.x + red[w].x;
                t.y = t.y + red[w].y;
            }
            jb.partial[b] = t;
        }
    }
    (void)slots;
}

template <typename Real, bool COMP, bool DD>
__device__ __forceinline__ void sum_wg_slot(const SumJob *jobs, int n_jobs, int b, Real *buf) {
    const int jx = __builtin_amdgcn_readfirstlane(find_job(jobs, n_jobs, b));
    const SumJob jb = load_uniform(jobs + jx);
    sum_wg_tile<Real, COMP, DD, 2, false, false>(jb, 0, b - jb.wave_base, buf);
}

template <typename Real, bool COMP, bool DD>
__global__ __launch_bounds__(256) void sum_wg_batch_kernel(const SumJob *jobs, int n_jobs,
                                                           int slots) {
    extern __shared__ float4 sum_lds[];
    const int b = xcd_block_id();
    if (b >= slots) return;
    sum_wg_slot<Real, COMP, DD>(jobs, n_jobs, b, (Real *)sum_lds);
}

// Persistent variant: workgroups pull tile slots from one atomic counter
// (lane 0 draws, the slot is broadcast through LDS) until all are handed out.
template <typename Real, bool COMP, bool DD>
__global__ __launch_bounds__(256) void sum_wg_persistent_kernel(const SumJob *jobs,
                                                                int n_jobs, int slots,
                                                                unsigned *counter) {
    extern __shared__ float4 sum_lds[];
    __shared__ int slot;
    for (;;) {
        if (threadIdx.x == 0) slot = (int)atomicAdd(counter, 1u);
        __syncthreads();
        const int b = slot;
        __syncthreads();
        if (b >= slots) break;
        sum_wg_slot<Real, COMP, DD>(jobs, n_jobs, b, (Real *)sum_lds);
    }
}

// ===========================================================================
// Matrix-core summation (binary32 output).  See the shape constants in
// few_internal.h: per knot interval and power p of u, the product of the
// coefficient matrix (rows: the real and imaginary part of each signed m;
// columns: (n, re/im)) with the matrix of harmonics (Re f^|n|, Im f^|n|) over
// the samples, f = e^{-i Phi_r}, on fp16 hi/lo operands with fp32
// accumulation; the sum over p is a Horner recurrence in v = 2 u - 1 (or one
// step within a block of samples) on the accumulators, and the rows are combined with e^{-i m Phi_phi}.
// ===========================================================================
typedef _Float16 mf_half8 __attribute__((ext_vector_type(8)));
typedef float mf_float4 __attribute__((ext_vector_type(4)));

// Fold and pack for the matrix-core path: workgroup 0 computes the interval
// starts and tile prefixes; each other workgroup folds one interval iv for
// one row tile mt (rows 8 mt .. 8 mt + 7, the signed m values m_r; numbering
// below) and writes its part of the operand table.
//
// Fold (Eqs. (9)-(10) for fixed viewing angles, Sec. IV): every term (m_r, n)
// is C = scale sum_contributors w A, with w = -2Y_{l, m_r} for a listed mode
// and (-1)^l -2Y_{l, m_r} for the mirror of a listed mode (m_r = -m, the
// amplitude conjugated), and the cubic written in v = 2 x / h_i - 1.
// The weights depend on (l, m_r) only, so the workgroup forms them once per
// row and l.  The folded values stay in LDS.
//
// Pack.  Row r is the pair of matrix rows 2r (real part) and 2r + 1
// (imaginary part).  For power p, column (a, c) multiplies Re w (c = 0) or
// Im w (c = 1), w = f^a, a = |n|.  The terms n = a and n = -a of the row
// (coefficients P and Q) contribute P w + Q conj(w) =
// ((Re P + Re Q) Re w + (Im Q - Im P) Im w) +
// i ((Im P + Im Q) Re w + (Re P - Re Q) Im w),
// so row 2r holds (Re P + Re Q, Im Q - Im P) and row 2r + 1 holds
// (Im P + Im Q, Re P - Re Q) (Q = 0 for a = 0).  Each pair of rows (signed m
// rows 2j and 2j + 1, which one lane of the product holds) is scaled by
// 2^-E, E the exponent of the pair's largest |coefficient| on the interval
// (so scaled values stay below 2), and stored in binary32; the summation cuts
// the values into fp16 hi and lo parts.  (One scale per interval would save
// the sum's multiplies, but the lo parts of the small rows then fall into fp16
// subnormals: error 5.1e-7 against 4.5e-7 on the one-year case.)  Layout, per
// interval: [mt][p][t][lane 64][8 values], lane l's operand fragment of
// v_mfma_f32_16x16x32_f16: matrix row l % 16 of the tile, columns
// a = 16 t + 4 (l / 16) + i / 2 and c = i % 2 for value i.  MfInfo holds 2^E
// and the largest |scaled value| of every fragment (mt, p, t), from which the
// summation decides which products a fragment needs (found as bit patterns: a
// NaN counts as the largest value, so it is never left out).
constexpr int kFoldPackThreads = 512;
constexpr int kFoldSegs = 64;                       // segments of a row tile kept in LDS

__device__ void fold_pack_body(const PrepJob &jb, int b) {
    if (b == 0) {
        prep_intervals(jb);
        return;
    }
    // workgroup 1 + 8 (kMfMT (iv / 8) + mt) + iv % 8 folds row tile mt of
    // interval iv: the tiles of one interval are 8 workgroups apart and so run
    // on one XCD (workgroup b runs on XCD b mod 8), whose L2 then serves the
    // coefficient rows that several tiles read (a mode's own and mirror terms)
    const int c = b - 1, q = c >> 3;
    const int mt = q % kMfMT, iv = 8 * (q / kMfMT) + (c & 7);
    if (iv >= jb.K - 1) return;                     // uniform per workgroup
    constexpr int NL = kMaxL + 1, NN = 2 * kMfA;    // l = 0..30; n + kMfA - 1 in [0, NN - 1)
    __shared__ double2 yw[8][NL];
    __shared__ double cf[8][NN][8];
    __shared__ double rsc[8];
    __shared__ int rowm[9];
    __shared__ int rowmv[8];                        // m_r of the tile's rows
    __shared__ double2 trig[9];                     // (cos, sin) of theta / 2 and of m_r phi
    __shared__ int2 segv[kFoldSegs];
    const int tid = threadIdx.x;
    const int r0 = 8 * mt;
    // the tile's segments [g0, g1); its terms are one contiguous run [t0, t1)
    // (uniform values: scalar loads)
    const int g0 = jb.mrows[min(r0, jb.n_mrows)].y, g1 = jb.mrows[min(r0 + 8, jb.n_mrows)].y;
    const int t0 = g0 < jb.n_segs ? jb.segs[g0].w : jb.n_terms;
    const int t1 = g1 < jb.n_segs ? jb.segs[g1].w : jb.n_terms;
    // This lane's first term: its contributor range is requested first, its
    // first three contributor indices once that has arrived (after the first
    // barrier) and before the weights are formed (from LDS only), so that the
    // rows can be requested as soon as the weights are in place.
    int tt = t0 + tid;
    int ea = 0, eb = 0;
    if (tt < t1) {
        ea = jb.term_ptr[tt];
        eb = jb.term_ptr[tt + 1];
    }
    // the tile's segments and its rows' (m, first segment), both requested
    // before either is used (every lane loads, at clamped indices, so that
    // no load sits under a branch)
    const int4 S = jb.segs[min(g0 + tid, max(g1 - 1, 0))];
    const int2 R = jb.mrows[min(r0 + min(tid, 8), jb.n_mrows)];
    if (tid < g1 - g0 && tid < kFoldSegs) segv[tid] = make_int2(S.w, S.y);
    if (tid < 9) {
        const int r = r0 + tid;
        rowm[tid] = R.y;                            // first segment
        const int m = r < jb.n_mrows ? R.x : 0;
        if (tid < 8) rowmv[tid] = m;
        double sv, cv;
        if (tid == 8)
            sincos(0.5 * jb.theta, &sv, &cv);
        else
            sincos((double)m * jb.phi, &sv, &cv);
        trig[tid] = make_double2(cv, sv);
    }
    for (int x = tid; x < 8 * NN * 8; x += blockDim.x) (&cf[0][0][0])[x] = 0.0;
    __syncthreads();
    // (clamped, unconditional loads; indices past eb are never used)
    int2 src[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) src[j] = jb.term_src[min(ea + j, max(eb - 1, 0))];
    for (int x = tid; x < 8 * NL; x += blockDim.x) {
        const int k = x / NL, l = x % NL, r = r0 + k;
        double yr = 0.0, yi = 0.0;
        if (r < jb.n_mrows) {
            const int m = rowmv[k];
            if (l >= 2 && l >= abs(m) && l <= jb.l_max)
                few_swsh_m2_cs(l, m, trig[8].x, trig[8].y, trig[k].x, trig[k].y, &yr, &yi);
        }
        yw[k][l] = make_double2(yr, yi);
    }
    __syncthreads();
    // the tile's segments (first term, n of the first term) in LDS when few
    const bool seg_lds = g1 - g0 <= kFoldSegs;
    auto seg_of = [&](int g) {
        if (seg_lds) return make_int2(segv[g - g0].x, segv[g - g0].y);
        const int4 S = jb.segs[g];
        return make_int2(S.w, S.y);
    };
    const double h = jb.t[iv + 1] - jb.t[iv];
    // acoef [K-1][4][2M] (matrix-core requests): coefficient p of mode k at
    // arow[p * 2M + 2k + {0, 1}], so lanes taking consecutive modes read
    // contiguous memory in each of the four planes
    const size_t ps = 2 * (size_t)jb.M;
    const double *arow = jb.acoef + (size_t)iv * 4 * ps;
    auto load8 = [&](int mode, double *a) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double2 v = *(const double2 *)(arow + p * ps + 2 * (size_t)mode);
            a[2 * p] = v.x;
            a[2 * p + 1] = v.y;
        }
    };
    for (; tt < t1; tt += blockDim.x) {
        if (tt != t0 + tid) {
            ea = jb.term_ptr[tt];
            eb = jb.term_ptr[tt + 1];
#pragma unroll
            for (int j = 0; j < 3; ++j)
                src[j] = ea + j < eb ? jb.term_src[ea + j] : make_int2(0, 0);
        }
        int g = g0;
        while (g + 1 < g1 && seg_of(g + 1).x <= tt) ++g;
        const int2 S = seg_of(g);
        int k = 0;
        while (k + 1 < 8 && rowm[k + 1] <= g) ++k;
        const int n = S.y + (tt - S.x);
        double acc[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = 0.0;
        auto add = [&](int2 cs, const double *a) {
            const int l = cs.y & 255, mir = (cs.y >> 16) & 1;
            double2 w = yw[k][l];
            if (mir && (l & 1)) w = make_double2(-w.x, -w.y);
            const double sgn = mir ? -1.0 : 1.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double ar = a[2 * q], ai = sgn * a[2 * q + 1];
                acc[2 * q] += w.x * ar - w.y * ai;
                acc[2 * q + 1] += w.x * ai + w.y * ar;
            }
        };
        // three contributors at a time, added in contributor order: their
        // coefficient rows are requested, then the next three indices (so
        // that those arrive while these rows do), then the rows are added
        for (int e = ea; e < eb; e += 3) {
            double av[3][8];
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (e + j < eb) load8(src[j].x, av[j]);
            int2 nsrc[3];
#pragma unroll
            for (int j = 0; j < 3; ++j)
                nsrc[j] = e + 3 + j < eb ? jb.term_src[e + 3 + j] : make_int2(0, 0);
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (e + j < eb) add(src[j], av[j]);
#pragma unroll
            for (int j = 0; j < 3; ++j) src[j] = nsrc[j];
        }
        // overall factor; coefficients of v = 2 x / h - 1 in [-1, 1]
        double *dst = cf[k][n + kMfA - 1];
        const double hh = 0.5 * h;
        double f = jb.scale, fi = jb.scale_im;
        double b[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            b[2 * q] = acc[2 * q] * f - acc[2 * q + 1] * fi;
            b[2 * q + 1] = acc[2 * q] * fi + acc[2 * q + 1] * f;
            f *= hh;
            fi *= hh;
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {               // (v + 1)^q expanded
            const double b1 = b[2 + c], b2 = b[4 + c], b3 = b[6 + c];
            dst[c] = b[c] + (b1 + (b2 + b3));
            dst[2 + c] = b1 + (2.0 * b2 + 3.0 * b3);
            dst[4 + c] = b2 + 3.0 * b3;
            dst[6 + c] = b3;
        }
    }
    __syncthreads();
    {
        const int k = tid >> 5, sub = tid & 31;     // 8 rows x 32 lanes
        double mx = 0.0;
        if (k < 8)
            for (int x = sub; x < NN * 8; x += 32) mx = fmax(mx, fabs((&cf[k][0][0])[x]));
        for (int off = 16; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 32));
        // one scale for the row pair 2j, 2j + 1 (rows k and k ^ 1, the two
        // rows one lane of the product holds): the epilogue applies it once
        mx = fmax(mx, __shfl_xor(mx, 32));
        if (k < 8 && sub == 0) {
            int e = 0;
            double sc = 0.0;
            float ms = 0.0f;
            if (mx > 0.0) {
                frexp(mx, &e);
                sc = ldexp(1.0, -e);
                ms = (float)ldexp(1.0, e);
            }
            rsc[k] = sc;
            if ((k & 1) == 0) jb.minfo[iv].scale[(r0 + k) >> 1] = ms;
        }
    }
    __syncthreads();
    float *dst = jb.mtab + ((size_t)iv * kMfMT + mt) * (4 * kMfT * 512);
    for (int it = tid; it < 4 * kMfT * 64; it += blockDim.x) {
        const int ln = it & 63, t = (it >> 6) % kMfT, p = (it >> 6) / kMfT;   // one wave: one (p, t)
        const int kk = (ln & 15) >> 1, comp = ln & 1, g = ln >> 4;
        const double sc = rsc[kk];
        float o[8];
        unsigned big = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int a = 16 * t + 4 * g + j;
            const double pr = cf[kk][a + kMfA - 1][2 * p], pi = cf[kk][a + kMfA - 1][2 * p + 1];
            double qr = 0.0, qi = 0.0;
            if (a > 0) {
                qr = cf[kk][-a + kMfA - 1][2 * p];
                qi = cf[kk][-a + kMfA - 1][2 * p + 1];
            }
            o[2 * j] = (float)((comp == 0 ? pr + qr : pi + qi) * sc);
            o[2 * j + 1] = (float)((comp == 0 ? qi - pi : pr - qr) * sc);
            big = max(big, max(__float_as_uint(o[2 * j]) & 0x7fffffffu,
                               __float_as_uint(o[2 * j + 1]) & 0x7fffffffu));
        }
        float4 *d = (float4 *)(dst + ((size_t)p * kMfT + t) * 512 + (size_t)ln * 8);
        d[0] = make_float4(o[0], o[1], o[2], o[3]);
        d[1] = make_float4(o[4], o[5], o[6], o[7]);
        for (int off = kWave / 2; off > 0; off >>= 1) big = max(big, (unsigned)__shfl_xor((int)big, off));
        if (ln == 0)
            jb.minfo[iv].top[(mt * 4 + p) * kMfT + t] =
                (unsigned short)min((big + 0xffffu) >> 16, 0x7fffu);
    }
}

// 512 lanes: about one folded term per lane (the fold's dependent loads
// dominate), two operand items per lane in the pack; at most 128 registers,
// so two workgroups fit a compute unit (the grid is slightly larger than the
// number of compute units).

__global__ __launch_bounds__(kFoldPackThreads) __attribute__((amdgpu_waves_per_eu(4)))
void fold_pack_kernel(PrepJob jb) {
    fold_pack_body(jb, blockIdx.x);
}

__global__ __launch_bounds__(kFoldPackThreads) __attribute__((amdgpu_waves_per_eu(4)))
void fold_pack_batch_kernel(const PrepJob *jobs) {
    const PrepJob jb = jobs[blockIdx.y];
    fold_pack_body(jb, blockIdx.x);
}

// Complex product with one rounding per component (fused multiply-add).
__device__ __forceinline__ void cmulf(float ar, float ai, float br, float bi, float *cr,
                                      float *ci) {
    *cr = __builtin_fmaf(ar, br, -(ai * bi));
    *ci = __builtin_fmaf(ar, bi, ai * br);
}

// e^{-i v} in binary32 for a binary64 phase v, |v| < 2^50: v = q pi/2 + r, q
// the nearest integer of v 2/pi and r = v - q pi/2 with pi/2 = 2pi_hi/4 +
// 2pi_lo/4 (both quarters exact), so |r| <= pi/4 up to rounding; sin r and
// cos r from their Taylor series in binary32 (terms to r^9 and r^10: the first
// omitted term is below 2e-9 for |r| <= pi/4), then the quadrant: e^{-iv} is
// (cos r, -sin r) times (-i)^q.  q comes from adding 1.5 2^52 to v 2/pi in
// one rounding (the sum's unit in the last place is 1, so its low mantissa
// bits hold q, and q mod 4 is its two lowest).  No branch.
__device__ __forceinline__ void phasor_f32(double v, float *re, float *im) {
    constexpr double kRound = 6755399441055744.0;           // 1.5 * 2^52
    const double qs = fma(v, FEW_TWO_OVER_PI, kRound);
    const double q = qs - kRound;
    const double rd = fma(-q, 0.25 * FEW_TWO_PI_LO, fma(-q, 0.25 * FEW_TWO_PI_HI, v));
    const int qm = (int)(__builtin_bit_cast(unsigned long long, qs) & 3);   // q mod 4
    const float r = (float)rd, r2 = r * r;
    float ps = __builtin_fmaf(r2, 1.0f / 362880.0f, -1.0f / 5040.0f);
    ps = __builtin_fmaf(ps, r2, 1.0f / 120.0f);
    ps = __builtin_fmaf(ps, r2, -1.0f / 6.0f);
    const float sn = __builtin_fmaf(r * r2, ps, r);
    float pc = __builtin_fmaf(r2, -1.0f / 3628800.0f, 1.0f / 40320.0f);
    pc = __builtin_fmaf(pc, r2, -1.0f / 720.0f);
    pc = __builtin_fmaf(pc, r2, 1.0f / 24.0f);
    pc = __builtin_fmaf(pc, r2, -0.5f);
    const float cs = __builtin_fmaf(pc, r2, 1.0f);
    // cos v, sin v for q mod 4 = 0, 1, 2, 3: (c, s), (-s, c), (-c, -s), (s, -c)
    const bool swap = qm & 1;
    const float a = swap ? sn : cs, b = swap ? cs : sn;
    const float cv = (qm == 1 || qm == 2) ? -a : a;
    const float sv = (qm >= 2) ? -b : b;
    *re = cv;
    *im = -sv;
}

// fp16 hi/lo parts of a pair of binary32 values, packed as two fp16 values per
// 32-bit word: hi = fp16(a), lo = fp16(a - hi) (the difference is exact in
// binary32), about 22 significant bits together.  The differences read the
// packed hi halves directly (v_fma_mix_f32, written out because the compiler
// unpacks them first).  Four instructions of 4.4 clocks per pair; forming lo
// with v_fma_mixlo_f16 / mixhi takes one instruction less but those issue every
// 8.4 clocks (rates measured with three waves per SIMD).
typedef _Float16 mf_half2 __attribute__((ext_vector_type(2)));
typedef float mf_f2 __attribute__((ext_vector_type(2)));
typedef unsigned mf_u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ unsigned pack_half2(float a0, float a1) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector((mf_f2){a0, a1}, mf_half2));
}
__device__ __forceinline__ void split_pair(float a0, float a1, unsigned &hi, unsigned &lo) {
    const unsigned h = pack_half2(a0, a1);
    float l0, l1;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[0,0,1]" : "=v"(l0) : "v"(a0), "v"(h));
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
        : "=v"(l1)
        : "v"(a1), "v"(h));
    hi = h;
    lo = pack_half2(l0, l1);
}

// Per-wave LDS area of the per-sample values of one round (64 samples, one per
// lane): f = e^{-i Phi_r} and its powers f^2, f^3 (steps inside a lane group's
// four columns), f^{4g} (g = 0..3, the group's first column; g = 0 stays 1),
// f^16; E = e^{-i Phi_phi}, E^4 and E^8 (for rows of arbitrary m the reduced
// Phi_phi, binary64, in place of E^8); the coefficient variable v (or s).
constexpr int kMfSPW = kMfNT * 16;                  // samples per wave and round
static_assert(kMfNT == 4, "one sample per lane");
struct MfSampleArea {
    float2 f[kMfSPW], f2[kMfSPW], f3[kMfSPW], f16[kMfSPW], c[4][kMfSPW];
    float2 e[kMfSPW], e4[kMfSPW], e8[kMfSPW];
    float v[kMfSPW];
};

// Exchange of the upper 32 lanes of a with the lower 32 of b, and of the odd
// 16-lane rows of a with the even ones of b.
__device__ __forceinline__ void lane_swap32(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a),
                                                    __builtin_bit_cast(unsigned, b), false, false);
    a = __builtin_bit_cast(float, (unsigned)r[0]);
    b = __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ void lane_swap16(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a),
                                                    __builtin_bit_cast(unsigned, b), false, false);
    a = __builtin_bit_cast(float, (unsigned)r[0]);
    b = __builtin_bit_cast(float, (unsigned)r[1]);
}

// A wave-uniform value in scalar registers.
__device__ __forceinline__ float uniform_f32(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform_f64(double v) { return lane_value(v, 0); }

// How the products of an interval are formed.
//
// Static tables.  A fragment (row tile mt, power p, step t) takes all three
// hi/lo products if some |value| reaches kMfSmall = 2^-12 of its row pair's
// scale S (the power of two above the pair's largest coefficient), else
// hi * hi alone, and none if it holds only zeros.  Below 2^-12, hi = fp16(value)
// alone resolves it to 2^-24 of the scale, the resolution that hi + lo gives
// values near the scale, and the lo part of the harmonics (below 2^-12 of
// their modulus 1) would add less than 2^-24 too, the size of the lo * lo
// products that are left out everywhere.  A spline's higher powers are small
// on smooth data: at 100 knots over a year p = 2 and 3 take one product each,
// 8 in place of 12.
//
// Blocks.  Where the data allow it, the cubic is written about the centre v_0
// of a block of consecutive samples, in s = (v - v_0) / w in [-1, 1], w the
// block's half width in v:
//   C(v) = T_0 + s T_1,  T_0 = b_0 + v_0 b_1 + (v_0^2 + w^2/2) b_2 + (v_0^3 + 3 w^2 v_0 / 2) b_3,
//   T_1 = w (b_1 + 2 v_0 b_2 + (3 v_0^2 + 3 w^2 / 4) b_3)
// (s^2 replaced by 1/2 and s^3 by 3 s / 4, their best constant and linear
// approximations), which is off by at most (|b_2| + 3 |b_3|) w^2 / 2 + |b_3|
// w^3 / 4.  Blocks are as long as keeps that below kMfBlockRest = 2^-25 S and
// |T_1| below kMfBlockSlope = 2^-11 S in every fragment; T_1 then needs one
// product, so a block takes 4 products and one Horner step in place of 8 to 12
// and 3.  (Its rounding to fp16 and the missing lo part of the columns are
// 2^-23 S each, 2^-22 S |s| together.  Neither this nor the products left out of
// static tables shows in the result, whose error is that of the binary32
// harmonics: over 96 full lists, smooth, decaying and noisy, of 0.4 and 3 million
// samples, the rms and the largest error are within 1 % of those with static
// tables and all three products, and of those with blocks a fourth as wide.)  The launch is
// limited by power, which goes with the products (one set of them cost 28.5 us
// on 12.6 million samples, everything else 270 us).  The 72 registers of
// T_0 (hi, lo) and T_1 stay in the wave, which forms them from the interval's
// binary32 values (staged in LDS) whenever its samples enter another block:
// about 400 vector instructions, against 560 for a round of 64 samples.  Sharing the tables
// between waves through LDS instead, formed one block ahead, cost more in
// barriers and reads than it saved (644 us against 515 with static tables).
constexpr float kMfSmall = 0x1p-12f;
constexpr float kMfBlockRest = 0x1p-25f;
constexpr float kMfBlockSlope = 0x1p-11f;
constexpr int kMfMinBlock = 2;          // shortest block, in rounds of 64 samples
constexpr int kMfMaxBlock = 1 << 20;

// Per-interval values.
struct MfInterval {
    double ti, inv_h2;      // knot time, 2 / h
    unsigned any, big;      // static tables: bit (mt * 4 + p) * T + t
    int block;              // rounds per block, 0: static tables
};

// LDS: the interval's binary32 values, [mt][p][t][half of 4 values][lane 64],
// or (static) the same values as fp16, [mt][p][t][hi, lo][lane 64][8].
// Binary32 values of one interval (or one polar index of it).
constexpr size_t mf_table_bytes(int MT, int T) { return (size_t)MT * 4 * T * 2048; }

// The operand values of fold_pack staged for the blocks.
__device__ __forceinline__ void mf_stage(const float *tab, float4 *lds) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));       // (addresses formed here, not kept through the rounds)
    for (int v = tid; v < (int)(kMfIntervalFloats / 4); v += 64 * kMfWaves)
        lds[(v & ~127) | (v & 1) << 6 | ((v >> 1) & 63)] = ((const float4 *)tab)[v];
}

// fp16 parts of a lane's 8 operand values of one fragment, stored as in a static
// table (d: the fragment's hi part of this lane).
__device__ __forceinline__ void mf_store_parts(float4 a, float4 b, float4 *d) {
    unsigned hi[4], lo[4];
    split_pair(a.x, a.y, hi[0], lo[0]);
    split_pair(a.z, a.w, hi[1], lo[1]);
    split_pair(b.x, b.y, hi[2], lo[2]);
    split_pair(b.z, b.w, hi[3], lo[3]);
    ((uint4 *)d)[0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    ((uint4 *)d)[64] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// The operand values of fold_pack staged as a static table.
__device__ __forceinline__ void mf_stage_static(const float *tab, float4 *lds) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int it = 0; it < (int)(kMfIntervalFloats / 8); it += 64 * kMfWaves) {
        const int x = it + tid;
        const float4 *v = (const float4 *)tab + 2 * x;
        mf_store_parts(v[0], v[1], lds + (x >> 6) * 128 + (x & 63));
    }
}
static_assert(kMfIntervalFloats / 8 % (64 * kMfWaves) == 0, "whole turns");

// Staged values -> static table, in place (each lane rewrites what it read).
template <int MT, int T>
__device__ __forceinline__ void mf_convert(float4 *lds) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    for (int it = tid; it < MT * 4 * T * 64; it += 64 * kMfWaves) {
        float4 *d = lds + (it >> 6) * 128 + (it & 63);
        const float4 a = d[0], b = d[64];
        mf_store_parts(a, b, d);
    }
}

// LDS of the requests whose operand values are formed here from the folded
// terms of prepare_kernel: the term of every (row, n) of one polar index, the
// largest |coefficient| of each row pair (as bits) and 2^E, the fragments'
// largest scaled values.
template <int MT, int T>
struct MfTerms {
    int idx[8 * MT][32 * T];        // n + 16 T; -1: no term
    unsigned pmax[4 * MT];
    float un[4 * MT];
    unsigned top[MT * 4 * T];
};

// Cubic in u = x / h -> cubic in v = 2 u - 1.
__device__ __forceinline__ void mf_recentre(float a0, float a1, float a2, float a3, float *b) {
    const float h1 = 0.5f * a1, h2 = 0.25f * a2, h3 = 0.125f * a3;
    b[0] = a0 + (h1 + (h2 + h3));
    b[1] = h1 + __builtin_fmaf(2.0f, h2, 3.0f * h3);
    b[2] = __builtin_fmaf(3.0f, h3, h2);
    b[3] = h3;
}

__device__ __forceinline__ unsigned abs_bits(float x) { return __float_as_uint(x) & 0x7fffffffu; }

// max over the lanes of groups of 2^steps
template <int STEPS>
__device__ __forceinline__ unsigned lanes_max(unsigned v) {
#pragma unroll
    for (int i = 0; i < STEPS; ++i) v = max(v, (unsigned)__shfl_xor((int)v, 1 << i));
    return v;
}

// Terms of polar index kp into idx[row][n + half] (rows of `stride`); the waves
// take its segments in turn.
__device__ __forceinline__ void mf_terms_scatter(const SumJob &jb, int kp, int half, int stride,
                                                 int *idx, int lane, int wave) {
    int turn = 0;
    for (int g0 = 0; g0 < jb.n_segs; g0 += kWave) {
        const int4 S = jb.segs[min(g0 + lane, jb.n_segs - 1)];
        unsigned long long hit = __ballot(g0 + lane < jb.n_segs && seg_k(S.x) == kp);
        for (; hit; hit &= hit - 1, ++turn) {
            if ((turn & (kMfWaves - 1)) != wave) continue;
            const int src = __ffsll((long long)hit) - 1;
            const int row = __builtin_amdgcn_readlane(S.x, src) - 256 * kp - jb.mf_m0;
            const int n_lo = __builtin_amdgcn_readlane(S.y, src);
            const int len = __builtin_amdgcn_readlane(S.z, src);
            const int first = __builtin_amdgcn_readlane(S.w, src);
            for (int q = lane; q < len; q += kWave) idx[row * stride + n_lo + q + half] = first + q;
        }
    }
}

// The operand values of interval iv and polar index kp (0 in Schwarzschild),
// from the binary32 fold table: the values that fold_pack writes, formed in
// binary32.  M.idx holds -1 everywhere on entry and on return.  A lane takes
// the columns n = +-a of one row; a wave 8 rows by 8 of a, so that both maxima
// are reductions over lanes.  Latency bound (the segments, the terms, then
// the two maxima: four barriers).
template <int MT, int T>
__device__ __forceinline__ void mf_terms_stage(const SumJob &jb, int iv, int kp,
                                               MfTerms<MT, T> &M, float4 *lds) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));       // (addresses formed here, not kept through the rounds)
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    __syncthreads();                                // the previous values no longer read
    if (tid < 4 * MT) M.pmax[tid] = 0u;
    if (tid < MT * 4 * T) M.top[tid] = 0u;
    mf_terms_scatter(jb, kp, 16 * T, 32 * T, &M.idx[0][0], lane, wave);
    __syncthreads();
    constexpr int kTasks = MT * T * 2, kTurns = (kTasks + kMfWaves - 1) / kMfWaves;
    // (terms are stored in reverse order, 8 values each)
    const float4 *last = (const float4 *)jb.table + ((size_t)iv * jb.n_terms + jb.n_terms - 1) * 2;
    float4 v[kTurns][4];
#pragma unroll
    for (int q = 0; q < kTurns; ++q) {
        const int task = min(wave + q * kMfWaves, kTasks - 1);      // (mt, t, half of the a)
        const int row = 8 * (task / (2 * T)) + (lane >> 3), a = 8 * (task % (2 * T)) + (lane & 7);
        int *ip = &M.idx[row][16 * T + a], *iq = &M.idx[row][16 * T - a];
        const int tp = *ip, tq = a > 0 ? *iq : -1;
        const float4 *cp = last - 2 * (size_t)max(tp, 0), *cq = last - 2 * (size_t)max(tq, 0);
        v[q][0] = cp[0];
        v[q][1] = cp[1];
        v[q][2] = cq[0];
        v[q][3] = cq[1];
        if (tp < 0) v[q][0] = v[q][1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (tq < 0) v[q][2] = v[q][3] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < kTurns; ++q) {
        if (wave + q * kMfWaves >= kTasks) continue;
        const int task = wave + q * kMfWaves;
        const int row = 8 * (task / (2 * T)) + (lane >> 3), a = 8 * (task % (2 * T)) + (lane & 7);
        M.idx[row][16 * T + a] = -1;
        M.idx[row][16 * T - a] = -1;
        unsigned m = 0;
#pragma unroll
        for (int h = 0; h < 4; h += 2) {
            float b[4], c[4];
            mf_recentre(v[q][h].x, v[q][h].z, v[q][h + 1].x, v[q][h + 1].z, b);
            mf_recentre(v[q][h].y, v[q][h].w, v[q][h + 1].y, v[q][h + 1].w, c);
#pragma unroll
            for (int i = 0; i < 4; ++i) m = max(m, max(abs_bits(b[i]), abs_bits(c[i])));
        }
        m = lanes_max<4>(m);                        // the 8 columns of two rows
        if ((lane & 15) == 0) atomicMax(&M.pmax[row >> 1], m);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kTurns; ++q) {
        if (wave + q * kMfWaves >= kTasks) continue;
        const int task = wave + q * kMfWaves, mt = task / (2 * T), ta = task % (2 * T);
        const int r = lane >> 3, a = 8 * ta + (lane & 7), t = ta >> 1;
        // scale 2^-E, E the exponent of the row pair's largest value (NaN and
        // infinity: none)
        const float mx = __uint_as_float(M.pmax[4 * mt + (r >> 1)]);
        int e = 0;
        if (mx > 0.0f && mx < INFINITY) frexpf(mx, &e);
        e = min(max(e, -126), 127);
        const float sc = ldexpf(1.0f, -e);
        if ((lane & 15) == 0) M.un[4 * mt + (r >> 1)] = ldexpf(1.0f, e);
        // columns per power: (Re P + Re Q, Im Q - Im P) of row component 0,
        // (Im P + Im Q, Re P - Re Q) of component 1
        const float4 p0 = v[q][0], p1 = v[q][1], q0 = v[q][2], q1 = v[q][3];
        float o[2][2][4];
        mf_recentre(p0.x + q0.x, p0.z + q0.z, p1.x + q1.x, p1.z + q1.z, o[0][0]);
        mf_recentre(q0.y - p0.y, q0.w - p0.w, q1.y - p1.y, q1.w - p1.w, o[0][1]);
        mf_recentre(p0.y + q0.y, p0.w + q0.w, p1.y + q1.y, p1.w + q1.w, o[1][0]);
        mf_recentre(p0.x - q0.x, p0.z - q0.z, p1.x - q1.x, p1.z - q1.z, o[1][1]);
        // a = 16 t + 4 g + j: fragment lane 2 r + component + 16 g, values
        // 2 j and 2 j + 1 (half j >> 1 of the staged fragment)
        const int g = (a >> 2) & 3, j = a & 3;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            unsigned big = 0;
            float4 *f = lds + ((mt * 4 + p) * T + t) * 128 + 64 * (j >> 1) + 2 * r + 16 * g;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float x = o[c][0][p] * sc, y = o[c][1][p] * sc;
                big = max(big, max(abs_bits(x), abs_bits(y)));
                ((float2 *)(f + c))[j & 1] = make_float2(x, y);
            }
            big = lanes_max<6>(big);
            if (lane == 0) atomicMax(&M.top[(mt * 4 + p) * T + t], big);
        }
    }
    __syncthreads();
}

// The operand registers of a block: T_0 (hi, lo) and T_1 per row tile and step.
template <int MT, int T>
struct MfBlock {
    mf_u4 t1[MT][T], h0[MT][T], l0[MT][T];
};

// Form them for block centre v0 and half width w from the staged values.
template <int MT, int T>
__device__ __forceinline__ void mf_block_form(const float4 *lds, double v0, double w,
                                              MfBlock<MT, T> &B) {
    const int lane = threadIdx.x & (kWave - 1);
    const double vv = v0 * v0, ww = w * w;
    const float k1 = uniform_f32((float)v0), k2 = uniform_f32((float)fma(0.5, ww, vv)),
                k3 = uniform_f32((float)(v0 * fma(1.5, ww, vv)));
    const float q1 = uniform_f32((float)w), q2 = uniform_f32((float)(w * 2.0 * v0)),
                q3 = uniform_f32((float)(w * fma(0.75, ww, 3.0 * vv)));
    const float4 *src = lds + lane;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            float4 b[4][2];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const float4 *q = src + ((mt * 4 + p) * T + t) * 128;
                b[p][0] = q[0];
                b[p][1] = q[64];
            }
            const float *b0 = (const float *)b[0], *b1 = (const float *)b[1];
            const float *b2 = (const float *)b[2], *b3 = (const float *)b[3];
            float T0[8], T1[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                T0[i] = __builtin_fmaf(k3, b3[i], __builtin_fmaf(k2, b2[i], __builtin_fmaf(k1, b1[i], b0[i])));
                T1[i] = __builtin_fmaf(q3, b3[i], __builtin_fmaf(q2, b2[i], q1 * b1[i]));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                unsigned h, l;
                split_pair(T0[2 * i], T0[2 * i + 1], h, l);
                B.h0[mt][t][i] = h;
                B.l0[mt][t][i] = l;
                B.t1[mt][t][i] = pack_half2(T1[2 * i], T1[2 * i + 1]);
            }
            __builtin_amdgcn_sched_barrier(0);      // (one fragment's values at a time)
        }
}

// What a lane keeps of its own sample until the end of the round: z0 =
// e^{-i m_0 Phi_phi}, E^2, and for generic Kerr Theta = e^{-i Phi_theta}.
struct MfOwn {
    float z0r, z0i, e2r, e2i, tr, ti;
};

// Generic Kerr: the sum over the polar index k is a Horner recurrence in Theta
// on the sums over (m, n) of each k, highest k first, with the waves' running
// values in LDS (hp, one per sample of kMfKerrRounds rounds).
constexpr int kMfKerrRounds = 12;
struct MfPolar {
    float2 *hp;             // this round's running values
    bool first, last;       // highest, lowest k
    int k0;                 // lowest k
};

// First part of a round: lane l forms the values of sample wbase + l (phases,
// harmonics and their powers) into the wave's LDS area.  z0 and E^2 (and
// Theta) stay in registers: the same lane holds the sample at the end.
template <bool CONSEC, bool KERR>
__device__ __forceinline__ MfOwn mf_samples(const SumJob &jb, int iv, double ti, double vscale,
                                            double vshift, long long wbase, long long e,
                                            int m0, const MfPolar &po, MfSampleArea *sa) {
    const int lane = threadIdx.x & (kWave - 1);
    const FEW_AS4 double *pc = cptr(jb.pcoef) + (size_t)iv * (KERR ? 24 : 16);
    MfOwn own{1.0f, 0.0f, 1.0f, 0.0f, 1.0f, 0.0f};
    // (wbase and e are whole numbers below 2^53: exact)
    const double jd = fmin((double)wbase + (double)lane, (double)(e - 1));
    const double tj = __dadd_rn(jb.t_start, __dmul_rn(jd, jb.dt));
    const double x = tj - ti;
    const double pf = phase_raw(pc, x);
    const double pr = phase_raw(pc + 8, x);
    float er, ei, fr, fi;
    phasor_f32(pf, &er, &ei);
    phasor_f32(pr, &fr, &fi);
    float f2r, f2i, f3r, f3i, f4r, f4i, f8r, f8i, f12r, f12i, f16r, f16i;
    cmulf(fr, fi, fr, fi, &f2r, &f2i);
    cmulf(f2r, f2i, fr, fi, &f3r, &f3i);
    cmulf(f2r, f2i, f2r, f2i, &f4r, &f4i);
    cmulf(f4r, f4i, f4r, f4i, &f8r, &f8i);
    cmulf(f8r, f8i, f4r, f4i, &f12r, &f12i);
    cmulf(f8r, f8i, f8r, f8i, &f16r, &f16i);
    sa->v[lane] = (float)fma(x, vscale, vshift);
    sa->f[lane] = make_float2(fr, fi);
    sa->f2[lane] = make_float2(f2r, f2i);
    sa->f3[lane] = make_float2(f3r, f3i);
    sa->f16[lane] = make_float2(f16r, f16i);
    sa->c[1][lane] = make_float2(f4r, f4i);
    sa->c[2][lane] = make_float2(f8r, f8i);
    sa->c[3][lane] = make_float2(f12r, f12i);
    sa->e[lane] = make_float2(er, ei);
    if constexpr (CONSEC) {
        const int am0 = m0 < 0 ? -m0 : m0;
        // Rows of consecutive m (m_r = m_0 + r): every z_r is a power of
        // E = e^{-i Phi_phi}.  z_0 = E^{m_0} by binary powering (E^{-1} =
        // conj E), so each z_r carries m_r times the phase error of E, at
        // most max |m| of it.
        float e4r, e4i, e8r, e8i;
        cmulf(er, ei, er, ei, &own.e2r, &own.e2i);
        cmulf(own.e2r, own.e2i, own.e2r, own.e2i, &e4r, &e4i);
        cmulf(e4r, e4i, e4r, e4i, &e8r, &e8i);
        if (!KERR || po.last) {
            float br = e8r, bi = e8i;
            auto take = [&](float qr, float qi) {
                float nr, ni;
                cmulf(own.z0r, own.z0i, qr, qi, &nr, &ni);
                own.z0r = nr;
                own.z0i = ni;
            };
            if (am0 & 1) take(er, ei);
            if (am0 & 2) take(own.e2r, own.e2i);
            if (am0 & 4) take(e4r, e4i);
            for (int bit = 8; bit <= am0; bit <<= 1) {
                if (am0 & bit) take(br, bi);
                float nr, ni;
                cmulf(br, bi, br, bi, &nr, &ni);
                br = nr;
                bi = ni;
            }
            if (m0 < 0) own.z0i = -own.z0i;
        }
        sa->e4[lane] = make_float2(e4r, e4i);
        sa->e8[lane] = make_float2(e8r, e8i);
    } else {
        // rows of arbitrary m carry their whole phase themselves
        sa->e4[lane] = make_float2(1.0f, 0.0f);
        ((double *)sa->e8)[lane] = d_reduce_2pi(pf);
    }
    if constexpr (KERR) {
        const double pt = phase_raw(pc + 16, x);
        phasor_f32(pt, &own.tr, &own.ti);
        if (po.last && po.k0 != 0) {
            float zr, zi, kr, ki;
            phasor_f32((double)po.k0 * d_reduce_2pi(pt), &kr, &ki);
            cmulf(own.z0r, own.z0i, kr, ki, &zr, &zi);
            own.z0r = zr;
            own.z0i = zi;
        }
    }
    __builtin_amdgcn_wave_barrier();
    return own;
}

// The operand columns of sample tile nt: powers of f for every step, fp16 hi
// and lo pairs.  Lane group g = l / 16 holds |n| = 16 t + 4 g + j, j < 4, of
// step t: f^{16 t + 4 g} times f^j (the same fragment serves n and -n).
template <int T>
__device__ __forceinline__ void mf_columns(const MfSampleArea *sa, int nt, mf_u4 (&bh)[T],
                                           mf_u4 (&bl)[T]) {
    const int lane = threadIdx.x & (kWave - 1);
    const int g = lane >> 4, sl = 16 * nt + (lane & 15);
    const float2 f1 = sa->f[sl], f2 = sa->f2[sl], f3 = sa->f3[sl];
    const float2 c0 = sa->c[g][sl];
    float w[8];
    w[0] = c0.x;
    w[1] = c0.y;
    cmulf(c0.x, c0.y, f1.x, f1.y, &w[2], &w[3]);
    cmulf(c0.x, c0.y, f2.x, f2.y, &w[4], &w[5]);
    cmulf(c0.x, c0.y, f3.x, f3.y, &w[6], &w[7]);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (t > 0) {
            const float2 fs = sa->f16[sl];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float nr, ni;
                cmulf(w[2 * i], w[2 * i + 1], fs.x, fs.y, &nr, &ni);
                w[2 * i] = nr;
                w[2 * i + 1] = ni;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned h, l;
            split_pair(w[2 * i], w[2 * i + 1], h, l);
            bh[t][i] = h;
            bl[t][i] = l;
        }
    }
}

// Rows of tile mt -> the lane's value of its column in sample tile nt.  The
// lane holds rows r = 8 mt + 2g (a0 + i b0) and r + 1 (a1 + i b1), which share
// the scale se.
template <bool CONSEC, int MT>
__device__ __forceinline__ void mf_rows(const mf_float4 &acc, float se, int mt, int nt,
                                        const int *mm, const MfSampleArea *sa, float &qr,
                                        float &qi) {
    const int lane = threadIdx.x & (kWave - 1);
    const int g = lane >> 4, sl = 16 * nt + (lane & 15);
    const float2 E = sa->e[sl];
    const float a0 = acc[0], b0 = acc[1], a1 = acc[2], b1 = acc[3];
    if constexpr (CONSEC) {
        // z_r = z_0 E^{2g} E^{8 mt} (E for the odd row): Horner in E^8 over
        // the tiles of s (a0 + i b0 + E (a1 + i b1))
        const float wr = se * __builtin_fmaf(E.x, a1, __builtin_fmaf(-E.y, b1, a0));
        const float wi = se * __builtin_fmaf(E.x, b1, __builtin_fmaf(E.y, a1, b0));
        if (mt == MT - 1) {
            qr = wr;
            qi = wi;
        } else {
            const float2 E8 = sa->e8[sl];
            const float nr = __builtin_fmaf(qr, E8.x, __builtin_fmaf(-qi, E8.y, wr));
            const float ni = __builtin_fmaf(qr, E8.y, __builtin_fmaf(qi, E8.x, wi));
            qr = nr;
            qi = ni;
        }
    } else {
        // rows of arbitrary m: one phasor per row (the odd row from the even
        // one when its m is the next integer)
        const double spf = ((const double *)sa->e8)[sl];
        const int me = mm[8 * mt + 2 * g], mo = mm[8 * mt + 2 * g + 1];
        float zr, zi, yr, yi;
        phasor_f32((double)me * spf, &zr, &zi);
        if (mo == me + 1)
            cmulf(zr, zi, E.x, E.y, &yr, &yi);
        else
            phasor_f32((double)mo * spf, &yr, &yi);
        zr = zr * se;
        zi = zi * se;
        yr = yr * se;
        yi = yi * se;
        if (mt == MT - 1) qr = qi = 0.0f;
        qr = __builtin_fmaf(zr, a0, __builtin_fmaf(-zi, b0, qr));
        qi = __builtin_fmaf(zr, b0, __builtin_fmaf(zi, a0, qi));
        qr = __builtin_fmaf(yr, a1, __builtin_fmaf(-yi, b1, qr));
        qi = __builtin_fmaf(yr, b1, __builtin_fmaf(yi, a1, qi));
    }
}

// Last part of a round.  Join the lane groups, h = z_0 ((q_0 + E^4 q_2) +
// E^2 (q_1 + E^4 q_3)): swapping halves between tiles P and Q leaves (P: g 0, 1;
// Q: g 0, 1) in one register and (P: g 2, 3; Q: g 2, 3) in the other; swapping
// rows between the pairs (0, 2) and (1, 3) then leaves lane l with sample l.
// Stores h, or returns this lane's binary64 inner-product sums with the data
// dv (INNER).  Generic Kerr: the Horner step in Theta, and only the lowest k
// goes on to h.
template <bool INNER, bool KERR>
__device__ __forceinline__ double2 mf_finish(const SumJob &jb, const float *qr, const float *qi,
                                             const MfOwn &own, const MfSampleArea *sa,
                                             long long jo, bool valid, float2 dv,
                                             const MfPolar &po) {
    const int lane = threadIdx.x & (kWave - 1), col = lane & 15;
    auto join4 = [&](int a, int b, float *yr, float *yi) {
        float pr = qr[a], pi = qi[a], ur = qr[b], ui = qi[b];
        lane_swap32(pr, ur);
        lane_swap32(pi, ui);
        const float2 E4 = sa->e4[16 * (lane < 32 ? a : b) + col];
        *yr = __builtin_fmaf(E4.x, ur, __builtin_fmaf(-E4.y, ui, pr));
        *yi = __builtin_fmaf(E4.x, ui, __builtin_fmaf(E4.y, ur, pi));
    };
    float xr, xi, yr, yi, hr, hq;
    join4(0, 2, &xr, &xi);
    join4(1, 3, &yr, &yi);
    lane_swap16(xr, yr);
    lane_swap16(xi, yi);
    float sr = __builtin_fmaf(own.e2r, yr, __builtin_fmaf(-own.e2i, yi, xr));
    float si = __builtin_fmaf(own.e2r, yi, __builtin_fmaf(own.e2i, yr, xi));
    if constexpr (KERR) {
        if (!po.first) {
            const float2 q = po.hp[lane];
            const float nr = __builtin_fmaf(q.x, own.tr, __builtin_fmaf(-q.y, own.ti, sr));
            si = __builtin_fmaf(q.x, own.ti, __builtin_fmaf(q.y, own.tr, si));
            sr = nr;
        }
        if (!po.last) {
            po.hp[lane] = make_float2(sr, si);
            __builtin_amdgcn_wave_barrier();
            return make_double2(0.0, 0.0);
        }
    }
    cmulf(sr, si, own.z0r, own.z0i, &hr, &hq);
    double dh = 0.0, hh = 0.0;
    if (valid) {
        if constexpr (INNER) {
            const double vr = hr, vi = hq, dr = dv.x, di = dv.y;
            dh = dr * vr + di * vi;
            hh = vr * vr + vi * vi;
        } else {
            ((float2 *)jb.out)[jo] = make_float2(hr, hq);
        }
    }
    // the area is rewritten by the next round only after these reads
    __builtin_amdgcn_wave_barrier();
    return make_double2(dh, hh);
}

// INNER: the lane's data sample, requested at the start of the round so that
// its latency passes under the products (every lane loads, at a clamped index:
// under a branch the compiler would wait for it at the join).
template <bool INNER>
__device__ __forceinline__ float2 mf_data(const SumJob &jb, long long jo, long long e) {
    if constexpr (INNER) return ((const float2 *)jb.data)[min(jo, e - 1)];
    return make_float2(0.0f, 0.0f);
}

// One round of a wave: the 64 samples wbase + l (valid below e) in four tiles
// of 16, with the interval's static table in LDS.  The row tiles are taken one
// after the other, the highest first: the accumulators of a tile (16
// registers) run a Horner recurrence in v over p = 3 .. 0, then the lane's two
// rows are combined and added into its running value.  The LDS accesses of
// one wave complete in order, so its area needs no barrier.
template <bool INNER, bool CONSEC, int MT, int T, bool KERR>
__device__ __forceinline__ double2 mf_round_static(const SumJob &jb, int iv, const MfInterval &I,
                                                   long long wbase, long long e,
                                                   const float4 *lds, const float *msc,
                                                   const int *mm, const MfPolar &po,
                                                   MfSampleArea *sa) {
    const int lane = threadIdx.x & (kWave - 1);
    const long long jo = wbase + lane;
    const float2 dv = mf_data<INNER>(jb, jo, e);
    const MfOwn own = mf_samples<CONSEC, KERR>(jb, iv, I.ti, I.inv_h2, -1.0, wbase, e, mm[0], po,
                                              sa);
    mf_u4 bh[kMfNT][T], bl[kMfNT][T];
    float vv[kMfNT];
#pragma unroll
    for (int nt = 0; nt < kMfNT; ++nt) {
        vv[nt] = sa->v[16 * nt + (lane & 15)];
        mf_columns<T>(sa, nt, bh[nt], bl[nt]);
    }
    float qr[kMfNT], qi[kMfNT];
#pragma unroll
    for (int mt = MT - 1; mt >= 0; --mt) {
        mf_float4 acc[kMfNT];
        // acc[nt] += A B_nt for the four sample tiles; the first product
        // starts from zero (no accumulator to clear)
        auto products = [&](float4 A, const mf_u4 (&B)[kMfNT][T], int t, bool first) {
#pragma unroll
            for (int nt = 0; nt < kMfNT; ++nt)
                acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                    __builtin_bit_cast(mf_half8, A), __builtin_bit_cast(mf_half8, B[nt][t]),
                    first ? mf_float4{0.0f, 0.0f, 0.0f, 0.0f} : acc[nt], 0, 0, 0);
        };
        // fragment k of the tile, p descending
        const float4 *fp = lds + (size_t)mt * 4 * T * 128 + lane;
        auto at = [](int k) { return ((3 - k / T) * T + k % T) * 128; };
        // (opaque here, so that the compiler does not keep a condition per
        // fragment in scalar registers across the whole loop over rounds)
        unsigned any = I.any >> (mt * 4 * T), big = I.big >> (mt * 4 * T);
        asm volatile("" : "+s"(any), "+s"(big));
        constexpr int NF = 4 * T;
        float4 ch = fp[at(0)], cl = fp[at(0) + 64];
#pragma unroll
        for (int k = 0; k < NF; ++k) {
            const int t = k % T, p = 3 - k / T;
            float4 nh = ch, nl = cl;
            if (k + 1 < NF) {
                nh = fp[at(k + 1)];
                nl = fp[at(k + 1) + 64];
            }
            // keep the next fragment's reads ahead of this fragment's products
            __builtin_amdgcn_sched_barrier(0);
            if (k == 0) {
                products(ch, bh, t, true);
            } else if (t == 0) {
                // Horner step: every accumulator element of tile nt times v
#pragma unroll
                for (int nt = 0; nt < kMfNT; ++nt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[nt][i] = acc[nt][i] * vv[nt];
            }
            if ((big >> (p * T + t)) & 1) {
                products(cl, bh, t, false);
                products(ch, bl, t, false);
            }
            if (k != 0 && ((any >> (p * T + t)) & 1)) products(ch, bh, t, false);
            __builtin_amdgcn_sched_barrier(0);
            ch = nh;
            cl = nl;
        }
        const float se = msc[4 * mt + (lane >> 4)];
#pragma unroll
        for (int nt = 0; nt < kMfNT; ++nt) 
            mf_rows<CONSEC, MT>(acc[nt], se, mt, nt, mm, sa, qr[nt], qi[nt]);
    }
    return mf_finish<INNER, KERR>(jb, qr, qi, own, sa, jo, jo < e, dv, po);
}

// The same round within one block (operands in registers, s in place of v),
// one sample tile after the other: the columns, T_1 and T_0 of the three row
// tiles (independent accumulators), the rows.
template <bool INNER, int MT, int T, bool KERR>
__device__ __forceinline__ double2 mf_round_block(const SumJob &jb, int iv, double ti,
                                                  double vscale, double vshift,
                                                  const MfBlock<MT, T> &B, long long wbase,
                                                  long long e, const float *msc, const int *mm,
                                                  const MfPolar &po, MfSampleArea *sa) {
    const int lane = threadIdx.x & (kWave - 1);
    const long long jo = wbase + lane;
    const float2 dv = mf_data<INNER>(jb, jo, e);
    const MfOwn own = mf_samples<true, KERR>(jb, iv, ti, vscale, vshift, wbase, e, mm[0], po, sa);
    float se[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) se[mt] = msc[4 * mt + (lane >> 4)];
    float qr[kMfNT], qi[kMfNT];
#pragma unroll
    for (int nt = 0; nt < kMfNT; ++nt) {
        mf_u4 bh[T], bl[T];
        mf_columns<T>(sa, nt, bh, bl);
        const float s = sa->v[16 * nt + (lane & 15)];
        mf_float4 acc[MT];
        auto products = [&](const mf_u4 (&A)[MT][T], const mf_u4 (&b)[T], int t, bool first) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                    __builtin_bit_cast(mf_half8, A[mt][t]), __builtin_bit_cast(mf_half8, b[t]),
                    first ? mf_float4{0.0f, 0.0f, 0.0f, 0.0f} : acc[mt], 0, 0, 0);
        };
#pragma unroll
        for (int t = 0; t < T; ++t) products(B.t1, bh, t, t == 0);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[mt][i] = acc[mt][i] * s;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            products(B.l0, bh, t, false);
            products(B.h0, bl, t, false);
            products(B.h0, bh, t, false);
        }
#pragma unroll
        for (int mt = MT - 1; mt >= 0; --mt)
            mf_rows<true, MT>(acc[mt], se[mt], mt, nt, mm, sa, qr[nt], qi[nt]);
    }
    return mf_finish<INNER, KERR>(jb, qr, qi, own, sa, jo, jo < e, dv, po);
}

// The constants of interval iv and which products it takes, from mx(f), the
// largest |scaled value| of fragment f = (mt 4 + p) T + t (every wave forms
// the same).
template <bool CONSEC, int MT, int T, typename Max>
__device__ __forceinline__ MfInterval mf_interval(const SumJob &jb, int iv, Max mx) {
    const int lane = threadIdx.x & (kWave - 1);
    MfInterval I;
    I.ti = uniform_f64(jb.t[iv]);
    I.inv_h2 = uniform_f64(2.0 / (jb.t[iv + 1] - I.ti));
    {
        constexpr int NF = MT * 4 * T;
        const float v = mx(min(lane, NF - 1));
        I.any = (unsigned)__ballot(lane < NF && !(v == 0.0f));
        I.big = (unsigned)__ballot(lane < NF && !(v < kMfSmall));
    }
    I.block = 0;
    if constexpr (CONSEC) {
        // the widest block (half width w in v) that every fragment (mt, t) allows
        constexpr int NF = MT * T;
        const int f = min(lane, NF - 1), mt = f / T, t = f % T;
        const float b1 = mx((mt * 4 + 1) * T + t), b2 = mx((mt * 4 + 2) * T + t);
        const float b3 = mx((mt * 4 + 3) * T + t);
        const float w1 = kMfBlockSlope / (b1 + 2.0f * b2 + 3.75f * b3);
        const float w2 = sqrtf(kMfBlockRest / (0.5f * b2 + 1.75f * b3));    // (w <= 1)
        // (NaN and infinite values: no block)
        float w = w1 > 0.0f && w2 > 0.0f ? fminf(fminf(w1, w2), 1.0f) : 0.0f;
        for (int off = 4; off > 0; off >>= 1) w = fminf(w, __shfl_xor(w, off));
        w = uniform_f32(w);
        // half width of a round in v
        const double unit = 0.5 * kMfSPW * jb.dt * I.inv_h2;
        const double r = fmin((double)w / unit, (double)kMfMaxBlock);
        const int k = (int)r;
        I.block = __builtin_amdgcn_readfirstlane(k >= kMfMinBlock ? k : 0);
    }
    return I;
}

// Rounds [ra, rb) of interval iv (samples a .. end - 1, valid below e) on one
// wave, within blocks; each(r): the polar state of round r, add(v): takes its
// inner-product sums.
template <bool INNER, int MT, int T, bool KERR, typename Each, typename Add>
__device__ __forceinline__ void mf_blocks(const SumJob &jb, int iv, const MfInterval &I,
                                          long long a, long long end, long long e, int ra, int rb,
                                          const float4 *lds, const float *msc, const int *mm,
                                          MfSampleArea *sa, Each each, Add add) {
    const double x0 = dev_sample_time(jb.t_start, jb.dt, a) - I.ti;
    const double w = uniform_f64(0.5 * kMfSPW * I.block * jb.dt * I.inv_h2);
    const double vscale = uniform_f64(I.inv_h2 / w);
    for (int r = ra; r < rb;) {
        // the block of round r, centred at the middle of its samples (the last
        // one's end with the interval, so |v0| <= 1)
        const int k = r / I.block, re = min(rb, (k + 1) * I.block);
        const long long j0 = (long long)k * I.block * kMfSPW;
        const long long j1 = min(j0 + (long long)I.block * kMfSPW, end - a);
        const double mid = 0.5 * (double)(j0 + j1 - 1);
        const double v0 = uniform_f64(fma(fma(mid, jb.dt, x0), I.inv_h2, -1.0));
        const double vshift = uniform_f64(-(1.0 + v0) / w);
        MfBlock<MT, T> B;
        mf_block_form<MT, T>(lds, v0, w, B);
        for (; r < re; ++r)
            add(mf_round_block<INNER, MT, T, KERR>(jb, iv, I.ti, vscale, vshift, B,
                                                   a + (long long)r * kMfSPW, e, msc, mm, each(r),
                                                   sa));
    }
}

// Samples [lo, hi) of one job (matrix-core path), from interval `first` on.  Every
// lane of the workgroup runs the same loops over intervals (lo, hi uniform).
// INNER: each lane's binary64 sums accumulate in its LDS slot
// iacc[threadIdx.x] (zeroed by the caller), which keeps them out of the
// registers of the product loop.
template <bool INNER, bool CONSEC>
__device__ void mf_range(const SumJob &jb, long long lo, long long hi, int first, float4 *lds,
                         float *msc, int *mm, double2 *iacc) {
    constexpr int MT = kMfMT, T = kMfT;
    if (lo >= hi) return;
    // the waves' sample areas follow the tables in LDS
    const int wave = threadIdx.x / kWave;
    MfSampleArea *sa = (MfSampleArea *)((char *)lds + mf_table_bytes(MT, T)) + wave;
    sa->c[0][threadIdx.x & (kWave - 1)] = make_float2(1.0f, 0.0f);
    __syncthreads();                                // rows of a previous job no longer read
    if ((int)threadIdx.x < kMfRows) {
        const int r = threadIdx.x;
        const FEW_AS4 int2 *mr = cptr(jb.mrows);
        mm[r] = r < jb.n_mrows ? mr[r].x : mr[jb.n_mrows - 1].x + (r - jb.n_mrows + 1);
    }
    const FEW_AS4 long long *st = cptr(jb.starts);
    const MfPolar po{nullptr, true, true, 0};
    auto add = [&](double2 v) {
        if constexpr (INNER) {
            double2 a = iacc[threadIdx.x];
            a.x = a.x + v.x;
            a.y = a.y + v.y;
            iacc[threadIdx.x] = a;
        }
    };
    for (int iv = first; iv <= jb.K - 2 && lo < hi; ++iv) {
        const long long a = st[iv], end = st[iv + 1], e = min(hi, end);
        if (e <= lo) continue;
        const unsigned short *top = jb.minfo[iv].top;
        const MfInterval I = mf_interval<CONSEC, MT, T>(
            jb, iv, [&](int f) { return __uint_as_float((unsigned)top[f] << 16); });
        __syncthreads();                            // previous interval no longer read
        if ((int)threadIdx.x < kMfRows / 2) msc[threadIdx.x] = jb.minfo[iv].scale[threadIdx.x];
        const float *tab = jb.mtab + (size_t)iv * kMfIntervalFloats;
        if (I.block == 0)
            mf_stage_static(tab, lds);
        else
            mf_stage(tab, lds);
        __syncthreads();
        if (I.block == 0) {
            // (a wave whose samples of a round all lie past the end skips it)
            for (long long base = lo + (long long)wave * kMfSPW; base < e; base += kMfRound)
                add(mf_round_static<INNER, CONSEC, MT, T, false>(jb, iv, I, base, e, lds, msc, mm,
                                                                 po, sa));
        } else if constexpr (CONSEC) {
            // the waves take equal contiguous runs of rounds
            const int r0 = (int)((lo - a) / kMfSPW);
            const long long n = (e - lo + kMfSPW - 1) / kMfSPW;
            mf_blocks<INNER, MT, T, false>(
                jb, iv, I, a, end, e, r0 + (int)(n * wave / kMfWaves),
                r0 + (int)(n * (wave + 1) / kMfWaves), lds, msc, mm, sa,
                [&](int) -> const MfPolar & { return po; }, add);
        }
        lo = e;
    }
}

// The same for requests summed from the binary32 fold table of
// prepare_kernel (rows of consecutive m): short mode lists, whose operand
// table would not fit the space of their fold table, and generic Kerr, one
// polar index k after the other.  Each workgroup forms the operand values of
// its intervals itself (latency; what a visit costs is stated at mf_terms_path).  In Kerr
// the waves' running sums of 12 rounds at a time stay in LDS, so a (interval,
// k) is staged once per 6144 samples.  Measured against the vector kernel:
// 225 terms on 1.26 million samples 86 -> 46 us (shape 2 x 2), 34587 Kerr
// modes (9 x 1281 terms) on 3.16 million 7230 -> 1000 us (3 x 2); the error
// against binary64 falls too, 8.1e-7 -> 2.6e-7 and 1.6e-6 -> 4.6e-7.
template <bool INNER, int MT, int T, bool KERR>
__device__ void mf_range_terms(const SumJob &jb, long long lo, long long hi, int first,
                               float4 *lds, double2 *iacc) {
    if (lo >= hi) return;
    __shared__ MfTerms<MT, T> M;
    const int wave = threadIdx.x / kWave;
    MfSampleArea *sa = (MfSampleArea *)((char *)lds + mf_table_bytes(MT, T)) + wave;
    float2 *hp = (float2 *)((char *)lds + mf_table_bytes(MT, T) + kMfWaves * sizeof(MfSampleArea)) +
                 wave * kMfKerrRounds * kMfSPW;
    __syncthreads();        // areas of a previous job of another shape no longer read
    sa->c[0][threadIdx.x & (kWave - 1)] = make_float2(1.0f, 0.0f);
    const int mm[1] = {jb.mf_m0};
    const FEW_AS4 long long *st = cptr(jb.starts);
    auto add = [&](double2 v) {
        if constexpr (INNER) {
            double2 a = iacc[threadIdx.x];
            a.x = a.x + v.x;
            a.y = a.y + v.y;
            iacc[threadIdx.x] = a;
        }
    };
    for (int x = threadIdx.x; x < 8 * MT * 32 * T; x += 64 * kMfWaves) (&M.idx[0][0])[x] = -1;
    // operand values of (interval, polar index) and how its products are formed
    auto stage = [&](int iv, int kp) {
        mf_terms_stage<MT, T>(jb, iv, kp, M, lds);
        const MfInterval I = mf_interval<true, MT, T>(
            jb, iv, [&](int f) { return __uint_as_float(M.top[f]); });
        if (I.block == 0) {
            mf_convert<MT, T>(lds);
            __syncthreads();
        }
        return I;
    };
    for (int iv = first; iv <= jb.K - 2 && lo < hi; ++iv) {
        const long long a = st[iv], end = st[iv + 1], e = min(hi, end);
        if (e <= lo) continue;
        // the waves take equal contiguous runs of rounds
        const int r0 = (int)((lo - a) / kMfSPW);
        const int n = (int)((e - lo + kMfSPW - 1) / kMfSPW);
        const int ra = r0 + (int)((long long)n * wave / kMfWaves);
        const int rb = r0 + (int)((long long)n * (wave + 1) / kMfWaves);
        // (generic Kerr: at most kMfKerrRounds rounds of each wave at a time)
        const int most = (n + kMfWaves - 1) / kMfWaves, step = KERR ? kMfKerrRounds : most;
        for (int c = 0; c < most; c += step) {      // uniform per workgroup
            const int ca = min(rb, ra + c), cb = min(rb, ca + step);
            for (int q = KERR ? jb.mf_nk - 1 : 0; q >= 0; --q) {
                const MfInterval I = stage(iv, jb.mf_k0 + q);
                MfPolar po{hp, !KERR || q == jb.mf_nk - 1, !KERR || q == 0, jb.mf_k0};
                auto each = [&](int r) -> const MfPolar & {
                    if constexpr (KERR) po.hp = hp + (r - ca) * kMfSPW;
                    return po;
                };
                if (I.block == 0) {
                    for (int r = ca; r < cb; ++r)
                        add(mf_round_static<INNER, true, MT, T, KERR>(
                            jb, iv, I, a + (long long)r * kMfSPW, e, lds, M.un, mm, each(r), sa));
                } else {
                    mf_blocks<INNER, MT, T, KERR>(jb, iv, I, a, end, e, ca, cb, lds, M.un, mm, sa,
                                                  each, add);
                }
            }
        }
        lo = e;
    }
}

// Share r of G of [0, total): workgroup b runs on XCD b mod 8 and takes share
// (b mod 8) G/8 + b/8, so each XCD works through one contiguous eighth.
__device__ __forceinline__ void mf_share(long long total, long long *lo, long long *hi) {
    const int G = gridDim.x, b = blockIdx.x;
    const int r = (G % 8 == 0) ? (b & 7) * (G >> 3) + (b >> 3) : b;
    *lo = total * r / G;
    *hi = total * (r + 1) / G;
}

// Launches whose XCD split follows the weights: a multiple of 8 workgroups
// (XCD b mod 8 takes workgroup b), at most kMfBalanceWG, and weights within
// [1/4, 4].
__device__ __forceinline__ bool mf_balanced(const SumJob &jb) {
    if (jb.btime == nullptr || gridDim.x % 8 != 0 || gridDim.x > kMfBalanceWG) return false;
    for (int x = 0; x < 8; ++x)
        if (!(jb.bw[x] >= 0.25f && jb.bw[x] <= 4.0f)) return false;
    return true;
}

// Share of workgroup b with the weights wl: XCD x takes the samples
// [X_x, X_{x+1}), X_x = floor(total W_x / W_8) with W the running sum of the
// weights (X_0 = 0, X_8 = total), in equal contiguous slots of its G/8
// workgroups.
__device__ __forceinline__ void mf_share_w(const float *wl, long long total, long long *lo,
                                           long long *hi) {
    const int G = gridDim.x, b = blockIdx.x;
    const int x = b & 7, j = b >> 3, S = G >> 3;
    double cw = 0.0, all = 0.0;
    for (int i = 0; i < 8; ++i) {
        const double w = wl[i];
        if (i < x) cw += w;
        all += w;
    }
    const long long a = x == 0 ? 0 : (long long)((double)total * (cw / all));
    const long long e = x == 7 ? total : (long long)((double)total * ((cw + (double)wl[x]) / all));
    *lo = a + (e - a) * j / S;
    *hi = a + (e - a) * (j + 1) / S;
}

// A job is shared out in units: an interval counts its samples and a gap before
// them (mf_gap), so that a share holds fewer samples where it has more
// intervals to form operands for.  Units [u0, u1) -> samples [lo, hi), both moved
// up to the grid of rounds (64 samples from the first one of their interval), so
// that every round belongs to one workgroup and a sample's block does not depend
// on how the samples are shared out; iv: the interval of lo (or the one before
// it).  Both searches run in step: a chain of scalar loads is what a short
// launch waits for.
__device__ __forceinline__ void mf_units(const SumJob &jb, long long u0, long long u1,
                                         long long gap, long long *lo, long long *hi, int *iv) {
    const FEW_AS4 long long *st = cptr(jb.starts);
    int a0 = 0, a1 = 0;
    for (int step = 512; step > 0; step >>= 1) {    // (K <= 1024)
        const int q0 = min(a0 + step, jb.K - 2), q1 = min(a1 + step, jb.K - 2);
        if (st[q0] + gap * q0 <= u0) a0 = q0;
        if (st[q1] + gap * q1 <= u1) a1 = q1;
    }
    auto sample = [&](int i, long long u) {
        const long long a = st[i], r = max(u - gap * (i + 1) - a, 0ll);
        return min((long long)st[i + 1], a + (r + kMfSPW - 1) / kMfSPW * kMfSPW);
    };
    *lo = sample(a0, u0);
    *hi = sample(a1, u1);
    *iv = a0;
}

// A single-request launch: this workgroup's share of the samples through
// range(lo, hi, first interval), its time reported, and (INNER) its sums of iacc in
// partial.  gap: of mf_units.
template <bool INNER, typename Range>
__device__ __forceinline__ void mf_single(const SumJob &jb, double2 *iacc, long long gap,
                                          Range range) {
    if constexpr (INNER) iacc[threadIdx.x] = make_double2(0.0, 0.0);
    long long lo, hi, u0, u1;
    int iv;
    // the inner-product launch keeps the equal split (its binary64 sums
    // then do not depend on the weights)
    const unsigned long long t0 = wall_clock64();
    const long long units = jb.n + gap * (jb.K - 1);
    if (!INNER && mf_balanced(jb))
        mf_share_w(jb.bw, units, &u0, &u1);
    else
        mf_share(units, &u0, &u1);
    mf_units(jb, u0, u1, gap, &lo, &hi, &iv);
    range(lo, hi, iv);
    if (!INNER && jb.btime != nullptr && (int)blockIdx.x < kMfBalanceWG) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long dt = min(wall_clock64() - t0, (1ull << kMfTagShift) - 1);
            jb.btime[blockIdx.x] = ((unsigned long long)jb.btag << kMfTagShift) | dt;
        }
    }
    if constexpr (INNER) {
        __shared__ double2 red[kMfWaves];
        double2 v = wave_sum(iacc[threadIdx.x]);
        if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            double2 t = red[0];
            for (int w = 1; w < kMfWaves; ++w) {
                t.x = t.x + red[w].x;
                t.y = t.y + red[w].y;
            }
            jb.partial[blockIdx.x] = t;
        }
    }
}

// A batched launch: the jobs' units, cost(job) each, laid end to end (job j from
// sample_base_j), split into equal shares; range(job, lo, hi, first interval).
// most: of the gaps.
template <typename Cost, typename Range>
__device__ __forceinline__ void mf_batch(const SumJob *jobs, int n_jobs, long long total, int most,
                                         Cost cost, Range range) {
    long long lo, hi;
    mf_share(total, &lo, &hi);
    int j = 0, top = n_jobs - 1;
    while (j < top) {
        const int mid = (j + top + 1) >> 1;
        if (*cptr(&jobs[mid].sample_base) <= lo) j = mid; else top = mid - 1;
    }
    for (; j < n_jobs; ++j) {
        const long long b0 = *cptr(&jobs[j].sample_base);
        if (b0 >= hi) break;
        const SumJob jb = load_uniform(jobs + j);
        const long long gap = mf_gap(jb.n, most), units = jb.n + gap * (jb.K - 1);
        // (a share's end and the next one's start round to the same unit)
        const long long c = cost(jb);
        const long long u0 = (max(lo, b0) - b0 + c - 1) / c;
        const long long u1 = (min(hi, b0 + units * c) - b0 + c - 1) / c;
        long long a, e;
        int iv;
        mf_units(jb, u0, u1, gap, &a, &e, &iv);
        if (a < e) range(jb, a, e, iv);
    }
}

// ---- binary64 on the matrix cores ------------------------------------------
// The same contraction from the binary64 fold table on
// v_mfma_f64_16x16x4_f64: 16 matrix rows (8 signed m, re/im) by 16 samples,
// two values of a = |n| (re/im columns) per product, f^a by a recurrence in
// f^2 per column lane.  Products and vector binary64 arithmetic share one unit
// (measured: they add), and it is the bound, so the count of binary64
// operations per term decides: the vector kernel spends 10 FMAs per term
// (cubic and recurrence), a product spends 2 per power of v (n and -n meet in
// one column pair).
//
// The cubic is written about the centre v0 of a block of 32 or 16 samples, with
// d = v - v0:
//   C(v) = T_0 + d T_1 + d^2 (b_2 + (3 v0 + d) b_3),
//   T_0 = C(v0), T_1 = C'(v0),
// T_0 and T_1 formed in binary64 from the staged b_p for each use (6 operations of
// 4 cycles against 4 or 2 products of 64).  The rest is small: |d| <= w, half the
// block's width in v.  Where (M_2 + 4 M_3) w^2 <= 2^-30 M_0 (M_p the largest |b_p| of the
// interval, M_0 of p <= 1) it is summed from fp16 hi + lo operands (22 bits) with
// binary32 harmonics and accumulation, at 1/16 of the binary64 products' cost: 4 binary64 operations per term in all.  The
// harmonics f^a and E^row are binary32 power chains of up to 31 and 24 steps, so
// a term's rest is good to 2^-19 at worst and adds up to 2^-49 M_0; the vector kernel's
// Horner recurrence rounds at 2^-53 of its running sum once per term it walks.
// Else T_2 = C''(v0) / 2 takes binary64 products too and only d^3 b_3 is left to
// fp16 (w^3 M_3 <= 2^-30 M_0), else all four powers take them.  Measured at the limits
// (cubics swept through them, modes of one size, 0.02 to 3 million samples): the
// largest error is 1.3e-15 to 4e-15, as with four powers everywhere, the vector
// kernel's 4e-15 to 1e-14.
// Measured (3843 modes, 1281 terms, 3.16 million samples): 1430 -> 920 us, of which
// the products 560 at the rate of a large binary64 matrix product.
struct MfPlan64 {
    int P;          // powers in binary64 products: 2, 3 or 4
    int nt;         // P = 2: sample tiles of 16 per block, 2 or 1
    bool lo3;       // b_3 of the rest takes all three fp16 products
};

template <int MT, int T>
struct MfTerms64 {
    int idx[8 * MT][32 * T];            // n + 16 T; -1: no term
    unsigned m01[4 * MT], m2[4 * MT], m3[4 * MT];   // largest |b_p| per row pair (binary32 bits)
    float un[4 * MT];                   // 2^E of the fp16 values
};

// Cubic in u -> cubic in v = 2 u - 1.
__device__ __forceinline__ void mf_recentre(double a0, double a1, double a2, double a3, double *b) {
    const double h1 = 0.5 * a1, h2 = 0.25 * a2, h3 = 0.125 * a3;
    b[0] = a0 + (h1 + (h2 + h3));
    b[1] = h1 + fma(2.0, h2, 3.0 * h3);
    b[2] = fma(3.0, h3, h2);
    b[3] = h3;
}

// LDS: base [mt][step][p][lane 64] doubles, then rest [mt][p - 2][t][hi, lo][lane 64][8].
static constexpr size_t mf64_base_bytes(int MT, int ns) { return (size_t)MT * ns * 2048; }
static constexpr size_t mf64_rest_bytes(int MT, int T) { return (size_t)MT * 2 * T * 2048; }

// How the interval's rounds are summed (every wave forms the same).
template <int MT, int T>
__device__ __forceinline__ MfPlan64 mf64_plan(const SumJob &jb, double inv_h2,
                                              const MfTerms64<MT, T> &M) {
    unsigned b01 = 0, b2 = 0, b3 = 0;
#pragma unroll
    for (int i = 0; i < 4 * MT; ++i) {
        b01 = max(b01, M.m01[i]);
        b2 = max(b2, M.m2[i]);
        b3 = max(b3, M.m3[i]);
    }
    const float M0 = uniform_f32(__uint_as_float(b01)), M2 = uniform_f32(__uint_as_float(b2)),
                M3 = uniform_f32(__uint_as_float(b3));
    // half width of a block of 32 samples.  Blocks do not end with the interval:
    // v0 lies up to 1 + w, and |3 v0 + d| = |3 v - 2 d| <= 3 + 2 w for |v| <= 1.  In
    // an interval of less than 64 samples (w > 1/2) the rest, small there for the
    // interval's sake alone, would be multiplied up again by d^2 and 3 v0 + d (an
    // interval of 8 samples: error 9e-13, of 1.5 samples 2e-9): no blocks.
    const float w = uniform_f32((float)(16.0 * jb.dt * inv_h2));
    MfPlan64 I{4, 1, true};
    // (NaN, infinite and tiny values: all in binary64)
    if (w <= 0.5f && M0 > 1e-30f && M0 < 1e30f && M2 < 1e30f && M3 < 1e30f) {
        const float lim = 0x1p-30f * M0, q = (M2 + 4.0f * M3) * w * w;
        if (q <= 4.0f * lim) {
            I.P = 2;
            I.nt = q <= lim ? 2 : 1;
        } else if (M3 * w * w * w <= lim) {
            I.P = 3;
        }
        const float u = I.nt == 2 ? w : 0.5f * w;
        I.lo3 = !(I.P == 2 && (M2 + 8192.0f * M3) * u * u <= lim);
    }
    return I;
}

// Operand values of interval iv and polar index kp: mf_terms_stage in binary64.
// Lane 16 k + rho of a product's left operand holds row rho = 4 i + g of (signed m
// 2 g + i / 2, component i % 2) and column k = 2 (a % 2) + component, so that a
// result lane (16 g + sample) holds both components of rows 2 g and 2 g + 1, as
// the fp16 products' does.
template <int MT, int T>
__device__ __forceinline__ MfPlan64 mf64_stage(const SumJob &jb, int iv, int kp, int ns,
                                               double inv_h2, MfTerms64<MT, T> &M, double *base,
                                               unsigned *rest) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));       // (addresses formed here, not kept through the rounds)
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    __syncthreads();                                // the previous values no longer read
    if (tid < 4 * MT) M.m01[tid] = M.m2[tid] = M.m3[tid] = 0u;
    mf_terms_scatter(jb, kp, 16 * T, 32 * T, &M.idx[0][0], lane, wave);
    __syncthreads();
    constexpr int kTasks = MT * T * 2, kTurns = (kTasks + kMfWaves - 1) / kMfWaves;
    const double2 *last = (const double2 *)jb.table + ((size_t)iv * jb.n_terms + jb.n_terms - 1) * 4;
    double2 v[kTurns][8];
#pragma unroll
    for (int q = 0; q < kTurns; ++q) {
        const int task = min(wave + q * kMfWaves, kTasks - 1);      // (mt, t, half of the a)
        const int row = 8 * (task / (2 * T)) + (lane >> 3), a = 8 * (task % (2 * T)) + (lane & 7);
        const int tp = M.idx[row][16 * T + a], tq = a > 0 ? M.idx[row][16 * T - a] : -1;
        const double2 *cp = last - 4 * (size_t)max(tp, 0), *cq = last - 4 * (size_t)max(tq, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[q][i] = cp[i];
            v[q][4 + i] = cq[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (tp < 0) v[q][i] = make_double2(0.0, 0.0);
            if (tq < 0) v[q][4 + i] = make_double2(0.0, 0.0);
        }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < kTurns; ++q) {
        if (wave + q * kMfWaves >= kTasks) continue;
        const int task = wave + q * kMfWaves;
        const int row = 8 * (task / (2 * T)) + (lane >> 3), a = 8 * (task % (2 * T)) + (lane & 7);
        M.idx[row][16 * T + a] = -1;
        M.idx[row][16 * T - a] = -1;
        unsigned m01 = 0, m2 = 0, m3 = 0;
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
            double b[4], c[4];
            mf_recentre(v[q][h].x, v[q][h + 1].x, v[q][h + 2].x, v[q][h + 3].x, b);
            mf_recentre(v[q][h].y, v[q][h + 1].y, v[q][h + 2].y, v[q][h + 3].y, c);
            auto up = [](unsigned m, double x, double y) {
                return max(m, max(abs_bits((float)x), abs_bits((float)y)));
            };
            m01 = up(up(m01, b[0], c[0]), b[1], c[1]);
            m2 = up(m2, b[2], c[2]);
            m3 = up(m3, b[3], c[3]);
        }
        m01 = lanes_max<4>(m01);                    // the 8 columns of two rows
        m2 = lanes_max<4>(m2);
        m3 = lanes_max<4>(m3);
        if ((lane & 15) == 0) {
            atomicMax(&M.m01[row >> 1], m01);
            atomicMax(&M.m2[row >> 1], m2);
            atomicMax(&M.m3[row >> 1], m3);
        }
    }
    __syncthreads();
    const MfPlan64 I = mf64_plan<MT, T>(jb, inv_h2, M);
#pragma unroll
    for (int q = 0; q < kTurns; ++q) {
        if (wave + q * kMfWaves >= kTasks) continue;
        const int task = wave + q * kMfWaves, mt = task / (2 * T), ta = task % (2 * T);
        const int r = lane >> 3, a = 8 * ta + (lane & 7), t = ta >> 1;
        // scale of the larger of b_2 and b_3, or of b_3 where it is summed alone (in
        // that of b_2 a b_3 of 2^-7 b_2 keeps only 17 bits, and three powers in
        // binary64 were off by 1.2e-14 of |h| near their limit, now 2.5e-15)
        const float m3 = __uint_as_float(M.m3[4 * mt + (r >> 1)]);
        const float mx = I.P == 3 ? m3 : fmaxf(__uint_as_float(M.m2[4 * mt + (r >> 1)]), m3);
        int e = 0;
        if (mx > 0.0f && mx < INFINITY) frexpf(mx, &e);
        e = min(max(e, -126), 127);
        const double sc = ldexp(1.0, -e);
        if ((lane & 15) == 0) M.un[4 * mt + (r >> 1)] = ldexpf(1.0f, e);
        // columns per power: (Re P + Re Q, Im Q - Im P) of row component 0,
        // (Im P + Im Q, Re P - Re Q) of component 1
        const double2 *P = v[q], *Q = v[q] + 4;
        double o[2][2][4];
        mf_recentre(P[0].x + Q[0].x, P[1].x + Q[1].x, P[2].x + Q[2].x, P[3].x + Q[3].x, o[0][0]);
        mf_recentre(Q[0].y - P[0].y, Q[1].y - P[1].y, Q[2].y - P[2].y, Q[3].y - P[3].y, o[0][1]);
        mf_recentre(P[0].y + Q[0].y, P[1].y + Q[1].y, P[2].y + Q[2].y, P[3].y + Q[3].y, o[1][0]);
        mf_recentre(P[0].x - Q[0].x, P[1].x - Q[1].x, P[2].x - Q[2].x, P[3].x - Q[3].x, o[1][1]);
        const int step = a >> 1, g = (a >> 2) & 3, j = a & 3;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (step < ns) {
                const int rho = 4 * (2 * (r & 1) + c) + (r >> 1);
                double *d = base + (size_t)(mt * ns + step) * 256 + rho + 32 * (a & 1);
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    d[64 * p] = o[c][0][p];
                    d[64 * p + 16] = o[c][1][p];
                }
            }
            // a = 16 t + 4 g + j: fragment lane 2 r + c + 16 g, values 2 j, 2 j + 1
#pragma unroll
            for (int p = 2; p < 4; ++p) {
                unsigned hi, lo;
                split_pair((float)(o[c][0][p] * sc), (float)(o[c][1][p] * sc), hi, lo);
                unsigned *f = rest + (((mt * 2 + p - 2) * T + t) * 128 + 2 * r + c + 16 * g) * 4 + j;
                f[0] = hi;
                f[256] = lo;
            }
        }
    }
    __syncthreads();
    return I;
}

__device__ __forceinline__ void cmul64(double ar, double ai, double br, double bi, double *r,
                                       double *i) {
    *r = fma(ar, br, -(ai * bi));
    *i = fma(ar, bi, ai * br);
}

struct MfPolar64 {
    double2 *hp;            // this round's running values
    bool first, last;       // highest, lowest k
    int k0;
};

// fp16 sum over |n| of the rest of one sample tile: the columns f^a.
template <int T>
__device__ __forceinline__ void mf64_columns(float fr, float fi, mf_u4 (&bh)[T], mf_u4 (&bl)[T]) {
    const int g = (threadIdx.x & (kWave - 1)) >> 4;
    float r2, i2, r3, i3, r4, i4, r8, i8, cr, ci;
    cmulf(fr, fi, fr, fi, &r2, &i2);
    cmulf(r2, i2, fr, fi, &r3, &i3);
    cmulf(r2, i2, r2, i2, &r4, &i4);
    cmulf(r4, i4, r4, i4, &r8, &i8);
    cmulf(g & 1 ? r4 : 1.0f, g & 1 ? i4 : 0.0f, g & 2 ? r8 : 1.0f, g & 2 ? i8 : 0.0f, &cr, &ci);
    float w[8] = {cr, ci};
    cmulf(cr, ci, fr, fi, &w[2], &w[3]);
    cmulf(cr, ci, r2, i2, &w[4], &w[5]);
    cmulf(cr, ci, r3, i3, &w[6], &w[7]);
    float r16, i16;
    cmulf(r8, i8, r8, i8, &r16, &i16);
#pragma unroll
    for (int t = 0; t < T; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (t > 0) {
                float nr, ni;
                cmulf(w[2 * i], w[2 * i + 1], r16, i16, &nr, &ni);
                w[2 * i] = nr;
                w[2 * i + 1] = ni;
            }
            unsigned h, l;
            split_pair(w[2 * i], w[2 * i + 1], h, l);
            bh[t][i] = h;
            bl[t][i] = l;
        }
    }
}

typedef double mf_double4 __attribute__((ext_vector_type(4)));

// 4 x 4 exchange between the 16-lane groups: x[q] of group g <- x[g] of group q.
__device__ __forceinline__ void lane_transpose(float (&x)[4]) {
    lane_swap32(x[0], x[2]);
    lane_swap32(x[1], x[3]);
    lane_swap16(x[0], x[1]);
    lane_swap16(x[2], x[3]);
}

// This lane's sample from the rows of one tile: c[i][g] holds component i % 2 of
// row 2 g + i / 2; sum over the 8 rows of E^row (the row's value), by Horner.
template <typename R>
__device__ __forceinline__ void mf64_rows(const R (&c)[4][4], R er, R ei, R *yr, R *yi) {
    R sr = c[2][3], si = c[3][3];
#pragma unroll
    for (int row = 6; row >= 0; --row) {
        const R vr = c[2 * (row & 1)][row >> 1], vi = c[2 * (row & 1) + 1][row >> 1];
        const R nr = fmar(sr, er, fmar(-si, ei, vr));
        si = fmar(sr, ei, fmar(si, er, vi));
        sr = nr;
    }
    *yr = sr;
    *yi = si;
}

// The rest of a round, sum of d^(P-2).. b_p f^a over fp16 operands, without its factor
// d^2 (P = 2) or d^3 (P = 3): this lane's sample.
template <int MT, int T, int P>
__device__ __forceinline__ void mf64_rest(const uint4 *rest, const float *un, bool lo3, float fr,
                                          float fi, float vq, float er, float ei, float e8r,
                                          float e8i, float *yr, float *yi) {
    const int lane = threadIdx.x & (kWave - 1), col = lane & 15, g = lane >> 4;
    mf_u4 bh[4][T], bl[4][T];
    float vv[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int src = 16 * nt + col;
        mf64_columns<T>(__shfl(fr, src), __shfl(fi, src), bh[nt], bl[nt]);
        vv[nt] = __shfl(vq, src);
    }
    float sr = 0.0f, si = 0.0f;
#pragma unroll 1
    for (int mt = MT - 1; mt >= 0; --mt) {
        mf_float4 s[4];
        auto prod = [&](uint4 A, const mf_u4 (&B)[4][T], int t) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                s[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                    __builtin_bit_cast(mf_half8, A), __builtin_bit_cast(mf_half8, B[nt][t]), s[nt],
                    0, 0, 0);
        };
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) s[nt] = mf_float4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int p = 3; p >= P; --p) {
            if (p == 2) {
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[nt][i] = s[nt][i] * vv[nt];
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint4 *f = rest + ((mt * 2 + p - 2) * T + t) * 128 + lane;
                const uint4 ah = f[0];
                if (p == 2 || lo3) {
                    prod(f[64], bh, t);
                    prod(ah, bl, t);
                }
                prod(ah, bh, t);
            }
        }
        const float u = un[4 * mt + g];
        float c[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) c[i][nt] = s[nt][i] * u;
            lane_transpose(c[i]);
        }
        float wr, wi;
        mf64_rows<float>(c, er, ei, &wr, &wi);
        const float nr = fmar(sr, e8r, fmar(-si, e8i, wr));
        si = fmar(sr, e8i, fmar(si, e8r, wi));
        sr = nr;
    }
    *yr = sr;
    *yi = si;
}

// One round of a wave: the 64 samples wbase + l, P powers in binary64, blocks of
// NT sample tiles (P = 4: none, v0 = 0).
template <bool INNER, int MT, int T, bool KERR, int P, int NT>
__device__ __forceinline__ double2 mf64_round(const SumJob &jb, int iv, double ti, double inv_h2,
                                              bool lo3, long long wbase, long long e, int ns,
                                              const double *base, const uint4 *rest,
                                              const float *un, const MfPolar64 &po) {
    const int lane = threadIdx.x & (kWave - 1), col = lane & 15, g = lane >> 4;
    const FEW_AS4 double *pc = cptr(jb.pcoef) + (size_t)iv * (KERR ? 24 : 16);
    const long long jo = wbase + lane;
    double2 dv = make_double2(0.0, 0.0);
    if constexpr (INNER) {
        if (jo < e) dv = ((const double2 *)jb.data)[jo];
    }
    // this lane's sample; v at the centre of the round's first block, and the
    // step from block to block
    const dd x = two_sum(dev_sample_time(jb.t_start, jb.dt, jo < e ? jo : e - 1), -ti);
    double vc = 0.0, vs = 0.0;
    if constexpr (P < 4) {
        const double xm = dev_sample_time(jb.t_start, jb.dt, wbase) - ti;
        vc = uniform_f64(fma(fma(0.5 * (16 * NT - 1), jb.dt, xm), inv_h2, -1.0));
        vs = uniform_f64(16.0 * NT * jb.dt * inv_h2);
    }
    const double v0 = fma((double)(g / NT), vs, vc);        // of this lane's block
    const double dl = fma(x.hi, inv_h2, -1.0) - v0;
    double z0r = 1.0, z0i = 0.0, tr = 1.0, tth = 0.0, Er, Ei, fr, fi;
    {
        const double pf = phase_eval<true>(pc, x), pr = phase_eval<true>(pc + 8, x);
        unit_phasor<double>(pf, &Er, &Ei);
        unit_phasor<double>(pr, &fr, &fi);
        if constexpr (KERR) {
            const double pt = phase_eval<true>(pc + 16, x);
            unit_phasor<double>(pt, &tr, &tth);
            if (po.last && po.k0 != 0)
                unit_phasor<double>(d_reduce_2pi((double)po.k0 * pt), &z0r, &z0i);
        }
    }
    double E8r, E8i, hr, hq;
    {
        double E2r, E2i, E4r, E4i;
        cmul64(Er, Ei, Er, Ei, &E2r, &E2i);
        cmul64(E2r, E2i, E2r, E2i, &E4r, &E4i);
        cmul64(E4r, E4i, E4r, E4i, &E8r, &E8i);
        if (!KERR || po.last) {
            // z_0 = E^{m_0} (e^{-i k_0 Phi_theta}) from the binary powers
            const int m0 = jb.mf_m0, am = m0 < 0 ? -m0 : m0;
            double ar = 1.0, ai = 0.0;
            auto take = [&](double r, double i) {
                double nr, ni;
                cmul64(ar, ai, r, i, &nr, &ni);
                ar = nr;
                ai = ni;
            };
            if (am & 1) take(Er, Ei);
            if (am & 2) take(E2r, E2i);
            if (am & 4) take(E4r, E4i);
            if (am & 8) take(E8r, E8i);
            if (am & 16) {
                take(E8r, E8i);
                take(E8r, E8i);
            }
            if (m0 < 0) ai = -ai;
            if (KERR && po.k0 != 0) take(z0r, z0i);
            z0r = ar;
            z0i = ai;
        }
    }
    float yr = 0.0f, yi = 0.0f;
    if constexpr (P < 4)
        mf64_rest<MT, T, P>(rest, un, lo3, (float)fr, (float)fi, (float)fma(3.0, v0, dl), (float)Er,
                            (float)Ei, (float)E8r, (float)E8i, &yr, &yi);
    double sr = 0.0, si = 0.0;
#pragma unroll 1
    for (int n0 = 0; n0 < 4; n0 += NT) {
        const double vb = uniform_f64(fma((double)(n0 / NT), vs, vc));
        mf_double4 acc[MT][P][NT];
        double own[NT], oth[NT], f2r[NT], f2i[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            // columns: lane group g holds component g % 2 of f^a, a = 2 s + g / 2
            // in step s
            const int src = 16 * (n0 + nt) + col;
            const double ar = __shfl(fr, src), ai = __shfl(fi, src);
            double i2;
            cmul64(ar, ai, ar, ai, &f2r[nt], &i2);
            const double pr = g & 2 ? ar : 1.0, pi = g & 2 ? ai : 0.0;
            own[nt] = g & 1 ? pi : pr;
            oth[nt] = g & 1 ? pr : pi;
            f2i[nt] = g & 1 ? i2 : -i2;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int p = 0; p < P; ++p) acc[mt][p][nt] = mf_double4{0.0, 0.0, 0.0, 0.0};
        }
        const double *b = base + lane;
#pragma unroll 1
        for (int s = 0; s < ns; ++s, b += 256) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const double *bm = b + (size_t)mt * ns * 256;
                const double b0 = bm[0], b1 = bm[64], b2 = bm[128], b3 = bm[192];
                double q[4] = {b0, b1, b2, b3};
                if constexpr (P < 4) {
                    const double h = fma(vb, b3, b2);
                    q[0] = fma(vb, fma(vb, h, b1), b0);
                    q[1] = fma(vb, fma(vb, b3, h + h), b1);
                    if constexpr (P == 3) q[2] = fma(vb, b3 + b3, h);
                }
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[mt][p][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            q[p], own[nt], acc[mt][p][nt], 0, 0, 0);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const double o = fma(own[nt], f2r[nt], oth[nt] * f2i[nt]);
                oth[nt] = fma(oth[nt], f2r[nt], -(own[nt] * f2i[nt]));
                own[nt] = o;
            }
        }
        // rows: z_r = z_0 E^{2g} E^{8 mt} (E for the odd row), Horner in E^8
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int src = 16 * (n0 + nt) + col;
            const double d = __shfl(dl, src), er = __shfl(Er, src), ei = __shfl(Ei, src);
            const double e8r = __shfl(E8r, src), e8i = __shfl(E8i, src);
            double yr = 0.0, yi = 0.0;
#pragma unroll
            for (int mt = MT - 1; mt >= 0; --mt) {
                double c[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    c[i] = acc[mt][P - 1][nt][i];
#pragma unroll
                    for (int p = P - 2; p >= 0; --p) c[i] = fma(d, c[i], acc[mt][p][nt][i]);
                }
                const double wr = fma(er, c[2], fma(-ei, c[3], c[0]));
                const double wi = fma(er, c[3], fma(ei, c[2], c[1]));
                const double nr = mt == MT - 1 ? wr : fma(yr, e8r, fma(-yi, e8i, wr));
                yi = mt == MT - 1 ? wi : fma(yr, e8i, fma(yi, e8r, wi));
                yr = nr;
            }
            // times E^{2g}, summed over the lane groups; the tile's own lanes keep it
            double e2r, e2i, e4r, e4i, gr, gi, hr, hi;
            cmul64(er, ei, er, ei, &e2r, &e2i);
            cmul64(e2r, e2i, e2r, e2i, &e4r, &e4i);
            cmul64(g & 1 ? e2r : 1.0, g & 1 ? e2i : 0.0, g & 2 ? e4r : 1.0, g & 2 ? e4i : 0.0, &gr, &gi);
            cmul64(yr, yi, gr, gi, &hr, &hi);
            hr = hr + __shfl_xor(hr, 16);
            hi = hi + __shfl_xor(hi, 16);
            hr = hr + __shfl_xor(hr, 32);
            hi = hi + __shfl_xor(hi, 32);
            sr = g == n0 + nt ? hr : sr;
            si = g == n0 + nt ? hi : si;
        }
    }
    if constexpr (P < 4) {
        const double w = P == 2 ? dl * dl : dl * dl * dl;
        sr = fma(w, (double)yr, sr);
        si = fma(w, (double)yi, si);
    }
    if constexpr (KERR) {
        if (!po.first) {
            const double2 q = po.hp[lane];
            const double nr = fma(q.x, tr, fma(-q.y, tth, sr));
            si = fma(q.x, tth, fma(q.y, tr, si));
            sr = nr;
        }
        if (!po.last) {
            po.hp[lane] = make_double2(sr, si);
            __builtin_amdgcn_wave_barrier();
            return make_double2(0.0, 0.0);
        }
    }
    cmul64(sr, si, z0r, z0i, &hr, &hq);
    double dh = 0.0, hh = 0.0;
    if (jo < e) {
        if constexpr (INNER) {
            dh = dv.x * hr + dv.y * hq;
            hh = hr * hr + hq * hq;
        } else {
            ((double2 *)jb.out)[jo] = make_double2(hr, hq);
        }
    }
    return make_double2(dh, hh);
}

constexpr int kMfKerrRounds64 = 3;

// Samples [lo, hi) of one job, from interval `first` on (mf_range_terms in
// binary64).
template <bool INNER, int MT, int T, bool KERR>
__device__ void mf_range_f64(const SumJob &jb, long long lo, long long hi, int first,
                             double *base, double2 *iacc) {
    if (lo >= hi) return;
    __shared__ MfTerms64<MT, T> M;
    const int wave = threadIdx.x / kWave, ns = jb.mf_ns;
    unsigned *rest = (unsigned *)((char *)base + mf64_base_bytes(MT, ns));
    double2 *hp = (double2 *)((char *)rest + mf64_rest_bytes(MT, T)) + wave * kMfKerrRounds64 * kMfSPW;
    const FEW_AS4 long long *st = cptr(jb.starts);
    for (int x = threadIdx.x; x < 8 * MT * 32 * T; x += 64 * kMfWaves) (&M.idx[0][0])[x] = -1;
    for (int iv = first; iv <= jb.K - 2 && lo < hi; ++iv) {
        const long long a = st[iv], end = st[iv + 1], e = min(hi, end);
        if (e <= lo) continue;
        const double ti = uniform_f64(jb.t[iv]);
        const double inv_h2 = uniform_f64(2.0 / (jb.t[iv + 1] - ti));
        const int r0 = (int)((lo - a) / kMfSPW);
        const int n = (int)((e - lo + kMfSPW - 1) / kMfSPW);
        const int ra = r0 + (int)((long long)n * wave / kMfWaves);
        const int rb = r0 + (int)((long long)n * (wave + 1) / kMfWaves);
        const int most = (n + kMfWaves - 1) / kMfWaves, step = KERR ? kMfKerrRounds64 : most;
        for (int c = 0; c < most; c += step) {      // uniform per workgroup
            const int ca = min(rb, ra + c), cb = min(rb, ca + step);
            for (int q = KERR ? jb.mf_nk - 1 : 0; q >= 0; --q) {
                const MfPlan64 I = mf64_stage<MT, T>(jb, iv, jb.mf_k0 + q, ns, inv_h2, M, base, rest);
                MfPolar64 po{hp, !KERR || q == jb.mf_nk - 1, !KERR || q == 0, jb.mf_k0};
                auto run = [&](auto P, auto NT) {
                    for (int r = ca; r < cb; ++r) {
                        if constexpr (KERR) po.hp = hp + (r - ca) * kMfSPW;
                        const double2 v = mf64_round<INNER, MT, T, KERR, decltype(P)::value, decltype(NT)::value>(
                            jb, iv, ti, inv_h2, I.lo3, a + (long long)r * kMfSPW, e, ns, base,
                            (const uint4 *)rest, M.un, po);
                        if constexpr (INNER) {
                            double2 s = iacc[threadIdx.x];
                            s.x = s.x + v.x;
                            s.y = s.y + v.y;
                            iacc[threadIdx.x] = s;
                        }
                    }
                };
                using std::integral_constant;
                if (I.P == 2 && I.nt == 2)
                    run(integral_constant<int, 2>{}, integral_constant<int, 2>{});
                else if (I.P == 2)
                    run(integral_constant<int, 2>{}, integral_constant<int, 1>{});
                else if (I.P == 3)
                    run(integral_constant<int, 3>{}, integral_constant<int, 2>{});
                else
                    run(integral_constant<int, 4>{}, integral_constant<int, 1>{});
            }
        }
        lo = e;
    }
}

template <bool INNER, bool CONSEC>
__global__ __launch_bounds__(64 * kMfWaves) void sum_mfma_kernel(SumJob jb) {
    extern __shared__ float4 mf_lds[];
    __shared__ float msc[kMfRows / 2];
    __shared__ int mm[kMfRows];
    __shared__ double2 iacc[INNER ? 64 * kMfWaves : 1];
    mf_single<INNER>(jb, iacc, mf_gap(jb.n, kMfGap), [&](long long lo, long long hi, int iv) {
        mf_range<INNER, CONSEC>(jb, lo, hi, iv, mf_lds, msc, mm, iacc);
    });
}

template <bool CONSEC>
__global__ __launch_bounds__(64 * kMfWaves) void sum_mfma_batch_kernel(const SumJob *jobs, int n_jobs,
                                                             long long total) {
    extern __shared__ float4 mf_lds[];
    __shared__ float msc[kMfRows / 2];
    __shared__ int mm[kMfRows];
    auto one = [](const SumJob &) { return 1ll; };
    mf_batch(jobs, n_jobs, total, kMfGap, one, [&](const SumJob &jb, long long a, long long e, int iv) {
        mf_range<false, CONSEC>(jb, a, e, iv, mf_lds, msc, mm, nullptr);
    });
}

template <bool INNER, int MT, int T, bool KERR>
__global__ __launch_bounds__(64 * kMfWaves) void sum_mfma_terms_kernel(SumJob jb) {
    extern __shared__ float4 mf_lds[];
    __shared__ double2 iacc[INNER ? 64 * kMfWaves : 1];
    mf_single<INNER>(jb, iacc, mf_gap(jb.n, kMfGapTerms), [&](long long lo, long long hi, int iv) {
        mf_range_terms<INNER, MT, T, KERR>(jb, lo, hi, iv, mf_lds, iacc);
    });
}

template <bool INNER, int MT, int T, bool KERR>
__global__ __launch_bounds__(64 * kMfWaves) void sum_mfma_f64_kernel(SumJob jb) {
    extern __shared__ float4 mf_lds[];
    __shared__ double2 iacc[INNER ? 64 * kMfWaves : 1];
    mf_single<INNER>(jb, iacc, mf_gap(jb.n, kMfGap), [&](long long lo, long long hi, int iv) {
        mf_range_f64<INNER, MT, T, KERR>(jb, lo, hi, iv, (double *)mf_lds, iacc);
    });
}

// Calls f(MT, T) with the smallest compiled shape that holds a request's rows
// and |n| (as std::integral_constants).
template <typename F>
__host__ __device__ static inline void mf_with_shape(int mt, int t, F f) {
    using std::integral_constant;
    using I1 = integral_constant<int, 1>;
    using I2 = integral_constant<int, 2>;
    using I3 = integral_constant<int, 3>;
    if (mt == 1 && t == 1) f(I1{}, I1{});
    else if (mt <= 2 && t == 1) f(I2{}, I1{});
    else if (mt <= 2) f(I2{}, I2{});
    else f(I3{}, I2{});
}

// Batches: one launch over all shapes (a workgroup per compute unit either way,
// and short requests of one shape would leave most of a launch of their own
// idle).
template <bool F64>
__global__ __launch_bounds__(64 * kMfWaves) void sum_mfma_terms_batch_kernel(const SumJob *jobs,
                                                                             int n_jobs,
                                                                             long long total) {
    extern __shared__ float4 mf_lds[];
    auto cost = [](const SumJob &jb) {
        return (long long)mf_terms_cost(jb.mf_terms, jb.mf_ns, F64);
    };
    mf_batch(jobs, n_jobs, total, F64 ? kMfGap : kMfGapTerms, cost,
             [&](const SumJob &jb, long long a, long long e, int iv) {
        auto run = [&](auto MT, auto T) {
            constexpr int mt = decltype(MT)::value, t = decltype(T)::value;
            if constexpr (F64)
                mf_range_f64<false, mt, t, false>(jb, a, e, iv, (double *)mf_lds, nullptr);
            else
                mf_range_terms<false, mt, t, false>(jb, a, e, iv, mf_lds, nullptr);
        };
        mf_with_shape(jb.mf_terms / 10, jb.mf_terms % 10, run);
    });
}

#pragma clang fp contract(on)

// ===========================================================================
// Mode selector (Sec. III D): per knot, order the modes by decreasing power
// |A|^2 (ties by increasing index), sum the powers sequentially in that order,
// and keep the shortest prefix that reaches (1 - eps) of the knot's total (at
// least the top mode).  The selection is the union over knots.  One workgroup
// of 1024 lanes per knot, in two stages.
//
// Bounded stage.  A mode j is kept iff S_j < (1 - eps) T, S_j the sequential
// sum of the powers ranked before it and T the sequential total.  Any sum of
// n non-negative binary64 values, in any order, is within (n - 1) u of the
// exact sum times the exact sum (u = 2^-53), so sums formed in another order
// (here: block reductions and LDS atomics) decide every comparison the same
// way unless they lie within a margin, taken as 8 (M + 4) u T, of the
// threshold.  The workgroup finds the last kept mode by a most-significant-
// digit radix select on the power's bits (non-negative binary64 values order
// as their bit patterns): per level, 8 bits below the candidates' common
// prefix are bucketed with the bucket power sums, and the last bucket whose
// preceding sum is below the threshold holds the last kept mode.  Each choice
// is checked against the margin on both sides; equal powers are ranked by
// index.  Latency bound (one workgroup per knot, a level is two barriers and
// two dependent reductions, about 4 us), so a level that leaves at most 64
// candidates is the last: each of them sums the powers ranked before its own
// (3843 modes, 100 knots: a call 20.6 -> 18.9 us).
//
// Sorted stage, taken only when some comparison falls inside the margin (or
// the total is 0 or not finite, or the plan asks for it): bitonic sort of
// (power, index) held in registers; one lane forms the binary64 partial sums
// in sorted order (values loaded 32 at a time, so only the chain of adds is
// serial) and every threshold decision is taken on exactly those sums.
// ===========================================================================
// No contraction: a power is re re + im im with each product rounded (with
// __dmul_rn, a plain product of another header, the sum was fused, and powers
// that differ in their last bits ranked in another order).
#pragma clang fp contract(off)
__device__ __forceinline__ bool sel_before(double ka, int ia, double kb, int ib) {
    return ka > kb || (ka == kb && ia < ib);
}

constexpr int kSelectThreads = 1024;

// One compare-exchange of the bitonic network from the side of the element at
// position p, whose partner (position p ^ stride) holds (kq, iq).
__device__ __forceinline__ void sel_exchange(double &kv, int &iv, double kq, int iq, int p,
                                             int stride, int size) {
    const bool lower = (p & stride) == 0;
    const int low = lower ? p : (p ^ stride);
    const bool up = (low & size) == 0;             // this run sorts in "before" order
    const bool mine_first = sel_before(kv, iv, kq, iq);
    if (mine_first != (lower == up)) {
        kv = kq;
        iv = iq;
    }
}

// N = 1024 R positions (R = 1, 2 or 4); lane t holds positions t + 1024 r in
// registers.  Partners closer than a wave are exchanged by shuffles, partners
// 1024 or more apart are in the lane's own registers, the rest go through LDS.
__device__ void select_sorted(const double *amp, int M, int N, double one_minus_eps, int *keep,
                              double *sel_lds) {
    double *key = sel_lds;
    int *idx = (int *)(sel_lds + N);
    __shared__ double total;
    __shared__ int below;
    const int tid = threadIdx.x;
    const int R = N / kSelectThreads;
    const size_t k = blockIdx.x;
    double kv[4];
    int iv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int p = tid + kSelectThreads * r;
        if (r < R && p < M) {
            const double re = amp[(k * M + p) * 2], im = amp[(k * M + p) * 2 + 1];
            kv[r] = re * re + im * im;
            iv[r] = p;
        } else {
            kv[r] = -1.0;           // below every power
            iv[r] = INT_MAX;
        }
    }
    for (int size = 2; size <= N; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            if (stride >= kSelectThreads) {
                const int rs = stride / kSelectThreads;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (r < R && (r & rs) == 0) {
                        const int r2 = r | rs;
                        const int p = tid + kSelectThreads * r;
                        const bool up = (p & size) == 0;
                        const bool sw = up ? sel_before(kv[r2], iv[r2], kv[r], iv[r])
                                           : sel_before(kv[r], iv[r], kv[r2], iv[r2]);
                        if (sw) {
                            const double tk = kv[r]; kv[r] = kv[r2]; kv[r2] = tk;
                            const int ti = iv[r]; iv[r] = iv[r2]; iv[r2] = ti;
                        }
                    }
                }
            } else if (stride >= kWave) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (r < R) {
                        key[tid + kSelectThreads * r] = kv[r];
                        idx[tid + kSelectThreads * r] = iv[r];
                    }
                }
                __syncthreads();
                double kq[4];
                int iq[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (r < R) {
                        const int q = (tid + kSelectThreads * r) ^ stride;
                        kq[r] = key[q];
                        iq[r] = idx[q];
                    }
                }
                __syncthreads();                    // reads done before the next writes
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (r < R)
                        sel_exchange(kv[r], iv[r], kq[r], iq[r], tid + kSelectThreads * r,
                                     stride, size);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (r < R) {
                        const double kq = __shfl_xor(kv[r], stride);
                        const int iq = __shfl_xor(iv[r], stride);
                        sel_exchange(kv[r], iv[r], kq, iq, tid + kSelectThreads * r, stride,
                                     size);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (r < R) {
            key[tid + kSelectThreads * r] = kv[r];
            idx[tid + kSelectThreads * r] = iv[r];
        }
    }
    __syncthreads();
    // sequential partial sums: key[j] becomes the sum of the powers before j.
    // One lane walks the sorted powers in blocks of 32 held in its registers,
    // so the serial part is the chain of binary64 adds alone.
    if (tid == 0) {
        constexpr int B = 32;
        double run = 0.0;
        int j = 0;
        for (; j + B <= M; j += B) {
            double v[B];
#pragma unroll
            for (int q = 0; q < B; ++q) v[q] = key[j + q];
#pragma unroll
            for (int q = 0; q < B; ++q) {
                const double before = run;
                run = __dadd_rn(run, v[q]);
                v[q] = before;
            }
#pragma unroll
            for (int q = 0; q < B; ++q) key[j + q] = v[q];
        }
        for (; j < M; ++j) {
            const double before = run;
            run = __dadd_rn(run, key[j]);
            key[j] = before;
        }
        total = run;
        below = 0;
    }
    __syncthreads();
    // kept: the modes whose preceding sum is below (1 - eps) total, a prefix
    // since the sums do not decrease; at least the top mode
    const double thr = __dmul_rn(one_minus_eps, total);
    int local = 0;
    for (int j = tid; j < M; j += kSelectThreads) local += key[j] < thr ? 1 : 0;
    if (local) atomicAdd(&below, local);
    __syncthreads();
    const int cut = below > 0 ? below : 1;
    for (int j = tid; j < cut; j += kSelectThreads) keep[idx[j]] = 1;
}

// Bounded stage of one knot (see above).  Returns false, uniformly over the
// workgroup and before writing anything, when the sorted stage must decide.
// ties: LDS scratch for up to 4096 indices.
__device__ bool select_bounded(const double *amp, int M, double one_minus_eps, int *keep,
                               int *ties) {
    constexpr int NW = kSelectThreads / kWave;
    __shared__ double bsum[256];
    __shared__ int bcnt[256];
    __shared__ double wsum[NW];
    __shared__ unsigned long long wand[NW], wor[NW];
    __shared__ double s_above;
    __shared__ unsigned long long s_pre, s_mask;
    __shared__ int s_state, s_count, s_nties, s_bad;
    constexpr int kFew = 64;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const size_t k = blockIdx.x;
    double pv[4];
    unsigned long long kb[4];
    bool ok[4];
    double loc = 0.0;
    unsigned long long a = ~0ull, o = 0ull;         // AND and OR of the candidates' bits
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int p = tid + kSelectThreads * r;
        ok[r] = p < M;
        pv[r] = 0.0;
        if (ok[r]) {
            const double re = amp[(k * M + p) * 2], im = amp[(k * M + p) * 2 + 1];
            pv[r] = re * re + im * im;
        }
        kb[r] = (unsigned long long)__double_as_longlong(pv[r]);
        loc += pv[r];
        if (ok[r]) {
            a &= kb[r];
            o |= kb[r];
        }
    }
    for (int off = kWave / 2; off > 0; off >>= 1) loc += __shfl_xor(loc, off);
    if (lane == 0) wsum[w] = loc;
    if (tid == 0) {
        s_above = 0.0;
        s_pre = 0ull;
        s_mask = 0ull;
        s_state = 0;
        s_bad = 0;
        s_nties = 0;
    }
    // a, o over the workgroup
    auto common = [&]() {
        for (int off = kWave / 2; off > 0; off >>= 1) {
            a &= (unsigned long long)__shfl_xor((long long)a, off);
            o |= (unsigned long long)__shfl_xor((long long)o, off);
        }
        if (lane == 0) {
            wand[w] = a;
            wor[w] = o;
        }
        if (tid < 256) {
            bsum[tid] = 0.0;
            bcnt[tid] = 0;
        }
        __syncthreads();
        a = ~0ull;
        o = 0ull;
        for (int i = 0; i < NW; ++i) {
            a &= wand[i];
            o |= wor[i];
        }
    };
    common();
    double T = 0.0;
    for (int i = 0; i < NW; ++i) T += wsum[i];      // (every thread, in one order)
    if (!(T > 0.0) || !(T < INFINITY)) return false;
    const double thr = __dmul_rn(one_minus_eps, T);
    const double margin = 8.0 * (double)(M + 4) * 0x1p-53 * T;
    // levels: the candidates are the modes whose masked bits equal s_pre
    for (bool first = true;; first = false) {
        const unsigned long long pre = s_pre, hm = s_mask;
        if (!first) {
            a = ~0ull;
            o = 0ull;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (ok[r] && (kb[r] & hm) == pre) {
                    a &= kb[r];
                    o |= kb[r];
                }
            common();
        }
        const unsigned long long diff = a ^ o;
        if (diff == 0ull) break;                    // the candidates share one power
        const int hb = 63 - __clzll((long long)diff);
        const int sh = hb >= 7 ? hb - 7 : 0;
        const unsigned long long keepm = ~0ull << (hb + 1);   // bits common to all candidates
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (ok[r] && (kb[r] & hm) == pre) {
                const int d = (int)((kb[r] >> sh) & 255ull);
                atomicAdd(&bsum[d], pv[r]);
                atomicAdd(&bcnt[d], 1);
            }
        __syncthreads();
        if (w == 0) {
            // rank order: e = 4 lane + i takes bucket 255 - e (larger powers first)
            double sv[4];
            int cv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sv[i] = bsum[255 - (4 * lane + i)];
                cv[i] = bcnt[255 - (4 * lane + i)];
            }
            double inc = ((sv[0] + sv[1]) + sv[2]) + sv[3];
            for (int off = 1; off < kWave; off <<= 1) {
                const double y = __shfl_up(inc, off);
                if (lane >= off) inc += y;
            }
            double run = __shfl_up(inc, 1);
            run = s_above + (lane == 0 ? 0.0 : run);
            double C[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                C[i] = run;
                run += sv[i];
            }
            // last rank below the threshold, and the next occupied one
            int best = -1, nxt = 0x7fffffff;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned long long m = __ballot(cv[i] > 0 && C[i] < thr);
                if (m) best = max(best, 4 * (63 - __clzll((long long)m)) + i);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned long long m = __ballot(cv[i] > 0 && 4 * lane + i > best);
                if (m) nxt = min(nxt, 4 * (__ffsll((long long)m) - 1) + i);
            }
            bool bad = best < 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = 4 * lane + i;
                if (e == best && !(C[i] < thr - margin)) bad = true;
                if (e == nxt && !(C[i] >= thr + margin)) bad = true;
            }
            bad = __any(bad);
            if (bad) {
                if (lane == 0) s_state = 2;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * lane + i == best) {
                        const unsigned long long d = (unsigned long long)(255 - best);
                        s_pre = (a & keepm) | (d << sh);
                        s_mask = sh > 0 ? (~0ull << sh) : ~0ull;
                        s_above = C[i];
                        s_count = cv[i];
                        s_state = cv[i] == 1 ? 1 : (sh == 0 ? 3 : (cv[i] <= kFew ? 4 : 0));
                    }
            }
        }
        __syncthreads();
        if (s_state != 0) break;
    }
    const int state = s_state;
    if (state == 2) return false;
    const unsigned long long pre = s_pre, hm = s_mask;
    if (state != 1) {
        // at most kFew candidates: each sums the powers ranked before its own; or
        // candidates of one power p: the one ranked q-th by index has q p before it
        const bool few = state == 4;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (ok[r] && (kb[r] & hm) == pre) {
                const int at = atomicAdd(&s_nties, 1);
                ties[at] = tid + kSelectThreads * r;
                if (few) bsum[at] = pv[r];
            }
        __syncthreads();
        const int nt = s_nties;
        const double above = s_above;
        bool bad = false;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (!(ok[r] && (kb[r] & hm) == pre)) continue;
            const int me = tid + kSelectThreads * r;
            double before = above;
            if (few) {
                for (int i = 0; i < nt; ++i)
                    before += sel_before(bsum[i], ties[i], pv[r], me) ? bsum[i] : 0.0;
            } else {
                int q = 0;
                for (int i = 0; i < nt; ++i) q += ties[i] < me ? 1 : 0;
                before = fma((double)q, pv[r], above);
            }
            if (!(before < thr - margin) && !(before >= thr + margin)) bad = true;
            ok[r] = before < thr;                   // from here: kept among the candidates
            kb[r] = pre;
        }
        if (bad) s_bad = 1;
        __syncthreads();
        if (s_bad) return false;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int p = tid + kSelectThreads * r;
            if (p >= M) continue;
            const unsigned long long km =
                (unsigned long long)__double_as_longlong(pv[r]) & hm;
            const bool cand = km == pre;
            if ((!cand && km > pre) || (cand && ok[r])) keep[p] = 1;
        }
        return true;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (ok[r] && (kb[r] & hm) >= pre) keep[tid + kSelectThreads * r] = 1;
    return true;
}

// One workgroup per knot; `sorted` forces the sorted stage.
__global__ __launch_bounds__(kSelectThreads) void select_kernel(const double *amp, int M, int N,
                                                                double one_minus_eps,
                                                                int sorted, int *keep) {
    extern __shared__ double sel_lds[];
    if (!sorted && select_bounded(amp, M, one_minus_eps, keep, (int *)sel_lds)) return;
    __syncthreads();                                // the bounded stage's LDS reads are done
    select_sorted(amp, M, N, one_minus_eps, keep, sel_lds);
}

#pragma clang fp contract(on)

__global__ void zero_u32_kernel(unsigned *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// ===========================================================================
// Launchers.
// ===========================================================================
static inline int round_up8(long long x) { return (int)((x + 7) / 8 * 8); }

// Upload of a request's host tables: `bytes` from pinned, host-coherent memory
// (read by the GPU over the host link) into device memory, by a kernel on the
// compute queue, so a small upload does not wait on a copy engine's signal.
// 16-byte words, then the remaining bytes one per lane.
__global__ __launch_bounds__(256) void upload_kernel(const unsigned char *src, unsigned char *dst,
                                                     long long bytes) {
    const long long n16 = bytes / 16;
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = tid; i < n16; i += stride)
        ((uint4 *)dst)[i] = ((const uint4 *)src)[i];
    if (tid < bytes - n16 * 16) dst[n16 * 16 + tid] = src[n16 * 16 + tid];
}

hipError_t launch_upload(const void *src, void *dst, size_t bytes, hipStream_t stream) {
    if (bytes == 0) return hipSuccess;
    const long long n16 = (long long)(bytes / 16);
    const int blocks = (int)std::max<long long>(1, std::min<long long>((n16 + 255) / 256, 128));
    hipLaunchKernelGGL(upload_kernel, dim3(blocks), dim3(256), 0, stream,
                       (const unsigned char *)src, (unsigned char *)dst, (long long)bytes);
    return hipGetLastError();
}

// Amplitude coefficients in the documented export layout: dst [K-1][M][4][2]
// from the matrix-core requests' internal [K-1][4][2M].
__global__ __launch_bounds__(256) void acoef_export_kernel(const double *src, double *dst,
                                                           long long K1, long long M) {
    const long long n = K1 * M * 8;
    for (long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x; x < n;
         x += (long long)gridDim.x * blockDim.x) {
        const long long c = x & 1, p = (x >> 1) & 3, k = (x >> 3) % M, i = (x >> 3) / M;
        dst[x] = src[(i * 4 + p) * 2 * M + 2 * k + c];
    }
}

hipError_t launch_acoef_export(const double *src, double *dst, int K, int M,
                               hipStream_t stream) {
    const long long n = (long long)(K - 1) * M * 8;
    const int blocks = (int)std::max<long long>(1, std::min<long long>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(acoef_export_kernel, dim3(blocks), dim3(256), 0, stream, src, dst,
                       (long long)(K - 1), (long long)M);
    return hipGetLastError();
}

static inline size_t fit_lds_bytes(int K) {
    // phase workgroups: 9 arrays of K; amplitude workgroups: 5 arrays of K
    size_t n = 9 * (size_t)K;
    if (K <= kFitStageKnots)    // 4 arrays of K, the chunk values, a 2 KB slot per wave
        n = std::max(n, 4 * (size_t)K + 2 * 4 * kWave + 8 + 4 * 4 * kWave);
    return sizeof(double) * n;
}

static void fit_lds_attributes() {
    static std::once_flag once;
    std::call_once(once, [] {
        const int bytes = (int)fit_lds_bytes(kFitStageKnots);
        for (const void *f : {(const void *)fit_kernel<0>, (const void *)fit_kernel<2>,
                              (const void *)fit_kernel<3>, (const void *)fit_batch_kernel<0>,
                              (const void *)fit_batch_kernel<2>, (const void *)fit_batch_kernel<3>})
            hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    });
}

// Rows per lane of the wave sweeps for K knots (0: one lane).
static int fit_rows(int K) { return K <= 2 * kWave ? 2 : K <= kFitStageKnots ? 3 : 0; }

template <int R>
static void launch_fit_rows(const FitJob &job, const double *t_host, hipStream_t stream) {
    FitKnots<R> kt;
    if (R > 0) std::memcpy(kt.t, t_host, sizeof(double) * job.K);
    hipLaunchKernelGGL(fit_kernel<R>, dim3(job.n_ph + job.amp_blocks), dim3(256),
                       fit_lds_bytes(job.K), stream, job, kt);
}

hipError_t launch_fit(const FitJob &job, const double *t_host, hipStream_t stream) {
    fit_lds_attributes();
    switch (fit_rows(job.K)) {
    case 2: launch_fit_rows<2>(job, t_host, stream); break;
    case 3: launch_fit_rows<3>(job, t_host, stream); break;
    default: launch_fit_rows<0>(job, t_host, stream);
    }
    return hipGetLastError();
}

hipError_t launch_fit_batch(const FitJob *jobs_dev, int n_jobs, int max_blocks, int max_K,
                            hipStream_t stream) {
    fit_lds_attributes();
    dim3 grid(kMaxPhases + max_blocks, n_jobs);
    // jobs of up to kFitStageKnots knots stage in LDS whatever max_K is
    const size_t bytes =
        std::max(fit_lds_bytes(max_K), fit_lds_bytes(std::min(max_K, kFitStageKnots)));
    const int R = fit_rows(max_K);
    hipLaunchKernelGGL(R == 2 ? fit_batch_kernel<2> : R == 3 ? fit_batch_kernel<3> : fit_batch_kernel<0>,
                       grid, dim3(256), bytes, stream, jobs_dev);
    return hipGetLastError();
}

hipError_t launch_prepare(const PrepJob &job, bool fp32, hipStream_t stream) {
    const dim3 grid(1 + job.fold_blocks);
    if (fp32)
        hipLaunchKernelGGL(prepare_kernel<float>, grid, dim3(256), 0, stream, job);
    else
        hipLaunchKernelGGL(prepare_kernel<double>, grid, dim3(256), 0, stream, job);
    return hipGetLastError();
}

hipError_t launch_prepare_batch(const PrepJob *jobs_dev, int n_jobs, int max_fold_blocks,
                                bool fp32, hipStream_t stream) {
    const dim3 grid(1 + max_fold_blocks, n_jobs);
    if (fp32)
        hipLaunchKernelGGL(prepare_batch_kernel<float>, grid, dim3(256), 0, stream, jobs_dev);
    else
        hipLaunchKernelGGL(prepare_batch_kernel<double>, grid, dim3(256), 0, stream, jobs_dev);
    return hipGetLastError();
}

static inline size_t sum_lds_bytes() { return sizeof(float) * 8 * (size_t)kChunkTerms; }

int sum_resident_workgroups(int n_ph) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    const void *fn = n_ph == 3 ? (const void *)sum_wg_kernel<float, true, false, 3, false>
                               : (const void *)sum_wg_kernel<float, true, false, 2, false>;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 256, sum_lds_bytes()) !=
        hipSuccess)
        return 0;
    return cus * per_cu;
}

hipError_t launch_sum(const SumJob &job, int slots, bool fp32, hipStream_t stream) {
    const long long parts = job.parts;
    const bool kerr = job.n_ph == 3;
    if (fp32) {
        const dim3 grid((unsigned)(parts * slots));
        if (kerr)
            hipLaunchKernelGGL((sum_wg_kernel<float, true, false, 3, false>), grid, dim3(256),
                               sum_lds_bytes(), stream, job, slots);
        else
            hipLaunchKernelGGL((sum_wg_kernel<float, true, false, 2, false>), grid, dim3(256),
                               sum_lds_bytes(), stream, job, slots);
    } else {
        const int waves_per_block = 256 / kWave;
        const long long blocks = (slots + waves_per_block - 1) / waves_per_block;
        const dim3 grid((unsigned)(parts * blocks));
        if (kerr)
            hipLaunchKernelGGL((sum_kernel<double, false, true, 3, false>), grid, dim3(256), 0,
                               stream, job, slots);
        else
            hipLaunchKernelGGL((sum_kernel<double, false, true, 2, false>), grid, dim3(256), 0,
                               stream, job, slots);
    }
    return hipGetLastError();
}

// Adds count partials in a fixed order (strided per lane, four loads in
// flight, then a tree in LDS) and writes out2 = factor * (x sum, y sum).
constexpr int kReduceThreads = 1024;
__global__ __launch_bounds__(kReduceThreads) void reduce_partials_kernel(const double2 *partial,
                                                                         long long count,
                                                                         double factor,
                                                                         double *out2) {
    __shared__ double2 red[kReduceThreads];
    double2 v = make_double2(0.0, 0.0);
    const long long step = blockDim.x;
    long long i = threadIdx.x;
    for (; i + 3 * step < count; i += 4 * step) {
        const double2 a = partial[i], b = partial[i + step], c = partial[i + 2 * step],
                      d = partial[i + 3 * step];
        v.x = v.x + a.x; v.y = v.y + a.y;
        v.x = v.x + b.x; v.y = v.y + b.y;
        v.x = v.x + c.x; v.y = v.y + c.y;
        v.x = v.x + d.x; v.y = v.y + d.y;
    }
    for (; i < count; i += step) {
        v.x = v.x + partial[i].x;
        v.y = v.y + partial[i].y;
    }
    red[threadIdx.x] = v;
    __syncthreads();
    for (int off = blockDim.x / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            red[threadIdx.x].x = red[threadIdx.x].x + red[threadIdx.x + off].x;
            red[threadIdx.x].y = red[threadIdx.x].y + red[threadIdx.x + off].y;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out2[0] = factor * red[0].x;
        out2[1] = factor * red[0].y;
    }
}

// Partial sums of the allocation-free inner product: a file-scope device
// array, one copy per GPU, held until the process ends.  Host code never
// passes `scratch` itself to a kernel (in host code the name is a host-side
// stand-in); it uses the device address hipGetSymbolAddress returns, looked up
// once per device by noalloc_scratch().
static __device__ __align__(256) double2 scratch[kNoAllocSlots];

hipError_t noalloc_scratch(int device, double2 **out) {
    static std::mutex mu;
    static double2 *addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(mu);
    if (!addr[device]) {
        int cur = 0;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;   // caller makes `device` current
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = (double2 *)p;
    }
    *out = addr[device];
    return hipSuccess;
}

long long inner_slots(int parts, int slots, bool fp32) {
    if (fp32) return (long long)parts * slots;
    const int waves_per_block = 256 / kWave;
    return (long long)parts * ((slots + waves_per_block - 1) / waves_per_block) * waves_per_block;
}

hipError_t launch_sum_inner(const SumJob &job, int slots, bool fp32, double two_dt,
                            double *out2, hipStream_t stream) {
    const long long parts = job.parts;
    const bool kerr = job.n_ph == 3;
    if (fp32) {
        const dim3 grid((unsigned)(parts * slots));
        if (kerr)
            hipLaunchKernelGGL((sum_wg_kernel<float, true, false, 3, true>), grid, dim3(256),
                               sum_lds_bytes(), stream, job, slots);
        else
            hipLaunchKernelGGL((sum_wg_kernel<float, true, false, 2, true>), grid, dim3(256),
                               sum_lds_bytes(), stream, job, slots);
    } else {
        const int waves_per_block = 256 / kWave;
        const long long blocks = (slots + waves_per_block - 1) / waves_per_block;
        const dim3 grid((unsigned)(parts * blocks));
        if (kerr)
            hipLaunchKernelGGL((sum_kernel<double, false, true, 3, true>), grid, dim3(256), 0,
                               stream, job, slots);
        else
            hipLaunchKernelGGL((sum_kernel<double, false, true, 2, true>), grid, dim3(256), 0,
                               stream, job, slots);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(kReduceThreads), 0, stream,
                       job.partial, inner_slots(job.parts, slots, fp32), two_dt, out2);
    return hipGetLastError();
}

// Workgroup 0 and the (interval, row tile) workgroups of a K-knot request,
// the intervals in groups of 8 (fold_pack_body).
static int fold_pack_blocks(int K) { return 1 + 8 * kMfMT * ((K - 1 + 7) / 8); }

hipError_t launch_fold_pack(const PrepJob &job, hipStream_t stream) {
    hipLaunchKernelGGL(fold_pack_kernel, dim3(fold_pack_blocks(job.K)), dim3(kFoldPackThreads), 0,
                       stream, job);
    return hipGetLastError();
}

hipError_t launch_fold_pack_batch(const PrepJob *jobs_dev, int n_jobs, int max_K,
                                  hipStream_t stream) {
    hipLaunchKernelGGL(fold_pack_batch_kernel, dim3(fold_pack_blocks(max_K), n_jobs),
                       dim3(kFoldPackThreads), 0, stream, jobs_dev);
    return hipGetLastError();
}

static constexpr size_t mf_lds_bytes() {
    return mf_table_bytes(kMfMT, kMfT) + kMfWaves * sizeof(MfSampleArea);
}

static constexpr size_t mf_terms_lds_bytes(int MT, int T, bool kerr) {
    return mf_table_bytes(MT, T) + kMfWaves * sizeof(MfSampleArea) +
           (kerr ? sizeof(float2) * kMfWaves * kMfKerrRounds * kMfSPW : 0);
}

static constexpr size_t mf_f64_lds_bytes(int MT, int T, int ns, bool kerr) {
    return mf64_base_bytes(MT, ns) + mf64_rest_bytes(MT, T) +
           (kerr ? sizeof(double2) * kMfWaves * kMfKerrRounds64 * kMfSPW : 0);
}


// One workgroup per compute unit (the operand table takes most of the LDS).
int mfma_workgroups() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    static std::once_flag once;
    std::call_once(once, [] {
        const void *fn[] = {(const void *)sum_mfma_kernel<false, true>,
                            (const void *)sum_mfma_kernel<false, false>,
                            (const void *)sum_mfma_kernel<true, true>,
                            (const void *)sum_mfma_kernel<true, false>,
                            (const void *)sum_mfma_batch_kernel<true>,
                            (const void *)sum_mfma_batch_kernel<false>};
        for (const void *f : fn)
            hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)mf_lds_bytes());
        for (int mt = 1; mt <= kMfMT; ++mt)
            for (int t = 1; t <= kMfT; ++t)
                mf_with_shape(mt, t, [](auto MT, auto T) {
                    constexpr int mtv = decltype(MT)::value, tv = decltype(T)::value;
                    auto set = [](const void *f, bool kerr) {
                        hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)mf_terms_lds_bytes(mtv, tv, kerr));
                    };
                    set((const void *)sum_mfma_terms_kernel<false, mtv, tv, false>, false);
                    set((const void *)sum_mfma_terms_kernel<true, mtv, tv, false>, false);
                    set((const void *)sum_mfma_terms_kernel<false, mtv, tv, true>, true);
                    set((const void *)sum_mfma_terms_kernel<true, mtv, tv, true>, true);
                    auto set64 = [](const void *f, bool kerr) {
                        hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)mf_f64_lds_bytes(mtv, tv, 8 * tv, kerr));
                    };
                    set64((const void *)sum_mfma_f64_kernel<false, mtv, tv, false>, false);
                    set64((const void *)sum_mfma_f64_kernel<true, mtv, tv, false>, false);
                    set64((const void *)sum_mfma_f64_kernel<false, mtv, tv, true>, true);
                    set64((const void *)sum_mfma_f64_kernel<true, mtv, tv, true>, true);
                });
        hipFuncSetAttribute((const void *)sum_mfma_terms_batch_kernel<false>,
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)mf_terms_lds_bytes(kMfMT, kMfT, false));
        hipFuncSetAttribute((const void *)sum_mfma_terms_batch_kernel<true>,
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)mf_f64_lds_bytes(kMfMT, kMfT, 8 * kMfT, false));
    });
    return cus;
}

// One request summed from its fold table.
template <bool INNER>
static void launch_terms(const SumJob &job, int n_wg, hipStream_t stream) {
    const dim3 grid(n_wg), block(64 * kMfWaves);
    const bool kerr = job.n_ph == 3;
    mf_with_shape(job.mf_terms / 10, job.mf_terms % 10, [&](auto MT, auto T) {
        constexpr int mt = decltype(MT)::value, t = decltype(T)::value;
        if (job.mf_f64) {
            const size_t lds = mf_f64_lds_bytes(mt, t, job.mf_ns, kerr);
            if (kerr)
                hipLaunchKernelGGL((sum_mfma_f64_kernel<INNER, mt, t, true>), grid, block, lds, stream, job);
            else
                hipLaunchKernelGGL((sum_mfma_f64_kernel<INNER, mt, t, false>), grid, block, lds, stream, job);
        } else {
            const size_t lds = mf_terms_lds_bytes(mt, t, kerr);
            if (kerr)
                hipLaunchKernelGGL((sum_mfma_terms_kernel<INNER, mt, t, true>), grid, block, lds, stream, job);
            else
                hipLaunchKernelGGL((sum_mfma_terms_kernel<INNER, mt, t, false>), grid, block, lds, stream, job);
        }
    });
}

hipError_t launch_sum_mfma(const SumJob &job, int n_wg, hipStream_t stream) {
    if (job.mf_terms)
        launch_terms<false>(job, n_wg, stream);
    else if (job.mf_consec)
        hipLaunchKernelGGL((sum_mfma_kernel<false, true>), dim3(n_wg), dim3(64 * kMfWaves),
                           mf_lds_bytes(), stream, job);
    else
        hipLaunchKernelGGL((sum_mfma_kernel<false, false>), dim3(n_wg), dim3(64 * kMfWaves),
                           mf_lds_bytes(), stream, job);
    return hipGetLastError();
}

hipError_t launch_sum_mfma_inner(const SumJob &job, int n_wg, double two_dt, double *out2,
                                 hipStream_t stream) {
    if (job.mf_terms)
        launch_terms<true>(job, n_wg, stream);
    else if (job.mf_consec)
        hipLaunchKernelGGL((sum_mfma_kernel<true, true>), dim3(n_wg), dim3(64 * kMfWaves),
                           mf_lds_bytes(), stream, job);
    else
        hipLaunchKernelGGL((sum_mfma_kernel<true, false>), dim3(n_wg), dim3(64 * kMfWaves),
                           mf_lds_bytes(), stream, job);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(kReduceThreads), 0, stream,
                       job.partial, (long long)n_wg, two_dt, out2);
    return hipGetLastError();
}

hipError_t launch_sum_mfma_batch(const SumJob *jobs_dev, int n_jobs, long long total, bool consec,
                                 int n_wg, hipStream_t stream) {
    if (consec)
        hipLaunchKernelGGL(sum_mfma_batch_kernel<true>, dim3(n_wg), dim3(64 * kMfWaves),
                           mf_lds_bytes(), stream, jobs_dev, n_jobs, total);
    else
        hipLaunchKernelGGL(sum_mfma_batch_kernel<false>, dim3(n_wg), dim3(64 * kMfWaves),
                           mf_lds_bytes(), stream, jobs_dev, n_jobs, total);
    return hipGetLastError();
}

hipError_t launch_sum_mfma_terms_batch(const SumJob *jobs_dev, int n_jobs, long long total,
                                       bool f64, int n_wg, hipStream_t stream) {
    const dim3 grid(n_wg), block(64 * kMfWaves);
    if (f64)
        hipLaunchKernelGGL(sum_mfma_terms_batch_kernel<true>, grid, block,
                           mf_f64_lds_bytes(kMfMT, kMfT, 8 * kMfT, false), stream, jobs_dev, n_jobs,
                           total);
    else
        hipLaunchKernelGGL(sum_mfma_terms_batch_kernel<false>, grid, block,
                           mf_terms_lds_bytes(kMfMT, kMfT, false), stream, jobs_dev, n_jobs, total);
    return hipGetLastError();
}

hipError_t launch_sum_batch(const SumJob *jobs_dev, int n_jobs, int total_slots, bool fp32,
                            bool persistent, unsigned *counter_dev, hipStream_t stream) {
    const int waves_per_block = 256 / kWave;
    if (!persistent) {
        if (fp32)
            hipLaunchKernelGGL((sum_wg_batch_kernel<float, true, false>),
                               dim3(round_up8(total_slots)), dim3(256), sum_lds_bytes(), stream,
                               jobs_dev, n_jobs, total_slots);
        else
            hipLaunchKernelGGL((sum_batch_kernel<double, false, true>),
                               dim3(round_up8((total_slots + waves_per_block - 1) / waves_per_block)),
                               dim3(256), 0, stream, jobs_dev, n_jobs, total_slots);
        return hipGetLastError();
    }
    // one resident grid: 256 CUs x 4 workgroups of 4 waves
    hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(64), 0, stream, counter_dev, 1);
    if (fp32) {
        int blocks = 256 * 4;
        if (blocks > total_slots) blocks = total_slots > 0 ? total_slots : 1;
        hipLaunchKernelGGL((sum_wg_persistent_kernel<float, true, false>),
                           dim3(blocks), dim3(256), sum_lds_bytes(), stream, jobs_dev, n_jobs,
                           total_slots, counter_dev);
    } else {
        int blocks = 256 * 8;
        const int needed = (total_slots + waves_per_block - 1) / waves_per_block;
        if (blocks > needed) blocks = needed > 0 ? needed : 1;
        hipLaunchKernelGGL((sum_persistent_kernel<double, false, true>),
                           dim3(blocks), dim3(256), 0, stream, jobs_dev, n_jobs, total_slots,
                           counter_dev);
    }
    return hipGetLastError();
}

hipError_t launch_select(const double *amp, int K, int M, double eps, bool sorted, int *keep,
                         hipStream_t stream) {
    int N = kSelectThreads;                 // 1024, 2048 or 4096 sort positions
    while (N < M) N <<= 1;
    hipLaunchKernelGGL(zero_u32_kernel, dim3((M + 255) / 256), dim3(256), 0, stream,
                       (unsigned *)keep, M);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds = (sizeof(double) + sizeof(int)) * (size_t)N;
    hipLaunchKernelGGL(select_kernel, dim3(K), dim3(kSelectThreads), lds, stream, amp, M, N,
                       1.0 - eps, sorted ? 1 : 0, keep);
    return hipGetLastError();
}

hipError_t launch_zero_u32(unsigned *p, int n, hipStream_t stream) {
    hipLaunchKernelGGL(zero_u32_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, p, n);
    return hipGetLastError();
}

}  // namespace few
