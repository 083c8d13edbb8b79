// L D L^T of one 64 x 64 complex symmetric block by a workgroup of four waves,
// with the inverse X = L^-1 of its unit lower triangle, and products with X.
// Used by the blocked factorisation above 64 loops (diagonal blocks) and by the
// solves of 33 to 64 loops with few systems (the whole matrix).
#pragma once
#include "internal.h"

namespace cosim {

namespace {

__device__ inline double2 zmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// acc - l * u
__device__ inline double2 zfms(double2 acc, double2 l, double2 u) {
    return make_double2(fma(-l.x, u.x, fma(l.y, u.y, acc.x)), fma(-l.x, u.y, fma(-l.y, u.x, acc.y)));
}
// acc + l * u
__device__ inline double2 zfma(double2 acc, double2 l, double2 u) {
    return make_double2(fma(l.x, u.x, fma(-l.y, u.y, acc.x)), fma(l.x, u.y, fma(l.y, u.x, acc.y)));
}
__device__ inline double2 zinv(double2 a) {
    const double d = 1.0 / (a.x * a.x + a.y * a.y);
    return make_double2(a.x * d, -a.y * d);
}

// Factor storage: complex128 (FP64 path) or complex64 (FP32 factor of the
// refined path); arithmetic outside the matrix cores is FP64 either way.
__device__ inline double2 ld2(double2 v) { return v; }
__device__ inline double2 ld2(float2 v) { return make_double2((double)v.x, (double)v.y); }
template <typename T2>
__device__ inline T2 st2(double2 v);
template <>
__device__ inline double2 st2<double2>(double2 v) {
    return v;
}
template <>
__device__ inline float2 st2<float2>(double2 v) {
    return make_float2((float)v.x, (float)v.y);
}
template <typename T2>
struct Scal;
template <>
struct Scal<double2> {
    typedef double type;
};
template <>
struct Scal<float2> {
    typedef float type;
};

// One 16x16x4 matrix-core step on FP64 or FP32 operands.  Operand lanes are
// laid out alike (A: row l % 16, k = l / 16; B: k = l / 16, column l % 16);
// accumulator element m of lane group g = l / 16 sits in row g + 4m (FP64)
// or 4g + m (FP32), column l % 16.
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ inline f64x4 mfma4(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <typename T>
struct Acc4;
template <>
struct Acc4<double> {
    typedef f64x4 type;
};
template <>
struct Acc4<float> {
    typedef f32x4 type;
};
template <typename T>
__device__ inline int acc_row(int g, int m) {
    return sizeof(T) == 8 ? g + 4 * m : 4 * g + m;
}

// 1/a of a pivot that is checked afterwards (block_min_pivot): hardware
// reciprocal and two Newton steps (error at the rounding of the result, no
// division sequence).
__device__ inline double2 zinv_nr(double2 a) {
    const double q = fma(a.x, a.x, a.y * a.y);
    double r = __builtin_amdgcn_rcp(q);
    r = fma(r, fma(-q, r, 1.0), r);
    r = fma(r, fma(-q, r, 1.0), r);
    return make_double2(a.x * r, -a.y * r);
}

// A sub-panel of 16 columns, and LDS of one block: two of them, the next one
// being factored while products with the last one are still running.
struct SubPanel {
    double2 sp[64][17];  // the columns (rows from their own block on)
    double2 sx[16][17];  // inverse of their unit lower triangle
    double2 sdi[16];     // 1/pivots
};
struct BlockLds {
    SubPanel sub[2];
    double2 st[64];  // right-hand side
    double2 sz[64];  // diagonal of the block of Z
    // pivot k, until the block of a later system is put here
    __device__ double2 pivot(int k) const { return sub[(k >> 4) & 1].sp[k][k & 15]; }
};

// L D L^T of the 16 x 16 symmetric block in rows p0 .. p0 + 15 of sp by one
// wave, and X = L^-1.  Lane l holds columns 4 (l / 16) + u, u < 4, of row
// l % 16, the whole symmetric block.  Step c subtracts l_r = a_rc / d_c times
// row c from the rows below it; a column that has been eliminated holds the
// matching column of X from then on (it starts as e_c), so each step costs
// four complex multiply-adds per lane, with row c reaching the lanes as 64-bit
// DPP broadcasts inside the 16-lane rows and column c through one exchange.  A
// serial chain of 16 steps, straight-line code: the lanes that hold column c
// store it as it stands at its own step (rows above c unused), the others
// store to their own places in sx, which the inverse overwrites at the end, so
// that no store needs a branch.
template <int C>
__device__ __forceinline__ double row_bcast(double x) {
    // DPP row_newbcast: lane C of each row of 16
    const long v = __double_as_longlong(x);
    return __longlong_as_double(__builtin_amdgcn_mov_dpp(v, 0x150 + C, 0xF, 0xF, true));
}
__device__ inline double lane_value(double x, int src) {  // src uniform over the wave
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), src),
                            __builtin_amdgcn_readlane(__double2loint(x), src));
}
template <int C>
__device__ __forceinline__ void ldl16_step(SubPanel &m, int p0, double2 (&a)[4], int r, int q) {
    constexpr int Q = C >> 2, U = C & 3;
    const double2 d = make_double2(lane_value(a[U].x, 16 * Q + C), lane_value(a[U].y, 16 * Q + C));
    const double2 col = make_double2(__shfl(a[U].x, 16 * Q + r), __shfl(a[U].y, 16 * Q + r));
    double2 *dst = q == Q ? &m.sp[p0 + r][4 * Q] : &m.sx[r][4 * q];
    dst[U] = a[U];
    const double2 inv = zinv_nr(d);
    const double2 l = r > C ? zmul(col, inv) : make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 1; k <= 4; ++k) {  // the next pivot's column first, column c last
        const int u = (U + k) & 3;
        const double2 row = make_double2(row_bcast<C>(a[u].x), row_bcast<C>(a[u].y));
        a[u] = zfms(a[u], l, row);
        if (u == U) {
            a[u].x = q == Q ? (r == C ? 1.0 : -l.x) : a[u].x;
            a[u].y = q == Q ? -l.y : a[u].y;
        }
    }
    if constexpr (C + 1 < 16) ldl16_step<C + 1>(m, p0, a, r, q);
}
__device__ __forceinline__ void ldl16(SubPanel &m, int p0, int lane) {
    const int r = lane & 15, q = lane >> 4;
    double2 a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = m.sp[p0 + r][4 * q + u];
    ldl16_step<0>(m, p0, a, r, q);
#pragma unroll
    for (int u = 0; u < 4; ++u) m.sx[r][4 * q + u] = a[u];
    if (lane < 16) m.sdi[lane] = zinv_nr(m.sp[p0 + lane][lane]);
}

// The 16-column blocks of a 64 x 64 diagonal block that wave w holds as
// (row block, column block) accumulators; every pair below or on the diagonal
// appears once, wave 1's three in transposed form, so that each wave has at
// most three products and two distinct column blocks.
__device__ inline int diag_rb(int w, int q) { return w == 3 ? 2 + q : (w == 2 ? 1 + q : q); }
__device__ inline int diag_cb(int w, int q) { return w == 3 ? 2 + q : (w == 2 ? 1 : (w == 1 ? 3 : 0)); }

// L D L^T and X = L^-1 of the block held as accumulators (diag_rb, diag_cb),
// in 16-column sub-panels p:
//   1. the waves put their accumulators of block column p into LDS;
//   2. wave 3 factors the 16 x 16 block (ldl16), while the others, a block
//      column j of the inverse each, turn the last sub-panel's X_pj = X_pp Y_pj
//      into the rows below, Y_rj -= L_rp X_pj (accumulators in the layout of
//      the B operand of both products), and store its results;
//   3. V_rp = A_rp X_pp^T, one row block per wave;
//   4. A_rc -= V_rp D^-1 V_cp^T on the accumulators still to come.
// Everything but the pivots' chain runs on FP64 matrix cores, also for
// complex64 storage.  Bounded by the chain of 64 pivots (2.4 us per 16, issue
// and latency of one wave; 4.2 with two 32-bit DPP moves per value, selects
// and the pivots' check inside the chain) and 12 barriers: 8 diagonal
// blocks with their input checks take 27.8 us (30.5 with steps 1 to 4 and the
// inverse one after the other, 54 eliminated in LDS with 80 barriers).
// X receives X^T ([64][64], the lower triangle of blocks of X), A with ROWS the
// rows D L^T of the upper triangle (row stride NP), D the 1/pivots; the pivots
// stay on the diagonal of each sub-panel of sp.
template <typename T2, bool ROWS>
__device__ __forceinline__ void ldl_block(BlockLds &m, f64x4 (&Cr)[3], f64x4 (&Ci)[3], T2 *__restrict__ X,
                                          T2 *__restrict__ A, int NP, double2 *__restrict__ D) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    f64x4 Yr[3], Yi[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) Yr[q] = Yi[q] = f64x4{0, 0, 0, 0};
    const int nq = wv < 2 ? 3 : 2;
    const int yj = wv == 0 ? 0 : (wv == 2 ? 1 : (wv == 1 ? 2 : 3));  // block column of the inverse
    // the accumulators of block column p -> its sub-panel
    auto put = [&](int p) {
        SubPanel &u = m.sub[p & 1];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (q >= nq) continue;
            const int rb = diag_rb(wv, q), cb = diag_cb(wv, q);
            if (min(rb, cb) != p) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double2 v = make_double2(Cr[q][e], Ci[q][e]);
                if (rb >= cb) u.sp[16 * rb + g + 4 * e][r16] = v;
                else u.sp[16 * cb + r16][g + 4 * e] = v;
            }
        }
    };
    // X_pj = X_pp Y_pj and the rows below of the inverse, Y_rj -= L_rp X_pj, for
    // the wave's block column j; D^-1 and the rows of U, by the first nw waves
    auto finish = [&](int p, int nw) {
        const SubPanel &u = m.sub[p & 1];
        if (yj <= p) {
            f64x4 xr = f64x4{0, 0, 0, 0}, xi = xr;
            if (yj == p) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double2 v = u.sx[g + 4 * e][r16];
                    xr[e] = v.x;
                    xi[e] = v.y;
                }
            } else {
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    if (t + 1 != p) continue;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double2 a = u.sx[r16][4 * e + g];
                        xr = mfma4(a.x, Yr[t][e], xr);
                        xi = mfma4(a.x, Yi[t][e], xi);
                        xr = mfma4(a.y, -Yi[t][e], xr);
                        xi = mfma4(a.y, Yr[t][e], xi);
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < 3; ++t) {  // row block t + 1
                if (t + 1 <= p) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double2 a = zmul(u.sp[16 * (t + 1) + r16][4 * e + g], u.sdi[4 * e + g]);
                    Yr[t] = mfma4(a.x, -xr[e], Yr[t]);
                    Yi[t] = mfma4(a.x, -xi[e], Yi[t]);
                    Yr[t] = mfma4(a.y, xi[e], Yr[t]);
                    Yi[t] = mfma4(a.y, -xr[e], Yi[t]);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                X[(16 * yj + r16) * 64 + 16 * p + g + 4 * e] = st2<T2>(make_double2(xr[e], xi[e]));
        }
        if (tid < 16) D[16 * p + tid] = u.sdi[tid];
        for (int c = tid >> 4; ROWS && c < 16; c += 4 * nw)
            for (int rr = 16 * p + r16; rr < 64; rr += 16) {
                if (rr < 16 * p + c) continue;
                A[(size_t)(16 * p + c) * NP + rr] = st2<T2>(u.sp[rr][c]);
            }
    };
    put(0);
    __syncthreads();
    for (int p = 0; p < 4; ++p) {
        SubPanel &u = m.sub[p & 1];
        if (wv == 3) ldl16(u, 16 * p, lane);
        else if (p > 0) finish(p - 1, 3);
        __syncthreads();
        if (p == 3) break;
        if (wv > p) {  // V of row block wv
            f64x4 vr = f64x4{0, 0, 0, 0}, vi = vr;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double2 a = u.sp[16 * wv + r16][4 * e + g], b = u.sx[r16][4 * e + g];
                vr = mfma4(a.x, b.x, vr);
                vi = mfma4(a.x, b.y, vi);
                vr = mfma4(a.y, -b.y, vr);
                vi = mfma4(a.y, b.x, vi);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) u.sp[16 * wv + g + 4 * e][r16] = make_double2(vr[e], vi[e]);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (q >= nq) continue;
            const int rb = diag_rb(wv, q), cb = diag_cb(wv, q);
            if (min(rb, cb) <= p) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double2 a = u.sp[16 * rb + r16][4 * e + g];
                const double2 b = zmul(u.sp[16 * cb + r16][4 * e + g], u.sdi[4 * e + g]);
                Cr[q] = mfma4(a.x, -b.x, Cr[q]);
                Ci[q] = mfma4(a.x, -b.y, Ci[q]);
                Cr[q] = mfma4(a.y, b.y, Cr[q]);
                Ci[q] = mfma4(a.y, -b.x, Ci[q]);
            }
        }
        put(p + 1);
        __syncthreads();
    }
    finish(3, 4);
    __syncthreads();
}

// Smallest |re| + |im| of the first n pivots, 0 if one is NaN or outside the
// range in which zinv_nr holds (its square has to be a normal number); one wave.
__device__ __forceinline__ double block_min_pivot(const BlockLds &m, int lane, int n) {
    const double2 d = m.pivot(lane);
    double v = fabs(d.x) + fabs(d.y);
    v = v > 1e-150 && v < 1e150 ? v : 0.0;
    v = lane < n ? v : __builtin_inf();
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmin(v, __shfl_xor(v, off));
    return v;
}

// X v of the block for a vector in LDS, from X^T as ldl_block leaves it; thread
// k < 64 returns entry k.  red: 256 entries of LDS.  Synchronises the
// workgroup once.
template <typename T2>
__device__ __forceinline__ double2 block_x_times(const T2 *X, const double2 *v, double2 *red, int tid) {
    const int rr = tid & 63, part = tid >> 6;
    double2 acc = make_double2(0.0, 0.0);
    if (part <= (rr >> 4))
        for (int c = 16 * part; c < 16 * part + 16; ++c) acc = zfma(acc, ld2(X[c * 64 + rr]), v[c]);
    red[part * 64 + rr] = acc;
    __syncthreads();
    double2 y = make_double2(0.0, 0.0);
    if (tid < 64) {
        y = red[tid];
        for (int e = 1; e < 4; ++e) {
            y.x += red[64 * e + tid].x;
            y.y += red[64 * e + tid].y;
        }
    }
    return y;
}

}  // namespace

}  // namespace cosim
