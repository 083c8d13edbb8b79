// S-parameter cosimulation pipeline (Sec. III, Eq. 2-10; Sec. III-A):
// exports S0 and per-port fields of an n0-port structure, a connecting network
// S_C = S_C,const + S_C,var with n1 external ports, per (configuration,
// frequency) system s = b F + f:
//   A = I - S_C11 S0,  x = A^-1 S_C12 exc  (Eq. 6),  B_comb = fields x  (Eq. 7),
// the loss of Eq. 1 on one component, and its gradient with respect to the
// variable entries through A^H lam = fields^H w (Eq. 8-10).
//
// Kernels:
//   k_sp_prep   per frequency: K = I - S_C11,const S0 and r0 = S_C12,const exc
//               (the constant parts; the variable entries are applied per
//               system) and S0, both transposed;
//   k_sp_lu     one wave per system: A = K minus the variable rows of S_C11 S0,
//               right-hand side r0 plus the variable entries of S_C12 exc, LU with
//               partial pivoting (largest |re| + |im|, ties to the lower row)
//               applied to the right-hand side as it goes, back substitution;
//               the factor is recorded;
//   k_sp_adjoint  one wave per system: the right-hand side from the
//               contraction's partial sums, A^H lam = r with the recorded
//               factor, and the gradient of every variable entry;
//   k_sp_fused  FP64: B_comb = fields x, the loss epilogue and fields^H w in one
//               pass over the rows of the loss component, on matrix cores;
//   rocBLAS complex GEMMs (per frequency, strided over frequencies, in P-chunks)
//               with k_sp_epilogue between them for FP32, and for the
//               materialised B_comb;
//   k_sp_reduce    fixed-order loss sums;
//   k_sp_rc, k_sp_rc_backward  the RC preprocessing of Eq. 2-3 and its chain rule.
#include <rocblas/rocblas.h>

#include <algorithm>
#include <type_traits>

#include "epilogue.h"
#include "internal.h"

namespace cosim {

namespace {

__device__ inline double2 zmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline double2 zmulc(double2 a, double2 b) {  // a conj(b)
    return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ inline double2 zfms(double2 acc, double2 l, double2 u) {  // acc - l u
    return make_double2(fma(-l.x, u.x, fma(l.y, u.y, acc.x)), fma(-l.x, u.y, fma(-l.y, u.x, acc.y)));
}
__device__ inline double2 zinv(double2 a) {
    const double d = 1.0 / (a.x * a.x + a.y * a.y);
    return make_double2(a.x * d, -a.y * d);
}

template <int CTRL>
__device__ inline int dpp_i(int x) {
    return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
}
// The lane with the largest m over the wave (m = -1, or >= 0 and no NaN), ties to
// the lower lane: the bits of such floats order like integers, so that the
// largest is a DPP maximum inside each row of 16 lanes and a scalar one of the
// four rows, and its lane the first set bit of a comparison.
__device__ inline int wave_amax(float m) {
    const int own = __float_as_int(m);
    int b = own;
    b = max(b, dpp_i<0xB1>(b));   // quad_perm [1,0,3,2]
    b = max(b, dpp_i<0x4E>(b));   // quad_perm [2,3,0,1]
    b = max(b, dpp_i<0x141>(b));  // row_half_mirror
    b = max(b, dpp_i<0x140>(b));  // row_mirror
    const int top = max(max(__builtin_amdgcn_readlane(b, 0), __builtin_amdgcn_readlane(b, 16)),
                        max(__builtin_amdgcn_readlane(b, 32), __builtin_amdgcn_readlane(b, 48)));
    return (int)__builtin_ctzll(__ballot(own == top));
}
__device__ inline double rl(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}
__device__ inline double2 rl2(double2 v, int src) { return make_double2(rl(v.x, src), rl(v.y, src)); }

// K[f] = I - S11c[f] S0[f] and S0[f], both stored transposed, and r0[f] =
// S12c[f] exc; grid (n0, F), 64 threads.
__global__ __launch_bounds__(64) void k_sp_prep(int n0, int n1, int F, const double2 *__restrict__ S0,
                                                const double2 *__restrict__ scc,
                                                const double2 *__restrict__ exc,
                                                double2 *__restrict__ KT, double2 *__restrict__ S0T,
                                                double2 *__restrict__ r0) {
    const int i = blockIdx.x, f = blockIdx.y, lane = threadIdx.x;
    const int N = n0 + n1;
    const double2 *S0f = S0 + (size_t)f * n0 * n0;
    const double2 *Sc = scc ? scc + (size_t)f * N * N + (size_t)i * N : nullptr;
    for (int j = lane; j < n0; j += 64) {
        double2 acc = make_double2(0.0, 0.0);
        if (Sc)
            for (int k = 0; k < n0; ++k) {
                const double2 a = Sc[k], b = S0f[(size_t)k * n0 + j];
                acc.x = fma(a.x, b.x, fma(-a.y, b.y, acc.x));
                acc.y = fma(a.x, b.y, fma(a.y, b.x, acc.y));
            }
        KT[((size_t)f * n0 + j) * n0 + i] = make_double2((i == j ? 1.0 : 0.0) - acc.x, -acc.y);
        S0T[((size_t)f * n0 + j) * n0 + i] = S0f[(size_t)i * n0 + j];
    }
    if (lane == 0) {
        double2 acc = make_double2(0.0, 0.0);
        if (Sc)
            for (int j = 0; j < n1; ++j) {
                const double2 a = Sc[n0 + j], b = exc[j];
                acc.x = fma(a.x, b.x, fma(-a.y, b.y, acc.x));
                acc.y = fma(a.x, b.y, fma(a.y, b.x, acc.y));
            }
        r0[(size_t)f * n0 + i] = acc;
    }
}

// 1/a by the hardware reciprocal and two Newton steps of |a|^2 where that is
// safe, else by division.
__device__ inline double2 zinv_fast(double2 a) {
    const double q = fma(a.x, a.x, a.y * a.y);
    if (__builtin_expect(q > 1e-280 && q < 1e280, 1)) {
        double r = __builtin_amdgcn_rcp(q);
        r = fma(r, fma(-q, r, 1.0), r);
        r = fma(r, fma(-q, r, 1.0), r);
        return make_double2(a.x * r, -a.y * r);
    }
    return zinv(a);
}
// Record of the LU of a launch's systems: factor rows [n0][n0] in the order of
// A's rows (row r holds U from the step that took it as pivot row on, and L
// before), pivot row and 1/pivot per step.
struct SpLu {
    double2 *f;
    int *piv;
    double2 *dinv;
};

// One system's elimination: lane r holds row r, 32 columns at a time in
// registers.  Rows are not exchanged; `step` is the step that took the lane's
// row as its pivot row (64: none yet).
struct SpElim {
    double2 t;       // right-hand side entry of the lane's row
    int step = 64;
    int pk = 0;      // lane k: pivot row of step k
    double2 dk;      // lane k: 1 / pivot of step k
    int flag = 0;
};
// Steps kbase .. kbase + cnt - 1 on a[0 .. W): each takes a[0] as its column,
// picks the pivot row, reads its entries as wave-uniform values and writes the
// updated columns one place to the left, so that the loop body is the same
// for every step.
template <int W>
__device__ __forceinline__ void sp_steps(double2 (&a)[32], SpElim &e, int kbase, int cnt, int n0, int lane,
                                         double2 *__restrict__ frow) {
#pragma unroll 1
    for (int k = kbase; k < kbase + cnt; ++k) {
        const bool open = e.step == 64 && lane < n0;
        float mg = -1.0f;
        if (open) {
            mg = (float)(fabs(a[0].x) + fabs(a[0].y));
            if (!(mg == mg)) mg = __builtin_inff();  // a NaN wins
        }
        const int p = wave_amax(mg);
        const double2 d = rl2(a[0], p);
        if (!(d.x != 0.0 || d.y != 0.0)) e.flag |= COSIM_SYS_SINGULAR;
        const double2 inv = zinv_fast(d);
        double2 l = zmul(a[0], inv);
        l.x = open && lane != p ? l.x : 0.0;
        l.y = open && lane != p ? l.y : 0.0;
        // (componentwise: a select of the struct would put the array in memory)
        const bool low = open && lane != p;
        const double2 fv = make_double2(low ? l.x : a[0].x, low ? l.y : a[0].y);
        if (lane < n0) frow[k] = fv;
        const double2 tp = rl2(e.t, p);
        e.t = zfms(e.t, l, tp);
#pragma unroll
        for (int j = 1; j < W; ++j) a[j - 1] = zfms(a[j], l, rl2(a[j], p));
        if (lane == p) e.step = k;
        if (lane == k) {
            e.pk = p;
            e.dk = inv;
        }
    }
}

// Columns c0 .. c0 + 31 of the lane's row of A (zero past n0); with RHS also
// the variable entries of the right-hand side.
template <bool RHS>
__device__ __forceinline__ void sp_load_columns(const SpDev &d, int f, const double2 *__restrict__ v, int lane,
                                                int c0, double2 (&a)[32], double2 &t) {
    const int n0 = d.n0;
    const double2 *KT = d.KT + (size_t)f * n0 * n0, *S0T = d.S0T + (size_t)f * n0 * n0;
    const bool in = lane < n0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const bool ok = in && c0 + j < n0;
        const double2 k = KT[ok ? (size_t)(c0 + j) * n0 + lane : 0];
        a[j].x = ok ? k.x : 0.0;
        a[j].y = ok ? k.y : 0.0;
    }
    int e = in ? d.rowptr[lane] : 0;
    const int end = in ? d.rowptr[lane + 1] : 0;
    for (; e < end; ++e) {  // each row's entries in their order
        const int i = d.rowent[e], c = d.iy[i];
        const double2 x = v[i];
        if (c < n0) {
#pragma unroll
            for (int j = 0; j < 32; ++j)
                if (c0 + j < n0) a[j] = zfms(a[j], x, S0T[(size_t)(c0 + j) * n0 + c]);
        } else if (RHS) {
            const double2 w = zmul(x, d.exc[c - n0]);
            t.x += w.x;
            t.y += w.y;
        }
    }
}

// One wave per system s = s0 + blockIdx.x: LU with partial pivoting, two halves
// of 32 columns one after the other, and the solution x of A x = S_C12 exc:
// writes X[s][n0] (FP64), the contraction's operand Xg[f][b][n0] (PREC 0:
// complex128, 1: complex64), the status and the record.  Without barriers the
// waves of a SIMD hide each other's pivot chains; the four-wave form with
// the matrix in LDS and three barriers per column took 592 us for 2,560
// systems of 64 ports, this one 248 (three waves per SIMD spill: 395).  For one
// system it is the chain of pivots that counts: the pivot search is integer
// maxima and one comparison (with the row carried beside the magnitude through
// shuffles 64 ports took 120 us, 100 now, the four-wave form 115), and the steps
// leave out the columns past n0 (16 ports, 3,000 x 2 systems: 113 us with all 32,
// 68 now, the four-wave form 99).
template <int PREC>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_sp_lu(
    SpDev d, int B, int s0, const double2 *__restrict__ values, double2 *__restrict__ X, void *Xg,
    SpLu rec, int32_t *__restrict__ status) {
    const int n0 = d.n0, lane = threadIdx.x, slot = blockIdx.x, s = s0 + slot;
    const int b = s / d.F, f = s - b * d.F;
    const double2 *v = values + (size_t)s * d.nvar;
    double2 *frow = rec.f + ((size_t)slot * n0 + min(lane, n0 - 1)) * n0;
    SpElim e;
    e.dk = make_double2(0.0, 0.0);
    e.t = lane < n0 ? d.r0[(size_t)f * n0 + lane] : make_double2(0.0, 0.0);
    double2 a[32];
    sp_load_columns<true>(d, f, v, lane, 0, a, e.t);
    // eight steps at a time, with the columns that are left (a multiple of 8)
    auto half = [&](int kbase) {
        int left = min(n0 - kbase, 32);  // > 0
        if (left > 24) {
            sp_steps<32>(a, e, kbase, 8, n0, lane, frow);
            kbase += 8;
            left -= 8;
        }
        if (left > 16) {
            sp_steps<24>(a, e, kbase, 8, n0, lane, frow);
            kbase += 8;
            left -= 8;
        }
        if (left > 8) {
            sp_steps<16>(a, e, kbase, 8, n0, lane, frow);
            kbase += 8;
            left -= 8;
        }
        sp_steps<8>(a, e, kbase, left, n0, lane, frow);
    };
    half(0);
    if (n0 > 32) {
        sp_load_columns<false>(d, f, v, lane, 32, a, e.t);
        // the steps of the first half on these columns (the first `w`)
        auto earlier = [&](auto w) {
            for (int k0 = 0; k0 < 32; k0 += 8) {
                double2 l8[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) l8[u] = frow[k0 + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int k = k0 + u;
                    const int p = __builtin_amdgcn_readlane(e.pk, k);
                    const double2 l = e.step > k ? l8[u] : make_double2(0.0, 0.0);
#pragma unroll
                    for (int j = 0; j < decltype(w)::value; ++j) a[j] = zfms(a[j], l, rl2(a[j], p));
                }
            }
        };
        if (n0 > 48) earlier(std::integral_constant<int, 32>{});
        else if (n0 > 40) earlier(std::integral_constant<int, 16>{});
        else earlier(std::integral_constant<int, 8>{});
        half(32);
    }
    // back substitution: x_k, then its column off the rows of earlier steps
    double2 x = make_double2(0.0, 0.0);
    double2 u8[8], next[8];  // the rows' entries of eight steps, and of the eight below
    auto rows = [&](int k1, double2 (&u)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) u[i] = frow[max(k1 - 1 - i, 0)];
    };
    rows(n0, u8);
    for (int k1 = n0; k1 > 0; k1 -= 8) {
        rows(k1 - 8, next);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k1 - 1 - u;
            if (k < 0) continue;  // uniform
            const int p = __builtin_amdgcn_readlane(e.pk, k);
            const double2 xk = zmul(rl2(e.t, p), rl2(e.dk, k));
            if (lane == k) x = xk;
            const double2 c = e.step < k ? u8[u] : make_double2(0.0, 0.0);
            e.t = zfms(e.t, c, xk);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) u8[u] = next[u];
    }
    int flag = e.flag;
    const bool finite = isfinite(x.x) && isfinite(x.y);
    if (__ballot(lane < n0 && !finite) != 0) flag |= COSIM_SYS_NONFINITE;
    if (flag & COSIM_SYS_SINGULAR) x = make_double2(__builtin_nan(""), __builtin_nan(""));
    if (lane == 0) status[s] = flag;
    if (lane < n0) {
        X[(size_t)s * n0 + lane] = x;
        const size_t o = ((size_t)f * B + b) * n0 + lane;
        if (PREC == 0) ((double2 *)Xg)[o] = x;
        else ((float2 *)Xg)[o] = make_float2((float)x.x, (float)x.y);
        rec.piv[(size_t)slot * n0 + lane] = e.pk;
        rec.dinv[(size_t)slot * n0 + lane] = e.dk;
    }
}

// t - conj(l) u
__device__ inline double2 zfmsc(double2 t, double2 l, double2 u) {
    return make_double2(fma(-l.x, u.x, fma(-l.y, u.y, t.x)), fma(-l.x, u.y, fma(l.y, u.x, t.y)));
}

// One wave per system s = s0 + i, four per block: r = rscale conj(sum over chunks
// of Rp[c][f][b][:]) (the chunks hold conj(fields^H w)), A^H lam = r with the
// record of k_sp_lu (A = P^T L U: U^H z = r, L^H v = z, lam at pivot row k is
// v_k; both sweeps take the recorded row of each step, lane k its entry k), and
// the gradient of every variable entry to grad[s][nvar].
template <int PREC>
__global__ __launch_bounds__(256) void k_sp_adjoint(SpDev d, int B, int s0, int count,
                                                    const double2 *__restrict__ X, const void *Rp,
                                                    int nchunk, double rscale, SpLu rec,
                                                    double2 *__restrict__ grad,
                                                    int32_t *__restrict__ status) {
    const int n0 = d.n0, F = d.F, nvar = d.nvar, lane = threadIdx.x & 63;
    const int slot = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (slot >= count) return;  // whole wave
    const int s = s0 + slot, b = s / F, f = s - b * F;
    const int li = min(lane, n0 - 1);
    double2 t = make_double2(0.0, 0.0);
    {
        double sr = 0.0, si = 0.0;
#pragma unroll 8
        for (int c = 0; c < nchunk; ++c) {
            const size_t o = (((size_t)c * F + f) * B + b) * n0 + li;
            if (PREC == 0) {
                const double2 r = ((const double2 *)Rp)[o];
                sr += r.x;
                si += r.y;
            } else {
                const float2 r = ((const float2 *)Rp)[o];
                sr += (double)r.x;
                si += (double)r.y;
            }
        }
        if (lane < n0) t = make_double2(rscale * sr, -rscale * si);
    }
    const double2 *__restrict__ fac = rec.f + (size_t)slot * n0 * n0;
    const int pk = rec.piv[(size_t)slot * n0 + li];
    const double2 dk = rec.dinv[(size_t)slot * n0 + li];
    auto load = [&](double2 (&q)[8], int j0) {  // entry `lane` of the rows of steps j0 .. j0 + 7
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int p = __builtin_amdgcn_readlane(pk, min(max(j0 + u, 0), n0 - 1));
            q[u] = fac[(size_t)p * n0 + li];
        }
    };
    double2 q[8], nq[8];
    load(q, 0);
    for (int j0 = 0; j0 < n0; j0 += 8) {  // U^H z = r
        load(nq, j0 + 8);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = j0 + u;
            if (j >= n0) continue;  // uniform
            const double2 z = zmulc(rl2(t, j), rl2(dk, j));
            const double2 w = zfmsc(t, q[u], z);
            if (lane == j) t = z;
            else if (lane > j) t = w;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) q[u] = nq[u];
    }
    load(q, n0 - 8);
    for (int j1 = n0; j1 > 0; j1 -= 8) {  // L^H v = z
        load(nq, j1 - 16);
#pragma unroll
        for (int u = 7; u >= 0; --u) {
            const int j = j1 - 8 + u;
            if (j < 0) continue;  // uniform
            const double2 vj = rl2(t, j);
            const double2 w = zfmsc(t, q[u], vj);
            if (lane < j) t = w;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) q[u] = nq[u];
    }
    // lam to the lane of its row
    const int to = 4 * (lane < n0 ? pk : lane);
    auto send = [&](double x) {
        return __hiloint2double(__builtin_amdgcn_ds_permute(to, __double2hiint(x)),
                                __builtin_amdgcn_ds_permute(to, __double2loint(x)));
    };
    double2 x = make_double2(send(t.x), send(t.y));
    int flag = status[s];
    const bool finite = isfinite(x.x) && isfinite(x.y);
    if (__ballot(lane < n0 && !finite) != 0) flag |= COSIM_SYS_NONFINITE;
    if (flag & COSIM_SYS_SINGULAR) x = make_double2(__builtin_nan(""), __builtin_nan(""));
    if (lane == 0) status[s] = flag;
    // gradient: 2 lam_r conj(exc_j) for S_C12 entries (r, n0 + j), 2 lam_r
    // conj((S0 x)_c) for S_C11 entries (r, c), 0 for S_C21 / S_C22 entries
    // y = S0 x once (lane c: row c, x broadcast from the forward solution)
    const double2 xs = lane < n0 ? X[(size_t)s * n0 + lane] : make_double2(0.0, 0.0);
    double2 y = make_double2(0.0, 0.0);
    const double2 *col = d.S0T + (size_t)f * n0 * n0 + li;
#pragma unroll 8
    for (int k = 0; k < n0; ++k) {
        const double2 a = col[(size_t)k * n0], xk = rl2(xs, k);
        y.x = fma(a.x, xk.x, fma(-a.y, xk.y, y.x));
        y.y = fma(a.x, xk.y, fma(a.y, xk.x, y.y));
    }
    // lane e % 64 forms entry e
    for (int e0 = 0; e0 < nvar; e0 += 64) {
        const int e = e0 + lane;
        const int r = e < nvar ? d.ix[e] : n0, c = e < nvar ? d.iy[e] : 0;
        // gathers from other lanes: every lane takes part in the shuffles
        const int rs = r < n0 ? r : 0, cs = c < n0 ? c : 0;
        const double2 lam = make_double2(__shfl(x.x, rs), __shfl(x.y, rs));
        const double2 yv = make_double2(__shfl(y.x, cs), __shfl(y.y, cs));
        if (e < nvar) {
            double2 g = make_double2(0.0, 0.0);
            if (r < n0) {
                const double2 gv = zmulc(lam, c >= n0 ? d.exc[c - n0] : yv);
                g = make_double2(2.0 * gv.x, 2.0 * gv.y);
            }
            grad[(size_t)s * nvar + e] = g;
        }
    }
}

// The FP64 contraction in one pass: B_comb = fields x for 64 configurations of
// one frequency per workgroup (16 per wave, x as matrix-core B operands in
// registers), the loss epilogue on the accumulators, and conj(fields^H w) from
// the same rows, whose accumulators are the B operand of the second product
// (see fused.hip: row q + 4 m in register m of lane group q).  The four real
// products of a complex one run as separate matrix-core operations; rows come
// in tiles of 16 through two LDS buffers, the next one loaded into registers
// while the current one is used.  NE: ports rounded up to 16.
//   Matrix-core issue bounds it (16 P n0 flops per system): 64 ports, 16,384
// points, 2,560 systems in 753 us (57 TFLOP/s), where two library products and the
// epilogue between them took 1.71 ms and moved B_comb through memory three
// times.
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ inline f64x4 mma64(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <int NE, int LOSS, bool GRAD>
__global__ __launch_bounds__(256, 2) void k_sp_fused(SpDev d, int B, int comp, int tiles_per_chunk,
                                                     const double2 *__restrict__ Xg,
                                                     const double *__restrict__ T,
                                                     double2 *__restrict__ Rp,
                                                     double *__restrict__ lpart) {
    constexpr int KS = NE / 4, IB = NE / 16, LD = NE + 1;
    constexpr int VPT = 16 * NE / 256;  // row entries per thread and tile
    __shared__ double2 sGb[2][16 * LD];
    __shared__ double sTb[2][16];
    const int n0 = d.n0, F = d.F, P = d.P;
    const int f = blockIdx.y, chunk = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, q = lane >> 4;
    const int b = blockIdx.x * 64 + 16 * wave + r16;  // this lane's configuration
    const int pb = chunk * tiles_per_chunk * 16;
    const int pe = min(P, pb + tiles_per_chunk * 16);
    const size_t prow = (size_t)d.ncomp * n0;
    const double2 *G = d.fields64 + (size_t)f * P * prow + (size_t)comp * n0;
    double xr[KS], xi[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        const int k = 4 * kk + q;
        double2 v = make_double2(0.0, 0.0);
        if (b < B && k < n0) v = Xg[((size_t)f * B + b) * n0 + k];
        xr[kk] = v.x;
        xi[kk] = v.y;
    }
    f64x4 rr[IB], ri[IB];
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) rr[ib] = ri[ib] = f64x4{0, 0, 0, 0};
    double lacc = 0.0;
    double2 stg[VPT];
    double tstg = 0.0;
    auto fetch = [&](int p0) {  // zero rows and targets past the last point
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const int e = threadIdx.x + 256 * u, row = e / NE, k = e % NE;
            const bool in = p0 + row < P && k < n0;
            stg[u] = in ? G[(size_t)(p0 + row) * prow + k] : make_double2(0.0, 0.0);
        }
        const int p = p0 + ((int)threadIdx.x & 15);
        tstg = p < P ? T[p] : 0.0;
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const int e = threadIdx.x + 256 * u;
            sGb[buf][(e / NE) * LD + e % NE] = stg[u];
        }
        if (threadIdx.x < 16) sTb[buf][threadIdx.x] = tstg;
    };
    fetch(pb);
    stash(0);
    __syncthreads();
    for (int p0 = pb, buf = 0; p0 < pe; p0 += 16, buf ^= 1) {
        const double2 *sG = sGb[buf];
        fetch(min(p0 + 16, pe - 1));  // past the chunk's end: not used
        f64x4 rx = f64x4{0, 0, 0, 0}, ry = rx, br = rx, bi = rx;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const double2 g = sG[r16 * LD + 4 * kk + q];
            rx = mma64(g.x, xr[kk], rx);
            bi = mma64(g.x, xi[kk], bi);
            ry = mma64(g.y, xi[kk], ry);
            bi = mma64(g.y, xr[kk], bi);
        }
        f64x4 ni;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            double vx = rx[m] - ry[m], vy = bi[m];
            lacc += epilogue<LOSS>(vx, vy, sTb[buf][q + 4 * m]);
            br[m] = vx;
            bi[m] = vy;
            ni[m] = -vy;
        }
        if (GRAD) {
            // G conj(w): re = Gr wr + Gi wi, im = Gi wr - Gr wi
#pragma unroll
            for (int ib = 0; ib < IB; ++ib)
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const double2 g = sG[(q + 4 * m) * LD + 16 * ib + r16];
                    rr[ib] = mma64(g.x, br[m], rr[ib]);
                    ri[ib] = mma64(g.y, br[m], ri[ib]);
                    rr[ib] = mma64(g.y, bi[m], rr[ib]);
                    ri[ib] = mma64(g.x, ni[m], ri[ib]);
                }
        }
        stash(buf ^ 1);
        __syncthreads();
    }
    lacc += __shfl_xor(lacc, 16);
    lacc += __shfl_xor(lacc, 32);
    if (b >= B) return;
    const size_t o = ((size_t)chunk * F + f) * B + b;
    if (q == 0) lpart[o] = lacc;
    if (GRAD) {
#pragma unroll
        for (int ib = 0; ib < IB; ++ib)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int k = 16 * ib + q + 4 * m;
                if (k < n0) Rp[o * n0 + k] = make_double2(rr[ib][m], ri[ib][m]);
            }
    }
}

// Loss terms of one P-chunk and conj(w) in place of B_comb (FP32); grid (B, F).
// Y[f][b][rows] holds B_comb of rows p0 .. p0 + nrows - 1 of the loss
// component; lpart[f][b] receives the chunk's sum of loss terms.
template <int LOSS>
__global__ __launch_bounds__(256) void k_sp_epilogue(int B, int F, int rows, int p0, int nrows,
                                                     float2 *__restrict__ Y,
                                                     const double *__restrict__ T,
                                                     double *__restrict__ lpart, bool grad) {
    __shared__ double red[4];
    const int b = blockIdx.x, f = blockIdx.y;
    const size_t base = ((size_t)f * B + b) * rows;
    double acc = 0.0;
    for (int p = threadIdx.x; p < nrows; p += 256) {
        float2 *y = Y + base + p;
        float vx = y->x, vy = y->y;
        acc += epilogue<LOSS>(vx, vy, (float)T[p0 + p]);
        if (grad) *y = make_float2(vx, -vy);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) lpart[(size_t)f * B + b] = (red[0] + red[1]) + (red[2] + red[3]);
}

// loss[b] = lscale * sum over chunks and f of lpart[c][f][b], one wave per
// configuration, lanes in a fixed shuffle tree.
__global__ __launch_bounds__(256) void k_sp_reduce(int B, int F, int nchunk,
                                                   const double *__restrict__ lpart, double lscale,
                                                   double *__restrict__ loss) {
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (b >= B) return;  // whole wave
    double acc = 0.0;
    for (int e = lane; e < F * nchunk; e += 64) acc += lpart[(size_t)e * B + b];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if (lane == 0) loss[b] = lscale * acc;
}

// Eq. 2-3 per (b, f, k)
__global__ void k_sp_rc(int B, int F, int n, const double *__restrict__ R, const double *__restrict__ C,
                        const double *__restrict__ omega, double z0, double2 *__restrict__ gam, int ld) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (size_t)B * F * n) return;
    const int k = (int)(t % n);
    const size_t sf = t / n;
    const int f = (int)(sf % F), b = (int)(sf / F);
    const double zr = R[k], zi = -1.0 / (omega[f] * C[(size_t)b * n + k]);
    // (zr - z0 + j zi) / (zr + z0 + j zi)
    const double2 num = make_double2(zr - z0, zi), den = make_double2(zr + z0, zi);
    gam[sf * ld + k] = zmul(num, zinv(den));
}

// gC[b][k] = sum over f of Re(conj(g) dGamma/dC), dGamma/dC = 2 z0/(Z_C + z0)^2 j/(w C^2)
__global__ void k_sp_rc_backward(int B, int F, int n, const double *__restrict__ R,
                                 const double *__restrict__ C, const double *__restrict__ omega,
                                 double z0, const double2 *__restrict__ g, int ld,
                                 double *__restrict__ gC) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (size_t)B * n) return;
    const int k = (int)(t % n), b = (int)(t / n);
    const double c = C[t];
    double acc = 0.0;
    for (int f = 0; f < F; ++f) {
        const double w = omega[f];
        const double2 den = make_double2(R[k] + z0, -1.0 / (w * c));
        const double2 inv = zinv(den);
        const double2 inv2 = zmul(inv, inv);
        const double s = 2.0 * z0 / (w * c * c);
        const double2 dg = make_double2(-s * inv2.y, s * inv2.x);  // j s inv2
        const double2 gv = g[((size_t)b * F + f) * ld + k];
        acc += gv.x * dg.x + gv.y * dg.y;  // Re(conj(g) dg)
    }
    gC[t] = acc;
}

__global__ void k_sp_to_c64(size_t count, const double2 *__restrict__ a, float2 *__restrict__ b) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) b[t] = make_float2((float)a[t].x, (float)a[t].y);
}

hipError_t blas(rocblas_status r) { return r == rocblas_status_success ? hipSuccess : hipErrorLaunchFailure; }

// C[f] (m x n, ldc) = op(A[f]) B[f] per frequency, column-major, complex
hipError_t cgemm(rocblas_handle h, int prec, rocblas_operation ta, int m, int n, int k, const void *A,
                 int lda, size_t sA, const void *Bm, int ldb, size_t sB, void *C, int ldc, size_t sC,
                 int batch) {
    if (prec == 0) {
        const rocblas_double_complex one(1.0, 0.0), zero(0.0, 0.0);
        return blas(rocblas_zgemm_strided_batched(
            h, ta, rocblas_operation_none, m, n, k, &one, (const rocblas_double_complex *)A, lda,
            (rocblas_stride)sA, (const rocblas_double_complex *)Bm, ldb, (rocblas_stride)sB, &zero,
            (rocblas_double_complex *)C, ldc, (rocblas_stride)sC, batch));
    }
    const rocblas_float_complex one(1.0f, 0.0f), zero(0.0f, 0.0f);
    return blas(rocblas_cgemm_strided_batched(
        h, ta, rocblas_operation_none, m, n, k, &one, (const rocblas_float_complex *)A, lda,
        (rocblas_stride)sA, (const rocblas_float_complex *)Bm, ldb, (rocblas_stride)sB, &zero,
        (rocblas_float_complex *)C, ldc, (rocblas_stride)sC, batch));
}

SpLu record(const SpWork &w) { return SpLu{w.lu, w.piv, w.dinv}; }

// Forward solves of the systems s0 .. s0 + count - 1 into the record's slots.
hipError_t launch_lu(const SpDev &d, const SpWork &w, int B, int s0, int count, const double2 *values,
                     int prec, int32_t *status, hipStream_t st) {
    if (prec == 0)
        hipLaunchKernelGGL(k_sp_lu<0>, dim3(count), dim3(64), 0, st, d, B, s0, values, w.X, w.Xg,
                           record(w), status);
    else
        hipLaunchKernelGGL(k_sp_lu<1>, dim3(count), dim3(64), 0, st, d, B, s0, values, w.X, w.Xg,
                           record(w), status);
    return hipGetLastError();
}

// The adjoint solves and gradients.  A batch beyond the record's capacity is
// factored again, slab by slab.
hipError_t launch_adjoint(const SpDev &d, const SpWork &w, int B, const double2 *values, int nchunk,
                          double rscale, int prec, double2 *grad, int32_t *status, hipStream_t st) {
    const int S = B * d.F;
    hipError_t e;
    for (int s0 = 0; s0 < S; s0 += w.slots) {
        const int count = std::min(w.slots, S - s0);
        if (S > w.slots && (e = launch_lu(d, w, B, s0, count, values, prec, status, st)) != hipSuccess)
            return e;
        const dim3 grid((count + 3) / 4);
        if (prec == 0)
            hipLaunchKernelGGL(k_sp_adjoint<0>, grid, dim3(256), 0, st, d, B, s0, count, w.X, w.Rp, nchunk,
                               rscale, record(w), grad, status);
        else
            hipLaunchKernelGGL(k_sp_adjoint<1>, grid, dim3(256), 0, st, d, B, s0, count, w.X, w.Rp, nchunk,
                               rscale, record(w), grad, status);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int NE>
hipError_t launch_fused(const SpDev &d, const SpWork &w, int B, const double *T, int comp, int loss_mode,
                        bool grad, hipStream_t st) {
    const int tiles = (d.P + 15) / 16, nck = sp_fused_chunks(d, B);
    const int tpc = (tiles + nck - 1) / nck;
    const dim3 grid((B + 63) / 64, d.F, (tiles + tpc - 1) / tpc);
    const double2 *x = (const double2 *)w.Xg;
    double2 *rp = (double2 *)w.Rp;
#define SP_FUSED(LS, GR)                                                                              \
    hipLaunchKernelGGL((k_sp_fused<NE, LS, GR>), grid, dim3(256), 0, st, d, B, comp, tpc, x, T, rp, \
                       w.lpart)
    if (loss_mode == COSIM_LOSS_MAG) {
        if (grad) SP_FUSED(COSIM_LOSS_MAG, true);
        else SP_FUSED(COSIM_LOSS_MAG, false);
    } else {
        if (grad) SP_FUSED(COSIM_LOSS_COMPLEX, true);
        else SP_FUSED(COSIM_LOSS_COMPLEX, false);
    }
#undef SP_FUSED
    return hipGetLastError();
}

}  // namespace

hipError_t sp_blas_create(void **handle) {
    rocblas_handle h = nullptr;
    if (rocblas_create_handle(&h) != rocblas_status_success) return hipErrorOutOfMemory;
    *handle = h;
    return hipSuccess;
}

void sp_blas_destroy(void *handle) {
    if (handle) (void)rocblas_destroy_handle((rocblas_handle)handle);
}

hipError_t sp_prep(const SpDev &d, const double2 *S0, const double2 *scc, hipStream_t st) {
    hipLaunchKernelGGL(k_sp_prep, dim3(d.n0, d.F), dim3(64), 0, st, d.n0, d.n1, d.F, S0, scc, d.exc,
                       d.KT, d.S0T, d.r0);
    return hipGetLastError();
}

// Chunks of whole 16-row tiles: the fewest whose workgroups fill the last round
// of resident ones (two per compute unit) to 95%, else the best fill; 64 at
// most, as the partial sums are written and read once per chunk.
int sp_fused_chunks(const SpDev &d, int B) {
    const long long wgs = (long long)((B + 63) / 64) * d.F, slots = 2LL * std::max(1, d.cus);
    const int tiles = (d.P + 15) / 16, most = std::min(tiles, 64);
    int best = 1;
    double fill = 0.0;
    for (int c = 1; c <= most; ++c) {
        const int tpc = (tiles + c - 1) / c, cc = (tiles + tpc - 1) / tpc;
        const long long n = wgs * cc;
        const double x = (double)n / (double)((n + slots - 1) / slots * slots);
        if (x > fill) {
            fill = x;
            best = cc;
        }
        if (x >= 0.95) break;
    }
    return best;
}

hipError_t sp_forward(const SpDev &d, const SpWork &w, int B, const double2 *values, int prec,
                      int32_t *status, hipStream_t st) {
    const int S = B * d.F;
    for (int s0 = 0; s0 < S; s0 += w.slots) {
        const hipError_t e = launch_lu(d, w, B, s0, std::min(w.slots, S - s0), values, prec, status, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t sp_field(void *handle, const SpDev &d, int B, const double2 *Xg64, double2 *out,
                    hipStream_t st) {
    rocblas_handle h = (rocblas_handle)handle;
    if (rocblas_set_stream(h, st) != rocblas_status_success) return hipErrorInvalidValue;
    const int m = d.P * d.ncomp;
    // out[b][f][p][c]: per frequency a (P ncomp) x B column-major block with ld F P ncomp
    return cgemm(h, 0, rocblas_operation_transpose, m, B, d.n0, d.fields64, d.n0,
                 (size_t)d.P * d.ncomp * d.n0, Xg64, d.n0, (size_t)B * d.n0, out, d.F * m, (size_t)m,
                 d.F);
}

hipError_t sp_loss_and_grad(void *handle, const SpDev &d, const SpWork &w, int B,
                            const double2 *values, const double *T, int comp, int loss_mode, int prec,
                            double *loss, double2 *grad, int32_t *status, hipStream_t st) {
    hipError_t e = sp_forward(d, w, B, values, prec, status, st);
    if (e != hipSuccess) return e;
    const double scale = 1.0 / ((double)d.F * d.P);
    if (prec == 0) {
        const bool g = grad != nullptr;
        switch ((d.n0 + 15) / 16) {
            case 1: e = launch_fused<16>(d, w, B, T, comp, loss_mode, g, st); break;
            case 2: e = launch_fused<32>(d, w, B, T, comp, loss_mode, g, st); break;
            case 3: e = launch_fused<48>(d, w, B, T, comp, loss_mode, g, st); break;
            default: e = launch_fused<64>(d, w, B, T, comp, loss_mode, g, st); break;
        }
        if (e != hipSuccess) return e;
        const int nck = sp_fused_chunks(d, B);
        hipLaunchKernelGGL(k_sp_reduce, dim3((B + 3) / 4), dim3(256), 0, st, B, d.F, nck, w.lpart,
                           scale, loss);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        return g ? launch_adjoint(d, w, B, values, nck, scale, 0, grad, status, st) : hipSuccess;
    }
    rocblas_handle h = (rocblas_handle)handle;
    if (rocblas_set_stream(h, st) != rocblas_status_success) return hipErrorInvalidValue;
    const void *fields = d.fields32;
    const size_t esz = sizeof(float2);
    const int lda = d.ncomp * d.n0;
    const size_t sA = (size_t)d.P * d.ncomp * d.n0;
    const bool want_grad = grad != nullptr;
    for (int c = 0; c < w.nchunk; ++c) {
        const int p0 = c * w.rows, nr = std::min(w.rows, d.P - p0);
        const char *A = (const char *)fields + ((size_t)p0 * d.ncomp + comp) * d.n0 * esz;
        // B_comb of the chunk: (nr x n0)(n0 x B) per frequency
        if ((e = cgemm(h, prec, rocblas_operation_transpose, nr, B, d.n0, A, lda, sA, w.Xg, d.n0,
                       (size_t)B * d.n0, w.Y, w.rows, (size_t)B * w.rows, d.F)) != hipSuccess)
            return e;
#define SP_EPI(LS)                                                                         \
    hipLaunchKernelGGL((k_sp_epilogue<LS>), dim3(B, d.F), dim3(256), 0, st, B, d.F, w.rows, \
                       p0, nr, (float2 *)w.Y, T, w.lpart + (size_t)c * d.F * B, want_grad)
        if (loss_mode == COSIM_LOSS_MAG) SP_EPI(COSIM_LOSS_MAG);
        else SP_EPI(COSIM_LOSS_COMPLEX);
#undef SP_EPI
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (!want_grad) continue;
        // conj(fields^H w) of the chunk: (n0 x nr)(nr x B) per frequency
        char *Rc = (char *)w.Rp + (size_t)c * d.F * B * d.n0 * esz;
        if ((e = cgemm(h, prec, rocblas_operation_none, d.n0, B, nr, A, lda, sA, w.Y, w.rows,
                       (size_t)B * w.rows, Rc, d.n0, (size_t)B * d.n0, d.F)) != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL(k_sp_reduce, dim3((B + 3) / 4), dim3(256), 0, st, B, d.F, w.nchunk, w.lpart,
                       scale, loss);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (!want_grad) return hipSuccess;
    return launch_adjoint(d, w, B, values, w.nchunk, scale, 1, grad, status, st);
}

hipError_t sp_to_c64(size_t count, const double2 *a, float2 *b, hipStream_t st) {
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sp_to_c64, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, count, a,
                       b);
    return hipGetLastError();
}

hipError_t sp_rc(int B, int F, int n, const double *R, const double *C, const double *omega,
                 double z0, double2 *gam, int ld, hipStream_t st) {
    const size_t t = (size_t)B * F * n;
    if (t == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sp_rc, dim3((unsigned)((t + 255) / 256)), dim3(256), 0, st, B, F, n, R, C,
                       omega, z0, gam, ld);
    return hipGetLastError();
}

hipError_t sp_rc_backward(int B, int F, int n, const double *R, const double *C, const double *omega,
                          double z0, const double2 *g, int ld, double *gC, hipStream_t st) {
    const size_t t = (size_t)B * n;
    if (t == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sp_rc_backward, dim3((unsigned)((t + 255) / 256)), dim3(256), 0, st, B, F, n,
                       R, C, omega, z0, g, ld, gC);
    return hipGetLastError();
}

}  // namespace cosim
