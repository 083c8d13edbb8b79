// Batched FP64 complex solves for more than 64 loops (NP a multiple of 64, up
// to kMaxLoopsBig): Z I = E - j w Phi (Eq. 6 in impedance form) and, Z being
// complex symmetric, the adjoint Z mu = r with the same factor.
//
// One workgroup per (configuration, frequency) system; Z and its factor live
// in HBM ([NP][NP] complex, row-major, per system).  Right-looking LU with
// partial pivoting in panels of kPW columns:
//   1. each panel column: arg-max of |re|+|im| below the diagonal (ties to the
//      lower row), the whole row swapped at once, multipliers scaled, the rest
//      of the panel updated (rank-1);
//   2. U12 = L11^-1 A12 (one thread per column);
//   3. A22 -= L21 U12 over 16x16 tiles staged in LDS.
// The result is P Z = L U with the swaps recorded in order; the solve kernel
// replays the swaps on the right-hand side and runs the two triangular solves
// in blocks of 16 rows (dot products against solved rows, then the 16x16
// diagonal block inside one wave).
//
// When every R_k > 0 the impedance is complex symmetric with a positive
// definite real part, and Z = L D L^T needs no row exchanges (as for the
// smaller systems).  big_factor then runs a blocked LDL^T in block rows of 64,
// U = D L^T in the upper triangle of the slot:
//   k_ldl_start: input flags and diagonal block 0;
//   k_ldl_step, one launch per block row b: U_b,i = X_b (Z_b,i - the rows
//   above) on matrix cores, X_b = L_bb^-1, and diagonal block b + 1;
//   k_ldl_trail, after every kSuper block rows: their update of the trailing
//   matrix.
// The forward substitution rides along with the diagonal blocks, so that the
// forward solve is one backward sweep (k_big_solve), the adjoint both sweeps.
// Systems whose smallest pivot is below 1e-5 of the largest |Z_kk| (or not
// finite), or whose input is invalid, are marked and re-factored by k_lu_big
// with pivoting.
//
// With refinement on, the same kernels run on a complex64 record (diagonal
// blocks in FP64; the tiles on FP32 matrix cores, half the bytes and twice the
// peak of FP64), and k_solve_refined turns the FP32 factor F into FP64
// solutions by iterative refinement:
// x = F^-1 b, then r = b - Z x in FP64 (Z formed on the fly from M, R, C and
// w; it is never stored in FP64) and x += F^-1 r until the next correction is
// predicted below tol |x|.  A system that does not converge is re-factored in
// FP64 with pivoting and solved again.
#include "internal.h"
#include "ldl_block.h"

namespace cosim {

namespace {

constexpr int kPW = 16;    // panel width
constexpr int kTB = 256;   // threads per workgroup
constexpr int kTS = 1024;  // threads per workgroup of the solves: one wave per row of a 16-row block

// One system's view of its instance: the operands of Z and of the right-hand
// side, and where its outputs go.  s is the system's index in its instance.
struct SysRef {
    int n, S, s;
    double w;
    const double *M, *R, *phi, *Cb;  // Cb: the capacitances of the system's configuration
    double2 *I;                      // the instance's [S][n] currents
    const void *rhs;                 // the instance's adjoint sums
    int nchunk;
    double rscale;
    double *gsys;
    double2 *mu;
    int32_t *status;  // the instance's [S] status
};

// The systems of one instance (grid index = system index).
struct OneInst {
    const double *M, *R, *phi, *C, *omega;
    double2 *I;
    const void *rhs;
    double *gsys;
    double2 *mu;
    int32_t *status;
    int n, F, S, nchunk;
    double rscale;
    __device__ SysRef ref(int g) const {
        const int b = g / F, f = g - b * F;
        return SysRef{n, S, g, omega[f], M, R, phi, C + (size_t)b * n, I, rhs, nchunk, rscale,
                      gsys, mu, status};
    }
};

// The systems of up to kGroupMax instances of one padded size, numbered
// instance after instance (GroupArgs, passed by value).
struct GroupSrc {
    GroupArgs g;
    __device__ SysRef ref(int gs) const {
        int j = 0;
        while (j + 1 < g.count && gs >= g.in[j + 1].s0) ++j;
        const GroupInst &e = g.in[j];
        const int s = gs - e.s0, b = s / e.F, f = s - b * e.F;
        return SysRef{e.n, e.S, s, e.omega[f], e.M, e.R, e.phi, e.C + (size_t)b * e.n, e.I, e.rhs,
                      e.nchunk, e.rscale, e.gsys, e.mu, e.status};
    }
};

// Arg-max of (m, idx) over the workgroup, ties to the lower index; every
// thread returns with the result.  sm/si: 4-entry LDS scratch.
__device__ inline void block_amax(double &m, int &idx, double *sm, int *si) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const double om = __shfl_xor(m, off);
        const int oi = __shfl_xor(idx, off);
        if (om > m || (om == m && oi < idx)) {
            m = om;
            idx = oi;
        }
    }
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sm[wv] = m;
        si[wv] = idx;
    }
    __syncthreads();
    m = sm[0];
    idx = si[0];
#pragma unroll
    for (int w = 1; w < kTB / 64; ++w)
        if (sm[w] > m || (sm[w] == m && si[w] < idx)) {
            m = sm[w];
            idx = si[w];
        }
    __syncthreads();
}

// FALLBACK: the launch for marked systems, usually none: held to 128 registers
// so that it does not wait for an empty SIMD beside other work (0.5 ms in a
// multi-instance call).  A launch for all systems keeps the 120 entries of L11
// in registers across the columns of step 2 (one wave per SIMD; 256 loops, 32
// systems: 2.25 ms against 2.61).
template <bool FALLBACK, class Src>
__global__ __launch_bounds__(kTB, FALLBACK ? 4 : 1) void k_lu_big(int NP, int S, Src src,
                                                double2 *__restrict__ Aall, int *__restrict__ pivall,
                                                const int *__restrict__ only, int want) {
    __shared__ double sm[kTB / 64];
    __shared__ int si[kTB / 64];
    __shared__ int sFlag;
    __shared__ double2 sU[kPW];
    __shared__ double2 sL11[kPW][kPW];
    __shared__ double2 sLt[16][kPW + 1];
    __shared__ double2 sUt[kPW][16 + 1];
    const int s = blockIdx.x;
    if (s >= S) return;  // whole workgroup
    if (only && only[s] != want) return;  // re-factor marked systems only
    const int tid = threadIdx.x;
    double2 *A = Aall + (size_t)s * NP * NP;
    int *piv = pivall + (size_t)s * NP;
    const SysRef r = src.ref(s);
    const int n = r.n;
    const double w = r.w;
    const double *__restrict__ M = r.M;
    const double *__restrict__ Rv = r.R;
    const double *__restrict__ Cb = r.Cb;
    if (tid == 0) sFlag = 0;
    __syncthreads();
    for (int k = tid; k < n; k += kTB) {
        const double c = Cb[k];
        if (isnan(c) || c == 0.0 || !isfinite(w) || w == 0.0) atomicOr(&sFlag, COSIM_SYS_BAD_INPUT);
        else if (c < 0.0) atomicOr(&sFlag, COSIM_SYS_NEGATIVE_C);
    }
    // Z = diag(R) + j w M + diag(1/(j w C)), identity padding
    for (size_t e = tid; e < (size_t)NP * NP; e += kTB) {
        const int i = (int)(e / NP), j = (int)(e - (size_t)i * NP);
        double zr = 0.0, zi = 0.0;
        if (i < n && j < n) {
            zi = w * M[(size_t)i * n + j];
            if (i == j) {
                zr = Rv[i];
                zi -= 1.0 / (w * Cb[i]);
            }
        } else if (i == j) {
            zr = 1.0;
        }
        A[e] = make_double2(zr, zi);
    }
    __syncthreads();

    for (int j0 = 0; j0 < NP; j0 += kPW) {
        // ---- 1. panel columns j0 .. j0 + kPW - 1
        for (int jj = 0; jj < kPW; ++jj) {
            const int j = j0 + jj;
            double m = -1.0;
            int idx = j;
            for (int i = j + tid; i < NP; i += kTB) {
                const double2 a = A[(size_t)i * NP + j];
                double mg = fabs(a.x) + fabs(a.y);
                if (!(mg == mg)) mg = __builtin_inf();
                if (mg > m) {
                    m = mg;
                    idx = i;
                }
            }
            block_amax(m, idx, sm, si);
            const int p = idx;
            if (tid == 0) piv[j] = p;
            if (p != j) {
                for (int c = tid; c < NP; c += kTB) {
                    const double2 t = A[(size_t)j * NP + c];
                    A[(size_t)j * NP + c] = A[(size_t)p * NP + c];
                    A[(size_t)p * NP + c] = t;
                }
            }
            __syncthreads();
            if (tid < kPW) sU[tid] = A[(size_t)j * NP + j0 + tid];
            __syncthreads();
            const double2 d = sU[jj];
            if (tid == 0 && !(d.x != 0.0 || d.y != 0.0)) atomicOr(&sFlag, COSIM_SYS_SINGULAR);
            const double2 inv = zinv(d);
            for (int i = j + 1 + tid; i < NP; i += kTB) {
                double2 *row = A + (size_t)i * NP + j0;
                const double2 l = zmul(row[jj], inv);
                row[jj] = l;
                for (int c = jj + 1; c < kPW; ++c) row[c] = zfms(row[c], l, sU[c]);
            }
            __syncthreads();
        }
        if (j0 + kPW >= NP) break;
        // ---- 2. U12 = L11^-1 A12
        for (int e = tid; e < kPW * kPW; e += kTB) {
            const int r = e / kPW, c = e - r * kPW;
            sL11[r][c] = A[(size_t)(j0 + r) * NP + j0 + c];
        }
        __syncthreads();
        for (int c = j0 + kPW + tid; c < NP; c += kTB) {
            if (FALLBACK) asm volatile("" ::: "memory");  // L11 stays in LDS
            double2 u[kPW];
#pragma unroll
            for (int r = 0; r < kPW; ++r) u[r] = A[(size_t)(j0 + r) * NP + c];
#pragma unroll
            for (int r = 1; r < kPW; ++r)
#pragma unroll
                for (int r2 = 0; r2 < r; ++r2) u[r] = zfms(u[r], sL11[r][r2], u[r2]);
#pragma unroll
            for (int r = 1; r < kPW; ++r) A[(size_t)(j0 + r) * NP + c] = u[r];
        }
        __syncthreads();
        // ---- 3. A22 -= L21 U12, tiles of 16 x 16
        const int base = j0 + kPW, nt = (NP - base) / 16;
        const int tr = tid >> 4, tc = tid & 15;
        for (int t = 0; t < nt * nt; ++t) {
            const int ti = t / nt, tj = t - ti * nt;
            const int r0 = base + 16 * ti, c0 = base + 16 * tj;
            sLt[tr][tc] = A[(size_t)(r0 + tr) * NP + j0 + tc];
            sUt[tr][tc] = A[(size_t)(j0 + tr) * NP + c0 + tc];
            __syncthreads();
            double2 acc = A[(size_t)(r0 + tr) * NP + c0 + tc];
#pragma unroll
            for (int k = 0; k < kPW; ++k) acc = zfms(acc, sLt[tr][k], sUt[k][tc]);
            A[(size_t)(r0 + tr) * NP + c0 + tc] = acc;
            __syncthreads();
        }
    }
    if (tid == 0) r.status[r.s] = sFlag;
}

// Entry (i, j) of Z = diag(R) + j w M + diag(1/(j w C)), identity padding.
__device__ inline double2 z_entry(const SysRef &r, int i, int j) {
    if (i < r.n && j < r.n) {
        double2 z = make_double2(0.0, r.w * r.M[(size_t)i * r.n + j]);
        if (i == j) {
            z.x = r.R[i];
            z.y -= 1.0 / (r.w * r.Cb[i]);
        }
        return z;
    }
    return make_double2(i == j ? 1.0 : 0.0, 0.0);
}

// The same entry in two parts, so that a tile's loads are issued together and
// without a branch: w M_ij off the diagonal (0 in the padding; the address
// stays inside M), and the diagonal entry, padding 1.
__device__ inline double z_off(const SysRef &r, int i, int j) {
    const double v = r.w * r.M[(size_t)min(i, r.n - 1) * r.n + min(j, r.n - 1)];
    return i < r.n && j < r.n ? v : 0.0;
}
__device__ inline double2 z_diag(const SysRef &r, int i) { return z_entry(r, i, i); }

// ---- blocked LDL^T --------------------------------------------------------
// Blocks of 64 rows, U = D L^T kept in the upper triangle of the system's
// slot (row-major, row stride NP).  Per system beside it: X^T = L_bb^-T of
// each diagonal block b ([NP/64][64][64]) and D^-1, y = L^-1 (E - j w Phi)
// ([2][NP]).
//
// Block row b is U_b,i = X_b (Z_b,i - sum_j U_j,b^T D_j^-1 U_j,i).  The sum
// runs over the rows of the current super-panel of kSuper blocks only; what
// the super-panels before it contribute has been subtracted from the tile in
// HBM by k_ldl_trail (a tile of the first super-panel is formed from M, R, C
// and w and never stored).  Against an update of the whole trailing matrix
// after every 64 columns this reads and writes it once per kSuper blocks.
constexpr int kSuper = 4;

// Entry k of the right-hand side less what the super-panels before block js
// contribute: E - j w Phi, later the running value that k_ldl_trail keeps in
// the place of y.
__device__ inline double2 rhs_base(const SysRef &r, int k, int js, const double2 *y) {
    if (js > 0) return y[k];
    return k < r.n ? loop_voltage(r.phi, r.n, k, r.w) : make_double2(0.0, 0.0);
}

// Accumulates sum over rows j0 <= j < j1 (a multiple of 64 apart) of
// u_ja d_j u_jb, d = D^-1, for NR pairs of 16-column blocks: pair q takes the
// rows' entries at column ca[q] as the A operand and those at cb[q] (cb[0]
// when NB == 1) times d_j as the B operand.  Lane l supplies row j + l / 16
// of each step of 4 rows and column l % 16 of the block (in ca, cb), so both
// operands are runs of 256 bytes.  The operands of two steps are loaded one
// pair ahead into the other of two register sets.  sd[j - j0] = d_j; with Y
// the lane also forms its share of sum_j (d_j u_jb) y_j for cb[0].
template <typename T2, typename T, int NR, int NB, bool Y>
__device__ __forceinline__ void acc_utu(const T2 *__restrict__ A, int NP, int j0, int j1,
                                        const int (&ca)[NR], const int (&cb)[NB],
                                        const double2 *sd, const double2 *sy, int g,
                                        typename Acc4<T>::type (&Cr)[NR],
                                        typename Acc4<T>::type (&Ci)[NR], double2 &yacc) {
    T2 a0[2][NR], b0[2][NB], a1[2][NR], b1[2][NB];
    auto load = [&](int j, T2 (&a)[2][NR], T2 (&b)[2][NB]) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const T2 *row = A + (size_t)(j + 4 * u + g) * NP;
#pragma unroll
            for (int q = 0; q < NR; ++q) a[u][q] = row[ca[q]];
#pragma unroll
            for (int t = 0; t < NB; ++t) b[u][t] = row[cb[t]];
        }
    };
    auto mul = [&](int j, const T2 (&a)[2][NR], const T2 (&b)[2][NB]) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const double2 d = sd[j - j0 + 4 * u + g];
            T br[NB], bi[NB];
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const double2 v = zmul(ld2(b[u][t]), d);
                if (Y && t == 0) yacc = zfma(yacc, v, sy[j - j0 + 4 * u + g]);
                br[t] = (T)v.x;
                bi[t] = (T)v.y;
            }
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                const int t = NB == 1 ? 0 : q;
                const T ar = (T)a[u][q].x, ai = (T)a[u][q].y;
                Cr[q] = mfma4(ar, br[t], Cr[q]);
                Ci[q] = mfma4(ar, bi[t], Ci[q]);
                Cr[q] = mfma4(ai, -bi[t], Cr[q]);
                Ci[q] = mfma4(ai, br[t], Ci[q]);
            }
        }
    };
    if (j0 >= j1) return;
    load(j0, a0, b0);
    for (int j = j0; j < j1; j += 16) {
        load(j + 8, a1, b1);
        mul(j, a0, b0);
        load(min(j + 16, j1 - 8), a0, b0);  // the last pass loads rows again (unused)
        mul(j + 8, a1, b1);
    }
}

// LDS of one workgroup of k_ldl_step.
struct LdlLds : BlockLds {
    double2 sd[64 * kSuper];  // D^-1 of the super-panel's rows
    double2 sy[64 * kSuper];  // y of the same rows
    double sm[kTB / 64];
    int si[kTB / 64];
    int flag;
};

// What a wave reads of Z (its diagonal entries excepted in the first
// super-panel: sz) and of the right-hand side (lanes of its first column
// block) for the diagonal block, loaded ahead of the sums over U: alone, behind
// them, these loads and their address chain took 5 us per block.
struct DiagIn {
    double2 z[3][4], b;
};
template <typename T2>
__device__ __forceinline__ void ldl_diag_load(int NP, const SysRef &sys, int ib, int js,
                                              const T2 *__restrict__ A, const double2 *__restrict__ D,
                                              DiagIn &in) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int g = lane >> 4, r16 = lane & 15, k0 = 64 * ib;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (q >= (wv < 2 ? 3 : 2)) continue;
        const int row = k0 + 16 * diag_rb(wv, q) + g, col = k0 + 16 * diag_cb(wv, q) + r16;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            in.z[q][e] = js == 0 ? make_double2(0.0, z_off(sys, row + 4 * e, col))
                                 : ld2(A[(size_t)(row + 4 * e) * NP + col]);
    }
    if (sizeof(T2) == sizeof(double2) && lane < 16)
        in.b = rhs_base(sys, k0 + 16 * diag_cb(wv, 0) + r16, js, D + NP);
}

// Diagonal block ib: Z_ii - sum over the super-panel's rows [64 js, 64 ib) of
// u d u^T, then ldl_block and y = X (E - j w Phi - L y).
template <typename T2>
__device__ __forceinline__ void ldl_diag(int NP, int n, int s, const DiagIn &in, int ib, int js, T2 *__restrict__ A,
                                         T2 *__restrict__ XT, double2 *__restrict__ D,
                                         int *__restrict__ fmt, double zmax, LdlLds &m) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    const int k0 = 64 * ib, j0 = 64 * js;
    f64x4 Cr[3], Ci[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) Cr[q] = Ci[q] = f64x4{0, 0, 0, 0};
    double2 yacc = make_double2(0.0, 0.0);
    constexpr bool kY = sizeof(T2) == sizeof(double2);
    {
        const int nq = wv < 2 ? 3 : 2;
        if (wv < 2) {
            const int ca[3] = {k0 + r16, k0 + 16 + r16, k0 + 32 + r16};
            const int cb[1] = {k0 + (wv == 1 ? 48 : 0) + r16};
            acc_utu<T2, double, 3, 1, kY>(A, NP, j0, k0, ca, cb, m.sd, m.sy, g, Cr, Ci, yacc);
        } else {
            f64x4 cr[2] = {Cr[0], Cr[0]}, ci[2] = {Cr[0], Cr[0]};
            if (wv == 2) {
                const int ca[2] = {k0 + 16 + r16, k0 + 32 + r16};
                const int cb[1] = {k0 + 16 + r16};
                acc_utu<T2, double, 2, 1, kY>(A, NP, j0, k0, ca, cb, m.sd, m.sy, g, cr, ci, yacc);
            } else {
                const int ca[2] = {k0 + 32 + r16, k0 + 48 + r16};
                acc_utu<T2, double, 2, 2, kY>(A, NP, j0, k0, ca, ca, m.sd, m.sy, g, cr, ci, yacc);
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                Cr[q] = cr[q];
                Ci[q] = ci[q];
            }
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (q >= nq) continue;
            const int row = 16 * diag_rb(wv, q) + g, col = 16 * diag_cb(wv, q) + r16;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double2 z = in.z[q][e];
                if (js == 0 && diag_rb(wv, q) == diag_cb(wv, q)) {
                    const double2 zd = m.sz[row + 4 * e];
                    z.x = row + 4 * e == col ? zd.x : 0.0;
                    z.y = row + 4 * e == col ? zd.y : z.y;
                }
                Cr[q][e] = z.x - Cr[q][e];
                Ci[q][e] = z.y - Ci[q][e];
            }
        }
    }
    if (kY) {  // st = E - j w Phi - L y (the columns of this wave's first B operand)
        yacc.x += __shfl_xor(yacc.x, 16);
        yacc.y += __shfl_xor(yacc.y, 16);
        yacc.x += __shfl_xor(yacc.x, 32);
        yacc.y += __shfl_xor(yacc.y, 32);
        if (lane < 16) {
            const int c = 16 * diag_cb(wv, 0) + r16;
            m.st[c] = make_double2(in.b.x - yacc.x, in.b.y - yacc.y);
        }
    }
    T2 *X = XT + (size_t)ib * 64 * 64;
    ldl_block<T2, true>(m, Cr, Ci, X, A + (size_t)k0 * NP + k0, NP, D + k0);
    if (wv == 0) {
        const double dmin = block_min_pivot(m, lane, n - k0);  // not the padding's pivots of 1
        if (lane == 0 && !(dmin >= 1e-5 * zmax)) fmt[s] = kFmtNeedsPivot;
    }
    if (kY) {
        const double2 y = block_x_times(X, m.st, m.sd, tid);
        if (tid < 64) D[NP + k0 + tid] = y;
    }
}

// Workgroups of a system consecutive on one XCD (workgroups are dealt to the
// 8 XCDs round robin): id -> system 8 (k / T) + id % 8, item k % T, k = id / 8.
// The rows of U that a system's tiles share then stay in that XCD's L2.
__device__ inline int xcd_system(int id, int T, int *item) {
    const int k = id >> 3;
    *item = k % T;
    return 8 * (k / T) + (id & 7);
}

// The same with the items t = 0 of all systems dealt first: they are the long
// ones (a step's diagonal block), and the short ones then fill in behind them
// instead of the launch ending on a few long ones.
__device__ inline int xcd_system_first(int id, int S, int T, int *item) {
    const int S8 = (S + 7) & ~7;
    if (id < S8) {
        *item = 0;
        return id;
    }
    const int s = xcd_system(id - S8, T - 1, item);
    ++*item;
    return s;
}

// The first step: input flags, the largest diagonal |Z_kk|, diagonal block 0.
template <typename T2, class Src>
__global__ __launch_bounds__(kTB, 2) void k_ldl_start(int NP, int S, Src src, T2 *__restrict__ Aall,
                                                      T2 *__restrict__ Xall, double2 *__restrict__ Dall,
                                                      int *__restrict__ fmt, double *__restrict__ zmax) {
    __shared__ LdlLds m;
    const int s = blockIdx.x, tid = threadIdx.x;
    if (s >= S) return;  // whole workgroup
    const SysRef r = src.ref(s);
    DiagIn in;
    ldl_diag_load(NP, r, 0, 0, Aall, Dall, in);
    if (tid == 0) m.flag = 0;
    __syncthreads();
    double zm = 0.0;
    for (int k = tid; k < r.n; k += kTB) {
        const double c = r.Cb[k];
        if (isnan(c) || c == 0.0 || !isfinite(r.w) || r.w == 0.0) atomicOr(&m.flag, COSIM_SYS_BAD_INPUT);
        else if (c < 0.0) atomicOr(&m.flag, COSIM_SYS_NEGATIVE_C);
        zm = fmax(zm, fabs(r.R[k]) + fabs(r.w * r.M[(size_t)k * r.n + k] - 1.0 / (r.w * c)));
    }
    int dummy = 0;
    block_amax(zm, dummy, m.sm, m.si);  // max over the workgroup (index unused)
    const int flag = m.flag;
    const bool bad = (flag & COSIM_SYS_BAD_INPUT) != 0;
    if (tid == 0) {
        r.status[r.s] = flag;
        fmt[s] = bad ? kFmtNeedsPivot : kFmtLDL;
        zmax[s] = zm;
    }
    if (bad) return;  // whole workgroup: left to the pivoted LU
    if (tid < 64) m.sz[tid] = z_diag(r, tid);
    __syncthreads();
    ldl_diag(NP, r.n, s, in, 0, 0, Aall + (size_t)s * NP * NP, Xall + (size_t)s * 64 * NP,
             Dall + (size_t)s * 2 * NP, fmt, zm, m);
}

// A 64 x 64 tile of the trailing matrix as accumulators: each wave holds 64
// rows of its 16 columns, so that block row b's product with X_b takes them
// as the B operand where they are.  base + rows (and yacc) as in acc_utu.
// DIAG: the tile may be a diagonal one.
template <typename T2, bool DIAG, bool Y>
__device__ __forceinline__ void ldl_tile(int NP, const SysRef &sys, int rb, int cbk, int js, int j1,
                                         const T2 *__restrict__ A, const double2 *sd,
                                         const double2 *sy, double2 &yacc, int g,
                                         int r16, int wv, typename Acc4<typename Scal<T2>::type>::type (&Cr)[4],
                                         typename Acc4<typename Scal<T2>::type>::type (&Ci)[4]) {
    typedef typename Scal<T2>::type T;
    typedef typename Acc4<T>::type V4;
    const int col = 64 * cbk + 16 * wv + r16;
    int ca[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        ca[q] = 64 * rb + 16 * q + r16;
        Cr[q] = Ci[q] = V4{0, 0, 0, 0};
    }
    const int cb[1] = {col};
    acc_utu<T2, T, 4, 1, Y>(A, NP, 64 * js, j1, ca, cb, sd, sy, g, Cr, Ci, yacc);
    // Z in batches of QB x 4 entries, the loads of a batch issued together; the
    // trailing update, with three waves per SIMD, has registers for one row of
    // blocks at a time (all four at two waves: 2.66 ms against 2.53, 1,024 loops).
    constexpr int QB = DIAG ? 1 : 4;
#pragma unroll
    for (int q0 = 0; q0 < 4; q0 += QB) {
        if (DIAG && js == 0 && rb == cbk) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double2 z = z_entry(sys, 64 * rb + 16 * q0 + acc_row<T>(g, e), col);
                Cr[q0][e] = (T)z.x - Cr[q0][e];
                Ci[q0][e] = (T)z.y - Ci[q0][e];
            }
        } else if (js == 0) {
            double zo[QB][4];
#pragma unroll
            for (int q = 0; q < QB; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    zo[q][e] = z_off(sys, 64 * rb + 16 * (q0 + q) + acc_row<T>(g, e), col);
#pragma unroll
            for (int q = 0; q < QB; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    Cr[q0 + q][e] = (T)0 - Cr[q0 + q][e];
                    Ci[q0 + q][e] = (T)zo[q][e] - Ci[q0 + q][e];
                }
        } else {
            T2 z[QB][4];
#pragma unroll
            for (int q = 0; q < QB; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    z[q][e] = A[(size_t)(64 * rb + 16 * (q0 + q) + acc_row<T>(g, e)) * NP + col];
#pragma unroll
            for (int q = 0; q < QB; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    Cr[q0 + q][e] = z[q][e].x - Cr[q0 + q][e];
                    Ci[q0 + q][e] = z[q][e].y - Ci[q0 + q][e];
                }
        }
    }
}

// Block row kb: workgroup t of a system forms U_kb,i of block column
// i = kb + 1 + t; the one with t = 0 goes on to diagonal block kb + 1 (its
// last operand), whose X the next launch needs, so that a step is one launch
// and the factorisation of the diagonal block runs beside the other tiles.
// FP64 matrix-core issue bounds it for many systems, the chain of the t = 0
// workgroup for few.  Factorisation of 256 systems of 1,024 loops (all steps):
// 8.2 ms where separate assembly, diagonal, panel and update launches after
// every 64 columns took 11.6, and 6.8 ms with the t = 0 workgroups dealt first
// and Z loaded in batches without branches; of 160 of 256 loops 0.43, 0.30 and
// now 0.26 ms.
template <typename T2, class Src>
__global__ __launch_bounds__(kTB, 2) void k_ldl_step(int NP, int S, Src src, int kb, int js, int T,
                                                     T2 *__restrict__ Aall, T2 *__restrict__ Xall,
                                                     double2 *__restrict__ Dall, int *__restrict__ fmt,
                                                     const double *__restrict__ zmax) {
    typedef typename Scal<T2>::type Ts;
    typedef typename Acc4<Ts>::type V4;
    __shared__ LdlLds m;
    int t;
    const int s = xcd_system_first(blockIdx.x, S, T, &t);
    if (s >= S) return;  // whole workgroup
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    if (tid == 0) m.flag = fmt[s];  // one read: the t = 0 workgroup may be marking the system
    __syncthreads();
    if (m.flag != kFmtLDL) return;  // whole workgroup
    const int ib = kb + 1 + t;
    T2 *A = Aall + (size_t)s * NP * NP;
    T2 *XT = Xall + (size_t)s * 64 * NP;
    double2 *D = Dall + (size_t)s * 2 * NP;
    for (int j = tid; j < 64 * (kb + 1 - js); j += kTB) {
        m.sd[j] = D[64 * js + j];
        if (t == 0) m.sy[j] = D[NP + 64 * js + j];
    }
    const SysRef sys = src.ref(s);
    if (t == 0 && js == 0 && tid < 64) m.sz[tid] = z_diag(sys, 64 * ib + tid);
    __syncthreads();
    {
        V4 Cr[4], Ci[4], Ur[4], Ui[4];
        double2 none = make_double2(0.0, 0.0);
        ldl_tile<T2, false, false>(NP, sys, kb, ib, js, 64 * kb, A, m.sd, nullptr, none, g, r16,
                                   wv, Cr, Ci);
        const T2 *X = XT + (size_t)kb * 64 * 64;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            Ur[rb] = Ui[rb] = V4{0, 0, 0, 0};
#pragma unroll
            for (int cb = 0; cb <= rb; ++cb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const T2 x = X[(16 * cb + acc_row<Ts>(g, e)) * 64 + 16 * rb + r16];
                    Ur[rb] = mfma4(x.x, Cr[cb][e], Ur[rb]);
                    Ui[rb] = mfma4(x.x, Ci[cb][e], Ui[rb]);
                    Ur[rb] = mfma4(-x.y, Ci[cb][e], Ur[rb]);
                    Ui[rb] = mfma4(x.y, Cr[cb][e], Ui[rb]);
                }
        }
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                T2 u;
                u.x = Ur[rb][e];
                u.y = Ui[rb][e];
                A[(size_t)(64 * kb + 16 * rb + acc_row<Ts>(g, e)) * NP + 64 * ib + 16 * wv + r16] = u;
            }
    }
    if (t != 0) return;  // whole workgroup
    __syncthreads();     // the rows of block kb are operands of the diagonal block
    DiagIn in;
    ldl_diag_load(NP, sys, ib, js, A, D, in);
    ldl_diag(NP, sys.n, s, in, ib, js, A, XT, D, fmt, zmax[s], m);
}

// After the super-panel of blocks js .. ns - 1: its rows subtracted from the
// tiles (r, c), ns <= r <= c, of the trailing matrix (all but the first
// diagonal tile, which the last step has taken care of), and from the
// right-hand side of the rows of the diagonal tiles.
template <typename T2, class Src>
__global__ __launch_bounds__(kTB, 3) void k_ldl_trail(int NP, int S, Src src, int js, int ns, int T,
                                                      T2 *__restrict__ Aall,
                                                      double2 *__restrict__ Dall,
                                                      const int *__restrict__ fmt) {
    typedef typename Scal<T2>::type Ts;
    typedef typename Acc4<Ts>::type V4;
    constexpr bool kY = sizeof(T2) == sizeof(double2);
    __shared__ double2 sd[64 * kSuper], sy[64 * kSuper];
    int t;
    const int s = xcd_system(blockIdx.x, T, &t);
    if (s >= S) return;  // whole workgroup
    if (fmt[s] != kFmtLDL) return;
    ++t;
    int tc = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
    while ((tc + 1) * (tc + 2) / 2 <= t) ++tc;
    while (tc * (tc + 1) / 2 > t) --tc;
    const int rb = ns + t - tc * (tc + 1) / 2, cb = ns + tc;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    T2 *A = Aall + (size_t)s * NP * NP;
    double2 *D = Dall + (size_t)s * 2 * NP;
    for (int j = tid; j < 64 * (ns - js); j += kTB) {
        sd[j] = D[64 * js + j];
        if (kY) sy[j] = D[NP + 64 * js + j];
    }
    const SysRef sys = src.ref(s);
    __syncthreads();
    V4 Cr[4], Ci[4];
    double2 yacc = make_double2(0.0, 0.0);
    ldl_tile<T2, true, kY>(NP, sys, rb, cb, js, 64 * ns, A, sd, sy, yacc, g, r16, wv, Cr, Ci);
    if (kY && rb == cb) {
        yacc.x += __shfl_xor(yacc.x, 16);
        yacc.y += __shfl_xor(yacc.y, 16);
        yacc.x += __shfl_xor(yacc.x, 32);
        yacc.y += __shfl_xor(yacc.y, 32);
        if (lane < 16) {
            const int k = 64 * cb + 16 * wv + r16;
            const double2 b = rhs_base(sys, k, js, D + NP);
            D[NP + k] = make_double2(b.x - yacc.x, b.y - yacc.y);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            T2 u;
            u.x = Cr[q][e];
            u.y = Ci[q][e];
            A[(size_t)(64 * rb + 16 * q + acc_row<Ts>(g, e)) * NP + 64 * cb + 16 * wv + r16] = u;
        }
}

// sx <- Z^-1 sx from the U, X, D^-1 record of one system (FWD: the sweep with
// L = U^T D^-1; BWD: the one with U), the vector in LDS, the kTS threads of the
// workgroup taking part, in blocks of 64 rows.  Forward: y_b = X_b t_b, then
// the rows of U_b times D^-1 y_b are taken off the rest of the vector, each
// wave 64 columns (fewer columns than waves: the 64 rows split over up to 16
// groups).  Backward: rows 4 w .. 4 w + 3 of the block against the solved
// entries per wave, x_b = X_b^T D^-1 (y_b - .).  Rows and X are loaded before
// the value they multiply is ready.  sred: kTS entries, sv: 64 entries of LDS.
//   Latency of the blocks bounds it for small NP (8 systems of 144 loops: 29
// us for both sweeps, 12 us for the backward one, where blocks of 16 rows
// against an explicit LU record took 110 and 79 us), the read of U per sweep
// for large NP (256 systems of 1,024: 720 and 364 us, 868 and 855 before;
// 2.1 GB per sweep).
template <typename T2, bool FWD, bool BWD>
__device__ __forceinline__ void ldl_apply_inverse(const T2 *__restrict__ U, const T2 *__restrict__ XT,
                                                  const double2 *__restrict__ dinv, int NP, double2 *sx,
                                                  double2 *sred, double2 *sv) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int nb = NP / 64;
    const double2 z = make_double2(0.0, 0.0);
    for (int b = 0; FWD && b < nb; ++b) {
        const T2 *X = XT + (size_t)b * 64 * 64;
        const int mb = nb - 1 - b;  // column blocks right of the diagonal
        const int kg = mb <= 1 ? 16 : mb == 2 ? 8 : mb <= 4 ? 4 : mb <= 8 ? 2 : 1;
        const int rows = 64 / kg;
        const bool act = wv < mb * kg;
        const int cbk = act ? wv % mb : 0, kgrp = act ? wv / mb : 0;
        const T2 *ub = U + (size_t)(64 * b + rows * kgrp) * NP + 64 * (b + (act ? 1 + cbk : 0)) + lane;
        T2 u[16], x[4];
        if (act) {
#pragma unroll
            for (int e = 0; e < 16; ++e) u[e] = ub[(size_t)(e < rows ? e : 0) * NP];
        }
        double2 acc = z;
        const bool low = (wv >> 2) <= (lane >> 4);  // X is lower triangular
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = X[(low ? (4 * wv + e) * 64 : 0) + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = zfma(acc, low ? ld2(x[e]) : z, sx[64 * b + 4 * wv + e]);
        sred[tid] = acc;
        __syncthreads();
        if (tid < 64) {
            double2 y = sred[tid];
#pragma unroll
            for (int e = 1; e < 16; ++e) {
                y.x += sred[64 * e + tid].x;
                y.y += sred[64 * e + tid].y;
            }
            sx[64 * b + tid] = y;
            sv[tid] = zmul(y, dinv[64 * b + tid]);
        }
        __syncthreads();
        if (mb == 0) break;  // uniform
        acc = z;
        if (act) {
            const double2 *v = sv + rows * kgrp;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (e < rows) acc = zfma(acc, ld2(u[e]), v[e]);
            for (int r0 = 16; r0 < rows; r0 += 16) {
#pragma unroll
                for (int e = 0; e < 16; ++e) u[e] = ub[(size_t)(r0 + e) * NP];
#pragma unroll
                for (int e = 0; e < 16; ++e) acc = zfma(acc, ld2(u[e]), v[r0 + e]);
            }
            sred[(kgrp * mb + cbk) * 64 + lane] = acc;
        }
        __syncthreads();
        if (tid < 64 * mb) {
            double2 t = sx[64 * (b + 1) + tid];
            for (int e = 0; e < kg; ++e) {
                t.x -= sred[e * 64 * mb + tid].x;
                t.y -= sred[e * 64 * mb + tid].y;
            }
            sx[64 * (b + 1) + tid] = t;
        }
        __syncthreads();
    }
    for (int b = nb - 1; BWD && b >= 0; --b) {
        const T2 *X = XT + (size_t)b * 64 * 64;
        const int mb = nb - 1 - b;
        const int c = tid >> 4, r16 = tid & 15;
        T2 x[4];  // X^T of column c (rows of block e >= c / 16)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = X[c * 64 + r16 + 16 * (e >= (c >> 4) ? e : 3)];
        const T2 *ub = U + (size_t)(64 * b + 4 * wv) * NP + 64 * (b + 1) + lane;
        double2 acc[4] = {z, z, z, z};
        for (int f = 0; f < mb; f += 3) {
            T2 u[3][4];
#pragma unroll
            for (int h = 0; h < 3; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    u[h][e] = ub[(size_t)e * NP + 64 * (f + h < mb ? f + h : f)];
#pragma unroll
            for (int h = 0; h < 3; ++h) {
                const double2 xv = f + h < mb ? sx[64 * (b + 1 + f + h) + lane] : z;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = zfma(acc[e], ld2(u[h][e]), xv);
            }
        }
        // sums over the lanes: 32-lane halves keep two rows each, 16-lane
        // quarters one, then the 16 lanes of each row
        const bool hi = lane & 32, odd = lane & 16;
        double2 p[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const double2 mine = hi ? acc[2 + e] : acc[e], give = hi ? acc[e] : acc[2 + e];
            p[e] = make_double2(mine.x + __shfl_xor(give.x, 32), mine.y + __shfl_xor(give.y, 32));
        }
        const double2 mine = odd ? p[1] : p[0], give = odd ? p[0] : p[1];
        double2 t = make_double2(mine.x + __shfl_xor(give.x, 16), mine.y + __shfl_xor(give.y, 16));
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) {
            t.x += __shfl_xor(t.x, off);
            t.y += __shfl_xor(t.y, off);
        }
        if (r16 == 0) {
            const int k = 4 * wv + 2 * (hi ? 1 : 0) + (odd ? 1 : 0);
            const double2 y = sx[64 * b + k];
            sv[k] = zmul(make_double2(y.x - t.x, y.y - t.y), dinv[64 * b + k]);
        }
        __syncthreads();
        double2 w = z;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            w = zfma(w, e >= (c >> 4) ? ld2(x[e]) : z, sv[r16 + 16 * e]);
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) {
            w.x += __shfl_xor(w.x, off);
            w.y += __shfl_xor(w.y, off);
        }
        if (r16 == 0) sx[64 * b + c] = w;
        __syncthreads();
    }
}

// sum of row[j] x[j] over j = j0, j0 + 64, ... < j1 (one lane of the wave
// that owns the row).  Rows have at most kMaxLoopsBig = 16 x 64 entries, so a
// lane has at most 16, loaded in two batches of 8 issued at once: the solves
// walk their blocks of rows one after another and each block is
// latency-bound; a batch is what fits the 128 registers a lane has in a
// 1,024-thread workgroup without spilling.
static_assert(kMaxLoopsBig <= kTS, "load_rhs: one thread per entry");
static_assert(kMaxLoopsBig <= 16 * 64, "at most 16 entries of a row per lane");
// Entries past j1 are loaded from column 0 (always inside the row) and both
// factors replaced by zero, so that the loads need no branches.
__device__ inline double2 dot_run(const double2 *__restrict__ row, const double2 *x, int j0, int j1) {
    constexpr int D = 8;
    const double2 z = make_double2(0.0, 0.0);
    double2 a0 = z, a1 = z;
#pragma unroll 1
    for (int e0 = 0; e0 < 16 && j0 + 64 * e0 < j1; e0 += D) {
        double2 v[D];
#pragma unroll
        for (int e = 0; e < D; ++e) {
            const int j = j0 + 64 * (e0 + e);
            v[e] = row[j < j1 ? j : 0];
        }
#pragma unroll
        for (int e = 0; e < D; e += 2) {
            const int j = j0 + 64 * (e0 + e);
            const bool in0 = j < j1, in1 = j + 64 < j1;
            a0 = zfma(a0, in0 ? v[e] : z, x[in0 ? j : 0]);
            a1 = zfma(a1, in1 ? v[e + 1] : z, x[in1 ? j + 64 : 0]);
        }
    }
    return make_double2(a0.x + a1.x, a0.y + a1.y);
}

// The same for a real row (a row of M) against a complex vector, in two
// batches of 8 loads.
__device__ inline double2 dot_real_run(const double *__restrict__ row, const double2 *x, int j0,
                                       int j1) {
    double r0 = 0.0, i0 = 0.0;
#pragma unroll 1
    for (int e0 = 0; e0 < 16 && j0 + 64 * e0 < j1; e0 += 8) {
        double v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = j0 + 64 * (e0 + e);
            v[e] = row[j < j1 ? j : 0];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = j0 + 64 * (e0 + e);
            const bool in = j < j1;
            const double m = in ? v[e] : 0.0;
            const double2 xv = x[in ? j : 0];
            r0 = fma(m, xv.x, r0);
            i0 = fma(m, xv.y, i0);
        }
    }
    return make_double2(r0, i0);
}

// Sum over the 64 lanes of a wave; every lane returns with it.
__device__ inline double2 wave_sum(double2 a) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        a.x += __shfl_xor(a.x, off);
        a.y += __shfl_xor(a.y, off);
    }
    return a;
}

// Right-hand side of system r into sx[0 .. NP): the loop voltage (forward) or
// rscale * conj(sum over chunks of (rr + j ri)) (adjoint; the chunks dealt to
// as many threads per entry as the workgroup has, added up through sred).
template <int RHS>
__device__ __forceinline__ void load_rhs(int NP, const SysRef &r, double2 *sx, double2 *sred) {
    const int tid = threadIdx.x;
    if (RHS == kRhsExcitation) {
        for (int k = tid; k < NP; k += kTS)
            sx[k] = k < r.n ? loop_voltage(r.phi, r.n, k, r.w) : make_double2(0.0, 0.0);
        return;
    }
    const double2 *part = (const double2 *)r.rhs + (size_t)r.s * NP;
    const int G = kTS / NP, k = tid % NP, c0 = tid / NP;  // NP <= kTS
    double2 a = make_double2(0.0, 0.0);
    if (c0 < G && k < r.n) {
#pragma unroll 4
        for (int c = c0; c < r.nchunk; c += G) {
            const double2 v = part[(size_t)c * r.S * NP + k];
            a.x += v.x;
            a.y += v.y;
        }
    }
    sred[tid] = a;
    __syncthreads();
    if (tid < NP) {
        for (int e = 1; e < G; ++e) {
            a.x += sred[e * NP + tid].x;
            a.y += sred[e * NP + tid].y;
        }
        sx[tid] = make_double2(r.rscale * a.x, -r.rscale * a.y);
    }
}

// sx <- U^-1 L^-1 P sx for one system's LU record A (unit lower L below the
// diagonal, U on and above it; the row swaps piv first), the vector
// in LDS, the kTS threads of the workgroup taking part: blocks of 16 rows,
// dot products against the solved rows (wave r takes row r of the block and
// stages its diagonal-block entries in LDS), then the 16x16 diagonal block
// inside wave 0.  st: 16 entries, sd: 16 x 17 entries of LDS scratch.
//   The blocks follow one another, so each block's loads of its rows are
// latency on the critical path.  With PF (rows of at most 64 kPf entries),
// the next block's row entries (kPf per lane) and diagonal-block entries are
// loaded while the current block's diagonal part is solved.  Swaps that move
// nothing are found by one vote and skipped.
constexpr int kPf = 4;
template <bool PF>
__device__ __forceinline__ void lu_apply_inverse(const double2 *__restrict__ A, const int *__restrict__ piv, int NP,
                                 double2 *sx, double2 *st, double2 (*sd)[17]) {
    const int tid = threadIdx.x;
    {
        int moved = 0;
        for (int j = tid; j < NP; j += kTS) moved |= piv[j] != j;
        if (__syncthreads_or(moved)) {
            if (tid == 0) {
                for (int j = 0; j < NP; ++j) {
                    const int p = piv[j];
                    if (p != j) {
                        const double2 t = sx[j];
                        sx[j] = sx[p];
                        sx[p] = t;
                    }
                }
            }
            __syncthreads();
        }
    }
    const int r = tid >> 6, q = tid & 63;
    const double2 z = make_double2(0.0, 0.0);
    // PF: entries j = j0 + 64 e (e < kPf) of row r0 + r inside [j0, j1)
    // (others from column 0, always inside the row, and zeroed when used),
    // and the diagonal-block entry of column r0 + (q & 15)
    double2 pf[kPf], pd;
    auto fetch = [&](int r0, int j0, int j1) {
        const double2 *row = A + (size_t)(r0 + r) * NP;
#pragma unroll
        for (int e = 0; e < kPf; ++e) {
            const int j = j0 + 64 * e;
            pf[e] = row[j < j1 ? j : 0];
        }
        pd = row[r0 + (q & 15)];
    };
    // row r0 + r against sx over [j0, j1) (PF: the prefetched entries)
    auto dot = [&](int r0, int j0, int j1) {
        double2 acc = z;
        if constexpr (PF) {
#pragma unroll
            for (int e = 0; e < kPf; ++e) {
                const int j = j0 + 64 * e;
                const bool in = j < j1;
                acc = zfma(acc, in ? pf[e] : z, sx[in ? j : 0]);
            }
        } else {
            acc = dot_run(A + (size_t)(r0 + r) * NP, sx, j0, j1);
        }
        return wave_sum(acc);
    };
    auto diag_entry = [&](int r0) {
        if constexpr (PF)
            return pd;
        else
            return A[(size_t)(r0 + r) * NP + r0 + (q & 15)];
    };
    // forward: L y = P b, L unit lower; block r0 uses columns [0, r0)
    if (PF) fetch(0, q, 0);
    for (int r0 = 0; r0 < NP; r0 += 16) {
        if (q < 16) sd[r][q] = diag_entry(r0);
        const double2 acc = dot(r0, q, r0);
        if (PF && r0 + 16 < NP) fetch(r0 + 16, q, r0 + 16);  // in flight across the diagonal block
        if (q == 0) st[r] = make_double2(sx[r0 + r].x - acc.x, sx[r0 + r].y - acc.y);
        __syncthreads();
        if (tid < 64) {
            const int l = tid & 15;
            double2 t = st[l];
#pragma unroll
            for (int k = 0; k < 15; ++k) {
                const double2 yk = make_double2(__shfl(t.x, k), __shfl(t.y, k));
                const double2 lk = l > k ? sd[l][k] : make_double2(0.0, 0.0);
                t = zfms(t, lk, yk);
            }
            if (tid < 16) sx[r0 + l] = t;
        }
        __syncthreads();
    }
    // backward: U x = y; block r0 uses columns [r0 + 16, NP)
    if (PF) fetch(NP - 16, NP + q, NP);
    for (int r0 = NP - 16; r0 >= 0; r0 -= 16) {
        if (q < 16) sd[r][q] = diag_entry(r0);
        const double2 acc = dot(r0, r0 + 16 + q, NP);
        if (PF && r0 >= 16) fetch(r0 - 16, r0 + q, NP);
        if (q == 0) st[r] = make_double2(sx[r0 + r].x - acc.x, sx[r0 + r].y - acc.y);
        __syncthreads();
        if (tid < 64) {
            const int l = tid & 15;
            double2 t = st[l];
#pragma unroll
            for (int k = 15; k >= 0; --k) {
                // lane k finishes x_k; the lanes of the rows above subtract its term
                if (l == k) t = zmul(t, zinv(sd[k][k]));
                const double2 xk = make_double2(__shfl(t.x, k), __shfl(t.y, k));
                const double2 uk = l < k ? sd[l][k] : make_double2(0.0, 0.0);
                t = zfms(t, uk, xk);
            }
            if (tid < 16) sx[r0 + l] = t;
        }
        __syncthreads();
    }
}

// Outputs of a solved system: forward I[s][k]; adjoint gsys[s][k] =
// 2 Re(mu_k I_k / (j w C_k^2)) (and mu when asked for); status bits.
template <int RHS>
__device__ __forceinline__ void write_solution(const SysRef &r, const double2 *sx, int *sFlag) {
    const int tid = threadIdx.x;
    const int n = r.n, s = r.s;
    const double w = r.w;
    const double *__restrict__ Cb = r.Cb;
    double2 *__restrict__ I = r.I;
    double *__restrict__ gsys = r.gsys;
    double2 *__restrict__ mu = r.mu;
    int32_t *__restrict__ status = r.status;
    const int flag = status[s];
    const bool bad = (flag & (COSIM_SYS_BAD_INPUT | COSIM_SYS_SINGULAR)) != 0;
    int oflag = 0;
    for (int k = tid; k < n; k += kTS) {
        double2 x = sx[k];
        if (bad) x = make_double2(__builtin_nan(""), __builtin_nan(""));
        if (RHS == kRhsExcitation) {
            I[(size_t)s * n + k] = x;
            if (!bad && !(isfinite(x.x) && isfinite(x.y))) oflag = COSIM_SYS_NONFINITE;
        } else {
            const double2 Ik = I[(size_t)s * n + k];
            const double ck = Cb[k];
            // 2 Re(mu I / (j w C^2)) = 2 Im(mu I) / (w C^2)
            const double g = 2.0 * (x.x * Ik.y + x.y * Ik.x) / (w * ck * ck);
            gsys[(size_t)s * n + k] = g;
            if (mu) mu[(size_t)s * n + k] = x;
            if (!bad && !isfinite(g)) oflag = COSIM_SYS_NONFINITE;
        }
    }
    if (oflag) atomicOr(sFlag, oflag);
    __syncthreads();
    if (tid == 0 && *sFlag) status[s] = flag | *sFlag;
}

// One workgroup per system (only those with only[s] == want when `only` is
// set): right-hand side, the triangular solves with the FP64 record, outputs.
// Systems whose fmt is kFmtLDL hold a U, X, D^-1 record, and the forward solve
// starts from the y that the factorisation left (its backward sweep only);
// the others hold a pivoted LU.
template <int RHS, class Src>
__global__ __launch_bounds__(kTS) void k_big_solve(int NP, int S, Src src,
                                                   const double2 *__restrict__ Aall,
                                                   const int *__restrict__ pivall,
                                                   const double2 *__restrict__ Xall,
                                                   const double2 *__restrict__ Dall,
                                                   const int *__restrict__ fmt,
                                                   const int *__restrict__ only, int want) {
    __shared__ double2 sx[kMaxLoopsBig];
    __shared__ double2 sred[kTS];
    __shared__ double2 st[64];
    __shared__ double2 sd[16][17];
    __shared__ int sFlag;
    const int s = blockIdx.x;
    if (s >= S) return;
    if (only && only[s] != want) return;
    const int tid = threadIdx.x;
    const SysRef r = src.ref(s);
    const double2 *A = Aall + (size_t)s * NP * NP;
    if (tid == 0) sFlag = 0;
    const bool ldl = fmt && fmt[s] == kFmtLDL;  // uniform
    if (ldl) {
        const double2 *XT = Xall + (size_t)s * 64 * NP, *D = Dall + (size_t)s * 2 * NP;
        if (RHS == kRhsExcitation) {
            if (tid < NP) sx[tid] = D[NP + tid];
            __syncthreads();
            ldl_apply_inverse<double2, false, true>(A, XT, D, NP, sx, sred, st);
        } else {
            load_rhs<RHS>(NP, r, sx, sred);
            __syncthreads();
            ldl_apply_inverse<double2, true, true>(A, XT, D, NP, sx, sred, st);
        }
    } else {
        load_rhs<RHS>(NP, r, sx, sred);
        __syncthreads();
        if (NP <= 64 * kPf)  // uniform over the launch
            lu_apply_inverse<true>(A, pivall + (size_t)s * NP, NP, sx, st, sd);
        else
            lu_apply_inverse<false>(A, pivall + (size_t)s * NP, NP, sx, st, sd);
    }
    write_solution<RHS>(r, sx, &sFlag);
}

// Largest of a and b over the kTS threads, NaN taken as +inf; every thread
// returns with both.  sm: 2 kTS/64 entries of LDS scratch.
__device__ inline void block_max2(double &a, double &b, double *sm) {
    if (!(a == a)) a = __builtin_inf();
    if (!(b == b)) b = __builtin_inf();
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        a = fmax(a, __shfl_xor(a, off));
        b = fmax(b, __shfl_xor(b, off));
    }
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sm[2 * wv] = a;
        sm[2 * wv + 1] = b;
    }
    __syncthreads();
    a = sm[0];
    b = sm[1];
#pragma unroll
    for (int v = 1; v < kTS / 64; ++v) {
        a = fmax(a, sm[2 * v]);
        b = fmax(b, sm[2 * v + 1]);
    }
    __syncthreads();
}

// Refined solve of the systems factored in FP32 (fmt kFmtLDL, record A32 of
// the blocked LDL^T): x = F^-1 b, then up to max_iter times
//   r = b - Z x   in FP64: (R_k - j/(w C_k)) x_k + j w (M x)_k, rows of M read
//                 by 16 threads each as in the triangular solves;
//   d = F^-1 r,   x += d.
// With d_0 = x_0 the corrections shrink geometrically by about
// |d_i| / |d_(i-1)|, so the error left after step i is estimated as
// |d_i|^2 / |d_(i-1)|; the system is done once that is at most tol |x| and
// |d_i| <= |d_(i-1)| / 2 (max norms).  A system that is not done after
// max_iter steps is marked fail_fmt, writes nothing and is left to the
// pivoted FP64 fallback.
template <int RHS>
__global__ __launch_bounds__(kTS) void k_solve_refined(int NP, int S, OneInst src,
                                                       const float2 *__restrict__ A32all,
                                                       const float2 *__restrict__ Xall,
                                                       const double2 *__restrict__ Dall,
                                                       int *__restrict__ fmt, int fail_fmt,
                                                       int max_iter, double tol) {
    __shared__ double2 sb[kMaxLoopsBig];
    __shared__ double2 sx[kMaxLoopsBig];
    __shared__ double2 sr[kMaxLoopsBig];
    __shared__ double2 sred[kTS];
    __shared__ double2 st[64];
    __shared__ double sm[2 * (kTS / 64)];
    __shared__ int sFlag;
    const int s = blockIdx.x;
    if (s >= S) return;
    if (fmt[s] != kFmtLDL) return;  // whole workgroup: handled by the FP64 record
    const int tid = threadIdx.x;
    const SysRef sys = src.ref(s);
    const int n = sys.n;
    const double w = sys.w;
    const double *__restrict__ M = sys.M;
    const double *__restrict__ Rv = sys.R;
    const double *__restrict__ Cb = sys.Cb;
    const float2 *A = A32all + (size_t)s * NP * NP;
    const float2 *XT = Xall + (size_t)s * 64 * NP;
    const double2 *D = Dall + (size_t)s * 2 * NP;
    load_rhs<RHS>(NP, sys, sr, sred);
    __syncthreads();
    for (int k = tid; k < NP; k += kTS) sb[k] = sr[k];
    if (tid == 0) sFlag = 0;
    __syncthreads();
    const int r = tid >> 6, q = tid & 63;  // wave r takes row r0 + r of each block
    bool done = false;
    double prev = 0.0;
    // step 0 solves for x_0 (d_0 = x_0); step i >= 1 for the correction d_i
    for (int it = 0; it <= max_iter; ++it) {
        ldl_apply_inverse<float2, true, true>(A, XT, D, NP, sr, sred, st);
        double dm = 0.0, xm = 0.0;
        for (int k = tid; k < NP; k += kTS) {
            const double2 d = sr[k];
            double2 x = it == 0 ? make_double2(0.0, 0.0) : sx[k];
            x.x += d.x;
            x.y += d.y;
            sx[k] = x;
            dm = fmax(dm, fabs(d.x) + fabs(d.y));
            xm = fmax(xm, fabs(x.x) + fabs(x.y));
            if (!(d.x == d.x && d.y == d.y)) dm = __builtin_inf();
        }
        block_max2(dm, xm, sm);  // also orders the x updates before the residual
        if (it > 0) done = dm < __builtin_inf() && dm * dm <= tol * xm * prev && dm <= 0.5 * prev;
        prev = dm;
        if (done || it == max_iter) break;
        // r = b - Z x
        for (int r0 = 0; r0 < NP; r0 += 16) {
            const int i = r0 + r;
            double2 acc = make_double2(0.0, 0.0);
            if (i < n) acc = dot_real_run(M + (size_t)i * n, sx, q, n);
            acc = wave_sum(acc);
            if (q == 0) {
                double2 v = make_double2(0.0, 0.0);
                if (i < n) {
                    const double2 xi = sx[i], bi = sb[i];
                    const double zr = Rv[i], zi = -1.0 / (w * Cb[i]);
                    // b - z_ii x_i - j w (M x)_i
                    v.x = bi.x - (zr * xi.x - zi * xi.y) + w * acc.y;
                    v.y = bi.y - (zr * xi.y + zi * xi.x) - w * acc.x;
                }
                sr[i] = v;
            }
        }
        __syncthreads();
    }
    if (!done) {
        if (tid == 0) fmt[s] = fail_fmt;
        return;  // whole workgroup
    }
    write_solution<RHS>(sys, sx, &sFlag);
}

}  // namespace

namespace {

OneInst one_inst(int n, int F, int S, const double *M, const double *R, const double *phi,
                 const double *C, const double *omega, double2 *I, const void *rhs, int nchunk,
                 double rscale, double *gsys, double2 *mu, int32_t *status) {
    OneInst o;
    o.M = M;
    o.R = R;
    o.phi = phi;
    o.C = C;
    o.omega = omega;
    o.I = I;
    o.rhs = rhs;
    o.gsys = gsys;
    o.mu = mu;
    o.status = status;
    o.n = n;
    o.F = F;
    o.S = S;
    o.nchunk = nchunk;
    o.rscale = rscale;
    return o;
}

template <class Src>
hipError_t lu_big_launch(int NP, int S, const Src &src, double2 *A_d, int *piv_d,
                         const int *only, int want, hipStream_t st) {
    if (only)
        hipLaunchKernelGGL((k_lu_big<true, Src>), dim3(S), dim3(kTB), 0, st, NP, S, src, A_d, piv_d,
                           only, want);
    else
        hipLaunchKernelGGL((k_lu_big<false, Src>), dim3(S), dim3(kTB), 0, st, NP, S, src, A_d, piv_d,
                           only, want);
    return hipGetLastError();
}

// Blocked LDL^T of the S systems in the storage type T2 (invalid input and
// small pivots are marked in fmt and left to the pivoted LU).
template <typename T2, class Src>
hipError_t blocked_ldl(const BigFactor &bf, int NP, int S, const Src &src, T2 *A_d, hipStream_t st) {
    T2 *X = (T2 *)bf.x;
    const int nb = NP / 64;
    hipLaunchKernelGGL((k_ldl_start<T2, Src>), dim3(S), dim3(kTB), 0, st, NP, S, src, A_d, X, bf.d,
                       bf.fmt, bf.zmax);
    hipError_t e = hipGetLastError();
    for (int kb = 0; e == hipSuccess && kb + 1 < nb; ++kb) {
        const int js = kb / kSuper * kSuper, T = nb - 1 - kb;
        hipLaunchKernelGGL((k_ldl_step<T2, Src>), dim3(8 * ((S + 7) / 8) * T), dim3(kTB), 0, st, NP,
                           S, src, kb, js, T, A_d, X, bf.d, bf.fmt, (const double *)bf.zmax);
        if ((e = hipGetLastError()) != hipSuccess) break;
        const int ns = js + kSuper;
        if (kb + 1 < ns || ns + 1 >= nb) continue;
        const int nt = nb - ns, Tt = nt * (nt + 1) / 2 - 1;
        hipLaunchKernelGGL((k_ldl_trail<T2, Src>), dim3(8 * ((S + 7) / 8) * Tt), dim3(kTB), 0, st, NP,
                           S, src, js, ns, Tt, A_d, bf.d, (const int *)bf.fmt);
        e = hipGetLastError();
    }
    return e;
}

template <class Src>
hipError_t big_solve_any(int rhs_kind, const BigFactor &bf, int NP, int S, const Src &src,
                         const double2 *A_d, const int *piv_d, const int *only, int want,
                         hipStream_t st) {
    const int *fmt = bf.ldl && !only ? bf.fmt : nullptr;
    const double2 *X = bf.x, *D = bf.d;
    if (rhs_kind == kRhsExcitation)
        hipLaunchKernelGGL((k_big_solve<kRhsExcitation, Src>), dim3(S), dim3(kTS), 0, st, NP, S, src,
                           A_d, piv_d, X, D, fmt, only, want);
    else
        hipLaunchKernelGGL((k_big_solve<kRhsPairs, Src>), dim3(S), dim3(kTS), 0, st, NP, S, src, A_d,
                           piv_d, X, D, fmt, only, want);
    return hipGetLastError();
}

hipError_t refined_any(int rhs_kind, const BigFactor &bf, const BigRefine &rf, int NP, int S,
                       const OneInst &src, int fail_fmt, hipStream_t st) {
    const float2 *X = (const float2 *)bf.x;
    const double2 *D = bf.d;
    if (rhs_kind == kRhsExcitation)
        hipLaunchKernelGGL(k_solve_refined<kRhsExcitation>, dim3(S), dim3(kTS), 0, st, NP, S, src,
                           (const float2 *)rf.A32, X, D, bf.fmt, fail_fmt, rf.max_iter, rf.tol);
    else
        hipLaunchKernelGGL(k_solve_refined<kRhsPairs>, dim3(S), dim3(kTS), 0, st, NP, S, src,
                           (const float2 *)rf.A32, X, D, bf.fmt, fail_fmt, rf.max_iter, rf.tol);
    return hipGetLastError();
}

}  // namespace

hipError_t big_factor(const BigFactor &bf, const BigRefine &rf, int NP, int n, int S, int F,
                      const double *M_d, const double *R_d, const double *phi_d, const double *C_d,
                      const double *omega_d, double2 *A_d, int *piv_d, int32_t *status_d,
                      hipStream_t st) {
    if (NP % 64 != 0 || NP > kMaxLoopsBig) return hipErrorInvalidValue;
    const OneInst src = one_inst(n, F, S, M_d, R_d, phi_d, C_d, omega_d, nullptr, nullptr, 0,
                                 0.0, nullptr, nullptr, status_d);
    if (!bf.ldl) return lu_big_launch(NP, S, src, A_d, piv_d, nullptr, 0, st);
    if (!bf.fmt || !bf.zmax || !bf.x || !bf.d) return hipErrorInvalidValue;
    if (rf.on && !rf.A32) return hipErrorInvalidValue;
    hipError_t e = rf.on ? blocked_ldl<float2>(bf, NP, S, src, (float2 *)rf.A32, st)
                         : blocked_ldl<double2>(bf, NP, S, src, A_d, st);
    if (e != hipSuccess) return e;
    // pivoted FP64 LU (from a fresh Z) for the systems marked on the way
    return lu_big_launch(NP, S, src, A_d, piv_d, bf.fmt, kFmtNeedsPivot, st);
}

hipError_t big_solve(const BigFactor &bf, const BigRefine &rf, int NP, int n, int S, int F,
                     const double *M_d, const double *R_d, const double *phi_d, const double *C_d,
                     const double *omega_d, double2 *A_d, int *piv_d, double2 *I_d, int rhs_kind,
                     const void *rhs_d, int nchunk, double rscale, double *gsys_d,
                     int32_t *status_d, hipStream_t st, double2 *mu_d) {
    if (NP % 64 != 0 || NP > kMaxLoopsBig) return hipErrorInvalidValue;
    const OneInst src = one_inst(n, F, S, M_d, R_d, phi_d, C_d, omega_d, I_d, rhs_d, nchunk,
                                 rscale, gsys_d, mu_d, status_d);
    if (!(bf.ldl && rf.on))
        return big_solve_any(rhs_kind, bf, NP, S, src, A_d, piv_d, nullptr, 0, st);
    const bool fwd = rhs_kind == kRhsExcitation;
    const int fail = fwd ? kFmtRefineFailed : kFmtRefineFailedAdj;
    hipError_t e;
    // 1. the FP32 records, refined
    if ((e = refined_any(rhs_kind, bf, rf, NP, S, src, fail, st)) != hipSuccess) return e;
    // 2. systems that already hold an FP64 record
    const int have[2] = {kFmtNeedsPivot, kFmtRefineFailed};
    for (int h = 0; h < (fwd ? 1 : 2); ++h)
        if ((e = big_solve_any(rhs_kind, bf, NP, S, src, A_d, piv_d, bf.fmt, have[h], st)) != hipSuccess)
            return e;
    // 3. systems whose refinement did not converge just now: pivoted FP64
    // record from a fresh Z, then the FP64 solve
    if ((e = lu_big_launch(NP, S, src, A_d, piv_d, bf.fmt, fail, st)) != hipSuccess) return e;
    return big_solve_any(rhs_kind, bf, NP, S, src, A_d, piv_d, bf.fmt, fail, st);
}

hipError_t big_group_factor(const BigFactor &bf, const GroupArgs &g, int NP, int S,
                            double2 *A_d, int *piv_d, hipStream_t st) {
    if (NP % 64 != 0 || NP > kMaxLoopsBig || g.count < 1 || g.count > kGroupMax || !bf.fmt ||
        !bf.zmax || !bf.x || !bf.d)
        return hipErrorInvalidValue;
    const GroupSrc src{g};
    hipError_t e = blocked_ldl<double2>(bf, NP, S, src, A_d, st);
    if (e != hipSuccess) return e;
    return lu_big_launch(NP, S, src, A_d, piv_d, bf.fmt, kFmtNeedsPivot, st);
}

hipError_t big_group_solve(const BigFactor &bf, const GroupArgs &g, int NP, int S,
                           const double2 *A_d, const int *piv_d, int rhs_kind, hipStream_t st) {
    if (NP % 64 != 0 || NP > kMaxLoopsBig || g.count < 1 || g.count > kGroupMax)
        return hipErrorInvalidValue;
    const GroupSrc src{g};
    return big_solve_any(rhs_kind, bf, NP, S, src, A_d, piv_d, nullptr, 0, st);
}

}  // namespace cosim
