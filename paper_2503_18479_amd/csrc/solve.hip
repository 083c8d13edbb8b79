// Batched FP64 complex solves of the loop impedance system (Eq. 6 in
// impedance form, Eq. 2 and 11 for Z) on gfx950.
//
// One workgroup per (configuration, frequency) system.  Z (NP x NP complex,
// NP = n padded to 16/32/64 with an identity block) lives in registers: thread
// (ti, tj) owns the 4x4 tile Z[4ti..4ti+3][4tj..4tj+3]; the NT threads of a
// column of tiles (a "column group") are consecutive lanes of one wave.
// Gauss-Jordan elimination with partial pivoting (pivot = largest |re|+|im|
// among rows not yet used; rows are never swapped) eliminates each column from
// every other row, so the solution is read off at the end as
// x_k = b'_{p_k} / pivot_k with no back substitution.  Columns are processed
// in panels of 4 (see k_gj); the right-hand side is carried by the column
// group holding column n-1.  Z is complex symmetric (M symmetric, R and C
// diagonal), so the same routine serves the adjoint system Z^T mu = r.
#include <type_traits>

#include "internal.h"
#include "ldl_block.h"

namespace cosim {

namespace {

__device__ inline double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline double2 cinv(double2 a) {
    const double d = 1.0 / (a.x * a.x + a.y * a.y);
    return make_double2(a.x * d, -a.y * d);
}
// 1/a for a pivot known to be a normal, finite number away from zero or
// flagged afterwards: hardware reciprocal and two Newton steps (relative error
// at the level of the rounding of the result), no IEEE division sequence.
__device__ inline double rcp_nr(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    r = fma(r, fma(-x, r, 1.0), r);
    return r;
}
__device__ inline double2 cinv_nr(double2 a) {
    const double d = rcp_nr(fma(a.x, a.x, a.y * a.y));
    return make_double2(a.x * d, -a.y * d);
}

template <int NP>
struct GJShape {
    static constexpr int NT = NP / 4;
    static constexpr int NTHR = NT * NT;
    static constexpr int BLOCK = NTHR < 64 ? 64 : NTHR;
};

// acc - l*u with explicit fused multiply-adds (4 per complex product)
__device__ inline double2 cfms(double2 acc, double2 l, double2 u) {
    double2 r;
    r.x = fma(-l.x, u.x, fma(l.y, u.y, acc.x));
    r.y = fma(-l.x, u.y, fma(-l.y, u.x, acc.y));
    return r;
}

template <int CTRL>
__device__ inline int dpp_i(int x) {
    return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
}

// (magnitude, row) arg-max step with a DPP partner; ties -> lower row
template <int CTRL>
__device__ inline void amax_step(float &m, int &idx) {
    const float m2 = __int_as_float(dpp_i<CTRL>(__float_as_int(m)));
    const int i2 = dpp_i<CTRL>(idx);
    const bool take = (m2 > m) || (m2 == m && i2 < idx);
    m = take ? m2 : m;
    idx = take ? i2 : idx;
}

// arg-max over the NT lanes of a column group (NT = 4, 8 or 16 consecutive
// lanes inside one DPP row); every lane of the group ends with the result
template <int NT>
__device__ inline void group_amax(float &m, int &idx) {
    amax_step<0xB1>(m, idx);                    // quad_perm [1,0,3,2]
    amax_step<0x4E>(m, idx);                    // quad_perm [2,3,0,1]
    if (NT >= 8) amax_step<0x141>(m, idx);      // row_half_mirror
    if (NT >= 16) amax_step<0x140>(m, idx);     // row_mirror
}

// value of a double held by lane `src` (wave-uniform index) for every lane
__device__ inline double readlane_d(double x, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), src);
    return __hiloint2double(hi, lo);
}

// ADJ = false: rhs = E - j w Phi (loop_voltage), writes I[s][k].
// ADJ = true : rhs = rscale * sum_c (rr - j ri) of rpart[c][s][:], writes
//              gsys[s][k] = 2 Re(mu_k I_k / (j w C_k^2)).
//
// Blocked Gauss-Jordan, panels of 4 columns.  Panel kt is owned by the lane
// group tj == kt, which runs the four pivot steps on its own 4 columns
// (arg-max by DPP, pivot-row entries by readlane, no barrier) and
// publishes the multiplier columns l_c (c = 0..3) and pivot rows p_c through
// LDS.  After one block barrier every other column group applies the
// composite rank-4 update  a_ij -= sum_c l_c[i] u_cj  with
//   u_cj = a_{p_c j} - sum_{c' < c} l_{c'}[p_c] u_{c' j}
// (the pivot row of step c as it stands after steps c' < c), i.e. u = W a_p
// with W = (I + N)^-1, N[c][c'] = l_{c'}[p_c]; the panel group publishes W.
// Column groups left of the panel hold only eliminated columns and skip the
// update.
// One system s (block-uniform) of a plan with n loops, S systems, F
// frequencies; the kernels below call it for their own system index.
template <int NP>
struct GjLds {
    static constexpr int NT = GJShape<NP>::NT;
    double2 sL[2][4][NP];      // multiplier columns of a panel
    int sP[2][4];              // pivot rows of a panel
    double2 sPiv[NP];
    int sKof[NP];
    double2 sU[NT][4][4][4];   // [group][step c][row in tile][col in tile]
    double2 sUu[NT][4][4];     // [group][step c][col in tile]: u_c of the group's columns
    double2 sW[2][4][4];       // W = (I + N)^-1, N[c][c'] = l_c'[p_c] (c' < c)
    double2 sRb[4][4];         // rhs tiles of the pivot-row owners
    int sFlag;
};
template <int NP, bool ADJ>
__device__ __forceinline__ void gj_system(
    GjLds<NP> &lds, int s, int n, int S, int F, const double *__restrict__ M, const double *__restrict__ Rv,
    const double *__restrict__ phi, const double *__restrict__ C,
    const double *__restrict__ omega, const double2 *__restrict__ Iin,
    const double2 *__restrict__ rpart, int nchunk, double rscale, double2 *__restrict__ Iout,
    double *__restrict__ gsys, int32_t *__restrict__ status, bool or_status,
    GJFactor fac, bool fallback_only) {
    constexpr int NT = GJShape<NP>::NT;
    constexpr int NTHR = GJShape<NP>::NTHR;
    // fallback launch: only systems the LDL^T fast path handed over
    if (fallback_only && fac.fmt[s] != kFmtNeedsPivot) return;  // uniform per block
    const int t = threadIdx.x;
    const bool act = t < NTHR;
    const int ti = t % NT, tj = t / NT;
    const int b = s / F, f = s - b * F;

    auto &sL = lds.sL;
    auto &sP = lds.sP;
    auto &sPiv = lds.sPiv;
    auto &sKof = lds.sKof;
    auto &sU = lds.sU;
    auto &sUu = lds.sUu;
    auto &sW = lds.sW;
    auto &sRb = lds.sRb;
    int &sFlag = lds.sFlag;

    if (t == 0) sFlag = 0;
    __syncthreads();

    const double w = omega[f];
    const double *Cb = C + (size_t)b * n;
    const int tb = (n - 1) >> 2;  // column group that carries the rhs

    // ---- build the tile of Z and the rhs ---------------------------------
    double2 a[4][4];
    double2 rhs[4];
    if (act) {
        int flag = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * ti + r;
            double dre = 0.0, dim = 0.0;
            if (i < n) {
                const double c = Cb[i];
                if (tj == 0) {
                    if (isnan(c) || c == 0.0 || !isfinite(w) || w == 0.0) flag |= COSIM_SYS_BAD_INPUT;
                    else if (c < 0.0) flag |= COSIM_SYS_NEGATIVE_C;
                }
                dre = Rv[i];
                dim = -1.0 / (w * c);  // 1/(j w C) = -j/(w C)
            }
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const int j = 4 * tj + cc;
                double2 z = make_double2(0.0, 0.0);
                if (i < n && j < n) {
                    z.y = w * M[(size_t)i * n + j];
                    if (i == j) {
                        z.x += dre;
                        z.y += dim;
                    }
                } else if (i == j) {
                    z.x = 1.0;  // identity padding
                }
                a[r][cc] = z;
            }
            rhs[r] = make_double2(0.0, 0.0);
            if (tj == tb && i < n) {
                if (!ADJ) {
                    rhs[r] = loop_voltage(phi, n, i, w);
                } else {
                    double rr = 0.0, ri = 0.0;
                    for (int c = 0; c < nchunk; ++c) {
                        const double2 v = rpart[((size_t)c * S + s) * NP + i];
                        rr += v.x;
                        ri += v.y;
                    }
                    rhs[r] = make_double2(rscale * rr, -rscale * ri);
                }
            }
        }
        if (flag) atomicOr(&sFlag, flag);
    }

    // ---- elimination, one panel of 4 columns per iteration ------------------
    uint64_t used = 0;
    for (int kt = 0; 4 * kt < n; ++kt) {
        const int buf = kt & 1;
        const int nc = min(4, n - 4 * kt);  // real columns in this panel
        // -- panel factorisation by the owning column group
        if (act && tj == kt) {
            // first lane of this column group (the group is the only active one here)
            const int gbase = __builtin_amdgcn_readfirstlane((int)(threadIdx.x & 63));
            int pc[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                pc[c] = 0;
                if (c >= nc) continue;  // uniform
                // pivot search on |re| + |im| rounded to float: any near-maximal
                // pivot is as good, and the float arg-max needs 2 DPP moves per round
                float best = -1.0f;
                int bi = 1 << 30;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 4 * ti + r;
                    if (i < n && !((used >> i) & 1ull)) {
                        float m = (float)(fabs(a[r][c].x) + fabs(a[r][c].y));
                        if (!(m == m)) m = __builtin_inff();  // NaN rows still yield a pivot
                        if (m > best) {
                            best = m;
                            bi = i;
                        }
                    }
                }
                group_amax<NT>(best, bi);
                // the group's lanes agree on the pivot: make it wave-uniform; an unused
                // valid row always exists and the clamp keeps the index in range
                int p = __builtin_amdgcn_readfirstlane(bi);
                p = p < n ? p : n - 1;
                const int pr = p & 3;
                const int src = gbase + (p >> 2);  // lane holding row p
                auto rowsel = [&](int cc, bool im) {
                    const double v0 = im ? a[0][cc].y : a[0][cc].x, v1 = im ? a[1][cc].y : a[1][cc].x;
                    const double v2 = im ? a[2][cc].y : a[2][cc].x, v3 = im ? a[3][cc].y : a[3][cc].x;
                    return pr == 0 ? v0 : (pr == 1 ? v1 : (pr == 2 ? v2 : v3));
                };
                const double2 piv = make_double2(readlane_d(rowsel(c, false), src),
                                                 readlane_d(rowsel(c, true), src));
                const bool sing = !(piv.x != 0.0 || piv.y != 0.0);
                const double2 inv = sing ? make_double2(0.0, 0.0) : cinv(piv);
                double2 l[4];
                double2 *lcol = fac.L ? fac.L + ((size_t)s * NP + 4 * kt + c) * NP : nullptr;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 4 * ti + r;
                    l[r] = (i == p) ? make_double2(0.0, 0.0) : cmul(a[r][c], inv);
                    sL[buf][c][i] = l[r];
                    if (lcol) lcol[i] = l[r];
                }
                // remaining panel columns: a_ic' -= l_i a_pc'
#pragma unroll
                for (int c2 = c + 1; c2 < 4; ++c2) {
                    const double2 up = make_double2(readlane_d(rowsel(c2, false), src),
                                                    readlane_d(rowsel(c2, true), src));
#pragma unroll
                    for (int r = 0; r < 4; ++r) a[r][c2] = cfms(a[r][c2], l[r], up);
                }
                used |= 1ull << p;
                pc[c] = p;
                if (ti == 0) {
                    sPiv[4 * kt + c] = piv;
                    sKof[p] = 4 * kt + c;
                    if (sing) atomicOr(&sFlag, COSIM_SYS_SINGULAR);
                    if (fac.L) {
                        fac.piv_row[(size_t)s * NP + 4 * kt + c] = p;
                        fac.piv_val[(size_t)s * NP + 4 * kt + c] = piv;
                    }
                }
            }
            if (ti == 0) {
#pragma unroll
                for (int c = 0; c < 4; ++c) sP[buf][c] = pc[c];
            }
            // W = (I + N)^-1 (unit lower triangular) so that the pivot rows as
            // they stand at their own step are u = W a_p (a_p: rows before the panel)
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (ti == 0) {
                double2 N[4][4], Wm[4][4];
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int c2 = 0; c2 < 4; ++c2) {
                        N[c][c2] = (c2 < c && c < nc) ? sL[buf][c2][pc[c]] : make_double2(0.0, 0.0);
                        Wm[c][c2] = make_double2(c == c2 ? 1.0 : 0.0, 0.0);
                    }
#pragma unroll
                for (int c = 1; c < 4; ++c)
#pragma unroll
                    for (int c2 = 0; c2 < c; ++c2) {
                        double2 v = make_double2(0.0, 0.0);
#pragma unroll
                        for (int c3 = c2; c3 < c; ++c3) v = cfms(v, N[c][c3], Wm[c3][c2]);
                        Wm[c][c2] = v;
                    }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int c2 = 0; c2 < 4; ++c2) sW[buf][c][c2] = Wm[c][c2];
            }
            if (nc < 4) {  // unused steps of a ragged last panel contribute nothing
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c >= nc)
#pragma unroll
                        for (int r = 0; r < 4; ++r) sL[buf][c][4 * ti + r] = make_double2(0.0, 0.0);
            }
        }
        __syncthreads();
        int pc[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) pc[c] = sP[buf][c];
        if (!(act && tj == kt)) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c < nc) used |= 1ull << pc[c];
        }
        const bool upd_tile = act && tj > kt;
        const bool upd_rhs = act && tj == tb;
        if (upd_tile || upd_rhs) {
            // pivot-row owners of this column group publish their tiles / rhs
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (c < nc && ti == (pc[c] >> 2)) {
                    if (upd_tile) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int cc = 0; cc < 4; ++cc) sU[tj][c][r][cc] = a[r][cc];
                    }
                    if (upd_rhs) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) sRb[c][r] = rhs[r];
                    }
                }
            }
            // writers and readers are lanes of one wave
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (upd_tile) {
                // lane ti forms u[c][cc] for c = ti / 4, cc = ti % 4 (NT >= 16), or a
                // strided share of the 16 entries (NT < 16)
                for (int e = ti; e < 16; e += NT) {
                    const int c = e >> 2, cc = e & 3;
                    double2 v = make_double2(0.0, 0.0);
                    if (c < nc) {
                        for (int c2 = 0; c2 <= c; ++c2) {
                            const double2 wv = sW[buf][c][c2];
                            const double2 ap = sU[tj][c2][pc[c2] & 3][cc];
                            v.x = fma(wv.x, ap.x, fma(-wv.y, ap.y, v.x));
                            v.y = fma(wv.x, ap.y, fma(wv.y, ap.x, v.y));
                        }
                    }
                    sUu[tj][c][cc] = v;
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (c >= nc) continue;  // uniform
                    double2 lr[4], uc[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) lr[r] = sL[buf][c][4 * ti + r];
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc) uc[cc] = sUu[tj][c][cc];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int cc = 0; cc < 4; ++cc) a[r][cc] = cfms(a[r][cc], lr[r], uc[cc]);
                }
            }
            if (upd_rhs) {
                double2 bp[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) bp[c] = c < nc ? sRb[c][pc[c] & 3] : make_double2(0.0, 0.0);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (c >= nc) continue;  // uniform
                    double2 ub = make_double2(0.0, 0.0);
#pragma unroll
                    for (int c2 = 0; c2 <= c; ++c2) {
                        const double2 wv = sW[buf][c][c2];
                        ub.x = fma(wv.x, bp[c2].x, fma(-wv.y, bp[c2].y, ub.x));
                        ub.y = fma(wv.x, bp[c2].y, fma(wv.y, bp[c2].x, ub.y));
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) rhs[r] = cfms(rhs[r], sL[buf][c][4 * ti + r], ub);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();

    // ---- solution and outputs ---------------------------------------------
    const int flag0 = sFlag;
    const bool bad = (flag0 & (COSIM_SYS_BAD_INPUT | COSIM_SYS_SINGULAR)) != 0;
    int oflag = 0;
    if (act && tj == tb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * ti + r;
            if (i >= n) continue;
            const int k = sKof[i];
            double2 x = cmul(rhs[r], cinv(sPiv[k]));
            if (bad) x = make_double2(__builtin_nan(""), __builtin_nan(""));
            if (!ADJ) {
                Iout[(size_t)s * n + k] = x;
                if (!bad && !(isfinite(x.x) && isfinite(x.y))) oflag |= COSIM_SYS_NONFINITE;
            } else {
                const double2 Ik = Iin[(size_t)s * n + k];
                const double ck = Cb[k];
                // 2 Re(mu I / (j w C^2)) = 2 Im(mu I) / (w C^2)
                const double g = 2.0 * (x.x * Ik.y + x.y * Ik.x) / (w * ck * ck);
                gsys[(size_t)s * n + k] = g;
                if (Iout) Iout[(size_t)s * n + k] = x;  // the adjoint solution mu, on request
                if (!bad && !isfinite(g)) oflag |= COSIM_SYS_NONFINITE;
            }
        }
    }
    if (oflag) atomicOr(&sFlag, oflag);
    __syncthreads();
    if (t == 0) {
        if (or_status) status[s] |= sFlag;
        else status[s] = sFlag;
        if (fac.L) fac.fmt[s] = kFmtGJ;
    }
}

// One block per system.
template <int NP, bool ADJ>
__global__ __launch_bounds__(GJShape<NP>::BLOCK) void k_gj(
    int n, int S, int F, const double *__restrict__ M, const double *__restrict__ Rv,
    const double *__restrict__ phi, const double *__restrict__ C,
    const double *__restrict__ omega, const double2 *__restrict__ Iin,
    const double2 *__restrict__ rpart, int nchunk, double rscale, double2 *__restrict__ Iout,
    double *__restrict__ gsys, int32_t *__restrict__ status, bool or_status, GJFactor fac) {
    __shared__ GjLds<NP> lds;
    gj_system<NP, ADJ>(lds, blockIdx.x, n, S, F, M, Rv, phi, C, omega, Iin, rpart, nchunk, rscale,
                       Iout, gsys, status, or_status, fac, false);
}

// Member of a group that holds global system sg (wave-uniform): members are
// stored in order of their first system s0.
__device__ __forceinline__ int group_member(const SmallGroup &g, int sg) {
    int i = 0;
    while (i + 1 < g.count && sg >= g.in[i + 1].s0) ++i;
    return i;
}

// The forward fallback: workgroup i looks at the records of systems
// kFbSystems i .. kFbSystems (i + 1) - 1 at once and eliminates the marked ones
// (usually none) in turn.  One workgroup per system took 47 us to find
// nothing among 86,016.
constexpr int kFbSystems = 32;
template <int NP, class Run>
__device__ __forceinline__ void fallback_systems(int S, const Run &run, const int *fmt_at_thread) {
    // fmt_at_thread: this thread's record word (threads below kFbSystems)
    const int t = threadIdx.x;
    __shared__ uint32_t sMask;
    if (t < 64) {
        const bool marked = fmt_at_thread && *fmt_at_thread == kFmtNeedsPivot;
        const uint64_t m = __ballot(marked);
        if (t == 0) sMask = (uint32_t)m;
    }
    __syncthreads();
    uint32_t mask = sMask;
    while (mask) {  // uniform
        const int j = __ffs((int)mask) - 1;
        mask &= mask - 1;
        run(blockIdx.x * kFbSystems + j);
        __syncthreads();
    }
}
static_assert(kFbSystems == 32, "one bit per system");

template <int NP>
__global__ __launch_bounds__(GJShape<NP>::BLOCK) void k_gj_fallback(
    int n, int S, int F, const double *__restrict__ M, const double *__restrict__ Rv,
    const double *__restrict__ phi, const double *__restrict__ C,
    const double *__restrict__ omega, double2 *__restrict__ I, int32_t *status, GJFactor fac,
    int32_t *__restrict__ rec_status) {
    __shared__ GjLds<NP> lds;
    const int s0 = blockIdx.x * kFbSystems + threadIdx.x;
    auto run = [&](int s) {
        gj_system<NP, false>(lds, s, n, S, F, M, Rv, phi, C, omega, nullptr, nullptr, 0, 0.0, I,
                             nullptr, status, false, fac, true);
    };
    const bool mine = threadIdx.x < kFbSystems && s0 < S;
    fallback_systems<NP>(S, run, mine ? fac.fmt + s0 : nullptr);
    // the record's copy of the status, final now (the marked systems' by the
    // barrier behind each)
    if (rec_status && mine) rec_status[s0] = status[s0];
}

// The same over the S systems of a group.
template <int NP>
__global__ __launch_bounds__(GJShape<NP>::BLOCK) void k_gj_group(SmallGroup g, int S) {
    __shared__ GjLds<NP> lds;
    const int s0 = blockIdx.x * kFbSystems + threadIdx.x;
    const int *fmt = nullptr;
    if (threadIdx.x < kFbSystems && s0 < S) {
        const SmallInst &e = g.in[group_member(g, s0)];
        fmt = e.fac.fmt + (s0 - e.s0);
    }
    auto run = [&](int sg) {
        const SmallInst &e = g.in[group_member(g, sg)];
        gj_system<NP, false>(lds, sg - e.s0, e.n, e.S, e.F, e.M, e.R, e.phi, e.C, e.omega, nullptr,
                             nullptr, 0, 0.0, e.I, nullptr, e.status, false, e.fac, true);
    };
    fallback_systems<NP>(S, run, fmt);
}

// Sum of a complex value over the 64 lanes of a wave (all lanes active):
// DPP butterflies inside each row of 16, then the four row sums.
template <int CTRL>
__device__ inline double dpp_sum_step(double v) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), CTRL, 0xF, 0xF, false);
    return v + __hiloint2double(hi, lo);
}
__device__ inline double wave_sum(double v) {
    v = dpp_sum_step<0xB1>(v);   // quad_perm [1,0,3,2]
    v = dpp_sum_step<0x4E>(v);   // quad_perm [2,3,0,1]
    v = dpp_sum_step<0x141>(v);  // row_half_mirror
    v = dpp_sum_step<0x140>(v);  // row_mirror
    return (readlane_d(v, 0) + readlane_d(v, 16)) + (readlane_d(v, 32) + readlane_d(v, 48));
}

template <int CTRL>
__device__ inline double dpp_d(double v) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
// One butterfly stage of a transposed reduction: lanes with `upper` keep the
// upper half of their values and send the lower half to the DPP partner,
// which does the opposite; each keeps the pair sum of its half.
template <int CTRL, int N>
__device__ inline void halve(const double (&v)[2 * N], double (&w)[N], bool upper) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const double send = upper ? v[j] : v[j + N];
        const double keep = upper ? v[j + N] : v[j];
        w[j] = keep + dpp_d<CTRL>(send);
    }
}
// Sixteen wave sums at once: returns, in lane l, the sum over all 64 lanes
// of v[l & 15].  Within each row of 16 lanes the partners are 15 - i
// (row_mirror), the mirror inside each half row, then i ^ 2 and i ^ 1, so
// lane i keeps value index i; the four row results are then added across
// rows (lane ^ 16, lane ^ 32).
__device__ inline double wave_sum16(const double (&v)[16], int lane) {
    double w8[8], w4[4], w2[2], w1[1];
    halve<0x140, 8>(v, w8, (lane & 8) != 0);
    halve<0x141, 4>(w8, w4, (lane & 4) != 0);
    halve<0x4E, 2>(w4, w2, (lane & 2) != 0);
    halve<0xB1, 1>(w2, w1, (lane & 1) != 0);
    double t = w1[0];
    t += __shfl_xor(t, 16);
    t += __shfl_xor(t, 32);
    return t;
}

// Back substitution L^T x = z with the packed LDL^T record Ls of one system,
// one wave, lane i holding z_i on entry and x_i on return (0 beyond n).
// Columns go in blocks of U = 8, [k0, k1), from the bottom.  The terms with
// i >= k1 (x_i final) of the block's 8 columns are summed over the lanes
// through LDS: lane i stores its 8 products L_{i,k0+u} x_i as row i of red
// (rows padded to 9 entries, so 16 consecutive lanes hit distinct banks),
// lane l adds up column l % 8 over every 8th row starting at row l / 8, and
// three butterfly steps combine the 8 partial sums.  The terms inside the
// block use L's 8x8 diagonal block, transposed through LDS (tr) so that lane
// k0 + u holds row entries L_{k0+ii, k0+u}, and x_{k0+ii} broadcast from its
// lane as soon as it is final.  Each lane reads only its own row of L
// (entries L_{lane,k}, 0 unless k < lane < n).  red: NP x 9 double2, tr: 64
// (NP = 64) or 128 double2 of the wave's LDS.
constexpr int kBsU = 8;
template <int NP>
__device__ __forceinline__ void bs_load(double2 (&l)[kBsU], const double2 *__restrict__ Ls, int n,
                                        int lane, int k0) {
#pragma unroll
    for (int u = 0; u < kBsU; ++u) {
        const int k = k0 + u;
        l[u] = (lane > k && lane < n) ? Ls[ldl_col(NP, k) + lane - k - 1] : make_double2(0.0, 0.0);
    }
}
// One block [k1 - U, k1) from l (the lanes' row entries of its columns);
// then k1 -= U.  Two LDS exchanges: (1) every lane stores its products and
// the block's lanes their rows of the diagonal block; (2) lane l stores the
// sum of column l % 8 over rows l / 8, l / 8 + 8, ..., and the block's lanes
// read their transposed row entries; then each block lane adds up the 8
// partial sums of its own column.
template <int NP>
__device__ __forceinline__ void bs_block(double2 &x, int &k1, const double2 (&l)[kBsU], int lane,
                                         double2 *red, double2 *tr) {
    constexpr int U = kBsU, RS = U + 1;
    const int cu = lane & (U - 1), part = lane / U;  // column and first row this lane sums
    const int k0 = k1 - U;
    const int ub = (lane - k0) & (U - 1);  // column of the block lane k0 + ub owns
    const bool ext = lane >= k1, blk = lane >= k0 && lane < k1;
    const double2 xe = make_double2(ext ? x.x : 0.0, ext ? x.y : 0.0);
    // U x U partial sums: in the pad column of red when it has 64 rows
    auto psum = [&](int i) -> double2 & { return NP >= 64 ? red[i * RS + U] : tr[U * U + i]; };
    if (lane < NP) {
#pragma unroll
        for (int u = 0; u < U; ++u) red[lane * RS + u] = cmul(l[u], xe);
    }
    if (blk) {
#pragma unroll
        for (int u = 0; u < U; ++u) tr[ub * U + u] = l[u];
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll
    for (int r = 0; r < NP / U; ++r) {
        const double2 t = red[(r * U + part) * RS + cu];
        acc.x += t.x;
        acc.y += t.y;
    }
    psum(part * U + cu) = acc;
    double2 t[U];
#pragma unroll
    for (int ii = 1; ii < U; ++ii) t[ii] = blk ? tr[ii * U + ub] : make_double2(0.0, 0.0);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (blk) {
        double er = 0.0, ei = 0.0;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const double2 e = psum(q * U + ub);
            er += e.x;
            ei += e.y;
        }
        x = make_double2(x.x - er, x.y - ei);
    }
#pragma unroll
    for (int ii = U - 1; ii >= 1; --ii) {
        const double2 xk = make_double2(readlane_d(x.x, k0 + ii), readlane_d(x.y, k0 + ii));
        x = cfms(x, t[ii], xk);  // t[ii] = 0 unless lane < k0 + ii in the block
    }
    // the next block's stores wait for this block's reads
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    k1 = k0;
}
// The columns left of the last whole block, one at a time by wave sums.
__device__ __forceinline__ double2 bs_tail(double2 x, int k1, const double2 *__restrict__ Ls,
                                           int NP, int n, int lane) {
    for (int k = k1 - 1; k >= 0; --k) {
        const double2 l = (lane > k && lane < n) ? Ls[ldl_col(NP, k) + lane - k - 1]
                                                 : make_double2(0.0, 0.0);
        const double pr = l.x * x.x - l.y * x.y;
        const double pi = l.x * x.y + l.y * x.x;
        const double sr = wave_sum(pr), si = wave_sum(pi);
        if (lane == k) x = make_double2(x.x - sr, x.y - si);
    }
    return x;
}
// Any n: loads run DEPTH (1 or 2) blocks ahead, from a ring of DEPTH + 1
// register sets that rotate without copies (the block loop is unrolled).
template <int NP, int DEPTH>
__device__ __forceinline__ double2 ldl_backward(double2 x, const double2 *__restrict__ Ls, int n,
                                                int lane, double2 *red, double2 *tr) {
    constexpr int U = kBsU;
    static_assert(DEPTH == 1 || DEPTH == 2, "one or two blocks ahead");
    int k1 = n;  // columns >= k1 are done
    double2 s0[U], s1[U], s2[U];
    if (n >= U) bs_load<NP>(s0, Ls, n, lane, n - U);
    if (DEPTH == 2 && n >= 2 * U) bs_load<NP>(s1, Ls, n, lane, n - 2 * U);
    auto step = [&](const double2(&l)[U], double2(&fill)[U]) {
        if (k1 - U >= DEPTH * U) bs_load<NP>(fill, Ls, n, lane, k1 - U - DEPTH * U);
        bs_block<NP>(x, k1, l, lane, red, tr);
    };
    while (k1 >= U) {
        if constexpr (DEPTH == 1) {
            step(s0, s1);
            if (k1 < U) break;
            step(s1, s0);
        } else {
            step(s0, s2);
            if (k1 < U) break;
            step(s1, s0);
            if (k1 < U) break;
            step(s2, s1);
        }
    }
    return bs_tail(x, k1, Ls, NP, n, lane);
}
// Complex-symmetric LDL^T factorisation without pivoting, Z = L D L^T.
// The Hermitian part of Z is diag(R) (j w M and 1/(j w C) are skew-Hermitian),
// so with every R_k > 0 each Schur complement keeps a positive-definite real
// part and no pivot can vanish; the elimination needs no row exchanges and
// touches only the lower triangle.
//
// One wave per system.  The lower triangle is held as NB(NB+1)/2 blocks of
// 16x16 (NB = NP/16), each as two FP64 matrix-core accumulators (real and
// imaginary part; lane l holds column l%16, rows g+4m, g = l/16, m = 0..3).
// Panels of 8 columns:
//   1. the lanes holding the panel's columns copy them to LDS;
//   2. lane r eliminates row r of the panel (diagonal block and below) column
//      by column, with the diagonal-block rows broadcast by readlane, giving
//      L and V = L D; their rows replace the panel's rows in LDS;
//   3. every lower block right of the panel takes the rank-8 update
//      A -= L21 V21^T as eight 16x16x4 FP64 MFMAs (complex = 4 real products
//      per 4 columns).
// Wider panels halve the LDS round trips and wave barriers per column, which
// with one wave per system are latency that the MFMAs do not hide.
// Columns left of the trailing part also receive updates; they are finished
// and never read again.  The factor is recorded (L by columns, D^-1) for
// k_forward and the adjoint, and the forward right-hand side b = E - j w Phi
// rides along: y = L^-1 b is formed panel by panel and z = D^-1 y is written
// to Z, so that k_forward only runs the backward substitution.  A system whose
// smallest pivot is below 1e-5 of its largest impedance diagonal (or is not
// finite) is marked for the pivoted fallback.
// The accumulators and the row state fit 256 registers, so two systems share
// a SIMD: one wave's panel elimination runs while the other's MFMAs do.
constexpr int kOneRound = 2048;  // systems resident at once: two waves on each of 1,024 SIMDs

// One wave's LDS.  Panel rows (A, then L21) and V21 rows; a row holds 8 entries
// padded to 9 (144 bytes), so that the row-per-lane accesses of 16 consecutive
// lanes fall on disjoint LDS banks.
template <int NP>
struct LdlWaveLds {
    double2 pan[NP][9], vv[NP][9];
};
// With KEEP (NP = 32) the lane's row of L stays in lrow (panel p, column 8 p +
// c; zero on and above the diagonal and on padding) and z = D^-1 y in zout, for
// a back substitution in the same wave; nothing is written to Z and status.
// Returns whether the system needs the pivoted fallback; flag_out: input flags.
template <int NP, bool KEEP>
__device__ __forceinline__ bool ldl_system(
    LdlWaveLds<NP> &lds, double2 (&lrow)[KEEP ? NP / 8 : 1][8], double2 &zout, int &flag_out,
    int s, int n, int F, const double *__restrict__ M, const double *__restrict__ Rv,
    const double *__restrict__ C, const double *__restrict__ omega,
    const double *__restrict__ phi, GJFactor fac, double2 *__restrict__ Z,
    int32_t *__restrict__ status) {
    constexpr int NB = NP / 16;
    constexpr int NBLK = NB * (NB + 1) / 2;
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63;
    constexpr int PW = 8;  // panel width
    const int b = s / F, f = s - b * F;
    const double w = omega[f];
    const double *Cb = C + (size_t)b * n;
    const int g = lane >> 4, c16 = lane & 15;

    // ---- Z in accumulator layout: block (bi, bj) at index bi (bi + 1) / 2 + bj.
    // Loads use clamped indices and no branches, so they are all in flight at
    // once; out-of-range entries are replaced by the identity padding.
    double rdg[NB], cdg[NB];  // R_j, 1/(w C_j) of column j = 16 bj + c16
#pragma unroll
    for (int bj = 0; bj < NB; ++bj) {
        const int j = min(16 * bj + c16, n - 1);
        rdg[bj] = Rv[j];
        cdg[bj] = Cb[j];
    }
    f64x4 Xr[NBLK], Xi[NBLK];
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = 0; bj <= bi; ++bj) {
            const int bx = bi * (bi + 1) / 2 + bj;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int i = 16 * bi + g + 4 * m, j = 16 * bj + c16;
                const double mij = M[(size_t)min(i, n - 1) * n + min(j, n - 1)];
                Xr[bx][m] = 0.0;
                Xi[bx][m] = (i < n && j < n) ? w * mij : 0.0;
            }
        }
#pragma unroll
    for (int bj = 0; bj < NB; ++bj) {
        const double xc = 1.0 / (w * cdg[bj]);
        const int bx = bj * (bj + 1) / 2 + bj;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            if (g + 4 * m == c16) {  // diagonal entry i = j = 16 bj + c16
                const bool real = 16 * bj + c16 < n;
                Xr[bx][m] = real ? rdg[bj] : 1.0;
                Xi[bx][m] = real ? Xi[bx][m] - xc : 0.0;
            }
        }
    }
    // input flags and the largest |re|+|im| diagonal entry (lane k handles k)
    int flag = 0;
    float zdiag = 0.0f;
    if (lane < n) {
        const double c = Cb[lane];
        if (isnan(c) || c == 0.0 || !isfinite(w) || w == 0.0) flag = COSIM_SYS_BAD_INPUT;
        else if (c < 0.0) flag = COSIM_SYS_NEGATIVE_C;
        zdiag = (float)(fabs(Rv[lane]) + fabs(w * M[(size_t)lane * n + lane] - 1.0 / (w * c)));
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        flag |= __shfl_xor(flag, off);
        zdiag = fmaxf(zdiag, __shfl_xor(zdiag, off));
    }
    // right-hand side b = E - j w Phi (lane i holds b_i), turned into y = L^-1 b
    // column by column as L is formed
    double2 y = lane < n ? loop_voltage(phi, n, lane, w) : make_double2(0.0, 0.0);
    double2 dk = make_double2(1.0, 0.0);  // D_i of the lane's own column

    auto &pan = lds.pan;
    auto &vv = lds.vv;
    if constexpr (KEEP) {
#pragma unroll
        for (int p = 0; p < NP / 8; ++p)
#pragma unroll
            for (int c = 0; c < 8; ++c) lrow[p][c] = make_double2(0.0, 0.0);
    }
    double2 *Ls = fac.L + (size_t)s * NP * NP;  // packed columns, see ldl_col
#pragma unroll
    for (int bc = 0; bc < NB; ++bc) {
#pragma unroll
        for (int h = 0; h < 16 / PW; ++h) {
            const int k0 = 16 * bc + PW * h;  // first column of the panel
            if (k0 >= n) break;               // uniform
            // 1. panel columns -> LDS (rows >= k0 matter)
            if (c16 >= PW * h && c16 < PW * h + PW) {
                const int c = c16 - PW * h;
                // real parts, then imaginary parts: 8-byte stores straight from
                // the accumulators (the empty asm keeps the two halves from
                // being merged into 16-byte stores, which need register copies)
#pragma unroll
                for (int bi = bc; bi < NB; ++bi) {
                    const int bx = bi * (bi + 1) / 2 + bc;
#pragma unroll
                    for (int m = 0; m < 4; ++m) pan[16 * bi + g + 4 * m][c].x = Xr[bx][m];
                }
                asm volatile("" ::: "memory");
#pragma unroll
                for (int bi = bc; bi < NB; ++bi) {
                    const int bx = bi * (bi + 1) / 2 + bc;
#pragma unroll
                    for (int m = 0; m < 4; ++m) pan[16 * bi + g + 4 * m][c].y = Xi[bx][m];
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // 2. lane r takes row r of the panel, column by column:
            //      V_rc = A_rc - sum_{j<c} L_rj V_cj,  D_c = V_cc,  L_rc = V_rc / D_c.
            //    Row c of V (entries j < c, stored by lane k0 + c in earlier
            //    columns) reaches every lane as broadcast LDS reads, D_c by
            //    readlane; V and L rows replace the panel rows in LDS as they
            //    are formed.  Rows above the panel end in the upper triangle or
            //    in eliminated columns, which are never read again, so every
            //    row is stored as it comes.
            const int r = lane, rr = min(r, NP - 1);
            double2 l[PW];
#pragma unroll
            for (int c = 0; c < PW; ++c) {
                if (KEEP && k0 + c >= n) {  // uniform: identity padding, nothing below the diagonal
                    l[c] = make_double2(0.0, 0.0);
                    if (r < NP) {
                        pan[r][c] = l[c];
                        vv[r][c] = l[c];
                    }
                    continue;
                }
                double2 v = pan[rr][c];
                double2 vc[PW];
#pragma unroll
                for (int j = 0; j < c; ++j) vc[j] = vv[k0 + c][j];
#pragma unroll
                for (int j = 0; j < c; ++j) v = cfms(v, l[j], vc[j]);
                const double2 d = make_double2(readlane_d(v.x, k0 + c), readlane_d(v.y, k0 + c));
                const double2 dinv = cinv_nr(d);
                l[c] = cmul(v, dinv);
                // L below the diagonal (rows of the diagonal block and below
                // it); the column's base is wave-uniform, so the store takes a
                // scalar base and the lane's constant offset
                double2 *col = Ls + (ldl_col(NP, k0 + c) - (k0 + c) - 1);
                if (r > k0 + c && r < NP) col[r] = l[c];
                if (r < NP) {
                    pan[r][c] = l[c];
                    vv[r][c] = v;
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            if constexpr (KEEP) {
#pragma unroll
                for (int c = 0; c < PW; ++c)
                    if (r > k0 + c && r < n) lrow[k0 / 8][c] = l[c];
            }
            // D_c = V_cc to the lane of column c (with KEEP the padded columns of a
            // last panel are not formed: 1 stays)
            if (r >= k0 && r < k0 + PW && (!KEEP || r < n)) dk = vv[r][r - k0];
            // forward substitution for the panel's columns: y_r -= L_rc y_c (r > k0 + c)
#pragma unroll
            for (int c = 0; c < PW; ++c) {
                const double2 yc = make_double2(readlane_d(y.x, k0 + c), readlane_d(y.y, k0 + c));
                const double2 yn = cfms(y, l[c], yc);
                const bool below = r > k0 + c;
                y.x = below ? yn.x : y.x;  // componentwise: a select of the
                y.y = below ? yn.y : y.y;  // vector struct goes through memory
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // 3. rank-PW update of every lower block right of the panel, as
            // PW / 4 steps of four 16x16x4 FP64 MFMAs; the operands of a block
            // row are read from LDS just before its MFMAs.  The last panel of
            // a block column leaves that column fully eliminated, so its
            // blocks are skipped.
            const int bj0 = h == 16 / PW - 1 ? bc + 1 : bc;
#pragma unroll
            for (int bi = bj0; bi < NB; ++bi) {
                double2 La[PW / 4];  // A operand: row c16 of block bi, k = g + 4 q
#pragma unroll
                for (int q = 0; q < PW / 4; ++q) La[q] = pan[16 * bi + c16][g + 4 * q];
#pragma unroll
                for (int bj = bj0; bj <= bi; ++bj) {
                    const int bx = bi * (bi + 1) / 2 + bj;
#pragma unroll
                    for (int q = 0; q < PW / 4; ++q) {
                        const double2 Vb = vv[16 * bj + c16][g + 4 * q];  // B operand: column c16 of block bj
                        Xr[bx] = __builtin_amdgcn_mfma_f64_16x16x4f64(-La[q].x, Vb.x, Xr[bx], 0, 0, 0);
                        Xr[bx] = __builtin_amdgcn_mfma_f64_16x16x4f64(La[q].y, Vb.y, Xr[bx], 0, 0, 0);
                        Xi[bx] = __builtin_amdgcn_mfma_f64_16x16x4f64(-La[q].x, Vb.y, Xi[bx], 0, 0, 0);
                        Xi[bx] = __builtin_amdgcn_mfma_f64_16x16x4f64(-La[q].y, Vb.x, Xi[bx], 0, 0, 0);
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    const double2 dl = cinv_nr(dk);  // the D^-1 the elimination used
    if (lane < NP) fac.piv_val[(size_t)s * NP + lane] = dl;  // D^-1 (1 on the padding)
    // smallest |re| + |im| pivot of the real columns
    double dmin = lane < n ? fabs(dk.x) + fabs(dk.y) : __builtin_inf();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) dmin = fmin(dmin, __shfl_xor(dmin, off));
    const bool pivot = (flag & COSIM_SYS_BAD_INPUT) || !(dmin >= 1e-5 * (double)zdiag);
    zout = cmul(y, dl);  // z = D^-1 L^-1 b
    flag_out = flag;
    if (!KEEP && lane < n) Z[(size_t)s * n + lane] = zout;
    if (lane == 0) {
        if (!KEEP) status[s] = flag;
        fac.fmt[s] = pivot ? kFmtNeedsPivot : kFmtLDL;
    }
    return pivot;
}

// The whole forward solve of one system of at most 32 loops by one wave, the
// block's only one: LDL^T, the back substitution from the rows of L in
// registers, and the pivoted elimination if it is needed.  One launch in place
// of three, and no read of the record: at these sizes the launches and the
// memory round trips between them are the time (64 systems of one loop: 12.4
// us in three launches).
union Small32Lds {
    LdlWaveLds<32> ldl;
    struct {
        double2 red[32 * 9], tr[128];
    } bs;
    GjLds<32> gj;
    __device__ Small32Lds() {}
};
__device__ __forceinline__ void small32_system(
    Small32Lds &lds, int s, int n, int S, int F, const double *__restrict__ M,
    const double *__restrict__ Rv, const double *__restrict__ C, const double *__restrict__ omega,
    const double *__restrict__ phi, const GJFactor &fac, double2 *__restrict__ I,
    int32_t *__restrict__ status, int32_t *__restrict__ rec_status) {
    const int lane = threadIdx.x;
    double2 lrow[4][8], x;
    int flag;
    const bool pivot = ldl_system<32, true>(lds.ldl, lrow, x, flag, s, n, F, M, Rv, C, omega, phi,
                                            fac, nullptr, nullptr);
    __syncthreads();
    if (pivot) {  // uniform
        gj_system<32, false>(lds.gj, s, n, S, F, M, Rv, phi, C, omega, nullptr, nullptr, 0, 0.0, I,
                             nullptr, status, false, fac, false);
        if (rec_status && lane == 0) rec_status[s] = status[s];
        return;
    }
    if (lane >= n) x = make_double2(0.0, 0.0);
#pragma unroll
    for (int p = 3; p >= 0; --p) {
        if (8 * p >= n) continue;  // uniform
        int k1 = 8 * p + 8;
        bs_block<32>(x, k1, lrow[p], lane, lds.bs.red, lds.bs.tr);
    }
    bool nonfinite = false;
    if (lane < n) {
        I[(size_t)s * n + lane] = x;
        nonfinite = !(isfinite(x.x) && isfinite(x.y));
    }
    const bool any = __ballot(nonfinite) != 0;
    if (lane == 0) {
        flag |= any ? COSIM_SYS_NONFINITE : 0;
        status[s] = flag;
        if (rec_status) rec_status[s] = flag;
    }
}
// WPE waves per SIMD: 2 while every system is resident at once (no spills on
// the single wave's way), 3 beyond (2,100 systems of 25 loops: 33 us against 39).
template <int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE))) void k_small32(
    int n, int S, int F, const double *__restrict__ M, const double *__restrict__ Rv,
    const double *__restrict__ C, const double *__restrict__ omega,
    const double *__restrict__ phi, GJFactor fac, double2 *__restrict__ I,
    int32_t *__restrict__ status, int32_t *__restrict__ rec_status) {
    __shared__ Small32Lds lds;
    small32_system(lds, blockIdx.x, n, S, F, M, Rv, C, omega, phi, fac, I, status, rec_status);
}
template <int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE))) void k_small32_group(
    SmallGroup g) {
    __shared__ Small32Lds lds;
    const int sg = blockIdx.x;
    const SmallInst &e = g.in[group_member(g, sg)];
    small32_system(lds, sg - e.s0, e.n, e.S, e.F, e.M, e.R, e.C, e.omega, e.phi, e.fac, e.I,
                   e.status, nullptr);
}

// ---- 33 to 64 loops, few systems -------------------------------------------
// A workgroup of four waves per system: L D L^T of the whole matrix on
// accumulators (ldl_block), with X = L^-1 recorded in place of L (kFmtInv), so
// that both triangular solves, here and in the adjoint, are products with X
// instead of chains of 64 columns; the pivoted elimination, if it is needed,
// runs in the same launch.  This is the shorter way through one system, but
// it takes more of the chip per system: 48 systems of 64 loops take 28.8 us
// forward and 8.8 us in the adjoint, where a wave per system, the launch for the
// pivoted ones and the replay take 47.4 and 25.2, while 1,152 take 98 and 30 us
// against 76 and 37 (512 workgroups are resident at once).
//   The line is drawn by what a plan has, not by what a launch has, so that a
// member of a group takes the route (and gets the bits) it has alone; it lies
// where groups of up to 256 members stop gaining.  Whole calls, 64 loops, 4,096
// points, us by this route / by the other:
//   systems   one plan   48 plans   128 plans   256 plans
//       8      45 / 71   290 / 305   457 / 501    706 / 758
//      12      45 / 72   296 / 310   502 / 523    824 / 796
//      16      46 / 72   303 / 314   552 / 538    907 / 826
//      24         -      344 / 328   673 / 593  1,137 / 917
//      48      48 / 76   484 / 400   992 / 742        -
// (12 systems, 256 plans: 838 us before there were two routes.)
constexpr int kFewSystems = 12;

union Small64Lds {
    struct {
        BlockLds b;
        double2 red[256], v[64];
        int pivot;
        bool nonfinite;
    } x;
    GjLds<64> gj;
    __device__ Small64Lds() {}
};

// X^T v for the record's X: thread t returns its share, rows 16 (t % 4) ..
// + 15 of column t / 4, loaded beforehand by block_xt_load; summed over the
// four threads by the caller.
__device__ __forceinline__ void block_xt_load(const double2 *X, int tid, double2 (&x)[16]) {
    const int c = tid >> 2, part = tid & 3;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        x[i] = part >= (c >> 4) ? X[c * 64 + 16 * part + i] : make_double2(0.0, 0.0);
}
__device__ __forceinline__ double2 block_xt_times(const double2 (&x)[16], const double2 *v, int tid) {
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < 16; ++i) acc = zfma(acc, x[i], v[16 * (tid & 3) + i]);
#pragma unroll
    for (int off = 1; off <= 2; off <<= 1) {
        acc.x += __shfl_xor(acc.x, off);
        acc.y += __shfl_xor(acc.y, off);
    }
    return acc;
}

__device__ __forceinline__ void small64_system(Small64Lds &lds, int s, int n, int S, int F,
                                               const double *__restrict__ M,
                                               const double *__restrict__ Rv,
                                               const double *__restrict__ phi,
                                               const double *__restrict__ C,
                                               const double *__restrict__ omega, const GJFactor &fac,
                                               double2 *__restrict__ I, int32_t *__restrict__ status,
                                               int32_t *__restrict__ rec_status) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    const int b = s / F, f = s - b * F;
    const double w = omega[f];
    const double *Cb = C + (size_t)b * n;
    auto &x = lds.x;
    // Z off the diagonal (clamped addresses, so that all loads are in flight)
    double zo[3][4];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * diag_rb(wv, q) + g + 4 * e, j = 16 * diag_cb(wv, q) + r16;
            if (q < (wv < 2 ? 3 : 2)) {
                const double v = w * M[(size_t)min(i, n - 1) * n + min(j, n - 1)];
                zo[q][e] = i < n && j < n ? v : 0.0;
            }
        }
    int flag = 0;       // of wave 0
    double zmax = 0.0;  // of wave 0
    if (wv == 0) {
        const int k = min(lane, n - 1);
        const double c = Cb[k], r = Rv[k], xm = w * M[(size_t)k * n + k];
        const double2 rhs = loop_voltage(phi, n, k, w);
        const bool real = lane < n;
        if (__ballot(real && (isnan(c) || c == 0.0 || !isfinite(w) || w == 0.0)))
            flag = COSIM_SYS_BAD_INPUT;
        if (__ballot(real && c < 0.0)) flag |= COSIM_SYS_NEGATIVE_C;
        const double xk = xm - 1.0 / (w * c);
        x.b.sz[lane].x = real ? r : 1.0;
        x.b.sz[lane].y = real ? xk : 0.0;
        x.b.st[lane].x = real ? rhs.x : 0.0;
        x.b.st[lane].y = real ? rhs.y : 0.0;
        zmax = real ? fabs(r) + fabs(xk) : 0.0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) zmax = fmax(zmax, __shfl_xor(zmax, off));
        if (lane == 0) {
            x.pivot = (flag & COSIM_SYS_BAD_INPUT) != 0;
            x.nonfinite = false;
        }
    }
    __syncthreads();
    double2 *X = fac.L + (size_t)s * 64 * 64;
    if (!x.pivot) {  // uniform
        f64x4 Cr[3], Ci[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            Cr[q] = Ci[q] = f64x4{0, 0, 0, 0};
            if (q >= (wv < 2 ? 3 : 2)) continue;
            const int row = 16 * diag_rb(wv, q) + g, col = 16 * diag_cb(wv, q) + r16;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                Ci[q][e] = zo[q][e];
                if (diag_rb(wv, q) == diag_cb(wv, q)) {
                    const double2 zd = x.b.sz[row + 4 * e];
                    Cr[q][e] = row + 4 * e == col ? zd.x : 0.0;
                    Ci[q][e] = row + 4 * e == col ? zd.y : zo[q][e];
                }
            }
        }
        ldl_block<double2, false>(x.b, Cr, Ci, X, nullptr, 64, fac.piv_val + (size_t)s * 64);
        if (wv == 0) {
            const double dmin = block_min_pivot(x.b, lane, n);
            if (lane == 0) x.pivot = !(dmin >= 1e-5 * zmax);
        }
        double2 xt[16];
        block_xt_load(X, tid, xt);
        const double2 y = block_x_times(X, x.b.st, x.red, tid);
        if (tid < 64) {
            x.v[tid] = zmul(y, zinv_nr(x.b.pivot(tid)));
        }
        __syncthreads();
        const double2 cur = block_xt_times(xt, x.v, tid);
        const int k = tid >> 2;
        if ((tid & 3) == 0 && k < n) {
            I[(size_t)s * n + k] = cur;
            if (!(isfinite(cur.x) && isfinite(cur.y))) x.nonfinite = true;
        }
        __syncthreads();
    }
    const bool pivot = x.pivot;
    if (tid == 0 && !pivot) {
        flag |= x.nonfinite ? COSIM_SYS_NONFINITE : 0;
        fac.fmt[s] = kFmtInv;
        status[s] = flag;
        if (rec_status) rec_status[s] = flag;
    }
    if (!pivot) return;  // uniform
    __syncthreads();     // every thread has read the flag: its memory is reused
    gj_system<64, false>(lds.gj, s, n, S, F, M, Rv, phi, C, omega, nullptr, nullptr, 0, 0.0, I,
                         nullptr, status, false, fac, false);
    if (rec_status && tid == 0) rec_status[s] = status[s];  // the thread that wrote it
}
static_assert(GJShape<64>::BLOCK == 256, "one workgroup for either elimination");

__global__ __launch_bounds__(256, 2) void k_small64(
    int n, int S, int F, const double *__restrict__ M, const double *__restrict__ Rv,
    const double *__restrict__ phi, const double *__restrict__ C,
    const double *__restrict__ omega, GJFactor fac, double2 *__restrict__ I,
    int32_t *__restrict__ status, int32_t *__restrict__ rec_status) {
    __shared__ Small64Lds lds;
    small64_system(lds, blockIdx.x, n, S, F, M, Rv, phi, C, omega, fac, I, status, rec_status);
}
// The members of a group that have few systems; as in every launch of a group,
// a member takes the same route as alone, so the results are the same bits.
__global__ __launch_bounds__(256, 2) void k_small64_group(SmallGroup g) {
    __shared__ Small64Lds lds;
    const int sg = blockIdx.x;
    const SmallInst &e = g.in[group_member(g, sg)];
    if (e.S > kFewSystems) return;  // whole workgroup: k_ldl_group's
    small64_system(lds, sg - e.s0, e.n, e.S, e.F, e.M, e.R, e.phi, e.C, e.omega, e.fac, e.I, e.status,
                   nullptr);
}

// Forward solve of a system in the LDL^T format from the z the factorisation
// left in I: x = L^-T z, written over it (systems handed to the pivoted
// fallback are skipped; it writes their I).  red, tr: as for ldl_backward.
template <int NP>
__device__ __forceinline__ void forward_system(int s, int n, GJFactor fac, double2 *__restrict__ I,
                                               int32_t *__restrict__ status, double2 *red,
                                               double2 *tr) {
    const int lane = threadIdx.x & 63;
    if (__builtin_amdgcn_readfirstlane(fac.fmt[s]) != kFmtLDL) return;
    double2 x = lane < n ? I[(size_t)s * n + lane] : make_double2(0.0, 0.0);
    x = ldl_backward<NP, 2>(x, fac.L + (size_t)s * NP * NP, n, lane, red, tr);
    bool nonfinite = false;
    if (lane < n) {
        I[(size_t)s * n + lane] = x;
        nonfinite = !(isfinite(x.x) && isfinite(x.y));
    }
    if (__ballot(nonfinite) != 0 && lane == 0) status[s] |= COSIM_SYS_NONFINITE;
}

template <int NP>
__global__ __launch_bounds__(256) void k_forward(int n, int S, GJFactor fac,
                                                 double2 *__restrict__ I,
                                                 int32_t *__restrict__ status) {
    const int s = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    __shared__ double2 sRed[4][NP * 9], sTr[4][64];
    if (s >= S) return;
    forward_system<NP>(s, n, fac, I, status, sRed[threadIdx.x >> 6], sTr[threadIdx.x >> 6]);
}

// One wave per system, four per block.  With FWD the wave goes on to the back
// substitution (forward_system) from the record it has just written: chosen
// where all systems are resident at once (kOneRound), so that only latency
// counts; for more, the separate launch hides the substitution's exchanges
// better, with three to four waves per SIMD.
template <int NP, bool FWD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_ldl(
    int n, int S, int F, const double *__restrict__ M, const double *__restrict__ Rv,
    const double *__restrict__ C, const double *__restrict__ omega,
    const double *__restrict__ phi, GJFactor fac, double2 *__restrict__ Z,
    int32_t *__restrict__ status) {
    __shared__ LdlWaveLds<NP> lds[4];
    const int s = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (s >= S) return;  // whole wave; the block never synchronises
    double2 none[1][8], z;
    int flag;
    ldl_system<NP, false>(lds[threadIdx.x >> 6], none, z, flag, s, n, F, M, Rv, C, omega, phi, fac,
                          Z, status);
    if constexpr (FWD) {
        __threadfence_block();  // this wave's record, z and status
        LdlWaveLds<NP> &w = lds[threadIdx.x >> 6];
        forward_system<NP>(s, n, fac, Z, status, &w.pan[0][0], &w.vv[0][0]);
    }
}

// The same over the S systems of a group of plans (each wave resolves its own
// member, so the waves of a block may serve different plans).
template <int NP>
__global__ __launch_bounds__(256) void k_forward_group(SmallGroup g, int S) {
    const int sg = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    __shared__ double2 sRed[4][NP * 9], sTr[4][64];
    if (sg >= S) return;
    const SmallInst &e = g.in[group_member(g, sg)];
    forward_system<NP>(sg - e.s0, e.n, e.fac, e.I, e.status, sRed[threadIdx.x >> 6],
                       sTr[threadIdx.x >> 6]);
}

template <int NP, bool FWD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_ldl_group(
    SmallGroup g, int S) {
    __shared__ LdlWaveLds<NP> lds[4];
    const int sg = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (sg >= S) return;
    const SmallInst &e = g.in[group_member(g, sg)];
    if (NP == 64 && e.S <= kFewSystems) return;  // whole wave: k_small64_group's
    double2 none[1][8], z;
    int flag;
    ldl_system<NP, false>(lds[threadIdx.x >> 6], none, z, flag, sg - e.s0, e.n, e.F, e.M, e.R, e.C,
                          e.omega, e.phi, e.fac, e.I, e.status);
    if constexpr (FWD) {
        __threadfence_block();
        LdlWaveLds<NP> &w = lds[threadIdx.x >> 6];
        forward_system<NP>(sg - e.s0, e.n, e.fac, e.I, e.status, &w.pan[0][0], &w.vv[0][0]);
    }
}

// Adjoint solve with a recorded factorisation, one wave per system, lane i
// holds component i; b = rscale * sum_c (rr - j ri) of rpart[c][s][:].
// Format kFmtLDL: y = L^-1 b by columns (readlane broadcast of y_k, one
// coalesced column load), z = D^-1 y, then L^T x = z (ldl_backward).
// Format kFmtGJ: replays the recorded Gauss-Jordan row operations
// b <- b - l_k b_{p_k}, then x_k = b_{p_k} / piv_k.
// Writes gsys[s][k] = 2 Re(mu_k I_k / (j w C_k^2)) and, if given, mu.
template <int NP>
__device__ __forceinline__ void replay_system(int s, int n, int S, int F, GJFactor fac,
                                              const double *__restrict__ C,
                                              const double *__restrict__ omega,
                                              const double2 *__restrict__ I,
                                              const double2 *__restrict__ rpart, int nchunk,
                                              double rscale, double *__restrict__ gsys,
                                              double2 *__restrict__ mu,
                                              int32_t *__restrict__ status,
                                              const int32_t *__restrict__ status_in,
                                              const FinalSums &fin) {
    __shared__ double2 sRed[4][NP * 9];  // per wave: the lane products of ldl_backward
    __shared__ double2 sTr[4][NP >= 64 ? 64 : 128];  // per wave: an 8x8 block of L, transposed
    const int lane = threadIdx.x & 63;
    const int fmt = __builtin_amdgcn_readfirstlane(fac.fmt[s]);
    const int b = s / F, f = s - b * F;
    const double w = omega[f];
    double2 x = make_double2(0.0, 0.0);
    {
        // the chunks dealt to the 64 / w lanes that share entry k, w = 8, 16, 32
        // or 64 >= n, and added across them by halves
        const int w = n <= 8 ? 8 : n <= 16 ? 16 : n <= 32 ? 32 : 64;
        const int k = lane & (w - 1);
        double rr = 0.0, ri = 0.0;
#pragma unroll 8
        for (int c = lane / w; c < nchunk; c += 64 / w) {
            const double2 v = rpart[((size_t)c * S + s) * NP + (k < NP ? k : 0)];
            rr += v.x;
            ri += v.y;
        }
        for (int off = 32; off >= w; off >>= 1) {
            rr += __shfl_xor(rr, off);
            ri += __shfl_xor(ri, off);
        }
        if (lane < n) x = make_double2(rscale * rr, -rscale * ri);
    }
    const double2 *__restrict__ Ls = fac.L + (size_t)s * NP * NP;
    constexpr int U = 8;
    if (fmt == kFmtLDL) {
        // column k of L as lane i sees it: L_ik for k < i < n, else 0
        auto lcol = [&](int k) {
            return (lane > k && lane < n) ? Ls[ldl_col(NP, k) + lane - k - 1] : make_double2(0.0, 0.0);
        };
        // Columns are loaded in groups of U; the next group's loads are in
        // flight while the current group is applied (cur / nxt registers).
        double2 cur[U], nxt[U];
        auto load_group = [&](double2(&l)[U], int k0) {
#pragma unroll
            for (int u = 0; u < U; ++u) l[u] = lcol(k0 + u);
        };
        // forward: y_i -= L_ik y_k for i > k
        const int nfg = n / U;  // full groups
        if (nfg > 0) load_group(cur, 0);
        int k0 = 0;
        for (; k0 + U <= n; k0 += U) {
            if (k0 + 2 * U <= n) load_group(nxt, k0 + U);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double2 yk = make_double2(readlane_d(x.x, k0 + u), readlane_d(x.y, k0 + u));
                x = cfms(x, cur[u], yk);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) cur[u] = nxt[u];
        }
        for (; k0 < n; ++k0) {
            const double2 l = lcol(k0);
            const double2 yk = make_double2(readlane_d(x.x, k0), readlane_d(x.y, k0));
            x = cfms(x, l, yk);
        }
        if (lane < n) x = cmul(x, fac.piv_val[(size_t)s * NP + lane]);  // D^-1
        x = ldl_backward<NP, 1>(x, Ls, n, lane, sRed[threadIdx.x >> 6], sTr[threadIdx.x >> 6]);
    } else {
        const int *__restrict__ Ps = fac.piv_row + (size_t)s * NP;
        int k0 = 0;
        for (; k0 + U <= n; k0 += U) {
            double2 l[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                l[u] = lane < NP ? Ls[(size_t)(k0 + u) * NP + lane] : make_double2(0.0, 0.0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = Ps[k0 + u];
                const double2 bp = make_double2(readlane_d(x.x, p), readlane_d(x.y, p));
                x = cfms(x, l[u], bp);
            }
        }
        for (; k0 < n; ++k0) {
            const double2 l = lane < NP ? Ls[(size_t)k0 * NP + lane] : make_double2(0.0, 0.0);
            const int p = Ps[k0];
            const double2 bp = make_double2(readlane_d(x.x, p), readlane_d(x.y, p));
            x = cfms(x, l, bp);
        }
        const int pk = lane < n ? Ps[lane] : 0;
        const double2 bpk = make_double2(__shfl(x.x, pk), __shfl(x.y, pk));
        x = lane < n ? cmul(bpk, cinv(fac.piv_val[(size_t)s * NP + lane])) : make_double2(0.0, 0.0);
    }
    const int flag = status_in[s];
    const bool bad = (flag & (COSIM_SYS_BAD_INPUT | COSIM_SYS_SINGULAR)) != 0;
    bool nonfinite = false;
    if (lane < n) {
        if (bad) x = make_double2(__builtin_nan(""), __builtin_nan(""));
        const double2 Ik = I[(size_t)s * n + lane];
        const double ck = C[(size_t)b * n + lane];
        // 2 Re(mu I / (j w C^2)) = 2 Im(mu I) / (w C^2)
        const double g = 2.0 * (x.x * Ik.y + x.y * Ik.x) / (w * ck * ck);
        // with one frequency the system's term is the configuration's gradient (a
        // sum that starts from 0, as reduce_config's, has no negative zero)
        if (fin.grad) fin.grad[(size_t)s * n + lane] = 0.0 + g;
        else gsys[(size_t)s * n + lane] = g;
        if (mu) mu[(size_t)s * n + lane] = x;
        nonfinite = !bad && !isfinite(g);
    }
    if (fin.grad) {  // and its partial losses the configuration's: the order of reduce_config
        double acc = 0.0;
        for (int c = lane; c < nchunk; c += 64) acc += fin.lpart[(size_t)c * S + s];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
        if (lane == 0) fin.loss[s] = fin.lscale * acc;
    }
    const bool any = __ballot(nonfinite) != 0;
    if ((any || status_in != status) && lane == 0) status[s] = flag | (any ? COSIM_SYS_NONFINITE : 0);
}

// The adjoint of one system with a kFmtInv record (small64_system) by a
// workgroup: mu = X^T D^-1 X b, b and the results as in replay_system, which
// takes the other records.  Both layouts of X are on their way while the
// partial sums are added up.
__device__ __forceinline__ void replay64_system(
    int s, int n, int S, int F, const GJFactor &fac, const double *__restrict__ C,
    const double *__restrict__ omega, const double2 *__restrict__ I, const double2 *__restrict__ rpart,
    int nchunk, double rscale, double *__restrict__ gsys, double2 *__restrict__ mu,
    int32_t *__restrict__ status, const int32_t *__restrict__ status_in, const FinalSums &fin) {
    __shared__ double2 red[256], v[64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (fac.fmt[s] != kFmtInv) {  // whole workgroup
        if (wv == 0)
            replay_system<64>(s, n, S, F, fac, C, omega, I, rpart, nchunk, rscale, gsys, mu, status,
                              status_in, fin);
        return;
    }
    const double2 *__restrict__ X = fac.L + (size_t)s * 64 * 64;
    double2 xn[16], xt[16];
#pragma unroll
    for (int c = 0; c < 16; ++c)
        xn[c] = wv <= (lane >> 4) ? X[(16 * wv + c) * 64 + lane] : make_double2(0.0, 0.0);
    block_xt_load(X, tid, xt);
    const int b = s / F, kk = min(lane, n - 1);
    const double w = omega[s - b * F];
    const double2 Ik = I[(size_t)s * n + kk];
    const double ck = C[(size_t)b * n + kk];
    const double2 dinv = fac.piv_val[(size_t)s * 64 + lane];
    const int flag = status_in[s];
    double rr = 0.0, ri = 0.0;
#pragma unroll 8
    for (int c = wv; c < nchunk; c += 4) {
        const double2 r = rpart[((size_t)c * S + s) * 64 + lane];
        rr += r.x;
        ri += r.y;
    }
    red[tid] = make_double2(rr, ri);
    __syncthreads();
    if (wv == 0) {
        double2 t = red[lane];
#pragma unroll
        for (int e = 1; e < 4; ++e) {
            t.x += red[64 * e + lane].x;
            t.y += red[64 * e + lane].y;
        }
        v[lane].x = lane < n ? rscale * t.x : 0.0;
        v[lane].y = lane < n ? -rscale * t.y : 0.0;
    }
    __syncthreads();
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll
    for (int c = 0; c < 16; ++c) acc = zfma(acc, xn[c], v[16 * wv + c]);
    red[tid] = acc;
    __syncthreads();
    if (wv == 0) {
        double2 t = red[lane];
#pragma unroll
        for (int e = 1; e < 4; ++e) {
            t.x += red[64 * e + lane].x;
            t.y += red[64 * e + lane].y;
        }
        v[lane] = zmul(t, dinv);
    }
    __syncthreads();
    const double2 m = block_xt_times(xt, v, tid);
    if ((tid & 3) == 0) red[tid >> 2] = m;
    __syncthreads();
    if (wv == 1 && fin.grad) {  // the order of reduce_config
        double sum = 0.0;
        for (int c = lane; c < nchunk; c += 64) sum += fin.lpart[(size_t)c * S + s];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
        if (lane == 0) fin.loss[s] = fin.lscale * sum;
    }
    if (wv != 0) return;
    const double2 x = red[lane];
    // 2 Re(mu I / (j w C^2)) = 2 Im(mu I) / (w C^2); a kFmtInv record has no
    // invalid input and no vanishing pivot
    const double gk = 2.0 * (x.x * Ik.y + x.y * Ik.x) / (w * ck * ck);
    if (lane < n) {
        if (fin.grad) fin.grad[(size_t)s * n + lane] = 0.0 + gk;  // see replay_system
        else gsys[(size_t)s * n + lane] = gk;
        if (mu) mu[(size_t)s * n + lane] = x;
    }
    const bool any = __ballot(lane < n && !isfinite(gk)) != 0;
    if ((any || status_in != status) && lane == 0) status[s] = flag | (any ? COSIM_SYS_NONFINITE : 0);
}

__global__ __launch_bounds__(256, 2) void k_replay64(
    int n, int S, int F, GJFactor fac, const double *__restrict__ C, const double *__restrict__ omega,
    const double2 *__restrict__ I, const double2 *__restrict__ rpart, int nchunk, double rscale,
    double *__restrict__ gsys, double2 *__restrict__ mu, int32_t *__restrict__ status,
    const int32_t *__restrict__ status_in, FinalSums fin) {
    replay64_system(blockIdx.x, n, S, F, fac, C, omega, I, rpart, nchunk, rscale, gsys, mu, status,
                    status_in, fin);
}
__global__ __launch_bounds__(256, 3) void k_replay64_group(SmallGroup g) {
    const int sg = blockIdx.x;
    const SmallInst &e = g.in[group_member(g, sg)];
    if (e.S > kFewSystems) return;  // whole workgroup
    replay64_system(sg - e.s0, e.n, e.S, e.F, e.fac, e.C, e.omega, e.I, e.rpart, e.nchunk, e.rscale,
                    e.gsys, e.mu, e.status, e.status, FinalSums{});
}

template <int NP>
__global__ __launch_bounds__(256) void k_replay_adjoint(int n, int S, int F, GJFactor fac,
                                                        const double *__restrict__ C,
                                                        const double *__restrict__ omega,
                                                        const double2 *__restrict__ I,
                                                        const double2 *__restrict__ rpart,
                                                        int nchunk, double rscale,
                                                        double *__restrict__ gsys,
                                                        double2 *__restrict__ mu,
                                                        int32_t *__restrict__ status,
                                                        const int32_t *__restrict__ status_in,
                                                        FinalSums fin) {
    const int s = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (s >= S) return;  // whole wave; no block-level synchronisation below
    replay_system<NP>(s, n, S, F, fac, C, omega, I, rpart, nchunk, rscale, gsys, mu, status, status_in,
                      fin);
}

template <int NP>
__global__ __launch_bounds__(256) void k_replay_adjoint_group(SmallGroup g, int S) {
    const int sg = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (sg >= S) return;
    const SmallInst &e = g.in[group_member(g, sg)];
    if (NP == 64 && e.S <= kFewSystems) return;  // whole wave: k_replay64_group's
    replay_system<NP>(sg - e.s0, e.n, e.S, e.F, e.fac, e.C, e.omega, e.I, e.rpart, e.nchunk,
                      e.rscale, e.gsys, e.mu, e.status, e.status, FinalSums{});
}

// One block per configuration b: dL/dC_b summed over frequencies per loop, and
// the loss over frequencies and P-chunks, each thread taking every kTR-th
// partial loss, the lanes of a wave combined by a fixed shuffle tree and the
// waves in order (every order is fixed, so repeated calls agree bit for bit;
// up to 64 partial losses it is the sum of the first wave alone, as
// replay_system forms it).
constexpr int kTR = 256;
__device__ __forceinline__ void reduce_config(int b, int n, int B, int F, int nchunk,
                                              const double *__restrict__ gsys,
                                              const double *__restrict__ lpart, double lscale,
                                              double *__restrict__ grad,
                                              double *__restrict__ loss) {
    __shared__ double sw[kTR / 64];
    const int S = B * F;
    double part = 0.0;
    if (loss) {
        const int m = F * nchunk;
#pragma unroll 4
        for (int e = threadIdx.x; e < m; e += kTR) {
            const int c = e / F, f = e - c * F;  // consecutive lanes: consecutive f
            part += lpart[(size_t)c * S + (size_t)b * F + f];
        }
    }
    if (grad) {
        for (int k = threadIdx.x; k < n; k += kTR) {
            double acc = 0.0;
#pragma unroll 4
            for (int f = 0; f < F; ++f) acc += gsys[((size_t)b * F + f) * n + k];
            grad[(size_t)b * n + k] = acc;
        }
    }
    if (loss) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
        if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = part;
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 1; w < kTR / 64; ++w) part += sw[w];
            loss[b] = lscale * part;
        }
    }
}

__global__ __launch_bounds__(kTR) void k_reduce(int n, int B, int F, int nchunk,
                                               const double *__restrict__ gsys,
                                               const double *__restrict__ lpart, double lscale,
                                               double *__restrict__ grad,
                                               double *__restrict__ loss) {
    reduce_config(blockIdx.x, n, B, F, nchunk, gsys, lpart, lscale, grad, loss);
}

__global__ __launch_bounds__(kTR) void k_reduce_group(ReduceGroup g) {
    const int bg = blockIdx.x;
    int i = 0;
    while (i + 1 < g.count && bg >= g.in[i + 1].b0) ++i;
    const ReduceInst &e = g.in[i];
    reduce_config(bg - e.b0, e.n, e.B, e.F, e.nchunk, e.gsys, e.lpart, e.lscale, e.grad, e.loss);
}

template <bool ADJ>
hipError_t launch_gj(int NP, int n, int S, int F, const double *M, const double *R,
                     const double *phi, const double *C, const double *omega, const double2 *Iin,
                     const double2 *rpart, int nchunk, double rscale, double2 *Iout,
                     double *gsys, int32_t *status, bool or_status, GJFactor fac,
                     hipStream_t st) {
    switch (NP) {
        case 32:
            hipLaunchKernelGGL((k_gj<32, ADJ>), dim3(S), dim3(GJShape<32>::BLOCK), 0, st, n, S,
                               F, M, R, phi, C, omega, Iin, rpart, nchunk, rscale, Iout, gsys,
                               status, or_status, fac);
            break;
        case 64:
            hipLaunchKernelGGL((k_gj<64, ADJ>), dim3(S), dim3(GJShape<64>::BLOCK), 0, st, n, S,
                               F, M, R, phi, C, omega, Iin, rpart, nchunk, rscale, Iout, gsys,
                               status, or_status, fac);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_solve_forward(int NP, int n, int S, int F, const double *M_d,
                                const double *R_d, const double *phi_d, const double *C_d,
                                const double *omega_d, double2 *I_d, int32_t *status_d,
                                GJFactor fac, hipStream_t st) {
    return launch_gj<false>(NP, n, S, F, M_d, R_d, phi_d, C_d, omega_d, nullptr, nullptr, 0, 0.0,
                            I_d, nullptr, status_d, false, fac, st);
}

hipError_t launch_ldl(int NP, int n, int S, int F, const double *M_d, const double *R_d,
                      const double *C_d, const double *omega_d, const double *phi_d, GJFactor fac,
                      double2 *I_d, int32_t *status_d, int32_t *rec_status_d, hipStream_t st) {
    const dim3 grid((S + 3) / 4);
    switch (NP) {
        case 32:
            if (S <= kOneRound)
                hipLaunchKernelGGL(k_small32<2>, dim3(S), dim3(64), 0, st, n, S, F, M_d, R_d, C_d,
                                   omega_d, phi_d, fac, I_d, status_d, rec_status_d);
            else
                hipLaunchKernelGGL(k_small32<3>, dim3(S), dim3(64), 0, st, n, S, F, M_d, R_d, C_d,
                                   omega_d, phi_d, fac, I_d, status_d, rec_status_d);
            return hipGetLastError();
        case 64:
            if (S <= kFewSystems) {
                hipLaunchKernelGGL(k_small64, dim3(S), dim3(256), 0, st, n, S, F, M_d, R_d, phi_d,
                                   C_d, omega_d, fac, I_d, status_d, rec_status_d);
                return hipGetLastError();
            }
            if (S <= kOneRound) {
                hipLaunchKernelGGL((k_ldl<64, true>), grid, dim3(256), 0, st, n, S, F, M_d, R_d,
                                   C_d, omega_d, phi_d, fac, I_d, status_d);
            } else {
                hipLaunchKernelGGL((k_ldl<64, false>), grid, dim3(256), 0, st, n, S, F, M_d, R_d,
                                   C_d, omega_d, phi_d, fac, I_d, status_d);
                hipLaunchKernelGGL(k_forward<64>, grid, dim3(256), 0, st, n, S, fac, I_d, status_d);
            }
            break;
        default:
            return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_gj_fallback<64>, dim3((S + kFbSystems - 1) / kFbSystems),
                       dim3(GJShape<64>::BLOCK), 0, st, n, S, F, M_d, R_d, phi_d, C_d, omega_d, I_d,
                       status_d, fac, rec_status_d);
    return hipGetLastError();
}

hipError_t launch_replay_adjoint(int NP, int n, int S, int F, GJFactor fac, const double *C_d,
                                 const double *omega_d, double2 *I_d, const double2 *rpart_d,
                                 int nchunk, double rscale, double *gsys_d, double2 *mu_d,
                                 int32_t *status_d, hipStream_t st, const FinalSums &fin,
                                 const int32_t *status_in_d) {
    if (!status_in_d) status_in_d = status_d;
    const dim3 grid((S + 3) / 4);
    switch (NP) {
        case 32:
            hipLaunchKernelGGL(k_replay_adjoint<32>, grid, dim3(256), 0, st, n, S, F, fac, C_d,
                               omega_d, I_d, rpart_d, nchunk, rscale, gsys_d, mu_d, status_d,
                               status_in_d, fin);
            break;
        case 64:
            // a call's factorisation and its replay have the same systems
            if (S <= kFewSystems) {
                hipLaunchKernelGGL(k_replay64, dim3(S), dim3(256), 0, st, n, S, F, fac, C_d, omega_d,
                                   I_d, rpart_d, nchunk, rscale, gsys_d, mu_d, status_d, status_in_d,
                                   fin);
                break;
            }
            hipLaunchKernelGGL(k_replay_adjoint<64>, grid, dim3(256), 0, st, n, S, F, fac, C_d,
                               omega_d, I_d, rpart_d, nchunk, rscale, gsys_d, mu_d, status_d,
                               status_in_d, fin);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_solve_adjoint(int NP, int n, int S, int F, const double *M_d,
                                const double *R_d, const double *C_d, const double *omega_d,
                                const double2 *I_d, const double2 *rpart_d, int nchunk,
                                double rscale, double *gsys_d, double2 *mu_d, int32_t *status_d,
                                bool or_status, hipStream_t st) {
    return launch_gj<true>(NP, n, S, F, M_d, R_d, nullptr, C_d, omega_d, I_d, rpart_d, nchunk,
                           rscale, mu_d, gsys_d, status_d, or_status, GJFactor{}, st);
}

hipError_t launch_reduce(int n, int B, int F, int nchunk, const double *gsys_d,
                         const double *lpart_d, double lscale, double *grad_d, double *loss_d,
                         hipStream_t st) {
    hipLaunchKernelGGL(k_reduce, dim3(B), dim3(kTR), 0, st, n, B, F, nchunk, gsys_d, lpart_d,
                       lscale, grad_d, loss_d);
    return hipGetLastError();
}

hipError_t launch_reduce_group(const ReduceGroup &g, int Btot, hipStream_t st) {
    if (Btot <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_group, dim3(Btot), dim3(kTR), 0, st, g);
    return hipGetLastError();
}

hipError_t launch_small_group(int NP, const SmallGroup &g, int S, SmallPhase phase,
                              hipStream_t st) {
    if (S <= 0) return hipSuccess;
    const dim3 wave_grid((S + 3) / 4);
    if (NP != 32 && NP != 64) return hipErrorInvalidValue;
    bool few = false, many = false;  // 33 to 64 loops: members on either side of kFewSystems
    for (int i = 0; i < g.count; ++i) (g.in[i].S <= kFewSystems ? few : many) = true;
    switch (phase) {
        case SmallPhase::Factor:
            if (NP == 32) {
                if (S <= kOneRound)
                    hipLaunchKernelGGL(k_small32_group<2>, dim3(S), dim3(64), 0, st, g);
                else
                    hipLaunchKernelGGL(k_small32_group<3>, dim3(S), dim3(64), 0, st, g);
                break;
            }
            if (few) hipLaunchKernelGGL(k_small64_group, dim3(S), dim3(256), 0, st, g);
            if (!many) break;
            if (S <= kOneRound) {
                hipLaunchKernelGGL((k_ldl_group<64, true>), wave_grid, dim3(256), 0, st, g, S);
            } else {
                hipLaunchKernelGGL((k_ldl_group<64, false>), wave_grid, dim3(256), 0, st, g, S);
                hipLaunchKernelGGL(k_forward_group<64>, wave_grid, dim3(256), 0, st, g, S);
            }
            hipLaunchKernelGGL(k_gj_group<64>, dim3((S + kFbSystems - 1) / kFbSystems),
                               dim3(GJShape<64>::BLOCK), 0, st, g, S);
            break;
        case SmallPhase::Adjoint:
            if (NP == 32) {
                hipLaunchKernelGGL(k_replay_adjoint_group<32>, wave_grid, dim3(256), 0, st, g, S);
                break;
            }
            if (few) hipLaunchKernelGGL(k_replay64_group, dim3(S), dim3(256), 0, st, g);
            if (many)
                hipLaunchKernelGGL(k_replay_adjoint_group<64>, wave_grid, dim3(256), 0, st, g, S);
            break;
    }
    return hipGetLastError();
}

}  // namespace cosim
