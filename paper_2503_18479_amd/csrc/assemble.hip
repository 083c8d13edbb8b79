// One-time operator assembly on gfx950: the Biot-Savart field matrix G and
// the Neumann inductance matrix M.  Both are plain-ALU kernels (FP64 sqrt,
// division and asinh dominate); they run once per geometry and point set, on
// the loops with straight runs of segments merged (merge_straight in abi.cpp).
#include <type_traits>

#include "epilogue.h"
#include "internal.h"

namespace cosim {

namespace {

// Round-to-nearest-even float -> bf16 bits (finite inputs).
__device__ inline uint16_t bf16_rne(float x) {
    uint32_t u = __float_as_uint(x);
    uint32_t lsb = (u >> 16) & 1u;
    u += 0x7FFFu + lsb;
    return (uint16_t)(u >> 16);
}
__device__ inline float bf16_to_f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// 1/x from the hardware reciprocal and two Newton steps (about 1 ulp), by
// division outside the range where they are safe.
__device__ inline double rcp_safe(double x) {
    if (__builtin_expect(x > 1e-280 && x < 1e280, 1)) {
        double r = __builtin_amdgcn_rcp(x);
        r = fma(r, fma(-x, r, 1.0), r);
        return fma(r, fma(-x, r, 1.0), r);
    }
    return 1.0 / x;
}

// Vector from a point to a vertex, its length and the reciprocal of that.
struct Arm {
    double x, y, z, l, il;
};
__device__ inline Arm arm(double x, double y, double z) {
    Arm a{x, y, z, 0.0, 0.0};
    mag_inv(fma(x, x, fma(y, y, z * z)), a.l, a.il);
    return a;
}

// Cartesian component `comp` (0 x, 1 y, 2 z) of the field per ampere of the
// straight filament v1 -> v2 at point p.  With a = v1 - p, b = v2 - p:
//   mu0/(4pi) (a x b)_comp (|a|+|b|) / (|a||b| (|a||b| + a.b)).
// For a.b < 0 the last factor is evaluated as (|a||b| - a.b)/|a x b|^2, its
// equal that does not cancel beside the filament.
__device__ inline double b_filament(int comp, const Arm &a, const Arm &b) {
    const double cx = a.y * b.z - a.z * b.y;
    const double cy = a.z * b.x - a.x * b.z;
    const double cz = a.x * b.y - a.y * b.x;
    const double dot = a.x * b.x + a.y * b.y + a.z * b.z;
    const double ab = a.l * b.l;
    const double num = dot >= 0.0 ? 1.0 : ab - dot;
    const double den = dot >= 0.0 ? ab + dot : cx * cx + cy * cy + cz * cz;
    const double cc = comp == 2 ? cz : comp == 1 ? cy : cx;
    return cc * (a.l + b.l) * (num * rcp_safe(den)) * (a.il * b.il);
}

// Block: 64 points x one chunk of KC = 32 or 64 loops (grid: points x chunks),
// 4 waves.  Wave w evaluates loops w, w+4, ... for the 64 points of its lanes
// (every lane of a wave walks the same vertices, so each vertex load is one
// cache line for the whole wave); the tile [64][KC] is staged in LDS and written
// out in 16-byte stores, row-major and transposed, so that a row segment of G
// and a column segment of each transposed copy are contiguous runs.  Copies
// the plan did not ask for are null and skipped.
//   FP64 vector work and the stores take about the same time: 256 loops of
// four segments at 65,536 points, every copy (539 MB), 224 us (square root and
// two divisions per segment, 8-byte and smaller stores: 261 us; 32 segments per
// loop: 1.81 ms).
constexpr int kGPts = 64;

template <int KC>
__global__ __launch_bounds__(256) void k_assemble_G(int n, int NP, int P, int P_pad, int comp,
                                                    const int32_t *__restrict__ seg_off,
                                                    const double *__restrict__ verts,
                                                    const double *__restrict__ pts,
                                                    double *__restrict__ G64,
                                                    float *__restrict__ G32,
                                                    uint16_t *__restrict__ Ghi,
                                                    uint16_t *__restrict__ Glo,
                                                    double *__restrict__ GT64,
                                                    float *__restrict__ GT32,
                                                    uint16_t *__restrict__ GThi,
                                                    uint16_t *__restrict__ GTlo) {
    __shared__ double tile[kGPts][KC + 1];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int p0 = blockIdx.x * kGPts, k0 = blockIdx.y * KC;
    const int p = p0 + lane;
    double px = 0.0, py = 0.0, pz = 0.0;
    if (p < P) {
        px = pts[3 * (size_t)p + 0];
        py = pts[3 * (size_t)p + 1];
        pz = pts[3 * (size_t)p + 2];
    }
    for (int kk = wave; kk < KC; kk += 4) {
        const int k = k0 + kk;
        double acc = 0.0;
        if (k < n && p < P) {
            const int v0 = seg_off[k], v1 = seg_off[k + 1];
            // distances are shared by neighbouring segments
            const Arm first = arm(verts[3 * v0] - px, verts[3 * v0 + 1] - py, verts[3 * v0 + 2] - pz);
            Arm a = first;
            for (int v = v0 + 1; v < v1; ++v) {
                const Arm b = arm(verts[3 * v] - px, verts[3 * v + 1] - py, verts[3 * v + 2] - pz);
                acc += b_filament(comp, a, b);
                a = b;
            }
            acc += b_filament(comp, a, first);  // closing segment
            acc *= kMu0Over4Pi;
        }
        tile[lane][kk] = acc;
    }
    __syncthreads();
    // NV consecutive entries of the tile's rows (TR: columns) per thread, E
    // such runs per row; P_pad is a multiple of 64, so every row exists
    auto split = [](double g, uint16_t &hi, uint16_t &lo) {
        const float g32 = (float)g;
        hi = bf16_rne(g32);
        lo = bf16_rne(g32 - bf16_to_f(hi));
    };
    auto put = [&](auto tr, double *__restrict__ o64, float *__restrict__ o32,
                   uint16_t *__restrict__ oh, uint16_t *__restrict__ ol) {
        constexpr bool TR = decltype(tr)::value;
        constexpr int ROWS = TR ? KC : kGPts, COLS = TR ? kGPts : KC;
        const size_t ld = TR ? (size_t)P_pad : (size_t)NP;
        const size_t o0 = TR ? (size_t)k0 * ld + p0 : (size_t)p0 * ld + k0;
        auto at = [&](int r, int c) { return TR ? tile[c][r] : tile[r][c]; };
        if (o64)
            for (int e = threadIdx.x; e < ROWS * COLS / 2; e += 256) {
                const int r = e / (COLS / 2), c = 2 * (e % (COLS / 2));
                *(double2 *)(o64 + o0 + r * ld + c) = make_double2(at(r, c), at(r, c + 1));
            }
        if (o32)
            for (int e = threadIdx.x; e < ROWS * COLS / 4; e += 256) {
                const int r = e / (COLS / 4), c = 4 * (e % (COLS / 4));
                *(float4 *)(o32 + o0 + r * ld + c) =
                    make_float4((float)at(r, c), (float)at(r, c + 1), (float)at(r, c + 2),
                                (float)at(r, c + 3));
            }
        if (oh)
            for (int e = threadIdx.x; e < ROWS * COLS / 8; e += 256) {
                const int r = e / (COLS / 8), c = 8 * (e % (COLS / 8));
                __attribute__((aligned(16))) uint16_t h[8], l[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) split(at(r, c + j), h[j], l[j]);
                auto pack = [](const uint16_t *v) {
                    return make_uint4(v[0] | (uint32_t)v[1] << 16, v[2] | (uint32_t)v[3] << 16,
                                      v[4] | (uint32_t)v[5] << 16, v[6] | (uint32_t)v[7] << 16);
                };
                *(uint4 *)(oh + o0 + r * ld + c) = pack(h);
                *(uint4 *)(ol + o0 + r * ld + c) = pack(l);
            }
    };
    put(std::false_type{}, G64, G32, Ghi, Glo);
    put(std::true_type{}, GT64, GT32, GThi, GTlo);
}

// ----------------------------------------------------------------------------
// Neumann mutual inductance of two straight filaments x1->x2, y1->y2 with the
// kernel 1/sqrt(|r - r'|^2 + a^2):
//   parallel:      Grover's closed form, four corner terms of
//                  F(u) = u asinh(u/d) - sqrt(u^2 + d^2); for d = 0 (collinear)
//                  F(u) = |u| ln|u| (the terms linear in |u| cancel);
//   perpendicular: exactly zero;
//   otherwise:     inner integral along y in closed form, outer integral along x
//                  by composite Gauss-Legendre on graded panels (neumann_skew).
// ----------------------------------------------------------------------------
struct V3 {
    double x, y, z;
};
__device__ inline V3 sub(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline double dot3(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline V3 scl(V3 a, double s) { return {a.x * s, a.y * s, a.z * s}; }
__device__ inline V3 add(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }

__device__ inline double cornerF(double u, double d) {
    if (d > 0.0) return u * asinh(u / d) - sqrt(u * u + d * d);
    double au = fabs(u);
    return au > 0.0 ? au * log(au) : 0.0;
}

__device__ inline V3 cross(V3 a, V3 b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}

// Integral over x = x1 + s u, 0 <= s <= L1, of the potential of the filament
// y1 -> y2 = y1 + L2 v (u, v unit, c = u.v, s2 = |u x v|^2 > 0):
//   f(s) = asinh((L2 - t0)/r) + asinh(t0/r),
// t0 the projection on the filament, r^2 = rho^2 + a^2 with rho the distance
// from its line; far from the filament, where the two terms cancel, as
// log(1 + 2 L2 / (R1 + R2 - L2)), R the distances to its ends.
//   f is singular at complex s only: c_j +- i d_j for the projections of the
// two ends (d = sqrt(distance^2 + a^2)) and, if the filament holds its point,
// for the closest approach of the lines (d = sqrt(distance^2 + a^2) / |u x v|;
// past an end the logarithms of r cancel).  A panel is no longer than its
// distance from the nearest of them, so 16 nodes leave an error of 4.2^-32 of
// the panel whatever the filaments' lengths are: panels grow geometrically
// away from a near crossing or a shared corner (about 2 log2(L / d) of them)
// and a filament seen from afar takes one.  Panels of one length, a quarter of
// the ends' distances and at most 64, lost all but 2 to 8 digits where whole
// sides cross or meet at a thin wire's radius, and took longer (plans of 64
// circles of 64 segments 8.5 ms against 2.1, of 64 turned squares 0.40 against
// 0.18; M of parallel squares does not come here).
__device__ double neumann_skew(V3 x1, V3 u, double L1, V3 y1, V3 v, double L2, double c, double s2,
                               double a, const GLRule &gl) {
    const V3 w0 = sub(x1, y1);
    const double p = dot3(w0, u), q = dot3(w0, v), a2 = a * a;
    double sc[3], sd[3];
    const double tc = (q - c * p) / s2;
    sc[0] = (c * q - p) / s2;
    const V3 gap = sub(add(w0, scl(u, sc[0])), scl(v, tc));
    sd[0] = tc >= 0.0 && tc <= L2 ? sqrt((dot3(gap, gap) + a2) / s2) : 1e300;
    const V3 e0 = sub(y1, x1), e1 = add(e0, scl(v, L2));
    sc[1] = dot3(e0, u);
    sc[2] = dot3(e1, u);
    const V3 h0 = sub(e0, scl(u, sc[1])), h1 = sub(e1, scl(u, sc[2]));
    sd[1] = sqrt(dot3(h0, h0) + a2);
    sd[2] = sqrt(dot3(h1, h1) + a2);
    // touching filaments (a = 0) would need panels without end: at least 2^-40 L1
    const double hmin = L1 * 0x1p-40;
    double acc = 0.0, s = 0.0;
    for (int k = 0; k < 400 && s < L1; ++k) {
        double h = L1 - s;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double g = sc[j] - s, d = sd[j];
            // behind s the distance is that of s; ahead, that of the panel's end,
            // and once the panel reaches past it, d
            h = fmin(h, d >= h ? h : g <= 0.0 ? sqrt(g * g + d * d) : d < g ? (g * g + d * d) / (2.0 * g) : d);
        }
        const bool last = fmax(h, hmin) >= L1 - s;
        h = last ? L1 - s : fmax(h, hmin);
        double part = 0.0;
        for (int i = 0; i < kGLOrder; ++i) {
            const V3 w = add(w0, scl(u, s + 0.5 * h * (1.0 + gl.x[i])));
            const double t0 = dot3(w, v), t1 = L2 - t0;
            const V3 n = cross(w, v);  // |n| = rho, without the cancellation of |w|^2 - t0^2
            const double r2 = dot3(n, n) + a2;
            const double R = sqrt(fma(t0, t0, r2)) + sqrt(fma(t1, t1, r2));
            double f;
            if (R >= 2.0 * L2) {
                f = log1p(2.0 * L2 / (R - L2));
            } else {
                double r = sqrt(r2);
                if (r == 0.0) r = 1e-300;
                f = asinh(t1 / r) + asinh(t0 / r);
            }
            part += gl.w[i] * f;
        }
        acc += 0.5 * h * part;
        s = last ? L1 : s + h;
    }
    return acc;
}

__device__ double neumann_pair(V3 x1, V3 x2, V3 y1, V3 y2, double a, const GLRule &gl) {
    V3 du = sub(x2, x1), dv = sub(y2, y1);
    const double L1 = sqrt(dot3(du, du)), L2 = sqrt(dot3(dv, dv));
    const V3 u = scl(du, 1.0 / L1), v = scl(dv, 1.0 / L2);
    const double c = dot3(u, v);
    const V3 cr = cross(u, v);
    const double s2 = dot3(cr, cr);
    if (s2 < 1e-24) {
        const double sgn = c > 0.0 ? 1.0 : -1.0;
        const V3 w = sub(y1, x1);
        const double along = dot3(w, u);
        const V3 perp = sub(w, scl(u, along));
        double d = sqrt(dot3(perp, perp) + a * a);
        if (d < 1e-12 * fmax(L1, L2)) d = 0.0;
        const double b1 = along, b2 = along + sgn * L2;
        const double lo = fmin(b1, b2), hi = fmax(b1, b2);
        const double val = cornerF(L1 - lo, d) - cornerF(L1 - hi, d) - cornerF(-lo, d) +
                           cornerF(-hi, d);
        return kMu0Over4Pi * sgn * val;
    }
    if (fabs(c) < 1e-12) return 0.0;
    return kMu0Over4Pi * c * neumann_skew(x1, u, L1, y1, v, L2, c, s2, a, gl);
}

// One group of TP threads per unordered loop pair (k <= l), striding over the
// segment pairs; a fixed-order tree reduction (deterministic).  TP follows the
// largest number of segment pairs: a wave for up to 64 (four-sided loops have
// 16), else a whole workgroup of up to 1,024 threads.
template <int TB, int TP>
__global__ __launch_bounds__(TB) void k_assemble_M(int n, const int32_t *__restrict__ seg_off,
                                                   const double *__restrict__ verts,
                                                   const double *__restrict__ wire_a, GLRule gl,
                                                   double *__restrict__ M) {
    __shared__ double red[TB];
    // linear pair index -> (k, l), k <= l, row-major over the upper triangle:
    // row k starts at k (2 n - k + 1) / 2
    const long long idx = (long long)blockIdx.x * (TB / TP) + threadIdx.x / TP;
    const long long pairs = (long long)n * (n + 1) / 2;
    const bool in = idx < pairs;
    const double m = 2.0 * n + 1.0;
    int k = (int)((m - sqrt(fmax(m * m - 8.0 * (double)idx, 0.0))) * 0.5);
    k = min(max(k, 0), n - 1);
    auto row = [&](long long r) { return r * (2LL * n - r + 1) / 2; };
    while (in && row(k) > idx) --k;
    while (in && k + 1 < n && row(k + 1) <= idx) ++k;
    double acc = 0.0;
    int l = 0;
    if (in) {
        l = k + (int)(idx - row(k));
        const int ka = seg_off[k], kn = seg_off[k + 1] - ka;
        const int la = seg_off[l], ln = seg_off[l + 1] - la;
        const double a = (k == l) ? wire_a[k] : 0.0;
        for (int e = threadIdx.x % TP; e < kn * ln; e += TP) {
            const int s = e / ln, t = e - s * ln;
            const int s2 = (s + 1 == kn) ? 0 : s + 1;
            const int t2 = (t + 1 == ln) ? 0 : t + 1;
            const double *p = verts + 3 * (size_t)(ka + s);
            const double *p2 = verts + 3 * (size_t)(ka + s2);
            const double *q = verts + 3 * (size_t)(la + t);
            const double *q2 = verts + 3 * (size_t)(la + t2);
            acc += neumann_pair({p[0], p[1], p[2]}, {p2[0], p2[1], p2[2]}, {q[0], q[1], q[2]},
                                {q2[0], q2[1], q2[2]}, a, gl);
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = TP / 2; w > 0; w >>= 1) {
        if ((int)(threadIdx.x % TP) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (in && threadIdx.x % TP == 0) {
        M[(size_t)k * n + l] = red[threadIdx.x];
        M[(size_t)l * n + k] = red[threadIdx.x];
    }
}

}  // namespace

hipError_t launch_assemble_G(int n, int NP, int P, int P_pad, int comp, const int32_t *seg_off_d,
                             const double *verts_d, const double *pts_d, double *G64,
                             float *G32, uint16_t *Ghi, uint16_t *Glo, double *GT64,
                             float *GT32, uint16_t *GThi, uint16_t *GTlo, hipStream_t st) {
    if (P_pad % kGPts != 0 || NP % 32 != 0 || (NP > 32 && NP % 64 != 0)) return hipErrorInvalidValue;
    const unsigned blocks = (unsigned)(P_pad / kGPts);
    if (NP == 32)
        hipLaunchKernelGGL(k_assemble_G<32>, dim3(blocks), dim3(256), 0, st, n, NP, P, P_pad, comp,
                           seg_off_d, verts_d, pts_d, G64, G32, Ghi, Glo, GT64, GT32, GThi, GTlo);
    else
        hipLaunchKernelGGL(k_assemble_G<64>, dim3(blocks, NP / 64), dim3(256), 0, st, n, NP, P,
                           P_pad, comp, seg_off_d, verts_d, pts_d, G64, G32, Ghi, Glo, GT64, GT32,
                           GThi, GTlo);
    return hipGetLastError();
}

hipError_t launch_assemble_M(int n, int max_segs, const int32_t *seg_off_d, const double *verts_d,
                             const double *wire_a_d, const GLRule &gl, double *M_d,
                             hipStream_t st) {
    const long long pairs = (long long)n * (n + 1) / 2;
    const long long sp = (long long)max_segs * max_segs;
    if (sp <= 64)
        hipLaunchKernelGGL((k_assemble_M<256, 64>), dim3((unsigned)((pairs + 3) / 4)), dim3(256), 0,
                           st, n, seg_off_d, verts_d, wire_a_d, gl, M_d);
    else if (sp <= 256)
        hipLaunchKernelGGL((k_assemble_M<256, 256>), dim3((unsigned)pairs), dim3(256), 0, st, n,
                           seg_off_d, verts_d, wire_a_d, gl, M_d);
    else
        hipLaunchKernelGGL((k_assemble_M<1024, 1024>), dim3((unsigned)pairs), dim3(1024), 0, st, n,
                           seg_off_d, verts_d, wire_a_d, gl, M_d);
    return hipGetLastError();
}

}  // namespace cosim
