// uSARA's denoiser (section "uSARA's handcrafted denoiser"): the prox of
// t ||w . Psi^dagger x||_1 + iota_+(x) for the SARA dictionary
// Psi = [Dirac, db1, ..., db8] / 3 (each basis an orthonormal 2D periodic
// wavelet transform with 4 levels), by sub-iterations of dual forward-backward
// with unit step (||Psi^dagger|| = 1):
//   x_k = max(0, z - Psi v_k),   v_{k+1} = clip(v_k + Psi^dagger x_k, -t w, t w),
// warm-started from the previous call's dual variable, and the reweighting of
// the log-sum penalty, w = rho / (rho + |Psi^dagger x|).
//
// Filters: the minimum-phase Daubechies low-pass filter with p vanishing
// moments (2p taps) is the spectral factor h(z) = sqrt(2) ((1+z)/2)^p Q(z)/Q(1)
// with Q's roots the roots outside the unit circle of z^{p-1} P_p((2-z-1/z)/4),
// P_p(y) = sum_{k<p} C(p-1+k, k) y^k; computed on the host (roots of P_p in y
// by Durand-Kerner in long double, then mapped to z) and checked for
// orthonormality before use. High-pass g[t] = (-1)^t h[L-1-t].
//
// Transform (all 8 wavelet bases in one launch per level): one level on an n x n
// block (row stride N) in both directions, each
// a[k] = sum_t h[t] x[(2k+t) mod n], d[k] = sum_t g[t] x[(2k+t) mod n],
// low half first; the top-left block goes on to the next level. The analysis
// writes only the low-low block for the next level and finalises every
// other coefficient in place: the dual update (clip), the new weight, or the
// plain coefficient. Synthesis runs the adjoint from the coarsest level, reading
// the coarse block from the previous level's result and the details from the
// coefficients; its last level sums the 8 bases and the Dirac part and
// applies max(0, z - .) with the Dirac dual update fused.
//
// Bound: memory. A sub-iteration cannot do without reading and writing the nine
// dual planes and reading the nine weights (470 MB in FP32 at 2048^2 with z and
// x: 97 us at the rate of a copy). One pass per level and both directions in LDS
// leave the low-low blocks and the tiles' borders as the only other traffic; with a
// pass per direction and a plane in between for every basis a sub-iteration moved
// 1.53 GB (counted) in 16 launches and took 370 us, this form moves 0.92 GB in 8 and
// takes 189 us (finest level 59 us analysis and 56 us synthesis, the three others
// 75 us).
#include <cmath>
#include <complex>
#include <limits>
#include <utility>

#include "ri_internal.h"

namespace ri {

namespace {

constexpr int NW = 8;          // wavelet bases (db1 .. db8)
constexpr int LEVELS = 4;
constexpr int LMAX = 16;

__constant__ double c_h64[NW][LMAX];
__constant__ double c_g64[NW][LMAX];
__constant__ float c_h32[NW][LMAX];
__constant__ float c_g32[NW][LMAX];

template <typename T> __device__ __forceinline__ T fh(int b, int t);
template <typename T> __device__ __forceinline__ T fg(int b, int t);
template <> __device__ __forceinline__ double fh<double>(int b, int t) { return c_h64[b][t]; }
template <> __device__ __forceinline__ double fg<double>(int b, int t) { return c_g64[b][t]; }
template <> __device__ __forceinline__ float fh<float>(int b, int t) { return c_h32[b][t]; }
template <> __device__ __forceinline__ float fg<float>(int b, int t) { return c_g32[b][t]; }

// f(integral_constant<int, i>) for i = 0 .. N-1, unrolled at compile time.
template <typename F, int... I>
__device__ __forceinline__ void static_for_(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) { static_for_(f, std::make_integer_sequence<int, N>{}); }

// 16 bytes of T as one LDS vector load; four elements of memory whose alignment is
// that of one element (coefficients and images may be caller buffers).
template <typename T>
using vec16 = T __attribute__((ext_vector_type(16 / sizeof(T))));
template <typename T>
using vec4 = T __attribute__((ext_vector_type(4)));
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) mem4 {
    vec4<T> v;
};
template <typename T>
__device__ __forceinline__ vec4<T> load4(const T *p) { return reinterpret_cast<const mem4<T> *>(p)->v; }
template <typename T>
__device__ __forceinline__ void store4(T *p, vec4<T> v) { reinterpret_cast<mem4<T> *>(p)->v = v; }

enum { FIN_DUAL = 0, FIN_WEIGHT = 1, FIN_COEF = 2 };
enum { SYN_PROX = 0, SYN_PLAIN = 1, SYN_LEVEL = 2 };

// Finalised coefficient of basis slot j (0 = Dirac) from its transform val
// (unscaled), its dual variable v and weight w.
template <typename T, int FIN>
__device__ __forceinline__ T final_value(T v, T w, T val, T scale, T par) {
    const T cval = val * scale;
    if (FIN == FIN_DUAL) {
        const T lim = par * w;
        return fmin(fmax(v + cval, -lim), lim);
    }
    return FIN == FIN_WEIGHT ? par / (par + fabs(cval)) : cval;
}
template <typename T, int FIN>
__device__ __forceinline__ void finalise(T *dst9, const T *w9, size_t i9, T val, T scale, T par) {
    if (FIN == FIN_DUAL) dst9[i9] = final_value<T, FIN>(dst9[i9], w9[i9], val, scale, par);
    else dst9[i9] = final_value<T, FIN>((T)0, (T)0, val, scale, par);
}

// f(std::integral_constant<int, L>) for the filter length L = 2 (b + 1) of basis b.
template <typename F>
__device__ __forceinline__ void with_length(int b, F &&f) {
    switch (b) {
        case 0: f(std::integral_constant<int, 2>{}); break;
        case 1: f(std::integral_constant<int, 4>{}); break;
        case 2: f(std::integral_constant<int, 6>{}); break;
        case 3: f(std::integral_constant<int, 8>{}); break;
        case 4: f(std::integral_constant<int, 10>{}); break;
        case 5: f(std::integral_constant<int, 12>{}); break;
        case 6: f(std::integral_constant<int, 14>{}); break;
        default: f(std::integral_constant<int, 16>{}); break;
    }
}

// One level in one pass: a workgroup transforms a tile in both directions and
// only coefficients and the low-low block touch memory. A tile has 64 low columns
// (128 columns of the level's block; a quadrant's rows are runs of 256 bytes in
// FP32) and 8 S low rows (16 S rows). The longest filter needs 14 rows and
// columns beyond the tile: with S = 4 1.2 times the work in each direction, about a third of
// the time the memory takes. The analysis runs columns first, so that the
// input goes straight from memory to registers, the synthesis rows first, so that
// the coefficients do.
constexpr int TC = 64;             // low columns of a tile
constexpr int KB = 8;              // low rows of a column strip: one thread's register window
constexpr int APITCH = 2 * TC + 16;

// E consecutive elements from 16-byte-aligned LDS.
template <typename T, int E>
__device__ __forceinline__ void lds_window(const T *p, T (&w)[E]) {
    constexpr int V = 16 / sizeof(T);
#pragma unroll
    for (int i = 0; i < E / V; ++i) {
        const vec16<T> v = reinterpret_cast<const vec16<T> *>(p)[i];
#pragma unroll
        for (int e = 0; e < V; ++e) w[i * V + e] = v[e];
    }
}

// Analysis of one level block (n x n, row stride N; basis stride in_bs, 0 for the
// image): low-low block into out (unless last) and every other coefficient
// finalised into dst9 (slot b + 1).
//   Column pass: thread = one column and one strip of KB low rows, whose
// 2 KB + L - 2 inputs stay in registers (for all bases with ALLB: the finest
// level's bases share their input); both halves' KB outputs go to LDS. 128 S
// threads have the tile's columns, a last wave the 16 columns beyond it.
//   Row pass: thread = four low columns of one row of each half, from 24-element
// windows in LDS (outputs need columns 2 k + t, t < L <= 16); its 16 results are
// finalised as 4-element vectors, whose dual variables and weights were
// asked for before the column pass. SMALL: blocks of n < 8, element by element.
template <typename T, int FIN, int S, bool ALLB, bool SMALL>
__global__ void __launch_bounds__(128 * S + 64)
k_ana(const T *__restrict__ in, int64_t in_bs, T *__restrict__ out, T *dst9, const T *__restrict__ w9, int N, int n,
      int last, T scale, T par) {
    __shared__ __attribute__((aligned(16))) T mid[2 * KB * S * APITCH];
    const int tid = threadIdx.x, half = n >> 1, m = n - 1;
    const bool main = tid < 128 * S;
    const int strip = main ? tid >> 7 : (tid - 128 * S) >> 4;
    const int lc = main ? tid & 127 : 128 + ((tid - 128 * S) & 15);
    const int k0 = (blockIdx.y * S + strip) * KB, gcol = (blockIdx.x * 2 * TC + lc) & m;
    const bool cact = strip < S && k0 < half;
    const int kr = tid >> 4, j = tid & 15;
    const int k = blockIdx.y * KB * S + kr, kc = blockIdx.x * TC + 4 * j;
    const bool ract = main && k < half && kc < half;
    const size_t NN = (size_t)N * N;
    T r[2 * KB + LMAX - 2];
    auto load = [&](const T *src, auto NRc) {
#pragma unroll
        for (int q = 0; q < decltype(NRc)::value; ++q) r[q] = src[(size_t)((2 * k0 + q) & m) * N + gcol];
    };
    auto basis = [&](int b, auto Lc) {
        constexpr int L = decltype(Lc)::value;
        const size_t e0 = (size_t)k * N + kc, dh = (size_t)half * N;
        T *d9 = dst9 + (size_t)(b + 1) * NN;
        const T *l9 = w9 + (size_t)(b + 1) * NN;
        vec4<T> v[4], w[4];
        if (!ALLB && cact) load(in + b * in_bs, std::integral_constant<int, 2 * KB + L - 2>{});
        if (FIN == FIN_DUAL && !SMALL && ract) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q == 0 && !last) continue;
                const size_t p = e0 + (q & 2 ? dh : 0) + (q & 1 ? half : 0);
                v[q] = load4<T>(d9 + p);
                w[q] = load4<T>(l9 + p);
            }
        }
        if (cact) {
            T *lo = mid + strip * KB * APITCH + lc, *hi = lo + KB * S * APITCH;
#pragma unroll
            for (int kk = 0; kk < KB; ++kk) {
                T a = 0, d = 0;
#pragma unroll
                for (int t = 0; t < L; ++t) {
                    a = fma(fh<T>(b, t), r[2 * kk + t], a);
                    d = fma(fg<T>(b, t), r[2 * kk + t], d);
                }
                lo[kk * APITCH] = a;
                hi[kk * APITCH] = d;
            }
        }
        __syncthreads();
        if (ract) {
#pragma unroll
            for (int vh = 0; vh < 2; ++vh) {
                T x[24];
                lds_window<T, 24>(mid + (vh * KB * S + kr) * APITCH + 8 * j, x);
                vec4<T> c[2];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    T a = 0, d = 0;
#pragma unroll
                    for (int t = 0; t < L; ++t) {
                        a = fma(fh<T>(b, t), x[2 * u + t], a);
                        d = fma(fg<T>(b, t), x[2 * u + t], d);
                    }
                    c[0][u] = a;
                    c[1][u] = d;
                }
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const size_t p = e0 + (vh ? dh : 0) + (hh ? half : 0);
                    const bool low = vh == 0 && hh == 0 && !last;
                    if (SMALL) {
                        for (int u = 0; u < 4; ++u)
                            if (kc + u < half) {
                                if (low) out[b * NN + e0 + u] = c[hh][u];
                                else finalise<T, FIN>(d9, l9, p + u, c[hh][u], scale, par);
                            }
                    } else if (low) {
                        store4<T>(out + b * NN + e0, c[hh]);
                    } else {
                        vec4<T> o;
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            o[u] = final_value<T, FIN>(v[2 * vh + hh][u], w[2 * vh + hh][u], c[hh][u], scale, par);
                        store4<T>(d9 + p, o);
                    }
                }
            }
        }
    };
    if (ALLB) {
        if (cact) load(in, std::integral_constant<int, 2 * KB + LMAX - 2>{});
        static_for<NW>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            if (b > 0) __syncthreads();       // the previous basis' windows are read
            basis(b, std::integral_constant<int, 2 * (b + 1)>{});
        });
    } else {
        with_length(blockIdx.z, [&](auto Lc) { basis(blockIdx.z, Lc); });
    }
}

// Dirac slot of the analysis (weights or plain coefficients).
template <typename T, int FIN>
__global__ void k_ana_dirac(const T *__restrict__ x, T *dst9, int64_t n, T scale, T par) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        finalise<T, FIN>(dst9, nullptr, (size_t)i, x[i], scale, par);
}

// Synthesis of one level block (n x n): the coarse block (rows and columns < n/2)
// from low (or from the coefficients at the coarsest level), the rest from
// the coefficients v9 (slot b + 1).
//   Row pass: thread = 8 outputs of one coefficient row, from the 12 elements of
// each half that they need, x[2u + par] = sum_{s2 < L/2} h[par + 2 s2] A[u - s2] +
// g[par + 2 s2] D[u - s2]; the 8 S rows of each half and the L/2 - 1 before them go
// to LDS. Column pass: thread = one column and 16 rows from windows of
// KB + L/2 - 1 elements of each half.
// SYN_LEVEL: to out (basis b = blockIdx.z). ALLB (the finest level): the sum over
// the bases stays in registers, and with the Dirac slot SYN_PLAIN gives
// x = scale * s, SYN_PROX x = max(0, z - scale * s) and the Dirac dual update
// v0 = clip(v0 + scale * x, -t w0, t w0). SMALL: n < 8, element by element.
template <typename T, int MODE>
__device__ __forceinline__ void syn_point(T *v9, const T *w9, const T *z, T *x, size_t p, T sum, T scale, T thr) {
    const T tot = v9[p] + sum;
    if (MODE == SYN_PLAIN) {
        x[p] = scale * tot;
    } else {
        const T xo = fmax((T)0, z[p] - scale * tot);
        x[p] = xo;
        const T lim = thr * w9[p];
        v9[p] = fmin(fmax(v9[p] + scale * xo, -lim), lim);
    }
}

template <typename T, int MODE, int S, bool SMALL>
__global__ void __launch_bounds__(128 * S)
k_syn(T *v9, const T *__restrict__ low, T *__restrict__ out, const T *__restrict__ w9, const T *__restrict__ z, int N,
      int n, int coarsest, T scale, T thr) {
    constexpr bool ALLB = MODE != SYN_LEVEL;
    constexpr int PITCH = 2 * TC;
    __shared__ __attribute__((aligned(16))) T mid[2 * (KB * S + LMAX / 2 - 1) * PITCH];
    const int tid = threadIdx.x, half = n >> 1, hm = half - 1;
    const int j = tid & 15, kbase = blockIdx.y * KB * S, u0 = blockIdx.x * TC + 4 * j;
    const int strip = tid >> 7, col = tid & 127;
    const int i0 = 2 * (kbase + strip * KB), gcol = blockIdx.x * 2 * TC + col;
    const size_t NN = (size_t)N * N;
    T acc[2 * KB] = {};
    auto basis = [&](int b, auto Lc) {
        constexpr int L = decltype(Lc)::value, S2 = L / 2, NR = KB * S + S2 - 1;
        constexpr int NV = 1 + (S2 - 1 + 3) / 4, W0 = 4 * (NV - 1);     // vectors of a window, its elements before u0
        const T *cf = v9 + (size_t)(b + 1) * NN;
        const T *lo = coarsest ? cf : low + b * NN;
        if (u0 < half) {
            for (int rr = tid >> 4; rr < 2 * NR; rr += KB * S) {
                const int vh = rr >= NR ? 1 : 0;
                const int k = (kbase - (S2 - 1) + rr - vh * NR) & hm;
                const T *ra = vh ? cf + (size_t)(half + k) * N : lo + (size_t)k * N;
                const T *rd = cf + (size_t)(vh * half + k) * N + half;
                T wa[4 * NV], wd[4 * NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    const int c0 = u0 - W0 + 4 * q;
                    vec4<T> va, vd;
                    if (SMALL) {
                        for (int e = 0; e < 4; ++e) {
                            va[e] = ra[(c0 + e) & hm];
                            vd[e] = rd[(c0 + e) & hm];
                        }
                    } else {
                        va = load4<T>(ra + (c0 & hm));
                        vd = load4<T>(rd + (c0 & hm));
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        wa[4 * q + e] = va[e];
                        wd[4 * q + e] = vd[e];
                    }
                }
                T x[8];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
#pragma unroll
                    for (int par = 0; par < 2; ++par) {
                        T v = 0;
#pragma unroll
                        for (int s2 = 0; s2 < S2; ++s2) {
                            v = fma(fh<T>(b, par + 2 * s2), wa[u + W0 - s2], v);
                            v = fma(fg<T>(b, par + 2 * s2), wd[u + W0 - s2], v);
                        }
                        x[2 * u + par] = v;
                    }
                }
                T *dst = mid + rr * PITCH + 8 * j;
                constexpr int V = 16 / sizeof(T);
#pragma unroll
                for (int q = 0; q < 8 / V; ++q) {
                    vec16<T> o;
#pragma unroll
                    for (int e = 0; e < V; ++e) o[e] = x[q * V + e];
                    reinterpret_cast<vec16<T> *>(dst)[q] = o;
                }
            }
        }
        __syncthreads();
        T ar[KB + S2 - 1], dr[KB + S2 - 1];
        const T *lp = mid + strip * KB * PITCH + col, *hp = lp + NR * PITCH;
#pragma unroll
        for (int q = 0; q < KB + S2 - 1; ++q) {
            ar[q] = lp[q * PITCH];
            dr[q] = hp[q * PITCH];
        }
#pragma unroll
        for (int u = 0; u < KB; ++u) {
#pragma unroll
            for (int par = 0; par < 2; ++par) {
                T v = acc[2 * u + par];
#pragma unroll
                for (int s2 = 0; s2 < S2; ++s2) {
                    v = fma(fh<T>(b, par + 2 * s2), ar[u - s2 + S2 - 1], v);
                    v = fma(fg<T>(b, par + 2 * s2), dr[u - s2 + S2 - 1], v);
                }
                acc[2 * u + par] = v;
            }
        }
    };
    if (ALLB) {
        static_for<NW>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            if (b > 0) __syncthreads();       // the previous basis' columns are read
            basis(b, std::integral_constant<int, 2 * (b + 1)>{});
        });
    } else {
        with_length(blockIdx.z, [&](auto Lc) { basis(blockIdx.z, Lc); });
    }
    if (gcol >= n) return;
#pragma unroll
    for (int u = 0; u < 2 * KB; ++u) {
        if (i0 + u >= n) break;
        const size_t p = (size_t)(i0 + u) * N + gcol;
        if constexpr (ALLB) syn_point<T, MODE>(v9, w9, z, out, p, acc[u], scale, thr);
        else out[blockIdx.z * NN + p] = acc[u];
    }
}

// The finest level's sum over the bases where their planes were written one by
// one, with the Dirac slot (x may be the first of the planes).
template <typename T, int MODE>
__global__ void __launch_bounds__(256) k_syn_sum(const T *planes, T *v9, const T *__restrict__ w9,
                                                 const T *__restrict__ z, T *x, int64_t n, T scale, T thr) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    T sum = 0;
#pragma unroll
    for (int b = 0; b < NW; ++b) sum += planes[b * n + p];
    syn_point<T, MODE>(v9, w9, z, x, (size_t)p, sum, scale, thr);
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// Filters on the host
// ---------------------------------------------------------------------------
using cld = std::complex<long double>;

// Roots of sum_k a[k] y^k (degree d = a.size() - 1 >= 1) by Durand-Kerner: until a
// sweep moves no root by more than a few roundings of its size (about 1; 13 sweeps
// at most for the filters here), and eight sweeps more, in which the last
// roundings settle (the filters come out the same to the last bit after 2000).
// Waiting for a step below 1e-24, which long double never takes, cost the first
// prox of every context 8.8 ms of host time.
std::vector<cld> poly_roots(const std::vector<long double> &a) {
    const int d = (int)a.size() - 1;
    std::vector<cld> r(d);
    const cld seed(0.4L, 0.9L);
    cld pw(1.0L, 0.0L);
    for (int i = 0; i < d; ++i) { r[i] = pw; pw *= seed; }
    auto eval = [&](cld y) {
        cld v = 0;
        for (int k = d; k >= 0; --k) v = v * y + a[k];
        return v / a[d];
    };
    for (int it = 0, settled = 0; it < 2000 && settled < 8; ++it) {
        long double moved = 0;
        for (int i = 0; i < d; ++i) {
            cld den = 1;
            for (int j = 0; j < d; ++j)
                if (j != i) den *= (r[i] - r[j]);
            const cld step = eval(r[i]) / den;
            r[i] -= step;
            moved = std::max(moved, std::abs(step));
        }
        if (moved <= 4 * std::numeric_limits<long double>::epsilon()) ++settled;
    }
    return r;
}

std::vector<double> daubechies(int p) {
    std::vector<cld> q(1, cld(1.0L, 0.0L));   // Q(z), increasing powers
    if (p > 1) {
        std::vector<long double> a(p);
        long double binom = 1;                 // C(p-1+k, k)
        for (int k = 0; k < p; ++k) {
            a[k] = binom;
            binom = binom * (long double)(p + k) / (long double)(k + 1);
        }
        for (const cld &y : poly_roots(a)) {
            const cld bq = 1.0L - 2.0L * y;
            const cld disc = std::sqrt(bq * bq - 1.0L);
            const cld z = std::abs(bq + disc) > 1.0L ? bq + disc : bq - disc;
            std::vector<cld> nq(q.size() + 1, cld(0));
            for (size_t i = 0; i < q.size(); ++i) {
                nq[i + 1] += q[i];
                nq[i] -= z * q[i];
            }
            q.swap(nq);
        }
    }
    std::vector<long double> h(q.size());
    for (size_t i = 0; i < q.size(); ++i) h[i] = q[i].real();
    for (int k = 0; k < p; ++k) {              // times (1 + z) / 2, p times
        std::vector<long double> nh(h.size() + 1, 0.0L);
        for (size_t i = 0; i < h.size(); ++i) {
            nh[i] += 0.5L * h[i];
            nh[i + 1] += 0.5L * h[i];
        }
        h.swap(nh);
    }
    long double sum = 0;
    for (long double v : h) sum += v;
    std::vector<double> out(h.size());
    for (size_t i = 0; i < h.size(); ++i) out[i] = (double)(h[i] * std::sqrt(2.0L) / sum);
    // orthonormality check: sum_k h[k] h[k + 2m] = delta_m
    for (int m = 0; m < p; ++m) {
        long double dot = 0;
        for (size_t k = 0; k + 2 * m < out.size(); ++k) dot += (long double)out[k] * out[k + 2 * m];
        if (std::fabs((double)dot - (m == 0 ? 1.0 : 0.0)) > 1e-13)
            throw Error(RI_EDEVICE, "Daubechies filter " + std::to_string(p) + " failed its orthonormality check");
    }
    return out;
}

void upload_filters(ri_ctx *c) {
    double h64[NW][LMAX] = {}, g64[NW][LMAX] = {};
    float h32[NW][LMAX] = {}, g32[NW][LMAX] = {};
    for (int b = 0; b < NW; ++b) {
        const std::vector<double> h = daubechies(b + 1);
        const int L = (int)h.size();
        for (int t = 0; t < L; ++t) {
            h64[b][t] = h[t];
            g64[b][t] = (t & 1 ? -1.0 : 1.0) * h[L - 1 - t];
            h32[b][t] = (float)h64[b][t];
            g32[b][t] = (float)g64[b][t];
        }
    }
    RI_CHECK_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_h64), h64, sizeof(h64)));
    RI_CHECK_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_g64), g64, sizeof(g64)));
    RI_CHECK_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_h32), h32, sizeof(h32)));
    RI_CHECK_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_g32), g32, sizeof(g32)));
    (void)c;
}

// launch(S, ALLB, SMALL) for the level block n. The finest level's bases in one
// workgroup (ALLB) read the image once and keep the sum of the synthesis in
// registers; it pays as soon as there is a workgroup per CU, if need be with half
// the tile's rows (S = 2). Five sub-iterations at N = 2048: 924 us in
// FP32 and 1774 us in FP64 against 1248 and 2354 us with a workgroup per basis and
// a sum over the planes; at N = 1024 with S = 2 409 and 533 us against 406 and 686;
// below, the workgroups are too few. Elsewhere the tallest tile that gives every CU
// a workgroup: asking for two or four a CU measured the same within 2%.
template <typename F>
void dispatch_tile(ri_ctx *c, int n, bool finest, F &&launch) {
    const int64_t t4 = (int64_t)cdiv(n, 2 * TC) * cdiv(n, 2 * KB * 4);   // tiles of S = 4
    using std::integral_constant;
    using no = std::false_type;
    using yes = std::true_type;
    const int cus = c->dev.cu_count;
    if (n < 8) launch(integral_constant<int, 1>{}, no{}, yes{});
    else if (finest && t4 >= cus) launch(integral_constant<int, 4>{}, yes{}, no{});
    else if (finest && t4 * 2 >= cus) launch(integral_constant<int, 2>{}, yes{}, no{});
    else if (t4 * NW >= cus) launch(integral_constant<int, 4>{}, no{}, no{});
    else if (t4 * NW * 2 >= cus) launch(integral_constant<int, 2>{}, no{}, no{});
    else launch(integral_constant<int, 1>{}, no{}, no{});
}

// A caller may transform in place, the image lying inside the coefficients. Tiles
// of one launch read what others of it write then, so such an image passes
// through a work array.
template <typename T>
bool inside(const T *x, const T *coef9, int N) {
    const size_t NN = (size_t)N * N;
    return x + NN > coef9 && x < coef9 + 9 * NN;
}
template <typename T>
void copy_image(T *out, const T *x, int N, hipStream_t s) {
    axpby<T>(out, x, (T)1, nullptr, (T)0, (int64_t)N * N, s);
}

// Psi^dagger x into dst9 (FIN selects the dual update, the weights or the plain coefficients).
template <typename T, int FIN>
void analysis(ri_ctx *c, const T *x, T *dst9, T par, bool dirac, hipStream_t s) {
    SaraState &st = c->sara;
    const int N = c->N;
    if (FIN == FIN_COEF && inside<T>(x, dst9, N)) {
        copy_image<T>((T *)st.tmp, x, N, s);   // the second level's output, free until then
        x = (T *)st.tmp;
    }
    const T scale = (T)(1.0 / 3.0);
    T *const buf[2] = {(T *)st.work, (T *)st.tmp};   // the low-low blocks of even and odd levels
    const T *w9 = (const T *)st.w;
    if (dirac)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_ana_dirac<T, FIN>), dim3(1024), dim3(256), 0, s, x, dst9,
                           (int64_t)N * N, scale, par);
    for (int l = 0; l < LEVELS; ++l) {
        const int n = N >> l, last = l == LEVELS - 1 ? 1 : 0;
        const T *in = l == 0 ? x : buf[(l + 1) & 1];
        const int64_t in_bs = l == 0 ? 0 : (int64_t)N * N;
        auto launch = [&](auto Sc, auto ALLBc, auto SMALLc) {
            constexpr int S = decltype(Sc)::value;
            constexpr bool ALLB = decltype(ALLBc)::value;
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_ana<T, FIN, S, ALLB, decltype(SMALLc)::value>),
                               dim3(cdiv(n, 2 * TC), cdiv(n, 2 * KB * S), ALLB ? 1 : NW), dim3(128 * S + 64), 0, s, in,
                               in_bs, buf[l & 1], dst9, w9, N, n, last, scale, par);
        };
        dispatch_tile(c, n, l == 0, launch);
    }
}

// Psi v9 (MODE SYN_PLAIN) or x = max(0, z - Psi v9) with the Dirac dual update (SYN_PROX).
template <typename T, int MODE>
void synthesis(ri_ctx *c, T *v9, const T *z, T *x, T thr, hipStream_t s) {
    SaraState &st = c->sara;
    const int N = c->N;
    const T scale = (T)(1.0 / 3.0);
    T *const buf[2] = {(T *)st.work, (T *)st.tmp};   // the blocks of even and odd levels
    const T *w9 = (const T *)st.w;
    T *const dst = MODE == SYN_PLAIN && inside<T>(x, v9, N) ? buf[0] : x;   // free at the finest level
    for (int l = LEVELS - 1; l >= 0; --l) {
        const int n = N >> l, coarsest = l == LEVELS - 1 ? 1 : 0;
        auto launch = [&](auto Sc, auto ALLBc, auto SMALLc) {
            constexpr int S = decltype(Sc)::value;
            constexpr bool ALLB = decltype(ALLBc)::value;
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_syn<T, ALLB ? MODE : (int)SYN_LEVEL, S, decltype(SMALLc)::value>),
                               dim3(cdiv(n, 2 * TC), cdiv(n, 2 * KB * S), ALLB ? 1 : NW), dim3(128 * S), 0, s, v9,
                               buf[(l + 1) & 1], ALLB ? dst : buf[l & 1], w9, z, N, n, coarsest, scale, thr);
            if (l == 0 && !ALLB)
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_syn_sum<T, MODE>), dim3(cdiv(N * N, 256)), dim3(256), 0, s, buf[0],
                                   v9, w9, z, dst, (int64_t)N * N, scale, thr);
        };
        dispatch_tile(c, n, l == 0, launch);
    }
    if (dst != x) copy_image<T>(x, dst, N, s);
}

}  // namespace

void sara_free(ri_ctx *c) {
    SaraState &st = c->sara;
    dev_free(c, st.v);
    dev_free(c, st.w);
    dev_free(c, st.work);
    dev_free(c, st.tmp);
    const int sub = st.sub_iters;
    st = SaraState{};
    st.sub_iters = sub;
}

void sara_setup(ri_ctx *c, int sub_iters, hipStream_t s) {
    if (c->N % 16 != 0) throw Error(RI_EUNSUPPORTED, "the SARA dictionary needs N divisible by 16");
    SaraState &st = c->sara;
    if (sub_iters > 0) st.sub_iters = sub_iters;
    const size_t eb = c->d.precision == 64 ? sizeof(double) : sizeof(float);
    const size_t NN = (size_t)c->N * c->N;
    if (!st.ready) {
        upload_filters(c);
        st.v = dev_alloc(c, eb * 9 * NN);
        st.w = dev_alloc(c, eb * 9 * NN);
        st.work = dev_alloc(c, eb * NW * NN);
        st.tmp = dev_alloc(c, eb * NW * NN);
        st.ready = true;
    }
    sara_reset(c, s);
}

void sara_reset(ri_ctx *c, hipStream_t s) {
    SaraState &st = c->sara;
    const int64_t n9 = 9 * (int64_t)c->N * c->N;
    if (c->d.precision == 64) {
        fill_real<double>((double *)st.v, n9, 0.0, s);
        fill_real<double>((double *)st.w, n9, 1.0, s);
    } else {
        fill_real<float>((float *)st.v, n9, 0.0f, s);
        fill_real<float>((float *)st.w, n9, 1.0f, s);
    }
}

template <typename T>
void sara_prox(ri_ctx *c, const T *z, T thr, T *x_out, hipStream_t s) {
    SaraState &st = c->sara;
    ProfScope ps(c, PROF_PROX, s);
    T *v9 = (T *)st.v;
    for (int k = 0; k < st.sub_iters; ++k) {
        synthesis<T, SYN_PROX>(c, v9, z, x_out, thr, s);
        analysis<T, FIN_DUAL>(c, x_out, v9, thr, false, s);
    }
}

template <typename T>
void sara_reweight(ri_ctx *c, const T *x, T rho, hipStream_t s) {
    ProfScope ps(c, PROF_OTHER, s);
    analysis<T, FIN_WEIGHT>(c, x, (T *)c->sara.w, rho, true, s);
}

template <typename T>
void sara_analysis(ri_ctx *c, const T *x, T *coef9, hipStream_t s) {
    analysis<T, FIN_COEF>(c, x, coef9, (T)0, true, s);
}

template <typename T>
void sara_synthesis(ri_ctx *c, const T *coef9, T *x, hipStream_t s) {
    synthesis<T, SYN_PLAIN>(c, const_cast<T *>(coef9), nullptr, x, (T)0, s);
}

template void sara_prox<float>(ri_ctx *, const float *, float, float *, hipStream_t);
template void sara_prox<double>(ri_ctx *, const double *, double, double *, hipStream_t);
template void sara_reweight<float>(ri_ctx *, const float *, float, hipStream_t);
template void sara_reweight<double>(ri_ctx *, const double *, double, hipStream_t);
template void sara_analysis<float>(ri_ctx *, const float *, float *, hipStream_t);
template void sara_analysis<double>(ri_ctx *, const double *, double *, hipStream_t);
template void sara_synthesis<float>(ri_ctx *, const float *, float *, hipStream_t);
template void sara_synthesis<double>(ri_ctx *, const double *, double *, hipStream_t);

}  // namespace ri
