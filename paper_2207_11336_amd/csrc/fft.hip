// F and F^dagger on the N' x N' grid (paper eq. 1: F is the DFT on the fine
// grid), fused with Z (zero padding + 1/kappa_hat correction) on the way in
// and with Z^dagger (crop, correction, real part) on the way out.
//
// Layout: grid row-major [ky][kx], wrap-centred (pixel n at cell n mod N').
// Rows: one workgroup per image row, the whole N'-point row in LDS, Stockham
// radix-16 passes (natural order in and out, twiddles from an FP64-computed
// table); the first pass reads global memory and the last one writes it
// directly. Only the N non-zero rows are transformed on the way in, and only
// the N needed rows on the way out.
// Columns: four-step decomposition N' = N1 * N2 over stripes of adjacent
// columns, so every global access is a contiguous row segment:
//   pass A: N1-point transforms along rows n2 + N2*n1, times W_{N'}^{n2 k1};
//   pass B: N2-point transforms along rows N2*k1 + n2, written to row k1 + N1*k2.
// For N' = 4096 and 8192 these are two launches with each column's points in registers
// (a few lanes per column, see k_colpass_a_reg); below, one launch with whole columns
// in LDS (k_colfft).
#include <type_traits>
#include <utility>

#include "ri_internal.h"

namespace ri {

namespace {

// exp(-2 pi i k / 16), k = 0..15 (exact constants of the 16th roots of unity)
__device__ constexpr double kRoot16[16][2] = {
    {1.0, 0.0},
    {0.92387953251128675613, -0.38268343236508977173},
    {0.70710678118654752440, -0.70710678118654752440},
    {0.38268343236508977173, -0.92387953251128675613},
    {0.0, -1.0},
    {-0.38268343236508977173, -0.92387953251128675613},
    {-0.70710678118654752440, -0.70710678118654752440},
    {-0.92387953251128675613, -0.38268343236508977173},
    {-1.0, 0.0},
    {-0.92387953251128675613, 0.38268343236508977173},
    {-0.70710678118654752440, 0.70710678118654752440},
    {-0.38268343236508977173, 0.92387953251128675613},
    {0.0, 1.0},
    {0.38268343236508977173, 0.92387953251128675613},
    {0.70710678118654752440, 0.70710678118654752440},
    {0.92387953251128675613, 0.38268343236508977173}};

constexpr int brev(int k, int bits) {
    int r = 0;
    for (int b = 0; b < bits; ++b) r |= ((k >> b) & 1) << (bits - 1 - b);
    return r;
}
constexpr int ilog2(int R) { return R <= 1 ? 0 : 1 + ilog2(R / 2); }

// Products of the forward transforms with their roundings spelled out, so that the
// same transform gives the same bits from whichever kernel the compiler builds it
// into (left to itself it contracts a sum of two products either way, and shares
// products where both parts of w are alike). XR: the real part's product that is
// rounded by itself is a.x b.x, else a.y b.y; XI: the imaginary part's is a.x b.y,
// else a.y b.x. No choice is more accurate than another. Which one a product takes
// (mul_root, the callers' arguments, kPassAyBx) follows the contractions that the
// compiler chose in the kernels whose visibilities the FP32 transforms reproduce bit
// for bit: ||Phi x - y||^2 is an FP64 sum, and other last bits of Phi x move it
// by 2e-9 (one pass rounded otherwise) to 1e-7 (the half-plane form).
template <bool XR, bool XI, typename T>
__device__ __forceinline__ cx<T> mulr(cx<T> a, cx<T> b) {
    return mk<T>(XR ? fma(a.y, -b.y, a.x * b.x) : fma(a.x, b.x, -(a.y * b.y)),
                 XI ? fma(a.y, b.x, a.x * b.y) : fma(a.x, b.y, a.y * b.x));
}
// Who transforms: anyone, the columns, or the first, the middle or the last pass of a row.
enum { MUL_ANY = 0, MUL_COLS, MUL_FIRST, MUL_MID, MUL_LAST };
// d w for the 16th root of unity with exponent e, at input m of the butterflies.
template <typename T, int X>
__device__ __forceinline__ cx<T> mul_root(cx<T> d, cx<T> w, int e, int m) {
    if (X == MUL_ANY) return d * w;
    if (X == MUL_COLS) return e > 4 ? mulr<false, false>(d, w) : mulr<false, true>(d, w);
    if (e == 5 || e == 7) return mulr<true, false>(d, w);
    if (X == MUL_FIRST) return (e & 1) ? mulr<false, true>(d, w) : mulr<false, false>(d, w);
    if ((X == MUL_LAST && e == 6) || m == 9 || m == 11) return mulr<false, false>(d, w);
    return mulr<true, true>(d, w);
}

// In-register R-point DFT, natural order in and out:
// V[k] = sum_r v[r] exp(-+ 2 pi i r k / R).
template <typename T, int R, int X = MUL_ANY>
__device__ __forceinline__ void dft_reg(cx<T> *v, bool inv) {
#pragma unroll
    for (int span = R / 2; span >= 1; span >>= 1) {
#pragma unroll
        for (int m = 0; m < R; ++m) {
            if (m & span) continue;
            const int mloc = m & (2 * span - 1);
            cx<T> a = v[m], b = v[m + span];
            v[m] = a + b;
            cx<T> d = a - b;
            const int e = mloc * (16 / (2 * span));
            if (e != 0) {
                cx<T> w = mk<T>((T)kRoot16[e][0], inv ? -(T)kRoot16[e][1] : (T)kRoot16[e][1]);
                d = mul_root<T, X>(d, w, e, m);
            }
            v[m + span] = d;
        }
    }
    cx<T> t[R];
#pragma unroll
    for (int k = 0; k < R; ++k) t[k] = v[brev(k, ilog2(R))];
#pragma unroll
    for (int k = 0; k < R; ++k) v[k] = t[k];
}

__device__ __forceinline__ bool in_band(int r, int N, int Np) { return r < N / 2 || r >= Np - N / 2; }

template <typename F, int... I>
__device__ __forceinline__ void static_for_(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) { static_for_(f, std::make_integer_sequence<int, N>{}); }

// Row transforms: one row of N' = 2^LOGNP points per workgroup, N'/16 threads (at
// least a wave). The first pass (radix 16, no twiddles) takes input j + r N'/16 of
// group j from ld(j, r), the last one (radix R, twiddle step j) hands output
// j + r N'/R to st(j, r, value); r is a compile-time constant in both, and both index
// patterns run contiguously over j, so the global accesses coalesce and none of
// them depends on a branch. The passes between are radix-16 Stockham passes in LDS. A pass's
// twiddles are asked for before the barrier in front of it.
// Bound by memory latency and, for large rows, bandwidth. With the loads inside the
// crop's branches and one runtime-sized kernel for all N' the rows took, in us in FP32, forwards
// (with the clearing of the output grid) and backwards at N' = 256: 7.8 and 9.2,
// now 4.0 and 3.8; at 2048: 16.5 and 12.0, now 12.9 and 8.1; at 8192: 239 and 119,
// now 168 and 89; FP64 at 512: 12.1 and 9.6, now 6.1 and 5.5.
// SPELL: with the products' roundings spelled out (mulr).
template <typename T, int LOGNP, bool SPELL = false>
struct RowFft {
    static constexpr int NP = 1 << LOGNP, NT = NP / 16 < 64 ? 64 : NP / 16;
    static constexpr int MID = (LOGNP - 5) / 4, R = 1 << (LOGNP - 4 - 4 * MID);
    static constexpr size_t LDS = sizeof(cx<T>) * (size_t)(NP + NP / 32);

    // LDS element of point i, padded by one element per 32 against bank conflicts
    static __device__ __forceinline__ int at(int i) { return i + (i >> 5); }

    // Twiddles of group j's radix-RR pass with Ns finished points: W^(step r), r = 1 .. RR - 1.
    template <int RR>
    static __device__ __forceinline__ void fetch(cx<T> *w, const cx<T> *__restrict__ tw, int step) {
#pragma unroll
        for (int r = 1; r < RR; ++r) w[r] = tw[step * r];
    }
    template <int RR, bool LAST>
    static __device__ __forceinline__ void twiddle(cx<T> *v, const cx<T> *w0, bool any, bool inv) {
        if (!any) return;
#pragma unroll
        for (int r = 1; r < RR; ++r) {
            cx<T> w = w0[r];
            if (inv) w.y = -w.y;
            v[r] = SPELL ? mulr<false, !LAST>(v[r], w) : v[r] * w;
        }
    }

    template <typename Load, typename Store>
    static __device__ __forceinline__ void run(cx<T> *s, const cx<T> *__restrict__ tw, bool inv, Load &&ld, Store &&st) {
        constexpr int NG = NP / 16, G = 16 / R, NL = NP / R;
        const int tid = threadIdx.x;
        const bool live = NT == NG || tid < NG;
        cx<T> v[16], w[16];
        if (live) {
            static_for<16>([&](auto r) { v[r] = ld(tid, r); });
            dft_reg<T, 16, SPELL ? MUL_FIRST : MUL_ANY>(v, inv);
#pragma unroll
            for (int r = 0; r < 16; ++r) s[at(16 * tid + r)] = v[r];
        }
        static_for<MID>([&](auto m) {
            constexpr int Ns = 16 << (4 * decltype(m)::value);
            const int jm = tid & (Ns - 1);
            if (live) fetch<16>(w, tw, jm * (NP / (Ns * 16)));
            __syncthreads();
            if (live) {
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = s[at(tid + r * NG)];
            }
            __syncthreads();
            if (live) {
                twiddle<16, false>(v, w, jm != 0, inv);
                dft_reg<T, 16, SPELL ? MUL_MID : MUL_ANY>(v, inv);
#pragma unroll
                for (int r = 0; r < 16; ++r) s[at((tid - jm) * 16 + jm + r * Ns)] = v[r];
            }
        });
#pragma unroll
        for (int i = 0; i < G; ++i)
            if (G * NT == NL || tid + i * NT < NL) fetch<R>(w + i * R, tw, tid + i * NT);
        __syncthreads();
        static_for<G>([&](auto i) {
            const int j = tid + decltype(i)::value * NT;
            if (G * NT != NL && j >= NL) return;
            cx<T> *u = v + decltype(i)::value * R;
#pragma unroll
            for (int r = 0; r < R; ++r) u[r] = s[at(j + r * NL)];
            twiddle<R, true>(u, w + decltype(i)::value * R, j != 0, inv);
            dft_reg<T, R, SPELL ? MUL_LAST : MUL_ANY>(u, inv);
            static_for<R>([&](auto r) { st(j, r, u[decltype(r)::value]); });
        });
    }
};

// The kernels of image side N'/2: pixel column ix = (gx + N/2) mod N' of grid column gx
// = j + r N'/16 lies in the image for r < 4 and r >= 12.

// Zero the output grid, the work counter and the partial sums, spread over the launch.
template <typename T>
__device__ __forceinline__ void clear_share(const Clear<T> &z) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x, i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint4 *g = reinterpret_cast<uint4 *>(z.grid);
    const int64_t n16 = z.n * (int64_t)sizeof(cx<T>) / 16;
    for (int64_t i = i0; i < n16; i += step) g[i] = make_uint4(0u, 0u, 0u, 0u);
    if (i0 == 0 && z.counter) *z.counter = 0;
    for (int64_t i = i0; i < z.npart; i += step) z.part[i] = 0.0;
}

template <typename T>
__global__ void k_clear(Clear<T> z) {
    clear_share<T>(z);
}

// Z then the row DFT of image row iy (blockIdx.x), written to row (iy - N/2) & rowmask
// (N' - 1: the grid row; N - 1: the N rows packed).
// With a w-stack's phase screen (chirp != NULL) the padded image is x c_s.
template <typename T, int LOGNP, bool CHIRP>
__global__ void __launch_bounds__((RowFft<T, LOGNP>::NT))
k_zpad_rowfft(const T *__restrict__ x, cx<T> *__restrict__ grid, const T *__restrict__ icorr,
              const cx<T> *__restrict__ tw, const cx<T> *__restrict__ chirp, int rowmask, Clear<T> z) {
    using F = RowFft<T, LOGNP, true>;
    extern __shared__ unsigned char smem_raw[];
    constexpr int Np = F::NP, N = Np / 2;
    const int iy = blockIdx.x;
    const T cy = icorr[iy];
    const T *xr = x + (size_t)iy * N;
    const cx<T> *chr = CHIRP ? chirp + (size_t)iy * N : nullptr;
    cx<T> *row = grid + (size_t)((iy - N / 2) & rowmask) * Np;
    F::run(reinterpret_cast<cx<T> *>(smem_raw), tw, false,
           [&](int j, auto r) -> cx<T> {
               if constexpr (r >= 4 && r < 12) return mk<T>((T)0, (T)0);
               const int ix = (j + r * (Np / 16) + N / 2) & (Np - 1);
               const T a = xr[ix] * icorr[ix] * cy;
               if (!CHIRP) {
                   T zero = 0;              // opaque: products that the compiler knows to be
                   asm("" : "+v"(zero));    // real would be contracted into the next butterflies
                   return mk<T>(a, zero);
               }
               const cx<T> ch = chr[ix];
               return mk<T>(a * ch.x, a * ch.y);
           },
           [&](int j, auto r, cx<T> v) { row[j + r * (Np / F::R)] = v; });
    clear_share<T>(z);
}

// Inverse row DFT of grid row (iy - N/2) mod N', then crop, correction, real part:
// out[iy][ix] = Re{row[(ix - N/2) mod N']} / (kappa_hat_x kappa_hat_y). With a
// w-stack's phase screen the value is Re{conj(c_s) row[...]} (Z_s^dagger), added
// to out when accumulate != 0 (the sum over stacks).
template <typename T, int LOGNP, bool CHIRP>
__global__ void __launch_bounds__((RowFft<T, LOGNP>::NT))
k_irowfft_crop(const cx<T> *__restrict__ grid, T *__restrict__ out, const T *__restrict__ icorr,
               const cx<T> *__restrict__ tw, const cx<T> *__restrict__ chirp, int accumulate) {
    using F = RowFft<T, LOGNP>;
    extern __shared__ unsigned char smem_raw[];
    constexpr int Np = F::NP, N = Np / 2;
    const int iy = blockIdx.x;
    const cx<T> *row = grid + (size_t)((iy - N / 2) & (Np - 1)) * Np;
    const T cy = icorr[iy];
    T *orow = out + (size_t)iy * N;
    const cx<T> *chr = CHIRP ? chirp + (size_t)iy * N : nullptr;
    F::run(reinterpret_cast<cx<T> *>(smem_raw), tw, true, [&](int j, auto r) { return row[j + r * (Np / 16)]; },
           [&](int j, auto r, cx<T> v) {
               const int ix = (j + r * (Np / F::R) + N / 2) & (Np - 1);   // the crop: image column ix < N
               if (ix >= N) return;
               T re = v.x;
               if (CHIRP) {
                   const cx<T> ch = chr[ix];
                   re = v.x * ch.x + v.y * ch.y;
               }
               const T val = re * icorr[ix] * cy;
               if (accumulate) orow[ix] += val;
               else orow[ix] = val;
           });
}

// ---------------------------------------------------------------------------
// Column transforms up to N' = 2048: a workgroup has CW whole columns in LDS, one
// read and one write of the grid. The arithmetic is that of the four-step form
// N' = N1 N2: N1-point transforms over the rows n2 + N2 n1, times W_{N'}^{n2 k1},
// N2-point transforms over n2, frequency k1 + N1 k2; each of the two by a radix-16
// pass (radix N1 or N2 below 16) and a radix-2 or -4 one. Neighbouring stripes run
// on one XCD (workgroups are dealt to the 8 XCDs in turn), whose L2 holds the lines
// they share. Bound by memory latency: 18 us at N' = 2048 in FP32 for 50 MB (10 us
// at the rate of a copy), 11 at 1024 and 5 at 256, with 4 columns of FP32 (2 of FP64) a
// workgroup; 8 columns measured 18, 11.5 and 5, and a launch for each of the two
// transforms with the grid in between 49, 29 and 18.
// ---------------------------------------------------------------------------
template <typename T, int LOGNP>
struct FullCol {
    static constexpr int NP = 1 << LOGNP, LOG1 = full_log_n1(LOGNP), N1 = 1 << LOG1, N2 = NP >> LOG1;
    static constexpr int LCW = sizeof(T) == 4 ? 2 : 1, CW = 1 << LCW;
    static constexpr int NT = NP * CW / 16 < 64 ? 64 : NP * CW / 16;
    static constexpr int RA = N1 < 16 ? N1 : 16, RA2 = N1 / RA, RB = N2 < 16 ? N2 : 16, RB2 = N2 / RB;
    static constexpr size_t LDS = sizeof(cx<T>) * (size_t)(NP + NP / 16) * CW;

    // LDS element of point i of column col (padded against bank conflicts of the 16-strided stores)
    static __device__ __forceinline__ int at(int i, int col) { return ((i + (i >> 4)) << LCW) + col; }

    // f(q, col, registers) for the thread's groups of a radix-R pass.
    template <int R, typename F>
    static __device__ __forceinline__ void groups(cx<T> *v, F &&f) {
#pragma unroll
        for (int i = 0; i < 16 / R; ++i) {
            const int g = threadIdx.x + i * NT;
            if (16 / R * NT > NP / R * CW && g >= NP / R * CW) continue;
            f(g >> LCW, g & (CW - 1), v + i * R);
        }
    }
    template <int R>
    static __device__ __forceinline__ void twiddle(cx<T> *v, const cx<T> *__restrict__ tw, int step, bool inv) {
        if (step == 0) return;
#pragma unroll
        for (int r = 1; r < R; ++r) {
            cx<T> w = tw[step * r];
            if (inv) w.y = -w.y;
            v[r] = mulr<false, true>(v[r], w);
        }
    }
};

// The stripe's columns: point row of column col from ld(row, col), frequency k1 + N1 k2 to st(k1, k2, col, value).
template <typename T, int LOGNP, typename Load, typename Store>
__device__ __forceinline__ void full_cols(cx<T> *s, const cx<T> *__restrict__ tw, bool inv, Load &&ld, Store &&st) {
    using C = FullCol<T, LOGNP>;
    constexpr int N1 = C::N1, N2 = C::N2, RA = C::RA, RA2 = C::RA2, RB = C::RB, RB2 = C::RB2;
    cx<T> v[16];
    C::template groups<RA>(v, [&](int q, int col, cx<T> *u) {
        const int j = q & (N1 / RA - 1), n2 = q / (N1 / RA);
#pragma unroll
        for (int r = 0; r < RA; ++r) u[r] = ld(n2 + N2 * (j + r * (N1 / RA)), col);
    });
    auto four_step = [&](cx<T> *u, int R, int n2, int k0, int dk) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cx<T> w = tw[n2 * (k0 + dk * r)];
            if (inv) w.y = -w.y;
            u[r] = mulr<false, false>(u[r], w);
        }
    };
    C::template groups<RA>(v, [&](int q, int col, cx<T> *u) {
        const int j = q & (N1 / RA - 1), n2 = q / (N1 / RA);
        dft_reg<T, RA, MUL_COLS>(u, inv);
        if (RA2 == 1) four_step(u, RA, n2, 0, 1);
#pragma unroll
        for (int r = 0; r < RA; ++r) s[C::at(n2 * N1 + RA * j + r, col)] = u[r];
    });
    __syncthreads();
    if constexpr (RA2 > 1) {
        C::template groups<RA2>(v, [&](int q, int col, cx<T> *u) {
            const int j = q & 15, n2 = q >> 4;
#pragma unroll
            for (int r = 0; r < RA2; ++r) u[r] = s[C::at(n2 * N1 + j + 16 * r, col)];
            C::template twiddle<RA2>(u, tw, j * N2, inv);
            dft_reg<T, RA2, MUL_COLS>(u, inv);
            four_step(u, RA2, n2, j, 16);
#pragma unroll
            for (int r = 0; r < RA2; ++r) s[C::at(n2 * N1 + j + 16 * r, col)] = u[r];
        });
        __syncthreads();
    }
    C::template groups<RB>(v, [&](int q, int col, cx<T> *u) {
        const int k1 = q & (N1 - 1), j = q >> C::LOG1;
#pragma unroll
        for (int r = 0; r < RB; ++r) u[r] = s[C::at((j + r * (N2 / RB)) * N1 + k1, col)];
        dft_reg<T, RB, MUL_COLS>(u, inv);
        if (RB2 == 1) {
#pragma unroll
            for (int r = 0; r < RB; ++r) st(k1, r, col, u[r]);
        }
    });
    if constexpr (RB2 > 1) {
        __syncthreads();
        C::template groups<RB>(v, [&](int q, int col, cx<T> *u) {
            const int k1 = q & (N1 - 1), j = q >> C::LOG1;
#pragma unroll
            for (int r = 0; r < RB; ++r) s[C::at((RB * j + r) * N1 + k1, col)] = u[r];
        });
        __syncthreads();
        C::template groups<RB2>(v, [&](int q, int col, cx<T> *u) {
            const int k1 = q & (N1 - 1), j = q >> C::LOG1;
#pragma unroll
            for (int r = 0; r < RB2; ++r) u[r] = s[C::at((j + 16 * r) * N1 + k1, col)];
            C::template twiddle<RB2>(u, tw, j * N1, inv);
            dft_reg<T, RB2, MUL_COLS>(u, inv);
#pragma unroll
            for (int r = 0; r < RB2; ++r) st(k1, j + 16 * r, col, u[r]);
        });
    }
}

// First column of the workgroup's stripe: neighbouring stripes on one XCD.
__device__ __forceinline__ int stripe_x0(int cw) {
    const int nb = gridDim.x;
    return ((nb & 7) ? (int)blockIdx.x : (int)(blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3)) * cw;
}

template <typename T, int LOGNP>
__global__ void __launch_bounds__((FullCol<T, LOGNP>::NT))
k_colfft(const cx<T> *in, cx<T> *out, const cx<T> *__restrict__ tw, int N, int band_in, int band_out, int inv) {
    using C = FullCol<T, LOGNP>;
    extern __shared__ unsigned char smem_raw[];
    constexpr int NP = C::NP;
    const bool permuted = out == in;
    const int x0 = stripe_x0(C::CW);
    full_cols<T, LOGNP>(
        reinterpret_cast<cx<T> *>(smem_raw), tw, inv != 0,
        [&](int row, int col) {
            return (!band_in || in_band(row, N, NP)) ? in[(size_t)row * NP + x0 + col] : mk<T>((T)0, (T)0);
        },
        [&](int k1, int k2, int col, cx<T> val) {
            const int k = k1 + C::N1 * k2, row = permuted ? C::N2 * k1 + k2 : k;
            if (!band_out || in_band(row, N, NP)) out[(size_t)row * NP + x0 + col] = val;
        });
}

// ---------------------------------------------------------------------------
// Column passes of the 4096- and 8192-point transforms (N1 = 64 or 128,
// N2 = 64) in registers: a one-wave workgroup takes 64/Q adjacent columns, Q
// lanes per column so that a lane holds at most 512 bytes of points (64 FP32
// or 32 FP64 complex values), so every load and store of the wave is a
// contiguous 512-byte row segment and no LDS or barrier is involved. Radix-2
// decimation in frequency, natural order in, bit-reversed out; twiddles come
// from the FP64-computed table.
// ---------------------------------------------------------------------------
//
// SPELL (64 points): with the products' roundings spelled out as the compiler contracts
// them in k_colpass_a_reg<float, 128, 2>: a.y b.y is rounded by itself in every real
// part; in the imaginary part of input j, stage by stage, a.y b.x where bit j is set
// here, else a.x b.y. The pattern has no meaning of its own (the order in which that
// kernel's values arise); it is what a kernel has to follow to give the same
// visibilities to the last bit.
constexpr uint64_t kPassAyBx[6] = {0, 0xFE00000000ull, 0xFE000E00FE0000ull, 0x60E0E0E020E0E00ull, 0x2220222022202220ull, 0};

template <typename T, int P, bool SPELL = false>
__device__ __forceinline__ void fftp_reg(cx<T> *v, const cx<T> *__restrict__ tw, int tw_mul, bool inv) {
    static_assert(!SPELL || P == 64, "the pattern is that of 64 points");
    static_for<ilog2(P)>([&](auto St) {
        constexpr int span = (P / 2) >> decltype(St)::value;
        static_for<P>([&](auto J) {
            constexpr int j = decltype(J)::value;
            if constexpr ((j & span) == 0) {
                const cx<T> a = v[j], b = v[j + span];
                v[j] = a + b;
                cx<T> d = a - b;
                constexpr int e = (j & (span - 1)) * ((P / 2) / span);
                if constexpr (e != 0) {
                    cx<T> w = tw[e * tw_mul];
                    if (inv) w.y = -w.y;
                    if constexpr (!SPELL) d = d * w;
                    else d = mulr<false, !((kPassAyBx[decltype(St)::value] >> j) & 1)>(d, w);
                }
                v[j + span] = d;
            }
        });
    });
}

// L-point transform of a column held by Q lanes (lane half h = 0 .. Q-1 holds
// points h P .. h P + P - 1, P = L / Q, the lanes of one column CPB = 64 / Q
// apart): the first log2 Q decimation-in-frequency stages pair lanes h and
// h ^ (s / P) by shuffles (span s = L/2 .. P), the rest run in registers.
// Afterwards point i of lane h holds frequency brev_P(i) Q + brev_Q(h).
template <typename T, int L, int Q>
__device__ __forceinline__ void fft_lanes(cx<T> *v, int h, const cx<T> *__restrict__ tw, int Np, bool inv) {
    constexpr int P = L / Q, CPB = 64 / Q;
    static_for<ilog2(Q)>([&](auto St) {
        constexpr int s = (L / 2) >> decltype(St)::value;   // span in points, >= P
        constexpr int hs = s / P;                            // partner distance in lane halves
        const bool upper = (h & hs) != 0;
        static_for<P>([&](auto I) {
            constexpr int i = decltype(I)::value;
            cx<T> o;
            o.x = __shfl_xor(v[i].x, hs * CPB);
            o.y = __shfl_xor(v[i].y, hs * CPB);
            if (!upper) {
                v[i] = v[i] + o;
            } else {
                cx<T> d = o - v[i];
                const int e = ((h * P + i) & (s - 1)) * ((L / 2) / s);   // W_{2s}^{j mod s} = W_L^{...}
                if (e != 0) {
                    cx<T> w = tw[e * (Np / L)];
                    if (inv) w.y = -w.y;
                    d = d * w;
                }
                v[i] = d;
            }
        });
    });
    fftp_reg<T, P>(v, tw, Np / P, inv);
}

// Pass A in place: rows n2 + N2 n1 -> L = N1-point transforms over n1, times W_{N'}^{n2 k1}, rows n2 + N2 k1.
template <typename T, int L, int Q>
__global__ void __launch_bounds__(64) k_colpass_a_reg(cx<T> *__restrict__ grid, const cx<T> *__restrict__ tw, int N,
                                                      int logNp, int band_in, int inv) {
    constexpr int P = L / Q, CPB = 64 / Q;
    const int Np = 1 << logNp, N2 = Np / L;
    const int h = threadIdx.x / CPB, c = blockIdx.x * CPB + threadIdx.x % CPB, n2 = blockIdx.y;
    cx<T> v[P];
    static_for<P>([&](auto I) {
        const int r = n2 + N2 * (h * P + decltype(I)::value);
        v[I] = (!band_in || in_band(r, N, Np)) ? grid[(size_t)r * Np + c] : mk<T>((T)0, (T)0);
    });
    fft_lanes<T, L, Q>(v, h, tw, Np, inv != 0);
    const int hb = brev(h, ilog2(Q));
    static_for<P>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const int k1 = brev(i, ilog2(P)) * Q + hb;
        cx<T> w = tw[n2 * k1];
        if (inv) w.y = -w.y;
        grid[(size_t)(n2 + N2 * k1) * Np + c] = v[i] * w;
    });
}

// Pass A of a 128-point column whose band input has 64 non-zero points (image
// side N = N'/2: points 32..95 are zero): the first radix-2 stage only selects
// and twists, so a lane holds one 64-point half, the even or (blockIdx.z = 1)
// the odd frequencies, and no value crosses lanes (the two halves write rows that
// the other reads, hence out of place, from the N packed band rows). All products
// round as in k_colpass_a_reg<float, 128, 2> (fftp_reg's SPELL; left to itself the
// compiler rounds the real part's other product where an input is negated, and other
// imaginary products: 85% of the visibilities at N = 4096 then differ in their last bits
// from those of the other kernel, and ||r||^2 by up to 2e-9). At N' = 8192 in FP32:
// 231 us, against 321 us with two lanes per column (average of both directions).
template <typename T>
__global__ void __launch_bounds__(64) k_colpass_a_band(const cx<T> *in, cx<T> *out, const cx<T> *__restrict__ tw,
                                                       int logNp) {
    const int Np = 1 << logNp, N2 = Np / 128;
    const int c = blockIdx.x * 64 + threadIdx.x, n2 = blockIdx.y, odd = blockIdx.z;
    cx<T> v[64];
    static_for<64>([&](auto I) {
        constexpr int i = decltype(I)::value;
        v[i] = in[(size_t)(n2 + N2 * i) * Np + c];
    });
    if (odd)
        static_for<64>([&](auto I) {
            constexpr int i = decltype(I)::value;
            cx<T> d = i < 32 ? v[i] : mk<T>(-v[i].x, -v[i].y);
            if constexpr (i != 0) d = mulr<false, true>(d, tw[i * (Np / 128)]);
            v[i] = d;
        });
    fftp_reg<T, 64, true>(v, tw, Np / 64, false);
    static_for<64>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const int k1 = brev(i, 6) * 2 + odd;
        out[(size_t)(n2 + N2 * k1) * Np + c] = mulr<false, true>(v[i], tw[n2 * k1]);
    });
}

// Pass B: rows L k1 + n2 (L = N2) -> L-point transforms over n2 -> rows k1 + N1 k2, or, in place
// (out == in), -> rows L k1 + k2. The wave has loaded all its points before it stores one.
template <typename T, int L, int Q>
__global__ void __launch_bounds__(64) k_colpass_b_reg(const cx<T> *in, cx<T> *out,
                                                      const cx<T> *__restrict__ tw, int N, int logNp, int band_out,
                                                      int inv) {
    constexpr int P = L / Q, CPB = 64 / Q;
    const int Np = 1 << logNp, N1 = Np / L;
    const int h = threadIdx.x / CPB, c = blockIdx.x * CPB + threadIdx.x % CPB, k1 = blockIdx.y;
    cx<T> v[P];
    static_for<P>([&](auto I) { v[I] = in[(size_t)(L * k1 + h * P + decltype(I)::value) * Np + c]; });
    fft_lanes<T, L, Q>(v, h, tw, Np, inv != 0);
    const int hb = brev(h, ilog2(Q));
    static_for<P>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const int k2 = brev(i, ilog2(P)) * Q + hb, r = out == in ? L * k1 + k2 : k1 + N1 * k2;
        if (!band_out || in_band(r, N, Np)) out[(size_t)r * Np + c] = v[i];
    });
}

// ---------------------------------------------------------------------------
// Half-plane transforms of a real image. F Z x is Hermitian, so only the
// columns kx = 0 .. N of the grid are formed, and on the way out only those
// carry the (mirrored) visibilities.
//
// Rows: two image rows a, b ride through one complex transform as a + i b and
// are separated by their symmetry. The columns kx = 0 and kx = N of the row
// spectra are real; the scratch holds them as one complex column 0.
//
// Columns: of the 2N grid rows only N are non-zero (forward) or wanted
// (adjoint), so the even and the odd ky of a column are N-point transforms
// of the same N inputs, the odd ones twisted by exp(-+ i pi n / N):
//   X[2k + p] = sum_n (w^{pn} x[n]) W_N^{nk},   x[n] = sum_p w^{-pn} (IDFT_N Y[2k + p])[n].
// One workgroup holds CW adjacent whole columns in LDS: one read of the
// scratch per parity and one write of the grid forward, one read of the grid
// and one write of the scratch back. Bound by memory latency and bandwidth; the
// adjoint's columns and rows take 59 + 21 us at N' = 4096 in FP32 (whole plane,
// two column passes: about 150), 189 + 89 at 8192 (about 680).
// ---------------------------------------------------------------------------
inline __device__ __host__ int scratch_pitch(int N) { return N >= 64 ? N + 16 : N; }

// Image rows 2 b and 2 b + 1 -> rows of the scratch (row index n mod N).
template <typename T, int LOGNP>
__global__ void __launch_bounds__((RowFft<T, LOGNP>::NT))
k_half_rows(const T *__restrict__ x, cx<T> *__restrict__ scr, const T *__restrict__ icorr,
            const cx<T> *__restrict__ tw, Clear<T> z) {
    using F = RowFft<T, LOGNP>;
    extern __shared__ unsigned char smem_raw[];
    cx<T> *s = reinterpret_cast<cx<T> *>(smem_raw);
    constexpr int Np = F::NP, N = Np / 2;
    const int iy = 2 * blockIdx.x;
    const T ca = icorr[iy], cb = icorr[iy + 1];
    const T *xa = x + (size_t)iy * N, *xb = xa + N;
    F::run(s, tw, false,
           [&](int j, auto r) -> cx<T> {
               if constexpr (r >= 4 && r < 12) return mk<T>((T)0, (T)0);
               const int ix = (j + r * (Np / 16) + N / 2) & (Np - 1);
               const T c = icorr[ix];
               return mk<T>(xa[ix] * c * ca, xb[ix] * c * cb);
           },
           [&](int j, auto r, cx<T> v) { s[F::at(j + r * (Np / F::R))] = v; });   // where the group read its inputs
    __syncthreads();
    cx<T> *ra = scr + (size_t)((iy - N / 2) & (N - 1)) * scratch_pitch(N);
    cx<T> *rb = ra + scratch_pitch(N);   // n and n + 1 are neighbours: n is even
#pragma unroll
    for (int i = 0; i < (N + F::NT - 1) / F::NT; ++i) {
        const int k = threadIdx.x + i * F::NT;
        if (N % F::NT != 0 && k >= N) break;
        const cx<T> p = s[F::at(k)], q = s[F::at(k == 0 ? N : Np - k)];
        if (k == 0) {
            ra[0] = mk<T>(p.x, q.x);
            rb[0] = mk<T>(p.y, q.y);
        } else {
            ra[k] = mk<T>((T)0.5 * (p.x + q.x), (T)0.5 * (p.y - q.y));
            rb[k] = mk<T>((T)0.5 * (p.y + q.y), (T)0.5 * (q.x - p.x));
        }
    }
    clear_share<T>(z);
}

// Rows of the scratch -> image rows 2 b and 2 b + 1: the real inverse row
// transforms of both half spectra as one complex one, cropped and corrected.
template <typename T, int LOGNP>
__global__ void __launch_bounds__((RowFft<T, LOGNP>::NT))
k_half_irows(const cx<T> *__restrict__ scr, T *__restrict__ out, const T *__restrict__ icorr,
             const cx<T> *__restrict__ tw) {
    using F = RowFft<T, LOGNP>;
    extern __shared__ unsigned char smem_raw[];
    constexpr int Np = F::NP, N = Np / 2;
    const int iy = 2 * blockIdx.x;
    const cx<T> *ra = scr + (size_t)((iy - N / 2) & (N - 1)) * scratch_pitch(N);
    const cx<T> *rb = ra + scratch_pitch(N);
    const T ca = icorr[iy], cb = icorr[iy + 1];
    T *oa = out + (size_t)iy * N, *ob = oa + N;
    F::run(reinterpret_cast<cx<T> *>(smem_raw), tw, true,
           [&](int j, auto r) -> cx<T> {
               // spectrum element k from element k or, conjugated, N' - k; the real k = 0
               // and k = N share element 0
               const int k = j + r * (Np / 16), e = r < 8 ? k : (Np - k) & (N - 1);
               cx<T> a = ra[e], b = rb[e];
               if (r >= 8) {
                   a.y = -a.y;
                   b.y = -b.y;
               }
               const cx<T> v = mk<T>((T)0.5 * (a.x - b.y), (T)0.5 * (a.y + b.x));
               if (r == 0) return j == 0 ? mk<T>(a.x, b.x) : v;
               if (r == 8) return j == 0 ? mk<T>(-a.y, -b.y) : v;
               return v;
           },
           [&](int j, auto r, cx<T> v) {
               const int ix = (j + r * (Np / F::R) + N / 2) & (Np - 1);
               const T c = icorr[ix & (N - 1)];
               if (ix >= N) return;
               oa[ix] = v.x * c * ca;
               ob[ix] = v.y * c * cb;
           });
}

// base[i] through a 32-bit byte offset (one address register instead of two).
template <typename T>
__device__ __forceinline__ T &at32(T *base, unsigned i) {
    using B = std::conditional_t<std::is_const<T>::value, const char, char>;
    return *reinterpret_cast<T *>(reinterpret_cast<B *>(base) + (size_t)(i * (unsigned)sizeof(T)));
}

// The same value, opaque to the compiler: addresses formed from it are
// computed again instead of being kept in registers from one transform to the next.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// log2 of the columns per workgroup: 4 (FP32, N' = 4096: 59 us against 61 with 8; 8192: 192
// against 234 with 2; FP64 forward at N = 256 and 1024: with 2 columns 15.8 against
// 10.2 and 17 against 13 us), 2 in FP64 at N = 4096, whose columns then fill 139 KB of LDS.
template <typename T>
constexpr int half_log_cw(int logN) { return sizeof(T) == 8 && logN > 11 ? 1 : 2; }
template <typename T>
constexpr int half_threads(int logN) {
    const int n = 1 << (logN + half_log_cw<T>(logN) - 4);
    return n < 64 ? 64 : n;
}

// Whole-column transforms: N = 2^LOGN points, CW columns in LDS.
template <typename T, int LOGN>
struct ColFft {
    static constexpr int N = 1 << LOGN, LCW = half_log_cw<T>(LOGN), CW = 1 << LCW, NT = half_threads<T>(LOGN);
    static constexpr int RL = LOGN == 4 ? 16 : 1 << (((LOGN - 1) & 3) + 1);   // last pass's radix
    static constexpr int SP = N >= 64 ? N + 16 : N;                           // scratch pitch
    static constexpr size_t LDS = sizeof(cx<T>) * ((size_t)(N + N / 16) * CW);

    // LDS element of point i of column col: CW elements of padding per 16
    // points, so that the first pass's stores (16 points apart per lane) spread
    // over the banks.
    static __device__ __forceinline__ int cidx(int i, int col) { return (i + (i >> 4)) * CW + col; }

    // One Stockham radix-R pass (Ns = points per finished sub-transform); LAST
    // leaves the outputs in v: output j + r N/R of group g = (j, col),
    // g = tid + i NT, in v[i R + r].
    template <int R, int NS, bool LAST>
    static __device__ __forceinline__ void pass(cx<T> *s, const cx<T> *__restrict__ tw2, bool inv, int tid, cx<T> (&v)[16]) {
        constexpr int G = 16 / R, ng = (N / R) * CW;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int g = tid + i * NT;
            if (G * NT > ng && g >= ng) continue;
            const int col = g & (CW - 1), j = g >> LCW, jm = j & (NS - 1);
#pragma unroll
            for (int r = 0; r < R; ++r) v[i * R + r] = s[cidx(j + r * (N / R), col)];
            const int step = 2 * jm * (N / (NS * R));
#pragma unroll
            for (int r = 1; r < R; ++r) {
                cx<T> w = at32(tw2, (unsigned)(step * r));
                if (inv) w.y = -w.y;
                v[i * R + r] = v[i * R + r] * w;
            }
            dft_reg<T, R>(v + i * R, inv);
        }
        __syncthreads();
        if (LAST) return;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int g = tid + i * NT;
            if (G * NT > ng && g >= ng) continue;
            const int col = g & (CW - 1), j = g >> LCW, jm = j & (NS - 1);
#pragma unroll
            for (int r = 0; r < R; ++r) s[cidx((j - jm) * R + jm + r * NS, col)] = v[i * R + r];
        }
        __syncthreads();
    }

    // v: inputs j + r N/16 of group (j, col) = tid on entry, the last
    // pass's outputs on return (read them with visit). s is free on entry and
    // on return.
    static __device__ __forceinline__ void run(cx<T> *s, const cx<T> *__restrict__ tw2, bool inv, int tid, cx<T> (&v)[16]) {
        dft_reg<T, 16>(v, inv);
        if constexpr (LOGN > 4) {
            const int g = tid, col = g & (CW - 1), j = g >> LCW;
            if (j < N / 16) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[cidx(16 * j + r, col)] = v[r];
            }
            __syncthreads();
            if constexpr (LOGN > 8) pass<16, 16, false>(s, tw2, inv, tid, v);
            pass<RL, N / RL, true>(s, tw2, inv, tid, v);
        }
    }

    // f(k, col, integral_constant<register>) for the thread's outputs.
    template <typename F>
    static __device__ __forceinline__ void visit(int tid, F &&f) {
        constexpr int ng = (N / RL) * CW;
        static_for<16 / RL>([&](auto I) {
            const int g = tid + decltype(I)::value * NT;
            if (16 / RL * NT > ng && g >= ng) return;
            static_for<RL>([&](auto Q) {
                f((g >> LCW) + decltype(Q)::value * (N / RL), g & (CW - 1),
                  std::integral_constant<int, decltype(I)::value * RL + decltype(Q)::value>{});
            });
        });
    }

    // exp(-2 pi i n / (2N)) of the row with index i = n mod N, n in [-N/2, N/2).
    static __device__ __forceinline__ cx<T> twist(const cx<T> *__restrict__ tw2, int i) {
        return at32(tw2, (unsigned)((i < N / 2 ? i : i + N) & (2 * N - 1)));
    }
};

// Scratch -> grid columns x0 .. x0 + CW - 1, the ky of one parity per workgroup.
// The two parities of a stripe and its neighbours run on one XCD (workgroups
// are dealt to the 8 XCDs in turn), whose L2 then holds the scratch lines they
// share. Stripe 0 also writes column kx = N.
template <typename T, int LOGN>
__global__ void __launch_bounds__((half_threads<T>(LOGN)))
k_half_cols(const cx<T> *__restrict__ scr, cx<T> *__restrict__ X, const cx<T> *__restrict__ tw2, int pitch) {
    using C = ColFft<T, LOGN>;
    extern __shared__ unsigned char smem_raw[];
    cx<T> *s = reinterpret_cast<cx<T> *>(smem_raw);
    constexpr int N = C::N;
    const int nb = gridDim.x, b = (nb & 7) ? (int)blockIdx.x : (int)(blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3);
    const int p = b & 1, x0 = (b >> 1) * C::CW, g = threadIdx.x, col0 = g & (C::CW - 1), j0 = g >> C::LCW;
    const bool live = j0 < N / 16;
    cx<T> v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
        v[r] = live ? at32(scr, (unsigned)((j0 + r * (N / 16)) * C::SP + x0 + col0)) : mk<T>((T)0, (T)0);
    if (p && live) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = v[r] * C::twist(tw2, j0 + r * (N / 16));
    }
    C::run(s, tw2, false, g, v);
    cx<T> *Xp = X + (size_t)p * pitch;
    if (x0 == 0) {
        // column 0 carries kx = 0 and kx = N (their row spectra are real)
        C::visit(g, [&](int k, int col, auto q) {
            if (col != 0) at32(Xp, (unsigned)(2 * k * pitch + col)) = v[q];
            else s[k] = v[q];
        });
        __syncthreads();
        for (int k = g; k < N; k += C::NT) {
            const cx<T> a = s[k], c = s[(N - k - p) & (N - 1)];
            at32(Xp, (unsigned)(2 * k * pitch)) = mk<T>((T)0.5 * (a.x + c.x), (T)0.5 * (a.y - c.y));
            at32(Xp, (unsigned)(2 * k * pitch + N)) = mk<T>((T)0.5 * (a.y + c.y), (T)0.5 * (c.x - a.x));
        }
    } else {
        C::visit(g, [&](int k, int col, auto q) { at32(Xp, (unsigned)(2 * k * pitch + x0 + col)) = v[q]; });
    }
}

// Grid columns -> scratch: the adjoint of k_half_cols. Column 0 takes the
// Hermitian parts of kx = 0 and kx = N (only the image's real part is wanted).
template <typename T, int LOGN>
__global__ void __launch_bounds__((half_threads<T>(LOGN)))
k_half_icols(const cx<T> *__restrict__ Y, cx<T> *__restrict__ scr, const cx<T> *__restrict__ tw2, int pitch) {
    using C = ColFft<T, LOGN>;
    extern __shared__ unsigned char smem_raw[];
    cx<T> *s = reinterpret_cast<cx<T> *>(smem_raw);
    constexpr int N = C::N;
    const int nb = gridDim.x, b = (nb & 7) ? (int)blockIdx.x : (int)(blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3);
    const int x0 = b * C::CW, g = threadIdx.x, col0 = g & (C::CW - 1), j0 = g >> C::LCW;
    const bool live = j0 < N / 16;
    auto load = [&](int p, cx<T>(&a)[16]) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ky = 2 * (j0 + r * (N / 16)) + p;
            a[r] = live ? at32(Y, (unsigned)(ky * pitch + x0 + col0)) : mk<T>((T)0, (T)0);
        }
        if (live && x0 + col0 == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int ky = 2 * (j0 + r * (N / 16)) + p, km = (2 * N - ky) & (2 * N - 1);
                const cx<T> m = Y[(size_t)km * pitch], b = Y[(size_t)ky * pitch + N], bm = Y[(size_t)km * pitch + N];
                const cx<T> h0 = mk<T>((T)0.5 * (a[r].x + m.x), (T)0.5 * (a[r].y - m.y));
                const cx<T> hn = mk<T>((T)0.5 * (b.x + bm.x), (T)0.5 * (b.y - bm.y));
                a[r] = mk<T>(h0.x - hn.y, h0.y + hn.x);
            }
        }
    };
    cx<T> ev[16], od[16];
    load(0, ev);
    load(1, od);
    C::run(s, tw2, true, g, ev);
    const int g2 = fresh(g);
    C::run(s, tw2, true, g2, od);
    C::visit(fresh(g2), [&](int i, int col, auto q) {
        at32(scr, (unsigned)(i * C::SP + x0 + col)) = ev[q] + mulc(od[q], C::twist(tw2, i));
    });
}

// k_half_icols up to N' = 2048 by whole columns (full_cols): the N' / 16 threads of
// a column do one transform where the two parities' N / 16 did two in turn. In us, FP32
// at N' = 256, 1024 and 2048: 8.7 -> 6.4, 16.3 -> 10.4, 19.0 -> 14.1; FP64 at 512 and 2048:
// 9.8 -> 9.0, 21.8 -> 19.5. Not tried for larger columns (4 of 4096 points in FP32 fill
// 139 KB of LDS, one workgroup per CU in either form).
template <typename T, int LOGNP>
__global__ void __launch_bounds__((FullCol<T, LOGNP>::NT))
k_half_icols_full(const cx<T> *__restrict__ Y, cx<T> *__restrict__ scr, const cx<T> *__restrict__ tw, int pitch) {
    using C = FullCol<T, LOGNP>;
    extern __shared__ unsigned char smem_raw[];
    constexpr int NP = C::NP, N = NP / 2;
    cx<T> *s = reinterpret_cast<cx<T> *>(smem_raw);
    const int x0 = stripe_x0(C::CW);
    auto st = [&](int k1, int k2, int col, cx<T> v) {
        const int n = k1 + C::N1 * k2;     // wanted: n in [-N/2, N/2) mod N'
        if (in_band(n, N, NP)) at32(scr, (unsigned)((n & (N - 1)) * scratch_pitch(N) + x0 + col)) = v;
    };
    if (x0 != 0) {
        full_cols<T, LOGNP>(s, tw, true, [&](int ky, int col) { return at32(Y, (unsigned)(ky * pitch + x0 + col)); }, st);
    } else {
        // every lane loads what column 0 needs: no load waits behind a branch
        full_cols<T, LOGNP>(
            s, tw, true,
            [&](int ky, int col) {
                const int km = (NP - ky) & (NP - 1);
                const cx<T> a = at32(Y, (unsigned)(ky * pitch + col)), m = at32(Y, (unsigned)(km * pitch));
                const cx<T> b = at32(Y, (unsigned)(ky * pitch + N)), bm = at32(Y, (unsigned)(km * pitch + N));
                const cx<T> h0 = mk<T>((T)0.5 * (a.x + m.x), (T)0.5 * (a.y - m.y));
                const cx<T> hn = mk<T>((T)0.5 * (b.x + bm.x), (T)0.5 * (b.y - bm.y));
                return col == 0 ? mk<T>(h0.x - hn.y, h0.y + hn.x) : a;
            },
            st);
    }
}

// The two column launches of image side N = 2^logN (16 .. 4096).
template <typename T, int LOGN>
void half_cols_launch(ri_ctx *c, Prec<T> &p, const cx<T> *in, cx<T> *out, bool inv, hipStream_t s) {
    using C = ColFft<T, LOGN>;
    const int stripes = C::N / C::CW, pitch = half_pitch(C::N);
    if constexpr (LOGN <= 10) {
        using F = FullCol<T, LOGN + 1>;
        if (inv)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_half_icols_full<T, LOGN + 1>), dim3(C::N / F::CW), dim3(F::NT), F::LDS, s,
                               in, out, p.tw, pitch);
    } else {
        if (inv)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_half_icols<T, LOGN>), dim3(stripes), dim3(C::NT), C::LDS, s, in, out,
                               p.tw, pitch);
    }
    if constexpr (std::is_same<T, double>::value) {   // FP32 images go forwards by the whole plane
        if (!inv)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_half_cols<T, LOGN>), dim3(2 * stripes), dim3(C::NT), C::LDS, s, in, out,
                               p.tw, pitch);
    }
}

template <typename T>
void half_cols(ri_ctx *c, Prec<T> &p, const cx<T> *in, cx<T> *out, bool inv, hipStream_t s) {
    switch (c->logNp - 1) {
        case 4: return half_cols_launch<T, 4>(c, p, in, out, inv, s);
        case 5: return half_cols_launch<T, 5>(c, p, in, out, inv, s);
        case 6: return half_cols_launch<T, 6>(c, p, in, out, inv, s);
        case 7: return half_cols_launch<T, 7>(c, p, in, out, inv, s);
        case 8: return half_cols_launch<T, 8>(c, p, in, out, inv, s);
        case 9: return half_cols_launch<T, 9>(c, p, in, out, inv, s);
        case 10: return half_cols_launch<T, 10>(c, p, in, out, inv, s);
        case 11: return half_cols_launch<T, 11>(c, p, in, out, inv, s);
        case 12: return half_cols_launch<T, 12>(c, p, in, out, inv, s);
        default: throw Error(RI_EUNSUPPORTED, "image side outside 16 .. 4096");
    }
}

template <typename T, int L>
constexpr int lanes_per_column() { return (L * (int)sizeof(cx<T>)) / 512 < 1 ? 1 : (L * (int)sizeof(cx<T>)) / 512; }


// Column transforms of grid_io (scratch) into grid_out; grid_out == grid_io
// leaves the second pass in place (permuted rows). band: the N packed band rows
// when they are the input (N' = 8192 in FP32, forward), else NULL.
template <typename T>
void colfft(ri_ctx *c, cx<T> *grid_io, cx<T> *grid_out, const cx<T> *tw, bool inv, bool band_in, bool band_out,
            hipStream_t s, const cx<T> *band = nullptr) {
    const int logNp = c->logNp, Np = c->Np;
    const int logN1 = full_log_n1(logNp), logN2 = logNp - logN1;
    if (logNp == 12 || logNp == 13) {
        // 4096 = 64 x 64 and 8192 = 128 x 64: both column passes in registers,
        // at most 64 complex FP32 (32 FP64) points per lane
        constexpr int QA4 = lanes_per_column<T, 64>(), QA8 = lanes_per_column<T, 128>();
        constexpr int QB = lanes_per_column<T, 64>();
        if (logNp == 12)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_colpass_a_reg<T, 64, QA4>), dim3(Np / (64 / QA4), 64), dim3(64), 0,
                               s, grid_io, tw, c->N, logNp, band_in ? 1 : 0, inv ? 1 : 0);
        else if (band != nullptr)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_colpass_a_band<T>), dim3(Np / 64, 64, 2), dim3(64), 0, s, band,
                               grid_io, tw, logNp);
        else
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_colpass_a_reg<T, 128, QA8>), dim3(Np / (64 / QA8), 64), dim3(64), 0,
                               s, grid_io, tw, c->N, logNp, band_in ? 1 : 0, inv ? 1 : 0);
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_colpass_b_reg<T, 64, QB>), dim3(Np / (64 / QB), Np / 64), dim3(64), 0, s,
                           (const cx<T> *)grid_io, grid_out, tw, c->N, logNp, band_out ? 1 : 0, inv ? 1 : 0);
        return;
    }
    auto launch = [&](auto LOGNP) {
        using C = FullCol<T, decltype(LOGNP)::value>;
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_colfft<T, decltype(LOGNP)::value>), dim3(Np / C::CW), dim3(C::NT), C::LDS,
                           s, (const cx<T> *)grid_io, grid_out, tw, c->N, band_in ? 1 : 0, band_out ? 1 : 0,
                           inv ? 1 : 0);
    };
    switch (logNp) {
        case 5: return launch(std::integral_constant<int, 5>{});
        case 6: return launch(std::integral_constant<int, 6>{});
        case 7: return launch(std::integral_constant<int, 7>{});
        case 8: return launch(std::integral_constant<int, 8>{});
        case 9: return launch(std::integral_constant<int, 9>{});
        case 10: return launch(std::integral_constant<int, 10>{});
        case 11: return launch(std::integral_constant<int, 11>{});
        default: throw Error(RI_EUNSUPPORTED, "image side outside 16 .. 4096");
    }
}

}  // namespace

// f(integral_constant<int, log2 N'>) for the context's N'.
template <typename F>
void with_log(int logNp, F &&f) {
    switch (logNp) {
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 9: return f(std::integral_constant<int, 9>{});
        case 10: return f(std::integral_constant<int, 10>{});
        case 11: return f(std::integral_constant<int, 11>{});
        case 12: return f(std::integral_constant<int, 12>{});
        case 13: return f(std::integral_constant<int, 13>{});
        default: throw Error(RI_EUNSUPPORTED, "image side outside 16 .. 4096");
    }
}

// Z and the row FFTs of x into dst (rows as k_zpad_rowfft places them).
template <typename T>
void launch_zpad_rows(ri_ctx *c, Prec<T> &p, const T *x, cx<T> *dst, const cx<T> *chirp, int rowmask,
                      const Clear<T> &z, hipStream_t s) {
    with_log(c->logNp, [&](auto LOG) {
        using F = RowFft<T, decltype(LOG)::value>;
        if (chirp)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_zpad_rowfft<T, decltype(LOG)::value, true>), dim3(c->N), dim3(F::NT),
                               F::LDS, s, x, dst, p.icorr, p.tw, chirp, rowmask, z);
        else
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_zpad_rowfft<T, decltype(LOG)::value, false>), dim3(c->N), dim3(F::NT),
                               F::LDS, s, x, dst, p.icorr, p.tw, chirp, rowmask, z);
    });
}

template <typename T>
void require_row_fits(ri_ctx *c) {
    if (sizeof(cx<T>) * (size_t)(c->Np + c->Np / 32) > (size_t)c->dev.lds_per_block)
        throw Error(RI_EUNSUPPORTED, "grid row does not fit the workgroup LDS");
}

// x (N x N) -> F Z_s x in p.gridB[s] for every w-stack s (row FFT into gridA band rows,
// columns A in place, B into gridB[s])
template <typename T>
void fwd_zpad_fft(ri_ctx *c, Prec<T> &p, const T *x, hipStream_t s) {
    const int Np = c->Np;
    ProfScope prof(c, PROF_FFT, s);
    require_row_fits<T>(c);
    // one FFT per w-stack (a single one without stacking); gridA is the scratch
    for (int st = 0; st < c->P; ++st) {
        launch_zpad_rows<T>(c, p, x, p.gridA, c->P > 1 ? p.chirp + (size_t)st * c->N * c->N : nullptr, Np - 1,
                            Clear<T>(), s);
        colfft<T>(c, p.gridA, p.gridB + (size_t)st * Np * Np, p.tw, false, true, false, s);
    }
}

// p.gridA (Y_s = G_s^H r, one full grid per w-stack) -> Re sum_s Z_s^dagger F^dagger Y_s
// into x (N x N); gridA is clobbered and gridB[0] serves as the scratch.
template <typename T>
void adj_fft_crop(ri_ctx *c, Prec<T> &p, T *x, hipStream_t s) {
    const int Np = c->Np;
    ProfScope prof(c, PROF_FFT, s);
    for (int st = 0; st < c->P; ++st) {
        const cx<T> *ch = c->P > 1 ? p.chirp + (size_t)st * c->N * c->N : nullptr;
        colfft<T>(c, p.gridA + (size_t)st * Np * Np, p.gridB, p.tw, true, false, true, s);
        with_log(c->logNp, [&](auto LOG) {
            using F = RowFft<T, decltype(LOG)::value>;
            if (ch)
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_irowfft_crop<T, decltype(LOG)::value, true>), dim3(c->N),
                                   dim3(F::NT), F::LDS, s, p.gridB, x, p.icorr, p.tw, ch, st > 0 ? 1 : 0);
            else
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_irowfft_crop<T, decltype(LOG)::value, false>), dim3(c->N),
                                   dim3(F::NT), F::LDS, s, p.gridB, x, p.icorr, p.tw, ch, st > 0 ? 1 : 0);
        });
    }
}

template <typename T>
Clear<T> pass_clear(ri_ctx *c, Prec<T> &p, bool with_grid, int32_t *counter, double *part) {
    Clear<T> z;
    z.grid = p.gridA;
    if (with_grid) z.n = c->P == 1 ? (int64_t)c->Np * half_pitch(c->N) : (int64_t)c->P * c->Np * c->Np;
    z.counter = counter;
    z.part = part;
    z.npart = part ? c->n_partials : 0;
    return z;
}

template <typename T>
void clear(const Clear<T> &z, hipStream_t s) {
    const int64_t n = std::max<int64_t>(z.n * (int64_t)sizeof(cx<T>) / 16, z.npart);
    hipLaunchKernelGGL(k_clear<T>, dim3((int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096))),
                       dim3(256), 0, s, z);
}

// The scratch lies in gridB behind the half-plane grid: N'(pitch) + N sp <= N'^2 cells.
template <typename T>
cx<T> *half_scratch(ri_ctx *c, Prec<T> &p) { return p.gridB + (size_t)c->Np * half_pitch(c->N); }

template <typename T>
void fwd_half_fft(ri_ctx *c, Prec<T> &p, const T *x, const Clear<T> &z, hipStream_t s) {
    const int N = c->N, Np = c->Np;
    ProfScope prof(c, PROF_FFT, s);
    cx<T> *scr = half_scratch<T>(c, p);
    with_log(c->logNp, [&](auto LOG) {
        using F = RowFft<T, decltype(LOG)::value>;
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_half_rows<T, decltype(LOG)::value>), dim3(c->N / 2), dim3(F::NT), F::LDS, s,
                           x, scr, p.icorr, p.tw, z);
    });
    half_cols<T>(c, p, scr, p.gridB, false, s);
}

template <typename T>
void adj_half_fft(ri_ctx *c, Prec<T> &p, T *x, hipStream_t s) {
    const int N = c->N, Np = c->Np;
    ProfScope prof(c, PROF_FFT, s);
    cx<T> *scr = half_scratch<T>(c, p);
    half_cols<T>(c, p, p.gridA, scr, true, s);
    with_log(c->logNp, [&](auto LOG) {
        using F = RowFft<T, decltype(LOG)::value>;
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_half_irows<T, decltype(LOG)::value>), dim3(c->N / 2), dim3(F::NT), F::LDS, s,
                           scr, x, p.icorr, p.tw);
    });
}

// Whole plane of one real image into gridB, all passes in place there (rows
// end permuted, see full_log_n1), which leaves gridA to be cleared by the row launch. At
// N' = 8192 in FP32 the row spectra pass through the part of gridA behind the
// half-plane output grid (k_colpass_a_band works out of place).
template <typename T>
void fwd_full_fft(ri_ctx *c, Prec<T> &p, const T *x, const Clear<T> &z, hipStream_t s) {
    ProfScope prof(c, PROF_FFT, s);
    cx<T> *band = nullptr;
    if (packs_band<T>(c)) band = p.gridA + (size_t)c->Np * half_pitch(c->N);
    launch_zpad_rows<T>(c, p, x, band ? band : p.gridB, nullptr, band ? c->N - 1 : c->Np - 1, z, s);
    colfft<T>(c, p.gridB, p.gridB, p.tw, false, true, false, s, band);
}

template <typename T>
void operator_fft(ri_ctx *c, Prec<T> &p, bool folded, const T *x, const Clear<T> &z, hipStream_t s) {
    require_row_fits<T>(c);
    if (c->P > 1) {   // each stack's image is complex (its phase screen)
        fwd_zpad_fft<T>(c, p, x, s);
        clear<T>(z, s);
        return;
    }
    if constexpr (std::is_same<T, double>::value) {
        if (folded) return fwd_half_fft<T>(c, p, x, z, s);
    }
    fwd_full_fft<T>(c, p, x, z, s);
}

template <typename T>
void operator_adj_fft(ri_ctx *c, Prec<T> &p, T *x, hipStream_t s) {
    if (c->P == 1) adj_half_fft<T>(c, p, x, s);
    else adj_fft_crop<T>(c, p, x, s);
}

template Clear<float> pass_clear<float>(ri_ctx *, Prec<float> &, bool, int32_t *, double *);
template Clear<double> pass_clear<double>(ri_ctx *, Prec<double> &, bool, int32_t *, double *);
template void clear<float>(const Clear<float> &, hipStream_t);
template void clear<double>(const Clear<double> &, hipStream_t);
template void operator_fft<float>(ri_ctx *, Prec<float> &, bool, const float *, const Clear<float> &, hipStream_t);
template void operator_fft<double>(ri_ctx *, Prec<double> &, bool, const double *, const Clear<double> &, hipStream_t);
template void operator_adj_fft<float>(ri_ctx *, Prec<float> &, float *, hipStream_t);
template void operator_adj_fft<double>(ri_ctx *, Prec<double> &, double *, hipStream_t);
template void fwd_zpad_fft<float>(ri_ctx *, Prec<float> &, const float *, hipStream_t);
template void fwd_zpad_fft<double>(ri_ctx *, Prec<double> &, const double *, hipStream_t);
template void adj_fft_crop<float>(ri_ctx *, Prec<float> &, float *, hipStream_t);
template void adj_fft_crop<double>(ri_ctx *, Prec<double> &, double *, hipStream_t);

}  // namespace ri
