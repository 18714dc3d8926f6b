// Batched dense objective on the matrix cores:
//   forward   Y = A X,  f = sum W (.) psi(Y)  (epilogue),  V = W (.) psi'(Y)
//   backward  G = fbar * A^T V
//
// Both products are m x m by m x n contractions on the matrix cores.  FP64:
// v_mfma_f64_16x16x4_f64.  FP32, small: v_mfma_f32_16x16x4_f32, 16 terms at a
// time.  FP32, large: each operand is split into three bfloat16 parts (8 + 8 +
// 8 bits, nearest) and eight of their nine products run on
// v_mfma_f32_16x16x32_bf16, 32 terms at a time, the leading parts' apart from
// the others.  Every FP32 sum is added into FP64 accumulators and the next
// starts from zero, so every longer accumulation is FP64.  A wave
// loads its operand fragments from global memory straight into the registers
// the instruction reads, a k-step or more ahead, so there is no LDS staging
// and no barrier in the k loop (but for the split of large FP32 tiles, whose
// waves share it); the nonlinearity and its derivative are fused
// into the forward epilogue, so neither Y nor psi(Y) round-trips through HBM;
// the objective is reduced per tile and then in a fixed order (deterministic).
#include <type_traits>

#include "device_common.hpp"
#include "launch.hpp"

namespace pg {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// The arithmetic of a product.
enum Arith {
    FP64 = 0,   // v_mfma_f64_16x16x4_f64
    FP32 = 1,   // v_mfma_f32_16x16x4_f32, 16 terms to a sum
    SPLIT = 2,  // FP32 operands in three bfloat16 parts, 32 terms to a sum
};

template <typename T>
struct Mfma;

template <>
struct Mfma<double> {
    using acc_t = d4;
    __device__ static acc_t mac(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // Output row (within the 16 x 16 block) of register r in lanes 16*g .. 16*g+15.
    __device__ static int row(int g, int r) { return g + 4 * r; }
};

template <>
struct Mfma<float> {
    using acc_t = f4;
    __device__ static acc_t mac(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ static int row(int g, int r) { return 4 * g + r; }
};

// 2^16 v = h + m + l, each the nearest bfloat16 of what is left: bfloat16 has
// FP32's exponents but ends at 2^-133, 16 places above FP32's last subnormal
// bit, so the factor keeps the low parts of the smallest values.  A value that
// the factor takes past the largest bfloat16, an infinity or a NaN has parts
// that are not finite, and so have the products (the caller then repeats
// them in FP32).
constexpr float kSplitScale = 65536.f;
struct Split {
    uint32_t h[4], m[4], l[4];  // two parts to a register
};
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, bf2));
}
__device__ __forceinline__ float low_bf16(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float high_bf16(uint32_t p) { return __builtin_bit_cast(float, p & 0xffff0000u); }
__device__ __forceinline__ bf8 parts(const uint32_t (&p)[4]) { return __builtin_bit_cast(bf8, p); }

__device__ __forceinline__ Split split3(const float (&v)[8]) {
    Split s;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float v0 = v[2 * e] * kSplitScale, v1 = v[2 * e + 1] * kSplitScale;
        s.h[e] = pack_bf16(v0, v1);
        const float r0 = v0 - low_bf16(s.h[e]), r1 = v1 - high_bf16(s.h[e]);
        s.m[e] = pack_bf16(r0, r1);
        s.l[e] = pack_bf16(r0 - low_bf16(s.m[e]), r1 - high_bf16(s.m[e]));
    }
    return s;
}

// 32 products per entry: the leading parts' in a sum of their own, which goes
// into the FP64 sums at once, and the other parts', some 2^-8 of it, in a sum
// that runs on for kLowSteps k-steps.  (In one sum the small products lose to
// the large ones: the instruction aligns eight terms at a time to their largest
// and truncates.)  Left out is l l, 2^-34 of a product.  Entry error of a
// gradient, rms over sum |a| |b|, against v_mfma_f32_16x16x4_f32 in sums of 16
// / one sum of the six largest products / this (1,056 x 1,000): a ~ N(0,1/m), b
// ~ U(-1,1) 3.5e-9 / 2.4e-9 / 1.6e-9; one term to an entry 2.52e-8 / 3.32e-8 /
// 2.53e-8 (largest 5.96e-8 / 1.45e-7 / 5.97e-8: the rounding of the result);
// sums that cancel 7.0e-10 / 1.2e-9 / 1.7e-11; rows and columns of magnitudes
// 2^-20 to 2^10 7.4e-9 / 7.7e-9 / 6.2e-9.  Operands log-uniform over e^+-10
// are the exception: 1.78e-8 / 2.16e-8 / 1.96e-8 (largest 1.39e-7 / 1.28e-7 /
// 1.30e-7).
constexpr int kLowSteps = 8;
__device__ __forceinline__ f4 mma_high(const Split& a, const Split& b) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(parts(a.h), parts(b.h), f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
}
__device__ __forceinline__ f4 mma_low(const Split& a, const Split& b, f4 c) {
    const bf8 ah = parts(a.h), am = parts(a.m), al = parts(a.l);
    const bf8 bh = parts(b.h), bm = parts(b.m), bl = parts(b.l);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bm, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bl, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bm, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bh, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bm, c, 0, 0, 0);
    return c;
}

enum Epi { EPI_FWD = 0, EPI_BWD = 1 };

// VN consecutive elements with the alignment of one (the compiler picks the
// widest load the target allows for it).
template <typename T, int VN>
__device__ __forceinline__ void load_vec(const T* __restrict__ p, T (&o)[VN]) {
    typedef T V __attribute__((ext_vector_type(VN), aligned(sizeof(T))));
    const V v = *reinterpret_cast<const V*>(p);
#pragma unroll
    for (int c = 0; c < VN; ++c) o[c] = v[c];
}
template <typename T>
__device__ __forceinline__ void load_vec(const T* __restrict__ p, T (&o)[1]) {
    o[0] = *p;
}

// Tile shape: a wave owns BX x BY MFMA blocks (16 BX x 16 BY of C); a
// workgroup has WM x WN such wave tiles and KW waves on each, which split the
// contraction among them and are summed through LDS.  D k-steps are in
// flight; the registers allow OCC waves per SIMD at least.
template <int BX_, int BY_, int WM_, int WN_, int KW_, int D64, int D32, int OCC_>
struct Shape {
    static constexpr int BX = BX_, BY = BY_, WM = WM_, WN = WN_, KW = KW_, OCC = OCC_;
    template <typename T>
    static constexpr int D = sizeof(T) == 8 ? D64 : D32;
    static constexpr int NWAVES = WM * WN * KW, NTHR = 64 * NWAVES;
    static constexpr int TM = 16 * BX * WM, TN = 16 * BY * WN;
};

// One k-step of both operands as a lane holds them.
template <typename T, int E, int BX, int BY>
struct Frag {
    T a[E][BX];
    T b[E][BY];
};

// C[M x N] = op(A)[M x K] * Bm[K x N].
//   TRANS_A == false: op(A)[i][k] = A[i * K + k]   (forward, A is m x m)
//   TRANS_A == true:  op(A)[i][k] = A[k * M + i]   (backward, A^T)
// A lane's rows of a block are i0 + 16 x + li (forward; consecutive k in one
// load) or i0 + BX li + x (backward; BX consecutive rows in one load); its
// columns are j0 + BY li + y, so operand B, C and W are read and written BY
// columns at a time.  A wave whose block would reach past the edge takes the
// last whole block instead and stores only its own part of it (a block of one
// 16 x 16 reads the last row or column again instead), so the loads need no
// bounds checks; the caller offers only shapes whose blocks fit C.
//
// Bound by the matrix cores in FP64 (67 TFLOP/s of 78.6 at 4096 x 1024, 59 with
// the tiles staged through LDS and a barrier per k-step), by the vector
// instructions of the split and the FP64 sums, beside the eight products, in
// FP32 (4,096 x 1,024: 530-580 us a gradient, 118-130 TFLOP/s; 1,323 on
// v_mfma_f32_16x16x4_f32; six products in one sum, which was less accurate, 456),
// and by latency below some 500 x 500: 257 x 129 takes 10.6 us per FP32 gradient.
template <typename T, int AR, bool TRANS_A, int EPI, typename S>
__global__ void __launch_bounds__(S::NTHR, S::OCC)
k_gemm_mfma(const T* __restrict__ A, const T* __restrict__ Bm, int64_t M, int64_t N, int64_t K,
            const T* __restrict__ W, double* __restrict__ partials, T* __restrict__ Vout,
            const double* __restrict__ fbar, T* __restrict__ Gout, int accumulate, int tiles_n,
            int64_t np, double* __restrict__ f_out) {
    using MF = Mfma<T>;
    using acc_t = typename MF::acc_t;
    constexpr int BX = S::BX, BY = S::BY, D = S::template D<T>, KW = S::KW;
    static_assert((AR == FP64) == (sizeof(T) == 8), "FP64 arithmetic for FP64 operands");
    // A k-step is 4 E deep; a lane (li, lk) holds E of them: consecutive ones,
    // or, for the FP32 instruction, every fourth, so that a 16-term sum takes
    // its terms in ascending k.
    constexpr int E = AR == SPLIT ? 8 : 4, KS = 4 * E;
    constexpr int kBase = AR == FP32 ? 1 : E, kStep = AR == FP32 ? 4 : 1;
    constexpr bool kWide = AR != FP64;
    using F = Frag<T, E, BX, BY>;
    // SPLIT, at least as many waves side by side as A blocks to a wave: they
    // have the same A rows, and BX of them split one block each for all, through
    // LDS.
    constexpr bool kShare = AR == SPLIT && BX > 2 && S::WN >= BX;
    static_assert(BX != 3 || kShare, "blocks of three rows only where they are read one by one");
    constexpr int kPartBytes = KW > 1 ? KW * S::WM * S::WN * BX * BY * 4 * 64 * 8 : 16;
    constexpr int kShareBytes = kShare ? KW * S::WM * 2 * BX * (int)sizeof(Split) * 64 : 16;
    __shared__ alignas(16) unsigned char smem[kPartBytes > kShareBytes ? kPartBytes : kShareBytes];
    __shared__ double red[16];
    // Backward: a workgroup past the tiles sums the forward's partials of f.
    const uint32_t tiles = gridDim.x - (EPI == EPI_BWD && f_out ? 1 : 0);
    if (EPI == EPI_BWD && blockIdx.x == tiles) {
        const double f = final_sum_block<false>(partials, np, red);
        if (threadIdx.x == 0) f_out[0] = f;
        return;
    }

    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int wmn = wid % (S::WM * S::WN), kw = wid / (S::WM * S::WN);
    const uint32_t tile = xcd_remap(blockIdx.x, tiles);
    // First row / column of wave block q, and of the whole block it reads.
    const int64_t ti = (int64_t)(tile / tiles_n) * S::TM, tj = (int64_t)(tile % tiles_n) * S::TN;
    auto own_i = [&](int q) { return ti + (q / S::WN) * (16 * BX); };
    auto own_j = [&](int q) { return tj + (q % S::WN) * (16 * BY); };
    auto low = [](int64_t a, int64_t b) { return a < b ? a : b; };
    auto read_i = [&](int64_t i) { return BX > 1 ? low(i, M - 16 * BX) : i; };
    auto read_j = [&](int64_t j) { return BY > 1 ? low(j, N - 16 * BY) : j; };
    const int64_t i0 = read_i(own_i(wmn)), j0 = read_j(own_j(wmn));
    const bool any = own_i(wmn) < M && own_j(wmn) < N;

    // This wave's k range: whole steps, the remainder of K with the last one.
    const int64_t steps = K / KS;
    const int64_t t0 = steps * kw / KW, t1 = steps * (kw + 1) / KW;
    const int64_t kbeg = t0 * KS, kend = kw == KW - 1 ? K : t1 * KS;

    const T* pa[TRANS_A ? 1 : BX];
    if constexpr (TRANS_A) {
        pa[0] = A + low(i0 + BX * li, M - BX) + (kbeg + kBase * lk) * M;
    } else {
#pragma unroll
        for (int x = 0; x < BX; ++x) pa[x] = A + low(i0 + 16 * x + li, M - 1) * K + (kbeg + kBase * lk);
    }
    const T* pb = Bm + low(j0 + BY * li, N - BY) + (kbeg + kBase * lk) * N;

    // FP64: the running sums; FP32 instruction: the 16-term sums; split: the
    // small parts' sums
    acc_t acc[BX][BY];
    double wide[kWide ? BX : 1][kWide ? BY : 1][4];
    auto clear = [&]() {
#pragma unroll
        for (int x = 0; x < BX; ++x)
#pragma unroll
            for (int y = 0; y < BY; ++y) {
                acc[x][y] = acc_t{0, 0, 0, 0};
                if constexpr (kWide)
#pragma unroll
                    for (int r = 0; r < 4; ++r) wide[x][y][r] = 0.0;
            }
    };
    clear();
    auto load = [&](F& f, int64_t t) {
        const int64_t k = t * KS;
        if constexpr (!TRANS_A) {
#pragma unroll
            for (int x = 0; x < BX; ++x) {
                if constexpr (kStep == 1) {
                    T v[E];
                    load_vec<T, E>(pa[x] + k, v);
#pragma unroll
                    for (int e = 0; e < E; ++e) f.a[e][x] = v[e];
                } else {
#pragma unroll
                    for (int e = 0; e < E; ++e) f.a[e][x] = pa[x][k + kStep * e];
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) load_vec(pa[0] + (k + kStep * e) * M, f.a[e]);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) load_vec(pb + (k + kStep * e) * N, f.b[e]);
    };
    // FP32: the 16-term sums (split: the small parts') into the FP64 ones.
    [[maybe_unused]] auto fold = [&]() {
#pragma unroll
        for (int x = 0; x < BX; ++x)
#pragma unroll
            for (int y = 0; y < BY; ++y) {
#pragma unroll
                for (int r = 0; r < 4; ++r) wide[x][y][r] += (double)acc[x][y][r];
                acc[x][y] = acc_t{0, 0, 0, 0};
            }
    };
    // The products of one k-step; next() is called once f has been read.
    auto mma = [&](const F& f, auto next) {
        if constexpr (AR != SPLIT) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int x = 0; x < BX; ++x)
#pragma unroll
                    for (int y = 0; y < BY; ++y) acc[x][y] = MF::mac(f.a[s][x], f.b[s][y], acc[x][y]);
            next();
            if constexpr (kWide) fold();
        } else {
            Split a[BX], b[BY];
#pragma unroll
            for (int x = 0; x < BX; ++x) {
                float v[E];
#pragma unroll
                for (int e = 0; e < E; ++e) v[e] = f.a[e][x];
                a[x] = split3(v);
            }
#pragma unroll
            for (int y = 0; y < BY; ++y) {
                float v[E];
#pragma unroll
                for (int e = 0; e < E; ++e) v[e] = f.b[e][y];
                b[y] = split3(v);
            }
            next();
#pragma unroll
            for (int y = 0; y < BY; ++y)
#pragma unroll
                for (int x = 0; x < BX; ++x) {
                    const f4 c = mma_high(a[x], b[y]);
                    acc[x][y] = mma_low(a[x], b[y], acc[x][y]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) wide[x][y][r] += (double)c[r];
                }
        }
    };
    const int64_t n = t1 - t0;
    if constexpr (kShare) {
        // One barrier per k-step.  Between two of them a wave multiplies step t
        // while it splits its share of step t + 1 into the other buffer and
        // loads step t + 2.  Every wave takes every barrier, also one past the
        // edge of C (it reads the last whole block) and one whose part of K is
        // a step shorter.
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        const int xs = wmn % S::WN;
        u4* const shared_a = reinterpret_cast<u4*>(smem) + (int64_t)(kw * S::WM + wmn / S::WN) * 2 * BX * 3 * 64 + lane;
        const bool splits_a = xs < BX;
        const int xa = splits_a ? xs : 0;
        const T* const own = TRANS_A ? pa[0] + xa : A + low(i0 + 16 * xa + li, M - 1) * K + (kbeg + kBase * lk);
        float ra[E], rb[E][BY];
        Split sb[BY];
        auto load1 = [&](int64_t t) {
            const int64_t k = t * KS;
            if (BX == S::WN || splits_a) {
                if constexpr (TRANS_A) {
#pragma unroll
                    for (int e = 0; e < E; ++e) ra[e] = own[(k + e) * M];
                } else {
                    load_vec<T, E>(own + k, ra);
                }
            }
#pragma unroll
            for (int e = 0; e < E; ++e) load_vec(pb + (k + e) * N, rb[e]);
        };
        auto share = [&](int64_t t, Split (&o)[BY]) {
            if (BX == S::WN || splits_a) {
                const Split a = split3(ra);
                u4* const q = shared_a + ((t & 1) * BX + xs) * 3 * 64;
                q[0] = u4{a.h[0], a.h[1], a.h[2], a.h[3]};
                q[64] = u4{a.m[0], a.m[1], a.m[2], a.m[3]};
                q[128] = u4{a.l[0], a.l[1], a.l[2], a.l[3]};
            }
#pragma unroll
            for (int y = 0; y < BY; ++y) {
                float v[E];
#pragma unroll
                for (int e = 0; e < E; ++e) v[e] = rb[e][y];
                o[y] = split3(v);
            }
        };
        auto multiply = [&](int64_t t) {
#pragma unroll
            for (int x = 0; x < BX; ++x) {
                const u4* const q = shared_a + ((t & 1) * BX + x) * 3 * 64;
                const u4 h = q[0], m = q[64], l = q[128];
                const Split a{{h[0], h[1], h[2], h[3]}, {m[0], m[1], m[2], m[3]}, {l[0], l[1], l[2], l[3]}};
#pragma unroll
                for (int y = 0; y < BY; ++y) {
                    const f4 c = mma_high(a, sb[y]);
                    acc[x][y] = mma_low(a, sb[y], acc[x][y]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) wide[x][y][r] += (double)c[r];
                }
            }
        };
        const int64_t nmin = steps / KW, nmax = (steps + KW - 1) / KW;
        if (n > 0) {
            load1(0);
            share(0, sb);
            if (n > 1) load1(1);
        }
        __syncthreads();
        int64_t t = 0;
        for (; t + 2 < nmin; ++t) {
            Split next[BY];
            share(t + 1, next);
            load1(t + 2);
            multiply(t);
            if ((t & (kLowSteps - 1)) == kLowSteps - 1) fold();
#pragma unroll
            for (int y = 0; y < BY; ++y) sb[y] = next[y];
            __syncthreads();
        }
        for (; t < nmax; ++t) {
            Split next[BY] = {};
            if (t + 1 < n) share(t + 1, next);
            if (t + 2 < n) load1(t + 2);
            if (t < n) multiply(t);
#pragma unroll
            for (int y = 0; y < BY; ++y) sb[y] = next[y];
            __syncthreads();
        }
    } else if (any) {
        F f[D];
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < n) load(f[d], d);
        int64_t t = 0;
        for (; t + 2 * D <= n; t += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) mma(f[d], [&] { load(f[d], t + d + D); });
            if constexpr (AR == SPLIT) {
                static_assert(kLowSteps % D == 0, "t is a multiple of D");
                if ((t & (kLowSteps - D)) == kLowSteps - D) fold();
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (t + d < n)
                mma(f[d], [&] {
                    if (t + d + D < n) load(f[d], t + d + D);
                });
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (t + d + D < n) mma(f[d], [] {});
    }
    if (any) {
        if (t1 * KS < kend) {
            // the last K % KS products: k past the end contributes zero
            const int64_t k0 = n * KS;
            F z;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int dk = kStep * e;
                const bool in = t1 * KS + kBase * lk + dk < K;
#pragma unroll
                for (int x = 0; x < BX; ++x)
                    z.a[e][x] = in ? (TRANS_A ? pa[0][(k0 + dk) * M + x] : pa[TRANS_A ? 0 : x][k0 + dk]) : T(0);
#pragma unroll
                for (int y = 0; y < BY; ++y) z.b[e][y] = in ? pb[(k0 + dk) * N + y] : T(0);
            }
            mma(z, [] {});
        }
        if constexpr (AR == SPLIT) {
            fold();
            // An operand or a sum that is not finite: the whole block again on
            // the FP32 instruction, whose infinities are those of the sums.
            bool bad = false;
#pragma unroll
            for (int x = 0; x < BX; ++x)
#pragma unroll
                for (int y = 0; y < BY; ++y)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        wide[x][y][r] *= 1.0 / ((double)kSplitScale * kSplitScale);
                        bad |= !__builtin_isfinite(wide[x][y][r]);
                    }
            if (__any(bad)) {
                clear();
                const int64_t ra = kbeg + E * lk, rb = ra;  // k of pa[.][0] and pb[0]
                for (int64_t k0 = kbeg; k0 < kend; k0 += 16) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const int64_t k = k0 + 4 * s + lk;
                        const bool in = k < kend;
                        T av[BX], bv[BY];
#pragma unroll
                        for (int x = 0; x < BX; ++x)
                            av[x] = in ? (TRANS_A ? pa[0][(k - ra) * M + x] : pa[TRANS_A ? 0 : x][k - ra]) : T(0);
#pragma unroll
                        for (int y = 0; y < BY; ++y) bv[y] = in ? pb[(k - rb) * N + y] : T(0);
#pragma unroll
                        for (int x = 0; x < BX; ++x)
#pragma unroll
                            for (int y = 0; y < BY; ++y)
                                acc[x][y] = MF::mac(av[x], bv[y], acc[x][y]);
                    }
                    fold();
                }
            }
        }
    }

    double tsum = 0.0;
    const double fb = (EPI == EPI_BWD && fbar) ? fbar[0] : 1.0;
    // Stores an entry of wave block q unless it belongs to another wave.
    auto emit = [&](int q, int64_t gi, int64_t gj, double c) {
        if (gi < own_i(q) || gi >= M || gj < own_j(q) || gj >= N) return;
        const int64_t o = gi * N + gj;
        if constexpr (EPI == EPI_FWD) {
            const double s2 = c * c, wv = to_f64(W[o]);
            tsum += wv * psi_from_sq(s2);
            if (Vout) Vout[o] = static_cast<T>(wv * dpsi_from(c, s2));
        } else {
            const double g = fb * c;
            Gout[o] = accumulate ? static_cast<T>(to_f64(Gout[o]) + g) : static_cast<T>(g);
        }
    };
    auto value = [&](int x, int y, int r) -> double {
        if constexpr (kWide)
            return wide[x][y][r];
        else
            return acc[x][y][r];
    };
    // Register r of lane (li, lk) holds row MF::row(lk, r) and column li of a
    // block: the FP64 instruction interleaves rows across registers (lk + 4r),
    // the FP32 one keeps them in consecutive registers (4 lk + r).
    auto row_of = [&](int x, int rho) { return TRANS_A ? BX * rho + x : 16 * x + rho; };
    if constexpr (KW == 1) {
#pragma unroll
        for (int x = 0; x < BX; ++x)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int y = 0; y < BY; ++y)
                    emit(wmn, i0 + row_of(x, MF::row(lk, r)), j0 + BY * li + y, value(x, y, r));
    } else {
        // The KW partial sums of each entry, added in ascending k order; the
        // entries are dealt to all the waves.
        constexpr int NS = S::WM * S::WN * BX * BY * 4;  // 64-entry slices of the tile
        static_assert(KW * NS * 64 * 8 == kPartBytes, "room for the partial sums");
        double(*const part)[NS][64] = reinterpret_cast<double(*)[NS][64]>(smem);
#pragma unroll
        for (int x = 0; x < BX; ++x)
#pragma unroll
            for (int y = 0; y < BY; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r) part[kw][((wmn * BX + x) * BY + y) * 4 + r][lane] = value(x, y, r);
        __syncthreads();
        for (int q = wid; q < NS; q += S::NWAVES) {
            double c = part[0][q][lane];
#pragma unroll
            for (int k = 1; k < KW; ++k) c += part[k][q][lane];
            const int r = q & 3, y = (q >> 2) % BY, x = (q >> 2) / BY % BX, w2 = (q >> 2) / (BX * BY);
            emit(w2, read_i(own_i(w2)) + row_of(x, MF::row(lk, r)), read_j(own_j(w2)) + BY * li + y, c);
        }
    }
    if constexpr (EPI == EPI_FWD) {
        const double s = block_sum<S::NTHR>(tsum, red);
        if (threadIdx.x == 0) partials[tile] = s;
    }
}

// A workgroup has eight waves in every shape; they share a tile by splitting
// it or the contraction (not one of a step or two: 16 x 256).  Large tiles move the fewest operand bytes, small
// ones fill the device when C is small.  Two workgroups per compute unit (four
// waves per SIMD) with one k-step in flight beat one with two or three for the
// middle shapes (3,000 x 500, FP64 / FP32: 64 x 32 341 / 255 -> 334 / 230 us,
// 32 x 32 381 / 308 -> 353 / 244 us).
using S0 = Shape<4, 2, 2, 4, 1, 2, 1, 2>;  // 128 x 128
using S1 = Shape<4, 2, 1, 4, 2, 2, 1, 2>;  // 64 x 128
using S2 = Shape<2, 2, 2, 2, 2, 1, 1, 4>;  // 64 x 64
using S3 = Shape<2, 2, 2, 1, 4, 1, 1, 4>;  // 64 x 32
using S4 = Shape<2, 2, 1, 1, 8, 1, 1, 4>;  // 32 x 32
using S5 = Shape<2, 1, 1, 1, 8, 3, 2, 2>;  // 32 x 16
using S6 = Shape<1, 1, 1, 1, 8, 4, 2, 2>;  // 16 x 16, the one that takes any size
using S7 = Shape<3, 2, 1, 4, 2, 2, 1, 2>;  // 48 x 128, split FP32 operands only
using S8 = Shape<1, 2, 1, 8, 1, 1, 1, 4>;  // 16 x 256, for contractions too short to share
struct ShapeInfo {
    int tm, tn, bx, by;
    double cost[3], entry[3];  // by Arith
};
template <typename S>
constexpr ShapeInfo info(double c64, double c32, double split, double e64, double e32, double esplit) {
    return {S::TM, S::TN, S::BX, S::BY, {c64, c32, split}, {e64, e32, esplit}};
}
constexpr double kNever = 1e9;  // not built

// Whether FP32 operands are split.  Gradients, FP32 instruction / split, us, each
// in its best shape: 300 x 300 13.5 / 17.7, 512 x 512 20.6 / 19.7, 700 x 700 37.4
// / 43.2, 900 x 900 79 / 65, 1,000 x 1,000 95 / 73, 2,000 x 540 217 / 131, 10,000 x
// 100 1,091 / 593; of few rows, 16 x 100,000 21 / 26, 48 x 100,000 52 / 82, 130 x
// 100,000 200 / 230, 200 x 20,000 117 / 118, 300 x 20,000 177 / 161, 500 x 20,000
// 376 / 302.  From 2^20 entries and 256 rows the split is the faster one at
// every shape tried; below, either may be, and the products keep the FP32
// instruction's bits.
bool splits(const BDenseView& b) { return b.dtype == F32 && b.m >= 256 && b.m * b.n >= (1 << 20); }
Arith arith(const BDenseView& b) { return b.dtype == F64 ? FP64 : splits(b) ? SPLIT : FP32; }
// cost, entry: picoseconds per product and, besides, per entry of a tile with
// every compute unit busy, fitted to whole gradients at 152 sizes from 1 x 1,000
// to 8,000 x 140 and 4,096 x 1,024 in every shape.  The rule below takes the
// best shape or one within 17% of it there, 1.2% on average.  (By the products
// alone it was 22% on average and a factor of nine where a short contraction
// meets many columns: 16 x 100,000, FP64 / FP32, 105 / 38 us in 16 x 16 tiles
// with eight waves to share 16 products, 24 / 21 in 16 x 256.)  kNever: a form
// that the rule takes at no size (gone through for m up to 270,000, n to 2e8).
constexpr ShapeInfo kShapes[] = {
    info<S0>(7.7, kNever, 3.8, 1600, 0, 1600),     info<S1>(7.6, kNever, 3.85, 2600, 0, 3000),
    info<S2>(8.3, 9.0, 5.1, 1900, 1900, 2500),     info<S3>(8.2, 8.8, 5.3, 2500, 2100, 3700),
    info<S4>(8.5, 8.5, 5.6, 3900, 3200, 6200),     info<S5>(14.4, 14.2, 8.6, 7800, 3500, 15500),
    info<S6>(19.8, 14.1, kNever, 15500, 4300, 0),  info<S7>(kNever, kNever, 4.15, 0, 0, 3650),
    info<S8>(14.8, 11.5, 7.5, 1400, 1300, 2200)};
constexpr int kNShapes = sizeof(kShapes) / sizeof(kShapes[0]);

int64_t tiles_of(const BDenseView& b, int sh) {
    const ShapeInfo& s = kShapes[sh];
    return ((b.m + s.tm - 1) / s.tm) * ((b.n + s.tn - 1) / s.tn);
}

}  // namespace

// The shape with the least time for its rounds of 256 tiles, one to a compute
// unit.  Measured gradients that the rule decides (FP64 / split, us): 3,000 x
// 500: 722 / 401 in 128 x 128 tiles (96 of them), 372 / 217 in 64 x 128 (188),
// - / 187 in 48 x 128 (252: one to nearly every compute unit), 320 / 238 in 64 x
// 32 (752); 4,096 x 1,024: 1,015 / 530 in 128 x 128, 1,116 / 750 in 64 x 64; 1,000 x
// 100, FP64 / FP32 instruction: 262 / 332 in 128 x 128, 24 / 28 in 32 x 16.
int bdense_shape(const BDenseView& b) {
    int best = 6;
    double tbest = 1e300;
    for (int i = 0; i < kNShapes; ++i) {
        const ShapeInfo& s = kShapes[i];
        if ((s.bx > 1 && b.m < 16 * s.bx) || (s.by > 1 && b.n < 16 * s.by)) continue;
        const double t = (double)((tiles_of(b, i) + 255) / 256) * s.tm * s.tn *
                         (2.0 * (double)b.m * s.cost[arith(b)] + s.entry[arith(b)]);
        if (t < tbest) {
            tbest = t;
            best = i;
        }
    }
    return best;
}

int64_t bdense_fwd_tiles(const BDenseView& b) { return tiles_of(b, b.shape); }

namespace {

template <typename T, int AR, bool TRANS, int EPI, typename S>
hipError_t launch_shape(const BDenseView& b, hipStream_t s, const T* A, const T* Bm, const T* W,
                        double* partials, T* V, const double* fbar, T* G, int accumulate, int64_t np,
                        double* f_out) {
    const int64_t tn = (b.n + S::TN - 1) / S::TN, nt = tn * ((b.m + S::TM - 1) / S::TM);
    if (nt > 0x7fffffffLL) return hipErrorInvalidValue;
    PG_LAUNCH((k_gemm_mfma<T, AR, TRANS, EPI, S>), dim3((unsigned)nt + (f_out ? 1 : 0)), dim3(S::NTHR), 0,
              s, A, Bm, b.m, b.n, b.m, W, partials, V, fbar, G, accumulate, (int)tn, np, f_out);
    return hipGetLastError();
}

template <typename T, int AR, bool TRANS, int EPI>
hipError_t launch_gemm(const BDenseView& b, hipStream_t s, const T* A, const T* Bm, const T* W,
                       double* partials, T* V, const double* fbar, T* G, int accumulate, int64_t np,
                       double* f_out) {
    switch (b.shape) {
        case 0:
            if constexpr (AR != FP32)
                return launch_shape<T, AR, TRANS, EPI, S0>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
            break;
        case 1:
            if constexpr (AR != FP32)
                return launch_shape<T, AR, TRANS, EPI, S1>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
            break;
        case 2: return launch_shape<T, AR, TRANS, EPI, S2>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
        case 3: return launch_shape<T, AR, TRANS, EPI, S3>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
        case 4: return launch_shape<T, AR, TRANS, EPI, S4>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
        case 5: return launch_shape<T, AR, TRANS, EPI, S5>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
        case 6:
            if constexpr (AR != SPLIT)
                return launch_shape<T, AR, TRANS, EPI, S6>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
            break;
        case 7:
            if constexpr (AR == SPLIT)
                return launch_shape<T, AR, TRANS, EPI, S7>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
            break;
        case 8: return launch_shape<T, AR, TRANS, EPI, S8>(b, s, A, Bm, W, partials, V, fbar, G, accumulate, np, f_out);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_bdense_fwd(const BDenseView& b, const void* X, double* partials, void* V,
                             hipStream_t s) {
    if (b.m == 0 || b.n == 0) return hipSuccess;
    if (b.dtype == F64)
        return launch_gemm<double, FP64, false, EPI_FWD>(b, s, (const double*)b.A, (const double*)X,
                                                   (const double*)b.W, partials, (double*)V, nullptr,
                                                   nullptr, 0, 0, nullptr);
    const float *A = (const float*)b.A, *Xp = (const float*)X, *W = (const float*)b.W;
    if (splits(b))
        return launch_gemm<float, SPLIT, false, EPI_FWD>(b, s, A, Xp, W, partials, (float*)V, nullptr,
                                                         nullptr, 0, 0, nullptr);
    return launch_gemm<float, FP32, false, EPI_FWD>(b, s, A, Xp, W, partials, (float*)V, nullptr,
                                                    nullptr, 0, 0, nullptr);
}

hipError_t launch_bdense_bwd(const BDenseView& b, const void* V, const double* fbar, void* G,
                             int accumulate, const double* partials, int64_t np, double* f_out,
                             hipStream_t s) {
    if (b.m == 0 || b.n == 0)
        return f_out ? launch_final_sum(partials, np, f_out, s) : hipSuccess;
    double* part = const_cast<double*>(partials);  // read only in the backward product
    if (b.dtype == F64)
        return launch_gemm<double, FP64, true, EPI_BWD>(b, s, (const double*)b.A, (const double*)V, nullptr,
                                                  part, nullptr, fbar, (double*)G, accumulate, np, f_out);
    const float *A = (const float*)b.A, *Vp = (const float*)V;
    if (splits(b))
        return launch_gemm<float, SPLIT, true, EPI_BWD>(b, s, A, Vp, nullptr, part, nullptr, fbar,
                                                        (float*)G, accumulate, np, f_out);
    return launch_gemm<float, FP32, true, EPI_BWD>(b, s, A, Vp, nullptr, part, nullptr, fbar,
                                                   (float*)G, accumulate, np, f_out);
}

}  // namespace pg
