// Dense row reduction with hierarchical (team / vector) parallelism:
//   f(x) = sum_i w_i psi((A x)_i),   grad = A^T (fbar w (.) psi'(A x)).
//
// Rows of at most kFusedElems elements per thread of the widest team run in
// one pass over A (k_dense_fused): a team -- one wave for short rows, a
// workgroup of 4 or 8 waves for longer ones -- takes U rows at a time, keeps
// its slice of x, of those rows and of the running column sums in registers,
// and reads A from HBM exactly once for f and the gradient together; the
// per-band column sums are then added in a fixed order (deterministic, no
// atomics).  Longer rows take two passes (k_dense_rows, k_dense_cols).
#include <type_traits>

#include "device_common.hpp"
#include "launch.hpp"

namespace pg {

namespace {

// Elements a thread of the widest team keeps of a row, of x and of the column
// sums: what the 256 registers a 512-thread workgroup has per thread hold.
template <typename T>
constexpr int kFusedElems = sizeof(T) == 8 ? 32 : 24;

constexpr int kRawBuffer = 0x00020000;  // flags word of a raw buffer resource (gfx9)

typedef int i4v __attribute__((ext_vector_type(4)));

// A slice of VN consecutive elements, read through a buffer resource that
// ends with the row: offsets past the end read zero, so the lanes beyond the
// row, and whole rows past the band, need no branch and touch no memory.
template <typename T, int VN>
struct Slice {
    T v[VN];
};

template <typename T, int VN>
__device__ __forceinline__ Slice<T, VN> buf_slice(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    constexpr int bytes = (int)sizeof(T) * VN;
    static_assert(bytes == 4 || bytes == 8 || bytes == 16, "one load per slice");
    if constexpr (bytes == 16)
        return __builtin_bit_cast(Slice<T, VN>, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
    else if constexpr (bytes == 8)
        return __builtin_bit_cast(Slice<T, VN>, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
    else
        return __builtin_bit_cast(Slice<T, VN>, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

// Row of the U (a power of two) that lane l holds after rows_reduce.
template <int U>
__device__ __forceinline__ constexpr int row_of_lane(int l) {
    int r = 0;
    for (int h = U / 2, b = 1; h >= 1; h >>= 1, b <<= 1)
        if (l & b) r += h;
    return r;
}

// Sums of U values over each group of L lanes (L = 64: the wave): while more
// than one value is left, a pair of lanes halves them (each keeps one half and
// receives the other lane's share of it), so U sums cost U - 1 + log2(L) -
// log2(U) exchanges instead of U log2(L).  Lane l returns the total of value
// row_of_lane<U>(l).  Fixed order.  (Recursive: as a loop over halves the
// array of values was still indexed at run time when the compiler placed it,
// and went to LDS.)
template <int U, int L, int MASK = 1>
__device__ __forceinline__ double rows_reduce(const double (&v)[U], int lane) {
    if constexpr (U > 1) {
        const bool up = (lane & MASK) != 0;
        double h[U / 2];
#pragma unroll
        for (int i = 0; i < U / 2; ++i) {
            const double keep = up ? v[i + U / 2] : v[i], give = up ? v[i] : v[i + U / 2];
            h[i] = keep + __shfl_xor(give, MASK, kWave);
        }
        return rows_reduce<U / 2, L, 2 * MASK>(h, lane);
    } else {
        double s = v[0];
#pragma unroll
        for (int m = MASK; m < L; m <<= 1) s += __shfl_xor(s, m, kWave);
        return s;
    }
}

__device__ __forceinline__ double lane_bcast(double v, int l) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// One pass over a band of rows.  NW: waves of a team (1: a workgroup holds
// four teams; more: the workgroup is the team).  A thread owns Q slices of VN
// elements of a row, U rows at a time.  colpart (GRAD) gets the band's column
// sums, partials its share of f.
//
// Bound by HBM reads of A.  One row per 512-thread workgroup at a time, each
// thread evaluating psi of it, left short rows waiting on two barriers and a
// logarithm per row.  So: U rows share one exchange, their psi' is evaluated
// once with a row per lane, psi is put off until 64 rows are there (a row per
// lane again), and rows of up to 512 elements need no barrier at all.
// Measured, FP64 gradient calls, before -> after: 50,003 x 301 3,466 -> 26.8 us
// (4.5 TB/s; the odd length took the two passes before), 20,000 x 1,000
// 134 -> 36.9 us, 5,000 x 5,001 530 -> 50.6 us, 10,000 x 10,000 157 -> 143 us
// (5.6 TB/s).
template <typename T, int VN, int Q, int U, int NW, bool GRAD>
__global__ void __launch_bounds__(NW == 1 ? 256 : 64 * NW)
k_dense_fused(DenseView d, const T* __restrict__ x, const double* __restrict__ fbar,
              double* __restrict__ partials, double* __restrict__ colpart, int nbands) {
    constexpr bool WG = NW > 1;
    constexpr int TEAMS = WG ? 1 : 4, TS = kWave * NW;
    // The next rows are loaded before these are reduced, while a second set
    // of row registers fits.
    constexpr bool PF = WG && VN * Q <= (VN == 4 ? 24 : 20);
    // x as FP64 while that fits the registers
    using XT = typename std::conditional<(VN * Q > 16), T, double>::type;
    __shared__ double red[WG ? 2 : 1][WG ? NW : 1][U];
    __shared__ double colred[WG || !GRAD ? 1 : TS * VN * Q];
    __shared__ double tred[TEAMS];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int t = WG ? (int)threadIdx.x : lane;
    const int team = WG ? 0 : wid;
    const T* __restrict__ A = static_cast<const T*>(d.A);
    const T* __restrict__ w = static_cast<const T*>(d.w);
    const int64_t cols = d.cols;
    const uint32_t row_bytes = (uint32_t)(cols * sizeof(T));
    const int g = blockIdx.x;
    const int64_t r0 = d.rows * g / nbands, r1 = d.rows * (g + 1) / nbands;
    const double fb = fbar ? fbar[0] : 1.0;

    XT xr[Q][VN];
    double acc[GRAD ? Q : 1][VN];
    uint32_t off[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t j = (int64_t)(t + TS * q) * VN;
        off[q] = (uint32_t)(j * sizeof(T));
#pragma unroll
        for (int c = 0; c < VN; ++c) xr[q][c] = j + c < cols ? (XT)x[j + c] : XT(0);
        if constexpr (GRAD)
#pragma unroll
            for (int c = 0; c < VN; ++c) acc[q][c] = 0.0;
    }
    using S = Slice<T, VN>;
    auto load_rows = [&](int64_t base, S (&dst)[U][Q]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = base + u < r1;
            const T* row = A + (in ? base + u : r0) * cols;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                (void*)row, (short)0, in ? (int)row_bytes : 0, kRawBuffer);
#pragma unroll
            for (int q = 0; q < Q; ++q) dst[u][q] = buf_slice<T, VN>(r, off[q]);
        }
    };
    const int myrow = row_of_lane<U>(lane & (U - 1));
    double tsum = 0.0, rk = 0.0, wk = 0.0;
    int slot = 0, phase = 0;
    auto step = [&](int64_t base, const S (&a)[U][Q], double wi) {
        double dot[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            dot[u] = 0.0;
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int c = 0; c < VN; ++c) dot[u] += to_f64(a[u][q].v[c]) * (double)xr[q][c];
        }
        double r = rows_reduce<U, kWave>(dot, lane);
        if constexpr (WG) {
            // Two buffers: a wave that runs ahead writes the other one, and
            // cannot reach this one again before every wave passed the next barrier.
            if (lane < U) red[phase][wid][lane] = r;
            __syncthreads();
            r = 0.0;
#pragma unroll
            for (int i = 0; i < NW; ++i) r += red[phase][i][lane & (U - 1)];
            phase ^= 1;
        }
        const bool have = base + myrow < r1;
        if (!WG || wid == 0) {
            if (lane / U == slot) {
                rk = have ? r : 0.0;
                wk = wi;
            }
            if (++slot == kWave / U) {
                tsum += wk * psi_from_sq(rk * rk);
                slot = 0;
                rk = wk = 0.0;
            }
        }
        if constexpr (GRAD) {
            const double v = fb * wi * dpsi_from(r, r * r);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (base + u >= r1) break;  // the same for the whole workgroup or wave
                const double vu = lane_bcast(v, row_of_lane<U>(u));
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int c = 0; c < VN; ++c) acc[q][c] += vu * to_f64(a[u][q].v[c]);
            }
        }
    };
    auto load_w = [&](int64_t base) { return base + myrow < r1 ? to_f64(w[base + myrow]) : 0.0; };

    constexpr int64_t kStride = (int64_t)TEAMS * U;
    int64_t base = r0 + (int64_t)team * U;
    if constexpr (PF) {
        S cur[U][Q], nxt[U][Q];
        double wc = 0.0, wn = 0.0;
        if (base < r1) {
            load_rows(base, cur);
            wc = load_w(base);
        }
        for (; base < r1; base += kStride) {
            if (base + kStride < r1) {
                load_rows(base + kStride, nxt);
                wn = load_w(base + kStride);
            }
            step(base, cur, wc);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < Q; ++q) cur[u][q] = nxt[u][q];
            wc = wn;
        }
    } else {
        for (; base < r1; base += kStride) {
            S cur[U][Q];
            load_rows(base, cur);
            step(base, cur, load_w(base));
        }
    }
    if (!WG || wid == 0) {
        tsum += wk * psi_from_sq(rk * rk);  // the rows of the last, partly filled 64
        tsum = wave_sum(tsum);
        if (lane == 0) tred[team] = tsum;
    }
    if constexpr (GRAD && !WG) {
#pragma unroll
        for (int k = 0; k < TEAMS; ++k) {
            if (wid == k) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int c = 0; c < VN; ++c) {
                        double& s = colred[(t + TS * q) * VN + c];
                        s = k == 0 ? acc[q][c] : s + acc[q][c];
                    }
            }
            __syncthreads();
        }
        double* out = colpart + (int64_t)g * cols;
        for (int j = threadIdx.x; j < (int)cols; j += 256) out[j] = colred[j];
    }
    if constexpr (GRAD && WG) {
        double* out = colpart + (int64_t)g * cols;
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int c = 0; c < VN; ++c) {
                const int64_t j = (int64_t)(t + TS * q) * VN + c;
                if (j < cols) out[j] = acc[q][c];
            }
    }
    if constexpr (!WG) __syncthreads();
    if (threadIdx.x == 0) {
        double s = tred[0];
#pragma unroll
        for (int k = 1; k < TEAMS; ++k) s += tred[k];
        partials[g] = s;
    }
}

// The same for rows of at most LPR slices: LPR lanes to a row, 64 / LPR rows
// side by side in a wave and U such sets at a time, so that short rows leave
// no lanes idle and every lane evaluates psi of a row of its own.  100,000 x 16
// gradient: 437 us with a workgroup to a row, 24.4 with a wave to a row, 8.9
// so (1.5 TB/s, two launches); FP32 453, 40.4, 9.7.
template <typename T, int VN, int LPR, bool GRAD>
__global__ void __launch_bounds__(256)
k_dense_narrow(DenseView d, const T* __restrict__ x, const double* __restrict__ fbar,
               double* __restrict__ partials, double* __restrict__ colpart, int nbands) {
    constexpr int G = kWave / LPR, U = 8, ROWS = G * U;  // rows of a wave at a time
    static_assert(U <= LPR, "a lane holds one row's sum");
    __shared__ double colred[GRAD ? 4 * LPR * VN : 1];
    __shared__ double tred[4];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int t = lane % LPR, grp = lane / LPR;
    const T* __restrict__ A = static_cast<const T*>(d.A);
    const T* __restrict__ w = static_cast<const T*>(d.w);
    const int cols = (int)d.cols;
    const uint32_t row_bytes = (uint32_t)(cols * sizeof(T));
    const int g = blockIdx.x;
    const int64_t r0 = d.rows * g / nbands, r1 = d.rows * (g + 1) / nbands;
    const double fb = fbar ? fbar[0] : 1.0;
    double xr[VN], acc[VN];
    const bool mine = t * VN < cols;
#pragma unroll
    for (int c = 0; c < VN; ++c) {
        xr[c] = mine ? to_f64(x[t * VN + c]) : 0.0;
        acc[c] = 0.0;
    }
    // Byte offset of this lane's slice in the first set of rows; lanes past
    // the row get one past any set (which reads zero).
    const uint32_t off = mine ? grp * row_bytes + (uint32_t)(t * VN * sizeof(T)) : 0x7ff00000u;
    const int myset = row_of_lane<U>(t & (U - 1));
    const bool holds = t < U;  // one lane per row
    double tsum = 0.0;
    for (int64_t base = r0 + (int64_t)wid * ROWS; base < r1; base += 4 * ROWS) {
        const int left = (int)(r1 - base < ROWS ? r1 - base : ROWS);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(A + base * cols), (short)0, (int)(left * row_bytes), kRawBuffer);
        Slice<T, VN> a[U];
        double dot[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = buf_slice<T, VN>(r, off + u * G * row_bytes);
        const int row = myset * G + grp;
        const double wi = row < left ? to_f64(w[base + row]) : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            dot[u] = 0.0;
#pragma unroll
            for (int c = 0; c < VN; ++c) dot[u] += to_f64(a[u].v[c]) * xr[c];
        }
        const double s = rows_reduce<U, LPR>(dot, lane), s2 = s * s;
        if (holds && row < left) tsum += wi * psi_from_sq(s2);
        if constexpr (GRAD) {
            // selects, not products with zero, keep the rows past the band out
            const double v = row < left ? fb * wi * dpsi_from(s, s2) : 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double vu = __shfl(v, grp * LPR + row_of_lane<U>(u), kWave);
#pragma unroll
                for (int c = 0; c < VN; ++c) acc[c] += vu * to_f64(a[u].v[c]);
            }
        }
    }
    tsum = wave_sum(tsum);
    if (lane == 0) tred[wid] = tsum;
    if constexpr (GRAD) {
#pragma unroll
        for (int c = 0; c < VN; ++c) {
            double s = acc[c];
#pragma unroll
            for (int m = LPR; m < kWave; m <<= 1) s += __shfl_xor(s, m, kWave);
            if (grp == 0) colred[(wid * LPR + t) * VN + c] = s;
        }
    }
    __syncthreads();
    if constexpr (GRAD) {
        constexpr int W = LPR * VN;
        for (int j = threadIdx.x; j < cols; j += 256)
            colpart[(int64_t)g * cols + j] =
                ((colred[j] + colred[W + j]) + colred[2 * W + j]) + colred[3 * W + j];
    }
    if (threadIdx.x == 0) partials[g] = ((tred[0] + tred[1]) + tred[2]) + tred[3];
}

// grad[j] (=|+=) sum of colpart[g, j] over the bands: kColSlices slices of
// consecutive bands, each summed in ascending order by one thread, then the
// slices added in ascending order (deterministic).  W columns per
// workgroup: few, so that short rows still spread over the device.  The
// first workgroup also sums the bands' shares of f (fixed order), which
// saves a gradient the launch of its own that a separate sum takes.
constexpr int kColBS = 512;

template <typename T, int kColW>
__global__ void __launch_bounds__(kColBS)
k_dense_colsum(const double* __restrict__ colpart, int nbands, int64_t cols, T* __restrict__ grad,
               int accumulate, const double* __restrict__ partials, int64_t np,
               double* __restrict__ f_out) {
    constexpr int kColSlices = kColBS / kColW;
    __shared__ double part[kColSlices][kColW];
    __shared__ double lds[kColBS / kWave];
    const int cx = threadIdx.x % kColW, y = threadIdx.x / kColW;
    const int64_t j = (int64_t)blockIdx.x * kColW + cx;
    double s = 0.0;
    if (j < cols) {
        const int g0 = nbands * y / kColSlices, g1 = nbands * (y + 1) / kColSlices;
        int g = g0;
        for (; g + 4 <= g1; g += 4) {  // four loads in flight, added in order
            double v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = colpart[(int64_t)(g + q) * cols + j];
#pragma unroll
            for (int q = 0; q < 4; ++q) s += v[q];
        }
        for (; g < g1; ++g) s += colpart[(int64_t)g * cols + j];
    }
    part[y][cx] = s;
    __syncthreads();
    if (y == 0 && j < cols) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kColSlices; ++q) t += part[q][cx];
        grad[j] = accumulate ? static_cast<T>(to_f64(grad[j]) + t) : static_cast<T>(t);
    }
    if (f_out && blockIdx.x == 0) {
        double v = 0.0;
        for (int64_t q = threadIdx.x; q < np; q += kColBS) v += partials[q];
        v = block_sum<kColBS>(v, lds);
        if (threadIdx.x == 0) f_out[0] = v;
    }
}

// Pass over rows of any length: a workgroup takes U rows at a time (they
// share the loads of x), rows dealt round-robin; f's share per workgroup
// and, when v != nullptr, v_i = fbar w_i psi'(r_i).  XA: x is aligned to the
// slices that the rows are read in, else it is read by element.
template <typename T, int VN, int U, int BS, bool XA>
__global__ void __launch_bounds__(BS)
k_dense_rows(DenseView d, const T* __restrict__ x, const double* __restrict__ fbar,
             double* __restrict__ partials, double* __restrict__ v) {
    constexpr int NW = BS / kWave;
    constexpr int D = 4;  // slices of each row in flight per thread
    struct alignas(sizeof(T) * VN) SV {
        T v[VN];
    };
    __shared__ double red[2][NW][U];
    const T* __restrict__ A = static_cast<const T*>(d.A);
    const T* __restrict__ w = static_cast<const T*>(d.w);
    const int64_t cols = d.cols, nvec = cols / VN;  // VN divides cols
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const double fb = fbar ? fbar[0] : 1.0;
    auto load_x = [&](int64_t j) {
        if constexpr (XA) return reinterpret_cast<const SV*>(x)[j];
        SV r;
#pragma unroll
        for (int c = 0; c < VN; ++c) r.v[c] = x[j * VN + c];
        return r;
    };
    double tsum = 0.0;
    int phase = 0;
    for (int64_t i0 = (int64_t)blockIdx.x * U; i0 < d.rows; i0 += (int64_t)gridDim.x * U) {
        const SV* row[U];
        double dot[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u < d.rows ? i0 + u : d.rows - 1;  // a repeat is not used
            row[u] = reinterpret_cast<const SV*>(A + i * cols);
            dot[u] = 0.0;
        }
        int64_t j = threadIdx.x;
        for (; j + (D - 1) * BS < nvec; j += D * BS) {
            SV xs[D], a[U][D];
#pragma unroll
            for (int q = 0; q < D; ++q) xs[q] = load_x(j + q * BS);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < D; ++q) a[u][q] = row[u][j + q * BS];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < D; ++q)
#pragma unroll
                    for (int c = 0; c < VN; ++c)
                        dot[u] += to_f64(a[u][q].v[c]) * to_f64(xs[q].v[c]);
        }
        for (; j < nvec; j += BS) {
            const SV xs = load_x(j);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const SV a = row[u][j];
#pragma unroll
                for (int c = 0; c < VN; ++c) dot[u] += to_f64(a.v[c]) * to_f64(xs.v[c]);
            }
        }
        const double r1 = rows_reduce<U, kWave>(dot, lane);
        if (lane < U) red[phase][wid][lane] = r1;
        __syncthreads();
        if ((int)threadIdx.x < U) {
            double r = 0.0;
#pragma unroll
            for (int k = 0; k < NW; ++k) r += red[phase][k][threadIdx.x];
            const int64_t i = i0 + row_of_lane<U>((int)threadIdx.x);
            if (i < d.rows) {
                const double s2 = r * r, wi = to_f64(w[i]);
                tsum += wi * psi_from_sq(s2);
                if (v) v[i] = fb * wi * dpsi_from(r, s2);
            }
        }
        phase ^= 1;  // the next rows use the other buffer: one barrier per step
    }
    if (wid == 0) {
        tsum = wave_sum(tsum);
        if (lane == 0) partials[blockIdx.x] = tsum;
    }
}

// Column sums of v_i A_i over a band of rows, 256 slices of columns per
// workgroup; bands enough to fill the device (four row slices of one
// workgroup each, 64 columns wide, left most of it idle: 2,000 x 20,001
// gradient 283 -> 113 us).  The bands are taken last first: the row pass ended
// there, so that part of A is the part still in the last-level cache.
template <typename T, int VN>
__global__ void __launch_bounds__(256)
k_dense_cols(DenseView d, const double* __restrict__ v, double* __restrict__ colpart) {
    constexpr int D = 8;
    struct alignas(sizeof(T) * VN) SV {
        T v[VN];
    };
    const int64_t nvec = d.cols / VN;
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int nb = gridDim.y, g = nb - 1 - (int)blockIdx.y;
    if (j >= nvec) return;
    const int64_t r0 = d.rows * g / nb, r1 = d.rows * (g + 1) / nb;
    const SV* __restrict__ A = reinterpret_cast<const SV*>(d.A) + j;
    double acc[VN];
#pragma unroll
    for (int c = 0; c < VN; ++c) acc[c] = 0.0;
    int64_t i = r0;
    for (; i + D <= r1; i += D) {
        SV a[D];
#pragma unroll
        for (int q = 0; q < D; ++q) a[q] = A[(i + q) * nvec];
#pragma unroll
        for (int q = 0; q < D; ++q) {
            const double vi = v[i + q];
#pragma unroll
            for (int c = 0; c < VN; ++c) acc[c] += vi * to_f64(a[q].v[c]);
        }
    }
    for (; i < r1; ++i) {
        const SV a = A[i * nvec];
        const double vi = v[i];
#pragma unroll
        for (int c = 0; c < VN; ++c) acc[c] += vi * to_f64(a.v[c]);
    }
    double* out = colpart + (int64_t)g * d.cols + j * VN;
#pragma unroll
    for (int c = 0; c < VN; ++c) out[c] = acc[c];
}

// Rows a team takes at a time, by the elements a thread holds of each.  More
// share an exchange and a barrier, fewer leave registers for the next rows.
// Gradients, us, with half of these / these / twice: FP64 50,000 x 301 26.1 / 26.8 /
// 26.9, 20,000 x 1,000 32.4 / 32.8 / 40.8, 10,000 x 4,000 64.0 / 58.5 / 143, 5,000 x
// 12,000 105 / 104 / 109, 3,000 x 16,000 91 / 91 / 171; FP32 50,000 x 301 20.0 / 23.1 /
// 22.6, 20,000 x 1,000 22.8 / 26.7 / 32.3, 10,000 x 4,000 40.9 / 38.5 / 50.9, 5,000 x
// 12,000 56 / 56 / 95.
constexpr int rows_at_once(int nw, int elems) {
    return nw == 1 ? (elems <= 2 ? 16 : elems <= 4 ? 8 : 4)
                   : (elems <= 4 ? 8 : elems <= 8 ? 4 : elems <= 12 ? 2 : 1);
}

template <typename T, int VN, int NW, int Q>
hipError_t launch_fused_q(const DenseView& d, const T* x, const double* fbar, int want_grad,
                          double* partials, double* colpart, int nbands, hipStream_t s) {
    constexpr int U = rows_at_once(NW, VN * Q), BS = NW == 1 ? 256 : 64 * NW;
    if (want_grad) {
        PG_LAUNCH((k_dense_fused<T, VN, Q, U, NW, true>), dim3(nbands), dim3(BS), 0, s, d, x, fbar,
                  partials, colpart, nbands);
        return hipGetLastError();
    }
    if constexpr (NW == 1) {
        PG_LAUNCH((k_dense_fused<T, VN, Q, U, NW, false>), dim3(nbands), dim3(BS), 0, s, d, x, fbar,
                  partials, nullptr, nbands);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;  // longer rows take k_dense_rows for f alone
}

template <typename T, int VN>
hipError_t launch_fused_vn(const DenseView& d, int nw, const T* x, const double* fbar, int want_grad,
                           double* partials, double* colpart, int nbands, hipStream_t s) {
    const int64_t per = (int64_t)kWave * nw * VN;
    const int64_t q = (d.cols + per - 1) / per;
#define PG_Q(NWV, QV)                                                                          \
    if constexpr (VN * (QV) <= kFusedElems<T>) {                                               \
        if (nw == NWV && q <= QV)                                                              \
            return launch_fused_q<T, VN, NWV, QV>(d, x, fbar, want_grad, partials, colpart,    \
                                                  nbands, s);                                  \
    }
    if constexpr (VN == 1) {
        PG_Q(1, 1) PG_Q(1, 2) PG_Q(1, 3) PG_Q(1, 4) PG_Q(1, 5) PG_Q(1, 6) PG_Q(1, 8)
        PG_Q(4, 3) PG_Q(4, 4) PG_Q(4, 6) PG_Q(4, 8)
        PG_Q(8, 5) PG_Q(8, 6) PG_Q(8, 8) PG_Q(8, 10) PG_Q(8, 12) PG_Q(8, 16) PG_Q(8, 20)
        PG_Q(8, 24) PG_Q(8, 32)
    } else {
        // With two elements to a slice, a row too long for fewer waves takes
        // two slices of four waves at least, three of eight.
        PG_Q(1, 1) PG_Q(1, 2)
        if constexpr (VN == 2) { PG_Q(1, 3) PG_Q(1, 4) }
        if constexpr (VN == 4) { PG_Q(4, 1) }
        PG_Q(4, 2)
        if constexpr (VN == 2) { PG_Q(4, 3) PG_Q(4, 4) }
        if constexpr (VN == 4) { PG_Q(8, 2) }
        PG_Q(8, 3) PG_Q(8, 4) PG_Q(8, 5) PG_Q(8, 6) PG_Q(8, 8) PG_Q(8, 10) PG_Q(8, 12)
        PG_Q(8, 16)
    }
#undef PG_Q
    return hipErrorInvalidValue;
}

template <typename T, int VN>
hipError_t launch_narrow_vn(const DenseView& d, int lpr, const T* x, const double* fbar,
                            int want_grad, double* partials, double* colpart, int nbands,
                            hipStream_t s) {
#define PG_LPR(L)                                                                              \
    if (lpr == L) {                                                                            \
        if (want_grad)                                                                         \
            PG_LAUNCH((k_dense_narrow<T, VN, L, true>), dim3(nbands), dim3(256), 0, s, d, x,   \
                      fbar, partials, colpart, nbands);                                        \
        else                                                                                   \
            PG_LAUNCH((k_dense_narrow<T, VN, L, false>), dim3(nbands), dim3(256), 0, s, d, x,  \
                      fbar, partials, nullptr, nbands);                                        \
        return hipGetLastError();                                                              \
    }
    PG_LPR(8) PG_LPR(16) PG_LPR(32)
#undef PG_LPR
    return hipErrorInvalidValue;
}

// Elements per load: whole 16-byte slices when the rows keep their alignment.
int slice_elems(const DenseView& d) {
    const int vn = d.dtype == F64 ? 2 : 4;
    return d.cols % vn == 0 ? vn : 1;
}

template <typename T>
hipError_t launch_fused_t(const DenseView& d, const DenseCfg& c, const void* x, const double* fbar,
                          int want_grad, double* partials, double* colpart, hipStream_t s) {
    constexpr int VN = 16 / sizeof(T);
    const T* xp = static_cast<const T*>(x);
    const bool vec = slice_elems(d) > 1;
    if (c.lanes < kWave)
        return vec ? launch_narrow_vn<T, VN>(d, c.lanes, xp, fbar, want_grad, partials, colpart, c.bands, s)
                   : launch_narrow_vn<T, 1>(d, c.lanes, xp, fbar, want_grad, partials, colpart, c.bands, s);
    return vec ? launch_fused_vn<T, VN>(d, c.nw, xp, fbar, want_grad, partials, colpart, c.bands, s)
               : launch_fused_vn<T, 1>(d, c.nw, xp, fbar, want_grad, partials, colpart, c.bands, s);
}

// Rows a workgroup of the row pass takes at a time, and its threads.  Many rows:
// four at a time, which share the loads of x.  Fewer than 1,024: one, so that
// more of the device reads; a wide workgroup each for very few very long ones
// (more than 48 slices for each of 256 threads).
// Objectives, us, FP64 / FP32, (4 rows, 256 threads) / (1, 256) / (1, 1,024): 100 x
// 60,000 28.6 / 18.9 / 15.4, 20.6 / 9.9 / 9.3; 300 x 60,000 31.0 / 28.8 / 32.2,
// 27.7 / 17.4 / 19.6; 100 x 20,001 (by element) FP32 10.0 / 8.9 / 7.8; 300 x 16,000 12.6 / 11.0 / 12.6; 1,000 x 514 7.9 / 7.9 / 10.4
// (the call's own 7.7); 1,000 x 16,000 22.5 / 23.0 / 26.4; 2,500 x 2,048 9.8 / 11.5 /
// 19.6; 5,000 x 16,000 109 / 122 / 134; 20,000 x 514 19.4 / 30.5 / 86.6.
struct RowPass {
    int u, bs;
};
RowPass row_pass(const DenseView& d) {
    if (d.rows >= 1024) return {4, 256};
    return {1, d.rows <= 128 && d.cols / slice_elems(d) > 12288 ? 1024 : 256};
}

template <typename T, int VN, bool XA>
hipError_t launch_rows_vn(const DenseView& d, const T* x, const double* fbar, double* partials,
                          double* v, int groups, hipStream_t s) {
    const RowPass r = row_pass(d);
    const dim3 grid(groups), block(r.bs);
    if (r.u == 4)
        PG_LAUNCH((k_dense_rows<T, VN, 4, 256, XA>), grid, block, 0, s, d, x, fbar, partials, v);
    else if (r.bs == 256)
        PG_LAUNCH((k_dense_rows<T, VN, 1, 256, XA>), grid, block, 0, s, d, x, fbar, partials, v);
    else
        PG_LAUNCH((k_dense_rows<T, VN, 1, 1024, XA>), grid, block, 0, s, d, x, fbar, partials, v);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_rows_t(const DenseView& d, const void* x, const double* fbar, double* partials,
                         double* v, int groups, hipStream_t s) {
    constexpr int VN = 16 / sizeof(T);
    const T* xp = static_cast<const T*>(x);
    if (slice_elems(d) != VN) return launch_rows_vn<T, 1, true>(d, xp, fbar, partials, v, groups, s);
    if ((uintptr_t)x % 16 == 0) return launch_rows_vn<T, VN, true>(d, xp, fbar, partials, v, groups, s);
    // x off the 16-byte grid; A by slice / by element, us: FP64 1,025 x 16,000 25.5 /
    // 30.3, 2,500 x 30,000 109 / 116; FP32 500 x 16,000 9.5 / 11.6, but 5,000 x
    // 16,000 57 / 53, 1,025 x 12,000 13.9 / 12.8.
    if (sizeof(T) == 8 || row_pass(d).u == 1)
        return launch_rows_vn<T, VN, false>(d, xp, fbar, partials, v, groups, s);
    return launch_rows_vn<T, 1, true>(d, xp, fbar, partials, v, groups, s);
}

template <typename T>
hipError_t launch_colsum_t(const double* colpart, int nbands, int64_t cols, T* grad, int accumulate,
                           const double* partials, int64_t np, double* f_out, hipStream_t s) {
    // Columns to a workgroup, 8 / 32, whole FP64 gradients, us: 50,000 x 301 26.6 /
    // 29.7, 20,000 x 1,000 32.5 / 34.6, 10,000 x 2,000 36.0 / 35.2, 5,000 x 4,000 32.3 /
    // 31.8, 5,000 x 6,000 45.6 / 44.3, 2,000 x 16,000 64.8 / 58.5.
    const int w = cols < 4096 ? 8 : 32;
    const dim3 grid((unsigned)((cols + w - 1) / w));
    if (w == 8)
        hipLaunchKernelGGL((k_dense_colsum<T, 8>), grid, dim3(kColBS), 0, s, colpart, nbands, cols,
                           grad, accumulate, partials, np, f_out);
    else
        hipLaunchKernelGGL((k_dense_colsum<T, 32>), grid, dim3(kColBS), 0, s, colpart, nbands, cols,
                           grad, accumulate, partials, np, f_out);
    return hipGetLastError();
}

}  // namespace

// How a dense objective of this shape runs.  A team is as narrow as its
// registers allow (8 elements per thread below 8 waves): narrower teams
// exchange less per row, and the waves of a compute unit then wait for
// different rows.  One pass up to where its registers spill badly: FP64 2,000
// rows take 70 us at 16,384 columns (one pass, 26 spilled) and 92 us at 16,386
// (two); FP32 at 16,386 took 229 us in one pass (276 spilled) and takes 48 us
// in two, so FP32 stops at 12,288.
DenseCfg dense_config(const DenseView& d) {
    DenseCfg c;
    const int64_t lim = d.dtype == F64 ? kFusedElems<double> : kFusedElems<float>;
    const int vn = slice_elems(d);
    c.nw = d.cols <= 8 * kWave ? 1 : d.cols <= 8 * 4 * kWave ? 4 : 8;
    c.fused = d.cols <= lim * 8 * kWave;
    // Lanes to a row when half a wave or less holds it.
    const int64_t slices = (d.cols + vn - 1) / vn;
    c.lanes = slices <= 8 ? 8 : slices <= 16 ? 16 : slices <= 32 ? 32 : kWave;
    const int64_t elems = (d.cols + (int64_t)kWave * c.nw - 1) / ((int64_t)kWave * c.nw);
    const int64_t step = c.lanes < kWave ? 4 * 8 * (kWave / c.lanes)
                                         : (c.nw == 1 ? 4 : 1) *
                                               rows_at_once(c.nw, (int)((elems + vn - 1) / vn * vn));
    // Resident workgroups fill the device (the registers of 8-wave teams
    // allow one per compute unit); fewer when the rows run out.
    const int64_t most = c.nw == 1 ? 1024 : c.nw == 4 ? 768 : 256;
    if (c.fused)
        c.bands = (int)std::max<int64_t>(1, std::min<int64_t>(most, (d.rows + step - 1) / step));
    else {
        const int64_t chunks = std::max<int64_t>(1, (d.cols / vn + 255) / 256);
        c.bands = (int)std::max<int64_t>(1, std::min<int64_t>(2048 / chunks, d.rows / 8));
    }
    const int64_t u = row_pass(d).u;
    c.row_groups = (int)std::max<int64_t>(1, std::min<int64_t>(2048, (d.rows + u - 1) / u));
    return c;
}

hipError_t launch_dense_fused(const DenseView& d, const DenseCfg& c, const void* x,
                              const double* fbar, int want_grad, double* partials,
                              double* colpart, hipStream_t s) {
    if (!c.fused) return hipErrorInvalidValue;
    if (d.rows == 0) return hipSuccess;
    return d.dtype == F64
               ? launch_fused_t<double>(d, c, x, fbar, want_grad, partials, colpart, s)
               : launch_fused_t<float>(d, c, x, fbar, want_grad, partials, colpart, s);
}

hipError_t launch_dense_colsum(const double* colpart, int nbands, int64_t cols, void* grad,
                               Dtype dt, int accumulate, const double* partials, int64_t np,
                               double* f_out, hipStream_t s) {
    if (cols == 0) return hipSuccess;
    return dt == F64 ? launch_colsum_t(colpart, nbands, cols, static_cast<double*>(grad), accumulate,
                                       partials, np, f_out, s)
                     : launch_colsum_t(colpart, nbands, cols, static_cast<float*>(grad), accumulate,
                                       partials, np, f_out, s);
}

hipError_t launch_dense_rows(const DenseView& d, const DenseCfg& c, const void* x,
                             const double* fbar, double* partials, double* v, hipStream_t s) {
    if (d.rows == 0) return hipSuccess;
    return d.dtype == F64 ? launch_rows_t<double>(d, x, fbar, partials, v, c.row_groups, s)
                          : launch_rows_t<float>(d, x, fbar, partials, v, c.row_groups, s);
}

hipError_t launch_dense_cols(const DenseView& d, const DenseCfg& c, const double* v,
                             double* colpart, hipStream_t s) {
    if (d.cols == 0) return hipSuccess;
    const int vn = slice_elems(d);
    const dim3 grid((unsigned)((d.cols / vn + 255) / 256), (unsigned)c.bands), block(256);
    if (d.dtype == F64) {
        if (vn == 2)
            hipLaunchKernelGGL((k_dense_cols<double, 2>), grid, block, 0, s, d, v, colpart);
        else
            hipLaunchKernelGGL((k_dense_cols<double, 1>), grid, block, 0, s, d, v, colpart);
    } else {
        if (vn == 4)
            hipLaunchKernelGGL((k_dense_cols<float, 4>), grid, block, 0, s, d, v, colpart);
        else
            hipLaunchKernelGGL((k_dense_cols<float, 1>), grid, block, 0, s, d, v, colpart);
    }
    return hipGetLastError();
}

}  // namespace pg
