// Kernels of composed programs.  Non-pointwise constructs (stencil, gather,
// scan) run one kernel each way; chains of pointwise constructs run as fused
// groups (k_group), which recompute their forward values in registers in the
// reverse pass instead of reading them from a tape.  Shadows are FP64; a
// shadow's first contribution in the reverse pass stores, later ones add
// (the generated code of section 4 zeroes every shadow and adds).
#include <algorithm>

#include "device_common.hpp"
#include "elem_tile.hpp"
#include "launch.hpp"

namespace pg {

namespace {

constexpr int kBS = kGroupBlock;

inline unsigned nblocks(int64_t n) { return (unsigned)((n + kBS - 1) / kBS); }

__device__ __forceinline__ double map_f(int fn, double s) {
    return fn == 0 ? s * s : psi_from_sq(s * s);
}
__device__ __forceinline__ double map_df(int fn, double s) {
    return fn == 0 ? 2.0 * s : dpsi_from(s, s * s);
}

__global__ void __launch_bounds__(kBS)
k_stencil(int64_t n, const double* __restrict__ a, ProgTaps taps, double* __restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
    for (int t = 0; t < taps.n; ++t) {
        const int64_t j = i + taps.off[t];
        if (j >= 0 && j < n) s += taps.coef[t] * a[j];
    }
    y[i] = s;
}

// ---------------------------------------------------------- reverse pass

// The reverse of a stencil reads ybar through several index expressions; it
// is rescheduled by the written index: abar_j += sum_t c_t ybar_{j - o_t}.
__global__ void __launch_bounds__(kBS)
k_r_stencil(int64_t n, const double* __restrict__ yb, ProgTaps taps, double* __restrict__ ab,
            int accumulate) {
    const int64_t j = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (j >= n) return;
    double s = 0.0;
    for (int t = 0; t < taps.n; ++t) {
        const int64_t i = j - taps.off[t];
        if (i >= 0 && i < n) s += taps.coef[t] * yb[i];
    }
    if (accumulate)
        ab[j] += s;
    else
        ab[j] = s;
}

// The reverse of a gather whose products lie in the order of its transposed
// connectivity, in C parts: entry n adds its run of each part, in ascending
// incidence order over all of them, and stores the sum (or adds it to what is
// there).  Streams the products, the first D of every run read ahead; a stale
// plan only clears here what k_gather_scatter then adds to.
//
// With C = kXcds the part is the XCD whose workgroups store the products
// (xcd_remap): in one list each 128-byte line collected its 16 products
// through several L2s, which write the line back in pieces.  Random rows of
// eight, 200,003 of them on 300,007 entries (1.6 M incidences), the group and
// this pass: 121 us with one atomic per incidence (13 G/s), 42.9 in one list,
// 35.6 in parts.  (Reading B and the adjoint through the incidence list
// instead of storing products: 7 us more than one list.)
template <int C>
__global__ void __launch_bounds__(kBS) k_gather_rev(GatherRev r) {
    constexpr int D = C == 1 ? 8 : 4;
    const int64_t n = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * kBS + threadIdx.x;
    if (n >= r.n_nodes) return;
    if (*r.stale) {
        if (!r.accumulate) r.out[n] = 0.0;
        return;
    }
    int32_t p0[C], p1[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        p0[c] = r.offs[c * r.n_nodes + n];
        p1[c] = r.offs[c * r.n_nodes + n + 1];
    }
    double v[C][D];
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
        for (int q = 0; q < D; ++q) v[c][q] = p0[c] + q < p1[c] ? r.prod[p0[c] + q] : 0.0;
    }
    const double was = r.accumulate ? r.out[n] : 0.0;
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
        for (int q = 0; q < D; ++q)
            if (p0[c] + q < p1[c]) s += v[c][q];
        for (int32_t p = p0[c] + D; p < p1[c]; p += D) {
            double w[D];
#pragma unroll
            for (int q = 0; q < D; ++q) w[q] = p + q < p1[c] ? r.prod[p + q] : 0.0;
#pragma unroll
            for (int q = 0; q < D; ++q)
                if (p + q < p1[c]) s += w[q];
        }
    }
    r.out[n] = r.accumulate ? was + s : s;
}

// Of each incidence of n_elems rows of k: its entry, and in which part of the
// products the workgroup that handles its row stores (key = part * n_nodes +
// entry).
__global__ void __launch_bounds__(kBS)
k_part_keys(const int32_t* __restrict__ conn, int64_t n_elems, int32_t k, int64_t n_nodes,
            int32_t* __restrict__ keys) {
    const int64_t blocks = (n_elems + kBS - 1) / kBS, q = blocks / kXcds, r = blocks % kXcds;
    for (int64_t i = (int64_t)blockIdx.x * kBS + threadIdx.x; i < n_elems * k;
         i += (int64_t)gridDim.x * kBS) {
        const int64_t b = i / k / kBS;  // parts 0 .. r - 1 have q + 1 workgroups, the rest q
        const int64_t part = b < r * (q + 1) ? b / (q + 1) : r + (b - r * (q + 1)) / q;
        keys[i] = (int32_t)(part * n_nodes + conn[i]);
    }
}

// The same by element with atomics, for a connectivity changed since the
// transposed one was built (nothing to do otherwise), which it tells the host.  With f_out, the first
// workgroup sums the partials of f instead, which saves that its launch.
__global__ void __launch_bounds__(kBS) k_gather_scatter(GatherRev r) {
    __shared__ double lds[16];
    const unsigned first = r.f_out ? 1 : 0;
    if (blockIdx.x < first) {
        const double f = final_sum_block<false>(r.partials, r.n_partials, lds);
        if (threadIdx.x == 0) *r.f_out = f;
        return;
    }
    if (!*r.stale) return;
    if (r.tell && blockIdx.x == first && threadIdx.x == 0) *r.tell = 1;
    for (int64_t e = (int64_t)(blockIdx.x - first) * kBS + threadIdx.x; e < r.n_elems;
         e += (int64_t)(gridDim.x - first) * kBS) {
        const double v = r.adj[e];
        for (int j = 0; j < r.k; ++j) atomic_add_f64(r.out + r.conn[e * r.k + j], r.B[e * r.k + j] * v);
    }
}

// ------------------------------------------------------------ prefix scan
//
// Inclusive scan over chunks of kScanItems entries: chunk totals, then each
// chunk's local scan offset by the sum of the totals before it.  Up to
// kScanDirect chunks the workgroup of a chunk adds those itself (two launches,
// one for a single chunk); beyond, one workgroup scans the totals in between.
// With rev set, entry i is read and written at n-1-i, which turns the prefix
// scan into the suffix scan of the reverse pass: abar_j += sum_{i >= j} ybar_i.
// Summation order is fixed.  Bound by the launches up to some 10^5 entries, then
// by memory.  A program of one scan and its reverse, us, with the middle launch
// and each thread's run read straight from memory, with the chunks added
// directly, and read by consecutive lanes as well: 1,000 entries 21, 12, 12; 10^6
// 50, 45, 39; 8 10^6 227, 201, 137.  16 10^6: 432, 397, 288; 30 10^6 (14,649
// chunks, the totals read 10^8 times): 821, 806, so the middle launch again.

constexpr int kScanPer = 8;
constexpr int kScanItems = kBS * kScanPer;
constexpr int64_t kScanDirect = 8192;

__device__ __forceinline__ int64_t scan_at(int64_t n, int64_t i, int rev) { return rev ? n - 1 - i : i; }

// Exclusive scan of one value per thread over the workgroup; *total gets the sum.
__device__ __forceinline__ double block_excl_scan(double v, double* lds, double* total) {
    constexpr int NW = kBS / kWave;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    double inc = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const double t = __shfl_up(inc, d, kWave);
        if (lane >= d) inc += t;
    }
    if (lane == kWave - 1) lds[w] = inc;
    __syncthreads();
    double off = 0.0, tot = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const double t = lds[i];
        if (i < w) off += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return off + (inc - v);
}

// The workgroup's sum of one value per thread, in every thread.
__device__ __forceinline__ double block_sum_all(double v, double* lds) {
    v = wave_sum(v);
    if ((threadIdx.x & (kWave - 1)) == 0) lds[threadIdx.x / kWave] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kBS / kWave; ++w) t += lds[w];
    __syncthreads();
    return t;
}

__global__ void __launch_bounds__(kBS)
k_scan_totals(int64_t n, const double* __restrict__ a, int rev, double* __restrict__ totals) {
    __shared__ double lds[kBS / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanItems + threadIdx.x;
    double v[kScanPer];
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        const int64_t i = base + q * kBS;
        v[q] = i < n ? a[scan_at(n, i, rev)] : 0.0;
    }
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) s += v[q];
    const double t = block_sum<kBS>(s, lds);
    if (threadIdx.x == 0) totals[blockIdx.x] = t;
}

__global__ void __launch_bounds__(kBS)
k_scan_top(int64_t nchunks, double* __restrict__ totals) {
    __shared__ double lds[kBS / kWave];
    double carry = 0.0;
    for (int64_t b = 0; b < nchunks; b += kBS) {
        const int64_t i = b + threadIdx.x;
        const double v = i < nchunks ? totals[i] : 0.0;
        double tot;
        const double ex = block_excl_scan(v, lds, &tot);
        if (i < nchunks) totals[i] = carry + ex;
        carry += tot;
    }
}

// DIRECT: totals holds the chunk totals; else their exclusive scan.
// accumulate 0: y = scan; 1: y += scan.  Consecutive lanes read and write
// consecutive entries; in between each thread scans kScanPer consecutive ones,
// turned through LDS (one pad entry per thread's run).
template <bool DIRECT>
__global__ void __launch_bounds__(kBS)
k_scan_apply(int64_t n, const double* __restrict__ a, int rev, const double* __restrict__ totals,
             double* __restrict__ y, int accumulate) {
    __shared__ double lds[kBS / kWave];
    __shared__ double turn[kBS * (kScanPer + 1)];
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kScanItems + tid;
    double v[kScanPer], was[kScanPer];
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        const int64_t i = base + q * kBS;
        v[q] = i < n ? a[scan_at(n, i, rev)] : 0.0;
        was[q] = accumulate && i < n ? y[scan_at(n, i, rev)] : 0.0;
    }
    double before = 0.0;
    if constexpr (DIRECT) {
        for (unsigned q = tid; q < blockIdx.x; q += kBS) before += totals[q];
        before = block_sum_all(before, lds);
    } else {
        before = totals[blockIdx.x];
    }
    const int at = tid / kScanPer * (kScanPer + 1) + tid % kScanPer;  // of entry q * kBS + tid
    constexpr int kStep = kBS / kScanPer * (kScanPer + 1);
    double* const mine = turn + tid * (kScanPer + 1);
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) turn[q * kStep + at] = v[q];
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        v[q] = mine[q];
        s += v[q];
    }
    double tot;
    double run = before + block_excl_scan(s, lds, &tot);
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        run += v[q];
        mine[q] = run;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        const int64_t i = base + q * kBS;
        const double r = turn[q * kStep + at];
        if (i < n) y[scan_at(n, i, rev)] = accumulate ? was[q] + r : r;
    }
}

hipError_t launch_scan(int64_t n, const double* a, int rev, double* scratch, double* y,
                       int accumulate, hipStream_t s) {
    const int64_t nchunks = prog_scan_chunks(n);
    const dim3 grid((unsigned)nchunks), block(kBS);
    if (nchunks > 1)
        hipLaunchKernelGGL(k_scan_totals, grid, block, 0, s, n, a, rev, scratch);
    if (nchunks <= kScanDirect) {
        hipLaunchKernelGGL(k_scan_apply<true>, grid, block, 0, s, n, a, rev, scratch, y, accumulate);
    } else {
        hipLaunchKernelGGL(k_scan_top, dim3(1), block, 0, s, nchunks, scratch);
        hipLaunchKernelGGL(k_scan_apply<false>, grid, block, 0, s, n, a, rev, scratch, y, accumulate);
    }
    return hipGetLastError();
}

// ------------------------------------------- segment sum and broadcast
//
// One 64-lane wave per segment, four segments per workgroup.  The segment
// sum reduces lane-strided partial sums with a fixed butterfly
// (deterministic); its reverse, and the broadcast, write each entry of the
// segment from the segment's value; the broadcast's reverse is the segment
// sum of the output shadow.

constexpr int kSegPerBlock = kBS / kWave;

__global__ void __launch_bounds__(kBS)
k_segsum(int64_t n_seg, const int64_t* __restrict__ offs, const double* __restrict__ a,
         double* __restrict__ y, int accumulate) {
    const int64_t s = (int64_t)blockIdx.x * kSegPerBlock + threadIdx.x / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (s >= n_seg) return;  // whole waves leave together
    const int64_t b = offs[s], e = offs[s + 1];
    double t = 0.0;
    for (int64_t i = b + lane; i < e; i += kWave) t += a[i];
    t = wave_sum(t);
    if (lane == 0) {
        if (accumulate)
            y[s] += t;
        else
            y[s] = t;
    }
}

__global__ void __launch_bounds__(kBS)
k_segbcast(int64_t n_seg, const int64_t* __restrict__ offs, const double* __restrict__ a,
           double* __restrict__ y, int accumulate) {
    const int64_t s = (int64_t)blockIdx.x * kSegPerBlock + threadIdx.x / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (s >= n_seg) return;
    const int64_t b = offs[s], e = offs[s + 1];
    const double v = a[s];
    for (int64_t i = b + lane; i < e; i += kWave) {
        if (accumulate)
            y[i] += v;
        else
            y[i] = v;
    }
}

__global__ void __launch_bounds__(kBS)
k_validate_offsets(const int64_t* __restrict__ offs, int64_t n_seg, int64_t n, int32_t* flag) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int bad = 0;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s <= n_seg; s += stride) {
        const int64_t o = offs[s];
        if (s == 0 && o != 0) bad = 1;
        if (s == n_seg && o != n) bad = 1;
        if (s < n_seg && offs[s + 1] < o) bad = 1;
        if (o < 0 || o > n) bad = 1;
    }
    if (bad) atomicOr(flag, 1);
}

inline unsigned seg_blocks(int64_t n_seg) { return (unsigned)((n_seg + kSegPerBlock - 1) / kSegPerBlock); }

// ------------------------------------------------------------ fused groups

// NS FP64 slots addressed by a wave-uniform index.  A private array indexed
// at run time would live in scratch memory; here every access is a switch on
// the uniform index whose cases use constant indices, so the slots stay in
// VGPRs and an access costs a few scalar branches.  (Chains of selects over
// the slots measured twice as slow on the 128^3 mesh program.)  Launches
// pick the smallest NS (4, 8 or 16) that holds the group's leaves and ops.
#define PG_CASES(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)
template <int NS>
struct Slots {
    double r[NS];
    __device__ __forceinline__ Slots() {
#pragma unroll
        for (int q = 0; q < NS; ++q) r[q] = 0.0;
    }
    __device__ __forceinline__ double get(int i) const {
        switch (i) {
#define PG_GET(q) \
    case q:       \
        if constexpr (q < NS) return r[q < NS ? q : 0]; else return 0.0;
            PG_CASES(PG_GET)
#undef PG_GET
        }
        return 0.0;
    }
    __device__ __forceinline__ void set(int i, double v) {
        switch (i) {
#define PG_SET(q) \
    case q:       \
        if constexpr (q < NS) r[q < NS ? q : 0] = v; break;
            PG_CASES(PG_SET)
#undef PG_SET
        }
    }
    __device__ __forceinline__ void add(int i, double v) {
        switch (i) {
#define PG_ADD(q) \
    case q:       \
        if constexpr (q < NS) r[q < NS ? q : 0] += v; break;
            PG_CASES(PG_ADD)
#undef PG_ADD
        }
    }
};
#undef PG_CASES
static_assert(kGSlots == 16, "at most sixteen slots");

// Row of the fused gather: K > 0 keeps it in registers (vector loads);
// K < 0 is the generic row length, read again in the reverse scatter.
template <int K>
struct GatherRow {
    static constexpr int N = K > 0 ? K : 1;
    int32_t c[N];
    double b[N];
};

// A gathered row of any length: four entries' loads are in flight at a time.
__device__ __forceinline__ double gather_any(const GroupDev& g, int64_t i) {
    const int k = g.gk;
    const int32_t* c = g.gconn + i * k;
    const double* b = g.gB + i * k;
    double u = 0.0;
    int j = 0;
    for (; j + 4 <= k; j += 4) {
        int32_t n[4];
        double bv[4], xv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) n[q] = c[j + q];
#pragma unroll
        for (int q = 0; q < 4; ++q) bv[q] = b[j + q];
#pragma unroll
        for (int q = 0; q < 4; ++q) xv[q] = g.gsrc[n[q]];
#pragma unroll
        for (int q = 0; q < 4; ++q) u += bv[q] * xv[q];
    }
    for (; j < k; ++j) u += b[j] * g.gsrc[c[j]];
    return u;
}

// The products of a gathered row with its adjoint, at their places in the
// transposed connectivity.
template <int K>
__device__ __forceinline__ void store_products(const GroupDev& g, int64_t i, const GatherRow<K>& row,
                                               double ub) {
    g.gather_adj[i] = ub;
    bool changed = false;
    if constexpr (K > 0) {
        int32_t pos[K], was[K];
        load_conn_row<double, K>(g.gather_pos, i, pos);
        load_conn_row<double, K>(g.conn_copy, i, was);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            g.gather_prod[pos[j]] = row.b[j] * ub;
            changed |= was[j] != row.c[j];
        }
    } else {
        for (int j = 0; j < g.gk; ++j) {
            const int64_t q = i * g.gk + j;
            g.gather_prod[g.gather_pos[q]] = g.gB[q] * ub;
            changed |= g.conn_copy[q] != g.gconn[q];
        }
    }
    if (changed) *g.stale = 1;
}

// The last workgroup to take the ticket sums the partials of f.
template <int BS>
__device__ __forceinline__ void sum_by_last(const GroupDev& g, double* lds, int* last_wg) {
    if (threadIdx.x == 0) {
        publish_wait();  // its partial
        *last_wg = take_ticket(g.ticket, (int)gridDim.x);
    }
    __syncthreads();
    if (*last_wg) {
        double v = 0.0;
        for (int q = threadIdx.x; q < (int)gridDim.x; q += BS) v += read_published(g.partials + q);
        v = block_sum<BS>(v, lds);
        if (threadIdx.x == 0) *g.f_out = v;
    }
}

// A larger group that scatters nothing.  The slots live in LDS, one column of
// BS entries per slot, so a run-time slot index is an address and the
// interpreter is a short loop; every load (leaves, export shadows, shadows
// that are added to, the ops) is issued before the first is waited for.  Bound
// by the interpreter's latency up to some 10^5 entries, by memory above.
//
// K: fused gather row length (0 none, -1 generic).
template <int K, int MODE>
__global__ void __launch_bounds__(kBS) k_group_lds(GroupDev g) {
    constexpr bool REV = MODE != G_FWD;
    constexpr bool FWD = MODE != G_REV;
    extern __shared__ double slots[];
    constexpr int kOpWords = (int)(sizeof(GOp) / 4);
    static_assert(kGOps * kOpWords <= kBS, "one word of the ops per thread");
    __shared__ alignas(16) uint32_t op_words[kGOps * kOpWords];
    const GOp* const ops = reinterpret_cast<const GOp*>(op_words);
    __shared__ double lds[kBS / kWave];
    __shared__ int last_wg;
    const int tid = threadIdx.x;
    const int64_t i = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * kBS + tid;
    const bool ok = i < g.n;
    const int L = g.n_leaves, ns = L + g.n_ops;
    double* const r = slots + tid;                      // forward values, slot s at r[s * kBS]
    double* const a = slots + (int64_t)ns * kBS + tid;  // adjoints (REV)
    uint32_t word = 0;
    if (tid < g.n_ops * kOpWords) word = reinterpret_cast<const uint32_t*>(g.ops)[tid];
    double lv[kGLeaves] = {};
    [[maybe_unused]] double sv[kGLeaves] = {}, ev[kGExports] = {};
    [[maybe_unused]] GatherRow<K> row;
    if (ok) {
        if constexpr (K > 0) {
            double xv[K];
            load_conn_row<double, K>(g.gconn, i, row.c);
            load_b_row<K>(g.gB, i, row.b);
#pragma unroll
            for (int j = 0; j < K; ++j) xv[j] = g.gsrc[row.c[j]];
#pragma unroll
            for (int l = 0; l < kGLeaves; ++l)
                if (l < L && l != g.gather_slot) lv[l] = g.leaf[l][i];
            double u = 0.0;
#pragma unroll
            for (int j = 0; j < K; ++j) u += row.b[j] * xv[j];
            r[g.gather_slot * kBS] = u;
        } else {
#pragma unroll
            for (int l = 0; l < kGLeaves; ++l)
                if (l < L && l != g.gather_slot) lv[l] = g.leaf[l][i];
            if constexpr (K < 0) {
                r[g.gather_slot * kBS] = gather_any(g, i);
            }
        }
        if constexpr (REV) {
#pragma unroll
            for (int x = 0; x < kGExports; ++x)
                if (x < g.n_exports && g.export_shadow[x]) ev[x] = g.export_shadow[x][i];
#pragma unroll
            for (int l = 0; l < kGLeaves; ++l)
                if (l < L && g.leaf_shadow[l] && g.leaf_acc[l]) sv[l] = g.leaf_shadow[l][i];
        }
    }
    if (tid < g.n_ops * kOpWords) op_words[tid] = word;
    __syncthreads();
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    if (ok) {
#pragma unroll
        for (int l = 0; l < kGLeaves; ++l)
            if (l < L && l != g.gather_slot) r[l * kBS] = lv[l];
        for (int j = 0; j < g.n_ops; ++j) {
            // the reverse recomputes only the values that it reads
            if (!FWD && !(g.needed >> j & 1)) continue;
            const GOp o = ops[j];
            const int kind = uni(o.kind);
            const double x = r[uni(o.a) * kBS];
            double v;
            if (kind == P_SCALE) {
                v = o.alpha * x;
            } else if (kind == P_MAP) {
                v = map_f(uni(o.fn), x);
            } else {
                const double y = r[uni(o.b) * kBS];
                v = kind == P_ADD ? o.alpha * x + o.beta * y : x * y;
            }
            r[(L + j) * kBS] = v;
        }
        if constexpr (FWD) {
            for (int x = 0; x < g.n_exports; ++x) g.export_val[x][i] = r[g.export_slot[x] * kBS];
        }
    }
    if constexpr (FWD) {
        if (g.sum_slot >= 0) {
            const double t = block_sum<kBS>(ok ? r[g.sum_slot * kBS] : 0.0, lds);
            if (tid == 0) publish(g.partials + blockIdx.x, t);
        }
    }
    if constexpr (REV) {
        if (ok) {
            for (int q = 0; q < ns; ++q) a[q * kBS] = 0.0;
            if (g.sum_slot >= 0) a[g.sum_slot * kBS] = g.seed ? *g.seed : 1.0;
#pragma unroll
            for (int x = 0; x < kGExports; ++x)
                if (x < g.n_exports && g.export_shadow[x]) a[g.export_slot[x] * kBS] += ev[x];
            for (int j = g.n_ops - 1; j >= 0; --j) {
                const GOp o = ops[j];
                const int kind = uni(o.kind), oa = uni(o.a) * kBS;
                const double yb = a[(L + j) * kBS];
                if (kind == P_SCALE) {
                    a[oa] += o.alpha * yb;
                } else if (kind == P_MAP) {
                    a[oa] += map_df(uni(o.fn), r[oa]) * yb;
                } else {
                    const int ob = uni(o.b) * kBS;
                    if (kind == P_ADD) {
                        a[oa] += o.alpha * yb;
                        a[ob] += o.beta * yb;
                    } else {
                        const double av = r[oa], bv = r[ob];
                        a[oa] += bv * yb;
                        a[ob] += av * yb;
                    }
                }
            }
#pragma unroll
            for (int l = 0; l < kGLeaves; ++l) {
                if (l >= L || l == g.gather_slot || !g.leaf_shadow[l]) continue;
                const double v = a[l * kBS];
                g.leaf_shadow[l][i] = g.leaf_acc[l] ? sv[l] + v : v;
            }
            if constexpr (K != 0)
                if (g.gather_adj) store_products<K>(g, i, row, a[g.gather_slot * kBS]);
        }
    }
    if constexpr (FWD) {
        if (g.sum_slot >= 0 && g.ticket) sum_by_last<kBS>(g, lds, &last_wg);
    }
}

// K: fused gather row length (0 none, -1 generic); NS: slots; BS: workgroup;
// S: slots of the LDS table of the fused gather's scatter (0 without one: no
// gather, a forward pass, or a gather whose adjoint is written to
// g.gather_adj for the pass over the transposed connectivity).
template <int K, int MODE, int BS, int NS, int S>
__global__ void __launch_bounds__(BS) k_group(GroupDev g) {
    constexpr bool REV = MODE != G_FWD;
    constexpr bool FWD = MODE != G_REV;
    constexpr bool AGG = S > 0;
    static_assert(!AGG || (REV && K != 0), "only the reverse of a fused gather scatters");
    constexpr int NL = NS < kGLeaves ? NS : kGLeaves;
    __shared__ double lds[BS / kWave];
    __shared__ int last_wg;
    __shared__ typename std::conditional<AGG, AggTableT<S>, int>::type tab;
    const bool scatter = AGG && g.gsrc_shadow != nullptr;
    const int64_t i = xcd_remap(blockIdx.x, gridDim.x) * BS + threadIdx.x;
    const bool ok = i < g.n;
    const int L = g.n_leaves;
    Slots<NS> r;
    GatherRow<K> row;
    // The reverse of a group without ops (a gather of its own) is linear: it
    // needs the gather rows but no forward values.
    const bool values = FWD || g.n_ops > 0;
    if (ok) {
        // Every load first: the gather row, the gathered entries (issued as
        // soon as the row's connectivity is in: the leaves' loads sit behind
        // branches, and issued before the gather they made the gather wait
        // for B as well), then the leaves.
        double xv[K > 0 ? K : 1];
        if constexpr (K > 0) {
            load_conn_row<double, K>(g.gconn, i, row.c);
            load_b_row<K>(g.gB, i, row.b);
            if (values) {
#pragma unroll
                for (int j = 0; j < K; ++j) xv[j] = g.gsrc[row.c[j]];
            }
        }
#pragma unroll
        for (int l = 0; l < NL; ++l)
            if (l < L && l != g.gather_slot) r.r[l] = g.leaf[l][i];
        if (!values) {
        } else if constexpr (K > 0) {
            double u = 0.0;
#pragma unroll
            for (int j = 0; j < K; ++j) u += row.b[j] * xv[j];
            r.set(g.gather_slot, u);
        } else if constexpr (K < 0) {
            r.set(g.gather_slot, gather_any(g, i));
        }
        (void)values;
        for (int j = 0; j < g.n_ops; ++j) {
            // the reverse recomputes only the values that it reads
            if (!FWD && !(g.needed >> j & 1)) continue;
            const GOp o = g.ops[j];
            const double x = r.get(o.a);
            double v;
            switch (o.kind) {
                case P_SCALE: v = o.alpha * x; break;
                case P_ADD: v = o.alpha * x + o.beta * r.get(o.b); break;
                case P_MUL: v = x * r.get(o.b); break;
                default: v = map_f(o.fn, x); break;
            }
            r.set(L + j, v);
        }
        if constexpr (FWD) {
            for (int x = 0; x < g.n_exports; ++x) g.export_val[x][i] = r.get(g.export_slot[x]);
        }
    }
    if constexpr (FWD) {
        if (g.sum_slot >= 0) {
            const double t = block_sum<BS>(ok ? r.get(g.sum_slot) : 0.0, lds);
            if (threadIdx.x == 0) publish(g.partials + blockIdx.x, t);
        }
    }
    if constexpr (REV) {
        Slots<NS> a;
        if (ok) {
            if (g.sum_slot >= 0) a.add(g.sum_slot, g.seed ? *g.seed : 1.0);
            for (int x = 0; x < g.n_exports; ++x)
                if (g.export_shadow[x]) a.add(g.export_slot[x], g.export_shadow[x][i]);
            for (int j = g.n_ops - 1; j >= 0; --j) {
                const GOp o = g.ops[j];
                const double yb = a.get(L + j);
                switch (o.kind) {
                    case P_SCALE: a.add(o.a, o.alpha * yb); break;
                    case P_ADD:
                        a.add(o.a, o.alpha * yb);
                        a.add(o.b, o.beta * yb);
                        break;
                    case P_MUL: {
                        const double av = r.get(o.a), bv = r.get(o.b);
                        a.add(o.a, bv * yb);
                        a.add(o.b, av * yb);
                        break;
                    }
                    default: a.add(o.a, map_df(o.fn, r.get(o.a)) * yb); break;
                }
            }
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                if (l >= L || l == g.gather_slot || !g.leaf_shadow[l]) continue;
                double* p = g.leaf_shadow[l] + i;
                if (g.leaf_acc[l])
                    *p += a.r[l];
                else
                    *p = a.r[l];
            }
        }
        if constexpr (REV && K != 0 && !AGG) {
            if (ok && g.gather_adj) store_products<K>(g, i, row, a.get(g.gather_slot));
        }
        if constexpr (AGG) {
            if (scatter) {
                // The table is cleared only now, so the loads above were not held up.
                agg_clear(tab);
                __syncthreads();
                if (ok) {
                    const double ub = a.get(g.gather_slot);
                    if constexpr (K > 0) {
                        double cc[K];
#pragma unroll
                        for (int j = 0; j < K; ++j) cc[j] = row.b[j] * ub;
                        agg_add_row<K>(tab, row.c, cc, g.gsrc_shadow, g.hash_shift);
                    } else {
                        for (int j = 0; j < g.gk; ++j)
                            agg_add(tab, g.gconn[i * g.gk + j], g.gB[i * g.gk + j] * ub,
                                    g.gsrc_shadow, g.hash_shift);
                    }
                }
                __syncthreads();
                agg_flush(tab, g.gsrc_shadow);
            }
        }
    }
    if constexpr (FWD) {
        if (g.sum_slot >= 0 && g.ticket) sum_by_last<BS>(g, lds, &last_wg);
    }
}

// Whether a launch scatters its fused gather with atomics (an inactive
// operand, or one delivered through the transposed connectivity, does not).
bool group_scatters(const GroupDev& g, int mode) {
    return g.gather_slot >= 0 && mode != G_FWD && g.gsrc_shadow && !g.gather_adj;
}

template <int K, int NS>
hipError_t launch_scatter(const GroupDev& g, int mode, hipStream_t s) {
    constexpr int BS = kGroupBlockScatter;
    const dim3 grid((unsigned)group_blocks(g.n, BS)), block(BS);
    const bool small = g.agg_slots == kAggSlotsSmall;
    if (mode == G_REV) {
        if (small)
            PG_LAUNCH((k_group<K, G_REV, BS, NS, kAggSlotsSmall>), grid, block, 0, s, g);
        else
            PG_LAUNCH((k_group<K, G_REV, BS, NS, kAggSlots>), grid, block, 0, s, g);
    } else {
        if (small)
            PG_LAUNCH((k_group<K, G_FWDREV, BS, NS, kAggSlotsSmall>), grid, block, 0, s, g);
        else
            PG_LAUNCH((k_group<K, G_FWDREV, BS, NS, kAggSlots>), grid, block, 0, s, g);
    }
    return hipGetLastError();
}

// Slots up to which a group that scatters nothing keeps them in registers.
// In LDS, with more, the mix program's five-op reverse takes 6.7 us at
// 300,007 entries (12.1 in registers) and the segment program's sum group 18.5
// at 10^6 (20.8); its one-op reverse would take 13.0 (9.9 in registers).
constexpr int kRegisterSlots = 4;

template <int K>
hipError_t launch_group_ns(const GroupDev& g, int mode, hipStream_t s) {
    const int need = g.n_leaves + g.n_ops;
    if constexpr (K != 0) {
        if (group_scatters(g, mode)) {
            if (need <= 4) return launch_scatter<K, 4>(g, mode, s);
            if (need <= 8) return launch_scatter<K, 8>(g, mode, s);
            return launch_scatter<K, 16>(g, mode, s);
        }
    }
    const dim3 grid((unsigned)group_blocks(g.n, kBS)), block(kBS);
    if (need <= kRegisterSlots) {
        constexpr int NS = kRegisterSlots;
        switch (mode) {
            case G_FWD: PG_LAUNCH((k_group<K, G_FWD, kBS, NS, 0>), grid, block, 0, s, g); break;
            case G_REV: PG_LAUNCH((k_group<K, G_REV, kBS, NS, 0>), grid, block, 0, s, g); break;
            default: PG_LAUNCH((k_group<K, G_FWDREV, kBS, NS, 0>), grid, block, 0, s, g); break;
        }
        return hipGetLastError();
    }
    const unsigned lds = (unsigned)(sizeof(double) * need * kBS * (mode == G_FWD ? 1 : 2));
    switch (mode) {
        case G_FWD: PG_LAUNCH((k_group_lds<K, G_FWD>), grid, block, lds, s, g); break;
        case G_REV: PG_LAUNCH((k_group_lds<K, G_REV>), grid, block, lds, s, g); break;
        default: PG_LAUNCH((k_group_lds<K, G_FWDREV>), grid, block, lds, s, g); break;
    }
    return hipGetLastError();
}

}  // namespace

int64_t prog_scan_chunks(int64_t n) { return (n + kScanItems - 1) / kScanItems; }

int prog_scan_launches(int64_t n) {
    const int64_t c = prog_scan_chunks(n);
    return c <= 1 ? (int)c : c <= kScanDirect ? 2 : 3;
}

int64_t group_blocks(int64_t n, int bs) { return (n + bs - 1) / bs; }

// A group with a fused gather scatters through the LDS table in its reverse
// pass; a larger workgroup combines more contributions per table clear and
// flush (512 threads measured best for eight-node rows, as for the mesh).
int group_block_size(const GroupDev& g, int mode) {
    return group_scatters(g, mode) ? kGroupBlockScatter : kGroupBlock;
}

hipError_t launch_group(const GroupDev& g, int mode, hipStream_t s) {
    if (g.n == 0) return hipSuccess;
    if (g.n_leaves + g.n_ops > kGSlots || g.n_leaves > kGLeaves || g.n_ops > kGOps)
        return hipErrorInvalidValue;
    if (g.gather_slot < 0) return launch_group_ns<0>(g, mode, s);
    const bool vec = (reinterpret_cast<uintptr_t>(g.gconn) % 16 == 0) &&
                     (reinterpret_cast<uintptr_t>(g.gB) % 16 == 0);
    if (vec) {
        switch (g.gk) {
            case 2: return launch_group_ns<2>(g, mode, s);
            case 3: return launch_group_ns<3>(g, mode, s);
            case 4: return launch_group_ns<4>(g, mode, s);
            case 8: return launch_group_ns<8>(g, mode, s);
            default: break;
        }
    }
    return launch_group_ns<-1>(g, mode, s);
}

hipError_t launch_part_keys(const int32_t* conn, int64_t n_elems, int32_t k, int64_t n_nodes,
                            int32_t* keys, hipStream_t s) {
    if (n_elems == 0) return hipSuccess;
    hipLaunchKernelGGL(k_part_keys, dim3(std::min(nblocks(n_elems * k), 8192u)), dim3(kBS), 0, s, conn,
                       n_elems, k, n_nodes, keys);
    return hipGetLastError();
}

hipError_t launch_gather_rev(const GatherRev& r, hipStream_t s) {
    if (r.n_nodes == 0) return hipSuccess;
    const dim3 grid(nblocks(r.n_nodes)), block(kBS);
    if (r.parts == 1)
        PG_LAUNCH(k_gather_rev<1>, grid, block, 0, s, r);
    else if (r.parts == kXcds)
        PG_LAUNCH(k_gather_rev<kXcds>, grid, block, 0, s, r);
    else
        return hipErrorInvalidValue;
    const unsigned scatter = std::min(nblocks(r.n_elems), 256u) + (r.f_out ? 1u : 0u);
    hipLaunchKernelGGL(k_gather_scatter, dim3(scatter), block, 0, s, r);
    return hipGetLastError();
}

hipError_t launch_prog_fwd(const ProgOpDev& o, hipStream_t s) {
    if (o.n == 0) return hipSuccess;
    switch (o.kind) {
        case P_STENCIL: hipLaunchKernelGGL(k_stencil, dim3(nblocks(o.n)), dim3(kBS), 0, s, o.n, o.a, o.taps, o.y); break;
        case P_SCAN: return launch_scan(o.n, o.a, 0, o.scratch, o.y, 0, s);
        case P_SEGSUM:
            hipLaunchKernelGGL(k_segsum, dim3(seg_blocks(o.n_seg)), dim3(kBS), 0, s, o.n_seg, o.offs, o.a, o.y, 0);
            break;
        case P_BCAST:
            hipLaunchKernelGGL(k_segbcast, dim3(seg_blocks(o.n_seg)), dim3(kBS), 0, s, o.n_seg, o.offs, o.a, o.y, 0);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_prog_rev(const ProgOpDev& o, hipStream_t s) {
    // a broadcast's reverse writes every segment's adjoint, even with no outputs
    if (o.kind == P_BCAST ? o.n_seg == 0 : o.n == 0) return hipSuccess;
    switch (o.kind) {
        case P_STENCIL: hipLaunchKernelGGL(k_r_stencil, dim3(nblocks(o.n)), dim3(kBS), 0, s, o.n, o.yb, o.taps, o.ab, o.accumulate); break;
        case P_SCAN: return launch_scan(o.n, o.yb, 1, o.scratch, o.ab, o.accumulate, s);
        case P_SEGSUM:  // reverse of a segment sum: broadcast of the output shadow
            hipLaunchKernelGGL(k_segbcast, dim3(seg_blocks(o.n_seg)), dim3(kBS), 0, s, o.n_seg, o.offs, o.yb, o.ab, o.accumulate);
            break;
        case P_BCAST:  // reverse of a broadcast: segment sum of the output shadow
            hipLaunchKernelGGL(k_segsum, dim3(seg_blocks(o.n_seg)), dim3(kBS), 0, s, o.n_seg, o.offs, o.yb, o.ab, o.accumulate);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_validate_offsets(const int64_t* offs, int64_t n_seg, int64_t n, int32_t* flag,
                                   hipStream_t s) {
    const int64_t g = std::min<int64_t>((n_seg + kBS) / kBS, 4096);
    hipLaunchKernelGGL(k_validate_offsets, dim3((unsigned)g), dim3(kBS), 0, s, offs, n_seg, n, flag);
    return hipGetLastError();
}

}  // namespace pg
