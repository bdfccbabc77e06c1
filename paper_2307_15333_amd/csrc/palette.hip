// Median-cut palette of the SH coefficients (the compressed octrees of
// Sec. 4.1, Heckbert's median cut).  Every leaf's SH row (3K values) is a point;
// in each of `bits` rounds every box is cut at the median of its widest
// dimension (ties: lowest dimension; members ordered by value, then leaf
// index; -0.0 == +0.0), the lower n/2 members going to box 2b and the rest to
// 2b + 1.  The palette entry of a box is the FP64 mean of its members rounded
// once to FP16; each leaf keeps the uint16 index of its box.
//
// Device layout: the rows stay where they are; the leaf ids are kept in box
// order (box b occupies positions [start[b], start[b+1]), its members in
// ascending id), and a round moves only them.  A round reads every row once
// (per-box minima and maxima, 16 bytes a lane) and one value of it again (the
// key, value bits << LB | leaf id, along the box's widest dimension), finds
// each box's median key by a radix select and partitions the ids stably.
//
// Boxes of more than SMALL members are shared by the workgroups of their
// chunks: one launch a digit, whose last workgroup picks it.  Once all boxes
// fit a workgroup, a round is one launch: a workgroup a box, its keys in
// registers.  On 0.87M FP32 rows of degree 3 and 12 rounds the kernels take 1.4 ms
// (41 us of a round for the 166 MB of rows: 4 TB/s through the permuted ids);
// moving the rows themselves every round took 11.6 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dot_device.h"

namespace dot {

namespace {

constexpr int PB = 256;       // threads per workgroup
constexpr int CH = 1024;      // positions per (box, chunk) workgroup
constexpr int PER = 4;        // keys per thread of a workgroup that holds a whole box
constexpr int WIDE = 1024;    // threads of that workgroup while boxes are large
constexpr int SMALL = WIDE * PER;
constexpr int SEL_BITS = 11, SEL_BINS = 1 << SEL_BITS;

// the median search of one box
struct BoxSel {
    uint64_t prefix;          // digits found so far, zeros below
    uint32_t rank;            // rank of the median among the keys that match them
    uint32_t ticket;          // workgroups of the current pass that are through
    int32_t dim;
    uint32_t done;            // rank 0: no matching key lies below the prefix
};

struct Bufs {
    uint32_t *ids, *ids2, *cnt, *off, *bsum, *tot;
    uint64_t* keys;
    uint32_t *start, *start2, *mm, *hist;
    BoxSel* sel;
};

__device__ __forceinline__ uint32_t ord_f32(float f) {
    if (f == 0.f) f = 0.f;   // -0.0 orders with +0.0
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unord_f32(uint32_t o) {
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// FP64 -> FP16 rounded once: an FP32 rounded to odd keeps enough bits for the
// final round-to-nearest-even not to be a double rounding
__device__ __forceinline__ uint16_t f64_to_f16(double x) {
    float f = __double2float_rz(x);
    if ((double)f != x) f = __uint_as_float(__float_as_uint(f) | 1u);
    return f32_to_f16(f);
}

__global__ void k_pal_ids(int64_t N, uint32_t* __restrict__ ids) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x)
        ids[i] = (uint32_t)i;
}

template <int DT>
__global__ void k_pal_sigma(const void* __restrict__ src, int64_t N, uint16_t* __restrict__ dst) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = f32_to_f16(load_sigma<DT>(src, i));
}

// mm is [nb][64][2]: minima start at all ones, maxima at zero
__global__ void k_pal_init(uint32_t* __restrict__ mm, uint32_t* __restrict__ hist, BoxSel* __restrict__ sel,
                           const uint32_t* __restrict__ start, int64_t nb) {
    const int64_t n = nb * SEL_BINS;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        hist[i] = 0u;
        if (i < nb * 64) {
            mm[2 * i] = 0xffffffffu;
            mm[2 * i + 1] = 0u;
        }
        if (i < nb) sel[i] = BoxSel{0ull, (start[i + 1] - start[i]) / 2, 0u, 0, 0u};
    }
}

// Minima and maxima (ordered bits) per dimension of the rows at positions
// [lo, hi) into smn/smx[64] in LDS.  Lanes take a 16-byte piece of a row each, as
// many rows a wave and load as fit; the rows of four loads are in flight.
template <int DT, int NT>
__device__ __forceinline__ void block_minmax(const uint4* __restrict__ sh, int pieces, const uint32_t* __restrict__ ids,
                                             int64_t lo, int64_t hi, uint32_t* smn, uint32_t* smx) {
    constexpr int E = DT == DOT_F32 ? 4 : 8, U = 4;
    if (threadIdx.x < 64) {
        smn[threadIdx.x] = 0xffffffffu;
        smx[threadIdx.x] = 0u;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int rpw = 64 / pieces, row = lane / pieces, q = lane - row * pieces;
    uint32_t mn[E], mx[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        mn[e] = 0xffffffffu;
        mx[e] = 0u;
    }
    if (row < rpw)
        for (int64_t r = lo + w * rpw + row; r < hi; r += (int64_t)U * (NT / 64) * rpw) {
            uint4 v[U];
            bool in[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t ru = r + (int64_t)u * (NT / 64) * rpw;
                in[u] = ru < hi;
                if (in[u]) v[u] = sh[(int64_t)ids[ru] * pieces + q];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!in[u]) continue;
                const uint32_t x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    float f;
                    if constexpr (DT == DOT_F32)
                        f = __uint_as_float(x[e]);
                    else {
                        const uint32_t h = (x[e >> 1] >> ((e & 1) * 16)) & 0xffffu;
                        f = DT == DOT_F16 ? f16_to_f32(h) : bf16_to_f32(h);
                    }
                    const uint32_t o = ord_f32(f);
                    mn[e] = min(mn[e], o);
                    mx[e] = max(mx[e], o);
                }
            }
        }
    if (row < rpw && mn[0] <= mx[0]) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            atomicMin(&smn[q * E + e], mn[e]);
            atomicMax(&smx[q * E + e], mx[e]);
        }
    }
    __syncthreads();
}

// The widest dimension (largest max - min in FP64, first of equals), found by
// one wave from lane d's minimum and maximum.
__device__ __forceinline__ int widest(uint32_t mn, uint32_t mx, int D) {
    const int lane = threadIdx.x & 63;
    double w = -1.0;
    if (lane < D) {
        const double x = (double)unord_f32(mx) - (double)unord_f32(mn);
        if (x > w) w = x;       // not a NaN
    }
    int d = lane;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double w2 = __shfl_xor(w, o, 64);
        const int d2 = __shfl_xor(d, o, 64);
        if (w2 > w || (w2 == w && d2 < d)) {
            w = w2;
            d = d2;
        }
    }
    return w < 0.0 ? 0 : d;
}

template <int DT>
__global__ __launch_bounds__(PB) void k_pal_minmax(const uint4* __restrict__ sh, int pieces, int D,
                                                   const uint32_t* __restrict__ ids, const uint32_t* __restrict__ start,
                                                   int cpb, uint32_t* __restrict__ mm) {
    __shared__ uint32_t smn[64], smx[64];
    const int b = blockIdx.x / cpb, c = blockIdx.x % cpb;
    const int64_t lo = (int64_t)start[b] + (int64_t)c * CH;
    const int64_t hi = lo + CH < (int64_t)start[b + 1] ? lo + CH : (int64_t)start[b + 1];
    if (lo >= hi) return;
    block_minmax<DT, PB>(sh, pieces, ids, lo, hi, smn, smx);
    if ((int)threadIdx.x < D) {
        atomicMin(&mm[((int64_t)b * 64 + threadIdx.x) * 2], smn[threadIdx.x]);
        atomicMax(&mm[((int64_t)b * 64 + threadIdx.x) * 2 + 1], smx[threadIdx.x]);
    }
}

// one wave per box
__global__ __launch_bounds__(PB) void k_pal_dim(const uint32_t* __restrict__ mm, int D, const uint32_t* __restrict__ start,
                                                int64_t nb, BoxSel* __restrict__ sel) {
    const int64_t b = blockIdx.x * (int64_t)(PB / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (b >= nb || start[b + 1] == start[b]) return;
    const int d = widest(mm[(b * 64 + lane) * 2], mm[(b * 64 + lane) * 2 + 1], D);
    if (lane == 0) sel[b].dim = d;
}

template <int DT>
__device__ __forceinline__ uint64_t row_key(const void* __restrict__ sh, int stride, int d, uint32_t id, int lb) {
    return ((uint64_t)ord_f32(load_sigma<DT>(sh, (int64_t)id * stride + d)) << lb) | id;
}

template <int DT>
__global__ __launch_bounds__(PB) void k_pal_keys(const void* __restrict__ sh, int stride, const uint32_t* __restrict__ ids,
                                                 const uint32_t* __restrict__ start, int cpb,
                                                 const BoxSel* __restrict__ sel, int lb, uint64_t* __restrict__ keys) {
    const int b = blockIdx.x / cpb, c = blockIdx.x % cpb;
    const int64_t lo = (int64_t)start[b] + (int64_t)c * CH, s1 = start[b + 1];
    const int d = sel[b].dim;
    for (int64_t i = lo + threadIdx.x; i < lo + CH && i < s1; i += PB) keys[i] = row_key<DT>(sh, stride, d, ids[i], lb);
}

// The bin of the histogram h (read through `at`) that holds `rank`, found by the
// workgroup; every thread gets the bin and the rank within it.
template <int NT, class At>
__device__ __forceinline__ void find_bin(At at, uint32_t rank, uint32_t* part, uint32_t* out, uint32_t& bin, uint32_t& in_bin) {
    constexpr int RUN = SEL_BINS / NT;
    uint32_t run = 0;
#pragma unroll
    for (int i = 0; i < RUN; ++i) run += at(threadIdx.x * RUN + i);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) part[w] = x;
    __syncthreads();
    uint32_t before = x - run;
    for (int j = 0; j < w; ++j) before += part[j];
    if (before <= rank && rank < before + run) {
        uint32_t d = threadIdx.x * RUN, c;
        while (rank >= before + (c = at(d))) {
            before += c;
            ++d;
        }
        out[0] = d;
        out[1] = rank - before;
    }
    __syncthreads();
    bin = out[0];
    in_bin = out[1];
    __syncthreads();
}

// One digit of the median search of every box that is not decided yet: the
// histogram of the keys that match the digits so far, then, in the last of the
// box's workgroups to finish, the digit holding the wanted rank.
__global__ __launch_bounds__(PB) void k_pal_select(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ start,
                                                   int cpb, int shift, int first, uint32_t* __restrict__ hist,
                                                   BoxSel* __restrict__ sel) {
    __shared__ uint32_t h[SEL_BINS];
    __shared__ uint32_t part[PB / 64], found[2];
    __shared__ int last;
    const int b = blockIdx.x / cpb, c = blockIdx.x % cpb;
    const int64_t lo = (int64_t)start[b] + (int64_t)c * CH, s1 = start[b + 1];
    const uint32_t chunks = (uint32_t)((s1 - (int64_t)start[b] + CH - 1) / CH);
    if (lo >= s1 || sel[b].done) return;
    for (int i = threadIdx.x; i < SEL_BINS; i += PB) h[i] = 0u;
    __syncthreads();
    const uint64_t pre = sel[b].prefix;
    const int up = shift + SEL_BITS;
    for (int64_t i = lo + threadIdx.x; i < lo + CH && i < s1; i += PB) {
        const uint64_t k = keys[i];
        if (first || (k >> up) == (pre >> up)) atomicAdd(&h[(k >> shift) & (SEL_BINS - 1)], 1u);
    }
    __syncthreads();
    uint32_t* hb = hist + (int64_t)b * SEL_BINS;
    for (int i = threadIdx.x; i < SEL_BINS; i += PB)
        if (h[i]) atomicAdd(&hb[i], h[i]);
    // this wave's additions are complete before the workgroup's ticket is drawn
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&sel[b].ticket, 1u) == chunks - 1u;
    __syncthreads();
    if (!last) return;
    uint32_t bin, rank;
    find_bin<PB>([&](int i) { return __hip_atomic_load(&hb[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }, sel[b].rank,
             part, found, bin, rank);
    for (int i = threadIdx.x; i < SEL_BINS; i += PB) hb[i] = 0u;
    if (threadIdx.x == 0) {
        sel[b].prefix = pre | ((uint64_t)bin << shift);
        sel[b].rank = rank;
        sel[b].ticket = 0u;
        sel[b].done = rank == 0u;
    }
}

// members of a chunk below the box's median
__global__ __launch_bounds__(PB) void k_pal_count(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ start,
                                                  int cpb, const BoxSel* __restrict__ sel, uint32_t* __restrict__ cnt) {
    __shared__ uint32_t part[PB / 64];
    const int b = blockIdx.x / cpb, c = blockIdx.x % cpb;
    const int64_t lo = (int64_t)start[b] + (int64_t)c * CH, s1 = start[b + 1];
    const uint64_t m = sel[b].prefix;
    uint32_t n = 0;
    for (int64_t i = lo + threadIdx.x; i < lo + CH && i < s1; i += PB) n += keys[i] < m ? 1u : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int j = 1; j < PB / 64; ++j) n += part[j];
        cnt[blockIdx.x] = n;
    }
}

// exclusive prefix over the workgroup
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t* part) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) part[w] = x;
    __syncthreads();
    uint32_t base = 0;
    for (int j = 0; j < w; ++j) base += part[j];
    return base + x - v;
}

// every member to its half, in order: lower members at the front of the box,
// upper members behind them.  `below`: lower members of the box before the
// thread's first position i0; a thread holds consecutive positions.
template <int NK>
__device__ __forceinline__ void place(const uint64_t (&k)[NK], const uint32_t (&id)[NK], int64_t i0, int64_t s0, int64_t s1,
                                      int64_t end, uint64_t m, uint32_t below, uint32_t* __restrict__ ids2) {
    const int64_t half = (s1 - s0) / 2;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        if (i0 + j >= end) continue;
        const bool low = k[j] < m;
        int64_t dst = low ? s0 + below : s0 + half + (i0 + j - s0) - below;
        below += low ? 1u : 0u;
        // exactly `half` members are below (the keys are distinct), so dst stays
        // in the box; the clamp only keeps a broken invariant in bounds
        dst = dst < s0 ? s0 : (dst >= s1 ? s1 - 1 : dst);
        ids2[dst] = id[j];
    }
}

__device__ __forceinline__ void split_start(int64_t b, int64_t nb, uint32_t s0, uint32_t s1, uint32_t* __restrict__ start2) {
    start2[2 * b] = s0;
    start2[2 * b + 1] = s0 + (s1 - s0) / 2;
    if (b == nb - 1) start2[2 * nb] = s1;
}

// off: exclusive prefix of cnt over all chunks
__global__ __launch_bounds__(PB) void k_pal_scatter(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ ids,
                                                    const uint32_t* __restrict__ start, int cpb, int64_t nb,
                                                    const BoxSel* __restrict__ sel, const uint32_t* __restrict__ off,
                                                    uint32_t* __restrict__ ids2, uint32_t* __restrict__ start2) {
    constexpr int NK = CH / PB;
    __shared__ uint32_t part[PB / 64];
    const int64_t b = blockIdx.x / cpb;
    const int c = blockIdx.x % cpb;
    const int64_t s0 = start[b], s1 = start[b + 1];
    if (c == 0 && threadIdx.x == 0) split_start(b, nb, (uint32_t)s0, (uint32_t)s1, start2);
    const int64_t lo = s0 + (int64_t)c * CH, end = lo + CH < s1 ? lo + CH : s1;
    const uint64_t m = sel[b].prefix;
    const int64_t i0 = lo + (int64_t)threadIdx.x * NK;
    uint64_t k[NK];
    uint32_t id[NK], n = 0;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        k[j] = ~0ull;
        if (i0 + j < end) {
            k[j] = keys[i0 + j];
            id[j] = ids[i0 + j];
            n += k[j] < m ? 1u : 0u;
        }
    }
    const uint32_t below = off[blockIdx.x] - off[b * cpb] + block_prefix(n, part);
    place<NK>(k, id, i0, s0, s1, end, m, below, ids2);
}

// a whole round of one box of at most NT * PER members
template <int DT, int NT>
__global__ __launch_bounds__(NT) void k_pal_round(const void* __restrict__ sh, int stride, int pieces, int D,
                                                  const uint32_t* __restrict__ ids, const uint32_t* __restrict__ start,
                                                  int64_t nb, int lb, int digits, uint32_t* __restrict__ ids2,
                                                  uint32_t* __restrict__ start2) {
    __shared__ uint32_t h[SEL_BINS];
    __shared__ uint32_t smn[64], smx[64], part[NT / 64], found[2];
    __shared__ int dim;
    const int64_t b = blockIdx.x;
    const int64_t s0 = start[b], s1 = start[b + 1];
    if (threadIdx.x == 0) split_start(b, nb, (uint32_t)s0, (uint32_t)s1, start2);
    if (s0 == s1) return;
    block_minmax<DT, NT>(static_cast<const uint4*>(sh), pieces, ids, s0, s1, smn, smx);
    if (threadIdx.x < 64) {
        const int d = widest(smn[threadIdx.x], smx[threadIdx.x], D);
        if (threadIdx.x == 0) dim = d;
    }
    __syncthreads();
    const int d = dim;
    // positions are dealt out evenly, a run a thread, so that small boxes use all threads
    const int run = (int)((s1 - s0 + NT - 1) / NT);
    const int64_t i0 = s0 + (int64_t)threadIdx.x * run;
    const int64_t end = i0 + run < s1 ? i0 + run : s1;
    uint64_t k[PER];
    uint32_t id[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        k[j] = ~0ull;
        if (i0 + j < end) {
            id[j] = ids[i0 + j];
            k[j] = row_key<DT>(sh, stride, d, id[j], lb);
        }
    }
    uint64_t m = 0ull;
    uint32_t rank = (uint32_t)((s1 - s0) / 2);
    for (int p = digits - 1; p >= 0 && rank > 0u; --p) {
        const int shift = p * SEL_BITS, up = shift + SEL_BITS;
        for (int i = threadIdx.x; i < SEL_BINS; i += NT) h[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (i0 + j < end && (p == digits - 1 || (k[j] >> up) == (m >> up)))
                atomicAdd(&h[(k[j] >> shift) & (SEL_BINS - 1)], 1u);
        __syncthreads();
        uint32_t bin;
        find_bin<NT>([&](int i) { return h[i]; }, rank, part, found, bin, rank);
        m |= (uint64_t)bin << shift;
    }
    uint32_t n = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) n += i0 + j < end && k[j] < m ? 1u : 0u;
    const uint32_t below = block_prefix(n, part);
    place<PER>(k, id, i0, s0, s1, end, m, below, ids2);
}

// one wave per box: lane d sums dimension d in FP64 in position order (eight
// rows in flight); the mean rounded once to FP16; every member's leaf gets the
// box index
template <int DT>
__global__ void k_pal_mean(const void* __restrict__ sh, int stride, const uint32_t* __restrict__ ids, int D, int pstride,
                           const uint32_t* __restrict__ start, int64_t nb, uint16_t* __restrict__ pal,
                           uint16_t* __restrict__ index) {
    constexpr int U = 8;
    const int64_t b = blockIdx.x * (int64_t)(blockDim.x / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (b >= nb) return;
    const uint32_t s0 = start[b], s1 = start[b + 1];
    if (lane < pstride) {
        uint16_t out = 0;
        if (lane < D && s1 > s0) {
            double acc = 0.0;
            uint32_t r = s0;
            for (; r + U <= s1; r += U) {
                float x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = load_sigma<DT>(sh, (int64_t)ids[r + u] * stride + lane);
#pragma unroll
                for (int u = 0; u < U; ++u) acc += (double)x[u];
            }
            for (; r < s1; ++r) acc += (double)load_sigma<DT>(sh, (int64_t)ids[r] * stride + lane);
            out = f64_to_f16(acc / (double)(s1 - s0));
        }
        pal[b * pstride + lane] = out;
    }
    for (uint32_t r = s0 + lane; r < s1; r += 64) index[ids[r]] = (uint16_t)b;
}

unsigned g1(int64_t n) {
    int64_t g = (n + PB - 1) / PB;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, 1 << 20));
}

// the rounds, the palette, the indices and the FP16 densities
template <int DT>
hipError_t cut(const dot_tree& t, Bufs B, int bits, int lb, int pstride, uint16_t* sig16, uint16_t* index, uint16_t* pal,
               hipStream_t s) {
    const int64_t N = t.n_leaves, P = (int64_t)1 << bits;
    const int D = 3 * (t.degree + 1) * (t.degree + 1);
    const int stride = t.sh_stride, pieces = stride * storage_bytes(t.storage) / 16;
    const uint4* rows = static_cast<const uint4*>(t.sh);
    const int digits = (32 + lb + SEL_BITS - 1) / SEL_BITS;
    hipLaunchKernelGGL(k_pal_sigma<DT>, dim3(g1(N)), dim3(PB), 0, s, t.sigma, N, sig16);
    hipError_t e = hipGetLastError();
    for (int r = 0; r < bits && e == hipSuccess; ++r) {
        const int64_t nb = (int64_t)1 << r;
        const int64_t maxn = (N + nb - 1) / nb;      // a box's members: N / nb rounded down or up
        if (maxn <= SMALL) {
            if (maxn <= PB * PER)
                hipLaunchKernelGGL((k_pal_round<DT, PB>), dim3((unsigned)nb), dim3(PB), 0, s, t.sh, stride, pieces, D, B.ids,
                                   B.start, nb, lb, digits, B.ids2, B.start2);
            else
                hipLaunchKernelGGL((k_pal_round<DT, WIDE>), dim3((unsigned)nb), dim3(WIDE), 0, s, t.sh, stride, pieces, D,
                                   B.ids, B.start, nb, lb, digits, B.ids2, B.start2);
            e = hipGetLastError();
        } else {
            const int cpb = (int)((maxn + CH - 1) / CH);
            const dim3 grid((unsigned)(nb * cpb));
            hipLaunchKernelGGL(k_pal_init, dim3(g1(nb * SEL_BINS)), dim3(PB), 0, s, B.mm, B.hist, B.sel, B.start, nb);
            hipLaunchKernelGGL(k_pal_minmax<DT>, grid, dim3(PB), 0, s, rows, pieces, D, B.ids, B.start, cpb, B.mm);
            hipLaunchKernelGGL(k_pal_dim, dim3((unsigned)((nb + 3) / 4)), dim3(PB), 0, s, B.mm, D, B.start, nb, B.sel);
            hipLaunchKernelGGL(k_pal_keys<DT>, grid, dim3(PB), 0, s, t.sh, stride, B.ids, B.start, cpb, B.sel, lb, B.keys);
            for (int p = digits - 1; p >= 0; --p)
                hipLaunchKernelGGL(k_pal_select, grid, dim3(PB), 0, s, B.keys, B.start, cpb, p * SEL_BITS,
                                   p == digits - 1 ? 1 : 0, B.hist, B.sel);
            hipLaunchKernelGGL(k_pal_count, grid, dim3(PB), 0, s, B.keys, B.start, cpb, B.sel, B.cnt);
            e = hipGetLastError();
            if (e == hipSuccess) e = scan_u32(B.cnt, B.off, nb * cpb, B.bsum, B.tot, s);
            if (e != hipSuccess) break;
            hipLaunchKernelGGL(k_pal_scatter, grid, dim3(PB), 0, s, B.keys, B.ids, B.start, cpb, nb, B.sel, B.off, B.ids2,
                               B.start2);
            e = hipGetLastError();
        }
        std::swap(B.ids, B.ids2);
        std::swap(B.start, B.start2);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pal_mean<DT>, dim3((unsigned)((P + 3) / 4)), dim3(PB), 0, s, t.sh, stride, B.ids, D, pstride,
                       B.start, P, pal, index);
    return hipGetLastError();
}

}  // namespace

// dst[r][d] = palette[index[row0 + r]][d] for rows [row0, row0 + rows), FP32
__global__ void k_pal_decode(const uint16_t* __restrict__ index, const uint16_t* __restrict__ pal, int pstride, int D,
                             int64_t rows, int64_t row0, float* __restrict__ dst) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < rows * D; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / D;
        const int d = (int)(i - r * D);
        dst[i] = f16_to_f32(pal[(int64_t)index[row0 + r] * pstride + d]);
    }
}

hipError_t launch_decode_palette(const dot_tree& t, float* dst, int64_t rows, int64_t row0, hipStream_t s) {
    if (rows == 0) return hipSuccess;
    const int D = 3 * (t.degree + 1) * (t.degree + 1);
    hipLaunchKernelGGL(k_pal_decode, dim3(g1(rows * D)), dim3(PB), 0, s, static_cast<const uint16_t*>(t.sh),
                       static_cast<const uint16_t*>(t.palette), t.sh_stride, D, rows, row0, dst);
    return hipGetLastError();
}

int quantize_sh(dot_tree& t, int bits, hipStream_t s) {
    const int64_t N = t.n_leaves;
    const int D = 3 * (t.degree + 1) * (t.degree + 1);
    const int64_t P = (int64_t)1 << bits;
    const int pstride = sh_stride_for(t.degree, DOT_F16);
    int lb = 1;
    while (((int64_t)1 << lb) < N) ++lb;
    const Alloc& al = t.alloc;
    // scratch
    struct Owned {
        const Alloc& al;
        void* p[24] = {};
        int n = 0;
        explicit Owned(const Alloc& a) : al(a) {}
        void* get(size_t bytes) {
            void* q = al.get(bytes);
            p[n++] = q;
            return q;
        }
        bool ok() const {
            for (int i = 0; i < n; ++i)
                if (!p[i]) return false;
            return true;
        }
        ~Owned() {
            for (int i = 0; i < n; ++i) al.put(p[i]);
        }
    } tmp(al);
    // chunks of the rounds whose boxes are shared by workgroups, and their boxes
    int64_t nb_big = 0, n_chunks = 0;
    for (int r = 0; r < bits; ++r) {
        const int64_t nb = (int64_t)1 << r, maxn = (N + nb - 1) / nb;
        if (maxn <= SMALL) break;
        nb_big = nb;
        n_chunks = std::max(n_chunks, nb * ((maxn + CH - 1) / CH));
    }
    Bufs B;
    B.ids = static_cast<uint32_t*>(tmp.get((size_t)N * 4));
    B.ids2 = static_cast<uint32_t*>(tmp.get((size_t)N * 4));
    B.start = static_cast<uint32_t*>(tmp.get((size_t)(P + 1) * 4));
    B.start2 = static_cast<uint32_t*>(tmp.get((size_t)(P + 1) * 4));
    B.keys = static_cast<uint64_t*>(tmp.get((size_t)(nb_big ? N : 0) * 8));
    B.cnt = static_cast<uint32_t*>(tmp.get((size_t)n_chunks * 4));
    B.off = static_cast<uint32_t*>(tmp.get((size_t)n_chunks * 4));
    B.bsum = static_cast<uint32_t*>(tmp.get((size_t)scan_scratch_elems(n_chunks) * 4));
    B.tot = static_cast<uint32_t*>(tmp.get(16));
    B.mm = static_cast<uint32_t*>(tmp.get((size_t)nb_big * 64 * 2 * 4));
    B.hist = static_cast<uint32_t*>(tmp.get((size_t)nb_big * SEL_BINS * 4));
    B.sel = static_cast<BoxSel*>(tmp.get((size_t)nb_big * sizeof(BoxSel)));
    // the new planes
    uint16_t* sig16 = static_cast<uint16_t*>(al.get((size_t)N * 2));
    uint16_t* index = static_cast<uint16_t*>(al.get((size_t)N * 2));
    uint16_t* pal = static_cast<uint16_t*>(al.get((size_t)P * pstride * 2));
    auto drop_new = [&]() {
        al.put(sig16);
        al.put(index);
        al.put(pal);
    };
    if (!tmp.ok() || !sig16 || !index || !pal) {
        drop_new();
        return fail(DOT_ENOMEM, "dot_quantize_sh: scratch allocation failed");
    }
    hipLaunchKernelGGL(k_pal_ids, dim3(g1(N)), dim3(PB), 0, s, N, B.ids);
    // start = {0, N}
    const uint32_t init[2] = {0u, (uint32_t)N};
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(B.start, init, sizeof(init), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);   // `init` is on the host stack
    if (e == hipSuccess)
        e = t.storage == DOT_F32   ? cut<DOT_F32>(t, B, bits, lb, pstride, sig16, index, pal, s)
            : t.storage == DOT_F16 ? cut<DOT_F16>(t, B, bits, lb, pstride, sig16, index, pal, s)
                                   : cut<DOT_BF16>(t, B, bits, lb, pstride, sig16, index, pal, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        drop_new();
        return hip_fail(e, "dot_quantize_sh");
    }
    al.put(t.sigma);
    al.put(t.sh);
    t.sigma = sig16;
    t.sh = index;
    t.palette = pal;
    t.palette_bits = bits;
    t.storage = DOT_PAL16;
    t.sh_stride = pstride;
    return DOT_OK;
}

}  // namespace dot
