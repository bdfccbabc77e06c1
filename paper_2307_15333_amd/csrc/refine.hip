// Octree refinement on the device (Sec. 3.2, Alg. 1: pruning, then sampling,
// both driven by the same per-leaf signal).
//
//   mark    an internal node merges iff its 8 children are leaves and all are
//           selected for pruning (signal <= tau, or < tau); with recursive
//           pruning (the paper's "(R)" option) merging repeats up the
//           hierarchy, which ends with every node whose subtree leaves are all
//           selected merged: the subtree's leaves are a contiguous DFS range,
//           so one prefix count of unselected leaves decides every node;
//   select  exact top-k of the 64-bit keys (~ord(signal) << 32 | leaf) over
//           the sampling candidates by an MSD radix select of up to 6 digits,
//           so ties in signal go to the lower leaf index;
//   rebuild new leaf and internal indices by exclusive prefix scans over the
//           old DFS order, then scatter: a merged group becomes one leaf with
//           the mean of its 8 rows (Eq. 3), a sampled leaf becomes an internal
//           node whose 8 children copy its row (Eq. 4).
// The result is numbered in DFS order, so its topology is canonical.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "dot_device.h"

namespace dot {

namespace {

constexpr int TPB = 256;

unsigned blocks_for(int64_t n, int per_thread = 1) {
    int64_t g = (n + (int64_t)TPB * per_thread - 1) / ((int64_t)TPB * per_thread);
    if (g > 1 << 20) g = 1 << 20;
    return (unsigned)(g < 1 ? 1 : g);
}

#define GRID_STRIDE(i, n) \
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

__device__ __forceinline__ bool selected(float s, float tau, int le) { return le ? (s <= tau) : (s < tau); }

// order-preserving map of a float to uint32 (ascending)
__device__ __forceinline__ uint32_t ord32(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
    GRID_STRIDE(i, n) p[i] = v;
}

// first / last leaf of each internal node's subtree and the node's depth
__global__ void k_node_meta(const int32_t* __restrict__ child, int64_t I, const uint8_t* __restrict__ leaf_depth,
                            int32_t* __restrict__ first, int32_t* __restrict__ last, int32_t* __restrict__ ndepth) {
    GRID_STRIDE(p, I) {
        int steps = 1;
        int32_t e = child[p * 8];
        while (e >= 0) {
            e = child[(int64_t)e * 8];
            ++steps;
        }
        first[p] = -1 - e;
        ndepth[p] = (int32_t)leaf_depth[-1 - e] - steps;
        e = child[p * 8 + 7];
        while (e >= 0) e = child[(int64_t)e * 8 + 7];
        last[p] = -1 - e;
    }
}

__global__ void k_node_parent(const int32_t* __restrict__ child, int64_t I, int32_t* __restrict__ parent) {
    GRID_STRIDE(j, I * 8) {
        int32_t e = child[j];
        if (e >= 0) parent[e] = (int32_t)(j >> 3);
    }
}

// everything a leaf starts with: whether it is left unselected by the pruning,
// its sampling key (all ones: not a candidate), no covering root, no node count
__global__ void k_leaf_init(const float* __restrict__ sig, const uint8_t* __restrict__ depth, int64_t L, float tau, int le,
                            int max_depth, uint32_t* __restrict__ u, uint64_t* __restrict__ keys,
                            int32_t* __restrict__ cover, uint32_t* __restrict__ hist_first) {
    GRID_STRIDE(l, L) {
        const float s = sig[l];
        const bool sel = selected(s, tau, le);
        u[l] = sel ? 0u : 1u;
        keys[l] = !sel && (int)depth[l] < max_depth ? (((uint64_t)(~ord32(s)) << 32) | (uint64_t)l) : ~0ull;
        cover[l] = -1;
        hist_first[l] = 0u;
    }
}

// merge roots and survivors.  all_sel[p]: no unselected leaf in [first, last].
__global__ void k_mark_merge(const int32_t* __restrict__ child, int64_t I, const int32_t* __restrict__ first,
                             const int32_t* __restrict__ last, const int32_t* __restrict__ parent,
                             const uint32_t* __restrict__ unsel, const uint32_t* __restrict__ pre_unsel,
                             int recursive, uint32_t* __restrict__ survive, uint32_t* __restrict__ root,
                             uint32_t* __restrict__ need) {
    GRID_STRIDE(p, I) {
        auto all_sel = [&](int64_t q) {
            int32_t f = first[q], l = last[q];
            return pre_unsel[l] + unsel[l] - pre_unsel[f] == 0u;
        };
        bool as = all_sel(p);
        bool r;
        if (recursive) {
            r = as && (p == 0 || !all_sel(parent[p]));
            survive[p] = as ? 0u : 1u;
            need[p] = as ? 1u : 0u;
        } else {
            bool leaves = true;
#pragma unroll
            for (int o = 0; o < 8; ++o) leaves &= child[p * 8 + o] < 0;
            r = as && leaves;
            survive[p] = r ? 0u : 1u;
            need[p] = r ? 1u : 0u;
        }
        root[p] = r ? 1u : 0u;
    }
}

// every leaf under a merge root records the root (roots' ranges are disjoint)
__global__ void k_cover(int64_t I, const uint32_t* __restrict__ root, const int32_t* __restrict__ first,
                        const int32_t* __restrict__ last, int32_t* __restrict__ cover) {
    GRID_STRIDE(p, I) {
        if (!root[p]) continue;
        for (int32_t l = first[p]; l <= last[p]; ++l) cover[l] = (int32_t)p;
    }
}

constexpr int SEL_BITS = 11, SEL_BINS = 1 << SEL_BITS;

struct SelState {
    unsigned long long prefix, mask;
    unsigned long long k_rem, k_eff;
    unsigned int done;         // the digits found so far decide every key
    unsigned int ticket;       // workgroups of the current pass that are through
    unsigned int hist[SEL_BINS];
};

// a word written by other workgroups' atomics of this launch
__device__ __forceinline__ unsigned int read_shared_word(unsigned int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One digit of the radix select: the histogram of the candidates that match the
// digits so far, then, in the last workgroup to finish, the digit holding the
// k_rem-th smallest.  When that digit's bin holds just the keys still wanted,
// every key is decided and the later passes return at once (distinct signals
// take three or four passes of six; each pass cost two launches and a serial
// walk of the bins before, 0.20 ms per selection from 3.5M keys in all).
__global__ __launch_bounds__(TPB) void k_select(const uint64_t* __restrict__ keys, int64_t L, int shift, int bits, int first,
                                                unsigned long long k_req, SelState* st) {
    __shared__ unsigned int h[SEL_BINS];
    __shared__ unsigned long long part[TPB];
    __shared__ int last;
    if (!first && st->done) return;
    const unsigned int bins = 1u << bits;
    for (unsigned int i = threadIdx.x; i < bins; i += TPB) h[i] = 0;
    __syncthreads();
    const unsigned long long prefix = st->prefix, mask = st->mask;
    GRID_STRIDE(l, L) {
        const uint64_t k = keys[l];
        if (k != ~0ull && (k & mask) == prefix) atomicAdd(&h[(k >> shift) & (bins - 1u)], 1u);
    }
    __syncthreads();
    for (unsigned int i = threadIdx.x; i < bins; i += TPB)
        if (h[i]) atomicAdd(&st->hist[i], h[i]);
    // this wave's additions are complete before the workgroup's ticket is drawn
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&st->ticket, 1u) == gridDim.x - 1u;
    __syncthreads();
    if (!last) return;
    // each thread a run of bins, the runs' sums scanned
    const unsigned int per = bins / TPB;
    unsigned long long run = 0;
    for (unsigned int i = 0; i < per; ++i) run += read_shared_word(&st->hist[threadIdx.x * per + i]);
    part[threadIdx.x] = run;
    __syncthreads();
    for (int o = 1; o < TPB; o <<= 1) {
        const unsigned long long y = (int)threadIdx.x >= o ? part[threadIdx.x - o] : 0ull;
        __syncthreads();
        part[threadIdx.x] += y;
        __syncthreads();
    }
    unsigned long long want = st->k_rem;
    if (first) want = k_req < part[TPB - 1] ? k_req : part[TPB - 1];
    const unsigned long long before = part[threadIdx.x] - run;
    __syncthreads();
    if (want == 0) {
        if (threadIdx.x == 0) {
            st->k_eff = 0;
            st->done = 1;
        }
    } else if (before < want && want <= before + run) {
        unsigned long long cum = before;
        unsigned int d = threadIdx.x * per, c = 0;
        while (cum + (c = read_shared_word(&st->hist[d])) < want) {
            cum += c;
            ++d;
        }
        unsigned long long p = prefix | ((unsigned long long)d << shift);
        if (c == want - cum) {
            p |= (1ull << shift) - 1ull;      // the whole bin
            st->done = 1;
        }
        if (first) st->k_eff = want;
        st->k_rem = want - cum;
        st->prefix = p;
        st->mask = mask | ((unsigned long long)(bins - 1u) << shift);
    }
    __syncthreads();
    for (unsigned int i = threadIdx.x; i < SEL_BINS; i += TPB) st->hist[i] = 0;
    if (threadIdx.x == 0) st->ticket = 0;
}

// new-leaf counts per old leaf, the split flags, and the deepest new leaf of
// each workgroup's part
__global__ void k_leaf_counts(int64_t L, const int32_t* __restrict__ cover, const int32_t* __restrict__ first,
                              const uint64_t* __restrict__ keys, const uint8_t* __restrict__ depth,
                              const int32_t* __restrict__ ndepth, const SelState* __restrict__ st,
                              uint32_t* __restrict__ cnt, uint32_t* __restrict__ split, uint32_t* __restrict__ deep) {
    __shared__ uint32_t part[TPB / WAVE];
    unsigned int d = 0u;
    const unsigned long long kstar = st->prefix;
    const bool any = st->k_eff > 0;
    GRID_STRIDE(l, L) {
        int32_t c = cover[l];
        bool sp = any && keys[l] != ~0ull && keys[l] <= kstar;
        split[l] = sp ? 1u : 0u;
        cnt[l] = c >= 0 ? (first[c] == (int32_t)l ? 1u : 0u) : (sp ? 8u : 1u);
        d = max(d, c >= 0 ? (unsigned int)ndepth[c] : depth[l] + (sp ? 1u : 0u));
    }
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) d = max(d, (unsigned int)__shfl_xor((int)d, o, WAVE));
    if ((threadIdx.x & (WAVE - 1)) == 0) part[threadIdx.x / WAVE] = d;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < TPB / WAVE; ++w) d = max(d, part[w]);
        deep[blockIdx.x] = d;
    }
}

__global__ void k_add_u32(uint32_t* __restrict__ a, const uint32_t* __restrict__ h, int64_t n) {
    GRID_STRIDE(i, n) a[i] += h[i];
}

__global__ void k_first_hist(int64_t I, const uint32_t* __restrict__ survive, const int32_t* __restrict__ first,
                             uint32_t* __restrict__ hist) {
    GRID_STRIDE(p, I) {
        if (survive[p]) atomicAdd(&hist[first[p]], 1u);
    }
}

// ---- rebuild ----
__global__ void k_child_internal(const int32_t* __restrict__ child, int64_t I, const uint32_t* __restrict__ survive,
                                 const int32_t* __restrict__ first, const uint32_t* __restrict__ rank_int,
                                 const uint32_t* __restrict__ rank_split, const uint32_t* __restrict__ split,
                                 const uint32_t* __restrict__ cnt_le, const uint32_t* __restrict__ nl,
                                 int32_t* __restrict__ out) {
    // a thread an entry: the entries of a node, and the leaves they name, lie together
    GRID_STRIDE(i, I * 8) {
        const int64_t p = i >> 3;
        if (!survive[p]) continue;
        const int64_t np = (int64_t)rank_int[p] + rank_split[first[p]];
        const int32_t e = child[i];
        int32_t v;
        if (e >= 0) {
            if (survive[e])
                v = (int32_t)(rank_int[e] + rank_split[first[e]]);
            else
                v = -1 - (int32_t)nl[first[e]];
        } else {
            const int64_t l = -1 - e;
            if (split[l])
                v = (int32_t)(rank_split[l] + cnt_le[l]);
            else
                v = -1 - (int32_t)nl[l];
        }
        out[np * 8 + (i & 7)] = v;
    }
}

__global__ void k_child_split(int64_t L, const uint32_t* __restrict__ split, const uint32_t* __restrict__ rank_split,
                              const uint32_t* __restrict__ cnt_le, const uint32_t* __restrict__ nl,
                              int32_t* __restrict__ out) {
    GRID_STRIDE(l, L) {
        if (!split[l]) continue;
        int64_t np = (int64_t)rank_split[l] + cnt_le[l];
#pragma unroll
        for (int o = 0; o < 8; ++o) out[np * 8 + o] = -1 - (int32_t)(nl[l] + o);
    }
}

template <int DT>
__device__ __forceinline__ double ld_elem(const void* p, int64_t i) {
    if constexpr (DT == DOT_F32)
        return (double)static_cast<const float*>(p)[i];
    else if constexpr (DT == DOT_F16)
        return (double)f16_to_f32(static_cast<const uint16_t*>(p)[i]);
    else
        return (double)bf16_to_f32(static_cast<const uint16_t*>(p)[i]);
}

// FP64 -> storage, round to nearest even, rounded once: FP32 directly; FP16 /
// BF16 through an FP32 rounded to odd (truncate, set the last bit if inexact),
// which carries enough bits that the final rounding is not a double rounding.
template <int DT>
__device__ __forceinline__ void st_elem(void* p, int64_t i, double x) {
    if constexpr (DT == DOT_F32) {
        static_cast<float*>(p)[i] = __double2float_rn(x);
    } else {
        float f = __double2float_rz(x);
        if ((double)f != x) f = __uint_as_float(__float_as_uint(f) | 1u);
        static_cast<uint16_t*>(p)[i] = DT == DOT_F16 ? f32_to_f16(f) : f32_to_bf16(f);
    }
}

// Rows move in 16-byte pieces, one thread a piece, so that a wave reads and
// writes whole lines (a thread a row touched a line per lane and instruction:
// 2.0 ms for the rows of a 3.5M-leaf tree of degree 3, 0.4 ms so).

// Values of merged nodes: the mean of the 8 children's rows (leaf rows, or node
// rows formed by the previous launch), summed pairwise in FP64 and rounded once
// to the storage type.  depth < 0: every merged node (its children are leaves);
// else those of one level, launched from the deepest up.
template <int DT>
__global__ __launch_bounds__(TPB) void k_node_values(const int32_t* __restrict__ child, int64_t I, int depth,
                                                     const int32_t* __restrict__ ndepth,
                                                     const uint32_t* __restrict__ need, int nv, int pieces,
                                                     const void* __restrict__ sig, const uint4* __restrict__ sh,
                                                     void* __restrict__ nsig, uint4* __restrict__ nsh) {
    constexpr int E = DT == DOT_F32 ? 4 : 8;      // elements per piece
    union Piece {
        uint4 v;
        float f[4];
        uint16_t h[8];
    };
    GRID_STRIDE(i, I * pieces) {
        // I <= 2^28 and at most 12 pieces a row: 32-bit division
        const int64_t p = (uint32_t)i / (uint32_t)pieces;
        const int q = (int)(i - p * pieces);
        if (!need[p] || (depth >= 0 && ndepth[p] != depth)) continue;
        int32_t e[8];
        Piece x[8], m;
#pragma unroll
        for (int o = 0; o < 8; ++o) e[o] = child[p * 8 + o];
#pragma unroll
        for (int o = 0; o < 8; ++o) x[o].v = e[o] < 0 ? sh[(int64_t)(-1 - e[o]) * pieces + q] : nsh[(int64_t)e[o] * pieces + q];
        auto mean = [&](auto at) {
            return (((at(0) + at(1)) + (at(2) + at(3))) + ((at(4) + at(5)) + (at(6) + at(7)))) * 0.125;
        };
#pragma unroll
        for (int k = 0; k < E; ++k)
            st_elem<DT>(&m, k, q * E + k < nv ? mean([&](int o) { return ld_elem<DT>(&x[o], k); }) : 0.0);
        nsh[i] = m.v;
        if (q == 0)
            st_elem<DT>(nsig, p, mean([&](int o) {
                return e[o] < 0 ? ld_elem<DT>(sig, -1 - e[o]) : ld_elem<DT>(nsig, (int64_t)e[o]);
            }));
    }
}

// where each new leaf's row comes from: an old leaf (>= 0), or merged node -1 - n
__global__ void k_sources(int64_t L, const int32_t* __restrict__ cover, const int32_t* __restrict__ first,
                          const uint32_t* __restrict__ split, const uint32_t* __restrict__ nl,
                          int32_t* __restrict__ src) {
    GRID_STRIDE(l, L) {
        const int32_t c = cover[l];
        const int64_t j = nl[l];
        if (c >= 0) {
            if (first[c] == (int32_t)l) src[j] = -1 - c;
        } else {
            const int reps = split[l] ? 8 : 1;
            for (int r = 0; r < reps; ++r) src[j + r] = (int32_t)l;
        }
    }
}

constexpr int EMIT_ROWS = 64;    // new leaves per workgroup

template <int DT>
__global__ __launch_bounds__(TPB) void k_emit_rows(int64_t L2, int pieces, int reinit, const int32_t* __restrict__ src,
                                                   const uint32_t* __restrict__ split,
                                                   const int32_t* __restrict__ ndepth,
                                                   const uint8_t* __restrict__ depth, const void* __restrict__ sig,
                                                   const uint4* __restrict__ sh, const void* __restrict__ nsig,
                                                   const uint4* __restrict__ nsh, void* __restrict__ sig2,
                                                   uint4* __restrict__ sh2, uint8_t* __restrict__ depth2) {
    const int64_t j0 = (int64_t)blockIdx.x * EMIT_ROWS;
    const int rows = (int)(L2 - j0 < EMIT_ROWS ? L2 - j0 : EMIT_ROWS);
    const uint32_t n = (uint32_t)(rows * pieces);
    uint4* out = sh2 + j0 * pieces;
#pragma unroll 4
    for (uint32_t t = threadIdx.x; t < n; t += TPB) {
        const uint32_t r = t / (uint32_t)pieces, q = t - r * (uint32_t)pieces;
        const int64_t s = src[j0 + r];
        // a leaf the refinement creates starts at zero in the ablation without fusion
        const bool fresh = reinit && (s < 0 || split[s]);
        out[t] = fresh ? make_uint4(0u, 0u, 0u, 0u) : s < 0 ? nsh[(-1 - s) * pieces + q] : sh[s * pieces + q];
    }
    for (int r = threadIdx.x; r < rows; r += TPB) {
        const int64_t j = j0 + r, s = src[j];
        const bool cut = s >= 0 && split[s];
        if (reinit && (s < 0 || cut))
            st_elem<DT>(sig2, j, 0.0);
        else
            st_elem<DT>(sig2, j, s < 0 ? ld_elem<DT>(nsig, -1 - s) : ld_elem<DT>(sig, s));
        depth2[j] = s < 0 ? (uint8_t)ndepth[-1 - s] : (uint8_t)(depth[s] + (cut ? 1 : 0));
    }
}

__global__ void k_totals(int64_t L, int64_t I, const uint32_t* __restrict__ nl, const uint32_t* __restrict__ cnt,
                         const uint32_t* __restrict__ tot_int, const uint32_t* __restrict__ tot_split,
                         const SelState* __restrict__ st, const uint32_t* __restrict__ deep, int n_deep,
                         unsigned long long* __restrict__ out) {
    uint32_t d = 0u;
    for (int i = threadIdx.x; i < n_deep; i += WAVE) d = max(d, deep[i]);
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) d = max(d, (uint32_t)__shfl_xor((int)d, o, WAVE));
    if (threadIdx.x != 0) return;
    out[0] = (unsigned long long)nl[L - 1] + cnt[L - 1];      // new leaves
    out[1] = (unsigned long long)(I > 0 ? *tot_int : 0u) + *tot_split;  // new internal nodes
    out[2] = (unsigned long long)(I > 0 ? (uint64_t)I - *tot_int : 0u);  // merged nodes
    out[3] = st->k_eff;
    out[4] = d;
}

// RAII list of temporaries from the tree's allocator
struct Temps {
    const Alloc& al;
    std::vector<void*> ps;
    bool ok = true;
    explicit Temps(const Alloc& a) : al(a) {}
    template <class T>
    T* get(int64_t n) {
        void* p = al.get((size_t)(n < 1 ? 1 : n) * sizeof(T));
        if (!p) ok = false;
        ps.push_back(p);
        return static_cast<T*>(p);
    }
    // give one back early
    template <class T>
    void put(T*& p) {
        for (void*& q : ps)
            if (q == p) {
                al.put(q);
                q = nullptr;
            }
        p = nullptr;
    }
    ~Temps() {
        for (void* p : ps) al.put(p);
    }
};

template <int DT>
hipError_t launch_values_emit(const dot_tree& t, int64_t L2, int64_t I, int nv, const dot_refine_params& p,
                              const int32_t* ndepth, const uint32_t* need, const uint32_t* split, const int32_t* src,
                              void* nsig, void* nsh, void* sig2, void* sh2, uint8_t* depth2, hipStream_t s) {
    const int pieces = t.sh_stride * storage_bytes(t.storage) / 16;
    const uint4* sh = static_cast<const uint4*>(t.sh);
    uint4* vsh = static_cast<uint4*>(nsh);
    auto values = [&](int depth) {
        hipLaunchKernelGGL(k_node_values<DT>, dim3(blocks_for(I * pieces)), dim3(TPB), 0, s, t.child, I, depth, ndepth,
                           need, nv, pieces, t.sigma, sh, nsig, vsh);
    };
    if (I > 0 && !p.reinit) {
        if (p.recursive)
            for (int d = std::min(t.max_depth, DOT_MAX_DEPTH) - 1; d >= 0; --d) values(d);
        else
            values(-1);
    }
    hipLaunchKernelGGL(k_emit_rows<DT>, dim3((unsigned)((L2 + EMIT_ROWS - 1) / EMIT_ROWS)), dim3(TPB), 0, s, L2, pieces,
                       p.reinit, src, split, ndepth, t.leaf_depth, t.sigma, sh, nsig, vsh, sig2,
                       static_cast<uint4*>(sh2), depth2);
    return hipGetLastError();
}

}  // namespace

int refine_tree(dot_tree& t, const float* signal, const dot_refine_params& p, dot_refine_stats* st_out,
                hipStream_t s) {
    const int64_t L = t.n_leaves, I = t.n_internal;
    const int64_t k_req = (int64_t)std::floor((double)p.sample_frac * (double)L);
    if (L + 7 * k_req > (int64_t)INT32_MAX || I + k_req > (int64_t)INT32_MAX / 8)
        return fail(DOT_EINVAL, "dot_refine: the refined tree would exceed 32-bit indices");
    const int nv = 3 * (t.degree + 1) * (t.degree + 1);
    const int stride = t.sh_stride;
    const int es = storage_bytes(t.storage);
    const int rec = p.recursive ? 1 : 0;

    Temps tmp(t.alloc);
    int32_t* first = tmp.get<int32_t>(I);
    int32_t* last = tmp.get<int32_t>(I);
    int32_t* ndepth = tmp.get<int32_t>(I);
    int32_t* parent = tmp.get<int32_t>(I);
    uint32_t* survive = tmp.get<uint32_t>(I);
    uint32_t* root = tmp.get<uint32_t>(I);
    uint32_t* need = tmp.get<uint32_t>(I);
    uint32_t* rank_int = tmp.get<uint32_t>(I);
    void* nsh = tmp.get<unsigned char>(std::max<int64_t>(I, 1) * stride * es);
    void* nsig = tmp.get<unsigned char>(std::max<int64_t>(I, 1) * es);
    uint32_t* unsel = tmp.get<uint32_t>(L);
    uint32_t* pre_unsel = tmp.get<uint32_t>(L);
    int32_t* cover = tmp.get<int32_t>(L);
    uint64_t* keys = tmp.get<uint64_t>(L);
    SelState* sel = tmp.get<SelState>(1);
    uint32_t* cnt = tmp.get<uint32_t>(L);
    uint32_t* split = tmp.get<uint32_t>(L);
    uint32_t* nl = tmp.get<uint32_t>(L);
    uint32_t* rank_split = tmp.get<uint32_t>(L);
    uint32_t* hist_first = tmp.get<uint32_t>(L);
    uint32_t* cnt_le = tmp.get<uint32_t>(L);
    uint32_t* bsum = tmp.get<uint32_t>(scan_scratch_elems(std::max(L, I)));
    uint32_t* tots = tmp.get<uint32_t>(8);
    constexpr int kDeepMax = 1024;
    uint32_t* deep = tmp.get<uint32_t>(kDeepMax);
    unsigned long long* totals = tmp.get<unsigned long long>(5);
    if (!tmp.ok) return fail(DOT_ENOMEM, "dot_refine: scratch allocation failed");

    // 1. tree metadata, merge marks, candidate keys
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(TPB), 0, s, tots, (int64_t)8, 0u);
    hipLaunchKernelGGL(k_leaf_init, dim3(blocks_for(L)), dim3(TPB), 0, s, signal, t.leaf_depth, L, p.prune_tau, p.prune_le,
                       p.max_depth, unsel, keys, cover, hist_first);
    hipError_t e = scan_u32(unsel, pre_unsel, L, bsum, &tots[4], s);
    if (e != hipSuccess) return hip_fail(e, "dot_refine: scan");
    if (I > 0) {
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(TPB), 0, s, reinterpret_cast<uint32_t*>(parent), (int64_t)1,
                           0xffffffffu);
        hipLaunchKernelGGL(k_node_parent, dim3(blocks_for(I * 8)), dim3(TPB), 0, s, t.child, I, parent);
        hipLaunchKernelGGL(k_node_meta, dim3(blocks_for(I)), dim3(TPB), 0, s, t.child, I, t.leaf_depth, first, last,
                           ndepth);
        hipLaunchKernelGGL(k_mark_merge, dim3(blocks_for(I)), dim3(TPB), 0, s, t.child, I, first, last, parent, unsel,
                           pre_unsel, rec, survive, root, need);
        hipLaunchKernelGGL(k_cover, dim3(blocks_for(I)), dim3(TPB), 0, s, I, root, first, last, cover);
    }
    // 2. exact top-k by radix select over the 64-bit keys: three digits of the
    // signal's 32 bits, three of the index
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(TPB), 0, s, reinterpret_cast<uint32_t*>(sel),
                       (int64_t)(sizeof(SelState) / 4), 0u);
    if (k_req > 0) {
        const unsigned g = (unsigned)std::min<int64_t>(blocks_for(L, 16), 1024);
        const int bits[6] = {11, 11, 10, 11, 11, 10};
        for (int pass = 0, shift = 64; pass < 6; ++pass) {
            shift -= bits[pass];
            hipLaunchKernelGGL(k_select, dim3(g), dim3(TPB), 0, s, keys, L, shift, bits[pass], pass == 0 ? 1 : 0,
                               (unsigned long long)k_req, sel);
        }
    }
    // 3. counts and scans
    const int n_deep = (int)std::min<int64_t>(blocks_for(L, 2), kDeepMax);
    hipLaunchKernelGGL(k_leaf_counts, dim3(n_deep), dim3(TPB), 0, s, L, cover, first, keys, t.leaf_depth, ndepth, sel, cnt,
                       split, deep);
    if (I > 0) hipLaunchKernelGGL(k_first_hist, dim3(blocks_for(I)), dim3(TPB), 0, s, I, survive, first, hist_first);
    e = scan_u32(cnt, nl, L, bsum, &tots[0], s);
    if (e == hipSuccess) e = scan_u32(split, rank_split, L, bsum, &tots[1], s);
    if (e == hipSuccess) e = scan_u32(hist_first, cnt_le, L, bsum, &tots[2], s);
    if (e == hipSuccess && I > 0) e = scan_u32(survive, rank_int, I, bsum, &tots[3], s);
    if (e != hipSuccess) return hip_fail(e, "dot_refine: scans");
    // cnt_le becomes inclusive: surviving nodes whose first leaf is <= l
    hipLaunchKernelGGL(k_add_u32, dim3(blocks_for(L)), dim3(TPB), 0, s, cnt_le, (const uint32_t*)hist_first, L);
    hipLaunchKernelGGL(k_totals, dim3(1), dim3(64), 0, s, L, I, nl, cnt, &tots[3], &tots[1], sel,
                       deep, n_deep, totals);
    unsigned long long h_tot[5];
    e = hipMemcpyAsync(h_tot, totals, sizeof(h_tot), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "dot_refine: sizes");
    const int64_t L2 = (int64_t)h_tot[0], I2 = (int64_t)h_tot[1];

    // 4. new planes; what only the counts needed goes back first, which makes room
    // for the list of sources (4 B per new leaf; 24 B per old leaf go back)
    tmp.put(keys);
    tmp.put(unsel);
    tmp.put(pre_unsel);
    tmp.put(cnt);
    tmp.put(hist_first);
    int32_t* child2 = static_cast<int32_t*>(t.alloc.get((size_t)std::max<int64_t>(I2, 1) * 32));
    void* sig2 = t.alloc.get((size_t)L2 * es);
    void* sh2 = t.alloc.get((size_t)L2 * stride * es);
    uint8_t* depth2 = static_cast<uint8_t*>(t.alloc.get((size_t)L2));
    int32_t* src = tmp.get<int32_t>(L2);
    auto drop_new = [&]() {
        t.alloc.put(child2);
        t.alloc.put(sig2);
        t.alloc.put(sh2);
        t.alloc.put(depth2);
    };
    if (!child2 || !sig2 || !sh2 || !depth2 || !src) {
        drop_new();
        return fail(DOT_ENOMEM, "dot_refine: allocation of the refined planes failed");
    }
    if (I > 0)
        hipLaunchKernelGGL(k_child_internal, dim3(blocks_for(I * 8)), dim3(TPB), 0, s, t.child, I, survive, first,
                           rank_int, rank_split, split, cnt_le, nl, child2);
    hipLaunchKernelGGL(k_child_split, dim3(blocks_for(L)), dim3(TPB), 0, s, L, split, rank_split, cnt_le, nl, child2);
    hipLaunchKernelGGL(k_sources, dim3(blocks_for(L)), dim3(TPB), 0, s, L, cover, first, split, nl, src);
    auto emit = [&](auto launch) {
        return launch(t, L2, I, nv, p, ndepth, need, split, src, nsig, nsh, sig2, sh2, depth2, s);
    };
    e = t.storage == DOT_F32   ? emit(launch_values_emit<DOT_F32>)
        : t.storage == DOT_F16 ? emit(launch_values_emit<DOT_F16>)
                               : emit(launch_values_emit<DOT_BF16>);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        drop_new();
        return hip_fail(e, "dot_refine: rebuild");
    }
    // 5. swap into the handle
    t.alloc.put(t.child);
    t.alloc.put(t.sigma);
    t.alloc.put(t.sh);
    t.alloc.put(t.leaf_depth);
    t.child = child2;
    t.sigma = sig2;
    t.sh = sh2;
    t.leaf_depth = depth2;
    t.n_leaves = L2;
    t.n_internal = I2;
    t.max_depth = (int32_t)h_tot[4];   // bounds the walk's steps and the levels of the links
    if (st_out) {
        st_out->leaves_before = L;
        st_out->leaves_after = L2;
        st_out->internal_after = I2;
        st_out->merged = (int64_t)h_tot[2];
        st_out->subdivided = (int64_t)h_tot[3];
    }
    // the old links described the old topology; without new ones the tree is
    // still complete and walks by re-descent
    return update_links(t, s);
}

}  // namespace dot
