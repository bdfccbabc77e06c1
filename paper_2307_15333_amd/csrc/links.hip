// Face-neighbour links of the leaves (see LINK_* in dot_internal.h), built
// top-down one level per launch.  A node's links are derived from its
// parent's: across a face that stays inside the parent the neighbour is the
// sibling; across a face of the parent the neighbour is the child (mirrored
// octant) of the parent's neighbour when that is an internal node, and the
// parent's neighbour itself, one level further up, when that is a leaf or the
// outside.  Each launch passes over all nodes in their own (depth-first) order
// and takes those of its level, so that neighbours in space, whose entries a
// wave reads, are neighbours in memory; the depths it passes on are the next
// launch's level.  (A list of each level's nodes, in the order an atomic gave
// them, read them scattered: 0.46 ms for 3.5M leaves, 0.23 ms so.)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dot_internal.h"

namespace dot {

namespace {

constexpr int TPB = 256;

__device__ __forceinline__ uint32_t link_of(int32_t entry, uint32_t up) {
    return entry >= 0 ? (uint32_t)entry : (LINK_LEAF | (up << LINK_ID_BITS) | (uint32_t)(-1 - entry));
}

// the root's faces are the boundary; every other depth is unknown yet
__global__ void k_links_init(uint32_t* __restrict__ nlinks, uint32_t* __restrict__ depth4, int64_t words) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < 6) nlinks[i] = LINK_OUT;
    for (int64_t w = i; w < words; w += (int64_t)gridDim.x * blockDim.x) depth4[w] = w == 0 ? 0xffffff00u : 0xffffffffu;
}

// one thread per (node, octant)
__global__ __launch_bounds__(TPB) void k_links_level(const int32_t* __restrict__ child, int64_t I, int level,
                                                     uint8_t* __restrict__ depth, uint32_t* __restrict__ nlinks,
                                                     uint32_t* __restrict__ links) {
    for (int64_t i = blockIdx.x * (int64_t)TPB + threadIdx.x; i < I * 8; i += (int64_t)gridDim.x * TPB) {
        const int64_t node = i >> 3;
        if (depth[node] != level) continue;
        const int o = (int)(i & 7);
        const int32_t e = child[i];
        uint32_t r[6];
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const int a = f >> 1, up = f & 1;
            const int m = o ^ (1 << a);           // octant across the face
            if (((o >> a) & 1) != up) {
                r[f] = link_of(child[node * 8 + m], 0u);   // sibling
            } else {
                const uint32_t q = nlinks[node * 6 + f];
                if (q == LINK_OUT)
                    r[f] = LINK_OUT;
                else if (q & LINK_LEAF)
                    r[f] = q + (1u << LINK_ID_BITS);       // the same leaf, one more level up
                else
                    r[f] = link_of(child[(int64_t)q * 8 + m], 0u);
            }
        }
        uint32_t* dst;
        if (e >= 0) {
            dst = nlinks + (int64_t)e * 6;
            depth[e] = (uint8_t)(level + 1);
        } else {
            dst = links + (int64_t)(-1 - e) * 6;
        }
        uint2* d2 = reinterpret_cast<uint2*>(dst);
        d2[0] = make_uint2(r[0], r[1]);
        d2[1] = make_uint2(r[2], r[3]);
        d2[2] = make_uint2(r[4], r[5]);
    }
}

}  // namespace

int update_links(dot_tree& t, hipStream_t s) {
    t.alloc.put(t.links);
    t.links = nullptr;
    if (!t.links_on || t.n_internal == 0 || t.n_leaves > LINK_MAX_LEAVES) return DOT_OK;
    const int64_t L = t.n_leaves, I = t.n_internal;
    uint32_t* links = static_cast<uint32_t*>(t.alloc.get((size_t)L * 6 * sizeof(uint32_t)));
    // scratch: links and depths of the internal nodes
    const int64_t words = (I + 3) / 4;
    const size_t scratch_bytes = (size_t)I * 6 * 4 + (size_t)words * 4;
    char* scratch = static_cast<char*>(t.alloc.get(scratch_bytes));
    if (!links || !scratch) {
        t.alloc.put(links);
        t.alloc.put(scratch);
        return fail(DOT_ENOMEM, "neighbour links: device allocation failed");
    }
    uint32_t* nlinks = reinterpret_cast<uint32_t*>(scratch);
    uint32_t* depth4 = nlinks + I * 6;
    hipLaunchKernelGGL(k_links_init, dim3((unsigned)std::min<int64_t>((words + TPB - 1) / TPB, 1024)), dim3(TPB), 0, s,
                       nlinks, depth4, words);
    // the deepest internal node is at depth max_depth - 1
    const int levels = std::min(std::max(t.max_depth, 1), DOT_MAX_DEPTH);
    const unsigned grid = (unsigned)std::min<int64_t>((I * 8 + TPB - 1) / TPB, 1 << 20);
    for (int d = 0; d < levels; ++d)
        hipLaunchKernelGGL(k_links_level, dim3(grid), dim3(TPB), 0, s, t.child, I, d, reinterpret_cast<uint8_t*>(depth4),
                           nlinks, links);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    t.alloc.put(scratch);
    if (e != hipSuccess) {
        t.alloc.put(links);
        return hip_fail(e, "neighbour links: build");
    }
    t.links = links;
    return DOT_OK;
}

}  // namespace dot
