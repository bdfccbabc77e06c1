// The forward walk: 64 rays of a wave step through the tree together, so that
// the lanes of a quad can fetch their leaves' rows for each other.
//
// What bounds it: the per-CU vector-memory address path (one cache-line lookup
// a cycle) and, where few waves are resident, the dependent chain link -> child
// -> leaf.  Hence
//  - every plane is read through a buffer descriptor: a lane that has nothing
//    to fetch passes an offset past the end, which costs no lookup and no
//    branch (so the loads of a step are issued unconditionally and can be
//    waited for one by one), and addresses are 32-bit;
//  - FP32 rows of degree 3 (12 pieces of 16 B) are fetched by quads: the four
//    lanes read 64 B of one leaf's row per instruction, one lookup instead of
//    one per lane, and each lane multiplies the four coefficients it gets of
//    each of the quad's four leaves with the same four basis functions of the
//    ray they belong to; two exchange steps inside the quad add the parts up;
//  - the next leaf is found (link, child descent) while the current leaf's row
//    is in flight, and the row is used after that; the geometry is free of
//    branches, and what it needs is not held across the row's flight.
// Measured against the lane-by-lane walk (traverse), same images, one MI355X:
// 8 random 800x800 views of 3.5M FP32 leaves of degree 3 1.68 -> 1.30 ms (cache
// lookups per launch 7.6e8 -> 4.3e8), a 64x64 view of 8.6k leaves 47 -> 26 us, a
// 333x217 view of 0.87M BF16 leaves 113 -> 68 us, a 1920x1080 view of 3.5M FP16
// leaves 648 -> 526 us.
#pragma once

#include "dot_device.h"

namespace dot {

using Rsrc = __amdgpu_buffer_rsrc_t;

// offset that no plane reaches (adding a row's immediate offsets does not wrap)
constexpr uint32_t OFF_NONE = 0xfffff000u;

__device__ __forceinline__ Rsrc plane_rsrc(const void* p, uint64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)(uint32_t)bytes, 0x00020000);
}

// waves per SIMD that the forward kernels are held to: as many as their registers
// allow without spills in the walk.  8 views of 800x800, us at 4 / 5 / 6 waves: FP32 of
// degree 3 1240 / 2500 / -, of degree 2 580 / 595 / -, FP16 965 / 945 / 1367, BF16
// 975 / 1012 / 1564, palette 901 / 897 / 1290 (degree 3 all); the rest is within 2 % at
// 3 to 6.
constexpr int fwd_waves(int dt, int deg) {
    if (deg <= 1) return 6;
    return dt == DOT_F32 || (dt == DOT_BF16 && deg == 3) ? 4 : 5;
}

template <int CTRL>
__device__ __forceinline__ int quad_i(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float quad_f(float v) {
    return __int_as_float(quad_i<CTRL>(__float_as_int(v)));
}
constexpr int QUAD_XOR1 = 0xb1, QUAD_XOR2 = 0x4e;    // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int quad_lane(int r) { return r * 0x55; }  // quad_perm [r,r,r,r]

// 3 x in one instruction (a 32-bit product takes a quarter-rate one)
__device__ __forceinline__ uint32_t times3(int x) {
    uint32_t r;
    asm("v_lshl_add_u32 %0, %1, 1, %1" : "=v"(r) : "v"(x));
    return r;
}

// Contributing segments of a training forward wait here for STAGE_STEPS steps of
// the wave: [step][thread], leaf (or -2 - leaf beyond the record capacity, -1:
// none), delta, tau and the colour.
constexpr int STAGE_STEPS = 4;
struct Stage {
    float4 a[STAGE_STEPS][BLOCK];
    float2 b[STAGE_STEPS][BLOCK];
};

// The ray's compositing state (see FwdSeg, which computes the same per lane).
// COLOUR = false: the weights alone (the signal pass), which need no row: 16
// views of 800x800 over 3.5M FP32 leaves 3.11 -> 1.43 ms.  SIGNAL: none, the largest
// weight of a leaf or the sum of its weights; in instantiations of their own, since the
// registers of the sums cost the other forms 3 to 6 %, and those of the maximum a 64x64
// view of FP16 leaves 55 us instead of 50.
enum { SIGNAL_NONE = 0, SIGNAL_MAX = 1, SIGNAL_SUM = 2 };
template <int DT, int DEG, bool COUNT = false, bool COLOUR = true, int SIGNAL = SIGNAL_NONE>
struct FwdWave {
    static constexpr int K = (DEG + 1) * (DEG + 1);
    static constexpr bool QUAD = DT == DOT_F32 && DEG == 3;
    static constexpr int ES = DT == DOT_F32 ? 4 : 2;
    static constexpr int RDT = DT == DOT_PAL16 ? DOT_F16 : DT;
    static constexpr int ROW_BYTES = row_stride<RDT>(3 * K) * ES;
    static constexpr int PIECES = ROW_BYTES / 16;
    using Piece = uint32_t __attribute__((ext_vector_type(4)));

    const TreeView& tv;
    const FwdArgs& a;
    Rsrc r_sigma, r_sh;
    float Y[K];       // QUAD: Y[4 r + j] = basis function 4 q + j of the ray of quad lane r (q: this lane)
    float S = 0.f, T = 1.f;
    float C[3] = {0.f, 0.f, 0.f};
    int n = 0;
    int fetched = 0;
    int64_t rid = 0;    // COUNT: the ray's index in the batch (record column)
    int nrec = 0;       // COUNT: composited segments recorded so far
    Stage* stage = nullptr;   // COUNT
    int staged = 0;           // COUNT: steps waiting in it (the same in all lanes)

    // a segment's data in flight
    struct Fetch {
        float sg, cur;
        Piece row[!COLOUR ? 1 : QUAD ? 12 : PIECES];
    };

    __device__ __forceinline__ FwdWave(const TreeView& tv_, const FwdArgs& a_) : tv(tv_), a(a_) {
        r_sigma = plane_rsrc(tv.sigma, (uint64_t)tv.n_leaves * ES);
        if constexpr (DT == DOT_PAL16)
            r_sh = plane_rsrc(tv.sh, (uint64_t)tv.n_leaves * 2);
        else
            r_sh = plane_rsrc(tv.sh, (uint64_t)tv.n_leaves * ROW_BYTES);
    }

    __device__ __forceinline__ void begin(const Ray& r) {
        if constexpr (!COLOUR) return;
        float B[K];
        sh_basis<DEG>((float)r.dx, (float)r.dy, (float)r.dz, B);
        if constexpr (QUAD) {
            const int q = threadIdx.x & 3;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float v[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) v[p] = B[4 * p + j];
                auto pick = [&](float x0, float x1, float x2, float x3) {
                    const float lo = (q & 1) ? x1 : x0, hi = (q & 1) ? x3 : x2;
                    return (q & 2) ? hi : lo;
                };
                Y[0 + j] = pick(quad_f<quad_lane(0)>(v[0]), quad_f<quad_lane(0)>(v[1]), quad_f<quad_lane(0)>(v[2]), quad_f<quad_lane(0)>(v[3]));
                Y[4 + j] = pick(quad_f<quad_lane(1)>(v[0]), quad_f<quad_lane(1)>(v[1]), quad_f<quad_lane(1)>(v[2]), quad_f<quad_lane(1)>(v[3]));
                Y[8 + j] = pick(quad_f<quad_lane(2)>(v[0]), quad_f<quad_lane(2)>(v[1]), quad_f<quad_lane(2)>(v[2]), quad_f<quad_lane(2)>(v[3]));
                Y[12 + j] = pick(quad_f<quad_lane(3)>(v[0]), quad_f<quad_lane(3)>(v[1]), quad_f<quad_lane(3)>(v[2]), quad_f<quad_lane(3)>(v[3]));
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) Y[k] = B[k];
        }
    }

    // The run of neighbouring lanes with this lane's key: its first lane, and the
    // first lane behind it.
    __device__ __forceinline__ static void run_of(int key, int& head, int& end) {
        const int lane = (int)__lane_id();
        const int prev = __builtin_amdgcn_update_dpp(~key, key, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
        const uint64_t heads = __ballot(key != prev);
        const uint64_t le = 2ull * (1ull << lane) - 1ull;        // lanes up to this one
        head = 63 - __builtin_clzll(heads & le);
        const uint64_t above = heads & ~le;
        end = above ? __builtin_ctzll(above) : WAVE;
    }

    // One counting atomic for each run of neighbouring lanes in the same leaf (the
    // device completes 15 to 27 G counting atomics a second; lanes next to each
    // other are neighbouring pixels).  key as in Stage; returns the slot of this
    // lane's segment relative to `base`, which the run's first lane holds.
    __device__ __forceinline__ int count_run(int key, uint32_t& base) const {
        const int lane = (int)__lane_id();
        int head, end;
        run_of(key, head, end);
        base = 0;
        if (head == lane && key != -1) {
            if (key >= 0)
                base = atomicAdd(&a.leaf_count[key], (uint32_t)(end - lane));
            else
                atomicAdd(&a.leaf_rest[-2 - key], (uint32_t)(end - lane));
        }
        return lane - head;
    }

    // A signal that sums: the weights of a run of lanes in one leaf are added up
    // first, one float addition in memory for each run.  Called by all lanes of the
    // wave.  Additions to one leaf queue up in memory, the more the faster the walk
    // issues them; an 800x800 view of 205k leaves, the signal alone: 3.4 ms with the
    // lane-by-lane walk and an addition a lane, 4.0 with this walk, 0.44 so.
    __device__ __forceinline__ void add_signal(int leaf, float w, bool in) const {
        const int key = in ? leaf : -1, lane = (int)__lane_id();
        int head, end;
        run_of(key, head, end);
        float v = in ? w : 0.f;
        for (int s = 1; __any(lane + s < end); s <<= 1) {
            const float x = __shfl_down(v, s, WAVE);
            if (lane + s < end) v += x;
        }
        if (in && head == lane) unsafeAtomicAdd(&a.signal[leaf], v);
    }

    // Count and record the staged steps: per leaf the segments whose gradient rows
    // the adjoint emits, each recorded one with the slot of its row in the leaf's
    // bucket.  A ray's records lie in groups of four, so writing several steps
    // together fills a group's lines while the L2 still holds them, and the atomics
    // of those steps are in flight together (forward of 2^20 cell-ordered rays of
    // 3.5M leaves, four waves a SIMD: 1468 us when every step writes and counts by
    // itself, 1348 so).
    // Called by all lanes of the wave.
    __device__ __forceinline__ void flush() {
        if constexpr (COUNT) {
            if (staged == 0) return;
            const int tid = threadIdx.x;
            int key[STAGE_STEPS], rank[STAGE_STEPS], n_key = 0;
            uint32_t base[STAGE_STEPS];
#pragma unroll
            for (int j = 0; j < STAGE_STEPS; ++j) {
                key[j] = j < staged ? __float_as_int(stage->a[j][tid].x) : -1;
                n_key += key[j] != -1;
            }
#pragma unroll
            for (int j = 0; j < STAGE_STEPS; ++j) rank[j] = count_run(key[j], base[j]);
            if (a.rec.a) {
                int at = nrec - n_key;
#pragma unroll
                for (int j = 0; j < STAGE_STEPS; ++j) {
                    if (key[j] >= 0) {
                        const int64_t i = a.rec.at(at, rid);
                        a.rec.a[i] = stage->a[j][tid];
                        a.rec.b[i] = stage->b[j][tid];
                    }
                    at += key[j] != -1;
                }
                at = nrec - n_key;
#pragma unroll
                for (int j = 0; j < STAGE_STEPS; ++j) {
                    const int head = (int)__lane_id() - rank[j];
                    const uint32_t b = (uint32_t)__builtin_amdgcn_ds_bpermute(head << 2, (int)base[j]);
                    if (key[j] >= 0) a.rec.slot[a.rec.at(at, rid)] = b + (uint32_t)rank[j];
                    at += key[j] != -1;
                }
            }
            staged = 0;
        }
    }

    template <int R>
    __device__ __forceinline__ void fetch_quad(uint32_t off, Fetch& f) {
        const uint32_t o = (uint32_t)quad_i<quad_lane(R)>((int)off) + (threadIdx.x & 3) * 16u;
#pragma unroll
        for (int c = 0; c < 3; ++c) f.row[3 * R + c] = __builtin_amdgcn_raw_buffer_load_b128(r_sh, o + 64u * c, 0, 0);
    }

    // byte offset of a leaf's row (times3 where the row is 3 2^n bytes)
    __device__ __forceinline__ uint32_t row_off(int leaf) const {
        constexpr int P = ROW_BYTES / 3;
        if constexpr (ROW_BYTES % 3 == 0 && (P & (P - 1)) == 0)
            return times3(leaf) * (uint32_t)P;
        else
            return (uint32_t)leaf * (uint32_t)ROW_BYTES;
    }

    // the stored signal, read for the max filter, in = false: nothing
    __device__ __forceinline__ void fetch_signal(int leaf, bool in, Fetch& f) {
        if constexpr (SIGNAL == SIGNAL_MAX) {
            const Rsrc rs = plane_rsrc(a.signal, (uint64_t)tv.n_leaves * 4);
            f.cur = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, in ? (uint32_t)leaf * 4u : OFF_NONE, 0, 0));
        }
    }

    // request the data of `leaf` (in = false: nothing)
    __device__ __forceinline__ void fetch(int leaf, bool in, Fetch& f) {
        const uint32_t so = in ? (uint32_t)leaf * ES : OFF_NONE;
        if constexpr (DT == DOT_F32)
            f.sg = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r_sigma, so, 0, 0));
        else {
            const uint32_t h = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r_sigma, so, 0, 0);
            f.sg = DT == DOT_BF16 ? bf16_to_f32(h) : f16_to_f32(h);
        }
        if constexpr (!COLOUR) {
        } else if constexpr (QUAD) {
            const uint32_t ro = row_off(leaf), off = in ? ro : OFF_NONE;
            fetch_quad<0>(off, f);
            fetch_quad<1>(off, f);
            fetch_quad<2>(off, f);
            fetch_quad<3>(off, f);
        } else {
            uint32_t off;
            Rsrc rr = r_sh;
            if constexpr (DT == DOT_PAL16) {
                // the row lives in the palette: one dependent load after the index
                const uint32_t pi = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r_sh, so, 0, 0);
                rr = plane_rsrc(tv.palette, (uint64_t)65536 * ROW_BYTES);
                const uint32_t ro = row_off((int)pi);
                off = in ? ro : OFF_NONE;
            } else {
                const uint32_t ro = row_off(leaf);
                off = in ? ro : OFF_NONE;
            }
#pragma unroll
            for (int c = 0; c < PIECES; ++c) f.row[c] = __builtin_amdgcn_raw_buffer_load_b128(rr, off + 16u * c, 0, 0);
        }
    }

    __device__ __forceinline__ float coef(const Fetch& f, int i) const {
        if constexpr (DT == DOT_F32) {
            return __uint_as_float(f.row[i >> 2][i & 3]);
        } else {
            const uint32_t w = f.row[i >> 3][(i >> 1) & 3];
            if constexpr (RDT == DOT_BF16) return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
            return f16_to_f32((i & 1) ? (w >> 16) : (w & 0xffffu));
        }
    }

    // sum_k sh[ch][k] Y_k for the three channels; QUAD: all lanes of the quad take part
    __device__ __forceinline__ void dots(const Fetch& f, float (&x)[3]) const {
        if constexpr (QUAD) {
            const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                float p[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const Piece v = f.row[3 * r + ch];
                    p[r] = __uint_as_float(v[0]) * Y[4 * r];
#pragma unroll
                    for (int j = 1; j < 4; ++j) p[r] = fmaf(__uint_as_float(v[j]), Y[4 * r + j], p[r]);
                }
                // keep the rays of this lane's parity, hand the others over; then the pair of its half
                const float s0 = (b0 ? p[1] : p[0]) + quad_f<QUAD_XOR1>(b0 ? p[0] : p[1]);
                const float s1 = (b0 ? p[3] : p[2]) + quad_f<QUAD_XOR1>(b0 ? p[2] : p[3]);
                x[ch] = (b1 ? s1 : s0) + quad_f<QUAD_XOR2>(b1 ? s0 : s1);
            }
        } else {
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) x[ch] = sh_dot<DT, DEG>([&](int k) { return coef(f, ch * K + k); }, Y);
        }
    }

    // composite the segment (in: this lane has one); false when the ray stops.
    // Called by all lanes of the wave.
    __device__ __forceinline__ bool shade(int leaf, float delta, bool in, const Fetch& f) {
        float x[3], cv[3] = {0.f, 0.f, 0.f};
        [[maybe_unused]] float ws = 0.f;
        if constexpr (COLOUR) dots(f, x);
        const float sg = fmaxf(f.sg, 0.f);
        const float tau = sg * delta;
        if (in) {
            ++n;
            fetched += tau > 0.f;
            const float Sn = S + tau;
            const float Tn = __expf(-Sn);
            const float w = fmaxf(T - Tn, 0.f);
            if constexpr (COLOUR) {
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) {
                    cv[ch] = sigmoidf_(x[ch]);
                    C[ch] = fmaf(w, cv[ch], C[ch]);
                }
            }
            if constexpr (SIGNAL == SIGNAL_SUM) ws = w;
            if constexpr (SIGNAL == SIGNAL_MAX) {
                // non-negative floats order like their bit patterns; skip the
                // atomic when the stored value already dominates
                if (w > f.cur) atomicMax(reinterpret_cast<unsigned int*>(&a.signal[leaf]), __float_as_uint(w));
            }
            S = Sn;
            T = Tn;
        }
        if constexpr (SIGNAL == SIGNAL_SUM) add_signal(leaf, ws, in);
        if constexpr (COUNT) {
            const bool counted = in && sg > 0.f;
            if (__any(counted)) {
                const bool record = counted && a.rec.a && nrec < a.rec.cap;
                const int key = record ? leaf : counted ? -2 - leaf : -1;
                stage->a[staged][threadIdx.x] = make_float4(__int_as_float(key), delta, tau, cv[0]);
                stage->b[staged][threadIdx.x] = make_float2(cv[1], cv[2]);
                nrec += counted && a.rec.a;
                if (++staged == STAGE_STEPS) flush();
            }
        }
        return !in || !(S > a.thr);
    }
};

__device__ __forceinline__ int med3(int x, int lo, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo), "v"(hi));
    return r;
}

// v_min_f64 / v_max_f64 as they are (fmin and fmax quiet their operands first)
__device__ __forceinline__ double min_f64(double x, double y) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}
__device__ __forceinline__ double max_f64(double x, double y) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}

// traverse() for FwdWave: called by all 64 lanes of the wave (live = false: a
// lane without a ray).  The same leaves, lengths and read counts as traverse().
template <bool LINKED, class Seg>
__device__ __forceinline__ void walk_fwd(const TreeView& tv, const Ray& r, bool live, int* __restrict__ stk, Seg& seg,
                                         int& desc) {
    const double LF = (double)LAT_N;
    const double sc = (double)tv.scale;
    double O[3] = {(r.ox - (double)tv.bmin[0]) * sc, (r.oy - (double)tv.bmin[1]) * sc, (r.oz - (double)tv.bmin[2]) * sc};
    double D[3] = {r.dx * sc + 0.0, r.dy * sc + 0.0, r.dz * sc + 0.0};    // no -0
    double inv[3];
    double t0 = 0.0, t1 = __builtin_huge_val();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // no direction (a zero vector, a broken camera): as in traverse, never left
        // along this axis, from its first cell.  Such a ray ends in its first leaf
        // with a NaN colour (its basis is NaN)
        const bool has = D[a] == D[a];
        D[a] = has ? D[a] : 0.0;
        O[a] = has ? O[a] : 0.0;
        if (D[a] != 0.0) {
            inv[a] = 1.0 / D[a];
            const double p = (0.0 - O[a]) * inv[a], q = (LF - O[a]) * inv[a];
            t0 = fmax(t0, fmin(p, q));
            t1 = fmin(t1, fmax(p, q));
        } else {
            inv[a] = __builtin_huge_val();
            if (O[a] < 0.0 || O[a] > LF) live = false;
        }
    }
    if (!(t0 < t1)) live = false;
    // re-origin at the entry point: positions O + s D for s in [0, t1 - t0]
#pragma unroll
    for (int a = 0; a < 3; ++a) O[a] = fma(t0, D[a], O[a]);
    const double s1 = t1 - t0;
    int c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) c[a] = min(max((int)floor(O[a]), 0), LAT_N - 1);
    // -1 on an axis the ray walks towards smaller coordinates (its exit plane is the near one), else 0
    const int back[3] = {D[0] < 0.0 ? -1 : 0, D[1] < 0.0 ? -1 : 0, D[2] < 0.0 ? -1 : 0};
    const uint32_t face0 = D[0] < 0.0 ? 0u : 4u, face1 = D[1] < 0.0 ? 8u : 12u, face2 = D[2] < 0.0 ? 16u : 20u;
    const Rsrc r_child = plane_rsrc(tv.child, (uint64_t)tv.n_internal * 32);
    const Rsrc r_links = plane_rsrc(tv.links, LINKED ? (uint64_t)tv.n_leaves * 24 : 0);

    double s = 0.0;
    uint32_t nd = 0;
    int k = 0;               // where a descent starts: node and its depth
    int leaf = 0, ld = 0;    // the leaf holding cell c, and its depth
    int reads = 0;
    auto descend = [&](bool go) {
        while (go) {
            const int sh = LAT - 1 - k;
            const uint32_t oct = (((uint32_t)c[0] >> sh) & 1u) | ((((uint32_t)c[1] >> sh) & 1u) << 1) |
                                 ((((uint32_t)c[2] >> sh) & 1u) << 2);
            const int e = (int)__builtin_amdgcn_raw_buffer_load_b32(r_child, nd * 32u + oct * 4u, 0, 0);
            ++reads;
            ++k;
            if (e < 0) {
                leaf = -1 - e;
                ld = k;
                go = false;
            } else {
                nd = (uint32_t)e;
                if constexpr (!LINKED) stk[k * BLOCK] = e;
            }
        }
    };
    if constexpr (!LINKED)
        if (tv.n_internal > 0) stk[0] = 0;
    descend(live && tv.n_internal > 0);
    if (live) desc += reads;
    for (int step = 0; step < tv.max_steps && __any(live); ++step) {
        const int cs = 1 << (LAT - ld);
        int lo[3], plane[3];
        double te[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = c[a] & -cs;
            plane[a] = lo[a] + (cs & ~back[a]);
            // an axis the ray does not move along: inf, or NaN on the plane itself; neither attains the minimum
            te[a] = ((double)plane[a] - O[a]) * inv[a];
        }
        const double tm = min_f64(te[0], min_f64(te[1], te[2]));
        const bool last = !live || !(tm < s1);      // an origin that is not a number crosses no plane
        const double e = min_f64(max_f64(tm, s), s1);
        const float delta = (float)(e - s);
        const bool h0 = te[0] == tm, h1 = te[1] == tm, h2 = te[2] == tm;
        const bool one = (int)h0 + (int)h1 + (int)h2 == 1;
        const bool in = live && delta > 0.f;
        // the cell behind the exit, before the loads: what it is computed from
        // need not stay in registers while the row is in flight
        const bool hit[3] = {h0, h1, h2};
        uint32_t diff = 0;
        int out = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            // truncation is floor for positive positions, and both clamp to lo below zero
            const int in_cell = med3((int)fma(tm, D[a], O[a]), lo[a], lo[a] | (cs - 1));
            const int m = hit[a] ? plane[a] + back[a] : in_cell;
            diff |= (uint32_t)(c[a] ^ m);
            out |= m;
            c[a] = m;
        }
        bool next = !last && ((uint32_t)out >> LAT) == 0u;
        const int here = leaf;
        typename Seg::Fetch f;
        seg.fetch_signal(leaf, in, f);
        uint32_t link = LINK_OUT;
        if constexpr (LINKED) {
            // 24 B per leaf; axis ax's far face at 8 ax + 4
            const bool follow = !last && one;
            const uint32_t at = (times3(leaf) << 3) + (h0 ? face0 : (h1 ? face1 : face2));
            link = __builtin_amdgcn_raw_buffer_load_b32(r_links, follow ? at : OFF_NONE, 0, 0);
            desc += follow;
            __builtin_amdgcn_sched_barrier(0);
        }
        seg.fetch(leaf, in, f);
        __builtin_amdgcn_sched_barrier(0);
        // find the next leaf while the row is in flight
        bool go = false;
        if constexpr (LINKED) {
            // a leaf across the one exit face; an internal node there, of the depth
            // of the leaf just left; or, through an edge or corner, from the root.
            // LINK_OUT is not reached (an interior face has a neighbour); ids are
            // checked so a bad link cannot reach outside the planes
            const bool to_leaf = one && (int)link < 0;
            nd = one ? link : 0u;
            k = one ? ld : 0;
            leaf = (int)(link & LINK_ID_MASK);
            const uint32_t id = to_leaf ? (uint32_t)leaf : nd;
            next = next && id < (uint32_t)(to_leaf ? tv.n_leaves : tv.n_internal);
            ld -= (int)((link >> LINK_ID_BITS) & 15u);
            go = !to_leaf;
        } else if (tv.n_internal > 0) {
            k = min(__clz(diff) - (32 - LAT), ld - 1);  // the deepest ancestor both cells share
            go = true;
            if (next) nd = (uint32_t)stk[k * BLOCK];
        }
        s = e;
        reads = 0;
        descend(go && next);
        if (!seg.shade(here, delta, in, f)) next = false;
        live = next;
        if (live) desc += reads;
    }
}

// One ray per lane through the tree, by the walk that fits it; called by all
// lanes of the wave.  LINKED: the caller knows that the tree is near and has
// links (the other walks are then not compiled in).
template <class Wave, class Lane, bool LINKED>
__device__ __forceinline__ void trace_pixel(const TreeView& tv, const FwdArgs& a, const Ray& r, bool live,
                                            int* __restrict__ stk, const float (&bg)[3], float (&rgb)[3]) {
    int desc = 0;
    auto out = [&](const auto& seg) {
#pragma unroll
        for (int c = 0; c < 3; ++c) rgb[c] = fmaf(seg.T, bg[c], seg.C[c]);
    };
    if (LINKED || tv.near) {
        Wave seg(tv, a);
        seg.begin(r);
        if (LINKED || tv.links)
            walk_fwd<true>(tv, r, live, stk, seg, desc);
        else
            walk_fwd<false>(tv, r, live, stk, seg, desc);
        out(seg);
    } else {
        Lane seg(tv, a);
        seg.begin(r);
        if (live) traverse(tv, r, stk, seg, desc);
        out(seg);
    }
}

}  // namespace dot
