// Adjoint kernels of libptmi: replay A of every camera path sample (its
// radiance, kept per path), then replay B from the same random numbers,
// gradients added with hardware fp32 atomics (see adjoint.h for the
// algorithm).
#include <type_traits>

#include "adjoint.h"
#include "wave.h"
#include "kernels.h"

namespace ptmi {

namespace {

// The sums that a wave collects before it adds them to global memory: per
// pending triangle three channel values, its place in the gradient and one
// byte of a table that finds equal places.
constexpr int kMergeSlots = 128;
struct MergeBuf {
    float v[3 * 64];
    uint32_t at[64];
    uint8_t slot[kMergeSlots];
};
static_assert(sizeof(MergeBuf) <= 8 * 64 * sizeof(uint2), "the wave's stack rows hold it (at least 8)");

// order of the wave's own LDS accesses (they execute in order; this keeps the compiler from moving them)
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Gradients go to global memory with hardware fp32 atomics, except two
// kinds of hot spots, which each block sums in LDS and adds once at the
// end: the light-sample emission terms of lights in the first kLdsLights
// entries of the light table (every visible light sample adds to one of
// them), and the albedo and emission terms of the kHotTris largest
// triangles (a ground plane or an area light is reached by a large share
// of all paths, and atomics on a few addresses are served one at a time).
// The others wait in registers for flush(), once per vertex.  Added one by
// one they bound replay B from records: 5.60 ms for a whole backward of 2.1M
// paths (512 x 512, 8 samples) over 1.02M triangles, 3.94 with them left out,
// since every lane of every instruction is a request of its own.  With three
// neighbouring lanes for the three channels of a triangle, which are one
// request, 4.51; with the wave's equal triangles (samples of one pixel) merged
// before, 4.04 (replay B 2.27 -> 0.80).  More than one copy of the sums in LDS
// gained nothing.
struct AtomicAcc {
    float* lds_light;  // 3 floats per light (local memory of the block)
    uint32_t n_lds;    // lights kept there
    float* lds_hot;    // [albedo, emission][3 * kHotTris] sums of the largest triangles
    uint32_t n_hot;
    float* g[2];       // albedo and emission gradient
    uint32_t at[2];    // this lane's pending triangle in g: 3 * id (kNone: none)
    float v[2][3];     // and its values
    static constexpr uint32_t kNone = 0xFFFFFFFFu;

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            at[w] = kNone;
            v[w][0] = v[w][1] = v[w][2] = 0.0f;
        }
    }
    __device__ __forceinline__ void add_tri(uint32_t hot, int which, int c, float* p, float x) {
        if (x == 0.0f) return;
        if (hot - 1u < n_hot) {
            atomicAdd(&lds_hot[which * 3 * kHotTris + 3 * (hot - 1u) + (uint32_t)c], x);
        } else {
            at[which] = (uint32_t)(p - g[which]) - (uint32_t)c;
            v[which][c] = x;
        }
    }
    __device__ __forceinline__ void add_light(uint32_t j, int c, float* p, float x) {
        if (x == 0.0f) return;
        if (j < n_lds)
            atomicAdd(&lds_light[3 * j + (uint32_t)c], x);
        else
            unsafeAtomicAdd(p, x);
    }
    // by all lanes of the wave together
    __device__ __forceinline__ void flush(int which, MergeBuf& m) {
        const bool has = at[which] != kNone;
        const uint64_t all = __ballot(has);
        if (all == 0ull) return;
        const uint32_t lane = lane_id(), me = rank_in(all), n = (uint32_t)__popcll(all);
        const uint32_t h = (at[which] * 2654435761u) >> 25;
        if (has) {
            m.at[me] = at[which];
            m.slot[h] = (uint8_t)me;  // one of the lanes that share it stays
#pragma unroll
            for (int c = 0; c < 3; ++c) m.v[3 * me + c] = v[which][c];
        }
        wave_lds_order();
        if (has) {
            const uint32_t w = m.slot[h];
            if (w != me && m.at[w] == at[which]) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    m.v[3 * me + c] = 0.0f;
                    if (v[which][c] != 0.0f) atomicAdd(&m.v[3 * w + c], v[which][c]);
                }
            }
        }
        wave_lds_order();
        for (uint32_t e = lane; e < 3u * n; e += 64u) {
            const uint32_t t = e / 3u;
            const float x = m.v[e];
            if (x != 0.0f) unsafeAtomicAdd(g[which] + m.at[t] + (e - 3u * t), x);
        }
        wave_lds_order();
    }
};

// How a replay's waves come by their paths, the next ones for the idle lanes of
// a wave (ballot idle, nidle of them); all lanes of the wave call take, which
// returns whether this lane gets path p, and more is false once there are none.
//
// The tracing replays: from a cursor in global memory, 64 paths at a time,
// since a path's rays take unequally long: 2.1M paths of the 1.02M-triangle
// scene 8.57 ms a backward, from the workgroups' fixed shares 10.80.  Up to
// two paths per lane of the grid, each wave's first 64 are dealt: all waves
// would ask the cursor at once, and it serves one at a time (480000 paths of a
// room 926 -> 786 us; of 50000 triangles 753 -> 635).  With more paths that
// costs up to 5 % (8.57 -> 9.05 ms: waves that start together go on together).
struct CursorPaths {
    unsigned long long* cursor;  // zero when the kernel starts
    uint32_t dealt;              // paths dealt before
    uint32_t npaths, next, end;  // the wave's 64
    bool more;
    __device__ __forceinline__ void open(unsigned long long* c, uint32_t n) {
        const uint32_t lanes = gridDim.x * blockDim.x;
        cursor = c;
        npaths = n;
        dealt = 0u;
        next = end = 0u;
        more = true;
        if (n / 2u <= lanes) {
            const uint32_t w = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
            const unsigned long long at = 64ull * __builtin_amdgcn_readfirstlane(w);
            dealt = lanes;
            end = (uint32_t)min(at + 64ull, (unsigned long long)n);
            next = (uint32_t)min(at, (unsigned long long)end);
        }
    }
    __device__ __forceinline__ bool take(uint64_t idle, uint32_t nidle, uint32_t& p) {
        if (next >= end) {
            unsigned long long base = 0ull;
            if (lane_id() == 0 && dealt < npaths) base = atomicAdd(cursor, 64ull);
            base = wave_broadcast_u64(base) + dealt;
            if (base >= (unsigned long long)npaths) {
                more = false;
                return false;
            }
            next = (uint32_t)base;
            end = (uint32_t)min(base + 64ull, (unsigned long long)npaths);
        }
        const uint32_t r = rank_in(idle), left = end - next;
        p = next + r;
        next += min(nidle, left);
        return r < left;
    }
};

// The replay from records, whose vertices all cost the same: from the
// workgroup's share (wave.h).  The cursor is served one wave at a time, about
// 11 ns each, which was most of this replay (see k_adjoint).
struct SharePaths {
    BlockShare share;
    uint32_t want;  // paths to take next at most
    bool more;
    __device__ __forceinline__ void open(uint32_t n, uint32_t simds, uint32_t* cursor) {
        share = open_share(n, simds, cursor);
        more = share.first < share.hi;
        want = share.start;
    }
    __device__ __forceinline__ bool take(uint64_t idle, uint32_t nidle, uint32_t& p) {
        const uint32_t n = min(nidle, want), c = share.take<true>(n, more);
        want = 64u;
        const uint32_t r = rank_in(idle);
        const uint64_t at = share.at_wide(c + r);
        p = (uint32_t)at;
        return r < n && at < share.hi;
    }
};

}  // namespace

// Replay A of every path: its radiance, into Lpath[path].  One loop trip =
// one path vertex; a lane whose path is done takes the next path of its
// wave's 64 (cursor[0]).  Five waves per SIMD, as the megakernel.  STORE: every
// vertex's intersection and light-sample visibility go to rec as well.
template <int LDS, bool ATTR, bool STORE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) k_adjoint_radiance(
    SceneView sc, CamView cam, PathParams pp, float4* __restrict__ Lpath, unsigned long long* __restrict__ cursor,
    uint2* __restrict__ ovf, int gcap, uint32_t* __restrict__ stats, VertexRecs rec) {
    extern __shared__ __align__(8) uint32_t smem[];
    const uint32_t nlanes = gridDim.x * blockDim.x;
    const uint32_t gtid = blockIdx.x * blockDim.x + threadIdx.x;
    TravStack<LDS> st =
        make_trav_stack<LDS>(reinterpret_cast<uint2*>(smem), (int)blockDim.x, ovf, gtid, (int)nlanes, gcap);
    const uint32_t npaths = (uint32_t)cam.W * (uint32_t)cam.H * (uint32_t)pp.spp;
    CursorPaths paths;
    paths.open(cursor, npaths);
    bool live = false;
    uint32_t path = 0, pix = 0, sample = 0, ne = 0, ns = 0;
    PathRun pr;
    while (true) {
        const uint64_t idle = __ballot(!live);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        if (paths.more && nidle > 0u) {
            uint32_t p = 0;
            if (paths.take(idle, nidle, p) && !live) {
                path = p;
                pix = path / (uint32_t)pp.spp;
                sample = pp.frame * (uint32_t)pp.spp + (path - pix * (uint32_t)pp.spp);
                path_begin(cam, pp, pix, sample, pr);
                live = true;
            }
        }
        if (__ballot(live) == 0ull) {
            if (!paths.more) break;
            continue;
        }
        if (!live) continue;
        if constexpr (STORE) {
            if (adjoint_a_vertex<LDS, ATTR>(sc, pp, pix, sample, path, pr, st, ne, ns, rec)) continue;
        } else {
            if (path_vertex<LDS, false, false, ATTR>(sc, pp, pix, sample, pr, st, ne, ns)) continue;
        }
        Lpath[path] = make_float4(pr.ps.L.x, pr.ps.L.y, pr.ps.L.z, 0.f);
        live = false;
    }
    // the rays of the paths (replay B traces the same ones again): one
    // atomic per wave for the whole kernel
    for (int off = 32; off > 0; off >>= 1) {
        ne += __shfl_xor(ne, off);
        ns += __shfl_xor(ns, off);
    }
    if (lane_id() == 0 && (ne | ns)) {
        atomicAdd(&stats[0], ne);
        atomicAdd(&stats[1], ns);
    }
    if (st.overflow) atomicOr(&stats[2], 1u);
}

// Replay B of every path, one vertex per loop trip (tracing, paths from
// cursor[1]), from the radiance replay A left in Lpath.  STORED: from replay
// A's records too, tracing no ray; then bound by the instructions of shading a
// vertex: 2.1M paths of the 1.02M-triangle scene 0.80 -> 0.72 ms, and 122880
// paths of a room (four bounces) 104 -> 77 us, when the paths came from the
// workgroups' shares instead of one global cursor.  Three waves per SIMD: 0.79
// ms and 71 us, five 1.2; refilling only once 16 or 32 lanes are idle the same
// or slower.
template <int LDS, bool ATTR, bool STORED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) k_adjoint(SceneView sc, CamView cam, PathParams pp,
                                                 const float* __restrict__ d_img, const float4* __restrict__ Lpath,
                                                 unsigned long long* __restrict__ cursor, uint32_t simds,
                                                 float* __restrict__ g_alb,
                                                 float* __restrict__ g_emi, uint2* __restrict__ ovf, int gcap,
                                                 uint32_t* __restrict__ stats, int count_rays, VertexRecs rec) {
    extern __shared__ __align__(8) uint32_t smem[];
    const uint32_t nlanes = gridDim.x * blockDim.x;
    const uint32_t gtid = blockIdx.x * blockDim.x + threadIdx.x;
    TravStack<LDS> st =
        make_trav_stack<LDS>(reinterpret_cast<uint2*>(smem), (int)blockDim.x, ovf, gtid, (int)nlanes, gcap);
    __shared__ float light_g[3 * kLdsLights];
    __shared__ float hot_g[2 * 3 * kHotTris];
    AtomicAcc acc;
    acc.lds_light = light_g;
    acc.n_lds = (uint32_t)min(max(sc.nl, 0), kLdsLights);
    acc.lds_hot = hot_g;
    acc.n_hot = (uint32_t)min(max(sc.n_hot, 0), kHotTris);
    acc.g[0] = g_alb;
    acc.g[1] = g_emi;
    // replay B traces no ray while it adds, so the wave's stack rows serve
    // as its merge buffer
    constexpr uint32_t kWaveLds = STORED ? (uint32_t)sizeof(MergeBuf) : (uint32_t)(LDS + 1) * kStackRow;
    MergeBuf& merge = *reinterpret_cast<MergeBuf*>(reinterpret_cast<char*>(smem) + (threadIdx.x >> 6) * kWaveLds);
    for (uint32_t j = threadIdx.x; j < 3 * acc.n_lds; j += blockDim.x) light_g[j] = 0.0f;
    for (uint32_t j = threadIdx.x; j < 2 * 3 * kHotTris; j += blockDim.x) hot_g[j] = 0.0f;
    __syncthreads();
    const uint32_t npaths = (uint32_t)cam.W * (uint32_t)cam.H * (uint32_t)pp.spp;
    const float fs = (float)pp.spp;
    __shared__ uint32_t share_cursor;
    std::conditional_t<STORED, SharePaths, CursorPaths> paths;
    if constexpr (STORED) paths.open(npaths, simds, &share_cursor);
    else paths.open(cursor + 1, npaths);
    bool live = false;
    AdjRun ar;
    uint32_t ne = 0, ns = 0;
    while (true) {
        const uint64_t idle = __ballot(!live);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        if (paths.more && nidle > 0u) {
            uint32_t p = 0;
            if (paths.take(idle, nidle, p) && !live) {
                const uint32_t pix = p / (uint32_t)pp.spp;
                const uint32_t s = p - pix * (uint32_t)pp.spp;
                const f3 delta = mk3(d_img[3 * (size_t)pix] / fs, d_img[3 * (size_t)pix + 1] / fs,
                                     d_img[3 * (size_t)pix + 2] / fs);
                adjoint_b_begin(cam, pp, pix, pp.frame * (uint32_t)pp.spp + s, delta, xyz(Lpath[p]), ar, p);
                live = true;
            }
        }
        if (__ballot(live) == 0ull) {
            if (!paths.more) break;
            continue;
        }
        acc.clear();
        if (live)
            live = adjoint_b_step<LDS, ATTR, AtomicAcc, false, STORED>(sc, pp, ar, g_alb, g_emi, st, acc, ne, ns, rec);
        acc.flush(0, merge);
        acc.flush(1, merge);
    }
    // with count_rays (replay A ran as the wavefront, which keeps its own
    // counters) the paths' rays are counted here (traced here, or by
    // replay A with its records), one atomic per wave
    if (count_rays) {
        for (int off = 32; off > 0; off >>= 1) {
            ne += __shfl_xor(ne, off);
            ns += __shfl_xor(ns, off);
        }
        if (lane_id() == 0 && (ne | ns)) {
            atomicAdd(&stats[0], ne);
            atomicAdd(&stats[1], ns);
        }
    }
    // every thread of the block is here: add the block's sums
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < 3 * acc.n_lds; j += blockDim.x) {
        const float v = light_g[j];
        if (v != 0.0f) unsafeAtomicAdd(g_emi + 3 * (size_t)sc.lights[j / 3u].id + j % 3u, v);
    }
    for (uint32_t j = threadIdx.x; j < 3 * acc.n_hot; j += blockDim.x) {
        const size_t at = 3 * (size_t)sc.hot_ids[j / 3u] + j % 3u;
        const float va = hot_g[j], ve = hot_g[3 * kHotTris + j];
        if (va != 0.0f) unsafeAtomicAdd(g_alb + at, va);
        if (ve != 0.0f) unsafeAtomicAdd(g_emi + at, ve);
    }
    if (st.overflow) atomicOr(&stats[2], 1u);
}

hipError_t launch_adjoint_radiance(int lds, dim3 grid, dim3 block, hipStream_t s, const SceneView& sc,
                                   const CamView& cam, const PathParams& pp, float4* Lpath,
                                   unsigned long long* cursor, uint2* ovf, int gcap, uint32_t* stats,
                                   const VertexRecs& rec) {
    size_t sm = trav_stack_lds_bytes(lds, (int)block.x);
#define K(N, A, S) \
    hipLaunchKernelGGL((k_adjoint_radiance<N, A, S>), grid, block, sm, s, sc, cam, pp, Lpath, cursor, ovf, gcap, stats, rec)
#define X(N)                                                  \
    if (lds == N) {                                           \
        if (rec.hit) {                                        \
            if (sc.attr_flags) K(N, true, true);              \
            else K(N, false, true);                           \
        } else {                                              \
            if (sc.attr_flags) K(N, true, false);             \
            else K(N, false, false);                          \
        }                                                     \
        return hipGetLastError();                             \
    }
    X(8) X(16) X(24) X(32)
#undef X
#undef K
    return hipErrorInvalidValue;
}

hipError_t launch_adjoint(int lds, dim3 grid, dim3 block, hipStream_t s, const SceneView& sc, const CamView& cam,
                          const PathParams& pp, const float* d_img, const float4* Lpath, unsigned long long* cursor,
                          uint32_t simds,
                          float* g_alb, float* g_emi, uint2* ovf, int gcap, uint32_t* stats, int count_rays,
                          const VertexRecs& rec) {
    // with the records replay B traces nothing: no traversal stack in LDS, merge buffers only
    const size_t sm = rec.hit ? sizeof(MergeBuf) * (block.x / 64u) : trav_stack_lds_bytes(lds, (int)block.x);
#define K(N, A, S)                                                                                               \
    hipLaunchKernelGGL((k_adjoint<N, A, S>), grid, block, sm, s, sc, cam, pp, d_img, Lpath, cursor, simds, g_alb, g_emi, \
                       ovf, gcap, stats, count_rays, rec)
    if (rec.hit) {
        if (sc.attr_flags) K(8, true, true);
        else K(8, false, true);
        return hipGetLastError();
    }
#define X(N)                                      \
    if (lds == N) {                               \
        if (sc.attr_flags) K(N, true, false);     \
        else K(N, false, false);                  \
        return hipGetLastError();                 \
    }
    X(8) X(16) X(24) X(32)
#undef X
#undef K
    return hipErrorInvalidValue;
}

}  // namespace ptmi
