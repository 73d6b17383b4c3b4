// Frames too small to fill the GPU: whole paths in one launch (device code,
// compiled with the render kernels).
#pragma once
#include "kernels.h"
#include "wave.h"
#include "wavefront.h"

namespace ptmi {

namespace {

// what the two waves of a workgroup hand each other
struct PairShared {
    float ray[6][64];          // light samples: origin, direction
    unsigned long long valid;  // lanes that have one
    unsigned long long seen;   // of these, the unoccluded ones
    uint32_t go;               // 0: no further vertex
    uint32_t overflow;         // a traversal stack of the second wave overflowed
    uint32_t rays[2][kSmallDepth + 2];
};

// barrier of the workgroup's two waves, each at its own place in the code
__device__ __forceinline__ void pair_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

}  // namespace

// One path per lane of a workgroup's first wave, to its end; the second wave
// traces the light samples of a vertex while the first traces the
// continuations.  Few paths are bound by latency alone: a vertex of a wave
// that has its SIMD to itself takes about 10 us for the extension, 6 for the
// shading and 8 for the light sample, and as separate launches another 10
// for starting and joining them.  So: as few lanes to a wave as keep every
// SIMD at one path wave, samples of a pixel side by side instead of one
// after the other, no launch between the vertices.  us a frame before and
// after: the Cornell room at 32 x 24, 2 spp 214 -> 74, at 128 x 128, 4 spp 238
// -> 86; the room with attributes at 131 x 97, 3 spp (megakernel) 694 -> 164.
// Three waves per SIMD (168 registers, three spilled; at four, 128, 10 %
// slower; two the same).
//
// A chunk of sa.per paths (whole pixels when there is an image) goes to a
// wave at a time, the first one by the workgroup's number.  Where there are
// more chunks than workgroups (whose spill areas bound them), the next ones
// come from a cursor, sa.next.
//
// sa.img: the pixels' means over their spp samples, added in sample order (and
// the running average sa.acc); else wb.L: every path's
// radiance.  wb.rec_*: the adjoint's kept intersections (or null).  The rays
// traced per bounce go to sa.rows (extension rays of bounces 0 .. D + 1, light
// samples of 0 .. D + 1, overflow flag), one row per workgroup: counters
// shared by all would be served one at a time, after one more launch that
// clears them.
template <int LDS, bool INST, bool ATTR>
__global__ void __launch_bounds__(kSmallBlock) __attribute__((amdgpu_waves_per_eu(3))) k_small(
    SceneView sc, CamView cam, PathParams pp, SmallArgs sa, WaveBufs wb, uint2* __restrict__ ovf, int gcap) {
    extern __shared__ __align__(8) uint32_t smem[];
    __shared__ uint32_t light_buf[3 * kLdsLights];
    __shared__ PairShared ps2;
    static_assert(sizeof light_buf + sizeof ps2 <= kSmallLdsBytes, "resident workgroups are counted by it");
    for (uint32_t j = threadIdx.x; j < 2u * (kSmallDepth + 2u); j += blockDim.x) (&ps2.rays[0][0])[j] = 0u;
    if (threadIdx.x == 0) ps2.overflow = 0u;
    __syncthreads();
    const LightCache lc = stage_lights(sc, light_buf);
    TravStack<LDS> st = make_trav_stack<LDS>(reinterpret_cast<uint2*>(smem), 64, ovf,
                                             blockIdx.x * blockDim.x + threadIdx.x, (int)(gridDim.x * blockDim.x), gcap);
    const uint32_t lane = lane_id();
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) != 0u) {
        // the second wave: light samples
        while (true) {
            pair_sync();
            if (__builtin_amdgcn_readfirstlane(ps2.go) == 0u) break;
            const bool has = (ps2.valid >> lane) & 1ull;
            bool seen = false;
            if (has)
                seen = !any_hit_t<LDS, false, INST>(sc, mk3(ps2.ray[0][lane], ps2.ray[1][lane], ps2.ray[2][lane]),
                                                    mk3(ps2.ray[3][lane], ps2.ray[4][lane], ps2.ray[5][lane]),
                                                    kShadowTmax, st);
            const unsigned long long m = __ballot(seen);
            if (lane == 0u) ps2.seen = m;
            if (st.overflow) ps2.overflow = 1u;
            pair_sync();
        }
        return;
    }
    const uint32_t spp = (uint32_t)pp.spp;
    for (uint32_t chunk = blockIdx.x; (uint64_t)chunk * sa.per < sa.npaths;) {
        const uint32_t path = chunk * sa.per + lane;
        const bool mine = lane < sa.per && path < sa.npaths;
        const uint32_t pix = path / spp, s = path - pix * spp;
        const uint32_t sample = pp.frame * spp + s;
        PathRun pr;
        path_begin(cam, pp, pix, sample, pr);
        bool cont = mine, has = false;  // the path goes on; its last vertex has a light sample
        f3 contrib;
        Hit h;
        for (uint32_t b = 0;; ++b) {
            const unsigned long long m = __ballot(cont);
            if (m != 0ull) {
                if (lane == 0u) ps2.rays[0][b] += (uint32_t)__popcll(m);
                if (cont) h = closest_hit_t<LDS, false, INST>(sc, pr.o, pr.d, INFINITY, st);
            }
            if (b > 0u) {
                pair_sync();  // the light samples of the vertex before are decided
                if (has) {
                    const bool seen = (ps2.seen >> lane) & 1ull;
                    if (seen) pr.ps.L = add3(pr.ps.L, contrib);
                    if (wb.rec_vis) wb.rec_vis[(size_t)(b - 1u) * wb.rec_n + path] = seen ? 1 : 0;
                }
            }
            if (m == 0ull) break;
            has = false;
            if (cont) {
                if (wb.rec_hit) wb.rec_hit[(size_t)b * wb.rec_n + path] = make_uint2(f2u(h.t), h.tri);
                ShadowReq sh;
                const VertexOut vo = shade_vertex<INST, ATTR>(sc, pp, pix, sample, (int)b + 1, pr.d, h, pr.ps, sh, lc);
                add_radiance(pr.ps, vo);
                if (sh.valid) {
                    has = true;
                    contrib = sh.contrib;
                    ps2.ray[0][lane] = sh.o.x;
                    ps2.ray[1][lane] = sh.o.y;
                    ps2.ray[2][lane] = sh.o.z;
                    ps2.ray[3][lane] = sh.d.x;
                    ps2.ray[4][lane] = sh.d.y;
                    ps2.ray[5][lane] = sh.d.z;
                }
                cont = vo.cont;
                pr.o = vo.o;
                pr.d = vo.d;
            }
            const unsigned long long v = __ballot(has);
            if (v == 0ull && __ballot(cont) == 0ull) break;
            if (lane == 0u) {
                ps2.rays[1][b] += (uint32_t)__popcll(v);
                ps2.valid = v;
                ps2.go = 1u;
            }
            pair_sync();
        }
        const f3 L = pr.ps.L;
        if (sa.img) {
            f3 sum = L;
            for (uint32_t j = 1; j < spp; ++j)
                sum = add3(sum, mk3(__shfl(L.x, (int)(lane + j)), __shfl(L.y, (int)(lane + j)), __shfl(L.z, (int)(lane + j))));
            const float fs = (float)spp;
            if (mine && s == 0u) store_pixel(sa.img, sa.acc, pix, mk3(sum.x / fs, sum.y / fs, sum.z / fs), pp.frame);
        } else if (mine) {
            wb.L[path] = make_float4(L.x, L.y, L.z, 0.f);
        }
        if (sa.next == nullptr) break;
        uint32_t taken = 0u;
        if (lane == 0u) taken = atomicAdd(sa.next, 1u);
        chunk = gridDim.x + __builtin_amdgcn_readfirstlane(taken);
    }
    if (lane == 0u) ps2.go = 0u;
    pair_sync();
    const bool over = __ballot(st.overflow != 0u) != 0ull || ps2.overflow != 0u;
    const uint32_t nb = (uint32_t)pp.D + 2u;
    uint32_t* row = sa.rows + (size_t)blockIdx.x * small_row_words(pp.D);
    for (uint32_t j = lane; j < nb; j += 64u) {
        row[j] = ps2.rays[0][j];
        row[nb + j] = ps2.rays[1][j];
    }
    if (lane == 0u) {
        row[2u * nb] = over ? 1u : 0u;
        if (over && sa.err) atomicOr(sa.err, 1u);
    }
}

hipError_t launch_small(int lds, uint32_t grid, hipStream_t s, const SceneView& sc, const CamView& cam,
                        const PathParams& pp, const SmallArgs& sa, const WaveBufs& wb, uint2* ovf, int gcap) {
    const size_t sm = trav_stack_lds_bytes(lds, kSmallBlock);
    const bool inst = sc.n_inst > 0, attr = sc.attr_flags != 0;
#define K(N, I, A) hipLaunchKernelGGL((k_small<N, I, A>), dim3(grid), dim3(kSmallBlock), sm, s, sc, cam, pp, sa, wb, ovf, gcap)
#define X(N)                                  \
    if (lds == N) {                           \
        if (inst && attr) K(N, true, true);   \
        else if (inst) K(N, true, false);     \
        else if (attr) K(N, false, true);     \
        else K(N, false, false);              \
        return hipGetLastError();             \
    }
    X(8) X(16) X(24) X(32)
#undef X
#undef K
    return hipErrorInvalidValue;
}

}  // namespace ptmi
