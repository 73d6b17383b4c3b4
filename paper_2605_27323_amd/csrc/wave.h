// Wave- and block-level helpers of the GPU kernels (device code only):
// lane ranks within a 64-lane ballot, the per-wave queue chunk of the
// persistent traversal kernels, and block-aggregated queue reservation.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"

namespace ptmi {

__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// position of this lane among the set lanes of a 64-bit ballot below it
__device__ __forceinline__ uint32_t rank_in(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// one atomic per wave reserves room for the wave's set lanes; every set
// lane gets base + its rank among them
__device__ __forceinline__ uint32_t wave_reserve(uint32_t* ctr, uint64_t m) {
    uint32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(ctr, (uint32_t)__popcll(m));
    base = __builtin_amdgcn_readfirstlane(base);
    return base + rank_in(m);
}

// Sum v over the 64 lanes of the wave (every lane calls this) and add the
// sum to *dst with one atomic.
__device__ __forceinline__ void wave_add_u64(unsigned long long* dst, uint32_t v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane_id() == 0 && v) atomicAdd(dst, (unsigned long long)v);
}

// lane 0's value, in every lane
__device__ __forceinline__ unsigned long long wave_broadcast_u64(unsigned long long v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

// A workgroup's share of a queue in the persistent traversal kernels.  The
// queue is cut into sections of 64 entries per wave that go to the
// workgroups in turn, and the waves of a workgroup take their section's
// entries, and then those of its next section, from one cursor in LDS.
// Every workgroup then has rays from all over the queue (all over the image,
// after raygen): with one contiguous part of the queue per wave, the waves
// that got the empty sky ended long before those that got the objects.
// Sections of 1024 entries gave 2.74 instead of 2.43 ms per frame of the
// 1.02M-triangle scene, sections of 64 the same.  Full waves also where the
// queue does not fill the grid: 65536 rays as 1024 waves of 64 took 247 us a
// frame of the Cornell room, as waves of 32 255, of 16 279, of 8 (every wave
// of the grid) 351.  Only a queue too short for one full wave per SIMD is cut
// into sections of fewer entries per wave: such a wave is alone on its SIMD
// and takes as many steps as its longest ray and their divergence ask for
// (1536 rays: 218 us a frame, in full waves 228).
// xcd_local (PT_FLAG_XCD_LOCAL): the dispatcher places workgroup b on XCD
// b mod 8 (each XCD has its own L2); the sections of one eighth of the queue
// go to the workgroups of one XCD, so that neighbouring rays share an L2.
// Grids that are not a multiple of 8 ignore it.
struct BlockShare {
    uint32_t first;   // first entry of the workgroup's first section
    uint32_t hi;      // end of the queue (of the XCD's eighth)
    uint32_t stride;  // entries from one of its sections to the next
    uint32_t lg;      // log2 of the entries of a section
    uint32_t start;   // entries a wave takes first
    __attribute__((address_space(3))) uint32_t* cursor;

    // queue position of the share's c-th entry (valid below hi)
    __device__ __forceinline__ uint32_t at(uint32_t c) const {
        return first + (c >> lg) * stride + (c & ((1u << lg) - 1u));
    }
    // the same where the queue may end within a section per workgroup of 2^32
    __device__ __forceinline__ uint64_t at_wide(uint32_t c) const {
        return (uint64_t)first + (uint64_t)(c >> lg) * stride + (c & ((1u << lg) - 1u));
    }
    // the next n entries of the share, for this wave: the index of the first
    // (wave-uniform); more = false once the share holds no further ones
    template <bool WIDE = false>
    __device__ __forceinline__ uint32_t take(uint32_t n, bool& more) const {
        uint32_t c = 0;
        if (lane_id() == 0) c = __hip_atomic_fetch_add(cursor, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        c = __builtin_amdgcn_readfirstlane(c);
        if constexpr (WIDE) more = at_wide(c + n) < hi;
        else more = at(c + n) < hi;
        return c;
    }
};

// simds: SIMDs of the device.  Every thread of the workgroup calls this (it
// synchronises the workgroup).
__device__ __forceinline__ BlockShare open_share(uint32_t count, uint32_t simds, uint32_t* cursor, int xcd_local = 0) {
    if (threadIdx.x == 0) *cursor = 0u;
    uint32_t blk = blockIdx.x, nblk = gridDim.x, lo = 0u, hi = count;
    if (xcd_local && (gridDim.x & 7u) == 0u) {
        const uint32_t part = (count + 7u) >> 3;
        lo = min((blk & 7u) * part, count);
        hi = min(lo + part, count);
        blk >>= 3;
        nblk >>= 3;
    }
    uint32_t lg = 6u;  // log2 of the entries per wave
    while (lg > 0u && (simds << (lg - 1u)) >= count) --lg;
    BlockShare s;
    s.start = 1u << lg;
    for (uint32_t w = blockDim.x >> 6; w > 1u; w = (w + 1u) >> 1) ++lg;
    s.lg = lg;
    s.stride = __builtin_amdgcn_readfirstlane(nblk << lg);
    s.first = __builtin_amdgcn_readfirstlane(lo + (blk << lg));
    s.hi = __builtin_amdgcn_readfirstlane(hi);
    s.cursor = (__attribute__((address_space(3))) uint32_t*)cursor;
    __syncthreads();
    return s;
}

// Block-aggregated reservation on two queue counters: every thread of the
// block calls this once per trip (it synchronises the block) with its
// wave's ballots m0, m1; one atomic per counter and block.  Returns the
// slots of this lane (valid where its bit is set).  `par` alternates
// between trips: the counts are double-buffered so that two barriers per
// trip suffice.  Blocks of at most 256 threads.
struct BlockReserve {
    uint32_t cnt[2][2][4];
    uint32_t base[2][2];
};

__device__ __forceinline__ void block_reserve2(BlockReserve& br, int par, uint32_t* c0, uint64_t m0, uint32_t* c1,
                                               uint64_t m1, uint32_t& j0, uint32_t& j1) {
    const uint32_t w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (lane_id() == 0) {
        br.cnt[par][0][w] = (uint32_t)__popcll(m0);
        br.cnt[par][1][w] = (uint32_t)__popcll(m1);
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        uint32_t tot = 0;
        for (uint32_t k = 0; k < nw; ++k) tot += br.cnt[par][threadIdx.x][k];
        br.base[par][threadIdx.x] = tot ? atomicAdd(threadIdx.x == 0 ? c0 : c1, tot) : 0u;
    }
    __syncthreads();
    uint32_t o0 = br.base[par][0], o1 = br.base[par][1];
    for (uint32_t k = 0; k < w; ++k) {
        o0 += br.cnt[par][0][k];
        o1 += br.cnt[par][1][k];
    }
    j0 = o0 + rank_in(m0);
    j1 = o1 + rank_in(m1);
}

// Stage the light table (CDF words, leaf-order and input triangle indices)
// in the block's LDS so that the light choice is a binary search in LDS.
// Every thread of the block must call this (it synchronises the block).
__device__ __forceinline__ LightCache stage_lights(const SceneView& sc, uint32_t* buf) {
    if (sc.nl <= 0 || sc.nl > kLdsLights) return no_light_cache();
    for (int j = threadIdx.x; j < sc.nl; j += blockDim.x) {
        const LightEntry e = sc.lights[j];
        buf[j] = e.cdf;
        buf[kLdsLights + j] = e.tri;
        buf[2 * kLdsLights + j] = e.id;
    }
    __syncthreads();
    LightCache lc;
    lc.cdf = (const lds_u32*)buf;
    lc.tri = (const lds_u32*)(buf + kLdsLights);
    lc.id = (const lds_u32*)(buf + 2 * kLdsLights);
    lc.n = sc.nl;
    return lc;
}

}  // namespace ptmi
