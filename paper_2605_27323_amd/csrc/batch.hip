// Batched persistent wavefront kernels (see batch.h): one pool of path
// slots shared by many jobs, refilled from a global cursor every iteration.
// The host captures a fixed number of iterations into a hipGraph and replays
// it until the device control block reports that every path has finished.
#include "batch.h"
#include "wave.h"

namespace ptmi {

namespace {

template <int LDS>
__device__ __forceinline__ TravStack<LDS> stack_b(uint32_t* smem, uint2* ovf, int gcap) {
    return make_trav_stack<LDS>(reinterpret_cast<uint2*>(smem), (int)blockDim.x, ovf,
                                blockIdx.x * blockDim.x + threadIdx.x, (int)(gridDim.x * blockDim.x), gcap);
}

// The paths that a workgroup ends, per job: counted in LDS and taken off the
// job's count once, at the end of the kernel; the lane whose subtraction
// reaches zero stamps the job's completion time (at most the rest of its last
// kernel late).  Taken off wave by wave as the paths ended, they bounded the
// shade and shadow stages, since atomics on the few counters of all jobs are
// served one at a time, about 11 ns each: a batch of eight 512 x 512 renders of
// 4 samples took 2.45 ms, now 1.86 (its largest shadow launch 359 -> 177 us,
// shade 215 -> 104).
constexpr int kMostJobs = 256;  // a path carries its job in 8 bits

struct JobsEnded {
    uint32_t* n;  // [kMostJobs], in LDS
    __device__ __forceinline__ void open() const {
        for (uint32_t j = threadIdx.x; j < (uint32_t)kMostJobs; j += blockDim.x) n[j] = 0u;
        __syncthreads();
    }
    __device__ __forceinline__ void add(uint32_t job) const { atomicAdd(&n[job], 1u); }
    __device__ __forceinline__ void close(const BatchBufs& bb) const {
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < (uint32_t)bb.njobs; j += blockDim.x) {
            const uint32_t k = n[j];
            if (k && atomicSub(&bb.remaining[j], k) == k) bb.done_ts[j] = wall_clock64();
        }
    }
};

}  // namespace

__global__ void k_batch_init(BatchBufs bb, uint32_t total) {
    const int t = threadIdx.x;
    if (t == 0) {
        BatchCtl& c = *bb.ctl;
        c.total = total;
        c.cursor = 0u;
        c.live[0] = c.live[1] = 0u;
        c.count = c.regen_first = c.regen_n = c.regen_path = c.shadow = 0u;
        c.done = 0u;
        c.iterations = 0u;
        c.err = 0u;
        c.t_start = wall_clock64();
    }
    for (int j = t; j < bb.njobs; j += blockDim.x) {
        bb.remaining[j] = bb.jobs[j].npaths;
        bb.done_ts[j] = 0ull;
    }
}

__global__ void k_batch_sched(BatchBufs bb, int q) {
    if (threadIdx.x == 0 && blockIdx.x == 0) batch_schedule(bb, q);
}

__global__ void __launch_bounds__(256) k_batch_regen(BatchBufs bb, int q) {
    const uint32_t n = bb.ctl->regen_n;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        batch_regen_item(bb, q, i);
}

// persistent traversal over the pool (see k_extend); a lane's scene is its
// path's job's scene, held in registers: at seven waves per SIMD nothing
// spills, at eight nine registers did (a batch of 8 scenes 2.49 and 2.82 ms)
template <int LDS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7)))
k_batch_extend(BatchBufs bb, int q, uint2* __restrict__ ovf, int gcap) {
    extern __shared__ __align__(8) uint32_t smem[];
    TravStack<LDS> st = stack_b<LDS>(smem, ovf, gcap);
    __shared__ uint32_t cursor;
    const BlockShare share = open_share(bb.ctl->count, bb.simds, &cursor);
    bool more = share.at(0u) < share.hi;
    uint32_t want = share.start;
    uint32_t item = 0, ref = kDoneRef;  // a lane without a ray
    SceneView sc{};
    Ray ray;
    Hit h;
    while (true) {
        const uint64_t idle = __ballot(ref == kDoneRef);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        if (more && (nidle >= kRefill || nidle == 64u)) {
            const uint32_t n = min(nidle, want), c = share.take(n, more);
            want = 64u;
            if (ref == kDoneRef) {
                const uint32_t r = rank_in(idle), i = share.at(c + r);
                if (r < n && i < share.hi) {
                    const float4 o4 = bb.ray_o[q][i], d4 = bb.ray_d[q][i];
                    sc = bb.jobs[f2u(bb.pst[q][i].w) >> 24].sc;
                    ray = make_ray(xyz(o4), xyz(d4));
                    closest_begin<LDS>(INFINITY, h, ref, st);
                    item = i;
                }
            }
        } else if (nidle == 64u) {
            break;
        }
        if (ref != kDoneRef) {
            closest_step<LDS>(sc, ray, INFINITY, h, ref, st);
            if (ref == kDoneRef) bb.hit[item] = make_float4(h.t, 0.f, 0.f, u2f(h.tri));
        }
    }
    if (st.overflow) atomicOr(&bb.ctl->err, 1u);
}

// slots of the next queue and of the shadow queue reserved once per block
// and trip (see k_shade)
// four waves per SIMD, as k_shade (without attributes: 128 VGPRs, no spill)
template <bool ATTR>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) k_batch_shade(BatchBufs bb, int q) {
    const uint32_t nlanes = gridDim.x * blockDim.x;
    const uint32_t count = bb.ctl->count;
    __shared__ BlockReserve br;
    __shared__ uint32_t ended_n[kMostJobs];
    const JobsEnded ended{ended_n};
    ended.open();
    int par = 0;
    for (uint32_t bbase = blockIdx.x * blockDim.x; bbase < count; bbase += nlanes, par ^= 1) {
        const uint32_t i = bbase + threadIdx.x;
        VertexOut vo;
        ShadowReq sh;
        PathState ps;
        vo.cont = false;
        sh.valid = false;
        uint32_t g = 0, meta = 0;
        bool finished = false;
        if (i < count) finished = batch_shade_item<ATTR>(bb, q, i, vo, sh, ps, g, meta);
        if (finished) ended.add(meta >> 24);
        const uint64_t mk = __ballot(vo.cont), ms = __ballot(sh.valid);
        uint32_t jc, js;
        block_reserve2(br, par, &bb.ctl->live[q ^ 1], mk, &bb.ctl->shadow, ms, jc, js);
        if (vo.cont) batch_write_continuation(bb, q ^ 1, jc, vo, ps, g, meta);
        if (sh.valid) batch_write_shadow(bb, js, sh, g, meta >> 24, !vo.cont);
    }
    ended.close(bb);
}

// persistent any-hit over the shadow records, some of which end their path
template <int LDS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7)))
k_batch_shadow(BatchBufs bb, uint2* __restrict__ ovf, int gcap) {
    extern __shared__ __align__(8) uint32_t smem[];
    TravStack<LDS> st = stack_b<LDS>(smem, ovf, gcap);
    __shared__ uint32_t cursor;
    __shared__ uint32_t ended_n[kMostJobs];
    const JobsEnded ended{ended_n};
    ended.open();
    const BlockShare share = open_share(bb.ctl->shadow, bb.simds, &cursor);
    bool more = share.at(0u) < share.hi;
    uint32_t want = share.start;
    uint32_t item = 0, ref = kDoneRef, tag = 0;  // a lane without a ray
    SceneView sc{};
    Ray ray;
    uint32_t occluded = 0u;
    while (true) {
        const uint64_t idle = __ballot(ref == kDoneRef);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        if (more && (nidle >= kRefill || nidle == 64u)) {
            const uint32_t n = min(nidle, want), c = share.take(n, more);
            want = 64u;
            if (ref == kDoneRef) {
                const uint32_t r = rank_in(idle), i = share.at(c + r);
                if (r < n && i < share.hi) {
                    const float4 o4 = bb.sh_o[i], d4 = bb.sh_d[i];
                    tag = f2u(d4.w);
                    sc = bb.jobs[tag & 0x7FFFFFFFu].sc;
                    ray = make_ray(xyz(o4), xyz(d4));
                    any_begin<LDS>(ref, st);
                    occluded = 0u;
                    item = i;
                }
            }
        } else if (nidle == 64u) {
            break;
        }
        if (ref != kDoneRef) {
            any_step<LDS>(sc, ray, kShadowTmax, ref, st, occluded);
            if (ref == kDoneRef) {
                if (!occluded) batch_shadow_add(bb, item);
                if (tag >> 31) ended.add(tag & 0x7FFFFFFFu);
            }
        }
    }
    ended.close(bb);
    if (st.overflow) atomicOr(&bb.ctl->err, 1u);
}

__global__ void __launch_bounds__(256) k_batch_accumulate(BatchBufs bb, uint32_t total_pix) {
    for (uint32_t gp = blockIdx.x * blockDim.x + threadIdx.x; gp < total_pix; gp += gridDim.x * blockDim.x)
        batch_accumulate_item(bb, gp);
}

hipError_t launch_batch_init(hipStream_t s, const BatchBufs& bb, uint32_t total) {
    hipLaunchKernelGGL(k_batch_init, dim3(1), dim3(256), 0, s, bb, total);
    return hipGetLastError();
}

// one iteration of the pool on queue parity q
hipError_t launch_batch_iteration(int lds, dim3 grid, dim3 block, hipStream_t s, const BatchBufs& bb, int q,
                                  uint2* ovf, int gcap, bool attr) {
    const size_t sm = trav_stack_lds_bytes(lds, (int)block.x);
    hipLaunchKernelGGL(k_batch_sched, dim3(1), dim3(64), 0, s, bb, q);
    hipLaunchKernelGGL(k_batch_regen, grid, block, 0, s, bb, q);
#define X(N)                                                                              \
    if (lds == N) {                                                                       \
        hipLaunchKernelGGL(k_batch_extend<N>, grid, block, sm, s, bb, q, ovf, gcap);      \
        if (attr)                                                                         \
            hipLaunchKernelGGL(k_batch_shade<true>, grid, block, 0, s, bb, q);            \
        else                                                                              \
            hipLaunchKernelGGL(k_batch_shade<false>, grid, block, 0, s, bb, q);           \
        hipLaunchKernelGGL(k_batch_shadow<N>, grid, block, sm, s, bb, ovf, gcap);         \
        return hipGetLastError();                                                         \
    }
    X(8) X(16) X(24) X(32)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_batch_accumulate(dim3 grid, dim3 block, hipStream_t s, const BatchBufs& bb, uint32_t total_pix) {
    hipLaunchKernelGGL(k_batch_accumulate, grid, block, 0, s, bb, total_pix);
    return hipGetLastError();
}

}  // namespace ptmi
