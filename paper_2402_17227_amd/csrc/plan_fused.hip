// The whole sampling plan of a small layer in ONE launch (Sec. 4.1 SampleA,
// Sec. 4.2 SampleW): every workgroup takes rows of G and X and writes their sums
// of squares (and the SampleW uniforms); the workgroup that finishes last then
// runs both samplers on the vectors the others left in memory.  A layer of
// BERT-base size needs seven launches otherwise, and the command processor
// starts only about one kernel every 2.5 us.
//
// The samplers are those of samplers.hpp, by the same workgroup size as the stand-alone kernels (1024
// threads, four elements each).  An earlier version kept 256-thread workgroups for the norm phase and ran
// the samplers on sixteen elements a thread: the tail is a chain of cross-lane and fp64 latencies in
// which four times the elements on a quarter of the wavefronts took about twice as long.
#include "rowsum.hpp"
#include "samplers.hpp"

namespace vcas {

namespace {

constexpr int kThreads = 1024;
constexpr int kSub = 32;       // first-level ticket counters
constexpr int kLine = 32;      // words between counters: every counter has a 128-byte line to itself

struct PlanArgs {
    const uint4 *G, *X;
    int groups_g, groups_x;       // 16-byte groups per row
    int N, T;
    double budget_a, budget_w;
    int token_sampling;
    UniformJob job;               // SampleW uniforms (stream 1); seed, layer, draw also serve SampleA
    uint32_t *tickets;            // kSub + 1 zeroed counters, kLine words apart
    float *gsq, *gnorm, *p;
    uint8_t *maskA;
    int32_t *idxA, *cntA;
    float *xsq, *score, *q;
    uint8_t *maskW;
    float *scaleW;
    int32_t *idxW, *cntW;
};

// Store that is written through to device-coherent memory (no dirty line stays in this XCD's L2).
__device__ __forceinline__ void store_through(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// SampleA then SampleW by the last workgroup; N <= 1024, R <= 1024 * E.
template <int E>
__device__ __forceinline__ void plan_tail(const PlanArgs &a, uint32_t draw)
{
    __shared__ SampleTable table;
    const int tid = threadIdx.x;
    const int N = a.N, T = a.T, R = N * T;
    // this thread's tokens: issued first, needed after SampleA
    float g[E], x[E], uu[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int t = min(tid + 1024 * j, R - 1);
        g[j] = a.gsq[t];
        x[j] = a.xsq[t];
        uu[j] = a.token_sampling ? a.job.uniforms[t] : 0.0f;
    }
    sampler_a_fast_body(a.gsq, N, T, a.budget_a, a.job.seed, a.job.layer, draw, a.gnorm, a.p, a.maskA, a.idxA, a.cntA, &table);
#pragma unroll
    for (int j = 0; j < E; ++j) {   // beside SampleA: the square roots do not wait for it
        g[j] = __builtin_sqrtf(g[j]);
        x[j] = __builtin_sqrtf(x[j]);
    }
    __syncthreads();
    const uint32_t magic = sample_magic(T);
    float sc[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int t = tid + 1024 * j;
        sc[j] = 0.0f;
        if (t < R) {
            const int i = sample_of(t, T, magic);
            if (table.keep[i]) {
                const float s1 = table.pinv[i] * g[j];
                sc[j] = s1 * x[j];
            } else {
                a.xsq[t] = 0.0f;
            }
            a.score[t] = sc[j];
        }
    }
    sample_w_finish<E>(sc, uu, &table, a.p, a.maskA, R, T, a.budget_w, a.token_sampling, a.q, a.maskW,
                              a.scaleW, a.idxW, a.cntW);
}

template <bool BF16, int CH>
__global__ __launch_bounds__(kThreads) void plan_fused_kernel(PlanArgs a)
{
    __shared__ int is_last;
    const int R = a.N * a.T;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t draw = a.job.draw + (a.job.draw_offset ? *a.job.draw_offset : 0u);
    if (a.job.uniforms)
        for (int r = blockIdx.x * kThreads + tid; r < R; r += gridDim.x * kThreads)
            store_through(a.job.uniforms + r,
                          philox_uniform(a.job.seed, a.job.layer, a.job.stream_id, draw, (uint32_t)r));
    // rows [0, R) are G's, [R, 2R) are X's; a wavefront takes two rows at a time so that the
    // loads of both are in flight together
    const int wave = blockIdx.x * (kThreads / 64) + (tid >> 6), nwaves = gridDim.x * (kThreads / 64);
    for (int w = wave; w < 2 * R; w += 2 * nwaves) {
        const int w2 = w + nwaves;
        const bool two = w2 < 2 * R;
        const bool sx0 = w >= R, sx1 = w2 >= R;
        const int row0 = sx0 ? w - R : w, row1 = sx1 ? w2 - R : w2;
        const int gr0 = sx0 ? a.groups_x : a.groups_g, gr1 = sx1 ? a.groups_x : a.groups_g;
        const uint4 *p0 = (sx0 ? a.X : a.G) + (int64_t)row0 * gr0;
        const uint4 *p1 = (sx1 ? a.X : a.G) + (int64_t)row1 * gr1;
        float acc0, acc1 = 0.0f;
        if (gr0 <= 64 * CH && gr1 <= 64 * CH) {
            uint4 v0[CH], v1[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int gidx = lane + 64 * j;
                v0[j] = gidx < gr0 ? p0[gidx] : make_uint4(0u, 0u, 0u, 0u);
                v1[j] = two && gidx < gr1 ? p1[gidx] : make_uint4(0u, 0u, 0u, 0u);
            }
            acc0 = chunk_sumsq<BF16, CH>(v0, (gr0 + 63) / 64);
            if (two) acc1 = chunk_sumsq<BF16, CH>(v1, (gr1 + 63) / 64);
        } else {
            acc0 = wave_row_sumsq<BF16, CH>(p0, gr0);
            if (two) acc1 = wave_row_sumsq<BF16, CH>(p1, gr1);
        }
        if (lane == 0) {
            store_through((sx0 ? a.xsq : a.gsq) + row0, acc0);
            if (two) store_through((sx1 ? a.xsq : a.gsq) + row1, acc1);
        }
    }
    // The results went out as write-through stores, so releasing them needs no L2 write-back
    // (which costs every workgroup microseconds): wait until this workgroup's stores are
    // acknowledged, then take a ticket.  Two levels of counters keep the atomics on one address
    // few: a workgroup that completes its first-level counter takes a ticket of the top one.
    // Only the workgroup that completes the top counter stays; it zeroes the counters for the
    // next launch and drops whatever stale lines its caches hold before it reads the vectors.
    __builtin_amdgcn_s_waitcnt(0);   // vmcnt = expcnt = lgkmcnt = 0
    __syncthreads();
    if (tid == 0) {
        const uint32_t sub = blockIdx.x % kSub;
        const uint32_t members = (gridDim.x - sub + kSub - 1) / kSub;
        const uint32_t used = gridDim.x < (uint32_t)kSub ? gridDim.x : (uint32_t)kSub;
        int last = 0;
        if (__hip_atomic_fetch_add(a.tickets + sub * kLine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
            members - 1)
            last = __hip_atomic_fetch_add(a.tickets + kSub * kLine, 1u, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT) == used - 1;
        if (last)
            for (int i = 0; i <= kSub; ++i)
                __hip_atomic_store(a.tickets + i * kLine, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        is_last = last;
    }
    __syncthreads();
    if (!is_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (R <= 1024) plan_tail<1>(a, draw);
    else plan_tail<4>(a, draw);
}

}  // namespace

// True when plan_fused handles this layer.
bool plan_fused_fits(int N, int T) { return N <= 1024 && (int64_t)N * T <= 4096; }

// Row norms of G and X, SampleA and SampleW of one layer in a single launch.  `tickets` are
// kPlanTicketBytes zeroed bytes of device memory that no other launch in flight uses; they are
// zero again when the launch has finished.
vcas_status plan_fused(const void *G, int K_out, const void *X, int K_in, int dtype, int N, int T, double budget_a,
                       double budget_w, int token_sampling, const vcas_rng &rng, float *uniforms, uint32_t *tickets,
                       const vcas_plan &pl, hipStream_t st)
{
    if (!plan_fused_fits(N, T)) return VCAS_EINVAL;
    const int per = dtype == VCAS_BF16 ? 8 : 4;
    PlanArgs a;
    a.G = static_cast<const uint4 *>(G);
    a.X = static_cast<const uint4 *>(X);
    a.groups_g = K_out / per;
    a.groups_x = K_in / per;
    a.N = N;
    a.T = T;
    a.budget_a = budget_a;
    a.budget_w = budget_w;
    a.token_sampling = token_sampling;
    a.job = {token_sampling ? uniforms : nullptr, rng.seed, rng.layer, 1u, rng.draw, rng.draw_offset};
    a.tickets = tickets;
    a.gsq = pl.gsq; a.gnorm = pl.gnorm; a.p = pl.p; a.maskA = pl.maskA; a.idxA = pl.idxA; a.cntA = pl.cntA;
    a.xsq = pl.xsq; a.score = pl.score; a.q = pl.q; a.maskW = pl.maskW; a.scaleW = pl.scaleW;
    a.idxW = pl.idxW; a.cntW = pl.cntW;
    const int R = N * T;
    const int need = ((a.groups_g > a.groups_x ? a.groups_g : a.groups_x) + 63) / 64;
    // two rows (a pair) per wavefront, sixteen wavefronts per workgroup
    const int blocks = (2 * R + 31) / 32;
#define VCAS_PLAN(B, C) hipLaunchKernelGGL((plan_fused_kernel<B, C>), dim3(blocks), dim3(kThreads), 0, st, a)
    if (dtype == VCAS_BF16) {
        if (need <= 2) VCAS_PLAN(true, 2);
        else if (need <= 4) VCAS_PLAN(true, 4);
        else VCAS_PLAN(true, 8);
    } else {
        if (need <= 2) VCAS_PLAN(false, 2);
        else if (need <= 4) VCAS_PLAN(false, 4);
        else VCAS_PLAN(false, 8);
    }
#undef VCAS_PLAN
    return launch_status();
}

}  // namespace vcas
