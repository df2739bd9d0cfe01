// fp32 gather-GEMMs of the VCAS backward pass (the fp32 configuration): small tiles on v_mfma_f32_32x32x2_f32, larger ones from
// bf16 parts.
// dgrad (Eq. 2, upper line) here and in f32_split.hpp, wgrad (Sec. 4.2) in wgrad_gather.hpp and f32_split.hpp.
// dgrad_f32_staged_kernel and wgrad_f32_far_kernel serve tensors that 32-bit buffer offsets do not reach: 64x64 output tiles, four
// wavefronts, operands staged through registers into k-major LDS tiles ([k][row], pitch 68 floats, so that fragment reads are 32 consecutive floats), contraction in steps of 16.
#include "f32_split.hpp"

namespace vcas {

// gemm_bf16.hip
vcas_status splitk_reduce(const float *partials, const int32_t *cntW, float *dW, int64_t R, int64_t elems, int splits,
                          int min_steps, int step, hipStream_t st);

namespace f32gemm {

constexpr int BM = 64, BN = 64, BKF = 16, PITCH = 68, NT = 256;
constexpr int TILE_FLOATS = BKF * PITCH;

__device__ __forceinline__ void mma_step(const float *As, const float *Bs, int wm0, int wn0, f32x16 &acc)
{
    const int lane = threadIdx.x & 63;
    const int r = lane & 31, h = lane >> 5;
#pragma unroll
    for (int kk = 0; kk < BKF; kk += 2) {
        const float a = As[(kk + h) * PITCH + wm0 + r];
        const float b = Bs[(kk + h) * PITCH + wn0 + r];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
    }
}

}  // namespace f32gemm

// ------------------------------------------------------------------ dgrad
//
// BM x BN output tile, WM x WN x WK wavefronts of one 32x32 block each.  The operand tiles go straight
// into LDS (buffer_load ... lds), NS stages of KSUB sub-tiles of 32 contraction elements.  Bound by the
// matrix cores (64 cycles for 2 elements of a 32x32 block); what keeps them busy is long steps (64
// elements between barriers) and several workgroups per CU, so two shallow stages beat a deep pipeline
// (768->3072, 4096 rows: 157 us = 123 TFLOP/s of 157 with two stages of 64, 179 with four of 32; the
// register-staged kernel with steps of 16 took 201).
// A sub-tile is
//   G: [row][32 k] rows of 128 bytes, slots swizzled by lds_off.  Lane half h of chunk c (8 elements)
//      reads slot 2c + h, four elements k = 8c + 4h + e, with one 16-byte read; the order of the
//      contraction is free, so MFMA e of the chunk takes element e of both halves.
//   W: [32 k][BN columns] as in memory; the two halves read rows k and k + 4 at once, which are put
//      into different banks by exchanging the halves of a 64-column row (BN = 64) or neighbouring
//      32-column rows (BN = 32) wherever bit 2 of k is set.
// WK > 1: the WK wavefronts of a block take different chunks of every step and their sums meet in LDS
// at the end, in wavefront order: a wavefront alone on its SIMD would be bound by its own chain of MFMAs.
template <int BM, int BN, int WM, int WN, int WK, int KSUB, int NS>
__device__ __forceinline__ void dgrad_direct_body(const DgradF32 &q)
{
    constexpr int NW = WM * WN * WK, NT = NW * 64, BKF = 32 * KSUB;
    static_assert(BM == WM * 32 && BN == WN * 32 && (BN == 32 || BN == 64), "one 32x32 block per wavefront");
    constexpr int AI = KSUB * BM / (8 * NW), BI = KSUB * BN / (8 * NW);   // LDS-direct loads per wavefront and step
    constexpr int B_ROWS = 256 / BN, B_SLOTS = BN / 4;         // k rows per W load, 16-byte slots per W row
    constexpr int SUB = (BM + BN) * 128, STAGE = KSUB * SUB, B_AT = BM * 128, B_PITCH = BN * 4;
    constexpr int LOADS = AI + BI, CHUNKS = 4 * KSUB / WK;
    static_assert(AI >= 1 && BI >= 1 && CHUNKS >= 1, "tile/wave mismatch");
    static_assert((WK - 1) * WM * WN * 4096 <= NS * STAGE, "the partial blocks meet in the operand stages");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int32_t *row_of = reinterpret_cast<int32_t *>(smem + NS * STAGE);
    float *scale_of = reinterpret_cast<float *>(row_of + BM);

    const float *G = q.G, *W = q.W, *p = q.p, *J = q.J;
    const int32_t *idxA = q.idxA;
    float *dX = q.dX;
    const int N = q.N, T = q.T, K_in = q.K_in, K_out = q.K_out, tiles_n = q.tiles_n;
    const int cnt = min(max(*q.cntA, 0), N);
    const int64_t M = (int64_t)cnt * T, R = (int64_t)N * T;
    const int compute = (int)((M + BM - 1) / BM) * tiles_n;
    const int compute8 = (compute + 7) / 8 * 8;
    if ((int)blockIdx.x >= compute8) {
        if (!q.fill_dropped) return;
        const int z = blockIdx.x - compute8;
        const int64_t d0 = (int64_t)(z / tiles_n) * BM;
        const int n0 = (z % tiles_n) * BN;
        if (d0 >= R - M) return;
        for (int r = threadIdx.x; r < BM; r += NT) {
            const int64_t d = d0 + r;
            row_of[r] = d < R - M ? nth_missing(idxA, cnt, (int)(d / T)) * T + (int)(d % T) : -1;
        }
        __syncthreads();
        for (int u = threadIdx.x; u < BM * (BN / 4); u += NT) {
            const int r = u / (BN / 4), col = n0 + (u % (BN / 4)) * 4;
            if (row_of[r] >= 0 && col < K_in)
                *reinterpret_cast<float4 *>(dX + (int64_t)row_of[r] * K_in + col) = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        return;
    }
    const int tile = xcd_remap(blockIdx.x, compute);
    if (tile >= compute) return;
    const int64_t m0 = (int64_t)(tile / tiles_n) * BM;
    const int n0 = (tile % tiles_n) * BN;
    float p_row = 0.0f;   // of row threadIdx.x: fetched here, needed in the epilogue only
    static_assert(NT >= BM, "a thread per row");
    if (threadIdx.x < BM) {
        const int64_t m = m0 + threadIdx.x;
        int32_t dst = -1;
        if (m < M) {
            const int s = idxA[m / T];
            if (s >= 0 && s < N) {
                dst = s * T + (int)(m % T);
                p_row = p[s];
            }
        }
        row_of[threadIdx.x] = dst;
    }
    __syncthreads();

    const i32x4 descG = raw_descriptor(G, (uint32_t)(R * K_out * 4));
    const i32x4 descW = raw_descriptor(W, (uint32_t)((int64_t)K_out * K_in * 4));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    // LDS row of k row k of W and slot XOR within it: involutions, so the lane that fills LDS row r,
    // slot s fetches k row place(r), slot s ^ flip(place(r))
    // load j of this wavefront: sub-tile and first row (of 8 rows of G, of B_ROWS k rows of W) within it
    auto a_sub = [&](int j) { return (wave * AI + j) / (BM / 8); };
    auto a_row = [&](int j) { return (wave * AI + j) % (BM / 8) * 8; };
    auto b_sub = [&](int j) { return (wave * BI + j) / (BN / 8); };
    auto b_row = [&](int j) { return (wave * BI + j) % (BN / 8) * B_ROWS; };
    auto place = [](int k) { return BN == 32 ? k ^ ((k >> 2) & 1) : k; };
    auto flip = [](int k) { return BN == 64 ? ((k >> 2) & 1) * 8 : 0; };
    uint32_t a_off[AI], b_off[BI];
#pragma unroll
    for (int j = 0; j < AI; ++j) {
        const int row = a_row(j) + (lane >> 3);
        const int32_t src = row_of[row];
        a_off[j] = src >= 0 ? (uint32_t)src * (uint32_t)K_out * 4u + (uint32_t)(a_sub(j) * 128 + ((lane & 7) ^ swz(row)) * 16) : kOutside;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
        const int krow = place(b_row(j) + lane / B_SLOTS);
        const int col = n0 + ((lane % B_SLOTS) ^ flip(krow)) * 4;
        b_off[j] = col < K_in ? ((uint32_t)(b_sub(j) * 32 + krow) * (uint32_t)K_in + (uint32_t)col) * 4u : kOutside;
    }
    const int steps = (K_out + BKF - 1) / BKF;
    const int tail_pieces = (K_out - (steps - 1) * BKF + 3) / 4;   // pieces of a G row that the last step still owns
    auto issue = [&](int stage, int step) {   // a step past the end fills a stage nobody reads and keeps the counts uniform
        const uint32_t kb = __builtin_amdgcn_readfirstlane(step * BKF * 4);
        const uint32_t wb = __builtin_amdgcn_readfirstlane(step * BKF * K_in * 4);
        const int pieces = step < steps - 1 ? 8 * KSUB : step == steps - 1 ? tail_pieces : 0;
#pragma unroll
        for (int j = 0; j < AI; ++j) {
            const int piece = a_sub(j) * 8 + ((lane & 7) ^ swz(a_row(j) + (lane >> 3)));
            const uint32_t dst = lds0 + stage * STAGE + a_sub(j) * SUB + a_row(j) * 128;
            lds_direct_load16(descG, __builtin_amdgcn_readfirstlane(dst), piece < pieces ? a_off[j] : kOutside, kb);
        }
#pragma unroll
        for (int j = 0; j < BI; ++j) {
            const uint32_t dst = lds0 + stage * STAGE + b_sub(j) * SUB + B_AT + b_row(j) * B_PITCH;
            lds_direct_load16(descW, __builtin_amdgcn_readfirstlane(dst), pieces ? b_off[j] : kOutside, wb);
        }
    };
#pragma unroll
    for (int d = 0; d < NS - 1; ++d) issue(d, d);

    const int wk = wave / (WM * WN), blk = wave % (WM * WN);
    const int wm0 = (blk / WN) * 32, wn0 = (blk % WN) * 32;
    const int r32 = lane & 31, h = lane >> 5;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    int stage = 0;
    for (int s = 0; s < steps; ++s) {
        wait_loads_outstanding<(NS - 2) * LOADS>();   // step s has landed, the younger ones may stay in flight
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage of step s - 1 has been read: its next loads go out now
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(stage == 0 ? NS - 1 : stage - 1, s + NS - 1);
        __builtin_amdgcn_sched_barrier(0);
        float4 a[CHUNKS];
        float b[CHUNKS][4];
#pragma unroll
        for (int q = 0; q < CHUNKS; ++q) {
            const int c = (wk * CHUNKS + q) & 3;
            const unsigned char *tileA = smem + stage * STAGE + ((wk * CHUNKS + q) >> 2) * SUB, *tileB = tileA + B_AT;
            a[q] = *reinterpret_cast<const float4 *>(tileA + lds_off(wm0 + r32, 2 * c + h));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 8 * c + 4 * h + e, col = wn0 + r32;
                b[q][e] = *reinterpret_cast<const float *>(tileB + place(k) * B_PITCH + (((col >> 2) ^ flip(k)) << 4) + (col & 3) * 4);
            }
        }
#pragma unroll
        for (int q = 0; q < CHUNKS; ++q) {
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q].x, b[q][0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q].y, b[q][1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q].z, b[q][2], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q].w, b[q][3], acc, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        stage = stage + 1 == NS ? 0 : stage + 1;
    }
    wait_loads_outstanding<0>();
    if (threadIdx.x < BM) scale_of[threadIdx.x] = 1.0f / p_row;
    __syncthreads();   // ... and every wavefront is done with the stages
    if (WK > 1) {
        float *part = reinterpret_cast<float *>(smem);
        if (wk > 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) part[(((wk - 1) * WM * WN + blk) * 16 + v) * 64 + lane] = acc[v];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int w = 1; w < WK; ++w)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = acc[v] + part[(((w - 1) * WM * WN + blk) * 16 + v) * 64 + lane];
    }
    const int col = n0 + wn0 + r32;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = wm0 + acc_row(v);
        if (row_of[r] >= 0 && col < K_in) {
            const int64_t at = (int64_t)row_of[r] * K_in + col;
            float val = acc[v] * scale_of[r];
            if (J) val = val * J[at];   // elementwise Jacobian of the layer below (App. E, proof of unbiasedness)
            dX[at] = val;
        }
    }
}

// Tiles whose wavefronts share the contraction: 32 rows with the body above, 64x64 from bf16 parts.
template <int BM, int BN, int WM, int WN, int WK>
__global__ __launch_bounds__(WM *WN *WK * 64) void dgrad_f32_kernel(DgradF32 q)
{
    if constexpr (BM == 64) dgrad_split_body<BM, BN, WM, WN, WK>(q, blockIdx.x);
    else dgrad_direct_body<BM, BN, WM, WN, WK, 2, WK == 8 ? 3 : 2>(q);
}

// Wide tiles from bf16 parts, eight wavefronts, OCC of them to a SIMD.  64x128 tiles are two workgroups to a CU, 128 VGPRs a wavefront: two
// values wait in scratch while the loops run, which do not touch it.
template <int BM, int BN, int OCC>
__global__ __launch_bounds__(512, OCC) void dgrad_f32_wide_kernel(DgradF32 q)
{
    dgrad_split_body<BM, BN, 2, 4, 1>(q, blockIdx.x);
}

// Both halves of a layer in one launch, see layer_bf16_kernel: dX in tiles of DM (64: as dgrad_f32_kernel, 128: as
// dgrad_f32_wide_kernel) in the ids below first_w, dW in tiles of DW.
template <int DM, int DW>
__global__ __launch_bounds__(512, 1) void layer_f32_kernel(DgradF32 q, GatherTask task, int first_w)
{
    if ((int)blockIdx.x < first_w) {
        if constexpr (DM == 64) dgrad_split_body<64, 64, 2, 2, 2>(q, blockIdx.x);
        else dgrad_split_body<128, 128, 2, 4, 1>(q, blockIdx.x);
    } else {
        if constexpr (DW == 64) wgrad_split_body<64, 64, 2, 2, 2, false>(task, (int)blockIdx.x - first_w);
        else wgrad_split_body<128, 128, 2, 4, 1, false>(task, (int)blockIdx.x - first_w);
    }
}

// dgrad for tensors of 2 GiB and more.
// grid: tiles_n * (ceil(R/64) + 1) + 8 workgroups.  The first ceil8(compute
// tiles) ids compute (spread over the XCDs), the next ones zero the rows of
// dropped samples, the rest exit.
__global__ __launch_bounds__(256) void dgrad_f32_staged_kernel(const float *__restrict__ G, const float *__restrict__ W,
                                                        const float *__restrict__ p,
                                                        const int32_t *__restrict__ idxA,
                                                        const int32_t *__restrict__ cntA, float *__restrict__ dX,
                                                        int N, int T, int K_in, int K_out, int tiles_n,
                                                        const float *__restrict__ J, int fill_dropped)
{
    using namespace f32gemm;
    __shared__ __attribute__((aligned(16))) float As[2][TILE_FLOATS];
    __shared__ __attribute__((aligned(16))) float Bs[2][TILE_FLOATS];
    __shared__ int32_t row_of[BM];
    __shared__ float scale_of[BM];

    const int cnt = min(max(*cntA, 0), N);
    const int64_t M = (int64_t)cnt * T, R = (int64_t)N * T;
    const int compute = (int)((M + BM - 1) / BM) * tiles_n;
    const int compute8 = (compute + 7) / 8 * 8;
    const int tid = threadIdx.x;

    if ((int)blockIdx.x >= compute8) {
        if (!fill_dropped) return;
        const int z = blockIdx.x - compute8;
        const int64_t d0 = (int64_t)(z / tiles_n) * BM;
        const int n0 = (z % tiles_n) * BN;
        if (d0 >= R - M) return;
        if (tid < BM) {
            const int64_t d = d0 + tid;
            row_of[tid] = d < R - M ? nth_missing(idxA, cnt, (int)(d / T)) * T + (int)(d % T) : -1;
        }
        __syncthreads();
        for (int u = tid; u < BM * (BN / 4); u += NT) {
            const int r = u / (BN / 4), col = n0 + (u % (BN / 4)) * 4;
            if (row_of[r] >= 0 && col < K_in)
                *reinterpret_cast<float4 *>(dX + (int64_t)row_of[r] * K_in + col) = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        return;
    }
    const int tile = xcd_remap(blockIdx.x, compute);
    if (tile >= compute) return;
    const int64_t m0 = (int64_t)(tile / tiles_n) * BM;
    const int n0 = (tile % tiles_n) * BN;
    if (tid < BM) {
        const int64_t m = m0 + tid;
        int32_t dst = -1;
        float sc = 0.0f;
        if (m < M) {
            const int s = idxA[m / T];
            if (s >= 0 && s < N) {
                dst = s * T + (int)(m % T);
                sc = 1.0f / (p[s]);
            }
        }
        row_of[tid] = dst;
        scale_of[tid] = sc;
    }
    __syncthreads();

    // G tile: 64 rows x 16 k, thread = (row tid/4, k-quad tid%4); W tile: 16 k x 64 cols, thread = (k tid/16, col-quad tid%16)
    const int a_row = tid >> 2, a_kq = tid & 3;
    const float *a_ptr = row_of[a_row] >= 0 ? G + (int64_t)row_of[a_row] * K_out : nullptr;
    const int b_k = tid >> 4, b_col = n0 + (tid & 15) * 4;
    // A step's MFMAs take a fifth of a microsecond and a workgroup often has its CU to itself, so the
    // global loads run DEPTH steps ahead of the step on the matrix cores, each step in a register set
    // of its own: set d holds step s = d (mod DEPTH) until the step before s has put it into LDS.
    constexpr int DEPTH = 4;
    float4 ra[DEPTH], rb[DEPTH];
    auto load = [&](int k0, float4 &qa, float4 &qb) {   // a step past the end loads zeros
        qa = make_float4(0.f, 0.f, 0.f, 0.f);
        qb = make_float4(0.f, 0.f, 0.f, 0.f);
        const int ka = k0 + a_kq * 4;
        if (a_ptr != nullptr && ka < K_out) qa = *reinterpret_cast<const float4 *>(a_ptr + ka);
        const int kb = k0 + b_k;
        if (kb < K_out && b_col < K_in) qb = *reinterpret_cast<const float4 *>(W + (int64_t)kb * K_in + b_col);
    };
    auto store = [&](int buf, const float4 &qa, const float4 &qb) {
        float *a = As[buf] + (a_kq * 4) * PITCH + a_row;
        a[0] = qa.x;
        a[PITCH] = qa.y;
        a[2 * PITCH] = qa.z;
        a[3 * PITCH] = qa.w;
        *reinterpret_cast<float4 *>(Bs[buf] + b_k * PITCH + (tid & 15) * 4) = qb;
    };

    const int wave = tid >> 6;
    const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;

    const int steps = (K_out + BKF - 1) / BKF;
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(d * BKF, ra[d], rb[d]);
    store(0, ra[0], rb[0]);
    __syncthreads();
    for (int s0 = 0; s0 < steps; s0 += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int s = s0 + d;
            if (s < steps) {   // the same for every thread
                const int cur = s & 1;
                load((s + DEPTH) * BKF, ra[d], rb[d]);   // set d (step s) went to LDS one step ago
                mma_step(As[cur], Bs[cur], wm0, wn0, acc);
                if (s + 1 < steps) store(cur ^ 1, ra[(d + 1) % DEPTH], rb[(d + 1) % DEPTH]);
                __syncthreads();
            }
        }
    }

    const int col = n0 + wn0 + (tid & 31);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = wm0 + acc_row(v);
        if (row_of[r] >= 0 && col < K_in) {
            const int64_t at = (int64_t)row_of[r] * K_in + col;
            float val = acc[v] * scale_of[r];
            if (J) val = val * J[at];   // elementwise Jacobian of the layer below (App. E, proof of unbiasedness)
            dX[at] = val;
        }
    }
}

// wgrad for tensors of 2 GiB and more.
// grid: splits * tiles workgroups rounded up to 8, split-major; see the bf16
// kernel for the split-K protocol (same partial buffers and reduction kernel).
__global__ __launch_bounds__(256) void wgrad_f32_far_kernel(const float *__restrict__ G, const float *__restrict__ X,
                                                        const float *__restrict__ row_scale,
                                                        const int32_t *__restrict__ idxW,
                                                        const int32_t *__restrict__ cntW, float *__restrict__ dW,
                                                        float *__restrict__ partials, int64_t R, int K_in, int K_out, int tiles_n, int tiles,
                                                        int splits, int min_steps)
{
    using namespace f32gemm;
    __shared__ __attribute__((aligned(16))) float As[2][TILE_FLOATS];
    __shared__ __attribute__((aligned(16))) float Bs[2][TILE_FLOATS];

    const int total = tiles * splits;
    const int id = xcd_remap(blockIdx.x, total);
    if (id >= total) return;
    const int split = id / tiles, tile = id % tiles;
    const int o0 = (tile / tiles_n) * BM, c0 = (tile % tiles_n) * BN;
    const int tid = threadIdx.x;

    const int64_t cnt = min((int64_t)max(*cntW, 0), R);
    const int steps_all = (int)((cnt + BKF - 1) / BKF);
    int per;
    const int active = wgrad_active_splits(steps_all, splits, min_steps, per);
    if (split >= active) return;
    const int s_begin = split * per, s_end = min(steps_all, s_begin + per);

    // both tiles: 16 tokens x 64 cols, thread = (token tid/16, col-quad tid%16)
    const int kk = tid >> 4, cq = (tid & 15) * 4;
    // Token indices and scales of CHUNK steps at a time go to LDS first (two dependent loads that
    // nothing else could hide); inside a chunk the row loads run DEPTH steps ahead of the MFMAs,
    // each step in a register set of its own, as in dgrad.
    constexpr int DEPTH = 4, CHUNK = 64;
    __shared__ int32_t tok_of[CHUNK * BKF];
    __shared__ float scale_of[CHUNK * BKF];
    float4 ra[DEPTH], rb[DEPTH];
    auto load = [&](int local_step, int local_steps, float4 &qa, float4 &qb) {   // past the chunk: zeros
        qa = make_float4(0.f, 0.f, 0.f, 0.f);
        qb = make_float4(0.f, 0.f, 0.f, 0.f);
        const int32_t t = local_step < local_steps ? tok_of[local_step * BKF + kk] : -1;
        if (t >= 0 && o0 + cq < K_out) qa = *reinterpret_cast<const float4 *>(G + (int64_t)t * K_out + o0 + cq);
        if (t >= 0 && c0 + cq < K_in) qb = *reinterpret_cast<const float4 *>(X + (int64_t)t * K_in + c0 + cq);
    };
    auto store = [&](int buf, int local_step, const float4 &qa, const float4 &qb) {
        const float sc = scale_of[local_step * BKF + kk];
        const float4 a = make_float4(qa.x * sc, qa.y * sc, qa.z * sc, qa.w * sc);
        *reinterpret_cast<float4 *>(As[buf] + kk * PITCH + cq) = a;
        *reinterpret_cast<float4 *>(Bs[buf] + kk * PITCH + cq) = qb;
    };

    const int wave = tid >> 6;
    const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;

    for (int chunk0 = s_begin; chunk0 < s_end; chunk0 += CHUNK) {
        const int local_steps = min(CHUNK, s_end - chunk0);
        __syncthreads();   // the previous chunk's table and tiles are no longer read
        for (int i = tid; i < local_steps * BKF; i += NT) {
            const int64_t k = (int64_t)chunk0 * BKF + i;
            int32_t t = -1;
            float sc = 0.0f;
            if (k < cnt) {
                const int32_t r = idxW[k];
                if (r >= 0 && r < R) {
                    t = r;
                    sc = row_scale[r];
                }
            }
            tok_of[i] = t;
            scale_of[i] = sc;
        }
        __syncthreads();
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) load(d, local_steps, ra[d], rb[d]);
        store(0, 0, ra[0], rb[0]);
        __syncthreads();
        for (int s0 = 0; s0 < local_steps; s0 += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                const int s = s0 + d;
                if (s < local_steps) {   // the same for every thread
                    const int cur = s & 1;
                    load(s + DEPTH, local_steps, ra[d], rb[d]);
                    mma_step(As[cur], Bs[cur], wm0, wn0, acc);
                    if (s + 1 < local_steps) store(cur ^ 1, s + 1, ra[(d + 1) % DEPTH], rb[(d + 1) % DEPTH]);
                    __syncthreads();
                }
            }
        }
    }

    float *dst = active == 1 ? dW : partials + (int64_t)split * K_out * K_in;
    const int c = c0 + wn0 + (tid & 31);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int o = o0 + wm0 + acc_row(v);
        if (o < K_out && c < K_in) dst[(int64_t)o * K_in + c] = acc[v];
    }
}

int wgrad_tiles_f32(int K_out, int K_in) { return ((K_out + 63) / 64) * ((K_in + 63) / 64); }

template <int BM, int BN, typename Kern>
static vcas_status launch_dgrad_f32(Kern kern, int threads, size_t operands, bool &allowed, DgradF32 q, hipStream_t st)
{
    const int64_t R = (int64_t)q.N * q.T;
    q.tiles_n = (q.K_in + BN - 1) / BN;
    const int64_t grid = q.tiles_n * ((R + BM - 1) / BM + 1) + 8;
    if (grid > (int64_t)1 << 30) return VCAS_EINVAL;
    const size_t lds = operands + BM * 8;   // behind the stages the row table and 1/p
    if (!allowed) {
        if (!allow_lds(kern, lds)) return VCAS_EHIP;
        allowed = true;
    }
    launch_timed(0, kern, dim3((unsigned)grid), dim3(threads), lds, st, q);
    return launch_status();
}

template <int BM, int BN, int WM, int WN, int WK>
static vcas_status launch_dgrad_shared(const DgradF32 &q, hipStream_t st)
{
    static bool allowed = false;
    constexpr size_t operands = BM == 64 ? split_lds(BM, BN, WK) : (WK == 8 ? 3 : 2) * 2 * (BM + BN) * 128;
    return launch_dgrad_f32<BM, BN>(dgrad_f32_kernel<BM, BN, WM, WN, WK>, WM * WN * WK * 64, operands, allowed, q, st);
}

template <int BM, int BN, int OCC>
static vcas_status launch_dgrad_wide(const DgradF32 &q, hipStream_t st)
{
    static bool allowed = false;
    return launch_dgrad_f32<BM, BN>(dgrad_f32_wide_kernel<BM, BN, OCC>, 512, split_lds(BM, BN, 1), allowed, q, st);
}

static int64_t tiles_of(int64_t rows, int K_in, int bm, int bn) { return (rows + bm - 1) / bm * ((K_in + bn - 1) / bn); }

// The largest tile that still gives most CUs one: larger tiles load and split fewer values per product.  All rows kept, us (rows x
// columns, contraction; 32x32 with eight wavefronts to a tile and 32x64 on the fp32 instruction, the others from bf16 parts;
// last the 64x64 tiles on the fp32 instruction that these replace):
//                        32x32   32x64   64x64  64x128 128x128 | 64x64 fp32
//    64x264,    136        6.3     6.9     8.4     9.0    11.4      8.4
//   256x768,    768       10.3    13.0    15.2    20.4    27.0     18.5
//   512x768,    768       16.8    13.6    15.3    20.2    27.0     18.8
//   300x1024,  4096       56.8    47.7    51.4    82.6   108       75.6
//  1024x768,    768       23.0    20.1    16.2    20.5    27.1     19.1
//  1024x768,   3072       67.2    62.0    44.7    64.0    83.1     58.7
//  4096x256,   1024       35.1    25.4    20.0    25.8    33.2     24.1
//  2048x768,    768       40.0    27.5    28.7    22.1    27.4     31.4
//  2048x768,   3072               96      84      78.5    87.3    118
//  4096x768,   3072              174     142     127     104      162
//  8192x1024,   264                       71      37.3    36.4     54
//  8192x1024,    64                       45      19.6    21.1     22
enum DgradF32Form { kShared32x32, kShared32x64, kShared64x64, kWide };   // each its own order of sums
static DgradF32Form dgrad_f32_form(int64_t rows, int K_in)
{
    if (tiles_of(rows, K_in, 32, 32) <= 256) return kShared32x32;
    if (tiles_of(rows, K_in, 32, 64) <= 256) return kShared32x64;
    return tiles_of(rows, K_in, 64, 64) <= 256 ? kShared64x64 : kWide;
}

vcas_status dgrad_f32(const vcas_shape &s, const void *G, const void *W, const float *p, const int32_t *idxA,
                      const int32_t *cntA, void *dX, const void *J, bool fill, int64_t expected_rows, hipStream_t st)
{
    const int64_t R = (int64_t)s.N * s.T;
    const int64_t rows = expected_rows > 0 && expected_rows < R ? expected_rows : R;
    if (!offsets_fit(s)) {   // larger tensors, which the fp32 calls have always taken
        const int tiles_n = (s.K_in + 63) / 64;
        const int64_t grid = tiles_n * ((R + 63) / 64 + 1) + 8;
        if (grid > (int64_t)1 << 30) return VCAS_EINVAL;
        launch_timed(0, dgrad_f32_staged_kernel, dim3((unsigned)grid), dim3(256), 0, st, static_cast<const float *>(G),
                     static_cast<const float *>(W), p, idxA, cntA, static_cast<float *>(dX), s.N, s.T, s.K_in, s.K_out,
                     tiles_n, static_cast<const float *>(J), fill ? 1 : 0);
        return launch_status();
    }
    DgradF32 q = {static_cast<const float *>(G), static_cast<const float *>(W), p, idxA, cntA, static_cast<float *>(dX),
                  static_cast<const float *>(J), s.N, s.T, s.K_in, s.K_out, 0, fill ? 1 : 0};
    switch (dgrad_f32_form(rows, s.K_in)) {
    case kShared32x32: return launch_dgrad_shared<32, 32, 1, 1, 8>(q, st);
    case kShared32x64: return launch_dgrad_shared<32, 64, 1, 2, 2>(q, st);
    case kShared64x64: return launch_dgrad_shared<64, 64, 2, 2, 2>(q, st);
    default: break;
    }
    // wide tiles (the same bits): two workgroups of 64x128 to a CU hide prologues and epilogues where a contraction is a few steps
    if (tiles_of(rows, s.K_in, 64, 128) <= 256 || s.K_out <= 128) return launch_dgrad_wide<64, 128, 4>(q, st);
    return launch_dgrad_wide<128, 128, 1>(q, st);
}

// Slices of 128x128 fp32 tiles: as many as give every CU at most one, eight at the most.
int wgrad_slices_large_f32(int K_out, int K_in, int64_t R, int fill)
{
    const int64_t tiles = gather_tiles(VCAS_F32, K_out, K_in, kLargeTile);
    int64_t n = (fill < 256 ? fill : 256) / tiles;
    if (n > R / kGatherMinTokens) n = R / kGatherMinTokens;
    return n > 8 ? 8 : n < 1 ? 1 : (int)n;
}

// Alone, reductions included, us (matrix, tokens; 32x32 tiles whose four wavefronts share each contraction, in slices;
// 64x64 and 128x128 tiles from bf16 parts, unsliced / in the best number of slices; what was taken before: 32x32, or 64x64
// on the fp32 instruction from 768 of them up):
//                       32x32     64x64        128x128     before
//   200x72,     100       5.7       7.0          9.6          5.7
//    72x456,   2000      11.3     30 / 11.7    63 / 16       11.3
//   256x256,   1024      10.4     18 / 10.5    36 / 13       10.4
//   384x576,     64       5.4       6.5                       5.4
//   384x576,    400      12.8      11.4                      12.8
//   384x576,   1000      16.4      18.5                      16.4
//   512x576,     64       6.0       6.5                       6.0
//   512x576,    400      13.7      11.4                      13.7
//   768x768,     64       7.1       6.7                       7.1
//   768x768,    256      10.3       9.2         13.7         10.3
//   768x768,   1024      25.0      18.4        36 / 21.8     25.0
//   768x768,   2048      42.4      30.8        65 / 27.1     42.4
//   768x768,   4096      77        55 / 51    123 / 38       77
//  1024x1024,  2048      53        34.8        65 / 35.2     53
//   768x3072,  1024      72        54.7        44.0          72
//  1608x1928,   170                28.2         15.2          24.1
//  4096x4096,   128                88          42.6          58.6
//  1536x768,    150      14.7      15.2         11.8, in three slices 15.4
//               400      22.5      21.9         19.2                  20.7
//               600                27.0         24.8                  23.1
//              1500                51.4         51.4                  31.8
//  2048x1024,   256      23.6      18.1         15.4, in two slices   23.4
//               600                30.4         27.2                  29.8
//               900                41.5         37.9                  35.1
//              3000               105           99.6                  77.2
// So 32x32 up to 64 tiles of 64x64 (100 where the tokens are few).  From 257 of those up (a second round of them) 128x128, in slices
// where what they save, 0.031 us a token, is more than adding them up costs.  In between by what a token costs: a 128x128 tile takes 2.2
// times as long for one as a 64x64 tile, and its slices and their reduction as long as 900 tokens.
static void wgrad_f32_form(const vcas_shape &s, int fill, int max_splits, int64_t tokens, GatherTile &tile, int32_t &splits)
{
    const int64_t R = (int64_t)s.N * s.T, t = tokens > 0 && tokens < R ? tokens : R;
    const int small = gather_tiles(VCAS_F32, s.K_out, s.K_in, kSmallTile), mid = gather_tiles(VCAS_F32, s.K_out, s.K_in, kMidTile);
    int slices = wgrad_slices_large_f32(s.K_out, s.K_in, R, fill);
    if (slices > max_splits) slices = max_splits;
    tile = kMidTile;
    splits = 1;
    if (mid <= 64 || (mid <= 100 && t <= 150)) {
        tile = kSmallTile;
        splits = (fill + fill / 3 + small - 1) / small;
        if (splits > max_splits) splits = max_splits;
    } else if (mid > 256) {
        tile = kLargeTile;
        const double saved = 0.031 * (double)t * (slices - 1) / slices, reduction = 4.5 + (double)slices * s.K_out * s.K_in / 600e3;
        if (saved > reduction) splits = slices;
    } else if ((double)t * (1.0 - 2.2 / slices) > 900.0) {
        tile = kLargeTile;
        splits = slices;
    }
}

static GatherTask wgrad_f32_task(const vcas_shape &s, const void *G, const void *X, const float *row_scale, const int32_t *idxW,
                                 const int32_t *cntW, float *dW)
{
    GatherTask q = {};
    q.G = G;
    q.X = X;
    q.row_scale = row_scale;
    q.idx = idxW;
    q.cnt = cntW;
    q.dst = dW;
    q.R = (int32_t)((int64_t)s.N * s.T);
    q.K_in = s.K_in;
    q.K_out = s.K_out;
    q.splits = 1;
    return q;
}

// max_splits: partial matrices there is room for; fill: workgroups the launch should have; tokens: how many are expected to be kept
// (0: unknown, all R)
vcas_status wgrad_f32(const vcas_shape &s, const void *G, const void *X, const float *row_scale, const int32_t *idxW,
                      const int32_t *cntW, float *dW, float *partials, int max_splits, int fill, int64_t tokens, hipStream_t st)
{
    constexpr int MIN_STEPS = 8;
    const int64_t R = (int64_t)s.N * s.T;
    if (offsets_fit(s)) {
        GatherTask q = wgrad_f32_task(s, G, X, row_scale, idxW, cntW, dW);
        q.partials = partials;
        GatherTile tile;
        wgrad_f32_form(s, fill, max_splits, tokens, tile, q.splits);
        const vcas_status rc = wgrad_gather(&q, 1, VCAS_F32, tile, false, st);
        if (rc != VCAS_OK) return rc;
        const int step = gather_step(VCAS_F32, tile);
        return splitk_reduce(partials, cntW, dW, R, (int64_t)s.K_out * s.K_in, q.splits, kGatherMinTokens / step, step, st);
    }
    int splits = max_splits;
    const int tiles_n = (s.K_in + 63) / 64;
    const int tiles = ((s.K_out + 63) / 64) * tiles_n;
    if (splits > 8) splits = 8;
    const int grid = (tiles * splits + 7) / 8 * 8;
    launch_timed(1, wgrad_f32_far_kernel, dim3(grid), dim3(256), 0, st, static_cast<const float *>(G),
                       static_cast<const float *>(X), row_scale, idxW, cntW, dW, partials, R, s.K_in, s.K_out, tiles_n,
                       tiles, splits, MIN_STEPS);
    if (hipGetLastError() != hipSuccess) return VCAS_EHIP;
    return splitk_reduce(partials, cntW, dW, R, (int64_t)s.K_out * s.K_in, splits, MIN_STEPS, f32gemm::BKF, st);
}

// Does an fp32 layer take both halves in one launch, and with which tiles?  Where each half's form (so that the bits are those of
// the halves apart) has one from bf16 parts, dW unsliced, and their tiles come to a CU each, a few left for more samples than
// expected.  Wide dX goes out in 128x128 tiles, which take longer than 64x128 ones: 0.007 us an element of the contraction,
// against a launch and 0.029 us a token for dW behind it.
bool layer_fits_f32(const vcas_shape &s, int64_t rows, int64_t tokens, int max_splits, int fill, int &dm, int &dw)
{
    if (!offsets_fit(s)) return false;
    const DgradF32Form form = dgrad_f32_form(rows, s.K_in);
    GatherTile tile;
    int32_t splits;
    wgrad_f32_form(s, fill, max_splits, tokens, tile, splits);
    if (form == kShared32x32 || form == kShared32x64 || tile == kSmallTile || splits > 1) return false;
    dm = form == kWide ? 128 : 64;
    dw = gather_edge(VCAS_F32, tile);
    if (form == kWide && tiles_of(rows, s.K_in, 64, 128) <= 256 && 7 * (int64_t)s.K_out > 5500 + 29 * tokens) return false;
    return tiles_of(rows, s.K_in, dm, dm) + gather_tiles(VCAS_F32, s.K_out, s.K_in, tile) <= 248;
}

template <int DM, int DW>
static vcas_status launch_layer_f32(DgradF32 q, GatherTask task, hipStream_t st)
{
    const int64_t R = (int64_t)q.N * q.T;
    q.tiles_n = (q.K_in + DM - 1) / DM;
    task.tiles_n = (q.K_in + DW - 1) / DW;
    task.tiles = (q.K_out + DW - 1) / DW * task.tiles_n;
    const int64_t first_w = (q.tiles_n * ((R + DM - 1) / DM + 1) + 15) / 8 * 8, grid = first_w + (task.tiles + 7) / 8 * 8;
    if (grid > (int64_t)1 << 30) return VCAS_EINVAL;
    constexpr size_t lds_d = split_lds(DM, DM, DM == 64 ? 2 : 1) + DM * 8, lds_w = split_lds(DW, DW, DW == 64 ? 2 : 1);
    constexpr size_t lds = lds_d > lds_w ? lds_d : lds_w;
    auto kern = layer_f32_kernel<DM, DW>;
    static bool allowed = false;
    if (!allowed) {
        if (!allow_lds(kern, lds)) return VCAS_EHIP;
        allowed = true;
    }
    launch_timed(0, kern, dim3((unsigned)grid), dim3(512), lds, st, q, task, (int)first_w);
    return launch_status();
}

// dX and dW of one layer whose plan is there, with the tiles of layer_fits_f32
vcas_status layer_f32(const vcas_shape &s, const void *G, const void *X, const void *W, const vcas_plan &pl, void *dX, float *dW,
                      int dm, int dw, hipStream_t st)
{
    const DgradF32 q = {static_cast<const float *>(G), static_cast<const float *>(W), pl.p, pl.idxA, pl.cntA, static_cast<float *>(dX),
                        nullptr, s.N, s.T, s.K_in, s.K_out, 0, 1};
    const GatherTask task = wgrad_f32_task(s, G, X, pl.scaleW, pl.idxW, pl.cntW, dW);
    if (dm == 64) return dw == 64 ? launch_layer_f32<64, 64>(q, task, st) : launch_layer_f32<64, 128>(q, task, st);
    return dw == 64 ? launch_layer_f32<128, 64>(q, task, st) : launch_layer_f32<128, 128>(q, task, st);
}

}  // namespace vcas
