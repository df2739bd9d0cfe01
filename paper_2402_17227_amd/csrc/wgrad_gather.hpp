// Weight gradient with both operands gathered through the kept list (gfx950, fp32 and bf16):
//   dW[o,c] = sum over k < *cnt of scale[t] * G[t,o] * X[t,c],  t = idx[k]          (Sec. 4.2)
// or, for the variance probe (Alg. 1), the squared distance of that product from a given matrix,
// without storing the product.
//
// Three kernels: 32x32 fp32 tiles here, larger fp32 ones in f32_split.hpp, bf16 in wgrad_staged.hpp.
#pragma once

#include "staged_loop.hpp"

namespace vcas {

// How many of the launched split-K slices do work for a given number of
// contraction steps, and how many steps each takes.  Used by the GEMMs and by
// the reduction so that both agree.
__host__ __device__ inline int wgrad_active_splits(int steps_all, int splits, int min_steps, int &per)
{
    int active = splits < steps_all / min_steps ? splits : steps_all / min_steps;
    if (active < 1) active = 1;
    per = (steps_all + active - 1) / active;
    if (per < 1) per = 1;
    active = (steps_all + per - 1) / per;
    return active < 1 ? 1 : active;
}

// One product of a launch (device view).
struct GatherTask {
    const void *G, *X;           // [R,K_out], [R,K_in]
    const float *row_scale;      // by token
    const int32_t *idx, *cnt;    // kept list and its length
    float *dst, *partials;       // dW, and [split][K_out][K_in] where more than one slice is active
    const float *exact;          // DIFF: the matrix the product is compared with,
    double *sq_out;              //       and one sum of squared differences per tile
    int32_t R, K_in, K_out;
    int32_t scale_g;             // bf16: nonzero: the scale goes to the G side, else to the X side
    int32_t tiles_n, tiles, splits;
    int32_t first_wg;            // first workgroup id of this task's range (a multiple of 8)
};

constexpr int kGatherMinTokens = 128;   // tokens a split-K slice has at least

__device__ __forceinline__ void lds_direct_load4(i32x4 desc, uint32_t lds_base, uint32_t voffset)
{
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds" : : "s"(lds_base), "v"(voffset), "s"(desc) : "memory", "m0");
}

// The end of a tile: its sums (of the wavefronts that hold some) to memory, or (DIFF) their squared distance from q.exact.  row0,
// col0: this wavefront's first row and column of dW; blk of `blocks`: which of the tile's blocks it holds.
template <int TM, int TN, bool DIFF>
__device__ __forceinline__ void gather_finish(const GatherTask &q, const f32x16 (&acc)[TM][TN], bool mine, int active, int split,
                                              int tile, int row0, int col0, int blk, int blocks, unsigned char *smem)
{
    const int lane = threadIdx.x & 63, lane32 = lane & 31, K_in = q.K_in, K_out = q.K_out;
    if constexpr (DIFF) {
        double sum = 0.0;
        if (mine) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int o = row0 + i * 32 + acc_row(v);
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int c = col0 + j * 32 + lane32;
                        if (o < K_out && c < K_in) {
                            const double d = (double)acc[i][j][v] - (double)q.exact[(int64_t)o * K_in + c];
                            sum += d * d;
                        }
                    }
                }
        }
        sum = wave_exchange_sum(sum);
        __syncthreads();   // everybody is done with the stages and the partial blocks
        double *wsum = reinterpret_cast<double *>(smem);
        if (lane == 0 && mine) wsum[blk] = sum;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int w = 0; w < blocks; ++w) s += wsum[w];
            q.sq_out[tile] = s;
        }
    } else {
        if (!mine) return;
        float *dst = active == 1 ? q.dst : q.partials + (int64_t)split * K_out * K_in;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int o = row0 + i * 32 + acc_row(v);
                if (o >= K_out) continue;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int c = col0 + j * 32 + lane32;
                    if (c < K_in) dst[(int64_t)o * K_in + c] = acc[i][j][v];
                }
            }
    }
}

// fp32, on the fp32 matrix instruction.  Both tiles of a step lie in LDS as [64 tokens][128 bytes of columns], written by
// LDS-direct loads one step ahead; a step's tokens come from a 64-entry table in LDS that is itself fetched four steps ahead, its
// token scales from a second table, gathered with the tiles, and are multiplied into G's fragments.  Two stages, one barrier per step.
// WM x WN wavefronts share the tile, WK of them each block: they take different parts of every step
// and their sums meet in LDS at the end, in wavefront order.
template <int SK, int WM, int WN, int WK, bool DIFF>
__device__ __forceinline__ void wgrad_gather_body(const GatherTask &q, int local_id)
{
    constexpr int NW = WM * WN * WK, E = 4, PA = 128, PB = 128;   // bytes of columns in a row of either tile
    constexpr int BM = PA / E, BN = PB / E;                       // columns of a tile
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int AI = SK * PA / 1024 / NW, BI = SK * PB / 1024 / NW;   // LDS-direct loads per wavefront and step
    constexpr int B_AT = SK * PA, STAGE = SK * (PA + PB);
    static_assert(AI >= 1 && BI >= 1 && TM >= 1 && TN >= 1, "tile/wave mismatch");
    static_assert((WK - 1) * WM * WN * TM * TN * 4096 <= 2 * STAGE, "the partial blocks meet in the operand stages");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int TOK_AT = 2 * STAGE, SCL_AT = TOK_AT + 4 * 256;
    int32_t *tok = reinterpret_cast<int32_t *>(smem + TOK_AT);   // [4][64], step st in slot st & 3
    float *scl = reinterpret_cast<float *>(smem + SCL_AT);       // [4][64], step st in slot st & 3
    const int total = q.tiles * q.splits;
    const int id = xcd_remap(local_id, total);
    if (id >= total) return;
    const int split = id / q.tiles, tile = id % q.tiles;
    const int K_in = q.K_in, K_out = q.K_out, R = q.R;
    int tile_o, tile_c;   // panels of 4 column tiles: an XCD's run of workgroups covers a squarish patch of dW
    panel_order_rt(tile, q.tiles / q.tiles_n, q.tiles_n, 4, tile_o, tile_c);
    const int o0 = tile_o * BM, c0 = tile_c * BN;

    const int cnt = min(max(*q.cnt, 0), R);
    const int steps_all = (cnt + SK - 1) / SK;
    int per;
    const int active = wgrad_active_splits(steps_all, q.splits, kGatherMinTokens / SK, per);
    if (split >= active) return;
    const int s_begin = split * per, s_end = min(steps_all, s_begin + per), steps = s_end - s_begin;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const i32x4 descG = raw_descriptor(q.G, (uint32_t)((int64_t)R * K_out * E));
    const i32x4 descX = raw_descriptor(q.X, (uint32_t)((int64_t)R * K_in * E));
    const i32x4 descI = raw_descriptor(q.idx, (uint32_t)cnt * 4u);        // entries past the count read as zero
    const i32x4 descS = raw_descriptor(q.row_scale, (uint32_t)R * 4u);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    // the two halves of a wavefront read tokens k and k + 4 at once (see below): neighbouring rows change places wherever bit 2 of k
    // is set
    auto place = [](int k) { return k ^ ((k >> 2) & 1); };
    // load j of this wavefront fills 1024 / pitch rows; lane's row and the column bytes it fetches there
    uint32_t a_col[AI], b_col[BI];
    int a_k[AI], b_k[BI];
#pragma unroll
    for (int j = 0; j < AI; ++j) {
        a_k[j] = place((wave * AI + j) * (1024 / PA) + lane / (PA / 16));
        const int col = o0 + lane % (PA / 16) * (16 / E);
        a_col[j] = col < K_out ? (uint32_t)col * E : kOutside;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
        b_k[j] = place((wave * BI + j) * (1024 / PB) + lane / (PB / 16));
        const int col = c0 + lane % (PB / 16) * (16 / E);
        b_col[j] = col < K_in ? (uint32_t)col * E : kOutside;
    }
    auto load_tokens = [&](int st) {   // wavefront 0: the tokens of step st into their table
        if (wave == 0 && st < steps) {
            const int k = (s_begin + st) * SK + lane;   // lanes past SK fetch ahead, and nobody reads what they fetched
            lds_direct_load4(descI, __builtin_amdgcn_readfirstlane(lds0 + TOK_AT + (st & 3) * 256), (uint32_t)k * 4u);
        }
    };
    // byte offsets of step st's loads, from its tokens (which have landed)
    uint32_t a_off[AI], b_off[BI], s_off = kOutside;
    auto aim = [&](int st) {
        const int k0 = (s_begin + st) * SK;
        const int32_t *t_of = tok + (st & 3) * 64;
#pragma unroll
        for (int j = 0; j < AI; ++j) {
            const uint32_t t = (uint32_t)t_of[a_k[j]];
            const bool in = k0 + a_k[j] < cnt && t < (uint32_t)R && a_col[j] != kOutside;
            a_off[j] = in ? t * (uint32_t)(K_out * E) + a_col[j] : kOutside;
        }
#pragma unroll
        for (int j = 0; j < BI; ++j) {
            const uint32_t t = (uint32_t)t_of[b_k[j]];
            const bool in = k0 + b_k[j] < cnt && t < (uint32_t)R && b_col[j] != kOutside;
            b_off[j] = in ? t * (uint32_t)(K_in * E) + b_col[j] : kOutside;
        }
        const uint32_t t = (uint32_t)t_of[lane];
        s_off = k0 + lane < cnt && t < (uint32_t)R ? t * 4u : kOutside;
    };
    auto issue = [&](int st) {   // tiles and scales of step st at the offsets aimed at
        if (st >= steps) return;
#pragma unroll
        for (int j = 0; j < AI; ++j)
            lds_direct_load16(descG, __builtin_amdgcn_readfirstlane(lds0 + (st & 1) * STAGE + (wave * AI + j) * 1024), a_off[j], 0u);
#pragma unroll
        for (int j = 0; j < BI; ++j)
            lds_direct_load16(descX, __builtin_amdgcn_readfirstlane(lds0 + (st & 1) * STAGE + B_AT + (wave * BI + j) * 1024), b_off[j], 0u);
        if (wave == NW - 1)
            lds_direct_load4(descS, __builtin_amdgcn_readfirstlane(lds0 + SCL_AT + (st & 3) * 256), s_off);
    };
    auto landed = [&]() {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    const int wk = wave / (WM * WN), blkw = wave % (WM * WN);
    const int wm0 = (blkw / WN) * (BM / WM), wn0 = (blkw % WN) * (BN / WN);
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // Fragments of two parts of a step are held at a time: part z of step st into set z & 1, then its MFMAs.
    // A part is 8 tokens; the WK wavefronts of a block take them in turn.
    constexpr int PARTS = SK / 8 / WK;
    static_assert(PARTS % 2 == 0, "two fragment sets alternate over an even number of parts");
    float a[2][4][TM], b[2][4][TN];   // four MFMAs per part and block
    float4 s4[2];
    auto read = [&](int st, int z) {
        const unsigned char *tileA = smem + (st & 1) * STAGE, *tileB = tileA + B_AT;
        const float *sc = scl + (st & 3) * 64;
        const int part = z * WK + wk;
        // half h of the wavefront takes tokens 4h + e of the part, e < 4: the order of the contraction
        // is free, and the four scales of a half are then one 16-byte read
        const int r32 = lane & 31, h = lane >> 5;
        auto cell = [&](const unsigned char *t, int pitch, int col, int k) {
            return *reinterpret_cast<const float *>(t + place(k) * pitch + col * E);
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 8 * part + 4 * h + e;
#pragma unroll
            for (int i = 0; i < TM; ++i) a[z & 1][e][i] = cell(tileA, PA, wm0 + i * 32 + r32, k);
#pragma unroll
            for (int i = 0; i < TN; ++i) b[z & 1][e][i] = cell(tileB, PB, wn0 + i * 32 + r32, k);
        }
        s4[z & 1] = *reinterpret_cast<const float4 *>(sc + 8 * part + 4 * h);
    };
    auto mma = [&](int z) {
        const float4 sv = s4[z & 1];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            a[z & 1][0][i] = a[z & 1][0][i] * sv.x;
            a[z & 1][1][i] = a[z & 1][1][i] * sv.y;
            a[z & 1][2][i] = a[z & 1][2][i] * sv.z;
            a[z & 1][3][i] = a[z & 1][3][i] * sv.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[z & 1][e][i], b[z & 1][e][j], acc[i][j], 0, 0, 0);
    };

    // The barrier of a step sits ahead of its LAST part, whose fragments every wavefront then holds in
    // registers: the stage is free for the loads of step s + 2, and the first fragments of step s + 1 are
    // read under the last part's MFMAs instead of behind a barrier with the matrix cores idle.
    for (int d = 0; d < 4; ++d) load_tokens(d);
    landed();
    aim(0);
    issue(0);
    aim(1);
    issue(1);
    aim(2);
    landed();   // (the tiles of step 1 need not have: once per slice)
    if (steps > 0) read(0, 0);
    for (int s = 0; s < steps; ++s) {
#pragma unroll
        for (int z = 0; z < PARTS; ++z) {
            if (z + 1 < PARTS) {
                read(s, z + 1);
            } else {
                landed();   // tiles and scales of step s + 1, tokens of step s + 3
                issue(s + 2);
                load_tokens(s + 4);
                __builtin_amdgcn_sched_barrier(0);
                if (s + 1 < steps) read(s + 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            mma(z);
            __builtin_amdgcn_sched_barrier(0);
        }
        aim(s + 3);
    }

    const bool mine = split_meet<TM, TN, WK>(smem, wk, blkw, WM * WN, acc);
    gather_finish<TM, TN, DIFF>(q, acc, mine, active, split, tile, o0 + wm0, c0 + wn0, blkw, WM * WN, smem);
}

// ---- host ---------------------------------------------------------------------------------
constexpr int kGatherBatch = 16;
struct GatherBatch {
    GatherTask task[kGatherBatch];
    int32_t n;
};

// Edges of the output tiles: bf16 64 and 128 columns; fp32 32 (fp32 matrix instructions, the wavefronts of a workgroup share the
// contraction), 64 and 128 (bf16 parts, f32_split.hpp).
enum GatherTile { kSmallTile, kMidTile, kLargeTile };   // bf16 has no middle one
inline int gather_edge(int dtype, GatherTile tile)
{
    return dtype == VCAS_BF16 ? (tile == kLargeTile ? 128 : 64) : tile == kLargeTile ? 128 : tile == kMidTile ? 64 : 32;
}
inline int gather_tiles(int dtype, int K_out, int K_in, GatherTile tile)
{
    const int edge = gather_edge(dtype, tile);
    return ((K_out + edge - 1) / edge) * ((K_in + edge - 1) / edge);
}
// Tokens per contraction step (the unit of a split-K slice).
inline int gather_step(int dtype, GatherTile tile) { return dtype == VCAS_F32 && tile == kLargeTile ? 32 : 64; }

// n <= kGatherBatch products of one type in one launch; `splits` of each task is set by the caller (1
// with diff).  diff: the squared distances from `exact`, gather_tiles(...) sums per task in sq_out.
vcas_status wgrad_gather(GatherTask *tasks, int n, int dtype, GatherTile tile, bool diff, hipStream_t st);

// Can a tensor of this shape be addressed by 32-bit buffer offsets?  (bf16: always, by the limits of the
// GEMM calls; fp32 calls take any size.)
inline bool offsets_fit(const vcas_shape &s)
{
    const int64_t R = (int64_t)s.N * s.T, kmax = s.K_in > s.K_out ? s.K_in : s.K_out;
    return R * kmax * elem_bytes(s.dtype) < ((int64_t)1 << 31) && (int64_t)s.K_in * s.K_out * 4 <= ((int64_t)1 << 30);
}

}  // namespace vcas
