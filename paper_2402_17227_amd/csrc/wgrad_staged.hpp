// bf16 weight gradient with both operands gathered through the kept list, the scaled one multiplied on its way through registers.
//
// The scale lies on the contraction axis, so one operand has to be multiplied by it before the matrix instruction, rounded once.
// Done to fragments (an earlier form) every wavefront that reads a value scales it again, 20 vector instructions a fragment: 21 an
// MFMA with 128x128 tiles, 52 with 64x64.  Here both tiles of a step pass through registers into LDS, each value once, and the
// kernel is bound by operand loads: 32 KiB a step of 64 tokens and 128x128 tile, 0.55 us alone on a CU, 0.67 with two workgroups.
// Scaled in fragments, packed by a launch of its own, and here, us: 768 -> 3072, 1024 tokens 24.6, 28.7, 18.5; 3072 -> 768, 1891 tokens
// 43.5, 30.6, 24.9; 1024x1024, 1638 tokens 21.4, 26.7, 13.6; sixteen products of 768x768, 2836 tokens (the variance probe) 122 and
// 91.  The same bits as scaled in fragments.  A long contraction of many tiles stays with the packed form: its 256x256 tiles load half
// as much for a product, and neither operand passes through registers (api.hip has both sides of the line).
#pragma once

#include "wgrad_gather.hpp"

namespace vcas {

// WM x WN wavefronts share the tile, WK of them each block (they take the slices of a step in turn and their sums meet in LDS).
// SCALE_G: G's values are the scaled ones, else X's.
template <int BM, int BN, int WM, int WN, int WK, bool DIFF, bool SCALE_G>
__device__ __forceinline__ void wgrad_staged_tile(const GatherTask &q, int local_id)
{
    constexpr int NW = WM * WN * WK, NT = NW * 64, TM = BM / WM / 32, TN = BN / WN / 32, SK = 64, KS = SK / 16 / WK;
    constexpr int B_AT = SK * BM * 2, STAGE = SK * (BM + BN) * 2;
    constexpr int AQ = SK * BM / 8 / NT, BQ = SK * BN / 8 / NT, A_K = NT * 8 / BM, B_K = NT * 8 / BN;   // loads per thread and step, tokens between them
    static_assert(AQ >= 1 && BQ >= 1 && TM >= 1 && TN >= 1, "tile/wave mismatch");
    static_assert(A_K % 4 == 0 && B_K % 4 == 0, "the slot XORs of a thread's tokens are one");
    static_assert(WK == 1 || (WK - 1) * WM * WN * TM * TN * 4096 <= 2 * STAGE, "the partial blocks meet in the operand stages");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int total = q.tiles * q.splits;
    const int id = xcd_remap(local_id, total);
    if (id >= total) return;
    const int split = id / q.tiles, tile = id % q.tiles;
    const int K_in = q.K_in, K_out = q.K_out, R = q.R, tid = threadIdx.x;
    int tile_o, tile_c;   // panels of 4 column tiles: an XCD's run of workgroups covers a squarish patch of dW
    panel_order_rt(tile, q.tiles / q.tiles_n, q.tiles_n, 4, tile_o, tile_c);
    const int o0 = tile_o * BM, c0 = tile_c * BN;

    const int cnt = min(max(*q.cnt, 0), R);
    const int steps_all = (cnt + SK - 1) / SK;
    int per;
    const int active = wgrad_active_splits(steps_all, q.splits, kGatherMinTokens / SK, per);
    if (split >= active) return;
    const int s_begin = split * per, s_end = min(steps_all, s_begin + per), steps = s_end - s_begin;
    const int k_begin = s_begin * SK, k_end = min(cnt, s_end * SK);

    const __amdgpu_buffer_rsrc_t bufG = buffer_of(q.G, (uint32_t)((int64_t)R * K_out * 2)), bufX = buffer_of(q.X, (uint32_t)((int64_t)R * K_in * 2));
    const __amdgpu_buffer_rsrc_t bufI = buffer_of(q.idx, (uint32_t)cnt * 4u), bufS = buffer_of(q.row_scale, (uint32_t)R * 4u);
    const int a_k = tid / (BM / 8), b_k = tid / (BN / 8), a_c = tid % (BM / 8) * 8, b_c = tid % (BN / 8) * 8;
    const uint32_t a_col = o0 + a_c < K_out ? (uint32_t)(o0 + a_c) * 2u : kOutside, b_col = c0 + b_c < K_in ? (uint32_t)(c0 + b_c) * 2u : kOutside;
    const uint32_t a_pitch = (uint32_t)K_out * 2u, b_pitch = (uint32_t)K_in * 2u;
    const int a_put = split_col_at<BM>(a_k, a_c), b_put = B_AT + split_col_at<BN>(b_k, b_c);
    // Value n of step s is token token(n) of the step; tok[n] holds its row: the kept-list entry is fetched a step ahead of the row
    // (and issued before the row of the step in front: loads return in order).  Entries past the count read as zero and are not used.
    constexpr int NQ = AQ + BQ;
    float4 raw[2][NQ];
    uint32_t scale[2][NQ], tok[NQ];
    auto token = [&](int n) { return n < AQ ? a_k + n * A_K : b_k + (n - AQ) * B_K; };
#pragma unroll
    for (int n = 0; n < NQ; ++n) tok[n] = buffer_load1(bufI, (uint32_t)(k_begin + token(n)) * 4u);
    auto load = [&](auto n_, auto set_, int s, auto fast_) {
        constexpr int n = decltype(n_)::value, set = decltype(set_)::value;
        const int k = k_begin + s * SK + token(n);
        const uint32_t t = tok[n];
        const bool in = (decltype(fast_)::value || k < k_end) && t < (uint32_t)R;
        tok[n] = buffer_load1(bufI, (uint32_t)(k + SK) * 4u);
        if constexpr ((n < AQ) == SCALE_G) scale[set][n] = buffer_load1(bufS, in ? t * 4u : kOutside);
        // rows < 2^24 and pitches < 2^14 (checked on the host); a column outside the matrix adds an offset that is outside too
        if constexpr (n < AQ) raw[set][n] = buffer_load4(bufG, in ? __umul24(t, a_pitch) + a_col : kOutside);
        else raw[set][n] = buffer_load4(bufX, in ? __umul24(t, b_pitch) + b_col : kOutside);
    };
    auto put = [&](auto n_, auto set_) {
        constexpr int n = decltype(n_)::value, set = decltype(set_)::value;
        u32x4 w = __builtin_bit_cast(u32x4, raw[set][n]);
        if constexpr ((n < AQ) == SCALE_G) {
            const float f = __uint_as_float(scale[set][n]);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = pack_bf16(bf16_lo(w[e]) * f, bf16_hi(w[e]) * f);
        }
        *reinterpret_cast<u32x4 *>(smem + set * STAGE + (n < AQ ? a_put + n * (A_K * BM * 2) : b_put + (n - AQ) * (B_K * BN * 2))) = w;
    };

    const int wave = tid >> 6, wk = wave / (WM * WN), blk = wave % (WM * WN);
    const int wm0 = (blk / WN) * (BM / WM), wn0 = (blk % WN) * (BN / WN);
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    bf16x8 a[2][TM], b[2][TN];
    auto frags = [&](int stage, int t, auto set_) {
        constexpr int set = decltype(set_)::value;
        const unsigned char *at = smem + stage * STAGE;
#pragma unroll
        for (int i = 0; i < TM; ++i) a[set][i] = split_col_frag<BM>(at, wm0 + i * 32, t * WK + wk);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[set][j] = split_col_frag<BN>(at + B_AT, wn0 + j * 32, t * WK + wk);
    };
    auto mma = [&](auto set_) {
        constexpr int set = decltype(set_)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[set][i], b[set][j], acc[i][j], 0, 0, 0);
    };
    staged_loop<NQ, KS, TM * TN, 2 * (TM + TN), 14, 1>(steps, (k_end - k_begin) / SK, load, put, frags, mma);
    const bool mine = split_meet<TM, TN, WK>(smem, wk, blk, WM * WN, acc);
    gather_finish<TM, TN, DIFF>(q, acc, mine, active, split, tile, o0 + wm0, c0 + wn0, blk, WM * WN, smem);
}

template <int BM, int BN, int WM, int WN, int WK, bool DIFF>
__device__ __forceinline__ void wgrad_staged_body(const GatherTask &q, int local_id)
{
    if (q.scale_g) wgrad_staged_tile<BM, BN, WM, WN, WK, DIFF, true>(q, local_id);
    else wgrad_staged_tile<BM, BN, WM, WN, WK, DIFF, false>(q, local_id);
}

// Two stages of both tiles.
constexpr size_t staged_lds(int BM, int BN) { return 2 * 64 * 2 * (size_t)(BM + BN); }

}  // namespace vcas
