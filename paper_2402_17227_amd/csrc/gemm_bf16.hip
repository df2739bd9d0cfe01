// bf16 MFMA gather-GEMM of the VCAS activation gradient (gfx950):
//   dgrad  dX[rows of kept samples] = (1/p_i) * G[row,:] W          (Eq. 2, upper line)
// A dense contraction over the kept rows only, on the matrix cores:
// v_mfma_f32_32x32x16_bf16, fp32 accumulation.  (The weight gradient is in wgrad_bf16.hip.)
//
// Tiling: a workgroup of WM x WN wavefronts owns a BM x BN output tile and walks the contraction
// in steps of 64, operand tiles double buffered in LDS.  The operand tiles never pass through
// registers: buffer loads write straight into LDS; W, which lies "the wrong way" for an MFMA
// lane (the contraction index is its slow dimension), stays as it is in memory, [64 k][columns],
// and ds_read_b64_tr_b16 transposes it on the way out.  The per-row 1/p goes into the epilogue.
#include <type_traits>

#include "mfma_common.hpp"

namespace vcas {

// ------------------------------------------------------------------ dgrad
//
// The operand tiles of dgrad never pass through registers: buffer loads write
// straight into LDS (16 bytes per lane, a wavefront fills 1 KiB of consecutive
// LDS per instruction).  G lands as [row][64 k] rows with the XOR slot swizzle
// realised by WHICH 16-byte piece of the row each lane fetches; W lands as it
// lies in memory, [64 k][BN n], its slots swizzled the same way, and is
// transposed on the way out of LDS by ds_read_b64_tr_b16 (a block of 16 lanes
// reads 4 k-rows x 16 columns and each lane receives one column's 4 k values).
// NS stages; the loads of step s+NS-1 are issued while step s is computed.  One
// barrier per step: before it every wavefront waits until its own loads of the
// step have landed (s_waitcnt vmcnt, the counter is in order), after it the
// stage computed in the previous step is free.
constexpr int kWholeStep = -100;   // SPQ: see below

// f(0), f(1), ... f(N-1) with the index as a constant
template <typename F, int... I>
__device__ __forceinline__ void for_constants_of(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void for_constants(F &&f)
{
    for_constants_of(f, std::make_integer_sequence<int, N>());
}

constexpr int kIdxStaged = 1024;   // kept-sample indices a workgroup stages in LDS ahead of the count

// One BM x BN output tile at (kept row m0, column n0).  idx_staged: the first `staged` entries of the kept list, in a
// stage that the prologue does not load before the row table is built.
// SPQ >= 0: one barrier at the top of every step; the loads of the next step are spread over the
// MFMAs of the first SPQ quarters of the current one (0: all issued right after the barrier).
// SPQ < 0 (two stages only): the barrier sits ahead of the step's LAST k-slice, the loads of the
// step after next go out one per -SPQ MFMAs from there, and the next step's first fragments are
// read under the last slice's MFMAs (256x256, one workgroup per CU: nothing else covers the
// wait for LDS behind a barrier there).
// SPQ = kWholeStep: all fragments of a step are read one step ahead.
template <int BM, int BN, int WM, int WN, int NS, int SPQ>
__device__ __forceinline__ void dgrad_bf16_tile(const uint16_t *__restrict__ G, const uint16_t *__restrict__ W,
                                                const float *__restrict__ p, const int32_t *__restrict__ idxA,
                                                const int32_t *idx_staged, int staged, uint16_t *__restrict__ dX,
                                                int N, int T, int K_in, int K_out, const uint16_t *__restrict__ J,
                                                float *__restrict__ sq_blocks, int64_t m0, int n0, int64_t M)
{
    constexpr int NW = WM * WN, NT = NW * 64;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int AI = BM / (8 * NW), BI = BN / (8 * NW);     // LDS-direct loads per wavefront and step
    constexpr int B_ROWS = 512 / BN, B_SLOTS = BN / 8;         // k rows per W load, 16-byte slots per W row
    // The stages of G lie in front of those of W, so that a stage is a constant within the 64 KiB that an LDS instruction
    // adds to its address register, and all stages share the registers.  The 256x256 tile then takes 217 VGPRs; with G and W
    // of a stage side by side, 64 KiB apart, it took 251, two wavefronts filled a SIMD, and the norm passes of a
    // stack's other streams waited for it to end (four chained layers of 1024x1024, 16 samples of 1024 rows: 315 and 302 us).
    constexpr int STAGE = (BM + BN) * 128, A_STAGE = BM * 128, B_STAGE = BN * 128, B_AT = NS * A_STAGE, B_PITCH = BN * 2;
    constexpr int LOADS = AI + BI;
    static_assert(AI >= 1 && BI >= 1 && BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile/wave mismatch");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int32_t *row_of = reinterpret_cast<int32_t *>(smem + NS * STAGE);
    float *scale_of = reinterpret_cast<float *>(row_of + BM);
    const int64_t R = (int64_t)N * T;
    __syncthreads();   // idx_staged complete
    for (int r = threadIdx.x; r < BM; r += NT) {
        const int64_t m = m0 + r;
        int32_t dst = -1;
        if (m < M) {
            const int j = (int)(m / T);
            const int s = j < staged ? idx_staged[j] : idxA[j];
            if (s >= 0 && s < N) dst = s * T + (int)(m % T);
        }
        row_of[r] = dst;
    }
    __syncthreads();

    const i32x4 descG = raw_descriptor(G, (uint32_t)(R * K_out * 2));
    const i32x4 descW = raw_descriptor(W, (uint32_t)((int64_t)K_out * K_in * 2));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    // G load j: rows (wave*AI + j)*8 + lane/8, LDS slot lane%8 <- the row's 16-byte piece (slot ^ swz)
    // W load j: k rows (wave*BI + j)*B_ROWS + lane/B_SLOTS, LDS slot lane%B_SLOTS <- column chunk (slot ^ wswz)
    uint32_t a_off[AI], b_off[BI];
#pragma unroll
    for (int j = 0; j < AI; ++j) {
        const int row = (wave * AI + j) * 8 + (lane >> 3);
        const int32_t src = row_of[row];
        a_off[j] = src >= 0 ? (uint32_t)src * (uint32_t)K_out * 2u + (uint32_t)(((lane & 7) ^ swz(row)) * 16) : kOutside;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
        const int krow = (wave * BI + j) * B_ROWS + lane / B_SLOTS;
        const int col = n0 + ((lane % B_SLOTS) ^ wswz(krow)) * 8;
        b_off[j] = col < K_in ? ((uint32_t)krow * (uint32_t)K_in + (uint32_t)col) * 2u : kOutside;
    }
    const int steps = (K_out + BK - 1) / BK;
    // 16-byte pieces of a G row that the last step still owns (8 unless K_out is ragged).  The
    // pieces behind them lie in the NEXT row of G: they meet zero rows of W, but zero times
    // whatever that row holds (a NaN, an Inf, a row nobody has written) is not zero, so they are
    // not fetched.
    const int tail_pieces = (K_out - (steps - 1) * BK + 7) / 8;
    // the d-th of the LOADS loads of contraction step `step` into stage `stage`: G and W pieces alternate
    auto issue_nth = [&](int d, int stage, int step) {
        const uint32_t a_dst = __builtin_amdgcn_readfirstlane(lds0 + stage * A_STAGE + wave * AI * 1024);
        const uint32_t b_dst = __builtin_amdgcn_readfirstlane(lds0 + B_AT + stage * B_STAGE + wave * BI * 1024);
        const uint32_t kb = __builtin_amdgcn_readfirstlane(step * BK * 2);
        const uint32_t wb = __builtin_amdgcn_readfirstlane(step * BK * K_in * 2);
        const int pieces = step == steps - 1 ? tail_pieces : 8;
        int seen = 0;
#pragma unroll
        for (int j = 0; j < (AI > BI ? AI : BI); ++j) {
            if (j < AI) {
                if (seen == d) {
                    const int piece = (lane & 7) ^ swz((wave * AI + j) * 8 + (lane >> 3));
                    lds_direct_load16(descG, a_dst + j * 1024, piece < pieces ? a_off[j] : kOutside, kb);
                }
                ++seen;
            }
            if (j < BI) {
                if (seen == d) lds_direct_load16(descW, b_dst + j * 1024, b_off[j], wb);
                ++seen;
            }
        }
    };
    // The same inside the unrolled part of a loop, where every load is whole and the stage is a constant: one
    // scalar add and the load.  With one or two wavefronts per SIMD a loop is bound by what it issues; the
    // lane reads, multiplies and selects of issue_nth for eight loads cost a 256x256 step 5 %, the steps
    // of smaller tiles up to a third.
    const uint32_t a_lds = __builtin_amdgcn_readfirstlane(lds0 + wave * AI * 1024);
    const uint32_t b_lds = __builtin_amdgcn_readfirstlane(lds0 + B_AT + wave * BI * 1024);
    auto issue_whole = [&](auto stage_, auto d_, uint32_t kb, uint32_t wb) {
        constexpr int d = decltype(d_)::value, stage = decltype(stage_)::value, LO = AI < BI ? AI : BI;
        // G and W alternate while both have loads left, then the rest of the longer one
        constexpr bool of_g = d < 2 * LO ? d % 2 == 0 : AI > BI;
        constexpr int j = d < 2 * LO ? d / 2 : d - LO;
        if constexpr (of_g) lds_direct_load16_at<stage * A_STAGE + j * 1024>(descG, a_lds, a_off[j], kb);
        else lds_direct_load16_at<stage * B_STAGE + j * 1024>(descW, b_lds, b_off[j], wb);
    };
    const uint32_t w_step = (uint32_t)BK * K_in * 2;   // bytes from a step of W to the next (of G: 2 BK)
    const int whole = steps - (tail_pieces < 8 ? 1 : 0);   // steps that fetch all of their 16-byte pieces
    // One k-slice's fragments out of a stage
    const int r32 = lane & 31, h = lane >> 5;
    const int blk = lane >> 4, sl = lane & 15;    // 16-lane block and lane within it
    const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
    // Byte offsets of a lane's piece of G at each k-slice, rows wm0 + r32: 64 rows on they are the same; 32 rows on the
    // XOR flips bit 2 of the slot, which is the piece of slice ks ^ 2.
    uint32_t a_at[BK / 16];
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) a_at[ks] = lds_off(wm0 + r32, ks * 2 + h);
    auto read_slice = [&](int stage, int ks, bf16x8(&fa)[TM], bf16x8(&fb)[TN]) {
        const unsigned char *tileA = smem + stage * A_STAGE;
        const unsigned char *tileB = smem + B_AT + stage * B_STAGE;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[i] = *reinterpret_cast<const bf16x8 *>(tileA + a_at[(i & 1) ? ks ^ 2 : ks] + i * 4096);
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            bf16x4 half[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int k = ks * 16 + (blk >> 1) * 8 + e * 4 + (sl >> 2);
                const int col = wn0 + i * 32 + (blk & 1) * 16 + (sl & 3) * 4;
                const unsigned char *src = tileB + k * B_PITCH + (((col >> 3) ^ wswz(k)) << 4) + (col & 7) * 2;
                half[e] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    (__attribute__((address_space(3))) bf16x4 *)(src));
            }
            fb[i] = __builtin_shufflevector(half[0], half[1], 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };
    // prologue: steps 0 .. NS-2 in flight (a step past the end fills a stage nobody reads and keeps the counts uniform)
#pragma unroll
    for (int d = 0; d < NS - 1; ++d)
#pragma unroll
        for (int q = 0; q < LOADS; ++q) issue_nth(q, d, d < steps ? d : steps + 64);
    // 1/p of the tile's rows is needed in the epilogue only: fetched behind the first tile loads
    for (int r = threadIdx.x; r < BM; r += NT) {
        const int32_t dst = row_of[r];
        scale_of[r] = dst >= 0 ? 1.0f / p[dst / T] : 0.0f;
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    constexpr int KS = BK / 16, MM = TM * TN, SPAN = KS * MM * (SPQ > 0 ? SPQ : 0) / 4;
    // One contraction step on stage `stage`; the loads of step `nstep` go to stage `nstage` (fast: whole
    // ones, at kb and wb).  Fragments of two k-slices are read ahead; load d goes out after MFMA number
    // d*SPAN/LOADS.
    auto step_body = [&](int stage, auto nstage_, int nstep, auto fast_, uint32_t kb, uint32_t wb) {
        bf16x8 a[2][TM], b[2][TN];
        auto issue = [&](auto d_) {
            if (decltype(fast_)::value) issue_whole(nstage_, d_, kb, wb);
            else issue_nth(decltype(d_)::value, decltype(nstage_)::value, nstep);
        };
        if (SPQ == 0) {
            for_constants<LOADS>([&](auto d_) { issue(d_); });
            __builtin_amdgcn_sched_barrier(0);
        }
        read_slice(stage, 0, a[0], b[0]);
        if (KS > 1) read_slice(stage, 1, a[1], b[1]);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks & 1][i], b[ks & 1][j], acc[i][j], 0, 0, 0);
                    if (SPQ > 0) {
                        const int m = ks * MM + i * TN + j;
                        for_constants<LOADS>([&](auto d_) {
                            if (decltype(d_)::value * SPAN / LOADS == m) {
                                __builtin_amdgcn_sched_barrier(0);
                                issue(d_);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        });
                    }
                }
            if (ks + 2 < KS) read_slice(stage, ks + 2, a[ks & 1], b[ks & 1]);
        }
    };

    if constexpr (SPQ == kWholeStep) {
        // Every fragment of a step is in registers before its first MFMA: the fragments of step s + 1 are read
        // while step s is on the matrix cores, and its stage is free for the loads of step s + NS as soon as
        // the barrier says that everybody holds it.
        static_assert(NS % 2 == 0, "fragment sets and stages repeat together");
        bf16x8 a[2][KS][TM], b[2][KS][TN];
        wait_loads_outstanding<(NS - 2) * LOADS>();
        __syncthreads();   // step 0 has landed (and nobody needs the staged kept list any more)
#pragma unroll
        for (int q = 0; q < LOADS; ++q) issue_nth(q, NS - 1, NS - 1 < steps ? NS - 1 : steps + 64);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) read_slice(0, ks, a[0][ks], b[0][ks]);
        uint32_t kb = NS * BK * 2, wb = NS * w_step;   // where step s + NS starts in G and W
        auto step = [&](int s, auto t_, auto fast_) {
            constexpr int t = decltype(t_)::value, P = t & 1;   // t = s mod NS
            constexpr bool fast = decltype(fast_)::value;
            wait_loads_outstanding<(NS - 2) * LOADS>();
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            const int after = s + NS < steps ? s + NS : steps + 64;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[P][ks][i], b[P][ks][j], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                read_slice((t + 1) % NS, ks, a[P ^ 1][ks], b[P ^ 1][ks]);
                for_constants<LOADS>([&](auto q_) {
                    constexpr int q = decltype(q_)::value;
                    if (q * KS / LOADS == ks) {
                        if (fast) issue_whole(t_, q_, kb, wb);
                        else issue_nth(q, t, after);
                    }
                });
                __builtin_amdgcn_sched_barrier(0);
            }
            kb += BK * 2;
            wb += w_step;
        };
        int s = 0;
        for (; s + 2 * NS <= whole; s += NS)
            for_constants<NS>([&](auto t_) { step(s + decltype(t_)::value, t_, std::true_type{}); });
        for (; s < steps; s += NS)
            for_constants<NS>([&](auto t_) {
                if (s + decltype(t_)::value < steps) step(s + decltype(t_)::value, t_, std::false_type{});
            });
    } else if constexpr (SPQ < 0) {
        // Two stages, the barrier ahead of the step's LAST k-slice.  By then every wavefront holds that
        // slice's fragments in registers, so the stage is free: the loads of step s+2 go out there, one
        // per MFMA, and the first fragments of step s+1 are read under the last slice's MFMAs, so that no wavefront sits behind the barrier waiting for LDS.
        static_assert(NS == 2 && KS >= 2 && KS % 2 == 0, "two fragment sets alternate over an even number of slices");
        static_assert(MM >= LOADS, "all of a step's loads go out during one slice");
        bf16x8 a[2][TM], b[2][TN];
        wait_loads_outstanding<0>();
        __syncthreads();                           // step 0 has landed
#pragma unroll
        for (int d = 0; d < LOADS; ++d) issue_nth(d, 1, 1 < steps ? 1 : steps + 64);
        read_slice(0, 0, a[0], b[0]);
        uint32_t kb = 2 * BK * 2, wb = 2 * w_step;   // where step s + 2 starts in G and W
        auto step = [&](int s, auto t_, auto fast_) {
            constexpr int cur = decltype(t_)::value;   // s mod 2
            constexpr bool fast = decltype(fast_)::value;
            const int after2 = s + 2 < steps ? s + 2 : steps + 64;
            __builtin_amdgcn_sched_barrier(0);
            read_slice(cur, 1, a[1], b[1]);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (ks == KS - 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    wait_loads_outstanding<0>();   // step s+1: all of its loads have been issued by now
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // ... and this stage has been read
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                    read_slice(cur ^ 1, 0, a[0], b[0]);
                }
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks & 1][i], b[ks & 1][j], acc[i][j], 0, 0, 0);
                        const int q = i * TN + j;   // one load per MFMA of the last slice
                        if (ks == KS - 1 && q < LOADS) {
                            __builtin_amdgcn_sched_barrier(0);
                            if (fast)
                                for_constants<LOADS>([&](auto q_) {
                                    if (decltype(q_)::value == q) issue_whole(t_, q_, kb, wb);
                                });
                            else
                                issue_nth(q, cur, after2);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                if (ks + 2 < KS) read_slice(cur, ks + 2, a[ks & 1], b[ks & 1]);
            }
            kb += BK * 2;
            wb += w_step;
        };
        int s = 0;
        for (; s + 4 <= whole; s += 2) {
            step(s, std::integral_constant<int, 0>(), std::true_type{});
            step(s + 1, std::integral_constant<int, 1>(), std::true_type{});
        }
        for (; s < steps; s += 2) {
            step(s, std::integral_constant<int, 0>(), std::false_type{});
            if (s + 1 < steps) step(s + 1, std::integral_constant<int, 1>(), std::false_type{});
        }
    } else {
        uint32_t kb = (NS - 1) * BK * 2, wb = (NS - 1) * w_step;   // where step s + NS - 1 starts in G and W
        auto step = [&](int s, auto t_, auto fast_) {
            constexpr int t = decltype(t_)::value;   // s mod NS
            // the NS-2 younger steps may stay in flight; step s must have landed
            wait_loads_outstanding<(NS - 2) * LOADS>();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const int nxt = s + NS - 1;
            __builtin_amdgcn_sched_barrier(0);
            step_body(t, std::integral_constant<int, (t + NS - 1) % NS>(), nxt < steps ? nxt : steps + 64, fast_, kb, wb);
            __builtin_amdgcn_sched_barrier(0);
            kb += BK * 2;
            wb += w_step;
        };
        int s = 0;
        for (; s + 2 * NS - 1 <= whole; s += NS)
            for_constants<NS>([&](auto t_) { step(s + decltype(t_)::value, t_, std::true_type{}); });
        for (; s < steps; s += NS)
            for_constants<NS>([&](auto t_) {
                if (s + decltype(t_)::value < steps) step(s + decltype(t_)::value, t_, std::false_type{});
            });
    }
    wait_loads_outstanding<0>();

    // Epilogue.  An MFMA lane holds one column of 16 rows, so stores straight from the
    // accumulators would be 64-byte pieces, 64 instructions per wavefront.  Instead every wavefront
    // passes its (TM*32) x 64 sub-tile through LDS (the operand stages are free by now): rounded
    // values in, 128-byte rows (whole cache lines) out, 16 bytes per lane.  Row `row` of the strip
    // keeps logical 16-byte slot s at slot s ^ esw(row), so that the two rows a write instruction
    // touches per half-wavefront fall into different banks.
    static_assert(TN == 2, "a staged row is 64 columns = 128 bytes");
    static_assert(NW * TM * 4096 <= NS * STAGE, "the output strips are staged in the operand stages");
    __syncthreads();   // every wavefront is done with the stages
    unsigned char *strip = smem + wave * (TM * 4096);
    auto esw = [](int row) { return (row & 1) << 2; };
    if (J) {
        // Elementwise Jacobian of the layer below (App. E, proof of unbiasedness), same layout as
        // dX: its sub-tile is fetched into the strip first (zeros for rows and columns that are not
        // stored), in the layout the results will have; each lane then picks up the values at its
        // own column and multiplies before the one rounding.
        const i32x4 descJ = raw_descriptor(J, (uint32_t)(R * K_in * 2));
        const uint32_t strip_lds = __builtin_amdgcn_readfirstlane(lds0 + wave * (TM * 4096));
#pragma unroll
        for (int q = 0; q < TM * 4; ++q) {
            const int row = q * 8 + (lane >> 3);
            const int32_t dst = row_of[wm0 + row];
            const int col = n0 + wn0 + (((lane & 7) ^ esw(row)) << 3);
            const uint32_t off = dst >= 0 && col < K_in ? ((uint32_t)dst * (uint32_t)K_in + (uint32_t)col) * 2u : kOutside;
            lds_direct_load16(descJ, strip_lds + q * 1024, off, 0u);
        }
        wait_loads_outstanding<0>();
        asm volatile("" ::: "memory");
    }
    // A lane rounds its column's values of two neighbouring rows into one dword; neighbouring lanes
    // then trade halves (one DPP move, one byte permute) so that each owns two adjacent columns of
    // one row.  A dropped row has scale 0 and a column past K_in met zero columns of W, so what is
    // not stored arrives as zero and counts as zero in the block sums.  All LDS reads of a group
    // of cells come before its writes: the compiler cannot tell the strip from the row tables.
    const bool odd = lane & 1;
    const uint32_t halves = odd ? 0x03020706u : 0x05040100u;   // even: (mine.lo, other.lo); odd: (other.hi, mine.hi)
    auto fill_strip = [&](auto with_jacobian) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float4 sc[4];
#pragma unroll
            for (int g = 0; g < 4; ++g)
                sc[g] = *reinterpret_cast<const float4 *>(scale_of + wm0 + i * 32 + g * 8 + (lane >> 5) * 4);
            uint16_t jw[16][TN];
            if (with_jacobian) {
                // the Jacobian's values at this lane's own column, rows acc_row(v)
#pragma unroll
                for (int v = 0; v < 16; ++v)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int row = i * 32 + acc_row(v);
                        const int slot = j * 4 + ((lane & 31) >> 3);
                        jw[v][j] = *reinterpret_cast<const uint16_t *>(strip + row * 128 + ((slot ^ esw(row)) << 4) +
                                                                      (lane & 7) * 2);
                    }
            }
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                const int row = i * 32 + acc_row(v) + (odd ? 1 : 0);
                const float sc_e = (v & 2) ? sc[v >> 2].z : sc[v >> 2].x, sc_o = (v & 2) ? sc[v >> 2].w : sc[v >> 2].y;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    float mine_e = acc[i][j][v] * sc_e, mine_o = acc[i][j][v + 1] * sc_o;
                    if (with_jacobian) {
                        mine_e = mine_e * __uint_as_float((uint32_t)jw[v][j] << 16);
                        mine_o = mine_o * __uint_as_float((uint32_t)jw[v + 1][j] << 16);
                    }
                    const uint32_t mine = pack_bf16(mine_e, mine_o);
                    const uint32_t other = __float_as_uint(dpp_move<0xB1>(__uint_as_float(mine)));
                    const int slot = j * 4 + ((lane & 31) >> 3);
                    *reinterpret_cast<uint32_t *>(strip + row * 128 + ((slot ^ esw(row)) << 4) + ((lane >> 1) & 3) * 4) =
                        __builtin_amdgcn_perm(other, mine, halves);
                }
            }
        }
    };
    if (J) fill_strip(std::true_type{});
    else fill_strip(std::false_type{});
    __builtin_amdgcn_wave_barrier();   // the strip is this wavefront's own: its LDS accesses execute in order
    int32_t dst_of[TM * 4];
    uint4 val[TM * 4];
#pragma unroll
    for (int q = 0; q < TM * 4; ++q) {
        const int row = q * 8 + (lane >> 3);
        dst_of[q] = row_of[wm0 + row];
        val[q] = *reinterpret_cast<const uint4 *>(strip + row * 128 + ((lane & 7) << 4));
    }
#pragma unroll
    for (int q = 0; q < TM * 4; ++q) {
        const int row = q * 8 + (lane >> 3);
        const int col = n0 + wn0 + (((lane & 7) ^ esw(row)) << 3);
        if (dst_of[q] >= 0 && col < K_in) *reinterpret_cast<uint4 *>(dX + (int64_t)dst_of[q] * K_in + col) = val[q];
    }
    if (sq_blocks) {
        // Sums of squares of the stored values by blocks of 64 columns (this wavefront's strip is
        // exactly one), pairwise with neighbours first: a lane adds its eight columns (three levels),
        // the eight lanes of a row the rest.  Four neighbouring blocks of a row lie side by side:
        // sq_blocks[((blk / 4) * R + row) * 4 + blk % 4].
        const int blk = (n0 + wn0) >> 6;
        const int nb = (K_in + 63) >> 6;
#pragma unroll
        for (int q = 0; q < TM * 4; ++q) {
            const uint4 w = val[q];
            const float q0 = bf16_lo(w.x) * bf16_lo(w.x), q1 = bf16_hi(w.x) * bf16_hi(w.x);
            const float q2 = bf16_lo(w.y) * bf16_lo(w.y), q3 = bf16_hi(w.y) * bf16_hi(w.y);
            const float q4 = bf16_lo(w.z) * bf16_lo(w.z), q5 = bf16_hi(w.z) * bf16_hi(w.z);
            const float q6 = bf16_lo(w.w) * bf16_lo(w.w), q7 = bf16_hi(w.w) * bf16_hi(w.w);
            float t = ((q0 + q1) + (q2 + q3)) + ((q4 + q5) + (q6 + q7));
            t = t + dpp_move<0xB1>(t);    // slots (0,1), (2,3), (4,5), (6,7)
            t = t + dpp_move<0x4E>(t);    // the two halves of each 32 columns
            t = t + dpp_move<0x141>(t);   // the two 32-column halves (the other quad of the row's eight lanes)
            if ((lane & 7) == 0 && dst_of[q] >= 0 && blk < nb)
                sq_blocks[((int64_t)(blk >> 2) * R + dst_of[q]) * 4 + (blk & 3)] = t;
        }
    }
}

// 256x256 tiles run one to a CU, and a last round of few tiles costs a whole round.  The kept count is known on the device
// only, so the kernel itself looks at the remainder: where it is at most half the CUs, its tiles go out as four 128x128
// quarters each (the tile that reads whole steps ahead, eight wavefronts, the same LDS; a quarter takes 0.27 of a tile).
// Measured alone, 65536 rows, without and with: 1024 <- 4096, 528 tiles 313 and 270 us, 576 tiles 329 and 278, 640 tiles 334
// and 316; 1024 <- 2048, 528 tiles 154 and 133; 1024 <- 1536, 576 tiles 142 and 135; 96 tiles of 1024 <- 4096 77 and 62.
// A short contraction has no rounds to speak of (prologues and epilogues let the CUs drift apart) and loses by the
// quarters' extra operand bytes: 4096 <- 1024, 272 tiles 77 and 80 us, 320 tiles 98 and 104.
constexpr int kTailCUs = 256, kTailContraction = 1536;
__device__ __forceinline__ int tail_tiles(int compute, int K_out)
{
    const int last = compute % kTailCUs;
    return K_out >= kTailContraction && last <= kTailCUs / 2 ? last : 0;
}

// grid: 1-D per layer, sized by dgrad_grid.  The first ceil8(compute
// tiles) ids compute (spread over the XCDs in contiguous runs; the quarters of the last round, if any, behind the whole
// tiles), the following ones write the zero rows of dropped samples, the rest exit.  QUARTERS: the last round may go out
// in quarters; the caller has sized the grid for them.
template <int BM, int BN, int WM, int WN, int NS, int SPQ, bool QUARTERS>
__device__ __forceinline__ void dgrad_bf16_body(const uint16_t *__restrict__ G, const uint16_t *__restrict__ W,
                                                const float *__restrict__ p, const int32_t *__restrict__ idxA,
                                                const int32_t *__restrict__ cntA, uint16_t *__restrict__ dX, int N,
                                                int T, int K_in, int K_out, int tiles_n,
                                                const uint16_t *__restrict__ J, int fill_dropped,
                                                const InlineSampleA &sa, float *__restrict__ sq_blocks)
{
    constexpr int NW = WM * WN, NT = NW * 64, STAGE = (BM + BN) * 128;
    constexpr bool kTail = QUARTERS && BM == 256;   // one workgroup per CU
    static_assert(BM * 128 >= kIdxStaged * 4, "index staging area does not fit a stage of G");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int32_t *row_of = reinterpret_cast<int32_t *>(smem + NS * STAGE);
    // The last stage is not loaded before the first barrier of the main loop; until then it
    // holds the kept-sample list, fetched together with the count instead of after it.
    int32_t *idx_staged = reinterpret_cast<int32_t *>(smem + (NS - 1) * BM * 128);
    const int staged = min(N, kIdxStaged);
    __shared__ float sa_norm[64], sa_p[64];
    __shared__ int32_t sa_idx[64];
    __shared__ int sa_count;
    int cnt;
    if (sa.gsq != nullptr || sa.lanes != nullptr) {
        // SampleA decided here, by every workgroup for itself (N <= 64: a few microseconds of one
        // wavefront's work), instead of by a launch of its own in front of this one; the first
        // workgroup writes the plan's fields for everybody else.  The sample norms are either given
        // or taken here from the row sums (4 N T bytes that sit in L2: short vectors only) or from
        // their lane sums (256 N bytes).
        const int lane_ = threadIdx.x & 63, wave_ = threadIdx.x >> 6;
        const uint32_t draw = sa.draw + (sa.draw_offset ? *sa.draw_offset : 0u);   // fetched beside the norms
        if (sa.lanes != nullptr) {
            float v[64 / NW];   // every load first
#pragma unroll
            for (int k = 0; k < 64 / NW; ++k) v[k] = sa.lanes[min(wave_ + k * NW, N - 1) * 64 + lane_];
#pragma unroll
            for (int k = 0; k < 64 / NW; ++k) {
                if (wave_ + k * NW >= N) break;
                const float norm = __builtin_sqrtf(wave_exchange_sum(v[k]));
                if (lane_ == 0) sa_norm[wave_ + k * NW] = norm;
            }
            __syncthreads();
        } else {
            if (T <= 128) sample_norms_batched<8, 2>(sa.gsq, wave_, NW, N, T, sa_norm);
            else sample_norms_batched<4, 8>(sa.gsq, wave_, NW, N, T, sa_norm);
            __syncthreads();
        }
        if (wave_ == 0) {
            const float a = lane_ < N ? sa_norm[lane_] : 0.0f;
            const SampleADecision d = sample_a_wave(a, N, sa.budget, sa.seed, sa.layer, draw);
            if (lane_ < N) sa_p[lane_] = d.pr;
            if (d.keep) sa_idx[d.below] = lane_;
            if (lane_ == 0) sa_count = d.count;
            if (blockIdx.x == 0) {
                if (lane_ < N) {
                    sa.gnorm[lane_] = a;
                    sa.p[lane_] = d.pr;
                    sa.maskA[lane_] = d.keep ? 1 : 0;
                }
                if (d.keep) sa.idxA[d.below] = lane_;
                if (lane_ == 0) *sa.cntA = d.count;
            }
        }
        __syncthreads();
        cnt = sa_count;
        idxA = idx_staged = sa_idx;   // the kept list lives in LDS from here on (N <= 64 entries)
        p = sa_p;
    } else {
        for (int j = threadIdx.x; j < staged; j += NT) idx_staged[j] = idxA[j];
        cnt = min(max(*cntA, 0), N);
    }
    const int64_t M = (int64_t)cnt * T;
    const int64_t R = (int64_t)N * T;
    const int compute = (int)((M + BM - 1) / BM) * tiles_n;
    const int tail = kTail ? tail_tiles(compute, K_out) : 0;   // tiles of the last round that go out as quarters
    // 8 ids per XCD for each quarter that an XCD gets, 32 at most (a CU each); the ones beyond 32 are second quarters
    const int per_xcd = (4 * tail + 7) / 8;
    const int whole8 = (compute - tail + 7) / 8 * 8, compute8 = whole8 + 8 * min(per_xcd, kTailCUs / 8);

    if ((int)blockIdx.x >= compute8) {
        // zero-fill duty: rows of the samples that are not in the kept list
        if (!fill_dropped) return;
        const int z = blockIdx.x - compute8;
        const int64_t d0 = (int64_t)(z / tiles_n) * BM;
        const int n0 = (z % tiles_n) * BN;
        if (d0 >= R - M) return;
        for (int r = threadIdx.x; r < BM; r += NT) {
            const int64_t d = d0 + r;
            int32_t dst = -1;
            if (d < R - M) dst = nth_missing(idxA, cnt, (int)(d / T)) * T + (int)(d % T);
            row_of[r] = dst;
        }
        __syncthreads();
        constexpr int CH = BN / 8;
        for (int u = threadIdx.x; u < BM * CH; u += NT) {
            const int r = u / CH, col = n0 + (u % CH) * 8;
            if (row_of[r] >= 0 && col < K_in)
                *reinterpret_cast<uint4 *>(dX + (int64_t)row_of[r] * K_in + col) = make_uint4(0u, 0u, 0u, 0u);
        }
        return;
    }
    const bool quarters = kTail && (int)blockIdx.x >= whole8;
    const int whole = compute - tail;
    const int id = (int)blockIdx.x - whole8;
    const int first = quarters ? (id & 7) * per_xcd + (id >> 3) : xcd_remap(blockIdx.x, whole);
    if (first >= (quarters ? 4 * tail : whole)) return;
    int tile_m, tile_n;
    // An XCD gets a contiguous run of tile ids and has an L2 of its own: a run that spans all
    // column tiles reads its rows of G once and W whole (W eight times in all); with the
    // columns in `a` panels an XCD reads 1/a of W and every row of G is read by `a` XCDs.
    // a*|G kept| + (8/a)*|W|, i.e. a*M + (8/a)*K_in, is least at a = 1, 2, 4 for M >= 4 K_in, >= K_in, below.
    const int a_panels = M >= 4 * (int64_t)K_in ? 1 : M >= K_in ? 2 : 4;
    const int panel = min(8, max(1, (tiles_n + a_panels - 1) / a_panels));
    if constexpr (kTail) {
        if (quarters) {
            for (int q = first; q < min(4 * tail, ((id & 7) + 1) * per_xcd); q += kTailCUs / 8) {
                panel_order_rt(whole + (q >> 2), compute / tiles_n, tiles_n, panel, tile_m, tile_n);
                const int64_t m0 = (int64_t)tile_m * BM + (q >> 1 & 1) * 128;
                const int n0 = tile_n * BN + (q & 1) * 128;
                // the operand stages of the first quarter lie over the staged list (if it is not SampleA's own)
                const int in_lds = q == first || idxA == sa_idx ? staged : 0;
                if (m0 < M && n0 < K_in)
                    dgrad_bf16_tile<128, 128, 4, 2, 4, kWholeStep>(G, W, p, idxA, idx_staged, in_lds, dX, N, T, K_in, K_out, J,
                                                                   sq_blocks, m0, n0, M);
                __syncthreads();   // the next one's row table and stages lie over this one's
            }
            return;
        }
    }
    panel_order_rt(first, compute / tiles_n, tiles_n, panel, tile_m, tile_n);
    const int n0 = tile_n * BN;
    const int64_t m0 = (int64_t)tile_m * BM;
    dgrad_bf16_tile<BM, BN, WM, WN, NS, SPQ>(G, W, p, idxA, idx_staged, staged, dX, N, T, K_in, K_out, J, sq_blocks, m0, n0, M);
}

template <int BM, int BN, int WM, int WN, int NS, int OCC, int SPQ>
__global__ __launch_bounds__(WM *WN * 64, OCC) void dgrad_bf16_kernel(const uint16_t *__restrict__ G,
                                                                  const uint16_t *__restrict__ W,
                                                                  const float *__restrict__ p,
                                                                  const int32_t *__restrict__ idxA,
                                                                  const int32_t *__restrict__ cntA,
                                                                  uint16_t *__restrict__ dX, int N, int T, int K_in,
                                                                  int K_out, int tiles_n,
                                                                  const uint16_t *__restrict__ J, int fill_dropped,
                                                                  InlineSampleA sa, float *__restrict__ sq_blocks)
{
    dgrad_bf16_body<BM, BN, WM, WN, NS, SPQ, true>(G, W, p, idxA, cntA, dX, N, T, K_in, K_out, tiles_n, J, fill_dropped, sa,
                                             sq_blocks);
}

// Several layers of one shape whose upstream gradients do not depend on each other (the Q, K and V
// projections of an attention block) in one launch: blockIdx.y picks the layer, everything else is the kernel above
// but the quarters (each layer knows its own count only, and what the others leave of the last round is not known).
template <int BM, int BN, int WM, int WN, int NS, int OCC, int SPQ>
__global__ __launch_bounds__(WM *WN * 64, OCC) void dgrad_bf16_group_kernel(DgradGroup grp, int N, int T, int K_in,
                                                                        int K_out, int tiles_n, int fill_dropped)
{
    const DgradProblem &q = grp.prob[blockIdx.y];
    dgrad_bf16_body<BM, BN, WM, WN, NS, SPQ, false>(q.G, q.W, q.p, q.idxA, q.cntA, q.dX, N, T, K_in, K_out, tiles_n, q.J,
                                             fill_dropped, q.sa, q.sq_blocks);
}

// ---------------------------------------------------------- host launchers

// Workgroup ids for a layer: `tiles` tiles if all rows are kept, and where the last round may go out as quarters the ids
// that these add (4 tail - tail, 193 at most at 63 tiles).  A whole round holds the quarters: without zero-fill duty
// behind them rounding up is enough.
template <int BM>
static int64_t dgrad_grid(int64_t tiles, int tiles_n, bool fill, int K_out)
{
    if (BM == 256 && K_out >= kTailContraction) tiles = fill ? tiles + 200 : (tiles + kTailCUs - 1) / kTailCUs * kTailCUs;
    // without zero-fill duty the ids past the compute tiles have nothing to do
    return tiles + (fill ? tiles_n : 0) + 8;
}

template <int BM, int BN, int WM, int WN, int NS, int OCC, int SPQ>
static vcas_status launch_dgrad(const vcas_shape &s, const void *G, const void *W, const float *p,
                                const int32_t *idxA, const int32_t *cntA, void *dX, const void *J, bool fill,
                                const InlineSampleA &sa, float *sq_blocks, hipStream_t st)
{
    const int64_t R = (int64_t)s.N * s.T;
    const int tiles_n = (s.K_in + BN - 1) / BN;
    const int64_t grid = dgrad_grid<BM>((R + BM - 1) / BM * tiles_n, tiles_n, fill, s.K_out);
    if (grid > (int64_t)1 << 30) return VCAS_EINVAL;
    const size_t lds = NS * (BM + BN) * 128 + BM * 8;
    auto kern = dgrad_bf16_kernel<BM, BN, WM, WN, NS, OCC, SPQ>;
    static bool allowed = false;
    if (!allowed) {
        if (!allow_lds(kern, lds)) return VCAS_EHIP;
        allowed = true;
    }
    launch_timed(0, kern, dim3((unsigned)grid), dim3(WM * WN * 64), lds, st, static_cast<const uint16_t *>(G),
                 static_cast<const uint16_t *>(W), p, idxA, cntA, static_cast<uint16_t *>(dX), s.N, s.T, s.K_in,
                 s.K_out, tiles_n, static_cast<const uint16_t *>(J), fill ? 1 : 0, sa, sq_blocks);
    return launch_status();
}

template <int BM, int BN, int WM, int WN, int NS, int OCC, int SPQ>
static vcas_status launch_dgrad_group(const vcas_shape &s, const DgradGroup &grp, int n, bool fill, hipStream_t st)
{
    const int64_t R = (int64_t)s.N * s.T;
    const int tiles_n = (s.K_in + BN - 1) / BN;
    // a multiple of 8 per layer, so that a workgroup's XCD is the same function of blockIdx.x in every layer
    const int64_t grid = (tiles_n * ((R + BM - 1) / BM + (fill ? 1 : 0)) + 8 + 7) / 8 * 8;
    if (grid > (int64_t)1 << 30) return VCAS_EINVAL;
    const size_t lds = NS * (BM + BN) * 128 + BM * 8;
    auto kern = dgrad_bf16_group_kernel<BM, BN, WM, WN, NS, OCC, SPQ>;
    static bool allowed = false;
    if (!allowed) {
        if (!allow_lds(kern, lds)) return VCAS_EHIP;
        allowed = true;
    }
    launch_timed(0, kern, dim3((unsigned)grid, (unsigned)n), dim3(WM * WN * 64), lds, st, grp, s.N, s.T, s.K_in,
                 s.K_out, tiles_n, fill ? 1 : 0);
    return launch_status();
}

enum DgradTile { kTile256, kTile128, kTile64, kTile128Whole, kTile64Whole };

// Which kernel for n layers of `rows` kept rows each, of R.  The larger tile moves fewer operand bytes per
// flop (loads into LDS and fragment reads out of it, not MFMAs, bound the smaller ones), so the largest
// that still fills the chip wins:
//  - 256x256 (one workgroup of eight wavefronts per CU) from 128 tiles up, half the CUs: inside a stack
//    other kernels take the rest (192 made a step 1-3 % longer).  Where the kept count is known on the
//    device only, the tiles of ALL rows are counted and half of them may be empty: 192.
//  - a contraction of less than 512 (eight steps): two stages.  The kernels that read whole steps ahead are twice the code
//    for a loop that is over before it pays.  64x128 tiles, contraction 128, 256, 320, 512, 1024: 8 tiles 6.2, 7.7, 8.0,
//    9.7, 10.5 us and reading ahead 7.1, 7.9, 8.7, 9.7, 10.2; 192 tiles 7.6, 9.0, 9.3, 10.0, 11.5 and 8.2, 9.0, 9.4, 10.1,
//    11.0.
//  - else one tile per CU and nothing else to hide its latencies: the kernels that read whole steps ahead
//    (kWholeStep), 64x128 up to 200 tiles, 128x128 up to 224.  A second round costs more than the better tile gains, and
//    more samples may be kept than expected, so the lines lie that much below 256; 64x128 tiles of ALL rows up to 256
//    are no risk.  K_in 1024, contraction 1024 and 3072, every row kept, us:
//      64x128 tiles     192          240          256          288             128x128 tiles  192          240          256          288
//      64x128 ahead   9.4  18.6    9.7  19.3   10.1  20.2   16.1  35.3
//      64x128        12.0  27.4   12.3  27.9   12.4  28.1   12.6  28.4                      12.9  28.7   13.4  30.8   13.7  31.4   17.3  45.6
//      128x128 ahead 10.4  21.2   10.6  21.5   10.6  21.5   10.7  21.9                      11.0  23.4   12.2  26.4   13.1  28.2   20.4  46.0
//      128x128                                                                              15.3  35.5   16.1  36.6   16.1  36.6   16.6  38.4
//    Forty draws of a sampled layer, 64x128 and 128x128 ahead: 32 samples, keep ratio 0.5, contraction 3072: 200 tiles expected
//    20.2 and 22.6, 216 23.0 and 22.7, 232 24.8 and 22.9; 13 samples of 130 rows, 1128 columns, contraction 3376, 207
//    expected and 243 of all rows 25.5 and 30.6.
//  - two workgroups per CU: 64x128 up to 256 tiles of 128x128, 128x128 beyond (the last columns; 8192 rows, 512 tiles, 30
//    and 24 us).
static DgradTile dgrad_tile(int64_t rows, int64_t R, int K_in, int K_out, int n, bool rows_known)
{
    auto tiles_of = [&](int64_t m, int bm, int bn) { return n * ((m + bm - 1) / bm) * ((K_in + bn - 1) / bn); };
    auto tiles = [&](int bm, int bn) { return tiles_of(rows, bm, bn); };
    if (tiles(256, 256) >= (rows_known ? 128 : 192)) return kTile256;
    if (K_out >= 512 && (tiles(64, 128) <= 200 || tiles_of(R, 64, 128) <= 256)) return kTile64Whole;
    if (K_out >= 512 && tiles(128, 128) <= 224) return kTile128Whole;
    return tiles(128, 128) > 256 ? kTile128 : kTile64;
}

// dgrad of n <= kMaxSiblings layers of shape s in one launch (see dgrad_bf16_group_kernel); the
// tile choice looks at the tiles of all of them together.
vcas_status dgrad_bf16_group(const vcas_shape &s, const DgradProblem *probs, int n, bool fill, int64_t expected_rows,
                             hipStream_t st)
{
    if (n < 1 || n > kMaxSiblings) return VCAS_EINVAL;
    DgradGroup grp = {};
    for (int i = 0; i < n; ++i) {
        if ((probs[i].sa.gsq || probs[i].sa.lanes) && s.N > 64) return VCAS_EINVAL;
        grp.prob[i] = probs[i];
    }
    const int64_t R = (int64_t)s.N * s.T;
    const int64_t rows = expected_rows > 0 && expected_rows < R ? expected_rows : R;
    switch (dgrad_tile(rows, R, s.K_in, s.K_out, n, true)) {
    case kTile256: return launch_dgrad_group<256, 256, 2, 4, 2, 1, -1>(s, grp, n, fill, st);
    case kTile64Whole: return launch_dgrad_group<64, 128, 2, 2, 4, 1, kWholeStep>(s, grp, n, fill, st);
    case kTile128Whole: return launch_dgrad_group<128, 128, 4, 2, 4, 1, kWholeStep>(s, grp, n, fill, st);
    case kTile128: return launch_dgrad_group<128, 128, 2, 2, 2, 2, 4>(s, grp, n, fill, st);
    default: return launch_dgrad_group<64, 128, 2, 2, 2, 2, 0>(s, grp, n, fill, st);
    }
}

// expected_rows: how many of the R rows the caller expects to be kept (R if unknown); it only
// steers the tile choice, any count is computed correctly by every variant.
// J: elementwise Jacobian [R, K_in] multiplied into dX, or null.  fill: write the zero rows of
// dropped samples (false: leave them as they are).
// sample_a (null: SampleA has been decided, p / idxA / cntA hold its outcome): the kernel decides
// it itself from the row sums or the sample norms and writes the plan's SampleA fields; N <= 64 only.
vcas_status dgrad_bf16(const vcas_shape &s, const void *G, const void *W, const float *p, const int32_t *idxA,
                       const int32_t *cntA, void *dX, const void *J, bool fill, int64_t expected_rows,
                       const InlineSampleA *sample_a, float *sq_blocks, hipStream_t st)
{
    InlineSampleA sa = {};
    sa.gsq = nullptr;
    if (sample_a) {
        if (s.N > 64) return VCAS_EINVAL;
        sa = *sample_a;
    }
    const int64_t R = (int64_t)s.N * s.T;
    const int64_t rows = expected_rows > 0 && expected_rows < R ? expected_rows : R;
    switch (dgrad_tile(rows, R, s.K_in, s.K_out, 1, expected_rows > 0)) {
    case kTile256: return launch_dgrad<256, 256, 2, 4, 2, 1, -1>(s, G, W, p, idxA, cntA, dX, J, fill, sa, sq_blocks, st);
    case kTile64Whole: return launch_dgrad<64, 128, 2, 2, 4, 1, kWholeStep>(s, G, W, p, idxA, cntA, dX, J, fill, sa, sq_blocks, st);
    case kTile128Whole: return launch_dgrad<128, 128, 4, 2, 4, 1, kWholeStep>(s, G, W, p, idxA, cntA, dX, J, fill, sa, sq_blocks, st);
    case kTile128: return launch_dgrad<128, 128, 2, 2, 2, 2, 4>(s, G, W, p, idxA, cntA, dX, J, fill, sa, sq_blocks, st);
    default: return launch_dgrad<64, 128, 2, 2, 2, 2, 0>(s, G, W, p, idxA, cntA, dX, J, fill, sa, sq_blocks, st);
    }
}

}  // namespace vcas
