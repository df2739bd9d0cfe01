// The two samplers by one workgroup of 1024 threads with the vector in registers (Sec. 4.1, 4.2): keep
// probabilities, Bernoulli masks, ascending kept lists.  Shared by the sampler kernels and by the
// fused planning kernel.  Element i of a vector belongs to thread i mod 1024 (its summation slot),
// ascending i inside a slot.
#pragma once

#include "sample_a_small.hpp"

namespace vcas {

// ---- block-wide sums over 1024 threads in a fixed order ---------------------
// Thread tid is "slot" tid.  Each 64-slot group (one wavefront) is combined by
// the neighbours-first tree, then the 16 group sums by the same kind of tree.
// Every thread returns the totals.  `bufd` / `bufi` are 16 values of LDS each;
// calls must alternate buffers or be separated by a barrier.
// `c_wave` is the wavefront's count, already the same in all its lanes.
__device__ __forceinline__ void block_totals_1024(double v, int c_wave, double *bufd, int *bufi, double &sum_v,
                                                  int &sum_c)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_exchange_sum(v);
    if (lane == 0) {
        bufd[wave] = v;
        bufi[wave] = c_wave;
    }
    __syncthreads();
    // every 16-lane row holds the 16 partials, one per lane, and adds them by the same tree
    // (quad swaps, then the two mirrors) instead of every lane reading and adding all 16
    double w = bufd[lane & 15];
    int c = bufi[lane & 15];
    w = w + dpp_move<0xB1>(w);
    w = w + dpp_move<0x4E>(w);
    w = w + dpp_move<0x141>(w);
    w = w + dpp_move<0x140>(w);
    c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);
    c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);
    c += __builtin_amdgcn_update_dpp(0, c, 0x141, 0xF, 0xF, true);
    c += __builtin_amdgcn_update_dpp(0, c, 0x140, 0xF, 0xF, true);
    sum_v = read_lane(w, 0);
    sum_c = __builtin_amdgcn_readlane(c, 0);
}

__device__ __forceinline__ void block_sum_pair_1024(double v, int c, double *bufd, int *bufi, double &sum_v, int &sum_c)
{
    block_totals_1024(v, wave_sum_int(c), bufd, bufi, sum_v, sum_c);
}

__device__ __forceinline__ int ballot_count(bool c) { return __builtin_popcountll(__ballot(c)); }

// What the rounds of the keep probabilities come to (Sec. 4.1: p ~ score, capped at one): an element is
// fixed at one in some round exactly if the largest c any round has tried pushes it to one (the
// product is monotone in c and in the score, rounding included), and the others get the last round's c.
// So two numbers stand for the whole vector, and no element carries a state from round to round.
// (Turning c_cap into the smallest float it caps, for a fp32 compare, costs a round more than it saves.)
struct KeepRule {
    double c_cap, c;
};

__device__ __forceinline__ float keep_prob(float a, const KeepRule &k)
{
    if (!(a > 0.0f)) return 0.0f;
    if (k.c_cap * (double)a >= 1.0) return 1.0f;
    const float p = (float)(k.c * (double)a);
    return p < 1.0f ? p : 1.0f;
}

// prob_i = min(1, c a_i) with sum prob = min(budget, #positive): c is found by rounds; every entry that the
// current c pushes to >= 1 is fixed at one, then c is recomputed from what is left, until a round
// fixes nothing.  Sums in fp64.  A round is one multiply, compare, select and add per element and one
// barrier.  a: thread tid's elements tid + 1024*j, j < E (zero past the end); whole workgroup calls.
template <int E>
__device__ __forceinline__ KeepRule keep_rule_regs(const float (&a)[E], double budget)
{
    __shared__ double sd[2][16];
    __shared__ int si[2][16];
    double part = 0.0;
    int cnt = 0;             // per wavefront, from ballots (scalar work, beside the vector sums)
    float open_max = 0.0f;   // largest score of this thread that is not fixed
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const bool pos = a[j] > 0.0f;
        const float v = pos ? a[j] : 0.0f;
        part += (double)v;
        cnt += ballot_count(pos);
        open_max = v > open_max ? v : open_max;
    }
    double S;
    int nonzero;
    block_totals_1024(part, cnt, sd[0], si[0], S, nonzero);
    if (budget >= (double)nonzero) return {__builtin_inf(), 0.0};   // every positive score is kept
    KeepRule k = {0.0, 0.0};
    int ncap = 0;
    cnt = 0;
    int flip = 1;
    for (;;) {
        const double rem = budget - (double)ncap;
        if (!(S > 0.0) || !(rem > 0.0)) {
            k.c = 0.0;
            return k;
        }
        k.c = rem / S;
        k.c_cap = k.c > k.c_cap ? k.c : k.c_cap;
        // A thread whose largest open score stays below one has nothing to fix, and its partial sum, the
        // same additions over the same values, is the one it already holds.  A wavefront without any
        // thread that fixes something skips the round's arithmetic (in the later rounds most of them).
        if (__ballot(k.c_cap * (double)open_max >= 1.0) != 0ull) {
            part = 0.0;
            open_max = 0.0f;
            cnt = 0;
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const bool cap = k.c_cap * (double)a[j] >= 1.0;
                const float v = cap || !(a[j] > 0.0f) ? 0.0f : a[j];
                part += (double)v;
                cnt += ballot_count(cap);
                open_max = v > open_max ? v : open_max;
            }
        }
        double S_next;
        int capped;
        block_totals_1024(part, cnt, sd[flip], si[flip], S_next, capped);
        flip ^= 1;
        if (capped == ncap) return k;
        ncap = capped;
        S = S_next;
    }
}

// The same from memory: every round reads the n scores again.
__device__ __forceinline__ KeepRule keep_rule_memory(const float *__restrict__ score, int n, double budget)
{
    __shared__ double sd[2][16];
    __shared__ int si[2][16];
    // the sum over what c_cap does not fix, and how many it fixes (c_cap = 0: how many scores are positive)
    auto pass = [&](double c_cap, double &part, int &cnt) {
        part = 0.0;
        cnt = 0;
        for (int i0 = threadIdx.x; i0 < n; i0 += 8 * 1024) {
            float a[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) a[j] = score[min(i0 + 1024 * j, n - 1)];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool pos = i0 + 1024 * j < n && a[j] > 0.0f;
                const bool cap = pos && c_cap * (double)a[j] >= 1.0;
                part += pos && !cap ? (double)a[j] : 0.0;
                cnt += c_cap == 0.0 ? pos : cap;
            }
        }
    };
    double part, S;
    int cnt, nonzero;
    pass(0.0, part, cnt);
    block_sum_pair_1024(part, cnt, sd[0], si[0], S, nonzero);
    if (budget >= (double)nonzero) return {__builtin_inf(), 0.0};   // every positive score is kept
    KeepRule k = {0.0, 0.0};
    int ncap = 0, flip = 1;
    for (;;) {
        const double rem = budget - (double)ncap;
        if (!(S > 0.0) || !(rem > 0.0)) {
            k.c = 0.0;
            return k;
        }
        k.c = rem / S;
        k.c_cap = k.c > k.c_cap ? k.c : k.c_cap;
        pass(k.c_cap, part, cnt);
        double S_next;
        int capped;
        block_sum_pair_1024(part, cnt, sd[flip], si[flip], S_next, capped);
        flip ^= 1;
        if (capped == ncap) return k;
        ncap = capped;
        S = S_next;
    }
}

// Ascending list of the kept indices and their count.  Bit j of `kept` = element j of this thread, index
// tid + 1024 j, so ascending order is j, then wavefront, then lane.  Every wavefront counts its kept
// lanes per j with a ballot; the first wavefront turns the 16 E counts into bases; a lane's position is
// its base plus the kept lanes below it.
template <int E>
__device__ __forceinline__ void compact_regs(uint32_t kept, int32_t *__restrict__ idx, int32_t *__restrict__ count)
{
    constexpr int CNT = 16 * E, PER = (CNT + 63) / 64;
    __shared__ int counts[CNT + 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int n = ballot_count((kept >> j) & 1);
        if (lane == 0) counts[j * 16 + wave] = n;
    }
    __syncthreads();
    if (wave == 0) {
        // lane L owns counts PER*L .. PER*L+PER-1; exclusive prefix of all of them, in place
        int c[PER], mine = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            c[q] = PER * lane + q < CNT ? counts[PER * lane + q] : 0;
            mine += c[q];
        }
        int incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += up;
        }
        int run = incl - mine;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (PER * lane + q < CNT) counts[PER * lane + q] = run;
            run += c[q];
        }
        if (lane == 63) counts[CNT] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const bool m = (kept >> j) & 1;
        const uint64_t b = __ballot(m);
        const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
        if (m) idx[counts[j * 16 + wave] + below] = (int)threadIdx.x + 1024 * j;
    }
    if (threadIdx.x == 0) *count = counts[CNT];
}

// ---- SampleA --------------------------------------------------------------------------------

// What SampleW needs to know of a sample, in LDS (N <= 1024).
struct SampleTable {
    float p[1024], pinv[1024];
    uint8_t keep[1024];
};

// SampleA for N <= 1024 (whole workgroup calls): norms from the row sums, probabilities, mask, kept
// list to memory, and to `table` (null: not wanted; complete after the caller's next barrier).
__device__ __forceinline__ void sampler_a_fast_body(const float *__restrict__ gsq, int N, int T, double budget,
                                                    uint64_t seed, uint32_t layer, uint32_t draw,
                                                    float *__restrict__ gnorm, float *__restrict__ p,
                                                    uint8_t *__restrict__ maskA, int32_t *__restrict__ idxA,
                                                    int32_t *__restrict__ cntA, SampleTable *table)
{
    __shared__ float gn[1024];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (T <= 128) sample_norms_batched<4, 2>(gsq, wave, 16, N, T, gn);
    else sample_norms_batched<2, 8>(gsq, wave, 16, N, T, gn);
    __syncthreads();
    if (N <= 64) {
        // one wavefront decides (see sample_a_small.hpp)
        if (wave != 0) return;
        const float a = lane < N ? gn[lane] : 0.0f;
        const SampleADecision d = sample_a_wave(a, N, budget, seed, layer, draw);
        if (lane < N) {
            gnorm[lane] = a;
            p[lane] = d.pr;
            maskA[lane] = d.keep ? 1 : 0;
            if (table) {
                table->p[lane] = d.pr;
                table->pinv[lane] = d.keep ? 1.0f / d.pr : 0.0f;
                table->keep[lane] = d.keep ? 1 : 0;
            }
        }
        if (d.keep) idxA[d.below] = lane;
        if (lane == 0) *cntA = d.count;
        return;
    }
    float a[1];
    a[0] = tid < N ? gn[tid] : 0.0f;
    const KeepRule rule = keep_rule_regs<1>(a, budget);
    bool m = false;
    if (tid < N) {
        const float pr = keep_prob(a[0], rule);
        m = philox_uniform(seed, layer, 0u, draw, (uint32_t)tid) < pr;
        gnorm[tid] = a[0];
        p[tid] = pr;
        maskA[tid] = m ? 1 : 0;
        if (table) {
            table->p[tid] = pr;
            table->pinv[tid] = m ? 1.0f / pr : 0.0f;
            table->keep[tid] = m ? 1 : 0;
        }
    }
    compact_regs<1>(m ? 1 : 0, idxA, cntA);
}

// ---- SampleW --------------------------------------------------------------------------------

// What the norm passes have left in the score and q arrays when SampleW starts (`roots_given`): the square roots of
// gsq and xsq for every row, taken before SampleA, and xsq itself is still there on dropped samples; or the scores,
// final (0 on dropped samples, whose xsq is 0 already).

// t / T for t * T < 2^32 with a multiplier the wavefront computes once (T > 1):
// t * (floor(2^32 / T) + 1) / 2^32 = t / T + t * e / 2^32 with 0 < e <= 1, and
// t / 2^32 < 1 / T keeps the sum below the next integer.
__device__ __forceinline__ uint32_t sample_magic(int T) { return T > 1 ? (uint32_t)(0x100000000ull / (uint32_t)T) + 1u : 0u; }
__device__ __forceinline__ int sample_of(int t, int T, uint32_t magic)
{
    return T > 1 ? (int)__umulhi((uint32_t)t, magic) : t;
}

// From the scores on: q, mask, scale and kept list.  a: this thread's scores (zero past the end), uu: its uniforms.
template <int E>
__device__ __forceinline__ void sample_w_finish(const float (&a)[E], const float (&uu)[E], const SampleTable *table,
                                                const float *__restrict__ p, const uint8_t *__restrict__ maskA, int R, int T,
                                                double budget, int token_sampling, float *__restrict__ q,
                                                uint8_t *__restrict__ maskW, float *__restrict__ scaleW,
                                                int32_t *__restrict__ idxW, int32_t *__restrict__ cntW)
{
    const int tid = threadIdx.x;
    const uint32_t magic = sample_magic(T);
    KeepRule rule = {0.0, 0.0};
    if (token_sampling) rule = keep_rule_regs<E>(a, budget);
    uint32_t kept = 0;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int t = tid + 1024 * j;
        if (t < R) {
            const int i = sample_of(t, T, magic);
            bool m;
            float qv;
            if (token_sampling) {
                qv = keep_prob(a[j], rule);
                m = uu[j] < qv;
            } else {
                m = table ? table->keep[i] != 0 : maskA[i] != 0;
                qv = m ? 1.0f : 0.0f;
            }
            kept |= (m ? 1u : 0u) << j;
            q[t] = qv;
            maskW[t] = m ? 1 : 0;
            scaleW[t] = m ? 1.0f / ((table ? table->p[i] : p[i]) * qv) : 0.0f;
        }
    }
    compact_regs<E>(kept, idxW, cntW);
}

// SampleW for R <= 1024*E (one workgroup of 1024).  The whole vector is this one
// workgroup's arithmetic, so everything per sample (1/p_i, the keep byte) is
// computed once into LDS when N <= 1024, and the square roots come from the
// many-workgroup norm pass.
template <int E>
__device__ __forceinline__ void sampler_w_fast_body(float *__restrict__ xsq, const float *__restrict__ p,
                                                    const uint8_t *__restrict__ maskA, const float *__restrict__ u,
                                                    int N, int T, double budget, int token_sampling, int roots_given,
                                                    float *__restrict__ score, float *__restrict__ q,
                                                    uint8_t *__restrict__ maskW, float *__restrict__ scaleW,
                                                    int32_t *__restrict__ idxW, int32_t *__restrict__ cntW)
{
    __shared__ SampleTable table;
    const int tid = threadIdx.x;
    const int R = N * T;
    const bool tabled = N <= 1024;
    const uint32_t magic = sample_magic(T);
    // Every load of the vectors first, with no condition on a loaded value in between, so that
    // they are all in flight together (rows past the end re-read the last row and are ignored).
    float a[E], rx[E], uu[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int t = min(tid + 1024 * j, R - 1);
        uu[j] = token_sampling ? u[t] : 0.0f;
        a[j] = score[t];
        rx[j] = roots_given ? q[t] : 0.0f;
    }
    if (tabled) {
        if (tid < N) {
            const float pi = p[tid];
            const uint8_t k = maskA[tid];
            table.p[tid] = pi;
            table.keep[tid] = k;
            table.pinv[tid] = k ? 1.0f / pi : 0.0f;
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int t = tid + 1024 * j;
        if (t >= R) {
            a[j] = 0.0f;
        } else if (roots_given) {
            const int i = sample_of(t, T, magic);
            const bool keep = tabled ? table.keep[i] != 0 : maskA[i] != 0;
            const float rg = a[j];
            a[j] = 0.0f;
            if (keep) {
                const float inv = tabled ? table.pinv[i] : 1.0f / p[i];
                const float s1 = inv * rg;
                a[j] = s1 * rx[j];
            } else {
                xsq[t] = 0.0f;
            }
            score[t] = a[j];
        }
    }
    sample_w_finish<E>(a, uu, tabled ? &table : nullptr, p, maskA, R, T, budget, token_sampling, q, maskW, scaleW, idxW, cntW);
}

}  // namespace vcas
