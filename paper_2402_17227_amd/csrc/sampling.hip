// Sampling kernels of the VCAS backward pass: capped-proportional keep
// probabilities (Sec. 4.1 p_i ~ ||G_i||_F, Sec. 4.2 q_t ~ leverage score),
// Philox Bernoulli masks, kept-row compaction, and the two small elementwise
// steps (leverage scores, per-row scale).  All vectors are at most R floats,
// so these kernels are latency-bound, not bandwidth-bound.
#include "groups.hpp"
#include "samplers.hpp"

namespace vcas {

// prob_i = min(1, c * score_i), sum prob = min(budget, #positive scores).
// c is found by rounds: every not-yet-fixed entry that the current c pushes to
// >= 1 is fixed at one, then c is recomputed from what is left, until a round
// fixes nothing.  Sums in fp64, slot = i mod 1024, ascending i inside a slot.
// While running, prob[i] == 1 marks "fixed at one" (each element is only ever
// touched by its own thread).  Single block of 1024 threads.
__device__ void keep_probs_block(const float *__restrict__ score, int n, double budget, float *__restrict__ prob)
{
    __shared__ double sd[2][16];
    __shared__ int si[2][16];
    const int tid = threadIdx.x;

    double part = 0.0;
    int cnt = 0;
    for (int i = tid; i < n; i += 1024) {
        float a = score[i];
        if (a > 0.0f) {
            part += (double)a;
            ++cnt;
        }
        prob[i] = 0.0f;
    }
    double S;
    int nonzero;
    block_sum_pair_1024(part, cnt, sd[0], si[0], S, nonzero);

    if (budget >= (double)nonzero) {
        for (int i = tid; i < n; i += 1024) prob[i] = score[i] > 0.0f ? 1.0f : 0.0f;
        return;
    }

    int ncap = 0;
    double c = 0.0;
    int flip = 1;
    for (;;) {
        const double rem = budget - (double)ncap;
        if (!(S > 0.0) || !(rem > 0.0)) {
            c = 0.0;
            break;
        }
        c = rem / S;
        part = 0.0;
        cnt = 0;
        for (int i = tid; i < n; i += 1024) {
            float a = score[i];
            if (a > 0.0f && prob[i] != 1.0f) {
                if (c * (double)a >= 1.0) {
                    prob[i] = 1.0f;
                    ++cnt;
                } else {
                    part += (double)a;
                }
            }
        }
        double S_next;
        int newly;
        block_sum_pair_1024(part, cnt, sd[flip], si[flip], S_next, newly);
        flip ^= 1;
        if (newly == 0) break;
        ncap += newly;
        S = S_next;
    }
    for (int i = tid; i < n; i += 1024) {
        float a = score[i];
        if (prob[i] == 1.0f) continue;
        float p = 0.0f;
        if (a > 0.0f) {
            p = (float)(c * (double)a);
            p = p < 1.0f ? p : 1.0f;
        }
        prob[i] = p;
    }
}

__global__ __launch_bounds__(1024) void keep_probs_kernel(const float *__restrict__ score, int n, double budget,
                                                          float *__restrict__ prob)
{
    keep_probs_block(score, n, budget, prob);
}

// mask[r] = [u_r < prob[r]]
__global__ __launch_bounds__(256) void bernoulli_mask_kernel(const float *__restrict__ prob, int n, uint64_t seed,
                                                             uint32_t layer, uint32_t stream_id, uint32_t draw,
                                                             const uint32_t *__restrict__ draw_offset,
                                                             uint8_t *__restrict__ mask)
{
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    if (draw_offset) draw += *draw_offset;
    const float u = philox_uniform(seed, layer, stream_id, draw, (uint32_t)r);
    mask[r] = u < prob[r] ? 1 : 0;
}

// Ascending list of the r with mask[r] != 0, and their count.  Single block of
// 1024 threads; thread tid owns the contiguous slice [tid*per, (tid+1)*per).
// Slice counts are scanned across the block (wave scan, then the 16 wave
// totals through LDS).
__device__ void compact_block(const uint8_t *__restrict__ mask, int n, int32_t *__restrict__ idx,
                              int32_t *__restrict__ count)
{
    __shared__ int wave_total[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (n + 1023) / 1024;
    const int lo = min(n, tid * per), hi = min(n, lo + per);
    int mine = 0;
    for (int r = lo; r < hi; ++r) mine += mask[r] != 0;
    int incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int up = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += up;
    }
    if (lane == 63) wave_total[wave] = incl;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        int t = wave_total[w];
        if (w < wave) before += t;
        total += t;
    }
    int pos = before + incl - mine;
    for (int r = lo; r < hi; ++r)
        if (mask[r] != 0) idx[pos++] = r;
    if (tid == 0) *count = total;
}

__global__ __launch_bounds__(1024) void compact_kernel(const uint8_t *__restrict__ mask, int n,
                                                       int32_t *__restrict__ idx, int32_t *__restrict__ count)
{
    compact_block(mask, n, idx, count);
}

// score[t] = maskA[i] * ((1/p[i]) * sqrt(gsq[t])) * sqrt(xsq[t])
__global__ __launch_bounds__(256) void leverage_kernel(const float *__restrict__ gsq, const float *__restrict__ xsq,
                                                       const float *__restrict__ p, const uint8_t *__restrict__ maskA,
                                                       int64_t R, int T, float *__restrict__ score)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= R) return;
    const int i = (int)(t / T);
    float s = 0.0f;
    if (maskA[i]) {
        const float inv = 1.0f / (p[i]);
        const float a = inv * __builtin_sqrtf(gsq[t]);
        s = a * __builtin_sqrtf(xsq[t]);
    }
    score[t] = s;
}

// scaleW[t] = maskW[t] ? 1/(p[i] q[t]) : 0
__global__ __launch_bounds__(256) void row_scale_kernel(const float *__restrict__ p, const float *__restrict__ q,
                                                        const uint8_t *__restrict__ maskW, int64_t R, int T,
                                                        float *__restrict__ scale)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= R) return;
    const int i = (int)(t / T);
    scale[t] = maskW[t] ? 1.0f / (p[i] * q[t]) : 0.0f;
}

// ---- fused single-workgroup samplers (used by vcas_linear_backward) -----------
// The vectors are at most R floats, so one workgroup of 1024 threads does the
// whole decision chain of a sampler in one launch instead of five.

__global__ __launch_bounds__(1024) void sampler_a_fast_kernel(const float *__restrict__ gsq, int N, int T,
                                                              double budget, uint64_t seed, uint32_t layer,
                                                              uint32_t draw, const uint32_t *__restrict__ draw_offset,
                                                              float *__restrict__ gnorm, float *__restrict__ p,
                                                              uint8_t *__restrict__ maskA, int32_t *__restrict__ idxA,
                                                              int32_t *__restrict__ cntA)
{
    if (draw_offset) draw += *draw_offset;
    sampler_a_fast_body(gsq, N, T, budget, seed, layer, draw, gnorm, p, maskA, idxA, cntA, nullptr);
}

// SampleA of up to kMaxSamplers layers with the same N and T, one workgroup per layer.
__global__ __launch_bounds__(1024) void sampler_a_group_kernel(SampleAGroup grp, int N, int T)
{
    const InlineSampleA &q = grp.prob[blockIdx.x];
    const uint32_t draw = q.draw + (q.draw_offset ? *q.draw_offset : 0u);
    sampler_a_fast_body(q.gsq, N, T, q.budget, q.seed, q.layer, draw, q.gnorm, q.p, q.maskA, q.idxA, q.cntA, nullptr);
}

// SampleW of up to kMaxSamplers layers of one shape, one workgroup per layer.
template <int E>
__global__ __launch_bounds__(1024) void sampler_w_group_kernel(SampleWGroup grp, int N, int T, int token_sampling,
                                                               int roots_given)
{
    const SampleWProblem &w = grp.prob[blockIdx.x];
    sampler_w_fast_body<E>(w.xsq, w.p, w.maskA, w.u, N, T, w.budget, token_sampling, roots_given, w.score, w.q, w.maskW,
                           w.scaleW, w.idxW, w.cntW);
}

// SampleA: ||G_i||_F from gsq, p, Bernoulli mask over samples, kept list.
__global__ __launch_bounds__(1024) void sampler_a_kernel(const float *__restrict__ gsq, int N, int T, double budget,
                                                         uint64_t seed, uint32_t layer, uint32_t draw,
                                                         const uint32_t *__restrict__ draw_offset,
                                                         float *__restrict__ gnorm, float *__restrict__ p,
                                                         uint8_t *__restrict__ maskA, int32_t *__restrict__ idxA,
                                                         int32_t *__restrict__ cntA)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (draw_offset) draw += *draw_offset;
    for (int i = wave; i < N; i += 16) {
        const float *row = gsq + (int64_t)i * T;
        float acc = 0.0f;
        for (int t = lane; t < T; t += 64) acc = acc + row[t];
        acc = wave_exchange_sum(acc);
        if (lane == 0) gnorm[i] = __builtin_sqrtf(acc);
    }
    __syncthreads();
    keep_probs_block(gnorm, N, budget, p);
    __syncthreads();
    for (int i = tid; i < N; i += 1024) maskA[i] = philox_uniform(seed, layer, 0u, draw, (uint32_t)i) < p[i] ? 1 : 0;
    __syncthreads();
    compact_block(maskA, N, idxA, cntA);
}

// ---- SampleW of more rows than one workgroup's registers hold comfortably ----------------------
// Only the rounds of the keep probabilities need the whole vector in one place.  Launches: scores
// (many workgroups, where the norm pass has not written them), the rounds (one workgroup: reads R
// floats and writes the two numbers of a KeepRule), what is elementwise given the rule (many
// workgroups), the kept list (many workgroups).  One workgroup for all of it took 227 us at R = 65536 from memory and 132 us with
// the scores in (spilling) registers; see sampler_w_group for the line.

// From the square roots that the norm pass has left.
__global__ __launch_bounds__(256) void sampler_w_scores_kernel(SampleWGroup grp, int R, int T)
{
    const SampleWProblem &w = grp.prob[blockIdx.y];
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= R) return;
    const int i = t / T;
    float s = 0.0f;
    if (w.maskA[i]) {
        const float inv = 1.0f / w.p[i];
        const float a = inv * w.score[t];
        s = a * w.q[t];
    } else {
        w.xsq[t] = 0.0f;
    }
    w.score[t] = s;
}

// E elements per thread in registers, or (E = 0) every round reads the scores again.
template <int E>
__global__ __launch_bounds__(1024) void sampler_w_rule_kernel(SampleWGroup grp, int R)
{
    const SampleWProblem &w = grp.prob[blockIdx.x];
    const int tid = threadIdx.x;
    KeepRule rule;
    if constexpr (E > 0) {
        float a[E];
#pragma unroll
        for (int j = 0; j < E; ++j) a[j] = w.score[min(tid + 1024 * j, R - 1)];
#pragma unroll
        for (int j = 0; j < E; ++j) a[j] = tid + 1024 * j < R ? a[j] : 0.0f;
        rule = keep_rule_regs<E>(a, w.budget);
    } else {
        rule = keep_rule_memory(w.score, R, w.budget);
    }
    if (tid == 0) {
        w.rule[0] = rule.c_cap;
        w.rule[1] = rule.c;
    }
}

// q, mask and scale of every row.  COUNTED: also how many of the workgroup's 256 rows are kept, over the first of their
// uniforms.
template <bool COUNTED>
__global__ __launch_bounds__(256) void sampler_w_apply_kernel(SampleWGroup grp, int R, int T, int token_sampling)
{
    const SampleWProblem &w = grp.prob[blockIdx.y];
    const int t = blockIdx.x * 256 + threadIdx.x;
    bool m = false;
    if (t < R) {
        const int i = t / T;
        float qv;
        if (token_sampling) {
            const KeepRule rule = {w.rule[0], w.rule[1]};
            qv = keep_prob(w.score[t], rule);
            m = w.u[t] < qv;
        } else {
            m = w.maskA[i] != 0;
            qv = m ? 1.0f : 0.0f;
        }
        w.q[t] = qv;
        w.maskW[t] = m ? 1 : 0;
        w.scaleW[t] = m ? 1.0f / (w.p[i] * qv) : 0.0f;
    }
    if constexpr (COUNTED) {
        __shared__ int wave_count[4];
        const int n = ballot_count(m);
        if ((threadIdx.x & 63) == 0) wave_count[threadIdx.x >> 6] = n;
        __syncthreads();   // ... and everybody has read its uniform
        if (threadIdx.x == 0) w.u[t] = __int_as_float((wave_count[0] + wave_count[1]) + (wave_count[2] + wave_count[3]));
    }
}

// Kept list of 1024 rows per workgroup.  The place of a row in the ascending list is the number of kept
// rows in front of it: every workgroup adds up the mask bytes before its own rows again, a few 16-byte
// loads per thread up to kListRows, which is cheaper than an exchange between workgroups.
__global__ __launch_bounds__(1024) void sampler_w_list_kernel(SampleWGroup grp, int R)
{
    __shared__ int wave_count[16], wave_before[16];
    const SampleWProblem &w = grp.prob[blockIdx.y];
    const uint8_t *mask = w.maskW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int first = blockIdx.x * 1024;
    // [0, head) and [head + 16 * vecs, first) byte by byte, the aligned part in between by 16
    const int head = min(first, (int)(-reinterpret_cast<uintptr_t>(mask) & 15u));
    const int vecs = (first - head) / 16, tail = head + 16 * vecs;
    int before = 0;
    for (int v = tid; v < vecs; v += 1024) {
        const uint4 b = *reinterpret_cast<const uint4 *>(mask + head + 16 * v);   // bytes of 0 and 1: a popcount adds them
        before += __builtin_popcount(b.x) + __builtin_popcount(b.y) + __builtin_popcount(b.z) + __builtin_popcount(b.w);
    }
    if (tid < head) before += mask[tid];
    if (tid < first - tail) before += mask[tail + tid];
    before = wave_sum_int(before);
    const int t = first + tid;
    const bool m = t < R && mask[t] != 0;
    const uint64_t b = __ballot(m);
    if (lane == 0) {
        wave_before[wave] = before;
        wave_count[wave] = __builtin_popcountll(b);
    }
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        base += wave_before[v] + (v < wave ? wave_count[v] : 0);
        total += wave_before[v] + wave_count[v];
    }
    if (m) w.idxW[base + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = t;
    if (tid == 0 && first + 1024 >= R) *w.cntW = total;
}

// The same for longer vectors, where adding up everything in front would be R^2 / 2048 bytes of reads: the counts that
// sampler_w_apply_kernel left for every 256 rows become places (one workgroup per layer), and every 256 rows go there.
__global__ __launch_bounds__(1024) void sampler_w_places_kernel(SampleWGroup grp, int R)
{
    __shared__ int wave_total[16];
    const SampleWProblem &w = grp.prob[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, blocks = (R + 255) / 256;
    int run = 0, next = tid < blocks ? __float_as_int(w.u[256 * tid]) : 0;
    for (int b0 = 0; b0 < blocks; b0 += 1024) {
        const int b = b0 + tid, mine = next;
        next = b + 1024 < blocks ? __float_as_int(w.u[256 * (b + 1024)]) : 0;
        int incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += up;
        }
        if (lane == 63) wave_total[wave] = incl;
        __syncthreads();
        int before = run;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            before += v < wave ? wave_total[v] : 0;
            run += wave_total[v];
        }
        if (b < blocks) w.u[256 * b] = __int_as_float(before + incl - mine);
        __syncthreads();   // the totals have been read
    }
    if (tid == 0) *w.cntW = run;
}

__global__ __launch_bounds__(256) void sampler_w_place_kernel(SampleWGroup grp, int R)
{
    __shared__ int wave_count[4];
    const SampleWProblem &w = grp.prob[blockIdx.y];
    const int t = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool m = t < R && w.maskW[t] != 0;
    const uint64_t b = __ballot(m);
    if (lane == 0) wave_count[wave] = __builtin_popcountll(b);
    int at = __float_as_int(w.u[blockIdx.x * 256]);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 3; ++v) at += v < wave ? wave_count[v] : 0;
    if (m) w.idxW[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = t;
}

// ---- host launchers ---------------------------------------------------------

vcas_status keep_probs(const float *score, int n, double budget, float *prob, hipStream_t st)
{
    hipLaunchKernelGGL(keep_probs_kernel, dim3(1), dim3(1024), 0, st, score, n, budget, prob);
    return launch_status();
}

vcas_status sample_compact(const float *prob, int n, const vcas_rng &rng, uint32_t stream_id, uint8_t *mask,
                           int32_t *idx, int32_t *count, hipStream_t st)
{
    if (n > 0) {
        hipLaunchKernelGGL(bernoulli_mask_kernel, dim3((n + 255) / 256), dim3(256), 0, st, prob, n, rng.seed,
                           rng.layer, stream_id, rng.draw, rng.draw_offset, mask);
        if (hipGetLastError() != hipSuccess) return VCAS_EHIP;
    }
    hipLaunchKernelGGL(compact_kernel, dim3(1), dim3(1024), 0, st, mask, n, idx, count);
    return launch_status();
}

vcas_status leverage_scores(const float *gsq, const float *xsq, const float *p, const uint8_t *maskA, int64_t R,
                            int T, float *score, hipStream_t st)
{
    hipLaunchKernelGGL(leverage_kernel, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, st, gsq, xsq, p, maskA, R, T,
                       score);
    return launch_status();
}

vcas_status row_scale(const float *p, const float *q, const uint8_t *maskW, int64_t R, int T, float *scale,
                      hipStream_t st)
{
    hipLaunchKernelGGL(row_scale_kernel, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, st, p, q, maskW, R, T,
                       scale);
    return launch_status();
}

vcas_status sampler_a(const float *gsq, int N, int T, double budget, const vcas_rng &rng, float *gnorm, float *p,
                      uint8_t *maskA, int32_t *idxA, int32_t *cntA, hipStream_t st)
{
    if (N <= 1024)
        hipLaunchKernelGGL(sampler_a_fast_kernel, dim3(1), dim3(1024), 0, st, gsq, N, T, budget, rng.seed, rng.layer,
                           rng.draw, rng.draw_offset, gnorm, p, maskA, idxA, cntA);
    else
        hipLaunchKernelGGL(sampler_a_kernel, dim3(1), dim3(1024), 0, st, gsq, N, T, budget, rng.seed, rng.layer,
                           rng.draw, rng.draw_offset, gnorm, p, maskA, idxA, cntA);
    return launch_status();
}

// sampler_a for n <= kMaxSamplers layers of N <= 1024 samples in one launch
vcas_status sampler_a_group(const SampleAGroup &grp, int n, int N, int T, hipStream_t st)
{
    if (n < 1 || n > kMaxSamplers || N > 1024) return VCAS_EINVAL;
    hipLaunchKernelGGL(sampler_a_group_kernel, dim3(n), dim3(1024), 0, st, grp, N, T);
    return launch_status();
}

// Norm pass, apply and list of one layer with cached norms, mask bytes against counts: 65536 rows 8.0 and 9.1 us, 131072 9.4
// and 9.5, 262144 12.6 and 11.0, 2^20 37 and 23, 2^24 5351 and 347.
constexpr int kListRows = 131072;

// SampleW of n <= kMaxSamplers layers with one N and T in one set of launches.  Up to 16384 rows one
// workgroup per layer does everything; beyond, see sampler_w_rule_kernel and what
// follows it.
vcas_status sampler_w_group(const SampleWGroup &grp, int n, int N, int T, int token_sampling, int roots_given, hipStream_t st)
{
    const int64_t R64 = (int64_t)N * T;
    if (n < 1 || n > kMaxSamplers || R64 > (int64_t)1 << 30) return VCAS_EINVAL;
    const int R = (int)R64;
#define VCAS_SAMPLER_W(E) \
    if (R <= 1024 * (E)) { \
        hipLaunchKernelGGL(sampler_w_group_kernel<E>, dim3(n), dim3(1024), 0, st, grp, N, T, token_sampling, \
                           roots_given); \
        return launch_status(); \
    }
    VCAS_SAMPLER_W(1)
    VCAS_SAMPLER_W(4)
    VCAS_SAMPLER_W(8)
    VCAS_SAMPLER_W(16)
#undef VCAS_SAMPLER_W
    if (roots_given) hipLaunchKernelGGL(sampler_w_scores_kernel, dim3((R + 255) / 256, n), dim3(256), 0, st, grp, R, T);
    if (token_sampling) {
        if (R <= 32768) hipLaunchKernelGGL(sampler_w_rule_kernel<32>, dim3(n), dim3(1024), 0, st, grp, R);
        else if (R <= 65536) hipLaunchKernelGGL(sampler_w_rule_kernel<64>, dim3(n), dim3(1024), 0, st, grp, R);
        else hipLaunchKernelGGL(sampler_w_rule_kernel<0>, dim3(n), dim3(1024), 0, st, grp, R);
    }
    const dim3 by256((R + 255) / 256, n);
    if (R <= kListRows) {
        hipLaunchKernelGGL(sampler_w_apply_kernel<false>, by256, dim3(256), 0, st, grp, R, T, token_sampling);
        hipLaunchKernelGGL(sampler_w_list_kernel, dim3((R + 1023) / 1024, n), dim3(1024), 0, st, grp, R);
    } else {
        hipLaunchKernelGGL(sampler_w_apply_kernel<true>, by256, dim3(256), 0, st, grp, R, T, token_sampling);
        hipLaunchKernelGGL(sampler_w_places_kernel, dim3(n), dim3(1024), 0, st, grp, R);
        hipLaunchKernelGGL(sampler_w_place_kernel, by256, dim3(256), 0, st, grp, R);
    }
    return launch_status();
}

}  // namespace vcas
