// Kernels of the variance probe (Sec. 4.1, Eq. 3, the Monte-Carlo lines of Alg. 1) between the samplers and the
// products.  All mask draws of a chunk go through every launch together: the row norms do not depend on the
// draw, and one draw's vectors and weight gradients are far too small to fill the chip (BERT-base and ViT
// shapes: 36 to 144 output tiles).  The products are formed by the gathering weight-gradient kernel in its
// comparing form, which adds up squared distances from the exact gradient instead of storing the draw's.
// Measured, a probe of 8 draws at 64x197, 768x768 bf16: 1438 us draw by draw (21 launches each, among them two
// norm passes and two 24 us comparisons by 32 workgroups), 225 us now, of which the comparing products 130.
#include "probe.hpp"

namespace vcas {

// Every token with scale one (the exact gradient), and the four results zeroed.
__global__ __launch_bounds__(256) void probe_begin_kernel(float *__restrict__ ones, int32_t *__restrict__ iota,
                                                          int32_t *__restrict__ cnt, double *__restrict__ out, int R)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < R) {
        ones[t] = 1.0f;
        iota[t] = t;
    }
    if (t == 0) *cnt = R;
    if (t < 4) out[t] = 0.0;
}

// SampleA of the draws is done: uniforms and scores of SampleW ((1/p_i) sqrt(gsq) sqrt(xsq), 0 on dropped
// samples), the list of the rows of kept samples, and (draw 0; the probabilities are the same in every
// draw) 1/p of every row.  blockIdx.y = draw.
__global__ __launch_bounds__(256) void probe_draws_kernel(ProbeDraws d, const float *__restrict__ gsq,
                                                          const float *__restrict__ xsq, float *__restrict__ scale_a,
                                                          int R, int T, uint64_t seed, uint32_t layer,
                                                          const uint32_t *__restrict__ draw_offset)
{
    const ProbeDraw &w = d.draw[blockIdx.y];
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= R) return;
    const uint32_t draw = w.index + (draw_offset ? *draw_offset : 0u);
    w.u[t] = philox_uniform(seed, layer, 1u, draw, (uint32_t)t);
    const int i = t / T;
    const float p = w.p[i];
    float s = 0.0f;
    if (w.maskA[i]) {
        const float inv = 1.0f / p;
        const float a = inv * __builtin_sqrtf(gsq[t]);
        s = a * __builtin_sqrtf(xsq[t]);
    }
    w.score[t] = s;
    if (blockIdx.y == 0) scale_a[t] = p > 0.0f ? 1.0f / p : 0.0f;
    const int rows = min(max(*w.cntA, 0) * T, R);
    if (t < rows) w.list_a[t] = w.idxA[i] * T + t % T;
    if (t == 0) *w.rows_a = rows;
}

// The closed forms of one draw (fp64, fixed order), one workgroup each: sum of (1 - p)/p gnorm^2 over p > 0, and Eq. 3
// under the draw's data mask, the sum of (1 - q)/q score^2 over q > 0.  Where the draw is the last one, also zeroes
// the norms of X of its dropped samples, as the plan wants.
__global__ __launch_bounds__(1024) void probe_closed_kernel(ProbeDraws d, int R, int N, int T, float *__restrict__ xsq, int last)
{
    __shared__ double sh[16], sh_a[16];
    const ProbeDraw &w = d.draw[blockIdx.x];
    double acc = 0.0;
    for (int t0 = threadIdx.x; t0 < R; t0 += 4 * 1024) {
        float q[4], s[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = min(t0 + 1024 * k, R - 1);
            q[k] = w.q[t];
            s[k] = w.score[t];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = t0 + 1024 * k;
            if (t >= R) continue;
            const double qd = q[k], v = s[k];
            if (qd > 0.0) acc += (1.0 - qd) / qd * (v * v);
            if ((int)blockIdx.x == last && !w.maskA[t / T]) xsq[t] = 0.0f;
        }
    }
    double acc_a = 0.0;
    for (int i = threadIdx.x; i < N; i += 1024) {
        const double pr = w.p[i], g = w.gnorm[i];
        if (pr > 0.0) acc_a += (1.0 - pr) / pr * (g * g);
    }
    acc = wave_exchange_sum(acc);
    acc_a = wave_exchange_sum(acc_a);
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6] = acc;
        sh_a[threadIdx.x >> 6] = acc_a;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        w.closed[0] = tree16(sh_a);
        w.closed[1] = tree16(sh);
    }
}

// Every probability that these closed forms sum over is 0 or 1: the draw can only be the exact gradient, and its distance is
// zero.  The kernels that form the two add in different orders, so that what they differ by is rounding.
__device__ __forceinline__ bool no_choice(const double *closed, int n)
{
    return closed[0] == 0.0 && (n < 2 || closed[1] == 0.0);
}

__device__ __forceinline__ double block_sum_256(double v, double *sh)
{
    v = wave_exchange_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Adds a chunk of n draws to the four results: tile sums of the products (draw k: SampleA only in
// sq[k * tiles ..], both samplers in sq[(n + k) * tiles ..]; null: added elsewhere), Eq. 3 of each draw,
// and with the first chunk the closed form over the samples (the same in every draw).
__global__ __launch_bounds__(256) void probe_finish_kernel(ProbeDraws d, int n, const double *__restrict__ sq, int tiles,
                                                           double weight, int first, double *__restrict__ out)
{
    __shared__ double sh[4];
    __shared__ int skip[2 * kProbeDraws];
    if (sq) {
        if ((int)threadIdx.x < 2 * n) skip[threadIdx.x] = no_choice(d.draw[threadIdx.x % n].closed, 1 + threadIdx.x / n);
        __syncthreads();
        for (int w = 0; w < 2; ++w) {
            double acc = 0.0;
            for (int i = threadIdx.x; i < n * tiles; i += 256) {
                const double one = sq[(int64_t)w * n * tiles + i];
                acc += skip[w * n + i / tiles] ? 0.0 : one;
            }
            acc = block_sum_256(acc, sh);
            if (threadIdx.x == 0) out[2 + w] += weight * acc;
        }
    }
    if (threadIdx.x == 0) {
        if (first) out[0] = d.draw[0].closed[0];
        double s = 0.0;
        for (int k = 0; k < n; ++k) s += d.draw[k].closed[1];
        out[1] += weight * s;
    }
}

// per-block partial sums of (a-b)^2, then a one-block pass adds them in order (products too large for
// the comparing kernel's 32-bit offsets)
__global__ __launch_bounds__(256) void sq_diff_partial_kernel(const float *__restrict__ a, const float *__restrict__ b,
                                                              int64_t n, double *__restrict__ partial)
{
    __shared__ double sh[4];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double d = (double)a[i] - (double)b[i];
        acc += d * d;
    }
    acc = block_sum_256(acc, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

__global__ __launch_bounds__(64) void sq_diff_final_kernel(const double *__restrict__ partial, int blocks,
                                                           double weight, const double *__restrict__ closed, int n_closed,
                                                           double *__restrict__ out)
{
    if (threadIdx.x != 0 || no_choice(closed, n_closed)) return;
    double s = 0.0;
    for (int i = 0; i < blocks; ++i) s += partial[i];
    *out += weight * s;
}

size_t probe_scratch_bytes(const vcas_shape &s) { return probe_chunk_bytes(s.N, (int64_t)s.N * s.T, probe_chunk(s)); }

// ---- host launchers ---------------------------------------------------------------------------

vcas_status probe_begin(float *ones, int32_t *iota, int32_t *cnt, double *out, int64_t R, hipStream_t st)
{
    hipLaunchKernelGGL(probe_begin_kernel, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, st, ones, iota, cnt, out, (int)R);
    return launch_status();
}

vcas_status probe_draws(const ProbeDraws &d, int n, const float *gsq, const float *xsq, float *scale_a, int64_t R, int T,
                        const vcas_rng &rng, hipStream_t st)
{
    hipLaunchKernelGGL(probe_draws_kernel, dim3((unsigned)((R + 255) / 256), n), dim3(256), 0, st, d, gsq, xsq, scale_a, (int)R, T,
                       rng.seed, rng.layer, rng.draw_offset);
    return launch_status();
}

vcas_status probe_closed(const ProbeDraws &d, int n, int64_t R, int N, int T, float *xsq, int last, hipStream_t st)
{
    hipLaunchKernelGGL(probe_closed_kernel, dim3(n), dim3(1024), 0, st, d, (int)R, N, T, xsq, last);
    return launch_status();
}

vcas_status probe_finish(const ProbeDraws &d, int n, const double *sq, int tiles, double weight, bool first, double *out,
                         hipStream_t st)
{
    hipLaunchKernelGGL(probe_finish_kernel, dim3(1), dim3(256), 0, st, d, n, sq, tiles, weight, first ? 1 : 0, out);
    return launch_status();
}

vcas_status sq_diff_add(const float *a, const float *b, int64_t n, double weight, double *partial, const double *closed,
                        int n_closed, double *out, hipStream_t st)
{
    const int blocks = 32;   // what `partial` has room for
    hipLaunchKernelGGL(sq_diff_partial_kernel, dim3(blocks), dim3(256), 0, st, a, b, n, partial);
    hipLaunchKernelGGL(sq_diff_final_kernel, dim3(1), dim3(64), 0, st, partial, blocks, weight, closed, n_closed, out);
    return launch_status();
}

}  // namespace vcas
