// Argument blocks and launchers of the variance probe (probe.hip).
#pragma once

#include "common.hpp"

namespace vcas {

constexpr int kProbeDraws = 8;   // mask draws that go through the launches together, at the most

// One mask draw: what SampleA has decided, and where SampleW's inputs and the lists go.
struct ProbeDraw {
    uint32_t index;            // rng.draw of this draw
    const float *p, *gnorm;
    const uint8_t *maskA;
    const int32_t *idxA, *cntA;
    float *u, *score;          // [R]
    const float *q;            // [R], SampleW's outcome
    int32_t *list_a, *rows_a;  // [R] rows of kept samples, and how many
    double *closed;            // [2] Sec. 4.1's variance under p, and Eq. 3 under this draw's data mask
};
struct ProbeDraws {
    ProbeDraw draw[kProbeDraws];
};

// Scratch of one draw in bytes (a multiple of 256): its SampleA and SampleW vectors.
inline size_t probe_pad(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
inline size_t probe_draw_bytes(int64_t N, int64_t R)
{
    return 5 * probe_pad(4 * R) + probe_pad(R) + 3 * probe_pad(4 * N) + probe_pad(N) + 256;
}
// n draws together: their vectors (those of the probe's last draw, or of a draw that goes alone, lie in the plan), a
// row list and a few words for each, and 1/p of every row.
inline size_t probe_chunk_bytes(int64_t N, int64_t R, int n)
{
    return (n > 1 ? n * probe_draw_bytes(N, R) : 0) + (n + 1) * probe_pad(4 * R) + n * 256;
}
// How many draws go together.  Their scratch is part of every layer's workspace: 64 MiB of it (eight draws of 328000 rows),
// or half of what the layer's G and X take.
inline int probe_chunk(const vcas_shape &s)
{
    const int64_t R = (int64_t)s.N * s.T;
    const size_t rows = (size_t)R * (s.K_in + s.K_out) * elem_bytes(s.dtype) / 2, room = rows > (64u << 20) ? rows : 64u << 20;
    int n = kProbeDraws;
    while (n > 1 && probe_chunk_bytes(s.N, R, n) > room) --n;
    return n;
}
vcas_status probe_begin(float *ones, int32_t *iota, int32_t *cnt, double *out, int64_t R, hipStream_t st);
vcas_status probe_draws(const ProbeDraws &d, int n, const float *gsq, const float *xsq, float *scale_a, int64_t R, int T,
                        const vcas_rng &rng, hipStream_t st);
// last: which of the n draws is the probe's last one (-1: none)
vcas_status probe_closed(const ProbeDraws &d, int n, int64_t R, int N, int T, float *xsq, int last, hipStream_t st);
vcas_status probe_finish(const ProbeDraws &d, int n, const double *sq, int tiles, double weight, bool first, double *out,
                         hipStream_t st);
// out += weight * ||a - b||^2 unless the first n_closed closed forms are all zero; partial: 32 doubles
vcas_status sq_diff_add(const float *a, const float *b, int64_t n, double weight, double *partial, const double *closed,
                        int n_closed, double *out, hipStream_t st);

}  // namespace vcas
