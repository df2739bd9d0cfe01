// Launches of the gathering weight gradient (wgrad_gather.hpp).
#include "wgrad_gather.hpp"

namespace vcas {

template <bool BF16, int PA, int PB, int SK, int WM, int WN, int WK, bool DIFF>
__global__ __launch_bounds__(WM *WN *WK * 64) void wgrad_gather_kernel(GatherBatch batch)
{
    // the task whose range holds this workgroup (ranges ascend)
    int p = 0;
    for (int i = 1; i < batch.n; ++i)
        if ((int)blockIdx.x >= batch.task[i].first_wg) p = i;
    const GatherTask &q = batch.task[p];
    wgrad_gather_body<BF16, PA, PB, SK, WM, WN, WK, DIFF>(q, (int)blockIdx.x - q.first_wg);
}

int gather_tiles(int dtype, int K_out, int K_in, bool large)
{
    const int edge = (dtype == VCAS_BF16 ? 64 : 32) * (large ? 2 : 1);
    return ((K_out + edge - 1) / edge) * ((K_in + edge - 1) / edge);
}

int gather_step(int dtype, bool large) { return dtype == VCAS_F32 && large ? 32 : 64; }

template <bool BF16, int PA, int PB, int SK, int WM, int WN, int WK, bool DIFF>
static vcas_status launch_gather(const GatherBatch &batch, int grid, hipStream_t st)
{
    const size_t lds = 2 * SK * (PA + PB) + 2048;
    auto kern = wgrad_gather_kernel<BF16, PA, PB, SK, WM, WN, WK, DIFF>;
    static bool allowed = false;
    if (!allowed) {
        if (!allow_lds(kern, lds)) return VCAS_EHIP;
        allowed = true;
    }
    launch_timed(1, kern, dim3((unsigned)grid), dim3(WM * WN * WK * 64), lds, st, batch);
    return launch_status();
}

vcas_status wgrad_gather(GatherTask *tasks, int n, int dtype, bool large, bool diff, hipStream_t st)
{
    if (n < 1 || n > kGatherBatch) return VCAS_EINVAL;
    const int edge = (dtype == VCAS_BF16 ? 64 : 32) * (large ? 2 : 1);
    GatherBatch batch = {};
    batch.n = n;
    int64_t grid = 0;
    for (int i = 0; i < n; ++i) {
        GatherTask &q = tasks[i];
        q.tiles_n = (q.K_in + edge - 1) / edge;
        q.tiles = ((q.K_out + edge - 1) / edge) * q.tiles_n;
        if (q.splits < 1 || diff) q.splits = 1;
        q.first_wg = (int32_t)grid;
        grid += ((int64_t)q.tiles * q.splits + 7) / 8 * 8;
        batch.task[i] = q;
    }
    if (grid > (int64_t)1 << 30) return VCAS_EINVAL;
    if (dtype == VCAS_BF16) {
        if (large) return diff ? launch_gather<true, 256, 256, 64, 2, 4, 1, true>(batch, (int)grid, st)
                               : launch_gather<true, 256, 256, 64, 2, 4, 1, false>(batch, (int)grid, st);
        return diff ? launch_gather<true, 128, 128, 64, 2, 2, 2, true>(batch, (int)grid, st)
                    : launch_gather<true, 128, 128, 64, 2, 2, 2, false>(batch, (int)grid, st);
    }
    if (large) return diff ? launch_gather<false, 256, 256, 32, 2, 2, 1, true>(batch, (int)grid, st)
                           : launch_gather<false, 256, 256, 32, 2, 2, 1, false>(batch, (int)grid, st);
    return diff ? launch_gather<false, 128, 128, 64, 1, 1, 4, true>(batch, (int)grid, st)
                : launch_gather<false, 128, 128, 64, 1, 1, 4, false>(batch, (int)grid, st);
}

}  // namespace vcas
