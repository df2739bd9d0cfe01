// Launches of the gathering weight gradient (wgrad_gather.hpp, f32_split.hpp, wgrad_staged.hpp).
#include "f32_split.hpp"
#include "wgrad_staged.hpp"

namespace vcas {

template <int SK, int WM, int WN, int WK, bool DIFF>
__global__ __launch_bounds__(WM *WN *WK * 64) void wgrad_gather_kernel(GatherBatch batch)
{
    // the task whose range holds this workgroup (ranges ascend)
    int p = 0;
    for (int i = 1; i < batch.n; ++i)
        if ((int)blockIdx.x >= batch.task[i].first_wg) p = i;
    const GatherTask &q = batch.task[p];
    wgrad_gather_body<SK, WM, WN, WK, DIFF>(q, (int)blockIdx.x - q.first_wg);
}

// bf16 (STAGED), or fp32 from the bf16 parts of its operands.
template <bool STAGED, int BM, int BN, int WM, int WN, int WK, bool DIFF>
__device__ __forceinline__ void wgrad_tile_of(const GatherBatch &batch)
{
    int p = 0;
    for (int i = 1; i < batch.n; ++i)
        if ((int)blockIdx.x >= batch.task[i].first_wg) p = i;
    const GatherTask &q = batch.task[p];
    if constexpr (STAGED) wgrad_staged_body<BM, BN, WM, WN, WK, DIFF>(q, (int)blockIdx.x - q.first_wg);
    else wgrad_split_body<BM, BN, WM, WN, WK, DIFF>(q, (int)blockIdx.x - q.first_wg);
}
template <int BM, int BN, int WM, int WN, int WK, bool DIFF>
__global__ __launch_bounds__(WM *WN *WK * 64, 4) void wgrad_staged_kernel(GatherBatch batch)
{
    wgrad_tile_of<true, BM, BN, WM, WN, WK, DIFF>(batch);
}
template <int BM, int BN, int WM, int WN, int WK, bool DIFF>
__global__ __launch_bounds__(512) void wgrad_split_kernel(GatherBatch batch)
{
    wgrad_tile_of<false, BM, BN, WM, WN, WK, DIFF>(batch);
}

template <typename Kern>
static vcas_status launch_tiles(Kern kern, int threads, size_t lds, bool &allowed, const GatherBatch &batch, int grid, hipStream_t st)
{
    if (!allowed) {
        if (!allow_lds(kern, lds)) return VCAS_EHIP;
        allowed = true;
    }
    launch_timed(1, kern, dim3((unsigned)grid), dim3(threads), lds, st, batch);
    return launch_status();
}

template <int BM, int BN, int WM, int WN, int WK, bool DIFF>
static vcas_status launch_split(const GatherBatch &batch, int grid, hipStream_t st)
{
    static_assert(WM * WN * WK == 8, "512 threads");
    static bool allowed = false;
    return launch_tiles(wgrad_split_kernel<BM, BN, WM, WN, WK, DIFF>, 512, split_lds(BM, BN, WK), allowed, batch, grid, st);
}

template <int BM, int BN, int WM, int WN, int WK, bool DIFF>
static vcas_status launch_staged(const GatherBatch &batch, int grid, hipStream_t st)
{
    static bool allowed = false;
    return launch_tiles(wgrad_staged_kernel<BM, BN, WM, WN, WK, DIFF>, WM * WN * WK * 64, staged_lds(BM, BN), allowed, batch, grid, st);
}

template <int SK, int WM, int WN, int WK, bool DIFF>
static vcas_status launch_gather(const GatherBatch &batch, int grid, hipStream_t st)
{
    const size_t lds = 2 * SK * 256 + 2048;   // two stages of both tiles, tokens and scales
    auto kern = wgrad_gather_kernel<SK, WM, WN, WK, DIFF>;
    static bool allowed = false;
    if (!allowed) {
        if (!allow_lds(kern, lds)) return VCAS_EHIP;
        allowed = true;
    }
    launch_timed(1, kern, dim3((unsigned)grid), dim3(WM * WN * WK * 64), lds, st, batch);
    return launch_status();
}

vcas_status wgrad_gather(GatherTask *tasks, int n, int dtype, GatherTile tile, bool diff, hipStream_t st)
{
    if (n < 1 || n > kGatherBatch) return VCAS_EINVAL;
    const int edge = gather_edge(dtype, tile);
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
        if (tile == kLargeTile) return diff ? launch_staged<128, 128, 2, 4, 1, true>(batch, (int)grid, st)
                                            : launch_staged<128, 128, 2, 4, 1, false>(batch, (int)grid, st);
        return diff ? launch_staged<64, 64, 2, 2, 2, true>(batch, (int)grid, st)
                    : launch_staged<64, 64, 2, 2, 2, false>(batch, (int)grid, st);
    }
    if (tile == kLargeTile) return diff ? launch_split<128, 128, 2, 4, 1, true>(batch, (int)grid, st)
                                          : launch_split<128, 128, 2, 4, 1, false>(batch, (int)grid, st);
    if (tile == kMidTile) return diff ? launch_split<64, 64, 2, 2, 2, true>(batch, (int)grid, st)
                                        : launch_split<64, 64, 2, 2, 2, false>(batch, (int)grid, st);
    return diff ? launch_gather<64, 1, 1, 4, true>(batch, (int)grid, st)
                : launch_gather<64, 1, 1, 4, false>(batch, (int)grid, st);
}

}  // namespace vcas
