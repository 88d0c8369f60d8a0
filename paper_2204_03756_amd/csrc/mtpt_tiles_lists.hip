// mtpt_tiles_lists.hip -- the neighbour-list variants of the 3-d row-sum and
// transfer passes (see mtpt_lists.h).
#include "mtpt_device.h"

namespace mtpt {

// The neighbour-list variants (3-d, FP64, isotropic; see mtpt_lists.h), held to
// the four waves per SIMD that their LDS allows.
__global__ __launch_bounds__(kListBlock, 4) void rowsum_list_k(SimArgs a)
{
    tile_body<3, 0, 1, false, false, false, true>(kernel_args(), xcd_block(blockIdx.x, gridDim.x));
}
template <int NS>
__global__ __launch_bounds__(kListBlock, 4) void transfer_list_k(SimArgs a)
{
    uint32_t blk = blockIdx.x, n = gridDim.x;
    if (a.fin_partials) {
        if (blk == 0) {
            finalize_body<kListBlock>(a, a.fin_partials, a.fin_counted != 0, a.nttiles, 0);
            return;
        }
        --blk;
        --n;
    }
    tile_body<3, 0, NS, true, false, false, true>(kernel_args(), xcd_block(blk, n));
}
__global__ __launch_bounds__(kListBlock) void rowsum_list_export_k(SimArgs a)
{
    tile_body<3, 0, 1, false, false, true, true>(a, xcd_block(blockIdx.x, gridDim.x));
}
template <int NS>
__global__ __launch_bounds__(kListBlock) void transfer_list_export_k(SimArgs a)
{
    tile_body<3, 0, NS, true, false, true, true>(a, xcd_block(blockIdx.x, gridDim.x));
}

hipError_t launch_lists(int ph, int ns, const SimArgs& a, hipStream_t s)
{
    const uint32_t grid = a.ntiles + (ph == PH_TRANSFER && a.fin_partials ? 1u : 0u);
    if (grid == 0 || a.n <= 0)
        return hipSuccess;
    if (ph == PH_ROWSUM) rowsum_list_k<<<grid, kListBlock, 0, s>>>(a);
    else if (ph != PH_TRANSFER) return hipErrorInvalidValue;
    else if (ns == 1) transfer_list_k<1><<<grid, kListBlock, 0, s>>>(a);
    else transfer_list_k<3><<<grid, kListBlock, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_lists_export(int ph, int ns, const SimArgs& a, hipStream_t s)
{
    const uint32_t grid = a.ntiles;
    if (grid == 0 || a.n <= 0)
        return hipSuccess;
    if (ph == PH_ROWSUM) rowsum_list_export_k<<<grid, kListBlock, 0, s>>>(a);
    else if (ph != PH_TRANSFER) return hipErrorInvalidValue;
    else if (ns == 1) transfer_list_export_k<1><<<grid, kListBlock, 0, s>>>(a);
    else transfer_list_export_k<3><<<grid, kListBlock, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace mtpt
