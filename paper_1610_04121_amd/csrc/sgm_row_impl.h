// The row kernel of one padded disparity range and its launcher (included by
// sgm_row_64.hip, sgm_row_128.hip and sgm_row_256.hip).
#pragma once

#include "sgm_row.h"

namespace sgm {

namespace {

using namespace dev;

template <int Dp, int NV, typename LT, bool NT, bool PAIR, bool SUB>
__global__ __launch_bounds__(512) void row_kernel(RowLaunch k) {
    extern __shared__ uint32_t row_smem[];
    __shared__ uint16_t p2lut[256];
    RowArgs a = k.l;
    int y = blockIdx.x;
    if (k.n > 0) {
        const BatchItem& it = k.items[find_item<&BatchItem::wta_blk0>(k.items, k.n, y)];
        y -= it.wta_blk0;
        const size_t plane = (size_t)it.W * it.H * Dp;
        const bool post = it.median || it.lrcheck, rb = y >= it.H;
        if (rb) y -= it.H;
        // right-base rows (full check): planes P .. 2P - 1, winners into D_R
        a = RowArgs{rb ? it.cost_r : it.cost,
                    static_cast<const LT*>(it.lbuf) + (rb ? plane * it.P : 0),
                    rb ? it.right : it.left,
                    rb ? it.dr : (post ? it.dl : it.out),
                    (it.lrcheck && !it.lr_full) ? it.dr : nullptr,
                    it.W, it.H, it.D, k.P1, k.P2, it.P, it.adaptive, SUB && !rb};
    } else if (y >= a.H) {
        y -= a.H;
        a = k.r;
    }
    for (int g = threadIdx.x; g < 256; g += blockDim.x)
        p2lut[g] = (uint16_t)(a.adaptive ? adaptive_p2((uint32_t)a.P1, (uint32_t)a.P2, (uint32_t)g) : (uint32_t)a.P2);
    __syncthreads();
    row_block<Dp, NV, LT, NT, PAIR, SUB>(a, y, row_smem, p2lut);
}

template <int Dp, int NV, bool SUB>
hipError_t launch_row_t(const RowLaunch& a, const RowVariant& v, int blocks, int waves, size_t smem, hipStream_t stream) {
    auto k = v.nt ? row_kernel<Dp, NV, uint16_t, true, false, SUB> : row_kernel<Dp, NV, uint16_t, false, false, SUB>;
    if (!v.l16) {
        if (v.pair)
            k = v.nt ? row_kernel<Dp, NV, uint8_t, true, true, SUB> : row_kernel<Dp, NV, uint8_t, false, true, SUB>;
        else
            k = v.nt ? row_kernel<Dp, NV, uint8_t, true, false, SUB> : row_kernel<Dp, NV, uint8_t, false, false, SUB>;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(64 * waves), smem, stream, a);
    return hipGetLastError();
}

template <int Dp>
hipError_t launch_row_dp(const RowLaunch& a, const RowVariant& v, int blocks, int waves, size_t smem, hipStream_t stream) {
    auto launch = v.n_paths == 2   ? (v.sub ? launch_row_t<Dp, 1, true> : launch_row_t<Dp, 1, false>)
                  : v.n_paths == 4 ? (v.sub ? launch_row_t<Dp, 2, true> : launch_row_t<Dp, 2, false>)
                                   : (v.sub ? launch_row_t<Dp, 6, true> : launch_row_t<Dp, 6, false>);
    return launch(a, v, blocks, waves, smem, stream);
}

}  // namespace

}  // namespace sgm
