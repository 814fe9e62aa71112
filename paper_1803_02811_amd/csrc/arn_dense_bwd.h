// The dense layers' backward pass in one launch: once d(pre_fc) exists, the fc layer's input gradient, its weight
// gradient, the head's weight gradient and the totals of the reported losses are independent of each other, so they
// are four ranges of workgroups of one grid.
#pragma once
#include "arn_gemm.h"
#include "arn_problems.h"
#include "arn_resident_conv.h"
#include "arn_small_kernels.h"

namespace arn {

constexpr int DENSE_THREADS = 256;

struct LossTotals {   // arguments of loss_finalize
    const float *partial;
    int blocks, B;
    float value_coef, entropy_coef;
    float *loss;
};

template <class Dgrad, class Wgrad, class HeadW>
struct DenseBackwardArgs {
    Dgrad dg;                       // fc input gradient
    int dg_x, dg_blocks;            // position tiles, workgroups
    Wgrad wg;                       // fc weight gradient
    float *wg_part;
    int wg_rows, wg_blocks;         // samples per batch split, workgroups
    HeadW hw;                   // head weight gradient
    float *hw_part;
    int hw_rows, hw_blocks;
    LossTotals loss;                // one workgroup
};

template <class Dgrad, class Wgrad, class HeadW>
__global__ __launch_bounds__(DENSE_THREADS) void dense_backward_kernel(const DenseBackwardArgs<Dgrad, Wgrad, HeadW> a) {
    // the weight gradients take as many stages as the input gradient's LDS holds
    constexpr int L1 = gemm_nt_lds_bytes<Dgrad>(), R2 = L1 / gemm_tn_stage_bytes<Wgrad>(), R3 = L1 / gemm_tn_stage_bytes<HeadW>();
    static_assert(NT_THREADS == DENSE_THREADS, "one block size for all ranges");
    __shared__ u32x4 lds[L1 / 16];
    int b = blockIdx.x;
    if (b < a.dg_blocks) {
        gemm_nt_body<Dgrad>(lds, a.dg, b % a.dg_x, b / a.dg_x, 0, a.dg_x, 1, 1);
        return;
    }
    b -= a.dg_blocks;
    if (b < a.wg_blocks) {
        constexpr int X = Wgrad::KP / Wgrad::BK2, Y = Wgrad::N1 / Wgrad::BN1;
        gemm_tn_body<Wgrad, R2>(lds, a.wg, a.wg_part, a.wg_rows, b % X, b / X % Y, b / (X * Y));
        return;
    }
    b -= a.wg_blocks;
    if (b < a.hw_blocks) {
        constexpr int X = HeadW::KP / HeadW::BK2;
        const int Y = a.hw.N1 / HeadW::BN1;
        gemm_tn_body<HeadW, R3>(lds, a.hw, a.hw_part, a.hw_rows, b % X, b / X % Y, b / (X * Y));
        return;
    }
    loss_finalize(a.loss.partial, a.loss.blocks, a.loss.B, a.loss.value_coef, a.loss.entropy_coef, a.loss.loss);
}

}  // namespace arn
