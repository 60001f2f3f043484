// The matmul bound on the binary64 matrix cores (linear_f64.hip), for outputs too small to fill the chip
// with the tiles of linear.hip.
#pragma once
#include "tao_host.hpp"

namespace tao {

struct LinearProblem {               // arguments of tao_bound_linear, validated
    const float* A; const float* W; const float* bias; float* tau;
    long M, N, K, lda, ldw, ldt;
    bool trans_w;
    long batch, strideA, strideW, strideT;
};
bool f64_route(const LinearProblem& p, int cus);          // is this kernel the faster one?
double linear_us(long M, long N, long K, long batch, int cus);     // what tao_bound_linear takes, contiguous operands
int f64_launch(const LinearProblem& p, const tao_fp_model& md, double gamma, int cus, hipStream_t st);

}  // namespace tao
