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
// The implicit patch matrix of a convolution: A is its channels-last input of batch x H x W x C (M = batch OH OW rows, K = R S C).
struct ConvRows { int H, W, C, OW, S, sh, sw, ph, pw, dh, dw; unsigned ohow; };
// bm, whole, slabs, fast: the FP32 tiles' rows, whether all of them are regular, whether they load 32 channels of a tap at a time, whether they
// accumulate in one chain
bool f64_conv_route(const LinearProblem& p, const ConvRows& cv, long xbytes, long bm, bool whole, bool slabs, bool fast, int cus);
int f64_conv_launch(const LinearProblem& p, const ConvRows& cv, long xbytes, const tao_fp_model& md, double gamma, int cus, hipStream_t st);
bool f64_route(const LinearProblem& p, int cus);          // is this kernel the faster one?
double linear_us(long M, long N, long K, long batch, int cus);     // what tao_bound_linear takes, contiguous operands
int f64_launch(const LinearProblem& p, const tao_fp_model& md, double gamma, int cus, hipStream_t st);

}  // namespace tao
