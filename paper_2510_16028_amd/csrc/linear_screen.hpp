// Screening of a checked matmul bound: one BF16 product decides the comparisons that six would (linear_screen.hip).
#pragma once
#include "tao_check.hpp"

namespace tao {

// An operand of the screening product.  Image: as tao_split_operand writes it (its blocks begin with their hi pieces).
// Rows: the binary32 matrix itself (16-byte aligned rows, whole groups of 32 k).
// Pixels: BF16 magnitudes [batch][H][W][C] of a convolution's input, whose patch matrix the operand is (C a multiple of 32).
struct ScreenPixels {
    int H, W, C, OW, S, sh, sw, ph, pw, dh, dw;
    unsigned ohow;
    int slabs;                 // C / 32
    unsigned zeros;            // offset in bytes of 64 bytes of zeros
};
struct ScreenOperand {
    const void* data;
    long batch_bytes;          // 0: shared
    long ld;                   // rows: elements between rows; otherwise 0
    const ScreenPixels* pixels;
};
constexpr long kScreenMaxLd = 1L << 22;      // rows of claims and outputs, and of binary32 operands: 32-bit offsets within a tile

struct ScreenCheck { const float* claimed; const float* ref; long ldy, strideY; double alpha, eps_rel; };

// A screened check divides the partial results among the screen (the first half) and the exact route behind it (the second);
// all of the check's workspace is zero before the screen.  The words of the counters that no check writes hold the flag that the
// screen could not settle every element and the exact route's counts of finished tiles and parts.
constexpr int kScreenSlots = kMaxCheckBlocks / 2;
constexpr int kOpenFlag = kMaxCheckBlocks - 1, kDoneFlag = kMaxCheckBlocks - 2, kMaxTileFlags = kMaxCheckBlocks - 2;
inline CheckWorkspace screened_second_half(const CheckWorkspace& w) {
    return {w.hist + (size_t)kScreenSlots * kBins, w.coarse + (size_t)kScreenSlots * kGroups, w.stats + kScreenSlots};
}

// Whether the screen can decide for these constants (u: the model's, cg: Gamma with its guard factor; see linear_screen.hip).
bool screen_usable(long K, double u, double cg, double alpha, double uflow);
int launch_screen(const ScreenOperand& A, const ScreenOperand& W, const float* bias, long M, long N, long K, long batch,
                  double cg, const ScreenCheck& chk, const CheckWorkspace& ws, hipStream_t st);

}  // namespace tao
