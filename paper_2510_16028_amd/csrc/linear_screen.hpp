// Screening of a checked matmul bound: one BF16 product decides the comparisons that six would (linear_screen.hip).
#pragma once
#include <cmath>
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

// A screened check keeps few partial results (they are cleared before and added up after each call): the first kScreenSlots, to which
// the screen adds, and the exact route its violations.  The words of the counters that no check writes hold, one for each of them, in how
// many tiles the screen left comparisons open, and how many of these the exact route has finished.
constexpr int kScreenSlots = 64;              // (32 cost perturbed claims of 1111 x 3001 2 us, 128 honest ones 0.4)
constexpr int kDoneFlag = kMaxCheckBlocks - 1;
static_assert(kScreenSlots == kWave, "a lane for each");
// The comparisons that the screen left open in a tile of the exact route (128 x 128 outputs; tiles row by row, batch entries one after
// the other).  All zero before the screen; zero after it where none is open.
constexpr int kOpenTile = 128, kOpenList = 14;
constexpr unsigned kNoPlace = ~0u;
struct OpenTile {
    unsigned state;            // bit 4 r + c: every comparison of block (r, c), 32 x 32; from bit 16 on: how many places were asked for
    unsigned arrived;          // parts of the reduction that the exact route has finished
    unsigned at[kOpenList];    // places: 128 row + column, or kNoPlace
};
static_assert(sizeof(OpenTile) == 64, "cleared in 16-byte words");
inline size_t open_tiles_of(long M, long N, long batch) {
    return (size_t)((M + kOpenTile - 1) / kOpenTile) * (size_t)((N + kOpenTile - 1) / kOpenTile) * (size_t)batch;
}
// What a launch before a check clears, in 16-byte words: of `slots` partial results the histograms and coarse counts, all counters, and
// a screened check's records.
struct ClearJob { void* at[4]; long words[4]; };
inline ClearJob clear_job(const CheckWorkspace& w, int slots, OpenTile* open = nullptr, size_t tiles = 0) {
    return {{w.hist, w.coarse, w.stats, open},
            {(long)slots * kBins / 4, (long)slots * kGroups / 4, (long)(kMaxCheckBlocks * sizeof(BlockStats) / 16), (long)(tiles * sizeof(OpenTile) / 16)}};
}
static_assert(kMaxCheckBlocks * sizeof(BlockStats) % 16 == 0, "cleared in 16-byte words");

// The real sum of |a||w| lies in [lower P, upper P] of the chain's result P (see linear_screen.hip).
constexpr int kScreenGroup = 32;              // reductions go by whole groups of 32 k
inline double accumulation_error(long K) { return (2.01 * (double)((K + kScreenGroup - 1) / kScreenGroup * kScreenGroup) / 8.0 + 8.0) * 0x1p-24; }
struct ScreenLimits { double lower, upper; };
inline ScreenLimits screen_limits(long K) {
    const double acc = accumulation_error(K), half = 0x1p-8;
    return {(1.0 - half) * (1.0 - half) / std::exp(acc), (1.0 + half) * (1.0 + half) / (1.0 - acc)};
}
// Whether the screen can decide for these constants (u: the model's, cg: Gamma with its guard factor): a bound inflated by its own 11.4u
// well within 2^-14, factors that stay ordinary in binary32 (bounds of at least 2^-120, limits below 2^109), absolute terms below 2^-20 of them.
inline bool screen_usable(long K, double u, double cg, double alpha, double uflow) {
    const double a = alpha * cg;
    return K > 0 && u <= 0x1p-20 && accumulation_error(K) <= 0x1p-6 && cg >= 0x1p-40 && cg <= 0x1p10 && a >= 0x1p-40 && a <= 0x1p20 &&
           uflow <= cg * (double)K * 0x1p-100;
}
int launch_screen(const ScreenOperand& A, const ScreenOperand& W, const float* bias, long M, long N, long K, long batch,
                  double cg, const ScreenCheck& chk, const CheckWorkspace& ws, OpenTile* open, hipStream_t st);

}  // namespace tao
