// Screening of a checked matmul bound: one BF16 product decides the comparisons that six would (linear_screen.hip).
#pragma once
#include <cmath>
#include "tao_check.hpp"

namespace tao {

// An operand of the screening product.  Image: as tao_split_operand writes it (its blocks begin with their hi pieces).
// Rows: the binary32 matrix itself (16-byte aligned rows, whole groups of 32 k).
// Pixels: BF16 magnitudes [batch][H][W][C] of a convolution's input, whose patch matrix the operand is (C a multiple of 32).
struct ScreenPixels {
    int H, W, C, OW, R, S, sh, sw, ph, pw, dh, dw;
    int r0, s0;                // the tap that its product begins with: the middle one, which lies in the padding last
    unsigned ohow;
    int slabs;                 // C / 32
    unsigned zeros;            // offset in bytes of 64 bytes of zeros
};
// Marks that say whether all of an operand is ordinary, that is below 2^32: the workgroups that cut it leave a byte each at the end of its
// image, kOrdinary if all that they read was (the sum of any eight neighbours, that is), and places without a workgroup hold that too.  An operand
// passes for ordinary only where all bytes say so: an image's leading pieces, which a caller that passes a part of a batch as an image of its
// own has in this place, never do (their sign bits are 0).
constexpr int kMarks = 512;
constexpr unsigned char kOrdinary = 0xa5;

// Words of the screen's LDS before its stages, whose place the strips of sums take in turn (rows of `strip` words, `cols` of them sums):
// the bins up to infinity's, 2040 (NaN is counted apart), and seven words more;
constexpr int kHistWords = 2048;
// words that count errors of 0, one for each lane, so that these need no ballots (three scalar instructions and a comparison an element:
// 8 x 8192 x 2048 over 128 234 -> 231 us).  Tiles of 64 x 64 have none and count by ballots: in all of their forms but one the
// workgroups of a compute unit fill the LDS to its last 64 bytes (the form for few tiles has room; its workgroups check one tile or two);
__host__ __device__ constexpr int spare_words(int blocks) { return blocks > 1 ? 64 : 0; }
// and, in forms that try first slabs, a bit for each tile that these left open.
constexpr int kEarlyWords = 8;
__host__ __device__ constexpr int words_before_stages(int blocks, bool early) { return kHistWords + spare_words(blocks) + (early ? kEarlyWords : 0); }
// The word to which a lane adds one for an error of 0: one of these, or, where there are none, a word that nobody reads, of the padding of the
// first strip's rows.
constexpr int kZeroRows = 22;
__host__ __device__ __forceinline__ constexpr int zero_word(int lane, int blocks, bool early, int cols, int strip) {
    return spare_words(blocks) ? kHistWords + lane : words_before_stages(blocks, early) + (lane % kZeroRows) * strip + cols + lane / kZeroRows;
}

struct ScreenOperand {
    const void* data;
    long batch_bytes;          // 0: shared
    long ld;                   // rows: elements between rows; otherwise 0
    const ScreenPixels* pixels;
    const unsigned char* marks;    // (rows: none)
};
constexpr long kScreenMaxLd = 1L << 22;      // rows of claims and outputs, and of binary32 operands: 32-bit offsets within a tile

struct ScreenCheck { const float* claimed; const float* ref; long ldy, strideY; double alpha, eps_rel; };

// A screened check keeps few partial results (they are cleared before and added up after each call): the first kScreenSlots, to which
// the screen adds, and the exact route its violations.  The words of the counters that no check writes hold, one for each of them, in how
// many tiles the screen left comparisons open, and how many of these the exact route has finished.
constexpr int kScreenSlots = 64;              // (32 cost perturbed claims of 1111 x 3001 2 us, 128 honest ones 0.4)
constexpr int kDoneFlag = kMaxCheckBlocks - 1;
static_assert(kScreenSlots == kWave, "a lane for each");
// The comparisons that the screen left open, a record per tile of the exact route (128 x 128 outputs; tiles row by row, batch entries one
// after the other), in the room of the partial results that a screened check does not use.  A record's first word is its state -- bit 4 r + c:
// every comparison of block (r, c), 32 x 32; from bit 16 on: how many places were asked for --, the second the number of parts of the
// reduction that the exact route has finished, the others are places: 128 row + column, or kNoPlace.  All zero before the screen.  Outputs of
// more tiles than fit so (0.4 G outputs) have their records where a short reduction's stored bound would lie, or records of the state
// alone; those of more than these (6.4 G, over more than 1024 k) are not screened.
constexpr int kOpenTile = 128, kOpenWords = 16;
constexpr unsigned kNoPlace = ~0u;
struct OpenRecords {
    unsigned* first;
    int words;                 // of a record: kOpenWords or 1
    __host__ __device__ unsigned* of(size_t tile) const { return first + tile * (size_t)words; }
    __host__ __device__ int places() const { return words == kOpenWords ? kOpenWords - 2 : 0; }
};
constexpr size_t kOpenRoom = (size_t)(kMaxCheckBlocks - kScreenSlots) * kBins;           // words
inline size_t open_tiles_of(long M, long N, long batch) {
    return (size_t)((M + kOpenTile - 1) / kOpenTile) * (size_t)((N + kOpenTile - 1) / kOpenTile) * (size_t)batch;
}
// bound, bound_bytes: the stored bound's place (16-byte aligned) and size.  words 0: no room.
inline OpenRecords open_records(const CheckWorkspace& w, size_t tiles, void* bound, size_t bound_bytes) {
    unsigned* const spare = w.hist + (size_t)kScreenSlots * kBins;
    if (tiles * kOpenWords <= kOpenRoom) return {spare, kOpenWords};
    if (tiles * kOpenWords * 4 <= bound_bytes) return {static_cast<unsigned*>(bound), kOpenWords};
    return {spare, tiles <= kOpenRoom ? 1 : 0};
}
// What a launch before a check clears, in 16-byte words: of `slots` partial results the histograms and coarse counts, all counters, and
// the records of `tiles` tiles.
struct ClearJob { void* at[4]; long words[4]; };
inline ClearJob clear_job(const CheckWorkspace& w, int slots, const OpenRecords& open = {nullptr, 0}, size_t tiles = 0) {
    return {{w.hist, w.coarse, w.stats, open.first},
            {(long)slots * kBins / 4, (long)slots * kGroups / 4, (long)(kMaxCheckBlocks * sizeof(BlockStats) / 16), (long)((tiles * open.words + 3) / 4)}};
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
bool screen_reads_marks(long M, long N, long K, long batch, bool rows, bool pixels);       // whether launch_screen's choice does
bool screen_reads_marks(long K);                             // whether it can, of prepared images of K columns
int launch_screen(const ScreenOperand& A, const ScreenOperand& W, const float* bias, long M, long N, long K, long batch,
                  double cg, const ScreenCheck& chk, const CheckWorkspace& ws, const OpenRecords& open, hipStream_t st);

}  // namespace tao
