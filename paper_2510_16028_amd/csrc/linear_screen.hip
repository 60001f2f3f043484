// The screen of a checked matmul bound (Sec. 3.1 reductions, checked as Sec. 5.4 and profiled as Sec. 5.3 say).
//
// A check needs of a bound only the answer to  d <= alpha tau,  and most answers do not hang on tau's last bits:
// honest claims stay far below their bounds, and a violation is rarely within a per cent of it.  The screen forms the sum
//     P = sum_k hi(a_k) hi(w_k),    hi(v) = |v| rounded to the nearest BF16 value,
// with one chain of v_mfma_f32_32x32x16_bf16 where the bound itself takes six products and their binary64 folds
// (linear_split.hip), and encloses the real sum S = sum_k |a_k||w_k| from both sides:
//   rounding of the operands:  |v| in hi(v) [1 - 2^-8, 1 + 2^-8], so S in P [(1 - 2^-8)^2, (1 + 2^-8)^2];
//   accumulation: the instruction's two steps of 8 k each err by at most 2.01u of the sum so far and 7u of the step's own
//     (the model that tao_selftest_matrix_core_bf16 re-checks); upwards these compound, so with acc = (2.01 Kp / 8 + 8) u the chain
//     returns a value in P [1 - acc, exp(acc)];
//   the bound's own slack: tau lies in [1, 1 + 1e-6] of Gamma (S + |b|) and its absolute terms are below 2^-20 of it;
//     2^-14 covers these and the few binary32 roundings of the comparison.
// Hence  d <= alpha cg (P lower + |b|)  proves that the exact check finds no violation and  d > alpha cg (P upper + |b|)
// that it finds one.  The enclosure holds where every operand is below 2^32 in magnitude (nothing overflows, and what
// operands below 2^-126 lose in BF16's subnormal range, 2^-134 each, weighs at most K 2^-101) and the sum at least
// Kp 2^-80; an element with d = 0 never violates a bound that is not NaN, and one whose d is NaN violates every bound.  Other
// comparisons -- a claim between the two limits, a smaller sum -- are left open, and so are all of a tile with a larger or
// non-finite operand or a bias beyond 2^60: a record per tile of the exact route (OpenRecords) keeps their places, and that route,
// enqueued behind the screen, decides these and nothing else.  So every profile is the exact route's, bit for bit.
// Part of the products is enough for most claims: their terms are not negative, so the sum over any k is a lower limit of the sum over all, and
//     d <= alpha cg (P' lower + |b|),   P' over the first 64 or 128 k,
// proves that there is no violation, whatever the rest -- but for operands that are infinite or NaN, so this way is taken only where the
// operands' marks say that all of both is ordinary (linear_screen.hpp).  Honest claims lie a thousand times below their bounds and are decided
// so; a tile with a claim that is not takes all products afterwards.  What bounds it then is the traffic of claims and outputs, not
// of operands (us of the whole call on images, all products / first slabs: 2048 x 12288 over 4096 235 -> 47, 201 MB at 4.3 TB/s; 2048 x 4096 over 1024 39 -> 24;
// 512 x 768 over 3072 26 -> 13; the 3 x 3 convolution of 32 x 56 x 56 x 256 203 -> 87).  The cost where it decides nothing: 1 us of a workgroup's time
// with tiles of 64 x 64, 3 with 128 x 128 (claims at 0.5 to 1.1 times their bounds, with the cut of A: 300 x 300 over 448 17.5 -> 18.5, 512 x 3072 over 768
// 22.0 -> 23.5, 2048 x 4096 over 1024 47.5 -> 50.2, 2048 x 12288 over 4096 the same within the spread).  A far-off claim that is found as a tile's first
// ones ends the first slabs of its workgroup: a proposer who spoils a corner of an output takes the gain from the later tiles of some workgroups,
// and no call takes longer than that.
// The errors' bins and maximum do not depend on tau: quick settlement as in tao_check.hpp, exact arithmetic where
// an estimate does not decide.
// A workgroup forms no further products and leaves all comparisons open once all of its wavefronts have found much open in a tile, or some
// in two tiles running: where that route forms most bounds anyway they are work for nothing (us of the whole call, every claim at its
// bound, with all products / so: 2048 x 12288 over 4096 1577 / 1425, the 3 x 3 convolution of 32 x 56 x 56 x 256 1378 / 1214, 8 x 8192 x 128
// over 2048 428 / 364; 8192 x 8192 over 8192, heavy-tailed operands and two thirds of the claims 1 % from their bounds, 7690 / 6990).
#include <cmath>
#include <type_traits>
#include "tao_device.hpp"
#include "tao_host.hpp"
#include "linear_screen.hpp"

namespace tao {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));     // 16-byte loads at 4-byte alignment
typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));

constexpr int SBK = kScreenGroup;
constexpr int kImageBlock = 3 * 128 * 64;               // bytes of an image's block of 128 rows x 32 k, three pieces
constexpr unsigned kLargeBf16 = (127u + 32u) << 7;      // 2^32: operands from here on are not screened
constexpr float kTinyPerStep = 0x1p-80f;
constexpr int kEarlyTiles = 32 * kEarlyWords;            // tiles of a workgroup that may be tried by their first slabs (2.1 G outputs)

__device__ __forceinline__ unsigned pack_abs_bf16(float even, float odd) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{fabsf(even), fabsf(odd)}), bf16x2));
}

// (what the compiler cannot see to be the same in all lanes, such as a word of LDS)
__device__ __forceinline__ unsigned same_in_all(unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); }

// ---- the product and its check ------------------------------------------------------------------
struct ScreenArgs {
    const char* A; const char* W;
    long stepA, stepW;                 // bytes between k groups (rows: 128; pixels: unused)
    long batchA, batchW;               // bytes between batch entries
    int last_blkA, last_blkW;          // image: the last block of an operand (tiles beyond it read that one)
    const unsigned* marksA; const unsigned* marksW;       // the operands' marks (pixels: both the filters'; rows: none)
    long ldA;                          // rows: bytes between rows
    ScreenPixels px;                   // pixels: the convolution
    long M, N;
    int groups;
    unsigned tiles_m, tiles_n, ntiles;
    const float* claimed; const float* ref; const float* bias;
    long ldy, strideY;
    int stream;                        // claims and outputs are more than the memory-side cache holds: streaming loads
    double eps_rel;
    float low, high, low_b, high_b, tiny;
    OpenRecords open; unsigned open_m, open_n;              // and how many tiles they are down and across
    unsigned int* hist; unsigned int* coarse; BlockStats* stats;
};

enum { IMAGE, ROWS, PIXELS };

// Waits until at most min(behind, MOST) slabs of COPIES copies each are outstanding.
template <int COPIES, int MOST>
__device__ __forceinline__ void wait_for_copies(int behind) {
    constexpr int n = COPIES * MOST;
    if constexpr (MOST == 0) {
        __builtin_amdgcn_s_waitcnt(0x0F70);
    } else {
        if (behind >= MOST) __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | (n >> 4 << 14));
        else wait_for_copies<COPIES, MOST - 1>(behind);
    }
}

// WVM x WVN wavefronts of RM x RN accumulator tiles of 32 x 32.  A stage holds a group of 32 k of the tile's operands as the images
// hold them (ROWS: of A the binary32 values, cut when a fragment is read; PIXELS: gathered from BF16 magnitudes of the input,
// taps in the padding from a line of zeros), GPS times; NST stages filled by 16-byte copies that go to LDS directly, requested
// NST - 1 stages ahead, one barrier per stage.  The matrix instruction takes W as its row operand, so a lane holds four consecutive columns
// of one row; the sums pass through LDS (32 rows of a wavefront at a time) so that claims and outputs are read along their
// rows.  Workgroups walk the tiles; each XCD (workgroups are dealt to them in turn) owns a contiguous eighth of them, eight
// tile rows deep, for its L2.
//
// UNDERFLOW: an estimated error may come down to 0 though claim and output differ (denominators of 2 and more next to the smallest
// subnormals), so an error of 0 is told by the difference; otherwise by the estimate, which then is 0 only if the difference is: with
// eps_rel <= 1 the denominator is at most 1 + 2^-20 where |output| is below 2^-20, and elsewhere a difference is at least 2^-25 of |output|.
// The test of the difference takes 1 to 2 % (33000 x 128 over 1056 with its cut 52.1 -> 53.1 us, 2048 x 12288 over 4096 228.5 -> 231.5), so forms
// that could go without it have an instantiation for either.
//
// EARLY: a workgroup walks its tiles with one slab of products each, requested while the tile before is checked (early_walk), up to one whose first
// claims exceed what the sums prove in numbers; from there on with all products; and then those of the first walk that
// are not decided once more, with all products and without the errors, which are settled.  Workgroups of 64 x 64 tiles, which have one each, or two, try
// the first one, unless its claims are far off by the size of the outputs.
//
// Forms that do so: 128 x 128, and few 64 x 64 tiles.  Not: 64 x 128 tiles of up to 256 k, whose time is the check's (8 x 8192 x 2048 over 128 231 -> 240 us, 22 spilled
// registers), 64 x 64 with four workgroups to a compute unit (128 registers: 19 spilled; 1111 x 3001 over 1001 40.7 -> 50.7), and rows, which are
// read whole in any case.
// Bytes behind the histogram: the stages, or the strips of sums with the slab that is requested under them.
constexpr int stage_bytes(int RM, int RN, int WVM, int WVN, int GPS, int NST, int SRC, bool EARLY) {
    const int group = WVM * RM * 32 * (SRC == ROWS ? 128 : 64) + WVN * RN * 32 * 64;
    const int early = EARLY && RM * RN > 1 ? WVM * WVN * RN * 4096 + GPS * group : 0;
    return early > NST * GPS * group ? early : NST * GPS * group;
}
template <int RM, int RN, int WVM, int WVN, int GPS, int NST, int PER_CU, int SRC, bool EARLY, bool UNDERFLOW>
__global__ __launch_bounds__(WVM * WVN * 64, WVM * WVN * PER_CU / 4) void screen_product(ScreenArgs p) {
    constexpr int WAVES = WVM * WVN, THREADS = WAVES * 64;
    constexpr int TM = WVM * RM * 32, TN = WVN * RN * 32;
    constexpr int ROWB = SRC == ROWS ? 128 : 64;                               // bytes of a row of A's slab
    constexpr int SLAB_A = TM * ROWB, SLAB_W = TN * 64, GROUP = SLAB_A + SLAB_W, STAGE = GPS * GROUP;
    constexpr int NA = SLAB_A / 1024 / WAVES, NW = SLAB_W / 1024 / WAVES;      // copies of a wavefront per group
    static_assert(NA * WAVES * 1024 == SLAB_A && NW * WAVES * 1024 == SLAB_W, "whole copies");
    constexpr bool ACROSS = RM * RN > 1, SPARE = spare_words(RM * RN) > 0, BY_ESTIMATE = SPARE && !UNDERFLOW;
    // a wavefront's strip of sums: 32 x COLS, rows padded, or (no padding: the LDS holds one workgroup more) their 16-byte units at u ^ (row & 15)
    constexpr int COLS = RN * 32, STRIP = COLS + (SPARE ? 0 : 4);
    static_assert(!SPARE || COLS == 64, "sixteen units to a row");
    static_assert(WAVES * 32 * STRIP * 4 <= stage_bytes(RM, RN, WVM, WVN, GPS, NST, SRC, EARLY), "the strips lie in the stages");
    constexpr int CHAINS = RM * RN == 1 ? 2 : 1;                               // (a single accumulator would be one serial chain)
    // Both halves of a group are read before its two products where the registers allow it: the wait for the second then passes under the
    // first product (64 x 200 over 8192 52.0 -> 46.0 us, 512 x 768 over 3072 28.4 -> 26.6).
    constexpr bool AHEAD = RM * RN == 1 && PER_CU == 2 && SRC == IMAGE;
    static_assert(!EARLY || THREADS == kMarks / 2, "a thread for four marks");
    static_assert(!EARLY || ACROSS || (NST == 2 && WAVES * 32 * STRIP * 4 <= STAGE), "a second slab beside the strips");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    unsigned int* const hist = reinterpret_cast<unsigned int*>(lds);
    constexpr int WORDS = words_before_stages(RM * RN, EARLY);
    unsigned int* const pending = hist + kHistWords + spare_words(RM * RN);      // tiles of which a first slab did not decide all, a bit each
    char* const stages = lds + WORDS * 4;
    char* const slab0 = stages + (ACROSS ? WAVES * 32 * STRIP * 4 : 0);        // a first slab's place (ACROSS: behind the strips)
    unsigned int& largest = hist[2041];                      // a lower bound of an error that occurs (its bits)
    // 1 + the last tile with an operand that is not screened (volatile, by measurement: the form for rows takes 49 us for 2007 x 128 over 5632 with it and
    // 53 without)
    volatile unsigned int& large_in = hist[2042];
    unsigned int& heavy = hist[2043];                        // wavefronts that had to leave whole blocks open
    unsigned int& refused = hist[2044];                      // 1 + the last tile of which the first slab would not decide much
    unsigned int& unordinary = hist[2045];                   // an operand may not be ordinary, or the first claims are far off
    unsigned int& some_pending = hist[2046];                 // whether any of `pending` is set
    auto now = [](unsigned int& word) __attribute__((always_inline)) { return same_in_all(newest(&word)); };        // (behind a barrier)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WVN, wn = wave % WVN;
    const int r32 = lane & 31, h = lane >> 5;
    for (int i = tid; i < WORDS / 4; i += THREADS) reinterpret_cast<uintx4*>(hist)[i] = uintx4{0, 0, 0, 0};
    unsigned marks = kOrdinary * 0x01010101u;
    if (EARLY) marks = (tid < kMarks / 4 ? p.marksA : p.marksW)[tid % (kMarks / 4)];        // (all lanes: behind a branch it would be waited for here)

    // fragments: lane (r32, h) holds k = 16 kg + 8 h .. + 7 of its row.  The first k half a wavefront takes is (wm ^ wn) & 1, so that
    // the first halves of all wavefronts cover every operand value of the tile: only those are looked at for large ones.
    const int swz = (r32 >> 2) & 3, swr = (r32 >> 1) & 7, flip = (wm ^ wn) & 1;
    int unitW[2], unitA[2][2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int kg = s ^ flip;
        unitW[s] = ((2 * kg + h) ^ swz) * 16;
        unitA[s][0] = SRC == ROWS ? ((4 * kg + 2 * h) ^ swr) * 16 : unitW[s];
        unitA[s][1] = SRC == ROWS ? ((4 * kg + 2 * h + 1) ^ swr) * 16 : 0;
    }
    const int fragA = (wm * RM * 32 + r32) * ROWB;
    const int fragW = SLAB_A + (wn * RN * 32 + r32) * 64;

    const QuickCheck qc(1.f, p.eps_rel);
    unsigned nans = 0, vio = 0, max_bits = 0, known = 0;
    int zeros = 0;                                           // elements with d = 0 (a lane's own, to be added to all_zeros)
    int all_zeros = 0;                                       // (the same in all lanes)
    float* strip = reinterpret_cast<float*>(stages) + wave * 32 * STRIP;
    // what stands for the bits of an error of 0, which is counted elsewhere: the middle of a "bin" that is a word of no bin (zero_word)
    static_assert(SPARE || (COLS + (kWave - 1) / kZeroRows < STRIP && kZeroRows <= 32), "in the padding of the first strip's rows");
    static_assert(WORDS + kZeroRows * STRIP < 4096, "twelve bits of bin");
    const unsigned zero_bits = (unsigned)zero_word(lane, RM * RN, EARLY, COLS, STRIP) << 20 | 0x80000u;
    // elements of a strip: a lane has four consecutive columns of one row per step
    constexpr int LPR = COLS / 4, RPI = 64 / LPR, STEPS = 32 / RPI;           // lanes per row, rows per step
    const int lrow = lane / LPR, lcol = (lane % LPR) * 4;
    const int srow = wm * RM * 32, scol = wn * COLS;

    const unsigned xcd = blockIdx.x & 7u, per = gridDim.x >> 3;
    const unsigned t_end = (unsigned)((unsigned long long)p.ntiles * (xcd + 1) >> 3);
    const unsigned per_z = p.tiles_m * p.tiles_n;
    unsigned opened = 0;                                     // records that this wavefront was the first to write to
    unsigned heavy_before = 0, by_before = 0;                // (as of the last tile, and by how many wavefronts in that one)
    int groups = p.groups;                                   // 0: the products are not formed any more
    // A tile: its place, and where its claims and outputs begin.
    struct Tile { unsigned z; long m0, n0; int rows_left, cols_left; const float* C; const float* Y; };
    auto tile_of = [&](unsigned t) __attribute__((always_inline)) {
        const unsigned z = t / per_z, b = t - z * per_z;
        const unsigned grp = b / (8 * p.tiles_n), in = b - grp * 8 * p.tiles_n;
        const unsigned deep = min(8u, p.tiles_m - grp * 8);
        const unsigned tx = in / deep, ty = grp * 8 + (in - tx * deep);
        const long m0 = (long)ty * TM, n0 = (long)tx * TN, at = (long)z * p.strideY + m0 * p.ldy + n0;
        return Tile{z, m0, n0, (int)min((long)TM, p.M - m0), (int)min((long)TN, p.N - n0), p.claimed + at, p.ref + at};
    };
    // claims and outputs of a strip; positions beyond the edge read the edge's elements
    const int ldy = (int)p.ldy;
    floatv4 cv[STEPS], rv[STEPS];
    auto fetch = [&](const Tile& T, int i, int k) __attribute__((always_inline)) {
        const int row = min(srow + i * 32 + lrow + k * RPI, T.rows_left - 1) * ldy, col = scol + lcol;
        if (col + 4 <= T.cols_left) {
            const floatx4u* cp = reinterpret_cast<const floatx4u*>(T.C + (unsigned)(row + col));        // (at any alignment)
            const floatx4u* rp = reinterpret_cast<const floatx4u*>(T.Y + (unsigned)(row + col));
            if (p.stream) { cv[k] = __builtin_nontemporal_load(cp); rv[k] = __builtin_nontemporal_load(rp); }
            else          { cv[k] = *cp; rv[k] = *rp; }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                unsigned at = (unsigned)(row + min(col + e, T.cols_left - 1));
                asm volatile("" : "+v"(at));                 // (the last two are the same: copied they were waited for, 1536 x 5119 over 512 28.0 -> 24.3 us)
                cv[k][e] = T.C[at]; rv[k][e] = T.Y[at];
            }
        }
    };
    // Sources of this wavefront's copies, scalar bases and 32-bit lane offsets, and how far they have come.
    struct Sources {
        const char* A[NA]; const char* W[NW];
        unsigned offA[NA];
        int pix_h[SRC == PIXELS ? NA : 1], pix_w[SRC == PIXELS ? NA : 1];     // PIXELS: input coordinates of tap (0, 0)
        int tap_c, tap_s, tap_r;
        int left;                                            // groups not requested yet
    };
    const unsigned off = lane * 16;
    auto sources_of = [&](const Tile& T, Sources& s) __attribute__((always_inline)) {
        s.tap_c = 0; s.tap_s = p.px.s0; s.tap_r = p.px.r0;   // (PIXELS: from the middle tap on; the first follows the last)
        s.left = p.groups;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int chunk = wave + i * WAVES;
            if (SRC == ROWS) {
                const int r = chunk * 8 + (lane >> 3);
                s.offA[i] = (unsigned)(min(r, T.rows_left - 1) * p.ldA) + ((unsigned)((lane & 7) ^ ((r >> 1) & 7))) * 16u;
                s.A[i] = p.A + T.z * p.batchA + T.m0 * p.ldA;
            } else if (SRC == PIXELS) {
                const int r = chunk * 16 + (lane >> 2);
                const unsigned m = (unsigned)T.m0 + (unsigned)min(r, T.rows_left - 1);
                const unsigned img = m / p.px.ohow, rem = m - img * p.px.ohow;
                const unsigned oh = rem / (unsigned)p.px.OW, ow = rem - oh * (unsigned)p.px.OW;
                s.pix_h[i] = (int)oh * p.px.sh - p.px.ph; s.pix_w[i] = (int)ow * p.px.sw - p.px.pw;
                // (modulo 2^32: a tap inside the input has an offset below 2^31)
                s.offA[i] = (unsigned)((((int)img * p.px.H + s.pix_h[i]) * p.px.W + s.pix_w[i])) * (unsigned)p.px.C * 2u +
                            (unsigned)((lane & 3) ^ ((r >> 2) & 3)) * 16u;
                s.A[i] = p.A;
            } else {
                const int row = (int)T.m0 + chunk * 16, blk = min(row >> 7, p.last_blkA);
                s.A[i] = p.A + T.z * p.batchA + (long)blk * kImageBlock + (row & 127) * 64;
                s.offA[i] = off;
            }
        }
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int row = (int)T.n0 + (wave + i * WAVES) * 16, blk = min(row >> 7, p.last_blkW);
            s.W[i] = p.W + T.z * p.batchW + (long)blk * kImageBlock + (row & 127) * 64;
            if (SRC == PIXELS) s.W[i] += (long)((p.px.r0 * p.px.S + p.px.s0) * p.px.slabs) * p.stepW;
        }
    };
    auto next_tap = [&](Sources& s) __attribute__((always_inline)) {
        if (++s.tap_c < p.px.slabs) return;
        s.tap_c = 0;
        if (++s.tap_s < p.px.S) return;
        s.tap_s = 0;
        if (++s.tap_r < p.px.R) return;
        s.tap_r = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) s.W[i] -= (long)p.groups * p.stepW;
    };
    // one stage's copies (a stage's groups beyond the last repeat it: their number is then the same for all)
    auto request = [&](Sources& s, const char* stage) __attribute__((always_inline)) {
#pragma unroll
        for (int sub = 0; sub < GPS; ++sub) {
            const unsigned dst = (unsigned)(size_t)(__attribute__((address_space(3))) char*)const_cast<char*>(stage) +
                                 (unsigned)(sub * GROUP) + (unsigned)wave * 1024u;
            const int dr = s.tap_r * p.px.dh, ds = s.tap_s * p.px.dw;
            const unsigned tap = (unsigned)((dr * p.px.W + ds) * p.px.C + s.tap_c * SBK) * 2u;
            const bool on = --s.left > 0;
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                unsigned o = s.offA[i];
                if (SRC == PIXELS) {
                    const bool inside = (unsigned)(s.pix_h[i] + dr) < (unsigned)p.px.H && (unsigned)(s.pix_w[i] + ds) < (unsigned)p.px.W;
                    o = inside ? o + tap : p.px.zeros;
                }
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                             :: "s"(dst + (unsigned)(i * WAVES * 1024)), "v"(o), "s"(s.A[i]) : "memory");
                if (SRC != PIXELS) s.A[i] += GPS == 1 || on ? p.stepA : 0;
            }
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                             :: "s"(dst + (unsigned)(SLAB_A + i * WAVES * 1024)), "v"(off), "s"(s.W[i]) : "memory");
                s.W[i] += GPS == 1 || on ? p.stepW : 0;
            }
            if (SRC == PIXELS && (GPS == 1 || on)) next_tap(s);
        }
    };
    // The sums, and the largest operands that went into them (packed, of a fragment's even and odd values).
    struct Sums { floatx16 acc[RM][RN], more; ushortx2 mostA[RM], mostW[RN]; };
    auto clear_sums = [&](Sums& s) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s.more[v] = 0.f;
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < RN; ++j) s.acc[i][j][v] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < RM; ++i) s.mostA[i] = ushortx2{0, 0};
#pragma unroll
        for (int j = 0; j < RN; ++j) s.mostW[j] = ushortx2{0, 0};
    };
    auto most = [&](ushortx2& m, const bf16x8& f) __attribute__((always_inline)) {
        const uintx4 u = __builtin_bit_cast(uintx4, f);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned two = u[j];                       // (a bit cast of the element itself takes the vector's first)
            m = __builtin_elementwise_max(m, __builtin_bit_cast(ushortx2, two));
        }
    };
    auto compute = [&](Sums& sums, const char* stage) __attribute__((always_inline)) {
        bf16x8 second_a, second_w;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            bf16x8 a[RM], w[RN];
#pragma unroll
            for (int i = 0; i < RM; ++i) {
                if (SRC == ROWS) {
                    const float4 x = *reinterpret_cast<const float4*>(stage + fragA + i * 32 * 128 + unitA[s][0]);
                    const float4 y = *reinterpret_cast<const float4*>(stage + fragA + i * 32 * 128 + unitA[s][1]);
                    a[i] = __builtin_bit_cast(bf16x8, (uintx4{pack_abs_bf16(x.x, x.y), pack_abs_bf16(x.z, x.w),
                                                              pack_abs_bf16(y.x, y.y), pack_abs_bf16(y.z, y.w)}));
                } else {
                    a[i] = *reinterpret_cast<const bf16x8*>(stage + fragA + i * 32 * 64 + unitA[s][0]);
                }
            }
#pragma unroll
            for (int j = 0; j < RN; ++j) w[j] = *reinterpret_cast<const bf16x8*>(stage + fragW + j * 32 * 64 + unitW[s]);
            if (AHEAD && s == 0) {
                second_a = *reinterpret_cast<const bf16x8*>(stage + fragA + unitA[1][0]);
                second_w = *reinterpret_cast<const bf16x8*>(stage + fragW + unitW[1]);
                __builtin_amdgcn_sched_barrier(0);           // (the compiler would wait for one half before it reads the other)
            }
            if (AHEAD && s == 1) { a[0] = second_a; w[0] = second_w; }
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < RN; ++j) {
                    floatx16& sum = CHAINS == 2 && s == 1 ? sums.more : sums.acc[i][j];
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[j], a[i], sum, 0, 0, 0);
                }
            if (s == 0) {
#pragma unroll
                for (int i = 0; i < RM; ++i) most(sums.mostA[i], a[i]);
#pragma unroll
                for (int j = 0; j < RN; ++j) most(sums.mostW[j], w[j]);
            }
        }
    };
    // Behind the products: their sum, whether there were operands that are not screened, of rows that exist, and the bias's share of the limits.
    floatv4 bl, bh;
    float bias_low;
    auto finish_sums = [&](const Tile& T, Sums& s) __attribute__((always_inline)) -> bool {
        if (CHAINS == 2) {
#pragma unroll
            for (int v = 0; v < 16; ++v) s.acc[0][0][v] += s.more[v];
        }
        bool large = false;
#pragma unroll
        for (int i = 0; i < RM; ++i)
            large |= srow + i * 32 + r32 < T.rows_left && (s.mostA[i][0] >= kLargeBf16 || s.mostA[i][1] >= kLargeBf16);
#pragma unroll
        for (int j = 0; j < RN; ++j)
            large |= scol + j * 32 + r32 < T.cols_left && (s.mostW[j][0] >= kLargeBf16 || s.mostW[j][1] >= kLargeBf16);
        bias_low = INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int col = scol + lcol + e;
            const float b = p.bias && col < T.cols_left ? fabsf(p.bias[T.n0 + col]) : 0.f;
            large |= !(b <= 0x1p60f);
            bl[e] = b * p.low_b; bh[e] = b * p.high_b;
            bias_low = fminf(bias_low, bl[e]);
        }
        return large;
    };
    // An error that occurs, to begin with (without one no element could be settled for the maximum): the largest of a lane's first
    // elements, lowered by what the estimate may be off.  All lanes take part, also those that have met an error on the exact way: the
    // reduction asks for all of them, and lane 0 puts the result down.
    auto first_error = [&]() __attribute__((always_inline)) {
        if (!__any(known == 0)) return;
        unsigned first = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float den = fabsf(rv[0][e]) + qc.eps;
            const unsigned bits = __float_as_uint(fabsf(cv[0][e] - rv[0][e]) * __builtin_amdgcn_rcpf(den));
            if (den <= 0x1p100f && bits <= 0x7f800000u && bits > 16u) first = max(first, bits - 16u);
        }
        // (rows and columns beyond the edge repeat elements that exist)
        // (one atomic of a wavefront: 256 lanes' on the one word took 2.3 us; 512 x 3072 over 768 24.05 -> 22.7 us with the histogram in lines below)
        first = wave_max(first);
        if (first && lane == 0) atomicMax(&largest, first);
    };
    auto put_strip = [&](const Sums& s, int i) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < RN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int unit = j * 8 + 2 * q + h;
                *reinterpret_cast<floatv4*>(strip + r32 * STRIP + (SPARE ? unit ^ (r32 & 15) : unit) * 4) =
                    floatv4{s.acc[i][j][4 * q], s.acc[i][j][4 * q + 1], s.acc[i][j][4 * q + 2], s.acc[i][j][4 * q + 3]};
            }
    };
    auto strip_sums = [&](int k) __attribute__((always_inline)) {
        const int row = lrow + k * RPI;
        return *reinterpret_cast<const floatv4*>(strip + row * STRIP + (SPARE ? (lcol / 4) ^ (row & 15) : lcol / 4) * 4);
    };

    using Places = typename std::conditional<(RM * STEPS * 4 > 32), unsigned long long, unsigned>::type;
    // Four elements of a lane: violations, and bins and maximum where the estimates decide (false: exact4).  Tests are made for the
    // four together first: a test per element costs as much as the estimate.  high: infinite where the sums are of some products only.
    auto check4 = [&](const floatv4& c, const floatv4& r, const floatv4& s, float high, Places& open, int step) __attribute__((always_inline)) -> bool {
        unsigned word[4], bits[4], edge[4], least[4];
        float over[4], den[4];
        int found = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float d = fabsf(c[e] - r[e]);
            den[e] = fabsf(r[e]) + qc.eps;
            bits[e] = __float_as_uint(d * __builtin_amdgcn_rcpf(den[e]));
            over[e] = fmaf(s[e], -p.low, d);
            if (BY_ESTIMATE) {
                const unsigned b = min(bits[e] - 1u, zero_bits);         // (one below: another bin only within 16 steps of an edge)
                edge[e] = (b + 17u) << 12;                   // (below 32 << 12 within 16 steps of a bin's edge)
                word[e] = b >> 20;
            } else {
                const bool zero = d == 0.f;                  // (an estimate of 0 where it is not: at an edge, and so left open)
                const unsigned b = zero ? zero_bits : bits[e];
                edge[e] = (b + 16u) << 12;
                word[e] = b >> 20;
                if (!SPARE) found += __popcll(__ballot(zero));
            }
            least[e] = __float_as_uint(s[e]);                // (sums are not negative)
        }
        if (!SPARE) {
            asm volatile("" : "+s"(found));                  // (counted here: masks kept until later exceed the scalar registers)
            all_zeros += found;
        }
        int inside = fmaxf(fmaxf(over[0], over[1]), fmaxf(over[2], over[3])) <= bias_low;
        inside &= min(min(least[0], least[1]), min(least[2], least[3])) >= __float_as_uint(p.tiny);
        const unsigned most_bits = max(max(bits[0], bits[1]), max(bits[2], bits[3]));      // (a NaN's are the largest)
        // (no larger than an error that occurs; or all 0, and then exactly: none comes down to 0, or the edges leave it open)
        int ok = most_bits <= max(known, 16u) - 16u;
        ok &= min(min(edge[0], edge[1]), min(edge[2], edge[3])) >= 32u << 12;
        ok &= fmaxf(fmaxf(den[0], den[1]), fmaxf(den[2], den[3])) <= 0x1p100f;
        if (!inside || most_bits > 0x7f800000u) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float d = fabsf(c[e] - r[e]);
                const bool sure = s[e] >= p.tiny, above = (d != d) | ((d > fmaf(s[e], high, bh[e])) & sure);
                vio += above;
                open |= (Places)!(above | (d == 0.f) | ((d <= fmaf(s[e], p.low, bl[e])) & sure)) << (4 * step + e);
            }
        }
        if (ok) {
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicAdd(&hist[word[e]], 1u);
        }
        return ok;
    };
    // The exact way for bins and maximum of step k of strip i, its elements read again.
    auto exact4 = [&](const Tile& T, int i, int k) __attribute__((always_inline)) {
        const int row = srow + i * 32 + lrow + k * RPI, col = scol + lcol;
        float c[4], r[4];
        bool in_range[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            in_range[e] = row < T.rows_left && col + e < T.cols_left;
            const unsigned at = in_range[e] ? (unsigned)(row * ldy + col + e) : 0u;
            c[e] = T.C[at]; r[e] = T.Y[at];
        }
        CheckedElement o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = check_arith<false>(c[e], r[e], 0.f, 1.0, p.eps_rel);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (!in_range[e]) { zeros += SPARE; continue; }                      // (not counted in check4, where elements with SPARE are if settled)
            if (!SPARE && c[e] == r[e] && fabsf(c[e]) < INFINITY) zeros -= 1;    // (counted in check4)
            nans += o[e].is_nan;
            if (!o[e].is_nan) { max_bits = max(max_bits, o[e].bits); atomicAdd(&hist[o[e].bin], 1u); }
        }
        if (max_bits > known) atomicMax(&largest, max_bits);
        known = max(known, newest(&largest));
    };
    // A tile's elements against its sums; what follows(i, k) is requested as registers become free.
    auto check_tile = [&](const Tile& T, const Sums& sums, float high, Places& open, auto&& before, auto&& follows) __attribute__((always_inline)) {
        unsigned again = 0;                                  // steps for exact4
#pragma unroll
        for (int i = 0; i < RM; ++i) {
            before(i);
            put_strip(sums, i);
            const int in_rows = max(0, min(32, T.rows_left - srow - i * 32)), in_cols = max(0, min(COLS, T.cols_left - scol));
            const bool whole = in_rows == 32 && in_cols == COLS;
            all_zeros -= 32 * COLS - in_rows * in_cols;      // (positions beyond the edge pass for zeros below)
#pragma unroll
            for (int k = 0; k < STEPS; ++k) {
                __builtin_amdgcn_sched_barrier(0);           // (side by side the steps' lane masks exceed the scalar registers)
                floatv4 s = strip_sums(k);
                if (!whole) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool out = lrow + k * RPI >= in_rows || lcol + e >= in_cols;
                        cv[k][e] = out ? 0.f : cv[k][e]; rv[k][e] = out ? 0.f : rv[k][e];
                        s[e] = out ? p.tiny : s[e];
                    }
                }
                if (!check4(cv[k], rv[k], s, high, open, i * STEPS + k)) again |= 1u << (i * STEPS + k);
                follows(i, k);
            }
        }
        while (again) {
            const int at = __ffs((int)again) - 1;
            again &= again - 1;
            exact4(T, at / STEPS, at % STEPS);
        }
    };

    // The first requests of a tile.  (The first step's claims go ahead: what waits for these does not wait for all of the chip's first tiles.)
    // Where a workgroup tries one tile only, the second slab is requested as well, for claims that turn out to be far off: what has been learnt of the
    // tile is then kept (300 x 300 over 448, the screen alone, 12.3 -> 11.5 us).  Where they do not its copies land beside the strips, unread.
    auto begin = [&](const Tile& T, Sources& src) __attribute__((always_inline)) {
        fetch(T, 0, 0);
        asm volatile("" ::: "memory");
        sources_of(T, src);
        request(src, slab0);
        if (!ACROSS) request(src, stages + STAGE);
#pragma unroll
        for (int k = 1; k < STEPS; ++k) fetch(T, 0, k);
    };

    // Whether, of a wavefront's first claims, `part` eighths of those that exist or more are further from their outputs than limit(e).
    auto far_off = [&](const Tile& T, int part, auto&& limit) __attribute__((always_inline)) -> bool {
        const int there = max(0, min(RPI, T.rows_left - srow)) * max(0, min(COLS, T.cols_left - scol));
        int n = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            n += __popcll(__ballot(srow + lrow < T.rows_left && scol + lcol + e < T.cols_left && fabsf(cv[0][e] - rv[0][e]) > limit(e)));
        return there && n * 8 >= there * part;
    };

    // ---- first slabs by themselves.  Tiles base, base + per, ...: how many of the next `n` went this way.
    auto early_walk = [&](unsigned base, unsigned n, Tile tile) __attribute__((always_inline)) -> unsigned {
        if (ACROSS) {
            Sources src;
            begin(tile, src);
        }
        for (unsigned at = 0;; ++at) {
            const unsigned t = base + at * per;
            // the copies are older than the claims and outputs behind the first step's (two loads a step at least), which stay on their way
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * (STEPS - 1)) : "memory");
            if (ACROSS && marks != kOrdinary * 0x01010101u) unordinary = 1;
            __syncthreads();
            Sums sums;
            clear_sums(sums);
#pragma unroll
            for (int sub = 0; sub < GPS; ++sub) compute(sums, slab0 + sub * GROUP);
            const bool large = finish_sums(tile, sums);
            first_error();
            // Whether many of these claims would be left pending, by the largest of the wavefront's first block of sums, of those that exist.
            // (Where an operand has no rows they are of whatever its image held before.)
            float most_sum = sums.acc[0][0][0];
            if (tile.rows_left >= TM && tile.cols_left >= TN) {
#pragma unroll
                for (int v = 1; v < 16; ++v) most_sum = fmaxf(most_sum, sums.acc[0][0][v]);
            } else {
                const int cols_there = srow + r32 < tile.rows_left ? tile.cols_left - scol - 4 * h : 0;
                most_sum = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) most_sum = fmaxf(most_sum, v / 4 * 8 + v % 4 < cols_there ? sums.acc[0][0][v] : 0.f);
            }
            most_sum = wave_max(most_sum);
            if (large || far_off(tile, 2, [&](int e) { return fmaf(most_sum, p.low, bl[e]); })) refused = t + 1;
            __syncthreads();                                 // every wavefront is done with the slab
            if (now(unordinary) != 0 || now(refused) == t + 1) return at;
            known = max(known, newest(&largest));
            const bool last = !ACROSS || at + 1 == n;
            const Tile next = ACROSS ? tile_of(last ? t : t + per) : tile;
            Places open = 0;
            check_tile(tile, sums, INFINITY, open,
                       [&](int i) __attribute__((always_inline)) {
                           if (ACROSS && i == RM - 1 && !last) {
                               Sources src;
                               sources_of(next, src);
                               request(src, slab0);
                           }
                       },
                       [&](int i, int k) __attribute__((always_inline)) {
                           if (i + 1 < RM) fetch(tile, i + 1, k);
                           else if (ACROSS && !last) fetch(next, 0, k);
                       });
            if (__any(open != 0) && lane == 0) { atomicOr(&pending[at / 32], 1u << (at & 31)); some_pending = 1; }
            if (last) return n;
            tile = next;
        }
    };

    // All products of a tile (begun: its first two slabs are under way).
    auto product = [&](Sources& src, Sums& sums, bool begun) __attribute__((always_inline)) {
        constexpr int COPIES = GPS * (NA + NW);
        const int slabs = (groups + GPS - 1) / GPS;
#pragma unroll
        for (int i = 0; i + 1 < NST; ++i)
            if (i < slabs && !(begun && i == 0)) request(src, stages + i * STAGE);
        int cur = 0;
#pragma unroll 1
        for (int g = 0; g < slabs; ++g) {
            // slab g has landed when only the copies of the slabs behind it are outstanding; the barrier publishes it and
            // separates the last reads of the stage before from its next fill
            wait_for_copies<COPIES, NST - 2>(slabs - 1 - g);
            __syncthreads();
            if (g + NST - 1 < slabs && !(begun && g == 0)) request(src, stages + (cur == 0 ? NST - 1 : cur - 1) * STAGE);
            compute(sums, stages + cur * STAGE);
#pragma unroll
            for (int sub = 1; sub < GPS; ++sub)
                if (g * GPS + sub < groups) compute(sums, stages + cur * STAGE + sub * GROUP);
            cur = cur == NST - 1 ? 0 : cur + 1;
        }
    };
    // A tile's start.  (All wavefronts have to read the same of `heavy` behind this barrier -- otherwise they would not meet at the same ones --,
    // and nothing else makes the compiler wait for an addition to it whose result is not used before it signals the barrier.)
    auto meet = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();                                     // the strips of the tile before have been read
        const unsigned heavy_now = now(heavy), by = heavy_now - heavy_before;
        if (by == WAVES || (by && by_before)) groups = 0;
        heavy_before = heavy_now; by_before = by;
    };
    // What was left open goes to the record of the 128 x 128 tile: a few comparisons by their places; many, or all of them, as the
    // wavefront's blocks, in which it then counts no violations.
    auto record = [&](const Tile& tile, Places open, bool none_decided, unsigned vio_before) __attribute__((always_inline)) {
        if (!(__any(open != 0) || none_decided)) return;
        unsigned* const rec = p.open.of(((size_t)tile.z * p.open_m + (unsigned)(tile.m0 >> 7)) * p.open_n + (unsigned)(tile.n0 >> 7));
        const unsigned places = (unsigned)p.open.places();
        const unsigned r0 = ((unsigned)tile.m0 & 127u) + srow, c0 = ((unsigned)tile.n0 & 127u) + scol;
        const unsigned mine = (unsigned)__popcll((unsigned long long)open), upto = (unsigned)wave_scan(mine), all = wave_sum(mine);
        unsigned was = 0;
        bool listed = !none_decided && all <= places;
        if (listed) {
            if (lane == 0) was = atomicAdd(rec, all << 16);
            was = __builtin_amdgcn_readfirstlane(was);
            listed = (was >> 16) + all <= places;
            unsigned at = (was >> 16) + upto - mine;
            for (Places left = open; left && at < places; left &= left - 1, ++at) {
                const int bit = __ffsll((unsigned long long)left) - 1, step = bit >> 2;
                const unsigned row = r0 + (unsigned)(step / STEPS * 32 + lrow + step % STEPS * RPI), col = c0 + (unsigned)(lcol + (bit & 3));
                rec[2 + at] = listed ? row << 7 | col : kNoPlace;
            }
            opened += was == 0;
        }
        if (!listed) {
            const unsigned before = was;
            constexpr unsigned across = (1u << RN) - 1u;
            const unsigned blocks = (RM == 2 ? across | across << 4 : across) << (r0 / 32 * 4 + c0 / 32);
            if (lane == 0) { was = atomicOr(rec, blocks); atomicAdd(&heavy, 1u); }
            was = __builtin_amdgcn_readfirstlane(was);
            opened += before == 0 && was == 0;
            vio = vio_before;
        }
    };

    unsigned t = (unsigned)((unsigned long long)p.ntiles * xcd >> 3) + (blockIdx.x >> 3);
    const unsigned t_first = t;
    bool begun = false, fetched = false;                     // the next tile's first slabs are on their way to their stages; its first claims and outputs are
    if (EARLY) __syncthreads();                              // (the words are clear)
    Tile tile;
    Sources src;
    if (EARLY && p.groups > GPS && t < t_end) {
        tile = tile_of(t);
        bool attempt = true;
        if (!ACROSS) {
            // First slabs are not tried where claims are far off from the start: an error of the share of the bound that they would prove is at
            // least that share of the output's own.  (By a wavefront's first elements, 5 in 8 of them.)
            begin(tile, src);
            const float part = p.low * (float)GPS / (float)p.groups;
            if (far_off(tile, 5, [&](int e) { return fabsf(rv[0][e]) * part; }) || marks != kOrdinary * 0x01010101u) unordinary = 1;
            __syncthreads();
            attempt = now(unordinary) == 0;
            begun = fetched = !attempt;
        }
        if (attempt) {
            const unsigned n = ACROSS ? min((unsigned)kEarlyTiles, (t_end - t + per - 1) / per) : 1u, went = early_walk(t, n, tile);
            t += per * went;
            fetched = went < n;
        }
    }
    // Claims and outputs of the first strip are requested before the product, and by tiles that are walked (the larger ones) while the last strip of the tile
    // before is checked, as its registers become free: a copy into LDS that is waited for has all older loads waited for too, so
    // requested behind the tile's barrier they held its first slab up (8 x 8192 x 2048 over 128 246 -> 233 us, the convolution of
    // 32 x 56 x 56 x 256 with its affine operator 317 -> 308; 512 x 3072 over 768, whose workgroups have a tile each, 22.8 -> 24).
    if (ACROSS && t < t_end) {
        tile = tile_of(t);
        if (!fetched) {
#pragma unroll
            for (int k = 0; k < STEPS; ++k) fetch(tile, 0, k);
        }
    }
    for (; t < t_end; t += per) {
        if (!ACROSS && !(EARLY && fetched)) {
            tile = tile_of(t);
#pragma unroll
            for (int k = 0; k < STEPS; ++k) fetch(tile, 0, k);
        }
        if (!(EARLY && begun)) sources_of(tile, src);
        Sums sums;
        clear_sums(sums);
        meet();
        product(src, sums, !ACROSS && begun);
        begun = fetched = false;
        const bool large = finish_sums(tile, sums);
        first_error();
        if (large) large_in = t + 1;
        __syncthreads();                                     // every wavefront is done with the stages
        known = max(known, newest(&largest));
        const bool none_decided = groups == 0 || large_in == t + 1;      // (its first half of k is one wavefront's, the tile's concern all the same)
        Places open = 0;                                     // comparisons that were not decided: bit 4 (i STEPS + k) + e
        const unsigned vio_before = vio;
        const bool last = t + per >= t_end;
        const Tile next = ACROSS ? tile_of(last ? t : t + per) : tile;
        check_tile(tile, sums, p.high, open, [](int) {},
                   [&](int i, int k) __attribute__((always_inline)) {
                       if (i + 1 < RM) fetch(tile, i + 1, k);       // the next strip's, as soon as the registers are free
                       else if (ACROSS && !last) fetch(next, 0, k);
                   });
        record(tile, open, none_decided, vio_before);
        if (ACROSS) tile = next;
    }
    if (EARLY && p.groups > GPS) {
        // Tiles of which a first slab did not decide all: all products, and the comparisons once more (the errors are settled).
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        const int words = now(some_pending) ? kEarlyWords : 0;
#pragma unroll 1
        for (int w = 0; w < words; ++w) {
            for (unsigned these = now(pending[w]); these; these &= these - 1) {
                const unsigned at = t_first + (unsigned)(w * 32 + __ffs((int)these) - 1) * per;
                const Tile again = tile_of(at);
                Sources src;
                sources_of(again, src);
                Sums sums;
                clear_sums(sums);
                meet();
                product(src, sums, false);
                if (finish_sums(again, sums)) large_in = at + 1;
                __syncthreads();                             // every wavefront is done with the stages
                const bool none_decided = groups == 0 || large_in == at + 1;
                Places open = 0;
                unsigned found = 0, counted = 0;             // violations, and NaN claims, which the first slab's check has counted
#pragma unroll
                for (int i = 0; i < RM; ++i) {
                    put_strip(sums, i);
#pragma unroll
                    for (int k = 0; k < STEPS; ++k) fetch(again, i, k);
#pragma unroll
                    for (int k = 0; k < STEPS; ++k) {
                        __builtin_amdgcn_sched_barrier(0);
                        const floatv4 s = strip_sums(k);
                        const int row = srow + i * 32 + lrow + k * RPI, col = scol + lcol;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float d = fabsf(cv[k][e] - rv[k][e]);
                            const bool in_range = row < again.rows_left && col + e < again.cols_left, nan = d != d;
                            const bool sure = s[e] >= p.tiny, above = (d > fmaf(s[e], p.high, bh[e])) & sure;
                            found += in_range & above;
                            counted += in_range & nan;
                            open |= (Places)(in_range & !(nan | above | (d == 0.f) | ((d <= fmaf(s[e], p.low, bl[e])) & sure))) << (4 * (i * STEPS + k) + e);
                        }
                    }
                }
                const unsigned vio_before = vio - counted;
                vio += found;
                record(again, open, none_decided, vio_before);
            }
        }
    }
    if (EARLY && !ACROSS) __builtin_amdgcn_s_waitcnt(0x0F70);       // (a second slab that nobody has read has landed)
    // this workgroup's counts to one of the partial results (integer atomics: the sums do not depend on the order)
    __syncthreads();
    if (SPARE && wave == 0) zeros += (int)hist[kHistWords + lane];
    zeros = wave_sum(zeros) + all_zeros;
    vio = wave_sum(vio); nans = wave_sum(nans); max_bits = wave_max(max_bits);
    const unsigned slot = blockIdx.x % (unsigned)kScreenSlots;
    if (lane == 0) {
        if (zeros) atomicAdd(&hist[0], (unsigned)zeros);
        if (nans) {
            atomicAdd(&p.hist[(size_t)slot * kBins + kBins - 1], nans);
            atomicAdd(&p.coarse[slot * kGroups + kGroups - 1], nans);
        }
        BlockStats* st = p.stats + slot;
        if (vio) atomicAdd(&st->violations, (unsigned long long)vio);
        if (nans) atomicAdd(&st->nans, (unsigned long long)nans);
        if (max_bits) atomicMax(&st->max_bits, max_bits);
        if (opened) atomicAdd(&st->flag, opened);
    }
    __syncthreads();
    // (a group of 64 bins to a wavefront: its atomics fall into two lines, and few groups are not empty.  With eight bins to a thread, and 256
    // lanes' atomics for the first error: 1111 x 3001 over 1001 with its cut 41.98 us, so 40.57)
    for (int base = wave * kWave; base < kBins; base += THREADS) {
        const int bin = base + lane;
        const unsigned cnt = bin <= 2040 ? hist[bin] : 0u;
        if (!__any(cnt != 0)) continue;
        if (cnt) atomicAdd(&p.hist[(size_t)slot * kBins + bin], cnt);
        const unsigned gsum = wave_sum(cnt);
        if (lane == 0) atomicAdd(&p.coarse[slot * kGroups + base / kWave], gsum);
    }
}

template <int RM, int RN, int WVM, int WVN, int GPS, int NST, int PER_CU, int SRC, bool EARLY, bool UNDERFLOW = spare_words(RM * RN) == 0>
int launch_config(ScreenArgs& p, long batch, hipStream_t st) {
    if (!UNDERFLOW && p.eps_rel > 1.0) return launch_config<RM, RN, WVM, WVN, GPS, NST, PER_CU, SRC, EARLY, true>(p, batch, st);
    constexpr int TM = WVM * RM * 32, TN = WVN * RN * 32;
    constexpr int lds_bytes = stage_bytes(RM, RN, WVM, WVN, GPS, NST, SRC, EARLY) + words_before_stages(RM * RN, EARLY) * 4;
    auto kernel = &screen_product<RM, RN, WVM, WVN, GPS, NST, PER_CU, SRC, EARLY, UNDERFLOW>;
    static OncePerDevice configured;
    const hipError_t e = configured.run([&] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (e != hipSuccess) { g_last_hip_error = (int)e; return TAO_ERR_LAUNCH; }
    p.tiles_m = (unsigned)((p.M + TM - 1) / TM); p.tiles_n = (unsigned)((p.N + TN - 1) / TN);
    const long ntiles = (long)p.tiles_m * p.tiles_n * batch;
    if (ntiles >= (1L << 30)) return TAO_ERR_SHAPE;
    p.ntiles = (unsigned)ntiles;
    long grid = (long)device_cus() * PER_CU & ~7L;
    if (grid < 8) grid = 8;
    const long want = (ntiles + 7) & ~7L;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(want < grid ? want : grid)), dim3(WVM * WVN * 64), lds_bytes, st, p);
    return launch_status();
}

enum Config { kRows64x128, kRows64x64, kPixels128x128, kPixels128x128Short, kPixels64x64, kImages64x128, kImages128x128, kImages64x64Few, kImages64x64Short, kImages64x64 };
// Tiles of 128 x 128, two workgroups to a compute unit, where they give every compute unit one (us of the whole call on images, with
// them / with 64 x 64: 2048 x 12288 over 4096 248 / 362, 2048 x 4096 over 4096 94 / 122, 1111 x 3001 over 1001, 216 tiles, 37 / 33);
// up to 256 k, where the check is most of the work, 64 x 128 and three (8 x 8192 x 2048 over 128 250, with 128 x 128 280; 228 now).
// Otherwise, and where a column tile would be half empty, 64 x 64: four to a compute unit, or two with four groups to a barrier
// where there are no more, as a group's copies, barrier and reads of LDS then are a chain that nothing else hides (512 x 3072 over
// 768 21, with a group to a barrier 24, with 128 x 128 31; 512 x 768 over 3072 29 / 37 / 57; 256 x 1024 over 8192 51 / 71 / 110).
// Few 64 x 64 tiles try first slabs, of 128 k, where there are four or more (512 x 768 over 416 18.2 -> 17.6, 300 x 300 over 1000 19.3 -> 15.9; with
// two, 912 x 64 over 228, the screen alone 9.2 -> 11.3).
// Convolutions of one slab, 64 k, have no first one to try: the form that does not has fewer registers to keep (1 x 1, 32 x 28 x 28 x 64 to 512, with its
// affine operator, 97.5 -> 94.9; of 96 channels 97.0 without, 96.7 with).
// A read as rows: 64 x 128 where they fill the chip (8 x 8192 x 128 over 2048 145, with 64 x 64 183), else 64 x 64 (12 x 512 x 64 over
// 512 22 / 26).
constexpr long kFewGroups = 8;                               // (up to which no form of images tries first slabs)
Config screen_config(long M, long N, long K, long batch, bool rows, bool pixels) {
    const long n = device_cus(), groups = (K + SBK - 1) / SBK;
    const long t128 = ((M + 127) / 128) * ((N + 127) / 128) * batch, t64 = ((M + 63) / 64) * ((N + 63) / 64) * batch;
    const bool wide = t128 >= n && N > 64;
    if (rows) return ((M + 63) / 64) * ((N + 127) / 128) * batch >= n && N > 64 ? kRows64x128 : kRows64x64;
    if (pixels) return !wide ? kPixels64x64 : groups > 2 ? kPixels128x128 : kPixels128x128Short;
    if (wide) return groups <= kFewGroups ? kImages64x128 : kImages128x128;
    return t64 > 2 * n ? kImages64x64 : groups > 12 ? kImages64x64Few : kImages64x64Short;
}

}  // namespace

bool screen_reads_marks(long M, long N, long K, long batch, bool rows, bool pixels) {
    const Config c = screen_config(M, N, K, batch, rows, pixels);
    return c == kPixels128x128 || c == kImages128x128 || c == kImages64x64Few;
}
// (an operand by itself, whose product is not known yet: the cut of 512 x 256 3.3 us with marks, 3.0 without, of 100000 x 64 12.0 / 10.8)
bool screen_reads_marks(long K) { return (K + SBK - 1) / SBK > kFewGroups; }

int launch_screen(const ScreenOperand& A, const ScreenOperand& W, const float* bias, long M, long N, long K, long batch,
                  double cg, const ScreenCheck& chk, const CheckWorkspace& ws, const OpenRecords& open, hipStream_t st) {
    const long groups = (K + SBK - 1) / SBK, blocksA = (M + 127) / 128, blocksW = (N + 127) / 128;
    ScreenArgs p = {};
    const bool rows = A.ld != 0, pixels = A.pixels != nullptr;
    if (pixels) p.px = *A.pixels;
    p.A = static_cast<const char*>(A.data); p.W = static_cast<const char*>(W.data);
    p.stepA = rows ? SBK * 4 : blocksA * kImageBlock; p.stepW = blocksW * kImageBlock;
    p.batchA = A.batch_bytes; p.batchW = W.batch_bytes;
    p.last_blkA = (int)blocksA - 1; p.last_blkW = (int)blocksW - 1;
    p.ldA = A.ld * 4;
    p.marksA = reinterpret_cast<const unsigned*>(A.marks); p.marksW = reinterpret_cast<const unsigned*>(W.marks);
    p.M = M; p.N = N; p.groups = (int)groups;
    p.claimed = chk.claimed; p.ref = chk.ref; p.bias = bias; p.ldy = chk.ldy; p.strideY = chk.strideY;
    // (8 x 8192 x 2048, 1.07 GB: 251 us with streaming loads, 267 without; 4096 x 4096 73.3 / 70.7, 12 x 512 x 512 20.3 / 18.0, 2048 x 12288 the same)
    p.stream = (double)M * (double)N * (double)batch * 8.0 > 0x1p28;
    p.eps_rel = chk.eps_rel;
    const double a = chk.alpha * cg;
    const ScreenLimits lim = screen_limits(K);
    p.low = (float)(a * lim.lower * (1.0 - 0x1p-14)); p.high = (float)(a * lim.upper * (1.0 + 0x1p-14));
    p.low_b = (float)(a * (1.0 - 0x1p-14)); p.high_b = (float)(a * (1.0 + 0x1p-14));
    p.tiny = (float)(groups * SBK) * kTinyPerStep;
    p.open = open; p.open_m = (unsigned)blocksA; p.open_n = (unsigned)blocksW;
    p.hist = ws.hist; p.coarse = ws.coarse; p.stats = ws.stats;
    if (chk.ldy >= kScreenMaxLd) return TAO_ERR_SHAPE;
    switch (screen_config(M, N, K, batch, rows, pixels)) {
        case kRows64x128:     return launch_config<1, 2, 2, 2, 1, 4, 2, ROWS, false>(p, batch, st);
        case kRows64x64:      return launch_config<1, 1, 2, 2, 2, 3, 2, ROWS, false>(p, batch, st);
        case kPixels128x128:  return launch_config<2, 2, 2, 2, 2, 2, 2, PIXELS, true>(p, batch, st);
        case kPixels128x128Short: return launch_config<2, 2, 2, 2, 2, 2, 2, PIXELS, false>(p, batch, st);
        case kPixels64x64:    return launch_config<1, 1, 2, 2, 2, 2, 4, PIXELS, false>(p, batch, st);
        case kImages64x128:   return launch_config<1, 2, 2, 2, 1, 3, 3, IMAGE, false>(p, batch, st);
        case kImages128x128:  return launch_config<2, 2, 2, 2, 2, 2, 2, IMAGE, true>(p, batch, st);
        case kImages64x64Few: return launch_config<1, 1, 2, 2, 4, 2, 2, IMAGE, true>(p, batch, st);
        case kImages64x64Short: return launch_config<1, 1, 2, 2, 4, 2, 2, IMAGE, false>(p, batch, st);
        case kImages64x64:    return launch_config<1, 1, 2, 2, 2, 2, 4, IMAGE, false>(p, batch, st);
    }
    return TAO_ERR_SHAPE;                                    // (not reached)
}

}  // namespace tao
