// tao_bound_linear_split: the matmul bound tau = Gamma(K') (|A| |W|^T + |bias|) (Sec. 3.1
// reductions; App. A.2 Eq. det-sum) on the BF16 matrix cores of gfx950, which run at 16 times the
// FP32 MFMA rate.
//
// Every binary32 magnitude is cut exactly into three BF16 pieces, a = hi + mid + lo, each the
// remainder of the one before rounded to nearest (hi non-negative, mid and lo signed: |mid| <= 2^-8 a,
// |lo| <= 2^-17 a), by a streaming pre-pass or while it is loaded.  The product of two operands is
// then the sum of nine BF16 x BF16 products, each exact in binary32; mid x lo, lo x mid and lo x lo
// together stay below 1.001u of it and are covered by the inflation, the other six go through
// v_mfma_f32_32x32x16_bf16:
//   main   hi x hi                        one instruction from a zero accumulator per 16 k-steps,
//                                         folded into a binary64 running sum right away;
//   cross  mid x mid, hi x lo, lo x hi, hi x mid, mid x hi (in magnitude together below 1.008 x 2^-7 of
//          the total)                     one chain of 10 instructions per 32 k-steps, then folded.
// (Pieces cut by masking instead are all non-negative, but then mid x lo reaches 8u and two more
// products are needed: 2048 x 4096 x 12288 with its check 1481 - 1522 us against 1343 - 1394 us with six.)
//
// Accuracy.  For non-negative operands the instruction was characterised on the device (280 000
// cases against exact rational arithmetic, all reproduced) as two sequential steps over k = 0..7
// and k = 8..15, each:  products truncated to 24 bits below the largest product exponent e_P of
// the step and summed exactly into P;  with e the larger of e_P and the accumulator's exponent,
// accumulator truncated to 24 bits and P to 31 bits below e (P dropped when the accumulator's
// exponent exceeds e_P by 28 or more);  sum rounded to nearest even.  Hence per instruction from
// a zero accumulator the result lies in [S (1 - 10u), S (1 + 2u)] (at most seven truncated
// products per step, each losing less than 2^-24 of the step's largest product; one rounding per
// step; a dropped second step is below 2u of the first).  With signed operands the same steps err, in
// either direction, by at most 7u of the step's sum of magnitudes for the truncated products and 2.01u of the sum
// of all magnitudes so far for the rest (u for the truncated accumulator, 2^-7 u for the truncated P and u for the
// rounding, or 2u for a dropped P alone).  A cross chain runs the three small products first in each half:
// 14 of its 20 steps have a hi x mid in the accumulator, so it errs by at most (7 + 14 x 2.01)u of its sum of
// magnitudes, 0.28u of the total; the six steps before are below 2^-15 of the total.  hi x hi is at most 1 + 2^-7
// of the total.  Altogether the sum lies in [S (1 - 11.36u), S (1 + 3.30u)]; the
// epilogue multiplies by 1/(1 - 11.4u) (and the binary64 slack), by Gamma and the guard factor
// and rounds up:  exact <= tau <= exact (1 + 11.4u + 3.3u + 2u + ...) < exact (1 + 16.75u) < exact (1 + 1e-6).
// tao_selftest_matrix_core_bf16 re-checks the instruction model on the device in use.  Operands below
// 2^-110 in magnitude lose low bits of their lo piece in BF16's subnormal range; that piece is then raised
// (see split_pack8), so the bound stays an upper bound but can exceed 1e-6 there.  Sums that reach
// down into the binary32 subnormal range carry an absolute error instead of a relative one; the
// epilogue adds a bound on it (see split_core), which is far below 1e-6 of any bound above 2^-120.
//
// A check needs only the comparisons d <= alpha tau.  Where the caller does not want tau, one BF16 product
// (linear_screen.hip) decides them first, and the kernels of this file form the bound only if it left one open
// (absgemm_settle*, launched behind it in either case, for the tiles that hold open ones; screened() holds the rule).
#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>
#include "tao_device.hpp"
#include "tao_host.hpp"
#include "linear_f64.hpp"
#include "linear_screen.hpp"
#include "tao_check.hpp"

namespace tao {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));

constexpr int kSplitThreads = 512;
constexpr int SBK = 32;                 // k-steps per group: two MFMA k-groups of 16
constexpr int SROW = 64;                // bytes per row of a slab (32 BF16 values); the four 16-byte units of row r
                                        // sit at positions c ^ ((r >> 2) & 3), which spreads the 16-byte reads of 16
                                        // consecutive rows over all LDS banks without padding
constexpr int STILE = 128;              // output rows and columns per workgroup
constexpr int kSlab = STILE * SROW;     // one operand, one piece
constexpr int kBlock = 3 * kSlab;       // one operand, three pieces: 24576 bytes, contiguous in the workspace
constexpr int kSplitStage = 2 * kBlock; // |A| hi, mid, lo, |W| hi, mid, lo: 49152 bytes
constexpr int kSplitStages = 3;         // 144 KB of LDS
constexpr long kEpilogueCheckMinK = 1025; // shorter reductions (up to 1024, as far as the plain bound walks its tiles), where no screen decides: the bound is stored and the streaming check reads it (see split_run)
constexpr long kMinGroupsPerPart = 4;   // a reduction cut into parts: at least 128 k-steps each
constexpr long kWalkMaxGroups = 32;     // reductions up to 1024 k-steps walk their tiles ...
constexpr int kWalkMinTilesPerCu = 4;   // ... when a compute unit has at least this many

#define TAO_MFMA_BF16(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)

// ---- pre-pass: binary32 -> BF16 blocks [k / 32][row / 128][piece][row % 128][32] with the 16-byte units of
// a row swizzled: the LDS image of a workgroup's slab; zero-padded to Kp columns ----------------------
// The three pieces of |v|: hi = |v| rounded to the nearest BF16 value, mid = the exact remainder (signed) rounded to
// nearest, lo = the exact second remainder, six significant bits, so that hi + mid + lo = |v| with
// |mid| <= 2^-8 |v| and |lo| <= 2^-17 |v|.  hi is kept finite (a value beyond the largest BF16 number leaves its
// excess to mid, which stays within that bound).  An infinite or NaN operand leaves an infinite or NaN mid and a NaN
// lo (inf - inf), so its outputs are never finite.  Where lo falls below BF16's subnormal step, 2^-133 (operands below
// 2^-110), it is rounded up and raised by one step more: the pieces then sum to at least |v| + 2^-133, which covers what
// the dropped products (split_run) can amount to there, relative to such an operand.
// Eight consecutive values -> the three 16-byte units of BF16 pieces.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_bf16(float even, float odd) {                 // both rounded to nearest even
    return __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{even, odd}), bf16x2));
}
__device__ __forceinline__ unsigned short lo_below_step(float r2) {
    if (!(r2 == r2)) return 0x7fc0u;
    const unsigned bits = __float_as_uint(r2);
    if (!(bits & 0xffffu)) return (unsigned short)(bits >> 16);
    const unsigned up = __float_as_uint(r2 + 0x1p-133f);                               // exact: multiples of 2^-149 below 2^-126
    return (unsigned short)((up + ((up >> 31) ? 0u : 0xffffu)) >> 16);                 // towards +infinity
}
__device__ __forceinline__ void split_pack8(const float (&v)[8], uintx4& H, uintx4& Mi, uintx4& L) {
    float r2[8];
    unsigned below = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        constexpr float kMaxBf16 = 0x1.fep127f;
        const float a0 = fabsf(v[2 * j]), a1 = fabsf(v[2 * j + 1]);
        H[j] = pack_bf16(fminf(a0, kMaxBf16), fminf(a1, kMaxBf16));
        const float r0 = a0 - __uint_as_float(H[j] << 16), r1 = a1 - __uint_as_float(H[j] & 0xffff0000u);
        Mi[j] = pack_bf16(r0, r1);
        r2[2 * j] = r0 - __uint_as_float(Mi[j] << 16);
        r2[2 * j + 1] = r1 - __uint_as_float(Mi[j] & 0xffff0000u);
        L[j] = __builtin_amdgcn_perm(__float_as_uint(r2[2 * j + 1]), __float_as_uint(r2[2 * j]), 0x07060302u);
        below |= __float_as_uint(r2[2 * j]) | __float_as_uint(r2[2 * j + 1]);
    }
    if (__builtin_expect((below & 0xffffu) != 0, 0)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) L[j] = lo_below_step(r2[2 * j]) | ((unsigned)lo_below_step(r2[2 * j + 1]) << 16);
    }
}

// One thread per 8 consecutive k of one row, for one or two operands in one launch; a workgroup's unit is 64 rows of one 32-k group,
// 4 KB contiguous per piece.  STRAIGHT: four threads to a row, 128 contiguous bytes; units run along k, so the workgroups in
// flight read rows on; of an operand of up to 16 rows and many units each is one wavefront's (4 x 100000 3.8 us, with a workgroup each 5.6;
// 8 x 4096, 128 units, 2.7 / 2.6).  TRANSPOSED: the source is [K][ld] with the row index running along its columns (W stored
// K x N); the lanes of a wavefront take the unit's rows.  MAGNITUDES: no image but the BF16 magnitudes alone, in the source's
// layout (K a multiple of 8, one row), and 64 bytes of zeros behind them.
// What bounds it: HBM for large operands, else one unit's latency -- its position takes scalar 32-bit arithmetic only (a thread's own
// 64-bit divisions, units of 256 k, which a short reduction leaves empty, and loads behind branches took 8 x 8192 x 128 19.2 us, now
// 13.6, 1111 x 1001 5.2, now 4.2, 8 x 128 x 2048 transposed 10.3, now 8.1; 12288 x 4096 103, at 4.9 TB/s, and 104 with marks, which cost 0.2 to 0.4 us
// where one unit's latency is all there is).
enum { STRAIGHT, TRANSPOSED, MAGNITUDES };
struct SplitOperand {
    const float* src; long rows, K, ld, batch, stride; unsigned short* dst; int form;
    unsigned char* marks; int nmarks;  // where this operand's workgroups say that all they have read is ordinary, a byte each (linear_screen.hpp)
    bool spread;                       // (launch_split3) units are dealt out to the workgroups' first parts, then to their second ones, and so on
    __host__ __device__ bool flat() const { return form == STRAIGHT && rows <= 16 && (K + SBK - 1) / SBK * batch >= 512; }
};
struct SplitOperands {
    SplitOperand op[2];
    long first[3];                     // workgroups [first[o], first[o + 1]) serve operand o
    ClearJob clear;                    // (words 0: nothing)
};
__device__ __forceinline__ void clear_words(const ClearJob& c, long i0, long step) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
        for (long i = i0; i < c.words[j]; i += step) static_cast<uintx4*>(c.at[j])[i] = uintx4{0, 0, 0, 0};
}
// A workgroup's mark, and the first one's for the places of those that there are not.  (__syncthreads_and has three barriers,
// this one: 512 x 768 3.8 -> 3.4 us.)
__device__ __forceinline__ void leave_mark(const SplitOperand& p, long wg, long wgs, bool ordinary) {
    __shared__ unsigned all_of_wave[16];
    const int lane = threadIdx.x & (kWave - 1), waves = blockDim.x / kWave;
    const unsigned all = __all(ordinary);
    if (lane == 0) all_of_wave[threadIdx.x / kWave] = all;
    __syncthreads();
    if (threadIdx.x < kWave) {
        const bool ok = __all(all_of_wave[lane < waves ? lane : 0]);
        if (lane == 0) p.marks[wg] = ok ? kOrdinary : 0;
    }
    if (wg == 0)
        for (long i = wgs + threadIdx.x; i < p.nmarks; i += blockDim.x) p.marks[i] = kOrdinary;
}
constexpr int kMostSplitThreads = 1024;
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));          // (16-byte loads need no more than 4-byte alignment)
template <bool MARKED>
__global__ __launch_bounds__(MARKED ? kMostSplitThreads : 256) void split3_bf16(SplitOperands a) {
    const int threads = MARKED ? (int)blockDim.x : 256;
    // (side job for the launch that follows: clears the partial results of a check, so that no launch of its own is needed for that)
    clear_words(a.clear, (long)blockIdx.x * threads + threadIdx.x, (long)gridDim.x * threads);
    const int o = (long)blockIdx.x >= a.first[1] ? 1 : 0;
    // (both operands' fields are requested at once: the choice would be one more step of the chain of scalar loads)
    const SplitOperand &q0 = a.op[0], &q1 = a.op[1];
    const SplitOperand p = {o ? q1.src : q0.src, o ? q1.rows : q0.rows, o ? q1.K : q0.K, o ? q1.ld : q0.ld, o ? q1.batch : q0.batch,
                            o ? q1.stride : q0.stride, o ? q1.dst : q0.dst, o ? q1.form : q0.form, o ? q1.marks : q0.marks, o ? q1.nmarks : q0.nmarks,
                            o ? q1.spread : q0.spread};
    const long wgs = o ? a.first[2] - a.first[1] : a.first[1], wg = o ? (long)blockIdx.x - a.first[1] : (long)blockIdx.x;
    // 256 threads take a unit at a time; a workgroup holds one to four such parts
    const long parts = threads >> 8, part = MARKED ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
    const long nblk = wgs * parts, blk = p.spread ? part * wgs + wg : wg * parts + part;
    const int tid = threadIdx.x & 255;
    bool ordinary = true;                                    // (by the sums of eight magnitudes)
    auto look = [&](float s) __attribute__((always_inline)) { if (MARKED) ordinary &= s < 0x1p32f; };
    if (p.form == MAGNITUDES) {
        for (long i = blk * 256 + tid; i < p.K / 8 + 4; i += nblk * 256) {
            uintx4 H = {0, 0, 0, 0};
            if (i < p.K / 8) {
                const floatx4u* q = reinterpret_cast<const floatx4u*>(p.src) + 2 * i;
                const floatx4u x = q[0], y = q[1];
                H = uintx4{pack_bf16(fabsf(x[0]), fabsf(x[1])), pack_bf16(fabsf(x[2]), fabsf(x[3])),
                           pack_bf16(fabsf(y[0]), fabsf(y[1])), pack_bf16(fabsf(y[2]), fabsf(y[3]))};
                look(fabsf(x[0]) + fabsf(x[1]) + fabsf(x[2]) + fabsf(x[3]) + fabsf(y[0]) + fabsf(y[1]) + fabsf(y[2]) + fabsf(y[3]));
            }
            reinterpret_cast<uintx4*>(p.dst)[i] = H;
        }
        if (MARKED) leave_mark(p, wg, wgs, ordinary);
        return;
    }
    const bool trans = p.form == TRANSPOSED;
    const unsigned groups = (unsigned)((p.K + SBK - 1) / SBK), rgroups = (unsigned)((p.rows + 63) >> 6);
    const long rblocks = (p.rows + STILE - 1) / STILE;
    // rows up to the next multiple of four are zeros: the product's epilogue looks at its sums by groups of four rows
    const long rows4 = (p.rows + 3) & ~3L;
    const unsigned units = (unsigned)(groups * (unsigned long long)rgroups * p.batch);
    const bool flat = p.flat();
    const int urow = trans ? tid & 63 : (flat ? tid & 63 : tid) >> 2, uch = trans ? tid >> 6 : tid & 3;
    const unsigned first = flat ? (unsigned)blk * 4 + __builtin_amdgcn_readfirstlane(tid >> 6) : (unsigned)blk;
    for (unsigned u = first; u < units; u += (unsigned)nblk * (flat ? 4 : 1)) {
        const unsigned rz = u / groups, g = u - rz * groups, z = rz / rgroups, rg = rz - z * rgroups;
        const long row = (long)rg * 64 + urow, k0 = (long)g * SBK + uch * 8;
        if (row >= rows4) continue;
        const float* s = p.src + z * p.stride;
        float v[8];
        // (positions beyond the operand read its last row or element: loads without branches all leave at once)
        const long rc = row < p.rows ? row : p.rows - 1;
        if (!trans && k0 + 8 <= p.K) {
            const floatx4u* q = reinterpret_cast<const floatx4u*>(s + rc * p.ld + k0);
            const floatx4u x = q[0], y = q[1];
#pragma unroll
            for (int j = 0; j < 4; ++j) { v[j] = row < p.rows ? x[j] : 0.f; v[4 + j] = row < p.rows ? y[j] : 0.f; }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const long kc = k0 + j < p.K ? k0 + j : p.K - 1;
                v[j] = trans ? s[kc * p.ld + rc] : s[rc * p.ld + kc];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = row < p.rows && k0 + j < p.K ? v[j] : 0.f;
        }
        uintx4 H, Mi, L;
        split_pack8(v, H, Mi, L);
        look(fabsf(v[0]) + fabsf(v[1]) + fabsf(v[2]) + fabsf(v[3]) + fabsf(v[4]) + fabsf(v[5]) + fabsf(v[6]) + fabsf(v[7]));
        const long r = row & (STILE - 1);
        const long unit = uch ^ ((r >> 2) & 3);
        unsigned short* d = p.dst + (((long)z * groups + g) * rblocks + (row >> 7)) * (kBlock / 2) + r * (SROW / 2) + unit * 8;
        *reinterpret_cast<uintx4*>(d) = H;
        *reinterpret_cast<uintx4*>(d + (kSlab / 2)) = Mi;
        *reinterpret_cast<uintx4*>(d + 2 * (kSlab / 2)) = L;
    }
    if (MARKED) leave_mark(p, wg, wgs, ordinary);
}

// ---- the product ----------------------------------------------------------------------------
struct SplitArgs {
    const unsigned short* A3; const unsigned short* W3;     // blocks of |A| and |W| (see the pre-pass)
    const float* bias; float* tau;
    long M, N, Kp, ldt, strideT;
    long batchA3, batchW3;            // elements between batch entries (0 for a shared W)
    unsigned tiles_n, tiles_m;
    // tau = Gamma ((S + s) infl + |bias|) guard + underflow, with s the absolute part of the accumulation's
    // error (for a positive / for an exactly zero sum), as host-folded constants, each rounded up:
    // tau = fma(S, c1, fma(cg, (S > 0 ? si : si0) + |bias|, uflow))
    double c1, cg, si, si0, uflow;
    // CHECK instantiation: the claimed and the re-executed output (layout ldy / strideY), the check's
    // parameters and the partial results of the leaf check in the caller's workspace
    const float* claimed; const float* ref;
    long ldy, strideY;
    double alpha, eps_rel;
    unsigned int* ws_hist; unsigned int* ws_coarse; BlockStats* ws_stats; unsigned check_slots;
    // PARTIAL instantiation (the reduction cut into `ksplit` parts of `gpp` groups, one workgroup per
    // tile and part): binary64 partial sums [part][batch][M][N]
    unsigned ntiles; int ksplit; long gpp;
    double* partial;
    // workgroup -> tile: slots per super-tile (8 patches of ph x pw tiles), per batch entry, patches side by side
    unsigned slots, slots_per_z, super_rows, pw, ph, npx, linear;
    // AREG instantiations: the binary32 A operand itself (row stride lda, batch stride strideA, in
    // elements); A3 is then unused
    const float* Af; long lda, strideA;
    // CONV instantiations: Af is the channels-last input x[batch][H][W][C] of a convolution and row m of
    // the implicit patch matrix is output pixel (image, oh, ow); a 32-wide k slab is 32 consecutive
    // channels of one filter tap (C a multiple of 32)
    int cH, cW, cC, cOW, cS, csh, csw, cph, cpw, cdh, cdw; unsigned cohow;
};

// The constant term of the bound for a column with |bias| = ab, and the bound of a sum S (SplitArgs).
__device__ __forceinline__ double bound_offset(const SplitArgs& p, double s_abs, double ab) {
    return fma(p.cg, s_abs + ab, p.uflow);
}
__device__ __forceinline__ double bound_of_sum(const SplitArgs& p, double sv, double off_pos, double off_zero) {
    return fma(sv, p.c1, sv != 0.0 ? off_pos : off_zero);
}

// Sums beyond binary32.  hi is rounded up, so hi x hi can overflow where the magnitudes' own product (or the sum of 16 of
// them) does not, and an infinite main term meets an infinite cross term of the other sign: a sum that is not finite
// is formed again in binary64 from the same pieces (the products of two binary32 values are exact there, and every addition
// errs by 2^-53, far inside the inflation).  It stays NaN where an operand is not finite.
// Eight pieces' sums, exact: |v| (or the raised value of split_pack8).
__device__ __forceinline__ void piece_sums(const uintx4& H, const uintx4& Mi, const uintx4& L, double (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[2 * j] = (double)__uint_as_float(H[j] << 16) + (double)__uint_as_float(Mi[j] << 16) + (double)__uint_as_float(L[j] << 16);
        v[2 * j + 1] = (double)__uint_as_float(H[j] & 0xffff0000u) + (double)__uint_as_float(Mi[j] & 0xffff0000u) +
                       (double)__uint_as_float(L[j] & 0xffff0000u);
    }
}
// The same of an image: unit `unit` (8 consecutive k) of group g of a row; base: the batch entry, blocks: its 128-row blocks.
__device__ __forceinline__ void image_values(const unsigned short* base, long blocks, long row, long g, int unit, double (&v)[8]) {
    const int r = (int)(row & (STILE - 1));
    const unsigned short* at = base + (g * blocks + row / STILE) * (kBlock / 2) + r * (SROW / 2) + (unit ^ ((r >> 2) & 3)) * 8;
    piece_sums(*reinterpret_cast<const uintx4*>(at), *reinterpret_cast<const uintx4*>(at + kSlab / 2),
               *reinterpret_cast<const uintx4*>(at + kSlab), v);
}
// Where a convolution's patch row begins: input coordinates of filter tap (0, 0), offset of that pixel's first channel.
__device__ __forceinline__ void patch_origin(const SplitArgs& p, unsigned row, int& ih0, int& iw0, long& base) {
    const unsigned img = row / p.cohow, rem = row - img * p.cohow;
    const unsigned oh = rem / (unsigned)p.cOW, ow = rem - oh * (unsigned)p.cOW;
    ih0 = (int)oh * p.csh - p.cph; iw0 = (int)ow * p.csw - p.cpw;
    base = (((long)img * p.cH + ih0) * p.cW + iw0) * p.cC;
}
// The eight values' place of k group g, unit `unit`, of a patch row (inside: false for a tap in the zero padding, whose
// address is then the input's first).
__device__ __forceinline__ const float* patch_values(const SplitArgs& p, int ih0, int iw0, long base, long g, int unit, bool& inside) {
    const unsigned k0 = (unsigned)(g * SBK);
    const unsigned tap = k0 / (unsigned)p.cC, c0 = k0 - tap * (unsigned)p.cC;
    const unsigned r = tap / (unsigned)p.cS, sx = tap - r * (unsigned)p.cS;
    const int dr = (int)r * p.cdh, ds = (int)sx * p.cdw;
    inside = (unsigned)(ih0 + dr) < (unsigned)p.cH && (unsigned)(iw0 + ds) < (unsigned)p.cW;
    return p.Af + (inside ? base + ((long)dr * p.cW + ds) * p.cC + c0 : 0L) + unit * 8;
}
// One output's operands: where they lie, and the products of unit `unit` of group g added to s.
template <bool AREG, bool CONV>
struct OutputOperands {
    long row, col, blocksA, blocksW, base = 0;
    const unsigned short* w; const unsigned short* a; const float* af;
    int ih0 = 0, iw0 = 0;
    __device__ __forceinline__ OutputOperands(const SplitArgs& p, long row_, long col_, unsigned z)
        : row(row_), col(col_), blocksA((p.M + STILE - 1) / STILE), blocksW((p.N + STILE - 1) / STILE),
          w(p.W3 + (long)z * p.batchW3), a(p.A3 + (long)z * p.batchA3), af(p.Af + (long)z * p.strideA + row_ * p.lda) {
        if (CONV) patch_origin(p, (unsigned)row, ih0, iw0, base);
    }
    __device__ __forceinline__ double add(const SplitArgs& p, long g, int unit, double s) const {
        double av[8], wv[8];
        if (AREG) {
            bool inside = true;
            const float* src = CONV ? patch_values(p, ih0, iw0, base, g, unit, inside) : af + g * SBK + unit * 8;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = inside ? src[j] : 0.f;
            uintx4 H, Mi, L;
            split_pack8(v, H, Mi, L);
            piece_sums(H, Mi, L, av);
        } else {
            image_values(a, blocksA, row, g, unit, av);
        }
        image_values(w, blocksW, col, g, unit, wv);
#pragma unroll
        for (int j = 0; j < 8; ++j) s = fma(av[j], wv[j], s);
        return s;
    }
};
template <bool AREG, bool CONV>
__device__ __forceinline__ double sum_in_binary64(const SplitArgs& p, long row, long col, unsigned z, long g0, long ngroup) {
    const OutputOperands<AREG, CONV> operands(p, row, col, z);
    double s = 0.0;
#pragma unroll 1
    for (long g = g0; g < g0 + ngroup; ++g) {
#pragma unroll 1
        for (int unit = 0; unit < 4; ++unit) s = operands.add(p, g, unit, s);
        if (s != s) break;
    }
    return s;
}

// check_one with the histogram layout of the CHECK instantiation below (16-bit counters, bin b in
// half b & 1 of word (b >> 1) * 4 + copy).
__device__ __forceinline__ void check_one_packed(float c, float r, float t, double alpha, double eps_rel,
                                                 unsigned int* hist, int copy, ThreadAcc& acc) {
    const CheckedElement o = check_arith<false>(c, r, t, alpha, eps_rel);
    acc.violations += o.violation;
    acc.nans += o.is_nan;
    if (!o.is_nan) acc.max_bits = max(acc.max_bits, o.bits);
    atomicAdd(&hist[(o.bin >> 1) * 4 + copy], (o.bin & 1) ? 0x10000u : 1u);
}

// Slot t -> tile (first row and column, batch entry); false if the slot has none (see absgemm_split_slot).
__device__ __forceinline__ bool locate_tile(const SplitArgs& p, unsigned t, unsigned& tm0, unsigned& tn0, unsigned& tz) {
    const unsigned zp = t / p.slots_per_z, bb = t - zp * p.slots_per_z;
    if (p.linear) {                                          // fewer tiles than compute units: row by row, no empty slot
        const unsigned ty = bb / p.tiles_n, tx = bb - ty * p.tiles_n;
        tn0 = tx * STILE; tm0 = ty * STILE; tz = zp;
        return true;
    }
    const unsigned sup = bb / p.slots, w8 = bb - sup * p.slots;
    const unsigned xcd = w8 & 7u, j = w8 >> 3;
    const unsigned ly = (xcd / p.npx) * p.ph + j / p.pw, lx = (xcd % p.npx) * p.pw + j % p.pw;
    const unsigned sband = sup / p.super_rows, srow = sup - sband * p.super_rows;
    const unsigned ty = srow * 16u + ly, tx = sband * 16u + lx;
    tn0 = tx * STILE; tm0 = ty * STILE; tz = zp;
    return ly < 16u && lx < 16u && ty < p.tiles_m && tx < p.tiles_n;
}

// Adds a workgroup's histogram (CHECK, below) to a partial result: non-empty bins; a wavefront covers one group of 64 bins.
__device__ __forceinline__ void flush_packed(const SplitArgs& p, const unsigned int* chk_hist) {
    const int tid = threadIdx.x, lane = tid & 63;
    const unsigned slot = blockIdx.x % p.check_slots;
    for (int b = tid; b < kBins; b += kSplitThreads) {
        unsigned int cnt = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) cnt += (chk_hist[(b >> 1) * 4 + c] >> (16 * (b & 1))) & 0xffffu;
        if (cnt) atomicAdd(&p.ws_hist[(size_t)slot * kBins + b], cnt);
        const unsigned int gsum = wave_sum(cnt);
        if (lane == 0 && gsum) atomicAdd(&p.ws_coarse[slot * kGroups + b / kBinsPerReduceBlock], gsum);
    }
}
__device__ __forceinline__ void flush_counters(const SplitArgs& p, const ThreadAcc& acc) {
    const unsigned slot = blockIdx.x % p.check_slots;
    const unsigned int vio = wave_sum(acc.violations), nn = wave_sum(acc.nans), mx = wave_max(acc.max_bits);
    if ((threadIdx.x & 63) == 0) {
        BlockStats* st = p.ws_stats + slot;
        if (vio) atomicAdd(&st->violations, (unsigned long long)vio);
        if (nn) atomicAdd(&st->nans, (unsigned long long)nn);
        if (mx) atomicMax(&st->max_bits, mx);
    }
}

template <bool SHARED>
__device__ __forceinline__ void store_sum(double* at, double s) {
    if (SHARED) __hip_atomic_store(at, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *at = s;
}

// The work of slot `wg` of `nwg` (false: the slot has no tile), by all threads of a workgroup.  lds: the stages; chk: the
// histogram (CHECK) or what is to be compared (OPEN).
// CHECK: the epilogue also runs the leaf check of Sec. 5.4 and the relative-error profile of Sec. 5.3
// on every bound it has just formed (the binary32 value the plain instantiation would store), against
// `claimed` and `ref`, with a 2048-bin histogram in the 16 KB of LDS the three stages leave free; tau
// itself is stored only if p.tau is not NULL.  Workgroups add their counts to one of p.check_slots
// partial results (integer atomics: the sums do not depend on the order), which profile_reduce
// finishes as it does for the streaming check.
// OPEN (with CHECK): behind a screen; only the comparisons whose bits are set in `chk` (a word per 32 columns of a row of the tile) are
// made, and of the profile only violations are counted.
// PARTIAL: launches with fewer tiles than compute units cut the reduction into parts; a workgroup
// then leaves the binary64 sums of its part in the workspace, and split_combine -- behind a screen the tile's last
// workgroup (SHARED: the sums are for another workgroup of the same launch) -- adds the parts, forms the bound and, if asked, checks it.
// WALK: the plain bound as the host launches it.  A workgroup takes the slots blockIdx.x,
// + gridDim.x, ... and its pipeline of slabs runs on across the tile boundaries: with a workgroup
// per slot that is one tile, with a workgroup per compute unit (short reductions) a walk over many.
// AREG: the A operand is not read from a prepared image but from its binary32 matrix: every thread
// loads 8 consecutive k of one row of the slab two groups ahead, cuts them into the three pieces in
// registers one group ahead and writes them to the stage in the image's layout.  For products
// whose A operand is used by one or two column tiles only (a 128-column output, e.g. attention
// probabilities times values), where a pre-pass over A (10 bytes per element written and read back)
// costs more than the product.  One tile per workgroup (no walk), whole groups only (K a multiple
// of 32), 16-byte aligned rows: the host checks all of it.
// CONV (with AREG): the A operand is the implicit patch matrix of a convolution, gathered from the
// channels-last input while loading; taps in the zero padding contribute zeros.
template <bool CHECK, bool PARTIAL, bool WALK, bool AREG, bool CONV, bool SHARED = false, bool OPEN = false>
__device__ __forceinline__ bool absgemm_split_slot(const SplitArgs& p, unsigned wg, unsigned nwg, char* lds, unsigned int* chk) {
    static_assert(CHECK || !OPEN, "a check of what is open");
    static_assert(!CONV || AREG, "the patch matrix exists only as a gather");
    static_assert(!(CHECK && PARTIAL), "the parts are checked when they are added");
    static_assert(!(WALK && (CHECK || PARTIAL)), "only the plain bound walks tiles");
    static_assert(!(AREG && WALK), "the in-load split keeps one tile per workgroup");
    // CHECK: four copies of the 2048-bin histogram with 16-bit counters (a tile has 16384 elements, so
    // none overflows), two bins to a word and the four copies of a word in consecutive banks: 16 KB,
    // all the LDS the stages leave.  The copy is chosen by the lane; errors crowd into a few bins, and
    // a single copy serialised the workgroup's atomics.
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;                 // 4 x 2 wavefronts, two 32x32 tiles each (along N)
    const int r32 = lane & 31, h = lane >> 5;

    // Workgroup -> tiles.  The output is walked in super-tiles of up to 16 x 16 tiles (column bands of
    // 16, rows running down a band): the workgroups in flight then read about 16 + 16 operand blocks
    // per group instead of a few rows times every column, which re-read all of W for every wave of
    // tiles.  Workgroups are dealt round-robin to the eight XCDs, each with its own L2: a super-tile is
    // cut into eight patches (ph rows x pw columns, npx of them side by side) and XCD x takes patch x,
    // so its tiles share ph + pw blocks (4 + 8 for a full super-tile).  Slots that fall beyond the
    // output's edge belong to no tile.  (A walk's stride is a multiple of 8, so a workgroup stays
    // with its XCD's patches.)  CHECK and PARTIAL calls take one slot (and part).
    const long part = PARTIAL ? wg / p.ntiles : 0;
    unsigned m0 = 0, n0 = 0, z = 0;                          // first row and column of the tile, batch entry
    auto locate = [&](unsigned t, unsigned& tm0, unsigned& tn0, unsigned& tz) __attribute__((always_inline)) -> bool {
        return locate_tile(p, t, tm0, tn0, tz);
    };
    // first slot at or after t (stepping by the grid) that holds a tile; p.ntiles if there is none
    auto next_tile = [&](unsigned t, unsigned& tm0, unsigned& tn0, unsigned& tz) __attribute__((always_inline)) -> unsigned {
        if (!WALK) return (t < p.ntiles && locate(t, tm0, tn0, tz)) ? t : p.ntiles;
        while (t < p.ntiles && !locate(t, tm0, tn0, tz)) t += nwg;
        return t < p.ntiles ? t : p.ntiles;
    };
    unsigned t = next_tile(PARTIAL ? wg % p.ntiles : wg, m0, n0, z);
    if (t >= p.ntiles) return false;                             // whole workgroup
    if (CHECK && !OPEN) {
        for (int i = threadIdx.x; i < kBins * 2; i += kSplitThreads) chk[i] = 0;
        __syncthreads();
    }
    // groups [g0, g0 + ngroup) of the reduction
    const long all_groups = p.Kp / SBK;
    const long g0 = PARTIAL ? part * p.gpp : 0;
    const long ngroup = PARTIAL ? (all_groups - g0 < p.gpp ? all_groups - g0 : p.gpp) : all_groups;

    // global -> LDS without a stop in registers: the workspace holds, per group and 128-row block,
    // the LDS image of the three pieces (24576 contiguous bytes); every wavefront copies three 1 KB
    // pieces of it per operand with 16-byte loads that write lane i's data at the wavefront's LDS
    // base + 16 i.
    const long blocksA = (p.M + STILE - 1) / STILE, blocksW = (p.N + STILE - 1) / STILE;
    const long stepA = blocksA * kBlock, stepW = blocksW * kBlock;            // bytes between groups
    auto request = [&](char* stage, unsigned tm0, unsigned tn0, unsigned tz, long g) __attribute__((always_inline)) {
        const char* a = reinterpret_cast<const char*>(p.A3 + (long)tz * p.batchA3) + (long)(tm0 / STILE) * kBlock + tid * 16 + (g0 + g) * stepA;
        const char* w = reinterpret_cast<const char*>(p.W3 + (long)tz * p.batchW3) + (long)(tn0 / STILE) * kBlock + tid * 16 + (g0 + g) * stepW;
        // (written as assembly: the compiler would otherwise wait for all outstanding copies before
        // every barrier, which is exactly the overlap this pipeline exists for; the waits are the
        // explicit s_waitcnt instructions below)
        const unsigned dst = __builtin_amdgcn_readfirstlane(
            (unsigned)(size_t)(__attribute__((address_space(3))) char*)(stage) + (unsigned)wave * 1024u);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (!AREG)
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                             :: "s"(dst + (unsigned)(i * kSplitThreads * 16)), "v"(a + i * kSplitThreads * 16) : "memory");
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                         :: "s"(dst + (unsigned)(kBlock + i * kSplitThreads * 16)), "v"(w + i * kSplitThreads * 16) : "memory");
        }
    };
    // AREG: thread -> row tid / 4 of the tile, k chunk tid % 4 of the group (8 consecutive k: 32
    // bytes).  Ordinary loads, which the compiler tracks: it waits for them where their registers are
    // first used (commit_a, one group after the request).  Rows beyond M read the last row instead
    // (their outputs are never stored).
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    // CONV: input coordinates of filter tap (0, 0) for this thread's patch row and the offset of that
    // pixel's first channel (a row beyond M never has a tap inside)
    int cv_ih0 = 0, cv_iw0 = 0; long cv_base = 0;
    if (CONV) {
        const long m = (long)m0 + (tid >> 2);
        patch_origin(p, m < p.M ? (unsigned)m : 0u, cv_ih0, cv_iw0, cv_base);
        if (m >= p.M) cv_ih0 = -(1 << 30);
    }
    // `inside`: CONV only, whether the slab's tap lies inside the input for this row (else the loaded
    // values are replaced by zeros when the slab is cut)
    auto fetch_a = [&](floatx4& lo4, floatx4& hi4, bool& inside, long g) __attribute__((always_inline)) {
        const float* src;
        if (CONV) {
            src = patch_values(p, cv_ih0, cv_iw0, cv_base, g, tid & 3, inside);
        } else {
            inside = true;
            long row = (long)m0 + (tid >> 2);
            row = row < p.M ? row : p.M - 1;
            src = p.Af + (long)z * p.strideA + row * p.lda + (g0 + g) * SBK + (tid & 3) * 8;
        }
        lo4 = reinterpret_cast<const floatx4*>(src)[0];
        hi4 = reinterpret_cast<const floatx4*>(src)[1];
    };
    auto commit_a = [&](char* stage, const floatx4& lo4, const floatx4& hi4, bool inside) __attribute__((always_inline)) {
        float v[8] = {lo4[0], lo4[1], lo4[2], lo4[3], hi4[0], hi4[1], hi4[2], hi4[3]};
        if (CONV) {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = inside ? v[j] : 0.f;
        }
        uintx4 H, Mi, L;
        split_pack8(v, H, Mi, L);
        const int r = tid >> 2;
        const int o = r * SROW + (((tid & 3) ^ ((r >> 2) & 3)) * 16);
        *reinterpret_cast<uintx4*>(stage + o) = H;
        *reinterpret_cast<uintx4*>(stage + kSlab + o) = Mi;
        *reinterpret_cast<uintx4*>(stage + 2 * kSlab + o) = L;
    };

    double S[2][16];
    floatx16 X[2], D[2], zero;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        zero[v] = 0.f;
#pragma unroll
        for (int tj = 0; tj < 2; ++tj) { S[tj][v] = 0.0; X[tj][v] = 0.f; D[tj][v] = 0.f; }
    }
    // operand fragments: lane (r32, h) holds k = 16 kg + 8 h .. + 7 of its row: unit 2 kg + h, swizzled
    const int swz = (r32 >> 2) & 3;
    const int unit0 = (h ^ swz) * 16, unit1 = ((2 + h) ^ swz) * 16;
    const int fragA = (wm * 32 + r32) * SROW;
    const int fragW = kBlock + (wn * 64 + r32) * SROW;
    auto frag = [&](const char* stage, int off) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8*>(stage + off);
    };
    // One group (32 k-steps) of both tiles of the wavefront, in four parts (k half, tile): a part
    // issues the six matrix-core instructions of its tile (hi x hi from zero into D, the five
    // cross products into the chain X, the small ones first) and, in their shadow, folds into the binary64 sums what the
    // OTHER tile finished one part earlier: its D always, its chain X where the chain has just ended
    // (tile 0's ends in the third part, tile 1's in the fourth and is folded in the first part of the
    // next group).  A matrix-core instruction occupies its pipe for 32 cycles, in which the SIMD
    // issues up to eight vector instructions; folding a result right after the instruction that
    // produced it instead stalls the wavefront until that instruction has drained (measured: the loop
    // runs at the matrix cores' own pace with this order and 19 % slower without).  The scheduling
    // directives ask for exactly that interleaving: one matrix-core instruction, then 6 or 11 vector
    // instructions.
    auto fold = [&](double (&acc)[16], const floatx16& part) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] += (double)part[v];
    };
    auto compute = [&](const char* stage) __attribute__((always_inline)) {
#pragma unroll
        for (int kg = 0; kg < 2; ++kg) {
            bf16x8 a[3], b[2][3];
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const int unit = kg == 0 ? unit0 : unit1;
                a[s] = frag(stage, s * kSlab + fragA + unit);
                b[0][s] = frag(stage, s * kSlab + fragW + unit);
                b[1][s] = frag(stage, s * kSlab + fragW + 32 * SROW + unit);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int o = t ^ 1;
                const bool chain_ended = (kg == 0) == (t == 0);  // parts (0, 0) and (1, 1)
                fold(S[o], D[o]);
                if (chain_ended) fold(S[o], X[o]);
                D[t] = TAO_MFMA_BF16(a[0], b[t][0], zero);
                // the cross products: the three of the order of 2^-16, then hi x mid and mid x hi
                X[t] = TAO_MFMA_BF16(a[1], b[t][1], kg == 0 ? zero : X[t]);
                X[t] = TAO_MFMA_BF16(a[0], b[t][2], X[t]);
                X[t] = TAO_MFMA_BF16(a[2], b[t][0], X[t]);
                X[t] = TAO_MFMA_BF16(a[0], b[t][1], X[t]);
                X[t] = TAO_MFMA_BF16(a[1], b[t][0], X[t]);
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                     // one MFMA
                    if (chain_ended) __builtin_amdgcn_sched_group_barrier(0x002, 11, 0);   // vector ALU
                    else             __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
                }
            }
        }
    };

    // Three LDS stages.  The slabs of a workgroup's tiles form one sequence: slab j of it is requested
    // at the top of group j - 2 into stage j % 3 and used in group j, so the first two slabs of the
    // next tile are on their way while this tile's last groups and its epilogue run.  At the top of
    // a group a wavefront waits until only its six youngest requests (slab j + 1) are outstanding,
    // so its part of slab j has landed; the barrier then publishes the slab and separates the last
    // reads of stage (j + 2) % 3 (group j - 1) from its next fill.  The first group of a later tile
    // waits for everything instead: the epilogue before it has issued loads, stores and atomics of
    // its own, which count in the same counter.
    // AREG: slab j's A part is requested into registers at the top of group j - 2 (after the copies of
    // slab j - 1's A part have been cut and written), cut into its pieces and written to stage j % 3 at
    // the top of group j - 1, and used in group j.
    floatx4 ar0[2], ar1[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) { ar0[i] = floatx4{0.f, 0.f, 0.f, 0.f}; ar1[i] = ar0[i]; }
    bool in0 = true, in1 = true;
    if (AREG) {
        if (ngroup > 0) { fetch_a(ar0[0], ar0[1], in0, 0); request(lds, m0, n0, z, 0); }
        if (ngroup > 1) { fetch_a(ar1[0], ar1[1], in1, 1); request(lds + kSplitStage, m0, n0, z, 1); }
        if (ngroup > 0) commit_a(lds, ar0[0], ar0[1], in0);
    } else {
        if (ngroup > 0) request(lds, m0, n0, z, 0);
        if (ngroup > 1) request(lds + kSplitStage, m0, n0, z, 1);
    }
    int cur = 0;
    bool first = true;
    unsigned top = 0;                                        // largest upper half of a sum (see the epilogue)
    ThreadAcc acc;
    const long nbatch = PARTIAL ? (long)(p.ntiles / p.slots_per_z) : 1;
#pragma unroll 1
    for (;;) {
        float pc[CHECK ? 2 : 1][CHECK ? 16 : 1], pr[CHECK ? 2 : 1][CHECK ? 16 : 1];
        unsigned m1 = 0, n1 = 0, z1 = 0;
        const unsigned tnext = WALK ? next_tile(t + nwg, m1, n1, z1) : p.ntiles;
        const bool more = WALK && tnext < p.ntiles;          // (the host walks tiles only if ngroup >= 2)
        // CHECK: the tile's claimed and re-executed values, requested before the last group so that their
        // latency passes under its arithmetic (the first 32-column half; the second half is requested
        // after that group, keeping 32 registers free during it).  Element (tj, v) of a lane: row m0 + wm*32 + 8*(v/4) + 4*h + v%4,
        // column n0 + wn*64 + tj*32 + r32 (the accumulator layout of a 32x32 tile).
        const float* __restrict__ Cl = CHECK ? p.claimed + (long)z * p.strideY : nullptr;
        const float* __restrict__ Rf = CHECK ? p.ref + (long)z * p.strideY : nullptr;
        // (Rows and columns beyond the edge read the edge's element instead: the epilogue does not
        // use them.  The empty asm statements keep the address arithmetic at the point of use: hoisted
        // out of the loops it would occupy a hundred registers through the whole reduction.)
        auto prefetch_claims = [&](int tj) __attribute__((always_inline)) {
            unsigned mo = m0, no = n0;
            int lrow = wm * 32 + 4 * h, lcol = wn * 64 + r32;
            asm volatile("" : "+s"(mo), "+s"(no), "+v"(lrow), "+v"(lcol));
            const long col = (long)no + lcol + tj * 32;
            const long colc = col < p.N ? col : p.N - 1;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const long row = (long)mo + lrow + 8 * (v >> 2) + (v & 3);
                const long rowc = row < p.M ? row : p.M - 1;
                pc[tj][v] = Cl[rowc * p.ldy + colc];
                pr[tj][v] = Rf[rowc * p.ldy + colc];
            }
        };
        // (the last group stands apart from the loop: the registers of the prefetched values are then
        // occupied in that copy of the arithmetic only)
        if (AREG) {
            // one group that is not the tile's last: slab g is used, slab g + 1 (register set `nset`,
            // requested one group ago) is cut and written to its stage, slab g + 2 requested
            auto body = [&](long g, floatx4 (&nset)[2], bool& nin, floatx4 (&fset)[2], bool& fin) __attribute__((always_inline)) {
                __builtin_amdgcn_s_waitcnt(0x0F75);               // vmcnt(5): all of slab g has landed
                __syncthreads();
                const int nxt2 = cur == 0 ? 2 : cur - 1, nxt1 = cur == 2 ? 0 : cur + 1;
                commit_a(lds + nxt1 * kSplitStage, nset[0], nset[1], nin);     // (the compiler waits for nset's loads here)
                if (g + 2 < ngroup) {
                    fetch_a(fset[0], fset[1], fin, g + 2);
                    request(lds + nxt2 * kSplitStage, m0, n0, z, g + 2);
                }
                compute(lds + cur * kSplitStage);
                cur = nxt1;
            };
            long g = 0;
#pragma unroll 1
            for (; g + 2 < ngroup; g += 2) { body(g, ar1, in1, ar0, in0); body(g + 1, ar0, in0, ar1, in1); }
            if (g + 1 < ngroup) body(g, ar1, in1, ar0, in0);
        } else {
#pragma unroll 1
        for (long g = 0; g + 1 < ngroup; ++g) {
            if (g == 0 && !first) __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
            else                  __builtin_amdgcn_s_waitcnt(0x0F76);      // vmcnt(6)
            __syncthreads();
            const int nxt2 = cur == 0 ? 2 : cur - 1;          // (cur + 2) % 3
            if (g + 2 < ngroup)  request(lds + nxt2 * kSplitStage, m0, n0, z, g + 2);
            else if (more)       request(lds + nxt2 * kSplitStage, m1, n1, z1, 0);
            compute(lds + cur * kSplitStage);
            cur = cur == 2 ? 0 : cur + 1;
        }
        }
        float bias_c[2] = {0.f, 0.f};
        if (!PARTIAL && p.bias) {
#pragma unroll
            for (int tj = 0; tj < 2; ++tj) {
                const long col = (long)n0 + wn * 64 + tj * 32 + r32;
                bias_c[tj] = p.bias[col < p.N ? col : p.N - 1];
            }
        }
        if (ngroup > 0) {
            if ((ngroup == 1 && !first) || !more) __builtin_amdgcn_s_waitcnt(0x0F70);
            else                                  __builtin_amdgcn_s_waitcnt(0x0F76);
            __syncthreads();
            const int nxt2 = cur == 0 ? 2 : cur - 1;
            if (more) request(lds + nxt2 * kSplitStage, m1, n1, z1, 1);
            if (CHECK) prefetch_claims(0);
            compute(lds + cur * kSplitStage);
            cur = cur == 2 ? 0 : cur + 1;
        } else if (CHECK) {
            prefetch_claims(0);
        }
        if (CHECK) prefetch_claims(1);                       // the second half passes under the first half's check
        fold(S[1], D[1]);                                    // what the last part left unfolded
        fold(S[1], X[1]);

        // Sums that are not finite: first whether there are any (a negative one, left by sums below 2^-126, passes for one), by
        // groups of four rows that exist (an image's rows end with zeros up to a multiple of four; what lies beyond is arbitrary).
        {
            const long rows_left = p.M - m0 - wm * 32 - 4 * h, cols_left = p.N - n0 - wn * 64 - r32;
#pragma unroll
            for (int tj = 0; tj < 2; ++tj) {
                unsigned most = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    unsigned four = 0;
#pragma unroll
                    for (int v = 0; v < 4; ++v) four = max(four, (unsigned)__double2hiint(S[tj][4 * b + v]));
                    most = max(most, 8 * b < rows_left ? four : 0u);
                }
                top = max(top, 32 * tj < cols_left ? most : 0u);
            }
        }
        if (CHECK && __builtin_expect(__any(top >= 0x7ff00000u), 0)) {
            // (positions and arguments in vector registers, the arguments read again: scalar ones would be taken from the loops)
            typedef const SplitArgs __attribute__((address_space(1)))* ArgsPtr;
            ArgsPtr q = (ArgsPtr)(size_t)__builtin_amdgcn_kernarg_segment_ptr();
            long row0 = (long)m0 + wm * 32 + 4 * h, col0 = (long)n0 + wn * 64 + r32, first_group = g0, groups = ngroup;
            unsigned zz = z;
            asm volatile("" : "+v"(q), "+v"(row0), "+v"(col0), "+v"(zz), "+v"(first_group), "+v"(groups));
            const SplitArgs& pa = *(const SplitArgs*)q;
            unsigned again = 0;
#pragma unroll
            for (int e = 0; e < 32; ++e) again |= (((unsigned)__double2hiint(S[e >> 4][e & 15]) & 0x7fffffffu) + 0x100000u) >> 31 << e;
            unsigned rows = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) rows |= ((1u << (int)max(0L, min(4L, pa.M - row0 - 8 * b))) - 1u) << (4 * b);
            again &= (col0 < pa.N ? rows : 0u) | (col0 + 32 < pa.N ? rows << 16 : 0u);
            if (__any(again != 0)) {
#pragma unroll 1
                for (int e = 0; e < 32; ++e) {
                    if (((again >> e) & 1u) == 0) continue;
                    const double s = sum_in_binary64<AREG, CONV>(pa, row0 + 8 * ((e & 15) >> 2) + (e & 3), col0 + (e >> 4) * 32, zz, first_group, groups);
#pragma unroll
                    for (int w = 0; w < 32; ++w) S[w >> 4][w & 15] = w == e ? s : S[w >> 4][w & 15];
                }
            }
        }

        // epilogue: D[i][j] of a 32x32 tile sits in lane (j + 32*((i/4)%2)), register 4*(i/8) + i%4
        float* __restrict__ T = p.tau ? p.tau + (long)z * p.strideT : nullptr;
        unsigned me = m0, ne = n0;
        int erow = wm * 32 + 4 * h, ecol = wn * 64 + r32;
        asm volatile("" : "+s"(me), "+s"(ne), "+v"(erow), "+v"(ecol));     // (as above)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj) {
            const long col = (long)ne + ecol + tj * 32;
            const double ab = fabs((double)bias_c[tj]);
            const double off_pos = bound_offset(p, p.si, ab), off_zero = bound_offset(p, p.si0, ab);
            const unsigned int* asked = chk + erow * (STILE / 32) + wn * 2 + tj;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const long row = (long)me + erow + 8 * (v >> 2) + (v & 3);
                if (OPEN) {
                    if (row < p.M && col < p.N && (asked[(8 * (v >> 2) + (v & 3)) * (STILE / 32)] >> r32 & 1u)) {
                        const float t32 = up32(bound_of_sum(p, S[tj][v], off_pos, off_zero));
                        acc.violations += !(fabs((double)pc[tj][v] - (double)pr[tj][v]) <= p.alpha * (double)t32);
                    }
                    continue;
                }
                if (PARTIAL) {
                    if (row < p.M && col < p.N) store_sum<SHARED>(p.partial + ((part * nbatch + z) * p.M + row) * p.N + col, S[tj][v]);
                    continue;
                }
                if (row < p.M && col < p.N) {
                    const float t32 = up32(bound_of_sum(p, S[tj][v], off_pos, off_zero));
                    if (!CHECK) {
                        T[row * p.ldt + col] = t32;
                    } else {
                        if (T) T[row * p.ldt + col] = t32;
                        check_one_packed(pc[tj][v], pr[tj][v], t32, p.alpha, p.eps_rel, chk, lane & 3, acc);
                    }
                }
            }
        }
        if (CHECK && !OPEN) {
            __syncthreads();
            flush_packed(p, chk);
        }
        if (!more) break;
        // Everything this tile has in flight ends here (the next tile's first two slabs were requested
        // long ago), so that no load or store of this tile counts in the next tile's waits.
        __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
        t = tnext; m0 = m1; n0 = n1; z = z1; first = false;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
#pragma unroll
            for (int tj = 0; tj < 2; ++tj) { S[tj][v] = 0.0; X[tj][v] = 0.f; D[tj][v] = 0.f; }
        }
    }
    // Plain bounds: the elements whose stored value is not finite once more, after the walk.  (Among the loops this code cost
    // the loops their schedule -- 1111 x 1001 x 3001: 64 against 59 us; positions and arguments are taken anew so that nothing of
    // it lives through them: else 4 spilled registers in the convolution, 988 against 978 us at 32 x 56 x 56 x 256.)
    if (!CHECK && __builtin_expect(__any(top >= 0x7ff00000u), 0)) {
        __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): what this wavefront stored is in place
        typedef const SplitArgs __attribute__((address_space(1)))* ArgsPtr;
        ArgsPtr q = (ArgsPtr)(size_t)__builtin_amdgcn_kernarg_segment_ptr();
        int lid = threadIdx.x;
        asm volatile("" : "+v"(q), "+v"(lid));
        const SplitArgs& pa = *(const SplitArgs*)q;
        const int lrow = (lid >> 7) * 32 + ((lid >> 5) & 1) * 4, lcol = ((lid >> 6) & 1) * 64 + (lid & 31);
        unsigned mt, nt, zt;
        for (unsigned tt = next_tile(PARTIAL ? wg % p.ntiles : wg, mt, nt, zt); tt < p.ntiles;
             tt = WALK ? next_tile(tt + nwg, mt, nt, zt) : p.ntiles) {
#pragma unroll 1
            for (int e = 0; e < 32; ++e) {
                const long row = (long)mt + lrow + 8 * ((e & 15) >> 2) + (e & 3), col = (long)nt + lcol + (e >> 4) * 32;
                if (row >= pa.M || col >= pa.N) continue;
                if (PARTIAL) {
                    double* at = pa.partial + ((part * nbatch + zt) * pa.M + row) * pa.N + col;
                    if (!(fabs(*at) < (double)INFINITY)) store_sum<SHARED>(at, sum_in_binary64<AREG, CONV>(pa, row, col, zt, g0, ngroup));
                } else {
                    float* at = pa.tau + (long)zt * pa.strideT + row * pa.ldt + col;
                    if (fabsf(*at) < INFINITY) continue;
                    const double ab = pa.bias ? fabs((double)pa.bias[col]) : 0.0;
                    const double s = sum_in_binary64<AREG, CONV>(pa, row, col, zt, g0, ngroup);
                    *at = up32(bound_of_sum(pa, s, bound_offset(pa, pa.si, ab), bound_offset(pa, pa.si0, ab)));
                }
            }
        }
    }
    if (CHECK) flush_counters(p, acc);
    return true;
}

template <bool CHECK, bool PARTIAL = false, bool WALK = false, bool AREG = false, bool CONV = false>
__global__ __launch_bounds__(kSplitThreads) void absgemm_split(SplitArgs p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ unsigned int chk_hist[CHECK ? kBins * 2 : 1];
    absgemm_split_slot<CHECK, PARTIAL, WALK, AREG, CONV>(p, blockIdx.x, gridDim.x, lds, chk_hist);
}

// ---- behind a screen (linear_screen.hip) -------------------------------------------------------
// One launch that settles the check.  Its first workgroups form the profile of the screen's partial results; where no comparison is open
// nothing else happens.  The tiles with open ones are taken one by one: places that the real sum decides are done with it, for the others the
// bound is formed by the code above.  What is found there are violations alone; the workgroup that finishes the last such tile (counted in the
// workspace; nobody waits) adds them up.
struct SettleArgs {
    CheckWorkspace check;
    OpenRecords open;
    ProfileSize size;
    tao_profile* out;
};
__device__ __forceinline__ size_t open_index(const SplitArgs& p, unsigned m0, unsigned n0, unsigned z) {
    static_assert(STILE == kOpenTile, "a record per tile");
    return ((size_t)z * p.tiles_m + m0 / STILE) * p.tiles_n + n0 / STILE;
}
// How many tiles have open comparisons; the profile but for what their violations change.
__device__ __forceinline__ unsigned screened_profile(const SettleArgs& r, char* lds) {
    const BlockStats& mine = r.check.stats[threadIdx.x & (kWave - 1)];
    if (blockIdx.x >= (unsigned)kGroups) return wave_sum(mine.flag);
    ProfileGroup<kSplitThreads, kScreenSlots> group(r.check, kScreenSlots, blockIdx.x);      // (on its way before the counts are known)
    const unsigned tiles = wave_sum(mine.flag);
    group.finish(r.size, r.out, reinterpret_cast<unsigned long long*>(lds), tiles == 0);
    if (tiles) __syncthreads();                              // (its sums have been read)
    return tiles;
}
// What workgroups exchange within a launch goes past the XCDs' caches (atomics and write-through stores of agent scope), so a count that
// follows its completion publishes it; a release fence would write back an L2 for every workgroup (100 us of them at 256).
__device__ __forceinline__ unsigned publish(unsigned int* count, unsigned add, unsigned int& word) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0): this wavefront's are complete
    __syncthreads();
    if (threadIdx.x == 0) word = __hip_atomic_fetch_add(count, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
    __syncthreads();
    return word;
}
// Counts `done` more tiles, whose violations this workgroup has added; the workgroup that completes the count adds all of them up.
__device__ __forceinline__ void tiles_done(const SettleArgs& r, unsigned tiles, unsigned done, unsigned int& word) {
    if (publish(&r.check.stats[kDoneFlag].flag, done, word) != tiles) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (threadIdx.x < kWave) {
        const unsigned long long v = wave_sum(__hip_atomic_load(&r.check.stats[threadIdx.x].violations, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (threadIdx.x == 0) { r.out->violations = v; r.out->accept = v == 0 ? 1u : 0u; }
    }
}
// A comparison by the real sum of its products, by a wavefront: 0 or 1 violations, or -1 where the sum does not decide.  The sum of
// binary64 products is exact but for 2^-40 of it; the one that the bound is formed of lies within 11.4u below and 3.3u above (and 8u more
// where operands below 2^-110 were raised), so the bound lies between those of the sum's limits 2^-20 off, as both are formed alike.
template <bool AREG, bool CONV>
__device__ __forceinline__ int decide_by_sum(const SplitArgs& p, unsigned row, unsigned col, unsigned z) {
    const OutputOperands<AREG, CONV> operands(p, row, col, z);
    const int units = (int)(p.Kp / 8), lane = threadIdx.x & 63;
    double s = 0.0;
    for (int u = lane; u < units; u += kWave) s = operands.add(p, u >> 2, u & 3, s);
    s = wave_sum(s);
    if (!(s >= (double)p.Kp * 0x1p-80 && s <= 0x1p120)) return -1;
    const double ab = p.bias ? fabs((double)p.bias[col]) : 0.0, off = bound_offset(p, p.si, ab);
    const long at = (long)z * p.strideY + (long)row * p.ldy + col;
    const double d = fabs((double)p.claimed[at] - (double)p.ref[at]);
    if (d <= p.alpha * (double)up32(bound_of_sum(p, s * (1.0 - 0x1p-20), off, off))) return 0;
    if (!(d <= p.alpha * (double)up32(bound_of_sum(p, s * (1.0 + 0x1p-20), off, off)))) return 1;
    return -1;
}
// The open comparisons of a tile: `todo` receives those that take the bound itself, counts[0] the violations among the others.
// Returns whether any are left.
struct OpenLds { unsigned int todo[STILE * STILE / 32], counts[2], word; };
template <bool AREG, bool CONV>
__device__ __forceinline__ bool sift_open(const SplitArgs& p, const OpenRecords& open, const unsigned* rec, unsigned state, unsigned m0, unsigned n0, unsigned z, OpenLds& o) {
    static_assert(STILE * STILE / 32 == kSplitThreads, "a word a thread");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned blocks = state & 0xffffu;
    __syncthreads();                                         // (the tile before has read its words)
    o.todo[tid] = blocks >> ((tid >> 7) * 4 + (tid & 3)) & 1u ? ~0u : 0u;
    if (tid == 0) { o.counts[0] = 0; o.counts[1] = blocks; }
    __syncthreads();
    const int n = min((int)(state >> 16), open.places());
    if (n == 0) return true;
    for (int e = wave; e < n; e += kSplitThreads / kWave) {
        const unsigned at = rec[2 + e];
        if (at == kNoPlace) continue;
        // (with whole blocks the bound is formed in any case)
        const int v = blocks ? -1 : decide_by_sum<AREG, CONV>(p, m0 + (at >> 7), n0 + (at & 127u), z);
        if (lane == 0 && v > 0) atomicAdd(&o.counts[0], 1u);
        if (lane == 0 && v < 0) { atomicOr(&o.todo[at >> 5], 1u << (at & 31u)); o.counts[1] = 1; }
    }
    __syncthreads();
    return o.counts[1] != 0;
}
__device__ __forceinline__ void add_violations(const SplitArgs& p, unsigned n) {
    if (threadIdx.x == 0 && n) atomicAdd(&p.ws_stats[blockIdx.x % p.check_slots].violations, (unsigned long long)n);
}
// On images a workgroup per compute unit walks the slots (where nothing is open, thousands would only be given LDS and leave); the
// in-load forms have no registers for that (39 spilled instead of 12) and take a workgroup per slot.
template <bool AREG, bool CONV>
__global__ __launch_bounds__(kSplitThreads) void absgemm_settle(SplitArgs p, SettleArgs r) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ OpenLds o;
    const unsigned tiles = screened_profile(r, lds);
    if (tiles == 0) return;
    unsigned done = 0, m0, n0, z;
    if (AREG) {
        if (blockIdx.x >= p.ntiles || !locate_tile(p, blockIdx.x, m0, n0, z)) return;
        const unsigned* rec = r.open.of(open_index(p, m0, n0, z));
        const unsigned state = rec[0];
        if (state == 0) return;
        if (sift_open<AREG, CONV>(p, r.open, rec, state, m0, n0, z, o)) absgemm_split_slot<true, false, false, AREG, CONV, false, true>(p, blockIdx.x, gridDim.x, lds, o.todo);
        add_violations(p, o.counts[0]);
        done = 1;
    } else {
        // (64 slots' records at a time, one a lane; all wavefronts see the same)
        for (unsigned first = blockIdx.x; first < p.ntiles; first += gridDim.x * kWave) {
            const unsigned slot = first + (threadIdx.x & 63) * gridDim.x;
            const unsigned states = slot < p.ntiles && locate_tile(p, slot, m0, n0, z) ? r.open.of(open_index(p, m0, n0, z))[0] : 0u;
            for (unsigned long long left = __ballot(states != 0); left; left &= left - 1) {
                // (the arguments are read anew for each tile: kept in registers through it they cost the loop of the product some)
                typedef const SplitArgs __attribute__((address_space(4)))* ArgsPtr;
                ArgsPtr q = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
                asm volatile("" : "+s"(q));
                const SplitArgs& a = *(const SplitArgs*)q;
                const int at = __ffsll(left) - 1;
                const unsigned wg = first + (unsigned)at * gridDim.x, state = (unsigned)__builtin_amdgcn_readlane((int)states, at);
                locate_tile(a, wg, m0, n0, z);
                if (sift_open<AREG, CONV>(a, r.open, r.open.of(open_index(a, m0, n0, z)), state, m0, n0, z, o)) {
                    absgemm_split_slot<true, false, false, AREG, CONV, false, true>(a, wg, gridDim.x, lds, o.todo);
                    __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): nothing of it counts in the next tile's waits
                }
                add_violations(a, o.counts[0]);
                ++done;
            }
        }
    }
    if (done) tiles_done(r, tiles, done, o.word);
}
// The reduction in parts: every workgroup of an open tile sifts its places (all come to the same), leaves its part's sums in the workspace if any
// are left, and the one that brings the tile's last part adds them in split_combine's order and compares.
template <bool AREG>
__global__ __launch_bounds__(kSplitThreads) void absgemm_settle_parts(SplitArgs p, SettleArgs r) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ OpenLds o;
    const unsigned tiles = screened_profile(r, lds);
    if (tiles == 0 || blockIdx.x >= p.ntiles * (unsigned)p.ksplit) return;
    unsigned m0, n0, z;
    const unsigned slot = blockIdx.x % p.ntiles;
    if (!locate_tile(p, slot, m0, n0, z)) return;
    unsigned* rec = r.open.of(open_index(p, m0, n0, z));     // (so few tiles have whole records)
    const unsigned state = rec[0];
    if (state == 0) return;
    ThreadAcc acc;
    if (sift_open<AREG, false>(p, r.open, rec, state, m0, n0, z, o)) {
        absgemm_split_slot<false, true, false, AREG, false, true>(p, blockIdx.x, gridDim.x, lds, nullptr);
        if (publish(rec + 1, 1u, o.word) != (unsigned)p.ksplit) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const long per = p.M * p.N, total = per * (long)(p.ntiles / p.slots_per_z);
        // a thread has a column of every fourth row, eight of them at a time: the loads' latency is what the loop waits for
        constexpr int BATCH = 8, RSTEP = kSplitThreads / STILE;
        const int lcol = threadIdx.x & (STILE - 1), lrow = threadIdx.x / STILE;
        const long col = (long)n0 + lcol;
        const double ab = p.bias && col < p.N ? fabs((double)p.bias[col]) : 0.0;
        const double off_pos = bound_offset(p, p.si, ab), off_zero = bound_offset(p, p.si0, ab);
#pragma unroll 1
        for (int i0 = 0; i0 < STILE / RSTEP; i0 += BATCH) {
            double sv[BATCH];
            float c[BATCH], rf[BATCH];
            long at[BATCH];
            unsigned asked = 0;
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int row = lrow + (i0 + i) * RSTEP;
                if (m0 + row < p.M && col < p.N) asked |= (o.todo[row * (STILE / 32) + (lcol >> 5)] >> (lcol & 31) & 1u) << i;
            }
            if (!asked) continue;
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const long row = min((long)m0 + lrow + (i0 + i) * RSTEP, p.M - 1), y = (long)z * p.strideY + row * p.ldy + col;
                at[i] = (long)z * per + row * p.N + col;
                sv[i] = 0.0; c[i] = p.claimed[y]; rf[i] = p.ref[y];
            }
            for (int k = 0; k < p.ksplit; ++k)
#pragma unroll
                for (int i = 0; i < BATCH; ++i) sv[i] += p.partial[(long)k * total + at[i]];
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const float t32 = up32(bound_of_sum(p, sv[i], off_pos, off_zero));
                acc.violations += (asked >> i & 1u) && !(fabs((double)c[i] - (double)rf[i]) <= p.alpha * (double)t32);
            }
        }
        flush_counters(p, acc);
    } else if (blockIdx.x >= p.ntiles) {
        return;                                              // (a tile that needs no sums is its first part's)
    }
    add_violations(p, o.counts[0]);
    tiles_done(r, tiles, 1u, o.word);
}

// Adds the parts of a PARTIAL launch in a fixed order and forms the bound exactly as the epilogue
// above does; CHECK: checks it on the spot, in the structure of the streaming check pass.
template <bool CHECK>
__global__ __launch_bounds__(kCheckThreads) void split_combine(SplitArgs p, long batch) {
    __shared__ unsigned int hist[CHECK ? kBins * kReplicas : 1];
    __shared__ unsigned int red[CHECK ? 3 * (kCheckThreads / kWave) : 1];
    if (CHECK) {
        for (int i = threadIdx.x; i < kBins * kReplicas; i += kCheckThreads) hist[i] = 0;
        __syncthreads();
    }
    ThreadAcc acc;
    const int rep = threadIdx.x & (kReplicas - 1);
    const long per = p.M * p.N, total = per * batch;
    // (total < 2^32: a reduction is cut into parts only where the tiles are fewer than the compute units;
    // 64-bit divisions would cost an order of magnitude more)
    for (long i = (long)blockIdx.x * kCheckThreads + threadIdx.x; i < total; i += (long)gridDim.x * kCheckThreads) {
        const unsigned ui = (unsigned)i, uz = ui / (unsigned)per, rc = ui - uz * (unsigned)per, ur = rc / (unsigned)p.N;
        const long z = uz, row = ur, col = rc - ur * (unsigned)p.N;
        double sv = 0.0;
        for (int k = 0; k < p.ksplit; ++k) sv += p.partial[(long)k * total + i];
        const double ab = p.bias ? fabs((double)p.bias[col]) : 0.0;
        const float t32 = up32(bound_of_sum(p, sv, bound_offset(p, p.si, ab), bound_offset(p, p.si0, ab)));
        if (p.tau) p.tau[z * p.strideT + row * p.ldt + col] = t32;
        if (CHECK) {
            const long y = z * p.strideY + row * p.ldy + col;
            check_one(p.claimed[y], p.ref[y], t32, p.alpha, p.eps_rel, hist, rep, acc);
        }
    }
    if (CHECK) {
        flush_block_stats(acc, red, p.ws_stats);
        flush_histogram(hist, p.ws_hist + (size_t)blockIdx.x * kBins, p.ws_coarse + blockIdx.x * kGroups);
    }
}

__global__ __launch_bounds__(256) void clear_check(ClearJob c) { clear_words(c, (long)blockIdx.x * 256 + threadIdx.x, (long)gridDim.x * 256); }
static void launch_clear(const ClearJob& c, hipStream_t st) {
    hipLaunchKernelGGL(clear_check, dim3((unsigned)std::max(1L, (c.words[0] + 511) / 512)), dim3(256), 0, st, c);
}

// ---- instruction self test ------------------------------------------------------------------
// One wavefront per case: every row of A holds a[0..15], every column of B holds b[0..15], every
// accumulator element c; all outputs are then the same number.
struct Bf16Case { unsigned short a[16], b[16]; float c; };
__global__ __launch_bounds__(256) void bf16_mfma_probe(const Bf16Case* __restrict__ cs, float* __restrict__ d, int n) {
    const int w = blockIdx.x * 4 + threadIdx.x / 64;
    if (w >= n) return;
    const int lane = threadIdx.x % 64, g = lane / 32;
    typedef short shortx8 __attribute__((ext_vector_type(8)));
    shortx8 sa, sb;
    for (int e = 0; e < 8; ++e) { sa[e] = (short)cs[w].a[8 * g + e]; sb[e] = (short)cs[w].b[8 * g + e]; }
    floatx16 acc;
    for (int v = 0; v < 16; ++v) acc[v] = cs[w].c;
    acc = TAO_MFMA_BF16(__builtin_bit_cast(bf16x8, sa), __builtin_bit_cast(bf16x8, sb), acc);
    if (lane == 37) d[w] = acc[9];
}

// Host model of the instruction for non-negative normal operands, in exact integer arithmetic:
// values are integers in units of 2^-kScale.
typedef unsigned __int128 u128;
constexpr int kScale = 72;
static int top_bit(u128 v) { int b = -1; while (v) { v >>= 1; ++b; } return b; }
static u128 chop(u128 v, int e) {                  // clear everything below 2^e
    const int sh = e + kScale;
    return sh <= 0 ? v : (sh >= 128 ? (u128)0 : (v >> sh) << sh);
}
static u128 round24(u128 v) {                      // to 24 significant bits, ties to even
    const int tb = top_bit(v);
    if (tb < 24) return v;
    const int sh = tb - 23;
    u128 q = v >> sh;
    const u128 rem = v & (((u128)1 << sh) - 1), half = (u128)1 << (sh - 1);
    if (rem > half || (rem == half && (q & 1))) ++q;
    return q << sh;
}
static u128 model_step(u128 acc, const u128* prod, const int* pexp) {
    int eP = -100000;
    for (int k = 0; k < 8; ++k) if (prod[k] != 0 && pexp[k] > eP) eP = pexp[k];
    if (eP == -100000) return acc;
    u128 P = 0;
    for (int k = 0; k < 8; ++k) P += chop(prod[k], eP - 24);
    if (acc == 0) return round24(P);
    const int ce = top_bit(acc) - kScale;
    if (ce - eP >= 28) return acc;
    const int e = ce > eP ? ce : eP;
    return round24(chop(acc, e - 24) + chop(P, e - 31));
}

}  // namespace tao

extern "C" {

size_t tao_selftest_workspace_bytes(long cases) {
    if (cases <= 0) cases = 3072;
    const size_t bf16 = (size_t)cases * (sizeof(tao::Bf16Case) + sizeof(float)) + 256;
    return bf16 < 8192 ? 8192 : bf16;       // (the FP32 self test needs 5.6 KB)
}

int tao_selftest_matrix_core_bf16(unsigned* report, long cases, void* ws, size_t ws_bytes, void* stream) {
    using namespace tao;
    if (!report) return TAO_ERR_NULL;
    if (cases < 0 || cases > (1L << 24)) return TAO_ERR_SHAPE;
    if (cases == 0) cases = 3072;
    if (!ws || !aligned(ws, 256) || ws_bytes < tao_selftest_workspace_bytes(cases)) return TAO_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const int kCases = (int)cases;
    std::vector<Bf16Case> hc(kCases);
    std::vector<float> hd(kCases);
    unsigned long long lcg = 0x2545F4914F6CDD1Dull;
    auto rnd = [&]() { lcg = lcg * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(lcg >> 33); };
    auto bf = [](int e, unsigned man7) { return (unsigned short)(((127 + e) << 7) | (man7 & 127u)); };
    auto f32 = [](int e, unsigned man23) { const unsigned u = ((unsigned)(127 + e) << 23) | (man23 & 0x7fffffu); float f; memcpy(&f, &u, 4); return f; };
    // four seeded families of non-negative operands: narrow exponents; wide exponents; products far
    // below an accumulator of the order of 1; products and sums in the binary32 subnormal range; and a fifth
    // of signed operands over the exponents of the second (the cross products)
    for (int i = 0; i < kCases; ++i) {
        Bf16Case& c = hc[i];
        const int fam = i % 5;
        const int shift = 20 + (int)(rnd() % 10);
        for (int k = 0; k < 16; ++k) {
            if (fam == 0)      { c.a[k] = bf((int)(rnd() % 3) - 1, rnd()); c.b[k] = bf((int)(rnd() % 3) - 1, rnd()); }     // narrow
            else if (fam == 1) { c.a[k] = bf((int)(rnd() % 25) - 12, rnd()); c.b[k] = bf((int)(rnd() % 25) - 12, rnd()); } // wide
            else if (fam == 2) { c.a[k] = bf(-(shift / 2) + (int)(rnd() % 3) - 1, rnd()); c.b[k] = bf(-(shift - shift / 2), rnd()); }  // far below c
            else if (fam == 3) { c.a[k] = bf(-75 + (int)(rnd() % 11), rnd()); c.b[k] = bf(-75 + (int)(rnd() % 11), rnd()); }           // 2^-150 .. 2^-128
            else {
                const int w = i % 2 ? 25 : 3;
                c.a[k] = bf((int)(rnd() % w) - w / 2, rnd()); c.b[k] = bf((int)(rnd() % w) - w / 2, rnd());
                c.b[k] |= (unsigned short)((rnd() & 1u) << 15);
            }
        }
        c.c = fam == 3 ? 0.f : fam == 2 ? f32(0, rnd()) : fam == 4 ? ((i & 2) ? -1.f : 1.f) * f32((int)(rnd() % 25) - 12, rnd()) : ((i & 1) ? f32((int)(rnd() % 25) - 12, rnd()) : 0.f);
    }
    Bf16Case* dc = static_cast<Bf16Case*>(ws);
    float* dd = reinterpret_cast<float*>(static_cast<char*>(ws) + ((size_t)kCases * sizeof(Bf16Case) + 255) / 256 * 256);
    auto fail = [&](hipError_t e) { g_last_hip_error = (int)e; return TAO_ERR_LAUNCH; };
    hipError_t e;
    if ((e = hipMemcpyAsync(dc, hc.data(), (size_t)kCases * sizeof(Bf16Case), hipMemcpyHostToDevice, st)) != hipSuccess) return fail(e);
    hipLaunchKernelGGL(bf16_mfma_probe, dim3((kCases + 3) / 4), dim3(256), 0, st, dc, dd, kCases);
    if ((e = hipGetLastError()) != hipSuccess) return fail(e);
    if ((e = hipMemcpyAsync(hd.data(), dd, (size_t)kCases * sizeof(float), hipMemcpyDeviceToHost, st)) != hipSuccess) return fail(e);
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return fail(e);

    auto to_int = [](float f) -> u128 {                       // positive normal binary32 -> units of 2^-kScale
        unsigned u; memcpy(&u, &f, 4);
        if (f == 0.f) return 0;
        const int ex = (int)((u >> 23) & 255) - 127;
        const u128 m = (u & 0x7fffffu) | 0x800000u;
        const int sh = kScale + ex - 23;
        return sh >= 0 ? m << sh : m >> -sh;                  // (what cancellation leaves: low bits zero)
    };
    bool exact = true, within = true, tiny = true;
    for (int i = 0; i < kCases; ++i) {
        const Bf16Case& c = hc[i];
        if (i % 5 == 3) {
            // subnormal range: the exact sum (16 products of 16 bits within 22 binades: exact in
            // binary64) against the result, in steps of 2^-149
            double sum = 0.0;
            for (int k = 0; k < 16; ++k) {
                const int ea = (int)((c.a[k] >> 7) & 255) - 127, eb = (int)((c.b[k] >> 7) & 255) - 127;
                sum += std::ldexp((double)(((c.a[k] & 127u) | 128u) * ((c.b[k] & 127u) | 128u)), ea + eb - 14);
            }
            if (!(std::fabs((double)hd[i] - sum) <= 2.0 * 0x1p-149)) tiny = false;
            continue;
        }
        if (i % 5 == 4) {
            // signed operands: within 2 x 2.01u + 7u < 11.25u of the sum of all magnitudes
            __int128 sum = c.c < 0.f ? -(__int128)to_int(-c.c) : (__int128)to_int(c.c);
            u128 mag = to_int(std::fabs(c.c));
            for (int k = 0; k < 16; ++k) {
                const int ea = (int)((c.a[k] >> 7) & 255) - 127, eb = (int)((c.b[k] >> 7) & 255) - 127;
                const u128 v = (u128)(((c.a[k] & 127u) | 128u) * ((c.b[k] & 127u) | 128u)) << (kScale + ea + eb - 14);
                sum += (c.b[k] & 0x8000u) ? -(__int128)v : (__int128)v;
                mag += v;
            }
            const __int128 got = hd[i] < 0.f ? -(__int128)to_int(-hd[i]) : (__int128)to_int(hd[i]);
            const __int128 off = got > sum ? got - sum : sum - got;
            if (!((u128)off <= (mag >> 26) * 45u)) within = false;
            continue;
        }
        u128 prod[16]; int pexp[16];
        u128 sum = to_int(c.c);
        for (int k = 0; k < 16; ++k) {
            const int ea = (int)((c.a[k] >> 7) & 255) - 127, eb = (int)((c.b[k] >> 7) & 255) - 127;
            const u128 ma = (c.a[k] & 127u) | 128u, mb = (c.b[k] & 127u) | 128u;
            prod[k] = (ma * mb) << (kScale + ea + eb - 14);
            pexp[k] = ea + eb;
            sum += prod[k];
        }
        u128 acc = to_int(c.c);
        acc = model_step(acc, prod, pexp);
        acc = model_step(acc, prod + 8, pexp + 8);
        const u128 got = to_int(hd[i]);
        if (!(hd[i] > 0.f) || got != acc) exact = false;
        if (c.c == 0.f) {
            // [S (1 - 10u), S (1 + 2u)] with u = 2^-24, in integers: got * 2^24 against S * (2^24 -+ ...)
            const u128 lo = (sum >> 24) * ((1u << 24) - 10), hi = (sum >> 24) * ((1u << 24) + 2) + ((u128)1 << 30);
            if (got < lo || got > hi) within = false;
        }
    }
    *report = (exact ? 1u : 0u) | (within ? 2u : 0u) | (tiny ? 4u : 0u);
    return TAO_OK;
}

}  // extern "C"

namespace tao {
inline size_t round_up_256(size_t b) { return (b + 255) / 256 * 256; }
// Parts the reduction is cut into: launches with fewer 128 x 128 tiles than compute units take as
// many parts as fill the chip, each at least kMinGroupsPerPart groups long.
static int split_k_parts(long M, long N, long K, long batch) {
    if (M <= 0 || N <= 0 || K <= 0 || batch <= 0) return 1;
    const long tiles = ((M + STILE - 1) / STILE) * ((N + STILE - 1) / STILE) * batch;
    const long groups = (K + SBK - 1) / SBK;
    const long cus = device_cus();
    if (tiles >= cus) return 1;
    long parts = cus / tiles;
    if (parts > groups / kMinGroupsPerPart) parts = groups / kMinGroupsPerPart;
    if (parts > 16) parts = 16;
    return parts < 2 ? 1 : (int)parts;
}
}  // namespace tao

namespace tao {
// ---- workspace layout -------------------------------------------------------------------------
// An operand image: per 32 k-steps and 128-row block the LDS image of the three pieces (kBlock bytes),
// batch entries one after the other; at the end 512 bytes of marks (kMarks).
static size_t image_bytes(long rows, long K, long batch) {
    if (rows <= 0 || K <= 0 || batch <= 0) return 0;
    const long Kp = (K + SBK - 1) / SBK * SBK;
    const __int128 blocks = (__int128)(Kp / SBK) * ((rows + STILE - 1) / STILE) * batch;
    if (blocks * kBlock + 512 >= ((__int128)1 << 62)) return 0;
    return round_up_256((size_t)(blocks * kBlock) + kMarks);
}
static unsigned char* image_marks(const void* image, long rows, long K, long batch) {
    return static_cast<unsigned char*>(const_cast<void*>(image)) + (size_t)((K + SBK - 1) / SBK) * (size_t)((rows + STILE - 1) / STILE) * (size_t)batch * kBlock;
}
// What the product itself needs beyond the images: the binary64 partial sums of a reduction cut into
// parts and, with a check, the check's partial results and (short reductions) the stored bound.
static size_t core_workspace_bytes(long M, long N, long K, long batch, bool check) {
    if (M <= 0 || N <= 0 || batch <= 0) return check ? round_up_256(check_workspace_bytes()) : 0;
    const int parts = split_k_parts(M, N, K, batch);
    size_t b = parts >= 2 ? round_up_256((size_t)parts * (size_t)batch * (size_t)M * (size_t)N * sizeof(double)) : 0;
    if (check) {
        b += round_up_256(check_workspace_bytes());
        if (K < kEpilogueCheckMinK) b += round_up_256((size_t)M * N * batch * 4);
    }
    return b;
}
// The records of what a screen leaves open, within that, and what the launch before the screen clears.
static OpenRecords core_open_records(const CheckWorkspace& cw, long M, long N, long K, long batch) {
    const size_t bound = K < kEpilogueCheckMinK ? round_up_256((size_t)M * N * batch * 4) : 0;
    return open_records(cw, open_tiles_of(M, N, batch), reinterpret_cast<char*>(cw.hist) + round_up_256(check_workspace_bytes()), bound);
}
static ClearJob screen_clear(const CheckWorkspace& cw, long M, long N, long K, long batch) {
    return clear_job(cw, kScreenSlots, core_open_records(cw, M, N, K, batch), open_tiles_of(M, N, batch));
}
}  // namespace tao

extern "C" {

size_t tao_split_image_bytes(long rows, long K, long batch) { return tao::image_bytes(rows, K, batch); }

size_t tao_linear_split_workspace_bytes(long M, long N, long K, long batch, int shared_w) {
    if (M <= 0 || N <= 0 || K < 0 || batch <= 0) return 0;
    if (K == 0) return 0;
    const size_t a = tao::image_bytes(M, K, batch), w = tao::image_bytes(N, K, shared_w ? 1 : batch);
    if (a == 0 || w == 0) return 0;
    return a + w + tao::core_workspace_bytes(M, N, K, batch, false);
}

size_t tao_linear_images_workspace_bytes(long M, long N, long K, long batch) {
    return tao::core_workspace_bytes(M, N, K, batch, false);
}
size_t tao_check_linear_images_workspace_bytes(long M, long N, long K, long batch) {
    return tao::core_workspace_bytes(M, N, K, batch, true);
}

int tao_linear_split_preferred(long M, long N, long K, long batch) {
    // The BF16 path has one tile shape (128 x 128) and pays a pre-pass of 10 bytes per operand
    // element: it wins when the tiles fill the chip and each operand slab is shared by at least
    // two of them.  Launches with fewer tiles than compute units cut the reduction into parts; they count when the
    // parts fill the chip.
    if (M <= 0 || N <= 0 || K <= 0 || batch <= 0) return 0;
    const long tiles = ((M + tao::STILE - 1) / tao::STILE) * ((N + tao::STILE - 1) / tao::STILE) * batch;
    // (a single column tile pays when its A operand can be split while it is loaded: a long reduction of whole groups)
    // (even half a column tile counts where the tiles are so few that the reduction is cut into four parts or more; with 128
    // tiles in two parts -- 8 x 2048 x 128 over K = 2048 -- the pre-pass over A outweighs the gain: 0.137 against 0.111 ms)
    const bool n_ok = N >= 2 * tao::STILE || (N >= tao::STILE && K % tao::SBK == 0 && K / tao::SBK > tao::kWalkMaxGroups &&
                                              tao::split_k_parts(M, N, K, batch) < 2) ||
                      (N >= tao::STILE / 2 && tao::split_k_parts(M, N, K, batch) >= 4);
    // (a long reduction cut into parts also pays on half the chip: 512 x 768 x 3072 0.045 against 0.057 ms)
    const long parts = tao::split_k_parts(M, N, K, batch), cus = tao::device_cus();
    const bool fills = tiles * parts >= cus || (parts >= 2 && tiles * parts * 2 >= cus);
    if (!(fills && M >= 2 * tao::STILE && n_ok && K >= 64)) return 0;
    // What is left is small enough in places for the binary64 matrix cores of tao_bound_linear, which need no pre-pass and no parts
    // (us, BF16 path / tao_bound_linear: 12 x 512 x 64 over K = 512 28 / 17, 1024 x 512 over 512 29 / 18, 256 x 1024 over 1024
    // 30 / 15, 4 x 1024 x 64 over 1024 35 / 15; 512 x 3072 over 768 42 / 42, 1024 x 1024 over 1024 38 / 55).  Estimate of the BF16
    // path, fitted to 51 shapes: launches, operand images, groups of the walk, partial sums.  The line lies below equal times,
    // as the checked entry points save a launch and the bound's traffic on this path: 512 x 768 over 768 takes 28 / 21, with
    // the check 35 / 31 (this path kept), 512 x 512 over 4096 45 / 44, with the check 53 / 54.
    const double groups = (double)((K + tao::SBK - 1) / tao::SBK), elements = ((double)M + (double)N) * (double)K * (double)batch;
    const double rounds = std::ceil((double)(tiles * parts) / (double)cus);
    const double split_us = 14.0 + 1.47e-6 * elements + 1.56 * rounds * std::ceil(groups / (double)parts) +
                            (parts >= 2 ? 2.0 + 1.84e-6 * (double)parts * (double)M * (double)N * (double)batch : 0.0);
    return tao::linear_us(M, N, K, batch, (int)cus) >= 0.66 * split_us;
}

}  // extern "C"

namespace tao {
// The fused check: NULL for the plain bound.
struct SplitCheckHost {
    const float* claimed; const float* ref; long ldy, strideY; double alpha, eps_rel; tao_profile* out;
};

// What 256 threads of split3_bf16 take at a time.
static long split_blocks(const SplitOperand& p) {
    const long units = (p.K + SBK - 1) / SBK * ((p.rows + 63) / 64) * p.batch;
    return p.form == MAGNITUDES ? (p.K / 8 + 4 + 255) / 256 : p.flat() ? (units + 3) / 4 : units;
}
// Launches split3_bf16 for one or two operands: src [batch][rows][K] with row stride ld (STRAIGHT) or
// [batch][K][rows] (TRANSPOSED) -> image.  clear: the side job described at the kernel.
// A workgroup that leaves a mark: as many as there are marks, two to a compute unit, of as many parts of 256 threads as give every unit one, up to four.
// Dealt out to the workgroups' first parts, then to their second ones, the last units find all compute units (us on the device; a quarter of the
// workgroups, of 1024 threads, as soon as the marks were too few / so / without marks: 1111 x 1001, 576 units, 5.5 / 4.9 / 4.5, 3072 x 768 7.3 / 6.0 / 5.7,
// 1500 x 1500 7.4 / 6.3 / 6.0).  A walk of several rounds keeps neighbouring units together (12288 x 4096 104, dealt out 112; 2048 x 4096, cold, 16.0 and 18.7).
static void launch_split3(const SplitOperand* ops, int n, const ClearJob& clear, hipStream_t st) {
    SplitOperands a = {};
    a.clear = clear;
    const bool marked = ops[0].nmarks > 0;
    long parts = 1, first = 0;
    for (int o = 0; o < n && marked; ++o) parts = std::max(parts, (split_blocks(ops[o]) + ops[o].nmarks - 1) / ops[o].nmarks);
    parts = std::min(parts, (long)kMostSplitThreads / 256);
    for (int o = 0; o < n; ++o) {
        const long blocks = split_blocks(ops[o]), most = marked ? ops[o].nmarks : 256L * 64;
        // (an operand beside a longer one leaves no part of its workgroups idle, whose places that one could have: 1892 x 2560 beside 576 x 2560 13.6 -> 12.0 us)
        const long wgs = std::clamp((blocks + most - 1) / most < parts ? (blocks + parts - 1) / parts : blocks, 1L, most);
        a.op[o] = ops[o];
        a.op[o].spread = blocks <= wgs * parts;
        a.first[o] = first;
        first += wgs;
    }
    for (int o = n; o < 3; ++o) a.first[o] = first;
    if (marked) hipLaunchKernelGGL(split3_bf16<true>, dim3((unsigned)first), dim3((unsigned)parts * 256), 0, st, a);
    else        hipLaunchKernelGGL(split3_bf16<false>, dim3((unsigned)first), dim3(256), 0, st, a);
}

// The product on prepared images.  ws: what core_workspace_bytes(M, N, K, batch, chk != NULL) asks for.
// cleared: the check's partial results in ws are zero already (the caller's pre-pass cleared them).
// tau / ldt / strideT: the caller's layout (validated by the caller); with a check they describe y_ref and
// claimed as well when tau is stored.
// Af != NULL: the A operand is split while it is loaded (AREG instantiations; the caller has
// checked in_load_split_ok); A3 is then unused.
// screened: a screen has been enqueued with this workspace; one launch here settles the check.
struct ConvHost { int H, W, C, OW, S, sh, sw, ph, pw, dh, dw; unsigned ohow; };
// cv != NULL (with Af): Af is a convolution's channels-last input and A its implicit patch matrix.
static int split_core(const unsigned short* A3, const unsigned short* W3, const float* bias, float* tau,
                      long M, long N, long K, long ldt, long batch, long strideT, bool shared_w,
                      const tao_fp_model& md, void* ws, void* stream, const SplitCheckHost* chk, bool cleared,
                      const float* Af = nullptr, long lda = 0, long strideA = 0, const ConvHost* cv = nullptr,
                      bool screened = false) {
    const long Kp_ = K + (bias ? 1 : 0);
    const double c = gamma_up(Kp_, md);
    if (!(c == c)) return TAO_ERR_K_RANGE;
    hipStream_t st = (hipStream_t)stream;
    const int parts = split_k_parts(M, N, K, batch);
    char* wsb = static_cast<char*>(ws);
    const size_t partial_bytes = parts >= 2 ? round_up_256((size_t)parts * (size_t)batch * (size_t)M * (size_t)N * sizeof(double)) : 0;
    CheckWorkspace cw = {};
    bool two_pass = false;
    void* check_ws = nullptr;
    if (chk) {
        check_ws = wsb + partial_bytes;
        cw = carve_check_workspace(check_ws);
        // Short reductions: in the epilogue the check is arithmetic that nothing overlaps (about 70
        // instructions per element on a compute unit whose matrix cores idle meanwhile), while the
        // streaming check spends the same arithmetic under its loads and the plain bound walks its
        // tiles.  Up to K = 1024 the bound is therefore stored (in the workspace unless the caller
        // wants it) and checked by that pass: the same results, field for field, 5 - 9 % sooner at K = 128 ... 512
        // (8 x 8192 x 2048 over 128 608 against 666 us) and the same within 2 % at 1024 (2048 x 12288 410 / 419, 4096 x 4096 277 / 274);
        // beyond, the two routes take the same time (2048 x 12288 over 2048 747 / 745, over 4096 1422 / 1416) and the epilogue
        // saves the memory of the stored bound.
        // (A reduction cut into parts is checked by the pass that adds the parts, whatever its length.)
        two_pass = !screened && parts < 2 && K < kEpilogueCheckMinK && !(md.flags & TAO_FLAG_CHECK_IN_EPILOGUE) &&
                   chk->ldy == N && (batch == 1 || chk->strideY == M * N);
        if (two_pass && !tau) {
            tau = reinterpret_cast<float*>(static_cast<char*>(check_ws) + round_up_256(check_workspace_bytes()));
            ldt = N; strideT = M * N;
        }
    }
    const long Kp = (K + SBK - 1) / SBK * SBK;
    const long tiles_n = (N + STILE - 1) / STILE, tiles_m = (M + STILE - 1) / STILE;
    const long ntiles = tiles_n * tiles_m * batch;
    if (ntiles >= (1L << 31)) return TAO_ERR_SHAPE;
    const long blocksA = (M + STILE - 1) / STILE, blocksW = (N + STILE - 1) / STILE;

    SplitArgs p;
    p.A3 = A3; p.W3 = W3; p.bias = bias; p.tau = tau;
    p.Af = Af; p.lda = lda; p.strideA = strideA;
    p.cH = p.cW = p.cC = p.cOW = p.cS = p.csh = p.csw = p.cph = p.cpw = p.cdh = p.cdw = 0; p.cohow = 1;
    if (cv) {
        p.cH = cv->H; p.cW = cv->W; p.cC = cv->C; p.cOW = cv->OW; p.cS = cv->S; p.csh = cv->sh; p.csw = cv->sw;
        p.cph = cv->ph; p.cpw = cv->pw; p.cdh = cv->dh; p.cdw = cv->dw; p.cohow = cv->ohow;
    }
    p.M = M; p.N = N; p.Kp = Kp; p.ldt = ldt; p.strideT = strideT;
    p.batchA3 = (Kp / SBK) * blocksA * (kBlock / 2); p.batchW3 = shared_w ? 0 : (Kp / SBK) * blocksW * (kBlock / 2);
    p.tiles_n = (unsigned)tiles_n; p.tiles_m = (unsigned)tiles_m;
    const double u = md.u;
    // lower factor of the accumulation: (1 - 11.4u) for the matrix-core steps and the dropped products (10.08u main,
    // 0.28u cross, 1.001u dropped), 2^-53 per binary64 addition (three per 32 k-steps and output element)
    const double f64 = (double)(3 * (Kp / SBK) + 4 + 16);             // + the additions of up to 16 parts
    const double lower = (1.0 - 11.4 * u) * (1.0 - f64 * 0x1p-53);
    const double infl = widen(1.0 / (lower * (1.0 - 0x1p-52)));
    p.uflow = (md.flags & TAO_FLAG_UNDERFLOW_TERMS) ? widen((double)Kp_ * 0x1p-149) : 0.0;
    // Results in the binary32 subnormal range: the instruction keeps subnormal operands, products
    // and sums (gradual underflow) and then errs absolutely, by less than one step of 2^-149 per
    // instruction (probed like the model above: 160 000 cases with products between 2^-160 and
    // 2^-120); two steps are budgeted for each of the 12 instructions an output element sees per
    // 32 k-steps, and some to spare.  Added to every sum but an exact zero (the signed cross products can leave a sum
    // this far below zero); to an exactly zero sum only when the caller asked for
    // underflow terms (otherwise such a sum is taken as the exact zero of zero operands).
    const double sabs = K > 0 ? ((double)Kp + 32.0) * 0x1p-149 : 0.0;
    // The folded constants; every product is rounded up with room for the two or three roundings of its
    // evaluation on the device, and the guard factor (2^-32) stays far above all of them.
    p.c1 = widen(c * infl * kGuard);
    p.cg = widen(c * kGuard);
    p.si = widen(sabs * infl);
    p.si0 = (md.flags & TAO_FLAG_UNDERFLOW_TERMS) ? p.si : 0.0;

    constexpr int lds_bytes = kSplitStages * kSplitStage;
    static OncePerDevice configured;      // the dynamic LDS limit of the three instantiations, once per device
    {
        const hipError_t e = configured.run([] {
            hipError_t r = hipFuncSetAttribute(reinterpret_cast<const void*>(&absgemm_split<false, false, true>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            if (r == hipSuccess)
                r = hipFuncSetAttribute(reinterpret_cast<const void*>(&absgemm_split<true>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            if (r == hipSuccess)
                r = hipFuncSetAttribute(reinterpret_cast<const void*>(&absgemm_split<false, true>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            if (r == hipSuccess)
                r = hipFuncSetAttribute(reinterpret_cast<const void*>(&absgemm_split<false, false, false, true>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            if (r == hipSuccess)
                r = hipFuncSetAttribute(reinterpret_cast<const void*>(&absgemm_split<true, false, false, true>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            if (r == hipSuccess)
                r = hipFuncSetAttribute(reinterpret_cast<const void*>(&absgemm_split<false, false, false, true, true>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            if (r == hipSuccess)
                r = hipFuncSetAttribute(reinterpret_cast<const void*>(&absgemm_split<true, false, false, true, true>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            for (const void* settling : {reinterpret_cast<const void*>(&absgemm_settle<false, false>), reinterpret_cast<const void*>(&absgemm_settle<true, false>),
                                         reinterpret_cast<const void*>(&absgemm_settle<true, true>), reinterpret_cast<const void*>(&absgemm_settle_parts<false>), reinterpret_cast<const void*>(&absgemm_settle_parts<true>)})
                if (r == hipSuccess) r = hipFuncSetAttribute(settling, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            return r;
        });
        if (e != hipSuccess) { g_last_hip_error = (int)e; return TAO_ERR_LAUNCH; }
    }
    p.claimed = nullptr; p.ref = nullptr; p.ldy = 0; p.strideY = 0; p.alpha = 0.0; p.eps_rel = 0.0;
    p.ws_hist = nullptr; p.ws_coarse = nullptr; p.ws_stats = nullptr; p.check_slots = kMaxCheckBlocks;
    p.ksplit = 1; p.gpp = Kp / SBK; p.partial = nullptr;
    {
        const unsigned gw = (unsigned)(tiles_n < 16 ? tiles_n : 16), gh = (unsigned)(tiles_m < 16 ? tiles_m : 16);
        p.pw = gw < 8 ? gw : 8;
        p.npx = (gw + p.pw - 1) / p.pw;                              // 1 or 2
        const unsigned npy = 8 / p.npx;
        p.ph = (gh + npy - 1) / npy;
        p.slots = 8 * p.ph * p.pw;
        p.super_rows = (unsigned)((tiles_m + 15) / 16);
        long per_z = (long)p.super_rows * ((tiles_n + 15) / 16) * p.slots;
        // A patch pattern that leaves slots empty costs a launch of less than one round dearly (an empty
        // workgroup still has to be given a compute unit's LDS before it can leave): such launches, whose
        // tiles all run at once anyway, take their tiles row by row.
        p.linear = (tiles_m * tiles_n < per_z && tiles_m * tiles_n < (long)device_cus()) ? 1u : 0u;
        if (p.linear) per_z = tiles_m * tiles_n;
        if (per_z * batch * 16 >= (1L << 31)) return TAO_ERR_SHAPE;
        p.slots_per_z = (unsigned)per_z;
        p.ntiles = (unsigned)(per_z * batch);                        // workgroups of one part
    }
    const SplitCheckHost* epi = two_pass ? nullptr : chk;      // the check inside these launches, if any
    if (epi) {
        p.claimed = chk->claimed; p.ref = chk->ref; p.ldy = chk->ldy; p.strideY = chk->strideY;
        p.alpha = chk->alpha; p.eps_rel = chk->eps_rel;
        p.ws_hist = cw.hist; p.ws_coarse = cw.coarse; p.ws_stats = cw.stats;
        if (screened) p.check_slots = kScreenSlots;
    }
    // the streaming check of a stored bound, after the launches that store it
    auto then_check = [&]() -> int {
        const int lrc = launch_status();
        if (lrc != TAO_OK || !two_pass) return lrc;
        return tao_check_and_profile(chk->claimed, chk->ref, tau, M * N * batch, chk->alpha, chk->eps_rel, chk->out,
                                     check_ws, check_workspace_bytes(), stream);
    };
    const SettleArgs settle = {cw, screened ? core_open_records(cw, M, N, K, batch) : OpenRecords{}, profile_size((unsigned long long)((__int128)M * N * batch)), chk ? chk->out : nullptr};
    if (parts >= 2) {
        // the reduction in parts, then one pass that adds them and forms (and checks) the bound
        const long groups = Kp / SBK;
        if (M * N * batch >= (1L << 32)) return TAO_ERR_SHAPE;      // (cannot happen: fewer tiles than compute units)
        p.ksplit = parts; p.gpp = (groups + parts - 1) / parts;
        p.ksplit = (int)((groups + p.gpp - 1) / p.gpp);             // no empty part
        p.partial = reinterpret_cast<double*>(wsb);
        if (screened) {
            if (settle.open.words != kOpenWords) return TAO_ERR_SHAPE;      // (cannot happen, as above: the parts are counted in whole records)
            const long wgs = (long)p.ntiles * p.ksplit;              // (the profile's 32 groups have a workgroup each)
            const dim3 grid((unsigned)(wgs < kGroups ? kGroups : wgs));
            if (Af) hipLaunchKernelGGL(absgemm_settle_parts<true>, grid, dim3(kSplitThreads), lds_bytes, st, p, settle);
            else    hipLaunchKernelGGL(absgemm_settle_parts<false>, grid, dim3(kSplitThreads), lds_bytes, st, p, settle);
            return launch_status();
        }
        hipLaunchKernelGGL((absgemm_split<false, true>), dim3(p.ntiles * (unsigned)p.ksplit), dim3(kSplitThreads), lds_bytes, st, p);
        const long total = M * N * batch;
        long want = (total + (long)kCheckThreads * 2 - 1) / ((long)kCheckThreads * 2);   // (a few elements per thread: outputs that need parts are small)
        const int nblocks = (int)(want < 1 ? 1 : (want > kMaxCheckBlocks ? kMaxCheckBlocks : want));
        if (epi) {
            hipLaunchKernelGGL(split_combine<true>, dim3(nblocks), dim3(kCheckThreads), 0, st, p, batch);
            launch_profile_reduce(cw, nblocks, (unsigned long long)total, chk->out, st);
        } else {
            hipLaunchKernelGGL(split_combine<false>, dim3(nblocks), dim3(kCheckThreads), 0, st, p, batch);
        }
        return then_check();
    }
    if (!epi) {
        // One workgroup per slot; short reductions with many tiles per compute unit instead walk their
        // tiles with one workgroup per compute unit (a multiple of 8, so a workgroup stays with its
        // XCD's patches), which takes the launch of a workgroup and the latency of its first slabs off
        // the critical path of every tile.  (Long reductions lose more to the fixed assignment of
        // tiles than they gain; the checking instantiation's epilogue is arithmetic that a walk
        // cannot hide.)  The walk needs two groups per tile.
        const long groups = Kp / SBK;
        const unsigned cus = (unsigned)device_cus() & ~7u;
        const bool walk = !Af && groups >= 2 && groups <= kWalkMaxGroups && cus >= 8 && (long)p.ntiles >= (long)kWalkMinTilesPerCu * cus;
        // (one instantiation for both: with a workgroup per slot its walk ends after the first tile)
        if (Af && cv) hipLaunchKernelGGL((absgemm_split<false, false, false, true, true>), dim3(p.ntiles), dim3(kSplitThreads), lds_bytes, st, p);
        else if (Af)  hipLaunchKernelGGL((absgemm_split<false, false, false, true>), dim3(p.ntiles), dim3(kSplitThreads), lds_bytes, st, p);
        else          hipLaunchKernelGGL((absgemm_split<false, false, true>), dim3(walk ? cus : p.ntiles), dim3(kSplitThreads), lds_bytes, st, p);
        return then_check();
    }
    if (screened) {
        const unsigned cus = (unsigned)device_cus() & ~7u, g = Af || p.ntiles < cus ? p.ntiles : cus;      // (see absgemm_settle)
        const dim3 grid(g < (unsigned)kGroups ? (unsigned)kGroups : g);
        if (Af && cv) hipLaunchKernelGGL((absgemm_settle<true, true>), grid, dim3(kSplitThreads), lds_bytes, st, p, settle);
        else if (Af)  hipLaunchKernelGGL((absgemm_settle<true, false>), grid, dim3(kSplitThreads), lds_bytes, st, p, settle);
        else          hipLaunchKernelGGL((absgemm_settle<false, false>), grid, dim3(kSplitThreads), lds_bytes, st, p, settle);
        return launch_status();
    }
    const int slots = kMaxCheckBlocks;                       // workgroup b adds to partial result b % 256
    if (!cleared) launch_clear(clear_job(cw, kMaxCheckBlocks), st);
    if (Af && cv) hipLaunchKernelGGL((absgemm_split<true, false, false, true, true>), dim3(p.ntiles), dim3(kSplitThreads), lds_bytes, st, p);
    else if (Af)  hipLaunchKernelGGL((absgemm_split<true, false, false, true>), dim3(p.ntiles), dim3(kSplitThreads), lds_bytes, st, p);
    else          hipLaunchKernelGGL((absgemm_split<true>), dim3(p.ntiles), dim3(kSplitThreads), lds_bytes, st, p);
    launch_profile_reduce(cw, slots, (unsigned long long)((__int128)M * N * batch), chk->out, st);
    return launch_status();
}

// Does split_core, with a check, clear the check's partial results itself (false) or expect them
// cleared (an epilogue check without parts: the caller's pre-pass can do it on the side)?
static bool epilogue_check_without_parts(long M, long N, long K, long batch, const tao_fp_model& md, const SplitCheckHost* chk) {
    if (!chk) return false;
    const bool two_pass = K < kEpilogueCheckMinK && !(md.flags & TAO_FLAG_CHECK_IN_EPILOGUE) &&
                          chk->ldy == N && (batch == 1 || chk->strideY == M * N);
    return !two_pass && split_k_parts(M, N, K, batch) < 2;
}

// The screen of a checked bound (linear_screen.hip).  Whether one goes ahead of the exact route: the bound itself is not asked for,
// and its constants allow it.
static bool screened(long M, long N, long K, long batch, const float* bias, const float* tau, const tao_fp_model& md, const SplitCheckHost* chk) {
    if (!chk || tau || K <= 0 || core_open_records({}, M, N, K, batch).words == 0 || (md.flags & TAO_FLAG_CHECK_IN_EPILOGUE) || chk->ldy >= kScreenMaxLd) return false;
    const long Kp_ = K + (bias ? 1 : 0);
    const double uflow = (md.flags & TAO_FLAG_UNDERFLOW_TERMS) ? (double)Kp_ * 0x1p-148 : 0.0;
    return screen_usable(K, md.u, gamma_up(Kp_, md) * kGuard, chk->alpha, uflow);
}
// The check's workspace within what core_workspace_bytes asks for; the screen's launches want all of it cleared.
static CheckWorkspace core_check_workspace(void* rest, long M, long N, long K, long batch) {
    const int parts = split_k_parts(M, N, K, batch);
    const size_t partial_bytes = parts >= 2 ? round_up_256((size_t)parts * (size_t)batch * (size_t)M * (size_t)N * sizeof(double)) : 0;
    return carve_check_workspace(static_cast<char*>(rest) + partial_bytes);
}
static int run_screen(const ScreenOperand& A, const ScreenOperand& W, const float* bias, long M, long N, long K, long batch,
                      const tao_fp_model& md, const SplitCheckHost* chk, const CheckWorkspace& cw, hipStream_t st) {
    const ScreenCheck sc = {chk->claimed, chk->ref, chk->ldy, chk->strideY, chk->alpha, chk->eps_rel};
    return launch_screen(A, W, bias, M, N, K, batch, gamma_up(K + (bias ? 1 : 0), md) * kGuard, sc, cw, core_open_records(cw, M, N, K, batch), st);
}

// Validation shared by the entry points below (everything but the operands themselves).
static int split_validate(const float* bias, float* tau, long M, long N, long K, long ldt, long batch, long strideT,
                          const tao_fp_model& md, const SplitCheckHost* chk) {
    if (M < 0 || N < 0 || K < 0 || batch < 0) return TAO_ERR_SHAPE;
    if (tau || !chk) {
        if (ldt < N || strideT < 0) return TAO_ERR_SHAPE;
        if (batch > 1 && strideT < M * ldt - (ldt - N)) return TAO_ERR_SHAPE;   // outputs would overlap
    }
    const double c = gamma_up(K + (bias ? 1 : 0), md);
    if (!(c == c)) return TAO_ERR_K_RANGE;
    if (chk) {
        if (!chk->out) return TAO_ERR_NULL;
        if (!aligned(chk->out, 8)) return TAO_ERR_ALIGN;
        if (chk->ldy < N || chk->strideY < 0 || !(chk->alpha >= 0.0) || !std::isfinite(chk->alpha) ||
            !(chk->eps_rel >= 0.0) || !std::isfinite(chk->eps_rel)) return TAO_ERR_SHAPE;
        if ((__int128)M * N * batch >= ((__int128)1 << 36)) return TAO_ERR_SHAPE;   // 32-bit partial counters
    }
    // descriptor ranges (128 rows of a plane) and the per-thread offsets must fit 32 bits
    const long Kp = (K + SBK - 1) / SBK * SBK;
    if ((__int128)STILE * Kp * 2 >= ((__int128)1 << 31)) return TAO_ERR_SHAPE;
    return TAO_OK;
}

// An empty product: nothing to bound; with a check, the profile of an empty tensor.
static int split_empty(const SplitCheckHost* chk, void* check_ws, void* stream) {
    if (!chk) return TAO_OK;
    hipStream_t st = (hipStream_t)stream;
    const CheckWorkspace cw = carve_check_workspace(check_ws);
    launch_clear(clear_job(cw, 1), st);
    launch_profile_reduce(cw, 1, 0ull, chk->out, st);
    return launch_status();
}

static int split_run(const float* A, const float* W, const float* bias, float* tau,
                     long M, long N, long K, long lda, long ldw, long ldt, int trans_w,
                     long batch, long strideA, long strideW, long strideT,
                     const tao_fp_model* model, void* ws, size_t ws_bytes, void* stream, const SplitCheckHost* chk) {
    tao_fp_model md;
    int rc = resolve_model(model, &md);
    if (rc != TAO_OK) return rc;
    if (M < 0 || N < 0 || K < 0 || batch < 0) return TAO_ERR_SHAPE;
    if (lda < K || ldw < (trans_w ? N : K)) return TAO_ERR_SHAPE;
    if (strideA < 0 || strideW < 0) return TAO_ERR_SHAPE;
    rc = split_validate(bias, tau, M, N, K, ldt, batch, strideT, md, chk);
    if (rc != TAO_OK) return rc;
    const bool shared_w = (strideW == 0) || batch == 1;
    const bool empty = M == 0 || N == 0 || batch == 0;
    const size_t bytesA = (K > 0 && !empty) ? image_bytes(M, K, batch) : 0;
    const size_t bytesW = (K > 0 && !empty) ? image_bytes(N, K, shared_w ? 1 : batch) : 0;
    if (K > 0 && !empty && (bytesA == 0 || bytesW == 0)) return TAO_ERR_WORKSPACE;
    const size_t need = bytesA + bytesW + core_workspace_bytes(M, N, K, batch, chk != nullptr);
    if (need > 0 && (!ws || !aligned(ws, 256) || ws_bytes < need)) return TAO_ERR_WORKSPACE;
    if (empty) return split_empty(chk, ws, stream);
    if ((!chk && !tau) || (K > 0 && (!A || !W))) return TAO_ERR_NULL;
    if (chk && (!chk->claimed || !chk->ref)) return TAO_ERR_NULL;
    if (!aligned(A, 4) || !aligned(W, 4) || !aligned(bias, 4) || !aligned(tau, 4)) return TAO_ERR_ALIGN;
    if (chk && (!aligned(chk->claimed, 4) || !aligned(chk->ref, 4))) return TAO_ERR_ALIGN;

    char* wsb = static_cast<char*>(ws);
    unsigned short* A3 = reinterpret_cast<unsigned short*>(wsb);
    unsigned short* W3 = reinterpret_cast<unsigned short*>(wsb + bytesA);
    void* rest = wsb + bytesA + bytesW;
    hipStream_t st = (hipStream_t)stream;
    // An A operand that only one or two column tiles use is split while the product loads it (no
    // pre-pass over it, no image): whole groups, 16-byte aligned rows, and, without a screen, the reduction in one part and
    // not a launch whose short reduction is better served by the tile walk.
    const bool rows_ok = K > 0 && K % SBK == 0 && N <= 2 * STILE && aligned(A, 16) && lda % 4 == 0 && strideA % 4 == 0 &&
                         (__int128)M * lda < ((__int128)1 << 40);
    const bool scr = screened(M, N, K, batch, bias, tau, md, chk) && !(rows_ok && lda >= kScreenMaxLd);
    const bool in_load = rows_ok && (scr || (split_k_parts(M, N, K, batch) < 2 && K / SBK > kWalkMaxGroups));
    const CheckWorkspace cw = core_check_workspace(rest, M, N, K, batch);
    bool cleared = false;
    if (K > 0) {
        // the operand pre-pass also clears the partial results of a screen and of an epilogue check (no parts: those
        // are checked by the combining pass, which needs none)
        cleared = scr || epilogue_check_without_parts(M, N, K, batch, md, chk);
        const int nmarks = scr && screen_reads_marks(M, N, K, batch, in_load, false) ? kMarks : 0;
        const SplitOperand ops[2] = {{W, N, K, ldw, shared_w ? 1 : batch, strideW, W3, trans_w ? TRANSPOSED : STRAIGHT, image_marks(W3, N, K, shared_w ? 1 : batch), nmarks},
                                     {A, M, K, lda, batch, strideA, A3, STRAIGHT, image_marks(A3, M, K, batch), nmarks}};
        launch_split3(ops, in_load ? 1 : 2, scr ? screen_clear(cw, M, N, K, batch) : cleared ? clear_job(cw, kMaxCheckBlocks) : ClearJob{}, st);
    }
    if (scr) {
        const long groups = (K + SBK - 1) / SBK;
        ScreenOperand oa = {A3, groups * ((M + STILE - 1) / STILE) * kBlock, 0, nullptr, image_marks(A3, M, K, batch)};
        if (in_load) oa = {A, strideA * 4, lda, nullptr, nullptr};
        const ScreenOperand ow = {W3, shared_w ? 0 : groups * ((N + STILE - 1) / STILE) * kBlock, 0, nullptr, image_marks(W3, N, K, shared_w ? 1 : batch)};
        rc = run_screen(oa, ow, bias, M, N, K, batch, md, chk, cw, st);
        if (rc != TAO_OK) return rc;
    }
    return split_core(A3, W3, bias, tau, M, N, K, ldt, batch, strideT, shared_w, md, rest, stream, chk, cleared,
                      in_load ? A : nullptr, lda, strideA, nullptr, scr);
}

// The same on images the caller has prepared with tao_split_operand.
static int images_run(const void* A_image, const void* W_image, const float* bias, float* tau,
                      long M, long N, long K, long ldt, long batch, long strideT, int shared_w,
                      const tao_fp_model* model, void* ws, size_t ws_bytes, void* stream, const SplitCheckHost* chk) {
    tao_fp_model md;
    int rc = resolve_model(model, &md);
    if (rc != TAO_OK) return rc;
    rc = split_validate(bias, tau, M, N, K, ldt, batch, strideT, md, chk);
    if (rc != TAO_OK) return rc;
    const bool sw = shared_w != 0 || batch == 1;
    const size_t need = core_workspace_bytes(M, N, K, batch, chk != nullptr);
    if (need > 0 && (!ws || !aligned(ws, 256) || ws_bytes < need)) return TAO_ERR_WORKSPACE;
    if (M == 0 || N == 0 || batch == 0) return split_empty(chk, ws, stream);
    if ((!chk && !tau) || (K > 0 && (!A_image || !W_image))) return TAO_ERR_NULL;
    if (chk && (!chk->claimed || !chk->ref)) return TAO_ERR_NULL;
    if (!aligned(A_image, 256) || !aligned(W_image, 256) || !aligned(bias, 4) || !aligned(tau, 4)) return TAO_ERR_ALIGN;
    if (chk && (!aligned(chk->claimed, 4) || !aligned(chk->ref, 4))) return TAO_ERR_ALIGN;
    const unsigned short* A3 = static_cast<const unsigned short*>(A_image);
    const unsigned short* W3 = static_cast<const unsigned short*>(W_image);
    bool cleared = false;
    const bool scr = screened(M, N, K, batch, bias, tau, md, chk);
    if (scr) {
        hipStream_t st = (hipStream_t)stream;
        const CheckWorkspace cw = core_check_workspace(ws, M, N, K, batch);
        cleared = true;
        launch_clear(screen_clear(cw, M, N, K, batch), st);
        const long groups = (K + SBK - 1) / SBK;
        const ScreenOperand oa = {A3, groups * ((M + STILE - 1) / STILE) * kBlock, 0, nullptr, image_marks(A3, M, K, batch)};
        const ScreenOperand ow = {W3, sw ? 0 : groups * ((N + STILE - 1) / STILE) * kBlock, 0, nullptr, image_marks(W3, N, K, sw ? 1 : batch)};
        rc = run_screen(oa, ow, bias, M, N, K, batch, md, chk, cw, st);
        if (rc != TAO_OK) return rc;
    }
    return split_core(A3, W3, bias, tau, M, N, K, ldt, batch, strideT, sw, md, ws, stream, chk, cleared,
                      nullptr, 0, 0, nullptr, scr);
}
}  // namespace tao

extern "C" {

int tao_split_operand(const float* src, long rows, long K, long ld, int trans, long batch, long stride,
                      void* image, size_t image_bytes, void* stream) {
    using namespace tao;
    if (rows < 0 || K < 0 || batch < 0 || stride < 0) return TAO_ERR_SHAPE;
    if (ld < (trans ? rows : K)) return TAO_ERR_SHAPE;
    if (rows == 0 || K == 0 || batch == 0) return TAO_OK;
    const long Kp = (K + SBK - 1) / SBK * SBK;
    if ((__int128)STILE * Kp * 2 >= ((__int128)1 << 31)) return TAO_ERR_SHAPE;
    if (!src) return TAO_ERR_NULL;
    if (!aligned(src, 4)) return TAO_ERR_ALIGN;
    const size_t need = tao::image_bytes(rows, K, batch);
    if (need == 0 || !image || !aligned(image, 256) || image_bytes < need) return TAO_ERR_WORKSPACE;
    if (batch >= 65536) return TAO_ERR_SHAPE;                      // (an image's limit, whatever a launch could take)
    const SplitOperand op = {src, rows, K, ld, batch, stride, static_cast<unsigned short*>(image), trans ? TRANSPOSED : STRAIGHT,
                             image_marks(image, rows, K, batch), screen_reads_marks(K) ? kMarks : 0};
    launch_split3(&op, 1, ClearJob{}, (hipStream_t)stream);
    return launch_status();
}

int tao_bound_linear_images(const void* A_image, const void* W_image, const float* bias, float* tau,
                            long M, long N, long K, long ldt, long batch, long strideT, int shared_w,
                            const tao_fp_model* model, void* ws, size_t ws_bytes, void* stream) {
    return tao::images_run(A_image, W_image, bias, tau, M, N, K, ldt, batch, strideT, shared_w, model, ws, ws_bytes, stream, nullptr);
}

int tao_bound_check_linear_images(const void* A_image, const void* W_image, const float* bias, const float* y_ref,
                                  const float* claimed, float* tau, long M, long N, long K, long ldy, long batch,
                                  long strideY, int shared_w, double alpha, double eps_rel, const tao_fp_model* model,
                                  tao_profile* out, void* ws, size_t ws_bytes, void* stream) {
    tao::SplitCheckHost chk = {claimed, y_ref, ldy, strideY, alpha, eps_rel, out};
    return tao::images_run(A_image, W_image, bias, tau, M, N, K, ldy, batch, strideY, shared_w, model, ws, ws_bytes, stream, &chk);
}

}  // extern "C"

namespace tao {
// The convolution bound on the BF16 matrix cores: the filters' image is written into ws by the
// pre-pass, the patch matrix is gathered and cut into pieces while the product loads it.
static bool conv_split_ok(long M, long N, long K, long C, long batch_hwc, const float* x) {
    // whole 32-channel slabs inside one tap, the reduction in one part (enough tiles), 16-byte aligned
    // pixels, 32-bit pixel arithmetic in the kernel
    return C % SBK == 0 && K / SBK >= 1 && split_k_parts(M, N, K, 1) < 2 && aligned(x, 16) && batch_hwc < (1L << 40);
}
// What the screen of a checked convolution takes behind the rest of the workspace: the input's BF16 magnitudes and a line of zeros
// (0: offsets beyond 31 bits, no screen).
static size_t conv_pixel_bytes(long batch, long H, long W, long C) {
    const __int128 b = (__int128)batch * H * W * C * 2 + 64;
    return b < ((__int128)1 << 31) ? (size_t)b : 0;
}
static int conv_split_run(const float* x, const float* w, const float* bias, float* tau,
                          long batch, long H, long W, long C, long Cout, long R, long S,
                          long stride_h, long stride_w, long pad_h, long pad_w, long dil_h, long dil_w,
                          const tao_fp_model* model, void* ws, size_t ws_bytes, void* stream, const SplitCheckHost* chk) {
    tao_fp_model md;
    int rc = resolve_model(model, &md);
    if (rc != TAO_OK) return rc;
    long OH = 0, OW = 0, M = 0, K = 0;
    rc = conv_geometry(batch, H, W, C, Cout, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, &OH, &OW, &M, &K);
    if (rc != TAO_OK) return rc;
    const long N = Cout;
    rc = split_validate(bias, tau, M, N, K, N, 1, M * N, md, chk);
    if (rc != TAO_OK) return rc;
    const bool empty = M == 0 || N == 0;
    if (!empty && !conv_split_ok(M, N, K, C, batch * H * W * C, x)) return TAO_ERR_SHAPE;
    const size_t bytesW = empty ? 0 : image_bytes(N, K, 1);
    const size_t need = bytesW + core_workspace_bytes(M, N, K, 1, chk != nullptr);
    if (need > 0 && (!ws || !aligned(ws, 256) || ws_bytes < need)) return TAO_ERR_WORKSPACE;
    if (empty) return split_empty(chk, ws, stream);
    if ((!chk && !tau) || !x || !w) return TAO_ERR_NULL;
    if (chk && (!chk->claimed || !chk->ref)) return TAO_ERR_NULL;
    if (!aligned(w, 4) || !aligned(bias, 4) || !aligned(tau, 4)) return TAO_ERR_ALIGN;
    if (chk && (!aligned(chk->claimed, 4) || !aligned(chk->ref, 4))) return TAO_ERR_ALIGN;
    char* wsb = static_cast<char*>(ws);
    unsigned short* W3 = reinterpret_cast<unsigned short*>(wsb);
    void* rest = wsb + bytesW;
    ConvHost cv;
    cv.H = (int)H; cv.W = (int)W; cv.C = (int)C; cv.OW = (int)OW; cv.S = (int)S;
    cv.sh = (int)stride_h; cv.sw = (int)stride_w; cv.ph = (int)pad_h; cv.pw = (int)pad_w; cv.dh = (int)dil_h; cv.dw = (int)dil_w;
    cv.ohow = (unsigned)(OH * OW);
    // (a workspace without room for the input's magnitudes, as the exact route needs none, gets no screen)
    const size_t pixel_bytes = conv_pixel_bytes(batch, H, W, C), pixels_at = round_up_256(need);
    const bool scr = pixel_bytes > 0 && ws_bytes >= pixels_at + pixel_bytes && screened(M, N, K, 1, bias, tau, md, chk);
    const bool cleared = scr || epilogue_check_without_parts(M, N, K, 1, md, chk);
    const CheckWorkspace cw = carve_check_workspace(rest);
    unsigned short* px = reinterpret_cast<unsigned short*>(wsb + pixels_at);
    // (the input's magnitudes have no place for marks: both operands' lie behind the filters' image)
    unsigned char* const marks = image_marks(W3, N, K, 1);
    const long units = (K + SBK - 1) / SBK * ((N + 63) / 64);
    const int own = (int)std::min((units + 3) / 4, kMarks / 2L), nmarks = scr && screen_reads_marks(M, N, K, 1, false, true) ? kMarks : 0;
    const SplitOperand ops[2] = {{w, N, K, K, 1, 0, W3, STRAIGHT, marks, std::min(own, nmarks)},
                                 {x, 1, batch * H * W * C, 0, 1, 0, px, MAGNITUDES, marks + own, std::max(0, nmarks - own)}};
    launch_split3(ops, scr ? 2 : 1, scr ? screen_clear(cw, M, N, K, 1) : cleared ? clear_job(cw, kMaxCheckBlocks) : ClearJob{}, (hipStream_t)stream);
    if (scr) {
        const ScreenPixels pixels = {cv.H, cv.W, cv.C, cv.OW, (int)R, cv.S, cv.sh, cv.sw, cv.ph, cv.pw, cv.dh, cv.dw, (int)R / 2, cv.S / 2, cv.ohow, cv.C / SBK,
                                     (unsigned)(batch * H * W * C * 2)};
        const ScreenOperand oa = {px, 0, 0, &pixels, marks}, ow = {W3, 0, 0, nullptr, marks};
        rc = run_screen(oa, ow, bias, M, N, K, 1, md, chk, cw, (hipStream_t)stream);
        if (rc != TAO_OK) return rc;
    }
    return split_core(nullptr, W3, bias, tau, M, N, K, N, 1, M * N, true, md, rest, stream, chk, cleared, x, K, 0, &cv, scr);
}
}  // namespace tao

extern "C" {

int tao_conv2d_split_supported(long batch, long H, long W, long C, long Cout, long R, long S,
                               long stride_h, long stride_w, long pad_h, long pad_w, long dil_h, long dil_w) {
    long OH = 0, OW = 0, M = 0, K = 0;
    if (tao::conv_geometry(batch, H, W, C, Cout, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, &OH, &OW, &M, &K) != TAO_OK) return 0;
    if (M == 0 || Cout == 0) return 1;
    return tao::conv_split_ok(M, Cout, K, C, batch * H * W * C, nullptr) ? 1 : 0;
}

size_t tao_conv2d_split_workspace_bytes(long batch, long H, long W, long C, long Cout, long R, long S,
                                        long stride_h, long stride_w, long pad_h, long pad_w, long dil_h, long dil_w,
                                        int with_check) {
    long OH = 0, OW = 0, M = 0, K = 0;
    if (tao::conv_geometry(batch, H, W, C, Cout, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, &OH, &OW, &M, &K) != TAO_OK) return 0;
    const size_t img = (M == 0 || Cout == 0) ? 0 : tao::image_bytes(Cout, K, 1);
    const size_t need = img + tao::core_workspace_bytes(M, Cout, K, 1, with_check != 0);
    return with_check && img ? tao::round_up_256(need) + tao::conv_pixel_bytes(batch, H, W, C) : need;
}

int tao_bound_conv2d_split(const float* x, const float* w, const float* bias, float* tau,
                           long batch, long H, long W, long C, long Cout, long R, long S,
                           long stride_h, long stride_w, long pad_h, long pad_w, long dil_h, long dil_w,
                           const tao_fp_model* model, void* ws, size_t ws_bytes, void* stream) {
    return tao::conv_split_run(x, w, bias, tau, batch, H, W, C, Cout, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w,
                               model, ws, ws_bytes, stream, nullptr);
}

int tao_bound_check_conv2d(const float* x, const float* w, const float* bias, const float* y_ref, const float* claimed,
                           float* tau, long batch, long H, long W, long C, long Cout, long R, long S,
                           long stride_h, long stride_w, long pad_h, long pad_w, long dil_h, long dil_w,
                           double alpha, double eps_rel, const tao_fp_model* model, tao_profile* out,
                           void* ws, size_t ws_bytes, void* stream) {
    // (y_ref, claimed and tau are [batch][OH][OW][Cout] contiguous: rows of Cout, one batch entry in matrix terms)
    tao::SplitCheckHost chk = {claimed, y_ref, Cout, 0, alpha, eps_rel, out};
    return tao::conv_split_run(x, w, bias, tau, batch, H, W, C, Cout, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w,
                               model, ws, ws_bytes, stream, &chk);
}

int tao_bound_linear_split(const float* A, const float* W, const float* bias, float* tau,
                           long M, long N, long K, long lda, long ldw, long ldt, int trans_w,
                           long batch, long strideA, long strideW, long strideT,
                           const tao_fp_model* model, void* ws, size_t ws_bytes, void* stream) {
    return tao::split_run(A, W, bias, tau, M, N, K, lda, ldw, ldt, trans_w, batch, strideA, strideW, strideT,
                          model, ws, ws_bytes, stream, nullptr);
}

size_t tao_bound_check_linear_workspace_bytes(long M, long N, long K, long batch, int shared_w) {
    if (M < 0 || N < 0 || K < 0 || batch < 0) return 0;
    const bool empty = M == 0 || N == 0 || batch == 0;
    const size_t a = (K > 0 && !empty) ? tao::image_bytes(M, K, batch) : 0;
    const size_t w = (K > 0 && !empty) ? tao::image_bytes(N, K, shared_w ? 1 : batch) : 0;
    if (K > 0 && !empty && (a == 0 || w == 0)) return 0;
    return a + w + tao::core_workspace_bytes(M, N, K, batch, true);
}

int tao_bound_check_linear_in_epilogue(long M, long N, long K, long batch) {
    return (K >= tao::kEpilogueCheckMinK || tao::split_k_parts(M, N, K, batch) >= 2) ? 1 : 0;
}

int tao_bound_check_linear(const float* A, const float* W, const float* bias, const float* y_ref,
                           const float* claimed, float* tau,
                           long M, long N, long K, long lda, long ldw, long ldy, int trans_w,
                           long batch, long strideA, long strideW, long strideY,
                           double alpha, double eps_rel, const tao_fp_model* model, tao_profile* out,
                           void* ws, size_t ws_bytes, void* stream) {
    tao::SplitCheckHost chk = {claimed, y_ref, ldy, strideY, alpha, eps_rel, out};
    return tao::split_run(A, W, bias, tau, M, N, K, lda, ldw, ldy, trans_w, batch, strideA, strideW, strideY,
                          model, ws, ws_bytes, stream, &chk);
}

}  // extern "C"
