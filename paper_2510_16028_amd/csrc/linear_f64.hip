// tao_bound_linear on the binary64 matrix cores, for products whose output is too small for the
// 128 x 128 (or 64 x 128) tiles of linear.hip to fill the chip: a decode step's projections, small layers.
//
// What bounds them: the weights have to be read once (M = 8 rows against a 4096 x 4096 weight: 64 MB,
// 13 us at the rate a large copy reaches here), while the tiles of the FP32 kernel leave 32 workgroups
// walking the whole reduction one after the other (381 us for that product, whatever M up to 128).  Here a
// workgroup owns a small tile (16 to 64 rows x 16 to 64 columns) and its wavefronts divide the
// reduction: each streams its own 32-k chunks of both operands from global memory straight into
// registers, double-buffered, and the wavefronts' sums meet in LDS once at the end.  No operand goes through
// LDS: a weight value is used by one wavefront only.
//
// Arithmetic: v_mfma_f64_16x16x4_f64 on the magnitudes converted to binary64.  The product of two binary32
// values is exact there and every addition errs by less than 2^-52 of the sum of non-negative terms, so
// the computed sum lies in [S (1 - m), S (1 + m)] with m = (K + 64) 2^-52 < 2^-27, against 7 x 2^-24 for
// the FP32 scheme: the bound is tighter, and no partial sum can be subnormal (a product of two binary32
// subnormals is 2^-298), so the absolute term of the FP32 scheme disappears.  The instruction runs at half
// the rate of the FP32 one and without that scheme's folding: 78.6 against 96 TFLOP/s reached.
#include <type_traits>
#include "linear_f64.hpp"
#include "tao_device.hpp"

namespace tao {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kF64Chunk = 32;        // k per chunk: one 128-byte line of a row

struct F64Args {
    const float* A; const float* W; const float* bias; float* tau;
    long M, N, K, lda, ldw, ldt, strideA, strideW, strideT;
    unsigned tiles_m, tiles_n;
    unsigned items, share;           // tiles of all batch entries, of one XCD
    double c;                        // Gamma(K') guard, upper
    double infl;                     // reciprocal of the lower rounding factor
    double uflow;                    // TAO_FLAG_UNDERFLOW_TERMS
    ConvRows cv; unsigned xbytes;    // a convolution's patch matrix: A is its input
};

// Where the rows of A come from: a matrix, or the channels-last input of a convolution, of whose patch matrix a row is an output pixel's taps
// -- gathered four channels at a time (C a multiple of 4, 16-byte aligned), or each by itself.  Taps in the zero padding and k beyond the
// reduction are read outside the buffer's descriptor, which returns zeros.
enum { MATRIX, PATCHES4, PATCHES };
constexpr unsigned kOutside = 0xfffffff0u;

// Four consecutive values of a row from column k on; FULL: all of them lie inside it, else zeros beyond K.
template <bool VEC, bool FULL>
__device__ __forceinline__ float4 row4(const float* __restrict__ row, long k, long K) {
    if (FULL && VEC) return *reinterpret_cast<const float4*>(row + k);
    if (FULL) return make_float4(row[k], row[k + 1], row[k + 2], row[k + 3]);
    return make_float4(k < K ? row[k] : 0.f, k + 1 < K ? row[k + 1] : 0.f, k + 2 < K ? row[k + 2] : 0.f, k + 3 < K ? row[k + 3] : 0.f);
}

// WAVES wavefronts; the workgroup's tile is MT x NT matrix tiles of 16 x 16.  Lane l of a wavefront holds
// row (column) l % 16 of a matrix tile; k runs over the lane's quarter l / 16 and its four loaded values.
// (Which k a lane holds does not matter as long as both operands agree.)
// TRANS: W is [K][N].  A convolution's rows are gathered tap by tap (SRC): a lane's four k lie in one tap, or each in its own.
template <bool TRANS, bool VEC, int MT, int NT, int WAVES, int SRC = MATRIX>
__global__ __launch_bounds__(WAVES * 64) void absgemm_f64(F64Args p) {
    // the wavefronts' sums; with eight matrix tiles the upper half of the wavefronts hands its sums to the lower first
    constexpr int SLOTS = MT * NT > 4 ? WAVES / 2 : WAVES;
    __shared__ double part[SLOTS][MT * NT * 256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    // Workgroups are dealt round-robin to the eight XCDs, each with its own L2: XCD x takes the x-th contiguous eighth of the
    // tiles, row tiles first, so that those that share a slab of W meet in one.  (By columns -- column tile tn on XCD tn % 8 --
    // outputs of fewer than eight column tiles left XCDs idle: 65536 x 256 x 16 (M x K x N) 148 us against 22 now, 64
    // products of 512 x 512 x 64 230 against 60; wide outputs as before.)
    const unsigned item = (blockIdx.x & 7) * p.share + (blockIdx.x >> 3);
    if (item >= p.items) return;                                       // whole workgroup
    const unsigned column = item / p.tiles_m, tm = item - column * p.tiles_m;
    const unsigned zb = column / p.tiles_n, tn = column - zb * p.tiles_n;
    const long z = zb;
    const long m0 = (long)tm * (MT * 16), n0 = (long)tn * (NT * 16);
    const float* Ab = p.A + z * p.strideA;
    const float* Wb = p.W + z * p.strideW;
    const float* arow[MT];
    int pix_h[MT], pix_w[MT];                                          // input coordinates of tap (0, 0)
    unsigned pix[MT];                                                  // and its byte offset (modulo 2^32: a tap inside the input has one below 2^31)
    const __amdgpu_buffer_rsrc_t dx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.A), 0, (int)p.xbytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < MT; ++i) {                                     // rows beyond the edge repeat the last one
        const long m = m0 + i * 16 + r, mc = m < p.M ? m : p.M - 1;
        if (SRC == MATRIX) {
            arow[i] = Ab + mc * p.lda;
        } else {
            const unsigned row = (unsigned)mc, img = row / p.cv.ohow, rem = row - img * p.cv.ohow;
            const unsigned oh = rem / (unsigned)p.cv.OW, ow = rem - oh * (unsigned)p.cv.OW;
            pix_h[i] = (int)oh * p.cv.sh - p.cv.ph; pix_w[i] = (int)ow * p.cv.sw - p.cv.pw;
            pix[i] = ((img * (unsigned)p.cv.H + (unsigned)pix_h[i]) * (unsigned)p.cv.W + (unsigned)pix_w[i]) * (unsigned)p.cv.C * 4u;
        }
    }
    // the tap of the k'th column of the patch matrix: its shift against tap (0, 0), and the byte offset of its channel
    struct Tap { int dr, ds; unsigned off; bool real; };
    auto tap_of = [&](unsigned k) __attribute__((always_inline)) {
        const unsigned tap = k / (unsigned)p.cv.C, c = k - tap * (unsigned)p.cv.C, fr = tap / (unsigned)p.cv.S, fs = tap - fr * (unsigned)p.cv.S;
        const int dr = (int)fr * p.cv.dh, ds = (int)fs * p.cv.dw;
        return Tap{dr, ds, (((unsigned)dr * (unsigned)p.cv.W + (unsigned)ds) * (unsigned)p.cv.C + c) * 4u, (long)k < p.K};
    };
    auto offset_of = [&](int i, const Tap& t) __attribute__((always_inline)) {
        const bool inside = t.real && (unsigned)(pix_h[i] + t.dr) < (unsigned)p.cv.H && (unsigned)(pix_w[i] + t.ds) < (unsigned)p.cv.W;
        return (int)(inside ? pix[i] + t.off : kOutside);
    };
    const float* wrow[NT];                                             // row of W (!TRANS)
    unsigned wcol[NT];                                                 // byte offset of the column in the lane's first k row (TRANS)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const long n = n0 + j * 16 + r, nc = n < p.N ? n : p.N - 1;
        wrow[j] = Wb + (TRANS ? 0 : nc * p.ldw);
        wcol[j] = TRANS ? (unsigned)(nc + q * 4 * p.ldw) * 4u : 0u;    // (the host keeps this in 32 bits)
    }

    doublex4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};

    // One chunk: A as two vectors of four k per row, half a chunk apart; W likewise, or (TRANS) eight k of NT columns.
    float4 a[2][MT][2];
    float w[2][NT][8];
    auto load = [&](auto full, int s, long k0) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full)::value;
        if (SRC == MATRIX) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) a[s][i][hf] = row4<VEC, FULL>(arow[i], k0 + hf * 16 + q * 4, p.K);
        } else {
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const unsigned k = (unsigned)k0 + hf * 16 + q * 4;
                if (SRC == PATCHES4) {
                    const Tap t = tap_of(k);
#pragma unroll
                    for (int i = 0; i < MT; ++i)
                        a[s][i][hf] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(dx, offset_of(i, t), 0, 0));
                } else {
                    const Tap t0 = tap_of(k), t1 = tap_of(k + 1), t2 = tap_of(k + 2), t3 = tap_of(k + 3);
                    auto one = [&](int i, const Tap& t) { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(dx, offset_of(i, t), 0, 0)); };
#pragma unroll
                    for (int i = 0; i < MT; ++i) a[s][i][hf] = make_float4(one(i, t0), one(i, t1), one(i, t2), one(i, t3));
                }
            }
        }
        if (!TRANS) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
                    const float4 v = row4<VEC, FULL>(wrow[j], k0 + hf * 16 + q * 4, p.K);
                    w[s][j][4 * hf] = v.x; w[s][j][4 * hf + 1] = v.y; w[s][j][4 * hf + 2] = v.z; w[s][j][4 * hf + 3] = v.w;
                }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const long ks = k0 + (e >> 2) * 16 + (e & 3);              // the lane's k is ks + 4 q
                long krow = ks * p.ldw;
                asm("" : "+s"(krow));                                      // (one scalar base per k: else the compiler keeps a 64-bit pointer per load)
                const char* base = reinterpret_cast<const char*>(Wb + krow);
#pragma unroll
                for (int j = 0; j < NT; ++j) w[s][j][e] = (FULL || ks + q * 4 < p.K) ? *reinterpret_cast<const float*>(base + wcol[j]) : 0.f;
            }
        }
        __builtin_amdgcn_sched_barrier(0);                                 // (the loads stay ahead of the arithmetic they overlap)
    };
    auto multiply = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            double ad[MT], wd[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const float4 v = a[s][i][e >> 2];
                ad[i] = fabs((double)((e & 3) == 0 ? v.x : (e & 3) == 1 ? v.y : (e & 3) == 2 ? v.z : v.w));
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) wd[j] = fabs((double)w[s][j][e]);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ad[i], wd[j], acc[i][j], 0, 0, 0);
        }
    };
    // whole chunks double-buffered, then the ragged one, which belongs to one wavefront
    const long step = (long)WAVES * kF64Chunk;
    const long whole = p.K / kF64Chunk * kF64Chunk;
    long k0 = (long)__builtin_amdgcn_readfirstlane(wave) * kF64Chunk;
    if (k0 < whole) {
        load(std::true_type(), 0, k0);
        // (nothing conditional inside: the compiler then waits for the older chunk only)
        for (; k0 + 2 * step < whole; k0 += 2 * step) {
            load(std::true_type(), 1, k0 + step);
            multiply(0);
            load(std::true_type(), 0, k0 + 2 * step);
            multiply(1);
        }
        if (k0 + step < whole) {
            load(std::true_type(), 1, k0 + step);
            multiply(0);
            multiply(1);
            k0 += step;
        } else {
            multiply(0);
        }
        k0 += step;
    }
    if (k0 < p.K) {
        load(std::false_type(), 0, k0);
        multiply(0);
    }
    // register v of a matrix tile: row lane / 16 + 4 v, column lane % 16
    const long chunks = (p.K + kF64Chunk - 1) / kF64Chunk;
    int holders = chunks < WAVES ? (int)chunks : WAVES;                // wavefronts that had a chunk
    auto each = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) f(acc[i][j], v, (i * NT + j) * 256 + v * 64 + lane);
    };
    if (SLOTS < WAVES && holders > SLOTS) {
        if (wave >= SLOTS && wave < holders) each([&](doublex4& x, int v, int at) { part[wave - SLOTS][at] = x[v]; });
        __syncthreads();
        if (wave + SLOTS < holders) each([&](doublex4& x, int v, int at) { x[v] += part[wave][at]; });
        holders = SLOTS;                                               // (a wavefront reads and writes its own slot only)
    }
    if (wave < holders) each([&](doublex4& x, int v, int at) { part[wave][at] = x[v]; });
    __syncthreads();
    // every output element: the wavefronts' sums in a fixed order, then the bound
    for (int t = threadIdx.x; t < MT * NT * 256; t += WAVES * 64) {
        double s = 0.0;
        for (int g = 0; g < holders; ++g) s += part[g][t];
        const int tile = t >> 8, i = tile / NT, j = tile % NT, v = (t >> 6) & 3, l = t & 63;
        const long row = m0 + i * 16 + (l >> 4) + 4 * v;
        const long col = n0 + j * 16 + (l & 15);
        if (row < p.M && col < p.N) {
            const double ab = p.bias ? fabs((double)p.bias[col]) : 0.0;
            p.tau[z * p.strideT + row * p.ldt + col] = up32((s * p.infl + ab) * p.c + p.uflow);
        }
    }
}

// Tile of a problem: as many rows as M asks for, fewer while the workgroups would not fill the chip, then as
// many columns as still leave one workgroup per compute unit.  64 x 32 outputs (one workgroup resident per
// compute unit) run at 61 TFLOP/s, 64 x 16 at 54 (more operand bytes from L2 per product): the larger tile
// where its last round is not the emptier one (M = 255, K = 4096: N = 4096 148 against 159 us, but N = 3072, K = 768
// 39 against 31).  Up to 32 rows the weights' bytes decide, not the tile.
struct F64Tile { int mt, nt; long tiles_m, tiles_n; double rounds, tflops; };
static F64Tile f64_tile(long M, long N, long batch, int cus) {
    F64Tile t;
    t.mt = M > 32 ? 4 : M > 16 ? 2 : 1;
    auto count = [&](int mt, int nt) { return ((M + 16 * mt - 1) / (16 * mt)) * ((N + 16 * nt - 1) / (16 * nt)) * batch; };
    auto rounds = [&](int mt, int nt) { return (double)((count(mt, nt) + cus - 1) / cus); };
    while (t.mt > 1 && count(t.mt, 1) < cus) t.mt /= 2;
    t.nt = 1;
    if (t.mt == 4) { if (rounds(4, 2) * 2.0 / 61.0 < rounds(4, 1) / 54.0) t.nt = 2; }
    else           { while (t.mt * t.nt < 4 && count(t.mt, 2 * t.nt) >= cus) t.nt *= 2; }
    t.tiles_m = (M + 16 * t.mt - 1) / (16 * t.mt);
    t.tiles_n = (N + 16 * t.nt - 1) / (16 * t.nt);
    t.rounds = rounds(t.mt, t.nt);
    t.tflops = t.mt * t.nt == 8 ? 61.0 : 54.0;
    return t;
}

static void f64_args(const F64Tile& t, const LinearProblem& q, const tao_fp_model& md, double gamma, F64Args& p) {
    p.A = q.A; p.W = q.W; p.bias = q.bias; p.tau = q.tau;
    p.M = q.M; p.N = q.N; p.K = q.K; p.lda = q.lda; p.ldw = q.ldw; p.ldt = q.ldt;
    p.strideA = q.strideA; p.strideW = q.strideW; p.strideT = q.strideT;
    p.tiles_m = (unsigned)t.tiles_m; p.tiles_n = (unsigned)t.tiles_n;
    // every addition of non-negative terms within 2^-52 (1 for the product, K - 1 additions in the instruction's
    // chain, a few more where the wavefronts' sums meet)
    const double lower = 1.0 - ((double)q.K + 64.0) * 0x1p-52;
    p.infl = widen(1.0 / lower);
    p.c = widen(gamma * kGuard);
    p.uflow = (md.flags & TAO_FLAG_UNDERFLOW_TERMS) ? widen((double)(q.K + (q.bias ? 1 : 0)) * 0x1p-149) : 0.0;
    p.items = (unsigned)(t.tiles_m * t.tiles_n * q.batch);             // (the routes: below 2^30)
    p.share = (p.items + 7) / 8;
}

// Times in us as measured on both sides of the line at 480 shapes (8 ... 65536 rows, 16 ... 12288 columns, K = 32 ... 8192, up to
// 1024 batch entries), fitted so that the chosen side is within 1.15 of the better one, mostly the better one: a round of
// workgroups here takes its products at 1.09 times the rate above and, per matrix tile, 0.38 for first loads and the meeting of the
// wavefronts' sums, up to 0.6 more for a long reduction and 0.48 for a ragged last chunk; a round of the FP32 tiles
// takes 1.5 (64 rows) or 2.95 per 32 k-steps, 1.18 times that with ragged tiles and 1.43 times with unaligned rows, and 2.5 or 2
// besides.  (us, here / FP32 tiles: 8 x 4096 x 4096 (M x K x N) 17 / 381, 128 x 4096 x 4096 75 / 194, 65536 x 512 x 32 62 / 112,
// 1000 x 1000 x 1000 55 / 66, 255 x 8192 x 8192 521 / 519; 65536 x 147 x 64 89 / 50, 250 x 1024 x 12288 147 / 111,
// 145 x 60 x 1065 x 5 entries 17 / 9.)
struct LinearTimes { double f64, fp32; };
static LinearTimes linear_times(const F64Tile& t, long M, long N, long K, long batch, bool vec, int cus) {
    const double k = (double)K;
    const int matrix_tiles = t.mt * t.nt;
    LinearTimes r;
    r.f64 = t.rounds * matrix_tiles * (0.92 * 512.0 * k * (double)cus / (t.tflops * 1e6) + 0.38 + 0.6 * std::fmin(k / 1024.0, 1.0) +
                                       (K % kF64Chunk ? 0.48 : 0.0));
    auto fp32 = [&](long rows, double per_group, double besides) {
        const double rounds = (double)((((M + rows - 1) / rows) * ((N + 127) / 128) * batch + cus - 1) / cus);
        const bool clean = vec && M % rows == 0 && N % 128 == 0 && K % 32 == 0;
        return rounds * ((double)((K + 31) / 32) * per_group * (clean ? 1.0 : vec ? 1.18 : 1.43) + besides);
    };
    r.fp32 = fp32(128, 2.95, 2.0);
    if (M > 64) r.fp32 = std::fmin(r.fp32, fp32(64, 1.5, 2.5));
    return r;
}
// 16-byte loads of both operands
static bool vector_rows(const LinearProblem& p) {
    return aligned(p.A, 16) && p.lda % 4 == 0 && p.strideA % 4 == 0 && aligned(p.W, 16) && p.ldw % 4 == 0 && p.strideW % 4 == 0;
}
bool f64_route(const LinearProblem& p, int cus) {
    if (p.batch >= 65536 || p.K < 1) return false;
    if (p.trans_w && p.N + 16 * p.ldw >= (1L << 30)) return false;     // (32-bit column offsets)
    const F64Tile t = f64_tile(p.M, p.N, p.batch, cus);
    if (t.rounds * (double)cus >= 0x1p30) return false;                // (32-bit tile numbers)
    const LinearTimes r = linear_times(t, p.M, p.N, p.K, p.batch, vector_rows(p) && p.K % 4 == 0, cus);
    return r.f64 < r.fp32;
}
double linear_us(long M, long N, long K, long batch, int cus) {
    const LinearTimes r = linear_times(f64_tile(M, N, batch, cus), M, N, K, batch, K % 4 == 0, cus);
    return std::fmin(r.f64, r.fp32);
}

template <bool TRANS, bool VEC, int SRC>
static void f64_dispatch(const F64Tile& t, hipStream_t st, const F64Args& p) {
    const dim3 grid(p.share * 8);
#define TAO_F64(MT, NT, WAVES) hipLaunchKernelGGL((absgemm_f64<TRANS, VEC, MT, NT, WAVES, SRC>), grid, dim3(WAVES * 64), 0, st, p)
    if (t.mt == 1)      { if (t.nt == 1) TAO_F64(1, 1, 16); else if (t.nt == 2) TAO_F64(1, 2, 16); else TAO_F64(1, 4, 8); }
    else if (t.mt == 2) { if (t.nt == 1) TAO_F64(2, 1, 16); else TAO_F64(2, 2, 8); }
    else                { if (t.nt == 1) TAO_F64(4, 1, 8); else TAO_F64(4, 2, 8); }
#undef TAO_F64
}

int f64_launch(const LinearProblem& q, const tao_fp_model& md, double gamma, int cus, hipStream_t st) {
    const F64Tile t = f64_tile(q.M, q.N, q.batch, cus);
    F64Args p = {};
    f64_args(t, q, md, gamma, p);
    const bool vec = vector_rows(q);
    if (q.trans_w) { if (vec) f64_dispatch<true, true, MATRIX>(t, st, p); else f64_dispatch<true, false, MATRIX>(t, st, p); }
    else           { if (vec) f64_dispatch<false, true, MATRIX>(t, st, p); else f64_dispatch<false, false, MATRIX>(t, st, p); }
    return launch_status();
}

static bool patches_by_four(const LinearProblem& p, const ConvRows& cv) { return cv.C % 4 == 0 && aligned(p.A, 16) && aligned(p.W, 16); }
// The FP32 tiles of a convolution (bm rows each, whole: rows, columns and slabs regular; slabs: 32 channels of a tap at a time): times of a
// round as measured at 220 shapes (49 ... 250 000 rows, 64 ... 512 columns, K = 3 ... 4608, fitted to 15 %), us per 32 k and besides.
// fast: one accumulation chain (TAO_FLAG_FAST_ACCUM), at 56 shapes 0.73 to 0.87 of that where tiles are whole, otherwise 0.85 to 0.98, the lower the longer
// the reduction.
static double conv_fp32_us(long bm, bool whole, bool slabs, bool vec, bool fast, long M, long N, long K, int cus) {
    const double chain = !fast ? 1.0 : whole ? 0.74 : 0.87;
    const double rounds = chain * (double)((((M + bm - 1) / bm) * ((N + 127) / 128) + cus - 1) / cus), groups = (double)((K + 31) / 32);
    if (bm == 64) return rounds * (whole ? groups * 1.5 + 2.5 : slabs ? groups * 2.5 + 2.5 : vec ? groups * 2.65 + 6.5 : groups * 3.05 + 4.5);
    return rounds * (whole ? groups * 2.95 + 2.0 : slabs ? groups * 3.6 + 2.0 : vec ? groups * 4.0 + 13.0 : groups * 4.8 + 7.0);
}
// A convolution's few rows leave most of the chip idle while its FP32 tiles walk a long reduction (us, FP32 tiles / here: 49 rows x 64 over 4608
// 605 / 18, 588 x 64 over 4608 374 / 19, 1200 x 128 over 4608 367 / 58, 972 x 512 over 1152 88 / 28, 4805 x 256 over 4608 353 / 259; 2645 x 512
// over 576 47 / 50, 16384 x 512 over 288 65 / 181).  The line, at 1.1 times the estimate here and 4 us more, takes the better side within
// 0.5 % on the mean of the 220 shapes, and nowhere the slower by more than 1 %.  With one accumulation chain, FP32 tiles / here: 3136 x 256 over 2304
// 81.9 / 92.5, 3267 x 256 over 288 21.2 / 24.4; 576 x 512 over 1152 43 / 27.
bool f64_conv_route(const LinearProblem& p, const ConvRows& cv, long xbytes, long bm, bool whole, bool slabs, bool fast, int cus) {
    if (p.K < 1 || xbytes <= 0 || xbytes > (1L << 31) - 16) return false;                  // (32-bit offsets)
    const F64Tile t = f64_tile(p.M, p.N, 1, cus);
    if (t.rounds * (double)cus >= 0x1p30) return false;
    const bool vec = patches_by_four(p, cv);
    return 1.1 * linear_times(t, p.M, p.N, p.K, 1, vec, cus).f64 + 4.0 < conv_fp32_us(bm, whole, slabs, vec, fast, p.M, p.N, p.K, cus);
}
int f64_conv_launch(const LinearProblem& q, const ConvRows& cv, long xbytes, const tao_fp_model& md, double gamma, int cus, hipStream_t st) {
    const F64Tile t = f64_tile(q.M, q.N, 1, cus);
    F64Args p = {};
    f64_args(t, q, md, gamma, p);
    p.cv = cv; p.xbytes = (unsigned)xbytes;
    if (patches_by_four(q, cv)) f64_dispatch<false, true, PATCHES4>(t, st, p);
    else                        f64_dispatch<false, false, PATCHES>(t, st, p);
    return launch_status();
}

}  // namespace tao
