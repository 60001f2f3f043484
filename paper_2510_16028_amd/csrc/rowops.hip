// Row-wise bound kernels: tao_bound_softmax and tao_bound_norm.
//
// One "row group" of TPR threads (a wavefront, or a whole 256-thread workgroup
// for long rows) owns one row.  The row is read once with 16-byte loads and
// kept in registers (V vectors per thread); row statistics are accumulated in
// binary64 and combined over the lanes by register moves (plus one LDS exchange when the
// group spans four wavefronts); the bound is written once.  HBM traffic is the
// algorithmic minimum: each input element read once, each tau written once.
// Rows longer than 8192 columns take the V == 0 variant, which re-reads the row
// from global memory in each pass instead of caching it.
//
// Formulas: Sec. 3.1 softmax template closed to second order; LayerNorm,
// RMSNorm, BatchNorm-affine, sum and mean (operators of App. A.3) from the
// primitive rule of Sec. 3.1 with Gamma(n-1) for the reductions (App. A.2).
#include <type_traits>
#include "tao_check.hpp"
#include "tao_device.hpp"
#include "tao_host.hpp"

namespace tao {

constexpr int kRowThreads = 256;
// One-pass checks: rows that one workgroup takes in one trip (two of short rows), so that it forms the profile itself (finish_pass): GPU us
// alone / with the finalising kernel: 4 x 768 6.4 / 10.4, 8 x 768 10.4 / 10.4 (and one launch less to enqueue), 4 x 4096, two trips,
// 14.4 / 12.6.
constexpr long alone_row_groups(long cols) { return cols <= 1024 ? 2 : 1; }

struct RowConsts {
    double u;          // unit roundoff
    double G;          // Gamma(cols - 1), upper
    double inv1mu;     // >= 1/(1-u)
    double ce_u;       // c_exp * u
    double inv1mce;    // >= 1/(1 - c_exp u)
    double cd_u;       // c_div * u
    double inv1mcd;    // >= 1/(1 - c_div u)
    double cr_u;       // c_rsqrt * u
    double eps;        // (double)(float)eps
    double inv_n;      // 1/cols (nearest; covered by the guard factor)
    double mean_f;     // c_div u / (1 - c_div u), upper
    double m;          // rounding margin of a bound of this row length (see make_consts)
    float quick_alpha; // the one-pass checks: alpha of the estimates
    int apart;         // ... and rows between those of neighbouring row groups of a workgroup (row_blocks)
};

// Factors of the final upper rounding (up32g) for a rounding margin m.
struct UpFactors {
    double mul, sub;
    __device__ __forceinline__ explicit UpFactors(double m) : mul(1.0 + 0x1p-24 + fmax(0x1p-32, 2.0 * m)), sub(1.0 + m) {}
};

// ---- reductions over the TPR threads of a row group (result in every thread) ----
template <int TPR>
__device__ __forceinline__ void group_sum(double* v, int count, double* smem) {
    for (int i = 0; i < count; ++i) v[i] = wave_sum(v[i]);
    if (TPR > kWave) {
        const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
        // every reduction of a kernel has its own 16-double slot of smem, so one barrier is enough
        if (lane == 0) for (int i = 0; i < count; ++i) smem[wave * 4 + i] = v[i];
        __syncthreads();
        for (int i = 0; i < count; ++i) {
            double s = 0;
            for (int w = 0; w < TPR / kWave; ++w) s += smem[w * 4 + i];
            v[i] = s;
        }
    }
}
template <int TPR>
__device__ __forceinline__ void group_max_or(float& m, int& flag, double* smem) {
    m = wave_max(m);
    flag = wave_or(flag);
    if (TPR > kWave) {
        const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
        if (lane == 0) { smem[wave * 4] = (double)m; smem[wave * 4 + 1] = (double)flag; }
        __syncthreads();
        float mm = -INFINITY; int ff = 0;
        for (int w = 0; w < TPR / kWave; ++w) { mm = fmaxf(mm, (float)smem[w * 4]); ff |= (int)smem[w * 4 + 1]; }
        m = mm; flag = ff;
    }
}

#define TAO_ROW_PROLOGUE                                                              \
    constexpr int RPB = kRowThreads / TPR;                                            \
    constexpr bool CACHED = (V > 0);                                                  \
    __shared__ double smem[2 * 16]; /* one slot per reduction of the kernel */        \
    const int lt = threadIdx.x % TPR;                                                 \
    const long row = (long)blockIdx.x * RPB + threadIdx.x / TPR;                      \
    const bool active = row < rows;                                                   \
    const long limit = active ? cols : 0; /* idle groups see an empty row */          \
    const long roff = active ? row * ld : 0;                                          \
    const int nv = CACHED ? V : (int)((cols + TPR * 4 - 1) / (TPR * 4));              \
    (void)smem;

#define TAO_VEC_INDEX(v) (((long)(v) * TPR + lt) * 4)

// ------------------------------------------------------------------ softmax
template <int TPR, int V>
__global__ __launch_bounds__(kRowThreads) void softmax_bound(
    const float* __restrict__ x, const float* __restrict__ y, float* __restrict__ tau,
    long rows, long cols, long ld, int vec_ok, RowConsts k) {
    TAO_ROW_PROLOGUE
    float4 xv[CACHED ? V : 1], yv[CACHED ? V : 1];
    float m = -INFINITY; int bad = 0;
    for (int v = 0; v < nv; ++v) {
        const float4 X = load4<CACHED>(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, -INFINITY);
        if (CACHED) { xv[v] = X; yv[v] = load4<true>(y + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f); }
        const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) { bad |= (e[c] != e[c]) | (e[c] == INFINITY); m = fmaxf(m, e[c]); }
    }
    group_max_or<TPR>(m, bad, smem);
    if (m == -INFINITY) bad = 1;
    // a = u(|x| + |m|) and rho = (a(1+a) + c u)/(1 - c u) as three fused multiply-adds:
    //   a = fma(u, |x|, u|m|);  rho = fma(fma(a, a, a), inv, c u inv)
    const double uam = k.u * fabs((double)m);
    const double ce_inv = k.ce_u * k.inv1mce;
    double acc[2] = {0.0, 0.0};                                  // sum q, sum rho q
    // q and rho of the cached elements are kept for the last pass only while registers allow
    // (a wavefront-wide row of 2048 columns recomputes them: six operations per element)
    constexpr bool KEEP = CACHED && V <= 4;
    double qv[KEEP ? V * 4 : 1], rv[KEEP ? V * 4 : 1];
    // masked entries (x = -inf) take |x| = 0 and y = 0: then q = 0 drops them from both sums
    // and from tau without a select on binary64 values
    auto q_rho = [&](float xe, float ye, double& q, double& rho) __attribute__((always_inline)) {
        const bool masked = xe == -INFINITY;
        const double ax = (double)(masked ? 0.f : fabsf(xe));
        const double a = fma(k.u, ax, uam);
        rho = fma(fma(a, a, a), k.inv1mce, ce_inv);
        q = (double)(masked ? 0.f : fabsf(ye)) * k.inv1mu;
    };
    for (int v = 0; v < nv; ++v) {
        const float4 X = CACHED ? xv[v] : load4(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, -INFINITY);
        const float4 Y = CACHED ? yv[v] : load4(y + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        const float xe[4] = {X.x, X.y, X.z, X.w}, ye[4] = {Y.x, Y.y, Y.z, Y.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double q, rho;
            q_rho(xe[c], ye[c], q, rho);
            acc[0] += q; acc[1] = fma(rho, q, acc[1]);
            if (KEEP) { qv[v * 4 + c] = q; rv[v * 4 + c] = rho; }
        }
    }
    group_sum<TPR>(acc, 2, smem + 16);
    const double sigma = k.G * acc[0] + (1.0 + k.G) * acc[1];
    if (!(sigma < 1.0)) bad = 1;
    // tau = q rho + q (1+rho) sfac + u y  with y = q (1-u) <= q:
    //     = q (rho (1 + sfac) + (sfac + u)); a row without a finite bound gets NaN through the
    // two row constants (0 * NaN = NaN also covers its masked entries)
    const double sfac = sigma / (1.0 - sigma);
    const double w1 = bad ? NAN : 1.0 + sfac;
    const double w0 = bad ? NAN : sfac + k.u;
    // (an error of the sums enters sfac amplified by 1/(1 - sigma): the margin follows)
    const UpFactors up(k.m * (1.0 + 2.0 / (1.0 - sigma)));
    for (int v = 0; v < nv; ++v) {
        float4 X = make_float4(0.f, 0.f, 0.f, 0.f), Y = X;
        if (!CACHED) {
            X = load4(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, -INFINITY);
            Y = load4(y + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        } else if (!KEEP) {
            X = xv[v]; Y = yv[v];
        }
        const float xe[4] = {X.x, X.y, X.z, X.w}, ye[4] = {Y.x, Y.y, Y.z, Y.w};
        float te[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double q, rho;
            if (KEEP) { q = qv[v * 4 + c]; rho = rv[v * 4 + c]; }
            else q_rho(xe[c], ye[c], q, rho);
            te[c] = up32g(q * fma(rho, w1, w0), up.mul, up.sub);
        }
        store4(tau + roff, TAO_VEC_INDEX(v), limit, vec_ok, make_float4(te[0], te[1], te[2], te[3]));
    }
}

// ---- softmax bound checked in registers (the bound is never stored) --------------------------
// Same arithmetic as softmax_bound element by element (a row's sums in an order of their own, see norm_check), followed by the leaf check of
// tao_check_and_profile on (claimed, y, tau) with tau first rounded to binary32 as it would have
// been stored.  Workgroups of 1024 threads walk the rows (1024 / TPR at a time), keep the
// histogram of relative errors in LDS and leave one partial per workgroup, like the streaming
// check pass; the same finalising kernel turns the partials into the profile.  HBM traffic:
// x, y and claimed read once (12 B per element), nothing written.
// QUICK: most elements are settled in binary32 (QuickCheck), with a lower estimate of the bound; the
// others form the bound in binary64 as softmax_bound does.  FULL: aligned rows of whole vectors.
// What bounds it: HBM, 5.6 TB/s on 65536 causal or dense rows of 2048 columns (462 -> 286 us, 16384 x 1024 83 -> 50 us,
// 8192 x 4096 131 -> 110 us).  Before, a wavefront waited for each of its loads (a test for the row's
// end around every one of them), four wavefronts met at three barriers per row, and an element took 58 vector instructions.
template <int TPR>
__device__ __forceinline__ void wide_group_sum(double* v, int count, double* smem) {
    constexpr int STEPS = TPR >= kWave ? 6 : TPR == 32 ? 5 : 4;       // (a row group is 16 lanes at least)
    for (int i = 0; i < count; ++i) v[i] = wave_all<0, STEPS>(v[i], [](double a, double b) { return a + b; });
    if (TPR > kWave) {
        const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
        const int first = (threadIdx.x / TPR) * (TPR / kWave);       // first wavefront of this row group
        if (lane == 0) for (int i = 0; i < count; ++i) smem[wave * 4 + i] = v[i];
        __syncthreads();
        for (int i = 0; i < count; ++i) {
            double s = 0;
            for (int w = 0; w < TPR / kWave; ++w) s += smem[(first + w) * 4 + i];
            v[i] = s;
        }
    }
}
template <int TPR>
__device__ __forceinline__ void wide_group_max_or(float& m, int& flag, double* smem) {
    m = wave_max(m);
    flag = wave_or(flag);
    if (TPR > kWave) {
        const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
        const int first = (threadIdx.x / TPR) * (TPR / kWave);
        if (lane == 0) { smem[wave * 4] = (double)m; smem[wave * 4 + 1] = (double)flag; }
        __syncthreads();
        float mm = -INFINITY; int ff = 0;
        for (int w = 0; w < TPR / kWave; ++w) { mm = fmaxf(mm, (float)smem[(first + w) * 4]); ff |= (int)smem[(first + w) * 4 + 1]; }
        m = mm; flag = ff;
    }
}

// The four values of a thread's vector, loaded without a branch: from clamped positions that exist; row_fill then
// replaces those that are not the thread's.  (Behind a test for the row's end every load waited for the one before it.)
// WHOLE: 16-byte aligned rows of whole vectors, four consecutive columns from idx on.  ANY: four consecutive columns by one 16-byte load
// as well, at any alignment, of rows of four columns or more; a vector that the row's end cuts is read from the row's last four columns, of which
// the first belong to the vector before it.  SINGLE: the columns idx, idx + step, ..., with step the row group's size: neighbouring threads
// read neighbouring columns, four loads to a vector, but a row that ends early in its last vectors is spread more evenly (row_form).
// last: the last position of a vector or (SINGLE) value.
enum { SINGLE, WHOLE, ANY };
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
template <int FULL, bool STREAM, int STEP, class Idx>
__device__ __forceinline__ float4 row_vec(const float* __restrict__ row, Idx idx, Idx last) {
    if (FULL == WHOLE) {
        const float4* p = reinterpret_cast<const float4*>(row + min(idx, last));
        return STREAM ? ntload4(p) : *p;
    }
    if (FULL == ANY) {
        const floatx4u* p = reinterpret_cast<const floatx4u*>(row + min(idx, last));
        if (STREAM) return __builtin_bit_cast(float4, __builtin_nontemporal_load(p));
        return __builtin_bit_cast(float4, *p);
    }
    return make_float4(row[min(idx, last)], row[min((Idx)(idx + STEP), last)], row[min((Idx)(idx + 2 * STEP), last)], row[min((Idx)(idx + 3 * STEP), last)]);
}
// Whether value c of the vector at idx is the thread's; and whether all four are.
template <int FULL, int STEP, class Idx>
__device__ __forceinline__ bool row_has(Idx idx, Idx limit, Idx last, int c) {
    return FULL == WHOLE ? idx < limit : FULL == ANY ? idx < limit && idx - min(idx, last) <= (Idx)c : idx + c * STEP < limit;
}
// How many of the vector at idx, inside the row, belong to the one before; and a bit for each that does not.
template <int FULL, class Idx>
__device__ __forceinline__ unsigned row_others(Idx idx, Idx last) { return FULL == ANY ? (unsigned)(idx - min(idx, last)) : 0u; }
// A vector's claims, outputs and estimates for quick_check_four.
template <int FULL>
__device__ __forceinline__ void leave_others(unsigned others, floatv4& c, floatv4& y, floatv4& at) {
    if (FULL != ANY) return;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const bool other = (unsigned)i < others;
        c[i] = other ? 0.f : c[i]; y[i] = other ? 0.f : y[i]; at[i] = other ? 0.f : at[i];
    }
}
template <int FULL, int STEP, class Idx>
__device__ __forceinline__ float4 row_fill(float4 r, Idx idx, Idx limit, Idx last, float fill) {
    auto has = [&](int c) __attribute__((always_inline)) { return row_has<FULL, STEP>(idx, limit, last, c); };
    return make_float4(has(0) ? r.x : fill, has(1) ? r.y : fill, has(2) ? r.z : fill, has(3) ? r.w : fill);
}
#define TAO_VEC_IDX(v) (FULL ? ((Idx)(v) * TPR + lt) * 4 : (Idx)(v) * (4 * TPR) + lt)

template <int TPR, int V, int FULL, bool QUICK>
__global__ __launch_bounds__(kCheckThreads) void softmax_check(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ claimed,
    long rows, long cols, long ld, RowConsts k, double alpha, double eps_rel,
    PassOut pass) {
    using Idx = typename std::conditional<(V > 0), int, long>::type;     // columns: a cached row has at most 8192
    constexpr bool CACHED = (V > 0), CLAIMS = CACHED && V <= 4 && (QUICK || V == 1);   // claims requested with the row
    // the next rows are requested while these are worked on, where the registers allow it
    constexpr bool PIPE = V == 1 || (V == 2 && TPR < 1024);
    __shared__ unsigned int hist[kBins * kReplicas];
    __shared__ unsigned int red[kRedWords];
    __shared__ double smem[2 * 4 * (kCheckThreads / kWave)];       // one slot per reduction of a row
    __shared__ unsigned int largest;
    const int tid = threadIdx.x;
    const QuickCheck qc(k.quick_alpha, eps_rel);
    unsigned known = 0;
    for (int i = tid; i < kBins * kReplicas; i += kCheckThreads) hist[i] = 0;
    if (tid == 0) largest = 0;
    __syncthreads();
    ThreadAcc acc_chk;
    unsigned beyond = 0;                                     // counted in bin 0, but another vector's
    const int rep = tid & (kReplicas - 1);
    const int nv = CACHED ? V : (int)((cols + TPR * 4 - 1) / (TPR * 4));
    // Row group s of workgroup b, of G: rows b + s G, b + (s + all) G, ..., so that what is left for the last trip falls to all workgroups; or, k.apart being 1,
    // neighbouring rows.  A wavefront of whole rows goes by its first one, a workgroup whose row groups meet at barriers by the first of all.
    // (OWN: no lane of a wavefront asks whether there is its row; with four vectors the scheduling that comes of it is worse: 8192 x 1024 36.0 us, 30.8 without.)
    constexpr bool OWN = TPR == kWave && V != 4;
    const int lead = TPR <= kWave ? __builtin_amdgcn_readfirstlane(tid / kWave) * (kWave / TPR) : 0;
    const long trip = (long)gridDim.x * (kCheckThreads / TPR), mine = (long)k.apart * (tid / TPR - lead);
    const long first = (long)blockIdx.x * (k.apart == 1 ? kCheckThreads / TPR : 1) + (long)k.apart * lead;
    float4 xn[PIPE ? V : 1], yn[PIPE ? V : 1], cn[PIPE && CLAIMS ? V : 1];
    auto request = [&](long rb, float4* xr, float4* yr, float4* cr) __attribute__((always_inline)) {
        int lt = tid % TPR;
        asm volatile("" : "+v"(lt));
        const long row = OWN ? rb : rb + mine, roff = (OWN || row < rows ? row : rows - 1) * ld;
        const Idx last = (Idx)cols - (FULL ? 4 : 1);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            xr[v] = row_vec<FULL, true, TPR>(x + roff, TAO_VEC_IDX(v), last);
            yr[v] = row_vec<FULL, true, TPR>(y + roff, TAO_VEC_IDX(v), last);
            if (CLAIMS) cr[v] = row_vec<FULL, true, TPR>(claimed + roff, TAO_VEC_IDX(v), last);
        }
    };
    if (PIPE && first < rows) request(first, xn, yn, cn);
    // (every thread of a workgroup takes the same number of trips where the reductions hold barriers)
    for (long rb = first; rb < rows; rb += trip) {
        int lt = tid % TPR;
        if (CACHED) asm volatile("" : "+v"(lt));            // (positions are formed anew for every row and pass: hoisted they would take the registers of the row)
        const long row = OWN ? rb : rb + mine;
        const bool active = OWN || row < rows;
        const Idx limit = active ? (Idx)cols : 0, last = (Idx)cols - (FULL ? 4 : 1);
        const long roff = (active ? row : rows - 1) * ld;
        float4 xv[CACHED ? V : 1], yv[CACHED ? V : 1], cv[CLAIMS ? V : 1];
        float m = -INFINITY; int bad = 0;
        if (PIPE) {
#pragma unroll
            for (int v = 0; v < nv; ++v) {
                xv[v] = xn[v]; yv[v] = yn[v];
                if (CLAIMS) cv[v] = cn[v];
            }
            if (rb + trip < rows) request(rb + trip, xn, yn, cn);
            __builtin_amdgcn_sched_barrier(0);
        } else if (CACHED) {
#pragma unroll
            for (int v = 0; v < nv; ++v) {
                xv[v] = row_vec<FULL, true, TPR>(x + roff, TAO_VEC_IDX(v), last);
                yv[v] = row_vec<FULL, true, TPR>(y + roff, TAO_VEC_IDX(v), last);
                if (CLAIMS) cv[v] = row_vec<FULL, true, TPR>(claimed + roff, TAO_VEC_IDX(v), last);
            }
            __builtin_amdgcn_sched_barrier(0);               // (all requests leave before the first is waited for)
        }
        for (int v = 0; v < nv; ++v) {
            const float4 X = row_fill<FULL, TPR>(CACHED ? xv[v] : row_vec<FULL, false, TPR>(x + roff, TAO_VEC_IDX(v), last), TAO_VEC_IDX(v), limit, last, -INFINITY);
            if (CACHED) { xv[v] = X; yv[v] = row_fill<FULL, TPR>(yv[v], TAO_VEC_IDX(v), limit, last, 0.f); }
            const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) { bad |= (e[c] != e[c]) | (e[c] == INFINITY); m = fmaxf(m, e[c]); }
        }
        wide_group_max_or<TPR>(m, bad, smem);
        if (m == -INFINITY) bad = 1;
        const double uam = k.u * fabs((double)m);
        const double ce_inv = k.ce_u * k.inv1mce;
        double acc[2] = {0.0, 0.0};
        auto q_rho = [&](float xe, float ye, double& q, double& rho) __attribute__((always_inline)) {
            const bool masked = xe == -INFINITY;
            const double ax = (double)(masked ? 0.f : fabsf(xe));
            const double a = fma(k.u, ax, uam);
            rho = fma(fma(a, a, a), k.inv1mce, ce_inv);
            q = (double)(masked ? 0.f : fabsf(ye)) * k.inv1mu;
        };
        for (int v = 0; v < nv; ++v) {
            const float4 X = CACHED ? xv[v] : row_fill<FULL, TPR>(row_vec<FULL, false, TPR>(x + roff, TAO_VEC_IDX(v), last), TAO_VEC_IDX(v), limit, last, -INFINITY);
            const float4 Y = CACHED ? yv[v] : row_fill<FULL, TPR>(row_vec<FULL, false, TPR>(y + roff, TAO_VEC_IDX(v), last), TAO_VEC_IDX(v), limit, last, 0.f);
            const float xe[4] = {X.x, X.y, X.z, X.w}, ye[4] = {Y.x, Y.y, Y.z, Y.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                double q, rho;
                q_rho(xe[c], ye[c], q, rho);
                acc[0] += q; acc[1] = fma(rho, q, acc[1]);
            }
        }
        wide_group_sum<TPR>(acc, 2, smem + 4 * (kCheckThreads / kWave));
        const double sigma = k.G * acc[0] + (1.0 + k.G) * acc[1];
        if (!(sigma < 1.0)) bad = 1;
        const double sfac = sigma / (1.0 - sigma);
        const double w1 = bad ? NAN : 1.0 + sfac;
        const double w0 = bad ? NAN : sfac + k.u;
        const UpFactors up(k.m * (1.0 + 2.0 / (1.0 - sigma)));
        // alpha tau = |y| (rho w1 + w0) from below, in binary32 (rho held finite: a mask of the lowest finite value
        // has no square there)
        const float w1f = (float)(w1 * k.inv1mu) * qc.alpha, w0f = (float)(w0 * k.inv1mu) * qc.alpha;
        const float uf = (float)k.u, uamf = (float)uam, invf = (float)k.inv1mce, cef = (float)ce_inv;
        if (QUICK) known = newest(&largest);
        if (CACHED) asm volatile("" : "+v"(lt));
        float4 next = make_float4(0.f, 0.f, 0.f, 0.f);       // the next vector's claims are on their way while one is checked
        if (!CLAIMS) next = row_vec<FULL, true, TPR>(claimed + roff, TAO_VEC_IDX(0), last);
        for (int v = 0; v < nv; ++v) {
            const Idx idx = TAO_VEC_IDX(v);
            const float4 C = CLAIMS ? cv[v] : next;
            if (!CLAIMS && v + 1 < nv) next = row_vec<FULL, true, TPR>(claimed + roff, TAO_VEC_IDX(v + 1), last);
            if (idx >= limit) continue;
            const float4 X = CACHED ? xv[v] : row_vec<FULL, false, TPR>(x + roff, idx, last);
            const float4 Y = CACHED ? yv[v] : row_vec<FULL, false, TPR>(y + roff, idx, last);
            floatv4 xe = {X.x, X.y, X.z, X.w}, ye = {Y.x, Y.y, Y.z, Y.w}, ce = {C.x, C.y, C.z, C.w};
            asm volatile("" : "+v"(xe), "+v"(ye));           // (keeps the first pass's binary64 values from living on until here)
            auto tau = [&](int c) __attribute__((always_inline)) {
                double q, rho;
                q_rho(xe[c], ye[c], q, rho);
                return up32g(q * fma(rho, w1, w0), up.mul, up.sub);
            };
            const unsigned others = row_others<FULL>(idx, last), own = 15u & 15u << others;
            if (FULL != SINGLE || idx + 3 * TPR < limit) {
                if (!QUICK) {
                    const float c4[4] = {ce[0], ce[1], ce[2], ce[3]}, y4[4] = {ye[0], ye[1], ye[2], ye[3]};
                    const float t4[4] = {tau(0), tau(1), tau(2), tau(3)};
                    check_four(c4, y4, t4, alpha, eps_rel, hist, rep, acc_chk, own);
                    continue;
                }
                floatv4 at;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float a = fmaf(uf, fabsf(xe[c]), uamf);
                    const float rho = fminf(fmaf(fmaf(a, a, a), invf, cef), 0x1p60f);
                    at[c] = (xe[c] == -INFINITY ? 0.f : fabsf(ye[c])) * fmaf(rho, w1f, w0f);
                }
                leave_others<FULL>(others, ce, ye, at);
                if (quick_check_four<(V == 1 || (V == 2 && TPR < 1024))>(ce, ye, at, tau, qc, alpha, eps_rel, hist, rep, acc_chk, &largest, known, known != 0, own)) beyond += others;
                continue;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (!row_has<FULL, TPR>(idx, limit, last, c)) continue;
                check_one(ce[c], ye[c], tau(c), alpha, eps_rel, hist, rep, acc_chk);
            }
        }
    }
    if (FULL == ANY && QUICK && beyond) atomicSub(&hist[rep], beyond);
    __syncthreads();
    finish_pass(hist, acc_chk, red, pass);
}

// tail shared by LayerNorm and RMSNorm: from v*, E_v to (r*, E_r, R); ok = finite bound
// amp: how much a relative error of the row sums is amplified on its way into E_r (the sums enter
// through the difference w_lo = w - E_w, and E_r falls with w_lo at most like its power -3/2)
__device__ __forceinline__ bool rsqrt_tail(double vstar, double E_v, const RowConsts& k,
                                           double& rs, double& E_r, double& R, double& amp) {
    const double w = vstar + k.eps;
    const double E_w = (E_v + k.u * w) * k.inv1mu;
    const double w_lo = w - E_w;
    const bool ok = w_lo > 0.0;
    amp = (w + E_w) / w_lo;
    const double inv_s = 1.0 / sqrt(w_lo);
    const double inv_s3 = inv_s / w_lo;
    E_r = 0.5 * E_w * inv_s3 + k.cr_u * inv_s;
    rs = 1.0 / sqrt(w);
    R = rs + E_r;
    return ok;
}

// ------------------------------------------------------------------ LayerNorm
// Chain of the template (E_s, E_mu, E_d, D, E_q, Q, E_t, E_v, E_w, w_lo, E_r, R, E_h, H, E_p).
// Per element only |d| = |x - mu| varies, and everything downstream is a polynomial in it with
// non-negative coefficients:
//   E_d = u' |d| + E'      (u' = u/(1-u), E' = E_mu/(1-u));   D = |d| + E_d = (1+u')|d| + E'
// so the two sums the variance bound needs,
//   sum Q   = (1+u) sum D^2,   sum E_q = sum E_d(|d| + D) + u sum D^2,
// follow from n, sum|d| and sum d^2, and the per-element tail
//   E_p/|g| = (1+u) E_h + u r|d|,  E_h = D (E_r + u R) + r E_d
// collapses to K1 |d| + K0.  Same real-number formula as the step-by-step chain; the different
// binary64 rounding (a few 2^-53) is covered by the rounding margin of up32g.
// From E_mu, sum|d|, sum d^2 to the per-element coefficients: E_p/|g| = K1 |d| + K0.
__device__ __forceinline__ void layernorm_tail(double E_mu, double s_ad, double s_d2, double n, const RowConsts& k,
                                               double& K1, double& K0, double& amp, double* rs_out = nullptr) {
    const double up = k.u * k.inv1mu, Ep = E_mu * k.inv1mu;       // u', E'
    const double c1 = 1.0 + up;
    const double sD2 = c1 * c1 * s_d2 + 2.0 * c1 * Ep * s_ad + n * Ep * Ep;           // sum D^2
    const double sEdD = up * (1.0 + c1) * s_d2 + Ep * (up + 1.0 + c1) * s_ad + n * Ep * Ep;  // sum E_d(|d|+D)
    const double E_t = k.G * (1.0 + k.u) * sD2 + sEdD + k.u * sD2;
    const double vstar = s_d2 * k.inv_n;
    const double E_v = (E_t * k.inv_n + k.cd_u * vstar) * k.inv1mcd;
    double rs, E_r, R;
    const bool ok = rsqrt_tail(vstar, E_v, k, rs, E_r, R, amp);
    const double hc = E_r + k.u * R;                              // E_h = D hc + r E_d
    K1 = (1.0 + k.u) * (c1 * hc + rs * up) + k.u * rs;
    K0 = ok ? (1.0 + k.u) * Ep * (hc + rs) : NAN;                 // NaN row when the bound is not finite
    if (rs_out) *rs_out = rs;
}

// GROUPED (GroupNorm): a row is one (sample, group) of a channel-major tensor, cols = channels per
// group x positions; column c takes the affine scale of channel (row % groups) * cpg + c / hw.
struct GroupGeom { unsigned hw, cpg, groups; };
// NOY: the caller has no re-executed output; the fresh-rounding term u|y| is then taken at the upper
// bound Y = (|d| r |g| + E_p + |b|)(1+u) of |y| over all canonical executions (b: the additive term,
// which enters a bound only here).
template <int TPR, int V, bool GROUPED, bool NOY = false>
__device__ __forceinline__ void layernorm_body(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ g,
    float* __restrict__ tau, long rows, long cols, long ld, int vec_ok, int vec_g, const RowConsts& k,
    GroupGeom gg, const float* __restrict__ b = nullptr, int vec_b = 0) {
    static_assert(!(NOY && GROUPED), "GroupNorm takes the re-executed output");
    TAO_ROW_PROLOGUE
    // the four scales of the vector that starts at column idx
    const float* gb = (GROUPED && g && active) ? g + (unsigned long)(row % (long)gg.groups) * gg.cpg : g;
    auto scales = [&](long idx) {
        if (!g) return make_float4(1.f, 1.f, 1.f, 1.f);
        if (!GROUPED) return load4(g, idx, limit, vec_g, 1.f);
        float ge[4] = {1.f, 1.f, 1.f, 1.f};
        if (idx < limit) {
            unsigned ch = (unsigned)idx / gg.hw, rem = (unsigned)idx - ch * gg.hw;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (idx + c < limit) ge[c] = gb[ch];
                if (++rem == gg.hw) { rem = 0; ++ch; }
            }
        }
        return make_float4(ge[0], ge[1], ge[2], ge[3]);
    };
    // a cached row also requests y and g up front: their latency then overlaps the reductions
    constexpr bool CACHE_Y = CACHED;
    float4 xv[CACHED ? V : 1], yv[CACHE_Y ? V : 1], gv[CACHE_Y ? V : 1];
    double a1[2] = {0.0, 0.0};                                   // sum x, sum |x|
    for (int v = 0; v < nv; ++v) {
        const float4 X = load4<CACHED>(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        if (CACHED) xv[v] = X;
        if (CACHE_Y) {
            // (without y the registers hold |b| instead)
            yv[v] = NOY ? (b ? load4(b, TAO_VEC_INDEX(v), limit, vec_b, 0.f) : make_float4(0.f, 0.f, 0.f, 0.f))
                        : load4<true>(y + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
            gv[v] = scales(TAO_VEC_INDEX(v));
        }
        const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) { a1[0] += (double)e[c]; a1[1] += (double)fabsf(e[c]); }
    }
    group_sum<TPR>(a1, 2, smem);
    const double n = (double)cols;
    const double mu = a1[0] * k.inv_n;
    const double E_mu = ((k.G * a1[1]) * k.inv_n + k.cd_u * fabs(mu)) * k.inv1mcd;
    double a2[2] = {0.0, 0.0};                                   // sum |d|, sum d^2
    for (int v = 0; v < nv; ++v) {
        const float4 X = CACHED ? xv[v] : load4(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            // padding lanes (beyond the row) hold x = 0 and must not count: d = 0 for them
            const double d = (TAO_VEC_INDEX(v) + c < limit) ? (double)e[c] - mu : 0.0;
            a2[0] += fabs(d);
            a2[1] = fma(d, d, a2[1]);
        }
    }
    group_sum<TPR>(a2, 2, smem + 16);
    double K1, K0, amp, rs;
    layernorm_tail(E_mu, a2[0], a2[1], n, k, K1, K0, amp, &rs);
    const UpFactors up(k.m * (1.0 + 2.0 * amp));
    for (int v = 0; v < nv; ++v) {
        const float4 X = CACHED ? xv[v] : load4(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        const float4 Y = CACHE_Y ? yv[v]
                       : NOY ? (b ? load4(b, TAO_VEC_INDEX(v), limit, vec_b, 0.f) : make_float4(0.f, 0.f, 0.f, 0.f))
                             : load4<true>(y + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        const float4 Gv = CACHE_Y ? gv[v] : scales(TAO_VEC_INDEX(v));
        const float xe[4] = {X.x, X.y, X.z, X.w}, ye[4] = {Y.x, Y.y, Y.z, Y.w};
        const float ge[4] = {Gv.x, Gv.y, Gv.z, Gv.w};
        float te[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double ad = fabs((double)xe[c] - mu);
            const double ag = (double)fabsf(ge[c]);
            const double ep = ag * fma(K1, ad, K0);
            // |y|, or its upper bound (|d| r |g| + E_p + |b|)(1+u)
            const double Yb = NOY ? (ad * rs * ag + ep + (double)fabsf(ye[c])) * (1.0 + k.u) : (double)fabsf(ye[c]);
            te[c] = up32g(fma(k.u, Yb, ep), up.mul, up.sub);
        }
        store4(tau + roff, TAO_VEC_INDEX(v), limit, vec_ok, make_float4(te[0], te[1], te[2], te[3]));
    }
}
template <int TPR, int V>
__global__ __launch_bounds__(kRowThreads) void layernorm_bound(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ g,
    float* __restrict__ tau, long rows, long cols, long ld, int vec_ok, int vec_g, RowConsts k) {
    layernorm_body<TPR, V, false>(x, y, g, tau, rows, cols, ld, vec_ok, vec_g, k, GroupGeom());
}
template <int TPR, int V>
__global__ __launch_bounds__(kRowThreads) void layernorm_bound_noy(
    const float* __restrict__ x, const float* __restrict__ g, const float* __restrict__ b,
    float* __restrict__ tau, long rows, long cols, long ld, int vec_ok, int vec_g, int vec_b, RowConsts k) {
    layernorm_body<TPR, V, false, true>(x, nullptr, g, tau, rows, cols, ld, vec_ok, vec_g, k, GroupGeom(), b, vec_b);
}
template <int TPR, int V>
__global__ __launch_bounds__(kRowThreads) void groupnorm_bound(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ g,
    float* __restrict__ tau, long rows, long cols, long ld, int vec_ok, RowConsts k, GroupGeom gg) {
    layernorm_body<TPR, V, true>(x, y, g, tau, rows, cols, ld, vec_ok, 0, k, gg);
}

// ---- GroupNorm rows longer than the cached variants hold: the row is cut into chunks of
// kChunk columns, one workgroup each, so that a few very long rows still fill the chip.  Three
// passes, each reading its chunk once: (a) sum x, sum |x|; (b) the mean from the partials of
// (a), then sum |d|, sum d^2; (c) all four sums, the row's coefficients, the bound.  Partials
// live in a caller-supplied workspace, four binary64 values per (row, chunk); every workgroup
// adds them up in the same order, so all chunks of a row see identical row constants.
constexpr long kSplitMaxRows = 512;                            // from here on one workgroup per row
constexpr int kChunkVecs = 8;                                  // float4 per thread
constexpr long kChunk = (long)kRowThreads * kChunkVecs * 4;    // 8192 columns

struct ChunkPos { long row, c0, limit; int s; };
__device__ __forceinline__ ChunkPos chunk_pos(long cols, unsigned nchunk) {
    ChunkPos p;
    p.row = blockIdx.x / nchunk; p.s = (int)(blockIdx.x % nchunk);
    p.c0 = (long)p.s * kChunk;
    p.limit = cols - p.c0 < kChunk ? cols - p.c0 : kChunk;      // columns of this chunk
    return p;
}
// sum over the chunks of a row of partial `which` .. `which + 1` (same order in every workgroup)
__device__ __forceinline__ void chunk_totals(const double* __restrict__ part, unsigned nchunk, int which,
                                             double* out2, double* smem) {
    double a[2] = {0.0, 0.0};
    for (unsigned s = threadIdx.x; s < nchunk; s += kRowThreads) { a[0] += part[s * 4 + which]; a[1] += part[s * 4 + which + 1]; }
    group_sum<kRowThreads>(a, 2, smem);
    out2[0] = a[0]; out2[1] = a[1];
}
__global__ __launch_bounds__(kRowThreads) void groupnorm_sums_a(const float* __restrict__ x, double* __restrict__ ws,
                                                                long cols, unsigned nchunk, int vec_ok) {
    __shared__ double smem[16];
    const ChunkPos p = chunk_pos(cols, nchunk);
    const float* xr = x + p.row * cols + p.c0;
    double a[2] = {0.0, 0.0};
#pragma unroll
    for (int v = 0; v < kChunkVecs; ++v) {
        const float4 X = load4<false>(xr, ((long)v * kRowThreads + threadIdx.x) * 4, p.limit, vec_ok, 0.f);
        const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) { a[0] += (double)e[c]; a[1] += (double)fabsf(e[c]); }
    }
    group_sum<kRowThreads>(a, 2, smem);
    if (threadIdx.x == 0) { double* o = ws + ((long)blockIdx.x) * 4; o[0] = a[0]; o[1] = a[1]; }
}
__global__ __launch_bounds__(kRowThreads) void groupnorm_sums_b(const float* __restrict__ x, double* __restrict__ ws,
                                                                long cols, unsigned nchunk, int vec_ok, RowConsts k) {
    __shared__ double smem[32];
    const ChunkPos p = chunk_pos(cols, nchunk);
    double t[2];
    chunk_totals(ws + p.row * nchunk * 4, nchunk, 0, t, smem);
    const double mu = t[0] * k.inv_n;
    const float* xr = x + p.row * cols + p.c0;
    double a[2] = {0.0, 0.0};
#pragma unroll
    for (int v = 0; v < kChunkVecs; ++v) {
        const long idx = ((long)v * kRowThreads + threadIdx.x) * 4;
        const float4 X = load4<false>(xr, idx, p.limit, vec_ok, 0.f);
        const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double d = (idx + c < p.limit) ? (double)e[c] - mu : 0.0;
            a[0] += fabs(d);
            a[1] = fma(d, d, a[1]);
        }
    }
    group_sum<kRowThreads>(a, 2, smem + 16);
    if (threadIdx.x == 0) { double* o = ws + ((long)blockIdx.x) * 4; o[2] = a[0]; o[3] = a[1]; }
}
__global__ __launch_bounds__(kRowThreads) void groupnorm_apply(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ g, float* __restrict__ tau,
    const double* __restrict__ ws, long cols, unsigned nchunk, int vec_ok, RowConsts k, GroupGeom gg) {
    __shared__ double smem[32];
    const ChunkPos p = chunk_pos(cols, nchunk);
    double t1[2], t2[2];
    chunk_totals(ws + p.row * nchunk * 4, nchunk, 0, t1, smem);
    chunk_totals(ws + p.row * nchunk * 4, nchunk, 2, t2, smem + 16);
    const double n = (double)cols;
    const double mu = t1[0] * k.inv_n;
    const double E_mu = ((k.G * t1[1]) * k.inv_n + k.cd_u * fabs(mu)) * k.inv1mcd;
    double K1, K0, amp;
    layernorm_tail(E_mu, t2[0], t2[1], n, k, K1, K0, amp);
    const UpFactors up(k.m * (1.0 + 2.0 * amp));
    const long roff = p.row * cols + p.c0;
    const float* gb = g ? g + (unsigned long)(p.row % (long)gg.groups) * gg.cpg : nullptr;
#pragma unroll 2
    for (int v = 0; v < kChunkVecs; ++v) {
        const long idx = ((long)v * kRowThreads + threadIdx.x) * 4;
        if (idx >= p.limit) break;
        const float4 X = load4<true>(x + roff, idx, p.limit, vec_ok, 0.f);
        const float4 Y = load4<true>(y + roff, idx, p.limit, vec_ok, 0.f);
        float ge[4] = {1.f, 1.f, 1.f, 1.f};
        if (gb) {
            const unsigned col = (unsigned)(p.c0 + idx);
            unsigned ch = col / gg.hw, rem = col - ch * gg.hw;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (idx + c < p.limit) ge[c] = gb[ch];
                if (++rem == gg.hw) { rem = 0; ++ch; }
            }
        }
        const float xe[4] = {X.x, X.y, X.z, X.w}, ye[4] = {Y.x, Y.y, Y.z, Y.w};
        float te[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double ad = fabs((double)xe[c] - mu);
            const double ep = (double)fabsf(ge[c]) * fma(K1, ad, K0);
            te[c] = up32g(fma(k.u, (double)fabsf(ye[c]), ep), up.mul, up.sub);
        }
        store4(tau + roff, idx, p.limit, vec_ok, make_float4(te[0], te[1], te[2], te[3]));
    }
}

// ------------------------------------------------------------------ RMSNorm
// NOY: no re-executed output; u|y| is taken at Y = |x g| R (1+u)^2 >= |y|.
template <int TPR, int V, bool NOY>
__device__ __forceinline__ void rmsnorm_body(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ g,
    float* __restrict__ tau, long rows, long cols, long ld, int vec_ok, int vec_g, const RowConsts& k) {
    TAO_ROW_PROLOGUE
    float4 xv[CACHED ? V : 1], yv[(CACHED && !NOY) ? V : 1], gv[CACHED ? V : 1];
    double a1[1] = {0.0};
    for (int v = 0; v < nv; ++v) {
        const float4 X = load4<CACHED>(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        if (CACHED) {
            xv[v] = X;
            if (!NOY) yv[v] = load4<true>(y + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
            gv[v] = g ? load4(g, TAO_VEC_INDEX(v), limit, vec_g, 1.f) : make_float4(1.f, 1.f, 1.f, 1.f);
        }
        const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) a1[0] += (double)e[c] * (double)e[c];
    }
    group_sum<TPR>(a1, 1, smem);
    const double E_t = (k.G * (1.0 + k.u) + k.u) * a1[0];
    const double vstar = a1[0] * k.inv_n;
    const double E_v = (E_t * k.inv_n + k.cd_u * vstar) * k.inv1mcd;
    double rs, E_r, R, amp;
    const bool ok = rsqrt_tail(vstar, E_v, k, rs, E_r, R, amp);
    const double f = E_r + k.u * R;
    const double fy = k.u * R * (1.0 + k.u) * (1.0 + k.u);           // NOY: u Y / |x g|
    const UpFactors up(k.m * (1.0 + 2.0 * amp));
    for (int v = 0; v < nv; ++v) {
        const float4 X = CACHED ? xv[v] : load4(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        const float4 Y = NOY ? make_float4(0.f, 0.f, 0.f, 0.f)
                             : (CACHED ? yv[v] : load4<true>(y + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f));
        const float4 Gv = CACHED ? gv[v] : (g ? load4(g, TAO_VEC_INDEX(v), limit, vec_g, 1.f) : make_float4(1.f, 1.f, 1.f, 1.f));
        const float xe[4] = {X.x, X.y, X.z, X.w}, ye[4] = {Y.x, Y.y, Y.z, Y.w};
        const float ge[4] = {Gv.x, Gv.y, Gv.z, Gv.w};
        float te[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double xg = fabs((double)xe[c] * (double)ge[c]);
            const double t = NOY ? xg * f + xg * fy : xg * f + k.u * fabs((double)ye[c]);
            te[c] = ok ? up32g(t, up.mul, up.sub) : NAN;
        }
        store4(tau + roff, TAO_VEC_INDEX(v), limit, vec_ok, make_float4(te[0], te[1], te[2], te[3]));
    }
}
template <int TPR, int V>
__global__ __launch_bounds__(kRowThreads) void rmsnorm_bound(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ g,
    float* __restrict__ tau, long rows, long cols, long ld, int vec_ok, int vec_g, RowConsts k) {
    rmsnorm_body<TPR, V, false>(x, y, g, tau, rows, cols, ld, vec_ok, vec_g, k);
}
template <int TPR, int V>
__global__ __launch_bounds__(kRowThreads) void rmsnorm_bound_noy(
    const float* __restrict__ x, const float* __restrict__ g,
    float* __restrict__ tau, long rows, long cols, long ld, int vec_ok, int vec_g, RowConsts k) {
    rmsnorm_body<TPR, V, true>(x, nullptr, g, tau, rows, cols, ld, vec_ok, vec_g, k);
}

// LayerNorm / RMSNorm bounds checked on the spot: the structure of softmax_check (1024-thread
// workgroups that walk the rows, kCheckThreads / TPR rows at a time, one partial histogram each)
// with the arithmetic of layernorm_body / rmsnorm_bound per element.  A row's sums may be added in another order (row groups
// of another size, ragged rows read column by column): the bound compared is the binary32 value the bound kernels
// store or, rarely, its neighbour.  FULL, QUICK: as there.
// What bounds it: HBM for many rows (32768 x 768: LayerNorm 180 -> 90 us, RMSNorm 128 -> 65 us; LayerNorm 8192 x 2048 170 -> 67 us,
// whose rows are now kept instead of read again), the chain of one row -- loads, two reductions, a square root and divisions in
// binary64 -- for few (2048 x 4096 RMSNorm 34.4 -> 29.7 us with its finalising launch), which is why the next rows are requested early.
template <bool RMS, int TPR, int V, int FULL, bool QUICK>
__global__ __launch_bounds__(kCheckThreads) void norm_check(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ g, const float* __restrict__ claimed,
    long rows, long cols, long ld, RowConsts k, double alpha, double eps_rel,
    PassOut pass) {
    using Idx = typename std::conditional<(V > 0), int, long>::type;     // columns: a cached row has at most 8192
    constexpr bool CACHED = (V > 0), CLAIMS = CACHED && V <= 4 && QUICK;  // claims requested with the row
    // the next rows are requested while these are worked on, where the registers allow it
    constexpr bool PIPE = V == 1 || (V == 2 && RMS);
    __shared__ unsigned int hist[kBins * kReplicas];
    __shared__ unsigned int red[kRedWords];
    __shared__ double smem[2 * 4 * (kCheckThreads / kWave)];       // one slot per reduction of a row
    __shared__ unsigned int largest;
    const int tid = threadIdx.x;
    const QuickCheck qc(k.quick_alpha, eps_rel);
    unsigned known = 0;
    for (int i = tid; i < kBins * kReplicas; i += kCheckThreads) hist[i] = 0;
    if (tid == 0) largest = 0;
    __syncthreads();
    ThreadAcc acc_chk;
    unsigned beyond = 0;                                     // counted in bin 0, but another vector's
    const int rep = tid & (kReplicas - 1);
    const int nv = CACHED ? V : (int)((cols + TPR * 4 - 1) / (TPR * 4));
    // Row group s of workgroup b, of G: rows b + s G, b + (s + all) G, ..., so that what is left for the last trip falls to all workgroups; or, k.apart being 1,
    // neighbouring rows.  A wavefront of whole rows goes by its first one, a workgroup whose row groups meet at barriers by the first of all.
    const int lead = TPR <= kWave ? __builtin_amdgcn_readfirstlane(tid / kWave) * (kWave / TPR) : 0;
    const long trip = (long)gridDim.x * (kCheckThreads / TPR), mine = (long)k.apart * (tid / TPR - lead);
    const long first = (long)blockIdx.x * (k.apart == 1 ? kCheckThreads / TPR : 1) + (long)k.apart * lead;
    const double n = (double)cols;
    float4 xn[PIPE ? V : 1], yn[PIPE ? V : 1], cn[PIPE && CLAIMS ? V : 1];
    auto request = [&](long rb, float4* xr, float4* yr, float4* cr) __attribute__((always_inline)) {
        int lt = tid % TPR;
        asm volatile("" : "+v"(lt));
        const long row = TPR == kWave ? rb : rb + mine, roff = (TPR == kWave || row < rows ? row : rows - 1) * ld;
        const Idx last = (Idx)cols - (FULL ? 4 : 1);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            xr[v] = row_vec<FULL, true, TPR>(x + roff, TAO_VEC_IDX(v), last);
            yr[v] = row_vec<FULL, true, TPR>(y + roff, TAO_VEC_IDX(v), last);
            if (CLAIMS) cr[v] = row_vec<FULL, true, TPR>(claimed + roff, TAO_VEC_IDX(v), last);
        }
    };
    if (PIPE && first < rows) request(first, xn, yn, cn);
    // (every thread of a workgroup takes the same number of trips where the reductions hold barriers)
    for (long rb = first; rb < rows; rb += trip) {
        int lt = tid % TPR;
        if (CACHED) asm volatile("" : "+v"(lt));            // (positions are formed anew for every row and pass, as in softmax_check)
        const long row = TPR == kWave ? rb : rb + mine;
        const bool active = TPR == kWave || row < rows;
        const Idx limit = active ? (Idx)cols : 0, last = (Idx)cols - (FULL ? 4 : 1);
        const long roff = (active ? row : rows - 1) * ld;
        float4 xv[CACHED ? V : 1], yv[CACHED ? V : 1], cv[CLAIMS ? V : 1], gv[CLAIMS ? V : 1];
        double a1[2] = {0.0, 0.0};                 // RMS: sum x^2;  LayerNorm: sum x, sum |x|
        auto scales = [&](Idx idx) { return g ? row_vec<FULL, false, TPR>(g, idx, last) : make_float4(1.f, 1.f, 1.f, 1.f); };
        if (PIPE) {
#pragma unroll
            for (int v = 0; v < nv; ++v) {
                xv[v] = xn[v]; yv[v] = yn[v];
                if (CLAIMS) { cv[v] = cn[v]; gv[v] = scales(TAO_VEC_IDX(v)); }
            }
            if (rb + trip < rows) request(rb + trip, xn, yn, cn);
            __builtin_amdgcn_sched_barrier(0);
        } else if (CACHED) {
#pragma unroll
            for (int v = 0; v < nv; ++v) {
                xv[v] = row_vec<FULL, true, TPR>(x + roff, TAO_VEC_IDX(v), last);
                yv[v] = row_vec<FULL, true, TPR>(y + roff, TAO_VEC_IDX(v), last);
                if (CLAIMS) { cv[v] = row_vec<FULL, true, TPR>(claimed + roff, TAO_VEC_IDX(v), last); gv[v] = scales(TAO_VEC_IDX(v)); }
            }
            __builtin_amdgcn_sched_barrier(0);               // (all requests leave before the first is waited for)
        }
        for (int v = 0; v < nv; ++v) {
            const float4 X = row_fill<FULL, TPR>(CACHED ? xv[v] : row_vec<FULL, false, TPR>(x + roff, TAO_VEC_IDX(v), last), TAO_VEC_IDX(v), limit, last, 0.f);
            if (CACHED) xv[v] = X;
            const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (RMS) a1[0] += (double)e[c] * (double)e[c];
                else { a1[0] += (double)e[c]; a1[1] += (double)fabsf(e[c]); }
            }
        }
        wide_group_sum<TPR>(a1, RMS ? 1 : 2, smem);
        double mu = 0.0, K1 = 0.0, K0 = 0.0, f = 0.0, amp = 1.0;
        bool ok = true;
        if (RMS) {
            const double E_t = (k.G * (1.0 + k.u) + k.u) * a1[0];
            const double vstar = a1[0] * k.inv_n;
            const double E_v = (E_t * k.inv_n + k.cd_u * vstar) * k.inv1mcd;
            double rs, E_r, R;
            ok = rsqrt_tail(vstar, E_v, k, rs, E_r, R, amp);
            f = E_r + k.u * R;
        } else {
            mu = a1[0] * k.inv_n;
            const double E_mu = ((k.G * a1[1]) * k.inv_n + k.cd_u * fabs(mu)) * k.inv1mcd;
            double a2[2] = {0.0, 0.0};                                   // sum |d|, sum d^2
            for (int v = 0; v < nv; ++v) {
                const float4 X = CACHED ? xv[v] : row_fill<FULL, TPR>(row_vec<FULL, false, TPR>(x + roff, TAO_VEC_IDX(v), last), TAO_VEC_IDX(v), limit, last, 0.f);
                const float e[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double d = row_has<FULL, TPR>(TAO_VEC_IDX(v), limit, last, c) ? (double)e[c] - mu : 0.0;
                    a2[0] += fabs(d);
                    a2[1] = fma(d, d, a2[1]);
                }
            }
            wide_group_sum<TPR>(a2, 2, smem + 4 * (kCheckThreads / kWave));
            layernorm_tail(E_mu, a2[0], a2[1], n, k, K1, K0, amp);
        }
        const UpFactors up(k.m * (1.0 + 2.0 * amp));
        // alpha tau from below, in binary32: |x g| f + u |y|, or |g| (K1 |x - mu| + K0) + u |y| with the difference's
        // own rounding taken off.  The factor of a row has to be an ordinary number (else NaN: nothing of the row is
        // settled): a subnormal one has lost bits, and a large one magnifies what a subnormal product |x g| has
        // lost (2^-150; with f alpha below 2^55 that stays far below the 2^-90 of quick_settled).  What mu, the conversions and
        // the products of the LayerNorm row lose there is taken off K0.
        const float uf = (float)k.u * qc.alpha;
        const float factor = (float)(RMS ? f : K1);
        const float scaled = (ok && factor >= 0x1p-90f && factor <= 0x1p25f ? factor : NAN) * qc.alpha;
        const float ff = scaled, muf = (float)mu, K1f = scaled;
        const float K0f = (float)(K0 - 0x1p-22 * K1 * (fabs(mu) + 0x1p-126)) * qc.alpha - 0x1p-140f;
        if (QUICK) known = newest(&largest);
        if (CACHED) asm volatile("" : "+v"(lt));
        float4 next = make_float4(0.f, 0.f, 0.f, 0.f), next_g = next;    // the next vector's claims are on their way while one is checked
        constexpr bool AHEAD = CACHED && !CLAIMS;
        if (AHEAD) { next = row_vec<FULL, true, TPR>(claimed + roff, TAO_VEC_IDX(0), last); next_g = scales(TAO_VEC_IDX(0)); }
        for (int v = 0; v < nv; ++v) {
            const Idx idx = TAO_VEC_IDX(v);
            const float4 C = CLAIMS ? cv[v] : AHEAD ? next : row_vec<FULL, true, TPR>(claimed + roff, idx, last);
            const float4 Gv = CLAIMS ? gv[v] : AHEAD ? next_g : scales(idx);
            if (AHEAD && v + 1 < nv) { next = row_vec<FULL, true, TPR>(claimed + roff, TAO_VEC_IDX(v + 1), last); next_g = scales(TAO_VEC_IDX(v + 1)); }
            if (idx >= limit) continue;
            const float4 X = CACHED ? xv[v] : row_vec<FULL, false, TPR>(x + roff, idx, last);
            const float4 Y = CACHED ? yv[v] : row_vec<FULL, true, TPR>(y + roff, idx, last);
            floatv4 xe = {X.x, X.y, X.z, X.w}, ye = {Y.x, Y.y, Y.z, Y.w}, ge = {Gv.x, Gv.y, Gv.z, Gv.w}, ce = {C.x, C.y, C.z, C.w};
            asm volatile("" : "+v"(xe), "+v"(ye));           // (keeps the first pass's binary64 values from living on until here)
            auto tau = [&](int c) __attribute__((always_inline)) {
                if (RMS) {
                    const double xg = fabs((double)xe[c] * (double)ge[c]);
                    const double tt = xg * f + k.u * fabs((double)ye[c]);
                    return ok ? up32g(tt, up.mul, up.sub) : NAN;
                }
                const double ad = fabs((double)xe[c] - mu);
                const double ep = (double)fabsf(ge[c]) * fma(K1, ad, K0);
                return up32g(fma(k.u, (double)fabsf(ye[c]), ep), up.mul, up.sub);
            };
            const unsigned others = row_others<FULL>(idx, last), own = 15u & 15u << others;
            if (QUICK && (FULL != SINGLE || idx + 3 * TPR < limit)) {
                floatv4 at;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (RMS) at[c] = fmaf(fabsf(xe[c] * ge[c]), ff, uf * fabsf(ye[c]));
                    else     at[c] = fmaf(fabsf(ge[c]), fmaf(K1f, fabsf(xe[c] - muf), K0f), uf * fabsf(ye[c]));
                }
                leave_others<FULL>(others, ce, ye, at);
                if (quick_check_four<(V == 1 || (V == 2 && TPR < 1024))>(ce, ye, at, tau, qc, alpha, eps_rel, hist, rep, acc_chk, &largest, known, known != 0, own)) beyond += others;
                continue;
            }
            if (CACHED && (FULL != SINGLE || idx + 3 * TPR < limit)) {
                const float c4[4] = {ce[0], ce[1], ce[2], ce[3]}, y4[4] = {ye[0], ye[1], ye[2], ye[3]};
                const float t4[4] = {tau(0), tau(1), tau(2), tau(3)};
                check_four(c4, y4, t4, alpha, eps_rel, hist, rep, acc_chk, own);
                continue;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {                    // (rows re-read from memory: no registers for four side by side)
                if (!row_has<FULL, TPR>(idx, limit, last, c)) continue;
                check_one(ce[c], ye[c], tau(c), alpha, eps_rel, hist, rep, acc_chk);
            }
        }
    }
    if (FULL == ANY && QUICK && beyond) atomicSub(&hist[rep], beyond);
    __syncthreads();
    finish_pass(hist, acc_chk, red, pass);
}

// ------------------------------------------------------------------ sum / mean
template <int TPR, int V>
__global__ __launch_bounds__(kRowThreads) void summean_bound(
    const float* __restrict__ x, const float* __restrict__ y, float* __restrict__ tau,
    long rows, long cols, long ld, int vec_ok, int is_mean, RowConsts k) {
    TAO_ROW_PROLOGUE
    double a1[1] = {0.0};
    for (int v = 0; v < nv; ++v) {
        const float4 X = load4<true>(x + roff, TAO_VEC_INDEX(v), limit, vec_ok, 0.f);
        a1[0] += fabs((double)X.x) + fabs((double)X.y) + fabs((double)X.z) + fabs((double)X.w);
    }
    group_sum<TPR>(a1, 1, smem);
    if (active && lt == 0) {
        double t = k.G * a1[0];
        // (mean without y: |y| <= (sum|x| / n)(1 + Gamma)(1 + c_div u))
        if (is_mean) t = t * k.inv_n + (y ? fabs((double)y[row]) : a1[0] * k.inv_n * (1.0 + k.G) * (1.0 + k.cd_u)) * k.mean_f;
        const UpFactors up(k.m);
        tau[row] = up32g(t, up.mul, up.sub);
    }
}

// ------------------------------------------------------------------ BatchNorm-affine
// tau = u |x s_c| (1+u) + u |y|, column c = flat index mod cols; one thread per 4 columns.
// NOY: no re-executed output (y is then the shift t or NULL, indexed by column like s): u|y| is taken at
// Y = (|x s|(1+u) + |t|)(1+u) >= |y|.
template <bool NOY>
__global__ __launch_bounds__(kRowThreads) void bn_affine_bound(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ s,
    float* __restrict__ tau, long rows, long cols, long ld, int vec_ok, int vec_s, double u) {
    const long vpr = (cols + 3) / 4;                       // vectors per row
    const long total = rows * vpr;
    // flat grid-stride walk over (row, vector) pairs; the pair is advanced by additions only
    // (one division per thread, before the loop)
    const long stride = (long)gridDim.x * blockDim.x;
    const long srow = stride / vpr, sjv = stride - srow * vpr;
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    long row = i / vpr, jv = i - row * vpr;
    for (; i < total; i += stride, row += srow, jv += sjv) {
        if (jv >= vpr) { jv -= vpr; ++row; }
        const long j = jv * 4;
        const float4 X = load4<true>(x + row * ld, j, cols, vec_ok, 0.f);
        const float4 Y = NOY ? (y ? load4(y, j, cols, 0, 0.f) : make_float4(0.f, 0.f, 0.f, 0.f))
                             : load4<true>(y + row * ld, j, cols, vec_ok, 0.f);
        const float4 S = load4(s, j, cols, vec_s, 0.f);
        const float xe[4] = {X.x, X.y, X.z, X.w}, ye[4] = {Y.x, Y.y, Y.z, Y.w}, se[4] = {S.x, S.y, S.z, S.w};
        float te[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double xs = fabs((double)xe[c] * (double)se[c]);
            const double Yb = NOY ? (xs * (1.0 + u) + fabs((double)ye[c])) * (1.0 + u) : fabs((double)ye[c]);
            const double t = u * xs * (1.0 + u) + u * Yb;
            te[c] = up32g(t, kUpMul, 1.0 + 0x1p-48);
        }
        store4(tau + row * ld, j, cols, vec_ok, make_float4(te[0], te[1], te[2], te[3]));
    }
}

// How a ragged row is read whose group holds V vectors of 4 TPR columns: by vectors unless most of the last one would be empty (us, by single
// values / by vectors: LayerNorm 30000 x 511 58.2 / 51.5, 6442 x 861 48.1 / 38.8, softmax of 4 x 2045 x 2045 with its products 175 / 158; but LayerNorm
// 10000 x 1031 58.4 / 63.2, 30000 x 259 45.7 / 48.8, 155 x 3233 13.8 / 14.5).  A wavefront's rows of one vector to a lane by single values where these are one or
// two to a lane, or three in a few rows: a lane with values takes four by vectors, and the others wait for it (softmax 38 x 51 8.8 / 10.1, 100000 x 51 60.0 / 68.7,
// 65536 x 65 46.8 / 48.7, 3000 x 190 10.1 / 10.8, 24576 x 190 24.9 / 25.9, but 49152 x 190 41.9 / 41.0 and 16384 x 193 23.9 / 21.6; LayerNorm 300 x 129 9.7 / 10.0, 32768 x 129 37.1 / 36.2).
constexpr long kFewRaggedRows = 6L * kMaxCheckBlocks * (kCheckThreads / kWave);
static int row_form(bool whole, long rows, long cols, long tpr, long V) {
    if (whole) return WHOLE;
    if (cols < 4) return SINGLE;
    if (V == 1 && tpr == kWave) return cols <= 2 * kWave || (cols <= 3 * kWave && rows < kFewRaggedRows) ? SINGLE : ANY;
    return V == 2 && cols * 5 < tpr * V * 4 * 4 ? SINGLE : ANY;
}
// The one-pass checks of rows.  Quick settlement pays from eight rows per row group on, four where that is a wavefront; below, too many elements are
// among the first a workgroup sees and the second route is only more code to fetch (us with / without: softmax 512 x 512
// 20 / 16, RMSNorm 4096 x 768 28 / 25, but RMSNorm 8192 x 2048 55 / 59, 8192 x 4096 94 / 109).
// From two rows per wavefront on a row of 513 to 1024 (softmax: 2048) columns belongs to one wavefront -- no barrier, the
// wavefronts of a workgroup drift apart, so that some load while others calculate; fewer rows are divided
// among four wavefronts, which fill the chip sooner (8192 x 1024 34 against 46 us, 4096 x 2048 45 against 40).
// Rows of the norms of up to 64 and 128 columns belong to 16 and 32 lanes (a wavefront each, most of whose lanes then held nothing: RMSNorm 161713 x 56
// 96.9 us, now 35.3, LayerNorm 130000 x 64 121.7 / 37.6, 100000 x 100 88.5 / 49.1, RMSNorm 60 x 61 10.7 / 8.0).
// Workgroups of a one-pass check, `groups` rows at a time each.  Where all rows fit one trip with workgroups to spare, they go to more of these, down to
// kFewestElements each, as far as that takes rows off the fullest one.  Few rows wait for the arithmetic of the compute unit that has most of them, many end
// with a trip that only some have; with a workgroup's rows as far apart as there are workgroups that trip is everybody's, and the wavefronts that have none
// in it are done (softmax / RMSNorm, us, with neighbouring rows and so: 6144 x 512, one trip and a half, 20.5 / 19.1 and 16.8 / 15.8; 9000 x 512 26.7 / 24.2 and 22.1 / 20.5;
// 21696 x 1356 92.4 / 100 and 79.9 / 100; 16384 x 1024 47.6 / 46.4 and 45.6 / 42.6; 64 x 1500, on 16 workgroups and on 64,
// 13.6 / 12.5 and 11.3 / 10.2; 512 x 768 10.9 / 10.6 and 10.5 / 10.2).  Where the last trip is a full one neighbouring rows stay together
// (RMSNorm 2048 x 4096 31.3, 31.8 apart, 16384 x 512 29.6 / 30.1, softmax 8192 x 2048 56.5 / 61.2, 16384 x 300 30.0 / 30.6), but for a wavefront's rows of four
// vectors, which drift apart the more (softmax 8192 x 1024 38.8 / 33.9, 12288 x 1024 44.3 / 42.3, LayerNorm 16384 x 1024 47.1 / 44.2).
constexpr long kFewestElements = 1024;
static int row_blocks(long rows, long cols, int tpr, RowConsts& k) {
    const int groups = kCheckThreads / tpr;
    const long full = (rows + groups - 1) / groups;
    long blocks = full <= alone_row_groups(cols) ? 1 : full < kMaxCheckBlocks ? full : kMaxCheckBlocks;
    if (blocks > 1 && blocks < kMaxCheckBlocks) {
        const long most = rows < kMaxCheckBlocks ? rows : (long)kMaxCheckBlocks, spread = rows * cols / kFewestElements;
        blocks = spread < blocks ? blocks : spread < most ? spread : most;
        const long each = (rows + blocks - 1) / blocks;
        blocks = (rows + each - 1) / each;
    }
    const bool four_vectors = tpr == kWave && cols > 512 && cols <= 1024;
    k.apart = !four_vectors && rows % (blocks * groups) == 0 ? 1 : (int)blocks;
    return (int)blocks;
}
constexpr long kWaveRows = 2L * kMaxCheckBlocks * (kCheckThreads / kWave);
static bool quick_pays(long rows, int tpr) { return rows >= (tpr <= kWave ? 4L : 8L) * kMaxCheckBlocks * (kCheckThreads / tpr); }

// Pick the row-group shape for a row length and launch KERNEL<TPR, V>.  A single wavefront owns
// a row of up to WMAX columns (no barrier, no LDS exchange); longer rows take a workgroup.
// Measured: beyond 1024 columns the registers of a wavefront-wide cached row cut the occupancy
// to two wavefronts per SIMD and the kernels lose a third of their bandwidth, so WMAX = 1024.
// Rows of 513 .. 768 columns (a common hidden size) take three vectors per lane rather than four:
// fewer registers, one more wavefront per SIMD (LayerNorm 62 -> 68 %, RMSNorm 67 -> 75 % of the HBM roofline).
#define TAO_DISPATCH_ROWS(KERNEL, WMAX, rows, cols, stream, ...)                                    \
    do {                                                                                            \
        const long c_ = (cols);                                                                     \
        auto grid_ = [&](int tpr) { return dim3((unsigned)(((rows) + (kRowThreads / tpr) - 1) / (kRowThreads / tpr))); }; \
        if (c_ <= 256)       hipLaunchKernelGGL((KERNEL<64, 1>), grid_(64), dim3(kRowThreads), 0, stream, __VA_ARGS__);   \
        else if (c_ <= 512)  hipLaunchKernelGGL((KERNEL<64, 2>), grid_(64), dim3(kRowThreads), 0, stream, __VA_ARGS__);   \
        else if (c_ <= 768)  hipLaunchKernelGGL((KERNEL<64, 3>), grid_(64), dim3(kRowThreads), 0, stream, __VA_ARGS__);   \
        else if (c_ <= 1024) hipLaunchKernelGGL((KERNEL<64, 4>), grid_(64), dim3(kRowThreads), 0, stream, __VA_ARGS__);   \
        else if (c_ <= 2048 && WMAX >= 2048) hipLaunchKernelGGL((KERNEL<64, 8>), grid_(64), dim3(kRowThreads), 0, stream, __VA_ARGS__);  \
        else if (c_ <= 4096 && WMAX >= 4096) hipLaunchKernelGGL((KERNEL<64, 16>), grid_(64), dim3(kRowThreads), 0, stream, __VA_ARGS__); \
        else if (c_ <= 2048) hipLaunchKernelGGL((KERNEL<256, 2>), grid_(256), dim3(kRowThreads), 0, stream, __VA_ARGS__); \
        else if (c_ <= 4096) hipLaunchKernelGGL((KERNEL<256, 4>), grid_(256), dim3(kRowThreads), 0, stream, __VA_ARGS__); \
        else if (c_ <= 8192) hipLaunchKernelGGL((KERNEL<256, 8>), grid_(256), dim3(kRowThreads), 0, stream, __VA_ARGS__); \
        else                 hipLaunchKernelGGL((KERNEL<256, 0>), grid_(256), dim3(kRowThreads), 0, stream, __VA_ARGS__); \
    } while (0)

// variance: the operator divides by a computed variance (LayerNorm, RMSNorm, GroupNorm).  Its
// template subtracts the variance's own error bound, about Gamma(n-1) times the variance, from the
// variance: beyond Gamma(n-1) = 1/2 the difference has lost its relative accuracy (and soon its
// sign), so such rows are refused rather than bounded by noise.
static int make_consts(const tao_fp_model& md, long cols, double eps, RowConsts* k, bool variance = false) {
    const double G = gamma_up(cols - 1, md);
    if (!(G == G) || (variance && G > 0.5)) return TAO_ERR_K_RANGE;
    const double u = md.u;
    k->u = u; k->G = G;
    k->inv1mu = widen(1.0 / (1.0 - u));
    k->ce_u = md.c_exp * u;
    k->inv1mce = widen(1.0 / (1.0 - md.c_exp * u));
    k->cd_u = md.c_div * u;
    k->inv1mcd = widen(1.0 / (1.0 - md.c_div * u));
    k->cr_u = md.c_rsqrt * u;
    k->eps = (double)(float)eps;
    k->inv_n = 1.0 / (double)cols;
    k->mean_f = widen(k->cd_u * k->inv1mcd);
    // Rounding margin of the emitted bound.  The row sums are formed here in round-to-nearest
    // binary64 (each thread a sequential part, then a tree: at most cols 2^-53 below the real sum),
    // and a reference that adds the row sequentially with upward rounding sits up to cols 2^-52
    // above it; the scalar chain after the sums adds a few dozen roundings.  m covers both for a
    // bound that depends on the sums with unit sensitivity; the kernels scale it where a sum enters
    // through a difference (1 - sigma of the softmax, the lower end w_lo of the variance).
    k->m = ((double)cols + 130.0) * 0x1p-51;
    k->quick_alpha = NAN;
    k->apart = 1;                                            // (no launch leaves it open, one of no rows either: row_blocks chooses for the others)
    if (!(md.c_exp * u < 0.5) || !(md.c_div * u < 0.5)) return TAO_ERR_MODEL;
    return TAO_OK;
}

}  // namespace tao

extern "C" {

int tao_bound_softmax(const float* x, const float* y_ref, float* tau, long rows, long cols, long ld,
                      const tao_fp_model* model, void* stream) {
    using namespace tao;
    tao_fp_model md;
    int rc = resolve_model(model, &md);
    if (rc != TAO_OK) return rc;
    if (rows < 0 || cols < 0 || ld < cols) return TAO_ERR_SHAPE;
    if (rows == 0 || cols == 0) return TAO_OK;
    if (!x || !y_ref || !tau) return TAO_ERR_NULL;
    if (!aligned(x, 4) || !aligned(y_ref, 4) || !aligned(tau, 4)) return TAO_ERR_ALIGN;
    RowConsts k;
    rc = make_consts(md, cols, 0.0, &k);
    if (rc != TAO_OK) return rc;
    const int vec_ok = aligned(x, 16) && aligned(y_ref, 16) && aligned(tau, 16) && (ld % 4 == 0);
    hipStream_t st = (hipStream_t)stream;
    TAO_DISPATCH_ROWS(softmax_bound, 1024, rows, cols, st, x, y_ref, tau, rows, cols, ld, vec_ok, k);
    return launch_status();
}

int tao_bound_norm(int kind, const float* x, const float* y_ref, const float* gamma_or_scale,
                   const float* beta_or_shift, double eps, float* tau, long rows, long cols, long ld,
                   const tao_fp_model* model, void* stream) {
    using namespace tao;
    tao_fp_model md;
    int rc = resolve_model(model, &md);
    if (rc != TAO_OK) return rc;
    if (kind < TAO_NORM_LAYERNORM || kind > TAO_NORM_MEAN) return TAO_ERR_KIND;
    if (rows < 0 || cols < 0 || ld < cols) return TAO_ERR_SHAPE;
    if (rows == 0) return TAO_OK;
    if (cols == 0 && kind != TAO_NORM_SUM && kind != TAO_NORM_MEAN) return TAO_OK;
    if (cols == 0) return TAO_ERR_SHAPE;
    if (!x || !tau) return TAO_ERR_NULL;
    if (kind == TAO_NORM_BN_AFFINE && !gamma_or_scale) return TAO_ERR_NULL;
    if (!aligned(x, 4) || !aligned(y_ref, 4) || !aligned(tau, 4) || !aligned(gamma_or_scale, 4) || !aligned(beta_or_shift, 4))
        return TAO_ERR_ALIGN;
    if (!(eps >= 0.0) || !std::isfinite(eps)) return TAO_ERR_SHAPE;
    RowConsts k;
    rc = make_consts(md, cols, eps, &k, kind == TAO_NORM_LAYERNORM || kind == TAO_NORM_RMSNORM);
    if (rc != TAO_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    const int vec_x = aligned(x, 16) && (ld % 4 == 0);
    const int vec_ok = vec_x && aligned(y_ref, 16) && aligned(tau, 16);      // (a NULL y_ref counts as aligned)
    const int vec_g = aligned(gamma_or_scale, 16), vec_b = aligned(beta_or_shift, 16);
    const float* g = gamma_or_scale;
    const float* b = beta_or_shift;
    switch (kind) {
        case TAO_NORM_LAYERNORM:
            if (y_ref) TAO_DISPATCH_ROWS(layernorm_bound, 1024, rows, cols, st, x, y_ref, g, tau, rows, cols, ld, vec_ok, vec_g, k);
            else       TAO_DISPATCH_ROWS(layernorm_bound_noy, 1024, rows, cols, st, x, g, b, tau, rows, cols, ld, vec_ok, vec_g, vec_b, k);
            break;
        case TAO_NORM_RMSNORM:
            if (y_ref) TAO_DISPATCH_ROWS(rmsnorm_bound, 1024, rows, cols, st, x, y_ref, g, tau, rows, cols, ld, vec_ok, vec_g, k);
            else       TAO_DISPATCH_ROWS(rmsnorm_bound_noy, 1024, rows, cols, st, x, g, tau, rows, cols, ld, vec_ok, vec_g, k);
            break;
        case TAO_NORM_BN_AFFINE: {
            const long total = rows * ((cols + 3) / 4);
            long blocks = (total + kRowThreads - 1) / kRowThreads;
            if (blocks > 256L * 64) blocks = 256L * 64;    // grid-stride beyond 64 workgroups per CU
            if (y_ref) hipLaunchKernelGGL(bn_affine_bound<false>, dim3((unsigned)blocks), dim3(kRowThreads), 0, st, x, y_ref, g,
                                          tau, rows, cols, ld, vec_ok, vec_g, md.u);
            else       hipLaunchKernelGGL(bn_affine_bound<true>, dim3((unsigned)blocks), dim3(kRowThreads), 0, st, x, b, g,
                                          tau, rows, cols, ld, vec_ok, vec_g, md.u);
            break;
        }
        default: {
            const int is_mean = (kind == TAO_NORM_MEAN);
            TAO_DISPATCH_ROWS(summean_bound, 1024, rows, cols, st, x, y_ref, tau, rows, cols, ld, vec_x, is_mean, k);
            break;
        }
    }
    return launch_status();
}

size_t tao_groupnorm_workspace_bytes(long batch, long channels, long positions, long groups) {
    using namespace tao;
    if (batch <= 0 || channels <= 0 || positions <= 0 || groups < 1 || channels % groups) return 0;
    const __int128 cols = (__int128)(channels / groups) * positions;
    if (cols <= 8192 || cols >= (1L << 31) || batch * groups >= kSplitMaxRows) return 0;   // the row kernels need none
    const long nchunk = (long)((cols + kChunk - 1) / kChunk);
    return (size_t)batch * (size_t)groups * (size_t)nchunk * 4 * sizeof(double);
}

int tao_bound_groupnorm(const float* x, const float* y_ref, const float* gamma, const float* beta, double eps,
                        float* tau, long batch, long channels, long positions, long groups,
                        const tao_fp_model* model, void* ws, size_t ws_bytes, void* stream) {
    using namespace tao;
    (void)beta;
    tao_fp_model md;
    int rc = resolve_model(model, &md);
    if (rc != TAO_OK) return rc;
    if (batch < 0 || channels < 0 || positions < 0 || groups < 1 || channels % groups) return TAO_ERR_SHAPE;
    const long cpg = channels / groups;
    if (positions >= (1L << 31) || cpg >= (1L << 31) || groups >= (1L << 31)) return TAO_ERR_SHAPE;
    if ((__int128)cpg * positions >= (1L << 31) || (__int128)batch * groups >= (1L << 40)) return TAO_ERR_SHAPE;
    const long rows = batch * groups, cols = cpg * positions;
    if (rows == 0 || cols == 0) return TAO_OK;
    if (!x || !tau || !y_ref) return TAO_ERR_NULL;
    if (!aligned(x, 4) || !aligned(y_ref, 4) || !aligned(tau, 4) || !aligned(gamma, 4)) return TAO_ERR_ALIGN;
    if (!(eps >= 0.0) || !std::isfinite(eps)) return TAO_ERR_SHAPE;
    RowConsts k;
    rc = make_consts(md, cols, eps, &k, true);
    if (rc != TAO_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    const int vec_ok = aligned(x, 16) && aligned(y_ref, 16) && aligned(tau, 16) && (cols % 4 == 0);
    GroupGeom gg;
    gg.hw = (unsigned)positions; gg.cpg = (unsigned)cpg; gg.groups = (unsigned)groups;
    // rows the cached variants hold, or enough rows to fill the chip with one workgroup each
    // (measured: 1024 rows of 25088 run at 42 % of the HBM roofline that way, 32 % in chunks;
    // 256 rows of 40960 at 20 % against 32 %)
    if (cols <= 8192 || rows >= kSplitMaxRows) {
        TAO_DISPATCH_ROWS(groupnorm_bound, 1024, rows, cols, st, x, y_ref, gamma, tau, rows, cols, cols, vec_ok, k, gg);
        return launch_status();
    }
    const long nchunk = (cols + kChunk - 1) / kChunk;
    if ((__int128)rows * nchunk >= (1L << 31)) return TAO_ERR_SHAPE;
    const size_t need = (size_t)rows * (size_t)nchunk * 4 * sizeof(double);
    if (!ws || ws_bytes < need || !aligned(ws, 8)) return TAO_ERR_WORKSPACE;
    double* part = static_cast<double*>(ws);
    const dim3 grid((unsigned)(rows * nchunk)), blk(kRowThreads);
    hipLaunchKernelGGL(groupnorm_sums_a, grid, blk, 0, st, x, part, cols, (unsigned)nchunk, vec_ok);
    hipLaunchKernelGGL(groupnorm_sums_b, grid, blk, 0, st, x, part, cols, (unsigned)nchunk, vec_ok, k);
    hipLaunchKernelGGL(groupnorm_apply, grid, blk, 0, st, x, y_ref, gamma, tau, part, cols, (unsigned)nchunk, vec_ok, k, gg);
    return launch_status();
}

int tao_bound_check_norm(int kind, const float* x, const float* y_ref, const float* gamma, const float* beta,
                         double eps, const float* claimed, long rows, long cols, long ld,
                         double alpha, double eps_rel, const tao_fp_model* model, tao_profile* out,
                         void* ws, size_t ws_bytes, void* stream) {
    using namespace tao;
    (void)beta;
    tao_fp_model md;
    int rc = resolve_model(model, &md);
    if (rc != TAO_OK) return rc;
    if (kind != TAO_NORM_LAYERNORM && kind != TAO_NORM_RMSNORM) return TAO_ERR_KIND;
    if (!out || !ws) return out ? TAO_ERR_WORKSPACE : TAO_ERR_NULL;
    if (rows < 0 || cols < 0 || ld < cols || !(eps >= 0.0) || !std::isfinite(eps)) return TAO_ERR_SHAPE;
    if (!(alpha >= 0.0) || !std::isfinite(alpha) || !(eps_rel >= 0.0) || !std::isfinite(eps_rel)) return TAO_ERR_SHAPE;
    const long n = rows * cols;
    if (rows > 0 && cols > 0 && n / cols != rows) return TAO_ERR_SHAPE;
    if (n >= (1L << 36)) return TAO_ERR_SHAPE;                      // 32-bit per-workgroup counters
    if (n > 0 && (!x || !y_ref || !claimed)) return TAO_ERR_NULL;
    if (!aligned(x, 4) || !aligned(y_ref, 4) || !aligned(claimed, 4) || !aligned(gamma, 4) || !aligned(out, 8))
        return TAO_ERR_ALIGN;
    if (!aligned(ws, 256) || ws_bytes < check_workspace_bytes()) return TAO_ERR_WORKSPACE;
    RowConsts k;
    rc = make_consts(md, cols > 0 ? cols : 1, eps, &k, true);
    if (rc != TAO_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    const bool full = aligned(x, 16) && aligned(y_ref, 16) && aligned(claimed, 16) && aligned(gamma, 16) && (ld % 4 == 0) && (cols % 4 == 0);
    k.quick_alpha = quick_alpha(alpha, md);
    const CheckWorkspace w = carve_check_workspace(ws);
    int nblocks = 1;
    const bool rms = kind == TAO_NORM_RMSNORM;
    auto launch = [&](auto kernel, int tpr, long r, long c, long l) {
        nblocks = row_blocks(r, c, tpr, k);
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(kCheckThreads), 0, st, x, y_ref, gamma, claimed, r, c, l,
                           k, alpha, eps_rel, pass_out(w, nblocks, n, out));
    };
    auto quick = [&](int tpr) { return quick_pays(rows, tpr); };
#define TAO_NORM_CHECK_Q(RMS, TPR, V, Q) \
    do {                                                                                                    \
        const int form = row_form(full, rows, cols, TPR, V);                                                \
        if (form == WHOLE)    launch(norm_check<RMS, TPR, V, WHOLE, Q>, TPR, rows, cols, ld);               \
        else if (form == ANY) launch(norm_check<RMS, TPR, V, ANY, Q>, TPR, rows, cols, ld);                 \
        else                  launch(norm_check<RMS, TPR, V, V == 2 || (V == 1 && TPR == kWave) ? SINGLE : ANY, Q>, TPR, rows, cols, ld); \
    } while (0)
#define TAO_NORM_CHECK(RMS, TPR, V) do { if (quick(TPR)) TAO_NORM_CHECK_Q(RMS, TPR, V, true); else TAO_NORM_CHECK_Q(RMS, TPR, V, false); } while (0)
#define TAO_NORM_CHECK_ROWS(RMS)                                                                            \
    do {                                                                                                    \
        if (cols < 4)                        launch(norm_check<RMS, 64, 1, SINGLE, false>, 64, rows, cols, ld); \
        else if (cols <= 64)                 TAO_NORM_CHECK(RMS, 16, 1);                                    \
        else if (cols <= 128)                TAO_NORM_CHECK(RMS, 32, 1);                                    \
        else if (cols <= 256)                TAO_NORM_CHECK(RMS, 64, 1);                                    \
        else if (cols <= 512)                TAO_NORM_CHECK(RMS, 64, 2);                                    \
        else if (cols <= 1024 && rows >= kWaveRows) TAO_NORM_CHECK_Q(RMS, 64, 4, true);                    \
        else if (cols <= 1024)               TAO_NORM_CHECK(RMS, 256, 1);                                   \
        else if (cols <= 2048)               TAO_NORM_CHECK(RMS, 256, 2);                                   \
        else if (cols <= 4096)               TAO_NORM_CHECK(RMS, 512, 2);                                   \
        else if (cols <= 8192 && RMS)        TAO_NORM_CHECK(RMS, 1024, 2);                                  \
        else                                 TAO_NORM_CHECK_Q(RMS, 1024, 0, false);                         \
    } while (0)
    if (n == 0) {
        if (rms) launch(norm_check<true, 64, 1, SINGLE, false>, 64, 0L, 1L, 1L); else launch(norm_check<false, 64, 1, SINGLE, false>, 64, 0L, 1L, 1L);
    } else if (rms) {
        TAO_NORM_CHECK_ROWS(true);
    } else {
        TAO_NORM_CHECK_ROWS(false);
    }
#undef TAO_NORM_CHECK_ROWS
#undef TAO_NORM_CHECK_Q
#undef TAO_NORM_CHECK
    launch_finish(w, nblocks, n, out, st);
    return launch_status();
}

int tao_bound_check_softmax(const float* x, const float* y_ref, const float* claimed, long rows, long cols, long ld,
                            double alpha, double eps_rel, const tao_fp_model* model, tao_profile* out,
                            void* ws, size_t ws_bytes, void* stream) {
    using namespace tao;
    tao_fp_model md;
    int rc = resolve_model(model, &md);
    if (rc != TAO_OK) return rc;
    if (!out || !ws) return out ? TAO_ERR_WORKSPACE : TAO_ERR_NULL;
    if (rows < 0 || cols < 0 || ld < cols || !(eps_rel >= 0.0)) return TAO_ERR_SHAPE;
    const long n = rows * cols;
    if (rows > 0 && cols > 0 && n / cols != rows) return TAO_ERR_SHAPE;
    if (n >= (1L << 36)) return TAO_ERR_SHAPE;                      // 32-bit per-workgroup counters
    if (n > 0 && (!x || !y_ref || !claimed)) return TAO_ERR_NULL;
    if (!aligned(x, 4) || !aligned(y_ref, 4) || !aligned(claimed, 4) || !aligned(out, 8)) return TAO_ERR_ALIGN;
    if (!aligned(ws, 256) || ws_bytes < check_workspace_bytes()) return TAO_ERR_WORKSPACE;
    RowConsts k;
    rc = make_consts(md, cols > 0 ? cols : 1, 0.0, &k);
    if (rc != TAO_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    k.quick_alpha = quick_alpha(alpha, md);
    const CheckWorkspace w = carve_check_workspace(ws);
    const bool full = aligned(x, 16) && aligned(y_ref, 16) && aligned(claimed, 16) && (ld % 4 == 0) && (cols % 4 == 0);
    int nblocks = 1;
    if (n > 0) {
        auto launch = [&](auto kernel, int tpr) {
            nblocks = row_blocks(rows, cols, tpr, k);
            hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(kCheckThreads), 0, st, x, y_ref, claimed, rows, cols, ld,
                               k, alpha, eps_rel, pass_out(w, nblocks, n, out));
        };
        auto quick = [&](int tpr) { return quick_pays(rows, tpr); };
#define TAO_SOFTMAX_CHECK_Q(TPR, V, Q) \
    do {                                                                                        \
        const int form = row_form(full, rows, cols, TPR, V);                                    \
        if (form == WHOLE)    launch(softmax_check<TPR, V, WHOLE, Q>, TPR);                     \
        else if (form == ANY) launch(softmax_check<TPR, V, ANY, Q>, TPR);                       \
        else                  launch(softmax_check<TPR, V, V == 2 || (V == 1 && TPR == kWave) ? SINGLE : ANY, Q>, TPR); \
    } while (0)
#define TAO_SOFTMAX_CHECK(TPR, V) do { if (quick(TPR)) TAO_SOFTMAX_CHECK_Q(TPR, V, true); else TAO_SOFTMAX_CHECK_Q(TPR, V, false); } while (0)
        if (cols < 4)          launch(softmax_check<64, 1, SINGLE, false>, 64);
        else if (cols <= 256)  TAO_SOFTMAX_CHECK(64, 1);
        else if (cols <= 512)  TAO_SOFTMAX_CHECK(64, 2);
        else if (cols <= 1024 && rows >= kWaveRows) TAO_SOFTMAX_CHECK_Q(64, 4, true);
        else if (cols <= 1024) TAO_SOFTMAX_CHECK(256, 1);
        else if (cols <= 2048 && rows >= kWaveRows) TAO_SOFTMAX_CHECK_Q(64, 8, true);
        else if (cols <= 2048) TAO_SOFTMAX_CHECK(256, 2);
        else if (cols <= 4096) TAO_SOFTMAX_CHECK(512, 2);
        else if (cols <= 8192) TAO_SOFTMAX_CHECK(1024, 2);
        else                   TAO_SOFTMAX_CHECK_Q(1024, 0, false);
#undef TAO_SOFTMAX_CHECK
#undef TAO_SOFTMAX_CHECK_Q
    } else {
        // nothing to examine: an empty partial, so that the profile reports n = 0
        hipLaunchKernelGGL((softmax_check<64, 1, SINGLE, false>), dim3(1), dim3(kCheckThreads), 0, st, x, y_ref, claimed, 0L, 1L, 1L,
                           k, alpha, eps_rel, pass_out(w, nblocks, n, out));
    }
    launch_finish(w, nblocks, n, out, st);
    return launch_status();
}

}  // extern "C"
