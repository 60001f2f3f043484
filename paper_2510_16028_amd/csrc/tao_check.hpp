// Pieces of the leaf check (Sec. 5.4) and relative-error profile (Sec. 5.3; Sec. 3.2 Eq. 2) shared by
// the streaming check pass and by bound kernels that check their bound in registers instead of
// storing it: the per-element step, the per-workgroup counters, the workspace layout and the
// launch of the finalising kernel.
#pragma once
#include "tao_hist.hpp"
#include "tao_host.hpp"

namespace tao {

constexpr int kCheckThreads = 1024;          // one workgroup per CU: one partial histogram per CU
constexpr int kMaxCheckBlocks = kMaxPartials;
constexpr int kReduceBlocks = kGroups;

struct BlockStats {          // one per pass-1 workgroup, in the workspace after the histograms
    unsigned long long violations;
    unsigned long long nans;
    unsigned int max_bits;   // bit pattern of the largest non-NaN error (errors are >= 0)
    unsigned int flag;       // not a counter: no pass writes it (linear_screen.hpp)
};

struct ThreadAcc {
    unsigned int violations = 0, nans = 0, max_bits = 0;
};

// The arithmetic of one element: violation flag, bin of the relative error, its bits.  A claimed
// value that equals the re-executed one bit for bit (and is finite) has d = 0 exactly, so the error is
// 0 (NaN for 0/0) without the binary64 division; whole wavefronts of such elements -- the masked
// half of a causal softmax, exact operators -- skip the division's instructions altogether.
// SHORTCUT = false leaves the test out: straight-line code, which a caller that unrolls many elements
// (the matrix kernel's epilogue) wants more than the shortcut.
struct CheckedElement { bool violation, is_nan; unsigned int bin, bits; };
template <bool SHORTCUT = true>
__device__ __forceinline__ CheckedElement check_arith(float c, float r, float t, double alpha, double eps_rel) {
    CheckedElement o;
    const double rd = (double)r;
    const double T = alpha * (double)t;
    const double den = fabs(rd) + eps_rel;
    if (SHORTCUT && c == r && fabsf(c) != INFINITY) {
        o.violation = !(0.0 <= T);
        o.is_nan = !(den > 0.0);                             // 0/0
        o.bits = 0u;
        o.bin = o.is_nan ? (unsigned)(kBins - 1) : 0u;
        return o;
    }
    const double d = fabs((double)c - rd);
    o.violation = !(d <= T);
    const double e = d / den;
    const float e32 = (float)e;
    o.bin = error_bin(e32, o.is_nan);
    o.bits = __float_as_uint(e32);
    return o;
}

// Four elements at once, as straight-line code: the four chains of dependent binary64 operations are
// independent of one another, so the compiler interleaves them and a wavefront does not sit out the
// latency of every operation of every element in turn (element by element, each behind its own test
// for the shortcut, that is what happened).  The shortcut is taken for the four together or not at
// all; the full arithmetic returns the shortcut's result for an element that qualifies (d = 0, e = 0 or
// 0/0), so the profile does not depend on the route.
// own: a bit for each that counts (all of them, unless a row's end cuts the four).
template <int R = kReplicas>
__device__ __forceinline__ void check_four(const float (&c)[4], const float (&r)[4], const float (&t)[4], double alpha,
                                           double eps_rel, unsigned int* hist, int rep, ThreadAcc& acc, unsigned own = 15u) {
    bool same = true;
#pragma unroll
    for (int i = 0; i < 4; ++i) same = same && c[i] == r[i] && fabsf(c[i]) != INFINITY;
    CheckedElement o[4];
    if (same) {
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = check_arith<true>(c[i], r[i], t[i], alpha, eps_rel);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = check_arith<false>(c[i], r[i], t[i], alpha, eps_rel);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned int mine = own >> i & 1u;
        acc.violations += o[i].violation & mine;
        acc.nans += o[i].is_nan & mine;
        acc.max_bits = max(acc.max_bits, o[i].is_nan || !mine ? 0u : o[i].bits);
        atomicAdd(&hist[o[i].bin * R + rep], mine);
    }
}

// R: copies of every bin in the LDS histogram `hist` (copy `rep` is used).
template <int R = kReplicas>
__device__ __forceinline__ void check_one(float c, float r, float t, double alpha, double eps_rel,
                                          unsigned int* hist, int rep, ThreadAcc& acc) {
    const CheckedElement o = check_arith(c, r, t, alpha, eps_rel);
    acc.violations += o.violation;
    acc.nans += o.is_nan;
    if (!o.is_nan) acc.max_bits = max(acc.max_bits, o.bits);
    atomicAdd(&hist[o.bin * R + rep], 1u);
}

// Quick settlement of an element in binary32.  The check's results do not need the error of every element to the
// last bit: the histogram takes its leading 11 bits, the maximum is one element's, and a violation is a comparison.  A
// binary32 estimate of the error (relative error below 2^-21: a subtraction, an addition, v_rcp_f32 and a
// product) and a lower estimate of alpha tau therefore decide, unless the estimate lies within 16 steps of an edge of
// its bin, might exceed the largest error the workgroup has seen exactly so far, is not clearly below alpha tau, or
// is no ordinary number; such elements (about one in 2^15, and the first ones) take check_arith, so the results are
// the same bit for bit.  About 18 instructions instead of 35, a dozen of them a binary64 division.
// alpha for the estimates: lowered by 2^-18; NaN, which settles nothing, unless it is an ordinary factor (a NaN alpha
// admits no element and an infinite one none whose bound is 0, which no estimate tells apart) and the model's
// constants, which the estimates take as binary32 factors, are ordinary too.
inline float quick_alpha(double alpha, const tao_fp_model& m) {
    auto ordinary = [](double c) { return c == 0.0 || c >= 0x1p-20; };
    const bool ok = alpha >= 0x1p-30 && alpha <= 0x1p30 && m.u >= 0x1p-40 && ordinary(m.c_exp) && ordinary(m.c_erf) && ordinary(m.c_rsqrt) &&
                    ordinary(m.c_div) && ordinary(m.c_log) && ordinary(m.c_sin) && ordinary(m.c_cos) && ordinary(m.c_tanh) && ordinary(m.c_pow);
    return ok ? (float)(alpha * (1.0 - 0x1p-18)) : NAN;
}
struct QuickCheck {
    float alpha, eps;
    __device__ __forceinline__ QuickCheck(float a, double e)
        : alpha(a), eps(e >= 0x1p-60 && e <= 0x1p60 ? (float)e : INFINITY) {}   // (an infinite eps settles nothing)
};
// at <= alpha tau (1 + 2^-18), or beyond 2^120 (an overflow on the way: settles nothing, nor does NaN); known: bits of an error that occurs.  bin: the error's bin.
__device__ __forceinline__ bool quick_settled(float c, float r, float at, const QuickCheck& q, unsigned known, unsigned& bin) {
    const float d = fabsf(c - r);
    const float den = fabsf(r) + q.eps;
    const unsigned bits = __float_as_uint(d * __builtin_amdgcn_rcpf(den));
    bin = bits >> 20;
    const bool zero = d == 0.f;                              // exactly: c == r
    const unsigned t = bits + 16u;
    const float lhs = zero ? 0.f : fmaf(d, 1.f + 0x1p-16f, 0x1p-90f);     // (a bound near the subnormal range settles nothing)
    return lhs <= at && at <= 0x1p120f && den <= 0x1p100f && (zero || ((t & 0xfffffu) >= 32u && t <= known));
}
typedef float floatv4 __attribute__((ext_vector_type(4)));      // (indexed by a variable it stays in registers)
// Four elements: settled together or checked exactly, with tau(i) the binary32 bound of element i.  largest: the
// workgroup's largest exactly computed error (LDS), known: this thread's copy, no newer than it needs to be.  WIDE: the
// exact way takes the four side by side, for kernels that have the registers (small tensors see little else);
// otherwise one after the other in a loop, as four binary64 divisions would set the kernel's register count.
// attempt: false goes the exact way at once (before any error is known, known == 0, only equal values can be settled).
// own: as in check_four; with any that does not count the caller passes 0 for its c, r and at, and the estimates, which take it for an error of
// 0, add one to bin 0 for it (`beyond`, to be taken off).
// Returns whether the estimates settled them.
template <bool WIDE, int R = kReplicas, class Tau>
__device__ __forceinline__ bool quick_check_four(floatv4 c, floatv4 r, floatv4 at, Tau&& tau,
                                                 const QuickCheck& q, double alpha, double eps_rel, unsigned int* hist, int rep,
                                                 ThreadAcc& acc, unsigned int* largest, unsigned& known, bool attempt, unsigned own = 15u) {
    if (attempt) {
        unsigned bin[4];
        bool ok = true;
#pragma unroll
        for (int i = 0; i < 4; ++i) ok &= quick_settled(c[i], r[i], at[i], q, known, bin[i]);
        if (ok) {
#pragma unroll
            for (int i = 0; i < 4; ++i) atomicAdd(&hist[bin[i] * R + rep], 1u);
            return true;
        }
    }
    if (WIDE) {
        const float c4[4] = {c[0], c[1], c[2], c[3]}, r4[4] = {r[0], r[1], r[2], r[3]};
        const float t4[4] = {tau(0), tau(1), tau(2), tau(3)};
        check_four<R>(c4, r4, t4, alpha, eps_rel, hist, rep, acc, own);
    } else {
#pragma unroll 1
        for (int i = 0; i < 4; ++i)
            if (own >> i & 1u) check_one<R>(c[i], r[i], tau(i), alpha, eps_rel, hist, rep, acc);
    }
    if (acc.max_bits > known) atomicMax(largest, acc.max_bits);
    known = max(known, acc.max_bits);
    return false;
}
__device__ __forceinline__ unsigned newest(unsigned int* largest) {
    return __hip_atomic_load(largest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Workgroup totals of the per-thread counters (kCheckThreads threads) into ws_stats[blockIdx.x];
// red: 3 * (kCheckThreads / kWave) words of LDS.  Contains one barrier.
__device__ __forceinline__ void flush_block_stats(const ThreadAcc& acc, unsigned int* red, BlockStats* __restrict__ ws_stats) {
    const int tid = threadIdx.x;
    const unsigned int v = wave_sum(acc.violations), q = wave_sum(acc.nans), m = wave_max(acc.max_bits);
    const int wave = tid / kWave;
    if ((tid & (kWave - 1)) == 0) { red[wave * 3] = v; red[wave * 3 + 1] = q; red[wave * 3 + 2] = m; }
    __syncthreads();
    static_assert(kCheckThreads / kWave == 16, "a row of lanes reads the wavefronts' totals");
    if (tid < 16) {
        const unsigned long long vs = wave_all<0, 4>((unsigned long long)red[tid * 3], [](unsigned long long a, unsigned long long b) { return a + b; });
        const unsigned long long qs = wave_all<0, 4>((unsigned long long)red[tid * 3 + 1], [](unsigned long long a, unsigned long long b) { return a + b; });
        const unsigned int ms = wave_all<0, 4>(red[tid * 3 + 2], [](unsigned int a, unsigned int b) { return max(a, b); });
        if (tid == 0) {
            BlockStats& o = ws_stats[blockIdx.x];
            o.violations = vs; o.nans = qs; o.max_bits = ms;
        }
    }
}

// The caller's workspace: kMaxCheckBlocks partial histograms, their coarse group counts, the counters.
struct CheckWorkspace {
    unsigned int* hist; unsigned int* coarse; BlockStats* stats;
};
constexpr size_t check_workspace_bytes() {
    return (size_t)kMaxCheckBlocks * ((kBins + kGroups) * sizeof(unsigned int) + sizeof(BlockStats));
}
inline CheckWorkspace carve_check_workspace(void* ws) {
    CheckWorkspace w;
    w.hist = (unsigned int*)ws;
    w.coarse = w.hist + (size_t)kMaxCheckBlocks * kBins;
    w.stats = (BlockStats*)(w.coarse + (size_t)kMaxCheckBlocks * kGroups);
    return w;
}
// What the finalising kernel needs to know of the tensor: its size and the nearest ranks of p50, p99 and p99.9.
struct ProfileSize { unsigned long long n; Ranks<3> ranks; };
inline ProfileSize profile_size(unsigned long long n) { return {n, {{rank_of(n, 1, 2), rank_of(n, 99, 100), rank_of(n, 999, 1000)}}}; }
// Group `grp` of the profile of the partial results of `nblocks` (at most PARTIALS) pass-1 workgroups, by one workgroup of
// THREADS threads; group 0 brings the scalar fields.  Loads first (construct it early), then finish().
// smem: profile_smem_words(THREADS) 64-bit words.
constexpr int profile_smem_words(int threads) { return threads + 4 * (threads / kWave); }
template <int THREADS, int PARTIALS>
struct ProfileGroup {
    GroupLoads<THREADS, PARTIALS> loads;
    unsigned long long v = 0, q = 0;
    unsigned int m = 0;
    int grp;
    __device__ __forceinline__ ProfileGroup(const CheckWorkspace& w, int nblocks, int g) : loads(w.hist, w.coarse, nblocks, g), grp(g) {
        if (grp == 0) {                                      // counters of pass 1
#pragma unroll
            for (int k = threadIdx.x; k < PARTIALS; k += THREADS)
                if (k < nblocks) { v += w.stats[k].violations; q += w.stats[k].nans; m = max(m, w.stats[k].max_bits); }
        }
    }
    // counted: all violations are in the partial results (else violations and accept are left to the caller)
    __device__ __forceinline__ void finish(const ProfileSize& size, tao_profile* out, unsigned long long* smem, bool counted = true) {
        constexpr int WAVES = THREADS / kWave;
        const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
        unsigned long long* wv = smem + THREADS + WAVES;
        unsigned long long* wq = wv + WAVES;
        unsigned int* wm = reinterpret_cast<unsigned int*>(wq + WAVES);
        if (grp == 0) {
            v = wave_sum(v); q = wave_sum(q); m = wave_max(m);
            if (lane == 0) { wv[wave] = v; wq[wave] = q; wm[wave] = m; }
        }
        // the three bin and three edge fields of tao_profile are consecutive
        reduce_group<3>(loads, grp, out->hist, size.ranks, &out->p50_bin, &out->p50, smem);
        if (grp == 0 && tid == kWave) {                      // (reduce_group's barrier lies between; not the wavefront that takes the bins)
            v = 0; q = 0; m = 0;
#pragma unroll
            for (int k = 0; k < WAVES; ++k) { v += wv[k]; q += wq[k]; m = max(m, wm[k]); }
            out->n = size.n;
            if (counted) { out->violations = v; out->accept = (v == 0) ? 1u : 0u; }
            out->nan_count = q;
            out->max_rel = __uint_as_float(m);
            out->pad_ = 0;
            if (size.n == 0) {
                out->p50_bin = out->p99_bin = out->p999_bin = 0;
                out->p50 = out->p99 = out->p999 = bin_upper_edge(0);
            }
        }
    }
};
// What a check pass leaves: partial results, or (alone) the profile itself.
struct PassOut {
    CheckWorkspace w;
    tao_profile* alone;
    ProfileSize size;
};
// The end of a check pass (kCheckThreads threads): its workgroup's LDS histogram and counters to the partial results, or, where it is the
// only one, the profile from them at once: a small tensor's check is then one launch.  GPU us with the finalising kernel / alone: streaming check of
// 100 elements 8.2 / 2.9, 8192 9.4 / 5.0, 16384 7.9 / 7.5 (and 24576 7.9 / 10); GELU, whose bound is longer, of 8192 9.5 / 8.4.
// red: kRedWords words of LDS.
constexpr long kAloneElements = 16384;
constexpr int kRedWords = 4 * (kCheckThreads / kWave);
__device__ __forceinline__ void finish_pass(const unsigned int* hist, const ThreadAcc& acc, unsigned int* red, const PassOut& o) {
    if (!o.alone) {
        flush_block_stats(acc, red, o.w.stats);
        flush_histogram(hist, o.w.hist + (size_t)blockIdx.x * kBins, o.w.coarse + blockIdx.x * kGroups);
        return;
    }
    static_assert(kBins == 2 * kCheckThreads && kCheckThreads / kWave == 16, "two bins a thread, a row of lanes for the wavefronts");
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    __syncthreads();                                         // (the histogram is complete)
    unsigned int c[2] = {0, 0};
#pragma unroll
    for (int r = 0; r < kReplicas; ++r) { c[0] += hist[2 * tid * kReplicas + r]; c[1] += hist[(2 * tid + 1) * kReplicas + r]; }
    const unsigned int mine = c[0] + c[1];                   // (at most kAloneMost elements: every sum here fits 32 bits)
    const unsigned int upto = (unsigned int)wave_scan(mine);
    const unsigned int v = wave_sum(acc.violations), q = wave_sum(acc.nans), m = wave_max(acc.max_bits);
    if (lane == kWave - 1) { red[wave * 4] = v; red[wave * 4 + 1] = q; red[wave * 4 + 2] = m; red[wave * 4 + 3] = upto; }
    __syncthreads();
    const auto sum = [](unsigned int a, unsigned int b) { return a + b; };
    const int other = lane & 15;                             // every row of lanes holds the 16 wavefronts' totals
    const unsigned int before = wave_all<0, 4>(other < wave ? red[other * 4 + 3] : 0u, sum);
    unsigned long long below = before + upto - mine;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const unsigned int bin = 2 * tid + j;
        o.alone->hist[bin] = c[j];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const unsigned long long r = o.size.ranks.at[i];
            if (below < r && r <= below + c[j]) { (&o.alone->p50_bin)[i] = bin; (&o.alone->p50)[i] = bin_upper_edge(bin); }
        }
        below += c[j];
    }
    if (wave == 0) {
        const unsigned int vs = wave_all<0, 4>(red[other * 4], sum), qs = wave_all<0, 4>(red[other * 4 + 1], sum);
        const unsigned int ms = wave_all<0, 4>(red[other * 4 + 2], [](unsigned int a, unsigned int b) { return max(a, b); });
        if (lane == 0) {
            tao_profile* out = o.alone;
            out->n = o.size.n; out->violations = vs; out->nan_count = qs;
            out->max_rel = __uint_as_float(ms); out->accept = vs == 0 ? 1u : 0u; out->pad_ = 0;
            if (o.size.n == 0) {
                out->p50_bin = out->p99_bin = out->p999_bin = 0;
                out->p50 = out->p99 = out->p999 = bin_upper_edge(0);
            }
        }
    }
}
// Enqueue the finalising kernel over the partials of `nblocks` pass-1 workgroups (defined with the check pass).
void launch_profile_reduce(const CheckWorkspace& w, int nblocks, unsigned long long n, tao_profile* out, hipStream_t st);
// One workgroup forms the profile itself where it is alone, in sums of 32 bits; a longer tensor that one workgroup takes (a single row of
// any length) goes through the finalising kernel, which adds in 64.
constexpr long kAloneMost = 0xffffffffL;
inline bool forms_profile(int nblocks, long n) { return nblocks == 1 && n <= kAloneMost; }
// The outputs of a pass of `nblocks` workgroups over n elements, and the finalising kernel where the pass does not end with the profile.
inline PassOut pass_out(const CheckWorkspace& w, int nblocks, long n, tao_profile* out) {
    return {w, forms_profile(nblocks, n) ? out : nullptr, profile_size((unsigned long long)n)};
}
inline void launch_finish(const CheckWorkspace& w, int nblocks, long n, tao_profile* out, hipStream_t st) {
    if (!forms_profile(nblocks, n)) launch_profile_reduce(w, nblocks, (unsigned long long)n, out, st);
}

}  // namespace tao
