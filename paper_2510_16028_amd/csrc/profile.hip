// tao_profile_errors: absolute and relative element-wise errors between two outputs of one
// operator (Sec. 3.2 Eq. 1-2), their percentile profiles on the 22-point grid
// P = {1, 5, 10, ..., 95, 99, 100} (Sec. 3.2 / Sec. 5.3) and the selection statistic
//     p_max = max_p { p_abs(p)/thr_abs(p), p_rel(p)/thr_rel(p) },   offending iff p_max > 1
// that the dispute game uses to pick the child to descend into (Sec. 5.3).
//
// Pass 1 (errors_pass): grid-stride over 16-byte vectors of both inputs; per element IEEE
// binary64 arithmetic (no contraction), two lane-replicated 2048-bin LDS histograms, partial
// histograms and counters to the workspace (no global atomics: the result does not depend on
// scheduling).  Pass 2 (errors_reduce): one workgroup per 64 bins of either histogram sums the
// partials and locates the 22 nearest-rank percentiles; the last of them to finish has the exact
// maxima, percentile values capped by the maximum and threshold ratios.
#include "tao_hist.hpp"
#include "tao_host.hpp"

namespace tao {

constexpr int kErrThreads = 1024;            // one workgroup per CU
constexpr int kErrReplicas = 4;              // two histograms of 4 x 2048 counters: 64 KB of LDS
constexpr int kGrid = TAO_NGRID;

struct ErrStats {            // one per pass-1 workgroup
    unsigned int nans;                         // (n < 2^36: at most 2^28 elements each)
    unsigned int done;                         // the first one's: workgroups of pass 2 that have finished
    unsigned int max_abs_bits, max_rel_bits;   // bit patterns of the largest non-NaN errors (>= 0)
};
static_assert(sizeof(ErrStats) == 16, "as the workspace's size counts them");

inline unsigned int grid_percent(int g) {
    return g == 0 ? 1u : (g <= 19 ? 5u * (unsigned)g : (g == 20 ? 99u : 100u));
}

__device__ __forceinline__ void error_one(float c, float r, double eps_rel, unsigned int* hist_a,
                                          unsigned int* hist_r, int rep, unsigned int& nans,
                                          unsigned int& max_a, unsigned int& max_r) {
    const double cd = (double)c, rd = (double)r;
    const double d = fabs(cd - rd);
    const double den = fabs(rd) + eps_rel;
    const double e = d / den;
    const float a32 = (float)d, e32 = (float)e;
    bool an, en;
    const unsigned int ba = error_bin(a32, an), be = error_bin(e32, en);
    nans += en;
    if (!en) max_r = max(max_r, __float_as_uint(e32));
    if (!an) max_a = max(max_a, __float_as_uint(a32));
    atomicAdd(&hist_a[ba * kErrReplicas + rep], 1u);
    atomicAdd(&hist_r[be * kErrReplicas + rep], 1u);
}

__global__ __launch_bounds__(kErrThreads) void errors_pass(
    const float* __restrict__ claimed, const float* __restrict__ ref, long n, int vec_ok, double eps_rel,
    unsigned int* __restrict__ ws_hist_a, unsigned int* __restrict__ ws_hist_r,
    unsigned int* __restrict__ ws_coarse_a, unsigned int* __restrict__ ws_coarse_r,
    ErrStats* __restrict__ ws_stats) {
    __shared__ unsigned int hist_a[kBins * kErrReplicas], hist_r[kBins * kErrReplicas];
    __shared__ unsigned int red[3 * (kErrThreads / kWave)];
    const int tid = threadIdx.x;
    for (int i = tid; i < kBins * kErrReplicas; i += kErrThreads) { hist_a[i] = 0; hist_r[i] = 0; }
    __syncthreads();

    unsigned int nans = 0, max_a = 0, max_r = 0;
    const int rep = tid & (kErrReplicas - 1);
    const long nvec = vec_ok ? (n >> 2) : 0;
    const long stride = (long)gridDim.x * kErrThreads;
    const auto four = [&](const float4& c4, const float4& r4) __attribute__((always_inline)) {
        error_one(c4.x, r4.x, eps_rel, hist_a, hist_r, rep, nans, max_a, max_r);
        error_one(c4.y, r4.y, eps_rel, hist_a, hist_r, rep, nans, max_a, max_r);
        error_one(c4.z, r4.z, eps_rel, hist_a, hist_r, rep, nans, max_a, max_r);
        error_one(c4.w, r4.w, eps_rel, hist_a, hist_r, rep, nans, max_a, max_r);
    };
    const float4* const cv = reinterpret_cast<const float4*>(claimed);
    const float4* const rv = reinterpret_cast<const float4*>(ref);
    long i = (long)blockIdx.x * kErrThreads + tid;
    for (; i + stride < nvec; i += 2 * stride) {               // (two of each under way: 8.4 M elements 16.2 us, one 17.4)
        const float4 c0 = ntload4(cv + i), r0 = ntload4(rv + i), c1 = ntload4(cv + i + stride), r1 = ntload4(rv + i + stride);
        four(c0, r0);
        four(c1, r1);
    }
    if (i < nvec) four(ntload4(cv + i), ntload4(rv + i));
    // scalar remainder (everything when the inputs are not 16-byte aligned)
    for (i = (nvec << 2) + (long)blockIdx.x * kErrThreads + tid; i < n; i += stride)
        error_one(claimed[i], ref[i], eps_rel, hist_a, hist_r, rep, nans, max_a, max_r);

    nans = wave_sum(nans); max_a = wave_max(max_a); max_r = wave_max(max_r);
    const int wave = tid / kWave;
    if ((tid & (kWave - 1)) == 0) { red[wave * 3] = nans; red[wave * 3 + 1] = max_a; red[wave * 3 + 2] = max_r; }
    __syncthreads();
    static_assert(kErrThreads / kWave == 16, "a row of lanes reads the wavefronts' totals");
    if (tid < 16) {
        const unsigned int ns = wave_all<0, 4>(red[tid * 3], [](unsigned int a, unsigned int b) { return a + b; });
        const auto larger = [](unsigned int a, unsigned int b) { return max(a, b); };
        const unsigned int as = wave_all<0, 4>(red[tid * 3 + 1], larger), rs = wave_all<0, 4>(red[tid * 3 + 2], larger);
        if (tid == 0) ws_stats[blockIdx.x] = ErrStats{ns, 0u, as, rs};
    }
    flush_histogram<kErrReplicas>(hist_a, ws_hist_a + (size_t)blockIdx.x * kBins, ws_coarse_a + blockIdx.x * kGroups);
    flush_histogram<kErrReplicas>(hist_r, ws_hist_r + (size_t)blockIdx.x * kBins, ws_coarse_r + blockIdx.x * kGroups);
}

// One wavefront, a lane per grid point (a thread that takes the 22 points and their divisions in turn needs 9 us, this 4).
__device__ __forceinline__ void errors_finalize(const ErrStats* ws_stats, int nblocks, unsigned long long n, const float* __restrict__ thr_abs,
                                                const float* __restrict__ thr_rel, tao_error_profile* out) {
    static_assert(kGrid <= kWave, "a lane per grid point");
    const int lane = threadIdx.x, g = lane < kGrid ? lane : 0;
    unsigned int ba = out->abs_bin[g], br = out->rel_bin[g];
    float pa = out->abs_p[g], pr = out->rel_p[g];
    const bool with_thr = thr_abs && thr_rel;
    const float ta = with_thr ? thr_abs[g] : 0.f, tr = with_thr ? thr_rel[g] : 0.f;
    unsigned long long qn = 0; unsigned int ma = 0, mr = 0;
#pragma unroll
    for (int j = 0; j < kMaxPartials / kWave; ++j) {
        const int k = lane + j * kWave;
        if (k < nblocks) { qn += ws_stats[k].nans; ma = max(ma, ws_stats[k].max_abs_bits); mr = max(mr, ws_stats[k].max_rel_bits); }
    }
    qn = wave_sum(qn); ma = wave_max(ma); mr = wave_max(mr);
    const float max_abs = __uint_as_float(ma), max_rel = __uint_as_float(mr);
    if (n == 0) { ba = br = 0; pa = pr = bin_upper_edge(0); }
    // a percentile cannot exceed the exact maximum (p = 100 is the maximum itself)
    if (n > 0 && ba < (unsigned)(kBins - 1) && pa > max_abs) pa = max_abs;
    if (n > 0 && br < (unsigned)(kBins - 1) && pr > max_rel) pr = max_rel;
    double pmax = NAN;                                       // the largest ratio that is not NaN (0/0), NaN if there is none
    const auto larger = [](double a, double b) { return a == a && !(b > a) ? a : b; };
    if (with_thr && lane < kGrid) pmax = larger((double)pa / (double)ta, (double)pr / (double)tr);
    pmax = wave_all(pmax, larger);
    if (lane < kGrid) { out->abs_bin[g] = ba; out->rel_bin[g] = br; out->abs_p[g] = pa; out->rel_p[g] = pr; }
    if (lane != 0) return;
    out->n = n; out->nan_count = qn; out->max_abs = max_abs; out->max_rel = max_rel; out->pad_ = 0;
    out->p_max = pmax;
    out->offending = (pmax > 1.0) ? 1u : 0u;
}

// workgroups 0 .. 31: absolute-error histogram; 32 .. 63: relative-error histogram.  The last one to finish sees the others' percentiles
// (fences on both sides of the count); in a launch of its own that part took 2 to 4 us, and the host 3.6.
__global__ __launch_bounds__(kReduceThreads) void errors_reduce(
    const unsigned int* __restrict__ ws_hist_a, const unsigned int* __restrict__ ws_hist_r,
    const unsigned int* __restrict__ ws_coarse_a, const unsigned int* __restrict__ ws_coarse_r,
    ErrStats* ws_stats, int nblocks, unsigned long long n, Ranks<kGrid> ranks, const float* __restrict__ thr_abs,
    const float* __restrict__ thr_rel, tao_error_profile* out) {
    __shared__ unsigned long long smem[kReduceThreads + kReduceWaves];
    const bool rel = blockIdx.x >= (unsigned)kGroups;
    const int grp = rel ? blockIdx.x - kGroups : blockIdx.x;
    const GroupLoads<kReduceThreads, kMaxPartials> loads(rel ? ws_hist_r : ws_hist_a, rel ? ws_coarse_r : ws_coarse_a, nblocks, grp);
    reduce_group<kGrid>(loads, grp, rel ? out->hist_rel : out->hist_abs, ranks, rel ? out->rel_bin : out->abs_bin,
                        rel ? out->rel_p : out->abs_p, smem);
    if (threadIdx.x >= kWave) return;                          // (the first wavefront has written the results)
    __threadfence();
    unsigned finished = 0;
    if (threadIdx.x == 0) finished = atomicAdd(&ws_stats[0].done, 1u);
    if (__builtin_amdgcn_readfirstlane(finished) != gridDim.x - 1) return;
    __threadfence();
    errors_finalize(ws_stats, nblocks, n, thr_abs, thr_rel, out);
}

// Calibration (Sec. 3.2): per grid point the maximum over the runs' percentile values (NaN entries
// skipped) and alpha times it, the product one binary64 multiplication rounded up to binary32.
// One thread per (kind, grid point); the runs are read with independent strided loads.
__global__ __launch_bounds__(64) void calibrate_kernel(const tao_error_profile* __restrict__ profiles, long count,
                                                       double alpha, float* __restrict__ env_abs,
                                                       float* __restrict__ env_rel, float* __restrict__ thr_abs,
                                                       float* __restrict__ thr_rel) {
    const int t = threadIdx.x;
    if (t >= 2 * kGrid) return;
    const bool rel = t >= kGrid;
    const int g = rel ? t - kGrid : t;
    float m = NAN;
    for (long r = 0; r < count; ++r) {
        const float v = rel ? profiles[r].rel_p[g] : profiles[r].abs_p[g];
        if (v == v && !(m >= v)) m = v;
    }
    float* env = rel ? env_rel : env_abs;
    if (env) env[g] = m;
    (rel ? thr_rel : thr_abs)[g] = up32(alpha * (double)m);
}

}  // namespace tao

extern "C" {

int tao_calibrate_thresholds(const tao_error_profile* profiles, long count, double alpha,
                             float* env_abs, float* env_rel, float* thr_abs, float* thr_rel, void* stream) {
    using namespace tao;
    if (count < 1 || !(alpha >= 0.0) || !std::isfinite(alpha)) return TAO_ERR_SHAPE;
    if (!profiles || !thr_abs || !thr_rel) return TAO_ERR_NULL;
    if (!aligned(profiles, 8) || !aligned(env_abs, 4) || !aligned(env_rel, 4) || !aligned(thr_abs, 4) || !aligned(thr_rel, 4))
        return TAO_ERR_ALIGN;
    hipLaunchKernelGGL(calibrate_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, profiles, count, alpha,
                       env_abs, env_rel, thr_abs, thr_rel);
    return launch_status();
}

size_t tao_profile_workspace_bytes(long n) {
    (void)n;
    return (size_t)tao::kMaxPartials *
           (2 * (tao::kBins + tao::kGroups) * sizeof(unsigned int) + sizeof(tao::ErrStats));
}

int tao_profile_errors(const float* claimed, const float* ref, long n, double eps_rel,
                       const float* thr_abs, const float* thr_rel, tao_error_profile* out,
                       void* ws, size_t ws_bytes, void* stream) {
    using namespace tao;
    if (!out || !ws) return out ? TAO_ERR_WORKSPACE : TAO_ERR_NULL;
    if (n < 0 || !(eps_rel >= 0.0)) return TAO_ERR_SHAPE;       // a negative or NaN eps_rel has no meaning
    if (n > 0 && (!claimed || !ref)) return TAO_ERR_NULL;
    if ((thr_abs == nullptr) != (thr_rel == nullptr)) return TAO_ERR_NULL;
    if (!aligned(claimed, 4) || !aligned(ref, 4) || !aligned(thr_abs, 4) || !aligned(thr_rel, 4) || !aligned(out, 8))
        return TAO_ERR_ALIGN;
    if (!aligned(ws, 256) || ws_bytes < tao_profile_workspace_bytes(n)) return TAO_ERR_WORKSPACE;
    if (n >= (1L << 36)) return TAO_ERR_SHAPE;   // 32-bit per-workgroup counters
    hipStream_t st = (hipStream_t)stream;
    const int vec_ok = aligned(claimed, 16) && aligned(ref, 16);
    // (one vector per thread before another workgroup, as in the check pass: 65536 elements 16.0 against 19.6 us with four)
    long want = (n + (long)kErrThreads * 4 - 1) / ((long)kErrThreads * 4);
    const int nblocks = (int)(want < 1 ? 1 : (want > kMaxPartials ? kMaxPartials : want));
    unsigned int* ws_hist_a = (unsigned int*)ws;
    unsigned int* ws_hist_r = ws_hist_a + (size_t)kMaxPartials * kBins;
    unsigned int* ws_coarse_a = ws_hist_r + (size_t)kMaxPartials * kBins;
    unsigned int* ws_coarse_r = ws_coarse_a + (size_t)kMaxPartials * kGroups;
    ErrStats* ws_stats = (ErrStats*)(ws_coarse_r + (size_t)kMaxPartials * kGroups);
    hipLaunchKernelGGL(errors_pass, dim3(nblocks), dim3(kErrThreads), 0, st, claimed, ref, n, vec_ok, eps_rel,
                       ws_hist_a, ws_hist_r, ws_coarse_a, ws_coarse_r, ws_stats);
    Ranks<kGrid> ranks;
    for (int g = 0; g < kGrid; ++g) ranks.at[g] = rank_of((unsigned long long)n, grid_percent(g), 100);
    hipLaunchKernelGGL(errors_reduce, dim3(2 * kGroups), dim3(kReduceThreads), 0, st, ws_hist_a, ws_hist_r,
                       ws_coarse_a, ws_coarse_r, ws_stats, nblocks, (unsigned long long)n, ranks, thr_abs, thr_rel, out);
    return launch_status();
}

}  // extern "C"
