// Projections of a tentative perturbation onto the verifier's admissible sets (Sec. 4.4).
//
//   project_clip       (i)  clip(delta, -alpha tau, alpha tau): one streaming pass.
//   project_empirical  (ii) cap the k-th smallest magnitude by the cap curve of Sec. 4.2 at rank
//                      (k - 1/2)/n, after a running maximum over k, and put sign and place back.
//
// (ii) needs an element's rank, i.e. a stable sort of the magnitudes, but only where its cap may bind.  A
// histogram over the leading 11 bits (eight bins to an octave) gives the first rank of every bin;
// caps do not decrease with the rank, so a bin whose largest magnitude stays within the cap of its first rank
// needs no ranks at all.  The elements of the other bins, the candidates, are sorted; a candidate's rank is
// its place among them plus the number of others in lower bins.  With a heavy upper tail over a calibrated
// threshold that is a tenth of the tensor; where every bin is a candidate the histogram is the only extra work.
// (8.4 M elements: none capped 257 -> 74 us, a heavy tail against calibrated thresholds 260 -> 104 us, all capped 343 -> 350 us;
// 67 M: 1608 -> 325, 1621 -> 354, 2406 -> 2415 us.  Since the counting pass leaves each
// tile its candidates closed up, and the first scatter reads those and not delta: none capped 74 -> 67 us, 34 M 168 -> 147, 67 M 325 -> 287;
// where most is sorted, and no tile is closed up, 67 M and 134 M take 0.3 % longer.)  What bounds it now (8.4 M elements, a heavy tail 86 us): two passes over delta, 30 us, and the latencies of some fifteen launches.
// The sort is a least-significant-digit radix sort of the 31 magnitude bits (a non-negative binary32 orders like
// its bit pattern, NaN above infinity) in four 8-bit passes; the payload is the element's index
// with its sign bit on top.  Per pass: count (digit histogram per tile), scan (of each digit's counters over
// the tiles; the digits' own totals are scanned by every workgroup of the next kernel), scatter (stable
// rank inside the tile by wave-wide digit matching, elements
// reordered in LDS so that runs of one digit leave as contiguous writes).  The first pass drops
// what is no candidate: its count kernel reads delta (and copies it to out when the two differ) and leaves tiles of few
// candidates closed up, its scatter kernel reads those, and delta where a tile is not closed up.  The last pass writes no
// sorted array at all: the destination of an element gives its rank, so the cap is evaluated there and only the
// elements that exceed their cap are written, straight to out[index] -- the one access of the
// whole path that is random, 4 bytes per 64-byte line, and therefore kept to the elements that
// need it.
//
// The running maximum over ranks needs no scan: the cap curve is piecewise linear in the rank and
// every operation of its formula is monotone under rounding, so inside one segment of the curve
// the computed caps are monotone and the maximum over the ranks up to k is the larger of
// C(first rank of the segment), C(k) and the maxima of the earlier segments (their first and last
// ranks).  A one-wave kernel tabulates those per segment.
#include "tao_device.hpp"
#include "tao_host.hpp"

namespace tao {

constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortItems = 16;                                // per thread
constexpr int kSortTile = kSortThreads * kSortItems;          // 4096 elements per workgroup
constexpr int kRadix = 256;
constexpr int kScanChunk = kSortThreads * 16;                 // counters per step of a scan
constexpr int kMagBins = 2048;                                // bins of the leading 11 magnitude bits
constexpr int kMagShift = 20;
constexpr int kXcds = 8;
// Up to which a scatter pass adds up the tiles' counters itself and the candidates' launch the workgroups' histograms: ten launches for fifteen
// (a usual tail / all capped, us: 50000 elements 58.3 / 107 by fifteen launches, 43.8 / 95.5 so; 262144 64.6 / 111 and 48.9 / 108; at 128 tiles
// 500000 elements 59.5 / 114 and 57.5 / 122).
constexpr int kFewTiles = 64;
constexpr int kCountCopies = 4;                               // histogram copies per wave in radix_count
constexpr int kCountStride = kRadix + 4;                      // copy c of digit d in LDS bank (d + 4c) % 32

// One segment of the cap curve: ranks whose r lies in (p0, p0 + dp].
struct CapSeg {
    double c0, dc, p0, dp;     // C(r) = c0 + dc * ((r - p0) / dp)
    double head;               // max of the caps of all earlier ranks' segments and of this one's first rank
    double inv_dp;             // ~ 1 / dp, for estimates only
};
struct CapTable {
    CapSeg seg[TAO_NGRID];
    double n;                  // (double)n
    double percent_per_rank;   // ~ 100 / n, for estimates only
};

__device__ __forceinline__ double grid_percent(int j) {      // P = {1, 5, 10, ..., 95, 99, 100}
    return j < 0 ? 0.0 : j == 0 ? 1.0 : j < 20 ? 5.0 * j : j == 20 ? 99.0 : 100.0;
}
__device__ __forceinline__ double rank_percent(double k, double n) { return ((k - 0.5) / n) * 100.0; }

// first knot j with r <= P[j]  (r <= 100 always)
__device__ __forceinline__ int segment_of(double r) {
    int j = (int)(r * 0.2);                                   // near r / 5, then settled by comparisons
    j = j < 0 ? 0 : j > TAO_NGRID - 1 ? TAO_NGRID - 1 : j;
    while (j < TAO_NGRID - 1 && r > grid_percent(j)) ++j;
    while (j > 0 && r <= grid_percent(j - 1)) --j;
    return j;
}
__device__ __forceinline__ double cap_in_segment(const CapSeg& s, double r) {
    return s.c0 + s.dc * ((r - s.p0) / s.dp);
}

// Largest binary32 value <= c, for c >= 0.
__device__ __forceinline__ float down32(double c) {
    float f = (float)c;
    if ((double)f > c) f = __uint_as_float(__float_as_uint(f) - 1u);
    return f;
}

// Fills *tab (global or LDS); called by all threads of a workgroup of at least 64, ends with a barrier.
__device__ __forceinline__ void build_cap_table(const float* __restrict__ thr, double alpha, long n, CapTable* tab) {
    __shared__ double seg_max[TAO_NGRID];
    __shared__ long first_rank[TAO_NGRID + 1];
    const int j = threadIdx.x;
    const double dn = (double)n;
    CapSeg s = {};
    if (j < TAO_NGRID) {
        const double c1 = (double)thr[j] * alpha;
        const double c0 = j == 0 ? 0.0 : (double)thr[j - 1] * alpha;
        s.c0 = c0; s.dc = c1 - c0; s.p0 = grid_percent(j - 1); s.dp = grid_percent(j) - grid_percent(j - 1);
        // smallest rank k in [1, n + 1] with r_k > P[j - 1]  (r_k is nondecreasing in k): near n P / 100 + 1/2, then settled by comparisons
        // (by bisection, some 23 divisions one after the other, the kernel took 1.5 us more)
        long k = min(max((long)(dn * (s.p0 * 0.01) + 0.5), 1L), n + 1);
        while (k <= n && !(rank_percent((double)k, dn) > s.p0)) ++k;
        while (k > 1 && rank_percent((double)(k - 1), dn) > s.p0) --k;
        first_rank[j] = k;
    }
    if (j == TAO_NGRID) first_rank[j] = n + 1;
    __syncthreads();
    double cfirst = 0.0;
    if (j < TAO_NGRID) {
        const long kf = first_rank[j], kl = first_rank[j + 1] - 1;
        double m = 0.0;                                       // caps are non-negative: 0 is neutral
        if (kf <= kl) {
            cfirst = cap_in_segment(s, rank_percent((double)kf, dn));
            m = fmax(cfirst, cap_in_segment(s, rank_percent((double)kl, dn)));
        }
        seg_max[j] = m;
    }
    __syncthreads();
    if (j < TAO_NGRID) {
        double head = cfirst;
        for (int e = 0; e < j; ++e) head = fmax(head, seg_max[e]);
        s.head = head;
        s.inv_dp = 1.0 / s.dp;
        tab->seg[j] = s;
    }
    if (j == 0) { tab->n = dn; tab->percent_per_rank = 100.0 / dn; }
    __syncthreads();
}

// The magnitudes' histogram and what follows from it (in the workspace).
struct MagTable {
    unsigned count[kMagBins];
    unsigned others_below[kMagBins];       // elements of lower bins that are no candidates
    unsigned flag[kMagBins / 32];          // one bit per bin: candidates
    unsigned candidates;
    unsigned digit_total[kRadix];          // of the pass under way
};

__global__ void __launch_bounds__(kWave) cap_table_kernel(const float* __restrict__ thr, double alpha, long n,
                                                          CapTable* __restrict__ tab, MagTable* __restrict__ mag) {
    for (int i = threadIdx.x; i < kMagBins; i += kWave) mag->count[i] = 0;
    build_cap_table(thr, alpha, n, tab);
}

// Histogram of the leading magnitude bits: 4 bytes per element read, one set of integer atomics per workgroup (PARTS: a histogram of
// its own instead, which no launch has to clear beforehand).
template <bool PARTS>
__global__ void __launch_bounds__(1024) magnitude_bins(const float* __restrict__ delta, long n, int vec_ok, MagTable* __restrict__ mag,
                                                       unsigned* __restrict__ parts) {
    constexpr int kCopies = 4;
    __shared__ unsigned cnt[kMagBins * kCopies];
    for (int i = threadIdx.x; i < kMagBins * kCopies; i += 1024) cnt[i] = 0;
    __syncthreads();
    const int copy = threadIdx.x & (kCopies - 1);
    const unsigned* src = reinterpret_cast<const unsigned*>(delta);
    auto add = [&](unsigned v) __attribute__((always_inline)) { atomicAdd(&cnt[((v & 0x7fffffffu) >> kMagShift) * kCopies + copy], 1u); };
    const long nvec = vec_ok ? n >> 2 : 0, stride = (long)gridDim.x * 1024;
    long i = (long)blockIdx.x * 1024 + threadIdx.x;
    for (; i + 3 * stride < nvec; i += 4 * stride) {           // (four loads under way: 8.4 M elements 10.8 us, two 11.5)
        uint4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = reinterpret_cast<const uint4*>(src)[i + j * stride];
#pragma unroll
        for (int j = 0; j < 4; ++j) { add(v[j].x); add(v[j].y); add(v[j].z); add(v[j].w); }
    }
    for (; i < nvec; i += stride) { const uint4 a = reinterpret_cast<const uint4*>(src)[i]; add(a.x); add(a.y); add(a.z); add(a.w); }
    for (long e = (nvec << 2) + (long)blockIdx.x * 1024 + threadIdx.x; e < n; e += stride) add(src[e]);
    __syncthreads();
    for (int b = threadIdx.x; b < kMagBins; b += 1024) {
        unsigned t = 0;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) t += cnt[b * kCopies + c];
        if (PARTS) parts[(size_t)blockIdx.x * kMagBins + b] = t;
        else if (t) atomicAdd(&mag->count[b], t);
    }
}

// ---- (i) -------------------------------------------------------------------------------------

__device__ __forceinline__ float clip_one(float d, float t, double alpha) {
    const float a = fabsf(d);
    const double cap = (double)t * alpha;
    const float r = (double)a > cap ? down32(cap) : a;        // NaN compares false and stays
    return copysignf(r, d);
}

__global__ void __launch_bounds__(256) project_clip_kernel(const float* __restrict__ delta, const float* __restrict__ tau,
                                                           double alpha, float* __restrict__ out, long n, int vec_ok) {
    const long stride = (long)gridDim.x * blockDim.x * 4;
    for (long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4; i < n; i += stride) {
        const float4 d = load4<true>(delta, i, n, vec_ok, 0.f);
        const float4 t = load4<true>(tau, i, n, vec_ok, 0.f);
        float4 r;
        r.x = clip_one(d.x, t.x, alpha); r.y = clip_one(d.y, t.y, alpha);
        r.z = clip_one(d.z, t.z, alpha); r.w = clip_one(d.w, t.w, alpha);
        store4(out, i, n, vec_ok, r);
    }
}

// ---- (ii): radix sort passes --------------------------------------------------------------------

// What a pass works on: all of the tensor in the first one, then the candidates.  Few candidates take tiles of a
// quarter or half the size: some 768 tiles, to fill the chip, but no more than the tensor's own (the grid and the
// counters are sized for those).
struct PassShape { long n; int items; long tiles, row; };      // elements, elements per thread, tiles; counters per digit (16-byte rows)
inline __host__ __device__ long counter_row(long tiles) { return (tiles + 3) & ~3L; }
template <bool FIRST>
__device__ __forceinline__ PassShape pass_shape(long all, const MagTable* __restrict__ mag) {
    PassShape p = {all, kSortItems, 0, 0};
    if (!FIRST) {
        p.n = (long)mag->candidates;
        p.items = p.n <= 768L * kSortThreads * 4 && p.n * 4 <= all ? 4 : p.n <= 768L * kSortThreads * 8 && p.n * 2 <= all ? 8 : kSortItems;
    }
    const int tile = p.items * kSortThreads;
    p.tiles = (p.n + tile - 1) / tile;
    p.row = counter_row(p.tiles);
    return p;
}

// Workgroups are dealt round-robin to the eight XCDs; giving XCD x the x-th contiguous eighth of
// the tiles keeps the counter cache lines that neighbouring tiles share inside one L2.
__device__ __forceinline__ long tile_of_block(long tiles_per_xcd) {
    const long i = blockIdx.x / kXcds;                         // (the grid is sized for the whole tensor: -1 beyond a pass's tiles)
    return i < tiles_per_xcd ? (long)(blockIdx.x % kXcds) * tiles_per_xcd + i : -1;
}

// A first pass's tile with few candidates leaves them closed up in the place of its keys and payloads in the second pair of buffers
// (free until the second pass), with how many there are in the last key's place, where no key has the top bit; the scatter kernel then reads
// those and not delta again.  Up to a quarter of the tile, beyond which writing and reading 16 bytes per candidate is more than reading
// 4 per element; tiles that are not read in whole vectors do not either.
constexpr unsigned kClosedUp = 1u << 31, kNotClosedUp = ~0u;
constexpr int kMostClosedUp = kSortTile / 4;
// (no tile is looked at where most of the tensor is to be sorted)
__device__ __forceinline__ bool closes_up(const MagTable* __restrict__ mag, long n) { return (long)mag->candidates * 2 <= n; }

// Digit histogram of every tile: hist[digit * row + tile].  Counting does not depend on the
// order inside the tile, so a thread takes four runs of four consecutive keys (16-byte loads, all
// issued before the first is used).  The first pass also copies delta to out on the way.
template <bool FIRST>
__global__ void __launch_bounds__(kSortThreads) radix_count(const float* delta, const unsigned* __restrict__ keys,
                                                            long all, int shift, int vec_ok, const MagTable* __restrict__ mag,
                                                            unsigned* __restrict__ hist, unsigned* copy_to,
                                                            unsigned* __restrict__ closed_keys, unsigned* __restrict__ closed_vals) {
    __shared__ unsigned piece[FIRST ? kSortItems / 4 : 1][kSortWaves];
    __shared__ unsigned cnt[kSortWaves][kCountCopies][kCountStride];
    __shared__ unsigned flag[FIRST ? kMagBins / 32 : 1];
    const PassShape shape = pass_shape<FIRST>(all, mag);
    const long n = shape.n, tiles = shape.tiles;
    const int items = FIRST ? kSortItems : shape.items;
    const long tile = tile_of_block((tiles + kXcds - 1) / kXcds);
    if (tile < 0 || tile >= tiles) return;                     // whole workgroup
    unsigned flags = 0;                                        // (requested ahead of the keys, put down behind them)
    if (FIRST && threadIdx.x < kMagBins / 32) flags = mag->flag[threadIdx.x];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    for (int d = lane; d < kCountCopies * kCountStride; d += kWave) (&cnt[wave][0][0])[d] = 0;
    __builtin_amdgcn_wave_barrier();
    const unsigned* src = FIRST ? reinterpret_cast<const unsigned*>(delta) : keys;
    const long tile_base = tile * (items * kSortThreads);
    unsigned key[kSortItems];
    const bool full = tile_base + items * kSortThreads <= n;
    bool closed = false;                                       // FIRST: counted as closed up
    if (full && vec_ok) {
#pragma unroll
        for (int q = 0; q < kSortItems / 4; ++q) {
            const long e = tile_base + ((long)q * kSortThreads + threadIdx.x) * 4;
            if (4 * q >= items) continue;
            const uint4 v = *reinterpret_cast<const uint4*>(src + e);
            if (FIRST && copy_to) *reinterpret_cast<uint4*>(copy_to + e) = v;
            key[4 * q] = v.x; key[4 * q + 1] = v.y; key[4 * q + 2] = v.z; key[4 * q + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kSortItems; ++i) {
            const long e = tile_base + (long)i * kSortThreads + threadIdx.x;
            key[i] = i < items && e < n ? src[e] : 0u;
            if (FIRST && copy_to && e < n) copy_to[e] = key[i];
        }
    }
    if (FIRST) {
        if (threadIdx.x < kMagBins / 32) flag[threadIdx.x] = flags;
        __syncthreads();
        // A tile's candidates, where they are few, in order (by vector of the thread, thread, place in the vector): closed up in LDS, and
        // then stored and counted from there, as sixteen steps with a tenth of the lanes each cost more than the loads
        const unsigned long long lanes_below = (1ull << lane) - 1ull;
        unsigned mine = 0, at[kSortItems / 4];                 // mine: a bit per key
        const bool closing = closes_up(mag, n), whole = closing && full && vec_ok;
        unsigned count = 0;
        if (whole) {                                           // (the same in the whole workgroup)
#pragma unroll
            for (int q = 0; q < kSortItems / 4; ++q) {
                unsigned all = 0;
                at[q] = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned bin = (key[4 * q + j] & 0x7fffffffu) >> kMagShift;
                    const bool c = (flag[bin >> 5] >> (bin & 31)) & 1u;
                    const unsigned long long b = __ballot(c);
                    mine |= (unsigned)c << (4 * q + j);
                    at[q] += (unsigned)__popcll(b & lanes_below);
                    all += (unsigned)__popcll(b);
                }
                if (lane == 0) piece[q][wave] = all;
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kSortItems / 4; ++q)
#pragma unroll
                for (int w = 0; w < kSortWaves; ++w) {
                    if (w == wave) at[q] += count;
                    count += piece[q][w];
                }
        }
        closed = whole && count <= (unsigned)kMostClosedUp;
        if (closing && threadIdx.x == 0) closed_keys[min(tile_base + kSortTile, n) - 1] = closed ? kClosedUp | count : kNotClosedUp;
        if (closed) {
            // (they lie in the counters of the other wavefronts: all count in the first one's; with room of their own fewer workgroups fit)
            unsigned* const found_key = &cnt[1][0][0];
            unsigned short* const found_at = reinterpret_cast<unsigned short*>(&cnt[2][0][0]);
            static_assert(kMostClosedUp <= kCountCopies * kCountStride, "in a wavefront's counters");
#pragma unroll
            for (int i = 0; i < kSortItems; ++i) {
                if ((mine >> i) & 1u) {
                    const unsigned to = at[i / 4] + (unsigned)__popc(mine >> (i & ~3) & ((1u << (i & 3)) - 1u));
                    found_key[to] = key[i];
                    found_at[to] = (unsigned short)(((i >> 2) * kSortThreads + threadIdx.x) * 4 + (i & 3));
                }
            }
            __syncthreads();
            for (unsigned e = threadIdx.x; e < count; e += kSortThreads) {
                const unsigned k = found_key[e];
                closed_keys[tile_base + e] = k & 0x7fffffffu;
                closed_vals[tile_base + e] = ((unsigned)tile_base + found_at[e]) | (k & 0x80000000u);
                atomicAdd(&cnt[0][lane & (kCountCopies - 1)][(k >> shift) & (kRadix - 1)], 1u);          // (the first digit: no sign in it)
            }
        }
    }
    if (!closed) {
#pragma unroll
        for (int i = 0; i < kSortItems; ++i) {
            if (i < items) {
                // element index of key[i] in the scalar layout (the vector layout is only used on full tiles)
                bool valid = full || tile_base + (long)i * kSortThreads + threadIdx.x < n;
                if (FIRST) {
                    const unsigned bin = (key[i] & 0x7fffffffu) >> kMagShift;
                    valid = valid && ((flag[bin >> 5] >> (bin & 31)) & 1u);
                }
                const unsigned d = ((FIRST ? key[i] & 0x7fffffffu : key[i]) >> shift) & (kRadix - 1);
                // A wave whose valid lanes all hold one digit (the rule in the top byte of narrow data) adds
                // once.  Otherwise LDS atomics, spread over eight copies of the histogram chosen by the lane
                // (a few distinct digits per wave -- exponent bytes, trailing zero bytes of deviations that are
                // differences of nearby values -- would serialise 64 atomics on a handful of addresses); the
                // copies are 260 counters apart, so equal digits of different copies fall into different banks.
                const unsigned long long vmask = __ballot(valid);
                if (vmask != 0) {
                    const unsigned d0 = __shfl(d, (int)__builtin_ctzll(vmask), kWave);
                    if (__ballot(valid && d == d0) == vmask) {
                        if (lane == (int)__builtin_ctzll(vmask)) cnt[wave][0][d0] += (unsigned)__popcll(vmask);
                    } else if (valid) {
                        atomicAdd(&cnt[wave][lane & (kCountCopies - 1)][d], 1u);
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
    __syncthreads();
    const int d = threadIdx.x;                                 // kSortThreads == kRadix
    unsigned total = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w)
#pragma unroll
        for (int c = 0; c < kCountCopies; ++c) total += w == 0 || !closed ? cnt[w][c][d] : 0u;
    hist[(long)d * shape.row + tile] = total;
}

// Exclusive scan of one value per thread over a workgroup of WAVES wavefronts; ends with a barrier.
// (By row shifts, and with the wavefronts' totals read at once: through LDS permutes and in a loop over the totals a projection of
// 8.4 M elements took 96.5 us against 90.9, one of 50000 62.8 against 58.3.)
template <int WAVES>
__device__ __forceinline__ unsigned block_exclusive_scan(unsigned v, unsigned* wave_tot, unsigned& block_total) {
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const unsigned inc = wave_scan(v);
    if (lane == kWave - 1) wave_tot[wave] = inc;
    __syncthreads();
    unsigned before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { const unsigned t = wave_tot[w]; before += w < wave ? t : 0u; all += t; }
    __syncthreads();
    block_total = all;
    return before + inc - v;
}

// Whether some element of a magnitude bin of `count` elements, the first of them at 0-based rank `first`, may exceed its cap.
__device__ __forceinline__ bool holds_candidates(const CapTable& tab, unsigned bin, unsigned count, unsigned first) {
    if (count == 0 || bin >= (0x7f800000u >> kMagShift) + 1u) return false;                // (NaN stays whatever its rank)
    const float top = bin == (0x7f800000u >> kMagShift) ? INFINITY : __uint_as_float(((bin + 1u) << kMagShift) - 1u);
    const double r = rank_percent((double)first + 1.0, tab.n);
    const CapSeg& sg = tab.seg[segment_of(r)];
    return !((double)top <= fmax(sg.head, cap_in_segment(sg, r)));
}
// Thread t of 1024 has the flags of bins 2 t and 2 t + 1: 16 threads make a word.
__device__ __forceinline__ void leave_flags(bool c0, bool c1, unsigned* flag) {
    const int t = threadIdx.x;
    unsigned bits = ((unsigned)c0 | ((unsigned)c1 << 1)) << 2 * (t & 15);
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) bits |= __shfl_xor(bits, o, kWave);
    if ((t & 15) == 0) flag[t >> 4] = bits;
}

// First rank of every bin, the bins whose elements may exceed their caps, and the numbers that lead from a
// candidate's place to its rank.  One workgroup; thread t has bins 2 t and 2 t + 1.  PARTS: the histogram is the sum of `nparts`
// workgroups', and the cap table is built here.
template <bool PARTS>
__global__ void __launch_bounds__(1024) find_candidates(const float* __restrict__ thr, double alpha, long n, CapTable* __restrict__ tab,
                                                        MagTable* __restrict__ mag, const unsigned* __restrict__ parts, int nparts) {
    static_assert(kMagBins == 2 * 1024, "two bins per thread");
    __shared__ CapTable stab;
    __shared__ __align__(16) unsigned wave_tot[1024 / kWave];
    const int t = threadIdx.x;
    unsigned n0 = 0, n1 = 0, total;
    if (PARTS) {
#pragma unroll 4
        for (int k = 0; k < nparts; ++k) {
            const uint2 c = reinterpret_cast<const uint2*>(parts + (size_t)k * kMagBins)[t];
            n0 += c.x; n1 += c.y;
        }
        build_cap_table(thr, alpha, n, &stab);                 // ends with a barrier
        if (t < (int)(sizeof(CapTable) / sizeof(double))) reinterpret_cast<double*>(tab)[t] = reinterpret_cast<const double*>(&stab)[t];
    } else {
        n0 = mag->count[2 * t]; n1 = mag->count[2 * t + 1];
    }
    const CapTable& caps = PARTS ? stab : *tab;
    const unsigned first0 = block_exclusive_scan<1024 / kWave>(n0 + n1, wave_tot, total), first1 = first0 + n0;
    const bool c0 = holds_candidates(caps, 2 * t, n0, first0), c1 = holds_candidates(caps, 2 * t + 1, n1, first1);
    const unsigned o0 = c0 ? 0u : n0, o1 = c1 ? 0u : n1;
    const unsigned below = block_exclusive_scan<1024 / kWave>(o0 + o1, wave_tot, total);
    mag->others_below[2 * t] = below;
    mag->others_below[2 * t + 1] = below + o0;
    if (t == 0) mag->candidates = (unsigned)n - total;
    leave_flags(c0, c1, mag->flag);
}

// Exclusive scan of one digit's counters over the tiles; workgroup d has digit d.
template <bool FIRST>
__global__ void __launch_bounds__(kSortThreads) scan_digit(unsigned* __restrict__ hist, long n, MagTable* __restrict__ mag) {
    __shared__ __align__(16) unsigned wave_tot[kSortWaves];
    const PassShape shape = pass_shape<FIRST>(n, mag);
    const long tiles = shape.tiles;
    unsigned* c = hist + (long)blockIdx.x * shape.row;
    unsigned carry = 0;
    // 16 consecutive counters per thread, in 16-byte loads (16384 tiles: 34 us counter by counter, 14 so), or one
    const bool few = tiles <= kSortThreads;
    for (long base = 0; base < tiles; base += kScanChunk) {     // uniform trip count
        const long e0 = base + (few ? (long)threadIdx.x : (long)threadIdx.x * 16);
        unsigned v[16], s = 0;
        if (!few && e0 + 16 <= tiles) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint4 r = reinterpret_cast<const uint4*>(c + e0)[q];
                v[4 * q] = r.x; v[4 * q + 1] = r.y; v[4 * q + 2] = r.z; v[4 * q + 3] = r.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = (!few || i == 0) && e0 + i < tiles ? c[e0 + i] : 0u;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) s += v[i];
        unsigned total;
        unsigned run = carry + block_exclusive_scan<kSortWaves>(s, wave_tot, total);
#pragma unroll
        for (int i = 0; i < 16; ++i) { const unsigned t = v[i]; v[i] = run; run += t; }
        if (!few && e0 + 16 <= tiles) {
#pragma unroll
            for (int q = 0; q < 4; ++q) reinterpret_cast<uint4*>(c + e0)[q] = make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((!few || i == 0) && e0 + i < tiles) c[e0 + i] = v[i];
        }
        carry += total;
    }
    if (threadIdx.x == 0) mag->digit_total[blockIdx.x] = carry;
}

// LDS of one tile's pass: TILE elements in the hands of WAVES wavefronts.
template <int WAVES, int TILE, class Payload>
struct TileSort {
    unsigned skey[TILE];
    Payload sval[TILE];
    unsigned cnt[WAVES][kRadix];             // per wave: running count, then the wave's offset in the digit's run
    unsigned tile_excl[kRadix];              // first tile-local position of a digit
    alignas(16) unsigned wave_tot[WAVES];
};

// One stable counting-sort step of a tile on the digit at `shift`: with `items` elements per thread, element i of
// lane l of wave w is the tile's element (w * items + i) * 64 + l (`valid_count` of them exist); on return sh.skey / sh.sval
// hold the tile ordered by digit, equal digits in their old order, and sh.tile_excl the start of
// every digit's run.  All threads of the workgroup call it; it ends with a barrier.
template <int WAVES, int TILE, class Payload>
__device__ __forceinline__ void tile_sort_step(TileSort<WAVES, TILE, Payload>& sh, const unsigned (&key)[kSortItems],
                                               const Payload (&val)[kSortItems], int items, int valid_count, int shift) {
    static_assert(WAVES * kWave >= kRadix && WAVES * kWave * kSortItems == TILE, "a thread per digit");
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    for (int d = lane; d < kRadix; d += kWave) sh.cnt[wave][d] = 0;
    __builtin_amdgcn_wave_barrier();
    const int first = wave * (items * kWave) + lane;
    unsigned short rank[kSortItems];
    // Stable rank of every element among those of its wave with the same digit: the elements of a
    // wave are ordered by (i, lane), which is their order in memory.  Eight ballots find the lanes
    // that share a digit; the lowest of them advances the wave's counter.  (By halves of the ballots and a sign-extended bit this is
    // four instructions per bit; selects of 64-bit words were seven: 8.4 M elements all capped 335 -> 315 us.)
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        if (i < items) {                                       // (uniform)
            const bool valid = first + i * kWave < valid_count;
            const unsigned d = (key[i] >> shift) & (kRadix - 1);
            const unsigned long long there = __ballot(valid);
            unsigned same_lo = (unsigned)there, same_hi = (unsigned)(there >> 32);
#pragma unroll
            for (int b = 0; b < 8; ++b) {                          // (halves and a mask: two three-operand instructions per bit)
                const unsigned bit = (unsigned)((int)(key[i] << (31 - shift - b)) >> 31);
                const unsigned long long bal = __ballot(bit != 0u);
                same_lo &= ~((unsigned)bal ^ bit);
                same_hi &= ~((unsigned)(bal >> 32) ^ bit);
            }
            const unsigned below = __builtin_amdgcn_mbcnt_hi(same_hi, __builtin_amdgcn_mbcnt_lo(same_lo, 0u));
            const unsigned prev = valid ? sh.cnt[wave][d] : 0u;
            const unsigned r = prev + below;
            __builtin_amdgcn_wave_barrier();                       // all reads of this round before its writes
            if (valid && below == 0) sh.cnt[wave][d] = prev + (unsigned)(__popc(same_lo) + __popc(same_hi));
            rank[i] = (unsigned short)r;
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    {   // per digit: offsets of the waves inside the digit's run, the run's place in the tile
        const int d = threadIdx.x;
        const bool has = WAVES * kWave == kRadix || d < kRadix;
        unsigned run = 0;
        if (has) {
#pragma unroll
            for (int w = 0; w < WAVES; ++w) { const unsigned t = sh.cnt[w][d]; sh.cnt[w][d] = run; run += t; }
        }
        unsigned total;
        const unsigned before = block_exclusive_scan<WAVES>(run, sh.wave_tot, total);
        if (has) sh.tile_excl[d] = before;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        if (i < items && first + i * kWave < valid_count) {
            const unsigned d = (key[i] >> shift) & (kRadix - 1);
            const unsigned pos = sh.tile_excl[d] + sh.cnt[wave][d] + rank[i];
            if (pos < (unsigned)TILE) { sh.skey[pos] = key[i]; sh.sval[pos] = val[i]; }
        }
    }
    __syncthreads();
}

// The element of 0-based rank `rank0` with magnitude bits k and payload v: write its capped value
// if it exceeds its cap (out already holds delta).  Most of the work is two
// binary64 divisions; an estimate with reciprocals (error far below the margin used) first sorts
// out the elements that are clearly under their cap.
__device__ __forceinline__ void cap_and_store(const CapTable& tab, unsigned rank0, unsigned k, unsigned v, long n,
                                              float* out) {
    const float a = __uint_as_float(k);
    const unsigned idx = v & 0x7fffffffu;
    if ((long)idx >= n) return;                                // cannot happen
    const double kk = (double)rank0 + 0.5;
    const double re = kk * tab.percent_per_rank;
    const CapSeg se = tab.seg[segment_of(re)];
    const double ce = fmax(se.head, se.c0 + se.dc * ((re - se.p0) * se.inv_dp));
    const bool near_knot = fabs(re - se.p0) < 1e-6 || fabs(re - (se.p0 + se.dp)) < 1e-6;
    if (!near_knot && (double)a < ce - (fabs(se.dc) + ce) * 1e-9) return;
    const double r = rank_percent((double)rank0 + 1.0, tab.n);
    const CapSeg s = tab.seg[segment_of(r)];
    const double cap = fmax(s.head, cap_in_segment(s, r));
    if ((double)a > cap) out[idx] = __uint_as_float(__float_as_uint(down32(cap)) | (v & 0x80000000u));       // NaN compares false and stays
}

// Scatter pass.  `hist` holds the scanned counters: hist[d * row + tile] elements with digit d lie in the tiles before.
// FEW: it holds the counters themselves, of at most kFewTiles tiles, and every workgroup adds up a digit's row per thread; a launch
// takes the host 3.6 us, and tensors of that size wait for it.
// The first pass sorts the tile's candidates: as the counting pass left them, or closed up here, in LDS and in order.
template <bool FIRST, bool LAST, bool FEW>
__global__ void __launch_bounds__(kSortThreads, LAST ? 3 : 4) radix_scatter(const float* delta,
                                                              const unsigned* __restrict__ keys_in, const unsigned* __restrict__ vals_in,
                                                              unsigned* __restrict__ keys_out, unsigned* __restrict__ vals_out,
                                                              long total, int shift, const unsigned* __restrict__ hist,
                                                              const MagTable* __restrict__ mag, const CapTable* __restrict__ tab, float* out) {
    __shared__ TileSort<kSortWaves, kSortTile, unsigned> sh;
    __shared__ unsigned dest_off[kRadix];                      // global destination minus tile-local position
    __shared__ CapTable stab;                                  // LAST: the cap table, read per element
    __shared__ double run_cap[LAST ? kRadix : 1];
    __shared__ unsigned flag[FIRST ? kMagBins / 32 : 1];
    const PassShape shape = pass_shape<FIRST>(total, mag);
    const long n = shape.n, tiles = shape.tiles;
    const long tile = tile_of_block((tiles + kXcds - 1) / kXcds);
    if (tile < 0 || tile >= tiles) return;                     // whole workgroup
    if (LAST) {
        static_assert(sizeof(CapTable) % sizeof(double) == 0 && sizeof(CapTable) / sizeof(double) <= kSortThreads, "one double per thread");
        if (threadIdx.x < sizeof(CapTable) / sizeof(double))
            reinterpret_cast<double*>(&stab)[threadIdx.x] = reinterpret_cast<const double*>(tab)[threadIdx.x];
        // visible after the barriers of the sort step
    }
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    unsigned digit_total = 0, digit_before = 0;                // kSortThreads == kRadix
    if (FEW) {
        const uint4* const row = reinterpret_cast<const uint4*>(hist + (long)threadIdx.x * shape.row);
#pragma unroll 4
        for (int q = 0; q < (int)(shape.row / 4); ++q) {
            const uint4 c = row[q];
            const unsigned v[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {                      // (the row's last counters, past the tiles, hold anything)
                digit_total += 4 * q + j < (int)tiles ? v[j] : 0u;
                digit_before += 4 * q + j < (int)tile ? v[j] : 0u;
            }
        }
    } else {
        digit_total = mag->digit_total[threadIdx.x];
        digit_before = hist[(long)threadIdx.x * shape.row + tile];
    }
    int items = FIRST ? kSortItems : shape.items;
    const long tile_base = tile * (items * kSortThreads);
    const long base = tile_base + (long)wave * (items * kWave) + lane;
    const long left = n - tile_base;
    int count = left < items * kSortThreads ? (int)left : items * kSortThreads;

    unsigned key[kSortItems], val[kSortItems];
    if (FIRST) {
        // (requested before it is known whether they are needed: behind that answer they were one more latency for every tile)
        unsigned flags = 0;
        if (threadIdx.x < kMagBins / 32) flags = mag->flag[threadIdx.x];
        const unsigned found = closes_up(mag, n) ? keys_in[tile_base + count - 1] : kNotClosedUp;
        if (found != kNotClosedUp) {
            count = (int)min(found & ~kClosedUp, (unsigned)kMostClosedUp);
            items = (count + kSortThreads - 1) / kSortThreads;
#pragma unroll
            for (int i = 0; i < kSortItems; ++i) {
                const int e = (wave * items + i) * kWave + lane;
                key[i] = 0xffffffffu; val[i] = 0;
                if (i < items && e < count) { key[i] = keys_in[tile_base + e]; val[i] = vals_in[tile_base + e]; }
            }
        } else {
            // every wavefront closes up its quarter of the tile in its quarter of the LDS arrays ...
            const unsigned* src = reinterpret_cast<const unsigned*>(delta) + tile_base;
            const unsigned long long lanes_below = (1ull << lane) - 1ull;
            unsigned at = 0;
#pragma unroll
            for (int i = 0; i < kSortItems; ++i) {
                const int e = wave * (kSortItems * kWave) + i * kWave + lane;
                key[i] = e < count ? src[e] : 0xffffffffu;         // (a NaN: never a candidate)
            }
            if (threadIdx.x < kMagBins / 32) flag[threadIdx.x] = flags;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kSortItems; ++i) {
                const int e = wave * (kSortItems * kWave) + i * kWave + lane;
                const unsigned k = key[i] & 0x7fffffffu, bin = k >> kMagShift;
                const bool c = e < count && ((flag[bin >> 5] >> (bin & 31)) & 1u);
                const unsigned long long b = __ballot(c);
                if (c) {
                    const unsigned pos = wave * (kSortItems * kWave) + at + (unsigned)__popcll(b & lanes_below);
                    sh.skey[pos] = k;
                    sh.sval[pos] = ((unsigned)tile_base + (unsigned)e) | (key[i] & 0x80000000u);
                }
                at += (unsigned)__popcll(b);
            }
            if (lane == 0) sh.wave_tot[wave] = at;
            __syncthreads();
            // ... and the workgroup takes the four pieces one after the other
            const int p1 = (int)sh.wave_tot[0], p2 = p1 + (int)sh.wave_tot[1], p3 = p2 + (int)sh.wave_tot[2];
            count = p3 + (int)sh.wave_tot[3];
            items = (count + kSortThreads - 1) / kSortThreads;
#pragma unroll
            for (int i = 0; i < kSortItems; ++i) {
                const int e = (wave * items + i) * kWave + lane;
                key[i] = 0xffffffffu; val[i] = 0;
                if (i < items && e < count) {
                    const int from = e < p1 ? e : e < p2 ? e - p1 + kSortItems * kWave : e < p3 ? e - p2 + 2 * kSortItems * kWave : e - p3 + 3 * kSortItems * kWave;
                    key[i] = sh.skey[from]; val[i] = sh.sval[from];
                }
            }
            __syncthreads();                                   // (wave_tot and the tile are written again)
        }
    } else {
#pragma unroll
        for (int i = 0; i < kSortItems; ++i) {
            const long e = base + (long)i * kWave;
            key[i] = 0xffffffffu; val[i] = 0;
            if (i < items && e < n) { key[i] = keys_in[e]; val[i] = vals_in[e]; }
        }
    }
    tile_sort_step(sh, key, val, items, count, shift);
    {
        unsigned sum;
        const unsigned first_dest = block_exclusive_scan<kSortWaves>(digit_total, sh.wave_tot, sum) + digit_before;
        dest_off[threadIdx.x] = first_dest - sh.tile_excl[threadIdx.x];
        if (LAST) {
            // Caps do not decrease with the rank: the exact cap of a rank that all elements of this tile with digit d
            // reach or exceed is a lower bound for theirs, and most elements are settled by one comparison with it.
            static_assert(kMagShift >= 16 && kMagShift <= 24, "a digit of the last pass is a run of bins");
            const unsigned low_bin = (unsigned)threadIdx.x << (24 - kMagShift);
            const unsigned rank0 = first_dest + (low_bin < (unsigned)kMagBins ? mag->others_below[low_bin] : 0u);
            const double r = rank_percent((double)rank0 + 1.0, stab.n);
            const CapSeg s = stab.seg[segment_of(r)];
            run_cap[threadIdx.x] = (long)rank0 < total ? fmax(s.head, cap_in_segment(s, r)) : 0.0;
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < count; j += kSortThreads) {
        const unsigned k = sh.skey[j], v = sh.sval[j];
        const unsigned d = (k >> shift) & (kRadix - 1);
        const unsigned dest = dest_off[d] + (unsigned)j;
        if ((long)dest >= total) continue;                     // cannot happen with consistent counters
        if (!LAST) {
            keys_out[dest] = k;
            vals_out[dest] = v;
        } else {
            if ((double)__uint_as_float(k) <= run_cap[d]) continue;
            const unsigned rank0 = dest + (n == total ? 0u : mag->others_below[min(k >> kMagShift, (unsigned)kMagBins - 1u)]);
            cap_and_store(stab, rank0, k, v, total, out);
        }
    }
}

// Tensors of at most 16384 elements: all of it in LDS by one workgroup, cap table and candidates included.  Nothing is busy
// here: it is a chain of some 30 barriers and LDS round trips, about 2.5 us per pass of few candidates, and 12 where 16384
// are ranked (the payload is 16 bits, so that they fit).  Four wavefronts that ranked every element of up to 4096, and fifteen launches above, took, in us, the usual
// heavy tail / nothing capped / all capped: 1000 elements 31.3 / 30.8 / 32.8, now 20.5 / 6.8 / 21.7; 4096 40.2 / 39.7 / 47.8, now 21.2 / 7.4 / 35.0;
// 16384 59.9 / 42.0 / 115, now 23.7 / 9.4 / 87.  (16385, by launches: 41.4 / 28.9 / 93.)
constexpr int kOneWaves = 16, kOneThreads = kOneWaves * kWave, kOneTile = kOneThreads * kSortItems;
__global__ void __launch_bounds__(kOneThreads) project_one_tile(const float* delta, const float* __restrict__ thr, double alpha,
                                                                int n, float* out) {
    static_assert(kMagBins == 2 * kOneThreads, "two bins per thread");
    constexpr int kCopies = 4;                                 // of the magnitudes' histogram, in the place of the keys
    __shared__ TileSort<kOneWaves, kOneTile, unsigned short> sh;
    static_assert(kCopies * kMagBins <= kOneTile && kOneTile <= 0x8000, "room for the histogram; index and sign in 16 bits");
    __shared__ unsigned others_below[kMagBins], flag[kMagBins / 32];
    __shared__ CapTable tab;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const unsigned long long lanes_below = (1ull << lane) - 1ull;
    int items = (n + kOneThreads - 1) / kOneThreads;           // (uniform)
    unsigned key[kSortItems];
    unsigned short val[kSortItems];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const int e = (wave * items + i) * kWave + lane;
        key[i] = i < items && e < n ? __float_as_uint(delta[e]) : 0xffffffffu;
    }
    for (int b = tid; b < kCopies * kMagBins; b += kOneThreads) sh.skey[b] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const int e = (wave * items + i) * kWave + lane;
        if (i < items && e < n) {
            if (out != delta) out[e] = __uint_as_float(key[i]);
            atomicAdd(&sh.skey[((key[i] & 0x7fffffffu) >> kMagShift) * kCopies + (lane & (kCopies - 1))], 1u);
        }
    }
    build_cap_table(thr, alpha, n, &tab);                      // ends with a barrier
    unsigned n0 = 0, n1 = 0, total;
#pragma unroll
    for (int c = 0; c < kCopies; ++c) { n0 += sh.skey[2 * tid * kCopies + c]; n1 += sh.skey[(2 * tid + 1) * kCopies + c]; }
    const unsigned first0 = block_exclusive_scan<kOneWaves>(n0 + n1, sh.wave_tot, total), first1 = first0 + n0;
    const bool c0 = holds_candidates(tab, 2 * tid, n0, first0), c1 = holds_candidates(tab, 2 * tid + 1, n1, first1);
    leave_flags(c0, c1, flag);
    const unsigned o0 = c0 ? 0u : n0, o1 = c1 ? 0u : n1;
    const unsigned below = block_exclusive_scan<kOneWaves>(o0 + o1, sh.wave_tot, total);
    others_below[2 * tid] = below;
    others_below[2 * tid + 1] = below + o0;
    __syncthreads();
    const int count = n - (int)total;
    if (count == 0) return;                                    // whole workgroup
    // the candidates closed up, in order
    unsigned mine = 0, in_wave = 0;                            // mine: a bit per key
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const int e = (wave * items + i) * kWave + lane;
        const unsigned bin = (key[i] & 0x7fffffffu) >> kMagShift;
        const bool c = i < items && e < n && ((flag[bin >> 5] >> (bin & 31)) & 1u);
        mine |= (unsigned)c << i;
        in_wave += (unsigned)__popcll(__ballot(c));
    }
    if (lane == 0) sh.wave_tot[wave] = in_wave;
    __syncthreads();
    unsigned at = 0;
    for (int w = 0; w < wave; ++w) at += sh.wave_tot[w];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const bool c = (mine >> i) & 1u;
        const unsigned long long b = __ballot(c);
        if (c) {
            const unsigned to = at + (unsigned)__popcll(b & lanes_below);
            sh.skey[to] = key[i] & 0x7fffffffu;
            sh.sval[to] = (unsigned short)(((wave * items + i) * kWave + lane) | (key[i] >> 31 << 15));
        }
        at += (unsigned)__popcll(b);
    }
    __syncthreads();
    items = (count + kOneThreads - 1) / kOneThreads;
    const int first = wave * (items * kWave) + lane;
#pragma unroll 1
    for (int pass = 0; pass < 4; ++pass) {
#pragma unroll
        for (int i = 0; i < kSortItems; ++i) {
            const int e = first + i * kWave;
            key[i] = 0xffffffffu; val[i] = 0;
            if (i < items && e < count) { key[i] = sh.skey[e]; val[i] = sh.sval[e]; }
        }
        // (what is read here is written again behind two barriers of the step)
        tile_sort_step(sh, key, val, items, count, 8 * pass);
    }
    for (int j = tid; j < count; j += kOneThreads) {
        const unsigned k = sh.skey[j], v = sh.sval[j];
        const unsigned rank0 = (unsigned)j + (count == n ? 0u : others_below[min(k >> kMagShift, (unsigned)kMagBins - 1u)]);
        cap_and_store(tab, rank0, k, (v & 0x7fffu) | (v >> 15 << 31), n, out);
    }
}

struct ProjectWorkspace {
    CapTable* tab;
    MagTable* mag;
    unsigned *hist, *keys_a, *vals_a, *keys_b, *vals_b;
    long tiles;
};

// The twelve launches behind the candidates, eight where the tiles are few.
template <bool FEW>
inline void sort_and_cap(const float* delta, long n, int vec_in, float* out, const ProjectWorkspace& w, hipStream_t st) {
    const long per_xcd = (w.tiles + kXcds - 1) / kXcds;
    const dim3 grid((unsigned)(per_xcd * kXcds)), blk(kSortThreads), digits(kRadix);
    unsigned* kin = nullptr; unsigned* vin = nullptr;
    unsigned* kout = w.keys_a; unsigned* vout = w.vals_a;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 8 * pass;
        if (pass == 0) {
            hipLaunchKernelGGL((radix_count<true>), grid, blk, 0, st, delta, kin, n, shift, (int)(vec_in && aligned(out, 16)), w.mag,
                               w.hist, out != delta ? reinterpret_cast<unsigned*>(out) : nullptr, w.keys_b, w.vals_b);
            if (!FEW) hipLaunchKernelGGL((scan_digit<true>), digits, blk, 0, st, w.hist, n, w.mag);
            hipLaunchKernelGGL((radix_scatter<true, false, FEW>), grid, blk, 0, st, delta, w.keys_b, w.vals_b, kout, vout, n, shift, w.hist, w.mag, w.tab, out);
        } else {
            hipLaunchKernelGGL((radix_count<false>), grid, blk, 0, st, delta, kin, n, shift, 1, w.mag, w.hist, nullptr, nullptr, nullptr);
            if (!FEW) hipLaunchKernelGGL((scan_digit<false>), digits, blk, 0, st, w.hist, n, w.mag);
            if (pass < 3) hipLaunchKernelGGL((radix_scatter<false, false, FEW>), grid, blk, 0, st, delta, kin, vin, kout, vout, n, shift, w.hist, w.mag, w.tab, out);
            else          hipLaunchKernelGGL((radix_scatter<false, true, FEW>), grid, blk, 0, st, delta, kin, vin, kout, vout, n, shift, w.hist, w.mag, w.tab, out);
        }
        kin = kout; vin = vout;
        kout = kin == w.keys_a ? w.keys_b : w.keys_a;
        vout = vin == w.vals_a ? w.vals_b : w.vals_a;
    }
}

inline size_t round256(size_t b) { return (b + 255) / 256 * 256; }

inline size_t carve_project(long n, char* ws, ProjectWorkspace* w) {
    const long tiles = (n + kSortTile - 1) / kSortTile;
    const long counters = counter_row(tiles) * kRadix;
    size_t off = 0;
    auto take = [&](size_t bytes) { char* p = ws ? ws + off : nullptr; off += round256(bytes); return p; };
    char* tab = take(sizeof(CapTable));
    char* mag = take(sizeof(MagTable));
    char* hist = take((size_t)counters * 4);
    char* ka = take((size_t)n * 4); char* va = take((size_t)n * 4);
    char* kb = take((size_t)n * 4); char* vb = take((size_t)n * 4);
    if (w) {
        w->tab = (CapTable*)tab; w->mag = (MagTable*)mag; w->hist = (unsigned*)hist;
        w->keys_a = (unsigned*)ka; w->vals_a = (unsigned*)va; w->keys_b = (unsigned*)kb; w->vals_b = (unsigned*)vb;
        w->tiles = tiles;
    }
    return off;
}

}  // namespace tao

extern "C" {

int tao_project_clip(const float* delta, const float* tau, double alpha, float* out, long n, void* stream) {
    using namespace tao;
    if (n < 0 || !(alpha >= 0.0) || !std::isfinite(alpha)) return TAO_ERR_SHAPE;
    if (n == 0) return TAO_OK;
    if (!delta || !tau || !out) return TAO_ERR_NULL;
    if (!aligned(delta, 4) || !aligned(tau, 4) || !aligned(out, 4)) return TAO_ERR_ALIGN;
    const int vec_ok = aligned(delta, 16) && aligned(tau, 16) && aligned(out, 16);
    long blocks = (n + 1023) / 1024;
    if (blocks > 256L * 32) blocks = 256L * 32;
    hipLaunchKernelGGL(project_clip_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       delta, tau, alpha, out, n, vec_ok);
    return launch_status();
}

size_t tao_project_workspace_bytes(long n) {
    if (n <= 0 || n >= (1L << 31)) return 0;
    return tao::carve_project(n, nullptr, nullptr);
}

int tao_project_empirical(const float* delta, const float* thr_abs, double alpha, float* out, long n,
                          void* ws, size_t ws_bytes, void* stream) {
    using namespace tao;
    if (n < 0 || n >= (1L << 31) || !(alpha >= 0.0) || !std::isfinite(alpha)) return TAO_ERR_SHAPE;
    if (n == 0) return TAO_OK;
    if (!delta || !thr_abs || !out) return TAO_ERR_NULL;
    if (!aligned(delta, 4) || !aligned(thr_abs, 4) || !aligned(out, 4)) return TAO_ERR_ALIGN;
    if (!ws || !aligned(ws, 256) || ws_bytes < tao_project_workspace_bytes(n)) return TAO_ERR_WORKSPACE;
    if (n <= kOneTile) {
        hipLaunchKernelGGL(project_one_tile, dim3(1), dim3(kOneThreads), 0, (hipStream_t)stream, delta, thr_abs, alpha,
                           (int)n, out);
        return launch_status();
    }
    ProjectWorkspace w;
    carve_project(n, (char*)ws, &w);
    hipStream_t st = (hipStream_t)stream;
    const int vec_in = aligned(delta, 16);
    const long want = (n + 8191) / 8192;                        // two vectors per thread before another workgroup is worth it
    const unsigned blocks = (unsigned)(want < 256 ? want : 256);
    if (w.tiles <= kFewTiles) {
        // (the workgroups' histograms lie in the place of the first sorted keys: 8192 bytes of at least 4 * 8192)
        static_assert(kMagBins <= 8192 && kFewTiles * kSortTile <= 256 * 8192, "a histogram in the place of its elements' keys");
        hipLaunchKernelGGL((magnitude_bins<true>), dim3(blocks), dim3(1024), 0, st, delta, n, vec_in, w.mag, w.keys_a);
        hipLaunchKernelGGL((find_candidates<true>), dim3(1), dim3(1024), 0, st, thr_abs, alpha, n, w.tab, w.mag, w.keys_a, (int)blocks);
        sort_and_cap<true>(delta, n, vec_in, out, w, st);
    } else {
        hipLaunchKernelGGL(cap_table_kernel, dim3(1), dim3(kWave), 0, st, thr_abs, alpha, n, w.tab, w.mag);
        hipLaunchKernelGGL((magnitude_bins<false>), dim3(blocks), dim3(1024), 0, st, delta, n, vec_in, w.mag, nullptr);
        hipLaunchKernelGGL((find_candidates<false>), dim3(1), dim3(1024), 0, st, thr_abs, alpha, n, w.tab, w.mag, nullptr, 0);
        sort_and_cap<false>(delta, n, vec_in, out, w, st);
    }
    return launch_status();
}

}  // extern "C"
