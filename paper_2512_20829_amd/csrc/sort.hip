// Device-wide exclusive scan and stable LSD radix sort of (u32 key, u32 value)
// pairs, written for 64-wide wavefronts.  Both are deterministic: ranks inside
// a block come from wavefront ballots in item order, never from atomics.
#include <type_traits>

#include "internal.hpp"

namespace flp {

// ------------------------------------------------------------------ scan
constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kScanBlock = kScanThreads * kScanItems;   // 1024 elements per block

__device__ inline uint32_t wave_incl_scan(uint32_t v, int lane)
{
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        uint32_t t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive scan of one 1024-element block in place; writes the block total.
__global__ __launch_bounds__(kScanThreads) void k_scan_block(uint32_t* data, int64_t n, uint32_t* sums)
{
    __shared__ uint32_t wsum[kScanThreads / kWave];
    int t = threadIdx.x, lane = t % kWave, wv = t / kWave;
    int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)t * kScanItems;
    uint32_t v[kScanItems];
    uint32_t tot = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? data[base + k] : 0u;
        tot += v[k];
    }
    uint32_t inc = wave_incl_scan(tot, lane);
    if (lane == kWave - 1) wsum[wv] = inc;
    __syncthreads();
    uint32_t woff = 0;
    for (int w = 0; w < wv; ++w) woff += wsum[w];
    uint32_t run = woff + inc - tot;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) data[base + k] = run;
        run += v[k];
    }
    if (t == kScanThreads - 1) sums[blockIdx.x] = woff + inc;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_add(uint32_t* data, int64_t n, const uint32_t* offs)
{
    int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems;
    uint32_t o = offs[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < n) data[base + k] += o;
}

int64_t scan_tmp_words(int64_t n)
{
    int64_t words = 0;
    while (n > 1) {
        n = (n + kScanBlock - 1) / kScanBlock;
        words += n + 1;
    }
    return words + 1;
}

hipError_t launch_exclusive_scan_u32(uint32_t* data, int64_t n, uint32_t* tmp, int64_t tmp_words,
                                     hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    if (nb + 1 > tmp_words) return hipErrorInvalidValue;
    FLA_LAUNCH(k_scan_block, dim3((unsigned)nb), dim3(kScanThreads), 0, s, data, n, tmp);
    if (nb > 1) {
        hipError_t e = launch_exclusive_scan_u32(tmp, nb, tmp + nb + 1, tmp_words - nb - 1, s);
        if (e != hipSuccess) return e;
        FLA_LAUNCH(k_scan_add, dim3((unsigned)nb), dim3(kScanThreads), 0, s, data, n, tmp);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ radix sort
constexpr int kSortThreads = 256;
constexpr int kDigits = 256;
// Items per thread of a block.  Up to kSortFewItems keys the blocks are a
// quarter as long where the caller has room for their histograms, so that a
// small sort has blocks enough for the compute units: with 30 blocks of 4096
// every round of 256 waits for the one before, 16 times (120k keys: a scatter
// 16 -> 6 us).
constexpr int kSortItemsMany = 16, kSortItemsFew = 4;
constexpr int64_t kSortFewItems = 1 << 18;

static int64_t sort_blocks(int64_t n, int items)
{
    const int64_t tile = (int64_t)kSortThreads * items;
    return (n + tile - 1) / tile;
}

int64_t radix_hist_words(int64_t n) { return sort_blocks(n, kSortItemsMany) * kDigits; }

// Per-block digit histogram, stored digit-major: hist[d * nblocks + b].
template <int kSortItems>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint32_t* keys, int64_t n, int shift,
                                                           uint32_t* hist, int nblocks)
{
    __shared__ uint32_t cnt[kDigits];
    int t = threadIdx.x;
    cnt[t] = 0;
    __syncthreads();
    int64_t base = (int64_t)blockIdx.x * kSortThreads * kSortItems;
    for (int k = 0; k < kSortItems; ++k) {
        int64_t i = base + (int64_t)k * kSortThreads + t;
        if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & 0xFF], 1u);
    }
    __syncthreads();
    hist[(int64_t)t * nblocks + blockIdx.x] = cnt[t];
}

// Stable scatter.  Items are visited in rounds of 256 consecutive items;
// inside a wave the rank among equal digits comes from 8 ballots, across
// the 4 waves of a round from a prefix over per-wave counts.
template <int kSortItems>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(const uint32_t* keys, const uint32_t* vals,
                                                              int64_t n, int shift, const uint32_t* offs,
                                                              int nblocks, uint32_t* keys_out,
                                                              uint32_t* vals_out)
{
    constexpr int NW = kSortThreads / kWave;
    __shared__ uint32_t run[kDigits];
    __shared__ uint32_t wcnt[NW][kDigits];
    int t = threadIdx.x, lane = t % kWave, wv = t / kWave;
    run[t] = offs[(int64_t)t * nblocks + blockIdx.x];
    int64_t base = (int64_t)blockIdx.x * kSortThreads * kSortItems;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int k = 0; k < kSortItems; ++k) {
        for (int w = 0; w < NW; ++w) wcnt[w][t] = 0;
        __syncthreads();
        int64_t i = base + (int64_t)k * kSortThreads + t;
        bool valid = i < n;
        uint32_t key = valid ? keys[i] : 0u;
        uint32_t val = valid ? vals[i] : 0u;
        uint32_t d = (key >> shift) & 0xFF;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            uint64_t bal = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? bal : ~bal;
        }
        uint32_t rank = (uint32_t)__popcll(peers & lt);
        if (valid && rank == 0) wcnt[wv][d] = (uint32_t)__popcll(peers);
        __syncthreads();
        if (valid) {
            uint32_t pos = run[d] + rank;
            for (int w = 0; w < wv; ++w) pos += wcnt[w][d];
            keys_out[pos] = key;
            vals_out[pos] = val;
        }
        __syncthreads();
        uint32_t add = 0;
        for (int w = 0; w < NW; ++w) add += wcnt[w][t];
        run[t] += add;
        __syncthreads();
    }
}

hipError_t radix_sort_pairs(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                            int64_t n, int key_bits, uint32_t* hist, int64_t hist_words,
                            uint32_t* scan_tmp, int64_t scan_tmp_words_, hipStream_t s,
                            bool* result_in_alt, uint32_t* spare, int64_t spare_words)
{
    *result_in_alt = false;
    if (n <= 1) return hipSuccess;
    bool few = false;
    if (n <= kSortFewItems) {
        const int64_t hw = sort_blocks(n, kSortItemsFew) * kDigits, sw = scan_tmp_words(hw);
        few = hw + sw <= spare_words;
        if (few) {
            hist = spare;
            hist_words = hw;
            scan_tmp = spare + hw;
            scan_tmp_words_ = sw;
        }
    }
    const int nblocks = (int)sort_blocks(n, few ? kSortItemsFew : kSortItemsMany);
    if ((int64_t)nblocks * kDigits > hist_words) return hipErrorInvalidValue;
    uint32_t *ka = keys, *va = vals, *kb = keys_alt, *vb = vals_alt;
    auto pass = [&](auto items, int shift) -> hipError_t {
        constexpr int K = decltype(items)::value;
        FLA_LAUNCH((k_radix_hist<K>), dim3(nblocks), dim3(kSortThreads), 0, s, ka, n, shift, hist, nblocks);
        hipError_t e = launch_exclusive_scan_u32(hist, (int64_t)nblocks * kDigits, scan_tmp, scan_tmp_words_, s);
        if (e != hipSuccess) return e;
        FLA_LAUNCH((k_radix_scatter<K>), dim3(nblocks), dim3(kSortThreads), 0, s, ka, va, n, shift, hist, nblocks, kb,
                   vb);
        return hipSuccess;
    };
    for (int shift = 0; shift < key_bits; shift += 8) {
        const hipError_t e = few ? pass(std::integral_constant<int, kSortItemsFew>{}, shift)
                                 : pass(std::integral_constant<int, kSortItemsMany>{}, shift);
        if (e != hipSuccess) return e;
        uint32_t* tk = ka; ka = kb; kb = tk;
        uint32_t* tv = va; va = vb; vb = tv;
        *result_in_alt = !*result_in_alt;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ small sort
// Up to kSortSmall keys in one workgroup: the stable sort, the bucket bounds
// (first position of every bucket b in [0, nb]) and the largest non-empty class
// in one launch instead of the six or more of the passes above and two: 4096
// keys of 9 bits take 10 us, in their own launches they took 49.  Bound by the
// chain of its steps: one workgroup, two passes.  Named for the scatter that it
// does in LDS and the bounds that it writes.
// Each wave keeps 64 K consecutive items in order; a pass ranks them by ballots
// and a running count per wave and digit, scans the counts digit-major and
// moves the items in LDS.
constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / kWave;
constexpr int kSmallBuckets = 1 << 14;
template <int K>
__global__ __launch_bounds__(kSmallThreads) void k_radix_scatter_bounds(uint32_t* keys, uint32_t* vals, int n, int bits, int db,
                                                            uint32_t nb, int per_class, uint32_t* bstart,
                                                            unsigned long long* max_class)
{
    constexpr int N = kSmallThreads * K;
    __shared__ uint32_t sk[N], sv[N];
    __shared__ uint32_t cnt[kDigits * kSmallWaves];
    __shared__ uint32_t wsum[kSmallWaves];
    const int t = threadIdx.x, lane = t % kWave, wv = t / kWave;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t key[K], val[K], pos[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = wv * kWave * K + k * kWave + lane;
        key[k] = i < n ? keys[i] : 0u;
        val[k] = i < n ? vals[i] : 0u;
    }
    const int nc = kSmallWaves << db;      // counts: digit-major, 16 waves each
    for (int shift = 0; shift < bits; shift += db) {
        for (int i = t; i < nc; i += kSmallThreads) cnt[i] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = wv * kWave * K + k * kWave + lane;
            const bool valid = i < n;
            const uint32_t d = (key[k] >> shift) & ((1u << db) - 1u);
            uint64_t peers = __ballot(valid);
            for (int b = 0; b < db; ++b) {
                const uint64_t bal = __ballot((d >> b) & 1u);
                peers &= ((d >> b) & 1u) ? bal : ~bal;
            }
            const uint32_t rank = (uint32_t)__popcll(peers & lt);
            const uint32_t before = cnt[d * kSmallWaves + wv];
            pos[k] = before + rank;
            wave_sync();
            if (valid && rank == 0) cnt[d * kSmallWaves + wv] = before + (uint32_t)__popcll(peers);
            wave_sync();
        }
        __syncthreads();
        // exclusive scan of the counts, 4 a thread
        uint32_t c[4], tot = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = 4 * t + j < nc ? cnt[4 * t + j] : 0u;
            tot += c[j];
        }
        const uint32_t inc = wave_incl_scan(tot, lane);
        if (lane == kWave - 1) wsum[wv] = inc;
        __syncthreads();
        uint32_t run = inc - tot;
        for (int w = 0; w < wv; ++w) run += wsum[w];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (4 * t + j < nc) cnt[4 * t + j] = run;
            run += c[j];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = wv * kWave * K + k * kWave + lane;
            if (i < n) {
                const uint32_t d = (key[k] >> shift) & ((1u << db) - 1u);
                const uint32_t at = cnt[d * kSmallWaves + wv] + pos[k];
                sk[at] = key[k];
                sv[at] = val[k];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = wv * kWave * K + k * kWave + lane;
            key[k] = i < n ? sk[i] : 0u;
            val[k] = i < n ? sv[i] : 0u;
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = wv * kWave * K + k * kWave + lane;
        if (i < n) {
            keys[i] = key[k];
            vals[i] = val[k];
            sk[i] = key[k];                // also where no pass ran
        }
    }
    __syncthreads();
    auto first_at = [&](uint32_t b) {
        int lo = 0, hi = n;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sk[mid] < b)
                lo = mid + 1;
            else
                hi = mid;
        }
        return (uint32_t)lo;
    };
    for (uint32_t b = t; b <= nb; b += kSmallThreads) bstart[b] = first_at(b);
    if (t == 0) {
        const uint32_t live = first_at(nb);    // keys past the buckets have no support
        *max_class = live ? sk[live - 1] / (uint32_t)per_class : 0u;
    }
}

// Keys that the small sort takes: what one workgroup holds in LDS, and buckets
// few enough for its bounds.
bool sort_is_small(int64_t n, uint32_t nb)
{
    return n >= 1 && n <= 8 * kSmallThreads && nb <= (uint32_t)kSmallBuckets;
}

hipError_t launch_sort_small(uint32_t* keys, uint32_t* vals, int64_t n, int key_bits, uint32_t nb, int per_class,
                             uint32_t* bstart, unsigned long long* max_class, hipStream_t s)
{
    const int passes = (key_bits + 7) / 8, db = passes > 0 ? (key_bits + passes - 1) / passes : 1;
    auto run = [&](auto items) {
        constexpr int K = decltype(items)::value;
        FLA_LAUNCH((k_radix_scatter_bounds<K>), dim3(1), dim3(kSmallThreads), 0, s, keys, vals, (int)n, key_bits, db, nb,
                   per_class, bstart, max_class);
    };
    if (n <= kSmallThreads)
        run(std::integral_constant<int, 1>{});
    else if (n <= 4 * kSmallThreads)
        run(std::integral_constant<int, 4>{});
    else
        run(std::integral_constant<int, 8>{});
    return hipGetLastError();
}

}  // namespace flp
