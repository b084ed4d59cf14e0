// Stable sort of (key, uint32 value) pairs by a range of key bits.
//
// Up to 1024 pairs, and up to kMergeMost pairs where the radix sort would take
// kMergePasses passes: tiles of 1024 sorted by one workgroup each, then merges
// of up to eight sorted runs, in which every pair finds its place by binary
// searches in the other runs.  Bound by launches and latency: at 2*10^4 pairs
// of 63-bit keys three launches take 43 us where the radix sort's 24 take 87;
// at 24 bits its nine take 39 us against 41, and at 1000 pairs 34 against 14.
//
// Else: LSD radix sort, 8-bit digits.  One pass = three launches:
//   hist    : per tile of keys, a 256-bin digit histogram (LDS atomics),
//             stored digit-major so that one row holds a digit's tile counts;
//   scan    : one workgroup per digit scans its row of tile counts and leaves
//             the row's total;
//   scatter : per tile, keys are ranked stably inside each wavefront with
//             ballots (8 ballots identify the lanes sharing a digit, the
//             popcount of those below a lane is its rank), the tile is
//             reordered by digit in LDS and written out in digit runs, so
//             consecutive lanes write consecutive addresses.
// At 10^7 keys of 63 bits 1.0 ms -> 0.69 ms (hist 21, scatter 64 us a pass; 240
// MB a pass is 46 us at the rate of a copy), at 10^6 0.24 -> 0.15 ms, against
// tiles of 16 keys per thread at every size, keys and values of a tile in LDS
// at once, and a separate launch for the digit totals.
// Sorting is what the paper names as the decisive construction cost (Section
// 2.6: switching to a vendor sort took construction from 17 s to 0.02 s).
#include <algorithm>

#include "device_util.hpp"
#include "internal.hpp"

namespace ax {
namespace {

constexpr int kSortBlock = 256;
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;
static_assert(kSortBlock == kRadix, "one thread per digit in the per-tile steps");

// Keys per thread of a radix tile.  A tile of 16 per thread writes digit runs
// of 16 keys on average, but few tiles leave compute units idle (256 of them), or
// each alone with its latency.  63 and 24 bits with 4, 8 and 16 per thread, us:
// 600000 keys 146 152 188 and 67 68 81; 786432 157 154 192 and 72 69 83; 2^20 189
// 166 188 and 83 74 85; 1.9*10^6 281 212 218 and 118 91 95; 2*10^6 290 221 220 and
// 122 94 96; 2.05*10^6 316 236 226 and 131 99 97; 2^22 525 394 356 and 203 155 129.
// So 8 from 1.5 tiles of 8 a compute unit on, 16 from 1.94 tiles of 16; the 992
// tiles of 8 below that fit the allocation-free nearest search's workspace of 1
// MiB, which holds 1015.
constexpr int64_t kItems8Least = 3 << 18, kItems16Least = 31 << 16;
inline int sort_items(int64_t n) { return n < kItems8Least ? 4 : (n < kItems16Least ? 8 : 16); }
inline int64_t sort_tiles(int64_t n, int items) { return (n + kSortBlock * items - 1) / (kSortBlock * items); }

template <typename K, int ITEMS>
__global__ __launch_bounds__(kSortBlock) void radix_hist(const K *__restrict__ keys, int64_t n, int shift,
                                                         uint32_t mask, uint32_t *__restrict__ tile_hist,
                                                         int num_tiles)
{
    __shared__ uint32_t h[kRadix];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (kSortBlock * ITEMS);
#pragma unroll 4
    for (int j = 0; j < ITEMS; ++j) {
        int64_t i = base + (int64_t)j * kSortBlock + threadIdx.x;
        if (i < n)
            atomicAdd(&h[(uint32_t)(keys[i] >> shift) & mask], 1u);
    }
    __syncthreads();
    tile_hist[(int64_t)threadIdx.x * num_tiles + blockIdx.x] = h[threadIdx.x];
}

// In place: tile_hist[d][t] <- sum_{t' < t} tile_hist[d][t'], and digit_total[d]
// the row's sum: one workgroup per digit.
__global__ __launch_bounds__(kSortBlock) void radix_scan(uint32_t *__restrict__ tile_hist,
                                                         uint32_t *__restrict__ digit_total, int num_tiles)
{
    __shared__ uint32_t wsum[kSortBlock / kWave];
    const int d = blockIdx.x;
    uint32_t carry = 0;
    uint32_t *row = tile_hist + (int64_t)d * num_tiles;
    constexpr int PER = 4;
    for (int start = 0; start < num_tiles; start += kSortBlock * PER) {
        const int i0 = start + (int)threadIdx.x * PER;
        uint32_t x[PER];
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            x[k] = (i0 + k < num_tiles) ? row[i0 + k] : 0u;
            s += x[k];
        }
        uint32_t chunk = 0;
        uint32_t run = carry + block_exclusive_scan<kSortBlock>(s, wsum, &chunk);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (i0 + k < num_tiles)
                row[i0 + k] = run;
            run += x[k];
        }
        carry += chunk;
    }
    if (threadIdx.x == 0)
        digit_total[d] = carry;
}

// The keys of a tile, then their values, pass through one LDS array, which
// leaves room for twice as many workgroups as one array for each.
template <typename K, int ITEMS>
__global__ __launch_bounds__(kSortBlock) void radix_scatter(const K *__restrict__ keys_in,
                                                            const uint32_t *__restrict__ vals_in,
                                                            K *__restrict__ keys_out, uint32_t *__restrict__ vals_out,
                                                            int64_t n, int shift, uint32_t mask,
                                                            const uint32_t *__restrict__ tile_off,
                                                            const uint32_t *__restrict__ digit_total, int num_tiles)
{
    constexpr int TILE = kSortBlock * ITEMS;
    constexpr int W = kSortBlock / kWave;  // wavefronts per tile
    constexpr int PER_WAVE = TILE / W;     // contiguous keys per wavefront
    constexpr int ROUNDS = PER_WAVE / kWave;
    __shared__ K s_keys[TILE];
    __shared__ uint32_t s_wcnt[W][kRadix];
    __shared__ uint32_t s_dstart[kRadix];
    __shared__ uint32_t s_goff[kRadix];
    __shared__ uint32_t s_wsum[W];
    uint32_t *s_vals = reinterpret_cast<uint32_t *>(s_keys);

    const int lane = lane_id(), w = wave_id();
    for (int i = threadIdx.x; i < W * kRadix; i += kSortBlock)
        (&s_wcnt[0][0])[i] = 0;
    uint32_t all = 0;  // keys of smaller digits + keys of this digit in earlier tiles
    s_goff[threadIdx.x] = tile_off[(int64_t)threadIdx.x * num_tiles + blockIdx.x] +
                          block_exclusive_scan<kSortBlock>(digit_total[threadIdx.x], s_wsum, &all);
    __syncthreads();

    const int64_t tile_base = (int64_t)blockIdx.x * TILE;
    const int64_t wbase = tile_base + (int64_t)w * PER_WAVE;
    const uint64_t lt = lanemask_lt();
    K k[ROUNDS];
    uint32_t v[ROUNDS];
    uint32_t rank[ROUNDS];
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int64_t i = wbase + (int64_t)j * kWave + lane;
        k[j] = i < n ? keys_in[i] : K(0);
        v[j] = i < n ? vals_in[i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int64_t i = wbase + (int64_t)j * kWave + lane;
        const bool valid = i < n;
        const uint32_t d = (uint32_t)(k[j] >> shift) & mask;
        // lanes of this round holding the same digit
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t r = (uint32_t)__popcll(peers & lt);
        uint32_t prior = 0;
        if (valid && r == 0)
            prior = atomicAdd(&s_wcnt[w][d], (uint32_t)__popcll(peers));
        const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
        prior = __shfl(prior, leader, kWave);
        rank[j] = prior + r;
    }
    __syncthreads();
    {
        // per digit: exclusive prefix over wavefronts, then over digits
        const int d = threadIdx.x;
        uint32_t run = 0;
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
            const uint32_t c = s_wcnt[ww][d];
            s_wcnt[ww][d] = run;
            run += c;
        }
        uint32_t tot = 0;
        s_dstart[d] = block_exclusive_scan<kSortBlock>(run, s_wsum, &tot);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int64_t i = wbase + (int64_t)j * kWave + lane;
        const uint32_t d = (uint32_t)(k[j] >> shift) & mask;
        rank[j] += s_dstart[d] + s_wcnt[w][d];  // place in the tile
        if (i < n && rank[j] < (uint32_t)TILE)
            s_keys[rank[j]] = k[j];
    }
    __syncthreads();
    const int64_t left = n - tile_base;
    const int tile_n = left < TILE ? (int)left : TILE;
    uint32_t to[ITEMS];  // where the tile's p-th pair goes
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int p = j * kSortBlock + (int)threadIdx.x;
        to[j] = 0xffffffffu;
        if (p < tile_n) {
            const K key = s_keys[p];
            const uint32_t d = (uint32_t)(key >> shift) & mask;
            to[j] = s_goff[d] + (uint32_t)(p - (int)s_dstart[d]);
            if ((int64_t)to[j] < n)
                keys_out[to[j]] = key;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int64_t i = wbase + (int64_t)j * kWave + lane;
        if (i < n && rank[j] < (uint32_t)TILE)
            s_vals[rank[j]] = v[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int p = j * kSortBlock + (int)threadIdx.x;
        if (p < tile_n && (int64_t)to[j] < n)
            vals_out[to[j]] = s_vals[p];
    }
}

// ---- merge sort of few pairs -----------------------------------------------

constexpr int64_t kMergeMost = 65536;
constexpr int kMergePasses = 5;
constexpr int kMergeTile = 1024;  // one pair per thread
constexpr int kMergeWays = 8;

template <typename K>
__device__ __forceinline__ K shfl_xor_key(K x, int j)
{
    if constexpr (sizeof(K) == 8)
        return ((K)__shfl_xor((uint32_t)(x >> 32), j, kWave) << 32) | __shfl_xor((uint32_t)x, j, kWave);
    else
        return __shfl_xor(x, j, kWave);
}

// Sort each tile by (key bits, place in the tile): a bitonic network over one
// pair per thread, its steps within a wavefront by shuffles and the ten wider
// ones through LDS.
template <typename K>
__global__ __launch_bounds__(kMergeTile) void merge_tiles(K *__restrict__ keys, uint32_t *__restrict__ vals, int n,
                                                          int shift, K mask)
{
    __shared__ K s_key[kMergeTile];
    __shared__ uint16_t s_at[kMergeTile];
    const int t = threadIdx.x, base = blockIdx.x * kMergeTile;
    const bool valid = base + t < n;
    K x = valid ? (K)((keys[base + t] >> shift) & mask) : (K)~(K)0;
    uint32_t at = valid ? t : t + kMergeTile;  // places past the end sort behind every pair
    for (int k = 2; k <= kMergeTile; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            K y;
            uint32_t yat;
            if (j < kWave) {
                y = shfl_xor_key(x, j);
                yat = __shfl_xor(at, j, kWave);
            } else {
                __syncthreads();
                s_key[t] = x;
                s_at[t] = (uint16_t)at;
                __syncthreads();
                y = s_key[t ^ j];
                yat = s_at[t ^ j];
            }
            const bool less = y < x || (y == x && yat < at);  // the partner comes first
            if (less == (((t & j) == 0) == ((t & k) == 0))) {
                x = y;
                at = yat;
            }
        }
    // the whole keys and the values of the pairs now at t (places past the end stay past the end)
    const bool take = at < kMergeTile;
    const K key = take ? keys[base + at] : K(0);
    const uint32_t val = take ? vals[base + at] : 0u;
    __syncthreads();
    if (take && base + t < n) {
        keys[base + t] = key;
        vals[base + t] = val;
    }
}

// Merge groups of kMergeWays sorted runs of `len` pairs (a power of two).  A
// pair's place in the group is its place in its own run, plus the pairs of
// earlier runs not after it and of later runs before it; the searches of the
// other runs advance together.
template <typename K>
__global__ __launch_bounds__(256) void merge_runs(const K *__restrict__ keys, const uint32_t *__restrict__ vals,
                                                  K *__restrict__ keys_out, uint32_t *__restrict__ vals_out, int n,
                                                  int log_len, int shift, K mask)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n)
        return;
    const K key = keys[i];
    const K x = (K)((key >> shift) & mask);
    const int len = 1 << log_len, own = i >> log_len, first = own & ~(kMergeWays - 1);
    int at[kMergeWays];
#pragma unroll
    for (int r = 0; r < kMergeWays; ++r)
        at[r] = 0;
    for (int step = len; step > 0; step >>= 1) {
#pragma unroll
        for (int r = 0; r < kMergeWays; ++r) {
            const int run = first + r;
            // the (at + step)-th pair of the run, if it has one, counts when it comes before x
            const int p = (run << log_len) + at[r] + step - 1;
            if (run != own && at[r] + step <= len && p < n) {
                const K y = (K)((keys[p] >> shift) & mask);
                if (y < x || (run < own && y == x))
                    at[r] += step;
            }
        }
    }
    int to = (first << log_len) + (i - (own << log_len));
#pragma unroll
    for (int r = 0; r < kMergeWays; ++r)
        to += at[r];
    if (to < n) {
        keys_out[to] = key;
        vals_out[to] = vals[i];
    }
}

template <typename K>
hipError_t merge_sort_pairs(K *keys, uint32_t *vals, K *keys_alt, uint32_t *vals_alt, int n, int begin, int end,
                            hipStream_t s, bool *in_alt)
{
    const int bits = end - begin;
    const K mask = bits >= (int)sizeof(K) * 8 ? (K)~(K)0 : (K)(((K)1 << bits) - 1);
    merge_tiles<K><<<(n + kMergeTile - 1) / kMergeTile, kMergeTile, 0, s>>>(keys, vals, n, begin, mask);
    K *kin = keys, *kout = keys_alt;
    uint32_t *vin = vals, *vout = vals_alt;
    for (int log_len = 10; (1 << log_len) < n; log_len += 3) {
        static_assert(kMergeTile == 1 << 10 && kMergeWays == 1 << 3, "run lengths");
        merge_runs<K><<<(n + 255) / 256, 256, 0, s>>>(kin, vin, kout, vout, n, log_len, begin, mask);
        K *tk = kin;
        kin = kout;
        kout = tk;
        uint32_t *tv = vin;
        vin = vout;
        vout = tv;
    }
    *in_alt = kin != keys;
    return hipGetLastError();
}

template <typename K, int ITEMS>
void radix_pass(const K *kin, const uint32_t *vin, K *kout, uint32_t *vout, int64_t n, int shift, uint32_t mask,
                uint32_t *tile_hist, uint32_t *totals, int tiles, hipStream_t s)
{
    radix_hist<K, ITEMS><<<tiles, kSortBlock, 0, s>>>(kin, n, shift, mask, tile_hist, tiles);
    radix_scan<<<kRadix, kSortBlock, 0, s>>>(tile_hist, totals, tiles);
    radix_scatter<K, ITEMS><<<tiles, kSortBlock, 0, s>>>(kin, vin, kout, vout, n, shift, mask, tile_hist, totals,
                                                         tiles);
}

}  // namespace

size_t radix_workspace_bytes(int64_t n)
{
    // enough for any smaller n too: a workspace is reserved for the largest call
    int64_t tiles = sort_tiles(std::min(n, kItems8Least), 4);
    if (n >= kItems8Least)
        tiles = std::max(tiles, sort_tiles(std::min(n, kItems16Least), 8));
    if (n >= kItems16Least)
        tiles = std::max(tiles, sort_tiles(n, 16));
    return (size_t)(tiles * kRadix + 8 * kRadix) * sizeof(uint32_t) + 256;
}

template <typename K>
hipError_t radix_sort_pairs(K *keys, uint32_t *vals, K *keys_alt, uint32_t *vals_alt, int64_t n, int begin, int end,
                            void *workspace, hipStream_t s, bool *in_alt)
{
    *in_alt = false;
    if (n <= 1 || end <= begin)
        return hipSuccess;
    if (n > (int64_t)UINT32_MAX)
        return hipErrorInvalidValue;
    const int passes = (end - begin + kRadixBits - 1) / kRadixBits;
    if (passes > 8)
        return hipErrorInvalidValue;
    if (n <= kMergeTile || (n <= kMergeMost && passes >= kMergePasses))
        return merge_sort_pairs<K>(keys, vals, keys_alt, vals_alt, (int)n, begin, end, s, in_alt);
    const int items = sort_items(n);
    const int tiles = (int)sort_tiles(n, items);
    uint32_t *tile_hist = static_cast<uint32_t *>(workspace);
    uint32_t *totals = tile_hist + (size_t)tiles * kRadix;
    K *kin = keys, *kout = keys_alt;
    uint32_t *vin = vals, *vout = vals_alt;
    for (int p = 0; p < passes; ++p) {
        const int shift = begin + p * kRadixBits;
        const int bits = (end - shift) < kRadixBits ? (end - shift) : kRadixBits;
        const uint32_t mask = (1u << bits) - 1u;
        if (items == 4)
            radix_pass<K, 4>(kin, vin, kout, vout, n, shift, mask, tile_hist, totals + p * kRadix, tiles, s);
        else if (items == 8)
            radix_pass<K, 8>(kin, vin, kout, vout, n, shift, mask, tile_hist, totals + p * kRadix, tiles, s);
        else
            radix_pass<K, 16>(kin, vin, kout, vout, n, shift, mask, tile_hist, totals + p * kRadix, tiles, s);
        K *tk = kin;
        kin = kout;
        kout = tk;
        uint32_t *tv = vin;
        vin = vout;
        vout = tv;
    }
    *in_alt = (passes & 1) != 0;
    return hipGetLastError();
}

template hipError_t radix_sort_pairs<uint64_t>(uint64_t *, uint32_t *, uint64_t *, uint32_t *, int64_t, int, int,
                                               void *, hipStream_t, bool *);
template hipError_t radix_sort_pairs<uint32_t>(uint32_t *, uint32_t *, uint32_t *, uint32_t *, int64_t, int, int,
                                               void *, hipStream_t, bool *);

}  // namespace ax
