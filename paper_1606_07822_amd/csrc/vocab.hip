// Vocabulary: id histogram, (count desc, id asc) ordering, id -> index map, token remap.
//
// Counting follows "for each wordid v in text" (Algorithm 1) and the mintf
// setting of §4.1. The order is produced by a radix sort of the ids by their
// counts in device memory; the sort is a one-off per corpus.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "w2v_internal.h"
#include "w2v_scan.h"

namespace w2v {
namespace {

constexpr int kHotBins = 36864;   // ids below this are counted in LDS first (Zipf-ranked ids are hot); 144 KiB
constexpr int64_t kRemapHotTokens = 16'000'000;
constexpr int kCountThreads = 1024;   // one workgroup per CU (the bins take most of its LDS)

__global__ __launch_bounds__(kCountThreads) void k_count(const int32_t *__restrict__ tok, int64_t n,
                                                         int32_t id_space, unsigned long long *__restrict__ counts,
                                                         unsigned long long *__restrict__ bad) {
    __shared__ uint32_t hot[kHotBins];
    const int nhot = id_space < kHotBins ? id_space : kHotBins;
    for (int i = threadIdx.x; i < nhot; i += blockDim.x) hot[i] = 0;
    __syncthreads();
    uint32_t my_bad = 0;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x * 4;
    for (int64_t base = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) * 4; base < n;
         base += stride) {
        int32_t t[4];
        if (base + 3 < n && ((reinterpret_cast<uintptr_t>(tok + base) & 15) == 0)) {
            const int4 q = *reinterpret_cast<const int4 *>(tok + base);
            t[0] = q.x; t[1] = q.y; t[2] = q.z; t[3] = q.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) t[k] = (base + k < n) ? tok[base + k] : -2;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t v = t[k];
            if (v == -2 && base + k >= n) continue;
            if (v < 0 || v >= id_space) {
                ++my_bad;
            } else if (v < nhot) {
                atomicAdd(&hot[v], 1u);
            } else {
                atomicAdd(&counts[v], 1ull);
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nhot; i += blockDim.x)
        if (hot[i]) atomicAdd(&counts[i], static_cast<unsigned long long>(hot[i]));
    if (my_bad) atomicAdd(bad, static_cast<unsigned long long>(my_bad));
}

// Long texts over large id spaces: the same, but an id at or past kHotBins goes to the workgroup's list instead of
// to memory's atomics, which bound k_count (1e8 tokens over 1M ids, 18 % of them past the bins: 944 us, 150 without
// them). The lists are partitioned into kBuckets ranges of ids and each range is counted in LDS by one workgroup,
// 400 us in all. The lists lie in the first half of the remapped text's place, workgroup g's at g * cap, their
// partition in the second half; what a full list cannot take is added to memory.
constexpr int kBuckets = 256;
constexpr int kListGroups = 256;   // workgroups, and lists
constexpr int64_t kListTokens = 8'000'000;
constexpr int64_t kListTokensMost = int64_t(1) << 32;

__global__ __launch_bounds__(kCountThreads) void k_count_lists(const int32_t *__restrict__ tok, int64_t n, int32_t id_space,
                                                               unsigned long long *__restrict__ counts,
                                                               unsigned long long *__restrict__ bad,
                                                               int32_t *__restrict__ lists, int64_t cap,
                                                               int32_t *__restrict__ lengths) {
    __shared__ uint32_t hot[kHotBins];
    __shared__ uint32_t s_n;
    for (int i = threadIdx.x; i < kHotBins; i += blockDim.x) hot[i] = 0;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    uint32_t my_bad = 0;
    int32_t *list = lists + blockIdx.x * cap;
    const int lane = lane_id();
    constexpr int kAhead = 2;   // groups of four tokens of each thread in flight
    const int64_t step = static_cast<int64_t>(gridDim.x) * kCountThreads * 4;
    const bool aligned = (reinterpret_cast<uintptr_t>(tok) & 15) == 0;
    for (int64_t b0 = static_cast<int64_t>(blockIdx.x) * kCountThreads * 4; b0 < n; b0 += kAhead * step) {
        int32_t t[kAhead][4];
#pragma unroll
        for (int g = 0; g < kAhead; ++g) {
            const int64_t base = b0 + g * step + threadIdx.x * 4;
            if (aligned && base + 3 < n) {
                const int4 q = *reinterpret_cast<const int4 *>(tok + base);
                t[g][0] = q.x; t[g][1] = q.y; t[g][2] = q.z; t[g][3] = q.w;
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) t[g][k] = base + k < n ? tok[base + k] : -2;   // -2: past the text
            }
        }
#pragma unroll
        for (int g = 0; g < kAhead; ++g) {
            uint64_t cold[4];
            uint32_t total = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t v = t[g][k];
                const bool past = b0 + g * step + threadIdx.x * 4 + k >= n;
                const bool ok = !past && v >= 0 && v < id_space;
                if (!past && !ok) ++my_bad;
                if (ok && v < kHotBins) atomicAdd(&hot[v], 1u);
                cold[k] = __ballot(ok && v >= kHotBins);
                total += static_cast<uint32_t>(__popcll(cold[k]));
            }
            uint32_t at = 0;
            if (lane == 0 && total) at = atomicAdd(&s_n, total);
            at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if ((cold[k] >> lane) & 1ull) {
                    const uint32_t i = at + static_cast<uint32_t>(__popcll(cold[k] & ((1ull << lane) - 1ull)));
                    if (i < cap) list[i] = t[g][k];
                    else atomicAdd(&counts[t[g][k]], 1ull);
                }
                at += static_cast<uint32_t>(__popcll(cold[k]));
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kHotBins; i += blockDim.x)
        if (hot[i]) atomicAdd(&counts[i], static_cast<unsigned long long>(hot[i]));
    if (threadIdx.x == 0) lengths[blockIdx.x] = static_cast<int32_t>(min(static_cast<int64_t>(s_n), cap));
    if (my_bad) atomicAdd(bad, static_cast<unsigned long long>(my_bad));
}

// Bucket sizes of each list: hist[bucket * kListGroups + list].
__global__ __launch_bounds__(kCountThreads) void k_bucket_counts(const int32_t *__restrict__ lists, int64_t cap,
                                                                 const int32_t *__restrict__ lengths, int32_t width,
                                                                 uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[kBuckets];
    if (threadIdx.x < kBuckets) h[threadIdx.x] = 0;
    __syncthreads();
    const int32_t *list = lists + blockIdx.x * cap;
    const int32_t n = lengths[blockIdx.x];
#pragma unroll 8
    for (int32_t i = threadIdx.x; i < n; i += kCountThreads) atomicAdd(&h[list[i] / width], 1u);
    __syncthreads();
    if (threadIdx.x < kBuckets) hist[threadIdx.x * kListGroups + blockIdx.x] = h[threadIdx.x];
}

// Order: ids by count descending, then id ascending; ids below min_count (key 0) come last, in any order. A
// stable radix sort of the ids (in ascending order at the start) by their keys, 8 bits a pass from the lowest, and
// only as many passes as the largest possible count, the number of tokens, has digits. Each pass: every tile's
// digit counts, their scan over (digit, tile), and the tiles' stable scatter. What bounds it is the chain of its
// launches: at 1M ids and 1e8 tokens (4 passes) it takes 125 us with the placing of the words;
// a bitonic sort of 16-byte records in 55 launches took 640.
constexpr int kDigits = 256;
constexpr int kTileThreads = 1024;
constexpr int kTileWaves = kTileThreads / kWave;
constexpr int kPerThread = 4;
constexpr int kTile = kTileThreads * kPerThread;   // ids of a workgroup: 256 consecutive ones a wavefront
constexpr int kWaveIds = kWave * kPerThread;

__device__ __forceinline__ int64_t sort_key(int64_t count, int64_t min_count) { return count >= min_count ? count : 0; }

// digit of a key in descending order
__device__ __forceinline__ int key_digit(int64_t key, int shift) {
    return (kDigits - 1) - static_cast<int>((key >> shift) & (kDigits - 1));
}

// The lanes (of those with `in`) that hold the same digit.
__device__ __forceinline__ uint64_t same_digit(int digit, bool in) {
    uint64_t m = __ballot(in);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t set = __ballot((digit >> b) & 1);
        m &= ((digit >> b) & 1) ? set : ~set;
    }
    return m;
}

// Stable places of a tile's ids for one digit, by one workgroup of kTileThreads. Element k of a thread is the
// wavefront's k-th row of 64. first(digit) gives where the tile's ids of a digit start. counts: LDS
// [kTileWaves][kDigits].
template <class First>
__device__ __forceinline__ void tile_places(const int (&digit)[kPerThread], const bool (&in)[kPerThread],
                                            uint32_t (*counts)[kDigits], First first, uint32_t (&place)[kPerThread]) {
    const int wid = static_cast<int>(threadIdx.x / kWave);
    for (int i = threadIdx.x; i < kTileWaves * kDigits; i += kTileThreads) (&counts[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPerThread; ++k)
        if (in[k]) atomicAdd(&counts[wid][digit[k]], 1u);
    __syncthreads();
    if (threadIdx.x < kDigits) {
        uint32_t at = first(static_cast<int>(threadIdx.x));
        for (int w = 0; w < kTileWaves; ++w) {
            const uint32_t n = counts[w][threadIdx.x];
            counts[w][threadIdx.x] = at;
            at += n;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const uint64_t m = same_digit(digit[k], in[k]);
        const uint64_t below = m & ((1ull << lane_id()) - 1ull);
        place[k] = in[k] ? counts[wid][digit[k]] + static_cast<uint32_t>(__popcll(below)) : 0u;
        __builtin_amdgcn_wave_barrier();
        if (in[k] && below == 0) counts[wid][digit[k]] += static_cast<uint32_t>(__popcll(m));
        __builtin_amdgcn_wave_barrier();
    }
}

// Exclusive scan of the digits' counts by the first wavefront, four to a lane.
__device__ __forceinline__ void digit_starts(const uint32_t *n, uint32_t *first) {
    if (threadIdx.x < kWave) {
        uint32_t v[4], mine = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) mine += v[k] = n[4 * threadIdx.x + k];
        uint32_t inc = mine;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(inc, d, kWave);
            if (lane_id() >= d) inc += y;
        }
        uint32_t at = inc - mine;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            first[4 * threadIdx.x + k] = at;
            at += v[k];
        }
    }
}

__global__ __launch_bounds__(kTileThreads) void k_digit_counts(const int64_t *__restrict__ counts, int64_t min_count,
                                                               const int32_t *__restrict__ ids, int32_t n, int shift,
                                                               int32_t tiles, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[kDigits];
    if (threadIdx.x < kDigits) h[threadIdx.x] = 0;
    __syncthreads();
    const int32_t base = static_cast<int32_t>(blockIdx.x) * kTile;
    for (int32_t i = base + static_cast<int32_t>(threadIdx.x); i < min(n, base + kTile); i += kTileThreads)
        atomicAdd(&h[key_digit(sort_key(counts[ids ? ids[i] : i], min_count), shift)], 1u);
    __syncthreads();
    if (threadIdx.x < kDigits) hist[static_cast<int64_t>(threadIdx.x) * tiles + blockIdx.x] = h[threadIdx.x];
}

// One workgroup per digit: exclusive scan of its counts over the tiles, in place, and their sum.
constexpr int kRowThreads = 256;
__global__ __launch_bounds__(kRowThreads) void k_scan_digits(uint32_t *hist, int32_t tiles, uint32_t *__restrict__ sums) {
    __shared__ uint32_t wsum[kRowThreads / kWave];
    uint32_t *row = hist + static_cast<int64_t>(blockIdx.x) * tiles;
    const int lane = lane_id(), wid = static_cast<int>(threadIdx.x / kWave);
    uint32_t carry = 0;
    for (int32_t base = 0; base < tiles; base += kRowThreads) {
        const int64_t i = static_cast<int64_t>(base) + threadIdx.x;
        const uint32_t x = i < tiles ? row[i] : 0;
        uint32_t inc = x;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(inc, d, kWave);
            if (lane >= d) inc += y;
        }
        if (lane == kWave - 1) wsum[wid] = inc;
        __syncthreads();
        uint32_t before = carry, step = 0;
        for (int w = 0; w < kRowThreads / kWave; ++w) {
            before += w < wid ? wsum[w] : 0;
            step += wsum[w];
        }
        __syncthreads();   // wsum is rewritten by the next step
        if (i < tiles) row[i] = before + inc - x;
        carry += step;
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = carry;
}

// Each list's ids to their buckets (in any order within one); hist: the lists' starts within each bucket.
__global__ __launch_bounds__(kCountThreads) void k_bucket_ids(const int32_t *__restrict__ lists, int64_t cap,
                                                              const int32_t *__restrict__ lengths, int32_t width,
                                                              const uint32_t *__restrict__ hist,
                                                              const uint32_t *__restrict__ sums,
                                                              int32_t *__restrict__ out) {
    __shared__ uint32_t at[kBuckets];
    digit_starts(sums, at);
    __syncthreads();
    if (threadIdx.x < kBuckets) at[threadIdx.x] += hist[threadIdx.x * kListGroups + blockIdx.x];
    __syncthreads();
    const int32_t *list = lists + blockIdx.x * cap;
    const int32_t n = lengths[blockIdx.x];
    int32_t i = threadIdx.x;
    for (; i + 3 * kCountThreads < n; i += 4 * kCountThreads) {   // four ids of each thread in flight
        int32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = list[i + k * kCountThreads];
#pragma unroll
        for (int k = 0; k < 4; ++k) out[atomicAdd(&at[v[k] / width], 1u)] = v[k];
    }
    for (; i < n; i += kCountThreads) out[atomicAdd(&at[list[i] / width], 1u)] = list[i];
}

// One workgroup per bucket, the only one that adds to its ids' counts.
__global__ __launch_bounds__(kCountThreads) void k_count_bucket(const int32_t *__restrict__ ids, int32_t width,
                                                                int32_t id_space, const uint32_t *__restrict__ sums,
                                                                unsigned long long *__restrict__ counts) {
    __shared__ uint32_t bins[kHotBins];
    __shared__ uint32_t first[kBuckets];
    for (int i = threadIdx.x; i < width; i += kCountThreads) bins[i] = 0;
    digit_starts(sums, first);
    __syncthreads();
    const int32_t base = static_cast<int32_t>(blockIdx.x) * width;
    const uint32_t n = sums[blockIdx.x];
    const int32_t *mine = ids + first[blockIdx.x];
    uint32_t i0 = threadIdx.x;
    for (; i0 + 7 * kCountThreads < n; i0 += 8 * kCountThreads) {   // eight ids of each thread in flight
        int32_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = mine[i0 + k * kCountThreads];
#pragma unroll
        for (int k = 0; k < 8; ++k) atomicAdd(&bins[v[k] - base], 1u);
    }
    for (; i0 < n; i0 += kCountThreads) atomicAdd(&bins[mine[i0] - base], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < width && base + i < id_space; i += kCountThreads)
        if (bins[i]) counts[base + i] += bins[i];
}

__global__ __launch_bounds__(kTileThreads) void k_scatter_ids(const int64_t *__restrict__ counts, int64_t min_count,
                                                              const int32_t *__restrict__ ids, int32_t n, int shift,
                                                              int32_t tiles, const uint32_t *__restrict__ hist,
                                                              const uint32_t *__restrict__ sums,
                                                              int32_t *__restrict__ out) {
    __shared__ uint32_t s_counts[kTileWaves][kDigits];
    __shared__ uint32_t s_first[kDigits];
    digit_starts(sums, s_first);   // read after the barriers of tile_places
    int digit[kPerThread], id[kPerThread];
    bool in[kPerThread];
    uint32_t place[kPerThread];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kTile + (threadIdx.x / kWave) * kWaveIds + lane_id();
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int64_t i = base + k * kWave;
        in[k] = i < n;
        id[k] = in[k] ? (ids ? ids[i] : static_cast<int32_t>(i)) : 0;
        digit[k] = in[k] ? key_digit(sort_key(counts[id[k]], min_count), shift) : 0;
    }
    tile_places(digit, in, s_counts, [&](int d) {
        return s_first[d] + hist[static_cast<int64_t>(d) * tiles + blockIdx.x];
    }, place);
#pragma unroll
    for (int k = 0; k < kPerThread; ++k)
        if (in[k]) out[place[k]] = id[k];
}

// Vocabulary entry of position i of the order. The kept words come first.
__device__ __forceinline__ void place_word(const int64_t *__restrict__ counts, int64_t min_count, int32_t id, int32_t i,
                                           int32_t *__restrict__ vocab_ids, int64_t *__restrict__ vocab_counts,
                                           int32_t *__restrict__ id_to_vocab, int64_t &words, int64_t &total) {
    const int64_t c = counts[id];
    const bool kept = c >= min_count;
    vocab_ids[i] = kept ? id : -1;
    vocab_counts[i] = kept ? c : 0;
    id_to_vocab[id] = kept ? i : -1;
    words += kept ? 1 : 0;
    total += kept ? c : 0;
}

// One add per workgroup: thousands of adds to one address take longer than the rest of the kernel.
__device__ __forceinline__ void add_totals(int64_t words, int64_t total, unsigned long long *nv, unsigned long long *tw) {
    __shared__ unsigned long long s_sum[2];
    if (threadIdx.x < 2) s_sum[threadIdx.x] = 0;
    __syncthreads();
    words = wave_sum(words);
    total = wave_sum(total);
    if (lane_id() == 0 && words) {
        atomicAdd(&s_sum[0], static_cast<unsigned long long>(words));
        atomicAdd(&s_sum[1], static_cast<unsigned long long>(total));
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_sum[0]) {
        atomicAdd(nv, s_sum[0]);
        atomicAdd(tw, s_sum[1]);
    }
}

__global__ __launch_bounds__(kTileThreads) void k_finish_vocab(const int64_t *__restrict__ counts, int64_t min_count,
                                                      const int32_t *__restrict__ ids, int32_t n,
                                                      int32_t *__restrict__ vocab_ids, int64_t *__restrict__ vocab_counts,
                                                      int32_t *__restrict__ id_to_vocab,
                                                      unsigned long long *__restrict__ nv,
                                                      unsigned long long *__restrict__ tw) {
    int64_t words = 0, total = 0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        place_word(counts, min_count, ids[i], static_cast<int32_t>(i), vocab_ids, vocab_counts, id_to_vocab, words,
                   total);
    add_totals(words, total, nv, tw);
}

// Id spaces of one tile: the whole order and its words in one launch (1,000 ids, 3 passes: 17 us; the
// bitonic tile sort, the fill and the placing took 55).
__global__ __launch_bounds__(kTileThreads) void k_order_small(const int64_t *__restrict__ counts, int64_t min_count,
                                                              int32_t n, int bits, int32_t *__restrict__ vocab_ids,
                                                              int64_t *__restrict__ vocab_counts,
                                                              int32_t *__restrict__ id_to_vocab,
                                                              unsigned long long *__restrict__ nv,
                                                              unsigned long long *__restrict__ tw) {
    __shared__ uint32_t s_counts[kTileWaves][kDigits];
    __shared__ uint32_t s_hist[kDigits], s_first[kDigits];
    __shared__ int32_t s_ids[kTile];
    for (int32_t i = threadIdx.x; i < n; i += kTileThreads) s_ids[i] = i;
    for (int shift = 0; shift < bits; shift += 8) {
        int digit[kPerThread], id[kPerThread];
        bool in[kPerThread];
        uint32_t place[kPerThread];
        if (threadIdx.x < kDigits) s_hist[threadIdx.x] = 0;
        __syncthreads();
        const int base = (threadIdx.x / kWave) * kWaveIds + lane_id();
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            in[k] = base + k * kWave < n;
            id[k] = in[k] ? s_ids[base + k * kWave] : 0;
            digit[k] = in[k] ? key_digit(sort_key(counts[id[k]], min_count), shift) : 0;
            if (in[k]) atomicAdd(&s_hist[digit[k]], 1u);
        }
        __syncthreads();
        digit_starts(s_hist, s_first);
        __syncthreads();
        tile_places(digit, in, s_counts, [&](int d) { return s_first[d]; }, place);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPerThread; ++k)
            if (in[k]) s_ids[place[k]] = id[k];
        __syncthreads();
    }
    __syncthreads();
    int64_t words = 0, total = 0;
    for (int32_t i = threadIdx.x; i < n; i += kTileThreads)
        place_word(counts, min_count, s_ids[i], i, vocab_ids, vocab_counts, id_to_vocab, words, total);
    add_totals(words, total, nv, tw);
}

// Four tokens per thread and step (16-byte loads and stores where the stream is 16-byte aligned), so that
// each thread keeps four independent gathers from id_to_vocab in flight.
__global__ void k_remap(const int32_t *__restrict__ tok, int64_t n, const int32_t *__restrict__ id_to_vocab,
                        int32_t id_space, int32_t *__restrict__ out) {
    auto map = [&](int32_t v) { return (v >= 0 && v < id_space) ? id_to_vocab[v] : -1; };
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const bool aligned = ((reinterpret_cast<uintptr_t>(tok) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
    const int64_t nq = aligned ? n / 4 : 0;   // whole 16-byte groups
    for (int64_t q = tid; q < nq; q += stride) {
        const int4 t = reinterpret_cast<const int4 *>(tok)[q];
        reinterpret_cast<int4 *>(out)[q] = make_int4(map(t.x), map(t.y), map(t.z), map(t.w));
    }
    for (int64_t i = nq * 4 + tid; i < n; i += stride) out[i] = map(tok[i]);
}

// The same for long texts: the indices of the ids below kHotBins (most tokens of a text whose ids are ranks) are
// looked up in LDS, which every workgroup fills first, so it pays from some tokens per workgroup on. Gathers from
// the cache bound k_remap (1e8 tokens over 1M ids: 390 us); this takes 268, with one
// group of four tokens in flight per thread 308, and no less than k_remap below some 16 million tokens.
__global__ __launch_bounds__(kCountThreads) void k_remap_hot(const int32_t *__restrict__ tok, int64_t n,
                                                             const int32_t *__restrict__ id_to_vocab,
                                                             int32_t id_space, int32_t *__restrict__ out) {
    __shared__ int32_t hot[kHotBins];
    const int nhot = id_space < kHotBins ? id_space : kHotBins;
    for (int i = threadIdx.x; i < nhot; i += blockDim.x) hot[i] = id_to_vocab[i];
    __syncthreads();
    auto map = [&](int32_t v) {
        return v >= 0 && v < id_space ? (v < nhot ? hot[v] : id_to_vocab[v]) : -1;
    };
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const bool aligned = ((reinterpret_cast<uintptr_t>(tok) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
    const int64_t nq = aligned ? n / 4 : 0;   // whole 16-byte groups
    constexpr int kAhead = 4;   // groups of each thread in flight: one workgroup per compute unit has 16 wavefronts
    int64_t q = tid;
    for (; q + (kAhead - 1) * stride < nq; q += kAhead * stride) {
        int4 t[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) t[k] = reinterpret_cast<const int4 *>(tok)[q + k * stride];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) t[k] = make_int4(map(t[k].x), map(t[k].y), map(t[k].z), map(t[k].w));
#pragma unroll
        for (int k = 0; k < kAhead; ++k) reinterpret_cast<int4 *>(out)[q + k * stride] = t[k];
    }
    for (; q < nq; q += stride) {
        const int4 t = reinterpret_cast<const int4 *>(tok)[q];
        reinterpret_cast<int4 *>(out)[q] = make_int4(map(t.x), map(t.y), map(t.z), map(t.w));
    }
    for (int64_t i = nq * 4 + tid; i < n; i += stride) out[i] = map(tok[i]);
}

__global__ void k_zero_counts(unsigned long long *counts, int64_t n, unsigned long long *scal) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) counts[i] = 0;
    if (i < 4) scal[i] = 0;
}

}  // namespace

size_t vocab_workspace_bytes(int32_t id_space) {
    Carve c;
    c.take<int32_t>(static_cast<size_t>(id_space));   // two id lists, one pass reading the other's
    c.take<int32_t>(static_cast<size_t>(id_space));
    c.take<uint32_t>(static_cast<size_t>(ceil_div(id_space, kTile)) * kDigits);   // digit counts by digit and tile
    c.take<uint32_t>(kDigits);
    c.take<unsigned long long>(4);
    c.take<uint32_t>(kBuckets * kListGroups);   // the long texts' lists: bucket sizes, lengths
    c.take<int32_t>(kListGroups);
    return c.used();
}

int run_build_vocab(const int32_t *tokens, int64_t n_tokens, int32_t id_space, int64_t min_count,
                    int64_t *counts_by_id, int32_t *vocab_ids, int64_t *vocab_counts, int32_t *id_to_vocab,
                    int32_t *tokens_out, int32_t *V_host, int64_t *train_words_host, void *workspace,
                    hipStream_t s) {
    Carve c(workspace);
    const int32_t tiles = static_cast<int32_t>(ceil_div(id_space, kTile));
    int32_t *list[2] = {c.take<int32_t>(static_cast<size_t>(id_space)), c.take<int32_t>(static_cast<size_t>(id_space))};
    uint32_t *hist = c.take<uint32_t>(static_cast<size_t>(tiles) * kDigits);
    uint32_t *sums = c.take<uint32_t>(kDigits);
    unsigned long long *scal = c.take<unsigned long long>(4);   // bad, V, train_words
    uint32_t *bucket_hist = c.take<uint32_t>(kBuckets * kListGroups);
    int32_t *lengths = c.take<int32_t>(kListGroups);
    unsigned long long *counts = reinterpret_cast<unsigned long long *>(counts_by_id);

    k_zero_counts<<<static_cast<unsigned>(ceil_div(id_space, 256)), 256, 0, s>>>(counts, id_space, scal);
    W2V_LAUNCH_CHECK("zero");
    const int32_t width = static_cast<int32_t>(ceil_div(id_space, kBuckets));
    // Lists pay where memory's atomics would take most of the time: texts of some millions of tokens, with ids past
    // the bins, whose ranges fit LDS and whose remapped text has room for them (without one the atomics stay); places
    // in the lists' partition (at most half as many as tokens) are 32 bits. Whole call with and without them, us:
    //                          1e6 tokens   4e6          8e6          1.6e7        3.2e7
    //   200K ids, Zipf ranks   151 / 132    181 / 174    208 / 222    258 / 295    334 / 434
    //   1M ids, Zipf ranks     160 / 158    193 / 208    230 / 275    297 / 392    413 / 623
    //   50K ids, scattered     239 / 1183   236 / 522    823 / 8593   1454 / 17066 2683 / 33998
    //   50K ids, Zipf ranks    156 / 130    183 / 149    212 / 189    258 / 230    318 / 298
    //   36,865 ids, Zipf ranks 154 / 129    174 / 156    193 / 184    232 / 214    280 / 265
    // (scattered: the frequent ids lie anywhere). The lists cost some 20 us of launches where next to no id is past
    // the bins, which the ids' number does not tell; without them frequent ids there cost milliseconds.
    if (tokens_out && n_tokens >= kListTokens && n_tokens <= kListTokensMost && id_space > kHotBins &&
        width <= kHotBins) {
        const int64_t cap = std::min<int64_t>(n_tokens / 2 / kListGroups, INT32_MAX);
        int32_t *parted = tokens_out + n_tokens / 2;
        k_count_lists<<<kListGroups, kCountThreads, 0, s>>>(tokens, n_tokens, id_space, counts, scal + 0, tokens_out, cap,
                                                            lengths);
        k_bucket_counts<<<kListGroups, kCountThreads, 0, s>>>(tokens_out, cap, lengths, width, bucket_hist);
        k_scan_digits<<<kBuckets, kRowThreads, 0, s>>>(bucket_hist, kListGroups, sums);
        k_bucket_ids<<<kListGroups, kCountThreads, 0, s>>>(tokens_out, cap, lengths, width, bucket_hist, sums, parted);
        k_count_bucket<<<kBuckets, kCountThreads, 0, s>>>(parted, width, id_space, sums, counts);
        W2V_LAUNCH_CHECK("k_count_lists");
    } else if (n_tokens > 0) {
        const int cus = device_cu_count();
        const int64_t want = ceil_div(n_tokens, static_cast<int64_t>(kCountThreads) * 4 * 8);
        const unsigned grid = static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>(want, 1LL * cus)));
        k_count<<<grid, kCountThreads, 0, s>>>(tokens, n_tokens, id_space, counts, scal + 0);
        W2V_LAUNCH_CHECK("k_count");
    }
    int bits = 1;   // of the largest possible count
    while (bits < 63 && (n_tokens >> bits) != 0) ++bits;
    if (tiles == 1) {
        k_order_small<<<1, kTileThreads, 0, s>>>(counts_by_id, min_count, id_space, bits, vocab_ids, vocab_counts,
                                                 id_to_vocab, scal + 1, scal + 2);
        W2V_LAUNCH_CHECK("k_order_small");
    } else {
        const int32_t *ids = nullptr;   // the first pass reads the ids in order
        int to = 0;
        for (int shift = 0; shift < bits; shift += 8, to ^= 1) {
            k_digit_counts<<<static_cast<unsigned>(tiles), kTileThreads, 0, s>>>(counts_by_id, min_count, ids, id_space,
                                                                                 shift, tiles, hist);
            k_scan_digits<<<kDigits, kRowThreads, 0, s>>>(hist, tiles, sums);
            k_scatter_ids<<<static_cast<unsigned>(tiles), kTileThreads, 0, s>>>(counts_by_id, min_count, ids, id_space,
                                                                                shift, tiles, hist, sums, list[to]);
            W2V_LAUNCH_CHECK("sort pass");
            ids = list[to];
        }
        k_finish_vocab<<<static_cast<unsigned>(std::min<int64_t>(tiles, device_cu_count())), kTileThreads, 0, s>>>(
            counts_by_id, min_count, ids, id_space, vocab_ids, vocab_counts, id_to_vocab, scal + 1, scal + 2);
        W2V_LAUNCH_CHECK("k_finish_vocab");
    }
    if (tokens_out && n_tokens > 0) {
        if (n_tokens >= kRemapHotTokens) {
            k_remap_hot<<<static_cast<unsigned>(device_cu_count()), kCountThreads, 0, s>>>(tokens, n_tokens, id_to_vocab,
                                                                                           id_space, tokens_out);
        } else {
            const unsigned grid = static_cast<unsigned>(std::min<int64_t>(ceil_div(n_tokens, 4 * 256), 8192));
            k_remap<<<grid, 256, 0, s>>>(tokens, n_tokens, id_to_vocab, id_space, tokens_out);
        }
        W2V_LAUNCH_CHECK("k_remap");
    }
    unsigned long long h[3];
    W2V_HIP(hipMemcpyAsync(h, scal, sizeof(h), hipMemcpyDeviceToHost, s));
    W2V_HIP(hipStreamSynchronize(s));
    *V_host = static_cast<int32_t>(h[1]);
    *train_words_host = static_cast<int64_t>(h[2]);
    if (h[0] != 0)
        return fail(W2V_E_RANGE, std::to_string(h[0]) + " token(s) outside [0, id_space)");
    return W2V_OK;
}

}  // namespace w2v
