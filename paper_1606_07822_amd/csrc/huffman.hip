// Huffman tree of the vocabulary (§2: output layer of the hierarchical softmax).
//
// Construction rule: leaves in ascending count (vocabulary index V-1 first),
// inner nodes in creation order; each merge takes the smaller front twice, a
// leaf winning a count tie; the first child taken gets bit 0; merge a creates
// inner node a (root = V-2). The chain of merges is split into generations that
// are each computed in parallel (below). Parallel kernels then derive codes,
// offsets and points.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "w2v_internal.h"
#include "w2v_scan.h"

namespace w2v {
namespace {

// Generations. Both queues are in ascending order, and the inner queue is first in,
// first out. Call the inner nodes that exist when a generation starts (indices
// ih .. a-1) old. While an old node is still queued, the inner front is an old node,
// so every pick is the smaller of the leaf front and an old node: the picks are the
// stable merge S of the leaf queue with the old nodes (a leaf first on a tie), and
// merge a+j takes S[2j] (bit 0) and S[2j+1] (bit 1). S ends with the last old node,
// after the leaves whose count is at most its count. If S has odd length, its last
// element (the last old node) opens one more merge whose second pick is the smaller of
// the leaf front and the first node of this generation (node a), and the next
// generation starts. A Zipf vocabulary of 1M words takes 26 generations.
//
// Each generation makes the tree one level deeper (it consumes every old node), so a tree
// whose codes fit 64 bits takes at most kMaxGenerations of them.
//
// The workgroups of a cooperative launch share a generation in chunks of kChunk elements
// of S, each found by a search on the merge path (the i with A[i-1] <= B[k-i-1] and
// B[k-i-1] < A[i] at diagonal k, A the leaves, B the old nodes), and meet at a barrier
// after it; every workgroup computes the generation's extent and the next queue fronts
// itself, so only the node counts pass between them. What bounds it is the chain: per
// generation one search over the leaves (64 probes a step, four steps at V = 1M), one
// merge and one barrier. One workgroup walking the chunks in turn took 4.14 ms at
// V = 1M (992 chunks), this 0.27 ms.
constexpr int kMergeThreads = 1024;
constexpr int kChunk = 2 * kMergeThreads;   // elements of S per chunk: one merge per thread
constexpr int kMaxMergeGroups = 128;
constexpr int kMaxGenerations = 72;

// Entry of `up` that no merge has written. Counts whose sums pass 2^63 give queues that are not ascending, and
// the merge then takes some nodes twice and others never; k_huff_codes refuses a path through one of those.
constexpr uint32_t kNoParent = ~0u;

__global__ void k_check_descending(const int64_t *__restrict__ counts, int32_t V, uint2 *__restrict__ up,
                                   int32_t *__restrict__ flags) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < V) up[i] = make_uint2(kNoParent, kNoParent);   // two of the 2 V entries
    if (i + 1 < V && counts[i] < counts[i + 1]) atomicOr(&flags[2], 1);
}

// Leaves in ascending count: position p is vocabulary index V-1-p.
__device__ __forceinline__ int64_t leaf_val(const int64_t *__restrict__ counts, int32_t V, int32_t p) {
    return counts[V - 1 - p];
}

// Every workgroup's writes before the barrier are visible to every workgroup after it: each wavefront waits until
// its stores have reached the L2 (a workgroup's barrier alone does not wait for them), then one writes the L2 back
// for the readers on other dies. (A fence by every wavefront, each with a write-back: 1,117 instead of 400 us for
// the tree at V = 1M.) The launch is cooperative (all workgroups resident) and every workgroup passes the same
// number of barriers, so the wait ends.
__device__ __forceinline__ void grid_barrier(uint32_t *arrived, uint32_t target) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        while (__hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target)
            __builtin_amdgcn_s_sleep(1);
        __threadfence();
    }
    __syncthreads();
}

// up[node] = parent << 1 | bit; node v < V is a leaf (vocabulary index), V + a inner node a. The root's
// entry is not written.
__global__ __launch_bounds__(kMergeThreads) void k_huff_merge(const int64_t *__restrict__ counts, int32_t V,
                                                              uint32_t *__restrict__ up, int64_t *icount,
                                                              int32_t *flags, uint32_t *arrived) {
    __shared__ int64_t s_val[kChunk];          // the chunk's leaves, then its old nodes
    __shared__ int32_t s_leaves, s_i0, s_i1;   // leaves of the generation; leaves before this chunk and its end
    __shared__ int32_t s_take_leaf;
    if (flags[2]) return;                      // counts not in descending order: no tree
    const int tid = threadIdx.x, wid = tid / kWave;
    const int32_t groups = gridDim.x;
    uint32_t target = 0;
    // queue state, the same in every thread: leaf front pl, inner front ih, next merge a
    int32_t pl = 2, ih = 0, a = 1;
    if (blockIdx.x == 0 && tid == 0) {         // the first merge: two leaves
        up[V - 1] = 0;
        up[V - 2] = 1;
        icount[0] = leaf_val(counts, V, 0) + leaf_val(counts, V, 1);
    }
    grid_barrier(arrived, target += groups);
    for (int gen = 0; a < V - 1; ++gen) {
        if (gen == kMaxGenerations) {          // deeper than 64 levels
            if (blockIdx.x == 0 && tid == 0) atomicOr(&flags[1], 1);
            return;
        }
        const int32_t T = a - ih;              // old nodes ih .. a-1
        const int32_t left = V - pl;           // leaves not yet taken
        auto leaf = [&](int32_t i) { return leaf_val(counts, V, pl + i); };
        auto old_node = [&](int32_t i) { return icount[ih + i]; };
        // leaves among the first k elements of S (leaves above the last old node's count never come before it)
        auto leaves_before = [&](int32_t k) {
            return wave_partition_point(max(0, k - T), min(k, left),
                                        [&](int32_t m) { return leaf(m) <= old_node(k - m - 1); });
        };
        const int64_t most = static_cast<int64_t>(T) + left;   // no chunk starts or ends past this
        int64_t k0 = static_cast<int64_t>(blockIdx.x) * kChunk;
        if (wid == 0) {
            const int64_t last = old_node(T - 1);
            const int32_t n = wave_partition_point(0, left, [&](int32_t m) { return leaf(m) <= last; });
            if (tid == 0) s_leaves = n;
        } else if (wid == 1) {
            const int32_t n = k0 < most ? leaves_before(static_cast<int32_t>(k0)) : 0;
            if (lane_id() == 0) s_i0 = n;
        } else if (wid == 2) {
            const int32_t n = k0 + kChunk < most ? leaves_before(static_cast<int32_t>(k0 + kChunk)) : 0;
            if (lane_id() == 0) s_i1 = n;
        }
        __syncthreads();
        const int32_t nl = s_leaves;
        const int32_t M = (T + nl) >> 1;       // merges within S
        const bool odd = (T + nl) & 1;
        if (tid == 0) {
            bool take_leaf = false;
            if (odd) {
                // second pick of the last old node's merge: the leaf front, or node a (the two smallest of S;
                // there is one if S has three elements), a leaf winning a tie
                const bool fresh = M > 0;
                const bool more = nl < left;
                int64_t first = 0;
                if (fresh) {
                    const int64_t inf = INT64_MAX;
                    const int64_t l0 = nl > 0 ? leaf(0) : inf, l1 = nl > 1 ? leaf(1) : inf;
                    const int64_t b0 = old_node(0), b1 = T > 1 ? old_node(1) : inf;
                    first = l0 <= b0 ? l0 + (l1 <= b0 ? l1 : b0) : b0 + (l0 <= b1 ? l0 : b1);
                }
                const int64_t lf = more ? leaf(nl) : 0;
                take_leaf = more && (!fresh || lf <= first);
                if (blockIdx.x == 0) {
                    const int32_t m = a + M;
                    up[V + a - 1] = static_cast<uint32_t>(m) << 1;
                    up[take_leaf ? V - 1 - (pl + nl) : V + a] = static_cast<uint32_t>(m) << 1 | 1u;
                    icount[m] = old_node(T - 1) + (take_leaf ? lf : first);
                }
            }
            s_take_leaf = take_leaf;
        }
        for (bool begun = true; k0 < 2LL * M; k0 += static_cast<int64_t>(groups) * kChunk, begun = false) {
            if (!begun) {                      // not the first chunk of this workgroup: its searches
                __syncthreads();               // the chunk before is merged
                const int64_t at = wid == 0 ? k0 : k0 + kChunk;
                if (wid < 2) {
                    const int32_t n = at < most ? leaves_before(static_cast<int32_t>(at)) : 0;
                    if (lane_id() == 0) (wid == 0 ? s_i0 : s_i1) = n;
                }
                __syncthreads();
            }
            const bool ends = k0 + kChunk >= 2LL * M;   // S's last chunk: all leaves come before its end
            const int32_t n = static_cast<int32_t>(ends ? 2LL * M - k0 : kChunk);
            // (the clamps only matter for counts whose sums pass 63 bits and are not ascending: a search then ends
            // anywhere in its range, and every index still stays within its queue)
            const int32_t i0 = s_i0, i1 = max(i0, min(ends ? nl : s_i1, min(i0 + n, left)));
            const int32_t j0 = static_cast<int32_t>(k0) - i0;
            const int32_t lw = i1 - i0, iw = n - lw;
            for (int32_t t = tid; t < n; t += kMergeThreads)
                s_val[t] = t < lw ? leaf(i0 + t) : old_node(min(j0 + t - lw, T - 1));
            __syncthreads();
            if (2 * tid < n) {
                const int64_t *A = s_val, *B = s_val + lw;
                const int32_t k = 2 * tid;
                int32_t lo = max(0, k - iw), hi = min(k, lw);
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (A[mid] <= B[k - mid - 1]) lo = mid + 1;
                    else hi = mid;
                }
                int32_t i = lo;
                const int32_t m = a + static_cast<int32_t>(k0 / 2) + tid;
                int64_t sum = 0;
#pragma unroll
                for (int pick = 0; pick < 2; ++pick) {
                    const int32_t j = k + pick - i;
                    const bool is_leaf = i < lw && (j >= iw || A[i] <= B[j]);
                    sum += is_leaf ? A[i] : B[j];
                    up[is_leaf ? V - 1 - (pl + i0 + i) : V + ih + min(j0 + j, T - 1)] = static_cast<uint32_t>(m) << 1 | pick;
                    i += is_leaf;
                }
                icount[m] = sum;
            }
        }
        __syncthreads();
        const bool take_leaf = s_take_leaf != 0;
        pl += nl + (odd && take_leaf);
        ih += T + (odd && !take_leaf);         // node a leaves the queue when the last old node took it
        a += M + odd;
        if (a < V - 1) grid_barrier(arrived, target += groups);
    }
}

// codelen / code per leaf; error flag (code longer than 64, or a node that was never merged). Depth does not fall
// along the queues (the inner queue is first in, first out, so an earlier node's parent is never later), so the last
// word has the longest code.
__global__ void k_huff_codes(const uint32_t *__restrict__ up, int32_t V, uint8_t *__restrict__ codelen,
                             uint64_t *__restrict__ code, int32_t *__restrict__ flags) {
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    if (flags[1] | flags[2]) {   // no tree
        codelen[v] = 0;
        code[v] = 0;
        return;
    }
    const int32_t root = V + V - 2;
    int32_t node = v, depth = 0;
    uint64_t rev = 0;
    while (node != root) {
        const uint32_t u = up[node];
        if (depth >= 64 || u >> 1 > static_cast<uint32_t>(V - 2)) {
            atomicOr(&flags[3], 1);
            codelen[v] = 0;
            code[v] = 0;
            return;
        }
        rev |= static_cast<uint64_t>(u & 1u) << depth;
        ++depth;
        node = V + static_cast<int32_t>(u >> 1);
    }
    codelen[v] = static_cast<uint8_t>(depth);
    code[v] = depth ? (__brevll(rev) >> (64 - depth)) : 0;
    if (v == V - 1) flags[0] = depth;
}

// Exclusive prefix sum of codelen into point_off[0..V] in three passes: the sum of each tile of
// kScanTile code lengths, one block scanning the tile sums, and each tile's own scan plus its offset.
// (At V = 1M this takes well under 0.1 ms; the one-workgroup block_exclusive_scan that the smaller
// per-document scans use would take about 0.8 ms here.)
constexpr int kScanTile = 1024;

// inclusive block scan of one value per thread (kScanTile threads); returns the inclusive prefix, *sum the total
__device__ __forceinline__ int64_t block_incl_scan(int64_t x, int64_t *wsum, int64_t *sum) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int64_t inc = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) wsum[wid] = inc;
    __syncthreads();
    int64_t before = 0, total = 0;
    for (int w = 0; w < kScanTile / 64; ++w) {
        before += w < wid ? wsum[w] : 0;
        total += wsum[w];
    }
    *sum = total;
    __syncthreads();   // wsum is reused by the next call
    return before + inc;
}

__global__ __launch_bounds__(kScanTile) void k_scan_tiles(const uint8_t *__restrict__ codelen, int32_t V,
                                                          int64_t *__restrict__ tile_sum) {
    __shared__ int64_t wsum[kScanTile / 64];
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x;
    int64_t total;
    block_incl_scan(i < V ? codelen[i] : 0, wsum, &total);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// tile_sum -> exclusive tile offsets in place; *total = sum of all code lengths
__global__ __launch_bounds__(kScanTile) void k_scan_tile_sums(int64_t *__restrict__ tile_sum, int32_t n_tiles,
                                                              int64_t *__restrict__ total) {
    __shared__ int64_t wsum[kScanTile / 64];
    int64_t carry = 0;
    for (int32_t base = 0; base < n_tiles; base += kScanTile) {
        const int32_t i = base + threadIdx.x;
        const int64_t x = i < n_tiles ? tile_sum[i] : 0;
        int64_t chunk;
        const int64_t inc = block_incl_scan(x, wsum, &chunk);
        if (i < n_tiles) tile_sum[i] = carry + inc - x;
        carry += chunk;
    }
    if (threadIdx.x == 0) *total = carry;
}

__global__ __launch_bounds__(kScanTile) void k_scan_apply(const uint8_t *__restrict__ codelen, int32_t V,
                                                          const int64_t *__restrict__ tile_off,
                                                          const int64_t *__restrict__ total,
                                                          int32_t *__restrict__ point_off) {
    __shared__ int64_t wsum[kScanTile / 64];
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x;
    const int64_t x = i < V ? codelen[i] : 0;
    int64_t chunk;
    const int64_t inc = block_incl_scan(x, wsum, &chunk);
    if (i < V) point_off[i] = static_cast<int32_t>(tile_off[blockIdx.x] + inc - x);
    if (i == V) point_off[V] = static_cast<int32_t>(*total);
}

// Path nodes of every leaf, root first. The leaves of a workgroup own one stretch of `points`: it is filled in
// LDS and written out in order where it fits (codes of up to 32 turns on average); storing each node of a leaf
// straight to memory, 4 bytes at a stride of a code length, took 303 us at V = 1M, this 34 us.
constexpr int kPointLeaves = 256;
constexpr int kPointStage = 32 * kPointLeaves;
__global__ __launch_bounds__(kPointLeaves) void k_huff_points(const uint32_t *__restrict__ up, int32_t V,
                                                              const uint8_t *__restrict__ codelen,
                                                              const int32_t *__restrict__ point_off,
                                                              const int64_t *__restrict__ total, int64_t cap,
                                                              const int32_t *__restrict__ flags,
                                                              int32_t *__restrict__ points) {
    __shared__ int32_t stage[kPointStage];
    if (*total > cap || flags[1] || flags[2] || flags[3]) return;   // the caller reports the error
    const int32_t v0 = blockIdx.x * kPointLeaves;
    const int32_t v = v0 + static_cast<int32_t>(threadIdx.x);
    const int32_t base = point_off[v0], n = point_off[min(V, v0 + kPointLeaves)] - base;
    const bool staged = n <= kPointStage;
    if (v < V) {
        const int32_t at = point_off[v], len = codelen[v];
        int32_t node = v;
        for (int32_t s = len - 1; s >= 0; --s) {
            const int32_t p = static_cast<int32_t>(up[node] >> 1);
            if (staged) stage[at - base + s] = p;
            else points[at + s] = p;
            node = V + p;
        }
    }
    if (!staged) return;
    __syncthreads();
    for (int32_t i = threadIdx.x; i < n; i += kPointLeaves) points[base + i] = stage[i];
}

__global__ void k_zero_i32(int32_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

}  // namespace

size_t huffman_workspace_bytes(int32_t V) {
    Carve c;
    c.take<uint32_t>(2 * static_cast<size_t>(V));  // up
    c.take<int64_t>(static_cast<size_t>(V));       // icount
    c.take<int32_t>(8);                            // flags and the merge's barrier counter
    c.take<int64_t>(2);                            // total
    c.take<int64_t>(static_cast<size_t>(ceil_div(V, kScanTile)));   // tile sums of the code-length scan
    return c.used();
}

int run_build_huffman(const int64_t *vocab_counts, int32_t V, uint8_t *codelen, uint64_t *code, int32_t *point_off,
                      int32_t *points, int64_t points_cap, int64_t *points_len_host, int32_t *max_len_host,
                      void *workspace, hipStream_t s) {
    Carve c(workspace);
    uint32_t *up = c.take<uint32_t>(2 * static_cast<size_t>(V));
    int64_t *icount = c.take<int64_t>(static_cast<size_t>(V));
    int32_t *flags = c.take<int32_t>(8);
    int64_t *total = c.take<int64_t>(2);
    const int32_t n_tiles = static_cast<int32_t>(ceil_div(V, kScanTile));
    int64_t *tile_sum = c.take<int64_t>(static_cast<size_t>(n_tiles));
    uint32_t *arrived = reinterpret_cast<uint32_t *>(flags + 4);
    const unsigned gv = static_cast<unsigned>(ceil_div(V, 256));
    k_zero_i32<<<1, 64, 0, s>>>(flags, 8);
    k_check_descending<<<gv, 256, 0, s>>>(vocab_counts, V, reinterpret_cast<uint2 *>(up), flags);
    W2V_LAUNCH_CHECK("k_check_descending");
    // a workgroup per chunk of the largest possible generation (all leaves and half as many nodes), at most one
    // per two compute units
    const unsigned groups = static_cast<unsigned>(
        std::max<int64_t>(1, std::min<int64_t>(ceil_div(V, kChunk), std::min(kMaxMergeGroups, device_cu_count() / 2))));
    void *args[] = {&vocab_counts, &V, &up, &icount, &flags, &arrived};
    W2V_HIP(hipLaunchCooperativeKernel(reinterpret_cast<const void *>(k_huff_merge), dim3(groups),
                                       dim3(kMergeThreads), args, 0, s));
    k_huff_codes<<<gv, 256, 0, s>>>(up, V, codelen, code, flags);
    W2V_LAUNCH_CHECK("k_huff_codes");
    k_scan_tiles<<<static_cast<unsigned>(n_tiles), kScanTile, 0, s>>>(codelen, V, tile_sum);
    k_scan_tile_sums<<<1, kScanTile, 0, s>>>(tile_sum, n_tiles, total);
    // one more thread than V writes point_off[V]
    k_scan_apply<<<static_cast<unsigned>(ceil_div(static_cast<int64_t>(V) + 1, kScanTile)), kScanTile, 0, s>>>(
        codelen, V, tile_sum, total, point_off);
    W2V_LAUNCH_CHECK("k_scan_codelen");
    if (points) {   // writes nothing where the tree failed or points_cap is too small
        k_huff_points<<<static_cast<unsigned>(ceil_div(V, kPointLeaves)), kPointLeaves, 0, s>>>(
            up, V, codelen, point_off, total, points_cap, flags, points);
        W2V_LAUNCH_CHECK("k_huff_points");
    }
    int32_t hflags[4];
    int64_t htotal = 0;
    W2V_HIP(hipMemcpyAsync(hflags, flags, sizeof(hflags), hipMemcpyDeviceToHost, s));
    W2V_HIP(hipMemcpyAsync(&htotal, total, sizeof(htotal), hipMemcpyDeviceToHost, s));
    W2V_HIP(hipStreamSynchronize(s));
    if (hflags[2]) return fail(W2V_E_ARG, "vocab_counts must be in descending order");
    if (hflags[1] | hflags[3]) return fail(W2V_E_RANGE, "a Huffman code is longer than 64 bits");
    *points_len_host = htotal;
    *max_len_host = hflags[0];
    if (points && points_cap < htotal)
        return fail(W2V_E_ARG, "points_cap " + std::to_string(points_cap) + " < points length " +
                                   std::to_string(htotal));
    return W2V_OK;
}

}  // namespace w2v
