// Deterministic synchronous training mode and the HS log-likelihood evaluator.
//
// Synchronous mode: every gradient of a batch of B consecutive kept centres is
// taken against the model as it stood at the start of the batch; the changes
// are summed exactly as int64 fixed point (value * 2^kFrac, integer atomics
// commute, so the sums do not depend on scheduling) and applied after the
// batch: row = row + (float)(sum * 2^-kFrac).
//
// Log-likelihood: sum over the sampler's pairs (v, w) of
// log P(v | syn0[w]) = sum_j log sigmoid((1 - 2 t_j) syn0[w] . syn1[n_j]);
// dot products in fp32, logarithms and all sums in fp64, in a fixed order.
// CBOW's objective: the same hierarchical softmax (§2) with the mean h of the
// window words' vectors as input, one term log P(v | h) per centre that has a
// window; h and its dot products in fp64.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "w2v_internal.h"
#include "w2v_scan.h"
#include "w2v_tiles.h"

namespace w2v {

constexpr int kFrac = 40;   // fixed-point fraction bits of the synchronous-mode sums

struct SyncArgs {
    const float *syn0;
    const float *syn1;
    int32_t V, dim, stride;
    const uint8_t *codelen;
    const uint64_t *code;
    const int32_t *point_off;
    const int32_t *points;
    const int32_t *kept_vid;
    const uint32_t *kept_meta;
    const int32_t *doc_kept;
    const int64_t *kept_off;   // exclusive prefix of doc_kept
    int64_t n_docs;
    int32_t doc_len;
    int64_t first_raw, epoch_base;
    const float *alpha_tab;
    int64_t blk0;
    int64_t c_lo;              // global kept index of this launch's first centre
    unsigned long long *d0;    // [V][dim] fixed-point deltas of syn0
    unsigned long long *d1;    // [V-1][dim] of syn1
    int32_t *flag0, *flag1;    // touched rows
    int32_t *list0, *list1;
    int32_t *cnt;              // [2] list lengths of this batch
    unsigned long long *stats; // kept, pairs, nodes
};

namespace {

__device__ __forceinline__ unsigned long long to_fixed(double v) {
    return static_cast<unsigned long long>(__double2ll_rn(ldexp(v, kFrac)));
}

__device__ __forceinline__ void touch(int32_t *flag, int32_t *list, int32_t *cnt, int32_t r) {
    if (atomicExch(&flag[r], 1) == 0) list[atomicAdd(cnt, 1)] = r;
}

// One workgroup per centre, its eight wavefronts sharing the path: wavefront w takes the nodes w, w+8, ... and
// walks them once for a group of GW window words, whose dot products are reduced four at a time. The fixed-point
// sums are exact in any order, so a node's change is summed over the group's words in registers, and a word's
// over all nodes in registers and LDS, before one atomic add each. What bounds a batch is the 64-bit adds to the
// rows its centres share and then the chain of a centre's loads, products and adds: one wavefront per centre
// with an add per pair, node and column on either side took 206 us for 256 centres (V = 30K, d = 100, window 5);
// this takes about 17 (an epoch of 305 such batches 7.6 instead of 64.8 ms; with four wavefronts 8.4, and with
// the words' sums added by each of four or eight wavefronts 10.4 and 15.0).
constexpr int kSyncWaves = 8;
template <int NE, int GW>
__global__ __launch_bounds__(kSyncWaves *kWave) void k_sync_grad(SyncArgs a) {
    __shared__ unsigned long long s_dx[GW][NE * kWave];   // the group's words' changes over all nodes
    const int lane = lane_id(), wid = static_cast<int>(threadIdx.x / kWave);
    const int64_t gi = a.c_lo + blockIdx.x;
    // document of kept centre gi: last d with kept_off[d] <= gi
    const int64_t d = wave_partition_point(0, static_cast<int32_t>(a.n_docs),
                                           [&](int32_t m) { return a.kept_off[m] <= gi; }) - 1;
    const int j = static_cast<int>(gi - a.kept_off[d]);
    const int nk = a.doc_kept[d];
    const int64_t base = d * a.doc_len;
    const uint32_t meta = a.kept_meta[base + j];
    const int v = a.kept_vid[base + j];
    const int eff = static_cast<int>(meta >> 16);
    const int clo = max(0, j - eff), chi = min(nk - 1, j + eff);
    const int P = chi - clo;
    const int len = a.codelen[v];
    if (threadIdx.x == 0) {
        atomicAdd(&a.stats[0], 1ull);
        atomicAdd(&a.stats[1], static_cast<unsigned long long>(P));
        atomicAdd(&a.stats[2], static_cast<unsigned long long>(P) * len);
    }
    if (P == 0) return;
    const int64_t g = a.epoch_base + a.first_raw + base + static_cast<int64_t>(meta & 0xFFFFu);
    const float alpha = a.alpha_tab[g / 10000 - a.blk0];
    const uint64_t code = a.code[v];
    const int my_pt = (lane < len) ? a.points[a.point_off[v] + lane] : 0;
    const int cq = clo + lane + ((clo + lane >= j) ? 1 : 0);
    const int my_w = (lane < P) ? a.kept_vid[base + cq] : 0;   // lane q: the q-th window word
    if (wid == 0 && lane < P) touch(a.flag0, a.list0, a.cnt, my_w);
    if (wid == 1 && lane < len) touch(a.flag1, a.list1, a.cnt + 1, my_pt);
    for (int p0 = 0; p0 < P; p0 += GW) {
        const int n_words = min(GW, P - p0);
        if (p0 > 0) __syncthreads();   // the group before is written out
        for (int i = threadIdx.x; i < n_words * NE * kWave; i += blockDim.x) (&s_dx[0][0])[i] = 0;
        __syncthreads();
        float x[GW][NE];
        long long dx[GW][NE];
#pragma unroll
        for (int p = 0; p < GW; ++p) {
            const int w = __builtin_amdgcn_readlane(my_w, min(p0 + p, kWave - 1));
            const bool in = p0 + p < P;
            buf_load_row<NE>(x[p], row_rsrc(const_cast<float *>(a.syn0), in ? w : 0, a.stride, in ? a.dim * 4 : 0), lane);
#pragma unroll
            for (int i = 0; i < NE; ++i) dx[p][i] = 0;
        }
        auto load_node = [&](float(&y)[NE], int jn) {   // zeros past the path's end
            const int n = __builtin_amdgcn_readlane(my_pt, min(jn, kWave - 1));
            buf_load_row<NE>(y, row_rsrc(const_cast<float *>(a.syn1), jn < len ? n : 0, a.stride,
                                         jn < len ? a.dim * 4 : 0), lane);
        };
        float next[NE];
        load_node(next, wid);
        for (int jn = wid; jn < len; jn += kSyncWaves) {
            const int n = __builtin_amdgcn_readlane(my_pt, min(jn, kWave - 1));
            const float t = static_cast<float>((code >> jn) & 1ull);
            float y[NE];
            long long dy[NE];
#pragma unroll
            for (int i = 0; i < NE; ++i) y[i] = next[i];
            load_node(next, jn + kSyncWaves);
#pragma unroll
            for (int i = 0; i < NE; ++i) dy[i] = 0;
#pragma unroll
            for (int c = 0; c < GW; c += 4) {
                if (p0 + c < P) {
                    const float z = reduce4(dot_partial<NE>(x[c], y), dot_partial<NE>(x[c + 1], y),
                                            dot_partial<NE>(x[c + 2], y), dot_partial<NE>(x[c + 3], y));
                    const float f = 1.0f / (1.0f + expf(-z));
                    const float gr = (1.0f - t - f) * alpha;   // lanes 16 r ..: window word p0 + c + r
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (p0 + c + r < P) {
                            const double gp = static_cast<double>(__builtin_bit_cast(
                                float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, gr), 16 * r)));
#pragma unroll
                            for (int i = 0; i < NE; ++i) {
                                dy[i] += static_cast<long long>(to_fixed(gp * static_cast<double>(x[c + r][i])));
                                dx[c + r][i] += static_cast<long long>(to_fixed(gp * static_cast<double>(y[i])));
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int col = lane + i * kWave;
                if (col < a.dim)
                    atomicAdd(&a.d1[static_cast<int64_t>(n) * a.dim + col], static_cast<unsigned long long>(dy[i]));
            }
        }
        if (wid < len) {
#pragma unroll
            for (int p = 0; p < GW; ++p)
                if (p < n_words)
#pragma unroll
                    for (int i = 0; i < NE; ++i)
                        atomicAdd(&s_dx[p][lane + i * kWave], static_cast<unsigned long long>(dx[p][i]));
        }
        __syncthreads();
        for (int p = wid; p < n_words; p += kSyncWaves) {
            const int w = __builtin_amdgcn_readlane(my_w, p0 + p);
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int col = lane + i * kWave;
                if (col < a.dim) atomicAdd(&a.d0[static_cast<int64_t>(w) * a.dim + col], s_dx[p][col]);
            }
        }
    }
}

// one wave per touched row of either matrix: row += (float)(delta 2^-40); clear delta and flag, and the other
// batch parity's list lengths, which the next batch fills
__global__ __launch_bounds__(256) void k_sync_apply(SyncArgs a, float *syn0, float *syn1, int32_t *next_cnt) {
    const int lane = lane_id();
    const int n0 = a.cnt[0], n = n0 + a.cnt[1];
    if (blockIdx.x == 0 && threadIdx.x < 2) next_cnt[threadIdx.x] = 0;
    const int nw = gridDim.x * blockDim.x / kWave;
    for (int k = (blockIdx.x * blockDim.x + threadIdx.x) / kWave; k < n; k += nw) {
        const bool words = k < n0;
        const int r = words ? a.list0[k] : a.list1[k - n0];
        unsigned long long *dl = (words ? a.d0 : a.d1) + static_cast<int64_t>(r) * a.dim;
        float *row = (words ? syn0 : syn1) + static_cast<int64_t>(r) * a.stride;
        for (int col = lane; col < a.dim; col += kWave) {
            const double dv = ldexp(static_cast<double>(static_cast<long long>(dl[col])), -kFrac);
            row[col] = row[col] + static_cast<float>(dv);
            dl[col] = 0ull;
        }
        if (lane == 0) (words ? a.flag0 : a.flag1)[r] = 0;
    }
}

__global__ void k_reset_counts(int32_t *cnt) {
    if (threadIdx.x < 4) cnt[threadIdx.x] = 0;
}

__global__ void k_zero_u64_range(unsigned long long *p, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0;
}
__global__ void k_zero_i32_range(int32_t *p, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0;
}

// exclusive scan of per-document kept counts (int32) into int64 offsets
__global__ __launch_bounds__(kScanThreads) void k_scan_kept(const int32_t *__restrict__ in, int64_t n,
                                                            int64_t *__restrict__ out) {
    block_exclusive_scan(in, n, out);
}

using SyncFn = void (*)(SyncArgs);
// window words taken together: a whole window of half-width 5 where its rows and their 64-bit sums fit the
// registers
SyncFn pick_sync(int dim) {
    const int ne = (dim + kWave - 1) / kWave;
    if (ne <= 1) return k_sync_grad<1, 12>;
    if (ne <= 2) return k_sync_grad<2, 12>;
    if (ne <= 4) return k_sync_grad<4, 8>;
    if (ne <= 5) return k_sync_grad<5, 8>;
    if (ne <= 8) return k_sync_grad<8, 4>;
    return k_sync_grad<16, 4>;
}

}  // namespace

size_t sync_extra_bytes(int32_t V, int32_t dim, int64_t n_docs) {
    Carve c;
    c.take<int64_t>(static_cast<size_t>(n_docs));                        // kept_off
    c.take<unsigned long long>(static_cast<size_t>(V) * dim);            // d0
    c.take<unsigned long long>(static_cast<size_t>(V) * dim);            // d1
    c.take<int32_t>(static_cast<size_t>(V) * 4);                         // flags, lists
    c.take<int32_t>(4);                                                  // list lengths of even and odd batches
    return c.used();
}

int run_train_sync(const w2v_model *m, const w2v_params *p, const SampleBufs &b, int64_t n_tokens, Carve &c,
                   const float *alpha_tab, int64_t blk0, unsigned long long *tstats, hipStream_t s) {
    const int64_t n_docs = std::max<int64_t>(1, ceil_div(n_tokens, p->doc_len));
    SyncArgs a{};
    a.syn0 = m->syn0;
    a.syn1 = m->syn1;
    a.V = m->V;
    a.dim = m->dim;
    a.stride = m->row_stride;
    a.codelen = m->codelen;
    a.code = m->code;
    a.point_off = m->point_off;
    a.points = m->points;
    a.kept_vid = b.kept_vid;
    a.kept_meta = b.kept_meta;
    a.doc_kept = b.doc_kept;
    int64_t *kept_off = c.take<int64_t>(static_cast<size_t>(n_docs));
    a.kept_off = kept_off;
    a.n_docs = ceil_div(n_tokens, p->doc_len);
    a.doc_len = p->doc_len;
    a.first_raw = p->first_raw_index;
    a.epoch_base = static_cast<int64_t>(p->epoch) * p->corpus_tokens;
    a.alpha_tab = alpha_tab;
    a.blk0 = blk0;
    a.d0 = c.take<unsigned long long>(static_cast<size_t>(m->V) * m->dim);
    a.d1 = c.take<unsigned long long>(static_cast<size_t>(m->V) * m->dim);
    int32_t *fl = c.take<int32_t>(static_cast<size_t>(m->V) * 4);
    a.flag0 = fl;
    a.flag1 = fl + m->V;
    a.list0 = fl + 2 * static_cast<size_t>(m->V);
    a.list1 = fl + 3 * static_cast<size_t>(m->V);
    int32_t *cnt = c.take<int32_t>(4);
    a.stats = tstats;
    const unsigned zg = static_cast<unsigned>(std::min<int64_t>(8192, ceil_div(static_cast<int64_t>(m->V) * m->dim, 256)));
    k_zero_u64_range<<<zg, 256, 0, s>>>(a.d0, static_cast<int64_t>(m->V) * m->dim);
    k_zero_u64_range<<<zg, 256, 0, s>>>(a.d1, static_cast<int64_t>(m->V) * m->dim);
    k_zero_i32_range<<<static_cast<unsigned>(ceil_div(2LL * m->V, 256)), 256, 0, s>>>(fl, 2LL * m->V);
    k_reset_counts<<<1, 64, 0, s>>>(cnt);
    if (n_tokens <= 0) return W2V_OK;
    k_scan_kept<<<1, kScanThreads, 0, s>>>(b.doc_kept, a.n_docs, kept_off);
    W2V_LAUNCH_CHECK("sync setup");
    int64_t tot[4];
    W2V_HIP(hipMemcpyAsync(tot, b.totals, sizeof(tot), hipMemcpyDeviceToHost, s));
    W2V_HIP(hipStreamSynchronize(s));
    const int64_t kept = tot[2];
    SyncFn fn = pick_sync(m->dim);
    const unsigned ag = static_cast<unsigned>(std::max(1, device_cu_count() * 4));
    int parity = 0;
    for (int64_t lo = 0; lo < kept; lo += p->sync_batch, parity ^= 1) {
        const int64_t hi = std::min<int64_t>(kept, lo + p->sync_batch);
        a.cnt = cnt + 2 * parity;
        for (a.c_lo = lo; a.c_lo < hi; a.c_lo += kMaxGroups)
            hipLaunchKernelGGL(fn, dim3(static_cast<unsigned>(std::min(hi - a.c_lo, kMaxGroups))),
                               dim3(kSyncWaves * kWave), 0, s, a);
        k_sync_apply<<<ag, 256, 0, s>>>(a, m->syn0, m->syn1, cnt + 2 * (parity ^ 1));
        W2V_LAUNCH_CHECK("sync batch");
    }
    return W2V_OK;
}

// ------------------------------------------------------------- log-likelihood
namespace {

// Held-out evaluation work units: kLLSeg consecutive kept centres of a document, one wavefront each.
// Short units keep the read-only walk's latency spread over many wavefronts (8: 4.2 ms for the 1e6-token
// held-out corpus at V = 1M, d = 300; the training kernel's 128-centre units: 8.4 ms).
constexpr int kLLSeg = 8;
inline int32_t ll_segs_per_doc(int32_t doc_len) { return static_cast<int32_t>(ceil_div(doc_len, kLLSeg)); }

struct LLArgs {
    const float *syn0;
    const float *syn1;
    int32_t dim, stride;
    const uint8_t *codelen;
    const uint64_t *code;
    const int32_t *point_off;
    const int32_t *points;
    const int32_t *kept_vid;
    const uint32_t *kept_meta;
    const int32_t *doc_kept;
    int64_t n_units;        // work units: kLLSeg consecutive kept centres of one document
    int32_t segs_per_doc;
    int32_t doc_len;
    double *unit_ll;
    int64_t *unit_nodes;
    int64_t *unit_terms;    // CBOW: centres with a window, per unit
};

// The centres of a work unit, one a lane, and the words around them.
constexpr int kLLReach = 10;   // the widest window
struct LLUnit {
    int64_t base;
    int nk, j0, n;   // kept words of the document, the unit's first centre and number of centres
    int eff, len, po, sid;   // lane c: half-width, path length and offset of centre j0 + c; lane l: word at j0 - kLLReach + l
    int code_lo, code_hi;
};

__device__ __forceinline__ LLUnit ll_unit(const LLArgs &a, int64_t u, int lane) {
    LLUnit r{};
    const int64_t d = u / a.segs_per_doc;
    r.nk = a.doc_kept[d];
    r.j0 = static_cast<int>(u - d * a.segs_per_doc) * kLLSeg;
    r.n = min(kLLSeg, r.nk - r.j0);
    r.base = d * a.doc_len;
    if (r.n <= 0) return r;
    const int pos = r.j0 - kLLReach + lane;
    r.sid = lane < kLLSeg + 2 * kLLReach && pos >= 0 && pos < r.nk ? a.kept_vid[r.base + pos] : 0;
    if (lane < r.n) {
        const int v = a.kept_vid[r.base + r.j0 + lane];
        r.eff = static_cast<int>(a.kept_meta[r.base + r.j0 + lane] >> 16);
        r.len = a.codelen[v];
        r.po = a.point_off[v];
        const uint64_t code = a.code[v];
        r.code_lo = static_cast<int>(code);
        r.code_hi = static_cast<int>(code >> 32);
    }
    return r;
}

// Centre c's path: lane l, its l-th node.
__device__ __forceinline__ int ll_path(const LLArgs &a, const LLUnit &r, int c, int lane) {
    const int len = __builtin_amdgcn_readlane(r.len, c);
    return lane < len ? a.points[__builtin_amdgcn_readlane(r.po, c) + lane] : 0;
}

__device__ __forceinline__ uint64_t ll_code(const LLUnit &r, int c) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(r.code_lo, c)) |
           static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(r.code_hi, c))) << 32;
}

// Sum of log sigmoids as one logarithm: log sigmoid(u) = min(u, 0) - log(1 + exp(-|u|)), and the logarithms of
// many factors in (1, 2] are the logarithm of their product (a lane takes at most 5 groups x 4 blocks of nodes x
// kLLSeg centres = 160 factors, so the product stays below 2^160). A factor's sum and its product each round, so a
// factor adds up to 2^-52 to the sum's absolute error (beside the exponential's own). Below 2^-10, where that would
// show beside the term itself, the term is summed directly, by five terms of its series (the terms left out are below
// 2^-52 of it). Measured against log1p in 80 bits (2e7 terms, 4e5 lanes of 160 factors): the series is off by up to
// 2.6e-16 of the term, the factors by up to 6.6e-15 in all and by 1.8e-15 of their sum.
struct LogSigmoidSum {
    double sum = 0.0, product = 1.0;
    __device__ __forceinline__ void add(double u, bool live) {
        const double e = exp(-fabs(u));
        const double series = e * fma(e, fma(e, fma(e, fma(e, 0.2, -0.25), 1.0 / 3.0), -0.5), 1.0);
        const bool small = e < 0x1p-10;
        sum += live ? fmin(u, 0.0) - (small ? series : 0.0) : 0.0;
        product *= live && !small ? 1.0 + e : 1.0;
    }
    __device__ __forceinline__ double total() const { return sum - log(product); }
};

// Columns c0 + 64 t + 4 (lane / 4) .. + 3 of the row that this lane's place in its quad takes, zeros past dim: four
// rows a load, in the form that mfma4 multiplies. The first FULL tiles lie within the row.
template <int FULL, int NE>
__device__ __forceinline__ void load_quad_rows(f4 (&r)[NE], const float *m, int stride, int dim, int c0, int row, int lane) {
    const float *p = m + static_cast<int64_t>(row) * stride;
#pragma unroll
    for (int t = 0; t < NE; ++t) {
        r[t] = *reinterpret_cast<const f4 *>(p + quad_column(FULL, c0, t, lane, dim));
        if (t >= FULL) {
            const int col = c0 + t * kWave + (lane >> 2) * 4;
#pragma unroll
            for (int i = 0; i < 4; ++i) r[t][i] = col + i < dim ? r[t][i] : 0.0f;
        }
    }
}

// One wavefront per work unit (a fixed assignment, so the sums are the same from run to run), in steps of one
// centre, up to 4 G of its window words and up to 32 of its nodes: four node rows at a time, the next four loaded
// meanwhile, their products with four words in 32 bits on the matrix cores; then lane 16 i + n holds word i's
// product with node n (and 16 + n), and all lanes take their log sigmoids in 64 bits at once, while the next
// step's window rows and first nodes are on their way. A row is read four columns a lane, four rows an
// instruction. Rows above 512 floats (PANELS) go in panels of 512 columns whose products are added.
// What bounds it is the latency of the rows: with a lane per column, vector dot products reduced across lanes and
// the log sigmoids of one word at a time (18 of 64 lanes) the 1e6-token held-out corpus took 3.97 ms at V = 1M,
// d = 300, this 2.05 ms (three
// wavefronts per SIMD, forced: two, without a spilled register, take 2.9 ms; twelve words a step 2.15).
template <int NE, int G, int FULL, bool PANELS = false>
__global__ __launch_bounds__(256, NE <= 5 ? 3 : 2) void k_loglik(LLArgs a) {
    const int lane = lane_id();
    const int64_t wave0 = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = static_cast<int64_t>(gridDim.x) * blockDim.x / kWave;
    const int row = lane >> 4;
    for (int64_t u = wave0; u < a.n_units; u += nwaves) {
        const LLUnit r = ll_unit(a, u, lane);
        LogSigmoidSum acc;
        int64_t nodes = 0;
        // the step: centre c, its path and code, the window's start and words, words g0 .., nodes n0 ..
        int c = -1, pt = 0, len = 0, clo = 0, P = 0, g0 = 0, n0 = 0;
        int pt_next = r.n > 0 ? ll_path(a, r, 0, lane) : 0;
        f4 x[G][NE], y[NE];
        auto next_step = [&]() {   // false after the last one
            if (n0 + 32 < len) {
                n0 += 32;
                return true;
            }
            n0 = 0;
            g0 += 4 * G;
            while (g0 >= P) {
                if (++c >= r.n) return false;
                const int eff = __builtin_amdgcn_readlane(r.eff, c);
                clo = max(0, r.j0 + c - eff);
                P = min(r.nk - 1, r.j0 + c + eff) - clo;
                len = __builtin_amdgcn_readlane(r.len, c);
                g0 = 0;
                pt = pt_next;
                pt_next = ll_path(a, r, min(c + 1, r.n - 1), lane);
                nodes += static_cast<int64_t>(P) * len;
            }
            return true;
        };
        auto load_words = [&](int c0) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (g0 + 4 * g < P) {
                    const int q = g0 + 4 * g + (lane & 3);   // past the window: any row
                    const int k = clo + q - r.j0 + kLLReach + (clo + q >= r.j0 + c ? 1 : 0);
                    const int w = __shfl(r.sid, k, kWave);
                    load_quad_rows<FULL>(x[g], a.syn0, a.stride, a.dim, c0, q < P ? w : 0, lane);
                }
            }
        };
        auto load_nodes = [&](f4(&to)[NE], int first, int c0) {
            const int n = first + (lane & 3);                // past the path: any row
            const int nd = __shfl(pt, min(n, kWave - 1), kWave);
            load_quad_rows<FULL>(to, a.syn1, a.stride, a.dim, c0, n < len ? nd : 0, lane);
        };
        bool more = next_step();
        if (more) {
            load_words(0);
            load_nodes(y, 0, 0);
        }
        while (more) {
            float z[G][2];
#pragma unroll
            for (int g = 0; g < G; ++g) z[g][0] = z[g][1] = 0.0f;
            const int end = min(len, n0 + 32), nx = min(4 * G, P - g0);
            for (int c0 = 0; c0 < (PANELS ? a.dim : 1); c0 += NE * kWave) {
                if (PANELS && c0 > 0) {
                    load_words(c0);
                    load_nodes(y, n0, c0);
                }
                for (int n = n0; n < end; n += 4) {
                    f4 yn[NE];
                    load_nodes(yn, n + 4, c0);
                    const int k = (n - n0) >> 2;
                    const bool here = ((lane >> 2) & 3) == (k & 3), low = k < 4;
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if (4 * g < nx) {
                            f4 d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                            for (int t = 0; t < NE; ++t)
#pragma unroll
                                for (int i = 0; i < 4; ++i) d = mfma4(x[g][t][i], y[t][i], d);
                            const float sum = block_sum(d);
                            z[g][0] += here && low ? sum : 0.0f;
                            z[g][1] += here && !low ? sum : 0.0f;
                        }
                    }
#pragma unroll
                    for (int t = 0; t < NE; ++t) y[t] = yn[t];
                }
            }
            const uint64_t code = ll_code(r, c);
            const int first = n0, to = end;
            more = next_step();
            if (more) {
                load_words(0);
                load_nodes(y, n0, 0);
            }
            // (one group of words and sixteen nodes after another: the 64-bit work of all of them at once would
            // take a third of the registers)
#pragma unroll 1
            for (int half = 0; half < 2 && first + 16 * half < to; ++half) {
                const int n = first + 16 * half + (lane & 15);
                const bool minus = (code >> min(n, 63)) & 1ull;
#pragma unroll 1
                for (int g = 0; 4 * g < nx; ++g) {
                    float zg = half ? z[0][1] : z[0][0];
#pragma unroll
                    for (int k = 1; k < G; ++k) zg = g == k ? (half ? z[k][1] : z[k][0]) : zg;
                    acc.add(static_cast<double>(minus ? -zg : zg), n < to && 4 * g + row < nx);
                }
            }
        }
        const double sum = wave_sum(acc.total());
        if (lane == 0) {
            a.unit_ll[u] = sum;
            a.unit_nodes[u] = nodes;
        }
    }
}

// CBOW: one wavefront per work unit; per centre with a window, h = (sum of the window rows in ascending window
// order, fp64) / P, then one walk of the centre's path with fp64 dot products, four nodes at a time (up to 512 floats
// the next four rows loaded meanwhile: wider ones have no registers for them) and reduced together; lane 16 r + k
// keeps node 4 k + r. Node after node, each with a sum over the wavefront of its own, it took 2.11 ms for the
// 1e6-token held-out corpus at V = 100K, d = 300, this 1.2 (four wavefronts per SIMD; 1.7 with three). Window words
// four at a time pay for the words that a window does not have (1.3 ms; V = 100: 495 instead of 400 us for 3e5 tokens);
// above 512 floats the next nodes' rows and two wavefronts per SIMD took 1.57 ms for 3e5 tokens at d = 600, this 0.79.
template <int NE>
__global__ __launch_bounds__(256, NE <= 5 ? 4 : 3) void k_loglik_cbow(LLArgs a) {
    constexpr bool kAhead = NE <= 8;
    const int lane = lane_id();
    const int64_t wave0 = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = static_cast<int64_t>(gridDim.x) * blockDim.x / kWave;
    auto load = [&](float(&to)[NE], const float *m, int row, bool in) {
        buf_load_row<NE>(to, row_rsrc(const_cast<float *>(m), in ? row : 0, a.stride, in ? a.dim * 4 : 0), lane);
    };
    for (int64_t u = wave0; u < a.n_units; u += nwaves) {
        const LLUnit r = ll_unit(a, u, lane);
        LogSigmoidSum acc;
        int64_t nodes = 0, terms = 0;
        int pt_next = r.n > 0 ? ll_path(a, r, 0, lane) : 0;
        for (int c = 0; c < r.n; ++c) {
            const int j = r.j0 + c;
            const int eff = __builtin_amdgcn_readlane(r.eff, c), len = __builtin_amdgcn_readlane(r.len, c);
            const uint64_t code = ll_code(r, c);
            const int my_pt = pt_next;
            pt_next = ll_path(a, r, min(c + 1, r.n - 1), lane);
            const int clo = max(0, j - eff), chi = min(r.nk - 1, j + eff);
            const int P = chi - clo;
            if (P == 0) continue;
            float y[4][NE], yn[4][NE];
            auto load_nodes = [&](float(&to)[4][NE], int n0) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    load(to[i], a.syn1, __builtin_amdgcn_readlane(my_pt, min(n0 + i, kWave - 1)), n0 + i < len);
            };
            if (kAhead) load_nodes(y, 0);
            double h[NE];
#pragma unroll
            for (int i = 0; i < NE; ++i) h[i] = 0.0;
            for (int q = 0; q < P; ++q) {
                const int pos = clo + q + (clo + q >= j ? 1 : 0);
                float x[NE];
                load(x, a.syn0, __builtin_amdgcn_readlane(r.sid, pos - r.j0 + kLLReach), true);
#pragma unroll
                for (int i = 0; i < NE; ++i) h[i] += static_cast<double>(x[i]);
            }
#pragma unroll
            for (int i = 0; i < NE; ++i) h[i] = h[i] / static_cast<double>(P);
            double mine = 0.0;
            for (int n0 = 0; n0 < len; n0 += 4) {
                load_nodes(kAhead ? yn : y, kAhead ? n0 + 4 : n0);
                double z[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int i = 0; i < NE; ++i)
#pragma unroll
                    for (int k = 0; k < 4; ++k) z[k] += h[i] * static_cast<double>(y[k][i]);
                const double s = reduce4(z[0], z[1], z[2], z[3]);
                mine = (lane & 15) == (n0 >> 2) ? s : mine;
                if (kAhead) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
#pragma unroll
                        for (int i = 0; i < NE; ++i) y[k][i] = yn[k][i];
                }
            }
            const int n = 4 * (lane & 15) + (lane >> 4);
            acc.add(((code >> n) & 1ull) ? -mine : mine, n < len);
            nodes += len;
            terms += 1;
        }
        const double sum = wave_sum(acc.total());
        if (lane == 0) {
            a.unit_ll[u] = sum;
            a.unit_nodes[u] = nodes;
            a.unit_terms[u] = terms;
        }
    }
}

// Fixed-order sum of the work units' partials (terms: optional) in two passes: each workgroup adds the units of
// its stretch, in place (its first unit takes the sum), then one workgroup adds the stretches (at most one a
// thread). One workgroup over all units took 58 us for 125,000.
constexpr int kSumThreads = 1024;
__device__ __forceinline__ void block_sum3(double &a, int64_t &b, int64_t &t) {
    __shared__ double sl[kSumThreads];
    __shared__ int64_t sn[kSumThreads];
    __shared__ int64_t st_[kSumThreads];
    sl[threadIdx.x] = a;
    sn[threadIdx.x] = b;
    st_[threadIdx.x] = t;
    __syncthreads();
    for (int st = kSumThreads / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st) {
            sl[threadIdx.x] += sl[threadIdx.x + st];
            sn[threadIdx.x] += sn[threadIdx.x + st];
            st_[threadIdx.x] += st_[threadIdx.x + st];
        }
        __syncthreads();
    }
    a = sl[0];
    b = sn[0];
    t = st_[0];
}

__global__ __launch_bounds__(kSumThreads) void k_sum_units(double *ll, int64_t *nodes, int64_t *terms, int64_t n,
                                                           int64_t stretch) {
    const int64_t lo = blockIdx.x * stretch, hi = min(n, lo + stretch);
    double a = 0.0;
    int64_t b = 0, t = 0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += kSumThreads) {
        a += ll[i];
        b += nodes[i];
        if (terms) t += terms[i];
    }
    block_sum3(a, b, t);
    if (threadIdx.x == 0) {
        ll[lo] = a;
        nodes[lo] = b;
        if (terms) terms[lo] = t;
    }
}

__global__ __launch_bounds__(kSumThreads) void k_sum_stretches(const double *__restrict__ ll,
                                                               const int64_t *__restrict__ nodes,
                                                               const int64_t *__restrict__ terms, int64_t n,
                                                               int64_t stretch, double *__restrict__ out_ll,
                                                               int64_t *__restrict__ out_nodes,
                                                               int64_t *__restrict__ out_terms) {
    const int64_t i = threadIdx.x * stretch;
    double a = i < n ? ll[i] : 0.0;
    int64_t b = i < n ? nodes[i] : 0, t = terms && i < n ? terms[i] : 0;
    block_sum3(a, b, t);
    if (threadIdx.x == 0) {
        *out_ll = a;
        *out_nodes = b;
        *out_terms = t;
    }
}

using LLFn = void (*)(LLArgs);
// 4 groups of window words per step: all of a window of half-width 5 for rows of up to 128 floats, eight words above.
template <int I>
constexpr LLFn ll_variant() {
    constexpr LoglikTiles t = kLoglikTiles[I];
    return k_loglik<t.tiles, t.groups, t.full, t.panels>;
}
LLFn pick_ll(int dim) {
    constexpr LLFn fns[] = {ll_variant<0>(), ll_variant<1>(), ll_variant<2>(),
                            ll_variant<3>(), ll_variant<4>(), ll_variant<5>()};
    int i = 0;
    while (dim > kLoglikTiles[i].columns) ++i;   // dim <= 1024
    return fns[i];
}

LLFn pick_ll_cbow(int dim) {
    const int ne = (dim + kWave - 1) / kWave;
    if (ne <= 1) return k_loglik_cbow<1>;
    if (ne <= 2) return k_loglik_cbow<2>;
    if (ne <= 4) return k_loglik_cbow<4>;
    if (ne <= 5) return k_loglik_cbow<5>;
    if (ne <= 8) return k_loglik_cbow<8>;
    return k_loglik_cbow<16>;
}

}  // namespace

int64_t loglik_units(int64_t n_tokens, int32_t doc_len) {
    return std::max<int64_t>(1, ceil_div(n_tokens, doc_len)) * ll_segs_per_doc(doc_len);
}

size_t loglik_extra_bytes(int64_t n_units) {
    Carve c;
    c.take<double>(static_cast<size_t>(n_units));
    c.take<int64_t>(static_cast<size_t>(n_units));
    c.take<int64_t>(static_cast<size_t>(n_units));
    c.take<double>(1);
    c.take<int64_t>(2);
    return c.used();
}

int run_loglik(const w2v_model *m, const w2v_params *p, const SampleBufs &b, int64_t n_tokens, Carve &c,
               double *sum_ll_host, int64_t *n_pairs_host, int64_t *n_nodes_host, hipStream_t s) {
    const int64_t n_units = loglik_units(n_tokens, p->doc_len);
    LLArgs a{};
    a.syn0 = m->syn0;
    a.syn1 = m->syn1;
    a.dim = m->dim;
    a.stride = m->row_stride;
    a.codelen = m->codelen;
    a.code = m->code;
    a.point_off = m->point_off;
    a.points = m->points;
    a.kept_vid = b.kept_vid;
    a.kept_meta = b.kept_meta;
    a.doc_kept = b.doc_kept;
    a.segs_per_doc = ll_segs_per_doc(p->doc_len);
    a.n_units = n_tokens > 0 ? ceil_div(n_tokens, p->doc_len) * a.segs_per_doc : 0;
    a.doc_len = p->doc_len;
    a.unit_ll = c.take<double>(static_cast<size_t>(n_units));
    a.unit_nodes = c.take<int64_t>(static_cast<size_t>(n_units));
    a.unit_terms = c.take<int64_t>(static_cast<size_t>(n_units));
    double *out = c.take<double>(1);
    int64_t *out_nt = c.take<int64_t>(2);   // nodes, terms
    const bool cbow = p->arch == 1;
    if (a.n_units > 0) {
        // one unit per wavefront: the hardware hands out workgroups as others finish, which balances the
        // uneven units (a document's kept centres end in a partial unit, and units past them are empty)
        const unsigned grid = static_cast<unsigned>(std::min(ceil_div(a.n_units, 4), kMaxGroups));
        hipLaunchKernelGGL(cbow ? pick_ll_cbow(m->dim) : pick_ll(m->dim), dim3(grid), dim3(256), 0, s, a);
        W2V_LAUNCH_CHECK("k_loglik");
        int64_t *terms = cbow ? a.unit_terms : nullptr;
        const int64_t stretch = std::max<int64_t>(kSumThreads, ceil_div(a.n_units, kSumThreads));
        k_sum_units<<<static_cast<unsigned>(ceil_div(a.n_units, stretch)), kSumThreads, 0, s>>>(
            a.unit_ll, a.unit_nodes, terms, a.n_units, stretch);
        k_sum_stretches<<<1, kSumThreads, 0, s>>>(a.unit_ll, a.unit_nodes, terms, a.n_units, stretch, out, out_nt,
                                                  out_nt + 1);
        W2V_LAUNCH_CHECK("k_sum_units");
    }
    double hll = 0.0;
    int64_t nt[2] = {0, 0};
    int64_t tot[4] = {0, 0, 0, 0};
    if (a.n_units > 0) {
        W2V_HIP(hipMemcpyAsync(&hll, out, sizeof(hll), hipMemcpyDeviceToHost, s));
        W2V_HIP(hipMemcpyAsync(nt, out_nt, sizeof(nt), hipMemcpyDeviceToHost, s));
    }
    W2V_HIP(hipMemcpyAsync(tot, b.totals, sizeof(tot), hipMemcpyDeviceToHost, s));
    W2V_HIP(hipStreamSynchronize(s));
    const int64_t nn = nt[0];
    *sum_ll_host = hll;
    *n_pairs_host = cbow ? nt[1] : tot[3];
    if (n_nodes_host) *n_nodes_host = nn;
    return W2V_OK;
}

}  // namespace w2v
