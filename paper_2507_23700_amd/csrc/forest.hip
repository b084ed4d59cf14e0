// Forest queries: B batches of queries, batch b = queries [boff[b], boff[b+1])
// searched in tree btree[b] of a forest (radius btree-specific for reductions).
//
// 1. ordering: each query gets the key (batch << mbits) | Hilbert code of the
//    query inside its target tree's box, and one radix sort orders all
//    queries by batch, then along the curve inside the batch;
// 2. one launch over the sorted queries of all batches, each lane answering
//    one query (or a few neighbours) against its batch's tree, which the
//    sorted key names.  Workgroups are dealt to the XCDs in contiguous runs
//    (xcd_block), so each XCD's L2 holds few trees.
// Bound: as the walks of single trees (traverse_codes, knn_search_codes).  For
// 512 batches of 6.5*10^6 queries in all on 32 trees of 9.4*10^6 points, against a
// persistent grid over float nodes that took 256 sorted queries at a time from
// an atomic counter, spread every tree over all eight L2 caches and searched
// each query's batch: k = 8 3.8 -> 3.0 ms, count with distances 2.7 -> 1.65.
// The query path allocates nothing once the forest's workspace is reserved, and
// never synchronises, so it can be captured in a hipGraph.  Results use indices
// local to the target tree (value index minus the tree's first value), the
// same as querying that tree built on its own.
#include <algorithm>

#include "device_util.hpp"
#include "geometry.hpp"
#include "internal.hpp"
#include "profile.hpp"
#include "traverse.hpp"

namespace ax {
namespace {

constexpr int kForestBlock = 256;

__device__ __forceinline__ int batch_of(const int64_t *__restrict__ boff, int B, int64_t i)
{
    int lo = 0, hi = B;  // last b with boff[b] <= i
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (boff[mid] <= i)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Batches are contiguous, so a workgroup finds the batch of its first query by
// a search and the others step on from there.
template <int D, typename K>
__global__ __launch_bounds__(kForestBlock) void k_forest_codes(const float *__restrict__ q, int64_t m,
                                                               const int64_t *__restrict__ boff, int B,
                                                               const int32_t *__restrict__ btree, int T,
                                                               const TreeHeader *__restrict__ hdrs, int mbits,
                                                               K *__restrict__ codes, uint32_t *__restrict__ ids)
{
    __shared__ int s_first;
    const int bits = mbits / D;
    const int64_t base = (int64_t)blockIdx.x * kForestBlock;
    if (threadIdx.x == 0)
        s_first = batch_of(boff, B, base);
    __syncthreads();
    const int64_t i = base + threadIdx.x;
    if (i >= m)
        return;
    int b = s_first;
    for (int step = 0; step < 8 && b + 1 < B && boff[b + 1] <= i; ++step)
        ++b;
    if (b + 1 < B && boff[b + 1] <= i)  // many small batches
        b = batch_of(boff, B, i);
    const int t = btree[b];
    uint32_t c[D];
    if (t >= 0 && t < T && hdrs[t].n > 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const float lo = hdrs[t].lo[d], ext = hdrs[t].hi[d] - lo;
            c[d] = quantise(q[i * D + d], lo, ext > 0.0f ? 1.0f / ext : 0.0f, bits);
        }
    } else {
#pragma unroll
        for (int d = 0; d < D; ++d)
            c[d] = 0;
    }
    const K code = mbits <= 32 ? (K)hilbert_code<D>(c, bits) : (K)interleave<D>(c, bits);
    codes[i] = ((K)b << mbits) | code;
    ids[i] = (uint32_t)i;
}

// The sorted queries of a call: the permutation, and the keys it was sorted by,
// whose bits from mbits up are the batch.
struct ForestOrder {
    const uint32_t *perm;
    const void *keys;
    bool wide;  // 64-bit keys
    int mbits;
    __device__ __forceinline__ int batch(int64_t t) const
    {
        return wide ? (int)(static_cast<const uint64_t *>(keys)[t] >> mbits)
                    : (int)(static_cast<const uint32_t *>(keys)[t] >> mbits);
    }
};

// One thread takes NQ consecutive sorted positions, which usually share a batch
// and tree and are walked together; ones that straddle trees are walked one at
// a time.  FMT: 0 float nodes, 1 quantized, 2 four-wide (the last two with the
// walks of single trees; NQ up to 2 and 1).
template <int D, bool SUMDIST, int NQ, int FMT>
__global__ __launch_bounds__(kForestBlock) void k_forest_reduce(
    const Node<D> *__restrict__ nodes, const QNode<D> *__restrict__ qnodes, const Node4<D> *__restrict__ wnodes,
    const float *__restrict__ leaves, int kind, int n_nodes, const TreeHeader *__restrict__ hdrs, int T,
    const float *__restrict__ queries, int64_t m, ForestOrder order, int B, const int32_t *__restrict__ btree,
    const float *__restrict__ bradius, float scale, int32_t *__restrict__ counts, int64_t *__restrict__ sums,
    int stack_cap)
{
    extern __shared__ int s_stack[];
    const int64_t t0 = (xcd_block() * blockDim.x + threadIdx.x) * NQ;
    if (t0 >= m)
        return;
    int spill[kSpill];
    int64_t qi[NQ];
    int tr[NQ];
    Sphere<D> pred[NQ];
    bool same = true;
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
        qi[j] = t0 + j < m ? (int64_t)order.perm[t0 + j] : -1;
        tr[j] = -1;
        if (qi[j] >= 0 && qi[j] < m) {
            const int b = order.batch(t0 + j);
            if (b >= 0 && b < B) {
                tr[j] = btree[b] >= 0 && btree[b] < T ? btree[b] : -1;
                const float r = bradius[b];
                pred[j].load(queries, qi[j], r * r);
            } else {
                pred[j].dead();
            }
        } else {
            qi[j] = -1;
            pred[j].dead();
        }
        if (qi[j] >= 0 && tr[j] != tr[0])
            same = false;
    }
    int c[NQ];
    long long s[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
        c[j] = 0;
        s[j] = 0;
    }
    auto one = [&](const TreeHeader &h, const Sphere<D> &p, auto &f) {
        ShortStack<int> st(s_stack + threadIdx.x, blockDim.x, stack_cap, spill);
        if (FMT == 1)
            walk_quantized<D>(nodes, qnodes, h, n_nodes, leaves, kind, p, s_stack, stack_cap, spill, f);
        else if (FMT == 2)
            traverse_spatial4<D>(wnodes, h.root, n_nodes, p, st, f);
        else
            traverse_spatial<D>(nodes, h.root, n_nodes, p, st, f);
    };
    if (NQ > 1 && same && tr[0] >= 0) {
        auto f = [&](int j, int, float d2) {
#pragma unroll
            for (int jj = 0; jj < NQ; ++jj)
                if (jj == j) {
                    ++c[jj];
                    if (SUMDIST)
                        s[jj] += fixed_term(d2, scale);
                }
        };
        if (FMT == 1) {
            walk_quantized_packet<D, NQ>(nodes, qnodes, hdrs[tr[0]], n_nodes, leaves, kind, pred, s_stack, stack_cap,
                                         spill, f);
        } else {
            ShortStack<int> st(s_stack + threadIdx.x, blockDim.x, stack_cap, spill);
            traverse_spatial_packet<D, NQ>(nodes, hdrs[tr[0]].root, n_nodes, pred, st, f);
        }
    } else {
#pragma unroll
        for (int j = 0; j < NQ; ++j)
            if (qi[j] >= 0 && tr[j] >= 0) {
                auto f = [&](int, float d2) {
                    ++c[j];
                    if (SUMDIST)
                        s[j] += fixed_term(d2, scale);
                };
                one(hdrs[tr[j]], pred[j], f);
            }
    }
#pragma unroll
    for (int j = 0; j < NQ; ++j)
        if (qi[j] >= 0) {
            counts[qi[j]] = c[j];
            if (SUMDIST)
                sums[qi[j]] = s[j];
        }
}

template <int D, int K, int FMT>
__global__ __launch_bounds__(kForestBlock) void k_forest_knn(
    const Node<D> *__restrict__ nodes, const QNode<D> *__restrict__ qnodes, const Node4<D> *__restrict__ wnodes,
    int n_nodes, const float *__restrict__ leaves, int kind, const TreeHeader *__restrict__ hdrs, int T,
    const float *__restrict__ queries, int64_t m, ForestOrder order, int B, const int32_t *__restrict__ btree,
    int k_out, float *__restrict__ out_d2, int32_t *__restrict__ out_idx, int stack_cap, int seed,
    const uint64_t *__restrict__ keys, int mbits)
{
    extern __shared__ int s_stack[];
    const int64_t t = xcd_block() * blockDim.x + threadIdx.x;
    if (t >= m)
        return;
    const int64_t qi = order.perm[t];
    if (qi < 0 || qi >= m)
        return;
    KnnEntry spill[kSpill];
    const int b = order.batch(t);
    const int tr = b >= 0 && b < B ? btree[b] : -1;
    TopK<K> best;
    best.reset(INFINITY);
    int start = 0;
    if (tr >= 0 && tr < T) {
        const TreeHeader &h = hdrs[tr];
        start = h.start;
        float q[D];
#pragma unroll
        for (int d = 0; d < D; ++d)
            q[d] = queries[qi * D + d];
        ShortStack<KnnEntry> st(reinterpret_cast<KnnEntry *>(s_stack) + threadIdx.x, blockDim.x, stack_cap, spill);
        // the seed searches this tree's segment of the forest's sorted build keys
        const SeedKeys sk{keys, (uint64_t)tr << mbits, mbits / D};
        if (FMT == 1 && kind != ARBORX_BOXES && codes_serve(h)) {
            TopStack<KnnCode> ts(reinterpret_cast<KnnCode *>(s_stack) + threadIdx.x, blockDim.x, stack_cap,
                                 reinterpret_cast<KnnCode *>(spill), knn_code(-1, 0u));
            knn_search_codes<D, K>(qnodes, n_nodes, leaves, kind, h, q, best, ts, seed, sk);
        } else if (FMT == 1 && kind == ARBORX_BOXES)
            knn_search_q<D, K>(qnodes, n_nodes, leaves, h, q, best, st, seed, sk);
        else if (FMT == 2)
            knn_search4<D, K>(nodes, wnodes, n_nodes, leaves, kind, h, q, best, st, seed, sk);
        else
            knn_search<D, K>(nodes, n_nodes, leaves, kind, h, q, best, st, seed, sk);
    }
    best.store(k_out, out_d2 + qi * k_out, out_idx + qi * k_out, start);  // indices local to the tree
}

// Workspace layout for m queries:
//   codes[2][m] (K), ids[2][m] (u32), radix workspace.
template <typename K>
size_t forest_ws_bytes(int64_t m)
{
    const int64_t mm = m > 0 ? m : 1;
    return 2 * mm * sizeof(K) + 2 * mm * sizeof(uint32_t) + radix_workspace_bytes(mm) + 1024;
}

arborx_status reserve_ws(ForestDev &f, int64_t m, hipStream_t s)
{
    const size_t need = std::max(forest_ws_bytes<uint64_t>(m), forest_ws_bytes<uint32_t>(m));
    if (f.ws_bytes >= need)
        return ARBORX_OK;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
        return fail(ARBORX_E_NOMEM, "forest workspace too small during graph capture: call arborx_forest_reserve first");
    if (f.ws)
        dfree(f.ws, s);
    f.ws = nullptr;
    f.ws_bytes = 0;
    arborx_status st = dalloc(&f.ws, need, s);
    if (st == ARBORX_OK)
        f.ws_bytes = need;
    return st;
}

// Sorted order of the queries (by batch, then along the curve inside it).
template <int D, typename K>
arborx_status forest_order_keys(const ForestDev &f, const float *q, int64_t m, const int64_t *boff, int B,
                                const int32_t *btree, int bb, ForestOrder *order, hipStream_t s)
{
    const int64_t mm = m > 0 ? m : 1;
    uint8_t *p = static_cast<uint8_t *>(f.ws);
    K *codes = reinterpret_cast<K *>(p);
    K *codes2 = codes + mm;
    uint32_t *ids = reinterpret_cast<uint32_t *>(codes2 + mm);
    uint32_t *ids2 = ids + mm;
    uint8_t *rws = reinterpret_cast<uint8_t *>(ids2 + mm);
    rws = reinterpret_cast<uint8_t *>((reinterpret_cast<uintptr_t>(rws) + 255) & ~uintptr_t(255));
    const int kbits = (int)sizeof(K) * 8 - (sizeof(K) == 8 ? 1 : 0);
    int mbits = (kbits - bb) / D * D;
    if (mbits > 8 * D)
        mbits = 8 * D;  // 8 bits per dimension order the queries of one batch well enough
    ProfScope ps("forest_order", s);
    k_forest_codes<D, K><<<grid_for(m, kForestBlock, INT32_MAX), kForestBlock, 0, s>>>(q, m, boff, B, btree, f.T, f.hdrs,
                                                                                       mbits, codes, ids);
    bool alt = false;
    AX_HIP(radix_sort_pairs<K>(codes, ids, codes2, ids2, m, 0, mbits + bb, rws, s, &alt));
    *order = ForestOrder{alt ? ids2 : ids, alt ? codes2 : codes, sizeof(K) == 8, mbits};
    return ARBORX_OK;
}

template <int D>
arborx_status forest_order(const ForestDev &f, const float *q, int64_t m, const int64_t *boff, int B,
                           const int32_t *btree, ForestOrder *order, hipStream_t s)
{
    int bb = 1;
    while ((1 << bb) < B)
        ++bb;
    return bb <= 20 ? forest_order_keys<D, uint32_t>(f, q, m, boff, B, btree, bb, order, s)
                    : forest_order_keys<D, uint64_t>(f, q, m, boff, B, btree, bb, order, s);
}

template <int D>
arborx_status forest_reduce_impl(ForestDev &f, const float *q, int64_t m, const int64_t *boff, const int32_t *btree,
                                 const float *brad, int B, int op, int scale_bits, int32_t *counts, int64_t *sums,
                                 hipStream_t s)
{
    ForestOrder order;
    arborx_status st = forest_order<D>(f, q, m, boff, B, btree, &order, s);
    if (st != ARBORX_OK)
        return st;
    const Tuning &tu = tuning(OP_REDUCE);
    int block_unused = 0, cap = 0;
    launch_shape(OP_REDUCE, D, block_unused, cap);
    while (cap > 1 && (size_t)cap * kForestBlock * sizeof(int) > 65536)
        cap >>= 1;
    const size_t lds = (size_t)(cap > 2 ? cap : 2) * kForestBlock * sizeof(int);  // a TopStack has at least two slots
    const float scale = ldexpf(1.0f, scale_bits);
    ProfScope ps(op == ARBORX_COUNT_SUMDIST ? "forest_reduce_sumdist" : "forest_reduce_count", s);
    const Node<D> *nodes = static_cast<const Node<D> *>(f.nodes);
    const QNode<D> *qnodes = static_cast<const QNode<D> *>(f.qnodes);
    const Node4<D> *wnodes = static_cast<const Node4<D> *>(f.wnodes);
    const int nn = (int)(f.n > 0 ? f.n : 1);
    const int fmt = forest_format(OP_REDUCE, f);
    // as for single trees: up to 3D 4 queries a thread on float nodes; 1 on quantized ones
    int nq = tu.packet ? tu.packet : (D <= 3 && fmt != 1 ? 4 : 1);
    if (fmt == 2)
        nq = 1;
    else if (fmt == 1 && nq > 2)
        nq = 2;
#define AX_FR(SD, N, F)                                                                                          \
    k_forest_reduce<D, SD, N, F><<<grid_for((m + N - 1) / N, kForestBlock, INT32_MAX), kForestBlock, lds, s>>>(  \
        nodes, qnodes, wnodes, f.leaves, f.kind, nn, f.hdrs, f.T, q, m, order, B, btree, brad, scale, counts,    \
        sums, cap)
#define AX_FR_NODES(SD)           \
    do {                          \
        if (fmt == 2)             \
            AX_FR(SD, 1, 2);      \
        else if (fmt == 1) {      \
            if (nq == 2)          \
                AX_FR(SD, 2, 1);  \
            else                  \
                AX_FR(SD, 1, 1);  \
        } else if (nq == 4)       \
            AX_FR(SD, 4, 0);      \
        else if (nq == 2)         \
            AX_FR(SD, 2, 0);      \
        else                      \
            AX_FR(SD, 1, 0);      \
    } while (0)
    if (op == ARBORX_COUNT_SUMDIST)
        AX_FR_NODES(true);
    else
        AX_FR_NODES(false);
#undef AX_FR_NODES
#undef AX_FR
    AX_HIP(hipGetLastError());
    return ARBORX_OK;
}

template <int D, int K>
arborx_status forest_knn_launch(ForestDev &f, const float *q, int64_t m, const int64_t *boff, const int32_t *btree,
                                int B, int k, float *d2, int32_t *idx, hipStream_t s)
{
    ForestOrder order;
    if (boff) {
        const arborx_status st = forest_order<D>(f, q, m, boff, B, btree, &order, s);
        if (st != ARBORX_OK)
            return st;
    } else {  // the forest's own values: its build sorted them by tree and curve
        order = ForestOrder{f.ids, f.keys, true, f.mbits};
    }
    const Tuning &tu = tuning(OP_KNN);
    const int fmt = forest_format(OP_KNN, f);
    int block = 0, cap = 0;
    launch_shape(OP_KNN, D, block, cap);
    if (block > kForestBlock)
        block = kForestBlock;
    while (cap > 1 && (size_t)cap * block * sizeof(KnnEntry) > 65536)
        cap >>= 1;
    const size_t lds = (size_t)(cap > 2 ? cap : 2) * block * sizeof(KnnEntry);
    ProfScope ps("forest_knn", s);
#define AX_FKNN(F)                                                                                                  \
    k_forest_knn<D, K, F><<<grid_for(m, block, INT32_MAX), block, lds, s>>>(                                        \
        static_cast<const Node<D> *>(f.nodes), static_cast<const QNode<D> *>(f.qnodes),                             \
        static_cast<const Node4<D> *>(f.wnodes), (int)(f.n > 0 ? f.n : 1), f.leaves, f.kind, f.hdrs, f.T, q, m,     \
        order, B, btree, k, d2, idx, cap, tu.seed, f.keys, f.mbits)
    if (fmt == 1)
        AX_FKNN(1);
    else if (fmt == 2)
        AX_FKNN(2);
    else
        AX_FKNN(0);
#undef AX_FKNN
    AX_HIP(hipGetLastError());
    return ARBORX_OK;
}

template <int D>
arborx_status forest_knn_impl(ForestDev &f, const float *q, int64_t m, const int64_t *boff, const int32_t *btree,
                              int B, int k, float *d2, int32_t *idx, hipStream_t s)
{
    if (k <= 1)
        return forest_knn_launch<D, 1>(f, q, m, boff, btree, B, k, d2, idx, s);
    if (k <= 4)
        return forest_knn_launch<D, 4>(f, q, m, boff, btree, B, k, d2, idx, s);
    if (k <= 8)
        return forest_knn_launch<D, 8>(f, q, m, boff, btree, B, k, d2, idx, s);
    if (k <= 16)
        return forest_knn_launch<D, 16>(f, q, m, boff, btree, B, k, d2, idx, s);
    if (k <= 32)
        return forest_knn_launch<D, 32>(f, q, m, boff, btree, B, k, d2, idx, s);
    return forest_knn_launch<D, 64>(f, q, m, boff, btree, B, k, d2, idx, s);
}

}  // namespace

arborx_status forest_reserve(ForestDev &f, int64_t m, hipStream_t s) { return reserve_ws(f, m, s); }

arborx_status forest_query_reduce(ForestDev &f, const float *q, int64_t m, const int64_t *boff, const int32_t *btree,
                                  const float *brad, int B, int op, int scale_bits, int32_t *counts, int64_t *sums,
                                  hipStream_t s)
{
    if (m == 0)
        return ARBORX_OK;
    arborx_status st = check_nodes(f.qnodes, f.wnodes, f.n, forest_format(OP_REDUCE, f));
    if (st == ARBORX_OK)
        st = reserve_ws(f, m, s);
    if (st != ARBORX_OK)
        return st;
    switch (f.dim) {
    case 2: return forest_reduce_impl<2>(f, q, m, boff, btree, brad, B, op, scale_bits, counts, sums, s);
    case 3: return forest_reduce_impl<3>(f, q, m, boff, btree, brad, B, op, scale_bits, counts, sums, s);
    case 6: return forest_reduce_impl<6>(f, q, m, boff, btree, brad, B, op, scale_bits, counts, sums, s);
    default: return fail(ARBORX_E_UNSUPPORTED, "dimension not compiled in");
    }
}

arborx_status forest_query_knn(ForestDev &f, const float *q, int64_t m, const int64_t *boff, const int32_t *btree,
                               int B, int k, float *d2, int32_t *idx, hipStream_t s)
{
    if (m == 0)
        return ARBORX_OK;
    arborx_status st = check_nodes(f.qnodes, f.wnodes, f.n, forest_format(OP_KNN, f));
    if (st == ARBORX_OK && boff)
        st = reserve_ws(f, m, s);
    if (st != ARBORX_OK)
        return st;
    switch (f.dim) {
    case 2: return forest_knn_impl<2>(f, q, m, boff, btree, B, k, d2, idx, s);
    case 3: return forest_knn_impl<3>(f, q, m, boff, btree, B, k, d2, idx, s);
    case 6: return forest_knn_impl<6>(f, q, m, boff, btree, B, k, d2, idx, s);
    default: return fail(ARBORX_E_UNSUPPORTED, "dimension not compiled in");
    }
}

}  // namespace ax
