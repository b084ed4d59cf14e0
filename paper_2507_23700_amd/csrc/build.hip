// BVH construction (Section 2.6 of the ArborX 2.0 paper: 64-bit Morton codes,
// a sort, and Apetrei's bottom-up hierarchy construction).
//
//   1. scene bounds      : min/max per dimension over all values;
//   2. Morton-64         : quantise each value's centre to floor(63/D) bits per
//                          dimension and interleave;
//   3. radix sort        : stable sort of (code, value index);
//   4. hierarchy + refit : one thread per leaf climbs the tree.  Internal node
//                          p separates sorted leaves p and p+1.  A subtree over
//                          leaves [l, r] becomes the left child of node r or the
//                          right child of node l-1, whichever boundary is the
//                          smaller split key (the XOR of neighbouring codes,
//                          ties between equal codes broken by position).  Each
//                          thread writes its box into its slot of the parent
//                          and swaps an arrival word into the parent's flag;
//                          the first to arrive stops, the second merges the
//                          sibling's box and continues upwards.  Writing a
//                          leaf's box straight into its parent slot is the
//                          "leaf gather": leaves need no array of their own.
#include <algorithm>
#include <cstddef>
#include <vector>

#include "device_util.hpp"
#include "geometry.hpp"
#include "internal.hpp"
#include "profile.hpp"

namespace ax {
namespace {

constexpr int kBuildBlock = 256;

// Step of the 16-bit frame [lo, hi]: a hair above (hi - lo) / kQMax, so that the
// frame's end lo + kQMax * step is not below hi.
__device__ __forceinline__ float quant_scale(float lo, float hi)
{
    if (!(hi > lo))
        return 0.0f;
    const double extent = (double)hi - (double)lo;
    float s = (float)(extent * ((1.0 + 0x1p-18) / kQMax));
    while ((double)s * kQMax < extent * (1.0 + 0x1p-40))  // rounding of a tiny step
        s = nextafterf(s, INFINITY);
    return s;
}

// The frame of a tree: one step for every dimension, the largest of them, so
// that walks measure distances in codes (CodeMetric), unless some extent is
// below 1/256 of the largest; that keeps at least 256 codes across every
// extent, and the largest extent has no finer codes either way.  Else each
// dimension has its own step (the largest where it has no extent), and the
// walks weigh the gaps of the dimensions.
template <int D>
__device__ void quant_frame(const float *lo, const float *hi, TreeHeader &h)
{
    float most = 0.0f, least = INFINITY;
    for (int d = 0; d < D; ++d) {
        h.qscale[d] = quant_scale(lo[d], hi[d]);
        most = fmaxf(most, h.qscale[d]);
        if (h.qscale[d] > 0.0f)
            least = fminf(least, h.qscale[d]);
    }
    h.qinv = most > 0.0f && most < INFINITY ? 1.0 / (double)most : 0.0;
    h.even = most * (1.0f / 256.0f) <= least;
    for (int d = 0; d < D; ++d) {
        if (h.even || !(h.qscale[d] > 0.0f))
            h.qscale[d] = most;
        h.qweight[d] = (float)((double)h.qscale[d] * h.qinv);
        h.qinvs[d] = h.qinv > 0.0 ? 1.0 / (double)h.qscale[d] : 0.0;
    }
}

// One dimension of a frame: codes rounded outward, with a hair for the
// arithmetic here.  Where lo + code * step is at most x, so is its rounding to a
// float, x being one: the decoded box contains the true one as well, and no more
// is needed where a code is far below the spacing of floats.
struct CodeAxis {
    double lo, inv;
    __device__ __forceinline__ void set(float l, double i)
    {
        lo = l;
        inv = i;
    }
    __device__ __forceinline__ uint32_t down(float x) const
    {
        return (uint32_t)fmin(fmax(((double)x - lo) * inv - 0x1p-10, 0.0), (double)kQMax);
    }
    __device__ __forceinline__ uint32_t up(float x) const
    {
        return (double)x > lo ? (uint32_t)fmin(ceil(((double)x - lo) * inv + 0x1p-10), (double)kQMax) : 0u;
    }
};

template <int D>
struct CodeFrame {
    CodeAxis axis[D];
    __device__ __forceinline__ explicit CodeFrame(const TreeHeader &h)
    {
#pragma unroll
        for (int d = 0; d < D; ++d)
            axis[d].set(h.lo[d], h.qinvs[d]);
    }
};

template <int D>
__global__ __launch_bounds__(kBuildBlock) void bounds_partial(const float *__restrict__ values, int64_t n, int kind,
                                                              float *__restrict__ partial)
{
    __shared__ float s_lo[kBuildBlock / kWave][D];
    __shared__ float s_hi[kBuildBlock / kWave][D];
    float lo[D], hi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        lo[d] = INFINITY;
        hi[d] = -INFINITY;
    }
    const int stride_v = kind == ARBORX_BOXES ? 2 * D : D;
    const int hoff = kind == ARBORX_BOXES ? D : 0;
    for (int64_t i = (int64_t)blockIdx.x * kBuildBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBuildBlock) {
        const float *v = values + i * stride_v;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = fminf(lo[d], v[d]);
            hi[d] = fmaxf(hi[d], v[hoff + d]);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
            lo[d] = fminf(lo[d], __shfl_xor(lo[d], o, kWave));
            hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o, kWave));
        }
    }
    if (lane_id() == 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            s_lo[wave_id()][d] = lo[d];
            s_hi[wave_id()][d] = hi[d];
        }
    }
    __syncthreads();
    if (threadIdx.x < D) {
        const int d = threadIdx.x;
        float a = INFINITY, b = -INFINITY;
        for (int w = 0; w < kBuildBlock / kWave; ++w) {
            a = fminf(a, s_lo[w][d]);
            b = fmaxf(b, s_hi[w][d]);
        }
        partial[(int64_t)blockIdx.x * 2 * D + d] = a;
        partial[(int64_t)blockIdx.x * 2 * D + D + d] = b;
    }
}

template <int D>
__global__ __launch_bounds__(kBuildBlock) void bounds_final(const float *__restrict__ partial, int blocks, int64_t n,
                                                             TreeHeader *hdr)
{
    __shared__ float s_lo[kBuildBlock / kWave][D];
    __shared__ float s_hi[kBuildBlock / kWave][D];
    float a[D], b[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        a[d] = INFINITY;
        b[d] = -INFINITY;
    }
    for (int k = threadIdx.x; k < blocks; k += kBuildBlock)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            a[d] = fminf(a[d], partial[(int64_t)k * 2 * D + d]);
            b[d] = fmaxf(b[d], partial[(int64_t)k * 2 * D + D + d]);
        }
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
            a[d] = fminf(a[d], __shfl_xor(a[d], o, kWave));
            b[d] = fmaxf(b[d], __shfl_xor(b[d], o, kWave));
        }
    if (lane_id() == 0)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            s_lo[wave_id()][d] = a[d];
            s_hi[wave_id()][d] = b[d];
        }
    __syncthreads();
    const int d = threadIdx.x;
    if (d < D) {
        float lo = INFINITY, hi = -INFINITY;
        for (int w = 0; w < kBuildBlock / kWave; ++w) {
            lo = fminf(lo, s_lo[w][d]);
            hi = fmaxf(hi, s_hi[w][d]);
        }
        hdr->lo[d] = lo;
        hdr->hi[d] = hi;
        s_lo[0][d] = lo;
        s_hi[0][d] = hi;
    }
    __syncthreads();
    if (d == 0) {
        quant_frame<D>(s_lo[0], s_hi[0], *hdr);
        hdr->crowded = 0;
        hdr->n = (int32_t)n;
        hdr->root = n > 0 ? 0 : -1;
        hdr->height = 0;
        hdr->start = 0;
    }
}

// Codes of value centres (points: the point; boxes: the box centre).
template <int D>
__global__ __launch_bounds__(kBuildBlock) void morton_kernel(const float *__restrict__ values, int64_t n, int kind,
                                                             const float *__restrict__ blo,
                                                             const float *__restrict__ bhi,
                                                             uint64_t *__restrict__ codes, uint32_t *__restrict__ ids)
{
    constexpr int bits = 63 / D;
    float lo[D], inv[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        lo[d] = blo[d];
        const float ext = bhi[d] - blo[d];
        inv[d] = ext > 0.0f ? 1.0f / ext : 0.0f;
    }
    for (int64_t i = (int64_t)blockIdx.x * kBuildBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBuildBlock) {
        uint32_t c[D];
        if (kind == ARBORX_BOXES) {
            const float *v = values + i * 2 * D;
#pragma unroll
            for (int d = 0; d < D; ++d)
                c[d] = quantise(v[d] + 0.5f * (v[D + d] - v[d]), lo[d], inv[d], bits);
        } else {
            const float *v = values + i * D;
#pragma unroll
            for (int d = 0; d < D; ++d)
                c[d] = quantise(v[d], lo[d], inv[d], bits);
        }
        codes[i] = interleave<D>(c, bits);
        if (ids)
            ids[i] = (uint32_t)i;
    }
}

// Split key between sorted leaves i and i+1: code differences rank above
// position differences (equal codes), so the order is total once ties are
// broken by node index.
__device__ __forceinline__ uint64_t split_key(const uint64_t *__restrict__ codes, int i)
{
    const uint64_t x = codes[i] ^ codes[i + 1];
    return x ? (x | (1ull << 63)) : (uint64_t)(uint32_t)(i ^ (i + 1));
}

template <int D>
__global__ __launch_bounds__(kBuildBlock) void hierarchy_kernel(const uint64_t *__restrict__ codes,
                                                                const uint32_t *__restrict__ ids,
                                                                const float *__restrict__ values, int kind, int n,
                                                                Node<D> *nodes, float *__restrict__ leaves,
                                                                unsigned long long *flags, TreeHeader *hdr)
{
    const int i = blockIdx.x * kBuildBlock + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t id = ids[i];
    if (id >= (uint32_t)n)
        return;
    float lo[D], hi[D];
    if (kind == ARBORX_BOXES) {
        const float *v = values + (int64_t)id * 2 * D;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = v[d];
            hi[d] = v[D + d];
        }
    } else {
        const float *v = values + (int64_t)id * D;
#pragma unroll
        for (int d = 0; d < D; ++d)
            lo[d] = hi[d] = v[d];
    }
    int32_t ref = ~(int32_t)id;
    store_leaf<D>(leaves, i, kind, lo, hi, (int32_t)id);
    if (n == 1) {
        Node<D> &nd = nodes[0];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            nd.lo[0][d] = lo[d];
            nd.hi[0][d] = hi[d];
            nd.lo[1][d] = INFINITY;
            nd.hi[1][d] = -INFINITY;
        }
        nd.child[0] = ref;
        nd.child[1] = kEmptyRef;
        nd.range_l = 0;
        nd.range_r = 0;
        hdr->root = 0;
        hdr->height = 1;
        return;
    }
    int l = i, r = i, h = 0;
    while (true) {
        int p, side;
        if (l == 0 || (r != n - 1 && split_key(codes, r) < split_key(codes, l - 1))) {
            p = r;
            side = 0;
        } else {
            p = l - 1;
            side = 1;
        }
        Node<D> *np = nodes + p;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            np->lo[side][d] = lo[d];
            np->hi[side][d] = hi[d];
        }
        np->child[side] = ref;
        // arrival word: (height + 1) << 32 | the outer bound of this subtree's range
        const unsigned long long mine =
            ((unsigned long long)(uint32_t)(h + 1) << 32) | (uint32_t)(side == 0 ? l : r);
        const unsigned long long other =
            __hip_atomic_exchange(flags + p, mine, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (other == 0)
            return;  // first arrival: the sibling's thread finishes this node
        const int oh = (int)(other >> 32) - 1;
        const int ob = (int)(uint32_t)other;
        if (side == 0)
            r = ob;
        else
            l = ob;
        h = (h > oh ? h : oh) + 1;
        const int os = 1 - side;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = fminf(lo[d], np->lo[os][d]);
            hi[d] = fmaxf(hi[d], np->hi[os][d]);
        }
        np->range_l = l;
        np->range_r = r;
        ref = p;
        if (l == 0 && r == n - 1) {
            hdr->root = p;
            hdr->height = h;
            return;
        }
    }
}

// ---------------------------------------------------------------------------
// Two-phase form of the same climb.  The tree is identical to the single-pass
// kernel's; only where the arrival handoff happens differs.
//
// Phase 1: one workgroup per chunk of C consecutive sorted leaves.  Arrivals at
// splits p with both neighbours inside the chunk (cs <= p <= ce-2) hand off
// through LDS: flags and the two child slots of each local split live in
// shared memory, so the exchange needs only workgroup scope.  A split whose
// second child reaches outside the chunk gets a single arrival here; its slot
// and arrival word are written to global memory at the end ("pending").  A
// climb that reaches split cs-1 or ce-1 (the chunk's borders) stops and is
// recorded as one of at most two escapes of the chunk.
// Phase 2: one thread per escape continues the climb over the splits whose
// subtrees span chunks; a workgroup takes the escapes of kGroupChunks
// neighbouring chunks, whose climbs meet in LDS, and the next level takes what
// leaves the groups, until one group is left.
// ---------------------------------------------------------------------------

template <int D>
struct Escape {
    int32_t valid, p, side, l, r, h, ref, pad;
    float lo[D], hi[D];
};

constexpr unsigned long long kDone = 1ull << 63;  // above an arrival word; with the node's local leaf range

__device__ __forceinline__ unsigned long long arrival_word(int side, int h, int bound)
{
    return ((unsigned long long)side << 48) | ((unsigned long long)(uint32_t)(h + 1) << 32) | (uint32_t)bound;
}

// While a child waits in a node, the node's range words hold the split key at
// the child's outer bound (none, all ones, at an end of the tree): the climb
// that meets it needs that key next.
template <int D>
__device__ __forceinline__ void put_wait_key(Node<D> &nd, uint64_t key)
{
    nd.range_l = (int32_t)(uint32_t)key;
    nd.range_r = (int32_t)(uint32_t)(key >> 32);
}
template <int D>
__device__ __forceinline__ uint64_t wait_key(const Node<D> &nd)
{
    return ((uint64_t)(uint32_t)nd.range_r << 32) | (uint32_t)nd.range_l;
}

template <int D>
__device__ __forceinline__ void store_node(Node<D> *dst, const Node<D> &nd)
{
    float4 *d4 = reinterpret_cast<float4 *>(dst);
    const float4 *s4 = reinterpret_cast<const float4 *>(&nd);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(Node<D>) / 16); ++k)
        d4[k] = s4[k];
}

template <int D>
__device__ __forceinline__ void load_value_box(const float *values, int kind, uint32_t id, float *lo, float *hi)
{
    if (kind == ARBORX_BOXES) {
        const float *v = values + (int64_t)id * 2 * D;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = v[d];
            hi[d] = v[D + d];
        }
    } else {
        const float *v = values + (int64_t)id * D;
#pragma unroll
        for (int d = 0; d < D; ++d)
            lo[d] = hi[d] = v[d];
    }
}

// A tree is crowded where its frame is coarse for its points: some subtree of
// kCrowd or more values lies within kCrowdCodes codes, rounded outward, in
// every dimension (and not all in one place, where no box can be left out).
// In codes every box around there is next to every query, so a search leaves
// nothing out and meets the whole crowd; float boxes have no such limit (see
// codes_serve).  One stray point far from 10^6 uniform ones in 3D widens the
// frame until a code is 1/S of the mean spacing; nearest 8 over codes and over
// float nodes: S = 20 466 and 564 us, 7 621 and 703, 5 789 and 787, 4 899 and
// 808, 2.2 1956 and 1063, 1.1 4063 and 1064, where the largest subtree within
// four codes has 3, 6, 7, 9, 21 and 79 points.  With 10^4 of 10^6 points inside
// two codes 4960 and 482 us.
// It is looked for in the subtrees that lie in one chunk of the climb: some part
// of a crowd over several chunks does, and the second phase, one chain of steps,
// took 24.5 us instead of 21.2 at 2*10^4 points when it looked at every node.
constexpr uint32_t kCrowdCodes = 5;
constexpr int kCrowd = 8;
template <int D>
__device__ __forceinline__ bool is_crowd(const float *lo, const float *hi, uint32_t span, int values)
{
    bool apart = false;
#pragma unroll
    for (int d = 0; d < D; ++d)
        apart = apart || lo[d] < hi[d];
    return apart && span <= kCrowdCodes && values >= kCrowd;
}
template <int D>
__device__ __forceinline__ bool is_crowd(const float *lo, const float *hi, const CodeFrame<D> &frame, int values)
{
    uint32_t span = 0;
#pragma unroll
    for (int d = 0; d < D; ++d)
        span = max(span, frame.axis[d].up(hi[d]) - frame.axis[d].down(lo[d]));
    return is_crowd<D>(lo, hi, span, values);
}

// Quantized form of float node p of a tree with the given frame.  A point tree's
// leaf child keeps its point and reference unchanged (the point's float words
// fill that child's code bytes); a box tree's leaf child becomes its sorted
// leaf position: the left child of node p is leaf p, the right child leaf
// p + 1.  Returns whether a child is a crowd.
template <int D>
__device__ __forceinline__ bool store_qnode(QNode<D> *__restrict__ dst, const Node<D> &nd, int p, int kind,
                                            const CodeFrame<D> &frame)
{
    QNode<D> qn;
    bool crowd = false;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(qn.pad) / sizeof(qn.pad[0])); ++k)
        qn.pad[k] = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int32_t ref = nd.child[c];
        if (ref == kEmptyRef) {
#pragma unroll
            for (int d = 0; d < D; ++d)
                qn.w[c][d] = 0xffffffffu;
            qn.child[c] = kEmptyRef;
            continue;
        }
        if (ref < 0 && kind != ARBORX_BOXES) {
#pragma unroll
            for (int d = 0; d < D; ++d)
                qn.w[c][d] = __float_as_uint(nd.lo[c][d]);
            qn.child[c] = ref;
            continue;
        }
        uint32_t span = 0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const CodeAxis &a = frame.axis[d];
            const uint32_t lo = a.down(nd.lo[c][d]), hi = a.up(nd.hi[c][d]);
            qn.w[c][d] = lo | (((uint32_t)kQMax - hi) << 16);
            span = max(span, hi - lo);
        }
        crowd = crowd || is_crowd<D>(nd.lo[c], nd.hi[c], span, c == 0 ? p - nd.range_l + 1 : nd.range_r - p);
        qn.child[c] = ref >= 0 ? ref : ~(p + c);
    }
    float4 *d4 = reinterpret_cast<float4 *>(dst);
    const float4 *s4 = reinterpret_cast<const float4 *>(&qn);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(QNode<D>) / 16); ++k)
        d4[k] = s4[k];
    return crowd;
}

template <int D>
__device__ void write_single_leaf_tree(Node<D> *node, QNode<D> *qnode, int kind, TreeHeader *hdr, const float *lo,
                                       const float *hi, int32_t ref, int index)
{
    Node<D> nd;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        nd.lo[0][d] = lo[d];
        nd.hi[0][d] = hi[d];
        nd.lo[1][d] = INFINITY;
        nd.hi[1][d] = -INFINITY;
    }
    nd.child[0] = ref;
    nd.child[1] = kEmptyRef;
    nd.range_l = index;
    nd.range_r = index;
    store_node(node, nd);
    if (qnode)
        store_qnode<D>(qnode, nd, index, kind, CodeFrame<D>(*hdr));
    hdr->root = index;
    hdr->height = 1;
}

// Chunks whose border climbs one workgroup of the second phase takes, one
// thread for each of their two escapes.  Small groups: a compute unit serves
// about one lane's load a clock, and a workgroup of 1024 climbs waited on that
// (137 us for the one group of 10^6 points, against 2 launches of 25).
constexpr int kGroupChunks = 128;
constexpr int kTopBlock = 2 * kGroupChunks;
template <int D> constexpr int chunk_leaves() { return D <= 3 ? 1024 : 512; }

// Tree (segment) holding sorted leaf i: seg[s] <= i < seg[s+1].  Without
// segments the whole array is one tree.  Climbs never cross a tree's ends, so
// every tree of a forest gets its own root.
__device__ __forceinline__ void segment_of(int i, const int64_t *__restrict__ seg, int nseg, int n, int &s, int &ts,
                                           int &te)
{
    if (!seg) {
        s = 0;
        ts = 0;
        te = n - 1;
        return;
    }
    int lo = 0, hi = nseg;  // find the last s with seg[s] <= i
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seg[mid] <= i)
            lo = mid;
        else
            hi = mid;
    }
    s = lo;
    ts = (int)seg[lo];
    te = (int)seg[lo + 1] - 1;
}

// Float nodes -> quantized nodes, a pass over the finished tree, for the
// single-pass climb (the chunked one writes both forms itself).  Node p
// belongs to the tree holding sorted leaf p (a one-value tree's node sits at
// its own leaf position).
template <int D>
__global__ void quantize_nodes(const Node<D> *__restrict__ nodes, int n_nodes, const int64_t *__restrict__ seg,
                               int nseg, int n, int kind, TreeHeader *__restrict__ hdrs,
                               QNode<D> *__restrict__ qnodes)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_nodes)
        return;
    int sg, ts, te;
    segment_of(p < n ? p : n - 1, seg, nseg, n, sg, ts, te);
    Node<D> nd;
    load_node(nodes, p, nd);
    if (store_qnode<D>(qnodes + p, nd, p, kind, CodeFrame<D>(hdrs[sg])))
        hdrs[sg].crowded = 1;
}


// Four-wide node p from binary node p and its internal children (the tree
// is final).  Slot order: p's left subtree first, so a leaf slot keeps the
// sorted order of the leaves.
template <int D>
__global__ void widen_nodes(const Node<D> *__restrict__ nodes, int n_nodes, Node4<D> *__restrict__ wnodes)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_nodes)
        return;
    Node<D> nd;
    load_node(nodes, p, nd);
    Node4<D> w;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(w.pad) / sizeof(w.pad[0])); ++k)
        w.pad[k] = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        w.child[s] = kEmptyRef;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            w.lo[s][d] = INFINITY;
            w.hi[s][d] = -INFINITY;
        }
    }
    int k = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int32_t ref = nd.child[c];
        if (ref >= 0 && ref < n_nodes) {
            Node<D> ch;
            load_node(nodes, ref, ch);
#pragma unroll
            for (int g = 0; g < 2; ++g) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    w.lo[k][d] = ch.lo[g][d];
                    w.hi[k][d] = ch.hi[g][d];
                }
                w.child[k] = ch.child[g];
                ++k;
            }
        } else if (ref != kEmptyRef) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                w.lo[k][d] = nd.lo[c][d];
                w.hi[k][d] = nd.hi[c][d];
            }
            w.child[k] = ref;
            ++k;
        }
    }
    float4 *dst = reinterpret_cast<float4 *>(wnodes + p);
    const float4 *src = reinterpret_cast<const float4 *>(&w);
#pragma unroll
    for (int q = 0; q < (int)(sizeof(Node4<D>) / 16); ++q)
        dst[q] = src[q];
}

template <int D>
__global__ __launch_bounds__(chunk_leaves<D>()) void hierarchy_chunk_kernel(const uint64_t *__restrict__ codes,
                                                                      const uint32_t *__restrict__ ids,
                                                                      const float *__restrict__ values, int kind,
                                                                      int n, Node<D> *__restrict__ nodes,
                                                                      QNode<D> *__restrict__ qnodes,
                                                                      float *__restrict__ leaves,
                                                                      unsigned long long *__restrict__ gflags,
                                                                      Escape<D> *__restrict__ escapes,
                                                                      const int64_t *__restrict__ seg, int nseg,
                                                                      TreeHeader *hdrs)
{
    constexpr int C = chunk_leaves<D>();
    __shared__ uint64_t s_key[C + 1];             // split keys of splits cs-1 .. ce-1
    __shared__ unsigned long long s_flag[C];      // arrival words of local splits cs .. ce-2
    __shared__ float s_lo[C][2][D], s_hi[C][2][D];  // both child slots of each local split
    __shared__ int32_t s_ref[C][2];

    // one thread per leaf of the chunk, so every climb of the chunk runs at once
    const int cs = blockIdx.x * C;
    const int ce = min(n, cs + C);
    const int tid = threadIdx.x;
    for (int j = tid; j < C; j += C)
        s_flag[j] = 0;
    for (int j = tid; j <= C; j += C) {
        const int g = cs - 1 + j;
        s_key[j] = (g >= 0 && g <= ce - 1 && g <= n - 2) ? split_key(codes, g) : 0ull;
    }
    if (tid < 2)
        escapes[2 * blockIdx.x + tid].valid = 0;
    __syncthreads();

    for (int i = cs + tid; i < ce; i += C) {
        const uint32_t id = ids[i];
        if (id >= (uint32_t)n)
            continue;
        float lo[D], hi[D];
        load_value_box<D>(values, kind, id, lo, hi);
        store_leaf<D>(leaves, i, kind, lo, hi, (int32_t)id);
        int32_t ref = ~(int32_t)id;
        int sg, ts, te;
        segment_of(i, seg, nseg, n, sg, ts, te);
        if (ts == te) {  // a one-value tree: its node slot is the unused split at its end
            write_single_leaf_tree<D>(nodes + ts, qnodes ? qnodes + ts : nullptr, kind, hdrs + sg, lo, hi, ref, ts);
            continue;
        }
        int l = i, r = i, h = 0;
        while (true) {
            int p, side;
            if (l == ts || (r != te && s_key[r - cs + 1] < s_key[l - 1 - cs + 1])) {
                p = r;
                side = 0;
            } else {
                p = l - 1;
                side = 1;
            }
            if (p < cs || p > ce - 2) {  // a border split of the chunk: continue in phase 2
                Escape<D> &e = escapes[2 * blockIdx.x + (p >= cs ? 1 : 0)];
                e.p = p;
                e.side = side;
                e.l = l;
                e.r = r;
                e.h = h;
                e.ref = ref;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    e.lo[d] = lo[d];
                    e.hi[d] = hi[d];
                }
                e.valid = 1;
                break;
            }
            const int lp = p - cs;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                s_lo[lp][side][d] = lo[d];
                s_hi[lp][side][d] = hi[d];
            }
            s_ref[lp][side] = ref;
            const unsigned long long other = __hip_atomic_exchange(
                &s_flag[lp], arrival_word(side, h, side == 0 ? l : r), __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (other == 0)
                break;  // first arrival
            const int os = 1 - side;
            const int oh = (int)((other >> 32) & 0xffff) - 1;
            const int ob = (int)(uint32_t)other;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                lo[d] = fminf(lo[d], s_lo[lp][os][d]);
                hi[d] = fmaxf(hi[d], s_hi[lp][os][d]);
            }
            if (side == 0)
                r = ob;
            else
                l = ob;
            h = (h > oh ? h : oh) + 1;
            s_flag[lp] = kDone | ((unsigned long long)(l - cs) << 16) | (unsigned long long)(r - cs);
            ref = p;
            if (l == ts && r == te) {
                hdrs[sg].root = p;
                hdrs[sg].height = h;
                break;
            }
        }
    }
    __syncthreads();
    // Bound: memory (a 128-byte line for each 12-byte point, and the nodes, about 2.9 GB at 10^7 points, in 0.69 ms,
    // where this kernel and the pass that read its nodes back took 0.66 + 0.27 ms).
    // Both child slots of every finished split are in LDS: its nodes are written here, in order, in both forms
    // (stores inside the climb lengthened its chain of levels, and a later pass for the quantized form read every
    // node back).  Of a split with a single arrival, that child's slot is published for the second phase.
    for (int lp = tid; lp <= ce - 1 - cs; lp += C) {
        const int p = cs + lp;
        if (p > n - 2)
            break;
        const unsigned long long w = lp < ce - 1 - cs ? s_flag[lp] : 0;
        if (w & kDone) {
            Node<D> nd;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    nd.lo[c][d] = s_lo[lp][c][d];
                    nd.hi[c][d] = s_hi[lp][c][d];
                }
                nd.child[c] = s_ref[lp][c];
            }
            nd.range_l = cs + (int)((w >> 16) & 0xffff);
            nd.range_r = cs + (int)(w & 0xffff);
            store_node(nodes + p, nd);
            if (qnodes) {
                int sg, ts, te;
                segment_of(p, seg, nseg, n, sg, ts, te);
                if (store_qnode<D>(qnodes + p, nd, p, kind, CodeFrame<D>(hdrs[sg])))
                    hdrs[sg].crowded = 1;
            }
            continue;
        }
        gflags[p] = w;
        if (w != 0) {
            const int side = (int)(w >> 48);
            Node<D> *np = nodes + p;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                np->lo[side][d] = s_lo[lp][side][d];
                np->hi[side][d] = s_hi[lp][side][d];
            }
            np->child[side] = s_ref[lp][side];
            const int bound = (int)(uint32_t)w;  // l of a left child, r of a right one
            int sg, ts, te;
            segment_of(p, seg, nseg, n, sg, ts, te);
            put_wait_key(*np, side == 0 ? (bound == ts ? ~0ull : s_key[bound - cs]) :
                                          (bound == te ? ~0ull : s_key[bound - cs + 1]));
            if (qnodes && is_crowd<D>(s_lo[lp][side], s_hi[lp][side], CodeFrame<D>(hdrs[sg]),
                                      side == 0 ? p - bound + 1 : bound - p))
                hdrs[sg].crowded = 1;
        }
    }
}

// One level of the second phase: workgroup g continues the climbs of its
// escapes, two for each of kGroupChunks parts of the level below, over the
// splits inside its leaves [g * span, (g + 1) * span), and records those that
// leave them (at most two) as escapes of its own (out; NULL for the last
// level).
//
// A climb is a chain of dependent steps, so its latency is all that counts.
// A split's other child either waits in the node, left there by an earlier
// phase (its arrival word in gflags), or comes from another climb of this
// workgroup.  Those two meet in LDS: the first enters its number under the
// split in a hash table and stops, the second finds it there and takes its
// box.  No store of a climb is waited for, and none is read back before the
// kernel ends; what is still waiting then is written for the next level.
// (Arrivals exchanged in global memory, with the fences that needs across the
// XCDs' L2 caches, took 252 us at 10^7 points, 52 at 10^6, 27 at 2*10^4; this
// takes 100, 53 and 21, the quantized nodes of the second phase included.)
template <int D>
__global__ __launch_bounds__(kTopBlock) void hierarchy_top_kernel(const uint64_t *__restrict__ codes, int n, int kind,
                                                                  Node<D> *__restrict__ nodes,
                                                                  QNode<D> *__restrict__ qnodes,
                                                                  unsigned long long *__restrict__ gflags,
                                                                  const Escape<D> *__restrict__ escapes,
                                                                  int n_escapes, int64_t span,
                                                                  Escape<D> *__restrict__ out,
                                                                  const int64_t *__restrict__ seg, int nseg,
                                                                  TreeHeader *__restrict__ hdrs)
{
    constexpr int E = kTopBlock;                      // escapes of a workgroup
    constexpr int kTableBits = 9, kTable = 1 << kTableBits;
    static_assert(kTable >= 2 * E, "a climb enters the table once");
    __shared__ unsigned long long s_table[kTable];    // (split + 1) << 32 | climb; 0: free
    __shared__ float s_lo[D][E], s_hi[D][E];
    __shared__ int32_t s_ref[E];
    __shared__ unsigned long long s_word[E];          // arrival word of a climb that waits; 0: none, or met
    __shared__ uint64_t s_key[E];                     // split key at its outer bound
    __shared__ int32_t s_at[E];                       // the split it waits at

    const int tid = threadIdx.x;
    for (int i = tid; i < kTable; i += kTopBlock)
        s_table[i] = 0;
    s_word[tid] = 0;
    if (out && tid < 2)
        out[2 * blockIdx.x + tid].valid = 0;
    __syncthreads();

    const int64_t cs = (int64_t)blockIdx.x * span, ce = cs + span < n ? cs + span : n;
    const int64_t e_i = (int64_t)blockIdx.x * E + tid;
    if (e_i < n_escapes && escapes[e_i].valid) {  // climbs never wait for one another
        const Escape<D> &e = escapes[e_i];
        float lo[D], hi[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = e.lo[d];
            hi[d] = e.hi[d];
        }
        int p = e.p, side = e.side, l = e.l, r = e.r, h = e.h;
        int32_t ref = e.ref;
        int sg, ts, te;
        segment_of(l, seg, nseg, n, sg, ts, te);
        const CodeFrame<D> frame(hdrs[sg]);
        // split keys at the subtree's two ends (none at an end of the tree)
        uint64_t kl = l == ts ? ~0ull : split_key(codes, l - 1), kr = r == te ? ~0ull : split_key(codes, r);
        if (qnodes && is_crowd<D>(lo, hi, frame, r - l + 1))
            hdrs[sg].crowded = 1;
        // a climb visits at most n-1 splits
        for (int guard = 0; guard < n; ++guard) {
            if (p < 0 || p > n - 2)
                break;
            if (out && (p < cs || p > ce - 2)) {
                Escape<D> &o = out[2 * blockIdx.x + (p >= cs ? 1 : 0)];
                o.p = p;
                o.side = side;
                o.l = l;
                o.r = r;
                o.h = h;
                o.ref = ref;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    o.lo[d] = lo[d];
                    o.hi[d] = hi[d];
                }
                o.valid = 1;
                break;
            }
            Node<D> *np = nodes + p;
            unsigned long long other = gflags[p];
            Node<D> nd;  // the waiting child's words, if there is one
            load_node(nodes, p, nd);
            float slo[D], shi[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                slo[d] = side ? nd.lo[0][d] : nd.lo[1][d];
                shi[d] = side ? nd.hi[0][d] : nd.hi[1][d];
            }
            int32_t sref = side ? nd.child[0] : nd.child[1];
            uint64_t okey = wait_key(nd);
            if (other == 0) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    s_lo[d][tid] = lo[d];
                    s_hi[d][tid] = hi[d];
                }
                s_ref[tid] = ref;
                s_word[tid] = arrival_word(side, h, side == 0 ? l : r);
                s_at[tid] = p;
                s_key[tid] = side == 0 ? kl : kr;  // at its outer bound
                const unsigned long long mine = ((unsigned long long)(uint32_t)(p + 1) << 32) | (uint32_t)tid;
                uint32_t at = ((uint32_t)p * 2654435761u) >> (32 - kTableBits);  // borders differ in high bits only
                int sib = -1;
                for (int probe = 0; probe < kTable; ++probe) {  // at most E entries: a free one is found
                    unsigned long long seen = 0;
                    if (__hip_atomic_compare_exchange_strong(&s_table[at], &seen, mine, __ATOMIC_ACQ_REL,
                                                             __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP))
                        break;
                    if ((uint32_t)(seen >> 32) == (uint32_t)(p + 1)) {
                        sib = (int)(uint32_t)seen;
                        break;
                    }
                    at = (at + 1) & (kTable - 1);
                }
                if (sib < 0)  // first of the two
                    break;
                s_word[tid] = 0;
                other = s_word[sib];
                s_word[sib] = 0;
                okey = s_key[sib];
                sref = s_ref[sib];
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    slo[d] = s_lo[d][sib];
                    shi[d] = s_hi[d][sib];
                }
            }
            const int oh = (int)((other >> 32) & 0xffff) - 1;
            const int ob = (int)(uint32_t)other;
            if (side == 0)
                r = ob;
            else
                l = ob;
            h = (h > oh ? h : oh) + 1;
            if (side == 0)
                kr = okey;
            else
                kl = okey;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                nd.lo[0][d] = side == 0 ? lo[d] : slo[d];
                nd.hi[0][d] = side == 0 ? hi[d] : shi[d];
                nd.lo[1][d] = side == 0 ? slo[d] : lo[d];
                nd.hi[1][d] = side == 0 ? shi[d] : hi[d];
                lo[d] = fminf(lo[d], slo[d]);
                hi[d] = fmaxf(hi[d], shi[d]);
            }
            nd.child[0] = side == 0 ? ref : sref;
            nd.child[1] = side == 0 ? sref : ref;
            nd.range_l = l;
            nd.range_r = r;
            store_node(np, nd);
            if (qnodes)
                store_qnode<D>(qnodes + p, nd, p, kind, frame);
            ref = p;
            if (l == ts && r == te) {
                hdrs[sg].root = p;
                hdrs[sg].height = h;
                break;
            }
            if (l == ts || (r != te && kr < kl)) {
                p = r;
                side = 0;
            } else {
                p = l - 1;
                side = 1;
            }
        }
    }
    __syncthreads();
    const unsigned long long w = s_word[tid];
    if (w != 0) {
        const int side = (int)(w >> 48);
        Node<D> *np = nodes + s_at[tid];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            np->lo[side][d] = s_lo[d][tid];
            np->hi[side][d] = s_hi[d][tid];
        }
        np->child[side] = s_ref[tid];
        put_wait_key(*np, s_key[tid]);
        gflags[s_at[tid]] = w;
    }
}

// The second phase over all chunks: levels of groups of kGroupChunks, until one
// workgroup takes all that is left.  esc has room for escape_entries<D>(chunks).
template <int D>
void hierarchy_top(const uint64_t *codes, int n, int kind, Node<D> *nodes, QNode<D> *qnodes, unsigned long long *flags,
                   Escape<D> *esc, int chunks, const int64_t *seg, int nseg, TreeHeader *hdrs, hipStream_t s)
{
    int64_t span = chunk_leaves<D>();
    for (int parts = chunks; parts > 1;) {
        const int groups = (parts + kGroupChunks - 1) / kGroupChunks;
        span *= kGroupChunks;
        Escape<D> *out = groups > 1 ? esc + 2 * (size_t)parts : nullptr;
        hierarchy_top_kernel<D><<<groups, kTopBlock, 0, s>>>(codes, n, kind, nodes, qnodes, flags, esc, 2 * parts, span,
                                                             out, seg, nseg, hdrs);
        esc = out;
        parts = groups;
    }
}
template <int D>
size_t escape_entries(int chunks)
{
    constexpr int G = kGroupChunks;
    size_t all = 2 * (size_t)chunks;
    for (int parts = chunks; parts > 1; parts = (parts + G - 1) / G)
        all += 2 * (size_t)((parts + G - 1) / G);
    return all;
}

__global__ void empty_header(TreeHeader *hdr, int dim)
{
    for (int d = 0; d < kMaxDim; ++d)
        hdr->qscale[d] = 0.0f;
    hdr->qinv = 0.0;
    hdr->even = 1;
    hdr->crowded = 0;
    hdr->root = -1;
    hdr->height = 0;
    hdr->n = 0;
    hdr->start = 0;
    for (int d = 0; d < kMaxDim; ++d) {
        hdr->lo[d] = INFINITY;
        hdr->hi[d] = -INFINITY;
    }
    (void)dim;
}

template <int D>
arborx_status build_impl(const float *values, int64_t n, int kind, TreeDev &t, hipStream_t s)
{
    AX_HIP(hipGetLastError());  // clear stale errors from earlier user work
    arborx_status st = dalloc((void **)&t.hdr, sizeof(TreeHeader), s);
    if (st != ARBORX_OK)
        return st;
    t.n = n;
    t.dim = D;
    t.kind = kind;
    if (n == 0) {
        empty_header<<<1, 1, 0, s>>>(t.hdr, D);
        AX_HIP(hipGetLastError());
        return ARBORX_OK;
    }
    const int64_t nn = n > 1 ? n - 1 : 1;
    st = dalloc(&t.nodes, (size_t)nn * sizeof(Node<D>), s);
    if (st != ARBORX_OK)
        return st;
    st = dalloc((void **)&t.leaves, (size_t)n * leaf_floats(D, kind) * sizeof(float), s);
    if (st != ARBORX_OK)
        return st;
    const bool quantized = format_requested(1, D, kind, false), wide = format_requested(2, D, kind, false);
    if (quantized && (st = dalloc(&t.qnodes, (size_t)nn * sizeof(QNode<D>), s)) != ARBORX_OK)
        return st;
    if (wide && (st = dalloc(&t.wnodes, (size_t)nn * sizeof(Node4<D>), s)) != ARBORX_OK)
        return st;

    Temps tmp(s);
    const int pblocks = (int)grid_for(n, kBuildBlock, 1024);
    float *partial;
    uint64_t *codes, *codes2;
    uint32_t *ids, *ids2;
    unsigned long long *flags;
    uint8_t *ws;
    // the sorted codes stay with the tree: kNN finds a query's leaf position by binary search
    if ((st = dalloc((void **)&t.codes, (size_t)n * sizeof(uint64_t), s)) != ARBORX_OK)
        return st;
    codes = t.codes;
    if ((st = tmp.get(&partial, (size_t)pblocks * 2 * D)) != ARBORX_OK ||
        (st = tmp.get(&ids, n)) != ARBORX_OK || (st = tmp.get(&ids2, n)) != ARBORX_OK ||
        (st = tmp.get(&flags, nn)) != ARBORX_OK || (st = tmp.get(&ws, radix_workspace_bytes(n))) != ARBORX_OK ||
        (st = dalloc((void **)&codes2, (size_t)n * sizeof(uint64_t), s)) != ARBORX_OK)
        return st;
    tmp.adopt(codes2);

    {
        ProfScope ps("build_bounds", s);
        bounds_partial<D><<<pblocks, kBuildBlock, 0, s>>>(values, n, kind, partial);
        bounds_final<D><<<1, kBuildBlock, 0, s>>>(partial, pblocks, n, t.hdr);
    }
    const float *blo = reinterpret_cast<const float *>(reinterpret_cast<const char *>(t.hdr) + offsetof(TreeHeader, lo));
    const float *bhi = reinterpret_cast<const float *>(reinterpret_cast<const char *>(t.hdr) + offsetof(TreeHeader, hi));
    {
        ProfScope ps("build_morton", s);
        morton_kernel<D><<<grid_for(n, kBuildBlock, 65536), kBuildBlock, 0, s>>>(values, n, kind, blo, bhi, codes,
                                                                                ids);
    }
    bool alt = false;
    {
        ProfScope ps("build_sort", s);
        AX_HIP(radix_sort_pairs<uint64_t>(codes, ids, codes2, ids2, n, 0, (63 / D) * D, ws, s, &alt));
    }
    if (alt) {  // the tree keeps whichever buffer holds the result
        tmp.exchange(codes2, t.codes);
        t.codes = codes2;
        codes = codes2;
        ids = ids2;
    }
    Node<D> *nodes = static_cast<Node<D> *>(t.nodes);
    if (tuning(OP_SPATIAL).build == 1) {
        // single pass: every handoff through device-scope acquire/release
        fill_kernel<unsigned long long><<<grid_for(nn, 256, 65536), 256, 0, s>>>(flags, nn, 0ull);
        ProfScope ps("build_hierarchy", s);
        hierarchy_kernel<D><<<grid_for(n, kBuildBlock), kBuildBlock, 0, s>>>(codes, ids, values, kind, (int)n, nodes,
                                                                             t.leaves, flags, t.hdr);
    } else {
        constexpr int C = chunk_leaves<D>();
        const int chunks = (int)((n + C - 1) / C);
        Escape<D> *esc;
        if ((st = tmp.get(&esc, escape_entries<D>(chunks))) != ARBORX_OK)
            return st;
        ProfScope ps("build_hierarchy", s);
        QNode<D> *qnodes = static_cast<QNode<D> *>(t.qnodes);
        hierarchy_chunk_kernel<D><<<chunks, C, 0, s>>>(codes, ids, values, kind, (int)n, nodes, qnodes, t.leaves, flags,
                                                       esc, nullptr, 0, t.hdr);
        hierarchy_top<D>(codes, (int)n, kind, nodes, qnodes, flags, esc, chunks, nullptr, 0, t.hdr, s);
    }
    if (quantized && tuning(OP_SPATIAL).build == 1) {
        ProfScope ps("build_quantize", s);
        quantize_nodes<D><<<grid_for(nn, kBuildBlock), kBuildBlock, 0, s>>>(nodes, (int)nn, nullptr, 0, (int)n, t.kind,
                                                                            t.hdr, static_cast<QNode<D> *>(t.qnodes));
    }
    if (wide) {
        ProfScope ps("build_widen", s);
        widen_nodes<D><<<grid_for(nn, kBuildBlock), kBuildBlock, 0, s>>>(nodes, (int)nn,
                                                                         static_cast<Node4<D> *>(t.wnodes));
    }
    AX_HIP(hipGetLastError());
    return ARBORX_OK;
}

template <int D>
hipError_t morton_impl(const float *pts, int64_t n, const float *bounds, uint64_t *codes, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    morton_kernel<D><<<grid_for(n, kBuildBlock, 65536), kBuildBlock, 0, s>>>(pts, n, ARBORX_POINTS, bounds,
                                                                            bounds + D, codes, nullptr);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Forest build: many trees over one packed value array, tree t holding values
// [seg[t], seg[t+1]).  Work is cut into tiles that never straddle a tree so
// each workgroup knows its tree.  Per-tree bounds are reduced per tile and
// combined with atomics on order-preserving integer images of the floats;
// Morton keys are (tree << mbits) | tree-local code, so one global sort keeps
// every tree contiguous and Morton-ordered inside; the climb then stops at the
// tree ends (segment_of).
// ---------------------------------------------------------------------------

constexpr int kForestTile = 4096;

__device__ __forceinline__ uint32_t float_order(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float order_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

template <int D>
__global__ __launch_bounds__(kBuildBlock) void forest_tile_bounds(const float *__restrict__ values, int kind,
                                                                  const int32_t *__restrict__ tile_tree,
                                                                  const int32_t *__restrict__ tile_start,
                                                                  const int32_t *__restrict__ tile_end,
                                                                  uint32_t *__restrict__ tmin,
                                                                  uint32_t *__restrict__ tmax)
{
    __shared__ float s_lo[kBuildBlock / kWave][D];
    __shared__ float s_hi[kBuildBlock / kWave][D];
    const int b = blockIdx.x;
    const int t = tile_tree[b];
    float lo[D], hi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        lo[d] = INFINITY;
        hi[d] = -INFINITY;
    }
    const int stride_v = kind == ARBORX_BOXES ? 2 * D : D;
    const int hoff = kind == ARBORX_BOXES ? D : 0;
    for (int i = tile_start[b] + threadIdx.x; i < tile_end[b]; i += kBuildBlock) {
        const float *v = values + (int64_t)i * stride_v;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = fminf(lo[d], v[d]);
            hi[d] = fmaxf(hi[d], v[hoff + d]);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
            lo[d] = fminf(lo[d], __shfl_xor(lo[d], o, kWave));
            hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o, kWave));
        }
    }
    if (lane_id() == 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            s_lo[wave_id()][d] = lo[d];
            s_hi[wave_id()][d] = hi[d];
        }
    }
    __syncthreads();
    if (threadIdx.x < D) {
        const int d = threadIdx.x;
        float a = INFINITY, c = -INFINITY;
        for (int w = 0; w < kBuildBlock / kWave; ++w) {
            a = fminf(a, s_lo[w][d]);
            c = fmaxf(c, s_hi[w][d]);
        }
        atomicMin(&tmin[t * D + d], float_order(a));
        atomicMax(&tmax[t * D + d], float_order(c));
    }
}

template <int D>
__global__ void forest_headers(const int64_t *__restrict__ seg, int T, const uint32_t *__restrict__ tmin,
                               const uint32_t *__restrict__ tmax, TreeHeader *__restrict__ hdrs)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T)
        return;
    const int n = (int)(seg[t + 1] - seg[t]);
    TreeHeader &h = hdrs[t];
    h.n = n;
    h.start = (int)seg[t];
    h.root = -1;
    h.height = 0;
    for (int d = 0; d < kMaxDim; ++d) {
        h.lo[d] = (d < D && n > 0) ? order_float(tmin[t * D + d]) : INFINITY;
        h.hi[d] = (d < D && n > 0) ? order_float(tmax[t * D + d]) : -INFINITY;
        h.qscale[d] = 0.0f;
    }
    h.qinv = 0.0;
    h.even = 1;
    h.crowded = 0;
    if (n > 0)
        quant_frame<D>(h.lo, h.hi, h);
}

template <int D>
__global__ __launch_bounds__(kBuildBlock) void forest_tile_morton(const float *__restrict__ values, int kind,
                                                                  const int32_t *__restrict__ tile_tree,
                                                                  const int32_t *__restrict__ tile_start,
                                                                  const int32_t *__restrict__ tile_end,
                                                                  const TreeHeader *__restrict__ hdrs, int mbits,
                                                                  uint64_t *__restrict__ codes,
                                                                  uint32_t *__restrict__ ids)
{
    const int b = blockIdx.x;
    const int t = tile_tree[b];
    const int bits = mbits / D;
    float lo[D], inv[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        lo[d] = hdrs[t].lo[d];
        const float ext = hdrs[t].hi[d] - lo[d];
        inv[d] = ext > 0.0f ? 1.0f / ext : 0.0f;
    }
    for (int i = tile_start[b] + threadIdx.x; i < tile_end[b]; i += kBuildBlock) {
        uint32_t c[D];
        if (kind == ARBORX_BOXES) {
            const float *v = values + (int64_t)i * 2 * D;
#pragma unroll
            for (int d = 0; d < D; ++d)
                c[d] = quantise(v[d] + 0.5f * (v[D + d] - v[d]), lo[d], inv[d], bits);
        } else {
            const float *v = values + (int64_t)i * D;
#pragma unroll
            for (int d = 0; d < D; ++d)
                c[d] = quantise(v[d], lo[d], inv[d], bits);
        }
        codes[i] = ((uint64_t)t << mbits) | interleave<D>(c, bits);
        ids[i] = (uint32_t)i;
    }
}

// The segmentation the build uses, made valid whatever the caller's device
// array holds: seg[0] = 0, seg[T] = n, and in between the running maximum of
// the offsets clamped to [0, n], so segments never overlap or leave the value
// array (a valid array is copied unchanged).  One workgroup: an inclusive
// max-scan over chunks of its width.
constexpr int kSegBlock = 1024;

__global__ __launch_bounds__(kSegBlock) void forest_segments(const int64_t *__restrict__ off, int T, int64_t n,
                                                             int64_t *__restrict__ seg)
{
    __shared__ int64_t s_wmax[kSegBlock / kWave];
    __shared__ int64_t s_carry;
    if (threadIdx.x == 0)
        s_carry = 0;
    __syncthreads();
    for (int base = 0; base <= T; base += kSegBlock) {
        const int i = base + (int)threadIdx.x;
        int64_t v = 0;
        if (i == T)
            v = n;
        else if (i > 0 && i < T)
            v = off[i] < 0 ? 0 : (off[i] > n ? n : off[i]);
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {  // inclusive max-scan across the wavefront
            const int64_t u = __shfl_up(v, o, kWave);
            if (lane_id() >= o)
                v = u > v ? u : v;
        }
        if (lane_id() == kWave - 1)
            s_wmax[wave_id()] = v;
        __syncthreads();
        int64_t before = s_carry;
        for (int w = 0; w < wave_id(); ++w)
            before = s_wmax[w] > before ? s_wmax[w] : before;
        v = v > before ? v : before;
        if (i <= T)
            seg[i] = v;
        __syncthreads();
        if (threadIdx.x == kSegBlock - 1)
            s_carry = v;
        __syncthreads();
    }
}

// Tiles that never straddle a tree, from the device segmentation: tree t
// gets ceil(n_t / kForestTile) tiles, placed by an exclusive scan over the
// trees; entries up to max_tiles past the last are empty tiles (no values).
__global__ __launch_bounds__(kSegBlock) void forest_tiles(const int64_t *__restrict__ seg, int T, int max_tiles,
                                                          int32_t *__restrict__ tile_tree,
                                                          int32_t *__restrict__ tile_start,
                                                          int32_t *__restrict__ tile_end)
{
    __shared__ int32_t s_wsum[kSegBlock / kWave];
    __shared__ int32_t s_carry;
    if (threadIdx.x == 0)
        s_carry = 0;
    __syncthreads();
    for (int base = 0; base < T; base += kSegBlock) {
        const int t = base + (int)threadIdx.x;
        const int64_t a = t < T ? seg[t] : 0, e = t < T ? seg[t + 1] : 0;
        const int cnt = (int)((e - a + kForestTile - 1) / kForestTile);
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int u = __shfl_up(incl, o, kWave);
            if (lane_id() >= o)
                incl += u;
        }
        if (lane_id() == kWave - 1)
            s_wsum[wave_id()] = incl;
        __syncthreads();
        int before = s_carry;
        for (int w = 0; w < wave_id(); ++w)
            before += s_wsum[w];
        const int first = before + incl - cnt;
        for (int j = 0; j < cnt && first + j < max_tiles; ++j) {
            const int64_t ts = a + (int64_t)j * kForestTile;
            tile_tree[first + j] = t;
            tile_start[first + j] = (int32_t)ts;
            tile_end[first + j] = (int32_t)(e < ts + kForestTile ? e : ts + kForestTile);
        }
        __syncthreads();
        if (threadIdx.x == kSegBlock - 1)
            s_carry = before + incl;
        __syncthreads();
    }
    for (int j = s_carry + (int)threadIdx.x; j < max_tiles; j += kSegBlock) {
        tile_tree[j] = 0;
        tile_start[j] = 0;
        tile_end[j] = 0;
    }
}

// The build workspace of a forest of n values in T trees, carved from one
// block: tree bounds, tile tables, keys and ids (two each, for the sort),
// arrival flags, the sort's tile histograms, the climb's escapes, and the
// caller's offsets copied in by the build from host offsets.
struct ForestBuildWs {
    uint32_t *tmin, *tmax;
    int32_t *tiles;
    uint64_t *codes, *codes2;
    uint32_t *ids, *ids2;
    unsigned long long *flags;
    uint8_t *rws;
    void *esc;
    int64_t *offs;
};

template <int D>
size_t forest_build_ws(int64_t n, int T, int max_tiles, uint8_t *base, ForestBuildWs *w)
{
    const int64_t nn = n > 0 ? n : 1;
    const int chunks = (int)((nn + chunk_leaves<D>() - 1) / chunk_leaves<D>());
    size_t at = 0;
    auto take = [&](size_t bytes) {
        uint8_t *p = base ? base + at : nullptr;
        at += (bytes + 255) / 256 * 256;
        return p;
    };
    uint8_t *tmin = take(sizeof(uint32_t) * T * D), *tmax = take(sizeof(uint32_t) * T * D);
    uint8_t *tiles = take(sizeof(int32_t) * 3 * (size_t)max_tiles);
    uint8_t *codes = take(8 * nn), *codes2 = take(8 * nn), *ids = take(4 * nn), *ids2 = take(4 * nn);
    uint8_t *flags = take(8 * nn), *rws = take(radix_workspace_bytes(nn));
    uint8_t *esc = take(sizeof(Escape<D>) * escape_entries<D>(chunks)), *offs = take(sizeof(int64_t) * (T + 1));
    if (w) {
        w->tmin = reinterpret_cast<uint32_t *>(tmin);
        w->tmax = reinterpret_cast<uint32_t *>(tmax);
        w->tiles = reinterpret_cast<int32_t *>(tiles);
        w->codes = reinterpret_cast<uint64_t *>(codes);
        w->codes2 = reinterpret_cast<uint64_t *>(codes2);
        w->ids = reinterpret_cast<uint32_t *>(ids);
        w->ids2 = reinterpret_cast<uint32_t *>(ids2);
        w->flags = reinterpret_cast<unsigned long long *>(flags);
        w->rws = rws;
        w->esc = esc;
        w->offs = reinterpret_cast<int64_t *>(offs);
    }
    return at;
}

inline int forest_max_tiles(int64_t n, int T) { return (int)(n / kForestTile) + T + 1; }

// Every device allocation of a forest of n values in T trees: the structure
// and the build workspace.
template <int D>
arborx_status forest_alloc_impl(int64_t n, int T, int kind, ForestDev &f, hipStream_t s)
{
    f.n = n;
    f.dim = D;
    f.kind = kind;
    f.T = T;
    f.max_tiles = forest_max_tiles(n, T);
    arborx_status st;
    if ((st = dalloc((void **)&f.hdrs, sizeof(TreeHeader) * T, s)) != ARBORX_OK ||
        (st = dalloc((void **)&f.seg, sizeof(int64_t) * (T + 1), s)) != ARBORX_OK ||
        (st = dalloc(&f.nodes, (size_t)(n > 0 ? n : 1) * sizeof(Node<D>), s)) != ARBORX_OK ||
        (st = dalloc((void **)&f.leaves, (size_t)(n > 0 ? n : 1) * leaf_floats(D, kind) * sizeof(float), s)) !=
            ARBORX_OK)
        return st;
    const size_t nn = (size_t)(n > 0 ? n : 1);
    if (format_requested(1, D, kind, true) && (st = dalloc(&f.qnodes, nn * sizeof(QNode<D>), s)) != ARBORX_OK)
        return st;
    if (format_requested(2, D, kind, true) && (st = dalloc(&f.wnodes, nn * sizeof(Node4<D>), s)) != ARBORX_OK)
        return st;
    f.bws_bytes = forest_build_ws<D>(n, T, f.max_tiles, nullptr, nullptr);
    return dalloc(&f.bws, f.bws_bytes, s);
}

// Build the forest's trees in place from device-resident values and offsets:
// kernels only (no allocation, no host read, no copy), so the call can be
// captured in a graph and replayed with new contents of the same sizes.
template <int D>
arborx_status forest_rebuild_impl(const float *values, const int64_t *offs, ForestDev &f, hipStream_t s)
{
    AX_HIP(hipGetLastError());
    const int64_t n = f.n;
    const int T = f.T, kind = f.kind, tiles = f.max_tiles;
    ForestBuildWs w;
    forest_build_ws<D>(n, T, tiles, static_cast<uint8_t *>(f.bws), &w);
    int32_t *dtiles = w.tiles;
    forest_segments<<<1, kSegBlock, 0, s>>>(offs, T, n, f.seg);
    forest_tiles<<<1, kSegBlock, 0, s>>>(f.seg, T, tiles, dtiles, dtiles + tiles, dtiles + 2 * tiles);
    fill_kernel<uint32_t><<<grid_for((int64_t)T * D, 256), 256, 0, s>>>(w.tmin, (int64_t)T * D, 0xffffffffu);
    fill_kernel<uint32_t><<<grid_for((int64_t)T * D, 256), 256, 0, s>>>(w.tmax, (int64_t)T * D, 0u);
    {
        ProfScope ps("build_bounds", s);
        forest_tile_bounds<D><<<tiles, kBuildBlock, 0, s>>>(values, kind, dtiles, dtiles + tiles, dtiles + 2 * tiles,
                                                            w.tmin, w.tmax);
        forest_headers<D><<<grid_for(T, 256), 256, 0, s>>>(f.seg, T, w.tmin, w.tmax, f.hdrs);
    }
    AX_HIP(hipGetLastError());
    f.keys = nullptr;
    if (n == 0)
        return ARBORX_OK;
    int tb = 1;
    while ((1 << tb) < T)
        ++tb;
    const int mbits = (63 - tb) / D * D;
    uint64_t *codes = w.codes, *codes2 = w.codes2;
    uint32_t *ids = w.ids, *ids2 = w.ids2;
    {
        ProfScope ps("build_morton", s);
        forest_tile_morton<D><<<tiles, kBuildBlock, 0, s>>>(values, kind, dtiles, dtiles + tiles, dtiles + 2 * tiles,
                                                            f.hdrs, mbits, codes, ids);
    }
    bool alt = false;
    {
        ProfScope ps("build_sort", s);
        AX_HIP(radix_sort_pairs<uint64_t>(codes, ids, codes2, ids2, n, 0, mbits + tb, w.rws, s, &alt));
    }
    if (alt) {
        codes = codes2;
        ids = ids2;
    }
    f.keys = codes;  // kept in the build workspace until the next rebuild: kNN seeds search them
    f.mbits = mbits;
    f.ids = ids;
    constexpr int C = chunk_leaves<D>();
    const int chunks = (int)((n + C - 1) / C);
    Escape<D> *esc = static_cast<Escape<D> *>(w.esc);
    Node<D> *nodes = static_cast<Node<D> *>(f.nodes);
    ProfScope ps("build_hierarchy", s);
    QNode<D> *qnodes = static_cast<QNode<D> *>(f.qnodes);
    hierarchy_chunk_kernel<D><<<chunks, C, 0, s>>>(codes, ids, values, kind, (int)n, nodes, qnodes, f.leaves, w.flags,
                                                   esc, f.seg, T, f.hdrs);
    hierarchy_top<D>(codes, (int)n, kind, nodes, qnodes, w.flags, esc, chunks, f.seg, T, f.hdrs, s);
    if (f.wnodes)
        widen_nodes<D><<<grid_for(n, kBuildBlock), kBuildBlock, 0, s>>>(nodes, (int)n,
                                                                        static_cast<Node4<D> *>(f.wnodes));
    AX_HIP(hipGetLastError());
    return ARBORX_OK;
}

template <int D>
arborx_status forest_build_impl(const float *values, const int64_t *seg_host, int T, int kind, ForestDev &f,
                                hipStream_t s)
{
    arborx_status st = forest_alloc_impl<D>(seg_host[T], T, kind, f, s);
    if (st != ARBORX_OK)
        return st;
    ForestBuildWs w;
    forest_build_ws<D>(f.n, T, f.max_tiles, static_cast<uint8_t *>(f.bws), &w);
    AX_HIP(hipMemcpyAsync(w.offs, seg_host, sizeof(int64_t) * (T + 1), hipMemcpyHostToDevice, s));
    return forest_rebuild_impl<D>(values, w.offs, f, s);
}

}  // namespace

size_t node_bytes(int dim)
{
    switch (dim) {
    case 2: return sizeof(Node<2>);
    case 3: return sizeof(Node<3>);
    case 6: return sizeof(Node<6>);
    default: return 0;
    }
}

arborx_status build_tree(const float *values, int64_t n, int dim, int kind, TreeDev &t, hipStream_t s)
{
    switch (dim) {
    case 2: return build_impl<2>(values, n, kind, t, s);
    case 3: return build_impl<3>(values, n, kind, t, s);
    case 6: return build_impl<6>(values, n, kind, t, s);
    default: return fail(ARBORX_E_UNSUPPORTED, "dimension not compiled in");
    }
}

void forest_release(ForestDev &f, hipStream_t s)
{
    void *const blocks[] = {f.nodes, f.qnodes, f.wnodes, f.leaves, f.hdrs, f.seg, f.ws, f.bws};
    dfree_many(blocks, (int)(sizeof(blocks) / sizeof(blocks[0])), s);
    f.nodes = nullptr;
    f.qnodes = nullptr;
    f.wnodes = nullptr;
    f.leaves = nullptr;
    f.hdrs = nullptr;
    f.seg = nullptr;
    f.ws = nullptr;
    f.ws_bytes = 0;
    f.bws = nullptr;
    f.bws_bytes = 0;
}

arborx_status forest_alloc(int64_t n, int T, int dim, int kind, ForestDev &f, hipStream_t s)
{
    switch (dim) {
    case 2: return forest_alloc_impl<2>(n, T, kind, f, s);
    case 3: return forest_alloc_impl<3>(n, T, kind, f, s);
    case 6: return forest_alloc_impl<6>(n, T, kind, f, s);
    default: return fail(ARBORX_E_UNSUPPORTED, "dimension not compiled in");
    }
}

arborx_status forest_rebuild(const float *values, const int64_t *tree_offsets, ForestDev &f, hipStream_t s)
{
    switch (f.dim) {
    case 2: return forest_rebuild_impl<2>(values, tree_offsets, f, s);
    case 3: return forest_rebuild_impl<3>(values, tree_offsets, f, s);
    case 6: return forest_rebuild_impl<6>(values, tree_offsets, f, s);
    default: return fail(ARBORX_E_UNSUPPORTED, "dimension not compiled in");
    }
}

arborx_status build_forest(const float *values, const int64_t *seg_host, int T, int dim, int kind, ForestDev &f,
                           hipStream_t s)
{
    switch (dim) {
    case 2: return forest_build_impl<2>(values, seg_host, T, kind, f, s);
    case 3: return forest_build_impl<3>(values, seg_host, T, kind, f, s);
    case 6: return forest_build_impl<6>(values, seg_host, T, kind, f, s);
    default: return fail(ARBORX_E_UNSUPPORTED, "dimension not compiled in");
    }
}

hipError_t morton64_points(const float *pts, int64_t n, int dim, const float *bounds, uint64_t *codes, hipStream_t s)
{
    switch (dim) {
    case 2: return morton_impl<2>(pts, n, bounds, codes, s);
    case 3: return morton_impl<3>(pts, n, bounds, codes, s);
    case 6: return morton_impl<6>(pts, n, bounds, codes, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ax
