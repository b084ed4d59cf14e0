// Device-side traversal pieces shared by the single-tree and forest queries:
// the short stack, query predicates, the depth-first spatial walk, the sorted
// register buffers, and the seeded nearest-first kNN walk.
#pragma once

#include <type_traits>

#include "device_util.hpp"
#include "geometry.hpp"
#include "internal.hpp"

namespace ax {
namespace {

// Deepest tree the build can make.  Along a root-to-leaf path the split keys
// (code XOR of neighbouring leaves, or position XOR for equal codes) strictly
// decrease, and two splits with the same highest bit always have a larger
// split between them in sorted order, so no path repeats a highest bit: at
// most 63 code bits + 31 position bits + the leaf edge.
constexpr int kMaxTreeHeight = 95;
// Spill entries behind the LDS ring.  A binary walk pushes at most one entry
// per level, a four-wide walk at most three per four-wide level (two binary
// levels), so no walk ever holds more than 3 * ceil(95 / 2) = 144 deferred
// entries, even with a one-entry ring: the spill area never overflows.
constexpr int kSpill = 160;
static_assert(kSpill >= 3 * ((kMaxTreeHeight + 1) / 2), "spill area below the four-wide walk's bound");

// The ring indices live in registers; only the rarely used spill area (a
// separate private array owned by the caller) sits in scratch memory.  Keeping
// the array out of this struct lets the compiler hold the counters in
// registers instead of reloading them from scratch on every push and pop.
template <typename E>
struct ShortStack {
    E *lds;  // this thread's column: entry j at lds[j << shift] (the stride is the block size, a power of two)
    E *spill;
    int shift, mask;
    int base = 0, cnt = 0, ns = 0;
    __device__ ShortStack(E *col, int stride, int cap, E *spill_) : lds(col), spill(spill_), shift(__ffs(stride) - 1),
                                                                     mask(cap - 1) {}
    __device__ __forceinline__ bool empty() const { return cnt == 0 && ns == 0; }
    __device__ __forceinline__ void clear() { base = cnt = ns = 0; }
    __device__ __forceinline__ void push(E x)
    {
        if (cnt == mask + 1) {  // ring full: move the oldest LDS entry to the spill area
            if (ns < kSpill)    // always true (see kSpill); the check only keeps the store in bounds
                spill[ns++] = lds[(base & mask) << shift];
            ++base;
            --cnt;
        }
        lds[((base + cnt) & mask) << shift] = x;
        ++cnt;
    }
    // The newest spilled entry sits just below the ring's oldest one: when the
    // ring is empty it moves back first, so every pop reads LDS.
    __device__ __forceinline__ E pop()
    {
        if (cnt == 0) {
            --base;
            lds[(base & mask) << shift] = spill[--ns];
            cnt = 1;
        }
        --cnt;
        return lds[((base + cnt) & mask) << shift];
    }
};

// The deferred subtrees of a walk over codes.  A step reads the top before it
// knows whether it needs it, so that the read runs beside the node's fetch,
// and writes the entry above the top without asking whether it counts; moving
// `at` decides, with no branch.  at, lim and stride are LDS byte offsets in
// this thread's column of `slots` (at least 2) entries, words of type E; slot 0 holds the entry
// that ends the walk, the last one only what is written above a full stack.
// A stack of slots - 2 entries is full: deeper ones go to a private array and
// come back from it (the two branches below, taken only there).
template <typename E>
struct TopStack {
    typedef __attribute__((address_space(3))) char *Lds;
    Lds at;
    Lds lim;
    int stride;
    E *spill;
    int ns = 0;
    __device__ __forceinline__ TopStack(E *col, int threads, int slots, E *spill_, E end)
        : stride(threads * (int)sizeof(E)), spill(spill_)
    {
        at = (Lds)(__attribute__((address_space(3))) E *)col;
        lim = at + (slots > 2 ? slots - 2 : 0) * stride;
        *(__attribute__((address_space(3))) E *)at = end;
    }
    __device__ __forceinline__ E top() const { return *(__attribute__((address_space(3))) E *)at; }
    __device__ __forceinline__ void put(E x) const { *(__attribute__((address_space(3))) E *)(at + stride) = x; }
    // both: the entry put above the top stays; none: the top is taken
    __device__ __forceinline__ void move(bool both, bool none, E x, E &taken)
    {
        int by = both ? stride : (none ? -stride : 0);
        if (at == lim && (both || ns > 0)) {
            if (both) {
                if (ns < kSpill)  // always true (see kSpill); keeps the store in bounds
                    spill[ns] = x;
                ++ns;
                by = 0;
            } else if (none) {
                --ns;
                taken = spill[ns < kSpill ? ns : kSpill - 1];
                by = 0;
            }
        }
        at += by;
    }
};

// Blocks are dealt round-robin over the 8 XCDs; renumber them so that each
// XCD (and its L2) works on one contiguous run of ordered queries.
__device__ __forceinline__ int64_t xcd_block()
{
    constexpr int64_t X = 8;
    const int64_t b = blockIdx.x, G = gridDim.x;
    const int64_t q = G / X, r = G % X, x = b % X;
    return x * q + (x < r ? x : r) + b / X;
}

template <int D>
struct Sphere {
    float c[D];
    float r2;
    __device__ __forceinline__ bool hit(const float *lo, const float *hi, float &d2) const
    {
        d2 = box_d2<D>(c, lo, hi);
        return d2 <= r2;
    }
    __device__ __forceinline__ void load(const float *q, int64_t i, float rr)
    {
#pragma unroll
        for (int d = 0; d < D; ++d)
            c[d] = q[i * D + d];
        r2 = rr;
    }
    __device__ __forceinline__ void dead()  // matches nothing: d2 >= 0 > r2
    {
#pragma unroll
        for (int d = 0; d < D; ++d)
            c[d] = 0.0f;
        r2 = -1.0f;
    }
};

template <int D>
struct BoxQuery {
    float lo[D], hi[D];
    __device__ __forceinline__ bool hit(const float *blo, const float *bhi, float &d2) const
    {
        d2 = 0.0f;
        return boxes_overlap<D>(lo, hi, blo, bhi);
    }
    __device__ __forceinline__ void load(const float *q, int64_t i, float)
    {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = q[i * 2 * D + d];
            hi[d] = q[i * 2 * D + D + d];
        }
    }
    __device__ __forceinline__ void dead()  // an empty box overlaps nothing
    {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = INFINITY;
            hi[d] = -INFINITY;
        }
    }
};

// Squared distance from q to the point stored in a leaf child's words: box_d2
// of the degenerate box, bit for bit.
template <int D>
__device__ __forceinline__ float point_d2(const float *q, const uint32_t (&w)[D])
{
#pragma clang fp contract(off)
    float acc = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const float t = q[d] - __uint_as_float(w[d]);
        const float s = t * t;
        acc = acc + s;
    }
    return acc;
}

// A ray o + t*dir, t >= 0 (Section 2.5).  It meets a closed box when its slab
// intervals overlap: slabs taken in dimension order from tmin = 0, tmax =
// +inf, t1 = (lo - o)/dir and t2 = (hi - o)/dir with correctly rounded
// division, a zero direction component requiring lo <= o <= hi.  The entry
// parameter tmin is reported in the distance slot.  Subtraction and division
// are monotone, so a box inside another is met no earlier: pruning by a
// parent's box is exact.  An internal box only has to be entered whenever that
// test passes, so reach() multiplies by 1/dir and widens the result: t' =
// fl(x fl(1/dir)) is within a factor 1 +- 2^-22 of fl(x/dir), or 2^-147 where it
// is that small.  The walks divide for leaf boxes that pass reach() alone: a
// correctly rounded division is about ten instructions, and a step had twelve
// in 3D: the all-hits walk of 3*10^5 rays over 10^6 boxes 2.78 -> 2.41 ms.  Rays
// with components for which the bound does not hold take hit().
template <int D>
struct RayPred {
    float o[D], dir[D], inv[D];
    bool plain;  // reach() may multiply
    __device__ __forceinline__ void load(const float *rays, int64_t i, float)
    {
        plain = true;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            o[d] = rays[i * 2 * D + d];
            dir[d] = rays[i * 2 * D + D + d];
            const float a = fabsf(dir[d]);
            plain = plain && fabsf(o[d]) < INFINITY && (a == 0.0f || (a >= 0x1p-100f && a <= 0x1p100f));
            inv[d] = 1.0f / dir[d];
        }
    }
    __device__ __forceinline__ void dead()  // origin at +inf, no direction: outside every finite box
    {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            o[d] = INFINITY;
            dir[d] = inv[d] = 0.0f;
        }
        plain = false;
    }
    // True whenever hit() is, with t at most its t.  A NaN bound of a box acts as in hit().
    __device__ __forceinline__ bool reach(const float *lo, const float *hi, float &t) const
    {
        if (!plain)
            return hit(lo, hi, t);
        float tmin = 0.0f, tmax = INFINITY;
        bool inside = true;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (dir[k] == 0.0f) {
                inside = inside && !(o[k] < lo[k] || o[k] > hi[k]);
                continue;
            }
            const float t1 = (lo[k] - o[k]) * inv[k];
            const float t2 = (hi[k] - o[k]) * inv[k];
            const bool up = t1 < t2;
            tmin = fmaxf(tmin, up ? t1 : t2);
            tmax = fminf(tmax, up ? t2 : t1);
        }
        t = fmaf(tmin, 1.0f - 0x1p-20f, -0x1p-120f);
        return inside && tmin <= fmaf(tmax, 1.0f + 0x1p-20f, 0x1p-120f);
    }
    __device__ __forceinline__ bool hit(const float *lo, const float *hi, float &t) const
    {
        float tmin = 0.0f, tmax = INFINITY;
        bool inside = true;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (dir[k] == 0.0f) {
                inside = inside && !(o[k] < lo[k] || o[k] > hi[k]);
                continue;
            }
            const float t1 = (lo[k] - o[k]) / dir[k];
            const float t2 = (hi[k] - o[k]) / dir[k];
            const float tn = t1 < t2 ? t1 : t2, tf = t1 < t2 ? t2 : t1;
            tmin = tn > tmin ? tn : tmin;
            tmax = tf < tmax ? tf : tmax;
        }
        t = tmin;
        return inside && !(tmin > tmax);
    }
};

// The predicate's first test of a node's child box, and its test of one with
// child reference ref: for rays reach(), and for leaf boxes that pass it hit().
template <int D, class P>
__device__ __forceinline__ bool first_hit(const P &pred, const float *lo, const float *hi, float &d)
{
    if constexpr (std::is_same<P, RayPred<D>>::value)
        return pred.reach(lo, hi, d);
    else
        return pred.hit(lo, hi, d);
}
template <int D, class P>
__device__ __forceinline__ bool child_hit(const P &pred, const float *lo, const float *hi, int ref, float &d)
{
    bool h = first_hit<D>(pred, lo, hi, d);
    if (std::is_same<P, RayPred<D>>::value && h && ref < 0)
        h = pred.hit(lo, hi, d);
    return h;
}

// Exact test of the sorted leaf record `pos` (the value's own box) against
// the predicate, calling f(index, d2) on a match.
template <int D, class P, class F>
__device__ __forceinline__ void leaf_exact(const float *__restrict__ leaves, int kind, int pos, const P &pred, F &f)
{
    const float *lf = leaves + (int64_t)pos * leaf_floats(D, kind);
    float lo[D], hi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        lo[d] = lf[d];
        hi[d] = kind == ARBORX_BOXES ? lf[D + d] : lf[d];
    }
    float d2;
    if (pred.hit(lo, hi, d2))
        f(__float_as_int(lf[kind == ARBORX_BOXES ? 2 * D : D]), d2);
}

struct NeverStop {
    __device__ __forceinline__ constexpr bool operator()() const { return false; }
};

// Depth-first walk calling f(index, d2) on every matching value; with a stop
// functor, the walk ends as soon as stop() holds after a node's matches were
// reported (the early termination of Section 2.2).
// The next node is chosen and its fetch issued before the matches are reported
// (and a ray's leaf boxes divided for): 10^5 2D rays over 3*10^5 boxes 6.1 ->
// 5.2 ms, box overlaps of 10^6 2D boxes 190 -> 186 us.
// Rays over more boxes than the caches hold are bound by the bytes behind L2:
// neighbouring rays part after a few nodes, and all hits of 10^6 rays over 2*10^6
// boxes read 36 GB in 8.0 ms (a third of the fetches hit L2), nine tenths of the
// rate of a large copy.
// A depth-first walk enters each internal node at most once, so `limit`
// iterations (more than the node count) bound every walk even on a corrupt
// tree, and node indices are range-checked before use.
template <int D, class P, class F, class S = NeverStop>
__device__ __forceinline__ void traverse_spatial(const Node<D> *__restrict__ nodes, int root, int n_nodes,
                                                 const P &pred, ShortStack<int> &st, F &f, const S &stop = S())
{
    constexpr bool two = std::is_same<P, RayPred<D>>::value;  // leaf boxes that pass the first test take a second
    const unsigned last = (unsigned)n_nodes - 1u;
    int cur = root;
    Node<D> nd;
    load_node(nodes, (int)min((unsigned)cur, last), nd);
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur > last)
            break;
        const Node<D> at = nd;
        float d0, d1;
        const int c0 = at.child[0], c1 = at.child[1];
        const bool h0 = first_hit<D>(pred, at.lo[0], at.hi[0], d0);
        const bool h1 = first_hit<D>(pred, at.lo[1], at.hi[1], d1);
        if (h0 && c0 >= 0) {
            if (h1 && c1 >= 0)
                st.push(c1);
            cur = c0;
        } else if (h1 && c1 >= 0) {
            cur = c1;
        } else {
            cur = st.empty() ? -1 : st.pop();
        }
        load_node(nodes, (int)min((unsigned)cur, last), nd);  // in flight while the matches below are reported
        if (h0 && c0 < 0 && c0 != kEmptyRef && (!two || pred.hit(at.lo[0], at.hi[0], d0)))
            f(~c0, d0);
        if (h1 && c1 < 0 && c1 != kEmptyRef && (!two || pred.hit(at.lo[1], at.hi[1], d1)))
            f(~c1, d1);
        if (stop())
            break;
    }
}

// The depth-first walk over four-wide nodes: one fetch tests up to four
// subtrees; matching leaf slots are reported, the first matching internal slot
// is entered and the others are deferred on the stack.
template <int D, class P, class F>
__device__ __forceinline__ void traverse_spatial4(const Node4<D> *__restrict__ nodes, int root, int n_nodes,
                                                  const P &pred, ShortStack<int> &st, F &f)
{
    int cur = root;
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        Node4<D> nd;
        load_node4(nodes, cur, nd);
        int next = -1;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            float d;
            const bool h = pred.hit(nd.lo[s], nd.hi[s], d);
            const int c = nd.child[s];
            if (h && c < 0 && c != kEmptyRef)
                f(~c, d);
            if (h && c >= 0) {
                if (next >= 0)
                    st.push(next);
                next = c;
            }
        }
        cur = next >= 0 ? next : (st.empty() ? -1 : st.pop());
    }
}

// Packet walk: one thread answers NQ queries (Morton neighbours) in a single
// depth-first walk over the union of their paths.  A child is entered when
// any query's predicate admits it; leaves are tested per query, calling
// f(j, index, d2) for query j.  Neighbouring queries share most of their
// paths, so a thread makes fewer dependent node fetches per query.
template <int D, int NQ, class P, class F>
__device__ __forceinline__ void traverse_spatial_packet(const Node<D> *__restrict__ nodes, int root, int n_nodes,
                                                        const P (&pred)[NQ], ShortStack<int> &st, F &f)
{
    int cur = root;
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        Node<D> nd;
        load_node(nodes, cur, nd);
        const int c0 = nd.child[0], c1 = nd.child[1];
        bool g0 = false, g1 = false;
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            float d0, d1;
            const bool h0 = pred[j].hit(nd.lo[0], nd.hi[0], d0);
            const bool h1 = pred[j].hit(nd.lo[1], nd.hi[1], d1);
            if (h0 && c0 < 0 && c0 != kEmptyRef)
                f(j, ~c0, d0);
            if (h1 && c1 < 0 && c1 != kEmptyRef)
                f(j, ~c1, d1);
            g0 = g0 | h0;
            g1 = g1 | h1;
        }
        g0 = g0 && c0 >= 0;
        g1 = g1 && c1 >= 0;
        if (g0) {
            if (g1)
                st.push(c1);
            cur = c0;
        } else if (g1) {
            cur = c1;
        } else {
            if (st.empty())
                break;
            cur = st.pop();
        }
    }
}

// Wavefront-packet form of the walk: the 64 lanes (64 Morton-neighbouring
// queries) visit the union of their paths together.  The node index is the
// same in every lane, so each node is fetched once per wavefront through the
// scalar cache, and the stack of deferred nodes is one per wavefront in LDS.
// A stack entry is pushed only at a level where some lane needs both
// children, so its depth never exceeds the tree height (kMaxTreeHeight),
// below kWaveStack.  Lanes without a query
// (`active` false) carry a predicate that matches nothing.
constexpr int kWaveStack = 128;
static_assert(kWaveStack > kMaxTreeHeight, "wavefront stack below the tree height bound");

template <int D, class P, class F>
__device__ __forceinline__ void traverse_spatial_wave(const Node<D> *__restrict__ nodes, int root, int n_nodes,
                                                      const P &pred, int *wstack, F &f)
{
    int sp = 0;
    int cur = root;
    for (int iter = 0; iter <= n_nodes; ++iter) {
        cur = __builtin_amdgcn_readfirstlane(cur);
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        Node<D> nd;
        load_node(nodes, cur, nd);
        float d0, d1;
        bool h0 = pred.hit(nd.lo[0], nd.hi[0], d0);
        bool h1 = pred.hit(nd.lo[1], nd.hi[1], d1);
        const int c0 = nd.child[0], c1 = nd.child[1];
        if (c0 < 0) {
            if (h0 && c0 != kEmptyRef)
                f(~c0, d0);
            h0 = false;
        }
        if (c1 < 0) {
            if (h1 && c1 != kEmptyRef)
                f(~c1, d1);
            h1 = false;
        }
        const bool any0 = __ballot(h0) != 0, any1 = __ballot(h1) != 0;
        if (any0) {
            if (any1) {
                if (sp < kWaveStack)
                    wstack[sp] = c1;
                ++sp;
            }
            cur = c0;
        } else if (any1) {
            cur = c1;
        } else {
            if (sp == 0)
                break;
            --sp;
            cur = sp < kWaveStack ? wstack[sp] : -1;
        }
    }
}

// Stackless walk with ropes (the paper's spatial traversal, Section 2.6).  The
// walk position is a child slot (node p, side).  Its rope, the slot the
// depth-first order visits after the whole subtree in it, needs no storage:
// after (p, left) comes (p, right); the right child of p covers leaves
// [p + 1, range_r(p)], and the next subtree in leaf order is the right child
// of the node splitting leaves range_r(p) and range_r(p) + 1, i.e. (range_r(p),
// right), unless range_r(p) is the last leaf of the tree.  Every slot is tested
// at most once, so 2 * n_nodes steps bound the walk.
template <int D, class P, class F>
__device__ __forceinline__ void traverse_spatial_rope(const Node<D> *__restrict__ nodes, int root, int n_nodes,
                                                      int last_leaf, const P &pred, F &f)
{
    int p = root, side = 0;
    Node<D> nd;
    int loaded = -1;
    for (int iter = 0; iter <= 2 * n_nodes; ++iter) {
        if ((unsigned)p >= (unsigned)n_nodes)
            break;
        if (p != loaded) {
            load_node(nodes, p, nd);
            loaded = p;
        }
        float lo[D], hi[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = side ? nd.lo[1][d] : nd.lo[0][d];
            hi[d] = side ? nd.hi[1][d] : nd.hi[0][d];
        }
        const int c = side ? nd.child[1] : nd.child[0];
        float d2;
        if (c != kEmptyRef && pred.hit(lo, hi, d2)) {
            if (c >= 0) {
                p = c;
                side = 0;
                continue;
            }
            f(~c, d2);
        }
        if (side == 0) {
            side = 1;
        } else {
            if (nd.range_r >= last_leaf)
                break;
            p = nd.range_r;
        }
    }
}

// Pair-search walk (Section 2.6 names a dedicated traversal for searching
// pairs of objects) for the value at sorted position p of a single tree: the
// rope walk started at p's own rope.  In depth-first order the slot after leaf
// p is (node p, right side) -- node p separates leaves p and p + 1, whichever
// of nodes p - 1 and p holds the leaf -- and the ropes from there reach
// exactly the subtrees of positions p + 1 .. last_leaf.  So each unordered
// pair of values is met once, from its earlier position, and no walk touches
// the part of the tree before its own leaf.  f(q, index, d2) gets the
// partner's sorted position (a leaf in slot (node, side) sits at position
// node + side), its value index and its distance.
template <int D, class P, class F>
__device__ __forceinline__ void traverse_pairs_after(const Node<D> *__restrict__ nodes, int n_nodes, int p,
                                                     int last_leaf, const P &pred, F &f)
{
    if (p >= last_leaf)
        return;
    int cur = p, side = 1;
    Node<D> nd;
    int loaded = -1;
    for (int iter = 0; iter <= 2 * n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        if (cur != loaded) {
            load_node(nodes, cur, nd);
            loaded = cur;
        }
        float lo[D], hi[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lo[d] = side ? nd.lo[1][d] : nd.lo[0][d];
            hi[d] = side ? nd.hi[1][d] : nd.hi[0][d];
        }
        const int c = side ? nd.child[1] : nd.child[0];
        float d2;
        if (c != kEmptyRef && pred.hit(lo, hi, d2)) {
            if (c >= 0) {
                cur = c;
                side = 0;
                continue;
            }
            f(cur + side, ~c, d2);
        }
        if (side == 0) {
            side = 1;
        } else {
            if (nd.range_r >= last_leaf)
                break;
            cur = nd.range_r;
        }
    }
}

// Top-down packet form of the pair-search walk: one thread takes the NQ
// consecutive sorted positions p0 .. p0 + NQ - 1 of a single tree and walks
// from the root over the union of their paths.  Node c separates leaves c and
// c + 1, so its left child holds positions [range_l, c] and its right child
// [c + 1, range_r]; query j enters a child only if the child's box admits it
// and the child holds a position after p0 + j.  Each unordered pair is thus
// reported once, to the query at its earlier position, as
// f(j, partner position, partner index, d2); the walk over the shared upper
// levels is paid once per NQ queries.  Queries past the tree carry a
// predicate that matches nothing.
template <int D, int NQ, class P, class F>
__device__ __forceinline__ void traverse_pairs_packet(const Node<D> *__restrict__ nodes, int root, int n_nodes, int p0,
                                                      const P (&pred)[NQ], ShortStack<int> &st, F &f)
{
    int cur = root;
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        Node<D> nd;
        load_node(nodes, cur, nd);
        const int c0 = nd.child[0], c1 = nd.child[1];
        bool g0 = false, g1 = false;
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            float d0, d1;
            const bool h0 = cur > p0 + j && pred[j].hit(nd.lo[0], nd.hi[0], d0);
            const bool h1 = nd.range_r > p0 + j && pred[j].hit(nd.lo[1], nd.hi[1], d1);
            if (h0 && c0 < 0 && c0 != kEmptyRef)
                f(j, cur, ~c0, d0);
            if (h1 && c1 < 0 && c1 != kEmptyRef)
                f(j, cur + 1, ~c1, d1);
            g0 = g0 | h0;
            g1 = g1 | h1;
        }
        g0 = g0 && c0 >= 0;
        g1 = g1 && c1 >= 0;
        if (g0) {
            if (g1)
                st.push(c1);
            cur = c0;
        } else if (g1) {
            cur = c1;
        } else {
            if (st.empty())
                break;
            cur = st.pop();
        }
    }
}

// Both child boxes of a quantized node in the tree's frame; `points` says the
// tree holds points, whose leaf children are stored exactly.
template <int D>
__device__ __forceinline__ void qboxes(const QNode<D> &nd, bool points, const float *flo, const float *fsc,
                                       float (&lo)[2][D], float (&hi)[2][D])
{
    qchild<D>(nd, 0, points && nd.child[0] < 0, flo, fsc, lo[0], hi[0]);
    qchild<D>(nd, 1, points && nd.child[1] < 0, flo, fsc, lo[1], hi[1]);
}

// The short-stack walk over quantized nodes.  Internal child boxes decode to
// supersets of the true boxes, so no matching subtree is skipped.  A point
// tree's leaf child is exact in the node and reported from it; a box tree's
// leaf whose decoded box passes is tested exactly on its leaf record.  (An
// empty slot's bytes are never reported: its reference is checked first.)
// An optional stop functor ends the walk as in traverse_spatial.
template <int D, class P, class F, class S = NeverStop>
__device__ __forceinline__ void traverse_spatial_q(const QNode<D> *__restrict__ nodes, const TreeHeader &h,
                                                   int n_nodes, const float *__restrict__ leaves, int kind,
                                                   const P &pred, ShortStack<int> &st, F &f, const S &stop = S())
{
    const bool points = kind != ARBORX_BOXES;
    float flo[D], fsc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        flo[d] = h.lo[d];
        fsc[d] = h.qscale[d];
    }
    int cur = h.root;
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        QNode<D> nd;
        load_qnode(nodes, cur, nd);
        float lo[2][D], hi[2][D];
        qboxes<D>(nd, points, flo, fsc, lo, hi);
        float d0, d1;
        const int c0 = nd.child[0], c1 = nd.child[1];
        // a box tree's leaf box is decided by leaf_exact
        bool h0 = child_hit<D>(pred, lo[0], hi[0], points ? c0 : 0, d0);
        bool h1 = child_hit<D>(pred, lo[1], hi[1], points ? c1 : 0, d1);
        if (h0 && c0 < 0) {
            if (c0 != kEmptyRef) {
                if (points)
                    f(~c0, d0);
                else
                    leaf_exact<D>(leaves, kind, ~c0, pred, f);
            }
            h0 = false;
        }
        if (h1 && c1 < 0) {
            if (c1 != kEmptyRef) {
                if (points)
                    f(~c1, d1);
                else
                    leaf_exact<D>(leaves, kind, ~c1, pred, f);
            }
            h1 = false;
        }
        if (stop())
            break;
        if (h0) {
            if (h1)
                st.push(c1);
            cur = c0;
        } else if (h1) {
            cur = c1;
        } else {
            if (st.empty())
                break;
            cur = st.pop();
        }
    }
}

// Packet walk over the quantized nodes of a tree of boxes: as
// traverse_spatial_packet, one decode of the node's child boxes serving all NQ
// queries; leaves whose decoded box passes are decided on their records.
template <int D, int NQ, class P, class F>
__device__ __forceinline__ void traverse_spatial_packet_q(const QNode<D> *__restrict__ nodes, const TreeHeader &h,
                                                          int n_nodes, const float *__restrict__ leaves,
                                                          const P (&pred)[NQ], ShortStack<int> &st, F &f)
{
    float flo[D], fsc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        flo[d] = h.lo[d];
        fsc[d] = h.qscale[d];
    }
    int cur = h.root;
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        QNode<D> nd;
        load_qnode(nodes, cur, nd);
        float lo[2][D], hi[2][D];
        qboxes<D>(nd, false, flo, fsc, lo, hi);
        const int c0 = nd.child[0], c1 = nd.child[1];
        bool g0 = false, g1 = false;
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            float d0, d1;
            const bool h0 = pred[j].hit(lo[0], hi[0], d0);
            const bool h1 = pred[j].hit(lo[1], hi[1], d1);
            auto fj = [&](int idx, float d) { f(j, idx, d); };
            if (h0 && c0 < 0 && c0 != kEmptyRef)
                leaf_exact<D>(leaves, ARBORX_BOXES, ~c0, pred[j], fj);
            if (h1 && c1 < 0 && c1 != kEmptyRef)
                leaf_exact<D>(leaves, ARBORX_BOXES, ~c1, pred[j], fj);
            g0 = g0 | h0;
            g1 = g1 | h1;
        }
        g0 = g0 && c0 >= 0;
        g1 = g1 && c1 >= 0;
        if (g0) {
            if (g1)
                st.push(c1);
            cur = c0;
        } else if (g1) {
            cur = c1;
        } else {
            if (st.empty())
                break;
            cur = st.pop();
        }
    }
}

// Distances in the codes of a tree's frame, in units of its largest step: the
// sum of the squared gaps of the dimensions between a query's code words and a
// child's words is at most the squared distance.  In a frame with one step the
// sum is of whole numbers (a saturating pair subtraction and a dot product a
// dimension); in one with a step for each dimension it is of floats, every gap
// times its step (five instructions a dimension).
template <int D, bool EVEN>
struct CodeMetric {
    typedef uint32_t Sum;
    __device__ __forceinline__ explicit CodeMetric(const TreeHeader &) {}
    __device__ __forceinline__ double inv(const TreeHeader &h, int) const { return h.qinv; }
    __device__ __forceinline__ double weight(int) const { return 1.0; }
    __device__ __forceinline__ Sum gap2(const uint32_t (&q)[D], const uint32_t (&w)[D]) const
    {
        return code_gap2<D>(q, w);
    }
    // a bound on the sum from one on the squared distance, at least as large
    __device__ __forceinline__ static Sum bound(double r)
    {
        return r < 4294967295.0 ? (uint32_t)fmax(r, 0.0) : UINT32_MAX;
    }
};
template <int D>
struct CodeMetric<D, false> {
    typedef float Sum;
    float wt[D];
    __device__ __forceinline__ explicit CodeMetric(const TreeHeader &h)
    {
#pragma unroll
        for (int d = 0; d < D; ++d)
            wt[d] = h.qweight[d];
    }
    __device__ __forceinline__ double inv(const TreeHeader &h, int d) const { return h.qinvs[d]; }
    __device__ __forceinline__ double weight(int d) const { return (double)wt[d]; }
    __device__ __forceinline__ float gap(uint32_t q, uint32_t w, int d) const
    {
        const ushort2_t one = {1, 1};
        return (float)__builtin_amdgcn_udot2(code_gap(q, w), one, 0u, false) * wt[d];
    }
    __device__ __forceinline__ Sum gap2(const uint32_t (&q)[D], const uint32_t (&w)[D]) const
    {
        float acc = 0.0f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const float g = gap(q[d], w[d], d);
            acc = fmaf(g, g, acc);
        }
        return acc;
    }
    __device__ __forceinline__ static Sum bound(double r)
    {
        return r < 3.0e38 ? (float)(fmax(r, 0.0) * (1.0 + 0x1p-22)) : INFINITY;
    }
};

// A ball around a query in these codes: a box whose gaps sum to more than r2
// holds no value within the radius.  A value matches when its float32 squared
// distance, within a factor 1 +- 2^-20 and 16 * 2^-149 of the real one, is at
// most the ball's; a float sum of gaps is off by a factor of 1 +- 2^-20 too.  A
// query outside the frame takes the excess e past it off the gaps of that
// dimension: (e + g)^2 = e^2 + g (2 e + g), so r2 lacks the sum of the e^2, and
// a search whose radius is about e long also counts the middle terms
// (CodeExcess).  A ball that does not reach the frame meets only boxes that
// span it.
template <int D, class Sum>
struct CodeBall {
    uint32_t q[D];
    Sum r2;
};
template <int D, bool EVEN>
__device__ __forceinline__ void code_ball(const float (&c)[D], float r2, const TreeHeader &h,
                                          const CodeMetric<D, EVEN> &metric,
                                          CodeBall<D, typename CodeMetric<D, EVEN>::Sum> &ball)
{
    double past = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        double e;
        ball.q[d] = code_query(c[d], h.lo[d], metric.inv(h, d), e);
        e *= metric.weight(d) * (EVEN ? 1.0 : 1.0 - 0x1p-22);
        past += e * e;
    }
    const double r = ((double)r2 * (1.0 + (EVEN ? 0x1p-18 : 0x1p-17)) + 0x1p-144) * h.qinv * h.qinv *
                         (1.0 + 0x1p-30) + (EVEN ? 1.0 : 0.0) - fmin(past, 1.0e300);
    ball.r2 = metric.bound(r);
    if (r < 0.0) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            ball.q[d] = 0;
    }
}

// Depth-first walk of NQ neighbouring sphere queries over the quantized nodes
// of a tree of points, in the codes of its frame: an internal child costs one
// saturating pair subtraction and one dot product per dimension instead of
// twelve instructions to decode and test it, a leaf child its exact distance
// from the node's words; both are formed and one is taken.  The next node is
// chosen and its fetch issued before the matches of this one are reported:
// f(j, hit0, index0, d0, hit1, index1, d1) tells which of the node's leaf
// children query j matches.  With PAIRS it is the pair walk of the leaf at
// sorted position lpos: only later positions match, and f gets `at`, the
// position of the left leaf (the right one is at + 1), first; node c
// separates leaves c and c + 1, so a left child [l, c] is entered when c >
// lpos and a right one always (its range ends where its parent's does).
// Bound: two 16-byte loads a visit (four in 6D), which leave the compute unit
// at about 1.3 lane-loads a clock, then vector instructions (busy 0.6 of the
// time in the CSR count at 10^7 cube points).  Against the decoded boxes that
// walk fell from 1.5e9 to 1.0e9 vector instructions and from 3.28 to 2.70 ms;
// CSR with distances of 5*10^5 6D mixture points, build included, from 3.95
// to 3.09 ms; DBSCAN of 5*10^6 points from 5.3 to 4.7 ms.
template <int D, int NQ, bool PAIRS, bool EVEN, class F, class S = NeverStop>
__device__ __forceinline__ void traverse_codes(const QNode<D> *__restrict__ nodes, const TreeHeader &h, int n_nodes,
                                               const Sphere<D> (&pred)[NQ], int lpos, TopStack<int> &st, F &f,
                                               const S &stop = S())
{
    const CodeMetric<D, EVEN> metric(h);
    CodeBall<D, typename CodeMetric<D, EVEN>::Sum> ball[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j)
        code_ball<D, EVEN>(pred[j].c, pred[j].r2, h, metric, ball[j]);
    const unsigned last = (unsigned)n_nodes - 1u;
    int cur = h.root;
    QNode<D> nd;
    load_qnode(nodes, (int)min((unsigned)cur, last), nd);
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur > last)
            break;
        int deferred = st.top();
        const int c0 = nd.child[0], c1 = nd.child[1];
        st.put(c1);
        bool g0 = false, g1 = false, h0[NQ], h1[NQ];
        float d0[NQ], d1[NQ];
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            g0 = g0 | (metric.gap2(ball[j].q, nd.w[0]) <= ball[j].r2);
            g1 = g1 | (metric.gap2(ball[j].q, nd.w[1]) <= ball[j].r2);
            d0[j] = point_d2<D>(pred[j].c, nd.w[0]);
            d1[j] = point_d2<D>(pred[j].c, nd.w[1]);
            h0[j] = c0 < 0 && (!PAIRS || cur > lpos) && d0[j] <= pred[j].r2;
            h1[j] = c1 < 0 && (!PAIRS || cur >= lpos) && d1[j] <= pred[j].r2;
        }
        g0 = g0 && c0 >= 0 && (!PAIRS || cur > lpos);
        g1 = g1 && c1 >= 0;
        const int at = cur;
        st.move(g0 && g1, !(g0 || g1), c1, deferred);
        cur = g0 ? c0 : (g1 ? c1 : deferred);
        load_qnode(nodes, (int)min((unsigned)cur, last), nd);  // in flight while the matches below are reported
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            if constexpr (PAIRS)
                f(at, h0[j], ~c0, h1[j], ~c1);
            else
                f(j, h0[j], ~c0, d0[j], h1[j], ~c1, d1[j]);
        }
        if (stop())
            break;
    }
}

// A reporter for traverse_codes from f(j, index, d2): one call for a node's
// first match and a rarer one for a second, instead of one for each slot.
template <class F>
struct EachHit {
    F &f;
    __device__ __forceinline__ void operator()(int j, bool h0, int i0, float d0, bool h1, int i1, float d1) const
    {
        if (h0 || h1) {
            f(j, h0 ? i0 : i1, h0 ? d0 : d1);
            if (h0 && h1)
                f(j, i1, d1);
        }
    }
};
template <class F>
__device__ __forceinline__ EachHit<F> each_hit(F &f)
{
    return EachHit<F>{f};
}

// One term of the fixed-point distance sum: trunc(sqrtf(d2) * scale), scale
// a power of two.
__device__ __forceinline__ long long fixed_term(float d2, float scale)
{
    const float dist = sqrtf(d2);       // correctly rounded
    const float scaled = dist * scale;  // exact: scale is a power of two
    return (long long)(unsigned long long)scaled;  // scaled >= 0: the unsigned conversion is shorter
}

// Store x in slot k of buf (k < C), with static indices only.
template <int C, typename T>
__device__ __forceinline__ void append_at(T (&buf)[C], int k, T x)
{
#pragma unroll
    for (int s = 0; s < C; ++s)
        buf[s] = s == k ? x : buf[s];
}

// Ascending bitonic sorting network over C (a power of two) registers.
template <int C, typename T>
__device__ __forceinline__ void sort_network(T (&v)[C])
{
#pragma unroll
    for (int k = 2; k <= C; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const int l = i ^ j;
                if (l > i) {
                    const T a = v[i], b = v[l];
                    const bool up = (i & k) == 0;
                    const T lo = a < b ? a : b, hi = a < b ? b : a;
                    v[i] = up ? lo : hi;
                    v[l] = up ? hi : lo;
                }
            }
}

struct alignas(8) KnnEntry {  // read and written as one word, also as a KnnCode
    int32_t ref;
    float d2;
};
// A deferred subtree of a kNN walk over codes: its squared gap above its
// reference, one word of a TopStack.
typedef uint64_t KnnCode;
static_assert(sizeof(KnnCode) == sizeof(KnnEntry) && alignof(KnnCode) == alignof(KnnEntry),
              "the two share a stack area");
__device__ __forceinline__ KnnCode knn_code(int32_t ref, uint32_t gap2) { return ((uint64_t)gap2 << 32) | (uint32_t)ref; }

// Minimum and maximum of two top-k keys held as doubles.  The bit pattern of
// a float32 distance >= 0, up to +inf and the NaN 0x7fc00000, in the high word
// makes a positive finite double (its exponent field is at most 0x7fc), so the
// double order is the order of the 64-bit words, and one instruction each
// replaces a 64-bit compare and two selects.  A denormal (distance 0) keeps
// its bits: double denormals are always on.  Written as instructions because
// the library calls would canonicalise their operands first.
__device__ __forceinline__ double key_min(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double key_max(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The K best (distance, index) pairs of one query in ascending order, each
// packed as one 64-bit key, distance bits above index: the float32 bits of a
// distance >= 0 order like the distance itself, so comparing keys compares
// distances first and breaks ties by the smaller index.  The word is kept as a
// double (key_min).  An empty slot holds index INT32_MAX.
template <int K>
struct TopK {
    double key[K];

    __device__ static __forceinline__ double pack(float d, int id)
    {
        return __hiloint2double((int)__float_as_uint(d), id);
    }
    __device__ __forceinline__ void reset(float bound)
    {
#pragma unroll
        for (int s = 0; s < K; ++s)
            key[s] = pack(bound, INT32_MAX);
    }
    // distance of the K-th best: a box farther than this cannot contribute
    __device__ __forceinline__ float bound() const { return __int_as_float(__double2hiint(key[K - 1])); }
    // Insertion: slot s becomes the middle one of its key, its left neighbour's
    // and the new one, so a key above all of them changes nothing and no lane
    // needs a branch of its own.  In a wavefront some lane nearly always
    // inserts, and a candidate that gets in usually ranks near the end: the
    // slots are done in groups of eight from the back, until no lane goes on.
    // (Against 64-bit compares and selects slot by slot: 1000 queries of k = 10
    // in 2*10^4 points 111 -> 77 us, k = 16 at 10^7 points 8.6 -> 8.0 ms.)
    __device__ __forceinline__ void offer(float d, int id) { offer_key(pack(d, id)); }
    __device__ __forceinline__ void offer_key(double v)
    {
        if (!(v < key[K - 1]))
            return;
#pragma unroll
        for (int s = K - 1; s > 0; --s) {
            key[s] = key_min(key[s], key_max(key[s - 1], v));
            if (s % 8 == 0 && __ballot(v < key[s - 1]) == 0)
                return;
        }
        key[0] = key_min(key[0], v);
    }
    // Write the first k_out, indices relative to `base`; empty slots become (+inf, -1).
    __device__ __forceinline__ void store(int k_out, float *d2, int32_t *idx, int base) const
    {
#pragma unroll
        for (int s = 0; s < K; ++s) {
            if (s < k_out) {
                const int id = __double2loint(key[s]);
                const bool empty = id == INT32_MAX;
                d2[s] = empty ? INFINITY : __int_as_float(__double2hiint(key[s]));
                idx[s] = empty ? -1 : id - base;
            }
        }
    }
};

// Squared distance from q to the value stored in leaf record `pos`.
template <int D>
__device__ __forceinline__ float leaf_d2(const float *__restrict__ leaves, int kind, int64_t pos, const float *q)
{
    const float *lf = leaves + pos * leaf_floats(D, kind);
    float lo[D], hi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        lo[d] = lf[d];
        hi[d] = kind == ARBORX_BOXES ? lf[D + d] : lf[d];
    }
    return box_d2<D>(q, lo, hi);
}

// Sorted leaf keys a kNN seed searches for the query's position: a tree's
// Morton codes (no prefix, 63/D bits per dimension), or a forest's keys, whose
// segment for tree t holds (t << mbits) | the tree-local code (mbits/D bits per
// dimension, on that tree's bounds).  Without codes a greedy descent finds the
// position.
struct SeedKeys {
    const uint64_t *codes = nullptr;
    uint64_t prefix = 0;
    int bits = 0;
};

// Position of q among the sorted leaves of the tree of hdr: the first leaf
// whose key (the build's, on the tree's bounds) is not below q's, found by
// binary search over the tree's segment of the keys, clamped to the tree.
template <int D>
__device__ __forceinline__ int leaf_position(const SeedKeys &keys, const TreeHeader &hdr, const float *q)
{
    uint32_t c[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const float ext = hdr.hi[d] - hdr.lo[d];
        c[d] = quantise(q[d], hdr.lo[d], ext > 0.0f ? 1.0f / ext : 0.0f, keys.bits);
    }
    const uint64_t key = keys.prefix | interleave<D>(c, keys.bits);
    const uint64_t *__restrict__ codes = keys.codes;
    int lo = hdr.start, hi = hdr.start + hdr.n;  // first code >= key in [lo, hi)
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (codes[mid] < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo < hdr.start + hdr.n ? lo : hdr.start + hdr.n - 1;
}

// Width of the register window that selects the mode-0 seed bound: the
// smallest power of two holding 2K distances.
template <int K>
constexpr int seed_width()
{
    int w = 1;
    while (w < 2 * K)
        w <<= 1;
    return w;
}

// Bitonic compare-exchange network on register words, fully unrolled so
// that every index is a compile-time constant: sorts v[LO .. LO + N) (N a
// power of two) ascending if UP, else descending.  The words are the bit
// patterns of distances >= 0 (or NaN), which order as unsigned integers like
// the distances, NaN after +inf.
template <int W, int LO, int N, bool UP>
__device__ __forceinline__ void bitonic_sort_range(uint32_t (&v)[W])
{
#pragma unroll
    for (int k = 2; k <= N; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int l = i ^ j;
                if (l > i) {
                    const bool asc = ((i & k) == 0) == UP;
                    const uint32_t a = v[LO + i], b = v[LO + l];
                    const uint32_t mn = a < b ? a : b, mx = a < b ? b : a;
                    v[LO + i] = asc ? mn : mx;
                    v[LO + l] = asc ? mx : mn;
                }
            }
}

// Starting bound for the kNN walk from the sorted leaves around position pos
// (where a greedy descent towards q ends).  mode 0: the k-th smallest distance
// among the 2k leaves around pos; mode 2: the largest distance among the k
// leaves around pos (a looser bound).  Either is at least the true k-th
// neighbour distance, so the slots start as k copies of (bound, INT32_MAX),
// which admit every true result.  Needs n >= k.
//
// For k <= 16 the k-th smallest of the window is selected in registers with a
// sorting network (the distances' bit patterns sorted as unsigned words);
// when the window is exactly 2k wide only its two halves are sorted, one up
// and one down: the elementwise minima of the halves are then the k smallest
// of the window, so their maximum is the k-th smallest.
template <int D, int K>
__device__ __forceinline__ void seed_window(const float *__restrict__ leaves, int kind, const TreeHeader &hdr, int pos,
                                            const float *q, TopK<K> &best, int mode)
{
    const int lo_lim = hdr.start, hi_lim = hdr.start + hdr.n;
    if (mode == 2) {
        int w0 = pos - K / 2;
        w0 = w0 > hi_lim - K ? hi_lim - K : w0;
        w0 = w0 < lo_lim ? lo_lim : w0;
        float b = 0.0f;
#pragma unroll 4
        for (int p = w0; p < w0 + K; ++p)
            b = fmaxf(b, leaf_d2<D>(leaves, kind, p, q));
        best.reset(b);
        return;
    }
    int w0 = pos - K;
    w0 = w0 > hi_lim - 2 * K ? hi_lim - 2 * K : w0;
    w0 = w0 < lo_lim ? lo_lim : w0;
    const int w1 = (w0 + 2 * K < hi_lim) ? w0 + 2 * K : hi_lim;
    if constexpr (K <= 16) {
        constexpr int W = seed_width<K>();
        constexpr uint32_t kInfBits = 0x7f800000u;
        uint32_t v[W];
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const int p = w0 + i;
            v[i] = (i < 2 * K && p < w1) ? __float_as_uint(leaf_d2<D>(leaves, kind, p, q)) : kInfBits;
        }
        uint32_t kth;
        if constexpr (W == 2 * K && K > 1) {
            bitonic_sort_range<W, 0, K, true>(v);
            bitonic_sort_range<W, K, K, false>(v);
            kth = 0;
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const uint32_t mn = v[i] < v[K + i] ? v[i] : v[K + i];
                kth = mn > kth ? mn : kth;
            }
        } else {
            bitonic_sort_range<W, 0, W, true>(v);
            kth = v[K - 1];
        }
        best.reset(__uint_as_float(kth < kInfBits ? kth : kInfBits));
        return;
    }
    for (int p = w0; p < w1; ++p)
        best.offer(leaf_d2<D>(leaves, kind, p, q), p);  // distinct keys; only distances matter
    best.reset(best.bound());
}

// Seeding of a kNN walk: the query's position in the tree's sorted leaves
// (binary search over the kept leaf keys, a tree's codes or its segment of a
// forest's keys, or a greedy nearer-child descent when there are none); the K-th smallest distance among the 2K leaves around
// it bounds the K-th nearest distance from above, so the walk starts with that
// bound instead of +inf.  The heap then starts as K copies of
// (bound, INT32_MAX): every value at distance < bound, or == bound, orders
// before them, so all true results are still admitted, and none of the
// placeholders survive when the tree has at least K values.
template <int D, int K>
__device__ __forceinline__ void knn_seed(const Node<D> *__restrict__ nodes, int n_nodes,
                                         const float *__restrict__ leaves, int kind, const TreeHeader &hdr,
                                         const float *q, TopK<K> &best, int seed, const SeedKeys &keys)
{
    const int n = hdr.n;
    best.reset(INFINITY);
    if (seed != 1 && n >= K) {
        int cur = keys.codes ? -1 : hdr.root, pos = keys.codes ? leaf_position<D>(keys, hdr, q) : hdr.start;
        for (int iter = 0; iter <= n_nodes; ++iter) {
            if ((unsigned)cur >= (unsigned)n_nodes)
                break;
            Node<D> nd;
            load_node(nodes, cur, nd);
            const float d0 = box_d2<D>(q, nd.lo[0], nd.hi[0]);
            const float d1 = box_d2<D>(q, nd.lo[1], nd.hi[1]);
            const int go = d1 < d0 ? 1 : 0;
            const int c = go ? nd.child[1] : nd.child[0];
            if (c < 0) {
                pos = cur + go;  // node cur separates sorted leaves cur and cur + 1
                break;
            }
            cur = c;
        }
        // window of 2K leaves around pos inside [start, start + n)
        seed_window<D, K>(leaves, kind, hdr, pos, q, best, seed);
    }
}

// Nearest-first walk keeping the K best (d2, index) pairs sorted in
// registers; a subtree is skipped only if its box is strictly farther than the
// current K-th pair, so equal-distance values with smaller indices are found.
// Software-pipelined: the next node is chosen from the current node's box
// distances and the bound before this node's leaves are offered (a bound that
// can only be looser, so nothing is lost), its fetch is issued, and the leaf
// insertions and the stack push run while it is in flight.
template <int D, int K>
__device__ __forceinline__ void knn_search(const Node<D> *__restrict__ nodes, int n_nodes,
                                           const float *__restrict__ leaves, int kind, const TreeHeader &hdr,
                                           const float *q, TopK<K> &best, ShortStack<KnnEntry> &st, int seed,
                                           const SeedKeys &keys, int *visits = nullptr)
{
    knn_seed<D, K>(nodes, n_nodes, leaves, kind, hdr, q, best, seed, keys);
    if (hdr.n <= 0)
        return;
    int cur = hdr.root;
    Node<D> nd;
    if ((unsigned)cur < (unsigned)n_nodes)
        load_node(nodes, cur, nd);
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        if (visits)  // node fetches, for the walk statistics of the debug entry point
            ++*visits;
        const float d0 = box_d2<D>(q, nd.lo[0], nd.hi[0]);
        const float d1 = box_d2<D>(q, nd.lo[1], nd.hi[1]);
        const int c0 = nd.child[0], c1 = nd.child[1];
        const float bound = best.bound();
        const bool k0 = c0 >= 0 && !(d0 > bound);
        const bool k1 = c1 >= 0 && !(d1 > bound);
        int next = -1;
        if (k0 && k1) {
            const bool near1 = d1 < d0;
            st.push(near1 ? KnnEntry{c0, d0} : KnnEntry{c1, d1});
            next = near1 ? c1 : c0;
        } else if (k0) {
            next = c0;
        } else if (k1) {
            next = c1;
        } else {
            while (!st.empty()) {
                const KnnEntry e = st.pop();
                if (!(e.d2 > bound)) {
                    next = e.ref;
                    break;
                }
            }
        }
        if ((unsigned)next < (unsigned)n_nodes)
            load_node(nodes, next, nd);  // in flight during the insertions below
        if (c0 < 0 && c0 != kEmptyRef)
            best.offer(d0, ~c0);
        if (c1 < 0 && c1 != kEmptyRef)
            best.offer(d1, ~c1);
        cur = next;
    }
}

// Order two (distance, reference, admitted) candidates so that the first is
// the farther admitted one; candidates not admitted go last.
__device__ __forceinline__ void far_first(float &da, int &ra, bool &ka, float &db, int &rb, bool &kb)
{
    const bool swap = (kb && !ka) || (ka && kb && db > da);
    const float td = da;
    const int tr = ra;
    const bool tk = ka;
    da = swap ? db : da;
    ra = swap ? rb : ra;
    ka = swap ? kb : ka;
    db = swap ? td : db;
    rb = swap ? tr : rb;
    kb = swap ? tk : kb;
}

// kNN over four-wide nodes: leaf slots are offered; admitted internal slots
// are sorted farthest first, the nearest is entered and the others are pushed
// with their distances (the nearest of them on top).  Seeding as knn_search,
// on the binary nodes.
template <int D, int K>
__device__ __forceinline__ void knn_search4(const Node<D> *__restrict__ nodes, const Node4<D> *__restrict__ wnodes,
                                            int n_nodes, const float *__restrict__ leaves, int kind,
                                            const TreeHeader &hdr, const float *q, TopK<K> &best,
                                            ShortStack<KnnEntry> &st, int seed, const SeedKeys &keys)
{
    const int n = hdr.n;
    best.reset(INFINITY);
    if (n <= 0)
        return;
    if (seed != 1 && n >= K) {
        int cur = keys.codes ? -1 : hdr.root, pos = keys.codes ? leaf_position<D>(keys, hdr, q) : hdr.start;
        for (int iter = 0; iter <= n_nodes; ++iter) {
            if ((unsigned)cur >= (unsigned)n_nodes)
                break;
            Node<D> nd;
            load_node(nodes, cur, nd);
            const float d0 = box_d2<D>(q, nd.lo[0], nd.hi[0]);
            const float d1 = box_d2<D>(q, nd.lo[1], nd.hi[1]);
            const int go = d1 < d0 ? 1 : 0;
            const int c = go ? nd.child[1] : nd.child[0];
            if (c < 0) {
                pos = cur + go;
                break;
            }
            cur = c;
        }
        seed_window<D, K>(leaves, kind, hdr, pos, q, best, seed);
    }
    int cur = hdr.root;
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        Node4<D> nd;
        load_node4(wnodes, cur, nd);
        float d[4];
        int r[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            d[s] = box_d2<D>(q, nd.lo[s], nd.hi[s]);
            r[s] = nd.child[s];
            if (r[s] < 0 && r[s] != kEmptyRef)
                best.offer(d[s], ~r[s]);
        }
        const float bound = best.bound();
        bool k[4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            k[s] = r[s] >= 0 && !(d[s] > bound);
        // sorting network on four: farthest admitted first, not admitted last
        far_first(d[0], r[0], k[0], d[1], r[1], k[1]);
        far_first(d[2], r[2], k[2], d[3], r[3], k[3]);
        far_first(d[0], r[0], k[0], d[2], r[2], k[2]);
        far_first(d[1], r[1], k[1], d[3], r[3], k[3]);
        far_first(d[1], r[1], k[1], d[2], r[2], k[2]);
        int next = -1;
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (k[s]) {
                if (next >= 0)
                    st.push(KnnEntry{next, d[s - 1 >= 0 ? s - 1 : 0]});
                next = r[s];
            }
        if (next < 0) {
            while (!st.empty()) {
                const KnnEntry e = st.pop();
                if (!(e.d2 > best.bound())) {
                    next = e.ref;
                    break;
                }
            }
        }
        cur = next;
    }
}

__device__ __forceinline__ float wave_min(float v)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1)
        v = fminf(v, __shfl_xor(v, o, kWave));
    return v;
}

// Wavefront-packet kNN walk (single tree: every lane shares the root).  Each
// lane keeps its own top-K and bound; a child is entered when some lane's
// bound admits it.  The nearer child for most lanes goes first; the deferred
// child is stored with the smallest distance any lane has to it, and is
// skipped at pop time only when that distance exceeds every lane's bound.
// Seeding (per lane) is as in knn_search.
template <int D, int K>
__device__ __forceinline__ void knn_search_wave(const Node<D> *__restrict__ nodes, int n_nodes,
                                                const float *__restrict__ leaves, int kind, const TreeHeader &hdr,
                                                const float *q, bool active, TopK<K> &best,
                                                KnnEntry *wstack, int seed)
{
    const int n = hdr.n;
    best.reset(INFINITY);
    if (n <= 0)
        return;
    if (active && seed != 1 && n >= K) {
        int cur = hdr.root, pos = hdr.start;
        for (int iter = 0; iter <= n_nodes; ++iter) {
            if ((unsigned)cur >= (unsigned)n_nodes)
                break;
            Node<D> nd;
            load_node(nodes, cur, nd);
            const float d0 = box_d2<D>(q, nd.lo[0], nd.hi[0]);
            const float d1 = box_d2<D>(q, nd.lo[1], nd.hi[1]);
            const int go = d1 < d0 ? 1 : 0;
            const int c = go ? nd.child[1] : nd.child[0];
            if (c < 0) {
                pos = cur + go;
                break;
            }
            cur = c;
        }
        seed_window<D, K>(leaves, kind, hdr, pos, q, best, seed);
    }
    int sp = 0;
    int cur = hdr.root;
    for (int iter = 0; iter <= n_nodes; ++iter) {
        cur = __builtin_amdgcn_readfirstlane(cur);
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        Node<D> nd;
        load_node(nodes, cur, nd);
        const float d0 = box_d2<D>(q, nd.lo[0], nd.hi[0]);
        const float d1 = box_d2<D>(q, nd.lo[1], nd.hi[1]);
        const int c0 = nd.child[0], c1 = nd.child[1];
        if (active && c0 < 0 && c0 != kEmptyRef)
            best.offer(d0, ~c0);
        if (active && c1 < 0 && c1 != kEmptyRef)
            best.offer(d1, ~c1);
        const bool k0 = active && c0 >= 0 && !(d0 > best.bound());
        const bool k1 = active && c1 >= 0 && !(d1 > best.bound());
        const bool any0 = __ballot(k0) != 0, any1 = __ballot(k1) != 0;
        if (any0 && any1) {
            const bool want1 = (k0 || k1) && d1 < d0;
            const bool want0 = (k0 || k1) && !(d1 < d0);
            const bool first1 = __popcll(__ballot(want1)) > __popcll(__ballot(want0));
            const int far = first1 ? c0 : c1;
            const float dfar = wave_min(first1 ? (k0 ? d0 : INFINITY) : (k1 ? d1 : INFINITY));
            if (sp < kWaveStack)
                wstack[sp] = KnnEntry{far, dfar};
            ++sp;
            cur = first1 ? c1 : c0;
        } else if (any0) {
            cur = c0;
        } else if (any1) {
            cur = c1;
        } else {
            cur = -1;
            while (sp > 0) {
                --sp;
                const KnnEntry e = sp < kWaveStack ? wstack[sp] : KnnEntry{-1, INFINITY};
                if (__ballot(active && !(e.d2 > best.bound())) != 0) {
                    cur = e.ref;
                    break;
                }
            }
            if (cur < 0)
                break;
        }
    }
}

// The sums a kNN walk over codes orders and prunes by, as words whose order is
// theirs, and the bound on them from k d^2 + a (a NaN, infinity times a k of zero,
// bounds nothing): in a frame with one step, for a query inside it and for one
// past it; in a frame with a step for each dimension, for both.
template <int D>
struct KnnGap {
    const uint32_t (&q)[D];
    __device__ __forceinline__ uint32_t sum(const uint32_t (&w)[D]) const { return code_gap2<D>(q, w); }
    __device__ __forceinline__ uint32_t bound(float fb) const { return fb < 4.29e9f ? (uint32_t)fb : UINT32_MAX; }
};
template <int D>
struct KnnGapPast {
    const uint32_t (&q)[D];
    CodeExcess<D> ex;
    __device__ __forceinline__ uint32_t sum(const uint32_t (&w)[D]) const { return ex.gap2(q, w); }
    __device__ __forceinline__ uint32_t bound(float fb) const
    {
        return fb < 4.29e9f ? (uint32_t)fmaxf(fb, 0.0f) : UINT32_MAX;
    }
};
template <int D>
struct KnnGapUneven {
    const uint32_t (&q)[D];
    CodeMetric<D, false> metric;
    float e2[D];  // twice the excess, rounded down
    __device__ __forceinline__ uint32_t sum(const uint32_t (&w)[D]) const
    {
        float acc = 0.0f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const float g = metric.gap(q[d], w[d], d);
            acc = fmaf(g, g + e2[d], acc);
        }
        return __float_as_uint(acc);
    }
    __device__ __forceinline__ uint32_t bound(float fb) const
    {
        return __float_as_uint(fb < 3.0e38f ? fmaxf(fb, 0.0f) : INFINITY);
    }
};

// kNN over the quantized nodes of a tree of points in the codes of its frame
// (see traverse_codes): as knn_search, seeded and software-pipelined, with
// internal children ordered and pruned by their squared code gaps against the
// bound in codes, and leaf children offered with their exact distances.  The
// bound in codes, k d^2 + a, is rounded up in float32: k and a hold 1/s^2 with
// the margins of code_ball and more.  A wavefront with a query outside the
// frame counts the excesses past it (CodeExcess), or it would enter every node
// near the projection on the frame: k = 1 between clouds of unlike extents
// took 6.6 ms without them, 1.8 over float nodes.  Half the loads of the float nodes and no decoding:
// k = 16 at 10^7 cube points 7.3 -> 6.0 ms, and k = 8 over 2*10^6 6D mixture
// points, against decoded boxes, 7.1 -> 5.9 ms.  (Gathering admitted leaves in
// LDS and merging eight at a time with a sorting network took 13 % fewer
// vector instructions at k = 16, none fewer at k = 8, and 6.5 and 6.7 ms: the
// bound lags and the queue takes LDS.)
template <int D, int K, class G>
__device__ __forceinline__ void knn_walk_codes(const QNode<D> *__restrict__ nodes, int n_nodes, const TreeHeader &hdr,
                                               const float (&q)[D], TopK<K> &best, TopStack<KnnCode> &st, float k,
                                               float a, const G &gap)
{
    const unsigned last = (unsigned)n_nodes - 1u;
    int cur = hdr.root;
    QNode<D> nd;
    load_qnode(nodes, (int)min((unsigned)cur, last), nd);
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur > last)
            break;
        KnnCode deferred = st.top();
        const int c0 = nd.child[0], c1 = nd.child[1];
        const uint32_t s0 = gap.sum(nd.w[0]), s1 = gap.sum(nd.w[1]);
        // leaf children as keys, the other slots above every key; no slot is empty (its words are a NaN with an
        // exponent of 0x7ff, for which the key order fails): a frame with an extent holds two values at least
        const double none = TopK<K>::pack(__uint_as_float(0x7fc00000u), INT32_MAX);
        const double v0 = c0 < 0 ? TopK<K>::pack(point_d2<D>(q, nd.w[0]), ~c0) : none;
        const double v1 = c1 < 0 ? TopK<K>::pack(point_d2<D>(q, nd.w[1]), ~c1) : none;
        const uint32_t bound = gap.bound(fmaf(best.bound(), k, a));
        const bool k0 = c0 >= 0 && s0 <= bound;
        const bool k1 = c1 >= 0 && s1 <= bound;
        const bool near1 = k1 && (!k0 || s1 < s0);
        const KnnCode far = near1 ? knn_code(c0, s0) : knn_code(c1, s1);
        st.put(far);
        st.move(k0 && k1, !(k0 || k1), far, deferred);
        cur = near1 ? c1 : c0;
        if (!(k0 || k1)) {
            while ((uint32_t)(deferred >> 32) > bound) {  // the last entry is below every bound
                deferred = st.top();
                st.move(false, true, deferred, deferred);
            }
            cur = (int)(uint32_t)deferred;
        }
        load_qnode(nodes, (int)min((unsigned)cur, last), nd);  // in flight during the insertions below
        best.offer_key(key_min(v0, v1));
        best.offer_key(key_max(v0, v1));
    }
}

template <int D, int K>
__device__ __forceinline__ void knn_search_codes(const QNode<D> *__restrict__ nodes, int n_nodes,
                                                 const float *__restrict__ leaves, int kind, const TreeHeader &hdr,
                                                 const float (&q)[D], TopK<K> &best, TopStack<KnnCode> &st,
                                                 int seed, const SeedKeys &keys)
{
    best.reset(INFINITY);
    if (hdr.n <= 0)
        return;
    if (seed != 1 && hdr.n >= K)
        seed_window<D, K>(leaves, kind, hdr, leaf_position<D>(keys, hdr, q), q, best, seed);
    uint32_t qc[D];
    double e[D], past = 0.0;
    const double k = hdr.qinv * hdr.qinv * (1.0 + 0x1p-19), a = hdr.qinv * hdr.qinv * 0x1p-144;
    if (hdr.even) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            qc[d] = code_query(q[d], hdr.lo[d], hdr.qinv, e[d]);
            past += e[d] * e[d];
        }
        if (!__any(past > 1.0)) {
            knn_walk_codes<D, K>(nodes, n_nodes, hdr, q, best, st, (float)k, (float)(a + 2.0), KnnGap<D>{qc});
            return;
        }
        const KnnGapPast<D> gap{qc, CodeExcess<D>(e)};
        const double unit = ldexp(1.0, -(int)(gap.ex.shift & 15u));
        const double rest = (a + 2.0 - past * (1.0 - 0x1p-22)) * unit;
        knn_walk_codes<D, K>(nodes, n_nodes, hdr, q, best, st, (float)(k * unit), (float)fmax(rest + 1.0, -3.0e38), gap);
        return;
    }
    KnnGapUneven<D> gap{qc, CodeMetric<D, false>(hdr)};
#pragma unroll
    for (int d = 0; d < D; ++d) {
        qc[d] = code_query(q[d], hdr.lo[d], gap.metric.inv(hdr, d), e[d]);
        e[d] *= gap.metric.weight(d) * (1.0 - 0x1p-22);
        gap.e2[d] = (float)(2.0 * e[d] * (1.0 - 0x1p-23));
        past += e[d] * e[d];
    }
    knn_walk_codes<D, K>(nodes, n_nodes, hdr, q, best, st, (float)(k * (1.0 + 0x1p-18)),
                         (float)fmax(a + 0x1p-100 - past * (1.0 - 0x1p-22), -3.0e38), gap);
}

// kNN over the quantized nodes of a tree of boxes: as knn_search (seeded,
// software-pipelined), pruning with the decoded (larger) boxes; leaves that
// pass the bound are offered from their records.
template <int D, int K>
__device__ __forceinline__ void knn_search_q(const QNode<D> *__restrict__ nodes, int n_nodes,
                                             const float *__restrict__ leaves, const TreeHeader &hdr, const float *q,
                                             TopK<K> &best, ShortStack<KnnEntry> &st, int seed, const SeedKeys &keys)
{
    const int n = hdr.n;
    best.reset(INFINITY);
    if (n <= 0)
        return;
    constexpr int kind = ARBORX_BOXES;
    float flo[D], fsc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        flo[d] = hdr.lo[d];
        fsc[d] = hdr.qscale[d];
    }
    if (seed != 1 && n >= K) {
        int cur = keys.codes ? -1 : hdr.root, pos = keys.codes ? leaf_position<D>(keys, hdr, q) : hdr.start;
        for (int iter = 0; iter <= n_nodes; ++iter) {
            if ((unsigned)cur >= (unsigned)n_nodes)
                break;
            QNode<D> nd;
            load_qnode(nodes, cur, nd);
            float lo[2][D], hi[2][D];
            qboxes<D>(nd, false, flo, fsc, lo, hi);
            const float d0 = box_d2<D>(q, lo[0], hi[0]);
            const float d1 = box_d2<D>(q, lo[1], hi[1]);
            const int go = (d1 < d0 && nd.child[1] != kEmptyRef) ? 1 : 0;
            const int c = go ? nd.child[1] : nd.child[0];
            if (c < 0) {
                pos = cur + go;  // node cur separates sorted leaves cur and cur + 1
                break;
            }
            cur = c;
        }
        seed_window<D, K>(leaves, kind, hdr, pos, q, best, seed);
    }
    int cur = hdr.root;
    QNode<D> nd;
    if ((unsigned)cur < (unsigned)n_nodes)
        load_qnode(nodes, cur, nd);
    for (int iter = 0; iter <= n_nodes; ++iter) {
        if ((unsigned)cur >= (unsigned)n_nodes)
            break;
        float lo[2][D], hi[2][D];
        qboxes<D>(nd, false, flo, fsc, lo, hi);
        const float d0 = box_d2<D>(q, lo[0], hi[0]);
        const float d1 = box_d2<D>(q, lo[1], hi[1]);
        const int c0 = nd.child[0], c1 = nd.child[1];
        const float bound = best.bound();
        const bool k0 = c0 >= 0 && !(d0 > bound);
        const bool k1 = c1 >= 0 && !(d1 > bound);
        int next = -1;
        if (k0 && k1) {
            const bool near1 = d1 < d0;
            st.push(near1 ? KnnEntry{c0, d0} : KnnEntry{c1, d1});
            next = near1 ? c1 : c0;
        } else if (k0) {
            next = c0;
        } else if (k1) {
            next = c1;
        } else {
            while (!st.empty()) {
                const KnnEntry e = st.pop();
                if (!(e.d2 > bound)) {
                    next = e.ref;
                    break;
                }
            }
        }
        if ((unsigned)next < (unsigned)n_nodes)
            load_qnode(nodes, next, nd);  // in flight during the insertions below
        const int lf = leaf_floats(D, kind);
        if (c0 < 0 && c0 != kEmptyRef && !(d0 > best.bound()))
            best.offer(leaf_d2<D>(leaves, kind, ~c0, q), __float_as_int(leaves[(int64_t)(~c0) * lf + 2 * D]));
        if (c1 < 0 && c1 != kEmptyRef && !(d1 > best.bound()))
            best.offer(leaf_d2<D>(leaves, kind, ~c1, q), __float_as_int(leaves[(int64_t)(~c1) * lf + 2 * D]));
        cur = next;
    }
}

// Node slots of a single tree (one-value trees still have one node).
__device__ __forceinline__ int node_count(const TreeHeader *hdr) { return hdr->n > 1 ? hdr->n - 1 : 1; }

// Whether searches over points walk the codes of the tree's frame: no crowd of
// points is there that the codes cannot tell apart (store_qnode).  A ball much
// wider than a code meets few more boxes in codes than in floats: 10^6 uniform
// 3D points 4 codes apart, counts over codes and over float nodes 537 and 506 us
// at a radius of 5 codes, 938 and 955 at 8, 3622 and 4243 at 16; 2.2 codes apart
// 5626 and 5176 at 8, 26431 and 28397 at 16; 3*10^5 2D points 1.1 codes apart 79
// and 70 at 2, 122 and 126 at 4.  The nearest searches turn their bound into
// codes in float32, so 1/step^2 has to lie in its range.
template <int D> constexpr double kWideBall = D <= 2 ? 3.0 : 12.0;  // codes
constexpr double kLeastStep = 1e-19;
__device__ __forceinline__ bool codes_serve(const TreeHeader &h)
{
    return h.qinv != 0.0 && !h.crowded && h.qinv <= 1.0 / kLeastStep;
}
template <int D>
__device__ __forceinline__ bool codes_serve(const TreeHeader &h, float r2)
{
    return h.qinv != 0.0 && (!h.crowded || (double)r2 * h.qinv * h.qinv >= kWideBall<D> * kWideBall<D>);
}

// Walk of one query over a tree that holds quantized nodes: in codes for a
// sphere over points where they serve, else over the float nodes; other
// predicates and box values decode the boxes.
template <int D, class P, class F, class S = NeverStop>
__device__ __forceinline__ void walk_quantized(const Node<D> *__restrict__ nodes, const QNode<D> *__restrict__ qnodes,
                                               const TreeHeader &h, int n_nodes, const float *__restrict__ leaves,
                                               int kind, const P &pred, int *s_stack, int cap, int (&spill)[kSpill],
                                               F &f, const S &stop = S())
{
    if constexpr (std::is_same<P, Sphere<D>>::value) {
        if (kind != ARBORX_BOXES) {
            if (codes_serve<D>(h, pred.r2)) {
                TopStack<int> st(s_stack + threadIdx.x, blockDim.x, cap, spill, -1);
                auto g1 = [&](int, int idx, float d2) { f(idx, d2); };
                auto g = each_hit(g1);
                const P preds[1] = {pred};
                if (h.even)
                    traverse_codes<D, 1, false, true>(qnodes, h, n_nodes, preds, -1, st, g, stop);
                else
                    traverse_codes<D, 1, false, false>(qnodes, h, n_nodes, preds, -1, st, g, stop);
            } else {
                ShortStack<int> st(s_stack + threadIdx.x, blockDim.x, cap, spill);
                traverse_spatial<D>(nodes, h.root, n_nodes, pred, st, f, stop);
            }
            return;
        }
    }
    ShortStack<int> st(s_stack + threadIdx.x, blockDim.x, cap, spill);
    traverse_spatial_q<D>(qnodes, h, n_nodes, leaves, kind, pred, st, f, stop);
}

// The same for NQ neighbouring sphere queries of one thread.
template <int D, int NQ, class F>
__device__ __forceinline__ void walk_quantized_packet(const Node<D> *__restrict__ nodes,
                                                      const QNode<D> *__restrict__ qnodes, const TreeHeader &h,
                                                      int n_nodes, const float *__restrict__ leaves, int kind,
                                                      const Sphere<D> (&pred)[NQ], int *s_stack, int cap,
                                                      int (&spill)[kSpill], F &f)
{
    float r2 = pred[0].r2;  // idle ones have none
#pragma unroll
    for (int j = 1; j < NQ; ++j)
        r2 = fmaxf(r2, pred[j].r2);
    if (kind != ARBORX_BOXES && codes_serve<D>(h, r2)) {
        TopStack<int> st(s_stack + threadIdx.x, blockDim.x, cap, spill, -1);
        auto g = each_hit(f);
        if (h.even)
            traverse_codes<D, NQ, false, true>(qnodes, h, n_nodes, pred, -1, st, g);
        else
            traverse_codes<D, NQ, false, false>(qnodes, h, n_nodes, pred, -1, st, g);
        return;
    }
    ShortStack<int> st(s_stack + threadIdx.x, blockDim.x, cap, spill);
    if (kind != ARBORX_BOXES)
        traverse_spatial_packet<D, NQ>(nodes, h.root, n_nodes, pred, st, f);
    else
        traverse_spatial_packet_q<D, NQ>(qnodes, h, n_nodes, leaves, pred, st, f);
}

}  // namespace
}  // namespace ax
