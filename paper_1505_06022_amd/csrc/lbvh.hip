// GPU construction of the multiple-threaded BVH (Sec. 3.1) from sorted Morton
// codes: a linear BVH (Karras 2012's radix tree over the sorted centroid
// codes), the GPU build the paper names as future work (Sec. 4.1).  It
// produces the same device layout as the host SAH build -- six preorder copies
// of 16-byte quantised nodes, one per link set, and 48-byte triangles in leaf
// order -- so every traversal kernel and the renderer use it unchanged.
//
// Steps (all on the device, on the caller's stream):
//   1. triangle boxes; scene and centroid bounds and the quantisation grid
//      (block partials, one reduce)
//   2. 30-bit Morton code of each centroid; stable radix sort of the indices
//   3. radix tree: internal node i splits its key range at the highest
//      differing bit (keys made unique by their sorted position)
//   4. from the leaves up: boxes, triangle counts and collapsed subtree sizes.
//      A workgroup takes the subtrees that lie within its run of sorted leaves
//      and leaves their roots in a list, the next launch does the same over
//      runs 32 times as long, until one run covers all (no kernel waits on
//      another workgroup's writes)
//   5. subtrees of at most max_leaf triangles become leaves; each kept node's
//      index in the six preorders is the sum, over its ancestors, of 1 plus
//      the size of the earlier sibling when it is the later child (children
//      ordered by box centre along each set's direction, ties to the left);
//      quantised node records and triangle records
//   6. the four-child nodes of the wide walk
// The host reads back twice: the node count, for the allocation, and the end.
#include <hip/hip_runtime.h>
#include <hipcub/device/device_radix_sort.hpp>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "bvh_build.h"
#include "runtime.h"

namespace {

constexpr int kLb = 256, kReduce = 1024;

inline uint32_t lb_blocks(int64_t n) { return (uint32_t)((n + kLb - 1) / kLb); }

struct CentreMap {
    float lo[3], scale[3];  // cell = (c - lo) * scale, scale = 1024 / extent (0 for a flat axis)
};

struct QuantGrid {
    double qlo[3], qstep[3], pad;
};

// What the host reads back; zeroed before the first kernel.
struct LbOut {
    float lo[3], hi[3], qlo[3], qstep[3];
    QuantGrid grid;
    CentreMap cells;
    uint32_t bad;         // a walk too long, a full list or an index out of range
    int32_t n_nodes;      // collapsed size of the root
    uint32_t depth;
    unsigned long long leaves;
    double sah;
};

static_assert(sizeof(LbOut) % sizeof(int32_t) == 0, "read back as words");

// Per triangle: box [lo.xyz, hi.xyz]; per block: partial bounds of the
// vertices (vlo, vhi) and of the box centres (clo, chi).
__global__ __launch_bounds__(kLb) void k_lb_boxes(const float *__restrict__ verts, uint32_t n,
                                                  float *__restrict__ tbox, float *__restrict__ part,
                                                  uint4 *__restrict__ link) {
    __shared__ float red[kLb / 64][12];
    const uint32_t i = blockIdx.x * kLb + threadIdx.x;
    float v[12];
    for (int a = 0; a < 3; ++a) {
        v[a] = INFINITY;       // vertex lo
        v[3 + a] = -INFINITY;  // vertex hi
        v[6 + a] = INFINITY;   // centre lo
        v[9 + a] = -INFINITY;  // centre hi
    }
    if (i < n) {
        float lo[3], hi[3];
        for (int a = 0; a < 3; ++a) {
            float x0 = verts[9 * (size_t)i + a], x1 = verts[9 * (size_t)i + 3 + a], x2 = verts[9 * (size_t)i + 6 + a];
            lo[a] = fminf(fminf(x0, x1), x2);
            hi[a] = fmaxf(fmaxf(x0, x1), x2);
            tbox[6 * (size_t)i + a] = lo[a];
            tbox[6 * (size_t)i + 3 + a] = hi[a];
            float c = 0.5f * (lo[a] + hi[a]);
            v[a] = lo[a];
            v[3 + a] = hi[a];
            v[6 + a] = c;
            v[9 + a] = c;
        }
        link[2 * (size_t)i] = link[2 * (size_t)i + 1] = make_uint4(0u, 0u, ~0u, 0u);  // no parent yet
    }
    for (int off = 32; off > 0; off >>= 1)
        for (int a = 0; a < 3; ++a) {
            v[a] = fminf(v[a], __shfl_xor(v[a], off));
            v[3 + a] = fmaxf(v[3 + a], __shfl_xor(v[3 + a], off));
            v[6 + a] = fminf(v[6 + a], __shfl_xor(v[6 + a], off));
            v[9 + a] = fmaxf(v[9 + a], __shfl_xor(v[9 + a], off));
        }
    if ((threadIdx.x & 63) == 0)
        for (int c = 0; c < 12; ++c) red[threadIdx.x >> 6][c] = v[c];
    __syncthreads();
    if (threadIdx.x < 12) {
        const int c = threadIdx.x;
        const bool is_min = (c / 3) % 2 == 0;
        float r = red[0][c];
        for (int w = 1; w < kLb / 64; ++w) r = is_min ? fminf(r, red[w][c]) : fmaxf(r, red[w][c]);
        part[12 * (size_t)blockIdx.x + c] = r;
    }
}

// The scene's bounds, and from them the quantisation grid of the host build
// (padded scene box, 16-bit steps) and the Morton cells, in double precision as
// on the host.  One workgroup: a serial loop over the 512 partials of 131,072
// triangles took 68 us.
__global__ __launch_bounds__(kReduce) void k_lb_reduce(const float *__restrict__ part, uint32_t nblk,
                                                       LbOut *__restrict__ out) {
    __shared__ float red[kReduce / 64][12];
    float v[12];
    for (int c = 0; c < 12; ++c) v[c] = (c / 3) % 2 == 0 ? INFINITY : -INFINITY;
    for (uint32_t b = threadIdx.x; b < nblk; b += kReduce)
        for (int c = 0; c < 12; ++c) {
            const float x = part[12 * (size_t)b + c];
            v[c] = (c / 3) % 2 == 0 ? fminf(v[c], x) : fmaxf(v[c], x);
        }
    for (int off = 32; off > 0; off >>= 1)
        for (int c = 0; c < 12; ++c) {
            const float x = __shfl_xor(v[c], off);
            v[c] = (c / 3) % 2 == 0 ? fminf(v[c], x) : fmaxf(v[c], x);
        }
    if ((threadIdx.x & 63) == 0)
        for (int c = 0; c < 12; ++c) red[threadIdx.x >> 6][c] = v[c];
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kReduce / 64; ++w)
        for (int c = 0; c < 12; ++c)
            v[c] = (c / 3) % 2 == 0 ? fminf(v[c], red[w][c]) : fmaxf(v[c], red[w][c]);
    float ext = 0.0f, mag = 0.0f;
    for (int a = 0; a < 3; ++a) {
        ext = fmaxf(ext, v[3 + a] - v[a]);
        mag = fmaxf(mag, fmaxf(fabsf(v[a]), fabsf(v[3 + a])));
    }
    const double pad = fmax((double)ext * 0x1p-15, (double)mag * 0x1p-20) + 1e-30;
    out->grid.pad = pad;
    for (int a = 0; a < 3; ++a) {
        const double lo = (double)v[a] - pad, hi = (double)v[3 + a] + pad;
        float l = (float)lo;
        if ((double)l > lo) l = nextafterf(l, -INFINITY);
        float sf = (float)((hi - (double)l) / 65535.0);
        while ((double)l + 65535.0 * (double)sf < hi) sf = nextafterf(sf, INFINITY);
        out->lo[a] = v[a];
        out->hi[a] = v[3 + a];
        out->qlo[a] = l;
        out->qstep[a] = sf;
        out->grid.qlo[a] = (double)l;
        out->grid.qstep[a] = (double)sf;
        const float e = v[9 + a] - v[6 + a];
        out->cells.lo[a] = v[6 + a];
        out->cells.scale[a] = e > 0.0f ? 1024.0f / e : 0.0f;
    }
}

__device__ __forceinline__ uint32_t spread10(uint32_t v) {  // 10 bits -> every third bit
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__global__ __launch_bounds__(kLb) void k_lb_morton(const float *__restrict__ tbox, uint32_t n,
                                                   const LbOut *__restrict__ out,
                                                   uint32_t *__restrict__ code, uint32_t *__restrict__ idx) {
    const uint32_t i = blockIdx.x * kLb + threadIdx.x;
    if (i >= n) return;
    const CentreMap cm = out->cells;
    uint32_t q[3];
    for (int a = 0; a < 3; ++a) {
        float c = 0.5f * (tbox[6 * (size_t)i + a] + tbox[6 * (size_t)i + 3 + a]);
        float f = (c - cm.lo[a]) * cm.scale[a];
        q[a] = f >= 1023.0f ? 1023u : (f > 0.0f ? (uint32_t)f : 0u);
    }
    code[i] = spread10(q[0]) | (spread10(q[1]) << 1) | (spread10(q[2]) << 2);
    idx[i] = i;
}

// Length of the common prefix of sorted keys i and j, the key being the Morton
// code followed by the sorted position (so keys are unique); -1 outside.
__device__ __forceinline__ int lb_delta(const uint32_t *__restrict__ code, int n, int i, int j) {
    if (j < 0 || j >= n) return -1;
    uint32_t a = code[i], b = code[j];
    if (a != b) return __clz(a ^ b);
    return 32 + __clz((uint32_t)i ^ (uint32_t)j);
}

// Node numbering: internal nodes 0 .. n-2 (0 is the root), leaf k (sorted
// position k) is node n-1+k.  For n = 1 the single leaf is node 0.
// kids[i]: left child, right child, first and last sorted position of internal
// node i.  link[v].zw: parent of node v and the far end of the parent's range,
// its last position for a left child, the complement of its first for a right.
__global__ __launch_bounds__(kLb) void k_lb_tree(const uint32_t *__restrict__ code, int n, int4 *__restrict__ kids,
                                                 uint4 *__restrict__ link, uint32_t *__restrict__ seen) {
    const int i = (int)(blockIdx.x * kLb + threadIdx.x);
    if (i >= n - 1) return;
    const int d = lb_delta(code, n, i, i + 1) > lb_delta(code, n, i, i - 1) ? 1 : -1;
    const int dmin = lb_delta(code, n, i, i - d);
    int lmax = 2;
    while (lb_delta(code, n, i, i + lmax * d) > dmin) lmax *= 2;
    int l = 0;
    for (int t = lmax / 2; t >= 1; t /= 2)
        if (lb_delta(code, n, i, i + (l + t) * d) > dmin) l += t;
    const int j = i + l * d;
    const int dnode = lb_delta(code, n, i, j);
    int s = 0, t = l;
    do {
        t = (t + 1) / 2;
        if (lb_delta(code, n, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    const int gamma = i + s * d + min(d, 0);
    const int lo = min(i, j), hi = max(i, j);
    const int lc = lo == gamma ? n - 1 + gamma : gamma;
    const int rc = hi == gamma + 1 ? n - 1 + gamma + 1 : gamma + 1;
    kids[i] = make_int4(lc, rc, lo, hi);
    *(uint2 *)&link[lc].z = make_uint2((uint32_t)i, (uint32_t)hi);
    *(uint2 *)&link[rc].z = make_uint2((uint32_t)i, ~(uint32_t)lo);
    seen[i] = 0u;
}

// A radix tree over unique keys of at most 62 bits is at most 62 deep; the
// walks up the tree stop at kMaxWalk steps and flag an error instead.  At most
// two subtrees of each depth are whole within a run of leaves without their
// parents being so, which bounds a run's list of roots.
constexpr int kMaxWalk = 128;
constexpr uint32_t kRootCap = 128;

// A node on the way up: its box, triangle count and size in the collapsed tree
// (two 16-byte words in memory).
struct UpNode {
    float4 lo, hi;  // .w: count, size
};

__device__ __forceinline__ int up_count(const UpNode &u) { return __float_as_int(u.lo.w); }
__device__ __forceinline__ int up_size(const UpNode &u) { return __float_as_int(u.hi.w); }

// One launch of step 4: workgroup w completes the internal nodes whose leaves
// all lie in its run [w run, (w + 1) run).  The threads start at the leaves
// (kLeaves: run is kRun) or at the roots that the previous launch left for the
// 32 parts of the run; of the two children that reach a node the second
// completes it and goes on.  Only threads of one workgroup meet at a node, so
// the hand-over is ordered within the workgroup.  Bound by the chain of
// dependent accesses up the tree, two a level.  131,072 triangles: three
// launches, 62 us, where a launch for each of 22 depths over all nodes took 65 us
// and, with the gaps between them and the walk that found the depths, 290.
constexpr uint32_t kRun = 512, kRunGrowth = 32;

template <bool kLeaves>
__global__ __launch_bounds__(kRun) void k_lb_up(int n, uint32_t run, const float *__restrict__ tbox,
                                                const uint32_t *__restrict__ order, const int4 *__restrict__ kids,
                                                int max_leaf, UpNode *node, uint4 *link, uint32_t *seen,
                                                const uint32_t *__restrict__ roots_in,
                                                const uint32_t *__restrict__ n_in, uint32_t n_parts,
                                                uint32_t *__restrict__ roots_out, uint32_t *__restrict__ n_out,
                                                LbOut *__restrict__ out) {
    __shared__ uint32_t meet[kLeaves ? kRun : 1], n_roots;
    const int64_t c0 = (int64_t)blockIdx.x * run, c1 = min(c0 + (int64_t)run, (int64_t)n);
    if (threadIdx.x == 0) n_roots = 0u;
    if (kLeaves) meet[threadIdx.x] = 0u;
    __syncthreads();
    auto climb = [&](int v, UpNode u) {
        uint2 up = *(const uint2 *)&link[v].z;
        for (int step = 0; v != 0; ++step) {
            const int p = (int)up.x, end = (int)up.y;
            if (step >= kMaxWalk || p < 0 || p >= n - 1) {
                atomicOr(&out->bad, 1u);
                return;
            }
            if (end < 0 ? ~end < c0 : end >= c1) {  // a root of this run
                const uint32_t at = atomicAdd(&n_roots, 1u);
                if (at < kRootCap) roots_out[(size_t)blockIdx.x * kRootCap + at] = (uint32_t)v;
                else atomicOr(&out->bad, 1u);
                return;
            }
            // neither changes in this kernel: read beside the hand-over
            const int4 q = kids[p];
            up = *(const uint2 *)&link[p].z;
            // node p is at one end of its range, so within the run
            uint32_t *m = kLeaves ? &meet[(uint32_t)(p - c0) % kRun] : &seen[p];
            if (__hip_atomic_fetch_add(m, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) == 0u) return;
            const bool is_left = q.x == v;
            const UpNode w = node[is_left ? q.y : q.x];
            const UpNode &l = is_left ? u : w, &r = is_left ? w : u;
            // sets in which the right child comes first (s = 2 axis + negative): box
            // centres compared along the axis, ties to the left
            uint32_t rfirst = 0u;
            const float cl[3] = {l.lo.x + l.hi.x, l.lo.y + l.hi.y, l.lo.z + l.hi.z};
            const float cr[3] = {r.lo.x + r.hi.x, r.lo.y + r.hi.y, r.lo.z + r.hi.z};
            for (int a = 0; a < 3; ++a) {
                if (cr[a] < cl[a]) rfirst |= 1u << (2 * a);
                if (cr[a] > cl[a]) rfirst |= 1u << (2 * a + 1);
            }
            *(uint2 *)&link[q.x] = make_uint2((uint32_t)up_size(r), rfirst);
            *(uint2 *)&link[q.y] = make_uint2((uint32_t)up_size(l), ~rfirst & 63u);
            const int c = up_count(l) + up_count(r);
            UpNode t;
            t.lo = make_float4(fminf(l.lo.x, r.lo.x), fminf(l.lo.y, r.lo.y), fminf(l.lo.z, r.lo.z), __int_as_float(c));
            t.hi = make_float4(fmaxf(l.hi.x, r.hi.x), fmaxf(l.hi.y, r.hi.y), fmaxf(l.hi.z, r.hi.z),
                               __int_as_float(c <= max_leaf ? 1 : 1 + up_size(l) + up_size(r)));
            node[p] = t;
            u = t;
            v = p;
        }
        out->n_nodes = up_size(u);
    };
    if (kLeaves) {
        const int64_t k = c0 + threadIdx.x;
        if (k < c1) {
            const float *b = tbox + 6 * (size_t)order[k];
            UpNode u;
            u.lo = make_float4(b[0], b[1], b[2], __int_as_float(1));
            u.hi = make_float4(b[3], b[4], b[5], __int_as_float(1));
            const int v = (int)(n - 1 + k);
            node[v] = u;
            climb(v, u);
        }
    } else {
        constexpr uint32_t kPer = kRun / kRunGrowth;  // threads on one part's list
        const uint32_t part = blockIdx.x * kRunGrowth + threadIdx.x / kPer;
        const uint32_t count = part < n_parts ? min(n_in[part], kRootCap) : 0u;
        for (uint32_t j = threadIdx.x % kPer; j < count; j += kPer) {
            const uint32_t v = roots_in[(size_t)part * kRootCap + j];
            climb((int)v, node[v]);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) n_out[blockIdx.x] = min(n_roots, kRootCap);
}

__device__ __forceinline__ uint32_t lb_q_down(const QuantGrid &g, int a, double x) {
    double q = floor((x - g.qlo[a]) / g.qstep[a]);
    q = fmin(fmax(q, 0.0), 65535.0);
    while (q > 0.0 && g.qlo[a] + q * g.qstep[a] > x) q -= 1.0;
    return (uint32_t)q;
}

__device__ __forceinline__ uint32_t lb_q_up(const QuantGrid &g, int a, double x) {
    double q = ceil((x - g.qlo[a]) / g.qstep[a]);
    q = fmin(fmax(q, 0.0), 65535.0);
    while (q < 65535.0 && g.qlo[a] + q * g.qstep[a] < x) q += 1.0;
    return (uint32_t)q;
}

// Every kept node writes its record into each of the six preorders.  link[v]:
// size of v's sibling, the sets in which v comes after it, parent.  One 16-byte
// load per ancestor; the statistics are summed over the workgroup first (three
// additions to one address for every kept node, and ten loads per ancestor,
// made this 162 us for 131,072 triangles; now 46).
__global__ __launch_bounds__(kLb) void k_lb_thread(int n, int max_leaf, const uint4 *__restrict__ link,
                                                   const int4 *__restrict__ kids, const UpNode *__restrict__ node,
                                                   uint32_t n_nodes, double trav_cost, uint4 *__restrict__ nodes,
                                                   LbOut *__restrict__ out) {
    __shared__ double sum_sah[kLb / 64];
    __shared__ uint32_t sum_leaves[kLb / 64], max_dep[kLb / 64];
    const int64_t v = (int64_t)blockIdx.x * kLb + threadIdx.x;
    double sah = 0.0;
    uint32_t dep = 0u, leaves = 0u;
    auto place = [&]() {
        const UpNode u = node[v];
        const int cnt = up_count(u);
        const bool leaf = cnt <= max_leaf;
        uint4 up = link[v];
        if (v != 0) {
            if (up.z >= (uint32_t)(n - 1)) {  // every node but the root has an internal parent
                atomicOr(&out->bad, 1u);
                return;
            }
            if (leaf && __float_as_int(node[up.z].lo.w) <= max_leaf) return;  // inside a collapsed leaf
        }
        uint32_t idx[6] = {0, 0, 0, 0, 0, 0};
        for (uint32_t c = (uint32_t)v; c != 0u;) {
            if (up.z >= (uint32_t)(n - 1) || dep >= (uint32_t)kMaxWalk) {
                atomicOr(&out->bad, 1u);
                return;
            }
            for (int s = 0; s < 6; ++s) idx[s] += 1u + ((up.y >> s) & 1u ? up.x : 0u);
            dep++;
            c = up.z;
            if (c != 0u) up = link[c];
        }
        const QuantGrid &g = out->grid;
        const float lo[3] = {u.lo.x, u.lo.y, u.lo.z}, hi[3] = {u.hi.x, u.hi.y, u.hi.z};
        uint32_t lo3[3], hi3[3];
        for (int a = 0; a < 3; ++a) {
            lo3[a] = lb_q_down(g, a, (double)lo[a] - g.pad);
            hi3[a] = lb_q_up(g, a, (double)hi[a] + g.pad);
        }
        uint4 rec;
        rec.x = lo3[0] | (hi3[0] << 16);
        rec.y = lo3[1] | (hi3[1] << 16);
        rec.z = lo3[2] | (hi3[2] << 16);
        const uint32_t first = v >= n - 1 ? (uint32_t)(v - (n - 1)) : (uint32_t)kids[v].z;
        for (int s = 0; s < 6; ++s) {
            rec.w = leaf ? (0x80000000u | (first << 3) | (uint32_t)cnt) : idx[s] + (uint32_t)up_size(u);
            if (idx[s] < n_nodes) nodes[(size_t)s * n_nodes + idx[s]] = rec;
            else atomicOr(&out->bad, 1u);
        }
        // SAH cost with C_isect = 1, normalised by the root's area
        const UpNode top = node[0];
        const double e[3] = {(double)hi[0] - (double)lo[0], (double)hi[1] - (double)lo[1], (double)hi[2] - (double)lo[2]};
        const double r[3] = {(double)top.hi.x - (double)top.lo.x, (double)top.hi.y - (double)top.lo.y,
                             (double)top.hi.z - (double)top.lo.z};
        const double area = e[0] * e[1] + e[1] * e[2] + e[2] * e[0];
        const double root = r[0] * r[1] + r[1] * r[2] + r[2] * r[0];
        const double rel = root > 0.0 ? area / root : 1.0;
        sah = rel * (leaf ? (double)cnt : trav_cost);
        leaves = leaf ? 1u : 0u;
    };
    if (v < 2 * (int64_t)n - 1) place();
    for (int off = 32; off > 0; off >>= 1) {
        sah += __shfl_xor(sah, off);
        leaves += __shfl_xor(leaves, off);
        dep = max(dep, (uint32_t)__shfl_xor(dep, off));
    }
    if ((threadIdx.x & 63) == 0) {
        sum_sah[threadIdx.x >> 6] = sah;
        sum_leaves[threadIdx.x >> 6] = leaves;
        max_dep[threadIdx.x >> 6] = dep;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kLb / 64; ++w) {
        sah += sum_sah[w];
        leaves += sum_leaves[w];
        dep = max(dep, max_dep[w]);
    }
    if (sah != 0.0) unsafeAtomicAdd(&out->sah, sah);
    if (leaves) atomicAdd(&out->leaves, (unsigned long long)leaves);
    atomicMax(&out->depth, dep);
}

// Triangle records in leaf (sorted) order: v0, v1, v2, original index,
// material; and each triangle's place.
__global__ __launch_bounds__(kLb) void k_lb_tris(const float *__restrict__ verts, const uint32_t *__restrict__ mats,
                                                 const uint32_t *__restrict__ order, int n, float4 *__restrict__ tris,
                                                 int32_t *__restrict__ pos) {
    const int k = (int)(blockIdx.x * kLb + threadIdx.x);
    if (k >= n) return;
    const uint32_t t = order[k];
    const float *p = verts + 9 * (size_t)t;
    pos[t] = k;
    tris[3 * (size_t)k] = make_float4(p[0], p[1], p[2], p[3]);
    tris[3 * (size_t)k + 1] = make_float4(p[4], p[5], p[6], p[7]);
    tris[3 * (size_t)k + 2] = make_float4(p[8], __uint_as_float(t), __uint_as_float(mats ? mats[t] : 0u), 0.0f);
}

// The scratch buffers of a build, in one allocation.
struct Scratch {
    char *mem = nullptr;
    size_t size = 0;
    ~Scratch() {
        if (mem) (void)hipFree(mem);
    }
    size_t add(size_t bytes) {
        const size_t at = size;
        size += (bytes + 255) & ~(size_t)255;
        return at;
    }
    template <class T>
    T *at(size_t offset) const {
        return (T *)(mem + offset);
    }
};

}  // namespace

namespace pm {

int build_bvh_gpu(const float *verts_h, const uint32_t *mats_h, int64_t n_tri, int max_leaf, double trav_cost,
                  hipStream_t s, pm_bvh *b) {
    const auto t0 = std::chrono::steady_clock::now();
    const int n = (int)n_tri;
    const size_t n_int = (size_t)std::max(n - 1, 1), n_all = 2 * (size_t)n - 1;
    const size_t pos_words = ((size_t)n + 3) & ~(size_t)3;
    const uint32_t nblk = lb_blocks(n);
    const uint32_t n_runs = (uint32_t)(((int64_t)n + kRun - 1) / kRun);
    size_t sort_bytes = 0;
    PM_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, sort_bytes, (uint32_t *)nullptr, (uint32_t *)nullptr,
                                              (uint32_t *)nullptr, (uint32_t *)nullptr, n, 0, 30, s));
    Scratch sc;
    const size_t o_verts = sc.add(sizeof(float) * 9 * (size_t)n), o_mats = sc.add(sizeof(uint32_t) * (size_t)n),
                 o_tbox = sc.add(sizeof(float) * 6 * (size_t)n), o_part = sc.add(sizeof(float) * 12 * (size_t)nblk),
                 o_code = sc.add(sizeof(uint32_t) * (size_t)n), o_code_s = sc.add(sizeof(uint32_t) * (size_t)n),
                 o_idx = sc.add(sizeof(uint32_t) * (size_t)n), o_order = sc.add(sizeof(uint32_t) * (size_t)n),
                 o_sort = sc.add(sort_bytes), o_kids = sc.add(sizeof(int4) * n_int),
                 o_link = sc.add(sizeof(uint4) * (n_all + 1)), o_node = sc.add(sizeof(UpNode) * n_all),
                 o_seen = sc.add(sizeof(uint32_t) * n_int),
                 o_roots = sc.add(sizeof(uint32_t) * 2 * kRootCap * (size_t)n_runs),
                 o_nroots = sc.add(sizeof(uint32_t) * 2 * (size_t)n_runs),
                 // read back together at the end: each triangle's place, then LbOut
                 o_pos = sc.add(sizeof(int32_t) * pos_words + sizeof(LbOut)), o_out = o_pos + sizeof(int32_t) * pos_words;
    PM_HIP(hipMalloc(&sc.mem, sc.size));
    float *verts = sc.at<float>(o_verts), *tbox = sc.at<float>(o_tbox), *part = sc.at<float>(o_part);
    uint32_t *mats = mats_h ? sc.at<uint32_t>(o_mats) : nullptr, *code = sc.at<uint32_t>(o_code),
             *code_s = sc.at<uint32_t>(o_code_s), *idx = sc.at<uint32_t>(o_idx), *order = sc.at<uint32_t>(o_order),
             *seen = sc.at<uint32_t>(o_seen);
    int4 *kids = sc.at<int4>(o_kids);
    uint4 *link = sc.at<uint4>(o_link);
    UpNode *node = sc.at<UpNode>(o_node);
    uint32_t *roots[2] = {sc.at<uint32_t>(o_roots), sc.at<uint32_t>(o_roots) + kRootCap * (size_t)n_runs};
    uint32_t *n_roots[2] = {sc.at<uint32_t>(o_nroots), sc.at<uint32_t>(o_nroots) + n_runs};
    LbOut *out = sc.at<LbOut>(o_out);
    int32_t *pos = sc.at<int32_t>(o_pos);
    PM_HIP(hipMemcpyAsync(verts, verts_h, sizeof(float) * 9 * (size_t)n, hipMemcpyHostToDevice, s));
    if (mats_h) PM_HIP(hipMemcpyAsync(mats, mats_h, sizeof(uint32_t) * (size_t)n, hipMemcpyHostToDevice, s));
    PM_HIP(hipMemsetAsync(out, 0, sizeof(LbOut), s));

    // 1-2. boxes, bounds, Morton codes and a stable sort by code
    hipLaunchKernelGGL(k_lb_boxes, dim3(nblk), dim3(kLb), 0, s, (const float *)verts, (uint32_t)n, tbox, part, link);
    hipLaunchKernelGGL(k_lb_reduce, dim3(1), dim3(kReduce), 0, s, (const float *)part, nblk, out);
    hipLaunchKernelGGL(k_lb_morton, dim3(nblk), dim3(kLb), 0, s, (const float *)tbox, (uint32_t)n, (const LbOut *)out,
                       code, idx);
    PM_HIP(hipcub::DeviceRadixSort::SortPairs(sc.at<uint8_t>(o_sort), sort_bytes, code, code_s, idx, order, n, 0, 30,
                                              s));

    // 3-4. radix tree; boxes, counts and sizes from the leaves up
    if (n > 1)
        hipLaunchKernelGGL(k_lb_tree, dim3(lb_blocks(n - 1)), dim3(kLb), 0, s, (const uint32_t *)code_s, n, kids, link,
                           seen);
    hipLaunchKernelGGL((k_lb_up<true>), dim3(n_runs), dim3(kRun), 0, s, n, kRun, (const float *)tbox,
                       (const uint32_t *)order, (const int4 *)kids, max_leaf, node, link, seen,
                       (const uint32_t *)nullptr, (const uint32_t *)nullptr, 0u, roots[0], n_roots[0], out);
    uint32_t parts = n_runs, run = kRun;
    for (int from = 0; parts > 1; from ^= 1) {
        const uint32_t groups = (parts + kRunGrowth - 1) / kRunGrowth;
        run = groups > 1 ? run * kRunGrowth : (uint32_t)n;
        hipLaunchKernelGGL((k_lb_up<false>), dim3(groups), dim3(kRun), 0, s, n, run, (const float *)tbox,
                           (const uint32_t *)order, (const int4 *)kids, max_leaf, node, link, seen,
                           (const uint32_t *)roots[from], (const uint32_t *)n_roots[from], parts, roots[from ^ 1],
                           n_roots[from ^ 1], out);
        parts = groups;
    }
    PM_HIP(hipGetLastError());
    // host work and allocations while the kernels run
    PM_HIP(hipGetDevice(&b->device));
    PM_HIP(hipMalloc(&b->d_tris, sizeof(float4) * 3 * (size_t)n + kNextBytes));
    b->d_next = (uint32_t *)(b->d_tris + 3 * (size_t)n);
    std::vector<int32_t> back(pos_words + sizeof(LbOut) / sizeof(int32_t));
    LbOut r;
    PM_HIP(hipMemcpyAsync(&r, out, sizeof(r), hipMemcpyDeviceToHost, s));
    PM_HIP(hipStreamSynchronize(s));
    if (r.bad || r.n_nodes < 1 || (size_t)r.n_nodes > n_all)
        return set_error("GPU BVH build: inconsistent tree"), PM_ERR_STATE;

    // 5. records
    const uint32_t n_nodes = (uint32_t)r.n_nodes;
    // zeroed pad nodes after the six arrays (a packet walk reads the node after the one it visits),
    // then the four-child nodes of a small tree: at most one for each inner node
    const bool small = n_nodes <= kHostMerge;
    const size_t node_bytes = sizeof(uint4) * (kLinkSets * (size_t)n_nodes + pm::kPadNodes),
                 o_wide = (node_bytes + 255) & ~(size_t)255;
    PM_HIP(hipMalloc(&b->d_nodes, small ? o_wide + 4 * sizeof(uint4) * (n_nodes / 2 + 1) : node_bytes));
    PM_HIP(hipMemsetAsync(b->d_nodes + kLinkSets * (size_t)n_nodes, 0, sizeof(uint4) * pm::kPadNodes, s));
    hipLaunchKernelGGL(k_lb_thread, dim3(lb_blocks((int64_t)n_all)), dim3(kLb), 0, s, n, max_leaf,
                       (const uint4 *)link, (const int4 *)kids, (const UpNode *)node, n_nodes, trav_cost, b->d_nodes,
                       out);
    hipLaunchKernelGGL(k_lb_tris, dim3(nblk), dim3(kLb), 0, s, (const float *)verts, (const uint32_t *)mats,
                       (const uint32_t *)order, n, b->d_tris, pos);
    PM_HIP(hipGetLastError());
    b->n_tri = n_tri;
    b->n_refs = n_tri;
    b->n_nodes = n_nodes;
    b->max_leaf = max_leaf;
    for (int a = 0; a < 3; ++a) {
        b->lo[a] = r.lo[a];
        b->hi[a] = r.hi[a];
        b->qlo[a] = r.qlo[a];
        b->qstep[a] = r.qstep[a];
    }

    // 6. four-child nodes
    auto results = [&]() -> int {
        memcpy(&r, back.data() + pos_words, sizeof(r));
        return r.bad ? (set_error("GPU BVH build: inconsistent tree"), PM_ERR_STATE) : PM_OK;
    };
    if (small) {
        std::vector<uint32_t> binary(4 * (size_t)n_nodes), merged;
        PM_HIP(hipMemcpyAsync(binary.data(), b->d_nodes, sizeof(uint4) * n_nodes, hipMemcpyDeviceToHost, s));
        PM_HIP(hipMemcpyAsync(back.data(), pos, sizeof(int32_t) * back.size(), hipMemcpyDeviceToHost, s));
        PM_HIP(hipStreamSynchronize(s));
        if (int rc = results()) return rc;
        if (int rc = merge_wide_host(b, binary.data(), merged)) return rc;
        if (!merged.empty()) {
            b->n_wide = (int64_t)(merged.size() / 16);
            b->d_wide = (uint4 *)((char *)b->d_nodes + o_wide);
            b->wide_inside = true;
            PM_HIP(hipMemcpyAsync(b->d_wide, merged.data(), sizeof(uint32_t) * merged.size(), hipMemcpyHostToDevice, s));
            PM_HIP(hipStreamSynchronize(s));
        }
    } else {
        WideBuild wide;
        if (int rc = wide.launch(b, s)) return rc;  // (does not need the results read here)
        PM_HIP(hipMemcpyAsync(back.data(), pos, sizeof(int32_t) * back.size(), hipMemcpyDeviceToHost, s));
        if (int rc = wide.finish(b, s)) return rc;
        if (int rc = results()) return rc;
    }
    back.resize((size_t)n);
    b->pos_of = std::move(back);
    b->n_leaves = (int64_t)r.leaves;
    b->depth = (int32_t)r.depth;
    b->sah_cost = r.sah;
    b->build_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return PM_OK;
}

}  // namespace pm
