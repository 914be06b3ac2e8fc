// Four-child nodes for the wide walk, merged on the device from the binary
// tree of link set 0 (both builders' output), so that the boxes, leaves and
// triangle records are those of the binary tree.
//
// The tree is recovered from the preorder: the left child of inner node v is
// v + 1 and the right child the node after the left subtree (its skip link; a
// leaf is its own subtree).  From the root down, one launch per level, a wide
// node takes a binary node's two children and opens the inner child of largest
// box area until it has four; its inner children are the next level.  A wide
// node's index is the rank of its binary node among all wide nodes' in
// preorder, so the layout does not depend on the order of the atomics and a
// subtree is contiguous.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "runtime.h"
#include "sppm_scan.h"

namespace {

constexpr int kWb = 256;
// Levels tried before the tree is left to the binary walks (the 2^20-triangle
// soup has 13; a ray through a chain of 32 would need more stack than the wide
// walk has).  The level kernels launch in two parts, so that a shallow tree
// does not pay for the launches of the deepest.
constexpr uint32_t kWideLevels = 32, kWideLevelsFirst = 16;

struct Kids {
    uint32_t id[4];
    uint4 rec[4];
    int n;
};

struct GridStep {
    float s[3];
};

__device__ __forceinline__ bool is_leaf(const uint4 &q) { return (q.w >> 31) != 0u; }

__device__ __forceinline__ float box_area(const uint4 &q, const GridStep &g) {
    const float x = (float)((q.x >> 16) - (q.x & 0xffffu)) * g.s[0], y = (float)((q.y >> 16) - (q.y & 0xffffu)) * g.s[1],
                z = (float)((q.z >> 16) - (q.z & 0xffffu)) * g.s[2];
    return x * y + y * z + z * x;
}

// The (at most four) children of the wide node at binary node v.  A tree of
// one leaf gives that leaf as the only child.
__device__ __forceinline__ Kids wide_children(const uint4 *__restrict__ nodes, uint32_t v, const GridStep &g) {
    Kids k;
    const uint4 root = nodes[v];
    if (is_leaf(root)) {
        k.id[0] = v;
        k.rec[0] = root;
        k.n = 1;
        return k;
    }
    uint32_t open = v;
    int at = -1;  // slot of the opened node (its first child replaces it)
    k.n = 0;
    for (;;) {
        const uint32_t l = open + 1u;
        const uint4 ql = nodes[l];
        const uint32_t r = is_leaf(ql) ? l + 1u : ql.w;
        const uint4 qr = nodes[r];
        const int s = at < 0 ? k.n++ : at;
        k.id[s] = l;
        k.rec[s] = ql;
        k.id[k.n] = r;
        k.rec[k.n] = qr;
        k.n++;
        if (k.n == 4) break;
        at = -1;
        float best = -1.0f;
        for (int i = 0; i < k.n; ++i) {
            if (is_leaf(k.rec[i])) continue;
            const float a = box_area(k.rec[i], g);
            if (a > best) {
                best = a;
                at = i;
            }
        }
        if (at < 0) break;
        open = k.id[at];
    }
    return k;
}

__global__ __launch_bounds__(kWb) void k_wide_begin(uint32_t *__restrict__ cnt, uint32_t *__restrict__ roots,
                                                    uint32_t *__restrict__ flag, uint32_t n_flag) {
    for (uint32_t i = blockIdx.x * kWb + threadIdx.x; i < n_flag; i += gridDim.x * kWb) flag[i] = i == 0u ? 1u : 0u;
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i <= kWideLevels; i += kWb) cnt[i] = i == 0u ? 1u : 0u;
        if (threadIdx.x == 0) roots[0] = 0u;
    }
}

// Level `level`: roots[lo, hi) are its wide nodes (cnt[i] of level i); their
// inner children are appended after hi and counted in cnt[level + 1].  Every
// binary node is appended at most once, so at most n_inner entries are used.
__global__ __launch_bounds__(kWb) void k_wide_level(const uint4 *__restrict__ nodes, uint32_t level, GridStep g,
                                                    uint32_t *cnt, uint32_t *roots, uint32_t *__restrict__ flag) {
    uint32_t lo = 0u;
    for (uint32_t i = 0; i < level; ++i) lo += cnt[i];
    const uint32_t hi = lo + cnt[level];
    for (uint32_t j = lo + blockIdx.x * kWb + threadIdx.x; j < hi; j += gridDim.x * kWb) {
        const Kids k = wide_children(nodes, roots[j], g);
        for (int i = 0; i < k.n; ++i) {
            if (is_leaf(k.rec[i])) continue;
            const uint32_t at = atomicAdd(&cnt[level + 1u], 1u);
            roots[hi + at] = k.id[i];
            flag[k.id[i]] = 1u;
        }
    }
}

__global__ __launch_bounds__(kWb) void k_wide_emit(const uint4 *__restrict__ nodes, const uint32_t *__restrict__ roots,
                                                   uint32_t n_wide, const uint32_t *__restrict__ index, GridStep g,
                                                   uint4 *__restrict__ wide) {
    const uint32_t j = blockIdx.x * kWb + threadIdx.x;
    if (j >= n_wide) return;
    const uint32_t v = roots[j];
    const Kids k = wide_children(nodes, v, g);
    uint4 *out = wide + 4 * (size_t)index[v];
    for (int i = 0; i < 4; ++i) {
        // an unused slot: an inverted box, and a leaf of no triangles should its test pass all the same
        uint4 q = make_uint4(0x0000ffffu, 0x0000ffffu, 0x0000ffffu, 0x80000000u);
        if (i < k.n) {
            q = k.rec[i];
            if (!is_leaf(q)) q.w = index[k.id[i]];
        }
        out[i] = q;
    }
}

}  // namespace

namespace pm {

int build_wide(pm_bvh *b, hipStream_t s) {
    const uint32_t n = (uint32_t)b->n_nodes;
    const uint32_t tiles = (n + pmd::kScanTile - 1) / pmd::kScanTile, np = tiles * pmd::kScanTile;
    // one arena: flags, their exclusive scan (two arrays), tile sums, level counts, wide nodes' binary nodes
    const size_t words = (size_t)np + (np + 1) + np + (tiles + 1) + (kWideLevels + 1) + (n / 2 + 1);
    uint32_t *mem = nullptr;
    PM_HIP(hipMalloc(&mem, sizeof(uint32_t) * words));
    uint32_t *flag = mem, *index = flag + np, *fill = index + np + 1, *bsum = fill + np, *cnt = bsum + tiles + 1,
             *roots = cnt + kWideLevels + 1;
    GridStep g;
    for (int a = 0; a < 3; ++a) g.s[a] = b->qstep[a];
    uint32_t c[kWideLevels + 1];
    auto run = [&]() -> int {
        hipLaunchKernelGGL(k_wide_begin, dim3(std::min(np / kWb, 2048u)), dim3(kWb), 0, s, cnt, roots, flag, np);
        const uint32_t grid = std::max(1u, std::min((n + kWb - 1) / kWb, 1024u));
        uint32_t level = 0;
        // a tree of depth d has inner nodes on at most d levels
        const uint32_t most = std::min<uint32_t>(kWideLevels, (uint32_t)std::max(b->depth, 1));
        for (const uint32_t upto : {std::min(kWideLevelsFirst, most), most}) {
            for (; level < upto; ++level)
                hipLaunchKernelGGL(k_wide_level, dim3(grid), dim3(kWb), 0, s, (const uint4 *)b->d_nodes, level, g, cnt,
                                   roots, flag);
            PM_HIP(hipGetLastError());
            PM_HIP(hipMemcpyAsync(c, cnt, sizeof(c), hipMemcpyDeviceToHost, s));
            PM_HIP(hipStreamSynchronize(s));
            if (c[level] == 0u) break;
        }
        if (c[level] != 0u) return PM_OK;  // deeper than kWideLevels: binary walks only
        uint32_t total = 0;
        for (uint32_t i = 0; i < level; ++i) total += c[i];
        PM_HIP(hipMalloc(&b->d_wide, sizeof(uint4) * 4 * (size_t)total));
        b->n_wide = total;
        launch_bucket_scan(flag, index, fill, bsum, np, s);
        hipLaunchKernelGGL(k_wide_emit, dim3((total + kWb - 1) / kWb), dim3(kWb), 0, s, (const uint4 *)b->d_nodes,
                           (const uint32_t *)roots, total, (const uint32_t *)index, g, b->d_wide);
        PM_HIP(hipGetLastError());
        PM_HIP(hipStreamSynchronize(s));
        return PM_OK;
    };
    const int rc = run();
    (void)hipFree(mem);
    return rc;
}

}  // namespace pm
