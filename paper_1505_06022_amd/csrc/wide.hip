// Four-child nodes for the wide walk, merged on the device from the binary
// tree of link set 0 (both builders' output), so that the boxes, leaves and
// triangle records are those of the binary tree.
//
// The tree is recovered from the preorder: the left child of inner node v is
// v + 1 and the right child the node after the left subtree (its skip link; a
// leaf is its own subtree).  From the root down, a wide node takes a binary
// node's two children and opens the inner child of largest box area until it
// has four; its inner children become wide nodes.  A wide node's index is the
// rank of its binary node among all wide nodes' in preorder, so the layout does
// not depend on the order of the atomics and a subtree is contiguous.
//
// The descent is a chain of dependent reads, three for each level.  A workgroup
// expands its nodes in LDS through as many levels as it can: it hands nodes to
// the next launch only while too few workgroups have work (its list outgrows
// its threads) or when its list is full.  For 92,000 binary nodes two launches
// do it in 67 us where one launch for each of 16 levels took 117, and 160 with
// the gaps between them.
//
// A small tree (kHostMerge) is merged on the host by the same code: the launches,
// two allocations and two synchronisations of the merge were half of the build of
// a 36-triangle box.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "runtime.h"
#include "sppm_scan.h"

namespace {

constexpr int kWb = 256;
// Levels tried before the tree is left to the binary walks (the 2^20-triangle
// soup has 13; a ray through a chain of 32 would need more stack than the wide
// walk has).
constexpr uint32_t kWideLevels = 32;
// Launches before the first look at what is left, and workgroups of each.
constexpr uint32_t kWideFirst = 3, kWideGrid = 1024;
// Entries of a workgroup's list; the room of one round's children is kept free.
constexpr uint32_t kWideList = 4096, kWideRoom = 4 * kWb;

// Counters: [0, kWideLevels + 1) nodes handed to each launch, then flags.
constexpr uint32_t kWideDeep = kWideLevels + 1, kWideBad = kWideLevels + 2, kWideCounters = kWideLevels + 3;
struct Kids {
    uint32_t id[4];
    uint4 rec[4];
    int n;
};

struct GridStep {
    float s[3];
};

__host__ __device__ __forceinline__ bool is_leaf(const uint4 &q) { return (q.w >> 31) != 0u; }

__host__ __device__ __forceinline__ float box_area(const uint4 &q, const GridStep &g) {
    const float x = (float)((q.x >> 16) - (q.x & 0xffffu)) * g.s[0], y = (float)((q.y >> 16) - (q.y & 0xffffu)) * g.s[1],
                z = (float)((q.z >> 16) - (q.z & 0xffffu)) * g.s[2];
    return x * y + y * z + z * x;
}

// The (at most four) children of the wide node at binary node v.  A tree of
// one leaf gives that leaf as the only child.  A link outside the n nodes (an
// inconsistent tree) gives n = -1.
__host__ __device__ __forceinline__ Kids wide_children(const uint4 *__restrict__ nodes, uint32_t n, uint32_t v,
                                                       const GridStep &g) {
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
        if (l >= n) {
            k.n = -1;
            break;
        }
        const uint4 ql = nodes[l];
        const uint32_t r = is_leaf(ql) ? l + 1u : ql.w;
        if (r >= n) {
            k.n = -1;
            break;
        }
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

// Record i of the wide node with these children, an inner child's still with
// the binary node's link.
__host__ __device__ __forceinline__ uint4 wide_record(const Kids &k, int i) {
    // an unused slot: an inverted box, and a leaf of no triangles should its test pass all the same
    return i < k.n ? k.rec[i] : make_uint4(0x0000ffffu, 0x0000ffffu, 0x0000ffffu, 0x80000000u);
}

// A node to expand: binary node, level of its wide node.
__global__ __launch_bounds__(kWb) void k_wide_begin(uint32_t *__restrict__ cnt, uint2 *__restrict__ list,
                                                    uint32_t *__restrict__ flag, uint32_t n_flag) {
    for (uint32_t i = blockIdx.x * kWb + threadIdx.x; i < n_flag; i += gridDim.x * kWb) flag[i] = i == 0u ? 1u : 0u;
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i < kWideCounters; i += kWb) cnt[i] = i == 0u ? 1u : 0u;
        if (threadIdx.x == 0) list[0] = make_uint2(0u, 0u);
    }
}

// Expands the cnt[launch] nodes of `in`, whole subtrees where it can; what is
// left goes to `out` and cnt[launch + 1].  Every binary node is handed over at
// most once, so a list has room for all inner nodes.  Every node of `in` is
// expanded at least once, so launch kWideLevels has none left to hand over.
__global__ __launch_bounds__(kWb) void k_wide_expand(const uint4 *__restrict__ nodes, uint32_t n, uint32_t launch,
                                                     GridStep g, uint32_t *cnt, const uint2 *__restrict__ in,
                                                     uint2 *__restrict__ out, uint32_t *__restrict__ flag) {
    __shared__ uint2 list[kWideList];
    __shared__ uint32_t size, at;
    const uint32_t total = cnt[launch];
    // nodes for each workgroup: as few as spread over all of them
    const uint32_t piece = min(max((total + gridDim.x - 1u) / gridDim.x, 1u), (uint32_t)kWb);
    const uint32_t most = total < 4u * gridDim.x ? (uint32_t)kWb : kWideList - kWideRoom;
    for (uint32_t base = blockIdx.x * piece; base < total; base += gridDim.x * piece) {
        const uint32_t have = min(piece, total - base);
        if (threadIdx.x < have) list[threadIdx.x] = in[base + threadIdx.x];
        if (threadIdx.x == 0) size = have;
        __syncthreads();
        uint32_t m = have;
        while (m > 0u) {
            // the last entries, one to a thread
            const uint32_t take = min(m, (uint32_t)kWb);
            uint2 e = make_uint2(0u, 0u);
            if (threadIdx.x < take) e = list[m - take + threadIdx.x];
            __syncthreads();
            if (threadIdx.x == 0) size = m - take;
            __syncthreads();
            if (threadIdx.x < take) {
                const Kids k = wide_children(nodes, n, e.x, g);
                if (k.n < 0) atomicOr(&cnt[kWideBad], 1u);
                for (int i = 0; i < k.n; ++i) {
                    if (is_leaf(k.rec[i])) continue;
                    if (e.y + 1u >= kWideLevels) {
                        cnt[kWideDeep] = 1u;
                        continue;
                    }
                    list[atomicAdd(&size, 1u)] = make_uint2(k.id[i], e.y + 1u);  // at most kWideList: see `most`
                    flag[k.id[i]] = 1u;
                }
            }
            __syncthreads();
            m = size;
            if (m > most) {
                if (threadIdx.x == 0) at = atomicAdd(&cnt[launch + 1u], m);
                __syncthreads();
                for (uint32_t i = threadIdx.x; i < m; i += kWb) out[at + i] = list[i];
                m = 0u;
            }
            __syncthreads();
        }
    }
}

__global__ __launch_bounds__(kWb) void k_wide_emit(const uint4 *__restrict__ nodes, uint32_t n,
                                                   const uint32_t *__restrict__ flag,
                                                   const uint32_t *__restrict__ index, GridStep g,
                                                   uint4 *__restrict__ wide) {
    const uint32_t v = blockIdx.x * kWb + threadIdx.x;
    if (v >= n || flag[v] == 0u) return;
    const Kids k = wide_children(nodes, n, v, g);
    uint4 *out = wide + 4 * (size_t)index[v];
    for (int i = 0; i < 4; ++i) {
        uint4 q = wide_record(k, i);
        if (i < k.n && !is_leaf(q)) q.w = index[k.id[i]];
        out[i] = q;
    }
}

GridStep grid_step(const pm_bvh *b) {
    GridStep g;
    for (int a = 0; a < 3; ++a) g.s[a] = b->qstep[a];
    return g;
}

}  // namespace

namespace pm {

int merge_wide_host(const pm_bvh *b, const uint32_t *binary, std::vector<uint32_t> &out) {
    const uint4 *nodes = (const uint4 *)binary;
    const uint32_t n = (uint32_t)b->n_nodes;
    const GridStep g = grid_step(b);
    // in the order of the binary nodes: a node's inner children are taken in theirs, a subtree before the next
    struct Todo {
        uint32_t node, level, slot;  // slot: where its parent has its index
    };
    std::vector<Todo> todo;
    out.clear();
    out.reserve(4 * (size_t)n + 16);
    todo.push_back({0u, 0u, 0u});
    while (!todo.empty()) {
        const Todo e = todo.back();
        todo.pop_back();
        const Kids k = wide_children(nodes, n, e.node, g);
        if (k.n < 0) return set_error("inconsistent binary tree"), PM_ERR_STATE;
        const uint32_t at = (uint32_t)out.size();
        if (at) out[e.slot] = at / 16;
        out.resize(at + 16);
        const size_t first = todo.size();
        for (int i = 0; i < 4; ++i) {
            const uint4 q = wide_record(k, i);
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
            std::copy(w, w + 4, out.begin() + at + 4 * i);
            if (i < k.n && !is_leaf(k.rec[i])) todo.push_back({k.id[i], e.level + 1u, at + 4u * i + 3u});
        }
        if (todo.size() > first && e.level + 1u >= kWideLevels) return out.clear(), PM_OK;  // too deep
        std::sort(todo.begin() + first, todo.end(), [](const Todo &x, const Todo &y) { return x.node > y.node; });
    }
    return PM_OK;
}

WideBuild::~WideBuild() {
    if (mem_) (void)hipFree(mem_);
}

// *mem stays NULL where the device has no room: a BVH without four-child nodes
// takes the binary walks.
static int allocate(void **mem, size_t bytes) {
    const hipError_t e = hipMalloc(mem, bytes);
    if (e == hipSuccess) return PM_OK;
    *mem = nullptr;
    if (e != hipErrorOutOfMemory) return hip_fail(e, "hipMalloc");
    (void)hipGetLastError();
    return PM_OK;
}

int WideBuild::expand(const pm_bvh *b, hipStream_t s, uint32_t upto) {
    const GridStep g = grid_step(b);
    for (; launches_ < upto; ++launches_)
        hipLaunchKernelGGL(k_wide_expand, dim3(launches_ == 0 ? 1u : kWideGrid), dim3(kWb), 0, s,
                           (const uint4 *)b->d_nodes, n_, launches_, g, cnt_, (const uint2 *)list_[launches_ & 1u],
                           list_[(launches_ + 1u) & 1u], flag_);
    launch_bucket_scan(flag_, index_, fill_, bsum_, tiles_ * pmd::kScanTile, s);
    PM_HIP(hipGetLastError());
    return PM_OK;
}

int WideBuild::launch(const pm_bvh *b, hipStream_t s) {
    n_ = (uint32_t)b->n_nodes;
    tiles_ = (n_ + pmd::kScanTile - 1) / pmd::kScanTile;
    const uint32_t np = tiles_ * pmd::kScanTile;
    // one allocation: two lists of nodes, flags, their exclusive scan (two arrays), tile sums, counters
    const size_t list = n_ / 2 + 1;
    if (int rc = allocate(&mem_, sizeof(uint2) * 2 * list +
                                     sizeof(uint32_t) * ((size_t)np + (np + 1) + np + (tiles_ + 1) + kWideCounters)))
        return rc;
    if (!mem_) return PM_OK;
    list_[0] = (uint2 *)mem_;
    list_[1] = list_[0] + list;
    flag_ = (uint32_t *)(list_[1] + list);
    index_ = flag_ + np;
    fill_ = index_ + np + 1;
    bsum_ = fill_ + np;
    cnt_ = bsum_ + tiles_ + 1;
    hipLaunchKernelGGL(k_wide_begin, dim3(std::min(np / kWb, 2048u)), dim3(kWb), 0, s, cnt_, list_[0], flag_, np);
    // with at most kWb inner nodes the first workgroup keeps them all
    return expand(b, s, n_ / 2 <= (uint32_t)kWb ? 1u : kWideFirst);
}

int WideBuild::finish(pm_bvh *b, hipStream_t s) {
    uint32_t read[1 + kWideCounters], *const c = read + 1;  // wide nodes, then the counters
    if (!mem_) {
        PM_HIP(hipStreamSynchronize(s));
        return PM_OK;
    }
    for (;;) {
        PM_HIP(hipMemcpyAsync(read, bsum_ + tiles_, sizeof(read), hipMemcpyDeviceToHost, s));
        PM_HIP(hipStreamSynchronize(s));
        if (c[kWideBad]) return set_error("inconsistent binary tree"), PM_ERR_STATE;
        if (c[kWideDeep]) return PM_OK;  // deeper than kWideLevels: binary walks only
        if (launches_ == kWideLevels || c[launches_] == 0u) break;
        if (int rc = expand(b, s, std::min(launches_ + kWideFirst, kWideLevels))) return rc;
    }
    const GridStep g = grid_step(b);
    if (int rc = allocate((void **)&b->d_wide, sizeof(uint4) * 4 * (size_t)read[0])) return rc;
    if (!b->d_wide) return PM_OK;
    b->n_wide = read[0];
    hipLaunchKernelGGL(k_wide_emit, dim3((n_ + kWb - 1) / kWb), dim3(kWb), 0, s, (const uint4 *)b->d_nodes, n_,
                       (const uint32_t *)flag_, (const uint32_t *)index_, g, b->d_wide);
    PM_HIP(hipGetLastError());
    PM_HIP(hipStreamSynchronize(s));
    return PM_OK;
}

}  // namespace pm
