// The scene fingerprint's hash over a long run of 32-bit words, on the device.
//
// The hash is h' = (h ^ w) p mod 2^64 with p = 2^40 + 435 over words w < 2^32, a
// chain of one multiplication a word: 2.1 ms on the host for the 2.5 million
// words of 250,000 triangles.  It can be cut into segments all the same:
//  * the low 32 bits follow L' = 435 (L ^ w) mod 2^32, and bit i of L' depends
//    on bits 0 .. i only.  With the bits below 4 j of a segment's start known,
//    its next four bits are one of 16; all 16 are run, giving the segment's map
//    from these bits at its start to those at its end, and the maps are
//    followed from the first segment to the last: within a workgroup's 16
//    segments by the workgroup, over the workgroups by one lane.  Eight such
//    passes give every segment's low half.
//  * the high 32 bits follow H' = 435 H + (a term of L and w), so a segment
//    run from H = 0 (k_segment_ends) gives its effect on any H.
// For 250,000 triangles the kernels take 0.25 ms and the upload 0.2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "runtime.h"
#include "sppm_host.h"

namespace {

constexpr int kHashBlock = 256, kFollow = 512;
constexpr uint32_t kGroup = kHashBlock / 16;      // segments of a workgroup
constexpr uint32_t kMinSegment = 320;             // words; a multiple of 4
constexpr uint32_t kSegments = kFollow * kGroup;  // at most

__device__ __forceinline__ uint32_t times435(uint32_t x) {  // 435 = 3 (16 * 9 + 1)
    const uint32_t y = (x << 3) + x, z = (y << 4) + x;
    return (z << 1) + z;
}

__device__ __forceinline__ uint32_t map_at(unsigned long long m, uint32_t v) { return (uint32_t)(m >> (4u * v)) & 15u; }

// Pass j.  A map has 16 four-bit entries: the bits [4 j, 4 j + 4) of the low half
// after a segment (map) or a workgroup's 16 segments (all) for each value of them
// before it.  16 lanes a segment.  first[block]: the previous pass's bits before
// the workgroup's first segment, with which its segments' starts are completed;
// pass 8 does only that.
__global__ __launch_bounds__(kHashBlock) void k_nibble_maps(const uint32_t *__restrict__ words, uint32_t n, uint32_t seg,
                                                            uint32_t n_seg, int j, uint32_t *__restrict__ start,
                                                            unsigned long long *__restrict__ map,
                                                            unsigned long long *__restrict__ all,
                                                            const uint32_t *__restrict__ first) {
    __shared__ unsigned long long maps[kGroup];
    const uint32_t g = threadIdx.x >> 4, v = threadIdx.x & 15u, s = blockIdx.x * kGroup + g;
    const bool in = s < n_seg;
    uint32_t L = 0u;
    if (j > 0) {
        if (v == 0u && in) maps[g] = map[s];
        __syncthreads();
        if (in) {
            uint32_t r = first[blockIdx.x];
            for (uint32_t t = 0; t < g; ++t) r = map_at(maps[t], r);
            L = (j > 1 ? start[s] : 0u) | (r << (4 * (j - 1)));
        }
        __syncthreads();
        if (v == 0u && in) start[s] = L;
    }
    if (j == 8) return;
    L |= v << (4 * j);
    const uint32_t b = in ? s * seg : 0u, e = in ? min(b + seg, n) : 0u;
    uint32_t i = b;
    for (; i + 4u <= e; i += 4u) {
        const uint4 w = *(const uint4 *)(words + i);
        L = times435(L ^ w.x);
        L = times435(L ^ w.y);
        L = times435(L ^ w.z);
        L = times435(L ^ w.w);
    }
    for (; i < e; ++i) L = times435(L ^ words[i]);
    // (a segment past the end changes nothing)
    unsigned long long m = (unsigned long long)((L >> (4 * j)) & 15u) << (4u * v);
    for (int off = 1; off < 16; off <<= 1) m |= __shfl_xor(m, off);
    if (v == 0u) {
        maps[g] = m;
        if (in) map[s] = m;
    }
    __syncthreads();
    if (g != 0u) return;
    uint32_t r = v;
    for (uint32_t t = 0; t < kGroup; ++t) r = map_at(maps[t], r);
    m = (unsigned long long)r << (4u * v);
    for (int off = 1; off < 16; off <<= 1) m |= __shfl_xor(m, off);
    if (v == 0u) all[blockIdx.x] = m;
}

// Follows the workgroups' maps from v: first[i] is the value before map i.
__global__ __launch_bounds__(kFollow) void k_follow_maps(const unsigned long long *__restrict__ all, uint32_t n,
                                                         uint32_t v, uint32_t *__restrict__ first) {
    __shared__ unsigned long long maps[kFollow];
    __shared__ uint8_t at[kFollow];
    if (threadIdx.x < n) maps[threadIdx.x] = all[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0)
        for (uint32_t t = 0; t < n; t += 8) {
            unsigned long long m[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) m[u] = maps[t + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                at[t + u] = (uint8_t)v;
                v = map_at(m[u], v);
            }
        }
    __syncthreads();
    if (threadIdx.x < n) first[threadIdx.x] = at[threadIdx.x];
}

// The whole state after each segment from the low half start[s] and high half 0.
__global__ __launch_bounds__(64) void k_segment_ends(const uint32_t *__restrict__ words, uint32_t n, uint32_t seg,
                                                     uint32_t n_seg, const uint32_t *__restrict__ start,
                                                     unsigned long long *__restrict__ end) {
    const uint32_t s = blockIdx.x * 64u + threadIdx.x;
    if (s >= n_seg) return;
    const uint32_t b = s * seg, e = min(b + seg, n);
    unsigned long long h = start[s];
    uint32_t i = b;
    for (; i + 4u <= e; i += 4u) {
        const uint4 w = *(const uint4 *)(words + i);
        h = (h ^ w.x) * pm::kHashPrime;
        h = (h ^ w.y) * pm::kHashPrime;
        h = (h ^ w.z) * pm::kHashPrime;
        h = (h ^ w.w) * pm::kHashPrime;
    }
    for (; i < e; ++i) h = (h ^ words[i]) * pm::kHashPrime;
    end[s] = h;
}

}  // namespace

namespace pm {

DeviceHash::~DeviceHash() { release(); }

void DeviceHash::release() {
    if (mem_) (void)hipFree(mem_);
    mem_ = nullptr;
}

int DeviceHash::launch(uint64_t h, const void *a, size_t words_a, const void *b, size_t words_b, hipStream_t st) {
    h_ = h;
    n_ = (uint32_t)(words_a + words_b);
    seg_ = std::max(kMinSegment, (n_ / kSegments + 4u) & ~3u);
    n_seg_ = (n_ + seg_ - 1) / seg_;
    const uint32_t blocks = (n_seg_ + kGroup - 1) / kGroup;
    const size_t list = (size_t)blocks * kGroup;
    // the segments' maps (in the end their ends), the workgroups', starts, first bits, the words
    PM_HIP(hipMalloc(&mem_, sizeof(uint64_t) * (list + kFollow) + sizeof(uint32_t) * (list + kFollow + (size_t)n_)));
    unsigned long long *map = (unsigned long long *)mem_, *all = map + list;
    uint32_t *start = (uint32_t *)(all + kFollow), *first = start + list, *words = first + kFollow;
    PM_HIP(hipMemcpyAsync(words, a, sizeof(uint32_t) * words_a, hipMemcpyHostToDevice, st));
    PM_HIP(hipMemcpyAsync(words + words_a, b, sizeof(uint32_t) * words_b, hipMemcpyHostToDevice, st));
    for (int j = 0; j <= 8; ++j) {
        hipLaunchKernelGGL(k_nibble_maps, dim3(blocks), dim3(kHashBlock), 0, st, (const uint32_t *)words, n_, seg_,
                           n_seg_, j, start, map, all, (const uint32_t *)first);
        if (j < 8)
            hipLaunchKernelGGL(k_follow_maps, dim3(1), dim3(kFollow), 0, st, (const unsigned long long *)all, blocks,
                               (uint32_t)(h >> (4 * j)) & 15u, first);
    }
    hipLaunchKernelGGL(k_segment_ends, dim3((n_seg_ + 63) / 64), dim3(64), 0, st, (const uint32_t *)words, n_, seg_,
                       n_seg_, (const uint32_t *)start, map);
    PM_HIP(hipGetLastError());
    return PM_OK;
}

int DeviceHash::finish(uint64_t &h, hipStream_t st) {
    std::vector<uint64_t> end(n_seg_);
    PM_HIP(hipMemcpyAsync(end.data(), mem_, sizeof(uint64_t) * n_seg_, hipMemcpyDeviceToHost, st));
    PM_HIP(hipStreamSynchronize(st));
    uint32_t step = 1u;  // 435^seg
    for (uint32_t i = 0; i < seg_; ++i) step *= 435u;
    uint32_t high = (uint32_t)(h_ >> 32);
    for (uint32_t s = 0; s < n_seg_; ++s) {
        if (s + 1 == n_seg_) {
            step = 1u;
            for (uint32_t i = s * seg_; i < n_; ++i) step *= 435u;
        }
        high = high * step + (uint32_t)(end[s] >> 32);
    }
    h = (uint64_t)high << 32 | (uint32_t)end[n_seg_ - 1];
    return PM_OK;
}

}  // namespace pm
