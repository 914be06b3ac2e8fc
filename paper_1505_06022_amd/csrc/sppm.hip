// Stochastic progressive photon mapping on the device (Sec. 2): single-scene
// kernels (eye pass, photon pass, hashed-grid build, range query, progressive
// update, resolve, adjoint replay) and their host driver.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

#include "runtime.h"
#include "sppm.h"
#include "sppm_dev.h"
#include "sppm_host.h"
#include "sppm_scan.h"

namespace {

using namespace pmd;

// The kernels that trace paths have two forms.  kWide: the wide walk, with its
// stacks in LDS (24 KB a workgroup) and PM_PASS_WAVES; else the binary walk
// only, for handles whose rays never take the other (one link set forced, or a
// BVH without four-child nodes): its registers and the photons' LDS leave room
// for five waves a SIMD, and the eye pass for six.  One form for both took 2.25
// ms an iteration with one link set (1280x720, 2^20 photons, calls of 8) instead
// of 1.79, and 1.90 with the eye pass at five waves.
#define PM_STACK()                                                                          \
    __shared__ uint32_t wide_stack[kWide ? kBlock / 64 : 1][kWide ? kStackWords : 1];       \
    uint32_t *const stk = kWide ? wide_stack[threadIdx.x >> 6] : nullptr
// The same for the photons on their way to the store.
#define PM_SINK()                                   \
    __shared__ float4 photon_buf[kBlock / 64][kSinkWords]; \
    const PhotonSink sink{photon_buf[threadIdx.x >> 6], 0u}

template <bool kWide>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kWide ? 4 : 6)))
void k_eye(SppmDev d, uint32_t k, int32_t emission) {
    int64_t p = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    PM_STACK();
    eye_elem(d, k, p, p < d.P, emission != 0, stk);
}

// The statistics variants (PM_PROFILE_COUNT): the same work, plus counts of
// paths, rays, box and triangle tests, and of the range query's buckets and
// photons, added to d.stats once per wavefront.
__global__ __launch_bounds__(kBlock) void k_eye_stats(SppmDev d, uint32_t k, int32_t emission) {
    int64_t p = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    LaneStats ls;
    eye_elem<true>(d, k, p, p < d.P, emission != 0, nullptr, &ls);
    wave_stats_flush(d.stats + kStatEyePaths, ls);
}

// The wave's place in the grid, each XCD owning a contiguous range.
__device__ __forceinline__ int64_t wave_index() {
    return (int64_t)xcd_block(blockIdx.x, gridDim.x) * (kBlock / 64) + (threadIdx.x >> 6);
}

// One path per lane, the first per_wave lanes of each wave.
template <bool kRecord, bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon(SppmDev d, uint32_t k, uint32_t per_wave,
                                                               uint16_t *__restrict__ mat_tab,
                                                               long long *__restrict__ adj_tab) {
    const uint32_t lane = threadIdx.x & 63u;
    const int64_t n = wave_index() * per_wave + lane;
    PM_STACK();
    PM_SINK();
    photon_elem<kRecord>(d, k, (uint32_t)n, lane < per_wave && n < d.n_paths, mat_tab, adj_tab, stk, sink);
}

// Persistent photon lanes with path regeneration.
template <bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon_regen(SppmDev d, uint32_t k) {
    PM_STACK();
    PM_SINK();
    photon_regen_loop(d, k, d.refill, stk, sink);
}

__global__ __launch_bounds__(kBlock) void k_photon_regen_stats(SppmDev d, uint32_t k) {
    PM_SINK();
    photon_regen_loop<false, true>(d, k, d.refill, nullptr, sink);
}

// Two-phase photon pass (PM_PHOTON_TWO_PHASE): regeneration that sets the
// last paths of each wavefront aside once the path counter has run out, then
// a launch over the paths set aside.
template <bool kStats, bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon_head(SppmDev d, uint32_t k, PathQueue q) {
    PM_STACK();
    PM_SINK();
    photon_regen_loop<false, kStats, true>(d, k, d.refill, stk, sink, nullptr, nullptr, q);
}

template <bool kStats, bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon_tail(SppmDev d, PathQueue q) {
    PM_STACK();
    PM_SINK();
    photon_queue_loop<false, kStats>(d, q, (uint32_t)wave_index(), gridDim.x * (kBlock / 64), stk, sink, nullptr, nullptr);
}

// The same two launches, recording each path's stored-photon materials for
// the adjoint (a queued path keeps its row of the tables).
template <bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon_head_rec(SppmDev d, uint32_t k, PathQueue q,
                                                            uint16_t *__restrict__ mat_tab,
                                                            long long *__restrict__ adj_tab) {
    PM_STACK();
    PM_SINK();
    photon_regen_loop<true, false, true>(d, k, d.refill, stk, sink, mat_tab, adj_tab, q);
}

template <bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon_tail_rec(SppmDev d, PathQueue q,
                                                            uint16_t *__restrict__ mat_tab,
                                                            long long *__restrict__ adj_tab) {
    PM_STACK();
    PM_SINK();
    photon_queue_loop<true, false>(d, q, (uint32_t)wave_index(), gridDim.x * (kBlock / 64), stk, sink, mat_tab, adj_tab);
}

// Regeneration from a queue of started paths in LDS (PM_PHOTON_POOL): each
// wavefront owns kPoolWords x kPoolSlots words of the workgroup's LDS.
template <bool kStats>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_photon_pool(SppmDev d, uint32_t k) {
    __shared__ uint32_t pool[kBlock / 64][kPoolWords * kPoolSlots];
    photon_pool_loop<kStats>(d, k, pool[threadIdx.x >> 6]);
}

// Regeneration at ray granularity (PM_PHOTON_RAY_REGEN).
__global__ __launch_bounds__(kBlock) void k_photon_stream(SppmDev d, uint32_t k) {
    photon_stream_loop(d, k, d.refill);
}

__global__ __launch_bounds__(kBlock) void k_photon_stream_stats(SppmDev d, uint32_t k) {
    photon_stream_loop<true>(d, k, d.refill);
}

// The same, recording each path's stored-photon materials for the adjoint.
template <bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon_regen_rec(SppmDev d, uint32_t k, uint16_t *__restrict__ mat_tab,
                                                             long long *__restrict__ adj_tab) {
    PM_STACK();
    PM_SINK();
    photon_regen_loop<true>(d, k, d.refill, stk, sink, mat_tab, adj_tab);
}

// One pass of the one-bounce-per-pass schedule; the grid covers the slots
// with the same workgroup-to-slot map in every pass.
template <bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon_pass(SppmDev d, uint32_t k, PassSlots ps) {
    PM_STACK();
    PM_SINK();
    photon_pass_elem(d, k, ps, xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x, stk, sink);
}

// Paths no pass started, before the drain adds the paths still in flight.
__global__ void k_pass_tally(SppmDev d) {
    if (threadIdx.x == 0) d.counters[3] = d.n_paths - min(d.counters[2], d.n_paths);
}

template <bool kWide>
__global__ __launch_bounds__(kBlock) PM_PASS_WAVES void k_photon_drain(SppmDev d, uint32_t k, PassSlots ps) {
    PM_STACK();
    PM_SINK();
    photon_drain_elem(d, k, ps, xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x, stk, sink);
}

// Start of a photon pass: clear its store's photon count; handed: where the path
// counter starts (0; the default pass of few paths, which does not use it, leaves
// the number of its paths there).
__global__ void k_photon_begin(SppmDev d, uint32_t handed) {
    if (threadIdx.x == 0) {
        d.counters[0] = 0u;
        d.counters[2] = handed;
    }
}

// Start of an eye pass: clear the R_max accumulator.
__global__ void k_rmax_clear(SppmDev d) {
    if (threadIdx.x == 0) *d.r2max = 0ull;
}

// Frame setup: clear the photon and path counters and the R_max accumulator.
__global__ void k_begin(SppmDev d) {
    if (threadIdx.x == 0) {
        d.counters[0] = 0u;
        d.counters[2] = 0u;
        *d.r2max = 0ull;
    }
}

// Largest R^2 over valid hit points: a grid-stride maximum per lane, reduced
// across the workgroup, then one atomic per workgroup (positive doubles order
// like their bit patterns).  Launched with few workgroups so the atomics on
// the single result do not serialise.
constexpr uint32_t kRmaxBlocks = 512;

__global__ __launch_bounds__(kBlock) void k_rmax(SppmDev d, const double *__restrict__ R2src) {
    __shared__ unsigned long long part[kBlock / 64];
    unsigned long long v = 0ull;
    for (int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x; p < d.P; p += (int64_t)gridDim.x * kBlock) {
        unsigned long long x = rmax_lane(d, R2src, p);
        v = x > v ? x : v;
    }
    for (int off = 32; off > 0; off >>= 1) {
        unsigned long long o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) v = part[w] > v ? part[w] : v;
        if (v) atomicMax(d.r2max, v);
    }
}

__global__ __launch_bounds__(kBlock) void k_count(SppmDev d, uint32_t *__restrict__ cell_count) {
    uint32_t n_ph = stored_photons(d);
    Grid gr = make_grid(d);
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < n_ph; j += gridDim.x * kBlock) count_elem(d, gr, j, cell_count);
}

__global__ __launch_bounds__(kBlock) void k_scatter(SppmDev d, const uint32_t *__restrict__ start,
                                                    float4 *__restrict__ sorted) {
    uint32_t n_ph = stored_photons(d);
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < n_ph; j += gridDim.x * kBlock)
        scatter_elem(d, j, start, sorted);
}

// Every lane takes part (the wave may scan a dense hit point together); a wave
// takes kHits pixels.
template <int kHits, bool kStats>
__global__ __launch_bounds__(kBlock) void k_gather(SppmDev d, const uint32_t *__restrict__ start,
                                                   const float4 *__restrict__ sorted) {
    const int64_t wave = (int64_t)xcd_block(blockIdx.x, gridDim.x) * (kBlock / 64) + (threadIdx.x >> 6);
    Grid gr = make_grid(d);
    gather_wave<kHits, kStats>(d, gr, wave * kHits + (threadIdx.x & 63), start, sorted);
}

// Stochastic spatial hashing: clear the keys, insert every stored photon
// (count and smallest key per entry), record each entry's survivor, gather.
__global__ __launch_bounds__(kBlock) void k_sh_clear(SppmDev d, uint32_t T) {
    for (uint32_t e = blockIdx.x * kBlock + threadIdx.x; e < T; e += gridDim.x * kBlock)
        d.sh_key[d.table_off + e] = ~0ull;
}

__global__ __launch_bounds__(kBlock) void k_sh_insert(SppmDev d, uint32_t k, uint32_t *__restrict__ count) {
    uint32_t n_ph = stored_photons(d);
    Grid gr = make_grid(d);
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < n_ph; j += gridDim.x * kBlock)
        sh_insert_elem(d, gr, k, j, count);
}

__global__ __launch_bounds__(kBlock) void k_sh_pick(SppmDev d, uint32_t k) {
    uint32_t n_ph = stored_photons(d);
    Grid gr = make_grid(d);
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < n_ph; j += gridDim.x * kBlock) sh_pick_elem(d, gr, k, j);
}

__global__ __launch_bounds__(kBlock) void k_sh_gather(SppmDev d, const uint32_t *__restrict__ count) {
    int64_t p = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if (p >= d.P) return;
    Grid gr = make_grid(d);
    sh_gather_elem(d, gr, p, count);
}

__global__ __launch_bounds__(kBlock) void k_update(SppmDev d, double *__restrict__ hist) {
    int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p < d.P) update_elem(d, p, hist);
}

__global__ __launch_bounds__(kBlock) void k_resolve(SppmDev d, int32_t K, float *__restrict__ img) {
    int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p < d.P) img[p] = resolve_elem(d, p, K);
}

__global__ __launch_bounds__(kBlock) void k_init_state(SppmDev d, double r0sq) {
    int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= d.P) return;
    d.N[p] = 0.0;
    d.R2[p] = r0sq;
    d.tau[p] = 0.0;
    d.D[p] = 0.0;
}

// ---------------------------------------------------------------------------
// Adjoint (gradient of an image loss by replay).  With sampling held fixed the
// radiance of pixel p is sum_k sum_c c / (pi R2_{p,k} K) + D_p / K, each
// contribution c = W rho_h / pi * phi_j, where phi_j carries rho_m / q_m for
// every earlier diffuse bounce on m.  Per iteration the replayed gather adds
// G_h = g_h / (pi R2_{h,k} K) times c to the photon's (path, bounce) entry and
// to the hit point's own material; a per-path suffix sum then gives the
// earlier-bounce terms.  Dividing by rho_m is left to the end of the iteration.
//
// Every sum is an integer sum, so the gradient does not depend on the order of
// the atomics or of the photons in their buckets.  Each term G_h c is rounded
// on its own to a fixed point whose scale is a power of two chosen per
// iteration from two maxima (of |G_h| wk_h over hit points, of the flux over
// stored photons), so that no term exceeds 2^39 units.  A (path, bounce) entry
// is a signed 64-bit sum (fewer than 2^24 hit points reach one photon); the
// per-material sums are 96-bit (two 64-bit words: the low 32 bits of each
// addend, and the rest), and each iteration's are converted to double once
// and added to the gradient in iteration order.
// ---------------------------------------------------------------------------
constexpr int kAdjTermBits = 39;

using i128 = __int128;

__device__ __forceinline__ void wide_add(unsigned long long *lo, unsigned long long *hi, i128 v) {
    atomicAdd(lo, (unsigned long long)(uint32_t)(uint64_t)v);
    atomicAdd(hi, (unsigned long long)(long long)(v >> 32));
}

// Per-material 96-bit sums: accumulate in LDS, then add each workgroup's sums
// to the global pair with the carry of the low word moved into the high one.
struct WideLds {
    unsigned long long lo[kMaxAdjMat], hi[kMaxAdjMat];
};

__device__ __forceinline__ void wide_clear(WideLds &w, int n_mat) {
    for (int m = threadIdx.x; m < n_mat; m += kBlock) {
        w.lo[m] = 0ull;
        w.hi[m] = 0ull;
    }
    __syncthreads();
}

__device__ __forceinline__ void wide_flush(WideLds &w, int n_mat, unsigned long long *__restrict__ glob) {
    __syncthreads();
    for (int m = threadIdx.x; m < n_mat; m += kBlock) {
        const unsigned long long lo = w.lo[m], hi = w.hi[m];
        if (lo | hi) {
            atomicAdd(&glob[m], lo & 0xffffffffull);
            atomicAdd(&glob[n_mat + m], hi + (lo >> 32));
        }
    }
}

__device__ __forceinline__ double adj_G(const float *__restrict__ g, int64_t p, double r2, double K) {
    return (double)g[p] / ((kPiD * r2) * K);
}

// Clears the iteration's maxima and per-material sums.
__global__ void k_adj_begin(unsigned long long *__restrict__ adj_max, unsigned long long *__restrict__ wide,
                            int32_t n_mat) {
    for (int i = threadIdx.x; i < 2 * n_mat; i += blockDim.x) wide[i] = 0ull;
    if (threadIdx.x < 2) adj_max[threadIdx.x] = 0ull;
}

// Maximum of v over the workgroup (non-negative doubles compare as their bit
// patterns): one atomic per workgroup.
__device__ __forceinline__ void block_max_atomic(unsigned long long v, unsigned long long *__restrict__ out) {
    __shared__ unsigned long long wave_max[kBlock / 64];
    for (int off = 32; off > 0; off >>= 1) {
        unsigned long long o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) v = wave_max[w] > v ? wave_max[w] : v;
        if (v) atomicMax(out, v);
    }
}

// Workgroups of the two maxima below: a grid-stride loop each, so that at
// most this many same-address atomics are issued.
constexpr uint32_t kAdjMaxBlocks = 256;

// max over valid hit points of |G_h| wk_h (non-negative doubles order like
// their bit patterns, so the maximum is an integer maximum)
__global__ __launch_bounds__(kBlock) void k_adj_gmax(SppmDev d, const double *__restrict__ R2k,
                                                     const float *__restrict__ g, double K,
                                                     unsigned long long *__restrict__ adj_max) {
    unsigned long long v = 0ull;
    for (int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x; p < d.P; p += (int64_t)gridDim.x * kBlock) {
        float4 hn = d.hp_nrm[p];
        if (__float_as_int(hn.w) >= 0) {
            double a = fabs(adj_G(g, p, R2k[p], K)) * (double)d.hp_pos[p].w;
            unsigned long long b = (unsigned long long)__double_as_longlong(a);
            v = b > v ? b : v;
        }
    }
    block_max_atomic(v, &adj_max[0]);
}

// max flux over the stored photons
__global__ __launch_bounds__(kBlock) void k_adj_phimax(SppmDev d, unsigned long long *__restrict__ adj_max) {
    const uint32_t n = min(d.counters[0], d.cap);
    unsigned long long v = 0ull;
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        unsigned long long b = (unsigned long long)__double_as_longlong((double)d.store[2 * (size_t)i].w);
        v = b > v ? b : v;
    }
    block_max_atomic(v, &adj_max[1]);
}

// Scale 2^(39 - e) with 2^e above the product of the two maxima, so
// |G_h wk_h phi_j| * scale < 2^39 for every pair (0: nothing to add).
__global__ void k_adj_scale(const unsigned long long *__restrict__ adj_max, double *__restrict__ scale) {
    if (threadIdx.x == 0) {
        const double bound = __longlong_as_double((long long)adj_max[0]) * __longlong_as_double((long long)adj_max[1]);
        double sc = 0.0;
        if (bound > 0.0 && bound < 1e300) {
            int e;
            (void)frexp(bound, &e);  // bound < 2^e
            sc = ldexp(1.0, kAdjTermBits - e);
        }
        *scale = sc;
    }
}

// The adjoint's range query, bound by its chain of reads and by the additions
// to the photons' table entries.  On small images it is split over lanes and
// waves like the forward one (gather_wave): a hit point whose buckets hold many
// photons is scanned by its whole wave, 320x180 with 2^16 photons 187 -> 114 us
// an iteration.  With 64 hit points a wave every lane scans its own: at 1280x720
// with 2^20 photons the whole-wave scans, 23 more registers and the additions
// of a wave to few entries at once made it 908 us instead of 701.
template <int kHits>
__global__ __launch_bounds__(kBlock) void k_gather_adj(SppmDev d, const double *__restrict__ R2k,
                                                       const uint32_t *__restrict__ start,
                                                       const float4 *__restrict__ sorted, const float *__restrict__ g,
                                                       double K, const double *__restrict__ scale_p,
                                                       long long *__restrict__ adj_tab, int32_t n_mat,
                                                       unsigned long long *__restrict__ wide) {
    __shared__ WideLds lds;
    wide_clear(lds, n_mat);
    const double scale = *scale_p;
    const uint32_t lane = threadIdx.x & 63u;
    const int64_t p = wave_index() * kHits + lane;
    const bool in = p < d.P && lane < (uint32_t)kHits;
    const float4 hn = in ? d.hp_nrm[p] : make_float4(0.0f, 0.0f, 0.0f, __int_as_float(-1));
    const bool valid = __float_as_int(hn.w) >= 0 && g[p] != 0.0f && scale > 0.0;
    const Grid gr = make_grid(d);
    const int32_t mb = d.max_bounces;
    float4 hx = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    double r2 = 0.0, G = 0.0;
    DiscCells dc{};
    uint32_t load = 0u;
    if (valid) {
        hx = d.hp_pos[p];
        r2 = R2k[p];
        G = adj_G(g, p, r2, K);
        dc = disc_cells(gr, hx, r2);
        if (kHits < 64) load = disc_load(d, gr, dc, start);
    }
    // one photon's term of a hit point: to the photon's entry, and returned
    auto term = [&](double Gp, double wk, const float4 &a, const float4 &b) {
        const double cc = wk * (double)a.w;
        const long long q = __double2ll_rn((Gp * cc) * scale);
        const uint32_t meta = __float_as_uint(b.w);
        if (q) atomicAdd((unsigned long long *)&adj_tab[(size_t)(meta >> 5) * mb + (meta & 31u)], (unsigned long long)q);
        return q;
    };
    const bool coop = kHits < 64 && load >= coop_min(kHits);
    if (valid && !coop) {
        const double wk = (double)hx.w;
        i128 own = 0;
        auto add = [&](const float4 &a, const float4 &b) { own += term(G, wk, a, b); };
        for (uint32_t m = dc.uniq; m != 0u; m &= m - 1u)
            photons_of_bucket(d, disc_cell_bucket(gr, dc.c0, __builtin_ctz(m)), hx, hn, r2, start, sorted, add);
        if (own != 0) wide_add(&lds.lo[__float_as_uint(hn.w)], &lds.hi[__float_as_uint(hn.w)], own);
    }
    for (uint64_t todo = kHits < 64 ? __ballot(coop) : 0ull; todo != 0ull; todo &= todo - 1ull) {
        const int L = __ffsll((unsigned long long)todo) - 1;
        const double wk = (double)readlane_f(hx.w, L), Gp = readlane_d(G, L);
        i128 own = 0;
        wave_scan(d, gr, L, hx, hn, r2, dc, start, sorted,
                  [&](const float4 &a, const float4 &b) { own += term(Gp, wk, a, b); });
        // the lanes' sums, in the two parts that wide_add adds
        unsigned long long lo = (unsigned long long)(uint32_t)(uint64_t)own, hi = (unsigned long long)(long long)(own >> 32);
        for (int off = 32; off > 0; off >>= 1) {
            lo += __shfl_xor(lo, off);
            hi += __shfl_xor(hi, off);
        }
        if ((int)lane == L && (lo | hi) != 0ull) {
            atomicAdd(&lds.lo[__float_as_uint(hn.w)], lo);
            atomicAdd(&lds.hi[__float_as_uint(hn.w)], hi);
        }
    }
    wide_flush(lds, n_mat, wide);
}

inline auto gather_adj_of(int hits) {
    return hits == 64 ? k_gather_adj<64> : (hits == 16 ? k_gather_adj<16> : k_gather_adj<4>);
}

__global__ __launch_bounds__(kBlock) void k_path_adj(const uint16_t *__restrict__ mat_tab,
                                                     const long long *__restrict__ adj_tab, uint32_t n_paths,
                                                     int32_t max_bounces, int32_t n_mat,
                                                     unsigned long long *__restrict__ wide) {
    __shared__ WideLds lds;
    wide_clear(lds, n_mat);
    uint32_t n = blockIdx.x * kBlock + threadIdx.x;
    if (n < n_paths) {
        const uint16_t *row = mat_tab + (size_t)n * max_bounces;
        const long long *arow = adj_tab + (size_t)n * max_bounces;
        int end = 0;
        while (end < max_bounces && row[end] != kMatEnd) end++;
        i128 S = 0;  // sensitivity of the photons stored after bounce b
        for (int b = end - 1; b >= 0; --b) {
            uint32_t m = row[b];
            if (m == kMatNone) continue;
            if (S != 0) wide_add(&lds.lo[m], &lds.hi[m], S);
            S += arow[b];
        }
    }
    wide_flush(lds, n_mat, wide);
}

// grad_mat[m] += (iteration's integer sum for m) / scale / rho_m, one
// iteration after another (the order of these additions is fixed).
__global__ void k_adj_fold(const unsigned long long *__restrict__ wide, int32_t n_mat,
                           const double *__restrict__ scale_p, const float *__restrict__ mat_rho,
                           double *__restrict__ grad_mat) {
    const double scale = *scale_p;
    for (int m = threadIdx.x; m < n_mat; m += blockDim.x) {
        const unsigned long long lo = wide[m];
        const long long hi = (long long)(wide[n_mat + m] + (lo >> 32));
        if (scale > 0.0 && (hi != 0 || (lo & 0xffffffffull) != 0ull) && mat_rho[m] > 0.0f) {
            const double v = (double)hi * 4294967296.0 + (double)(lo & 0xffffffffull);
            grad_mat[m] += (v / scale) / (double)mat_rho[m];
        }
    }
}

// Per-workgroup partial sums of g_p L_p (every term of L_p is proportional to
// the emitted radiance); k_collect_grad adds them in a fixed order.
__global__ __launch_bounds__(kBlock) void k_le_grad(SppmDev d, double K, const float *__restrict__ g,
                                                    double *__restrict__ part) {
    __shared__ double lds[kBlock / 64];
    int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    double v = 0.0;
    if (p < d.P) v = (double)g[p] * (d.tau[p] / ((kPiD * d.R2[p]) * K) + d.D[p] / K);
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) t += lds[w];
        part[blockIdx.x] = t;
    }
}

__global__ void k_fill_f64(double *p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

struct ParamMats {
    uint8_t m[kMaxAdjMat];
};

// One workgroup of kMaxAdjMat threads: parameter gradients, and the emission
// gradient as a fixed-order sum of the partial sums of g L.
__global__ __launch_bounds__(kMaxAdjMat) void k_collect_grad(const double *__restrict__ grad_mat, ParamMats pm,
                                                             int32_t n_par, const double *__restrict__ le_part,
                                                             int32_t n_part, double inv_Le, double *__restrict__ out) {
    __shared__ double lds[kMaxAdjMat];
    const int i = threadIdx.x;
    double t = 0.0;
    for (int j = i; j < n_part; j += kMaxAdjMat) t += le_part[j];
    lds[i] = t;
    __syncthreads();
    for (int w = kMaxAdjMat / 2; w > 0; w >>= 1) {
        if (i < w) lds[i] += lds[i + w];
        __syncthreads();
    }
    if (i < n_par) out[i] = grad_mat[pm.m[i]];
    if (i == n_par) out[i] = lds[0] * inv_Le;
}

// The form of a kernel that a handle launches.
template <class K>
K *pick(const pm_sppm *s, K *wide, K *binary) {
    return s->wide ? wide : binary;
}

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + kBlock - 1) / kBlock); }
// Workgroups for n elements, per_wave to a wave.
inline uint32_t blocks_for_waves(int64_t n, uint32_t per_wave) {
    return (uint32_t)((n + (int64_t)per_wave * (kBlock / 64) - 1) / ((int64_t)per_wave * (kBlock / 64)));
}

// host float3 helpers with the same evaluation order as the device
struct H3 {
    float x, y, z;
};
inline H3 hsub(H3 a, H3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
inline float hdot(H3 a, H3 b) { return (a.x * b.x + a.y * b.y) + a.z * b.z; }
inline H3 hcross(H3 a, H3 b) { return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x}; }
inline H3 hnorm(H3 v) {
    float l = std::sqrt(hdot(v, v));
    return {v.x / l, v.y / l, v.z / l};
}

}  // namespace

namespace pm {

// Stream sets of released handles, kept for the next ones (at most kPoolSets).
//
// The runtime maps streams onto four hardware queues (its default), a new
// stream onto the queue with the fewest, and streams that share a queue run one
// after another.  The four streams of a set must lie on four queues: with the
// main stream on a photon pass's queue 8 iterations at 1280x720 take 10.5 ms
// instead of 9.0, and the caller's stream in place of the main one shares a
// queue with a photon pass in every third handle (10.9).  While one of the queues
// is already used by the default stream, the fourth stream of a fresh process
// would not get that queue but one of its own set's, so three more streams are
// created first, which even out the queues, and released afterwards.  That costs
// 300 us a set, so sets are kept: a set is used by one handle at a time, and only
// a set with no work and no capture under way is kept.
constexpr int kPoolSets = 4;
static std::mutex g_pool_mu;
static struct {
    int device;
    PassStreams set;
} g_pool[kPoolSets];
static int g_pool_n = 0;

static void destroy_streams(PassStreams &p) {
    for (hipStream_t *q : {&p.pass[0], &p.pass[1], &p.pass[2], &p.main}) {
        if (*q) (void)hipStreamDestroy(*q);
        *q = nullptr;
    }
}

// Whether the streams of a kept set still exist: a device reset ends them.
static bool alive(const PassStreams &p) {
    bool ok = true;
    for (hipStream_t q : {p.pass[0], p.pass[1], p.pass[2], p.main}) {
        const hipError_t e = hipStreamQuery(q);
        ok = ok && (e == hipSuccess || e == hipErrorNotReady);
    }
    (void)hipGetLastError();
    return ok;
}

// A set of streams of the current device.
static hipError_t take_streams(int device, PassStreams &out) {
    {
        std::lock_guard<std::mutex> lock(g_pool_mu);
        for (int i = g_pool_n - 1; i >= 0; --i)
            if (g_pool[i].device == device) {
                out = g_pool[i].set;
                g_pool[i] = g_pool[--g_pool_n];
                if (alive(out)) return hipSuccess;
                out = PassStreams{};
            }
    }
    hipStream_t even[3] = {};
    hipError_t e = hipSuccess;
    for (hipStream_t *q : {&even[0], &even[1], &even[2], &out.pass[0], &out.pass[1], &out.pass[2], &out.main})
        if (e == hipSuccess) e = hipStreamCreateWithFlags(q, hipStreamNonBlocking);
    for (hipStream_t q : even)
        if (q) (void)hipStreamDestroy(q);
    return e;
}

// Called once all work on the set's streams has ended.
static void give_streams(int device, PassStreams &p) {
    bool keep = true;
    for (hipStream_t q : {p.pass[0], p.pass[1], p.pass[2], p.main}) {
        hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
        keep = keep && q && hipStreamIsCapturing(q, &c) == hipSuccess && c == hipStreamCaptureStatusNone;
    }
    if (keep) {
        std::lock_guard<std::mutex> lock(g_pool_mu);
        if (g_pool_n < kPoolSets) {
            g_pool[g_pool_n].device = device;
            g_pool[g_pool_n++].set = p;
            p = PassStreams{};
            return;
        }
    }
    destroy_streams(p);
}

void sppm_free(pm_sppm *s) {
    // kernels of this handle may still be in flight on the caller's stream
    (void)hipDeviceSynchronize();
    if (s->arena) (void)hipFree(s->arena);
    for (hipEvent_t e : s->prof_ev)
        if (e) (void)hipEventDestroy(e);
    for (uint32_t i = 0; i < kRing; ++i)
        for (hipEvent_t e : {s->ev_ph[i], s->ev_scat[i], s->ev_eye[i], s->ev_upd[i]})
            if (e) (void)hipEventDestroy(e);
    give_streams(s->device, s->streams);
    for (hipEvent_t e : {s->ev_fork, s->ev_join})
        if (e) (void)hipEventDestroy(e);
    if (s->own_bvh && s->bvh) {
        free_bvh(s->bvh);
        delete s->bvh;
    }
    delete s;
}

int sppm_validate(const pm_scene_desc *d, const pm_sppm_params *p) {
    if (!d || !p) return set_error("scene and params must not be NULL"), PM_ERR_ARG;
    if (d->size < sizeof(pm_scene_desc) || p->size < sizeof(pm_sppm_params))
        return set_error("struct size field too small"), PM_ERR_ARG;
    if (!d->tri_verts || !d->tri_mat || d->n_tri < 1) return set_error("scene has no triangles"), PM_ERR_ARG;
    if (!d->mat_type || !d->mat_rho || !d->mat_q || !d->mat_Le || !d->mat_ior || d->n_mat < 1)
        return set_error("material arrays missing"), PM_ERR_ARG;
    for (int64_t i = 0; i < d->n_tri; ++i)
        if (d->tri_mat[i] >= (uint32_t)d->n_mat) return set_error("triangle material id out of range"), PM_ERR_ARG;
    for (int32_t m = 0; m < d->n_mat; ++m) {
        int t = d->mat_type[m];
        if (t < 0 || t > 2) return set_error("unknown material type"), PM_ERR_ARG;
        if (!(d->mat_rho[m] >= 0.0f && d->mat_rho[m] < 1.0f)) return set_error("albedo must be in [0,1)"), PM_ERR_ARG;
        if (!(d->mat_q[m] >= 0.0f && d->mat_q[m] <= 1.0f)) return set_error("RR probability must be in [0,1]"), PM_ERR_ARG;
        if (!(d->mat_Le[m] >= 0.0f) || !std::isfinite(d->mat_Le[m])) return set_error("Le must be finite and >= 0"), PM_ERR_ARG;
        if (t == PM_MAT_GLASS && !(d->mat_ior[m] > 0.0f)) return set_error("glass ior must be > 0"), PM_ERR_ARG;
    }
    if (d->width < 1 || d->height < 1 || (int64_t)d->width * d->height > (int64_t(1) << 28))
        return set_error("image size out of range"), PM_ERR_ARG;
    if (!(d->tan_half_fov > 0.0f) || !std::isfinite(d->tan_half_fov)) return set_error("tan_half_fov must be > 0"), PM_ERR_ARG;
    if (p->n_photons < 1 || p->n_photons > (int64_t(1) << 26)) return set_error("n_photons must be in [1, 2^26]"), PM_ERR_ARG;
    if (!(p->alpha > 0.0 && p->alpha <= 1.0)) return set_error("alpha must be in (0,1]"), PM_ERR_ARG;
    if (!(p->r0 > 0.0) || !std::isfinite(p->r0)) return set_error("r0 must be > 0"), PM_ERR_ARG;
    if (p->max_eye_depth < 1 || p->max_eye_depth > 64 || p->max_photon_bounces < 1 || p->max_photon_bounces > 32)
        return set_error("max_eye_depth must be in [1,64] and max_photon_bounces in [1,32]"), PM_ERR_ARG;
    if (p->fixed_shift < 0 || p->fixed_shift > 52) return set_error("fixed_shift must be in [0,52]"), PM_ERR_ARG;
    if (p->store_factor < 1 || p->n_photons * p->store_factor > (int64_t(1) << 30))
        return set_error("store_factor must be >= 1 and the store below 2^30 photons"), PM_ERR_ARG;
    if (d->bvh && d->bvh->n_tri != d->n_tri) return set_error("bvh was built over a different triangle count"), PM_ERR_ARG;
    if (p->photon_kernel < 0 || p->photon_kernel > PM_PHOTON_TWO_PHASE || p->refill < 0 || p->refill > 64)
        return set_error("photon_kernel must be 0..6 and refill 0..64"), PM_ERR_ARG;
    if (p->pass_threads < 0 || p->pass_threads > (1 << 26) || p->passes < 0 || p->passes > 1024)
        return set_error("pass_threads must be in [0, 2^26] and passes in [0, 1024]"), PM_ERR_ARG;
    if (p->photon_kernel != PM_PHOTON_PASSES && (p->pass_threads != 0 || p->passes != 0))
        return set_error("pass_threads and passes apply to photon_kernel PM_PHOTON_PASSES only"), PM_ERR_ARG;
    if (p->gather_mode != PM_GATHER_EXACT && p->gather_mode != PM_GATHER_STOCHASTIC)
        return set_error("gather_mode must be PM_GATHER_EXACT or PM_GATHER_STOCHASTIC"), PM_ERR_ARG;
    if (p->gather_mode == PM_GATHER_STOCHASTIC && p->record_iterations > 0)
        return set_error("the adjoint needs the exact gather (gather_mode 0)"), PM_ERR_ARG;
    if (p->profile < 0 || p->profile > (PM_PROFILE_COUNT | PM_PROFILE_TIME))
        return set_error("profile must be a combination of PM_PROFILE_COUNT and PM_PROFILE_TIME"), PM_ERR_ARG;
    if ((p->profile & PM_PROFILE_COUNT) &&
        (p->gather_mode != PM_GATHER_EXACT || p->photon_kernel == PM_PHOTON_PER_PATH || p->photon_kernel == PM_PHOTON_PASSES))
        return set_error("PM_PROFILE_COUNT counts the regenerating photon kernels and the exact gather"), PM_ERR_ARG;
    if (p->single_link_set < 0 || p->single_link_set > 6)
        return set_error("single_link_set must be 0 (by direction) or 1..6"), PM_ERR_ARG;
    if (p->record_iterations < 0 || p->record_iterations > 100000)
        return set_error("record_iterations must be in [0, 100000]"), PM_ERR_ARG;
    if (p->record_iterations > 0 && d->n_mat > kMaxAdjMat)
        return set_error("the adjoint supports at most 256 materials"), PM_ERR_ARG;
    // a photon's (path, bounce) entry sums at most one term of 2^39 units per pixel
    if (p->record_iterations > 0 && (int64_t)d->width * d->height >= (int64_t(1) << 24))
        return set_error("the adjoint supports images below 2^24 pixels"), PM_ERR_ARG;
    return PM_OK;
}

// A default photon pass of at most this many paths for each wave the device
// holds (4,096) runs in one launch that spreads them evenly over half of the
// waves (k_photon).  It ends with its longest path either way, but the two
// launches of full waves came one after another for every iteration.  Calls, two
// launches and one (ms): 8 iterations of 100,003 paths 3.6 and 3.1, 4 of 2^18
// paths 1.9 either way.  Beyond 64 paths a wave the regenerating launch fills its
// lanes better.
constexpr uint32_t kThinPaths = 64;

// The photon passes of a pipelined handle do not take the whole device: a wave
// of theirs keeps its slot (and its LDS) for most of a pass, and two passes, an
// eye pass and a range query are under way at once.  With all slots taken the
// eye pass, whose waves mostly wait, became the longest stage: 1.9 ms instead of
// 0.4.  1280x720, 2^20 photons, ms an iteration in calls of 8: all waves for
// either launch 1.20, half for the first and a quarter for the second 1.09 (3/4
// and 1/4 1.10, 3/8 and 1/4 1.10, 1/2 and 1/8 1.19).  The shares are the handle's,
// whatever its calls: with nothing beside it a pass would rather have the device.
// Calls of 1, 4 and 8 with half and a quarter, and with all and a half: 1.83,
// 1.16, 1.08 and 1.72, 1.18, 1.09; 400,000 photons 1.19, 0.76, 0.69 and 1.23,
// 0.80, 0.71; 1920x1080 with 2^22 5.57, 3.70, 3.53 and 4.74, 3.74, 3.49; 320x180
// with 2^20 1.58, 1.02, 0.89 and 1.38, 0.91, 0.90.
// With the binary walk, whose passes are bound by waiting and gain from more
// waves, all and a half: 1.79 in calls of 8 and 2.67 of 1; all and all 1.96 and
// 2.66, half and a quarter 1.91 and 3.09.
struct Shares {
    uint32_t head, tail;
};
static Shares shares_of(const pm_sppm *s) { return s->wide ? Shares{2, 4} : Shares{1, 2}; }

// The photon schedule a handle runs: the default is the two-phase pass on
// single-scene handles and regeneration for a batch member (whose photon
// stage the batch schedules).
static int32_t photon_kernel_of(const pm_sppm_params *p, bool own_grid) {
    if (p->photon_kernel != PM_PHOTON_AUTO) return p->photon_kernel;
    return own_grid ? PM_PHOTON_TWO_PHASE : PM_PHOTON_REGEN;
}

// The buffers of a handle lie in one allocation, each on a 256-byte boundary.
// Some 30 allocations and releases, up to 268 MB each, took 0.9 ms of a
// thumbnail render (333x187, 100,003 photons; create 0.82 -> 0.28 ms, release
// 0.78 -> 0.38) and 4.6 ms of the release of a recording handle at 1280x720
// with 2^20 photons (5.07 -> 0.47 ms).
class Arena {
  public:
    template <class T>
    void add(T *&ptr, size_t bytes) {
        parts_.push_back({&ptr, size_, [](void *at, char *mem) { *static_cast<T **>(at) = reinterpret_cast<T *>(mem); }});
        size_ += (bytes + 255) & ~(size_t)255;
    }
    hipError_t allocate(void **mem) {
        const hipError_t e = hipMalloc(mem, size_);
        if (e != hipSuccess) return *mem = nullptr, e;
        for (const Part &p : parts_) p.set(p.at, (char *)*mem + p.offset);
        return e;
    }

  private:
    struct Part {
        void *at;
        size_t offset;
        void (*set)(void *, char *);
    };
    std::vector<Part> parts_;
    size_t size_ = 0;
};

// 64-bit fingerprint of everything in a scene description that the render reads
// (FNV-1a over 32-bit words).  The triangles' words are one serial chain of
// multiplications, 8.4 us for 1,000 triangles on the host.  From kHashThread
// triangles on a thread runs it beside the creation of the handle (0.3 ms without
// it); from kDeviceHash on the device does, in less time than the chain takes
// there: creating the handle of 250,000 triangles went from 2.16 ms (with the
// thread) to 0.8, while for 13,600 the device takes longer (0.41 ms instead of
// 0.25).  Where the device has no room for the words the host does it.  The
// description is not read after finish().
class SceneFingerprint {
  public:
    static constexpr int64_t kHashThread = 8192, kDeviceHash = 1 << 15;
    ~SceneFingerprint() {
        if (thread_.joinable()) thread_.join();
    }
    int launch(const pm_scene_desc *d, hipStream_t st) {
        d_ = d;
        add(&d->n_tri, sizeof(d->n_tri));
        const size_t nt = (size_t)d->n_tri;
        device_ = d->n_tri >= kDeviceHash && d->n_tri < (int64_t(1) << 28);
        if (device_) {
            const int rc = hash_.launch(h_, d->tri_verts, 9 * nt, d->tri_mat, nt, st);
            if (rc != PM_ERR_NOMEM) return rc;
            (void)hipGetLastError();
            device_ = false;
        }
        if (d->n_tri >= kHashThread) try {
                thread_ = std::thread([this] { triangles(); });
            } catch (const std::system_error &) {  // no thread to be had: finish() does it
            }
        return PM_OK;
    }
    // Ends the device's part and gives its memory back; false: there was none.
    bool settle(hipStream_t st, int &rc) {
        if (!device_) return false;
        rc = hash_.finish(h_, st);
        hash_.release();
        device_ = false;
        settled_ = true;
        return true;
    }
    int finish(uint64_t &out, hipStream_t st) {
        int rc = PM_OK;
        if (settle(st, rc)) {
            if (rc) return rc;
        } else if (thread_.joinable()) {
            thread_.join();
        } else if (!settled_) {
            triangles();
        }
        const size_t nm = (size_t)d_->n_mat;
        add(&d_->n_mat, sizeof(d_->n_mat));
        add(d_->mat_type, sizeof(int32_t) * nm);
        add(d_->mat_rho, sizeof(float) * nm);
        add(d_->mat_q, sizeof(float) * nm);
        add(d_->mat_Le, sizeof(float) * nm);
        add(d_->mat_ior, sizeof(float) * nm);
        add(d_->cam_pos, sizeof(d_->cam_pos));
        add(d_->cam_look, sizeof(d_->cam_look));
        add(d_->cam_up, sizeof(d_->cam_up));
        add(&d_->tan_half_fov, sizeof(d_->tan_half_fov));
        add(&d_->width, sizeof(d_->width));
        add(&d_->height, sizeof(d_->height));
        out = h_;
        return PM_OK;
    }

  private:
    void triangles() {
        add(d_->tri_verts, sizeof(float) * 9 * (size_t)d_->n_tri);
        add(d_->tri_mat, sizeof(uint32_t) * (size_t)d_->n_tri);
    }
    void add(const void *p, size_t bytes) {  // whole words
        const uint8_t *b = (const uint8_t *)p;
        for (size_t i = 0; i + 4 <= bytes; i += 4) {
            uint32_t w;
            memcpy(&w, b + i, 4);
            h_ = (h_ ^ w) * kHashPrime;
        }
    }
    const pm_scene_desc *d_ = nullptr;
    uint64_t h_ = 0xcbf29ce484222325ull;
    bool device_ = false, settled_ = false;
    DeviceHash hash_;
    std::thread thread_;
};

int sppm_create_ex(const pm_scene_desc *d, const pm_sppm_params *p, hipStream_t st, bool own_grid, pm_sppm **out) {
    int rc = sppm_validate(d, p);
    if (rc) return rc;
    SceneFingerprint fingerprint;
    if ((rc = fingerprint.launch(d, st))) return rc;
    pm_sppm *s = new pm_sppm();
    s->prm = *p;
    auto fail = [&](int code) {
        sppm_free(s);
        return code;
    };
#define PM_HIPF(call)                                            \
    do {                                                         \
        hipError_t e_ = (call);                                  \
        if (e_ != hipSuccess) return fail(hip_fail(e_, #call));  \
    } while (0)
    if (d->bvh) {
        s->bvh = const_cast<pm_bvh *>(d->bvh);
    } else {
        HostBvh hb;
        std::string err;
        BuildOptions bo;
        if (!build_bvh_host(d->tri_verts, d->tri_mat, d->n_tri, bo, hb, err)) {
            set_error(err);
            return fail(PM_ERR_ARG);
        }
        s->bvh = new pm_bvh();
        s->own_bvh = true;
        if ((rc = upload_bvh(hb, st, s->bvh))) return fail(rc);
    }
    const pm_bvh *b = s->bvh;
    s->wide = b->d_wide != nullptr && p->single_link_set == 0;
    s->P = (int64_t)d->width * d->height;
    // emitters in original triangle order, by power = area * Le
    std::vector<uint32_t> epos;
    std::vector<double> ecdf;
    double acc = 0.0;
    for (int64_t i = 0; i < d->n_tri; ++i) {
        float Le = d->mat_Le[d->tri_mat[i]];
        if (!(Le > 0.0f)) continue;
        const float *v = d->tri_verts + 9 * i;
        H3 v0{v[0], v[1], v[2]}, v1{v[3], v[4], v[5]}, v2{v[6], v[7], v[8]};
        H3 c = hcross(hsub(v1, v0), hsub(v2, v0));
        float area = 0.5f * std::sqrt(hdot(c, c));
        acc += (double)area * (double)Le;
        epos.push_back((uint32_t)b->pos_of[i]);
        ecdf.push_back(acc);
    }
    H3 ext{b->hi[0] - b->lo[0], b->hi[1] - b->lo[1], b->hi[2] - b->lo[2]};
    float diag = std::sqrt(hdot(ext, ext));
    s->phi0 = (float)((kPiD * acc) / (double)p->n_photons);
    int64_t cap64 = p->n_photons * p->store_factor;
    s->cap = (uint32_t)cap64;
    uint32_t bits = 12;
    while (bits < 24 && (int64_t(1) << bits) < 4 * p->n_photons) bits++;
    s->table_bits = bits;
    const uint32_t T = 1u << bits;
    const uint32_t nb = T / kScanTile;
    const int32_t nm = d->n_mat;

    {
        int dev = 0, cus = 0, per_cu = 0;
        PM_HIPF(hipGetDevice(&dev));
        s->device = dev;
        PM_HIPF(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        const std::pair<uint32_t *, const void *> grids[] = {
            {&s->regen_grid, (const void *)pick(s, k_photon_regen<true>, k_photon_regen<false>)},
            {&s->regen_grid_rec, (const void *)pick(s, k_photon_regen_rec<true>, k_photon_regen_rec<false>)},
            {&s->stream_grid, (const void *)k_photon_stream},
            {&s->pool_grid, (const void *)k_photon_pool<false>},
            {&s->head_grid, (const void *)pick(s, k_photon_head<false, true>, k_photon_head<false, false>)},
            {&s->tail_grid, (const void *)pick(s, k_photon_tail<false, true>, k_photon_tail<false, false>)},
            {&s->head_grid_rec, (const void *)pick(s, k_photon_head_rec<true>, k_photon_head_rec<false>)},
            {&s->tail_grid_rec, (const void *)pick(s, k_photon_tail_rec<true>, k_photon_tail_rec<false>)}};
        for (const auto &g : grids) {
            PM_HIPF(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, g.second, kBlock, 0));
            *g.first = (uint32_t)std::max(1, cus * std::max(1, per_cu));
        }
    }
    const int32_t photon_kernel = photon_kernel_of(p, own_grid);
    const bool pipelined = own_grid && !(p->profile & PM_PROFILE_TIME);
    {
        const int64_t waves = (int64_t)s->head_grid * (kBlock / 64), np = p->n_photons;
        if (own_grid && p->photon_kernel == PM_PHOTON_AUTO && !(p->profile & PM_PROFILE_COUNT) &&
            np <= waves * kThinPaths)
            s->thin = (uint32_t)std::min<int64_t>(std::max<int64_t>((2 * np + waves - 1) / waves, kMinPathsPerWave),
                                                  kThinPaths);
        const Shares part = pipelined ? shares_of(s) : Shares{1, 1};
        for (uint32_t *head : {&s->head_grid, &s->head_grid_rec}) *head = std::max(1u, *head / part.head);
        for (uint32_t *tail : {&s->tail_grid, &s->tail_grid_rec}) *tail = std::max(1u, *tail / part.tail);
    }
    // a stream per slot (two where the photon passes share one): see photon_queue
    const uint32_t slots = !pipelined ? 1u : (photon_kernel == PM_PHOTON_TWO_PHASE ? kRing : 2u);
    if (own_grid) {
        for (uint32_t i = 0; i < std::max(slots, 2u); ++i) {
            for (hipEvent_t *e : {&s->ev_ph[i], &s->ev_scat[i], &s->ev_eye[i], &s->ev_upd[i]})
                PM_HIPF(hipEventCreateWithFlags(e, hipEventDisableTiming));
        }
        PM_HIPF(take_streams(s->device, s->streams));
        PM_HIPF(hipEventCreateWithFlags(&s->ev_fork, hipEventDisableTiming));
        PM_HIPF(hipEventCreateWithFlags(&s->ev_join, hipEventDisableTiming));
    }
    // one slot per thread of a pass; the paper runs one thread per pixel
    const uint32_t pass_slots = p->pass_threads > 0 ? (uint32_t)p->pass_threads
                                                    : (uint32_t)std::min<int64_t>(s->P, int64_t(1) << 26);
    // two-phase pass, per slot: a queue slot for every lane of the first
    // launch (each parks at most one path), then the queue's count
    const uint32_t queue_slots =
        (uint32_t)std::min<int64_t>(p->n_photons, (int64_t)std::max(s->head_grid, s->head_grid_rec) * kBlock);
    const size_t queue_bytes = (size_t)56 * queue_slots + 256;
    s->rec_iters = p->record_iterations;
    // a handle that does not fit with all slots makes do with fewer (one: an iteration at a time)
    s->ring = slots;
    for (;;) {
        Arena arena;
        arena.add(s->mat_type, sizeof(int32_t) * nm);
        arena.add(s->mat_f, sizeof(float) * 4 * nm);
        arena.add(s->emit_pos, sizeof(uint32_t) * std::max<size_t>(1, epos.size()));
        arena.add(s->emit_cdf, sizeof(double) * std::max<size_t>(1, ecdf.size()));
        arena.add(s->N, sizeof(double) * s->P);
        arena.add(s->R2, sizeof(double) * s->P);
        arena.add(s->tau, sizeof(double) * s->P);
        arena.add(s->D, sizeof(double) * s->P);
        for (uint32_t i = 0; i < s->ring; ++i) {
            arena.add(s->hp_pos[i], sizeof(float4) * s->P);
            arena.add(s->hp_nrm[i], sizeof(float4) * s->P);
            arena.add(s->emit[i], sizeof(double) * s->P);
            arena.add(s->store[i], sizeof(float4) * 2 * (size_t)cap64);
        }
        arena.add(s->counters, sizeof(uint32_t) * 4 * kRing);
        arena.add(s->r2max, sizeof(unsigned long long) * kRing);
        if (own_grid) {
            arena.add(s->cell_count, sizeof(uint32_t) * T);
            if (p->gather_mode == PM_GATHER_STOCHASTIC) {
                arena.add(s->sh_key, sizeof(unsigned long long) * T);
                arena.add(s->sh_surv, sizeof(uint32_t) * T);
            } else {
                arena.add(s->sorted, sizeof(float4) * 2 * (size_t)cap64);
                arena.add(s->cell_start, sizeof(uint32_t) * (T + 1));
                arena.add(s->cell_fill, sizeof(uint32_t) * T);
                arena.add(s->bsum, sizeof(uint32_t) * (nb + 1));
            }
        }
        arena.add(s->M, sizeof(uint32_t) * s->P);
        arena.add(s->Phi, sizeof(unsigned long long) * s->P);
        if (p->gather_mode == PM_GATHER_EXACT) arena.add(s->key_rank, sizeof(uint2) * (size_t)cap64);
        if (p->photon_kernel == PM_PHOTON_PASSES) arena.add(s->slot_mem, (size_t)56 * pass_slots);
        if (photon_kernel == PM_PHOTON_TWO_PHASE) arena.add(s->queue_mem, s->ring * queue_bytes);
        if (p->profile & PM_PROFILE_COUNT) arena.add(s->stats, sizeof(unsigned long long) * kStatCount);
        if (s->rec_iters > 0) {
            arena.add(s->R2_hist, sizeof(double) * (size_t)s->rec_iters * s->P);
            for (uint32_t i = 0; i < s->ring; ++i) {  // the adjoint overlaps iterations like the forward
                arena.add(s->adj_tab[i], sizeof(long long) * (size_t)p->n_photons * p->max_photon_bounces);
                arena.add(s->mat_tab[i], sizeof(uint16_t) * (size_t)p->n_photons * p->max_photon_bounces);
            }
            arena.add(s->grad_mat, sizeof(double) * (nm + 1));
            arena.add(s->adj_wide, sizeof(unsigned long long) * 2 * nm);
            arena.add(s->adj_max, sizeof(unsigned long long) * 2 * kRing);
            arena.add(s->adj_scale, sizeof(double));
            arena.add(s->le_part, sizeof(double) * blocks_for(s->P));
        }
        const hipError_t e = arena.allocate(&s->arena);
        if (e == hipSuccess) break;
        // first without the fingerprint's buffer beside it
        if (e == hipErrorOutOfMemory && fingerprint.settle(st, rc)) {
            if (rc) return fail(rc);
        } else if (s->ring == 1u || e != hipErrorOutOfMemory) {
            return fail(hip_fail(e, "hipMalloc"));
        } else {
            s->ring--;
        }
        (void)hipGetLastError();
    }

    if (p->photon_kernel == PM_PHOTON_PASSES) {
        const uint32_t S = pass_slots;
        char *m = (char *)s->slot_mem;
        s->slots.g = (int4 *)m;
        s->slots.o = (float4 *)(m + (size_t)16 * S);
        s->slots.w = (float4 *)(m + (size_t)32 * S);
        s->slots.nb = (uint2 *)(m + (size_t)48 * S);
        s->slots.S = S;
        const int64_t auto_pass = (p->n_photons + S - 1) / S + 8;
        s->n_pass = p->passes > 0 ? p->passes : (int32_t)std::min<int64_t>(auto_pass, 1024);
    }
    if (photon_kernel == PM_PHOTON_TWO_PHASE) {
        const uint32_t S = queue_slots;
        for (uint32_t i = 0; i < s->ring; ++i) {
            char *m = (char *)s->queue_mem + i * queue_bytes;
            PathQueue &q = s->queue[i];
            q.s.g = (int4 *)m;
            q.s.o = (float4 *)(m + (size_t)16 * S);
            q.s.w = (float4 *)(m + (size_t)32 * S);
            q.s.nb = (uint2 *)(m + (size_t)48 * S);
            q.s.S = S;
            q.cnt = (uint32_t *)(m + (size_t)56 * S);
        }
    }
    if (p->profile & PM_PROFILE_COUNT) {
        PM_HIPF(hipMemsetAsync(s->stats, 0, sizeof(unsigned long long) * kStatCount, st));
    }
    if (p->profile & PM_PROFILE_TIME)
        for (hipEvent_t &e : s->prof_ev) PM_HIPF(hipEventCreate(&e));
    s->n_mat = nm;
    s->rho_host.assign(d->mat_rho, d->mat_rho + nm);
    {
        int n_emit_mat = 0;
        double le = 0.0;
        for (int32_t m = 0; m < nm; ++m)
            if (d->mat_Le[m] > 0.0f) {
                n_emit_mat++;
                le = d->mat_Le[m];
            }
        s->le_single = n_emit_mat == 1 ? le : 0.0;
    }

    std::vector<float> mf(4 * (size_t)nm);
    for (int32_t m = 0; m < nm; ++m) {
        mf[m] = d->mat_rho[m];
        mf[nm + m] = d->mat_q[m];
        mf[2 * nm + m] = d->mat_Le[m];
        mf[3 * nm + m] = d->mat_ior[m];
    }
    PM_HIPF(hipMemcpyAsync(s->mat_type, d->mat_type, sizeof(int32_t) * nm, hipMemcpyHostToDevice, st));
    PM_HIPF(hipMemcpyAsync(s->mat_f, mf.data(), sizeof(float) * 4 * nm, hipMemcpyHostToDevice, st));
    if (!epos.empty()) {
        PM_HIPF(hipMemcpyAsync(s->emit_pos, epos.data(), sizeof(uint32_t) * epos.size(), hipMemcpyHostToDevice, st));
        PM_HIPF(hipMemcpyAsync(s->emit_cdf, ecdf.data(), sizeof(double) * ecdf.size(), hipMemcpyHostToDevice, st));
    }
    PM_HIPF(hipMemsetAsync(s->counters, 0, sizeof(uint32_t) * 4 * kRing, st));
    for (uint32_t i = 0; i < s->ring; ++i) PM_HIPF(hipMemsetAsync(s->hp_nrm[i], 0xff, sizeof(float4) * s->P, st));
    PM_HIPF(hipMemsetAsync(s->M, 0, sizeof(uint32_t) * s->P, st));
    PM_HIPF(hipMemsetAsync(s->Phi, 0, sizeof(unsigned long long) * s->P, st));
    PM_HIPF(hipMemsetAsync(s->r2max, 0, sizeof(unsigned long long) * kRing, st));

    SceneDev &sc = s->dev.sc;
    sc.bvh = make_device_bvh(b);
    sc.mat_type = s->mat_type;
    sc.mat_rho = s->mat_f;
    sc.mat_q = s->mat_f + nm;
    sc.mat_Le = s->mat_f + 2 * nm;
    sc.mat_ior = s->mat_f + 3 * nm;
    sc.emit_pos = s->emit_pos;
    sc.emit_cdf = s->emit_cdf;
    sc.n_emit = (int32_t)epos.size();
    sc.power = acc;
    sc.eps = 1e-5f * diag;
    for (int a = 0; a < 3; ++a) sc.lo[a] = b->lo[a];
    sc.ext = std::max(b->hi[0] - b->lo[0], std::max(b->hi[1] - b->lo[1], b->hi[2] - b->lo[2]));
    H3 pos{d->cam_pos[0], d->cam_pos[1], d->cam_pos[2]};
    H3 look{d->cam_look[0], d->cam_look[1], d->cam_look[2]};
    H3 up{d->cam_up[0], d->cam_up[1], d->cam_up[2]};
    H3 f = hnorm(hsub(look, pos));
    H3 r = hnorm(hcross(f, up));
    H3 u = hcross(r, f);
    sc.cpos = V3{pos.x, pos.y, pos.z};
    sc.cf = V3{f.x, f.y, f.z};
    sc.cr = V3{r.x, r.y, r.z};
    sc.cu = V3{u.x, u.y, u.z};
    sc.tanh_fov = d->tan_half_fov;
    sc.aspect = (float)d->width / (float)d->height;
    sc.W = d->width;
    sc.H = d->height;
    SppmDev &dv = s->dev;
    dv.seed = p->seed;
    dv.max_depth = p->max_eye_depth;
    dv.max_bounces = p->max_photon_bounces;
    dv.n_paths = (uint32_t)p->n_photons;
    dv.cap = s->cap;
    dv.phi0 = s->phi0;
    dv.alpha = p->alpha;
    dv.scale = std::ldexp(1.0, p->fixed_shift);
    dv.inv_scale = std::ldexp(1.0, -p->fixed_shift);
    dv.P = s->P;
    dv.mask = T - 1u;
    dv.table_off = 0;
    dv.photon_kernel = photon_kernel;
    // default schedule: 8.71 ms with 16, 8.87 with 32, 9.73 with 44 for 8 iterations at 1280x720 with 2^20 photons
    dv.refill = p->refill > 0 ? (uint32_t)p->refill : (p->photon_kernel == PM_PHOTON_AUTO ? 16u : 32u);
    dv.force_set = p->single_link_set - 1;
    // Binary walks only (one link set, ray regeneration, the pool, a BVH without
    // four-child nodes): paired node requests pay off on one large scene (2.65 ->
    // 2.55 ms an iteration of the 250k-triangle scene when all passes took that
    // walk) but not on the many small scenes of a batch, whose BVHs stay in cache
    // (24.5 -> 25.3 ms).
    dv.paired_walk = own_grid ? 1 : 0;
    dv.gather_mode = p->gather_mode;
    dv.sh_key = s->sh_key;
    dv.sh_surv = s->sh_surv;
    dv.hp_pos = s->hp_pos[0];
    dv.hp_nrm = s->hp_nrm[0];
    dv.emit = s->emit[0];
    dv.N = s->N;
    dv.R2 = s->R2;
    dv.tau = s->tau;
    dv.D = s->D;
    dv.store = s->store[0];
    dv.key_rank = s->key_rank;
    dv.counters = s->counters;
    dv.r2max = s->r2max;
    dv.M = s->M;
    dv.Phi = s->Phi;
    dv.stats = s->stats;
    hipLaunchKernelGGL(k_init_state, dim3(blocks_for(s->P)), dim3(kBlock), 0, st, dv, p->r0 * p->r0);
    PM_HIPF(hipGetLastError());
    if ((rc = fingerprint.finish(s->scene_hash, st))) return fail(rc);
    // host staging vectors go out of scope: finish the copies first
    PM_HIPF(hipStreamSynchronize(st));
#undef PM_HIPF
    *out = s;
    return PM_OK;
}

int sppm_create(const pm_scene_desc *d, const pm_sppm_params *p, hipStream_t st, pm_sppm **out) {
    return sppm_create_ex(d, p, st, true, out);
}

int sppm_destroy(pm_sppm *s) {
    if (!s) return set_error("NULL handle"), PM_ERR_ARG;
    sppm_free(s);
    return PM_OK;
}

int sppm_reset(pm_sppm *s, hipStream_t st) {
    hipLaunchKernelGGL(k_init_state, dim3(blocks_for(s->P)), dim3(kBlock), 0, st, s->dev, s->prm.r0 * s->prm.r0);
    PM_HIP(hipGetLastError());
    s->K = 0;
    return PM_OK;
}

// Device view of iteration k: its slot's photon store (with its block of four
// counters), hit points, seen emission and R_max.
static SppmDev iteration_view(const pm_sppm *s, uint32_t k) {
    SppmDev dk = s->dev;
    const uint32_t i = k % s->ring;
    dk.store = s->store[i];
    dk.counters = s->counters + 4 * i;
    dk.r2max = s->r2max + i;
    dk.hp_pos = s->hp_pos[i];
    dk.hp_nrm = s->hp_nrm[i];
    dk.emit = s->emit[i];
    return dk;
}

// The streams of iteration k's photon and eye pass beside the main stream.  A
// pipelined handle's iterations take them in turn, the eye pass of k on the one
// that the photon pass of k + 1 takes after it: every stream then has the same
// work, and a photon pass, whose last paths run long, overlaps the next two.
// (With one stream for all eye passes and two for the photon passes the eye
// passes' stream was the slowest.  The eye pass of k on the stream of k + 2: 0
// to 3% faster or slower in calls of 8 iterations, 11% slower in 4 of the
// stochastic gather at 640x360.)  Photon kernels whose passes share a workspace
// run them on one stream.
static hipStream_t photon_queue(const pm_sppm *s, uint32_t k) {
    return s->streams.pass[s->dev.photon_kernel == PM_PHOTON_TWO_PHASE ? k % s->ring : 0u];
}
static hipStream_t eye_queue(const pm_sppm *s, uint32_t k) {
    return s->streams.pass[s->dev.photon_kernel == PM_PHOTON_TWO_PHASE && s->ring > 1 ? (k + 1u) % s->ring : 1u];
}
// The stream of a pipelined call's grids, range queries and updates: the main
// stream, or the caller's where the call is being recorded into a graph.  The
// runtime keeps the streams of a recording in a tree below the one that began
// it and walks that tree at the end: main and a pass stream, each waiting for the
// other, would be each other's parent and the walk endless.
static hipStream_t work_stream(const pm_sppm *s, hipStream_t caller) {
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (caller && hipStreamIsCapturing(caller, &c) == hipSuccess && c != hipStreamCaptureStatusNone) return caller;
    return s->streams.main;
}

// The streams that a call has forked from its caller's so far.
struct Forked {
    hipStream_t q[kRing + 1];
    int n = 0;
};

// Forks the work stream and those that the first iterations from k0 on use from
// the caller's stream; a stream without work stays out of it (in a recording it
// could not be joined).
static hipError_t fork_streams(pm_sppm *s, uint32_t k0, uint32_t n_iter, hipStream_t work, hipStream_t st,
                               Forked &forked) {
    hipError_t e = hipEventRecord(s->ev_fork, st);
    for (hipStream_t q : {work, s->streams.pass[0], s->streams.pass[1], s->streams.pass[2]}) {
        bool used = q == work && q != st;
        for (uint32_t k = k0; k < k0 + std::min(n_iter, kRing); ++k)
            used = used || q == photon_queue(s, k) || q == eye_queue(s, k);
        if (!used || e != hipSuccess) continue;
        e = hipStreamWaitEvent(q, s->ev_fork, 0);
        if (e == hipSuccess) forked.q[forked.n++] = q;
    }
    return e;
}
// The work stream has waited for the others.
static hipError_t join_streams(pm_sppm *s, hipStream_t work, hipStream_t st) {
    if (work == st) return hipSuccess;
    hipError_t e = hipEventRecord(s->ev_join, work);
    return e == hipSuccess ? hipStreamWaitEvent(st, s->ev_join, 0) : e;
}
// A call that failed on the way: what it has enqueued still ends before
// anything that the caller enqueues later, and a recording has no loose ends.
static void join_after_error(pm_sppm *s, const Forked &forked, hipStream_t st) {
    for (int i = 0; i < forked.n; ++i)
        if (hipEventRecord(s->ev_join, forked.q[i]) == hipSuccess) (void)hipStreamWaitEvent(st, s->ev_join, 0);
}

// The photon pass of iteration k (its counters cleared first) on stream q.
static int enqueue_photon(pm_sppm *s, const SppmDev &dk, uint32_t k, bool count, hipStream_t q) {
    const uint32_t np = (uint32_t)s->prm.n_photons;
    hipLaunchKernelGGL(k_photon_begin, dim3(1), dim3(64), 0, q, dk, s->thin ? np : 0u);
    if (s->thin) {
        hipLaunchKernelGGL(pick(s, k_photon<false, true>, k_photon<false, false>), dim3(blocks_for_waves(np, s->thin)), dim3(kBlock), 0, q, dk, k, s->thin,
                           (uint16_t *)nullptr, (long long *)nullptr);
        PM_HIP(hipGetLastError());
        return PM_OK;
    }
    if (dk.photon_kernel == PM_PHOTON_TWO_PHASE) {
        const PathQueue &pq = s->queue[k % s->ring];
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, q, pq.cnt, 1u, 0u);
        if (count)
            hipLaunchKernelGGL((k_photon_head<true, false>), dim3(s->head_grid), dim3(kBlock), 0, q, dk, k, pq);
        else
            hipLaunchKernelGGL(pick(s, k_photon_head<false, true>, k_photon_head<false, false>), dim3(s->head_grid), dim3(kBlock), 0, q, dk, k, pq);
        if (count)
            hipLaunchKernelGGL((k_photon_tail<true, false>), dim3(s->tail_grid), dim3(kBlock), 0, q, dk, pq);
        else
            hipLaunchKernelGGL(pick(s, k_photon_tail<false, true>, k_photon_tail<false, false>), dim3(s->tail_grid), dim3(kBlock), 0, q, dk, pq);
    } else if (dk.photon_kernel == PM_PHOTON_RAY_REGEN) {
        if (count)
            hipLaunchKernelGGL(k_photon_stream_stats, dim3(s->stream_grid), dim3(kBlock), 0, q, dk, k);
        else
            hipLaunchKernelGGL(k_photon_stream, dim3(s->stream_grid), dim3(kBlock), 0, q, dk, k);
    } else if (dk.photon_kernel == PM_PHOTON_POOL) {
        if (count)
            hipLaunchKernelGGL(k_photon_pool<true>, dim3(s->pool_grid), dim3(kBlock), 0, q, dk, k);
        else
            hipLaunchKernelGGL(k_photon_pool<false>, dim3(s->pool_grid), dim3(kBlock), 0, q, dk, k);
    } else if (dk.photon_kernel == PM_PHOTON_REGEN) {
        if (count)
            hipLaunchKernelGGL(k_photon_regen_stats, dim3(s->regen_grid), dim3(kBlock), 0, q, dk, k);
        else
            hipLaunchKernelGGL(pick(s, k_photon_regen<true>, k_photon_regen<false>), dim3(s->regen_grid), dim3(kBlock), 0, q, dk, k);
    } else if (dk.photon_kernel == PM_PHOTON_PASSES) {
        const PassSlots &ps = s->slots;
        hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(2 * (int64_t)ps.S)), dim3(kBlock), 0, q, (uint32_t *)ps.nb,
                           2u * ps.S, kSlotIdle);
        for (int32_t j = 0; j < s->n_pass; ++j)
            hipLaunchKernelGGL(pick(s, k_photon_pass<true>, k_photon_pass<false>), dim3(blocks_for(ps.S)), dim3(kBlock), 0, q, dk, k, ps);
        hipLaunchKernelGGL(k_pass_tally, dim3(1), dim3(64), 0, q, dk);
        hipLaunchKernelGGL(pick(s, k_photon_drain<true>, k_photon_drain<false>), dim3(blocks_for(ps.S)), dim3(kBlock), 0, q, dk, k, ps);
    } else {
        hipLaunchKernelGGL(pick(s, k_photon<false, true>, k_photon<false, false>), dim3(blocks_for(np)), dim3(kBlock), 0, q, dk, k, 64u, (uint16_t *)nullptr,
                           (long long *)nullptr);
    }
    PM_HIP(hipGetLastError());
    return PM_OK;
}

// One call runs n_iter iterations.  Per iteration k: the eye pass and R_max,
// the photon pass, then the hashed grid, the range query and the update.  A
// pipelined handle has the last three on its main stream and the eye and photon
// passes of its iterations on three more (see photon_queue): they need nothing
// of the iterations before except a free slot, so up to `ring` of them overlap
// the grid, range query and update of k and each other, and the device stays
// full while the last paths of a pass run.  Events order the rest: the photon
// pass of k waits for the last reader of its slot's store (the scatter of
// k - ring, or its stochastic gather), the eye pass for the update of k - ring
// (it overwrites the hit points that k - ring read), and the grid of k for the
// eye pass and photon pass of k.  With two slots, and the second launches of all
// passes on one stream, the next pass waited out a whole photon pass: 8
// iterations at 1280x720 with 2^20 photons went from 10.6 to 8.8 ms, 4 of the
// stochastic gather at 640x360 with 2^18 from 2.2 to 1.8, with the shares of the
// device at shares_of.  At the end of the call the caller's stream has waited
// for every stream.  Results are those of the serial order.
static int run_iterations(pm_sppm *s, int32_t n_iter, hipStream_t caller, Forked &forked) {
    const uint32_t T = 1u << s->table_bits;
    const uint32_t ph_blocks = std::min<uint32_t>(blocks_for(s->cap), 256u * 64u);
    const bool count = (s->prm.profile & PM_PROFILE_COUNT) != 0, timed = (s->prm.profile & PM_PROFILE_TIME) != 0;
    const bool pipe = s->ring > 1;
    hipEvent_t *ev = s->prof_ev;
    const uint32_t k0 = (uint32_t)s->K;
    int rc;
    auto eye_pass = [&](const SppmDev &dv, uint32_t kk, hipStream_t q) {
        if (count)
            hipLaunchKernelGGL(k_eye_stats, dim3(blocks_for(s->P)), dim3(kBlock), 0, q, dv, kk, 1);
        else
            hipLaunchKernelGGL(pick(s, k_eye<true>, k_eye<false>), dim3(blocks_for(s->P)), dim3(kBlock), 0, q, dv, kk,
                               1);
    };
    // photon and eye pass of iteration k, once their slot's readers of ring
    // iterations ago (the first `ring` of a call follow all earlier work) are done
    auto ahead = [&](uint32_t kk) -> int {
        const uint32_t i = kk % s->ring;
        hipStream_t q = photon_queue(s, kk), eq = eye_queue(s, kk);
        if (kk >= k0 + s->ring) {
            PM_HIP(hipStreamWaitEvent(q, s->ev_scat[i], 0));
            PM_HIP(hipStreamWaitEvent(eq, s->ev_upd[i], 0));
        }
        if (int e = enqueue_photon(s, iteration_view(s, kk), kk, count, q)) return e;
        PM_HIP(hipEventRecord(s->ev_ph[i], q));
        eye_pass(iteration_view(s, kk), kk, eq);
        PM_HIP(hipEventRecord(s->ev_eye[i], eq));
        return PM_OK;
    };
    uint32_t sent = k0;  // iterations whose photon and eye passes are enqueued
    hipStream_t st = pipe ? work_stream(s, caller) : caller;
    if (pipe) PM_HIP(fork_streams(s, k0, (uint32_t)n_iter, st, caller, forked));
    for (int32_t it = 0; it < n_iter; ++it) {
        const uint32_t k = k0 + (uint32_t)it;
        const SppmDev dk = iteration_view(s, k);
        for (; pipe && sent < k0 + (uint32_t)n_iter && sent < k + s->ring; ++sent)
            if ((rc = ahead(sent))) return rc;
        if (timed) PM_HIP(hipEventRecord(ev[0], st));
        if (pipe) {
            // R_max over the radii after the update of k - 1 and the hit points of k
            PM_HIP(hipStreamWaitEvent(st, s->ev_eye[k % s->ring], 0));
            hipLaunchKernelGGL(k_rmax_clear, dim3(1), dim3(64), 0, st, dk);
            hipLaunchKernelGGL(k_rmax, dim3(std::min(blocks_for(s->P), kRmaxBlocks)), dim3(kBlock), 0, st, dk,
                               (const double *)s->R2);
        } else {
            // one iteration at a time: eye pass and R_max on a second stream, beside the photon pass:
            // they share no data, and the eye pass's long specular paths would
            // otherwise leave the device idle at its end
            hipStream_t side = s->streams.pass[1];
            PM_HIP(hipEventRecord(s->ev_fork, st));
            PM_HIP(hipStreamWaitEvent(side, s->ev_fork, 0));
            forked.q[0] = side;
            forked.n = 1;
            if (timed) PM_HIP(hipEventRecord(ev[1], side));
            hipLaunchKernelGGL(k_rmax_clear, dim3(1), dim3(64), 0, side, dk);
            eye_pass(dk, k, side);
            hipLaunchKernelGGL(k_rmax, dim3(std::min(blocks_for(s->P), kRmaxBlocks)), dim3(kBlock), 0, side, dk,
                               (const double *)s->R2);
            if (timed) PM_HIP(hipEventRecord(ev[2], side));
            PM_HIP(hipEventRecord(s->ev_join, side));
            if (timed) PM_HIP(hipEventRecord(ev[3], st));
            if ((rc = enqueue_photon(s, dk, k, count, st))) return rc;
            if (timed) PM_HIP(hipEventRecord(ev[4], st));
        }
        hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(T)), dim3(kBlock), 0, st, s->cell_count, T, 0u);
        if (!pipe) PM_HIP(hipStreamWaitEvent(st, s->ev_join, 0));
        if (pipe) PM_HIP(hipStreamWaitEvent(st, s->ev_ph[k % s->ring], 0));
        if (timed) PM_HIP(hipEventRecord(ev[5], st));
        if (dk.gather_mode == PM_GATHER_STOCHASTIC) {
            hipLaunchKernelGGL(k_sh_clear, dim3(std::min<uint32_t>(blocks_for(T), 4096u)), dim3(kBlock), 0, st, dk, T);
            hipLaunchKernelGGL(k_sh_insert, dim3(ph_blocks), dim3(kBlock), 0, st, dk, k, s->cell_count);
            hipLaunchKernelGGL(k_sh_pick, dim3(ph_blocks), dim3(kBlock), 0, st, dk, k);
            if (timed) PM_HIP(hipEventRecord(ev[6], st));
            hipLaunchKernelGGL(k_sh_gather, dim3(blocks_for(s->P)), dim3(kBlock), 0, st, dk,
                               (const uint32_t *)s->cell_count);
            // this gather reads the photon store itself: only now may the pass of k + ring refill it
            if (pipe) PM_HIP(hipEventRecord(s->ev_scat[k % s->ring], st));
        } else {
            hipLaunchKernelGGL(k_count, dim3(ph_blocks), dim3(kBlock), 0, st, dk, s->cell_count);
            launch_bucket_scan(s->cell_count, s->cell_start, s->cell_fill, s->bsum, T, st);
            hipLaunchKernelGGL(k_scatter, dim3(ph_blocks), dim3(kBlock), 0, st, dk, (const uint32_t *)s->cell_start,
                               s->sorted);
            if (pipe) PM_HIP(hipEventRecord(s->ev_scat[k % s->ring], st));
            if (timed) PM_HIP(hipEventRecord(ev[6], st));
            const int hits = hits_per_wave(s->P);
            auto gather = count        ? k_gather<64, true>
                          : hits == 64 ? k_gather<64, false>
                          : hits == 16 ? k_gather<16, false>
                                       : k_gather<4, false>;
            hipLaunchKernelGGL(gather, dim3(blocks_for(s->P * (64 / (count ? 64 : hits)))), dim3(kBlock), 0, st, dk,
                               (const uint32_t *)s->cell_start, (const float4 *)s->sorted);
        }
        if (timed) PM_HIP(hipEventRecord(ev[7], st));
        double *hist = (int32_t)k < s->rec_iters ? s->R2_hist + (size_t)k * s->P : nullptr;
        hipLaunchKernelGGL(k_update, dim3(blocks_for(s->P)), dim3(kBlock), 0, st, dk, hist);
        if (pipe) PM_HIP(hipEventRecord(s->ev_upd[k % s->ring], st));
        PM_HIP(hipGetLastError());
        if (timed) {  // wait for the iteration and add its stage times
            PM_HIP(hipEventRecord(ev[8], st));
            PM_HIP(hipEventSynchronize(ev[8]));
            float ms[kProfTimes];
            PM_HIP(hipEventElapsedTime(&ms[0], ev[1], ev[2]));  // eye pass + R_max (side stream)
            PM_HIP(hipEventElapsedTime(&ms[1], ev[3], ev[4]));  // photon pass
            PM_HIP(hipEventElapsedTime(&ms[2], ev[5], ev[6]));  // hashed grid
            PM_HIP(hipEventElapsedTime(&ms[3], ev[6], ev[7]));  // range query
            PM_HIP(hipEventElapsedTime(&ms[4], ev[7], ev[8]));  // update
            PM_HIP(hipEventElapsedTime(&ms[5], ev[0], ev[8]));  // whole iteration
            for (int i = 0; i < kProfTimes; ++i) s->prof_ms[i] += ms[i];
            s->prof_timed_iters++;
        }
        if (count) s->prof_counted_iters++;
        s->K++;
    }
    if (pipe) PM_HIP(join_streams(s, st, caller));
    return PM_OK;
}

int sppm_iterate(pm_sppm *s, int32_t n_iter, hipStream_t st) {
    if (!s || n_iter < 0) return set_error("invalid handle or iteration count"), PM_ERR_ARG;
    if (!s->cell_count) return set_error("handle belongs to a batch: iterate the batch"), PM_ERR_STATE;
    if (n_iter == 0) return PM_OK;
    Forked forked;
    const int rc = run_iterations(s, n_iter, st, forked);
    if (rc) join_after_error(s, forked, st);
    return rc;
}

int sppm_get_stats(pm_sppm *s, pm_sppm_stats *out, int32_t reset, hipStream_t st) {
    if (!s || !out) return set_error("NULL handle or output"), PM_ERR_ARG;
    if (out->size < sizeof(pm_sppm_stats)) return set_error("pm_sppm_stats.size too small"), PM_ERR_ARG;
    unsigned long long c[kStatCount] = {};
    if (s->stats) {
        PM_HIP(hipMemcpyAsync(c, s->stats, sizeof(c), hipMemcpyDeviceToHost, st));
        PM_HIP(hipStreamSynchronize(st));
    }
    const uint32_t size = out->size;
    memset(out, 0, sizeof(pm_sppm_stats));
    out->size = size;
    out->counted_iterations = s->prof_counted_iters;
    out->eye_paths = c[kStatEyePaths];
    out->eye_rays = c[kStatEyeRays];
    out->eye_box_tests = c[kStatEyeBoxes];
    out->eye_tri_tests = c[kStatEyeTris];
    out->photon_paths = c[kStatPhotonPaths];
    out->photon_rays = c[kStatPhotonRays];
    out->photon_box_tests = c[kStatPhotonBoxes];
    out->photon_tri_tests = c[kStatPhotonTris];
    out->gather_hit_points = c[kStatGatherHits];
    out->gather_buckets = c[kStatGatherBuckets];
    out->gather_examined = c[kStatGatherExamined];
    out->gather_accepted = c[kStatGatherAccepted];
    out->photons_stored = c[kStatPhotonStored];
    out->timed_iterations = s->prof_timed_iters;
    out->ms_eye = s->prof_ms[0];
    out->ms_photon = s->prof_ms[1];
    out->ms_grid = s->prof_ms[2];
    out->ms_gather = s->prof_ms[3];
    out->ms_update = s->prof_ms[4];
    out->ms_iteration = s->prof_ms[5];
    if (reset) {
        if (s->stats) {
            hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(kBlock), 0, st, (uint32_t *)s->stats, 2u * kStatCount, 0u);
            PM_HIP(hipGetLastError());
        }
        s->prof_counted_iters = s->prof_timed_iters = 0;
        for (double &m : s->prof_ms) m = 0.0;
    }
    return PM_OK;
}

int sppm_resolve(pm_sppm *s, float *image, hipStream_t st) {
    if (!s || !image) return set_error("invalid handle or image pointer"), PM_ERR_ARG;
    if (s->K == 0) return set_error("no iteration has run"), PM_ERR_STATE;
    hipLaunchKernelGGL(k_resolve, dim3(blocks_for(s->P)), dim3(kBlock), 0, st, s->dev, s->K, image);
    PM_HIP(hipGetLastError());
    return PM_OK;
}

int sppm_status(pm_sppm *s, hipStream_t st) {
    if (!s) return set_error("NULL handle"), PM_ERR_ARG;
    uint32_t c[4 * kRing];
    PM_HIP(hipMemcpyAsync(c, s->counters, sizeof(c), hipMemcpyDeviceToHost, st));
    PM_HIP(hipStreamSynchronize(st));
    const uint32_t flags = c[1] | c[5] | c[9];  // the sticky flags of all slots
    if (flags & 1u) return set_error("photon store overflow: raise store_factor"), PM_ERR_OVERFLOW;
    if (flags & 2u)
        return set_error("flux fixed-point overflow (a term or a pixel's sum passed 2^64): lower fixed_shift"),
               PM_ERR_OVERFLOW;
    return PM_OK;
}

// The adjoint's replay with consecutive iterations overlapped, as in the
// forward iteration: the replayed photon passes (each with its flux maximum)
// and the replayed eye passes (with R_max and the |G| wk maximum) of the next
// iterations run on their slots' streams beside the grid, gather and path sums
// of k, into the photon store, (path, bounce) tables, hit points and maxima of
// their slot (k % ring), once iteration k - ring has read them.  Every sum is
// an integer sum, so the gradient equals the serial schedule's bit for bit.
static int adjoint_overlapped(pm_sppm *s, const float *g, hipStream_t caller, Forked &forked) {
    hipStream_t st = work_stream(s, caller);
    const uint32_t T = 1u << s->table_bits;
    const uint32_t np = (uint32_t)s->prm.n_photons;
    const int32_t mb = s->prm.max_photon_bounces;
    const uint32_t ph_blocks = std::min<uint32_t>(blocks_for(s->cap), 256u * 64u);
    const uint32_t K = (uint32_t)s->K;
    const double Kd = (double)s->K;
    auto mat_of = [&](uint32_t k) { return s->mat_tab[k % s->ring]; };
    auto tab_of = [&](uint32_t k) { return s->adj_tab[k % s->ring]; };
    const int hits = hits_per_wave(s->P);
    auto max_of = [&](uint32_t k) { return s->adj_max + 2 * (k % s->ring); };
    // the replayed photon pass on its iteration's photon stream; the flux maximum follows it
    auto replay = [&](uint32_t k) -> int {
        const SppmDev dk = iteration_view(s, k);
        hipStream_t q = photon_queue(s, k);
        if (k >= s->ring) PM_HIP(hipStreamWaitEvent(q, s->ev_scat[k % s->ring], 0));
        hipLaunchKernelGGL(k_photon_begin, dim3(1), dim3(64), 0, q, dk, s->thin ? np : 0u);
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, q, (uint32_t *)(max_of(k) + 1), 2u, 0u);
        if (s->thin) {
            hipLaunchKernelGGL(pick(s, k_photon<true, true>, k_photon<true, false>), dim3(blocks_for_waves(np, s->thin)), dim3(kBlock), 0, q, dk, k, s->thin,
                               mat_of(k), tab_of(k));
        } else if (s->dev.photon_kernel == PM_PHOTON_TWO_PHASE) {
            const PathQueue &pq = s->queue[k % s->ring];
            hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, q, pq.cnt, 1u, 0u);
            hipLaunchKernelGGL(pick(s, k_photon_head_rec<true>, k_photon_head_rec<false>), dim3(s->head_grid_rec), dim3(kBlock), 0, q, dk, k, pq,
                               mat_of(k), tab_of(k));
            hipLaunchKernelGGL(pick(s, k_photon_tail_rec<true>, k_photon_tail_rec<false>), dim3(s->tail_grid_rec), dim3(kBlock), 0, q, dk, pq, mat_of(k),
                               tab_of(k));
        } else {
            hipLaunchKernelGGL(pick(s, k_photon_regen_rec<true>, k_photon_regen_rec<false>), dim3(s->regen_grid_rec), dim3(kBlock), 0, q, dk, k,
                               mat_of(k), tab_of(k));
        }
        hipLaunchKernelGGL(k_adj_phimax, dim3(std::min<uint32_t>(ph_blocks, kAdjMaxBlocks)), dim3(kBlock), 0, q, dk,
                           max_of(k));
        PM_HIP(hipGetLastError());
        PM_HIP(hipEventRecord(s->ev_ph[k % s->ring], q));
        return PM_OK;
    };
    // the replayed eye pass, R_max (over the recorded radii) and max |G| wk of
    // iteration k, on its eye stream, into the hit-point buffer, R_max
    // accumulator and maxima of k's slot
    auto eye_chain = [&](uint32_t k) -> int {
        const SppmDev dk = iteration_view(s, k);
        hipStream_t q = eye_queue(s, k);
        const double *R2k = s->R2_hist + (size_t)k * s->P;
        if (k >= s->ring) PM_HIP(hipStreamWaitEvent(q, s->ev_upd[k % s->ring], 0));
        hipLaunchKernelGGL(k_rmax_clear, dim3(1), dim3(64), 0, q, dk);
        hipLaunchKernelGGL(pick(s, k_eye<true>, k_eye<false>), dim3(blocks_for(s->P)), dim3(kBlock), 0, q, dk, k, 0);
        hipLaunchKernelGGL(k_rmax, dim3(std::min(blocks_for(s->P), kRmaxBlocks)), dim3(kBlock), 0, q, dk, R2k);
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, q, (uint32_t *)max_of(k), 2u, 0u);
        hipLaunchKernelGGL(k_adj_gmax, dim3(std::min<uint32_t>(blocks_for(s->P), kAdjMaxBlocks)), dim3(kBlock), 0,
                           q, dk, R2k, g, Kd, max_of(k));
        PM_HIP(hipGetLastError());
        PM_HIP(hipEventRecord(s->ev_eye[k % s->ring], q));
        return PM_OK;
    };
    PM_HIP(fork_streams(s, 0u, K, st, caller, forked));
    uint32_t sent = 0;  // iterations whose replays are enqueued
    for (uint32_t k = 0; k < K; ++k) {
        const SppmDev dk = iteration_view(s, k);
        const double *R2k = s->R2_hist + (size_t)k * s->P;
        // a replay reuses the slot (store, tables, hit points, maxima) that iteration k - ring read
        for (; sent < K && sent < k + s->ring; ++sent) {
            if (int rc = replay(sent)) return rc;
            if (int rc = eye_chain(sent)) return rc;
        }
        hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(T)), dim3(kBlock), 0, st, s->cell_count, T, 0u);
        hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(4 * s->n_mat)), dim3(kBlock), 0, st, (uint32_t *)s->adj_wide,
                           (uint32_t)(4 * s->n_mat), 0u);
        PM_HIP(hipStreamWaitEvent(st, s->ev_eye[k % s->ring], 0));
        PM_HIP(hipStreamWaitEvent(st, s->ev_ph[k % s->ring], 0));
        hipLaunchKernelGGL(k_adj_scale, dim3(1), dim3(64), 0, st, (const unsigned long long *)max_of(k), s->adj_scale);
        hipLaunchKernelGGL(k_count, dim3(ph_blocks), dim3(kBlock), 0, st, dk, s->cell_count);
        launch_bucket_scan(s->cell_count, s->cell_start, s->cell_fill, s->bsum, T, st);
        hipLaunchKernelGGL(k_scatter, dim3(ph_blocks), dim3(kBlock), 0, st, dk, (const uint32_t *)s->cell_start,
                           s->sorted);
        hipLaunchKernelGGL(gather_adj_of(hits), dim3(blocks_for(s->P * (64 / hits))), dim3(kBlock), 0, st, dk, R2k,
                           (const uint32_t *)s->cell_start, (const float4 *)s->sorted, g, Kd,
                           (const double *)s->adj_scale, tab_of(k), s->n_mat, s->adj_wide);
        PM_HIP(hipEventRecord(s->ev_upd[k % s->ring], st));
        hipLaunchKernelGGL(k_path_adj, dim3(blocks_for(np)), dim3(kBlock), 0, st, (const uint16_t *)mat_of(k),
                           (const long long *)tab_of(k), np, mb, s->n_mat, s->adj_wide);
        PM_HIP(hipEventRecord(s->ev_scat[k % s->ring], st));
        hipLaunchKernelGGL(k_adj_fold, dim3(1), dim3(kMaxAdjMat), 0, st, (const unsigned long long *)s->adj_wide,
                           s->n_mat, (const double *)s->adj_scale, dk.sc.mat_rho, s->grad_mat);
        PM_HIP(hipGetLastError());
    }
    PM_HIP(join_streams(s, st, caller));
    return PM_OK;
}

// The same, one iteration after another (a handle with one slot).
static int adjoint_serial(pm_sppm *s, const float *g, hipStream_t st, Forked &forked) {
    const uint32_t T = 1u << s->table_bits;
    const uint32_t np = (uint32_t)s->prm.n_photons;
    const int32_t mb = s->prm.max_photon_bounces;
    const uint32_t ph_blocks = std::min<uint32_t>(blocks_for(s->cap), 256u * 64u);
    const double K = (double)s->K;
    const SppmDev &d = s->dev;
    const int hits = hits_per_wave(s->P);
    for (int32_t k = 0; k < s->K; ++k) {
        const double *R2k = s->R2_hist + (size_t)k * s->P;
        hipLaunchKernelGGL(k_begin, dim3(1), dim3(64), 0, st, d);
        hipLaunchKernelGGL(k_adj_begin, dim3(1), dim3(kBlock), 0, st, s->adj_max, s->adj_wide, s->n_mat);
        hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(T)), dim3(kBlock), 0, st, s->cell_count, T, 0u);
        // replayed eye pass, R_max and max |G| wk beside the replayed photon pass, as in the forward iteration
        hipStream_t side = s->streams.pass[1];
        PM_HIP(hipEventRecord(s->ev_fork, st));
        PM_HIP(hipStreamWaitEvent(side, s->ev_fork, 0));
        forked.q[0] = side;
        forked.n = 1;
        hipLaunchKernelGGL(pick(s, k_eye<true>, k_eye<false>), dim3(blocks_for(s->P)), dim3(kBlock), 0, side, d, (uint32_t)k, 0);
        hipLaunchKernelGGL(k_rmax, dim3(std::min(blocks_for(s->P), kRmaxBlocks)), dim3(kBlock), 0, side, d, R2k);
        hipLaunchKernelGGL(k_adj_gmax, dim3(std::min<uint32_t>(blocks_for(s->P), kAdjMaxBlocks)), dim3(kBlock), 0,
                           side, d, R2k, g, K, s->adj_max);
        PM_HIP(hipEventRecord(s->ev_join, side));
        hipLaunchKernelGGL(pick(s, k_photon_regen_rec<true>, k_photon_regen_rec<false>), dim3(s->regen_grid_rec), dim3(kBlock), 0, st, d, (uint32_t)k,
                           s->mat_tab[0], s->adj_tab[0]);
        hipLaunchKernelGGL(k_adj_phimax, dim3(std::min<uint32_t>(ph_blocks, kAdjMaxBlocks)), dim3(kBlock), 0, st, d,
                           s->adj_max);
        PM_HIP(hipStreamWaitEvent(st, s->ev_join, 0));
        hipLaunchKernelGGL(k_adj_scale, dim3(1), dim3(64), 0, st, (const unsigned long long *)s->adj_max,
                           s->adj_scale);
        hipLaunchKernelGGL(k_count, dim3(ph_blocks), dim3(kBlock), 0, st, d, s->cell_count);
        launch_bucket_scan(s->cell_count, s->cell_start, s->cell_fill, s->bsum, T, st);
        hipLaunchKernelGGL(k_scatter, dim3(ph_blocks), dim3(kBlock), 0, st, d, (const uint32_t *)s->cell_start,
                           s->sorted);
        hipLaunchKernelGGL(gather_adj_of(hits), dim3(blocks_for(s->P * (64 / hits))), dim3(kBlock), 0, st, d, R2k,
                           (const uint32_t *)s->cell_start, (const float4 *)s->sorted, g, K,
                           (const double *)s->adj_scale, s->adj_tab[0], s->n_mat, s->adj_wide);
        hipLaunchKernelGGL(k_path_adj, dim3(blocks_for(np)), dim3(kBlock), 0, st, (const uint16_t *)s->mat_tab[0],
                           (const long long *)s->adj_tab[0], np, mb, s->n_mat, s->adj_wide);
        hipLaunchKernelGGL(k_adj_fold, dim3(1), dim3(kMaxAdjMat), 0, st, (const unsigned long long *)s->adj_wide,
                           s->n_mat, (const double *)s->adj_scale, d.sc.mat_rho, s->grad_mat);
        PM_HIP(hipGetLastError());
    }
    return PM_OK;
}

int sppm_adjoint(pm_sppm *s, const float *g, const int32_t *pmat, int32_t n_par, double *grad, hipStream_t st) {
    if (!s || !g || !grad || n_par < 0 || (n_par > 0 && !pmat))
        return set_error("invalid handle, gradient or parameter pointers"), PM_ERR_ARG;
    if (!s->cell_count) return set_error("handle belongs to a batch"), PM_ERR_STATE;
    if (s->K < 1) return set_error("no iteration has run"), PM_ERR_STATE;
    if (s->K > s->rec_iters)
        return set_error("the forward iterations were not recorded: set record_iterations >= K"), PM_ERR_STATE;
    if (n_par >= kMaxAdjMat) return set_error("too many parameters"), PM_ERR_ARG;
    for (int32_t i = 0; i < n_par; ++i) {
        if (pmat[i] < 0 || pmat[i] >= s->n_mat) return set_error("parameter material out of range"), PM_ERR_ARG;
        if (!(s->rho_host[pmat[i]] > 0.0f)) return set_error("albedo parameters must have rho > 0"), PM_ERR_ARG;
    }
    const double K = (double)s->K;
    const SppmDev &d = s->dev;
    ParamMats pms;
    for (int32_t i = 0; i < n_par; ++i) pms.m[i] = (uint8_t)pmat[i];
    hipLaunchKernelGGL(k_fill_f64, dim3(blocks_for(s->n_mat + 1)), dim3(kBlock), 0, st, s->grad_mat,
                       (int64_t)s->n_mat + 1);
    Forked forked;
    if (int rc = s->ring > 1 ? adjoint_overlapped(s, g, st, forked) : adjoint_serial(s, g, st, forked)) {
        join_after_error(s, forked, st);
        return rc;
    }
    const uint32_t n_part = blocks_for(s->P);
    hipLaunchKernelGGL(k_le_grad, dim3(n_part), dim3(kBlock), 0, st, d, K, g, s->le_part);
    hipLaunchKernelGGL(k_collect_grad, dim3(1), dim3(kMaxAdjMat), 0, st, s->grad_mat, pms, n_par,
                       (const double *)s->le_part, (int32_t)n_part, s->le_single > 0.0 ? 1.0 / s->le_single : 0.0,
                       grad);
    PM_HIP(hipGetLastError());
    return PM_OK;
}

namespace {

// Checkpoint layout: this header, then N, R2, tau, D (f64 [P] each), then
// n_hist recorded radii (f64 [n_hist][P]).
struct CheckpointHeader {
    char magic[8];  // "PMSPPMCK"
    uint32_t version, header_bytes;
    int64_t n_pixels, n_photons;
    uint64_t seed, scene_hash;
    double alpha, r0;
    int32_t fixed_shift, max_eye_depth, max_photon_bounces, record_iterations;
    int32_t iterations, n_hist;
    uint32_t overflow;
    int32_t gather_mode;
};
constexpr uint32_t kCheckpointVersion = 1;

uint64_t checkpoint_bytes(const pm_sppm *s, int32_t n_hist) {
    return sizeof(CheckpointHeader) + (uint64_t)(4 + n_hist) * (uint64_t)s->P * sizeof(double);
}

}  // namespace

int sppm_save(pm_sppm *s, void *buf, uint64_t *size, hipStream_t st) {
    if (!s || !size) return set_error("NULL handle or size pointer"), PM_ERR_ARG;
    if (!s->cell_count) return set_error("handle belongs to a batch"), PM_ERR_STATE;
    const int32_t n_hist = std::min(s->K, s->rec_iters);
    const uint64_t need = checkpoint_bytes(s, n_hist);
    if (!buf) {
        *size = need;
        return PM_OK;
    }
    if (*size < need) {
        *size = need;
        return set_error("checkpoint buffer too small (the required size is returned in *size)"), PM_ERR_ARG;
    }
    uint32_t c[4 * kRing];
    PM_HIP(hipMemcpyAsync(c, s->counters, sizeof(c), hipMemcpyDeviceToHost, st));
    CheckpointHeader h{};
    memcpy(h.magic, "PMSPPMCK", 8);
    h.version = kCheckpointVersion;
    h.header_bytes = sizeof(CheckpointHeader);
    h.n_pixels = s->P;
    h.n_photons = s->prm.n_photons;
    h.seed = s->prm.seed;
    h.scene_hash = s->scene_hash;
    h.alpha = s->prm.alpha;
    h.r0 = s->prm.r0;
    h.fixed_shift = s->prm.fixed_shift;
    h.max_eye_depth = s->prm.max_eye_depth;
    h.max_photon_bounces = s->prm.max_photon_bounces;
    h.record_iterations = s->rec_iters;
    h.iterations = s->K;
    h.n_hist = n_hist;
    h.gather_mode = s->prm.gather_mode;
    uint8_t *out = (uint8_t *)buf;
    const size_t pb = sizeof(double) * (size_t)s->P;
    const double *arrays[4] = {s->N, s->R2, s->tau, s->D};
    for (int a = 0; a < 4; ++a)
        PM_HIP(hipMemcpyAsync(out + sizeof(h) + a * pb, arrays[a], pb, hipMemcpyDeviceToHost, st));
    if (n_hist > 0)
        PM_HIP(hipMemcpyAsync(out + sizeof(h) + 4 * pb, s->R2_hist, pb * (size_t)n_hist, hipMemcpyDeviceToHost, st));
    PM_HIP(hipStreamSynchronize(st));
    h.overflow = c[1] | c[5] | c[9];  // the sticky flags of all slots, now that the copy has ended
    memcpy(out, &h, sizeof(h));
    *size = need;
    return PM_OK;
}

int sppm_load(pm_sppm *s, const void *buf, uint64_t size, hipStream_t st) {
    if (!s || !buf) return set_error("NULL handle or buffer"), PM_ERR_ARG;
    if (!s->cell_count) return set_error("handle belongs to a batch"), PM_ERR_STATE;
    CheckpointHeader h;
    if (size < sizeof(h)) return set_error("checkpoint too short"), PM_ERR_ARG;
    memcpy(&h, buf, sizeof(h));
    if (memcmp(h.magic, "PMSPPMCK", 8) != 0 || h.version != kCheckpointVersion || h.header_bytes != sizeof(h))
        return set_error("not a checkpoint of this format version"), PM_ERR_ARG;
    if (h.n_pixels != s->P || h.n_photons != s->prm.n_photons || h.seed != s->prm.seed ||
        h.scene_hash != s->scene_hash || h.alpha != s->prm.alpha || h.r0 != s->prm.r0 ||
        h.fixed_shift != s->prm.fixed_shift || h.max_eye_depth != s->prm.max_eye_depth ||
        h.max_photon_bounces != s->prm.max_photon_bounces || h.record_iterations != s->rec_iters ||
        h.gather_mode != s->prm.gather_mode)
        return set_error("checkpoint was taken from a handle with another scene or parameters"), PM_ERR_ARG;
    if (h.iterations < 0 || h.n_hist != std::min(h.iterations, s->rec_iters) ||
        size < checkpoint_bytes(s, h.n_hist))
        return set_error("checkpoint is truncated or inconsistent"), PM_ERR_ARG;
    const uint8_t *in = (const uint8_t *)buf;
    const size_t pb = sizeof(double) * (size_t)s->P;
    double *arrays[4] = {s->N, s->R2, s->tau, s->D};
    for (int a = 0; a < 4; ++a)
        PM_HIP(hipMemcpyAsync(arrays[a], in + sizeof(h) + a * pb, pb, hipMemcpyHostToDevice, st));
    if (h.n_hist > 0)
        PM_HIP(hipMemcpyAsync(s->R2_hist, in + sizeof(h) + 4 * pb, pb * (size_t)h.n_hist, hipMemcpyHostToDevice, st));
    if (h.overflow) PM_HIP(hipMemcpyAsync(s->counters + 1, &h.overflow, sizeof(h.overflow), hipMemcpyHostToDevice, st));
    PM_HIP(hipStreamSynchronize(st));
    s->K = h.iterations;
    return PM_OK;
}

int sppm_views(pm_sppm *s, pm_sppm_views *v) {
    if (!s || !v || v->size < sizeof(pm_sppm_views)) return set_error("invalid handle or views struct"), PM_ERR_ARG;
    v->n_pixels = s->P;
    v->iterations = s->K;
    v->photon_capacity = s->cap;
    v->table_size = int64_t(1) << s->table_bits;
    v->N = s->N;
    v->R2 = s->R2;
    v->tau = s->tau;
    v->D = s->D;
    // the last iteration's hit points, photon store and counters
    const uint32_t i = s->K > 0 ? (uint32_t)(s->K - 1) % s->ring : 0u;
    v->hp_pos = (float *)s->hp_pos[i];
    v->hp_nrm = (float *)s->hp_nrm[i];
    v->photons = (float *)s->store[i];
    v->photon_count = s->counters + 4 * i;
    v->gather_M = s->M;
    v->gather_Phi = (uint64_t *)s->Phi;
    return PM_OK;
}

}  // namespace pm
