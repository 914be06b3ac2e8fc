// Internal state of an SPPM handle (shared by the single-scene driver and the
// batched driver).
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "runtime.h"
#include "sppm_dev.h"

// Iterations of a pipelined handle that may be under way at once.
constexpr uint32_t kRing = 3;

// The streams of a handle.
struct PassStreams {
    hipStream_t pass[kRing] = {}, main = nullptr;
};

struct pm_sppm {
    pm_sppm_params prm{};
    pm_bvh *bvh = nullptr;
    bool own_bvh = false;
    pmd::SppmDev dev{};  // device view passed to the kernels
    int64_t P = 0;
    int32_t K = 0;
    uint32_t cap = 0;
    uint32_t table_bits = 0;
    uint32_t regen_grid = 1;      // workgroups of the regenerating photon kernel
    uint32_t regen_grid_rec = 1;  // and of its recording variant (adjoint replay)
    uint32_t stream_grid = 1;     // workgroups of the ray-granularity regenerating photon kernel
    uint32_t pool_grid = 1;       // workgroups of the LDS-queue photon kernel
    uint32_t head_grid = 1;       // workgroups of the two-phase pass's first launch
    uint32_t tail_grid = 1;       // and of its second
    uint32_t head_grid_rec = 1;   // the same two launches recording for the adjoint replay
    uint32_t tail_grid_rec = 1;
    bool wide = false;            // its rays take the wide walk (else the binary one)
    uint32_t thin = 0;            // paths per wave of a small default photon pass (one launch), else 0
    float phi0 = 0.0f;
    // device buffers, all within the one allocation `arena`
    void *arena = nullptr;
    int32_t *mat_type = nullptr;
    float *mat_f = nullptr;  // rho | q | Le | ior, each n_mat
    uint32_t *emit_pos = nullptr;
    double *emit_cdf = nullptr;
    double *N = nullptr, *R2 = nullptr, *tau = nullptr, *D = nullptr;
    // what iteration k writes before its grid is built lies in slot k % ring of
    // ring slots (1: an iteration at a time): hit points, emission, photon store, its block
    // of counters, R_max, the paths set aside and the adjoint's tables
    uint32_t ring = 1;
    float4 *hp_pos[kRing] = {}, *hp_nrm[kRing] = {};
    double *emit[kRing] = {};
    float4 *store[kRing] = {}, *sorted = nullptr;
    // streams beside the caller's (default priority), forked from and joined to
    // it by events: see photon_queue and eye_queue; events per slot: photon pass
    // done, eye pass done, photon store read, hit points read
    PassStreams streams;
    int device = 0;
    hipEvent_t ev_ph[kRing] = {}, ev_eye[kRing] = {}, ev_scat[kRing] = {}, ev_upd[kRing] = {};
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    // two-phase photon pass (PM_PHOTON_TWO_PHASE): queues for the paths set
    // aside by the first launch
    void *queue_mem = nullptr;
    pmd::PathQueue queue[kRing] = {};
    uint2 *key_rank = nullptr;  // exact gather: [cap] bucket and rank of each stored photon
    uint32_t *counters = nullptr;  // [kRing][4]: per photon store [0] photons stored, [1] sticky flags, [2] next path, [3] pass leftovers
    unsigned long long *r2max = nullptr;
    // bucket arrays (absent for a batch member, which uses the batch's)
    uint32_t *cell_count = nullptr, *cell_start = nullptr, *cell_fill = nullptr, *bsum = nullptr;
    uint32_t *M = nullptr;
    unsigned long long *Phi = nullptr;
    // adjoint recording / replay buffers (record_iterations > 0)
    int32_t rec_iters = 0;
    int32_t n_mat = 0;
    std::vector<float> rho_host;  // albedos (validation of adjoint parameters)
    double le_single = 0.0;  // Le of the single emitting material, 0 if not exactly one
    double *R2_hist = nullptr;    // [rec_iters][P] radius used in each iteration
    long long *adj_tab[kRing] = {};  // [n_photons][max_bounces] photon sensitivities (fixed point, see adj_*)
    uint16_t *mat_tab[kRing] = {};   // [n_photons][max_bounces] stored-photon materials
    double *grad_mat = nullptr;    // [n_mat + 1]; last entry: sum g L
    unsigned long long *adj_wide = nullptr;  // [2][n_mat] per-material integer sums of one iteration (lo | hi)
    unsigned long long *adj_max = nullptr;   // [kRing][2] per slot: max |G| wk over hit points, max
                                             // flux over photons (double bits)
    double *adj_scale = nullptr;             // [1] fixed-point scale of the current iteration
    double *le_part = nullptr;               // [blocks over pixels] partial sums of g L
    uint64_t scene_hash = 0;      // fingerprint of the scene description (checkpoint matching)
    unsigned long long *sh_key = nullptr;  // stochastic hashing (gather_mode 1): [T] keys
    uint32_t *sh_surv = nullptr;           // and [T] survivors
    // one-bounce-per-pass photon schedule (PM_PHOTON_PASSES): path slots and
    // the number of passes enqueued per iteration before the drain
    void *slot_mem = nullptr;
    pmd::PassSlots slots{};
    int32_t n_pass = 0;
    // profiling (params.profile): device counts, and stage times of each timed iteration
    unsigned long long *stats = nullptr;  // [pmd::kStatCount]
    hipEvent_t prof_ev[9] = {};
    double prof_ms[6] = {};
    int64_t prof_counted_iters = 0, prof_timed_iters = 0;
};

constexpr int kProfTimes = 6;

namespace pm {

// own_grid = false: no bucket arrays (a batch member uses the batch's arrays).
int sppm_create_ex(const pm_scene_desc *d, const pm_sppm_params *p, hipStream_t st, bool own_grid, pm_sppm **out);
void sppm_free(pm_sppm *s);
// Back to the initial state (N = 0, R^2 = r0^2, tau = 0, D = 0, K = 0).
int sppm_reset(pm_sppm *s, hipStream_t st);

constexpr uint64_t kHashPrime = 0x100000001b3ull;

// The hash h = (h ^ w) kHashPrime over the words a[0 .. words_a), b[0 .. words_b)
// (at least one, below 2^32 together) from the state h: launch() uploads them and
// enqueues the work on st (PM_ERR_NOMEM: none, for want of device memory),
// finish() waits for it and gives the final state, release() frees the memory.
class DeviceHash {
  public:
    DeviceHash() = default;
    DeviceHash(const DeviceHash &) = delete;
    ~DeviceHash();
    int launch(uint64_t h, const void *a, size_t words_a, const void *b, size_t words_b, hipStream_t st);
    int finish(uint64_t &h, hipStream_t st);
    void release();

  private:
    void *mem_ = nullptr;
    uint64_t h_ = 0;
    uint32_t n_ = 0, seg_ = 0, n_seg_ = 0;
};

}  // namespace pm
