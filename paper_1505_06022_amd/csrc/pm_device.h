// Device building blocks of the photon-mapping hot path (gfx950 / CDNA4).
//
// Floating-point rules (the same rules the method is specified with):
// float32 geometry, no contraction of a*b+c into FMA (explicit fmaf only in
// the conservative box test), correctly rounded division and square root,
// fixed evaluation order for dot/cross/normalize, no transcendental calls.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#pragma clang fp contract(off)

namespace pmd {

// ---------------------------------------------------------------------------
// Random numbers (Sec. 3.2): four multiplicative LCGs s <- a*s mod m, each
// evaluated with Schrage's decomposition (q = m div a, r = m mod a) exactly
// as the paper's float code does, but in 32-bit integers; output is the
// fractional part of s0/m0 - s1/m1 + s2/m2 - s3/m3 of the advanced state.
// ---------------------------------------------------------------------------
struct Rng {
    int32_t s0, s1, s2, s3;
};

enum : uint32_t { kKindEye = 1u, kKindPhoton = 2u };

__device__ __forceinline__ int32_t lcg_step(int32_t s, int32_t a, int32_t q, int32_t r, int32_t m) {
    int32_t hi = s / q;
    int32_t lo = s - hi * q;
    int32_t t = a * lo - r * hi;
    return t < 0 ? t + m : t;
}

// s / m rounded to nearest float, for a state 0 < s < m of one of the four
// generators: the product with the rounded reciprocal, corrected once by its
// exact fma residual (Markstein's division, IBM J. Res. Dev. 1990). For these
// four moduli it equals the IEEE quotient for every state (checked
// exhaustively on the host), in 3 instructions instead of the ~10 of a full
// division.
__device__ __forceinline__ float div_by_modulus(int32_t s, float m, float inv_m) {
    float x = (float)s;
    float q0 = x * inv_m;
    float r = __builtin_fmaf(-q0, m, x);
    return __builtin_fmaf(r, inv_m, q0);
}

__device__ __forceinline__ float rng_next(Rng &g) {
    g.s0 = lcg_step(g.s0, 3423, 1225, 1112, 4194287);
    g.s1 = lcg_step(g.s1, 2646, 1585, 367, 4194277);
    g.s2 = lcg_step(g.s2, 1707, 2457, 92, 4194191);
    g.s3 = lcg_step(g.s3, 1999, 2098, 265, 4194167);
    float f0 = div_by_modulus(g.s0, 4194287.0f, 1.0f / 4194287.0f);
    float f1 = div_by_modulus(g.s1, 4194277.0f, 1.0f / 4194277.0f);
    float f2 = div_by_modulus(g.s2, 4194191.0f, 1.0f / 4194191.0f);
    float f3 = div_by_modulus(g.s3, 4194167.0f, 1.0f / 4194167.0f);
    float x = ((f0 - f1) + f2) - f3;
    float u = x - floorf(x);
    return u >= 1.0f ? 0x1.fffffep-1f : u;
}

// splitmix64 (Steele, Lea, Flood 2014)
__device__ __forceinline__ uint64_t splitmix64(uint64_t &st) {
    uint64_t z = (st += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Per-stream state from a counter key: splitmix64 mixes (seed, kind,
// iteration, index) into a Marsaglia xorshift128 seed (the generator the
// paper seeds its per-thread states with), whose outputs 9..12 are reduced
// into [1, m_j - 1].
__device__ __forceinline__ Rng rng_seed(uint64_t seed, uint32_t kind, uint32_t k, uint64_t index) {
    uint64_t st = seed;
    uint64_t h = splitmix64(st);
    st = h ^ (((uint64_t)kind << 32) | (uint64_t)k);
    h = splitmix64(st);
    st = h ^ index;
    uint64_t w01 = splitmix64(st);
    uint64_t w23 = splitmix64(st);
    uint32_t x = (uint32_t)w01, y = (uint32_t)(w01 >> 32), z = (uint32_t)w23, w = (uint32_t)(w23 >> 32);
    if ((x | y | z | w) == 0u) x = 1u;
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        uint32_t t = x ^ (x << 11);
        x = y;
        y = z;
        z = w;
        w = (w ^ (w >> 19)) ^ (t ^ (t >> 8));
        if (i >= 8) o[i - 8] = w;
    }
    Rng g;
    g.s0 = (int32_t)(1u + o[0] % 4194286u);
    g.s1 = (int32_t)(1u + o[1] % 4194276u);
    g.s2 = (int32_t)(1u + o[2] % 4194190u);
    g.s3 = (int32_t)(1u + o[3] % 4194166u);
    return g;
}

// ---------------------------------------------------------------------------
// float3 arithmetic with a fixed evaluation order
// ---------------------------------------------------------------------------
struct V3 {
    float x, y, z;
};
__device__ __forceinline__ V3 v3(float x, float y, float z) { return V3{x, y, z}; }
__device__ __forceinline__ V3 vsub(V3 a, V3 b) { return v3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ float vdot(V3 a, V3 b) { return (a.x * b.x + a.y * b.y) + a.z * b.z; }
__device__ __forceinline__ V3 vcross(V3 a, V3 b) {
    return v3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ V3 vnorm(V3 v) {
    float l = sqrtf(vdot(v, v));
    return v3(v.x / l, v.y / l, v.z / l);
}
__device__ __forceinline__ V3 vneg(V3 a) { return v3(-a.x, -a.y, -a.z); }
__device__ __forceinline__ V3 vray(V3 o, float t, V3 d) { return v3(o.x + t * d.x, o.y + t * d.y, o.z + t * d.z); }

// ---------------------------------------------------------------------------
// Scene layout on the device
// ---------------------------------------------------------------------------
struct Tri {
    V3 v0, v1, v2;
    int32_t id;
    uint32_t mat;
};

// 48-byte triangle record: v0.xyz v1.x | v1.yz v2.xy | v2.z id mat 0
__device__ __forceinline__ Tri load_tri(const float4 *__restrict__ tris, uint32_t k) {
    const float4 *p = tris + 3 * (size_t)k;
    float4 a = p[0], b = p[1], c = p[2];
    Tri t;
    t.v0 = v3(a.x, a.y, a.z);
    t.v1 = v3(a.w, b.x, b.y);
    t.v2 = v3(b.z, b.w, c.x);
    t.id = __float_as_int(c.y);
    t.mat = __float_as_uint(c.z);
    return t;
}

// Edge vectors v1 - v0 and v2 - v0 (for the normal and for points on the
// triangle), rounded once per component.
__device__ __forceinline__ V3 tri_e1(const Tri &t) { return vsub(t.v1, t.v0); }
__device__ __forceinline__ V3 tri_e2(const Tri &t) { return vsub(t.v2, t.v0); }
__device__ __forceinline__ V3 tri_normal(const Tri &t) { return vnorm(vcross(tri_e1(t), tri_e2(t))); }

// Per-ray constants of the watertight triangle test: kz = the major axis of d
// (ties x, y, z, as for the link set), kx = kz + 1 and ky = kz + 2 (mod 3),
// and the shear that maps d onto the kz axis: sx = d_kx / d_kz,
// sy = d_ky / d_kz, sz = 1 / d_kz.
struct Shear {
    float sx, sy, sz;
    uint32_t kz;
};

__device__ __forceinline__ Shear ray_shear(V3 d) {
    const float ax = fabsf(d.x), ay = fabsf(d.y), az = fabsf(d.z);
    Shear h;
    h.kz = (ax >= ay && ax >= az) ? 0u : (ay >= az ? 1u : 2u);
    const float dz = h.kz == 0u ? d.x : (h.kz == 1u ? d.y : d.z);
    const float dx = h.kz == 0u ? d.y : (h.kz == 1u ? d.z : d.x);
    const float dy = h.kz == 0u ? d.z : (h.kz == 1u ? d.x : d.y);
    h.sx = dx / dz;
    h.sy = dy / dz;
    h.sz = 1.0f / dz;
    return h;
}

// a b - c d with a relative error of at most 2u (u = 2^-24; Kahan's 2x2
// determinant with one fused multiply-add for the rounding error of c d), so
// its sign is the exact value's sign.
__device__ __forceinline__ float det2(float a, float b, float c, float d) {
    const float w = c * d;
    const float e = fmaf(-c, d, w);
    const float f = fmaf(a, b, -w);
    return f + e;
}

// Vertex v seen from the ray: (x, y) its position in the plane sheared along
// d (the ray passes through (0, 0)) and z its distance along the kz axis.
__device__ __forceinline__ void shear_vertex(V3 v, V3 o, const Shear &h, float &x, float &y, float &z) {
    const V3 a = vsub(v, o);
    const float az = h.kz == 0u ? a.x : (h.kz == 1u ? a.y : a.z);
    const float ax = h.kz == 0u ? a.y : (h.kz == 1u ? a.z : a.x);
    const float ay = h.kz == 0u ? a.z : (h.kz == 1u ? a.x : a.y);
    x = fmaf(-h.sx, az, ax);
    y = fmaf(-h.sy, az, ay);
    z = az;
}

// Watertight ray/triangle test (two-sided; Woop, Benthin and Wald 2013, with
// the edge functions taken by det2).  The edge functions U, V, W are the
// doubled signed areas that the ray's point spans with each edge of the
// sheared triangle; their signs are exact for the sheared vertices, so the
// ray hits when all three agree, and an edge shared by two triangles has
// the same vertices and the opposite sign in both (no ray slips between
// them).  t = (U z0 + V z1 + W z2) / (U + V + W) (z scaled by sz), the
// depth of the point with those barycentric weights.
//
// Error bound (used by the traversal's box test): the point o + t d lies
// within 22u (t |d_a| + L) of a point of the triangle along every axis a
// (L its longest edge): the weights are the exact non-negative barycentric
// coordinates of the ray in the sheared, rounded vertices (relative error of
// U, V, W at most 2u), each sheared coordinate is within 3u (|t d_a| + L) of
// the exact one, and t within 16u (|t| + L / |d_kz|).
__device__ __forceinline__ bool wt_hit(V3 o, const Shear &h, const Tri &tr, float &t_out) {
    float ax, ay, az, bx, by, bz, cx, cy, cz;
    shear_vertex(tr.v0, o, h, ax, ay, az);
    shear_vertex(tr.v1, o, h, bx, by, bz);
    shear_vertex(tr.v2, o, h, cx, cy, cz);
    const float U = det2(cx, by, cy, bx);
    const float V = det2(ax, cy, ay, cx);
    const float W = det2(bx, ay, by, ax);
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    const float det = (U + V) + W;
    if (det == 0.0f) return false;
    const float T = fmaf(W, h.sz * cz, fmaf(V, h.sz * bz, U * (h.sz * az)));
    t_out = T / det;
    return true;
}

// Closest-hit acceptance: inside (tmin, tbest), ties in t to the lower index.
__device__ __forceinline__ bool accept_hit(float t, int32_t id, float tmin, float tbest, int32_t best) {
    if (!(t > tmin)) return false;
    if (t < tbest) return true;
    return t == tbest && best >= 0 && id < best;
}

// Link set of a ray: the principal direction = major axis of d (ties x, y,
// z), signed by that component (the cube-map lookup of Fig. "mtbvh").
__device__ __forceinline__ int link_set(V3 d) {
    float ax = fabsf(d.x), ay = fabsf(d.y), az = fabsf(d.z);
    if (ax >= ay && ax >= az) return d.x < 0.0f ? 1 : 0;
    if (ay >= az) return d.y < 0.0f ? 3 : 2;
    return d.z < 0.0f ? 5 : 4;
}

struct Bvh {
    const uint4 *nodes;   // [6][n_nodes] 16-byte nodes, then a pad node
    const uint4 *wide;    // [n_wide][4] four-child nodes (see wide_walk), or NULL
    const float4 *tris;   // [n_tri][3] float4
    uint32_t n_nodes;
    float qlo[3], qstep[3];  // node box grid: coordinate = qlo + q * qstep
    float inv_max[3];        // largest reciprocal direction used in the slab test (2^100 / qstep)
};

struct TraceStats {
    uint32_t boxes, tris;
};

// Stackless closest-hit traversal of one link set (Sec. 3.1, Fig. "mtbvh"):
// follow the hit link (next node) when the ray meets the node's box, else the
// miss (skip) link; at a leaf test its triangles and continue with the miss
// link.  The box test is conservative (padded boxes, a relative slack on the
// exit distance; the bound is at box_hit) so the result equals the
// brute-force closest hit.  Walker holds one lane's traversal state so that a persistent kernel
// can interleave node steps of different rays.  kPairTris: a leaf's triangle
// records are requested two at a time (more registers; it pays where leaves
// are full and the kernel's occupancy is already register-bound).
template <bool kPairTris>
struct WalkerT {
    const uint4 *nodes;
    uint32_t n, i;
    V3 o, d;
    Shear sh;                      // the triangle test's shear
    float sx, sy, sz, bx, by, bz;  // slab planes: t = q * s + b per axis
    uint32_t rx, ry, rz;           // byte selectors of each axis's entry plane (see plane)
    float tmin, tbest;
    int32_t best, exclude;
    uint32_t best_k;

    __device__ __forceinline__ void init(const Bvh &bvh, int set, V3 o_, V3 d_, float tmin_, float tmax_,
                                         int32_t exclude_) {
        nodes = bvh.nodes + (size_t)set * bvh.n_nodes;
        n = bvh.n_nodes;
        i = 0;
        o = o_;
        d = d_;
        sh = ray_shear(d_);
        // reciprocal direction; zero components replaced by a tiny signed
        // value, and the reciprocal kept small enough for 2^23 s to stay finite
        // (an axis so clamped moves less than a grid step, half the padding,
        // over any t below 2^100)
        float dx = fabsf(d.x) > 1e-30f ? d.x : copysignf(1e-30f, d.x);
        float dy = fabsf(d.y) > 1e-30f ? d.y : copysignf(1e-30f, d.y);
        float dz = fabsf(d.z) > 1e-30f ? d.z : copysignf(1e-30f, d.z);
        const float ix = clamp_inverse(1.0f / dx, bvh.inv_max[0]), iy = clamp_inverse(1.0f / dy, bvh.inv_max[1]),
                    iz = clamp_inverse(1.0f / dz, bvh.inv_max[2]);
        sx = bvh.qstep[0] * ix;
        sy = bvh.qstep[1] * iy;
        sz = bvh.qstep[2] * iz;
        // the planes come as 2^23 + q (see plane)
        bx = fmaf(-0x1p23f, sx, (bvh.qlo[0] - o.x) * ix);
        by = fmaf(-0x1p23f, sy, (bvh.qlo[1] - o.y) * iy);
        bz = fmaf(-0x1p23f, sz, (bvh.qlo[2] - o.z) * iz);
        select_planes();
        tmin = tmin_;
        tbest = tmax_;
        best = -1;
        best_k = 0;
        exclude = exclude_;
    }

    __device__ __forceinline__ static float clamp_inverse(float i, float most) { return fminf(fmaxf(i, -most), most); }

    // A 16-bit plane coordinate q as the float 2^23 + q, taken from either
    // half of an axis's word by one byte permute: the entry plane is the low
    // half, or the high one where the ray runs towards -axis, so entry and
    // exit distances need no min/max per axis.  (Rotating the word and
    // converting both halves took three instructions a plane pair instead of
    // two; the wide walk, 9 of 10 of its time in vector instructions, went
    // from 0.829 to 0.811 ms on the soup's 2^21 incoherent rays.)
    static constexpr uint32_t kLowHalf = 0x07060100u, kHighHalf = 0x07060302u;
    __device__ __forceinline__ void select_planes() {
        rx = sx < 0.0f ? kHighHalf : kLowHalf;
        ry = sy < 0.0f ? kHighHalf : kLowHalf;
        rz = sz < 0.0f ? kHighHalf : kLowHalf;
    }
    __device__ __forceinline__ static float plane(uint32_t word, uint32_t select) {
        return __uint_as_float(__builtin_amdgcn_perm(0x4b000000u, word, select));
    }

    __device__ __forceinline__ bool done() const { return i >= n; }

    // One node visit (and, at a leaf, its triangles).  Requires !done().
    // Next node: i + 1 after an inner-node hit or any leaf, else the skip link.
    template <bool kStats>
    __device__ __forceinline__ void step(const float4 *__restrict__ tris, TraceStats &st) {
        visit<kStats>(nodes[i], tris, st);
    }

    // The visit of node i once its record q has been loaded.
    template <bool kStats>
    __device__ __forceinline__ void visit(const uint4 &q, const float4 *__restrict__ tris, TraceStats &st) {
        const bool leaf = (q.w >> 31) != 0u;
        const bool hit = box_hit(q);
        if (kStats) st.boxes++;
        if (hit && leaf) leaf_tris<kStats>(tris, q.w, st);
        i = (hit || leaf) ? i + 1 : q.w;
    }

    // Slab test of a quantised node box against [tmin, tbest].  Each word
    // holds one axis as lo | hi << 16; plane() takes the entry and the exit
    // plane from the halves that the ray's direction names.
    //
    // Conservative: a plane distance fma(2^23 + q, s, b) is within 5u |t| +
    // 2u ext / |d_a| + s / 2 of the exact one (u = 2^-24, ext the scene
    // extent, for any ray origin): s is rounded once, and b = (lo - o) / d -
    // 2^23 s, with the same rounded s, once at the size of 2^23 s (the s / 2,
    // half a grid step, 128u ext / |d_a|) and once at that of (lo - o) / d.
    // An accepted triangle hit at
    // t puts o + t d within 22u (|t d_a| + L) of a point of the triangle along
    // each axis (see wt_hit), so inside the triangle's box grown by that
    // much.  The absolute parts (2u ext, 128u ext, 22u L: at most 169u ext in
    // all) are covered three times over by
    // the padding of every box (at least 2^-15 ext = 512u ext), and the relative parts,
    // at most 54u |t| in all, by the slack kBoxSlack = 256u on the exit
    // distance: every box that holds a triangle with an accepted hit at a t
    // in (tmin, tbest] passes, so the walk finds the brute-force closest hit.
    static constexpr float kBoxSlack = 0x1p-16f;
    __device__ __forceinline__ bool box_hit(const uint4 &q) const {
        float tn;
        return box_near(q, tn);
    }

    // The same test, with the entry distance in tn.
    __device__ __forceinline__ bool box_near(const uint4 &q, float &tn) const {
        constexpr uint32_t kOther = kLowHalf ^ kHighHalf;
        const float nx = fmaf(plane(q.x, rx), sx, bx), fx = fmaf(plane(q.x, rx ^ kOther), sx, bx);
        const float ny = fmaf(plane(q.y, ry), sy, by), fy = fmaf(plane(q.y, ry ^ kOther), sy, by);
        const float nz = fmaf(plane(q.z, rz), sz, bz), fz = fmaf(plane(q.z, rz ^ kOther), sz, bz);
        tn = fmaxf(fmaxf(nx, ny), fmaxf(nz, tmin));
        const float tf = fminf(fminf(fx, fy), fminf(fz, tbest));
        return tn <= fmaf(fabsf(tf), kBoxSlack, tf);
    }

    template <bool kStats>
    __device__ __forceinline__ void leaf_tris(const float4 *__restrict__ tris, uint32_t w, TraceStats &st) {
        uint32_t first = (w >> 3) & 0x0fffffffu, cnt = w & 7u;
        // the excluded triangle is checked after the test, so that a record's
        // words arrive in one round trip (a branch on the index first would
        // wait for it before loading the vertices)
        if constexpr (kPairTris) {
            for (uint32_t k = 0; k < cnt; k += 2) {
                const bool two = k + 1 < cnt;
                const Tri ta = load_tri(tris, first + k);
                const Tri tb = load_tri(tris, first + k + (two ? 1u : 0u));
                if (kStats) st.tris += two ? 2u : 1u;
                tri_test(ta, first + k);
                if (two) tri_test(tb, first + k + 1);
            }
        } else {
            for (uint32_t k = 0; k < cnt; ++k) {
                const Tri tr = load_tri(tris, first + k);
                if (kStats) st.tris++;
                tri_test(tr, first + k);
            }
        }
    }

    // Triangle record rec against the ray: the closest hit so far, ties in t
    // to the lower original index, the excluded triangle skipped.
    __device__ __forceinline__ void tri_test(const Tri &tr, uint32_t rec) {
        float t;
        if (wt_hit(o, sh, tr, t) && tr.id != exclude && accept_hit(t, tr.id, tmin, tbest, best)) {
            tbest = t;
            best = tr.id;
            best_k = rec;
        }
    }

    // A ray of the wide walk whose stack ran out: the stackless walk from the
    // root, keeping the closest hit found so far (testing a triangle again
    // changes nothing).
    __device__ __forceinline__ void finish_binary(const Bvh &bvh) {
        nodes = bvh.nodes + (size_t)link_set(d) * bvh.n_nodes;
        n = bvh.n_nodes;
        i = 0;
        TraceStats st{0u, 0u};
        while (!done()) step<false>(bvh.tris, st);
    }

    // Up to two node visits per memory round trip: nodes i and i + 1 are
    // loaded together; when the walk continues at i + 1 (an inner-node hit or
    // any leaf) that node is tested without waiting for another load.
    template <bool kStats>
    __device__ __forceinline__ void step2(const float4 *__restrict__ tris, TraceStats &st) {
        uint4 q0 = nodes[i];
        uint4 q1 = nodes[i + 1 < n ? i + 1 : i];
        if (kStats) st.boxes++;
        bool leaf = (q0.w >> 31) != 0u, hit = box_hit(q0);
        if (hit && leaf) leaf_tris<kStats>(tris, q0.w, st);
        if (!(hit || leaf)) {
            i = q0.w;
            return;
        }
        i = i + 1;
        if (i >= n) return;
        if (kStats) st.boxes++;
        leaf = (q1.w >> 31) != 0u;
        hit = box_hit(q1);
        if (hit && leaf) leaf_tris<kStats>(tris, q1.w, st);
        i = (hit || leaf) ? i + 1 : q1.w;
    }

    // The whole walk with postponed leaf tests.  The wave visits boxes until
    // at most `late` of its lanes are still looking for a leaf hit (and at
    // least one lane holds one); then every lane that holds a leaf tests its
    // triangles, all lanes together.  A lane that holds a leaf keeps visiting
    // boxes while others search and halts in front of its next leaf hit, which
    // it visits again after the tests.  The wave votes once per
    // kPostponedSteps box visits (fewer ballots and branches per visit; an
    // idle lane just waits a few steps longer).  Each round of visits advances
    // every searching lane, so the walk ends.  The closest hit under the
    // lower-index tie rule does not depend on the order of the visits: the
    // result is the one of step().
#ifndef PM_POSTPONED_STEPS
#define PM_POSTPONED_STEPS 8
#endif
    static constexpr int kPostponedSteps = PM_POSTPONED_STEPS;

    template <bool kStats>
    __device__ __forceinline__ void walk_postponed(const float4 *__restrict__ tris, uint32_t late, TraceStats &st) {
        uint32_t held = 0u;  // link word of a leaf hit not yet tested, or 0
        bool halted = false;
        for (;;) {
            for (;;) {
                const uint64_t searching = __ballot(i < n && held == 0u);
                if (searching == 0ull) break;
                if ((uint32_t)__popcll(searching) <= late && __ballot(held != 0u) != 0ull) break;
#pragma unroll
                for (int u = 0; u < kPostponedSteps; ++u) {
                    if (i < n && !halted) {
                        const uint4 q = nodes[i];
                        if (kStats) st.boxes++;
                        const bool leaf = (q.w >> 31) != 0u, hit = box_hit(q);
                        const bool leaf_hit = hit && leaf;
                        halted = leaf_hit && held != 0u;
                        held = (leaf_hit && held == 0u) ? q.w : held;
                        i = halted ? i : ((hit || leaf) ? i + 1 : q.w);
                    }
                }
            }
            if (__ballot(held != 0u) == 0ull) break;  // no lane searching and none holding: all done
            if (held != 0u) leaf_tris<kStats>(tris, held, st);
            held = 0u;
            halted = false;
        }
    }

    __device__ __forceinline__ float t_hit() const { return best >= 0 ? tbest : __builtin_inff(); }
};
using Walker = WalkerT<false>;

// ---------------------------------------------------------------------------
// Wide walk: the closest hit through nodes of four children (64 bytes: four
// records in the layout of the binary node, whose link word names an inner
// child's wide node or a leaf's triangles).  The nodes are the binary tree of
// link set 0 with levels merged (wide.hip), so the boxes and the box test,
// and with them the proof that no accepted hit is culled, are those of the
// binary walk; children are taken by entry distance and the rest wait on a
// stack in LDS.  The closest hit under the lower-index tie rule does not
// depend on the order, so the result is that of the stackless walk.
//
// The binary walks are bound by their chain of dependent node reads (every
// read names the next): an incoherent ray of the 2^20-triangle soup makes 111.
// Here it makes 24, to one array of 23 MB instead of six of 147 MB together.
// 2^21 such rays, bucketing included, went from 1.83 to 0.81 ms, the camera's
// 2^21 in 8x8 tiles from 0.34 (packets) to 0.27 ms.  Now the vector units, busy
// 98% of the time with 36% of their lanes, and the L1 data path, busy 91%, bind
// together, so that easing one does not help: finished lanes refilled (19% fewer
// instructions, 18% more L1 accesses) 0.93 ms, held leaves' triangles spread over
// the wave's lanes 0.84, nodes fetched to LDS by four lanes each (4 waves a SIMD)
// 1.02.
//
// Two shapes of the same walk:
//  * one ray per lane (four boxes per lane and step), leaf tests held until at
//    most `late` lanes still look for a leaf;
//  * four lanes per ray (quads), each lane testing one child box or one
//    triangle.  A wave with at most kQuadRays unfinished rays moves them to
//    quads: a step then costs half the instructions of the lane form, a leaf's
//    tests a quarter, so the last rays of a wave, whose latency nothing hides,
//    end sooner (without quads the 2^21 rays take 1.08 ms, with them for the
//    last 8 rays of a wave 0.90).
// ---------------------------------------------------------------------------
constexpr uint32_t kWideNone = 0x7fffffffu;  // no node: the walk has ended
// Stack entries per ray: 21 in use at most (a visit may write three more); the
// soups and the 250k-triangle scene need up to 18.  A ray that needs more
// takes the binary walk (with 16 entries the 2^18-triangle soup's 1% of such
// rays made its walk 30% slower; 32 leave fewer waves resident, 9% slower).
constexpr int kWideStack = 24;
constexpr uint32_t kQuadRays = 16;
// Kernels with the wide walk ask for 6 wavefronts per SIMD (at most 80
// registers): its stacks leave room for 26 per compute unit.
#define PM_WIDE_WAVES __attribute__((amdgpu_waves_per_eu(6)))

__device__ __forceinline__ uint32_t lane_index() {
    return __builtin_amdgcn_mbcnt_hi(0xffffffffu, __builtin_amdgcn_mbcnt_lo(0xffffffffu, 0u));
}

// The value of the lane whose index in the quad differs by kXor (1, 2 or 3).
template <int kXor>
__device__ __forceinline__ int quad_xor(int v) {
    constexpr int kCtrl = kXor == 1 ? 0xB1 : (kXor == 2 ? 0x4E : 0x1B);
    return __builtin_amdgcn_mov_dpp(v, kCtrl, 0xf, 0xf, true);
}
__device__ __forceinline__ float quad_min(float v) {
    v = fminf(v, __int_as_float(quad_xor<1>(__float_as_int(v))));
    return fminf(v, __int_as_float(quad_xor<2>(__float_as_int(v))));
}
__device__ __forceinline__ uint32_t quad_min(uint32_t v) {
    v = min(v, (uint32_t)quad_xor<1>((int)v));
    return min(v, (uint32_t)quad_xor<2>((int)v));
}
__device__ __forceinline__ float pull(uint32_t lane, float v) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute((int)(lane << 2), __float_as_int(v)));
}
__device__ __forceinline__ uint32_t pull(uint32_t lane, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(lane << 2), (int)v);
}

// Orders (ka, ra), (kb, rb) by key.
__device__ __forceinline__ void sort_pair(int &ka, uint32_t &ra, int &kb, uint32_t &rb) {
    const bool s = kb < ka;
    const int k0 = min(ka, kb), k1 = max(ka, kb);
    const uint32_t r0 = s ? rb : ra, r1 = s ? ra : rb;
    ka = k0;
    kb = k1;
    ra = r0;
    rb = r1;
}

// One visit of wide node cur by one lane: the nearest child hit becomes cur,
// the others go on the stack, farthest first; with no hit the top of the
// stack does.  Entry e of a ray's stack is col[64 e]; entry 0 is kWideNone.
template <class W>
__device__ __forceinline__ void wide_step(W &w, const uint4 *__restrict__ wide, uint32_t *col, uint32_t &cur,
                                          uint32_t &sp, bool &overflow) {
    const uint4 *p = wide + 4 * (size_t)cur;
    const uint4 q0 = p[0], q1 = p[1], q2 = p[2], q3 = p[3];
    const uint32_t top = col[(sp - 1u) * 64u];
    float t0, t1, t2, t3;
    const bool h0 = w.box_near(q0, t0), h1 = w.box_near(q1, t1), h2 = w.box_near(q2, t2), h3 = w.box_near(q3, t3);
    uint32_t r0 = h0 ? q0.w : kWideNone, r1 = h1 ? q1.w : kWideNone, r2 = h2 ? q2.w : kWideNone,
             r3 = h3 ? q3.w : kWideNone;
    // distances order as their bits (negative ones, possible with tmin < 0, among themselves in reverse, which only
    // costs time); misses are above every distance, so the hits come first
    int k0 = h0 ? __float_as_int(t0) : 0x7fffffff, k1 = h1 ? __float_as_int(t1) : 0x7fffffff,
        k2 = h2 ? __float_as_int(t2) : 0x7fffffff, k3 = h3 ? __float_as_int(t3) : 0x7fffffff;
    sort_pair(k0, r0, k1, r1);
    sort_pair(k2, r2, k3, r3);
    sort_pair(k0, r0, k2, r2);
    sort_pair(k1, r1, k3, r3);
    sort_pair(k1, r1, k2, r2);
    col[sp * 64u] = r3;
    sp += r3 != kWideNone ? 1u : 0u;
    col[sp * 64u] = r2;
    sp += r2 != kWideNone ? 1u : 0u;
    col[sp * 64u] = r1;
    sp += r1 != kWideNone ? 1u : 0u;
    const bool none = r0 == kWideNone;  // then nothing was pushed
    cur = none ? top : r0;
    sp -= none ? 1u : 0u;
    if (sp > (uint32_t)kWideStack - 3u) {  // a visit writes entries sp .. sp + 2
        overflow = true;
        cur = kWideNone;
    }
}

// The last rays of a wave (at most kQuadRays lanes with cur != kWideNone),
// four lanes each.  Called by all lanes of the wave; each ray's result returns
// to the lane it came from.  stk is the wave's stack; a ray keeps its lane's
// column.  All four lanes of a quad hold the same ray and the same cur and sp.
template <class W>
__device__ __forceinline__ void wide_quads(W &w, const uint4 *__restrict__ wide, const float4 *__restrict__ tris,
                                           uint32_t *stk, uint32_t &cur_io, uint32_t sp_io, bool &overflow_io) {
    const uint32_t lane = lane_index(), c = lane & 3u;
    const uint64_t busy0 = __ballot(cur_io != kWideNone);
    const uint32_t n_rays = (uint32_t)__popcll(busy0);
    const uint32_t rank0 = __builtin_amdgcn_mbcnt_hi((uint32_t)(busy0 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)busy0, 0u));
    const bool mine = cur_io != kWideNone;
    // quad g takes the g-th unfinished ray: its lane tells the quad's first lane
    // its own index (finished lanes address lane 3 of quad 15, which no ray uses as first lane)
    uint32_t owner = (uint32_t)__builtin_amdgcn_ds_permute((int)((mine ? 4u * rank0 : 63u) << 2), (int)lane);
    owner = (uint32_t)__builtin_amdgcn_mov_dpp((int)owner, 0x00, 0xf, 0xf, true);
    const bool has = (lane >> 2) < n_rays;
    owner = has ? owner : 0u;
    W x;
    x.o = v3(pull(owner, w.o.x), pull(owner, w.o.y), pull(owner, w.o.z));
    x.sh.sx = pull(owner, w.sh.sx);
    x.sh.sy = pull(owner, w.sh.sy);
    x.sh.sz = pull(owner, w.sh.sz);
    x.sh.kz = pull(owner, w.sh.kz);
    x.sx = pull(owner, w.sx);
    x.sy = pull(owner, w.sy);
    x.sz = pull(owner, w.sz);
    x.bx = pull(owner, w.bx);
    x.by = pull(owner, w.by);
    x.bz = pull(owner, w.bz);
    x.select_planes();
    x.tmin = pull(owner, w.tmin);
    x.tbest = pull(owner, w.tbest);
    x.best = (int32_t)pull(owner, (uint32_t)w.best);
    x.best_k = pull(owner, w.best_k);
    x.exclude = (int32_t)pull(owner, (uint32_t)w.exclude);
    uint32_t cur = pull(owner, cur_io), sp = pull(owner, sp_io);
    cur = has ? cur : kWideNone;
    uint32_t *col = stk + owner;
    bool overflow = false;
    for (;;) {
        const uint64_t busy = __ballot(cur != kWideNone);
        if (busy == 0ull) break;
        if (cur < kWideNone) {
            const uint4 q = wide[4 * (size_t)cur + c];
            const uint32_t top = col[(sp - 1u) * 64u];
            float tn;
            const bool h = x.box_near(q, tn);
            // unique keys: the entry distance's bits with the lane in the last two; a miss is above every distance
            const int key = h ? ((__float_as_int(tn) & ~3) | (int)c) : (int)(0x7ffffffcu | c);
            const uint32_t rank = (quad_xor<1>(key) < key ? 1u : 0u) + (quad_xor<2>(key) < key ? 1u : 0u) +
                                  (quad_xor<3>(key) < key ? 1u : 0u);
            const uint32_t nh = (uint32_t)__popc((uint32_t)(__ballot(h) >> (lane & 60u)) & 15u);
            if (h && rank != 0u) col[(sp + nh - 1u - rank) * 64u] = q.w;
            uint32_t nearest = (h && rank == 0u) ? q.w : 0u;  // no child's word is 0 (node 0 is the root)
            nearest |= (uint32_t)quad_xor<1>((int)nearest);
            nearest |= (uint32_t)quad_xor<2>((int)nearest);
            cur = nh != 0u ? nearest : top;
            sp = sp + nh - 1u;
            if (sp > (uint32_t)kWideStack - 3u) {
                overflow = true;
                cur = kWideNone;
            }
            // the quad's lanes read each other's entries
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        const uint64_t inner = __ballot(cur < kWideNone);
        if (2u * (uint32_t)__popcll(inner) > (uint32_t)__popcll(busy)) continue;
        if ((cur >> 31) != 0u) {
            const uint32_t first = (cur >> 3) & 0x0fffffffu, cnt = cur & 7u;
            float bt = __builtin_inff();
            uint32_t bid = 0xffffffffu, bk = 0xffffffffu;
            for (uint32_t k = c; k < cnt; k += 4u) {
                const Tri tr = load_tri(tris, first + k);
                float t;
                if (wt_hit(x.o, x.sh, tr, t) && tr.id != x.exclude && accept_hit(t, tr.id, x.tmin, x.tbest, x.best) &&
                    (t < bt || (t == bt && (uint32_t)tr.id < bid))) {
                    bt = t;
                    bid = (uint32_t)tr.id;
                    bk = first + k;
                }
            }
            const float m = quad_min(bt);
            const uint32_t id = quad_min(bt == m ? bid : 0xffffffffu);
            const uint32_t rec = quad_min(bt == m && bid == id ? bk : 0xffffffffu);
            if (id != 0xffffffffu) {
                x.tbest = m;
                x.best = (int32_t)id;
                x.best_k = rec;
            }
            cur = col[(sp - 1u) * 64u];
            sp -= 1u;
        }
    }
    const uint32_t from = 4u * rank0 & 63u;  // first lane of this lane's quad (unfinished lanes only)
    const float tb = pull(from, x.tbest);
    const uint32_t bi = pull(from, (uint32_t)x.best), bk = pull(from, x.best_k), ov = pull(from, overflow ? 1u : 0u);
    if (mine) {
        w.tbest = tb;
        w.best = (int32_t)bi;
        w.best_k = bk;
        overflow_io = overflow_io || ov != 0u;
        cur_io = kWideNone;
    }
}

// Node visits between two votes of the wave in the lane form (1 costs 8% on
// bucketed incoherent rays, 4 gains 1% there and loses 4% on camera rays).
constexpr int kWideSteps = 2;

// One lane's walk between two rounds: the node or leaf it goes on with, its
// stack, and a leaf set aside (0: none).
struct WideState {
    uint32_t cur = kWideNone, sp = 1u, held = 0u;
    bool overflow = false;

    __device__ __forceinline__ void start(uint32_t *col) {
        col[0] = kWideNone;
        cur = 0u;
        sp = 1u;
        held = 0u;
        overflow = false;
    }
    __device__ __forceinline__ bool busy() const { return cur != kWideNone || held != 0u; }
};

// One round of the lane form, called by all lanes of a wave of which some are
// busy: either kWideSteps node visits by the lanes at inner nodes, or, once
// at most `late` lanes are and some lane holds a leaf, the held leaves' tests.
// A lane that reaches a leaf sets it aside and goes on until it meets a second
// one (most leaves hold no hit, so the visits are rarely in vain).
template <class W>
__device__ __forceinline__ void wide_round(W &w, const uint4 *__restrict__ wide, const float4 *__restrict__ tris,
                                           uint32_t *col, WideState &s, uint32_t late) {
    const uint64_t inner = __ballot(s.cur < kWideNone);
    if (inner != 0ull && ((uint32_t)__popcll(inner) > late || __ballot(s.held != 0u) == 0ull)) {
#pragma unroll
        for (int u = 0; u < kWideSteps; ++u)
            if (s.cur < kWideNone) wide_step(w, wide, col, s.cur, s.sp, s.overflow);
    } else {
        TraceStats st{0u, 0u};
        if (s.held != 0u) w.template leaf_tris<false>(tris, s.held, st);
        s.held = 0u;
    }
    if ((s.cur >> 31) != 0u && s.held == 0u) {
        s.held = s.cur;
        s.cur = col[(s.sp - 1u) * 64u];
        s.sp -= 1u;
    }
}

// The last rays of a wave: on quads (at most kQuadRays lanes are busy).
template <class W>
__device__ __forceinline__ void wide_drain(W &w, const uint4 *__restrict__ wide, const float4 *__restrict__ tris,
                                           uint32_t *stk, WideState &s) {
    if (s.held != 0u) {  // the leaf set aside comes first
        if (s.cur != kWideNone) {
            stk[lane_index() + s.sp * 64u] = s.cur;
            s.sp += 1u;
        } else {
            s.sp = 1u;  // entry 0, taken when the walk ended, is still there
        }
        s.cur = s.held;
        s.held = 0u;
    }
    // the quads read the columns their lanes wrote
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    wide_quads(w, wide, tris, stk, s.cur, s.sp, s.overflow);
}

// The whole walk of one ray per lane, called by all lanes of a wave (active:
// this lane has a ray, initialised in w).  stk: the wave's stack in LDS, 64
// kWideStack words.  Returns true when this lane's stack ran out: the caller
// then finishes the ray with the binary walk from the root, which keeps the
// hits found so far.
template <class W>
__device__ __forceinline__ bool wide_walk(W &w, const uint4 *__restrict__ wide, const float4 *__restrict__ tris,
                                          uint32_t *stk, bool active, uint32_t late) {
    uint32_t *col = stk + lane_index();
    WideState s;
    if (active) s.start(col);
    while ((uint32_t)__popcll(__ballot(s.busy())) > kQuadRays) wide_round(w, wide, tris, col, s, late);
    if (__ballot(s.busy()) != 0ull) wide_drain(w, wide, tris, stk, s);
    return s.overflow;
}

// Packet walk, for a wave whose lanes all walk one link set (nodes = that
// set's node array, the same on every lane): the wave follows one node index,
// taking the hit link when any lane's box test passes and the skip link
// otherwise; at a leaf each lane whose own box test passes tests the
// triangles.  The nodes a lane meets are a superset of those of its own walk
// and its box tests use its own t_best, so its closest hit is unchanged.  The
// node index, the link words and so every branch are uniform across the wave,
// and all lanes read the same node and triangle records.
template <bool kStats>
__device__ __forceinline__ uint32_t packet_visit(Walker &w, const uint4 &q, uint32_t i,
                                                 const float4 *__restrict__ tris, TraceStats &st) {
    const uint32_t link = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.w);
    const bool hit = w.box_hit(q);
    if (kStats) st.boxes++;
    if ((link >> 31) != 0u) {
        if (hit) w.leaf_tris<kStats>(tris, link, st);
        return i + 1;
    }
    return __ballot(hit) != 0ull ? i + 1 : link;
}

// Nodes a packet walk requests at once (measured: 2 beats 1, 3, 4 and 5).
constexpr int kPacketRun = 2;

template <bool kStats>
__device__ __forceinline__ void walk_packet(Walker &w, const uint4 *__restrict__ nodes, uint32_t n,
                                            const float4 *__restrict__ tris, TraceStats &st) {
    constexpr int kRun = kPacketRun;
    uint32_t i = 0;
    while (i < n) {
        // nodes i .. i + kRun - 1 come in one request: each is the next node
        // after a hit or a leaf, which then costs no further round trip
        const uint4 *p = nodes + i;  // in bounds: the node arrays end with kRun - 1 pad nodes
        uint4 q[kRun];
#pragma unroll
        for (int k = 0; k < kRun; ++k) q[k] = p[k];
        uint32_t cur = packet_visit<kStats>(w, q[0], i, tris, st);
#pragma unroll
        for (int k = 1; k < kRun; ++k)
            if (cur == i + (uint32_t)k && cur < n) cur = packet_visit<kStats>(w, q[k], cur, tris, st);
        i = cur;
    }
    w.i = n;
}

// Two rays per lane walked in lockstep: both node records are requested
// before either box is tested, so each lane keeps two loads in flight.  A
// walker that has finished re-reads node 0 of its link set (an in-bounds,
// cached address) and is left unchanged until the other one finishes.
template <bool kStats>
__device__ __forceinline__ void walk_two(Walker &a, Walker &b, const float4 *__restrict__ tris, TraceStats &sa,
                                         TraceStats &sb) {
    for (;;) {
        const bool da = a.done(), db = b.done();
        if (da && db) break;
        const uint4 qa = a.nodes[da ? 0u : a.i];
        const uint4 qb = b.nodes[db ? 0u : b.i];
        if (!da) a.visit<kStats>(qa, tris, sa);
        if (!db) b.visit<kStats>(qb, tris, sb);
    }
}

// Returns the original index of the closest triangle (-1: none); t_out gets
// its distance (+inf on a miss) and k_out its position in the triangle array.
// paired: the walk requests nodes i and i + 1 together (step2); kPairTris:
// a leaf's triangle records two at a time.
template <bool kStats, bool kPairTris = false>
__device__ __forceinline__ int32_t closest_hit(const Bvh &bvh, int set, V3 o, V3 d, float tmin, float tmax,
                                               int32_t exclude, float &t_out, uint32_t &k_out, TraceStats &st,
                                               bool paired = false) {
    WalkerT<kPairTris> w;
    w.init(bvh, set, o, d, tmin, tmax, exclude);
    if (paired) {
        while (!w.done()) w.template step2<kStats>(bvh.tris, st);
    } else {
        while (!w.done()) w.template step<kStats>(bvh.tris, st);
    }
    t_out = w.t_hit();
    k_out = w.best_k;
    return w.best;
}

// Wave-aggregated counter increment for the lanes in `mask` (uniform across
// the wave): returns base + rank of this lane within mask.
__device__ __forceinline__ uint32_t wave_fetch_add(uint32_t *counter, uint64_t mask, bool member) {
    uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    int leader = __ffsll((unsigned long long)mask) - 1;
    uint32_t base = 0;
    if (member && rank == 0) base = atomicAdd(counter, (uint32_t)__popcll(mask));
    base = __shfl(base, leader);
    return base + rank;
}

// ---------------------------------------------------------------------------
// Sampling (only + - * / sqrt; the same rules as the method's definition)
// ---------------------------------------------------------------------------
// Orthonormal basis about unit n (Duff et al. 2017).
__device__ __forceinline__ void onb(V3 n, V3 &b1, V3 &b2) {
    float sign = copysignf(1.0f, n.z);
    float a = -1.0f / (sign + n.z);
    float b = n.x * n.y * a;
    b1 = v3(1.0f + sign * n.x * n.x * a, sign * b, -sign * n.x);
    b2 = v3(b, sign + n.y * n.y * a, -n.y);
}

// Cosine-weighted direction about unit n: disk point by rejection from the
// square (at most 64 tries), lifted to the hemisphere (Malley's method).
__device__ __forceinline__ V3 cosine_dir(V3 n, Rng &g) {
    float a = 0.0f, b = 0.0f, r2 = 0.0f;
    bool ok = false;
    for (int tries = 0; tries < 64; ++tries) {
        a = 2.0f * rng_next(g) - 1.0f;
        b = 2.0f * rng_next(g) - 1.0f;
        r2 = a * a + b * b;
        if (r2 < 1.0f) {
            ok = true;
            break;
        }
    }
    if (!ok) {
        a = 0.0f;
        b = 0.0f;
        r2 = 0.0f;
    }
    float z = sqrtf(1.0f - r2);
    V3 t1, t2;
    onb(n, t1, t2);
    V3 w = v3((a * t1.x + b * t2.x) + z * n.x, (a * t1.y + b * t2.y) + z * n.y, (a * t1.z + b * t2.z) + z * n.z);
    return vnorm(w);
}

__device__ __forceinline__ V3 reflect(V3 d, V3 n) {
    float c = 2.0f * vdot(d, n);
    return v3(d.x - c * n.x, d.y - c * n.y, d.z - c * n.z);
}

// Smooth dielectric: unpolarised Fresnel reflectance picks reflection or
// refraction with one draw (also drawn under total internal reflection).
__device__ __forceinline__ V3 glass_dir(V3 d, V3 n, float ior, Rng &g) {
    float cosi = -vdot(d, n);
    float eta, ci;
    V3 nn;
    if (cosi > 0.0f) {
        eta = 1.0f / ior;
        nn = n;
        ci = cosi;
    } else {
        eta = ior;
        nn = vneg(n);
        ci = -cosi;
    }
    float sin2t = (eta * eta) * (1.0f - ci * ci);
    float k = 1.0f - sin2t;
    float F = 1.0f, ct = 0.0f;
    if (k >= 0.0f) {
        ct = sqrtf(k);
        float rs = (eta * ci - ct) / (eta * ci + ct);
        float rp = (ci - eta * ct) / (ci + eta * ct);
        F = 0.5f * (rs * rs + rp * rp);
    }
    float u = rng_next(g);
    if (u < F) return reflect(d, n);
    float c = eta * ci - ct;
    return vnorm(v3(eta * d.x + c * nn.x, eta * d.y + c * nn.y, eta * d.z + c * nn.z));
}

constexpr float kInvPiF = 0.318309886183790671538f;
constexpr double kPiD = 3.14159265358979323846;

// XCD-aware block order: hardware hands consecutive workgroups to the 8 XCDs
// round robin; remap so each XCD (and its L2) owns a contiguous range.
__device__ __forceinline__ uint32_t xcd_block(uint32_t bid, uint32_t nblk) {
    uint32_t per = nblk >> 3, rem = nblk & 7u;
    uint32_t x = bid & 7u, k = bid >> 3;
    return x * per + (x < rem ? x : rem) + k;
}

}  // namespace pmd
