// Ray traversal kernels.
//
// One persistent kernel template serves three ray sources:
//  LensRays   thin-lens rays for the masked pixels (3.2.2, after Cook's
//             distributed ray tracing), count read from the compaction;
//  PinholeRays  all-in-focus rays, one per full-res pixel (the sharp raster
//             image of section 3, produced by ray casting);
//  RawRays    closest hit of caller-given rays.
//
// Scheduling: each lane owns one ray at a time and advances it up to three
// or four BVH nodes per loop iteration; when enough lanes of a wave are idle
// (16 by default, or all of them) the wave hands them the next rays of its
// pool, a run of 64 ray indices: its first run follows from the wave's number,
// the others it takes with one atomic whenever the pool is empty, so long rays
// do not hold a whole wave hostage (persistent threads with dynamic fetch).
// Eight device counters 256 B apart hand the runs out, an eighth of them each
// to an eighth of the blocks, so the takes of all waves do not queue on one
// address.  A launch with no more rays than lanes deals them evenly
// over its waves instead.  When no ray is left to hand out and at most half of
// a wave's lanes have one, the idle lanes share the others' rays, a pending
// subtree each: the end of a launch, and all of a small one, is then bound by
// the tree's depth and not by a ray's number of visits.  Thin-lens rays come
// from a generation kernel as 24-byte records (origin and direction); a lane
// that takes one derives the watertight test's shear and the slab reciprocals
// itself.  A finishing ray leaves its hit's leaf and distance (8 bytes) that
// the resolve or the G-buffer's shading expands, so no lane waits on scene
// loads for shading.
//
// Closest hit: binary radix tree; the traversal reads a 32-byte copy of each
// node holding both children's boxes in binary16, rounded outward (one fetch
// of two 16-byte words tests two boxes).  Near child first, far child pushed
// on a per-lane stack of 16, 24 or 32 entries in LDS, so a pop is always an
// LDS read.  When the stack is full its oldest 8 entries are dropped; when it
// later runs empty the lane finds the dropped work again by walking parent
// links upwards: at each ancestor reached from its near child (entry
// distances compared as when it was first visited) whose far child still
// passes the box test, that far child is the next subtree.  Every dropped
// entry is such a far child, and the box test only loses children as the
// best hit shrinks, so the walk visits at least the pending subtrees that can
// still hold the closest hit: any depth is exact with no memory beyond LDS.
// Each outer iteration advances a lane by up to three or four nodes (a launch
// knob), which spreads the wave-wide refill and batching decisions over
// several visits.  Leaf hits wait in a 4-entry per-lane queue and the
// triangle test runs when enough lanes of the wave have one (32 by default),
// or a queue is nearly full, or a lane has finished its traversal, so it
// executes with most lanes active instead of once per node visit for a few
// lanes; watertight ray/triangle
// test of Woop, Benthin & Wald (JCGT 2013), two-sided, t > 0, equal
// distances resolved to the smaller triangle id -- the same answer as brute
// force over all triangles.  Box tests are loosened by a relative margin so
// rounding never culls a box that holds the winning triangle.
#include "dof_internal.h"

namespace dof {
namespace {

SceneArgs scene_args(const SceneDev &s) { return SceneArgs{s.nleaf, s.tris, s.albedo, s.nodes16, s.parent}; }

__device__ inline float pick3(float x, float y, float z, int k) { return k == 0 ? x : (k == 1 ? y : z); }

// Entries of the ray's stack were dropped (found again through parent links).
constexpr uint32_t kDropped = 0x80000000u;

struct WRay {
    float o0, o1, o2;
    float sx, sy, sz;
    float ix, iy, iz;   // slab reciprocals (zero components replaced by 1e-20)
    float cnx, cny, cnz, cfx, cfy, cfz;   // slab offsets of the entry and exit planes (box_hit)
    // bits 0-4: 16 where the axis' entry plane is a node word's high half, else
    // 0 (a rotation reads no more of its count); bits 5-6 the watertight test's
    // axes: kx in swx, ky in swy, kz in swz; bit 31 of swx: kDropped
    uint32_t swx, swy, swz;
};

// The watertight test's axes: kz the largest direction component, kx and ky
// the next two in cyclic order, swapped when d[kz] < 0 (keeps the winding).
__device__ inline void wray_axes(const float d[3], int &kx, int &ky, int &kz)
{
    float ax = fabsf(d[0]), ay = fabsf(d[1]), az = fabsf(d[2]);
    kz = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
    kx = kz + 1 == 3 ? 0 : kz + 1;
    ky = kx + 1 == 3 ? 0 : kx + 1;
    if (pick3(d[0], d[1], d[2], kz) < 0.0f) { int t = kx; kx = ky; ky = t; }
}

// A plane p meets the ray at fma(p, 1/d, c) with c = -o/d.  c carries an
// absolute rounding error of at most 2^-24 |c|; it is moved outward by
// max(2^-21 |c|, 2^-30 |1/d|) (down for the entry plane, up for the exit
// plane, which one is which following the sign of 1/d), so the remaining
// errors are relative to the distance and covered by box_hit's exit margin.
// The second term widens each slab by 2^-30 in position: an axis the ray is
// parallel to (d = 0, reciprocal 1e20) then never culls a box whose slab holds
// the origin, faces included.  Needs the origin and the reciprocals; every
// construction of a WRay ends with it.
__device__ inline float slab_offset(float o, float inv, bool entry_if_positive)
{
    const float c = -(o * inv);
    const float e = fmaxf(fabsf(c) * 4.76837158203125e-07f, fabsf(inv) * 9.31322574615478515625e-10f);   // 2^-21, 2^-30
    return (inv > 0.0f) == entry_if_positive ? c - e : c + e;
}

__device__ inline void slab_offsets(WRay &r)
{
    const float clx = slab_offset(r.o0, r.ix, true), chx = slab_offset(r.o0, r.ix, false);
    const float cly = slab_offset(r.o1, r.iy, true), chy = slab_offset(r.o1, r.iy, false);
    const float clz = slab_offset(r.o2, r.iz, true), chz = slab_offset(r.o2, r.iz, false);
    const bool px = r.ix > 0.0f, py = r.iy > 0.0f, pz = r.iz > 0.0f;
    r.cnx = px ? clx : chx; r.cfx = px ? chx : clx; r.swx |= px ? 0u : 16u;
    r.cny = py ? cly : chy; r.cfy = py ? chy : cly; r.swy |= py ? 0u : 16u;
    r.cnz = pz ? clz : chz; r.cfz = pz ? chz : clz; r.swz |= pz ? 0u : 16u;
}

__device__ inline WRay make_wray(const float o[3], const float d[3])
{
    WRay r;
    r.o0 = o[0]; r.o1 = o[1]; r.o2 = o[2];
    int kx, ky, kz;
    wray_axes(d, kx, ky, kz);
    float dz = pick3(d[0], d[1], d[2], kz);
    r.swx = (uint32_t)kx << 5; r.swy = (uint32_t)ky << 5; r.swz = (uint32_t)kz << 5;
    r.sx = pick3(d[0], d[1], d[2], kx) / dz;
    r.sy = pick3(d[0], d[1], d[2], ky) / dz;
    r.sz = 1.0f / dz;
    r.ix = 1.0f / (d[0] != 0.0f ? d[0] : 1e-20f);
    r.iy = 1.0f / (d[1] != 0.0f ? d[1] : 1e-20f);
    r.iz = 1.0f / (d[2] != 0.0f ? d[2] : 1e-20f);
    slab_offsets(r);
    return r;
}

__device__ inline bool tri_hit(const WRay &r, float4 v0, float4 v1, float4 v2, float &tout)
{
    const int kx = (int)(r.swx >> 5 & 3u), ky = (int)(r.swy >> 5), kz = (int)(r.swz >> 5);
    float A0 = v0.x - r.o0, A1 = v0.y - r.o1, A2 = v0.z - r.o2;
    float B0 = v1.x - r.o0, B1 = v1.y - r.o1, B2 = v1.z - r.o2;
    float C0 = v2.x - r.o0, C1 = v2.y - r.o1, C2 = v2.z - r.o2;
    float Akz = pick3(A0, A1, A2, kz), Bkz = pick3(B0, B1, B2, kz), Ckz = pick3(C0, C1, C2, kz);
    float Ax = pick3(A0, A1, A2, kx) - r.sx * Akz;
    float Ay = pick3(A0, A1, A2, ky) - r.sy * Akz;
    float Bx = pick3(B0, B1, B2, kx) - r.sx * Bkz;
    float By = pick3(B0, B1, B2, ky) - r.sy * Bkz;
    float Cx = pick3(C0, C1, C2, kx) - r.sx * Ckz;
    float Cy = pick3(C0, C1, C2, ky) - r.sy * Ckz;
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if (U == 0.0f || V == 0.0f || W == 0.0f) {
        U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
        V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
        W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
    }
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    float det = U + V + W;
    if (det == 0.0f) return false;
    float Az = r.sz * Akz, Bz = r.sz * Bkz, Cz = r.sz * Ckz;
    float T = (U * Az + V * Bz) + W * Cz;
    float t = T / det;
    if (!(t > 0.0f) || !(t < INFINITY)) return false;
    tout = t;
    return true;
}

// The planes of a binary16 node word: low plane in the low half, high plane
// in the high half.  Converted exactly; the compiler folds the conversion into
// the slab test's fused multiply-add (a mixed-precision fma).
__device__ inline float lo16(uint32_t w) { return __half2float(__ushort_as_half((unsigned short)(w & 0xffffu))); }
__device__ inline float hi16(uint32_t w) { return __half2float(__ushort_as_half((unsigned short)(w >> 16))); }

// Conservative slab test of a binary16 box (three node words) against
// [0, limit]; returns the entry distance.  Each word's halves are swapped
// (alignbit by 16) where that axis' reciprocal is negative, so its low half is
// the entry plane and its high half the exit plane in every lane.  The slab
// distance is monotone in the plane (and the entry offset lies below the exit
// offset), so these are exactly the smaller and larger of the two distances:
// one swap per axis instead of a min and a max.  The test only culls, so it
// may use the hardware min/max (no NaN can arise: the reciprocals are
// finite); the exit distance is enlarged by 2^-20 relative to cover rounding.
__device__ inline bool box_hit(const WRay &r, uint32_t wx, uint32_t wy, uint32_t wz, float limit, float &tenter)
{
    wx = __builtin_amdgcn_alignbit(wx, wx, r.swx);
    wy = __builtin_amdgcn_alignbit(wy, wy, r.swy);
    wz = __builtin_amdgcn_alignbit(wz, wz, r.swz);
    float nx = fmaf(lo16(wx), r.ix, r.cnx), fx = fmaf(hi16(wx), r.ix, r.cfx);
    float ny = fmaf(lo16(wy), r.iy, r.cny), fy = fmaf(hi16(wy), r.iy, r.cfy);
    float nz = fmaf(lo16(wz), r.iz, r.cnz), fz = fmaf(hi16(wz), r.iz, r.cfz);
    float tn = fmaxf(fmaxf(nx, ny), nz);
    float tf = fminf(fminf(fx, fy), fz) * 1.00000095367431640625f;
    tenter = tn;
    // tn <= tf, tf >= 0 and tn <= limit (limit >= 0) in one comparison
    return fmaxf(tn, 0.0f) <= fminf(tf, limit);
}

// Slab tests of both children of a binary16 node.
__device__ inline void node_hits(const WRay &r, const BvhNode16 &nd, float limit, bool &hl, bool &hr, float &tl,
                                 float &tr)
{
    hl = box_hit(r, nd.a.x, nd.a.y, nd.a.z, limit, tl);
    hr = box_hit(r, nd.a.w, nd.b.x, nd.b.y, limit, tr);
}

struct Hit {
    float t;
    uint32_t id;    // original triangle id, ~0u = none
    uint32_t leaf;  // sorted position
};

__device__ inline void consider_leaf(const SceneArgs &S, const WRay &r, uint32_t leaf, Hit &h)
{
    float4 v0 = S.tris[3 * (size_t)leaf], v1 = S.tris[3 * (size_t)leaf + 1], v2 = S.tris[3 * (size_t)leaf + 2];
    float t;
    if (tri_hit(r, v0, v1, v2, t)) {
        uint32_t id = __float_as_uint(v0.w);
        if (t < h.t || (t == h.t && id < h.id)) {
            h.t = t;
            h.id = id;
            h.leaf = leaf;
        }
    }
}

struct Shaded {
    float r, g, b;
    float n0, n1, n2;
};

// A leaf's triangle (its id in the first vertex's w) and albedo.
struct LeafData {
    float4 v0, v1, v2, al;
};

__device__ inline LeafData load_leaf(const SceneArgs &S, uint32_t leaf)
{
    return {S.tris[3 * (size_t)leaf], S.tris[3 * (size_t)leaf + 1], S.tris[3 * (size_t)leaf + 2], S.albedo[leaf]};
}

// Lambert: two-sided geometric normal facing the ray, one directional light
// plus ambient.
__device__ inline Shaded shade(const LeafData &leaf, const SceneShade &sh, const float d[3])
{
    const float4 v0 = leaf.v0, v1 = leaf.v1, v2 = leaf.v2, al = leaf.al;
    float e10 = v1.x - v0.x, e11 = v1.y - v0.y, e12 = v1.z - v0.z;
    float e20 = v2.x - v0.x, e21 = v2.y - v0.y, e22 = v2.z - v0.z;
    float n0 = e11 * e22 - e12 * e21, n1 = e12 * e20 - e10 * e22, n2 = e10 * e21 - e11 * e20;
    float len = sqrtf((n0 * n0 + n1 * n1) + n2 * n2);
    n0 = n0 / len; n1 = n1 / len; n2 = n2 / len;
    if ((n0 * d[0] + n1 * d[1]) + n2 * d[2] > 0.0f) { n0 = -n0; n1 = -n1; n2 = -n2; }
    float ndl = -((n0 * sh.light_dir[0] + n1 * sh.light_dir[1]) + n2 * sh.light_dir[2]);
    if (!(ndl > 0.0f)) ndl = 0.0f;
    Shaded o;
    o.r = al.x * (sh.light_rad[0] * ndl + sh.ambient[0]);
    o.g = al.y * (sh.light_rad[1] * ndl + sh.ambient[1]);
    o.b = al.z * (sh.light_rad[2] * ndl + sh.ambient[2]);
    o.n0 = n0; o.n1 = n1; o.n2 = n2;
    return o;
}

__device__ inline uint32_t pcg_hash(uint32_t v)
{
    // PCG-RXS-M-XS hash (Jarzynski & Olano, "Hash Functions for GPU Rendering", JCGT 2020)
    uint32_t state = v * 747796405u + 2891336453u;
    uint32_t word = ((state >> ((state >> 28u) + 4u)) ^ state) * 277803737u;
    return (word >> 22u) ^ word;
}

__device__ inline bool in_aperture(const Aperture &ap, float x, float y)
{
    if (ap.blades < 3) return x * x + y * y < 1.0f;
    for (int i = 0; i < ap.blades; ++i)
        if (x * ap.nx[i] + y * ap.ny[i] > ap.apothem) return false;
    return true;
}

// Lens point by rejection from [-1, 1)^2 (24-bit lattice), at most 32 tries:
// try att of ray k of the pixel whose hashed seed is h.
constexpr uint32_t kLensTries = 32;

__device__ inline uint32_t lens_seed(uint32_t seed, uint32_t frame, uint32_t q)
{
    return pcg_hash(pcg_hash(pcg_hash(seed) ^ frame) ^ q);
}

__device__ inline bool lens_try(const Aperture &ap, uint32_t h, uint32_t k, uint32_t att, float &x, float &y)
{
    uint32_t a = pcg_hash(h ^ ((k << 8) | att));
    uint32_t b = pcg_hash(a);
    x = (float)(a >> 8) * (1.0f / 8388608.0f) - 1.0f;
    y = (float)(b >> 8) * (1.0f / 8388608.0f) - 1.0f;
    return in_aperture(ap, x, y);
}

// The tries att0, att0 + 1, ... of a ray; (0, 0) when none of the 32 lands.
__device__ inline void lens_point_from(const Aperture &ap, uint32_t h, uint32_t k, uint32_t att0, float &lx, float &ly)
{
    for (uint32_t att = att0; att < kLensTries; ++att) {
        float x, y;
        if (lens_try(ap, h, k, att, x, y)) {
            lx = x;
            ly = y;
            return;
        }
    }
    lx = 0.0f;
    ly = 0.0f;
}

__device__ inline void lens_point(const Aperture &ap, uint32_t seed, uint32_t frame, uint32_t q, uint32_t k,
                                  float &lx, float &ly)
{
    lens_point_from(ap, lens_seed(seed, frame, q), k, 0, lx, ly);
}

__device__ inline void st_rgba(void *p, int fmt, size_t i, float4 v)
{
    if (fmt == DOF_RGBA32F) {
        reinterpret_cast<float4 *>(p)[i] = v;
    } else {
        __half2 *h = reinterpret_cast<__half2 *>(p) + 2 * i;
        h[0] = __halves2half2(__float2half(v.x), __float2half(v.y));
        h[1] = __halves2half2(__float2half(v.z), __float2half(v.w));
    }
}

// ---------------------------------------------------------------- ray sources

// Thin-lens ray k of pixel q = y w + x of a w x h grid: the pixel's point on
// the focus plane (view depth d), a lens point from the counter hash of
// (seed, frame, q, k), the normalised direction between them.
// The pixel's point on the focus plane.
__device__ inline void focus_point(const FrameConst &fc, uint32_t q, uint32_t w, uint32_t h, float pf[3])
{
    const int x = (int)(q % w), y = (int)(q / w);
    float fv[3];
    pixel_dir(fc.cur, x, y, (int)w, (int)h, fv);
#pragma unroll
    for (int a = 0; a < 3; ++a) pf[a] = fc.cur.pos[a] + fv[a] * fc.d;
}

// The ray from lens point (lx, ly) through the focus-plane point pf.
__device__ inline void lens_through(const FrameConst &fc, const float pf[3], float lx, float ly, float o[3], float d[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) o[a] = fc.cur.pos[a] + fc.half_a * (lx * fc.cur.right[a] + ly * fc.cur.up[a]);
#pragma unroll
    for (int a = 0; a < 3; ++a) d[a] = pf[a] - o[a];
    float len = sqrtf((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]);
#pragma unroll
    for (int a = 0; a < 3; ++a) d[a] = d[a] / len;
}

__device__ inline void thin_lens_ray(const FrameConst &fc, uint32_t q, uint32_t w, uint32_t h, uint32_t k, float o[3],
                                     float d[3])
{
    float pf[3];
    focus_point(fc, q, w, h, pf);
    float lx, ly;
    lens_point(fc.ap, fc.seed, fc.frame, q, k, lx, ly);
    lens_through(fc, pf, lx, ly, o, d);
}

// Thin-lens ray r of a frame: its pixel from the ray -> pixel map, traced at
// half resolution.
__device__ inline void lens_ray(const FrameConst &fc, const uint32_t *queue, const uint32_t *ray_base,
                                const uint32_t *ray_pix, uint32_t r, float o[3], float d[3])
{
    const uint32_t j = ray_pix[r];
    thin_lens_ray(fc, queue[j], (uint32_t)fc.hw, (uint32_t)fc.hh, r - ray_base[j], o, d);
}

// Hit id, distance, shaded colour with view depth and hit position of a lens
// ray whose traversal left (leaf, t) (sky colour and +inf depth on a miss, for
// which data may be any leaf's).
__device__ inline void lens_shade(const LeafData &data, const FrameConst &fc, const float o[3], const float d[3],
                                  uint2 lt, int32_t &hit, float &t, float4 &col, float4 &pos)
{
    if (lt.x != ~0u) {
        t = __uint_as_float(lt.y);
        float P0 = o[0] + t * d[0], P1 = o[1] + t * d[1], P2 = o[2] + t * d[2];
        float z = ((P0 - fc.cur.pos[0]) * fc.cur.fwd[0] + (P1 - fc.cur.pos[1]) * fc.cur.fwd[1]) +
                  (P2 - fc.cur.pos[2]) * fc.cur.fwd[2];
        Shaded s = dof::shade(data, fc.shade, d);
        hit = (int32_t)__float_as_uint(data.v0.w);
        col = make_float4(s.r, s.g, s.b, z);
        pos = make_float4(P0, P1, P2, 0.0f);
    } else {
        hit = -1;
        t = INFINITY;
        col = make_float4(fc.shade.sky[0], fc.shade.sky[1], fc.shade.sky[2], INFINITY);
        pos = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
}

// A ray record is its origin and direction (24 B: a float4 and a float2
// plane); the traversal derives the watertight shear and the reciprocals when
// a lane takes the ray (six correctly rounded divides, shared by the lanes a
// refill starts), which costs less than moving them through memory.
__device__ inline void put_ray(float4 *rec0, float2 *rec1, uint32_t r, const float o[3], const float d[3])
{
    rec0[r] = make_float4(o[0], o[1], o[2], d[0]);
    rec1[r] = make_float2(d[1], d[2]);
}

__device__ inline void get_ray(const float4 *rec0, const float2 *rec1, uint32_t r, float o[3], float d[3])
{
    const float4 a = rec0[r];
    const float2 b = rec1[r];
    o[0] = a.x; o[1] = a.y; o[2] = a.z;
    d[0] = a.w; d[1] = b.x; d[2] = b.y;
}

// The traversal's result of a lens ray: leaf of the closest hit (~0u: none)
// and distance, one 8-byte store; the resolve expands it when it shades.
__device__ inline void put_lt(uint2 *lt, uint32_t r, const Hit &h)
{
    lt[r] = make_uint2(h.id == ~0u ? ~0u : h.leaf, __float_as_uint(h.t));
}

struct LensRays {
    static constexpr bool kPerLaneScene = false, kStats = true, kCoherent = true;
    const float4 *rec0;
    const float2 *rec1;
    uint2 *ray_lt;

    __device__ void ray(uint32_t r, float o[3], float d[3]) const { get_ray(rec0, rec1, r, o, d); }

    __device__ void finish(uint32_t r, const Hit &h) const { put_lt(ray_lt, r, h); }
};

// Lens rays of all frames of a batch: ray r belongs to the last job whose
// first ray is at or before r (found in an LDS copy of the jobs' first rays);
// each lane remembers its ray's job and traces against that job's scene.
struct BatchRays {
    static constexpr bool kPerLaneScene = true, kStats = true, kCoherent = true;
    const Job *jobs;
    const BatchHead *head;
    int njobs;

    __device__ static uint32_t *offsets()
    {
        __shared__ uint32_t off[kMaxBatch + 1];
        return off;
    }

    __device__ void init() const
    {
        uint32_t *off = offsets();
        for (int j = threadIdx.x; j <= njobs; j += blockDim.x) off[j] = head->ray_off[j];
        __syncthreads();
    }

    __device__ int job_of(uint32_t r) const
    {
        const uint32_t *off = offsets();
        int lo = 0, hi = njobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (off[mid] <= r) lo = mid;
            else hi = mid - 1;
        }
        return lo;
    }

    __device__ SceneArgs scene(int j) const { return jobs[j].scene; }

    __device__ void ray(uint32_t r, int j, float o[3], float d[3]) const
    {
        const Job &J = jobs[j];
        get_ray(J.P.rec0, J.P.rec1, r - offsets()[j], o, d);
    }

    __device__ void finish(uint32_t r, int j, const Hit &h) const
    {
        put_lt(jobs[j].P.ray_lt, r - offsets()[j], h);
    }
};

// A pinhole ray leaves its hit's leaf and distance in the pixel's own outputs
// (the first word of its normal, its depth); k_gbuffer_shade turns them into
// the G-buffer, so no lane of the traversal waits on scene loads for shading.
struct PinholeRays {
    static constexpr bool kPerLaneScene = false, kStats = false, kCoherent = true;
    ViewConst view;
    int32_t W, H;
    float *depth;
    uint32_t *normal;
    uint32_t stride;   // words per pixel of the normal image

    __device__ void ray(uint32_t p, float o[3], float d[3]) const
    {
        const int x = (int)(p % (uint32_t)W), y = (int)(p / (uint32_t)W);
        float fv[3];
        pixel_dir(view, x, y, W, H, fv);
        float len = sqrtf((fv[0] * fv[0] + fv[1] * fv[1]) + fv[2] * fv[2]);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            d[a] = fv[a] / len;
            o[a] = view.pos[a];
        }
    }

    __device__ void finish(uint32_t p, const Hit &h) const
    {
        depth[p] = h.t;
        normal[(size_t)p * stride] = h.id == ~0u ? ~0u : h.leaf;
    }
};

__global__ __launch_bounds__(256) void k_gbuffer_shade(SceneArgs S, SceneShade sh, PinholeRays src, void *colour, int cfmt,
                                                       int nfmt, uint32_t npx)
{
    const uint32_t p = blockIdx.x * 256u + threadIdx.x;
    if (p >= npx) return;
    const float t = src.depth[p];
    if (t < INFINITY) {
        // a caller may hand in one piece of memory for the two images it does
        // not want: the leaf's bound keeps the reads inside the scene then
        const uint32_t leaf = min(src.normal[(size_t)p * src.stride], (uint32_t)S.nleaf - 1u);
        float o[3], d[3];
        src.ray(p, o, d);
        const ViewConst &v = src.view;
        const float P0 = o[0] + t * d[0], P1 = o[1] + t * d[1], P2 = o[2] + t * d[2];
        const Shaded s = dof::shade(load_leaf(S, leaf), sh, d);
        st_rgba(colour, cfmt, p, make_float4(s.r, s.g, s.b, 1.0f));
        src.depth[p] = ((P0 - v.pos[0]) * v.fwd[0] + (P1 - v.pos[1]) * v.fwd[1]) + (P2 - v.pos[2]) * v.fwd[2];
        st_rgba(src.normal, nfmt, p, make_float4(s.n0, s.n1, s.n2, 0.0f));
    } else {   // the depth holds the miss's infinite distance
        st_rgba(colour, cfmt, p, make_float4(sh.sky[0], sh.sky[1], sh.sky[2], 1.0f));
        st_rgba(src.normal, nfmt, p, make_float4(0.0f, 0.0f, 0.0f, 0.0f));
    }
}

struct RawRays {
    static constexpr bool kPerLaneScene = false, kStats = false, kCoherent = false;
    const float *org, *dir;
    int32_t *hit;
    float *t;

    __device__ void ray(uint32_t i, float o[3], float d[3]) const
    {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            o[a] = org[3 * (size_t)i + a];
            d[a] = dir[3 * (size_t)i + a];
        }
    }

    __device__ void finish(uint32_t i, const Hit &h) const
    {
        hit[i] = h.id == ~0u ? -1 : (int32_t)h.id;
        t[i] = h.t;
    }
};

// The fully ray-traced image (ground truth of the accuracy judge): ray r of
// a chunk is sample k = r mod spp of full-res pixel p0 + r / spp, traced at
// full resolution with the frame's lens; its (leaf, t) result goes to lt[r].
struct RefRays {
    static constexpr bool kPerLaneScene = false, kStats = false, kCoherent = true;
    FrameConst fc;
    uint32_t p0, spp;
    uint2 *lt;

    __device__ void ray(uint32_t r, float o[3], float d[3]) const
    {
        thin_lens_ray(fc, p0 + r / spp, (uint32_t)fc.W, (uint32_t)fc.H, r % spp, o, d);
    }

    __device__ void finish(uint32_t r, const Hit &h) const { put_lt(lt, r, h); }
};

// Mean shaded colour of each pixel's spp rays of a chunk (binary64 sum in
// sample order, one rounding to binary32).
__global__ __launch_bounds__(256) void k_ref_average(SceneArgs S, RefRays src, uint32_t npx, void *colour, int cfmt)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= npx) return;
    double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0;
    for (uint32_t k = 0; k < src.spp; ++k) {
        const uint32_t r = i * src.spp + k;
        float o[3], d[3];
        src.ray(r, o, d);
        const uint2 lt = src.lt[r];
        int32_t hi;
        float t;
        float4 c, p;
        lens_shade(load_leaf(S, lt.x != ~0u ? lt.x : 0u), src.fc, o, d, lt, hi, t, c, p);
        acc0 += (double)c.x;
        acc1 += (double)c.y;
        acc2 += (double)c.z;
    }
    const double n = (double)src.spp;
    st_rgba(colour, cfmt, (size_t)src.p0 + i, make_float4((float)(acc0 / n), (float)(acc1 / n), (float)(acc2 / n), 1.0f));
}

// ---------------------------------------------------------------- ray generation

constexpr int kGenTB = 256;
constexpr int kGenMaxBlocks = 2048;

// Every thin-lens ray of a frame (the count is the compaction's ray total).
__global__ __launch_bounds__(kGenTB) void k_raygen(FrameConst fc, const uint32_t *queue, const uint32_t *ray_base,
                                                   const uint32_t *ray_pix, const uint32_t *count, float4 *rec0,
                                                   float2 *rec1)
{
    const uint32_t N = *count;
    for (uint32_t r = blockIdx.x * kGenTB + threadIdx.x; r < N; r += gridDim.x * kGenTB) {
        float o[3], d[3];
        lens_ray(fc, queue, ray_base, ray_pix, r, o, d);
        put_ray(rec0, rec1, r, o, d);
    }
}

// The same for a bladed aperture, whose lens points take more tries
// (rejection from the square keeps 65 % of them for a hexagon against 79 %
// for a circle).  A wave walks runs of up to kGenSpan rays (shorter when the
// frame has few rays, so every wave gets some); each ray first gets
// kGenFirst tries, the rays still without a point wait in a per-wave LDS
// list, and the wave then runs the remaining tries for them one per lane, so
// it does not spin for its unluckiest lane while the others idle.  Every ray
// gets the same tries in the same order as one lens_point call.
constexpr int kGenSpan = 512;
constexpr uint32_t kGenFirst = 2;

__global__ __launch_bounds__(kGenTB) void k_raygen_bladed(FrameConst fc, const uint32_t *queue,
                                                          const uint32_t *ray_base, const uint32_t *ray_pix,
                                                          const uint32_t *count, float4 *rec0, float2 *rec1)
{
    __shared__ uint32_t left[kGenTB / 64][kGenSpan];
    const uint32_t N = *count;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const uint32_t nwaves = gridDim.x * (kGenTB / 64);
    const uint32_t hw = (uint32_t)fc.hw, hh = (uint32_t)fc.hh;
    uint32_t span = ((N / nwaves + 1u) + 63u) & ~63u;
    span = span < (uint32_t)kGenSpan ? span : (uint32_t)kGenSpan;
    for (uint32_t base = (blockIdx.x * (kGenTB / 64) + w) * span; base < N; base += nwaves * span) {
        const uint32_t end = N - base < span ? N : base + span;
        uint32_t nleft = 0;   // wave-uniform
        for (uint32_t r0 = base; r0 < end; r0 += 64) {
            const uint32_t r = r0 + (uint32_t)lane;
            bool miss = false;
            if (r < end) {
                const uint32_t j = ray_pix[r], q = queue[j], k = r - ray_base[j];
                const uint32_t hs = lens_seed(fc.seed, fc.frame, q);
                float lx = 0.0f, ly = 0.0f;
                bool ok = false;
                for (uint32_t att = 0; att < kGenFirst && !ok; ++att) ok = lens_try(fc.ap, hs, k, att, lx, ly);
                if (ok) {
                    float pf[3], o[3], d[3];
                    focus_point(fc, q, hw, hh, pf);
                    lens_through(fc, pf, lx, ly, o, d);
                    put_ray(rec0, rec1, r, o, d);
                } else {
                    miss = true;
                }
            }
            const uint64_t m = __ballot(miss);
            if (miss) left[w][nleft + (uint32_t)__popcll(m & lt)] = r;
            nleft += (uint32_t)__popcll(m);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (uint32_t t = (uint32_t)lane; t < nleft; t += 64) {
            const uint32_t r = left[w][t];
            const uint32_t j = ray_pix[r], q = queue[j], k = r - ray_base[j];
            float lx, ly, pf[3], o[3], d[3];
            lens_point_from(fc.ap, lens_seed(fc.seed, fc.frame, q), k, kGenFirst, lx, ly);
            focus_point(fc, q, hw, hh, pf);
            lens_through(fc, pf, lx, ly, o, d);
            put_ray(rec0, rec1, r, o, d);
        }
        __builtin_amdgcn_wave_barrier();   // the list is rewritten by the next run
    }
}

__global__ __launch_bounds__(kGenTB) void kb_raygen(const Job *__restrict__ jobs, const BatchHead *head, int njobs)
{
    __shared__ uint32_t off[kMaxBatch + 1];
    for (int j = threadIdx.x; j <= njobs; j += kGenTB) off[j] = head->ray_off[j];
    __syncthreads();
    const uint32_t N = head->rays;
    for (uint32_t r = blockIdx.x * kGenTB + threadIdx.x; r < N; r += gridDim.x * kGenTB) {
        int lo = 0, hi = njobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (off[mid] <= r) lo = mid;
            else hi = mid - 1;
        }
        const Job &J = jobs[lo];
        const uint32_t k = r - off[lo];
        float o[3], d[3];
        lens_ray(J.fc, J.P.queue, J.P.ray_base, J.P.ray_pix, k, o, d);
        put_ray(J.P.rec0, J.P.rec1, k, o, d);
    }
}

// The compaction and the ray generation of a small frame in one launch: one
// block per 256 pixels in row-major order, whose first queue position and ray
// are the sums over the mask before them.  Ranks come from wave ballots (masked
// pixels) and wave prefix sums (rays), so the queue is ascending and the
// block's rays are one contiguous range, which it then generates itself, a map
// from ray to pixel kept in LDS.  A small frame's time is its launches': 7 us
// instead of the three kernels' 13 and two gaps.  256x256 113 -> 109 us a
// frame, 640x480 144 -> 137, 800x600 159 -> 154; the sums over the mask grow
// with the square of the frame, and at 960x960 (230400 half-res pixels) it is
// 218 -> 220: hence kSmallFrame.  compact_in_one says which frames take it.
constexpr int kSmallRays = 4096;   // rays of a window (16 per pixel)

__global__ __launch_bounds__(kGenTB) void k_compact_small(FrameConst fc, Planes P, const uint8_t *__restrict__ mask)
{
    __shared__ uint32_t wp[4], wr[4];
    __shared__ uint8_t s_pix[kSmallRays];   // ray of the window -> pixel of the block
    __shared__ uint32_t s_base[kGenTB];     // pixel of the block -> its first ray
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t hw = (uint32_t)fc.hw, hh = (uint32_t)fc.hh, np = hw * hh, q0 = blockIdx.x * kGenTB, q = q0 + (uint32_t)tid;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    // the traversal's counters start the frame at zero
    if (blockIdx.x == 0 && tid < kWorkParts) {
        uint32_t *c = P.counters + kCntWork + tid * kWorkStride;
        c[0] = 0u;
        for (int k = 0; k < kStatWords; ++k) c[kStatAt + k] = 0u;
        if (tid == 0) P.counters[kCntWild] = 0u;
    }
    const uint32_t n = q < np ? mask[q] : 0u;
    uint32_t before = 0, rays_before = 0;   // four pixels a word: the launch has shown the mask aligned
    const uint32_t *words = reinterpret_cast<const uint32_t *>(mask);
#pragma unroll 8
    for (uint32_t i = (uint32_t)tid; i < q0 / 4; i += kGenTB) {
        const uint32_t v = words[i];
        before += (uint32_t)__popc((((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u);
        rays_before = __builtin_amdgcn_sad_u8(v, 0u, rays_before);
    }
    for (int o = 32; o >= 1; o >>= 1) {
        before += __shfl_xor(before, o);
        rays_before += __shfl_xor(rays_before, o);
    }
    const uint64_t bal = __ballot(n > 0u);
    uint32_t incl = n;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    __shared__ uint32_t bp[4], br[4];
    if (lane == 63) {
        wp[w] = (uint32_t)__popcll(bal);
        wr[w] = incl;
        bp[w] = before;
        br[w] = rays_before;
    }
    __syncthreads();
    const uint32_t p0 = bp[0] + bp[1] + bp[2] + bp[3], r0 = br[0] + br[1] + br[2] + br[3];
    const uint32_t rays = wr[0] + wr[1] + wr[2] + wr[3];
    uint32_t pos = p0 + (uint32_t)__popcll(bal & lt), first = r0 + incl - n;
    for (int k = 0; k < w; ++k) { pos += wp[k]; first += wr[k]; }
    if (n > 0u) {
        P.queue[pos] = q;
        P.ray_base[pos] = first;
    }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) {
        P.counters[kCntMasked] = p0 + wp[0] + wp[1] + wp[2] + wp[3];
        P.counters[kCntRays] = r0 + rays;
    }
    s_base[tid] = first;
    for (uint32_t w0 = 0; w0 < rays; w0 += kSmallRays) {   // block-uniform
        const uint32_t wn = rays - w0 < (uint32_t)kSmallRays ? rays - w0 : (uint32_t)kSmallRays;
        const uint32_t k0 = first - r0;   // the pixel's rays within the window
        for (uint32_t k = k0 > w0 ? k0 : w0; k < k0 + n && k < w0 + wn; ++k) s_pix[k - w0] = (uint8_t)tid;
        __syncthreads();
        for (uint32_t t = (uint32_t)tid; t < wn; t += kGenTB) {
            const uint32_t px = s_pix[t], ray = r0 + w0 + t;
            float o[3], d[3];
            thin_lens_ray(fc, q0 + px, hw, hh, ray - s_base[px], o, d);
            put_ray(P.rec0, P.rec1, ray, o, d);
        }
        __syncthreads();   // the window's map is rewritten
    }
}

// Shading and resolve of a frame's lens rays in one pass: each block shades
// the rays of its 64 pixels straight into the resolve's LDS chunks (and, when
// the frame keeps them, into the per-ray planes), so nothing is read back.
// Bound by the latency of two loads that depend on each other, a ray's record
// and then its triangle, so a lane has kShadeRays rays in flight: at 3840x2160,
// beside the gather, 218 us a frame with one and 166 with two (four hold more
// registers and slow the gather's blocks down by as much).
constexpr int kShadeRays = 2;

__device__ inline void shade_resolve_block(const SceneArgs &S, const FrameConst &fc, const Planes &P,
                                           const uint8_t *__restrict__ mask, uint32_t bx)
{
    resolve_block(fc, P, mask, bx, [&](uint32_t c0, uint32_t c1, float4 *col, float4 *pos) {
        for (uint32_t b0 = c0 + threadIdx.x; b0 < c1; b0 += 64 * kShadeRays) {
            // a ray past the end repeats the last one
            uint2 lt[kShadeRays];
            float o[kShadeRays][3], d[kShadeRays][3];
            LeafData data[kShadeRays];
#pragma unroll
            for (int u = 0; u < kShadeRays; ++u) {
                const uint32_t r = min(b0 + 64u * u, c1 - 1u);
                lt[u] = P.ray_lt[r];
                get_ray(P.rec0, P.rec1, r, o[u], d[u]);
            }
#pragma unroll
            for (int u = 0; u < kShadeRays; ++u) data[u] = load_leaf(S, lt[u].x != ~0u ? lt[u].x : 0u);
#pragma unroll
            for (int u = 0; u < kShadeRays; ++u) {
                const uint32_t r = b0 + 64u * u;
                if (r >= c1) break;
                int32_t hi;
                float t;
                float4 c, p;
                lens_shade(data[u], fc, o[u], d[u], lt[u], hi, t, c, p);
                if (P.ray_hit) {   // per-ray planes kept for inspection (params.ray_records)
                    P.ray_hit[r] = hi;
                    P.ray_t[r] = t;
                    P.ray_col[r] = c;
                    P.ray_pos[r] = p;
                }
                p.w = hi >= 0 ? sat(0.5f + (fc.d - c.w) / fc.ramp) : -1.0f;
                c.w = coc_px(fc.cock, fc.d, c.w);
                col[r - c0] = c;
                pos[r - c0] = p;
            }
        }
    });
}

__global__ __launch_bounds__(64) void k_shade_resolve(SceneArgs S, FrameConst fc, Planes P,
                                                      const uint8_t *__restrict__ mask)
{
    shade_resolve_block(S, fc, P, mask, blockIdx.x);
}

__global__ __launch_bounds__(64) void kb_shade_resolve(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridResolve, blockIdx.x, bx, by)];
    shade_resolve_block(J.scene, J.fc, J.P, J.mask, bx);
}

int gen_blocks(int64_t max_rays)
{
    const int64_t b = (max_rays + kGenTB - 1) / kGenTB;
    return b < 1 ? 1 : (b > kGenMaxBlocks ? kGenMaxBlocks : (int)b);
}

// ---------------------------------------------------------------- persistent traversal

constexpr int kShareRows = 6;    // LDS stack rows that the work sharing's state takes
constexpr int kShareLanes = 32;  // busy lanes at which a wave without further rays starts to share
constexpr int kShareSteps = 4;   // most node visits per lane between two shares
// Visits between two shares: kShareSteps while at least kShareBusy lanes have
// work and the rays run side by side (Src::kCoherent), so that the few idle
// lanes cost less than the sharing: a 1920x1080 frame 434 -> 424 us, a 256x256
// view 31.7 -> 31.1.  Else 2: random rays' lengths differ more, and with four
// visits a million of them take 388 us instead of 377; four in every case take
// 22 us for a thousand instead of 20.
constexpr int kShareBusy = 48;
// Rays per wave below which a small launch uses fewer waves: the waves of a
// SIMD share its issue slots, and work sharing spreads a wave's rays over its
// lanes.  With 4 a wave 1000 random rays take 19.5 us (8: 20.4, 16: 21.6), a
// 256x256 frame 95 (3: 99, 8: 94), a 224x218 one among 319000 triangles 150
// (8: 153, 16: 177), a 256x256 view 30.6 (3: 31.3, 16: 30.4).
constexpr int kMinRays = 4;
constexpr int kDropChunk = 8;    // oldest stack entries dropped when the LDS stack is full
// Launch knobs (TraceKnobs, defaults in brackets): a wave refills when at
// least tk.refill lanes are idle [16], takes tk.grab rays from the work
// counters at a time [64], and runs its triangle tests when at least
// tk.leaf_batch lanes have one pending [32]; kStack LDS stack entries per
// lane [24]; kSteps node visits per lane per iteration [4]; tk.reverse
// hands the rays out from the end of the queue [for
// frames; the scene-level sources keep the queue order].  The last rays a
// persistent grid hands out set its tail: when they are cheap, every wave
// finishes at nearly the same time.

// Orders a wave's own LDS accesses (they execute in order; this keeps the
// compiler from moving or caching them).
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

typedef __attribute__((address_space(3))) uint32_t LdsWord;

__device__ inline LdsWord *lds_word(uint32_t address) { return (LdsWord *)(uintptr_t)address; }

// A lane mask as each lane's predicate.
__device__ inline bool lanes(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// work: slot 0 of the work-counter slots; stats and drops_out (or null):
// slot 0's node-visit and stack-drop statistics, a wave adding its totals to
// the slot of its block (b mod kWorkParts) when it finishes.
// What bounds it: at 3840x2160 the L1's lookups (0.9 a cycle and CU, the
// texture data unit busy 0.95 of the time); at 1920x1080, with 2.4 rays per
// lane, also the waves' uneven ends.  A visit takes about 50 vector
// instructions, where predicates kept as booleans in registers, index
// arithmetic for the stack and 64-bit node addresses made it 74: gathered over
// the launch 763 M instead of 949 M vector instructions at 4K, the traversal
// 1358 -> 1215 us there and 349 -> 240 us at 1080p (with the work sharing).
// Occupancy: 70 VGPRs a lane would let seven waves share a SIMD; the 24-entry
// stack's LDS allows six (12.5 KB a block), the 16-entry one's seven.  A
// batch's lanes also hold their scene's pointers; asking for six waves (80
// VGPRs) makes a 32-session batch 3.6 % faster.
// kFar: the nodes' byte offsets need more than 32 bits (kMaxNear leaves)
template <class Src, int kStack, int kSteps, bool kFar>
__global__ __launch_bounds__(kTB) __attribute__((amdgpu_waves_per_eu(Src::kPerLaneScene ? (kStack == 32 ? 1 : 6) : (kStack == 16 ? 7 : 1))))
void k_traverse(SceneArgs S, Src src, uint32_t count, const uint32_t *count_ptr,
                                                  uint32_t *work, unsigned long long *stats, uint32_t *drops_out,
                                                  TraceKnobs tk)
{
    constexpr uint32_t kRow = kTB * sizeof(uint32_t);   // bytes from one stack row to the next
    // The stack's fullness is looked at once per iteration, before its kSteps
    // visits push at most one entry each: entries are dropped above kRows -
    // kSteps.  The small stack gets rows for those pushes on top (20 rows and
    // seven waves still fit the LDS); with 12 entries a 1080p frame dropped so
    // often that it took 797 instead of 508 us.
    constexpr int kRows = kStack == 16 ? kStack + kSteps : kStack;
    // row 0 stays unused: an empty stack's top; the work sharing keeps 64-bit
    // words in two of the rows
    __shared__ alignas(16) uint32_t lds_stack[(kRows + 1) * kTB];
    const uint32_t grab = tk.grab;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t N = count_ptr ? *count_ptr : count;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    // LDS byte addresses: the lane's row 0 and its newest stack entry
    const uint32_t stk = (uint32_t)(uintptr_t)(LdsWord *)(lds_stack + tid);
    uint32_t top = stk;

    // rays [pool, pool_end) taken by this wave and not yet handed to a lane
    // (wave-uniform); a new batch of `grab` comes from the work counters only
    // when the pool is empty, so refills rarely touch an atomic
    uint32_t pool = 0, pool_end = 0;
    bool drained = false;   // the wave's work counter has passed N (wave-uniform)
    uint32_t item = 0, node = 0;
    WRay wr;
    Hit h;
    uint32_t visits = 0, tests = 0;
    // leaf hits of this lane not yet tested (tested when enough lanes have some)
    uint32_t q0 = 0, q1 = 0, q2 = 0, q3 = 0;
    // The lane's state in one word, so that "may visit a node" is one
    // comparison (state <= 2): how many leaf hits wait, + kNoNode when it has
    // no inner node left to visit, kNoRay when it has no ray.
    constexpr uint32_t kNoNode = 8, kNoRay = 16;
    uint32_t state = kNoRay;
    SceneArgs Sl = S;    // scene of the lane's ray (differs per lane in a batch)
    int job = 0;         // job of the lane's ray (batches)
    if constexpr (Src::kPerLaneScene) src.init();

    // One node visit: both children's slab tests, leaf hits to the queue, the
    // next node.  The lane's stack runs from the row after `bottom` to `top`
    // and has room for one more.  Written for few vector instructions, which
    // bound the kernel: predicates are lane masks combined on the scalar unit,
    // a push and a pop are each one masked add and one LDS access, and the
    // second leaf of a node with two leaf hits is queued behind a branch that
    // most waves skip.
    auto visit = [&](float limit, uint32_t bottom) __attribute__((always_inline)) {
        BvhNode16 nd;
        if constexpr (Src::kPerLaneScene || kFar) nd = Sl.nodes[node];
        else nd = *reinterpret_cast<const BvhNode16 *>(reinterpret_cast<const char *>(Sl.nodes) + (node << 5));
        if constexpr (Src::kStats) ++visits;
        float tl, tr;
        bool hl, hr;
        node_hits(wr, nd, limit, hl, hr, tl, tr);
        const uint32_t L = nd.b.z, R = nd.b.w;
        const uint64_t mhl = __ballot(hl), mhr = __ballot(hr);
        const uint64_t mll = __ballot((int32_t)L < 0), mlr = __ballot((int32_t)R < 0);
        const uint64_t mpl = mhl & mll, mpr = mhr & mlr, mil = mhl & ~mll, mir = mhr & ~mlr;
        // a leaf hit goes to the front of the queue (shift in)
        const bool pl = lanes(mpl), pa = lanes(mpl | mpr);
        q3 = pa ? q2 : q3; q2 = pa ? q1 : q2; q1 = pa ? q0 : q1; q0 = pa ? (pl ? L : R) : q0;
        state += pa ? 1u : 0u;
        if ((mpl & mpr) != 0ull) {
            const bool two = lanes(mpl & mpr);
            q3 = two ? q2 : q3; q2 = two ? q1 : q2; q1 = two ? q0 : q1; q0 = two ? R : q0;
            state += two ? 1u : 0u;
        }
        // next node: the near child when both are hit (the far one pushed),
        // else the one hit child, else the stack top; a lane with none of
        // these ends on its last node's right child
        const bool left = lanes(mil & (__ballot(tl <= tr) | ~mir));
        uint32_t next = left ? L : R, t = top;
        if (lanes(mil & mir)) {
            t += kRow;
            *lds_word(t) = left ? R : L;
        }
        const uint64_t none = ~(mil | mir) & __ballot(true), pop = none & __ballot(t != bottom);
        if (lanes(pop)) {
            next = *lds_word(t);
            t -= kRow;
        }
        node = next;
        top = t;
        state += lanes(none & ~pop) ? kNoNode : 0u;
    };
    // The oldest kDropChunk entries of a lane's stack go.
    auto drop = [&]() __attribute__((always_inline)) {
        for (uint32_t a = stk + kRow; a + kDropChunk * kRow <= top; a += kRow) *lds_word(a) = *lds_word(a + kDropChunk * kRow);
        top -= kDropChunk * kRow;
        wr.swx |= kDropped;
        if (Src::kStats && drops_out) atomicAdd(drops_out + (blockIdx.x % kWorkParts) * kWorkStride, 1u);
    };
    // A lane whose stack ran empty after a drop: up from its finished subtree
    // to the nearest ancestor whose far child is still pending.
    auto walk = [&](float limit) __attribute__((always_inline)) {
        uint32_t c = Sl.parent[(node & kLeaf) ? (size_t)(Sl.nleaf - 1) + (node & ~kLeaf) : (size_t)node];
        wr.swx &= ~kDropped;
        for (uint32_t a = Sl.parent[c]; a != ~0u; c = a, a = Sl.parent[a]) {
            const BvhNode16 pn = Sl.nodes[a];
            if constexpr (Src::kStats) ++visits;
            float ta, tb;
            bool ha, hb;
            node_hits(wr, pn, limit, ha, hb, ta, tb);
            const bool from_left = pn.b.z == c;
            const uint32_t other = from_left ? pn.b.w : pn.b.z;
            const bool came_near = from_left ? ta <= tb : !(ta <= tb);
            if (came_near && (other & kLeaf) == 0u && (from_left ? hb : ha)) {
                node = other;
                state -= kNoNode;
                wr.swx |= kDropped;
                break;
            }
        }
    };

    // A launch with no more rays than lanes deals them evenly over its waves,
    // without counters, and leaves waves idle rather than give each fewer than
    // so many.  A larger one gives every wave a first run and hands
    // out the others through the counters: run g of those is the k-th of
    // counter g mod parts, and a wave whose counter is past the last run takes
    // no more.  Takes are few because they are dear, one address taking an
    // atomic after the other: with the first runs taken too, and each wave
    // looking through all eight counters before it gave up, a 1920x1080 view
    // took 457 us instead of 421, a million rays 408 instead of 377.
    const uint32_t wave = blockIdx.x * (kTB / 64) + (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6), waves = gridDim.x * (kTB / 64);
    const uint32_t parts = min((uint32_t)kWorkParts, gridDim.x), part = blockIdx.x % parts;
    if (N <= gridDim.x * (uint32_t)kTB) {
        const uint32_t used = max(1u, min(waves, N / (uint32_t)kMinRays));
        pool = wave < used ? (uint32_t)((uint64_t)N * wave / used) : N;
        pool_end = wave < used ? (uint32_t)((uint64_t)N * (wave + 1) / used) : N;
        drained = true;
    } else {
        const uint64_t b = (uint64_t)wave * grab;
        pool = b < N ? (uint32_t)b : N;
        pool_end = N - pool < grab ? N : pool + grab;
    }
    // The wave's next rays, one a lane: rays [first, ready) of the pool.  All
    // lanes fetch (or make) 64 at once and a refill's lanes take theirs by
    // shuffle, instead of each refill waiting for its own with a quarter of
    // the lanes at work: 3840x2160 2246 -> 2193 us, the fully traced
    // 1280x720 image, whose rays are sampled here, 2484 -> 2425.  A batch's
    // lanes have no registers left for it.
    float po[3] = {0.0f, 0.0f, 0.0f}, pd[3] = {0.0f, 0.0f, 0.0f};
    uint32_t first = pool, ready = pool;
    while (true) {
        const uint64_t idle = __ballot(state >= kNoRay);
        if (!(drained && pool == pool_end) && (__popcll(idle) >= tk.refill || idle == ~0ull) && idle != 0ull) {
            if (pool == pool_end) {
                uint32_t base = N;
                if (lane == 0) {
                    const uint64_t k = atomicAdd(work + part * kWorkStride, 1u), b = (waves + k * parts + part) * grab;
                    base = b < N ? (uint32_t)b : N;
                }
                base = __builtin_amdgcn_readfirstlane(base);
                if (base >= N) {
                    drained = true;
                } else {
                    pool = base;
                    pool_end = N - base < grab ? N : base + grab;
                    ready = pool;
                }
            }
            if (!Src::kPerLaneScene && pool == ready && pool != pool_end) {
                first = pool;
                ready = pool_end - pool < 64u ? pool_end : pool + 64u;
                const uint32_t r = min(first + (uint32_t)lane, ready - 1u);
                if constexpr (!Src::kPerLaneScene) src.ray(tk.reverse ? N - 1u - r : r, po, pd);
            }
            const uint32_t avail = (Src::kPerLaneScene ? pool_end : ready) - pool;
            const uint32_t rank = (uint32_t)__popcll(idle & lt);
            float so[3], sd[3];
            if constexpr (!Src::kPerLaneScene) {
                const int from = (int)(pool + rank - first);   // below 64 where a ray is taken
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    so[a] = __shfl(po[a], from);
                    sd[a] = __shfl(pd[a], from);
                }
            }
            if (state >= kNoRay && rank < avail) {
                item = pool + rank;
                if (tk.reverse) item = N - 1u - item;   // pool + rank < N
                if constexpr (Src::kPerLaneScene) {
                    float o[3], d[3];
                    job = src.job_of(item);
                    Sl = src.scene(job);
                    src.ray(item, job, o, d);
                    wr = make_wray(o, d);
                } else {
                    wr = make_wray(so, sd);
                }
                h = Hit{INFINITY, ~0u, 0u};
                node = 0;
                top = stk;
                state = 0;
                if (Sl.nleaf == 1) {   // the only leaf
                    state = kNoNode + 1;
                    q0 = 0u;
                }
            }
            const uint32_t nidle = (uint32_t)__popcll(idle);
            pool += nidle < avail ? nidle : avail;
        }
        const uint64_t busy = __ballot(state < kNoRay);
        if (drained && pool == pool_end && __popcll(busy) <= (tk.leaf_batch > 1 ? kShareLanes : 0)) break;
        if (busy == 0ull) continue;
        // triangle tests, batched across the wave
        const bool want = (state & 7u) != 0u;
        if (__ballot(want && state >= 3u) != 0ull || __popcll(__ballot(want)) >= tk.leaf_batch) {
            if (want) {
                if constexpr (Src::kStats) ++tests;
                consider_leaf(Sl, wr, q0 & ~kLeaf, h);
                q0 = q1; q1 = q2; q2 = q3;
                --state;
            }
        }
        // prune against the best hit, 2^-10 relative slack
        const float limit = h.t * 1.0009765625f;
        if (top > stk + (kRows - kSteps) * kRow) drop();
#pragma unroll
        for (int step = 0; step < kSteps; ++step)
            if (state <= 2u) visit(limit, stk);
        if (state >= kNoNode && state < kNoRay && (int32_t)wr.swx < 0) walk(limit);
        if (state == kNoNode) {
            if constexpr (Src::kPerLaneScene) src.finish(item, job, h);
            else src.finish(item, h);
            state = kNoRay;
            top = stk;
        }
    }

    // Work sharing: no ray is left to hand out and at most kShareLanes lanes
    // of the wave still have one.  An idle lane takes the oldest stack entry
    // (the largest pending subtree) of a busy one, with its ray, and both go
    // on; a ray's best hit, the lanes at work on it and its hit's leaf live in
    // LDS under the lane that owns it, and the owner finishes the ray when the
    // last of them is through.  The closest hit does not depend on the order
    // of the visits, so neither does any result.  The last rows of the wave's
    // own stack columns hold that state.  A lane that drops entries walks on
    // past the subtree it was given, over work that others do too, and gives
    // none away itself.  With trace_leaf_batch 1 every ray stays with its lane,
    // so that the statistics follow from the rays alone.
    // 1000 rays among 866 triangles took 102 us, a node visit after the other
    // with 64 rays to a wave, and take 20; a 256 x 256 view's rays 103 and 31.
    if (__ballot(state < kNoRay) != 0ull) {
        constexpr int kTop = kRows - kShareRows;   // rows left to the stack
        static_assert(kRows - kDropChunk <= kTop && kDropChunk + kShareSteps <= kTop, "room for the shared state");
        const int wb = tid & ~63;   // the wave's first column
        auto key_of = [&](int l) __attribute__((always_inline)) {
            return reinterpret_cast<unsigned long long *>(lds_stack + (1 + kTop + (l >> 5)) * kTB + wb + 2 * (l & 31));
        };
        uint32_t *s_leaf = lds_stack + (kTop + 3) * kTB + wb, *s_work = lds_stack + (kTop + 4) * kTB + wb;
        uint32_t *s_from = lds_stack + (kTop + 5) * kTB + wb, *s_node = lds_stack + (kTop + 6) * kTB + wb;
        if (top > stk + kTop * kRow) drop();
        wave_sync();
        bool mine = state < kNoRay;   // the lane's own ray is unfinished
        *key_of(lane) = ((unsigned long long)__float_as_uint(h.t) << 32) | h.id;
        s_leaf[lane] = h.leaf;
        s_work[lane] = mine ? 1u : 0u;
        int owner = lane;
        uint32_t bottom = stk;   // the stack's first entry lies above; the rows below it were given away
        wave_sync();
        while (true) {
            const uint64_t live = __ballot(state < kNoRay);
            if (live == 0ull) break;
            const int steps = Src::kCoherent && __popcll(live) >= kShareBusy ? kShareSteps : 2;
            const bool can = state < kNoNode && top != bottom && (int32_t)wr.swx >= 0;
            const uint64_t donors = __ballot(can);
            if (donors != 0ull && live != ~0ull) {
                const int give = __popcll(donors & lt), take = __popcll(~live & lt);
                const int n = min(__popcll(donors), __popcll(~live));
                if (can && give < n) {
                    bottom += kRow;
                    s_from[give] = (uint32_t)lane;
                    s_node[give] = *lds_word(bottom);
                }
                wave_sync();
                const bool taker = state >= kNoRay && take < n;
                const int from = taker ? (int)s_from[take] : lane;
                const uint32_t first = taker ? s_node[take] : node;
                wave_sync();
                wr.o0 = __shfl(wr.o0, from); wr.o1 = __shfl(wr.o1, from); wr.o2 = __shfl(wr.o2, from);
                wr.sx = __shfl(wr.sx, from); wr.sy = __shfl(wr.sy, from); wr.sz = __shfl(wr.sz, from);
                wr.ix = __shfl(wr.ix, from); wr.iy = __shfl(wr.iy, from); wr.iz = __shfl(wr.iz, from);
                wr.cnx = __shfl(wr.cnx, from); wr.cny = __shfl(wr.cny, from); wr.cnz = __shfl(wr.cnz, from);
                wr.cfx = __shfl(wr.cfx, from); wr.cfy = __shfl(wr.cfy, from); wr.cfz = __shfl(wr.cfz, from);
                wr.swx = __shfl(wr.swx, from); wr.swy = __shfl(wr.swy, from); wr.swz = __shfl(wr.swz, from);
                owner = __shfl(owner, from);
                if constexpr (Src::kPerLaneScene) {
                    const int oj = __shfl(job, owner);
                    if (taker) Sl = src.scene(oj);
                }
                if (taker) {
                    node = first;
                    top = stk;
                    bottom = stk;
                    state = 0;
                    atomicAdd(&s_work[owner], 1u);
                }
            }
            const bool want = (state & 7u) != 0u;
            if (__ballot(want && state >= 3u) != 0ull || 2 * __popcll(__ballot(want)) >= __popcll(live)) {
                if (want) {
                    if constexpr (Src::kStats) ++tests;
                    unsigned long long *best = key_of(owner);
                    Hit g{__uint_as_float((uint32_t)(*best >> 32)), (uint32_t)*best, ~0u};
                    consider_leaf(Sl, wr, q0 & ~kLeaf, g);
                    const unsigned long long key = ((unsigned long long)__float_as_uint(g.t) << 32) | g.id;
                    if (g.leaf != ~0u) atomicMin(best, key);
                    wave_sync();
                    // of lanes that improve one ray together, the closest names the leaf
                    if (g.leaf != ~0u && *best == key) s_leaf[owner] = g.leaf;
                    q0 = q1; q1 = q2; q2 = q3;
                    --state;
                }
            }
            wave_sync();
            const float limit = __uint_as_float((uint32_t)(*key_of(owner) >> 32)) * 1.0009765625f;
            // room for the visits' pushes: the stack moves down over the rows
            // given away, and drops entries where those are too few
            const uint32_t most = (uint32_t)(kTop - steps) * kRow;
            if (top > stk + most && bottom != stk) {
                const uint32_t d = bottom - stk;
                for (uint32_t a = stk + kRow; a + d <= top; a += kRow) *lds_word(a) = *lds_word(a + d);
                top -= d;
                bottom = stk;
            }
            if (top > stk + most) drop();
#pragma unroll 1
            for (int step = 0; step < steps; ++step)
                if (state <= 2u) visit(limit, bottom);
            if (state >= kNoNode && state < kNoRay && (int32_t)wr.swx < 0) walk(limit);
            if (state == kNoNode) {
                state = kNoRay;
                atomicSub(&s_work[owner], 1u);
            }
            wave_sync();
            if (mine && s_work[lane] == 0u) {
                const unsigned long long key = *key_of(lane);
                h = Hit{__uint_as_float((uint32_t)(key >> 32)), (uint32_t)key, s_leaf[lane]};
                if constexpr (Src::kPerLaneScene) src.finish(item, job, h);
                else src.finish(item, h);
                mine = false;
            }
        }
    }
    if (Src::kStats && stats) {
        unsigned long long v = visits, t = tests;
        for (int off = 32; off >= 1; off >>= 1) {
            v += __shfl_xor(v, off);
            t += __shfl_xor(t, off);
        }
        if (lane == 0 && (v | t) != 0ull) {   // a scene of one leaf has tests and no nodes
            unsigned long long *slot = stats + (blockIdx.x % kWorkParts) * (kWorkStride / 2);
            atomicAdd(slot, v);
            atomicAdd(slot + 1, t);
        }
    }
}

__global__ void k_zero_work(uint32_t *work)
{
    if ((int)threadIdx.x < kWorkParts) work[threadIdx.x * kWorkStride] = 0u;
}

// First ray of every job of a batch (exclusive prefix of the jobs' ray
// counts), the batch total, and cleared traversal counters.
__global__ __launch_bounds__(64) void kb_ray_offsets(BatchHead *head, const Job *__restrict__ jobs, int njobs)
{
    const int lane = threadIdx.x;
    uint32_t acc = 0;
    for (int j0 = 0; j0 < njobs; j0 += 64) {
        const int j = j0 + lane;
        const uint32_t n = j < njobs ? jobs[j].P.counters[kCntRays] : 0u;
        uint32_t incl = n;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(incl, o);
            if (lane >= o) incl += u;
        }
        if (j < njobs) head->ray_off[j] = acc + incl - n;
        acc += __shfl(incl, 63);
    }
    if (lane < kWorkParts) {
        uint32_t *w = head->work + lane * kWorkStride;
        w[0] = 0u;
        for (int k = 0; k < kStatWords; ++k) w[kStatAt + k] = 0u;
    }
    if (lane == 0) {
        head->ray_off[njobs] = acc;
        head->rays = acc;
        head->visits = 0ull;
        head->tests = 0ull;
    }
}

int clamp_blocks(int blocks) { return blocks < 1 ? 1 : (blocks > kMaxTraceBlocks ? kMaxTraceBlocks : blocks); }

}  // namespace

// The traversal kernel of a ray source for a stack depth and a number of
// node visits per loop iteration: f(kernel).
template <class Src, int kStack, class F>
void with_steps(int steps, F f)
{
    if (steps == 3) f(k_traverse<Src, kStack, 3, false>);
    else f(k_traverse<Src, kStack, 4, false>);
}

// Trees of up to kMaxNear leaves keep a node's byte offset in 32 bits (one
// shift per visit in place of 64-bit address arithmetic); a larger one runs
// the default shape's 64-bit variant.
constexpr int32_t kMaxNear = 1 << 27;

template <class Src, class F>
void with_shape(int stack, int steps, int32_t nleaf, F f)
{
    if (!Src::kPerLaneScene && nleaf > kMaxNear) f(k_traverse<Src, kStackLds, kTraceSteps, !Src::kPerLaneScene>);
    else if (stack == 16) with_steps<Src, 16>(steps, f);
    else if (stack == 32) with_steps<Src, 32>(steps, f);
    else with_steps<Src, kStackLds>(steps, f);
}

// The sources without launch knobs run the default shape.
template <class Src, class F>
void with_default(int32_t nleaf, F f)
{
    if (nleaf > kMaxNear) f(k_traverse<Src, kStackLds, kTraceSteps, true>);
    else f(k_traverse<Src, kStackLds, kTraceSteps, false>);
}

// A traversal of few rays needs no more blocks than give each wave kMinRays
// of them.
int blocks_for(int blocks, int64_t rays)
{
    const int64_t per = (int64_t)kMinRays * (kTB / 64), need = (rays + per - 1) / per;
    return need < blocks ? (need < 1 ? 1 : (int)need) : blocks;
}

int trace_blocks_per_cu(bool batch, int stack, int steps)
{
    int n = 0;
    hipError_t e = hipSuccess;
    auto occ = [&](auto kern) { e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, kTB, 0); };
    if (batch) with_shape<BatchRays>(stack, steps, 0, occ);
    else with_shape<LensRays>(stack, steps, 0, occ);
    return e == hipSuccess ? n : 0;
}

hipError_t launch_trace(const SceneDev &s, const FrameConst &fc, const ScratchLayout &L, char *scratch, int blocks,
                        hipStream_t st)
{
    LensRays src;
    const Planes P = planes(fc, L, scratch);
    src.rec0 = P.rec0;
    src.rec1 = P.rec1;
    src.ray_lt = P.ray_lt;
    uint32_t *cnt = reinterpret_cast<uint32_t *>(scratch + L.counters);
    with_shape<LensRays>(fc.tk.stack, fc.tk.steps, s.nleaf, [&](auto kern) {
        kern<<<clamp_blocks(blocks), kTB, 0, st>>>(scene_args(s), src, 0u, cnt + kCntRays, cnt + kCntWork,
                                                  reinterpret_cast<unsigned long long *>(cnt + kCntWork + kStatAt),
                                                  cnt + kCntWork + kStatAt + 4, fc.tk);
    });
    return hipGetLastError();
}

hipError_t launch_compact_small(const FrameConst &fc, const ScratchLayout &L, char *scratch, const uint8_t *mask, hipStream_t st)
{
    const uint32_t np = (uint32_t)fc.hw * (uint32_t)fc.hh;
    k_compact_small<<<(np + kGenTB - 1) / kGenTB, kGenTB, 0, st>>>(fc, planes(fc, L, scratch), mask);
    return hipGetLastError();
}

hipError_t launch_raygen(const FrameConst &fc, const ScratchLayout &L, char *scratch, hipStream_t st)
{
    const Planes P = planes(fc, L, scratch);
    const int64_t max_rays = (int64_t)fc.hw * fc.hh * fc.m;
    if (fc.ap.blades >= 3)
        k_raygen_bladed<<<gen_blocks(max_rays), kGenTB, 0, st>>>(fc, P.queue, P.ray_base, P.ray_pix,
                                                                 P.counters + kCntRays, P.rec0, P.rec1);
    else
        k_raygen<<<gen_blocks(max_rays), kGenTB, 0, st>>>(fc, P.queue, P.ray_base, P.ray_pix, P.counters + kCntRays,
                                                           P.rec0, P.rec1);
    return hipGetLastError();
}

hipError_t launch_batch_shade_resolve(const Job *jobs, int njobs, const uint32_t *nblk, hipStream_t st)
{
    kb_shade_resolve<<<nblk[kGridResolve], 64, 0, st>>>(jobs, njobs);
    return hipGetLastError();
}

hipError_t launch_shade_resolve(const SceneDev &s, const FrameConst &fc, const ScratchLayout &L, char *scratch,
                                const uint8_t *mask, hipStream_t st)
{
    const Planes P = planes(fc, L, scratch);
    const int64_t np = (int64_t)fc.hw * fc.hh;
    k_shade_resolve<<<(unsigned)((np + 63) / 64), 64, 0, st>>>(scene_args(s), fc, P, mask);
    return hipGetLastError();
}

hipError_t launch_gbuffer(const SceneDev &s, const FrameConst &fc, void *colour, int cfmt, float *depth, void *normal,
                          int nfmt, int blocks, hipStream_t st)
{
    const PinholeRays src{fc.cur, fc.W, fc.H, depth, static_cast<uint32_t *>(normal), nfmt == DOF_RGBA32F ? 4u : 2u};
    const int64_t rays = (int64_t)fc.W * fc.H;
    blocks = blocks_for(clamp_blocks(blocks), rays);
    if (rays > (int64_t)blocks * kTB) k_zero_work<<<1, 64, 0, st>>>(s.aux);   // fewer are dealt without counters
    with_default<PinholeRays>(s.nleaf, [&](auto kern) {
        kern<<<blocks, kTB, 0, st>>>(scene_args(s), src, (uint32_t)rays, nullptr, s.aux, nullptr, nullptr, fc.tk);
    });
    k_gbuffer_shade<<<(unsigned)((rays + 255) / 256), 256, 0, st>>>(scene_args(s), fc.shade, src, colour, cfmt, nfmt, (uint32_t)rays);
    return hipGetLastError();
}

hipError_t launch_trace_rays(const SceneDev &s, int64_t n, const float *org, const float *dir, int32_t *hit, float *t,
                             int blocks, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    RawRays src{org, dir, hit, t};
    blocks = blocks_for(clamp_blocks(blocks), n);
    if (n > (int64_t)blocks * kTB) k_zero_work<<<1, 64, 0, st>>>(s.aux);
    TraceKnobs tk{kStackLds, 64u, 16, 32};
    with_default<RawRays>(s.nleaf, [&](auto kern) {
        kern<<<blocks, kTB, 0, st>>>(scene_args(s), src, (uint32_t)n, nullptr, s.aux, nullptr, nullptr, tk);
    });
    return hipGetLastError();
}

hipError_t launch_reference(const SceneDev &s, const FrameConst &fc, int spp, uint2 *lt, int64_t chunk_px, void *colour,
                            int cfmt, int blocks, hipStream_t st)
{
    const int64_t npx = (int64_t)fc.W * fc.H;
    for (int64_t p0 = 0; p0 < npx; p0 += chunk_px) {
        const uint32_t n = (uint32_t)(npx - p0 < chunk_px ? npx - p0 : chunk_px);
        RefRays src{fc, (uint32_t)p0, (uint32_t)spp, lt};
        k_zero_work<<<1, 64, 0, st>>>(s.aux);
        with_default<RefRays>(s.nleaf, [&](auto kern) {
            kern<<<clamp_blocks(blocks), kTB, 0, st>>>(scene_args(s), src, n * (uint32_t)spp, nullptr, s.aux, nullptr,
                                                       nullptr, fc.tk);
        });
        k_ref_average<<<(n + 255) / 256, 256, 0, st>>>(scene_args(s), src, n, colour, cfmt);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_batch_raygen(BatchHead *head, const Job *jobs, int njobs, int64_t max_rays, hipStream_t st)
{
    kb_ray_offsets<<<1, 64, 0, st>>>(head, jobs, njobs);
    kb_raygen<<<gen_blocks(max_rays), kGenTB, 0, st>>>(jobs, head, njobs);
    return hipGetLastError();
}

hipError_t launch_batch_trace(BatchHead *head, const Job *jobs, int njobs, int blocks, const TraceKnobs &tk,
                              hipStream_t st)
{
    BatchRays src{jobs, head, njobs};
    with_shape<BatchRays>(tk.stack, tk.steps, 0, [&](auto kern) {
        kern<<<clamp_blocks(blocks), kTB, 0, st>>>(SceneArgs{}, src, 0u, &head->rays, head->work,
                                                  reinterpret_cast<unsigned long long *>(head->work + kStatAt),
                                                  nullptr, tk);
    });
    return hipGetLastError();
}

}  // namespace dof
