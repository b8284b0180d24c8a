// LBVH build on the device: the acceleration structure that replaces the
// DXR build the paper times inside its Ray Trace pass (section 5.2).
//
//   leaf references (a triangle, or four clipped pieces of a long thin one:
//   early split clipping, Ernst & Greiner 2007) with their boxes, and their
//   centroid bounds -> 64-bit keys (a large-box flag in bit 63 over a 63-bit
//   Morton code, 21 bits per axis, of cubic cells) and the digit counts of
//   all eight radix passes -> stable LSD radix sort of (key, reference), one
//   launch per pass -> the references' triangles in leaf order and the binary
//   radix tree over the 96-bit keys key << 32 | reference, numbered as Karras
//   2012 numbers it, built bottom-up with its boxes (after Apetrei 2014).
//
// A scene of few references sorts in one workgroup instead.
//
// All results are bit-reproducible: min/max are compare-selects and the
// sort is stable, so the tree depends only on the input triangles.
#include <algorithm>
#include <utility>

#include "dof_internal.h"

namespace dof {
namespace {

constexpr int kThreads = 256;
constexpr int kPasses = 8;                 // 8-bit digits of a 64-bit key
constexpr int kKeyBlocks = 256, kKeyThreads = 1024;

__device__ inline void tri_box3(const float *v, float lo[3], float hi[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float x = v[a], y = v[3 + a], z = v[6 + a];
        float m = x;
        m = y < m ? y : m;
        m = z < m ? z : m;
        lo[a] = m;
        float M = x;
        M = y > M ? y : M;
        M = z > M ? z : M;
        hi[a] = M;
    }
}

__device__ inline float wave_min(float v)
{
    for (int o = 32; o >= 1; o >>= 1) v = fmin_cs(v, __shfl_xor(v, o));
    return v;
}

__device__ inline float wave_max(float v)
{
    for (int o = 32; o >= 1; o >>= 1) v = fmax_cs(v, __shfl_xor(v, o));
    return v;
}

// Box of the piece of triangle v inside the slab s0 <= x_K <= s1: on axis K
// the slab; on each other axis the range of the vertices inside the slab and
// of the points where edges cross its planes.  A crossing point is computed
// in binary32 and widened by 2^-20 (|edge extent| + |x|), more than its
// rounding error; the range is then clipped to the triangle's box.  So the
// box holds every point of the piece, and the pieces' boxes together hold
// the triangle: a ray that meets the triangle enters one of them.
template <int K>
__device__ inline void piece_box(const float *v, float s0, float s1, const float lo[3], const float hi[3], float *out)
{
    out[K] = s0;
    out[3 + K] = s1;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        if (m == K) continue;
        float pl = INFINITY, ph = -INFINITY;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const float vk = v[3 * i + K];
            if (vk >= s0 && vk <= s1) {
                const float x = v[3 * i + m];
                pl = x < pl ? x : pl;
                ph = x > ph ? x : ph;
            }
        }
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const float *p = v + 3 * e, *q = v + 3 * (e == 2 ? 0 : e + 1);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float pc = c ? s1 : s0;
                if ((p[K] < pc && pc < q[K]) || (q[K] < pc && pc < p[K])) {
                    const float t = (pc - p[K]) / (q[K] - p[K]);
                    const float d = q[m] - p[m];
                    const float x = p[m] + d * t;
                    const float g = (fabsf(d) + fabsf(x)) * 9.5367431640625e-07f;   // 2^-20
                    const float xl = x - g, xh = x + g;
                    pl = xl < pl ? xl : pl;
                    ph = xh > ph ? xh : ph;
                }
            }
        }
        pl = lo[m] > pl ? lo[m] : pl;
        ph = hi[m] < ph ? hi[m] : ph;
        if (pl > ph) {
            pl = lo[m];
            ph = hi[m];
        }
        out[m] = pl;
        out[3 + m] = ph;
    }
}

// The np pieces of a triangle cut into equal slabs of its box along axis K.
template <int K, class Put>
__device__ inline void cut_slabs(const float *v, const float lo[3], const float hi[3], int np, Put put)
{
    const float q = (hi[K] - lo[K]) * (1.0f / (float)np);
    float s0 = lo[K];
    for (int j = 0; j < np; ++j) {
        float s1 = hi[K];
        if (j + 1 < np) {
            const float x = lo[K] + q * (float)(j + 1);
            s1 = x < hi[K] ? x : hi[K];
        }
        float o[6];
        piece_box<K>(v, s0, s1, lo, hi, o);
        put(j, o);
        s0 = s1;
    }
}

// References of triangle i.  A triangle with one reference keeps its own box;
// one with 2, 4 or 8 is cut into that many equal slabs of its box along the
// longest axis (the first one on ties).  The references' box centres widen
// blo, bhi.
__device__ inline void emit_refs(const float *__restrict__ verts, int i, const uint32_t *__restrict__ ref_off,
                                 LeafRef *__restrict__ refs, float blo[3], float bhi[3])
{
    float v[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) v[k] = verts[9 * (size_t)i + k];
    float lo[3], hi[3];
    tri_box3(v, lo, hi);
    const uint32_t r0 = ref_off[i], nr = ref_off[i + 1] - r0;
    auto put = [&](int j, const float o[6]) __attribute__((always_inline)) {
        float4 *dst = reinterpret_cast<float4 *>(refs + r0 + j);
        dst[0] = make_float4(o[0], o[1], o[2], o[3]);
        dst[1] = make_float4(o[4], o[5], __uint_as_float((uint32_t)i), 0.0f);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float c = (o[a] + o[3 + a]) * 0.5f;
            blo[a] = fmin_cs(blo[a], c);
            bhi[a] = fmax_cs(bhi[a], c);
        }
    };
    if (nr == 1) {
        const float o[6] = {lo[0], lo[1], lo[2], hi[0], hi[1], hi[2]};
        put(0, o);
        return;
    }
    const float ext[3] = {hi[0] - lo[0], hi[1] - lo[1], hi[2] - lo[2]};
    const int np = nr <= 2 ? 2 : (nr <= 4 ? 4 : 8);   // 2, 4 or 8 (the host never writes another count)
    const float x01 = ext[1] > ext[0] ? ext[1] : ext[0];
    if (ext[2] > x01) cut_slabs<2>(v, lo, hi, np, put);
    else if (ext[1] > ext[0]) cut_slabs<1>(v, lo, hi, np, put);
    else cut_slabs<0>(v, lo, hi, np, put);
}

// A block's minimum of lo and maximum of hi, in every thread's lo and hi
// (red: 6 x the block's waves, in LDS).
template <int kWaves>
__device__ inline void block_bounds(float lo[3], float hi[3], float (*red)[kWaves])
{
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int a = 0; a < 3; ++a) {
        const float m = wave_min(lo[a]), M = wave_max(hi[a]);
        if (lane == 0) { red[a][w] = m; red[3 + a][w] = M; }
    }
    __syncthreads();
    for (int a = 0; a < 3; ++a) {
        lo[a] = red[a][0];
        hi[a] = red[3 + a][0];
        for (int k = 1; k < kWaves; ++k) {
            lo[a] = fmin_cs(lo[a], red[a][k]);
            hi[a] = fmax_cs(hi[a], red[3 + a][k]);
        }
    }
}

// All references, each block's centre bounds, and the sort's state cleared.
__global__ __launch_bounds__(kThreads) void k_emit(const float *__restrict__ verts, int nt, const uint32_t *__restrict__ ref_off,
                                                   LeafRef *__restrict__ refs, float *__restrict__ partial, uint32_t *__restrict__ clear, int64_t nclear)
{
    __shared__ float red[6][kThreads / 64];
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    const int64_t step = (int64_t)gridDim.x * kThreads, first = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    for (int64_t i = first; i < nclear; i += step) clear[i] = 0u;
    for (int64_t i = first; i < nt; i += step) emit_refs(verts, (int)i, ref_off, refs, lo, hi);
    block_bounds<kThreads / 64>(lo, hi, red);
    if (threadIdx.x < 6) partial[6 * blockIdx.x + threadIdx.x] = threadIdx.x < 3 ? lo[threadIdx.x] : hi[threadIdx.x - 3];
}

// The Morton grid of the centre bounds: origin, one scale for all three axes,
// 2^21 / (largest extent), so its cells are cubes, and the squared diagonal
// above which a box counts as large (a quarter of the bounds' diagonal,
// squared).
struct KeyGrid {
    float lo[3], inv, large;
};

__device__ inline KeyGrid key_grid(const float lo[3], const float hi[3])
{
    KeyGrid g;
    float ext[3];
    for (int a = 0; a < 3; ++a) {
        g.lo[a] = lo[a];
        ext[a] = hi[a] - lo[a];
    }
    const float e = fmax_cs(fmax_cs(ext[0], ext[1]), ext[2]);
    const float s2 = (ext[0] * ext[0] + ext[1] * ext[1]) + ext[2] * ext[2];
    g.inv = e > 0.0f ? 2097152.0f / e : 0.0f;
    g.large = s2 * 0.0625f;
    return g;
}

__device__ inline uint64_t spread_bits21(uint32_t v)
{
    uint64_t x = v & 0x1fffffu;
    x = (x | (x << 32)) & 0x001f00000000ffffull;
    x = (x | (x << 16)) & 0x001f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ inline uint64_t key_of(const LeafRef *refs, size_t i, const KeyGrid &g)
{
    const float4 p = reinterpret_cast<const float4 *>(refs + i)[0], b = reinterpret_cast<const float4 *>(refs + i)[1];
    const float bl[3] = {p.x, p.y, p.z}, bh[3] = {p.w, b.x, b.y};
    uint32_t q[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float c = (bl[a] + bh[a]) * 0.5f;
        float t = floorf((c - g.lo[a]) * g.inv);
        int qi = (int)t;
        q[a] = (uint32_t)(qi > 2097151 ? 2097151 : qi);
    }
    const float dx = bh[0] - bl[0], dy = bh[1] - bl[1], dz = bh[2] - bl[2];
    const uint64_t large = ((dx * dx + dy * dy) + dz * dz) > g.large ? 1ull : 0ull;
    return (large << 63) | (spread_bits21(q[0]) << 2) | (spread_bits21(q[1]) << 1) | spread_bits21(q[2]);
}

// ---------------------------------------------------------------- radix sort
// Stable LSD passes over 8-bit digits.  The digit counts of all passes do not
// depend on the order, so the key kernel counts them once; a pass is then one
// launch: each tile ranks its keys, publishes its digit counts and finds the
// counts of the tiles before it by looking back (Merrill & Garland 2016,
// Adinets & Merrill 2022), and stores its keys from LDS in digit order, so
// most stores of a wave fall into few runs.  At 1.94 M references a pass takes
// 22 us, where the ranking and the look-back (4.5 and 4.4 us of one block's 16)
// weigh more than the 47 MB it moves; a count, two scan and a scatter launch
// per pass took 43.

// Keys and reference indices, and per block the digit counts of all passes.
__global__ __launch_bounds__(kKeyThreads) void k_keys(const LeafRef *__restrict__ refs, int n,
                                                      const float *__restrict__ partial, int npartial,
                                                      uint64_t *__restrict__ keys, uint32_t *__restrict__ ids,
                                                      uint32_t *__restrict__ rows)
{
    __shared__ float red[6][kKeyThreads / 64];
    __shared__ uint32_t cnt[kPasses * 256];
    const int tid = threadIdx.x;
    for (int k = tid; k < kPasses * 256; k += kKeyThreads) cnt[k] = 0u;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int b = tid; b < npartial; b += kKeyThreads)
        for (int a = 0; a < 3; ++a) {
            lo[a] = fmin_cs(lo[a], partial[6 * b + a]);
            hi[a] = fmax_cs(hi[a], partial[6 * b + 3 + a]);
        }
    block_bounds<kKeyThreads / 64>(lo, hi, red);
    const KeyGrid g = key_grid(lo, hi);
    const int64_t step = (int64_t)gridDim.x * kKeyThreads;
    for (int64_t i = (int64_t)blockIdx.x * kKeyThreads + tid; i < n; i += step) {
        const uint64_t key = key_of(refs, (size_t)i, g);
        keys[i] = key;
        ids[i] = (uint32_t)i;
        // neighbouring references share their high digits: one add for a
        // wave whose lanes agree
        const uint64_t here = __ballot(true);
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const uint32_t d = (uint32_t)(key >> (8 * p)) & 0xffu;
            const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
            if (__ballot(d != d0) == 0ull) {
                if ((tid & 63) == __builtin_ctzll(here)) atomicAdd(&cnt[256 * p + d0], (uint32_t)__popcll(here));
            } else {
                atomicAdd(&cnt[256 * p + d], 1u);
            }
        }
    }
    __syncthreads();
    for (int k = tid; k < kPasses * 256; k += kKeyThreads) rows[(size_t)blockIdx.x * (kPasses * 256) + k] = cnt[k];
}

__device__ inline uint32_t wave_incl(uint32_t v, int lane)
{
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(v, o);
        if (lane >= o) v += u;
    }
    return v;
}

// Exclusive sum of v over threads 0..255 of a block (scr: 4 words of LDS);
// every thread calls it, the first 256 get their sum.
__device__ inline uint32_t scan256(uint32_t v, uint32_t *scr)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t incl = wave_incl(v, lane);
    if (w < 4 && lane == 63) scr[w] = incl;
    __syncthreads();
    uint32_t base = 0u;
    for (int k = 0; k < w && k < 4; ++k) base += scr[k];
    __syncthreads();
    return base + incl - v;
}

// First output place of every digit: block p sums pass p's columns of the key
// blocks' rows and scans the sums.
__global__ __launch_bounds__(1024) void k_digit_places(const uint32_t *__restrict__ rows, int nrows, uint32_t *__restrict__ first)
{
    __shared__ uint32_t part[4][256];
    __shared__ uint32_t scr[4];
    const int c = threadIdx.x & 255, g = threadIdx.x >> 8;
    uint32_t sum = 0u;
#pragma unroll 16
    for (int r = g; r < nrows; r += 4) sum += rows[(size_t)r * (kPasses * 256) + 256 * blockIdx.x + c];
    part[g][c] = sum;
    __syncthreads();
    const uint32_t all = g == 0 ? ((part[0][c] + part[1][c]) + part[2][c]) + part[3][c] : 0u;
    const uint32_t at = scan256(all, scr);
    if (g == 0) first[256 * blockIdx.x + c] = at;
}

// Ranks a lane's keys (at most kItems) by the digit at `shift`, a wave's keys
// being `rounds` rounds of 64 in order: rank[r] is the key's place among the wave's
// keys of its digit, cnt (256 words of LDS, the wave's own) their counts.
template <int kItems>
__device__ inline void wave_rank(const uint64_t key[kItems], const bool valid[kItems], int rounds, int shift, uint32_t *cnt,
                                 uint32_t rank[kItems])
{
    const int lane = threadIdx.x & 63;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int k = lane; k < 256; k += 64) cnt[k] = 0u;
    uint32_t below[kItems], peers[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        if (r >= rounds) continue;
        const uint32_t d = (uint32_t)(key[r] >> shift) & 0xffu;
        const uint64_t all = __ballot(valid[r]);
        uint32_t ml = (uint32_t)all, mh = (uint32_t)(all >> 32);   // the lanes that share the digit
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint32_t x = (uint32_t)((int32_t)(d << (31 - bit)) >> 31);   // all ones where the bit is set
            const uint64_t bb = __ballot(x != 0u);
            ml &= ~((uint32_t)bb ^ x);
            mh &= ~((uint32_t)(bb >> 32) ^ x);
        }
        const uint64_t match = (uint64_t)mh << 32 | ml;
        below[r] = (uint32_t)__popcll(match & lt);
        peers[r] = (uint32_t)__popcll(match);
    }
    // LDS accesses of a wave execute in order: all lanes read the count, then
    // each digit's first lane adds its keys
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        if (r >= rounds) continue;
        const uint32_t d = (uint32_t)(key[r] >> shift) & 0xffu;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint32_t before = valid[r] ? cnt[d] : 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (valid[r] && below[r] == 0u) cnt[d] = before + peers[r];
        rank[r] = before + below[r];
    }
}

// Look-back words: 0 nothing yet, count + 1 a tile's own count, bit 31 + sum
// the sum of the tile and all before it.
constexpr uint32_t kSumWord = 0x80000000u;

// One pass.  first: each digit's first output place; ticket: its tile counter; words:
// 256 look-back words per tile, all zero at first.  Tiles are numbered in the
// order in which blocks start, so a tile waits only for tiles whose blocks run
// already, and those publish their counts before they wait themselves.
template <int kWaves, int kItems>
__global__ __launch_bounds__(kWaves * 64) void k_sort_pass(const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                           uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int n,
                                                           int shift, const uint32_t *__restrict__ first, uint32_t *ticket,
                                                           uint32_t *words)
{
    constexpr int kTileKeys = kWaves * 64 * kItems;
    __shared__ uint64_t skey[kTileKeys];
    __shared__ uint32_t sval[kTileKeys];
    __shared__ uint32_t wcnt[kWaves][256];
    __shared__ uint32_t goff[256];    // digit -> output place of the tile's first key of it, less its place in the tile
    __shared__ uint32_t scr[4], s_tile;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    if (tid == 0) s_tile = atomicAdd(ticket, 1u);
    __syncthreads();
    const uint32_t tile = s_tile;
    const size_t base = (size_t)tile * kTileKeys + (size_t)w * (64 * kItems);
    uint64_t key[kItems];
    uint32_t val[kItems], rank[kItems];
    bool valid[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const size_t i = base + (size_t)r * 64 + lane;
        valid[r] = i < (size_t)n;
        key[r] = valid[r] ? kin[i] : 0ull;
        val[r] = valid[r] ? vin[i] : 0u;
    }
    wave_rank<kItems>(key, valid, kItems, shift, wcnt[w], rank);
    __syncthreads();
    // digit tid: the tile's count, the waves' first places, the place in the tile
    uint32_t count = 0u;
    if (tid < 256) {
        for (int k = 0; k < kWaves; ++k) {
            const uint32_t c = wcnt[k][tid];
            wcnt[k][tid] = count;
            count += c;
        }
        __hip_atomic_store(words + (size_t)tile * 256 + tid, tile == 0u ? (kSumWord | count) : count + 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint32_t place = scan256(count, scr);
    if (tid < 256) {
        for (int k = 0; k < kWaves; ++k) wcnt[k][tid] += place;
        uint32_t sum = 0u;
        // the tiles before, kLook at a time so that their loads overlap (2, 4, 8,
        // 16, 32: 444, 441, 445, 457, 473 us for a build of 1.94 M references)
        constexpr int kLook = 4;
        for (int64_t t = (int64_t)tile - 1; t >= 0;) {
            uint32_t got[kLook];
#pragma unroll
            for (int k = 0; k < kLook; ++k)
                got[k] = t - k >= 0 ? __hip_atomic_load(words + (size_t)(t - k) * 256 + tid, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT)
                                    : kSumWord;
            bool done = false;
            int used = 0;
#pragma unroll
            for (int k = 0; k < kLook; ++k) {
                if (!done && used == k && got[k] != 0u) {
                    ++used;
                    done = (got[k] & kSumWord) != 0u;
                    sum += done ? got[k] & ~kSumWord : got[k] - 1u;
                }
            }
            if (done) break;
            t -= used;
            if (used == 0) __builtin_amdgcn_s_sleep(1);
        }
        if (tile != 0u)
            __hip_atomic_store(words + (size_t)tile * 256 + tid, kSumWord | (sum + count), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        goff[tid] = first[tid] + sum - place;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r)
        if (valid[r]) {
            const uint32_t at = wcnt[w][(uint32_t)(key[r] >> shift) & 0xffu] + rank[r];
            skey[at] = key[r];
            sval[at] = val[r];
        }
    __syncthreads();
    const size_t left = (size_t)n - (size_t)tile * kTileKeys;
    const uint32_t m = left < (size_t)kTileKeys ? (uint32_t)left : (uint32_t)kTileKeys;
    for (uint32_t t = tid; t < m; t += kWaves * 64) {
        const uint64_t k = skey[t];
        const uint32_t at = goff[(uint32_t)(k >> shift) & 0xffu] + t;
        kout[at] = k;
        vout[at] = sval[t];
    }
}

// A scene of at most kSmallRefs references, sorted by one workgroup: the
// references, their keys in LDS, eight passes there (a pass whose digit is the
// same in all keys changes nothing), the sorted keys and indices out.  Few
// references leave the many launches of the general path nearly empty: a scene
// of 866 triangles built in 170 us, most of it launches, and builds in 39.
constexpr int kSmallRefs = 4096, kSmallThreads = 512, kSmallItems = kSmallRefs / kSmallThreads;

__global__ __launch_bounds__(kSmallThreads) void k_small_sort(const float *__restrict__ verts, int nt,
                                                              const uint32_t *__restrict__ ref_off, LeafRef *refs, int n,
                                                              uint64_t *__restrict__ keys, uint32_t *__restrict__ ids)
{
    constexpr int kWaves = kSmallThreads / 64;
    __shared__ uint64_t skey[kSmallRefs];
    __shared__ uint16_t sval[kSmallRefs];
    __shared__ uint32_t wcnt[kWaves][256];
    __shared__ float red[6][kWaves];
    __shared__ uint32_t scr[4], s_same;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = tid; i < nt; i += kSmallThreads) emit_refs(verts, i, ref_off, refs, lo, hi);
    block_bounds<kWaves>(lo, hi, red);
    const KeyGrid g = key_grid(lo, hi);
    __threadfence_block();
    __syncthreads();
    uint64_t key[kSmallItems];
    uint32_t val[kSmallItems], rank[kSmallItems];
    bool valid[kSmallItems];
    const int rounds = (n + kSmallThreads - 1) / kSmallThreads;   // a wave's keys: rounds x 64 in order
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        const int i = w * (64 * rounds) + r * 64 + lane;
        valid[r] = r < rounds && i < n;
        key[r] = valid[r] ? key_of(refs, (size_t)i, g) : 0ull;
        val[r] = valid[r] ? (uint32_t)i : 0u;
    }
    for (int shift = 0; shift < 64; shift += 8) {
        wave_rank<kSmallItems>(key, valid, rounds, shift, wcnt[w], rank);
        if (tid == 0) s_same = 0u;
        __syncthreads();
        uint32_t count = 0u;
        if (tid < 256) {
            for (int k = 0; k < kWaves; ++k) {
                const uint32_t c = wcnt[k][tid];
                wcnt[k][tid] = count;
                count += c;
            }
            if (count == (uint32_t)n) s_same = 1u;
        }
        const uint32_t place = scan256(count, scr);   // ends with a barrier
        const bool same = s_same != 0u;
        __syncthreads();
        if (same) continue;                            // block-uniform
        if (tid < 256)
            for (int k = 0; k < kWaves; ++k) wcnt[k][tid] += place;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSmallItems; ++r)
            if (valid[r]) {
                const uint32_t at = wcnt[w][(uint32_t)(key[r] >> shift) & 0xffu] + rank[r];
                skey[at] = key[r];
                sval[at] = (uint16_t)val[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSmallItems; ++r)
            if (valid[r]) {
                const int i = w * (64 * rounds) + r * 64 + lane;
                key[r] = skey[i];
                val[r] = sval[i];
            }
    }
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r)
        if (valid[r]) {
            const int i = w * (64 * rounds) + r * 64 + lane;
            keys[i] = key[r];
            ids[i] = val[r];
        }
}

// ---------------------------------------------------------------- hierarchy

// Length of the common prefix of the 96-bit keys (code << 32 | reference) of
// leaves i and j; -1 outside the array.
__device__ inline int delta96(const uint64_t *keys, const uint32_t *ids, int n, int i, int j)
{
    if (j < 0 || j >= n) return -1;
    uint64_t x = keys[i] ^ keys[j];
    if (x != 0ull) return __clzll(x);
    return 64 + __clz(ids[i] ^ ids[j]);
}

inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// The traversal's binary16 copy of the nodes.  Each plane is converted with
// directed rounding, low planes down and high planes up, and a result in the
// subnormal range goes outward to 0 or to the smallest normal (2^-14), so the
// copy holds every box whatever the device's binary16 denormal mode; a plane
// beyond the binary16 range becomes an infinite one on its side.
// Conversion towards zero is one instruction; away from zero is the next
// value where that was inexact.
__device__ inline uint32_t half_rtz(float x, float &back)
{
    const auto h = __builtin_amdgcn_cvt_pkrtz(x, 0.0f);
    back = (float)h[0];
    return (uint32_t)__builtin_bit_cast(unsigned short, h[0]);
}

constexpr float kHalfMin = 6.103515625e-05f;   // 2^-14, the smallest normal binary16

__device__ inline uint32_t plane_down(float x)
{
    float back;
    const uint32_t b = half_rtz(x, back);
    const uint32_t neg = x > -kHalfMin ? 0x8400u : b + (back != x ? 1u : 0u);
    const uint32_t pos = x < kHalfMin ? b & 0x8000u : b;   // keeps the sign of a zero
    return x < 0.0f ? neg : pos;
}

__device__ inline uint32_t plane_up(float x)
{
    float back;
    const uint32_t b = half_rtz(x, back);
    const uint32_t pos = x < kHalfMin ? 0x0400u : b + (back != x ? 1u : 0u);
    const uint32_t neg = x > -kHalfMin ? ((b & 0x7fffu) == 0u ? b : 0u) : b;   // upwards to -0, or from a subnormal to 0
    return x > 0.0f ? pos : neg;
}

__device__ inline uint32_t axis16(float lo, float hi) { return plane_down(lo) | (plane_up(hi) << 16); }

// The tree, bottom-up.  A node that covers leaves l..r hangs below the split
// between r and r + 1 (as a left child) or between l - 1 and l (as a right
// child), whichever pair of leaves has the longer common key prefix (the two
// are never equal: a node's neighbours on its two sides differ from it in
// opposite values of the bit after a common prefix of equal length).  So
// adjacent subtrees pair up at their split: the first to arrive leaves its
// range and box there and the second goes on with the union, knowing both
// children.  Karras' index of a node is its last leaf as a left child, its
// first as a right child, 0 for the root.
//
// A block merges kMergeThreads consecutive entries in LDS (no ordering wider
// than the workgroup is needed: on a multi-die GPU an agent-scope one writes
// back and invalidates a die's L2).  k_tree_blocks starts from leaves; the
// subtrees whose parents reach beyond the block are its exits, in order, and
// are the entries of k_tree_merge's blocks, whose exits k_tree_top's one
// workgroup merges round by round to the root.  At most 194 subtrees exit a
// block (up to 96 siblings along the path to the parent's range on either
// side and the last subtree, prefixes being 0..95 bits long).
// Bound by memory: the leaves' gathered triangles and 168 bytes stored per leaf
// take 134 us at 1.94 M references, the blocks' exits 53 more; Karras' searches,
// a leaf-to-root climb with global reads at each level, one workgroup for all
// nodes that span blocks, and kernels for the triangles and for the copy of
// the nodes took 83 + 165 + 464 + 56 + 28.
constexpr int kMergeThreads = 1024;
constexpr int kExitCap = 256;         // exit records per block
constexpr int kTopBlocks = 64;        // blocks up to which k_tree_top takes the exits of k_tree_blocks itself

struct Entry {        // 32 B: leaves l..r and their box
    uint32_t l, r;
    float lo[3], hi[3];
};

struct TreeOut {
    const uint64_t *keys;
    const uint32_t *ids;
    int n;
    BvhNode *nodes;
    BvhNode16 *nodes16;
    uint32_t *parent;
};

struct MergeLds {
    float box[12][kMergeThreads + 1];   // per split: left child's lo xyz, hi xyz, then the right one's
    uint32_t arrived[kMergeThreads + 1];   // 1: left child, 2: right child
    // per split: the left child's first entry, the right child's last one, each
    // with the common prefix beyond it (+ 1) in the upper half
    uint32_t first[kMergeThreads + 1], last[kMergeThreads + 1];
    uint32_t node_at[kMergeThreads];    // split -> index of its node, or ~0
    uint16_t exit_of[kMergeThreads];    // first entry of an exit -> split | side << 15, or kNone
    int8_t d[kMergeThreads + 2];        // common prefix before each entry (d[e]) and after the last
    uint32_t wsum[kMergeThreads / 64];
};
constexpr uint16_t kNone = 0xffffu;

// A node's record by the two lanes' worth of words that its boxes and links make.
__device__ inline uint4 node16_word(const MergeLds &m, int s, int part, uint32_t left, uint32_t right)
{
    if (part == 0)
        return make_uint4(axis16(m.box[0][s], m.box[3][s]), axis16(m.box[1][s], m.box[4][s]),
                          axis16(m.box[2][s], m.box[5][s]), axis16(m.box[6][s], m.box[9][s]));
    return make_uint4(axis16(m.box[7][s], m.box[10][s]), axis16(m.box[8][s], m.box[11][s]), left, right);
}

__device__ inline float4 node_word(const MergeLds &m, int s, int part, uint32_t left, uint32_t right, uint32_t l, uint32_t r)
{
    if (part == 0) return make_float4(m.box[0][s], m.box[3][s], m.box[1][s], m.box[4][s]);
    if (part == 1) return make_float4(m.box[6][s], m.box[9][s], m.box[7][s], m.box[10][s]);
    if (part == 2) return make_float4(m.box[2][s], m.box[5][s], m.box[8][s], m.box[11][s]);
    return make_float4(__uint_as_float(left), __uint_as_float(right), __uint_as_float(l), __uint_as_float(r));
}

// Merges the block's entries 0..count-1, thread e holding entry e (its box in
// lo, hi; before and, of the last one, after: the common prefix with the leaf
// on either side); lo_of(e) and hi_of(e) are any entry's first and last leaf.  The
// nodes found are written after all merges.  Exits go to `out` in order;
// returns their number.  Every thread of the block calls it; it ends with a
// barrier.
template <class Lo, class Hi>
__device__ inline uint32_t merge_entries(MergeLds &m, const TreeOut &T, int count, int before, int after, float lo[3],
                                         float hi[3], Lo lo_of, Hi hi_of, Entry *__restrict__ out)
{
    const int tid = threadIdx.x;
    for (int k = tid; k <= kMergeThreads; k += kMergeThreads) m.arrived[k] = 0u;
    m.node_at[tid] = ~0u;
    m.exit_of[tid] = kNone;
    if (tid < count) m.d[tid] = (int8_t)before;
    if (tid == count - 1) m.d[count] = (int8_t)after;
    __syncthreads();
    if (tid < count) {
        int el = tid, er = tid, split = -1;   // split: where the two children met (-1: an entry)
        int dl = m.d[tid], dr = m.d[tid + 1];
        while (true) {
            const bool root = dl < 0 && dr < 0, is_left = dr > dl;
            if (split >= 0) m.node_at[split] = root ? 0u : (is_left ? hi_of(er) : lo_of(el));
            if (root) break;
            const int s = is_left ? er : (el > 0 ? el - 1 : count);   // slot `count`: the split before entry 0
            const int side = is_left ? 0 : 6;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                m.box[side + a][s] = lo[a];
                m.box[side + 3 + a][s] = hi[a];
            }
            if (is_left) m.first[s] = (uint32_t)el | (uint32_t)(dl + 1) << 16;
            else m.last[s] = (uint32_t)er | (uint32_t)(dr + 1) << 16;
            // LDS accesses of a wave execute in order, so who sees the arrival
            // sees what was stored before it; nothing outside LDS is shared
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            const uint32_t old = __hip_atomic_fetch_add(&m.arrived[s], is_left ? 1u : 2u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (old == 0u) break;
            const uint32_t far = is_left ? m.last[s] : m.first[s];
            if (is_left) {
                er = (int)(far & 0xffffu);
                dr = (int)(far >> 16) - 1;
            } else {
                el = (int)(far & 0xffffu);
                dl = (int)(far >> 16) - 1;
            }
            split = s;
            // union(left, right) as compare-selects, left first
            for (int a = 0; a < 3; ++a) {
                const float L = m.box[a][s], R = m.box[6 + a][s], LH = m.box[3 + a][s], RH = m.box[9 + a][s];
                lo[a] = R < L ? R : L;
                hi[a] = RH > LH ? RH : LH;
            }
        }
    }
    __syncthreads();
    // one-sided splits hold the exits
    if (tid < count) {
        const uint32_t a = m.arrived[tid];
        if (a == 1u) m.exit_of[m.first[tid] & 0xffffu] = (uint16_t)tid;
        else if (a == 2u) m.exit_of[tid + 1] = (uint16_t)(tid | 0x8000);
    }
    if (tid == 0 && m.arrived[count] == 2u) m.exit_of[0] = (uint16_t)(count | 0x8000);
    // a record's four words by four lanes, so that a node is stored whole
    for (int t = tid; t < 4 * count; t += kMergeThreads) {
        const int s = t >> 2, part = t & 3;
        const uint32_t at = m.node_at[s];
        if (at == ~0u) continue;
        const uint32_t l = lo_of(m.first[s] & 0xffffu), r = hi_of(m.last[s] & 0xffffu), gl = hi_of(s);
        const uint32_t left = l == gl ? gl | kLeaf : gl, right = r == gl + 1 ? (gl + 1) | kLeaf : gl + 1;
        reinterpret_cast<float4 *>(T.nodes + at)[part] = node_word(m, s, part, left, right, l, r);
        if (part < 2) {
            reinterpret_cast<uint4 *>(T.nodes16 + at)[part] = node16_word(m, s, part, left, right);
        } else {
            const bool leaf = ((part == 2 ? left : right) & kLeaf) != 0u;
            const uint32_t c = part == 2 ? gl : gl + 1;
            T.parent[leaf ? (size_t)(T.n - 1) + c : (size_t)c] = at;
            if (part == 2 && l == 0u && r == (uint32_t)(T.n - 1)) T.parent[0] = ~0u;
        }
    }
    __syncthreads();
    const uint16_t ex = m.exit_of[tid];
    const bool has = ex != kNone;
    const uint64_t bal = __ballot(has);
    const int lane = tid & 63, w = tid >> 6;
    if (lane == 0) m.wsum[w] = (uint32_t)__popcll(bal);
    __syncthreads();
    uint32_t ahead = 0u, total = 0u;
    for (int k = 0; k < kMergeThreads / 64; ++k) {
        if (k < w) ahead += m.wsum[k];
        total += m.wsum[k];
    }
    if (has) {
        const uint32_t rank = ahead + (uint32_t)__popcll(bal & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
        const int s = ex & 0x7fff, side = (ex & 0x8000) ? 6 : 0;
        const int e1 = side ? (int)(m.last[s] & 0xffffu) : s;
        uint4 *dst = reinterpret_cast<uint4 *>(out + rank);
        dst[0] = make_uint4(lo_of(tid), hi_of(e1), __float_as_uint(m.box[side][s]), __float_as_uint(m.box[side + 1][s]));
        dst[1] = make_uint4(__float_as_uint(m.box[side + 2][s]), __float_as_uint(m.box[side + 3][s]),
                            __float_as_uint(m.box[side + 4][s]), __float_as_uint(m.box[side + 5][s]));
    }
    __syncthreads();
    return total;
}

// Leaves b0 .. b0 + 1023: their triangles and albedos in leaf order, and the
// subtrees among them.
__global__ __launch_bounds__(kMergeThreads) void k_tree_blocks(const float *__restrict__ verts, const float *__restrict__ alb,
                                                               const LeafRef *__restrict__ refs, TreeOut T,
                                                               float4 *__restrict__ tris, float4 *__restrict__ albedo,
                                                               Entry *__restrict__ exits, uint32_t *__restrict__ counts)
{
    __shared__ MergeLds m;
    const uint32_t b0 = blockIdx.x * (uint32_t)kMergeThreads;
    const int count = T.n - (int)b0 < kMergeThreads ? T.n - (int)b0 : kMergeThreads;
    float lo[3] = {0.0f, 0.0f, 0.0f}, hi[3] = {0.0f, 0.0f, 0.0f};
    int before = -1, after = -1;
    if ((int)threadIdx.x < count) {
        const size_t i = b0 + threadIdx.x;
        const float4 *ref = reinterpret_cast<const float4 *>(refs + T.ids[i]);
        const float4 p = ref[0], q = ref[1];
        before = delta96(T.keys, T.ids, T.n, (int)i, (int)i - 1);
        if ((int)threadIdx.x == count - 1) after = delta96(T.keys, T.ids, T.n, (int)i, (int)i + 1);
        lo[0] = p.x; lo[1] = p.y; lo[2] = p.z;
        hi[0] = p.w; hi[1] = q.x; hi[2] = q.y;
        const uint32_t id = __float_as_uint(q.z);
        const float *v = verts + 9 * (size_t)id, *a = alb + 3 * (size_t)id;
        tris[3 * i + 0] = make_float4(v[0], v[1], v[2], __uint_as_float(id));
        tris[3 * i + 1] = make_float4(v[3], v[4], v[5], 0.0f);
        tris[3 * i + 2] = make_float4(v[6], v[7], v[8], 0.0f);
        albedo[i] = make_float4(a[0], a[1], a[2], 0.0f);
    }
    auto leaf = [&](int e) { return b0 + (uint32_t)e; };
    const uint32_t n = merge_entries(m, T, count, before, after, lo, hi, leaf, leaf, exits + (size_t)blockIdx.x * kExitCap);
    if (threadIdx.x == 0) counts[blockIdx.x] = n;
}

// Exclusive sums of n counts by one workgroup of kMergeThreads; off[n] is the total.
__device__ inline void block_offsets(const uint32_t *counts, uint32_t n, uint32_t *off, uint32_t *wsum)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t carry = 0u;
    for (uint32_t c0 = 0; c0 < n; c0 += kMergeThreads) {
        const uint32_t i = c0 + (uint32_t)tid, v = i < n ? counts[i] : 0u;
        const uint32_t incl = wave_incl(v, lane);
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        uint32_t before = 0u, all = 0u;
        for (int k = 0; k < kMergeThreads / 64; ++k) {
            if (k < w) before += wsum[k];
            all += wsum[k];
        }
        if (i < n) off[i] = carry + before + incl - v;
        carry += all;
        __syncthreads();
    }
    if (tid == 0) off[n] = carry;
    __syncthreads();
}

__global__ __launch_bounds__(kMergeThreads) void k_exit_offsets(const uint32_t *counts, uint32_t n, uint32_t *off)
{
    __shared__ uint32_t wsum[kMergeThreads / 64];
    block_offsets(counts, n, off, wsum);
}

// Entry k of the concatenation of n blocks' exits.
__device__ inline Entry exit_at(const Entry *exits, const uint32_t *off, uint32_t n, uint32_t k)
{
    uint32_t a = 0, b = n - 1;
    while (a < b) {
        const uint32_t mid = (a + b + 1) >> 1;
        if (off[mid] <= k) a = mid;
        else b = mid - 1;
    }
    const uint4 *p = reinterpret_cast<const uint4 *>(exits + (size_t)a * kExitCap + (k - off[a]));
    const uint4 x = p[0], y = p[1];
    return Entry{x.x, x.y, {__uint_as_float(x.z), __uint_as_float(x.w), __uint_as_float(y.x)},
                 {__uint_as_float(y.y), __uint_as_float(y.z), __uint_as_float(y.w)}};
}

// A round of at most kMergeThreads entries, e being thread tid's.
__device__ inline uint32_t merge_round(MergeLds &m, uint32_t *el, uint32_t *er, const TreeOut &T, int count, Entry &e, Entry *out)
{
    int before = -1, after = -1;
    if ((int)threadIdx.x < count) {
        el[threadIdx.x] = e.l;
        er[threadIdx.x] = e.r;
        before = delta96(T.keys, T.ids, T.n, (int)e.l, (int)e.l - 1);
        if ((int)threadIdx.x == count - 1) after = delta96(T.keys, T.ids, T.n, (int)e.r, (int)e.r + 1);
    }
    __syncthreads();
    return merge_entries(m, T, count, before, after, e.lo, e.hi, [&](int k) { return el[k]; }, [&](int k) { return er[k]; }, out);
}

// Block b merges entries 1024 b .. of the n blocks' exits.
__global__ __launch_bounds__(kMergeThreads) void k_tree_merge(TreeOut T, const Entry *__restrict__ exits,
                                                              const uint32_t *__restrict__ off, uint32_t n, Entry *out,
                                                              uint32_t *__restrict__ counts)
{
    __shared__ MergeLds m;
    __shared__ uint32_t el[kMergeThreads], er[kMergeThreads];
    const uint32_t total = off[n], first = blockIdx.x * (uint32_t)kMergeThreads;
    if (first >= total) {   // the grid holds as many blocks as there can be
        if (threadIdx.x == 0) counts[blockIdx.x] = 0u;
        return;
    }
    const int count = total - first < (uint32_t)kMergeThreads ? (int)(total - first) : kMergeThreads;
    Entry e{};
    if ((int)threadIdx.x < count) e = exit_at(exits, off, n, first + threadIdx.x);
    const uint32_t got = merge_round(m, el, er, T, count, e, out + (size_t)blockIdx.x * kExitCap);
    if (threadIdx.x == 0) counts[blockIdx.x] = got;
}

// The n blocks' exits to the root, 1024 at a time: the exits of a round's
// pieces, one after the other, are the entries of the next round (in the
// buffers ping and pong by turns).  A round leaves at most 194 of 1024 entries.
__global__ __launch_bounds__(kMergeThreads) void k_tree_top(TreeOut T, const Entry *exits, const uint32_t *counts, uint32_t n,
                                                            uint32_t *off, Entry *ping, Entry *pong)
{
    __shared__ MergeLds m;
    __shared__ uint32_t el[kMergeThreads], er[kMergeThreads];
    block_offsets(counts, n, off, m.wsum);
    uint32_t total = off[n];
    for (int round = 0; total > 0u; ++round) {
        const Entry *in = (round & 1) ? ping : pong;
        Entry *out = (round & 1) ? pong : ping;
        uint32_t left = 0u;
        for (uint32_t first = 0; first < total; first += kMergeThreads) {
            const int count = total - first < (uint32_t)kMergeThreads ? (int)(total - first) : kMergeThreads;
            Entry e{};
            if ((int)threadIdx.x < count) e = round == 0 ? exit_at(exits, off, n, first + threadIdx.x) : in[first + threadIdx.x];
            left += merge_round(m, el, er, T, count, e, out + left);
        }
        total = left;   // 0 once the root is made
        __threadfence_block();
        __syncthreads();
    }
}

}  // namespace

// Words of the sort's state in SceneDev::hist (api.hip sizes it): the key
// blocks' digit rows, the digits' places, the passes' tickets, and per pass and
// tile 256 look-back words.
// Larger tiles look back over fewer others and store longer runs, smaller ones
// fill more of the chip: 1.94 M references build in 455, 490, 570 us with tiles
// of 8192, 4096, 2048 keys, 0.5 M in 255, 238, 250, 60 000 in 162, 141, 126.
int sort_tile(int64_t n) { return n > 1024 * 1024 ? 8192 : (n > 128 * 1024 ? 4096 : 2048); }

int64_t sort_words(int64_t n)
{
    const int64_t rows = std::min<int64_t>(kKeyBlocks, (n + kKeyThreads - 1) / kKeyThreads);
    // grows with n, also where the tile does
    const int64_t tiles = std::max(std::max((n + 8191) / 8192, std::min<int64_t>(256, (n + 4095) / 4096)),
                                   std::min<int64_t>(64, (n + 2047) / 2048));
    return (rows + 1) * (kPasses * 256) + 64 + kPasses * 256 * tiles;
}

// Bytes of SceneDev::keys_tmp: the sort's second key buffer, then the exits of
// the tree's blocks and, for k_tree_top, those of its first two rounds.
constexpr int64_t kExits = 194;   // most exits of a block

int64_t top_records(int64_t blocks) { return (std::min<int64_t>(blocks, kTopBlocks) * kExits + kMergeThreads - 1) / kMergeThreads * kExits; }

int64_t keys_tmp_bytes(int64_t n)
{
    const int64_t blocks = (n + kMergeThreads - 1) / kMergeThreads;
    return (int64_t)sizeof(Entry) * (blocks * kExitCap + 2 * top_records(blocks));
}

hipError_t launch_build_bvh(SceneDev &s, hipStream_t st)
{
    const int nt = s.ntri, n = s.nleaf;
    if (n <= kSmallRefs) {
        k_small_sort<<<1, kSmallThreads, 0, st>>>(s.verts_in, nt, s.ref_off, s.refs, n, s.keys, s.ids);
    } else {
        const int rows = std::min(kKeyBlocks, ceil_div(n, kKeyThreads));
        uint32_t *row = s.hist, *first = row + (size_t)rows * (kPasses * 256), *ticket = first + kPasses * 256, *words = ticket + 64;
        const int tiles = ceil_div(n, sort_tile(n));
        const int nb = std::min(s.bound_blocks, ceil_div(nt, kThreads));
        k_emit<<<nb, kThreads, 0, st>>>(s.verts_in, nt, s.ref_off, s.refs, s.bounds, ticket,
                                        64 + (int64_t)kPasses * 256 * tiles);
        k_keys<<<rows, kKeyThreads, 0, st>>>(s.refs, n, s.bounds, nb, s.keys, s.ids, row);
        k_digit_places<<<kPasses, 1024, 0, st>>>(row, rows, first);
        uint64_t *ka = s.keys, *kb = s.keys_tmp;
        uint32_t *va = s.ids, *vb = s.ids_tmp;
        for (int p = 0; p < kPasses; ++p) {
            uint32_t *w = words + (size_t)p * 256 * tiles;
            auto pass = [&](auto kern, int threads) {
                kern<<<tiles, threads, 0, st>>>(ka, va, kb, vb, n, 8 * p, first + 256 * p, ticket + p, w);
            };
            if (sort_tile(n) == 8192) pass(k_sort_pass<16, 8>, 1024);
            else if (sort_tile(n) == 4096) pass(k_sort_pass<8, 8>, 512);
            else pass(k_sort_pass<8, 4>, 512);
            std::swap(ka, kb);
            std::swap(va, vb);
        }
    }
    // the sort is over: its second buffers hold the exits, its state their counts
    const TreeOut T{s.keys, s.ids, n, s.nodes, s.nodes16, s.parent};
    const int blocks = ceil_div(n, kMergeThreads);
    Entry *exits = reinterpret_cast<Entry *>(s.keys_tmp), *exits2 = reinterpret_cast<Entry *>(s.ids_tmp);
    uint32_t *counts = s.hist, *off = counts + blocks;
    k_tree_blocks<<<blocks, kMergeThreads, 0, st>>>(s.verts_in, s.albedo_in, s.refs, T, s.tris, s.albedo, exits, counts);
    if (blocks > kTopBlocks) {
        const int merges = ceil_div((int64_t)blocks * kExits, kMergeThreads);
        uint32_t *counts2 = off + blocks + 1, *off2 = counts2 + merges;
        k_exit_offsets<<<1, kMergeThreads, 0, st>>>(counts, (uint32_t)blocks, off);
        k_tree_merge<<<merges, kMergeThreads, 0, st>>>(T, exits, off, (uint32_t)blocks, exits2, counts2);
        Entry *pong = exits + (size_t)kExitCap * ceil_div(merges, 2);
        k_tree_top<<<1, kMergeThreads, 0, st>>>(T, exits2, counts2, (uint32_t)merges, off2, exits, pong);
    } else if (blocks > 1) {
        Entry *ping = exits + (size_t)blocks * kExitCap;
        k_tree_top<<<1, kMergeThreads, 0, st>>>(T, exits, counts, (uint32_t)blocks, off, ping, ping + top_records(blocks));
    }
    return hipGetLastError();
}

}  // namespace dof
