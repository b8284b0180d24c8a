// Per-frame kernels of the hybrid depth-of-field pass, except the ray
// traversal (trace.hip).  Stage names follow section 3 of the paper:
//   A1  CoC + half-res reduce (+ per-tile max CoC)          3.1, 3.3 eq. 6
//   A2  tile-neighbourhood max CoC                          3.1.1
//   A3  9-tap bilateral prefilter                           3.1.1
//   A4  81-tap near/far gather, eq. (1)                     3.1.2
//   A5  3x3 median postfilter                               3.1.3
//   A6  ray mask, eqs. (2)-(4)                              3.2.1
//   A7  ordered compaction of masked pixels into a queue    (GPU dispatch)
//   A11 near/far resolve and hit ratio                      3.2.2
//   A12 temporal accumulation, reprojection, variance       3.2.3
//   A13 median, mip chain, spatial reconstruction, eq. (5)(8)  3.2.4
//   A14 composite, eqs. (6)(7)                              3.3
// Every floating-point expression is evaluated in the order written, in
// binary32 without contraction, so that index decisions (nearest texels,
// ray counts) are reproducible.
#include "dof_internal.h"

namespace dof {
namespace {

constexpr int kBX = 64, kBY = 4;   // pixel-kernel block: one wave per row

// The dispatcher deals workgroups round-robin to the 8 XCDs (workgroup i to
// XCD i mod 8), each with its own L2.  xcd_tile renumbers the tiles of a 2-D
// grid so that XCD x takes one contiguous run of them in row-major order:
// neighbouring tiles, whose tap footprints overlap, then share one L2 instead
// of fetching the same halo into several.  A bijection for any grid size, so
// only the order of the work changes.  Worth it for the wide, uniform-cost
// gather and for the mask (1920x1080 17.0 -> 15.5 us); kernels whose cost
// follows the ray mask keep the interleaved order, which spreads expensive
// regions over all XCDs, and so do those that the memory bounds, which bands
// spread unevenly over its channels (3840x2160: composite 78 -> 83 us, blur,
// median and mips 62 -> 71).
__device__ inline void xcd_tile(uint32_t &bx, uint32_t &by)
{
    const uint32_t gx = gridDim.x, n = gridDim.x * gridDim.y;
    const uint32_t id = blockIdx.x + blockIdx.y * gx;
    const uint32_t x = id % 8u, s = id / 8u, per = n / 8u, rem = n % 8u;
    const uint32_t t = x * per + (x < rem ? x : rem) + s;
    bx = t % gx;
    by = t / gx;
}

// The same for a batch's blocks, a 1-D grid over all of its items.
__device__ inline uint32_t xcd_block()
{
    const uint32_t n = gridDim.x, x = blockIdx.x % 8u, s = blockIdx.x / 8u, per = n / 8u, rem = n % 8u;
    return x * per + (x < rem ? x : rem) + s;
}

__device__ inline float4 ld_rgba(const void *p, int fmt, size_t i)
{
    if (fmt == DOF_RGBA32F) return reinterpret_cast<const float4 *>(p)[i];
    const __half *h = reinterpret_cast<const __half *>(p) + 4 * i;
    return make_float4(__half2float(h[0]), __half2float(h[1]), __half2float(h[2]), __half2float(h[3]));
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

__device__ inline float4 lerp4(float4 a, float4 b, float t)
{
    return make_float4(a.x + (b.x - a.x) * t, a.y + (b.y - a.y) * t, a.z + (b.z - a.z) * t, a.w + (b.w - a.w) * t);
}

__device__ inline float4 bilinear4(const float4 *img, int w, int h, float x, float y)
{
    float x0f = floorf(x), y0f = floorf(y);
    float fx = x - x0f, fy = y - y0f;
    int x0 = (int)x0f, y0 = (int)y0f;
    int x1 = clampi(x0 + 1, 0, w - 1), y1 = clampi(y0 + 1, 0, h - 1);
    x0 = clampi(x0, 0, w - 1);
    y0 = clampi(y0, 0, h - 1);
    // 32-bit texel indices: a frame has at most 2^30 pixels
    const float4 *r0 = img + (uint32_t)(y0 * w), *r1 = img + (uint32_t)(y1 * w);
    float4 a = r0[x0], b = r0[x1];
    float4 c = r1[x0], d = r1[x1];
    return lerp4(lerp4(a, b, fx), lerp4(c, d, fx), fy);
}

__device__ inline int nearest_idx(float s, int n) { return clampi((int)floorf(s + 0.5f), 0, n - 1); }

// Median of 9 by a max-min exchange network (19 compare-exchanges).
__device__ inline float median9(float p0, float p1, float p2, float p3, float p4, float p5, float p6, float p7,
                                float p8)
{
#define DOF_CX(a, b)                  \
    {                                 \
        float lo_ = fmin_cs(a, b);    \
        float hi_ = fmax_cs(a, b);    \
        a = lo_;                      \
        b = hi_;                      \
    }
    DOF_CX(p1, p2); DOF_CX(p4, p5); DOF_CX(p7, p8);
    DOF_CX(p0, p1); DOF_CX(p3, p4); DOF_CX(p6, p7);
    DOF_CX(p1, p2); DOF_CX(p4, p5); DOF_CX(p7, p8);
    DOF_CX(p0, p3); DOF_CX(p5, p8); DOF_CX(p4, p7);
    DOF_CX(p3, p6); DOF_CX(p1, p4); DOF_CX(p2, p5);
    DOF_CX(p4, p7); DOF_CX(p4, p2); DOF_CX(p6, p4);
    DOF_CX(p4, p2);
#undef DOF_CX
    return p4;
}

// Half-res texel of the previous view that sees p (a direction when is_dir).
__device__ inline int reproject(const ViewConst &pv, int hw, int hh, const float p[3], bool is_dir)
{
    float e[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) e[a] = is_dir ? p[a] : p[a] - pv.pos[a];
    float ex = (e[0] * pv.right[0] + e[1] * pv.right[1]) + e[2] * pv.right[2];
    float ey = (e[0] * pv.up[0] + e[1] * pv.up[1]) + e[2] * pv.up[2];
    float ez = (e[0] * pv.fwd[0] + e[1] * pv.fwd[1]) + e[2] * pv.fwd[2];
    if (!(ez > 0.0f)) return -1;
    float pu = (ex / ez) / pv.tanx;
    float pvv = (ey / ez) / pv.tany;
    float px = ((pu + 1.0f) * 0.5f) * (float)hw - 0.5f;
    float py = ((1.0f - pvv) * 0.5f) * (float)hh - 0.5f;
    float sx = px + 0.5f, sy = py + 0.5f;
    if (!(sx >= 0.0f && sx < (float)hw && sy >= 0.0f && sy < (float)hh)) return -1;
    return (int)floorf(sy) * hw + (int)floorf(sx);
}

// History planes: A (near rgb, h) | B (far rgb, age) | C (cN, cF, mu1, mu2) | D var
struct Hist {
    const float4 *A, *B, *C;
    const float *D;
};
struct HistW {
    float4 *A, *B, *C;
    float *D;
};
__device__ inline Hist hist_view(const void *h, size_t np)
{
    const float4 *p = reinterpret_cast<const float4 *>(h);
    return Hist{p, p + np, p + 2 * np, reinterpret_cast<const float *>(p + 3 * np)};
}
__device__ inline HistW hist_wview(void *h, size_t np)
{
    float4 *p = reinterpret_cast<float4 *>(h);
    return HistW{p, p + np, p + 2 * np, reinterpret_cast<float *>(p + 3 * np)};
}

}  // namespace

Planes planes(const FrameConst &fc, const ScratchLayout &L, char *s)
{
    size_t np = (size_t)fc.hw * fc.hh;
    Planes p;
    p.colr = reinterpret_cast<float4 *>(s + L.colr);
    p.zn = reinterpret_cast<float4 *>(s + L.zn);
    p.zh = reinterpret_cast<float *>(s + L.zh);
    p.tile_max = reinterpret_cast<float *>(s + L.tile_max);
    p.tile_dil = reinterpret_cast<float *>(s + L.tile_dil);
    p.pre = reinterpret_cast<float4 *>(s + L.pre);
    p.gather = reinterpret_cast<float4 *>(s + L.gather);
    p.ppmed = reinterpret_cast<float4 *>(s + L.ppmed);
    p.prev_idx = reinterpret_cast<int32_t *>(s + L.prev_idx);
    p.chunk_cnt = reinterpret_cast<uint2 *>(s + L.chunk_cnt);
    p.counters = reinterpret_cast<uint32_t *>(s + L.counters);
    p.queue = reinterpret_cast<uint32_t *>(s + L.queue);
    p.ray_base = reinterpret_cast<uint32_t *>(s + L.ray_base);
    p.ray_pix = reinterpret_cast<uint32_t *>(s + L.ray_pix);
    const bool rec = fc.ray_records != 0;
    p.ray_hit = rec ? reinterpret_cast<int32_t *>(s + L.ray_hit) : nullptr;
    p.ray_t = rec ? reinterpret_cast<float *>(s + L.ray_t) : nullptr;
    p.ray_col = rec ? reinterpret_cast<float4 *>(s + L.ray_col) : nullptr;
    p.ray_pos = rec ? reinterpret_cast<float4 *>(s + L.ray_pos) : nullptr;
    const size_t nr = np * (size_t)fc.m;
    p.rec0 = reinterpret_cast<float4 *>(s + L.ray_rec);
    p.rec1 = reinterpret_cast<float2 *>(p.rec0 + nr);
    p.ray_lt = reinterpret_cast<uint2 *>(s + L.ray_lt);
    float4 *res = reinterpret_cast<float4 *>(s + L.resolve);
    p.R0 = res; p.R1 = res + np; p.R2 = res + 2 * np; p.R3 = res + 3 * np;
    float4 *tmp = reinterpret_cast<float4 *>(s + L.temporal);
    p.T0 = tmp; p.T1 = tmp + np;
    p.var_blur = reinterpret_cast<float *>(s + L.var_blur);
    p.rtmed = reinterpret_cast<float4 *>(s + L.rtmed);
    p.mips = reinterpret_cast<float4 *>(s + L.mips);
    p.tap = reinterpret_cast<float2 *>(s + L.tap);
    p.gtex = reinterpret_cast<float4 *>(s + L.gtex);
    p.mask_raw = reinterpret_cast<uint8_t *>(s + L.mask_raw);
    p.comp = (fc.taa & DOF_TAA_FINAL) ? reinterpret_cast<float4 *>(s + L.comp) : nullptr;
    p.rast = (fc.taa & DOF_TAA_RASTER) ? reinterpret_cast<float4 *>(s + L.rast) : nullptr;
    p.pptaa = (fc.taa & DOF_TAA_POST) ? reinterpret_cast<float4 *>(s + L.pptaa) : nullptr;
    p.ppout = (fc.taa & DOF_TAA_POST) ? p.pptaa : p.ppmed;
    p.recon = reinterpret_cast<float4 *>(s + L.recon);
    return p;
}

dof_gbuffer resolved_gbuffer(const FrameConst &fc, const Planes &P, const dof_gbuffer &gb)
{
    dof_gbuffer g = gb;
    if (fc.taa & DOF_TAA_RASTER) {
        g.colour = P.rast;
        g.colour_format = DOF_RGBA32F;
    }
    return g;
}

namespace {


// ---------------------------------------------------------------- A1

__device__ inline void b_reduce(const FrameConst &fc, const dof_gbuffer &gb, const Planes &P, const uint32_t bx, const uint32_t by)
{
    const int x = bx * kTile + threadIdx.x, y = by * kTile + threadIdx.y;
    float ar = 0.0f;
    if (x < fc.hw && y < fc.hh) {
        const size_t W = (size_t)fc.W;
        size_t t[4] = {(size_t)(2 * y) * W + 2 * x, (size_t)(2 * y) * W + 2 * x + 1,
                       (size_t)(2 * y + 1) * W + 2 * x, (size_t)(2 * y + 1) * W + 2 * x + 1};
        float zz[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) zz[k] = gb.depth[t[k]];
        int sel = 0;
        float z = zz[0];
        if (zz[1] < z) { z = zz[1]; sel = 1; }
        if (zz[2] < z) { z = zz[2]; sel = 2; }
        if (zz[3] < z) { z = zz[3]; sel = 3; }
        float4 c0 = ld_rgba(gb.colour, gb.colour_format, t[0]), c1 = ld_rgba(gb.colour, gb.colour_format, t[1]);
        float4 c2 = ld_rgba(gb.colour, gb.colour_format, t[2]), c3 = ld_rgba(gb.colour, gb.colour_format, t[3]);
        size_t ts = sel == 0 ? t[0] : (sel == 1 ? t[1] : (sel == 2 ? t[2] : t[3]));
        float4 nn = ld_rgba(gb.normal, gb.normal_format, ts);
        float r = coc_px(fc.cock, fc.d, z) * 0.25f;
        r = fmin_cs(r, fc.r_max);
        r = z < fc.d ? -r : r;
        size_t i = (size_t)y * fc.hw + x;
        P.colr[i] = make_float4(((c0.x + c1.x) + (c2.x + c3.x)) * 0.25f, ((c0.y + c1.y) + (c2.y + c3.y)) * 0.25f,
                                ((c0.z + c1.z) + (c2.z + c3.z)) * 0.25f, r);
        P.zn[i] = make_float4(z, nn.x, nn.y, nn.z);
        P.zh[i] = z;
        ar = fabsf(r);
    }
    // per-tile maximum |r| (tile == block)
    __shared__ float red[4];
    const int tid = threadIdx.y * kTile + threadIdx.x;
    for (int o = 32; o >= 1; o >>= 1) ar = fmax_cs(ar, __shfl_xor(ar, o));
    if ((tid & 63) == 0) red[tid >> 6] = ar;
    __syncthreads();
    if (tid == 0) {
        float m = 0.0f;
        for (int k = 0; k < 4; ++k) m = fmax_cs(m, red[k]);
        P.tile_max[(size_t)by * fc.tw + bx] = m;
    }
}

__global__ __launch_bounds__(256) void k_reduce(FrameConst fc, dof_gbuffer gb, Planes P)
{
    b_reduce(fc, gb, P, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void kb_reduce(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridTiles, blockIdx.x, bx, by)];
    b_reduce(J.fc, J.gb, J.P, bx, by);
}

// ---------------------------------------------------------------- A2

__device__ inline void b_dilate(const FrameConst &fc, const Planes &P, const uint32_t bx, const uint32_t by)
{
    const int tx = bx * blockDim.x + threadIdx.x, ty = by * blockDim.y + threadIdx.y;
    if (tx >= fc.tw || ty >= fc.th) return;
    float m = 0.0f;
    for (int j = ty - fc.D; j <= ty + fc.D; ++j)
        for (int i = tx - fc.D; i <= tx + fc.D; ++i)
            if (i >= 0 && j >= 0 && i < fc.tw && j < fc.th) m = fmax_cs(m, P.tile_max[(size_t)j * fc.tw + i]);
    P.tile_dil[(size_t)ty * fc.tw + tx] = m;
}

__global__ void k_dilate(FrameConst fc, Planes P)
{
    b_dilate(fc, P, blockIdx.x, blockIdx.y);
}

__global__ void kb_dilate(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridDilate, blockIdx.x, bx, by)];
    b_dilate(J.fc, J.P, bx, by);
}

// ---------------------------------------------------------------- A3

// One block per 16 x 16 tile, whose tap spacing follows the tile's dilated
// radius: the texels that its 9 bilinear taps reach are staged in LDS (up to
// 28 x 28, tap distances to 5 texels; else they are read in global memory).
// dilate: the tile's dilated radius is found, and stored, here.  Bound by
// vector arithmetic, nine divisions a pixel among it; with its 36 texels a
// pixel read from the L1, and the dilation a launch of its own, a batch of
// eight frames of 1280x720 to 2560x1440 took 2565 us instead of 2544, a
// 1920x1080 frame 437 instead of 434.
constexpr int kPreLds = 28 * 28;

// The two texels of a bilinear tap's axis and the weight of the second, as
// bilinear4 takes them.
struct TapAxis {
    int a, b;
    float f;
};

__device__ inline TapAxis tap_axis(float s, int n)
{
    const float s0 = floorf(s);
    const int i = (int)s0;
    return {clampi(i, 0, n - 1), clampi(i + 1, 0, n - 1), s - s0};
}

__device__ inline void b_prefilter(const FrameConst &fc, const Planes &P, bool dilate, const uint32_t bx, const uint32_t by)
{
    __shared__ float4 tex[kPreLds];
    __shared__ float s_rn;
    const int tid = threadIdx.x, hw = fc.hw, hh = fc.hh;
    const int x0 = (int)bx * kTile, y0 = (int)by * kTile, x = x0 + tid % kTile, y = y0 + tid / kTile;
    const size_t tile = (size_t)by * fc.tw + bx;
    float Rn;
    if (dilate) {
        if (tid < 64) {
            const int i0 = max((int)bx - fc.D, 0), i1 = min((int)bx + fc.D, fc.tw - 1);
            const int j0 = max((int)by - fc.D, 0), j1 = min((int)by + fc.D, fc.th - 1), w = i1 - i0 + 1;
            float m = 0.0f;
            const int cells = fc.D >= 0 ? w * (j1 - j0 + 1) : 0;
            for (int e = tid; e < cells; e += 64) m = fmax_cs(m, P.tile_max[(size_t)(j0 + e / w) * fc.tw + i0 + e % w]);
            for (int o = 32; o >= 1; o >>= 1) m = fmax_cs(m, __shfl_xor(m, o));
            if (tid == 0) {
                s_rn = m;
                P.tile_dil[tile] = m;
            }
        }
        __syncthreads();
        Rn = s_rn;
    } else {
        Rn = P.tile_dil[tile];
    }
    float dpre = Rn * 0.25f;
    if (dpre < kSqrt2) dpre = kSqrt2;
    const float sp = dpre * 0.5f;
    // the texels between the outermost taps' (floor and clamp are monotone)
    const int wx = min(x0 + kTile - 1, hw - 1), wy = min(y0 + kTile - 1, hh - 1);
    const int bx0 = tap_axis((float)x0 - sp, hw).a, bx1 = tap_axis((float)wx + sp, hw).b;
    const int by0 = tap_axis((float)y0 - sp, hh).a, by1 = tap_axis((float)wy + sp, hh).b;
    const int bw = bx1 - bx0 + 1;
    // (while the coordinates are integers' too: a spacing of 2^31 wraps the
    // second texel's index round to the first)
    const bool staged = sp < 1073741824.0f && bw <= 28 && by1 - by0 + 1 <= 28;
    if (staged) {
        // 32 columns (28 at most in use) by 8 rows at a time
        const int c = tid & 31;
        if (c < bw)
            for (int r = tid >> 5; r <= by1 - by0; r += 8) tex[r * bw + c] = P.colr[(size_t)(by0 + r) * hw + bx0 + c];
    }
    __syncthreads();
    if (x >= hw || y >= hh) return;
    const size_t i = (size_t)y * hw + x;
    TapAxis tx[3], ty[3];
    for (int k = 0; k < 3; ++k) {
        tx[k] = tap_axis((float)x + (float)(k - 1) * sp, hw);
        ty[k] = tap_axis((float)y + (float)(k - 1) * sp, hh);
    }
    float ax = 0.0f, ay = 0.0f, az = 0.0f, sw = 0.0f;
    auto taps = [&](const float4 *img, int row, int ox, int oy) __attribute__((always_inline)) {
        const float rc = img[(size_t)(y - oy) * row + (x - ox)].w;
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
            const float4 *r0 = img + (size_t)(ty[dy].a - oy) * row, *r1 = img + (size_t)(ty[dy].b - oy) * row;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const int ca = tx[dx].a - ox, cb = tx[dx].b - ox;
                const float4 v = lerp4(lerp4(r0[ca], r0[cb], tx[dx].f), lerp4(r1[ca], r1[cb], tx[dx].f), ty[dy].f);
                const float w = 1.0f / (1.0f + fabsf(v.w - rc));
                ax = ax + w * v.x;
                ay = ay + w * v.y;
                az = az + w * v.z;
                sw = sw + w;
            }
        }
        return rc;
    };
    const float rc = staged ? taps(tex, bw, bx0, by0) : taps(P.colr, hw, 0, 0);
    const float4 pre = make_float4(ax / sw, ay / sw, az / sw, rc);
    P.pre[i] = pre;
    // the texel as the gather's taps read it, one 16-byte load: colour, the
    // radius's magnitude (the only part the gather uses) and, in its sign
    // bit, whether the pixel counts as a bright (specular) sample of the
    // bokeh share
    const bool bright = luma709(pre.x, pre.y, pre.z) > fc.l_spec;
    P.gtex[i] = make_float4(pre.x, pre.y, pre.z, __uint_as_float(__float_as_uint(fabsf(rc)) | (bright ? 0x80000000u : 0u)));
}

__global__ __launch_bounds__(256) void k_prefilter(FrameConst fc, Planes P, bool dilate)
{
    b_prefilter(fc, P, dilate, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void kb_prefilter(const Job *__restrict__ jobs, int njobs, bool dilate)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridTiles, blockIdx.x, bx, by)];
    b_prefilter(J.fc, J.P, dilate, bx, by);
}

// ---------------------------------------------------------------- A4

// One block of 256 threads per 16 x 16 tile of half-res pixels, the tile of
// the neighbourhood-maximum CoC, so the kernel radius R_n and with it every
// tap offset is the same for the whole block.  Each tap's texel column
// (per pixel column of the tile) and row (per pixel row) are computed once
// per block into LDS tables, with the same binary32 operations as the
// per-pixel definition, so the nearest-texel decisions are identical.  Each
// tap is one 16-byte load of the prefilter's gather texel (colour, radius
// magnitude, bright flag).  Optionally (launch knob gather_window) a tile
// whose taps stay within a win x win texel window first stages that window
// (texels and depths) in LDS and reads its taps there, in a kernel of its
// own; the other tiles read their taps from global memory (L1/L2) in a
// kernel that needs little LDS and so keeps many waves resident.  On the
// 1080p and 4K workloads the global reads are faster (the tiles that fit a
// window are the ones whose centres need the depth term, and the staging
// kernel holds fewer waves), so no staging is the default.
//
// Per tap, with D_fg = [|r_i| > dist] and D_bg = D_fg and [|r_c| > dist]:
// the two weights of eq. (1) add up to alpha when D_bg holds (foreground and
// background shares of one tap), to alpha (1 - w_bg) when only D_fg holds,
// and to 0 otherwise, so one weighted sum replaces the two and w_bg (with its
// division) is evaluated only where it matters.  Sums are reassociated
// relative to the per-pixel definition (tolerance parity); the weights'
// zero/non-zero pattern, and so the empty-kernel fallback, is unchanged.
// Whether a tile's taps fit a win x win texel window (win 0: no staging).
__device__ inline bool gather_fits(float Rn, int win) { return win > 0 && kTile + 2 * ((int)ceilf(Rn) + 1) <= win; }

// The taps of one ring (one distance): kBg when some lane of the wave has a
// centre radius at or below the ring's distance, so that its background taps
// need w_bg (a wave-uniform choice; the depth load and the division run only
// then).  sampleAlpha = 1 / max(|r|, 1/2)^2 with a hardware reciprocal
// (weights are normalised by their sum; tolerance parity).
//
// The depth term sat((zi - zc) / range) divides by a frame's constant: with its
// correctly rounded reciprocal, a product and two fused steps round the
// quotient as the division does (Markstein); kBg = kBgDivide divides, for
// ranges whose reciprocal could leave the normal numbers.  Distances beyond
// the range are cut to it, so an infinite one (the sky) gives 1 and no NaN, and
// what is no number (the sky's distance to itself) gives 0 as before.  The
// depths of four taps are loaded together with their texels: each behind its
// own branch, they came one after the other, and the kernel alone took 244 us
// at 3840x2160 and 62 at 1920x1080, now 162 and 45.  Bound by the L1's data
// return (0.9 of the time) next to vector arithmetic (0.8 instructions a clock
// and CU).  Eight waves a SIMD and four taps at a time; eight taps at a time
// in 64 registers take 2142 us a frame at 3840x2160, in 101 2065, two at a
// time 2078, four 2036.
enum : int { kBgNone = 0, kBgFast = 1, kBgDivide = 2 };

template <bool kLds, int kBg>
__device__ inline void gather_ring(const Planes &P, const float4 *s_tex, const float *s_z, const short *ixt,
                                   const short *iyt, int hw, int k0, int k1, float dist, bool centre_far, float zc,
                                   float range, float range_inv, float &v0, float &v1, float &v2, float &sw, float &ss)
{
#pragma unroll 4
    for (int k = k0; k < k1; ++k) {
        const int ix = ixt[k * kTile], iy = iyt[k * kTile];
        float4 ci;
        uint32_t j = 0;
        if constexpr (kLds) {
            j = (uint32_t)(iy + ix);
            ci = s_tex[j];
        } else {
            j = __umul24((uint32_t)iy, (uint32_t)hw) + (uint32_t)ix;
            ci = P.gtex[j];
        }
        const float ari = fabsf(ci.w);
        const float mr = fmax_cs(ari, 0.5f);
        const float alpha = __builtin_amdgcn_rcpf(mr * mr);
        float wb = alpha;
        if constexpr (kBg != kBgNone) {
            const float zi = kLds ? s_z[j] : P.zh[j];
            float behind;
            if constexpr (kBg == kBgDivide) {
                behind = sat((zi - zc) / range);
            } else {
                float v = zi - zc;
                v = v > range ? range : v;
                const float q = v * range_inv, t = fmaf(fmaf(-q, range, v), range_inv, q);
                behind = t > 0.0f ? t : 0.0f;
            }
            const float wd = alpha * (1.0f - behind);
            wb = centre_far ? alpha : wd;
        }
        const float w = ari > dist ? wb : 0.0f;
        v0 = fmaf(w, ci.x, v0);
        v1 = fmaf(w, ci.y, v1);
        v2 = fmaf(w, ci.z, v2);
        sw = sw + w;
        ss = ss + ((__float_as_uint(ci.w) >> 31) ? w : 0.0f);
    }
}

// kWin > 0: the LDS variant for the tiles that fit a kWin window; kWin = 0:
// the global variant for the tiles that do not fit fc.gather_win.
template <int kWin>
__device__ inline void b_gather(const FrameConst &fc, const Rings &rings, const Planes &P, const uint32_t tx,
                                const uint32_t ty)
{
    constexpr bool kLds = kWin > 0;
    // per tap: the texel column of each pixel column of the tile and the
    // texel row (LDS variant: window row times window width) of each pixel row
    __shared__ short s_ix[kRingTaps * kTile], s_iy[kRingTaps * kTile];
    __shared__ float4 s_tex[kLds ? kWin * kWin : 1];
    __shared__ float s_z[kLds ? kWin * kWin : 1];
    const int tid = threadIdx.x;
    const int x0 = (int)tx * kTile, y0 = (int)ty * kTile;
    const float Rn = P.tile_dil[(size_t)ty * fc.tw + tx];
    if (gather_fits(Rn, kLds ? kWin : fc.gather_win) != kLds) return;   // the other variant takes this tile
    // every tap lies within ceil(R_n) + 1 texels of its pixel (ring offsets <= 1 kernel radius)
    const int C = (int)ceilf(Rn) + 1;
    const int wx0 = max(x0 - C, 0), wx1 = min(x0 + kTile - 1 + C, fc.hw - 1);
    const int wy0 = max(y0 - C, 0), wy1 = min(y0 + kTile - 1 + C, fc.hh - 1);
    const int ww = wx1 - wx0 + 1;
    for (int e = tid; e < kRingTaps * 2 * kTile; e += 256) {
        const int k = e / (2 * kTile), c = e % (2 * kTile);
        if (c < kTile) {
            const int ix = nearest_idx((float)(x0 + c) + rings.ox[k] * Rn, fc.hw);
            s_ix[k * kTile + c] = (short)(kLds ? clampi(ix, wx0, wx1) - wx0 : ix);
        } else {
            const int iy = nearest_idx((float)(y0 + c - kTile) + rings.oy[k] * Rn, fc.hh);
            s_iy[k * kTile + c - kTile] = (short)(kLds ? (clampi(iy, wy0, wy1) - wy0) * ww : iy);
        }
    }
    if constexpr (kLds) {
        // rows of the window, 64 texels wide at a time (kWin <= 64)
        static_assert(kWin <= 64, "one pass of 64 columns per window row");
        const int c = tid & 63;
        if (c < ww)
            for (int r = tid >> 6; r <= wy1 - wy0; r += 4) {
                const size_t j = (size_t)(wy0 + r) * fc.hw + (wx0 + c);
                s_tex[r * ww + c] = P.gtex[j];
                s_z[r * ww + c] = P.zh[j];
            }
    }
    __syncthreads();
    const int lx = tid & (kTile - 1), ly = tid / kTile;
    const int x = x0 + lx, y = y0 + ly;
    if (x >= fc.hw || y >= fc.hh) return;
    const size_t i = (size_t)y * fc.hw + x;
    const float4 c0 = P.pre[i];
    const float zc = P.zh[i], arc = fabsf(c0.w);
    float v0 = 0.0f, v1 = 0.0f, v2 = 0.0f, sw = 0.0f, ss = 0.0f;
    // 0: divide
    const float range_inv = fc.depth_range > 1e-30f && fc.depth_range < 1e30f ? 1.0f / fc.depth_range : 0.0f;
    // rings of 1, 8, 16, 24, 32 taps, each at one distance
    constexpr int kRingStart[6] = {0, 1, 9, 25, 49, 81};
#pragma unroll
    for (int ring = 0; ring < 5; ++ring) {
        const int k0 = kRingStart[ring], k1 = kRingStart[ring + 1];
        const float dist = Rn * rings.frac[k0];
        const bool centre_far = arc > dist;   // background taps need the centre's radius too
        auto taps = [&](auto bg) __attribute__((always_inline)) {
            gather_ring<kLds, decltype(bg)::value>(P, s_tex, s_z, s_ix + lx, s_iy + ly, fc.hw, k0, k1, dist, centre_far, zc,
                                                   fc.depth_range, range_inv, v0, v1, v2, sw, ss);
        };
        if (__all(centre_far)) taps(std::integral_constant<int, kBgNone>{});
        else if (range_inv != 0.0f) taps(std::integral_constant<int, kBgFast>{});
        else taps(std::integral_constant<int, kBgDivide>{});
    }
    float4 o;
    if (sw > 0.0f) o = make_float4(v0 / sw, v1 / sw, v2 / sw, ss / sw);
    else o = make_float4(c0.x, c0.y, c0.z, 0.0f);
    P.gather[i] = o;
}

template <int kWin>
__global__ __launch_bounds__(256, kWin == 0 ? 8 : 1) void k_gather(FrameConst fc, Rings rings, Planes P)
{
    // every tile costs about the same, so contiguous bands per XCD stay
    // balanced and neighbouring tiles share their halo in one L2
    uint32_t bx, by;
    xcd_tile(bx, by);
    b_gather<kWin>(fc, rings, P, bx, by);
}

template <int kWin>
__global__ __launch_bounds__(256, kWin == 0 ? 8 : 1) void kb_gather(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridTiles, blockIdx.x, bx, by)];
    b_gather<kWin>(J.fc, J.grings, J.P, bx, by);
}

// Both variants of the gather: the LDS one for tiles that fit the window,
// the global one for the rest (grid: the tiles, or the batch's tile blocks).
template <class Launch>
void launch_gather_pair(int win, Launch launch)
{
    switch (win) {
    case 32: launch(std::integral_constant<int, 32>{}); break;
    case 40: launch(std::integral_constant<int, 40>{}); break;
    case 48: launch(std::integral_constant<int, 48>{}); break;
    default: break;
    }
    launch(std::integral_constant<int, 0>{});
}

// ---------------------------------------------------------------- A5

__device__ inline void b_median_pp(const FrameConst &fc, const Planes &P, const uint32_t bx, const uint32_t by)
{
    const int x = bx * kBX + threadIdx.x, y = by * kBY + threadIdx.y;
    if (x >= fc.hw || y >= fc.hh) return;
    float4 v[9];
    int n = 0;
    for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx)
            v[n++] = P.gather[(size_t)clampi(y + dy, 0, fc.hh - 1) * fc.hw + clampi(x + dx, 0, fc.hw - 1)];
    const size_t i = (size_t)y * fc.hw + x;
    P.ppmed[i] = make_float4(median9(v[0].x, v[1].x, v[2].x, v[3].x, v[4].x, v[5].x, v[6].x, v[7].x, v[8].x),
                             median9(v[0].y, v[1].y, v[2].y, v[3].y, v[4].y, v[5].y, v[6].y, v[7].y, v[8].y),
                             median9(v[0].z, v[1].z, v[2].z, v[3].z, v[4].z, v[5].z, v[6].z, v[7].z, v[8].z),
                             v[4].w);
}

__global__ __launch_bounds__(kBX *kBY) void k_median_pp(FrameConst fc, Planes P)
{
    b_median_pp(fc, P, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kBX *kBY) void kb_median_pp(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridHalf, blockIdx.x, bx, by)];
    b_median_pp(J.fc, J.P, bx, by);
}

// ---------------------------------------------------------------- A6

constexpr int kMaskHalo = 4, kMaskL = kTile + 2 * kMaskHalo;   // 24 x 24 LDS cells

// The mask's filters, each a sum from 0 in tap order: (1, 4, 6, 4, 1) / 16,
// (1, 4, 6, 4, 1) and (-1, -2, 0, 2, 1).  A product by 1/16 or 1/4 is exact
// (below 2^-122 it is not, but such gradients' squares are 0), so the fused
// form rounds as product and sum would; 2 v and 4 v can overflow (the disparity
// of a depth below 2^-126 of the focus distance), which a fused step would hide.
__device__ inline float gauss5(float a, float b, float c, float d, float e)
{
    return fmaf(0.0625f, e, fmaf(0.25f, d, fmaf(0.25f, b, 0.0f + 0.0625f * a) + 0.375f * c));
}

__device__ inline float smooth5(float a, float b, float c, float d, float e)
{
    return ((((0.0f + a) + 4.0f * b) + 6.0f * c) + 4.0f * d) + e;
}

__device__ inline float diff5(float a, float b, float c, float d, float e)
{
    return ((((0.0f - a) - 2.0f * b) + 0.0f * c) + 2.0f * d) + e;
}

// One block per 16 x 16 tile.  Bound by vector arithmetic (no contraction: the
// ray counts are exact) and LDS reads.  The derivative filter as two passes
// instead of 25 cells read by every pixel, and two arrays of cells instead of
// three (eight blocks a CU instead of five): 3840x2160 70 -> 44 us.
__device__ inline void b_mask(const FrameConst &fc, const Planes &P, const void *hist_in, uint8_t *mask, const uint32_t bx, const uint32_t by)
{
    __shared__ float4 F[kMaskL][kMaskL];
    __shared__ float4 Hh[kMaskL][kMaskL];
    const int hw = fc.hw, hh = fc.hh;
    const int ox = bx * kTile - kMaskHalo, oy = by * kTile - kMaskHalo;
    const int tid = threadIdx.y * kTile + threadIdx.x;
    // Cells hold values at clamped coordinates; a coordinate g maps to cell g - origin.
    for (int c = tid; c < kMaskL * kMaskL; c += 256) {
        int lx = c % kMaskL, ly = c / kMaskL;
        int gx = clampi(ox + lx, 0, hw - 1), gy = clampi(oy + ly, 0, hh - 1);
        float4 v = P.zn[(size_t)gy * hw + gx];
        F[ly][lx] = make_float4(fc.d / v.x, v.y, v.z, v.w);
    }
    __syncthreads();
    for (int c = tid; c < kMaskL * kMaskL; c += 256) {
        int lx = c % kMaskL, ly = c / kMaskL;
        if (lx < 2 || lx >= kMaskL - 2) continue;
        int cx = clampi(ox + lx, 0, hw - 1);
        float4 v[5];
        for (int j = 0; j < 5; ++j) v[j] = F[ly][clampi(cx + j - 2, 0, hw - 1) - ox];
        Hh[ly][lx] = make_float4(gauss5(v[0].x, v[1].x, v[2].x, v[3].x, v[4].x), gauss5(v[0].y, v[1].y, v[2].y, v[3].y, v[4].y),
                                 gauss5(v[0].z, v[1].z, v[2].z, v[3].z, v[4].z), gauss5(v[0].w, v[1].w, v[2].w, v[3].w, v[4].w));
    }
    __syncthreads();
    for (int c = tid; c < kMaskL * kMaskL; c += 256) {
        int lx = c % kMaskL, ly = c / kMaskL;
        if (lx < 2 || lx >= kMaskL - 2 || ly < 2 || ly >= kMaskL - 2) continue;
        int cy = clampi(oy + ly, 0, hh - 1);
        float4 v[5];
        for (int j = 0; j < 5; ++j) v[j] = Hh[clampi(cy + j - 2, 0, hh - 1) - oy][lx];
        F[ly][lx] = make_float4(gauss5(v[0].x, v[1].x, v[2].x, v[3].x, v[4].x), gauss5(v[0].y, v[1].y, v[2].y, v[3].y, v[4].y),
                                gauss5(v[0].z, v[1].z, v[2].z, v[3].z, v[4].z), gauss5(v[0].w, v[1].w, v[2].w, v[3].w, v[4].w));
    }
    __syncthreads();
    // The derivative filter's two horizontal passes, once per cell (a pixel's
    // five rows of them are its column's): differences to F's cells, smoothing
    // to Hh's, once every cell's are read.
    constexpr int kCells = kTile * (kMaskL - 4), kMine = (kCells + 255) / 256;
    float4 dif[kMine], smo[kMine];
#pragma unroll
    for (int m = 0; m < kMine; ++m) {
        const int c = tid + m * 256, lx = kMaskHalo + c % kTile, ly = 2 + c / kTile;
        if (c < kCells) {
            float4 v[5];
            for (int k = 0; k < 5; ++k) v[k] = F[ly][clampi(min(ox + lx, hw - 1) + k - 2, 0, hw - 1) - ox];
            dif[m] = make_float4(diff5(v[0].x, v[1].x, v[2].x, v[3].x, v[4].x), diff5(v[0].y, v[1].y, v[2].y, v[3].y, v[4].y),
                                 diff5(v[0].z, v[1].z, v[2].z, v[3].z, v[4].z), diff5(v[0].w, v[1].w, v[2].w, v[3].w, v[4].w));
            smo[m] = make_float4(smooth5(v[0].x, v[1].x, v[2].x, v[3].x, v[4].x), smooth5(v[0].y, v[1].y, v[2].y, v[3].y, v[4].y),
                                 smooth5(v[0].z, v[1].z, v[2].z, v[3].z, v[4].z), smooth5(v[0].w, v[1].w, v[2].w, v[3].w, v[4].w));
        }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kMine; ++m) {
        const int c = tid + m * 256, lx = kMaskHalo + c % kTile, ly = 2 + c / kTile;
        if (c < kCells) {
            F[ly][lx] = dif[m];
            Hh[ly][lx] = smo[m];
        }
    }
    __syncthreads();
    const int x = bx * kTile + threadIdx.x, y = by * kTile + threadIdx.y;
    if (x >= hw || y >= hh) return;
    float gx[4], gy[4];
    {
        float4 dv[5], sv[5];
        for (int r = 0; r < 5; ++r) {
            const int ly = clampi(y + r - 2, 0, hh - 1) - oy;
            dv[r] = F[ly][x - ox];
            sv[r] = Hh[ly][x - ox];
        }
        const float axv[4] = {smooth5(dv[0].x, dv[1].x, dv[2].x, dv[3].x, dv[4].x), smooth5(dv[0].y, dv[1].y, dv[2].y, dv[3].y, dv[4].y),
                              smooth5(dv[0].z, dv[1].z, dv[2].z, dv[3].z, dv[4].z), smooth5(dv[0].w, dv[1].w, dv[2].w, dv[3].w, dv[4].w)};
        const float ayv[4] = {diff5(sv[0].x, sv[1].x, sv[2].x, sv[3].x, sv[4].x), diff5(sv[0].y, sv[1].y, sv[2].y, sv[3].y, sv[4].y),
                              diff5(sv[0].z, sv[1].z, sv[2].z, sv[3].z, sv[4].z), diff5(sv[0].w, sv[1].w, sv[2].w, sv[3].w, sv[4].w)};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            gx[c] = axv[c] * 0.0078125f;
            gy[c] = ayv[c] * 0.0078125f;
        }
    }
    float dd = sqrtf(gx[0] * gx[0] + gy[0] * gy[0]);
    float an = 0.0f;
    for (int c = 1; c < 4; ++c) an = an + (gx[c] * gx[c] + gy[c] * gy[c]);
    float dn = sqrtf(an);
    float xx = (dd + dn) * fc.s;
    float xn = sat(1.0f - 1.0f / (xx + 1.0f));
    const size_t i = (size_t)y * hw + x;
    const float z = P.zh[i];
    int pi = -1;
    const size_t np = (size_t)hw * hh;
    if (fc.have_hist) {
        float fv[3], Pw[3];
        pixel_dir(fc.cur, x, y, hw, hh, fv);
        bool isdir = !(z < INFINITY);
#pragma unroll
        for (int a = 0; a < 3; ++a) Pw[a] = isdir ? fv[a] : fc.cur.pos[a] + z * fv[a];
        pi = reproject(fc.prev, hw, hh, Pw, isdir);
        if (pi >= 0 && !(hist_view(hist_in, np).B[pi].w > 0.0f)) pi = -1;
    }
    P.prev_idx[i] = pi;
    float var_prev = pi >= 0 ? hist_view(hist_in, np).D[pi] : 0.0f;
    float xf = sat(xn + var_prev * fc.var_mask_w) * (float)fc.m;
    int cnt = (int)floorf(xf + 0.5f);
    int near_oof = (z < fc.d) && (coc_px(fc.cock, fc.d, z) > kSqrt2);
    int n = cnt > near_oof ? cnt : near_oof;
    if (n > fc.m) n = fc.m;
    if (fc.mask_mode == DOF_MASK_FIXED) n = n > 0 ? fc.m : 0;
    if (fc.mask_mode == DOF_MASK_ALL) n = fc.m;
    mask[i] = (uint8_t)n;
}

__global__ __launch_bounds__(256) void k_mask(FrameConst fc, Planes P, const void *hist_in, uint8_t *mask)
{
    uint32_t bx, by;
    xcd_tile(bx, by);
    b_mask(fc, P, hist_in, mask, bx, by);
}

__global__ __launch_bounds__(256) void kb_mask(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridTiles, xcd_block(), bx, by)];
    b_mask(J.fc, J.P, J.hist_in, J.fc.mask_mode == DOF_MASK_DILATE ? J.P.mask_raw : J.mask, bx, by);
}

// ---------------------------------------------------------------- A6, dilated (5.3)
// One block per 16 x 16 tile: the tile's window of raw counts (radius R =
// its dilated max CoC radius, rounded up) goes to LDS, then a horizontal and
// a vertical running maximum give each pixel the largest count within R.

constexpr int kDilMax = 32;
constexpr int kDilSide = kTile + 2 * kDilMax;

__device__ inline void b_mask_dilate(const FrameConst &fc, const Planes &P, uint8_t *mask, const uint32_t bx,
                                     const uint32_t by)
{
    __shared__ uint8_t win[kDilSide * kDilSide];
    __shared__ uint8_t hor[kDilSide * kTile];
    const int hw = fc.hw, hh = fc.hh, tid = threadIdx.y * kTile + threadIdx.x;
    const int R = min((int)ceilf(P.tile_dil[(size_t)by * fc.tw + bx]), kDilMax);
    const int S = kTile + 2 * R;
    const int ox = (int)bx * kTile - R, oy = (int)by * kTile - R;
    for (int c = tid; c < S * S; c += kTile * kTile) {
        const int gx = ox + c % S, gy = oy + c / S;
        win[c] = (gx >= 0 && gy >= 0 && gx < hw && gy < hh) ? P.mask_raw[(size_t)gy * hw + gx] : (uint8_t)0;
    }
    __syncthreads();
    for (int c = tid; c < S * kTile; c += kTile * kTile) {
        const int row = c / kTile, col = c % kTile;
        uint8_t m = 0;
        for (int k = 0; k <= 2 * R; ++k) m = max(m, win[row * S + col + k]);
        hor[row * kTile + col] = m;
    }
    __syncthreads();
    const int x = (int)bx * kTile + threadIdx.x, y = (int)by * kTile + threadIdx.y;
    if (x >= hw || y >= hh) return;
    uint8_t m = 0;
    for (int k = 0; k <= 2 * R; ++k) m = max(m, hor[(threadIdx.y + k) * kTile + threadIdx.x]);
    mask[(size_t)y * hw + x] = m;
}

__global__ __launch_bounds__(256) void k_mask_dilate(FrameConst fc, Planes P, uint8_t *mask)
{
    b_mask_dilate(fc, P, mask, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void kb_mask_dilate(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridTiles, blockIdx.x, bx, by)];
    b_mask_dilate(J.fc, J.P, J.mask, bx, by);
}

// ---------------------------------------------------------------- A7

constexpr int kPixLds = 4096;   // staged ray->pixel entries per 256-pixel round (16 rays per pixel)
// Chunks of 1024 pixels in row-major order; ranks from wave ballots (masked
// pixels) and wave prefix sums (rays), so the queue is ascending.

__device__ inline uint32_t wave_incl_scan(uint32_t v, int lane)
{
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t u = __shfl_up(v, o);
        if (lane >= o) v += u;
    }
    return v;
}

__device__ inline void b_compact_count(int64_t np, const uint8_t *__restrict__ mask, const Planes &P, const uint32_t bx, const uint32_t by)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    size_t base = (size_t)bx * kChunk;
    uint32_t cp = 0, cr = 0;
    for (int r = 0; r < kChunk / 256; ++r) {
        size_t i = base + (size_t)r * 256 + tid;
        uint32_t n = i < (size_t)np ? mask[i] : 0u;
        cp += n > 0u;
        cr += n;
    }
    for (int o = 32; o >= 1; o >>= 1) {
        cp += __shfl_xor(cp, o);
        cr += __shfl_xor(cr, o);
    }
    __shared__ uint32_t sp[4], sr[4];
    if (lane == 0) { sp[w] = cp; sr[w] = cr; }
    __syncthreads();
    if (tid == 0) P.chunk_cnt[bx] = make_uint2(sp[0] + sp[1] + sp[2] + sp[3], sr[0] + sr[1] + sr[2] + sr[3]);
}

__global__ __launch_bounds__(256) void k_compact_count(int64_t np, const uint8_t *__restrict__ mask, Planes P)
{
    // the traversal's counters start the frame at zero (the totals of the
    // compaction are written by its last scatter block)
    if (blockIdx.x == 0 && threadIdx.x < kWorkParts) {
        uint32_t *w = P.counters + kCntWork + threadIdx.x * kWorkStride;
        w[0] = 0u;
        for (int k = 0; k < kStatWords; ++k) w[kStatAt + k] = 0u;
        if (threadIdx.x == 0) P.counters[kCntWild] = 0u;
    }
    b_compact_count(np, mask, P, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void kb_compact_count(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridChunk, blockIdx.x, bx, by)];
    if (bx == 0 && threadIdx.x == 0) J.P.counters[kCntWild] = 0u;
    b_compact_count((int64_t)J.fc.hw * J.fc.hh, J.mask, J.P, bx, by);
}

__device__ inline void b_compact_scatter(int64_t np, const uint8_t *__restrict__ mask, const Planes &P, const uint32_t bx,
                                         const uint32_t by, uint2 start)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    __shared__ uint32_t wp[4], wr[4];
    __shared__ uint32_t runp, runr;
    __shared__ uint32_t s_pix[kPixLds];   // ray -> queue position of one round's rays
    if (tid == 0) {
        runp = start.x;
        runr = start.y;
    }
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    size_t base = (size_t)bx * kChunk;
    for (int r = 0; r < kChunk / 256; ++r) {
        size_t i = base + (size_t)r * 256 + tid;
        uint32_t n = i < (size_t)np ? mask[i] : 0u;
        uint64_t bal = __ballot(n > 0u);
        uint32_t rank = (uint32_t)__popcll(bal & lt);
        uint32_t incl = wave_incl_scan(n, lane);
        if (lane == 63) { wp[w] = (uint32_t)__popcll(bal); wr[w] = incl; }
        __syncthreads();
        uint32_t op = runp, orr = runr;
        const uint32_t rbase = runr, round_rays = wr[0] + wr[1] + wr[2] + wr[3];
        // the round's rays are one contiguous range: stage their pixel map in
        // LDS and store it coalesced (rounds with more rays store directly)
        const bool staged = round_rays <= (uint32_t)kPixLds;
        for (int k = 0; k < w; ++k) { op += wp[k]; orr += wr[k]; }
        if (n > 0u) {
            uint32_t pos = op + rank;
            uint32_t rb = orr + incl - n;
            P.queue[pos] = (uint32_t)i;
            P.ray_base[pos] = rb;
            if (staged) {
                for (uint32_t k = 0; k < n; ++k) s_pix[rb - rbase + k] = pos;
            } else {
                for (uint32_t k = 0; k < n; ++k) P.ray_pix[rb + k] = pos;
            }
        }
        __syncthreads();
        if (staged)
            for (uint32_t t = tid; t < round_rays; t += 256) P.ray_pix[rbase + t] = s_pix[t];
        if (tid == 0) {
            runp += wp[0] + wp[1] + wp[2] + wp[3];
            runr += wr[0] + wr[1] + wr[2] + wr[3];
        }
        __syncthreads();
    }
}

// The scatter finds its chunk's offsets itself, summing the counts of the
// chunks before it (whole numbers: the same offsets as a scan), so there is no
// scan launch; the last chunk's block writes the totals.
__device__ inline void b_scatter_chunk(int64_t np, const uint8_t *__restrict__ mask, const Planes &P, const uint32_t bx,
                                       const uint32_t by, const uint32_t nchunks)
{
    __shared__ uint32_t sp[4], sr[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t cp = 0, cr = 0;
    for (uint32_t i = (uint32_t)tid; i < bx; i += 256) {
        const uint2 c = P.chunk_cnt[i];
        cp += c.x;
        cr += c.y;
    }
    for (int o = 32; o >= 1; o >>= 1) {
        cp += __shfl_xor(cp, o);
        cr += __shfl_xor(cr, o);
    }
    if (lane == 0) { sp[w] = cp; sr[w] = cr; }
    __syncthreads();
    const uint2 start = make_uint2(sp[0] + sp[1] + sp[2] + sp[3], sr[0] + sr[1] + sr[2] + sr[3]);
    if (bx == nchunks - 1 && tid == 0) {
        const uint2 c = P.chunk_cnt[bx];
        P.counters[kCntMasked] = start.x + c.x;
        P.counters[kCntRays] = start.y + c.y;
    }
    b_compact_scatter(np, mask, P, bx, by, start);
}

__global__ __launch_bounds__(256) void k_compact_scatter(int64_t np, const uint8_t *__restrict__ mask, Planes P)
{
    b_scatter_chunk(np, mask, P, blockIdx.x, blockIdx.y, gridDim.x);
}

__global__ __launch_bounds__(256) void kb_compact_scatter(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridChunk, blockIdx.x, bx, by)];
    const int64_t np = (int64_t)J.fc.hw * J.fc.hh;
    b_scatter_chunk(np, J.mask, J.P, bx, by, (uint32_t)((np + kChunk - 1) / kChunk));
}

// ---------------------------------------------------------------- A11

// ---------------------------------------------------------------- A12

// A frame with a ray-traced colour beyond this (or none at all: NaN) is
// marked "wild": sums over its taps might not be finite.
constexpr float kTameColour = 1e18f;

__device__ inline void b_temporal(const FrameConst &fc, const Planes &P, const uint8_t *__restrict__ mask,
                                                       const void *hist_in, void *hist_out, const uint32_t bx, const uint32_t by)
{
    const int x = bx * kBX + threadIdx.x, y = by * kBY + threadIdx.y;
    const int hw = fc.hw, hh = fc.hh;
    if (x >= hw || y >= hh) return;
    const size_t np = (size_t)hw * hh, i = (size_t)y * hw + x;
    HistW ho = hist_wview(hist_out, np);
    const int n = mask[i];
    const float4 z4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (n == 0) {
        P.T0[i] = z4; P.T1[i] = z4;
        ho.A[i] = z4; ho.B[i] = z4; ho.C[i] = z4;
        return;
    }
    const float4 r0 = P.R0[i], r1 = P.R1[i], r2 = P.R2[i], r3 = P.R3[i];
    const float N = r0.w, hcur = r1.w, nf = (float)n - N;
    const int pn = P.prev_idx[i];
    const bool vn = pn >= 0;
    float fpos[3];
    bool fvalid = r3.w > 0.0f;
    if (fvalid) {
        fpos[0] = r3.x; fpos[1] = r3.y; fpos[2] = r3.z;
    } else {
        float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f;
        int cnt = 0;
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) {
                int xx = x + dx, yy = y + dy;
                if ((dx == 0 && dy == 0) || xx < 0 || yy < 0 || xx >= hw || yy >= hh) continue;
                size_t k = (size_t)yy * hw + xx;
                if (mask[k]) {
                    float4 q3 = P.R3[k];
                    if (q3.w > 0.0f) {
                        a0 = a0 + q3.x; a1 = a1 + q3.y; a2 = a2 + q3.z;
                        ++cnt;
                    }
                }
            }
        if (cnt > 0) {
            fpos[0] = a0 / (float)cnt; fpos[1] = a1 / (float)cnt; fpos[2] = a2 / (float)cnt;
            fvalid = true;
        }
    }
    Hist hi = hist_view(hist_in, np);
    int pf = -1;
    if (fc.have_hist && fvalid) {
        pf = reproject(fc.prev, hw, hh, fpos, false);
        if (pf >= 0 && !(hi.B[pf].w > 0.0f)) pf = -1;
    }
    const bool vf = pf >= 0;
    const float ah = fc.alpha_h;
    float4 hNa = vn ? hi.A[pn] : z4, hNb = vn ? hi.B[pn] : z4, hNc = vn ? hi.C[pn] : z4;
    float4 hFb = vf ? hi.B[pf] : z4, hFc = vf ? hi.C[pf] : z4;
    const float cur_n[3] = {r0.x, r0.y, r0.z}, cur_f[3] = {r1.x, r1.y, r1.z};
    const float hn_[3] = {hNa.x, hNa.y, hNa.z}, hf_[3] = {hFb.x, hFb.y, hFb.z};
    float accN[3], accF[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        accN[c] = N > 0.0f ? (vn ? lerp1(cur_n[c], hn_[c], ah) : cur_n[c]) : (vn ? hn_[c] : 0.0f);
        accF[c] = nf > 0.0f ? (vf ? lerp1(cur_f[c], hf_[c], ah) : cur_f[c]) : (vf ? hf_[c] : 0.0f);
    }
    float accCN = N > 0.0f ? (vn ? lerp1(r2.x, hNc.x, ah) : r2.x) : (vn ? hNc.x : 0.0f);
    float accCF = nf > 0.0f ? (vf ? lerp1(r2.y, hFc.y, ah) : r2.y) : (vf ? hFc.y : 0.0f);
    float accH = vn ? lerp1(hcur, hNa.w, ah) : hcur;
    float huse = fc.motion ? hcur : accH;
    float crt[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) crt[c] = lerp1(accF[c], accN[c], huse);
    float ct = lerp1(accCF, accCN, huse);
    float l = luma709(crt[0], crt[1], crt[2]);
    float mu1 = vn ? lerp1(l, hNc.z, ah) : l;
    float mu2 = vn ? lerp1(l * l, hNc.w, ah) : l * l;
    float v = mu2 - mu1 * mu1;
    v = v > 0.0f ? v : 0.0f;
    float age = vn ? hNb.w + 1.0f : 1.0f;
    // what lets the reconstruction skip pixels whose blend weight is 0 (every
    // lane stores the same value)
    if (!(fmaxf(fmaxf(fabsf(crt[0]), fabsf(crt[1])), fabsf(crt[2])) <= kTameColour) || crt[0] != crt[0] || crt[1] != crt[1] ||
        crt[2] != crt[2])
        P.counters[kCntWild] = 1u;
    P.T0[i] = make_float4(crt[0], crt[1], crt[2], 1.0f);
    P.T1[i] = make_float4(ct, huse, v, 0.0f);
    ho.A[i] = make_float4(accN[0], accN[1], accN[2], accH);
    ho.B[i] = make_float4(accF[0], accF[1], accF[2], age);
    ho.C[i] = make_float4(accCN, accCF, mu1, mu2);
}

__global__ __launch_bounds__(kBX *kBY) void k_temporal(FrameConst fc, Planes P, const uint8_t *__restrict__ mask,
                                                       const void *hist_in, void *hist_out)
{
    b_temporal(fc, P, mask, hist_in, hist_out, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kBX *kBY) void kb_temporal(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridHalf, blockIdx.x, bx, by)];
    b_temporal(J.fc, J.P, J.mask, J.hist_in, J.hist_out, bx, by);
}

// ---------------------------------------------------------------- A12 blur + A13 median, mips
// One wave per 8 x 8 tile: variance blur (3x3 binomial), 3x3 median of the
// ray-traced colour (invalid neighbours replaced by the centre), level 0 of
// the validity-weighted mip chain, then levels 1..3 of the tile from LDS;
// also the 8-byte record (CoC or -inf, hit ratio) that the reconstruction
// reads for each of its taps.

__device__ inline void b_blur_median_mips(const FrameConst &fc, const Planes &P, void *hist_out, const uint32_t bx, const uint32_t by)
{
    const int tx = threadIdx.x & 7, ty = threadIdx.x >> 3;
    const int x = bx * 8 + tx, y = by * 8 + ty;
    const int hw = fc.hw, hh = fc.hh;
    const size_t np = (size_t)hw * hh;
    __shared__ float4 m0[8][8];
    __shared__ float4 m1[4][4];
    __shared__ float4 m2[2][2];
    if (x < hw && y < hh) {
        const size_t i = (size_t)y * hw + x;
        const float g3[3] = {0.25f, 0.5f, 0.25f};
        float acc = 0.0f;
        for (int r = 0; r < 3; ++r) {
            size_t row = (size_t)clampi(y + r - 1, 0, hh - 1) * hw;
            float hs = 0.0f;
            for (int k = 0; k < 3; ++k) hs = hs + g3[k] * P.T1[row + clampi(x + k - 1, 0, hw - 1)].z;
            acc = acc + g3[r] * hs;
        }
        P.var_blur[i] = acc;
        hist_wview(hist_out, np).D[i] = acc;
        float4 c = P.T0[i];
        const float4 t1 = P.T1[i];
        P.tap[i] = make_float2(c.w > 0.0f ? t1.x : -INFINITY, t1.y);
        float4 med = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (c.w > 0.0f) {
            float4 v[9];
            int n = 0;
            for (int dy = -1; dy <= 1; ++dy)
                for (int dx = -1; dx <= 1; ++dx) {
                    float4 t = P.T0[(size_t)clampi(y + dy, 0, hh - 1) * hw + clampi(x + dx, 0, hw - 1)];
                    v[n++] = t.w > 0.0f ? t : c;
                }
            med = make_float4(median9(v[0].x, v[1].x, v[2].x, v[3].x, v[4].x, v[5].x, v[6].x, v[7].x, v[8].x),
                              median9(v[0].y, v[1].y, v[2].y, v[3].y, v[4].y, v[5].y, v[6].y, v[7].y, v[8].y),
                              median9(v[0].z, v[1].z, v[2].z, v[3].z, v[4].z, v[5].z, v[6].z, v[7].z, v[8].z),
                              1.0f);
        }
        P.rtmed[i] = med;
        float4 pm = make_float4(med.x * med.w, med.y * med.w, med.z * med.w, med.w);
        P.mips[fc.moff[0] + i] = pm;
        m0[ty][tx] = pm;
    }
    __syncthreads();
    // level 1 (4 x 4 of this tile)
    if (threadIdx.x < 16) {
        const int lx = threadIdx.x & 3, ly = threadIdx.x >> 2;
        const int gx = bx * 4 + lx, gy = by * 4 + ly;
        if (gx < fc.mw[1] && gy < fc.mh[1]) {
            int x0 = 2 * gx, y0 = 2 * gy, x1 = clampi(2 * gx + 1, 0, fc.mw[0] - 1), y1 = clampi(2 * gy + 1, 0, fc.mh[0] - 1);
            float4 a = m0[y0 - by * 8][x0 - bx * 8], b = m0[y0 - by * 8][x1 - bx * 8];
            float4 c = m0[y1 - by * 8][x0 - bx * 8], d = m0[y1 - by * 8][x1 - bx * 8];
            float4 o = make_float4(((a.x + b.x) + (c.x + d.x)) * 0.25f, ((a.y + b.y) + (c.y + d.y)) * 0.25f,
                                   ((a.z + b.z) + (c.z + d.z)) * 0.25f, ((a.w + b.w) + (c.w + d.w)) * 0.25f);
            P.mips[fc.moff[1] + (size_t)gy * fc.mw[1] + gx] = o;
            m1[ly][lx] = o;
        }
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int lx = threadIdx.x & 1, ly = threadIdx.x >> 1;
        const int gx = bx * 2 + lx, gy = by * 2 + ly;
        if (gx < fc.mw[2] && gy < fc.mh[2]) {
            int x0 = 2 * gx, y0 = 2 * gy, x1 = clampi(2 * gx + 1, 0, fc.mw[1] - 1), y1 = clampi(2 * gy + 1, 0, fc.mh[1] - 1);
            float4 a = m1[y0 - by * 4][x0 - bx * 4], b = m1[y0 - by * 4][x1 - bx * 4];
            float4 c = m1[y1 - by * 4][x0 - bx * 4], d = m1[y1 - by * 4][x1 - bx * 4];
            float4 o = make_float4(((a.x + b.x) + (c.x + d.x)) * 0.25f, ((a.y + b.y) + (c.y + d.y)) * 0.25f,
                                   ((a.z + b.z) + (c.z + d.z)) * 0.25f, ((a.w + b.w) + (c.w + d.w)) * 0.25f);
            P.mips[fc.moff[2] + (size_t)gy * fc.mw[2] + gx] = o;
            m2[ly][lx] = o;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int gx = bx, gy = by;
        if (gx < fc.mw[3] && gy < fc.mh[3]) {
            int x0 = 2 * gx, y0 = 2 * gy, x1 = clampi(2 * gx + 1, 0, fc.mw[2] - 1), y1 = clampi(2 * gy + 1, 0, fc.mh[2] - 1);
            float4 a = m2[y0 - by * 2][x0 - bx * 2], b = m2[y0 - by * 2][x1 - bx * 2];
            float4 c = m2[y1 - by * 2][x0 - bx * 2], d = m2[y1 - by * 2][x1 - bx * 2];
            float4 o = make_float4(((a.x + b.x) + (c.x + d.x)) * 0.25f, ((a.y + b.y) + (c.y + d.y)) * 0.25f,
                                   ((a.z + b.z) + (c.z + d.z)) * 0.25f, ((a.w + b.w) + (c.w + d.w)) * 0.25f);
            P.mips[fc.moff[3] + (size_t)gy * fc.mw[3] + gx] = o;
        }
    }
}

__global__ __launch_bounds__(64) void k_blur_median_mips(FrameConst fc, Planes P, void *hist_out)
{
    b_blur_median_mips(fc, P, hist_out, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(64) void kb_blur_median_mips(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridMip, blockIdx.x, bx, by)];
    b_blur_median_mips(J.fc, J.P, J.hist_out, bx, by);
}

// ---------------------------------------------------------------- A13

// Tap positions are c + o * R with |o| <= 1 (ring radii k/4, k <= 4), and
// rounding is monotone, so they lie in [c - R, c + R] as computed in binary32;
// every later coordinate map is monotone too, so testing the two ends bounds
// every tap.  taps_inside: the nearest-pixel lookup of the tap plane needs no
// clamp.  mip_taps_inside: the bilinear mip lookup at scale sc needs none and
// reads only non-negative coordinates.
__device__ inline bool taps_inside(int c, float R, int n)
{
    const float lo = (float)c + (-R), hi = (float)c + R;
    return lo + 0.5f >= 0.0f && hi + 0.5f < (float)n;
}

__device__ inline bool mip_taps_inside(int c, float R, float sc, int n)
{
    const float lo = (float)c + (-R), hi = (float)c + R;
    return (lo + 0.5f) * sc - 0.5f >= 0.0f && (hi + 0.5f) * sc - 0.5f < (float)(n - 1);
}

typedef float Texel __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const Texel LdsTexel;

// A mip level as a pixel's taps read it: from global memory, or (Lds) from
// its box in LDS, whose texel (x, y) lies at LDS byte address
// at + 16 x + row y.
struct MipLevel {
    float sc;                  // 2^-level
    int w, h;                  // the level's size
    const Texel *img;          // global
    uint32_t at, row;          // LDS
    int x0, x1, y0, y1;        // the box: first and last column and row
};

// Adds f times the bilinear sample at (x, y) of a level to the channel sums:
// four texel weights applied with fused multiply-adds (equal to the nested
// lerps in exact arithmetic; the reconstruction's tolerance parity covers the
// rounding).  Inside: the caller has shown that no index needs a clamp.  From
// LDS the clamp is into the box, which holds every index that the block's taps
// reach after the clamp to the image, so it gives the same texels and every
// LDS access stays inside the box.
template <bool Inside, bool Lds>
__device__ inline void acc_bilinear(const MipLevel &L, float x, float y, float f, float &a0, float &a1, float &a2, float &a3)
{
    float fx, fy;
    Texel t00, t10, t01, t11;
    if (Inside) {
        const int xi = (int)x, yi = (int)y;
        fx = __builtin_amdgcn_fractf(x);
        fy = __builtin_amdgcn_fractf(y);
        if (Lds) {
            const uint32_t at = (uint32_t)(__mul24(yi, (int)L.row) + (int)(((uint32_t)xi << 4) + L.at));
            const LdsTexel *r0 = (const LdsTexel *)(uintptr_t)at, *r1 = (const LdsTexel *)(uintptr_t)(at + L.row);
            t00 = r0[0]; t10 = r0[1]; t01 = r1[0]; t11 = r1[1];
        } else {
            const Texel *r0 = L.img + (__mul24(yi, L.w) + xi), *r1 = r0 + L.w;
            t00 = r0[0]; t10 = r0[1]; t01 = r1[0]; t11 = r1[1];
        }
    } else {
        const float x0f = floorf(x), y0f = floorf(y);
        fx = x - x0f;
        fy = y - y0f;
        const int xi = (int)x0f, yi = (int)y0f;
        const int xa = clampi(xi, L.x0, L.x1), xb = clampi(xi + 1, L.x0, L.x1);
        const int ya = clampi(yi, L.y0, L.y1), yb = clampi(yi + 1, L.y0, L.y1);
        if (Lds) {
            const uint32_t ra = (uint32_t)__mul24(ya, (int)L.row) + L.at, rb = (uint32_t)__mul24(yb, (int)L.row) + L.at;
            t00 = *(const LdsTexel *)(uintptr_t)(ra + 16u * (uint32_t)xa);
            t10 = *(const LdsTexel *)(uintptr_t)(ra + 16u * (uint32_t)xb);
            t01 = *(const LdsTexel *)(uintptr_t)(rb + 16u * (uint32_t)xa);
            t11 = *(const LdsTexel *)(uintptr_t)(rb + 16u * (uint32_t)xb);
        } else {
            const size_t ra = (size_t)ya * L.w, rb = (size_t)yb * L.w;
            t00 = L.img[ra + xa]; t10 = L.img[ra + xb]; t01 = L.img[rb + xa]; t11 = L.img[rb + xb];
        }
    }
    const float wy1 = fy * f, wy0 = f - wy1;
    const float w11 = fx * wy1, w01 = wy1 - w11, w10 = fx * wy0, w00 = wy0 - w10;
    a0 = fmaf(t11.x, w11, fmaf(t01.x, w01, fmaf(t10.x, w10, fmaf(t00.x, w00, a0))));
    a1 = fmaf(t11.y, w11, fmaf(t01.y, w01, fmaf(t10.y, w10, fmaf(t00.y, w00, a1))));
    a2 = fmaf(t11.z, w11, fmaf(t01.z, w01, fmaf(t10.z, w10, fmaf(t00.z, w00, a2))));
    a3 = fmaf(t11.w, w11, fmaf(t01.w, w01, fmaf(t10.w, w10, fmaf(t00.w, w00, a3))));
}

// What a pixel's taps add up to.
struct TapSums {
    float a0, a1, a2, a3;   // weighted colour and weight of the mip samples
    float sh;               // hit ratios of the taps that count
    int n;                  // how many count

    __device__ void add(const TapSums &u)
    {
        a0 = a0 + u.a0; a1 = a1 + u.a1; a2 = a2 + u.a2; a3 = a3 + u.a3;
        sh = sh + u.sh;
        n += u.n;
    }
};

constexpr int kReconTaps = 2;      // ring taps an iteration
constexpr int kReconQuarter = 20;  // ring taps of a quarter

// Quarters [q0, q1) of one pixel's 81 taps in tap order (the first quarter
// starts with the centre), each summed by itself, kReconTaps at a time (every ring starts at an odd tap and holds
// an even number of taps at one distance).  Two at a time keep the kernel at 4
// waves per SIMD without spills: 3840x2160 takes 2269 us a frame with two,
// 2295 with one or four and 2286 with eight (3 waves).  Which texels a tap
// reads, and whether it counts, are decided exactly as in the per-pixel
// definition.  Every tap's fetches are issued (indices in bounds: clamped, or
// shown inside) and rejected taps weigh 0, so the loads of several taps can be
// in flight at once.  A tap counts when its pixel is ray traced and its CoC
// radius reaches the tap (pixels that are not carry -inf).  The scales are
// powers of two, so the fused coordinate maps round as a product and a
// difference would.
template <bool Inside, bool Lds>
__device__ inline TapSums recon_taps(int q0, int q1, int x, int y, float Rr, float fl, const MipLevel &L0, const MipLevel &L1, int hw,
                                     int hh, const Rings &rings, const float2 *tap)
{
    TapSums s = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0}, sum = s;
    const float omf = 1.0f - fl, xf = (float)x, yf = (float)y;
    auto one = [&](float sx, float sy, float2 tj, float reach) __attribute__((always_inline)) {
        const bool ok = tj.x >= reach;   // CoC diameter against four times the distance: a quarter of it is exact
        const float cx = sx + 0.5f, cy = sy + 0.5f;
        acc_bilinear<Inside, Lds>(L0, fmaf(cx, L0.sc, -0.5f), fmaf(cy, L0.sc, -0.5f), ok ? omf : 0.0f, s.a0, s.a1, s.a2, s.a3);
        acc_bilinear<Inside, Lds>(L1, fmaf(cx, L1.sc, -0.5f), fmaf(cy, L1.sc, -0.5f), ok ? fl : 0.0f, s.a0, s.a1, s.a2, s.a3);
        s.sh = s.sh + (ok ? tj.y : 0.0f);
        s.n += ok ? 1 : 0;
    };
    auto pixel = [&](float sx, float sy) __attribute__((always_inline)) {
        if (Inside) return tap[(uint32_t)(__umul24((int)(sy + 0.5f), hw) + (int)(sx + 0.5f))];
        return tap[(size_t)nearest_idx(sy, hh) * hw + nearest_idx(sx, hw)];
    };
    if (q0 == 0)
        one(xf + rings.ox[0] * Rr, yf + rings.oy[0] * Rr, pixel(xf + rings.ox[0] * Rr, yf + rings.oy[0] * Rr),
            4.0f * (Rr * rings.frac[0]));
#pragma unroll 1
    for (int q = q0; q < q1; ++q) {
        const int first = 1 + q * kReconQuarter;
#pragma unroll 1
        for (int k = first; k < first + kReconQuarter; k += kReconTaps) {
            const float reach = 4.0f * (Rr * rings.frac[k]);
            float sx[kReconTaps], sy[kReconTaps];
            float2 tj[kReconTaps];
#pragma unroll
            for (int t = 0; t < kReconTaps; ++t) {
                sx[t] = xf + rings.ox[k + t] * Rr;
                sy[t] = yf + rings.oy[k + t] * Rr;
                tj[t] = pixel(sx[t], sy[t]);
            }
#pragma unroll
            for (int t = 0; t < kReconTaps; ++t) one(sx[t], sy[t], tj[t], reach);
        }
        sum.add(s);
        s = TapSums{0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0};
    }
    return sum;
}

static_assert(1 + 4 * kReconQuarter == kRingTaps && kReconQuarter % kReconTaps == 0, "whole quarters");

constexpr int kReconSplit = 768;  // 16 x 16 tiles below which a frame's reconstruction takes 8 x 8 ones
// Mip texels that a block can stage in LDS (24 KB: six blocks a CU, so that
// blocks with few live pixels do not hold the others' place).  1200 leave too
// many of 3840x2160's blocks to global memory (2204 us a frame against 2156),
// 2368 let in four blocks a CU (2166; 1920x1080 443 against 437).
constexpr int kReconLds = 1520;

// Index range that the bilinear lookups of taps between coordinates lo and hi
// (one axis, already at the level's scale sc) reach after the clamp to
// [0, n - 1]: the coordinate map and floor are monotone, so the two ends bound
// every tap.
__device__ inline void mip_span(float lo, float hi, float sc, int n, int &a, int &b)
{
    a = clampi((int)floorf((lo + 0.5f) * sc - 0.5f), 0, n - 1);
    b = clampi((int)floorf((hi + 0.5f) * sc - 0.5f) + 1, 0, n - 1);
}

__device__ inline float wave_fmin(float v)
{
    for (int o = 32; o >= 1; o >>= 1) v = fminf(v, __shfl_xor(v, o));
    return v;
}

// One block of 256 threads per tile of kSide x kSide half-res pixels (a square
// footprint stages fewer halo texels than a row block): 16 x 16, a lane per
// pixel, or 8 x 8, whose pixels' taps the four waves share, a quarter each.
// Both add the quarters' sums in the same order, so a pixel's value does not
// depend on the tile.
//
// The output is the median blended with the taps' mean by a weight that
// follows the pixel's temporal variance; where the weight is 0 it is the
// median itself, and no tap is read (a frame whose colours might sum to
// something that is not finite reads them all: 0 times it is no 0).  The
// remaining pixels are packed into as few waves as hold them: at 1920x1080
// 46 % of the waves of traced pixels have none, at 3840x2160 1 %.  What is
// left is bound by vector issue, 81 instructions a tap (94 with the coordinate
// maps and texel weights written out), next to the LDS reads, 64 of the 81
// clocks that a tap of one wave takes a CU.  1920x1080: 121 -> 75 us,
// 3840x2160 344 -> 323, 256x256 37 -> 30.
template <int kSide>
__device__ inline void b_recon(const FrameConst &fc, const Rings &rings, const Planes &P, const uint32_t bx, const uint32_t by)
{
    // The block's mip footprint: per level, the index box of every bilinear
    // lookup its pixels' taps make (taps lie within R of the pixel on both
    // axes), staged in LDS when the boxes fit; else the taps read the mips
    // in global memory.
    __shared__ float4 tex[kReconLds];
    __shared__ float span[4][4][4];   // per wave and lower level, of the taps: least x, -(greatest x), least y, -(greatest y)
    __shared__ int box[4][4];         // per level: first and last column, first and last row
    __shared__ int base[5];           // per level: first LDS texel; [4]: texels in all
    __shared__ uint32_t wcount[4];
    __shared__ uint8_t list[256];     // the pixels that read taps
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int hw = fc.hw, hh = fc.hh, tx0 = (int)bx * kSide, ty0 = (int)by * kSide;
    {
        const int x = tx0 + tid % kSide, y = ty0 + tid / kSide;
        bool live = false;
        float Rr = 0.0f;
        int L0 = -1;
        if (x < hw && y < hh && tid < kSide * kSide) {
            const size_t i = (size_t)y * hw + x;
            const float2 t = P.tap[i];
            const bool traced = t.x != -INFINITY;
            if (traced) {
                const float bb = clampf(P.var_blur[i] * fc.var_recon_w, 0.0f, fc.b_max);
                live = bb != 0.0f || P.counters[kCntWild] != 0u;
            }
            if (live) {
                Rr = fmin_cs(t.x * 0.25f, fc.r_max);
                L0 = (int)floorf(clampf(t.x * fc.lod_scale, 0.0f, fc.lod_max));
                L0 = L0 > fc.lod_levels ? fc.lod_levels : L0;
            } else {
                float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (traced) {
                    o = P.rtmed[i];
                    o.w = t.y;
                }
                P.recon[i] = o;
            }
        }
        const uint64_t lives = __ballot(live);
        if (lane == 0) wcount[w] = (uint32_t)__popcll(lives);
        // the tap coordinates' ends per lower level
        for (int L = 0; L < 4; ++L) {
            float e[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
            if (__ballot(L0 == L) != 0ull) {
                if (L0 == L) {
                    // a radius that is no number counts as 0: its taps are
                    // clamped into the box too, which must not be empty
                    const float R = Rr == Rr ? Rr : 0.0f;
                    e[0] = (float)x + (-R);
                    e[1] = -((float)x + R);
                    e[2] = (float)y + (-R);
                    e[3] = -((float)y + R);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) e[k] = wave_fmin(e[k]);
            }
            if (lane < 4) span[w][L][lane] = lane == 0 ? e[0] : (lane == 1 ? e[1] : (lane == 2 ? e[2] : e[3]));
        }
        __syncthreads();
        uint32_t at = 0u;
        for (int k = 0; k < w; ++k) at += wcount[k];
        if (live) list[at + (uint32_t)__popcll(lives & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))))] = (uint8_t)tid;
    }
    const int nlive = (int)(wcount[0] + wcount[1] + wcount[2] + wcount[3]);
    if (nlive == 0) return;   // block-uniform
    if (tid < 4) {
        // level tid is read by pixels whose lower level it is or is next above
        int c0 = 0x7fffffff, c1 = -1, r0 = 0x7fffffff, r1 = -1;
        float sc = 1.0f;
        for (int k = 0; k < tid; ++k) sc = sc * 0.5f;
        for (int L = tid > 0 ? tid - 1 : 0; L <= tid; ++L) {
            // pixels of lower level L read levels L and min(L + 1, lod_levels)
            if (L != tid && !(L < fc.lod_levels)) continue;
            float e[4];
            for (int k = 0; k < 4; ++k) e[k] = fminf(fminf(span[0][L][k], span[1][L][k]), fminf(span[2][L][k], span[3][L][k]));
            if (e[0] == INFINITY) continue;
            int a, b;
            mip_span(e[0], -e[1], sc, fc.mw[tid], a, b);
            c0 = min(c0, a);
            c1 = max(c1, b);
            mip_span(e[2], -e[3], sc, fc.mh[tid], a, b);
            r0 = min(r0, a);
            r1 = max(r1, b);
        }
        box[tid][0] = c0; box[tid][1] = c1;
        box[tid][2] = r0; box[tid][3] = r1;
    }
    __syncthreads();
    if (tid == 0) {
        int n = 0;
        for (int L = 0; L < 4; ++L) {
            base[L] = n;
            if (box[L][1] >= box[L][0]) n += (box[L][1] - box[L][0] + 1) * (box[L][3] - box[L][2] + 1);
        }
        base[4] = n;
    }
    __syncthreads();
    const bool staged = base[4] <= kReconLds;
    if (staged) {
        for (int L = 0; L < 4; ++L) {
            if (box[L][1] < box[L][0]) continue;
            const int bw = box[L][1] - box[L][0] + 1, cnt = bw * (box[L][3] - box[L][2] + 1);
            const float4 *src = P.mips + fc.moff[L];
            for (int e = tid; e < cnt; e += 256) {
                const int r = e / bw, c = e - r * bw;
                tex[base[L] + e] = src[(size_t)(box[L][2] + r) * fc.mw[L] + box[L][0] + c];
            }
        }
    }
    __syncthreads();
    const int slot = kSide == 16 ? tid : lane;
    if (kSide == 16 && slot >= nlive) return;
    const int px = list[slot < nlive ? slot : 0], x = tx0 + px % kSide, y = ty0 + px / kSide;
    const size_t i = (size_t)y * hw + x;
    const float2 t1 = P.tap[i];
    const float ct = t1.x, hu = t1.y, Rr = fmin_cs(ct * 0.25f, fc.r_max);
    const float lod = clampf(ct * fc.lod_scale, 0.0f, fc.lod_max);
    int L0 = (int)floorf(lod);
    const int Lmax = fc.lod_levels;
    if (L0 > Lmax) L0 = Lmax;
    const int L1 = L0 < Lmax ? L0 + 1 : Lmax;
    const float fl = lod - (float)L0;
    auto level = [&](int L) {
        MipLevel m;
        m.sc = 1.0f;
        for (int k = 0; k < L; ++k) m.sc = m.sc * 0.5f;
        m.w = fc.mw[L];
        m.h = fc.mh[L];
        m.img = (const Texel *)(P.mips + fc.moff[L]);
        m.row = 0u;
        m.at = 0u;
        m.x0 = 0; m.x1 = m.w - 1;
        m.y0 = 0; m.y1 = m.h - 1;
        if (staged) {
            m.x0 = box[L][0]; m.x1 = box[L][1];
            m.y0 = box[L][2]; m.y1 = box[L][3];
            m.row = 16u * (uint32_t)(m.x1 - m.x0 + 1);
            m.at = (uint32_t)(uintptr_t)(LdsTexel *)(tex + base[L]) - m.row * (uint32_t)m.y0 - 16u * (uint32_t)m.x0;
        }
        return m;
    };
    const MipLevel m0 = level(L0), m1 = level(L1);
    // The interior paths are taken by a whole wave when every lane's taps
    // stay inside all planes it reads (same arithmetic, no clamps).
    const bool inside = hw < (1 << 24) && hh < (1 << 24) && taps_inside(x, Rr, hw) && taps_inside(y, Rr, hh) &&
                        mip_taps_inside(x, Rr, m0.sc, m0.w) && mip_taps_inside(y, Rr, m0.sc, m0.h) &&
                        mip_taps_inside(x, Rr, m1.sc, m1.w) && mip_taps_inside(y, Rr, m1.sc, m1.h);
    const bool all_inside = __ballot(!inside) == 0ull;
    const int q0 = kSide == 16 ? 0 : __builtin_amdgcn_readfirstlane(w), q1 = kSide == 16 ? 4 : q0 + 1;
    TapSums s;
    if (staged) {
        if (all_inside) s = recon_taps<true, true>(q0, q1, x, y, Rr, fl, m0, m1, hw, hh, rings, P.tap);
        else s = recon_taps<false, true>(q0, q1, x, y, Rr, fl, m0, m1, hw, hh, rings, P.tap);
    } else {
        if (all_inside) s = recon_taps<true, false>(q0, q1, x, y, Rr, fl, m0, m1, hw, hh, rings, P.tap);
        else s = recon_taps<false, false>(q0, q1, x, y, Rr, fl, m0, m1, hw, hh, rings, P.tap);
    }
    if constexpr (kSide != 16) {
        __shared__ TapSums part[3][64];
        if (w > 0) part[w - 1][lane] = s;
        __syncthreads();
        if (w > 0 || lane >= nlive) return;
#pragma unroll
        for (int q = 0; q < 3; ++q) s.add(part[q][lane]);
    }
    const float4 med = P.rtmed[i];
    float nb0 = s.a3 > 0.0f ? s.a0 / s.a3 : med.x, nb1 = s.a3 > 0.0f ? s.a1 / s.a3 : med.y, nb2 = s.a3 > 0.0f ? s.a2 / s.a3 : med.z;
    float hnb = s.n > 0 ? s.sh / (float)s.n : hu;
    float bb = clampf(P.var_blur[i] * fc.var_recon_w, 0.0f, fc.b_max);
    P.recon[i] = make_float4(lerp1(med.x, nb0, bb), lerp1(med.y, nb1, bb), lerp1(med.z, nb2, bb), lerp1(hu, hnb, bb));
}

template <int kSide>
__global__ __launch_bounds__(256, 4) void k_recon(FrameConst fc, Rings rings, Planes P)
{
    b_recon<kSide>(fc, rings, P, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256, 4) void kb_recon(const Job *__restrict__ jobs, int njobs, Rings rings)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridTiles, blockIdx.x, bx, by)];
    b_recon<16>(J.fc, rings, J.P, bx, by);
}

// ---------------------------------------------------------------- A14

__device__ inline void b_composite(const FrameConst &fc, const Planes &P, const dof_gbuffer &gb, const dof_frame_out &out, const uint32_t bx, const uint32_t by)
{
    const int x = bx * kBX + threadIdx.x, y = by * kBY + threadIdx.y;
    if (x >= fc.W || y >= fc.H) return;
    const int hw = fc.hw, hh = fc.hh;
    const size_t p = (size_t)y * fc.W + x;
    const float z = gb.depth[p];
    const float c = coc_px(fc.cock, fc.d, z);
    const float hx = (float)x * 0.5f - 0.25f, hy = (float)y * 0.5f - 0.25f;
    const float4 pp = bilinear4(P.ppout, hw, hh, hx, hy);
    const float x0f = floorf(hx), y0f = floorf(hy);
    const float fx = hx - x0f, fy = hy - y0f;
    const int x0 = (int)x0f, y0 = (int)y0f;
    const int xs[2] = {clampi(x0, 0, hw - 1), clampi(x0 + 1, 0, hw - 1)};
    const int ys[2] = {clampi(y0, 0, hh - 1), clampi(y0 + 1, 0, hh - 1)};
    const float wts[4] = {(1.0f - fx) * (1.0f - fy), fx * (1.0f - fy), (1.0f - fx) * fy, fx * fy};
    float sw = 0.0f, rc0 = 0.0f, rc1 = 0.0f, rc2 = 0.0f, rh = 0.0f, rct = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        size_t j = (size_t)ys[k >> 1] * hw + xs[k & 1];
        // validity (exactly 0 or 1) and CoC (0 where invalid) from the tap record
        const float2 tp = P.tap[j];
        const bool valid = tp.x != -INFINITY;
        float wv = valid ? wts[k] : 0.0f;
        float4 rj = P.recon[j];
        sw = sw + wv;
        rc0 = rc0 + wv * rj.x;
        rc1 = rc1 + wv * rj.y;
        rc2 = rc2 + wv * rj.z;
        rh = rh + wv * rj.w;
        rct = rct + wv * (valid ? tp.x : 0.0f);
    }
    const bool rtv = sw > 0.0f;
    if (rtv) {
        rc0 = rc0 / sw; rc1 = rc1 / sw; rc2 = rc2 / sw;
        rh = rh / sw;
        rct = rct / sw;
    }
    float4 o;
    if (c <= kSqrt2 && (!rtv || rct < kSqrt2)) {
        float4 g = ld_rgba(gb.colour, gb.colour_format, p);
        o = make_float4(g.x, g.y, g.z, 1.0f);
    } else if (!rtv) {
        o = make_float4(pp.x, pp.y, pp.z, 1.0f);
    } else if (z < fc.d) {
        o = make_float4(lerp1(rc0, pp.x, pp.w), lerp1(rc1, pp.y, pp.w), lerp1(rc2, pp.z, pp.w), 1.0f);
    } else {
        float t = sat(rh / fc.h_edge);
        float w = (t * t) * (3.0f - 2.0f * t);
        if (fc.composite_literal)   // the literal reading: a high hit ratio favours the post-process colour
            o = make_float4(lerp1(rc0, pp.x, w), lerp1(rc1, pp.y, w), lerp1(rc2, pp.z, w), 1.0f);
        else
            o = make_float4(lerp1(pp.x, rc0, w), lerp1(pp.y, rc1, w), lerp1(pp.z, rc2, w), 1.0f);
    }
    if (fc.taa & DOF_TAA_FINAL) P.comp[p] = o;
    else st_rgba(out.colour, out.colour_format, p, o);
}

__global__ __launch_bounds__(kBX *kBY) void k_composite(FrameConst fc, Planes P, dof_gbuffer gb, dof_frame_out out)
{
    // The frame's counters are final once the traversal has run: the first
    // thread writes the caller's stats record (masked px, rays, and the sums
    // of the traversal's statistics slots).
    if (out.stats && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.y == 0 && threadIdx.x == 0) {
        unsigned long long v = 0ull, t = 0ull;
        uint32_t drops = 0u;
        for (int p = 0; p < kWorkParts; ++p) {
            const uint32_t *w = P.counters + kCntWork + p * kWorkStride + kStatAt;
            v += *reinterpret_cast<const unsigned long long *>(w);
            t += *reinterpret_cast<const unsigned long long *>(w + 2);
            drops += w[4];
        }
        dof_stats *o = out.stats;
        o->masked_px = P.counters[kCntMasked];
        o->rays = P.counters[kCntRays];
        o->node_visits = v;
        o->tri_tests = t;
        o->stack_spills = drops;
    }
    b_composite(fc, P, gb, out, blockIdx.x, blockIdx.y);
}

// Also, with an item's first thread, its stats record: masked pixels and rays
// (the traversal's statistics of a batch are kept once, in its head, where the
// first item's sums the slots).
__global__ __launch_bounds__(kBX *kBY) void kb_composite(BatchHead *head, const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const int j = job_of_block(jobs, njobs, kGridFull, blockIdx.x, bx, by);
    const Job &J = jobs[j];
    if (bx == 0 && by == 0 && threadIdx.x == 0 && threadIdx.y == 0) {
        if (j == 0) {
            unsigned long long v = 0ull, t = 0ull;
            for (int p = 0; p < kWorkParts; ++p) {
                const uint32_t *w = head->work + p * kWorkStride + kStatAt;
                v += *reinterpret_cast<const unsigned long long *>(w);
                t += *reinterpret_cast<const unsigned long long *>(w + 2);
            }
            head->visits = v;
            head->tests = t;
        }
        if (dof_stats *o = J.out.stats) {
            o->masked_px = J.P.counters[kCntMasked];
            o->rays = J.P.counters[kCntRays];
            o->node_visits = 0;
            o->tri_tests = 0;
        }
    }
    b_composite(J.fc, J.P, J.gb, J.out, bx, by);
}

// ---------------------------------------------------------------- TAA
// Temporal anti-aliasing stages (3.4, after Karis 2014).  One resolve: the
// current image's colour at (x, y) of a w x h grid is blended with the
// history image of the same grid, fetched bilinearly where the pixel's point
// (view depth z through the jittered camera; its direction for the sky)
// lands in the previous camera -- none behind it or off the grid -- that
// history clamped per RGB channel to the current 3 x 3 range (clamp to
// edge), history weight 0.9.  cur(x, y) reads the current image.  The 4th
// channel is 1, or the current one's with keep_w.

__device__ inline size_t taa_plane_floats(const FrameConst &fc, int which)   // 0 final, 1 raster, 2 post-filter
{
    const size_t base = ((size_t)fc.hw * fc.hh * 13 + 3) & ~(size_t)3;   // the record, rounded up to 16 bytes
    return base + (size_t)which * 4 * (size_t)fc.W * fc.H;
}

template <class Cur>
__device__ inline float4 taa_resolve(const FrameConst &fc, const Cur &cur, float z, int x, int y, int w, int h,
                                     const float4 *hin, bool keep_w)
{
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
            const float4 v = cur(clampi(x + dx, 0, w - 1), clampi(y + dy, 0, h - 1));
            const float vv[3] = {v.x, v.y, v.z};
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                mn[c] = vv[c] < mn[c] ? vv[c] : mn[c];
                mx[c] = vv[c] > mx[c] ? vv[c] : mx[c];
            }
        }
    const float4 c0 = cur(x, y);
    bool valid = false;
    float4 hc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (hin) {
        float fv[3], Pw[3], e[3];
        pixel_dir(fc.cur, x, y, w, h, fv);
        const bool isdir = !(z < INFINITY);
#pragma unroll
        for (int a = 0; a < 3; ++a) Pw[a] = isdir ? fv[a] : fc.cur.pos[a] + z * fv[a];
#pragma unroll
        for (int a = 0; a < 3; ++a) e[a] = isdir ? Pw[a] : Pw[a] - fc.prev.pos[a];
        const float ex = (e[0] * fc.prev.right[0] + e[1] * fc.prev.right[1]) + e[2] * fc.prev.right[2];
        const float ey = (e[0] * fc.prev.up[0] + e[1] * fc.prev.up[1]) + e[2] * fc.prev.up[2];
        const float ez = (e[0] * fc.prev.fwd[0] + e[1] * fc.prev.fwd[1]) + e[2] * fc.prev.fwd[2];
        if (ez > 0.0f) {
            const float pu = (ex / ez) / fc.prev.tanx, pv = (ey / ez) / fc.prev.tany;
            const float px = ((pu + 1.0f) * 0.5f) * (float)w - 0.5f;
            const float py = ((1.0f - pv) * 0.5f) * (float)h - 0.5f;
            if (px + 0.5f >= 0.0f && px + 0.5f < (float)w && py + 0.5f >= 0.0f && py + 0.5f < (float)h) {
                hc = bilinear4(hin, w, h, px, py);
                valid = true;
            }
        }
    }
    const float cv[3] = {c0.x, c0.y, c0.z}, hv[3] = {hc.x, hc.y, hc.z};
    float o[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float v = cv[c];
        if (valid) {
            float t = hv[c];
            t = t > mn[c] ? t : mn[c];
            t = t < mx[c] ? t : mx[c];
            v = lerp1(cv[c], t, 0.9f);
        }
        o[c] = v;
    }
    return make_float4(o[0], o[1], o[2], keep_w ? c0.w : 1.0f);
}

__device__ inline const float4 *taa_history(const FrameConst &fc, const void *hist_in, int which)
{
    return (fc.have_hist && hist_in) ? reinterpret_cast<const float4 *>(static_cast<const float *>(hist_in) +
                                                                        taa_plane_floats(fc, which))
                                     : nullptr;
}

// The raster image before filtering (DOF_TAA_RASTER): G-buffer colour in,
// the resolved plane out (every later stage reads it).
__device__ inline void b_taa_raster(const FrameConst &fc, const Planes &P, const dof_gbuffer &gb, const void *hist_in,
                                    void *hist_out, const uint32_t bx, const uint32_t by)
{
    const int x = bx * kBX + threadIdx.x, y = by * kBY + threadIdx.y;
    const int W = fc.W, H = fc.H;
    if (x >= W || y >= H) return;
    const size_t p = (size_t)y * W + x;
    auto cur = [&](int xx, int yy) { return ld_rgba(gb.colour, gb.colour_format, (size_t)yy * W + xx); };
    const float4 r = taa_resolve(fc, cur, gb.depth[p], x, y, W, H, taa_history(fc, hist_in, 1), false);
    P.rast[p] = r;
    reinterpret_cast<float4 *>(static_cast<float *>(hist_out) + taa_plane_floats(fc, 1))[p] = r;
}

// The half-res post-filter output (DOF_TAA_POST); the quad's nearest depth
// locates each pixel.
__device__ inline void b_taa_post(const FrameConst &fc, const Planes &P, const void *hist_in, void *hist_out,
                                  const uint32_t bx, const uint32_t by)
{
    const int x = bx * kBX + threadIdx.x, y = by * kBY + threadIdx.y;
    const int hw = fc.hw, hh = fc.hh;
    if (x >= hw || y >= hh) return;
    const size_t i = (size_t)y * hw + x;
    auto cur = [&](int xx, int yy) { return P.ppmed[(size_t)yy * hw + xx]; };
    const float4 r = taa_resolve(fc, cur, P.zn[i].x, x, y, hw, hh, taa_history(fc, hist_in, 2), true);
    P.pptaa[i] = r;
    reinterpret_cast<float4 *>(static_cast<float *>(hist_out) + taa_plane_floats(fc, 2))[i] = r;
}

// The output after the composite (DOF_TAA_FINAL).
__device__ inline void b_taa_final(const FrameConst &fc, const Planes &P, const dof_gbuffer &gb, const void *hist_in,
                                   void *hist_out, const dof_frame_out &out, const uint32_t bx, const uint32_t by)
{
    const int x = bx * kBX + threadIdx.x, y = by * kBY + threadIdx.y;
    const int W = fc.W, H = fc.H;
    if (x >= W || y >= H) return;
    const size_t p = (size_t)y * W + x;
    auto cur = [&](int xx, int yy) { return P.comp[(size_t)yy * W + xx]; };
    const float4 r = taa_resolve(fc, cur, gb.depth[p], x, y, W, H, taa_history(fc, hist_in, 0), false);
    st_rgba(out.colour, out.colour_format, p, r);
    reinterpret_cast<float4 *>(static_cast<float *>(hist_out) + taa_plane_floats(fc, 0))[p] = r;
}

__global__ __launch_bounds__(kBX *kBY) void k_taa_raster(FrameConst fc, Planes P, dof_gbuffer gb, const void *hist_in,
                                                         void *hist_out)
{
    b_taa_raster(fc, P, gb, hist_in, hist_out, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kBX *kBY) void k_taa_post(FrameConst fc, Planes P, const void *hist_in, void *hist_out)
{
    b_taa_post(fc, P, hist_in, hist_out, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kBX *kBY) void k_taa_final(FrameConst fc, Planes P, dof_gbuffer gb, const void *hist_in,
                                                        void *hist_out, dof_frame_out out)
{
    b_taa_final(fc, P, gb, hist_in, hist_out, out, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kBX *kBY) void kb_taa_raster(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridFull, blockIdx.x, bx, by)];
    b_taa_raster(J.fc, J.P, J.gb_in, J.hist_in, J.hist_out, bx, by);
}

__global__ __launch_bounds__(kBX *kBY) void kb_taa_post(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridHalf, blockIdx.x, bx, by)];
    b_taa_post(J.fc, J.P, J.hist_in, J.hist_out, bx, by);
}

__global__ __launch_bounds__(kBX *kBY) void kb_taa_final(const Job *__restrict__ jobs, int njobs)
{
    uint32_t bx, by;
    const Job &J = jobs[job_of_block(jobs, njobs, kGridFull, blockIdx.x, bx, by)];
    b_taa_final(J.fc, J.P, J.gb, J.hist_in, J.hist_out, J.out, bx, by);
}

__global__ void k_fill_zero(float *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0f;
}

inline dim3 grid2(int w, int h, int bx, int by) { return dim3((w + bx - 1) / bx, (h + by - 1) / by); }

// Where one launch for the compaction and the ray generation is the faster
// way.  It saves two launches, 5 to 9 us, but a block then makes all rays of
// its 256 pixels, on at most 512 blocks where the general path has 2048, and a
// bladed aperture's without the general path's second pass for rays whose first
// tries fail.  Its frame's time against the general path's, at 128x128,
// 256x256, 512x512 and 724x724 (866 triangles, us):
//   circle, m 30, every pixel    178/176, 188/186, 273/280, 396/413
//   circle, m 128, every pixel   1.04, 1.02, 0.98, 0.96 of it
//   circle, m 64, adaptive       0.99, 0.98, 0.98, 0.98; m 128: 1.03, 1.00, 0.98, 0.98
//   6 blades, m 30, every pixel  247/182, 253/194, 339/292, 465/431
//   6 blades, m 30, adaptive     142/125, 147/134, 158/154, 182/180
// and with 3 to 16 blades, worst of them: every pixel m 3 0.94, 0.98, 0.98,
// 1.00, m 4 0.97, 1.01, 1.01, 1.02; dilated m 6 0.97, 1.00, 0.99, 1.00, m 8
// 1.01, 1.03, 1.00, 1.01; adaptive m 8 0.95, 0.98, 0.97, 0.99, m 12 1.04, 1.02,
// 0.99, 1.00.
bool compact_in_one(const FrameConst &fc)
{
    const int64_t np = (int64_t)fc.hw * fc.hh;
    if (np > kSmallFrame) return false;
    const bool adaptive = fc.mask_mode == DOF_MASK_ADAPTIVE, dilate = fc.mask_mode == DOF_MASK_DILATE;
    if (fc.ap.blades >= 3) return fc.m <= (adaptive ? 8 : (dilate ? 6 : 3));
    return np >= kSmallFrame / 2 || fc.m <= (adaptive ? 64 : 24);
}

}  // namespace

#define DOF_REC(k)                                          \
    do {                                                    \
        if (ev) {                                           \
            hipError_t e_ = hipEventRecord(ev[(k)], st);    \
            if (e_ != hipSuccess) return e_;                \
        }                                                   \
    } while (0)

hipError_t launch_frame_pre(const FrameConst &fc, const Rings &rings, const ScratchLayout &L, char *scratch,
                            const dof_gbuffer &gb, const void *hist_in, void *hist_out, uint8_t *mask, hipEvent_t *ev,
                            const SideStream *side, hipStream_t st)
{
    Planes P = planes(fc, L, scratch);
    const int64_t np = (int64_t)fc.hw * fc.hh;
    DOF_REC(0);
    if (fc.taa & DOF_TAA_RASTER)
        k_taa_raster<<<grid2(fc.W, fc.H, kBX, kBY), dim3(kBX, kBY), 0, st>>>(fc, P, gb, hist_in, hist_out);
    k_reduce<<<dim3(fc.tw, fc.th), dim3(kTile, kTile), 0, st>>>(fc, resolved_gbuffer(fc, P, gb), P);
    DOF_REC(1);
    // the dilated tile radii feed the prefilter and the gather, and the ray
    // mask only in its dilated mode: otherwise the prefilter finds them itself,
    // on the side stream
    const bool dil_side = side && fc.mask_mode != DOF_MASK_DILATE;
    if (!dil_side) k_dilate<<<grid2(fc.tw, fc.th, 16, 16), dim3(16, 16), 0, st>>>(fc, P);
    DOF_REC(2);
    // The post-process chain reads only the reduce's and the dilation's planes
    // and only the composite reads its result: with a side stream it is forked
    // after the ray generation, so it shares the GPU with the traversal and not
    // with the mask, compaction and generation that lead up to it.
    auto chain = [&](hipStream_t pst) -> hipError_t {
        k_prefilter<<<dim3(fc.tw, fc.th), 256, 0, pst>>>(fc, P, dil_side);
        DOF_REC(3);
        launch_gather_pair(fc.gather_win, [&](auto w) {
            k_gather<decltype(w)::value><<<dim3(fc.tw, fc.th), 256, 0, pst>>>(fc, rings, P);
        });
        DOF_REC(4);
        k_median_pp<<<grid2(fc.hw, fc.hh, kBX, kBY), dim3(kBX, kBY), 0, pst>>>(fc, P);
        if (fc.taa & DOF_TAA_POST)
            k_taa_post<<<grid2(fc.hw, fc.hh, kBX, kBY), dim3(kBX, kBY), 0, pst>>>(fc, P, hist_in, hist_out);
        return hipSuccess;
    };
    if (!side) {
        const hipError_t ec = chain(st);
        if (ec != hipSuccess) return ec;
    }
    DOF_REC(5);
    if (fc.mask_mode == DOF_MASK_DILATE) {
        k_mask<<<dim3(fc.tw, fc.th), dim3(kTile, kTile), 0, st>>>(fc, P, hist_in, P.mask_raw);
        k_mask_dilate<<<dim3(fc.tw, fc.th), dim3(kTile, kTile), 0, st>>>(fc, P, mask);
    } else {
        k_mask<<<dim3(fc.tw, fc.th), dim3(kTile, kTile), 0, st>>>(fc, P, hist_in, mask);
    }
    DOF_REC(6);
    hipError_t e;
    if (compact_in_one(fc) && reinterpret_cast<uintptr_t>(mask) % 4 == 0) {
        e = launch_compact_small(fc, L, scratch, mask, st);
    } else {
        k_compact_count<<<(unsigned)L.nchunks, 256, 0, st>>>(np, mask, P);
        k_compact_scatter<<<(unsigned)L.nchunks, 256, 0, st>>>(np, mask, P);
        e = launch_raygen(fc, L, scratch, st);
    }
    if (e != hipSuccess) return e;
    DOF_REC(7);
    if (side) {
        hipError_t e2 = hipEventRecord(side->fork, st);
        if (e2 == hipSuccess) e2 = hipStreamWaitEvent(side->stream, side->fork, 0);
        if (e2 != hipSuccess) return e2;
        e2 = chain(side->stream);
        if (e2 == hipSuccess) e2 = hipEventRecord(side->join, side->stream);
        if (e2 != hipSuccess) return e2;
    }
    return hipGetLastError();
}

hipError_t launch_frame_post(const SceneDev &sd, const FrameConst &fc, const Rings &rings, const ScratchLayout &L, char *scratch,
                             const dof_gbuffer &gb, const void *hist_in, void *hist_out, uint8_t *mask,
                             const dof_frame_out &out, hipEvent_t *ev, const SideStream *side, hipStream_t st)
{
    Planes P = planes(fc, L, scratch);
    DOF_REC(8);
    {
        const hipError_t e = launch_shade_resolve(sd, fc, L, scratch, mask, st);
        if (e != hipSuccess) return e;
    }
    DOF_REC(9);
    k_temporal<<<grid2(fc.hw, fc.hh, kBX, kBY), dim3(kBX, kBY), 0, st>>>(fc, P, mask, hist_in, hist_out);
    DOF_REC(10);
    k_blur_median_mips<<<grid2(fc.hw, fc.hh, 8, 8), 64, 0, st>>>(fc, P, hist_out);
    DOF_REC(11);
    // Four waves to a pixel where the 16 x 16 tiles leave the chip idle (it
    // holds 1024 blocks): 256x256 127 -> 114 us a frame, 800x600 166 -> 159;
    // at 960x960 (900 tiles) both take as long, at 1920x1080 450 -> 468.
    if (fc.tw * fc.th < kReconSplit) k_recon<8><<<grid2(fc.hw, fc.hh, 8, 8), 256, 0, st>>>(fc, rings, P);
    else k_recon<16><<<dim3(fc.tw, fc.th), 256, 0, st>>>(fc, rings, P);
    DOF_REC(12);
    if (side) {
        const hipError_t e = hipStreamWaitEvent(st, side->join, 0);   // the post-process chain is done
        if (e != hipSuccess) return e;
    }
    k_composite<<<grid2(fc.W, fc.H, kBX, kBY), dim3(kBX, kBY), 0, st>>>(fc, P, resolved_gbuffer(fc, P, gb), out);
    if (fc.taa & DOF_TAA_FINAL)
        k_taa_final<<<grid2(fc.W, fc.H, kBX, kBY), dim3(kBX, kBY), 0, st>>>(fc, P, gb, hist_in, hist_out, out);
    DOF_REC(13);
    return hipGetLastError();
}

hipError_t launch_history_reset(float *hist, int64_t nfloats, hipStream_t st)
{
    k_fill_zero<<<1024, 256, 0, st>>>(hist, nfloats);
    return hipGetLastError();
}

hipError_t launch_batch_chain(const Job *jobs, int njobs, const uint32_t *nblk, const Rings &rings, bool with_dilate,
                              int taa, int gather_win, hipStream_t st)
{
    kb_prefilter<<<nblk[kGridTiles], 256, 0, st>>>(jobs, njobs, with_dilate);
    launch_gather_pair(gather_win, [&](auto w) {
        kb_gather<decltype(w)::value><<<nblk[kGridTiles], 256, 0, st>>>(jobs, njobs);
    });
    kb_median_pp<<<nblk[kGridHalf], dim3(kBX, kBY), 0, st>>>(jobs, njobs);
    if (taa & DOF_TAA_POST) kb_taa_post<<<nblk[kGridHalf], dim3(kBX, kBY), 0, st>>>(jobs, njobs);
    return hipGetLastError();
}

hipError_t launch_batch_pre(const BatchHead *, const Job *jobs, int njobs, const uint32_t *nblk, const Rings &rings,
                            bool dilate, int taa, int gather_win, const SideStream *side, hipStream_t st)
{
    if (taa & DOF_TAA_RASTER) kb_taa_raster<<<nblk[kGridFull], dim3(kBX, kBY), 0, st>>>(jobs, njobs);
    kb_reduce<<<nblk[kGridTiles], dim3(kTile, kTile), 0, st>>>(jobs, njobs);
    // as in a frame: the prefilter finds the dilated radii itself unless the
    // ray mask reads them
    if (!side || dilate) kb_dilate<<<nblk[kGridDilate], dim3(16, 16), 0, st>>>(jobs, njobs);
    if (!side) {
        const hipError_t e = launch_batch_chain(jobs, njobs, nblk, rings, false, taa, gather_win, st);
        if (e != hipSuccess) return e;
    }
    kb_mask<<<nblk[kGridTiles], dim3(kTile, kTile), 0, st>>>(jobs, njobs);
    if (dilate) kb_mask_dilate<<<nblk[kGridTiles], dim3(kTile, kTile), 0, st>>>(jobs, njobs);
    kb_compact_count<<<nblk[kGridChunk], 256, 0, st>>>(jobs, njobs);
    kb_compact_scatter<<<nblk[kGridChunk], 256, 0, st>>>(jobs, njobs);
    return hipGetLastError();
}

hipError_t launch_batch_post(BatchHead *head, const Job *jobs, int njobs, const uint32_t *nblk, const Rings &rings,
                             int taa, const SideStream *side, hipStream_t st)
{
    {
        const hipError_t e = launch_batch_shade_resolve(jobs, njobs, nblk, st);
        if (e != hipSuccess) return e;
    }
    kb_temporal<<<nblk[kGridHalf], dim3(kBX, kBY), 0, st>>>(jobs, njobs);
    kb_blur_median_mips<<<nblk[kGridMip], 64, 0, st>>>(jobs, njobs);
    kb_recon<<<nblk[kGridTiles], 256, 0, st>>>(jobs, njobs, rings);
    if (side) {
        const hipError_t e = hipStreamWaitEvent(st, side->join, 0);   // the post-process chain is done
        if (e != hipSuccess) return e;
    }
    kb_composite<<<nblk[kGridFull], dim3(kBX, kBY), 0, st>>>(head, jobs, njobs);
    if (taa & DOF_TAA_FINAL) kb_taa_final<<<nblk[kGridFull], dim3(kBX, kBY), 0, st>>>(jobs, njobs);
    return hipGetLastError();
}

}  // namespace dof
