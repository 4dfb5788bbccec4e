// Relaxed (real-valued) forward model and its adjoint, for encoder-side
// refinement of the dequantised residual planes and per-block shifts.
//
// Relaxed model: parameters are a real residual for every SRV value,
// res[c][node][y][x] (BFS node order), and a real shift per motion-compensated
// block, shift[rec] = (dx, dy) in pixels (initially the quarter-pel vector / 4;
// Phase-shifted Motion Compensation).  A reference SRV equals its residual
// plane; a predictive SRV is phase * bilinear(reference, shifted) + its
// residual, without rounding; a sample is root + the sum of its path's SRVs;
// the colour inverse is the linear one (R = Y + Co/2 - Cg/2, G = Y + Cg/2,
// B = Y - Co/2 - Cg/2); nothing is clamped; rendering is the quadrilinear
// blend of the renderer.  Within a block every pixel has the same bilinear
// fraction (floor(x + dx) = x + floor(dx)), which both directions use.
//
// Adjoint, deterministic (the sort counts its digits, and the tables the views
// to walk, by integer atomics; nothing else is atomic):
//  1. views whose homographies separate by axis get per-view tables of the
//     columns and rows that reach each light-field column, row and view;
//  2. if some view does not separate, or the tables would cost more, its rays
//     emit one record per light-field view they blend, keyed by the sample at the top-left of
//     their 2x2 pixel footprint (ray * 4 + view corner), which a stable radix
//     sort groups by key;
//  3. every sample gathers the rays that reach it, view by view from the
//     tables, then from the records keyed at itself and at its left, upper
//     and upper-left neighbours in ray order, and applies the colour
//     transpose, writing the level-0 node gradients and, from registers, up
//     to two levels of their sums;
//  4. the remaining levels are summed level by level in fixed order;
//  5. each block's shift gradient is a fixed-order reduction over its pixels,
//     and the block leaves a record: phase, split shift, and whether any of
//     its gradients is non-zero;
//  6. each reference residual pulls the phase-signed bilinear transpose of
//     its predictive siblings' gradients, from the recorded blocks.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lf_internal.h"

#define AD_MAX_PARTS 1024  // partial maxima of the shift reduction
#define AD_SORT_WG 512     // workgroups of the record sort, each owning a range of the records
#define AD_SORT_T 1024     // threads of each
#define AD_TILE 16         // reference tile side of the pull kernel
#define AD_FAR 48          // reach up to which positions outside the image are folded (three tiles)

// n / d for 0 <= n < 2^20, d >= 1: (n + 1/2) / d is at least 1 / (2 d) from
// an integer, and the rounded reciprocal and product are off by less than
// (n / d) 2^-22
__device__ __forceinline__ int lf_small_div(int n, int d)
{
    return (int)(((float)n + 0.5f) * __builtin_amdgcn_rcpf((float)d));
}

__device__ __forceinline__ float ad_lerp(float p, float q, float f) { return fmaf(f, q - p, p); }

// Integer part of a shift component along an axis of n pixels, f its floor:
// clamped to [-n - 1, n], which leaves every clamped tap where it was and
// keeps pixel + shift + 1 an ordinary integer for every float (out of range,
// the conversion and the sum are undefined, and the address made of them is
// wild).
__device__ __forceinline__ int ad_whole(float f, int n) { return (int)fminf(fmaxf(f, (float)(-n - 1)), (float)n); }

// four (two) consecutive floats at any 4-byte aligned address, one load
typedef float ad_f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float ad_f2 __attribute__((ext_vector_type(2), aligned(4)));

// element i of a uniform base, i * sizeof(T) below 2^32: one scalar base and
// one 32-bit offset register per load
template <class T, class E>
__device__ __forceinline__ T ad_ld(const E* __restrict__ base, uint32_t i)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(E));
}

struct AdRay {
    int a0, a1, b0, b1, x0, x1, y0, y1;
    float fu, fv, fs, ft;
};

__device__ __forceinline__ AdRay ad_ray(const LfGeom& g, const float* __restrict__ cam, int i, int j)
{
    AdRay r;
    float u, v, s, t;
    lf_ray(cam, i, j, u, v, s, t);
    lf_axis(u, g.na, r.a0, r.a1, r.fu);
    lf_axis(v, g.nb, r.b0, r.b1, r.fv);
    lf_axis(s, g.w, r.x0, r.x1, r.fs);
    lf_axis(t, g.h, r.y0, r.y1, r.ft);
    return r;
}

// phase of record j of (channel c, level l): 2-bit codes, sixteen to a word
__device__ __forceinline__ int ad_phase_at(const LfGeom& g, const LfPtrs& p, int c, int l, uint32_t j)
{
    const uint32_t code = (p.mv[g.sig_word[c][l] + (j >> 4)] >> (2u * (j & 15u))) & 3u;
    return code == 0u ? 1 : (code == 1u ? -1 : 0);
}

// ---------------------------------------------------------------------------
// parameter export: dequantised residuals and vector / 4
// ---------------------------------------------------------------------------

__global__ void k_export_residual(LfGeom g, LfPtrs p, float* __restrict__ res)
{
    const int64_t plane = (int64_t)g.w * g.h;
    const int64_t total = 3 * (int64_t)g.n_nodes * plane;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t px = t % plane;
        const int node = (int)((t / plane) % g.n_nodes);
        const int c = (int)(t / (plane * g.n_nodes));
        int l = 0;
        while (node < g.node_base[l]) l++;
        const int y = (int)(px / g.w), x = (int)(px % g.w);
        const int blk = (y / g.bs) * g.nbx + x / g.bs, i = (y % g.bs) * g.bs + x % g.bs;
        res[t] = (float)lf_residual(g, p, c, l, node, blk, i);
    }
}

__global__ void k_export_shift(LfGeom g, LfPtrs p, int64_t n_rec, float2* __restrict__ shift)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rec) return;
    int c = 0, l = g.H - 1;
    while (c < 2 && r >= g.rec_base[c + 1][g.H - 1]) c++;
    while (l > 0 && r >= g.rec_base[c][l - 1]) l--;
    const uint32_t j = (uint32_t)(r - g.rec_base[c][l]);
    int mx, my, sg;
    lf_motion(g, p, c, l, j, mx, my, sg);
    shift[r] = make_float2((float)mx * 0.25f, (float)my * 0.25f);
}

extern "C" lf_status lf_export_params(const lf_handle* h, float* d_residual, float* d_shift, void* stream)
{
    if (!h || !d_residual || !d_shift) return lf_fail(LF_EINVAL, "null argument");
    if (lf_status cs = lf_require_full_chroma(h, "lf_export_params")) return cs;
    const LfGeom& g = h->L.g;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_export_residual, dim3(65536), dim3(256), 0, s, g, h->p, d_residual);
    if (h->L.n_rec > 0)
        hipLaunchKernelGGL(k_export_shift, dim3((unsigned)((h->L.n_rec + 255) / 256)), dim3(256), 0, s, g, h->p,
                           h->L.n_rec, (float2*)d_shift);
    return lf_check_launch("export_params");
}

// ---------------------------------------------------------------------------
// relaxed forward
// ---------------------------------------------------------------------------

// Relaxed SRV values of node (B, A) of level l, channel c, at the pixels
// (ys[k >> 1], xs[k & 1]): the residual plus the phase-signed bilinear
// prediction.  The four pixels' loads are issued together; the two taps of a
// row come in one (columns q and q + 1, q at most w - 2; see ad_srv_nodes).
__device__ __forceinline__ void ad_srv_quad(const LfGeom& g, const LfPtrs& p, const float* __restrict__ res,
                                            const float2* __restrict__ shift, int c, int l, int B, int A, const int ys[2],
                                            const int xs[2], float v[4])
{
    const int64_t plane = (int64_t)g.w * g.h;
    const float* S = res + ((int64_t)c * g.n_nodes + g.node_base[l] + B * g.na_l[l] + A) * plane;
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = S[ys[k >> 1] * g.w + xs[k & 1]];
    if (!((A | B) & 1)) return;
    const float* R = res + ((int64_t)c * g.n_nodes + g.node_base[l] + (B & ~1) * g.na_l[l] + (A & ~1)) * plane;
    const uint32_t j0 = (uint32_t)pred_ordinal(g.na_l[l], B, A) * (uint32_t)g.nblk;
    const float2* sh = shift + g.rec_base[c][l] + j0;
    int sg[4];
    float2 d[4];
    ad_f2 ta[4], tb[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int blk = (ys[k >> 1] >> g.bsl) * g.nbx + (xs[k & 1] >> g.bsl);
        sg[k] = ad_phase_at(g, p, c, l, j0 + (uint32_t)blk);
        d[k] = sh[blk];
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int x0 = xs[k & 1] + ad_whole(floorf(d[k].x), g.w), y0 = ys[k >> 1] + ad_whole(floorf(d[k].y), g.h);
        const int q = max(min(lf_clampi(x0, 0, g.w - 1), g.w - 2), 0);
        ta[k] = *reinterpret_cast<const ad_f2*>(R + lf_clampi(y0, 0, g.h - 1) * g.w + q);
        tb[k] = *reinterpret_cast<const ad_f2*>(R + lf_clampi(y0 + 1, 0, g.h - 1) * g.w + q);
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const float fdx = floorf(d[k].x), fx = d[k].x - fdx, fy = d[k].y - floorf(d[k].y);
        const int x0 = xs[k & 1] + ad_whole(fdx, g.w);
        const int xa = lf_clampi(x0, 0, g.w - 1), xb = lf_clampi(x0 + 1, 0, g.w - 1), q = max(min(xa, g.w - 2), 0);
        const float t = ad_lerp(ad_lerp(xa > q ? ta[k].y : ta[k].x, xb > q ? ta[k].y : ta[k].x, fx),
                                ad_lerp(xa > q ? tb[k].y : tb[k].x, xb > q ? tb[k].y : tb[k].x, fx), fy);
        if (sg[k]) v[k] += sg[k] > 0 ? t : -t;
    }
}

// One channel of the 16 samples of a ray (view k >> 2 = b0a0, b0a1, b1a0,
// b1a1, pixel k & 3): root plus the relaxed SRVs of levels 0 .. H-1, added in
// that order; views sharing a tree node share its evaluation.
__device__ __forceinline__ void ad_ray_channel(const LfGeom& g, const LfPtrs& p, const float* __restrict__ res,
                                               const float2* __restrict__ shift, const AdRay& r, int c, float acc[16])
{
    const int ys[2] = {r.y0, r.y1}, xs[2] = {r.x0, r.x1};
    const int64_t plane = (int64_t)g.w * g.h;
    const int H = g.H;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int b = (q & 2) ? r.b1 : r.b0, a = (q & 1) ? r.a1 : r.a0;
        const int16_t* rt = p.root + ((size_t)(c * g.root_nb + (b >> H)) * g.root_na + (a >> H)) * plane;
#pragma unroll
        for (int k = 0; k < 4; k++) acc[4 * q + k] = (float)rt[ys[k >> 1] * g.w + xs[k & 1]];
    }
    for (int l = 0; l < H; l++) {
        const bool eqA = (r.a0 >> l) == (r.a1 >> l), eqB = (r.b0 >> l) == (r.b1 >> l);
        float v[4][4];
        ad_srv_quad(g, p, res, shift, c, l, r.b0 >> l, r.a0 >> l, ys, xs, v[0]);
        if (!eqA) ad_srv_quad(g, p, res, shift, c, l, r.b0 >> l, r.a1 >> l, ys, xs, v[1]);
        if (!eqB) ad_srv_quad(g, p, res, shift, c, l, r.b1 >> l, r.a0 >> l, ys, xs, v[2]);
        if (!eqA && !eqB) ad_srv_quad(g, p, res, shift, c, l, r.b1 >> l, r.a1 >> l, ys, xs, v[3]);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            if (eqA) v[1][k] = v[0][k];
            if (eqB) v[2][k] = v[0][k];
            if (eqB) v[3][k] = v[1][k];
            else if (eqA) v[3][k] = v[2][k];
#pragma unroll
            for (int q = 0; q < 4; q++) acc[4 * q + k] += v[q][k];
        }
    }
}

// Relaxed SRVs of N nodes of level l at one pixel (block blk), all three
// channels: the residual plus the phase-signed bilinear prediction.  Level
// and nodes are uniform across the wave.  All residual, phase and shift loads
// are issued first, then all taps, so that a level costs two round trips to
// memory.  The two taps of a row come in one load: columns q and q + 1 with q
// at most w - 2 (a plane one column wide reads one element of the next plane;
// a reference with predictive siblings is never the buffer's last).
template <int N>
__device__ __forceinline__ void ad_srv_nodes(const LfGeom& g, const LfPtrs& p, const float* __restrict__ res,
                                             const float2* __restrict__ shift, int l, const int (&B)[N], const int (&A)[N],
                                             int y, int x, int blk, float (&o)[N][3])
{
    const int64_t plane = (int64_t)g.w * g.h;
    const float* level = res + (int64_t)g.node_base[l] * plane;
    uint32_t code[N][3];
    float2 d[N][3];
    ad_f2 ta[N][3], tb[N][3];
#pragma unroll
    for (int n = 0; n < N; n++) {
        const bool pred = (A[n] | B[n]) & 1;
        const uint32_t j0 = (uint32_t)pred_ordinal(g.na_l[l], B[n], A[n]) * (uint32_t)g.nblk;
#pragma unroll
        for (int c = 0; c < 3; c++) {
            o[n][c] = ad_ld<float>(level + ((int64_t)c * g.n_nodes + B[n] * g.na_l[l] + A[n]) * plane, (uint32_t)(y * g.w + x));
            if (pred) {
                const uint32_t j = j0 + (uint32_t)blk;
                code[n][c] = (ad_ld<uint32_t>(p.mv + g.sig_word[c][l], j >> 4) >> (2u * (j & 15u))) & 3u;
                d[n][c] = ad_ld<float2>(shift + g.rec_base[c][l] + j0, (uint32_t)blk);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < N; n++)
        if ((A[n] | B[n]) & 1)
#pragma unroll
            for (int c = 0; c < 3; c++) {
                const float* R = level + ((int64_t)c * g.n_nodes + (B[n] & ~1) * g.na_l[l] + (A[n] & ~1)) * plane;
                const int x0 = x + ad_whole(floorf(d[n][c].x), g.w), y0 = y + ad_whole(floorf(d[n][c].y), g.h);
                const int q = max(min(lf_clampi(x0, 0, g.w - 1), g.w - 2), 0);
                ta[n][c] = ad_ld<ad_f2>(R, (uint32_t)(lf_clampi(y0, 0, g.h - 1) * g.w + q));
                tb[n][c] = ad_ld<ad_f2>(R, (uint32_t)(lf_clampi(y0 + 1, 0, g.h - 1) * g.w + q));
            }
#pragma unroll
    for (int n = 0; n < N; n++)
        if ((A[n] | B[n]) & 1)
#pragma unroll
            for (int c = 0; c < 3; c++) {
                const float fdx = floorf(d[n][c].x), fx = d[n][c].x - fdx, fy = d[n][c].y - floorf(d[n][c].y);
                const int x0 = x + ad_whole(fdx, g.w);
                const int xa = lf_clampi(x0, 0, g.w - 1), xb = lf_clampi(x0 + 1, 0, g.w - 1), q = max(min(xa, g.w - 2), 0);
                const float v = ad_lerp(ad_lerp(xa > q ? ta[n][c].y : ta[n][c].x, xb > q ? ta[n][c].y : ta[n][c].x, fx),
                                        ad_lerp(xa > q ? tb[n][c].y : tb[n][c].x, xb > q ? tb[n][c].y : tb[n][c].x, fx), fy);
                if (code[n][c] < 2u) o[n][c] += code[n][c] == 0u ? v : -v;  // code 2, 3: no prediction
            }
}

// Colour of one sample; the (s, t) blend of a view's four samples (row
// major); the (u, v) blend of the four views, scaled and stored.
__device__ __forceinline__ void ad_rgb(float Y, float Co, float Cg, float (&o)[3])
{
    o[0] = Y + 0.5f * Co - 0.5f * Cg;
    o[1] = Y + 0.5f * Cg;
    o[2] = Y - 0.5f * Co - 0.5f * Cg;
}

__device__ __forceinline__ void ad_blend_view(const float (&sm)[4][3], const AdRay& ry, float (&vw)[3])
{
#pragma unroll
    for (int c = 0; c < 3; c++) vw[c] = ad_lerp(ad_lerp(sm[0][c], sm[1][c], ry.fs), ad_lerp(sm[2][c], sm[3][c], ry.fs), ry.ft);
}

__device__ __forceinline__ void ad_blend_store(const float (&vw)[4][3], const AdRay& ry, float* __restrict__ out, int64_t npix,
                                               int64_t px)
{
#pragma unroll
    for (int c = 0; c < 3; c++)
        out[c * npix + px] =
            ad_lerp(ad_lerp(vw[0][c], vw[1][c], ry.fu), ad_lerp(vw[2][c], vw[3][c], ry.fu), ry.fv) * (1.0f / 255.0f);
}

#define AD_RT 32             // screen tile of the relaxed render: AD_RT x 8 pixels, an 8x8 part per wave64
#define AD_STAGE 10176       // floats of LDS per workgroup: 40 KB with the boxes, four workgroups per CU
#define AD_MARK 0x7FC0DEADu  // NaN payload at a part's first pixel: left to the per-ray pass

typedef unsigned short ad_u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t ad_pk_min(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(ad_u16x2, a), __builtin_bit_cast(ad_u16x2, b)));
}
__device__ __forceinline__ uint32_t ad_pk_max(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ad_u16x2, a), __builtin_bit_cast(ad_u16x2, b)));
}

// Relaxed render of 32x8 screen tiles: the samples that a tile's rays read
// (every pixel of their bounding box, in every light-field view of theirs)
// are reconstructed once into LDS, one plane per channel and light-field
// view, and the rays blend from there.  Reconstructing them ray by ray
// evaluates three times as many samples at unit magnification.  A wave takes
// 64 box pixels at a time, in 2x2 light-field views, so that everything about
// a tree node is scalar and views sharing a node share its value; the three
// channels of up to four nodes are in flight together, because the chain of
// dependent loads (shift, then taps, per level) is what bounds a tile.
// A tile whose box exceeds the LDS (the rays' footprints spread over more than
// about 1.6 light-field pixels per ray) is marked for k_relaxed_rest, where
// each sample is read by about one ray.  The sums, and their order, are those
// of the per-ray pass.  16 views of 512x512 over 17x17x512x512: 2.19 -> 0.74
// ms, three views of 250x187 over 9x9x256x256: 0.146 -> 0.058 ms (all rays
// one by one before).  30 KB of LDS, five workgroups per CU: 0.72 and 0.059
// ms for this kernel, but tiles whose rays span 3x3 views then go to the
// per-ray pass: 0.90 and 0.097 ms in all.
__global__ void __launch_bounds__(256, 4) k_render_relaxed(LfGeom g, LfPtrs p, const float* __restrict__ res,
                                                           const float2* __restrict__ shift,
                                                           const float* __restrict__ cams, int wo, int ho, int tiles_x,
                                                           int tiles_y, int64_t n_tiles, float* __restrict__ out)
{
    __shared__ float stage[AD_STAGE];
    __shared__ uint32_t boxes[4][4];
    const int64_t npix = (int64_t)wo * ho;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int per = tiles_x * tiles_y, H = g.H;
    // XCD-aware order: each XCD takes a contiguous range of tiles (one tile a
    // workgroup, except in launches of more than 2^20 tiles)
    const int64_t per_xcd = (n_tiles + 7) / 8;
    for (int64_t k8 = blockIdx.x >> 3; k8 < per_xcd; k8 += gridDim.x >> 3) {
        const int64_t T = (int64_t)(blockIdx.x & 7) * per_xcd + k8;
        if (T >= n_tiles) return;
        const int v = (int)(T / per), tt = (int)(T - (int64_t)v * per);
        const int tyi = tt / tiles_x, txi = tt - tyi * tiles_x;
        const int i = txi * AD_RT + wv * 8 + (lane & 7), j = tyi * 8 + (lane >> 3);
        const AdRay ry = ad_ray(g, cams + 18 * (int64_t)v, min(i, wo - 1), min(j, ho - 1));  // dead lanes repeat the last pixel
        uint32_t m[4] = {(uint32_t)ry.a0 | ((uint32_t)ry.b0 << 16), (uint32_t)ry.a1 | ((uint32_t)ry.b1 << 16),
                         (uint32_t)ry.x0 | ((uint32_t)ry.y0 << 16), (uint32_t)ry.x1 | ((uint32_t)ry.y1 << 16)};
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1)
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t t = (uint32_t)__shfl_xor((int)m[k], s, 64);
                m[k] = (k & 1) ? ad_pk_max(m[k], t) : ad_pk_min(m[k], t);
            }
        if (lane == 0)
#pragma unroll
            for (int k = 0; k < 4; k++) boxes[wv][k] = m[k];
        __syncthreads();
        uint32_t box[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            uint32_t t = boxes[0][k];
            for (int w = 1; w < 4; w++) t = (k & 1) ? ad_pk_max(t, boxes[w][k]) : ad_pk_min(t, boxes[w][k]);
            box[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
        }
        const int amin = (int)(box[0] & 0xFFFFu), bmin = (int)(box[0] >> 16), amax = (int)(box[1] & 0xFFFFu),
                  bmax = (int)(box[1] >> 16);
        const int xmin = (int)(box[2] & 0xFFFFu), ymin = (int)(box[2] >> 16), nx = (int)(box[3] & 0xFFFFu) - xmin + 1,
                  ny = (int)(box[3] >> 16) - ymin + 1;
        const int nA = amax - amin + 1, nB = bmax - bmin + 1, nbox = nx * ny;
        float* o = out + (int64_t)v * 3 * npix;
        if (3 * (int64_t)nbox * nA * nB > AD_STAGE) {  // uniform
            if (lane == 0 && i < wo) o[(int64_t)j * wo + i] = __uint_as_float(AD_MARK);
            __syncthreads();  // the next tile rewrites the boxes
            continue;
        }
        const int cs = nA * nB * nbox;  // channel stride in LDS
        for (int e0 = wv * 64; e0 < nbox; e0 += 256) {
            const int e = min(e0 + lane, nbox - 1);  // past the end: the last pixel again (same value)
            const int yy = lf_small_div(e, nx);
            const int y = ymin + yy, x = xmin + e - yy * nx;
            const int blk = (y >> g.bsl) * g.nbx + (x >> g.bsl);
            for (int b = bmin; b <= bmax; b += 2)
                for (int a = amin; a <= amax; a += 2) {
                    const int b1 = min(b + 1, bmax), a1 = min(a + 1, amax);
                    float acc[4][3];
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const int bb = (q & 2) ? b1 : b, aa = (q & 1) ? a1 : a;
#pragma unroll
                        for (int c = 0; c < 3; c++)
                            acc[q][c] = (float)ad_ld<int16_t>(
                                p.root + ((size_t)(c * g.root_nb + (bb >> H)) * g.root_na + (aa >> H)) * ((size_t)g.w * g.h),
                                (uint32_t)(y * g.w + x));
                    }
                    for (int l = 0; l < H; l++) {
                        const int B0 = b >> l, B1 = b1 >> l, A0 = a >> l, A1 = a1 >> l;
                        if (B0 == B1 && A0 == A1) {  // uniform: views of the 2x2 that share the node share its value
                            float s[1][3];
                            ad_srv_nodes<1>(g, p, res, shift, l, {B0}, {A0}, y, x, blk, s);
#pragma unroll
                            for (int q = 0; q < 4; q++)
#pragma unroll
                                for (int c = 0; c < 3; c++) acc[q][c] += s[0][c];
                        } else if (B0 == B1 || A0 == A1) {
                            float s[2][3];
                            ad_srv_nodes<2>(g, p, res, shift, l, {B0, B1}, {A0, A1}, y, x, blk, s);
#pragma unroll
                            for (int q = 0; q < 4; q++)
#pragma unroll
                                for (int c = 0; c < 3; c++) {
                                    const bool second = B0 == B1 ? (q & 1) : (q & 2);
                                    acc[q][c] += second ? s[1][c] : s[0][c];
                                }
                        } else {
#pragma unroll
                            for (int h = 0; h < 2; h++) {
                                float s[2][3];
                                ad_srv_nodes<2>(g, p, res, shift, l, {h ? B1 : B0, h ? B1 : B0}, {A0, A1}, y, x, blk, s);
#pragma unroll
                                for (int q = 0; q < 2; q++)
#pragma unroll
                                    for (int c = 0; c < 3; c++) acc[2 * h + q][c] += s[q][c];
                            }
                        }
                    }
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const int bb = b + (q >> 1), aa = a + (q & 1);
                        if (bb <= bmax && aa <= amax)
#pragma unroll
                            for (int c = 0; c < 3; c++) stage[c * cs + ((bb - bmin) * nA + aa - amin) * nbox + e] = acc[q][c];
                    }
                }
        }
        __syncthreads();
        if (i < wo && j < ho) {
            float vw[4][3];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int b = (q & 2) ? ry.b1 : ry.b0, a = (q & 1) ? ry.a1 : ry.a0;
                const float* view = stage + ((b - bmin) * nA + a - amin) * nbox;
                float sm[4][3];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int y = (k & 2) ? ry.y1 : ry.y0, x = (k & 1) ? ry.x1 : ry.x0;
                    const float* s = view + (y - ymin) * nx + x - xmin;
                    ad_rgb(s[0], s[cs], s[2 * cs], sm[k]);
                }
                ad_blend_view(sm, ry, vw[q]);
                __builtin_amdgcn_sched_barrier(0);  // one view's samples in registers at a time
            }
            ad_blend_store(vw, ry, o, npix, (int64_t)j * wo + i);
        }
        __syncthreads();  // the next tile rewrites the boxes and the stage
    }
}

// Ray-by-ray render of the 8x8 parts that k_render_relaxed marked: a wave
// looks at `each` parts and renders the marked ones.  60 views of 64x64 over
// 17x17x512x512, every part marked: 0.22 ms (0.33 with the four pixels of a
// node read one after the other).
__global__ void __launch_bounds__(256) k_relaxed_rest(LfGeom g, LfPtrs p, const float* __restrict__ res,
                                                      const float2* __restrict__ shift, const float* __restrict__ cams,
                                                      int wo, int ho, int parts_x, int parts_y, int64_t n_parts, int each,
                                                      float* __restrict__ out)
{
    const int64_t npix = (int64_t)wo * ho;
    const int lane = threadIdx.x & 63;
    const int per = parts_x * parts_y;
    for (int64_t p0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * each; p0 < n_parts; p0 += (int64_t)gridDim.x * 4 * each) {
        bool mine = false;
        if (lane < each && p0 + lane < n_parts) {
            const int v = (int)((p0 + lane) / per), t = (int)((p0 + lane) - (int64_t)v * per);
            const int py = t / parts_x, px = t - py * parts_x;
            mine = __float_as_uint(out[(int64_t)v * 3 * npix + (int64_t)(py * 8) * wo + px * 8]) == AD_MARK;
        }
        for (uint64_t m = __ballot(mine); m; m &= m - 1) {
            const int64_t pt = p0 + __builtin_ctzll(m);
            const int v = (int)(pt / per), t = (int)(pt - (int64_t)v * per);
            const int py = t / parts_x, i = (t - py * parts_x) * 8 + (lane & 7), j = py * 8 + (lane >> 3);
            if (i >= wo || j >= ho) continue;
            const AdRay ry = ad_ray(g, cams + 18 * (int64_t)v, i, j);
            float Ys[16], Cos[16], Cgs[16];
            ad_ray_channel(g, p, res, shift, ry, 0, Ys);
            ad_ray_channel(g, p, res, shift, ry, 1, Cos);
            ad_ray_channel(g, p, res, shift, ry, 2, Cgs);
            float vw[4][3];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                float sm[4][3];
#pragma unroll
                for (int k = 0; k < 4; k++) ad_rgb(Ys[4 * q + k], Cos[4 * q + k], Cgs[4 * q + k], sm[k]);
                ad_blend_view(sm, ry, vw[q]);
            }
            ad_blend_store(vw, ry, out + (int64_t)v * 3 * npix, npix, (int64_t)j * wo + i);
        }
    }
}

extern "C" lf_status lf_render_relaxed(const lf_handle* h, const float* d_residual, const float* d_shift,
                                       const float* d_cams, int32_t n_views, int32_t width, int32_t height, float* d_out,
                                       void* stream)
{
    if (!h || !d_residual || !d_shift || n_views < 0 || width < 1 || height < 1) return lf_fail(LF_EINVAL, "bad argument");
    if (lf_status cs = lf_require_full_chroma(h, "lf_render_relaxed")) return cs;
    if (n_views == 0) return LF_OK;
    if (!d_cams || !d_out) return lf_fail(LF_EINVAL, "null buffer");
    const int64_t total = (int64_t)n_views * width * height;
    if ((total + 255) / 256 > 0x7FFFFFFF) return lf_fail(LF_EINVAL, "too many rays");
    const int tx = (width + AD_RT - 1) / AD_RT, ty = (height + 7) / 8, px = (width + 7) / 8;
    const int64_t n_tiles = (int64_t)n_views * tx * ty, n_parts = (int64_t)n_views * px * ty;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_render_relaxed, dim3((unsigned)std::min<int64_t>((n_tiles + 7) / 8 * 8, 1 << 20)), dim3(256), 0, s, h->L.g, h->p,
                       d_residual, (const float2*)d_shift, d_cams, width, height, tx, ty, n_tiles, d_out);
    // marked parts: one per wave while that fills the chip, then up to eight
    // (mostly unmarked) per wave
    const int each = (int)std::min<int64_t>(std::max<int64_t>(n_parts / 8192, 1), 8);
    const int64_t wgs = (n_parts + 4 * each - 1) / (4 * each);
    hipLaunchKernelGGL(k_relaxed_rest, dim3((unsigned)std::min<int64_t>(wgs, 1 << 20)), dim3(256), 0, s, h->L.g, h->p,
                       d_residual, (const float2*)d_shift, d_cams, width, height, px, ty, n_parts, each, d_out);
    return lf_check_launch("render_relaxed");
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------

struct BwdLayout {
    int64_t n_recs, n_samples;
    int passes;     // of the record sort, 8 bits each
    bool use_axes;  // build the separable views' tables
    int64_t o_kin, o_kout, o_vin, o_vout, o_hist, o_start, o_max, o_parts, o_rayf, o_brec;
    int64_t o_sep, o_col, o_row, o_rx, o_ry, o_ra, o_rb, o_count, o_list, total;
};

static int64_t al256(int64_t v) { return (v + 255) & ~(int64_t)255; }

static lf_status bwd_layout(const lf_handle* h, int nv, int wo, int ho, BwdLayout* B)
{
    const LfGeom& g = h->L.g;
    B->n_recs = (int64_t)nv * wo * ho * 4;
    B->n_samples = (int64_t)g.na * g.nb * g.w * g.h;
    // records are numbered with 32 bits: at most 2^31 - 1 (2^29 - 1 rays per call)
    if (B->n_recs > 0x7FFFFFFFll) return lf_fail(LF_EINVAL, "too many rays for one backward call (at most 2^29 - 1)");
    if (B->n_samples >= 0xFFFFFFFFll) return lf_fail(LF_EINVAL, "too many light-field samples");
    // the reference pull indexes its 16x16 tiles with 32-bit integers
    if (3 * (int64_t)g.n_refs * ((g.w + AD_TILE - 1) / AD_TILE) * ((g.h + AD_TILE - 1) / AD_TILE) > 0x7FFFFFFFll)
        return lf_fail(LF_EINVAL, "too many reference tiles for the adjoint");
    int eb = 1;  // keys 0 .. n_samples
    while (eb < 32 && ((int64_t)1 << eb) <= B->n_samples) eb++;
    B->passes = (eb + 7) / 8;
    // The separable views' gather walks, per sample, the views that reach its
    // light-field view: never worth it where a view's pixels are fewer than a
    // light-field view's samples / 256 (a view reaches four light-field views
    // or more), nor made where the tables would be larger than the records.
    // What the views of a call reach is known on the device (ad_by_records).
    const int64_t tables = (int64_t)nv * (16 * ((int64_t)wo + ho) + 8 * ((int64_t)g.w + g.h + g.na + g.nb) +
                                          4 * (int64_t)g.na * g.nb + 4);
    B->use_axes = (int64_t)wo * ho * 256 >= (int64_t)g.w * g.h && tables <= 16 * B->n_recs + (1 << 20);
    int64_t o = 0;
    auto take = [&](int64_t bytes) {
        const int64_t at = o;
        o += al256(bytes);
        return at;
    };
    B->o_kin = take(B->n_recs * 4);
    B->o_kout = take(B->n_recs * 4);
    B->o_vin = take(B->n_recs * 4);
    B->o_vout = take(B->n_recs * 4);
    B->o_hist = take(AD_SORT_WG * 256 * 4);
    B->o_start = take(B->n_samples * 4);
    B->o_max = take(256);  // AdFlags
    B->o_parts = take(AD_MAX_PARTS * 4);
    B->o_rayf = take(B->n_recs / 4 * 16);  // one float4 per ray
    B->o_brec = take(h->L.n_rec * 16);     // one split shift per predictive block
    const int64_t k = B->use_axes ? nv : 0;
    B->o_sep = take(k * 4);
    B->o_col = take(k * wo * 16);
    B->o_row = take(k * ho * 16);
    B->o_rx = take(k * g.w * 8);
    B->o_ry = take(k * g.h * 8);
    B->o_ra = take(k * g.na * 8);
    B->o_rb = take(k * g.nb * 8);
    B->o_count = take(k ? (int64_t)g.na * g.nb * 4 : 0);
    B->o_list = take(k * g.na * g.nb * 4);
    B->total = o;
    return LF_OK;
}

extern "C" lf_status lf_backward_workspace(const lf_handle* h, int32_t n_views, int32_t width, int32_t height,
                                           int64_t* bytes)
{
    if (!h || !bytes || n_views < 1 || width < 1 || height < 1) return lf_fail(LF_EINVAL, "bad argument");
    if (lf_status cs = lf_require_full_chroma(h, "lf_backward_workspace")) return cs;
    BwdLayout B;
    lf_status st = bwd_layout(h, n_views, width, height, &B);
    if (st != LF_OK) return st;
    *bytes = B.total;
    return LF_OK;
}

// The words at o_max of the workspace.
struct AdFlags {
    float maxshift;
    int general;    // 1: some view does not separate (set by k_ad_axes)
    int nan_shift;  // 1: some shift component is NaN
    int pad;
    unsigned long long walked;  // sum over the light-field views of the separating views that reach them (k_ad_lists)
};

// ---- rays whose axes separate ----
//
// With every third row (0, 0, 1) and no cross terms, a camera's (u, s) depend
// on the pixel column alone and (v, t) on the row alone, each monotone along
// its axis.  The rays reaching sample (b, a, y, x) are then the pixels of a
// rectangle: columns whose x0 is x - 1 or x and whose a0 is a - 1 or a, rows
// likewise, and their blend weights are products of a column and a row factor.
// Such views need no records and no sort: per view, tables of the columns and
// rows and of the intervals that reach each x, y, a and b.
struct AdAxes {
    AdFlags* flags;
    int all_general;  // 1: no tables, every view goes by records
    uint64_t most;    // largest flags->walked with which the tables pay
    int* sep;         // [nv] 1: the view's axes separate
    float4 *col, *row;      // [nv][wo], [nv][ho]: (x0 | a0 << 16, fs, fu), (y0 | b0 << 16, ft, fv)
    int2 *rx, *ry, *ra, *rb;  // [nv][w], [nv][h], [nv][na], [nv][nb]: first and past-the-last column or row
    int *count, *list;      // [nb na], [nb na][nv]: separating views that reach light-field view (b, a), in order
};

// Views that go by records: none (0), those that do not separate (1), or all
// (2).  The tables' gather walks, per sample, every view that reaches its
// light-field view, most of them for nothing when small frames span many
// light-field views: 35 ps per wave of 64 samples and view, where a record
// costs about 50 ps and the record route 8 ps per sample.  Over 17x17 of
// 512x512, 32x32 views that each span the whole grid: 100 of them 4.50 ms by
// the tables and 1.76 by records, 1500 85.2 and 3.8; views from one point
// each: 100 1.99 and 2.64, 1500 7.24 and 8.87.
__device__ __forceinline__ int ad_by_records(const AdAxes& t)
{
    if (t.all_general || t.flags->walked > t.most) return 2;
    return t.flags->general;
}

__device__ __forceinline__ bool ad_separates(const float* __restrict__ cam)
{
    bool ok = true;
#pragma unroll
    for (int h = 0; h < 18; h += 9) {
        ok = ok && cam[h + 6] == 0.0f && cam[h + 7] == 0.0f && cam[h + 8] == 1.0f && cam[h + 1] == 0.0f && cam[h + 3] == 0.0f;
        // finite: x - x is 0 only for finite x
        ok = ok && cam[h] - cam[h] == 0.0f && cam[h + 2] - cam[h + 2] == 0.0f && cam[h + 4] - cam[h + 4] == 0.0f &&
             cam[h + 5] - cam[h + 5] == 0.0f;
    }
    return ok;
}

// Lower neighbour and fraction along one axis of n samples: coordinate 0 (u)
// or 1 (v) of homography h at pixel column (row) i.
__device__ __forceinline__ int ad_axis_at(const float* __restrict__ h, int which, int i, int n, float* f)
{
    float x, y;
    int k0, k1;
    lf_ray_h(h, (float)i + 0.5f, (float)i + 0.5f, x, y);  // no cross terms: the other pixel coordinate does not enter
    lf_axis(which ? y : x, n, k0, k1, *f);
    return k0;
}

// Interval of i in [0, len) whose lower neighbour is k - 1 or k.
__device__ __forceinline__ int2 ad_interval(const float* __restrict__ h, int which, int len, int n, int k)
{
    const bool up = h[which ? 4 : 0] >= 0.0f;  // the neighbour grows (or stays) with i, else it falls
    int edge[2];
#pragma unroll
    for (int e = 0; e < 2; e++) {
        // first i whose neighbour is at least k - 1, then k + 1 (at most k, then k - 2)
        const int want = up ? k - 1 + 2 * e : k - 2 * e;
        int lo = 0, hi = len;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            float f;
            const int at = ad_axis_at(h, which, mid, n, &f);
            if (up ? at >= want : at <= want)
                hi = mid;
            else
                lo = mid + 1;
        }
        edge[e] = lo;
    }
    return make_int2(edge[0], edge[1]);
}

// Entry id of the tables (per entries a view): columns, rows, then the
// intervals.  The interval search costs 2 log2(len) coordinate evaluations.
__device__ __forceinline__ void ad_axes_entry(const LfGeom& g, const float* __restrict__ cams, int wo, int ho, const AdAxes& t,
                                              int64_t per, int64_t id)
{
    const int64_t v = id / per;
    int e = (int)(id - v * per);
    const float* cam = cams + 18 * v;
    const bool sep = ad_separates(cam);
    if (e == 0) {
        t.sep[v] = sep;
        if (!sep) t.flags->general = 1;  // cleared by an earlier kernel; every writer stores 1
    }
    if (!sep) return;
    float fc, fu;
    if (e < wo) {
        const int x0 = ad_axis_at(cam + 9, 0, e, g.w, &fc), a0 = ad_axis_at(cam, 0, e, g.na, &fu);
        t.col[v * wo + e] = make_float4(__int_as_float(x0 | (a0 << 16)), fc, fu, 0.0f);
        return;
    }
    e -= wo;
    if (e < ho) {
        const int y0 = ad_axis_at(cam + 9, 1, e, g.h, &fc), b0 = ad_axis_at(cam, 1, e, g.nb, &fu);
        t.row[v * ho + e] = make_float4(__int_as_float(y0 | (b0 << 16)), fc, fu, 0.0f);
        return;
    }
    e -= ho;
    if (e < g.w) {
        t.rx[v * g.w + e] = ad_interval(cam + 9, 0, wo, g.w, e);
        return;
    }
    e -= g.w;
    if (e < g.h) {
        t.ry[v * g.h + e] = ad_interval(cam + 9, 1, ho, g.h, e);
        return;
    }
    e -= g.h;
    if (e < g.na)
        t.ra[v * g.na + e] = ad_interval(cam, 0, wo, g.na, e);
    else
        t.rb[v * g.nb + e - g.na] = ad_interval(cam, 1, ho, g.nb, e - g.na);
}

__global__ void k_ad_axes(LfGeom g, const float* __restrict__ cams, int nv, int wo, int ho, AdAxes t)
{
    const int64_t per = (int64_t)wo + ho + g.w + g.h + g.na + g.nb;
    for (int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; id < per * nv; id += (int64_t)gridDim.x * blockDim.x)
        ad_axes_entry(g, cams, wo, ho, t, per, id);
}

// Separating views that reach each light-field view, in view order: one
// wave64 per light-field view.
__global__ void __launch_bounds__(256) k_ad_lists(LfGeom g, int nv, AdAxes t)
{
    const int k = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (k >= g.na * g.nb) return;  // uniform per wave
    const int b = k / g.na, a = k - b * g.na;
    int n = 0;
    for (int v0 = 0; v0 < nv; v0 += 64) {
        const int v = v0 + lane;
        bool hit = false;
        if (v < nv && t.sep[v]) {
            const int2 ra = t.ra[(int64_t)v * g.na + a], rb = t.rb[(int64_t)v * g.nb + b];
            hit = ra.x < ra.y && rb.x < rb.y;
        }
        const uint64_t m = __ballot(hit);
        if (hit) t.list[(int64_t)k * nv + n + __popcll(m & ((1ull << lane) - 1ull))] = v;
        n += __popcll(m);
    }
    if (lane == 0) {
        t.count[k] = n;
        if (n) atomicAdd(&t.flags->walked, (unsigned long long)n);
    }
}

// ---- the other rays: records sorted by the sample they reach ----
//
// A stable least-significant-digit radix sort of (key, record), 8 bits a
// pass, workgroups each owning one contiguous range of the
// records: count the range's digits, then scatter in order.  Every kernel
// returns at once when no view goes by records.
struct AdSort {
    uint32_t *kin, *kout, *vin, *vout;  // ping-pong; the sorted records end in kin, vin after an even number of passes
    uint32_t* hist;                     // [AD_SORT_WG][256]
    int64_t n;                          // records: 4 per ray
    int64_t per;                        // records per workgroup (a multiple of 4)
};

__device__ __forceinline__ void ad_sort_count(uint32_t (&h)[256], const uint32_t* __restrict__ keys, int64_t begin, int64_t end,
                                              int shift)
{
    for (int64_t i = begin + threadIdx.x; i < end; i += AD_SORT_T) atomicAdd(&h[(keys[i] >> shift) & 255u], 1u);
}

// Records and blend fractions of every ray (a view that goes by the tables
// gets the key past every sample), the first digit's counts, and the empty key
// table.
__global__ void __launch_bounds__(AD_SORT_T) k_ad_records(LfGeom g, const float* __restrict__ cams, int nv, int wo, int ho,
                                                          AdAxes t, AdSort s, float4* __restrict__ rayf,
                                                          uint32_t* __restrict__ start, int64_t n_samples)
{
    const int by = ad_by_records(t);
    if (!by) return;
    __shared__ uint32_t h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t npix = (int64_t)wo * ho, rays = npix * nv;
    const int64_t begin = (int64_t)blockIdx.x * s.per / 4, end = min(begin + s.per / 4, rays);
    for (int64_t r = begin + threadIdx.x; r < end; r += AD_SORT_T) {
        const int v = (int)(r / npix);
        const int64_t px = r - (int64_t)v * npix;
        const bool use = by == 2 || !t.sep[v];
        const AdRay ry = ad_ray(g, cams + 18 * (int64_t)v, (int)(px % wo), (int)(px / wo));
        rayf[r] = make_float4(ry.fu, ry.fv, ry.fs, ry.ft);  // the blend fractions, for the gather pass
        uint32_t key[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int b = (q & 2) ? ry.b1 : ry.b0, a = (q & 1) ? ry.a1 : ry.a0;
            key[q] = use ? (uint32_t)((((int64_t)b * g.na + a) * g.h + ry.y0) * g.w + ry.x0) : (uint32_t)n_samples;
            atomicAdd(&h[key[q] & 255u], 1u);
        }
        reinterpret_cast<uint4*>(s.kin)[r] = make_uint4(key[0], key[1], key[2], key[3]);
        const uint32_t r4 = (uint32_t)(r * 4);
        reinterpret_cast<uint4*>(s.vin)[r] = make_uint4(r4, r4 + 1u, r4 + 2u, r4 + 3u);
    }
    for (int64_t i = (int64_t)blockIdx.x * AD_SORT_T + threadIdx.x; i < n_samples; i += (int64_t)gridDim.x * AD_SORT_T)
        start[i] = 0xFFFFFFFFu;
    __syncthreads();
    if (threadIdx.x < 256) s.hist[blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

__global__ void __launch_bounds__(AD_SORT_T) k_ad_sort_count(AdAxes t, AdSort s,
                                                             const uint32_t* __restrict__ keys, int shift)
{
    if (!ad_by_records(t)) return;
    __shared__ uint32_t h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * s.per;
    ad_sort_count(h, keys, begin, min(begin + s.per, s.n), shift);
    __syncthreads();
    if (threadIdx.x < 256) s.hist[blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

__global__ void __launch_bounds__(AD_SORT_T) k_ad_sort_scatter(AdAxes t, AdSort s,
                                                               const uint32_t* __restrict__ ki, const uint32_t* __restrict__ vi,
                                                               uint32_t* __restrict__ ko, uint32_t* __restrict__ vo, int shift)
{
    if (!ad_by_records(t)) return;
    constexpr int W = AD_SORT_T / 64;
    __shared__ uint32_t base[256];          // next output place of each digit
    __shared__ uint32_t cnt[W][256];        // this step's digit counts per wave
    __shared__ uint32_t wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // digit d: records of it in the workgroups before this one, and in all
    {
        const int d = tid & 255, part = tid >> 8;  // four threads per digit, a quarter of the workgroups each
        uint32_t before = 0, all = 0;
        for (int w = part * (AD_SORT_WG / 4); w < (part + 1) * (AD_SORT_WG / 4); w++) {
            const uint32_t c = s.hist[w * 256 + d];
            all += c;
            before += w < (int)blockIdx.x ? c : 0u;
        }
        cnt[part][d] = before;
        cnt[4 + part][d] = all;
    }
    __syncthreads();
    uint32_t before = 0, all = 0, inc = 0;
    if (tid < 256) {
        for (int q = 0; q < 4; q++) {
            before += cnt[q][tid];
            all += cnt[4 + q][tid];
        }
        inc = all;  // inclusive scan over the 256 digits
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t up = (uint32_t)__shfl_up((int)inc, o, 64);
            if (lane >= o) inc += up;
        }
        if (lane == 63) wsum[wv] = inc;
    }
    __syncthreads();
    if (tid < 256) {
        for (int q = 0; q < wv; q++) inc += wsum[q];
        base[tid] = inc - all + before;
    }
    for (int i = tid; i < W * 256; i += AD_SORT_T) (&cnt[0][0])[i] = 0;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * s.per, end = min(begin + s.per, s.n);
    for (int64_t i0 = begin; i0 < end; i0 += AD_SORT_T) {
        const int64_t i = i0 + tid;
        const bool in = i < end;
        const uint32_t key = in ? ki[i] : 0u, val = in ? vi[i] : 0u;
        const uint32_t d = (key >> shift) & 255u;
        // lanes of the wave with the same digit
        uint64_t same = __ballot(in);
#pragma unroll
        for (int bit = 0; bit < 8; bit++) {
            const bool one = (d >> bit) & 1u;
            const uint64_t m = __ballot(one);
            same &= one ? m : ~m;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        if (in && rank == 0) cnt[wv][d] = (uint32_t)__popcll(same);
        __syncthreads();
        if (in) {
            uint32_t at = base[d] + (uint32_t)rank;
            for (int q = 0; q < wv; q++) at += cnt[q][d];
            ko[at] = key;
            vo[at] = val;
        }
        __syncthreads();
        if (tid < 256) {
            uint32_t sum = 0;
            for (int q = 0; q < W; q++) {
                sum += cnt[q][tid];
                cnt[q][tid] = 0;
            }
            base[tid] += sum;
        }
        __syncthreads();
    }
}

// first record of every key present
__global__ void k_ad_heads(AdAxes t, const uint32_t* __restrict__ keys, int64_t n,
                           int64_t n_samples, uint32_t* __restrict__ start)
{
    if (!ad_by_records(t)) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t k = keys[i];
        if ((int64_t)k < n_samples && (i == 0 || keys[i - 1] != k)) start[k] = (uint32_t)i;
    }
}

// Sample gradients and sums in one launch, or in two, always or where records
// are to be gathered: the sample gradients alone first, then the sums.
enum AdPass { AD_WHOLE, AD_LEAVES, AD_SUMS, AD_RECORD_LEAVES, AD_RECORD_SUMS };

struct AdGather {
    AdAxes t;
    const float4* rayf;
    const float* grad_out;
    const uint32_t *keys, *vals, *start;
    int64_t n_recs;
    int nv, wo, ho;
};

// Gradient of the RGB sample (b, a, y, x): over the separating views that
// reach view (b, a), the rectangle of their pixels that reach (y, x); then,
// if some view goes by records (by > 0), those keyed at the sample and at its
// left, upper and upper-left neighbours.  A record keyed at the
// footprint corner (y0, x0) reaches pixel corner (cy, cx) at (y0 + cy, x0 +
// cx), except along an axis of length 1, where both corners are pixel 0.
__device__ __forceinline__ void ad_sample(const LfGeom& g, const AdGather& G, int b, int a, int y, int x, int by,
                                          float (&acc)[3])
{
    const int64_t npix = (int64_t)G.wo * G.ho;
    acc[0] = acc[1] = acc[2] = 0.0f;
    if (by < 2) {
        const int k = b * g.na + a, n = G.t.count[k];
        for (int q = 0; q < n; q++) {
            const int v = __builtin_amdgcn_readfirstlane(G.t.list[(int64_t)k * G.nv + q]);
            const int2 ra = G.t.ra[(int64_t)v * g.na + a], rb = G.t.rb[(int64_t)v * g.nb + b];
            const int2 rx = G.t.rx[(int64_t)v * g.w + x], ry = G.t.ry[(int64_t)v * g.h + y];
            const int i0 = max(ra.x, rx.x), i1 = min(ra.y, rx.y), j0 = max(rb.x, ry.x), j1 = min(rb.y, ry.y);
            const float4* col = G.t.col + (int64_t)v * G.wo;
            const float4* row = G.t.row + (int64_t)v * G.ho;
            const float* go = G.grad_out + (int64_t)v * 3 * npix;
            for (int j = j0; j < j1; j++) {
                const float4 r = row[j];
                const int yb = __float_as_int(r.x);
                const float wy = ((yb & 0xFFFF) == y ? 1.0f - r.y : r.y) * ((yb >> 16) == b ? 1.0f - r.z : r.z);
                for (int i = i0; i < i1; i++) {
                    const float4 c = col[i];
                    const int xa = __float_as_int(c.x);
                    const float wx = ((xa & 0xFFFF) == x ? 1.0f - c.y : c.y) * ((xa >> 16) == a ? 1.0f - c.z : c.z);
                    const float wt = wy * wx * (1.0f / 255.0f);
                    const int64_t px = (int64_t)j * G.wo + i;
#pragma unroll
                    for (int ch = 0; ch < 3; ch++) acc[ch] = fmaf(wt, go[ch * npix + px], acc[ch]);
                }
            }
        }
    }
    if (!by) return;
    const int64_t S = (((int64_t)b * g.na + a) * g.h + y) * g.w + x;
    for (int cy = 0; cy < 2; cy++) {
        const int dy = g.h >= 2 ? cy : 0;
        if (y < dy) continue;
        for (int cx = 0; cx < 2; cx++) {
            const int dx = g.w >= 2 ? cx : 0;
            if (x < dx) continue;
            const uint32_t K = (uint32_t)(S - (int64_t)dy * g.w - dx);
            uint32_t j = G.start[K];
            if (j == 0xFFFFFFFFu) continue;
            for (; (int64_t)j < G.n_recs && G.keys[j] == K; j++) {
                const uint32_t val = G.vals[j];
                const int64_t ray = val >> 2;
                const int q = (int)(val & 3u);
                const int v = (int)(ray / npix);
                const int64_t px = ray - (int64_t)v * npix;
                const float4 f = G.rayf[ray];  // (fu, fv, fs, ft)
                const float wt = ((q & 2) ? f.y : 1.0f - f.y) * ((q & 1) ? f.x : 1.0f - f.x) *
                                 (cy ? f.w : 1.0f - f.w) * (cx ? f.z : 1.0f - f.z) * (1.0f / 255.0f);
#pragma unroll
                for (int c = 0; c < 3; c++) acc[c] = fmaf(wt, G.grad_out[((int64_t)v * 3 + c) * npix + px], acc[c]);
            }
        }
    }
}

// Sample gradients and the node gradients above them.  One thread per pixel
// and cluster of 2^D x 2^D light-field views: it gathers each view's sample
// gradient, applies the colour transpose, writes the level-0 gradient (zero
// where no ray reaches), and writes levels 1 .. D as the sums of the children
// it has in registers, so that no level is read back.  Bound by writing
// every gradient once: 1.2 GB in 0.43 ms for 17x17 views of 512x512, 16
// views (records for every ray, a library radix sort, one thread per sample
// and a pass per tree level: 2.05 ms).
template <int D>
__global__ void __launch_bounds__(256) k_ad_gather(LfGeom g, AdGather G, int clusters, AdPass pass, float* __restrict__ gres)
{
    const int by = ad_by_records(G.t);
    if (pass == AD_RECORD_LEAVES && !by) return;
    const bool there = pass == AD_SUMS || (pass == AD_RECORD_SUMS && by);  // the sample gradients are in gres
    const int px = (int)(blockIdx.x * 256 + threadIdx.x);
    const int plane = g.w * g.h;
    if (px >= plane) return;
    const int y = px / g.w, x = px - y * g.w;
    const int nac = (g.na + (1 << D) - 1) >> D;
    const int64_t cstride = (int64_t)g.n_nodes * plane;
    auto put = [&](int l, int Bl, int Al, const float (&v)[3]) {
        float* o = gres + (int64_t)(g.node_base[l] + Bl * g.na_l[l] + Al) * plane + px;
        o[0] = v[0];
        o[cstride] = v[1];
        o[2 * cstride] = v[2];
    };
    auto leaf = [&](int b, int a, float (&o)[3]) {
        if (D > 0 && there) {
            const float* in = gres + (int64_t)(g.node_base[0] + b * g.na + a) * plane + px;
            o[0] = in[0];
            o[1] = in[cstride];
            o[2] = in[2 * cstride];
            return;
        }
        float acc[3];
        ad_sample(g, G, b, a, y, x, by, acc);
        // colour transpose of R = Y + Co/2 - Cg/2, G = Y + Cg/2, B = Y - Co/2 - Cg/2
        o[0] = acc[0] + acc[1] + acc[2];
        o[1] = 0.5f * (acc[0] - acc[2]);
        o[2] = 0.5f * (acc[1] - acc[0] - acc[2]);
        put(0, b, a, o);
    };
    for (int cl = blockIdx.y; cl < clusters; cl += gridDim.y) {
        const int B = cl / nac, A = cl - B * nac;
        if (D == 0) {
            float o[3];
            leaf(B, A, o);
            continue;
        }
        float top[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int q2 = 0; q2 < (D == 2 ? 4 : 1); q2++) {
            const int B1 = D == 2 ? 2 * B + (q2 >> 1) : B, A1 = D == 2 ? 2 * A + (q2 & 1) : A;
            if (B1 >= g.nb_l[1] || A1 >= g.na_l[1]) continue;
            float mid[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll 1
            for (int q1 = 0; q1 < 4; q1++) {
                const int b = 2 * B1 + (q1 >> 1), a = 2 * A1 + (q1 & 1);
                if (b >= g.nb || a >= g.na) continue;
                float o[3];
                leaf(b, a, o);
#pragma unroll
                for (int c = 0; c < 3; c++) mid[c] += o[c];
            }
            put(1, B1, A1, mid);
#pragma unroll
            for (int c = 0; c < 3; c++) top[c] += mid[c];
        }
        if (D == 2) put(2, B, A, top);
    }
}

// node gradients of a level the gather pass does not reach: the sum of its
// children's
__global__ void k_ad_tree(LfGeom g, int l, float* __restrict__ gres)
{
    const int64_t plane = (int64_t)g.w * g.h;
    const int64_t nodes_l = (int64_t)g.na_l[l] * g.nb_l[l];
    const int64_t total = 3 * nodes_l * plane;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t px = t % plane;
        const int64_t loc = (t / plane) % nodes_l;
        const int c = (int)(t / (plane * nodes_l));
        const int B = (int)(loc / g.na_l[l]), A = (int)(loc % g.na_l[l]);
        float v = 0.0f;
        for (int jj = 0; jj < 2; jj++)
            for (int ii = 0; ii < 2; ii++) {
                const int Bc = 2 * B + jj, Ac = 2 * A + ii;
                if (Bc >= g.nb_l[l - 1] || Ac >= g.na_l[l - 1]) continue;
                v += gres[((int64_t)c * g.n_nodes + g.node_base[l - 1] + Bc * g.na_l[l - 1] + Ac) * plane + px];
            }
        gres[((int64_t)c * g.n_nodes + g.node_base[l] + loc) * plane + px] = v;
    }
}

// largest |shift| component, NaN left out: AD_MAX_PARTS workgroups write
// partial maxima, negative (or -0) where a component is NaN, then one
// workgroup reduces them (a maximum is exact in any order)
__global__ void k_ad_maxshift(const float2* __restrict__ shift, int64_t n, float* __restrict__ out)
{
    __shared__ float red[256];
    float m = 0.0f;
    bool nan = false;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const float2 s = shift[t];
        m = fmaxf(m, fmaxf(fabsf(s.x), fabsf(s.y)));
        nan |= s.x != s.x || s.y != s.y;
    }
    red[threadIdx.x] = m;
    nan = __syncthreads_or(nan);
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = nan ? -red[0] : red[0];
}

__global__ void k_ad_maxparts(const float* __restrict__ parts, int n, AdFlags* __restrict__ out)
{
    __shared__ float red[256];
    float m = 0.0f;
    bool nan = false;
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
        m = fmaxf(m, fabsf(parts[t]));
        nan |= __float_as_int(parts[t]) < 0;
    }
    red[threadIdx.x] = m;
    nan = __syncthreads_or(nan);
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = AdFlags{red[0], 0, nan, 0, 0};
}

// pixel range [lo, hi] of [k0, k1] whose tap (x + fd + o), clamped to [0, n-1], equals X
__device__ __forceinline__ void ad_tap_range(int X, int n, int fd, int o, int k0, int k1, int& lo, int& hi)
{
    if (n == 1) {
        lo = k0;
        hi = k1;
    } else if (X == 0) {
        lo = k0;
        hi = min(k1, -fd - o);
    } else if (X == n - 1) {
        lo = max(k0, n - 1 - fd - o);
        hi = k1;
    } else {
        lo = max(k0, X - fd - o);
        hi = min(k1, X - fd - o);
    }
}

// Phase and split shift of one predictive block: integer part (clamped, see
// ad_whole) and fractional part.
struct AdRec {
    int sg, ix, iy;
    float fx, fy;
};

__device__ __forceinline__ int4 ad_pack(const AdRec& d)
{
    return make_int4(d.sg, (d.ix & 0xFFFF) | (d.iy << 16), __float_as_int(d.fx), __float_as_int(d.fy));
}

__device__ __forceinline__ AdRec ad_unpack(int4 v)
{
    return AdRec{v.x, (int)(int16_t)(v.y & 0xFFFF), v.y >> 16, __int_as_float(v.z), __int_as_float(v.w)};
}

// Split shift of a block with phase sg; sg 0 leaves it empty.
__device__ __forceinline__ AdRec ad_split(const LfGeom& g, int sg, float2 s)
{
    AdRec d{sg, 0, 0, 0.0f, 0.0f};
    if (sg) {
        const float fdx = floorf(s.x), fdy = floorf(s.y);
        d.fx = s.x - fdx;
        d.fy = s.y - fdy;
        d.ix = ad_whole(fdx, g.w);
        d.iy = ad_whole(fdy, g.h);
    }
    return d;
}

// What pixel (X, Y) on the border of a reference pulls from one predictive
// block (row ky, column kx) with gradient plane gp: the bilinear weights of the
// block's taps that are clamped onto the pixel or land there times the
// gradients of their pixels, phase-signed.
__device__ __forceinline__ float ad_border_pull(const LfGeom& g, const float* gp, int X, int Y, int ky, int kx, const AdRec& d)
{
    float acc = 0.0f;
    const int bx0 = kx * g.bs, by0 = ky * g.bs;
    for (int oy = 0; oy < 2; oy++) {
        int ylo, yhi;
        ad_tap_range(Y, g.h, d.iy, oy, by0, by0 + g.bs - 1, ylo, yhi);
        if (ylo > yhi) continue;
        const float wy = oy ? d.fy : 1.0f - d.fy;
        for (int ox = 0; ox < 2; ox++) {
            int xlo, xhi;
            ad_tap_range(X, g.w, d.ix, ox, bx0, bx0 + g.bs - 1, xlo, xhi);
            if (xlo > xhi) continue;
            const float wxy = wy * (ox ? d.fx : 1.0f - d.fx);
            float sum = 0.0f;
            for (int y = ylo; y <= yhi; y++)
                for (int x = xlo; x <= xhi; x++) sum += gp[y * g.w + x];
            acc = fmaf(wxy, sum, acc);
        }
    }
    return d.sg > 0 ? acc : -acc;
}

// One kept block of the reference pull: its record and place (scalar, from
// lane src of the candidates) and the five rows by two columns of source
// gradients that the four positions (Y0 + k, X) of a lane read.  The tap
// (oy, ox) landing on position (Y0 + k, X) comes from source pixel
// (Y0 + k - iy - oy, X - ix - ox) alone, when that lies in the block: rows
// ys .. ys + 4, columns xs - 1 and xs; others count as zero.
struct AdTaps {
    AdRec q;
    int bx, by;  // the block's first column and row
    float s0[5], s1[5];

    __device__ __forceinline__ void load(const LfGeom& g, const float* gp, int4 v, int kx, int ky, int src, int X, int Y0)
    {
        bx = __builtin_amdgcn_readlane(kx, src) << g.bsl;
        by = __builtin_amdgcn_readlane(ky, src) << g.bsl;
        q = ad_unpack(make_int4(__builtin_amdgcn_readlane(v.x, src), __builtin_amdgcn_readlane(v.y, src),
                                __builtin_amdgcn_readlane(v.z, src), __builtin_amdgcn_readlane(v.w, src)));
        const int xs = X - q.ix, ys = Y0 - q.iy - 1;
        const bool x0 = (unsigned)(xs - bx) < (unsigned)g.bs, x1 = (unsigned)(xs - 1 - bx) < (unsigned)g.bs;
        const int first = ys * g.w + xs;
        // a row outside the block reads the plane's first two elements, unused;
        // a plane of one element the one before it and its own
        const int outside = g.w * g.h > 1 ? 0 : -1;
#pragma unroll
        for (int t = 0; t < 5; t++) {
            const bool y = (unsigned)(ys + t - by) < (unsigned)g.bs;
            // both columns in one load: (xs - 1, xs), or (xs - 2, xs - 1) when
            // xs is past the block (a predictive plane is never the buffer's
            // first, so an element before it is still inside the buffer)
            const int at = y && (x0 || x1) ? first + t * g.w - (x0 ? 1 : 2) : outside;
            const ad_f2 a = *reinterpret_cast<const ad_f2*>(gp + at);
            s0[t] = y && x0 ? a.y : 0.0f;
            s1[t] = y && x1 ? (x0 ? a.x : a.y) : 0.0f;
        }
    }

    // far: pixels on the image border (live, not inner) collect every tap
    // clamped onto them here, instead of from the positions outside the image
    __device__ __forceinline__ void add(const LfGeom& g, const float* gp, bool far, const bool (&live)[4],
                                        const bool (&inner)[4], int X, int Y0, float (&acc)[4]) const
    {
        const float sg = (float)q.sg, gx = 1.0f - q.fx, gy = 1.0f - q.fy;
        const float w00 = sg * (gy * gx), w01 = sg * (gy * q.fx), w10 = sg * (q.fy * gx), w11 = sg * (q.fy * q.fx);
        float blk[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            blk[k] = w00 * s0[k + 1];
            blk[k] = fmaf(w01, s1[k + 1], blk[k]);
            blk[k] = fmaf(w10, s0[k], blk[k]);
            blk[k] = fmaf(w11, s1[k], blk[k]);
        }
        if (!far && w00 * 0.0f == 0.0f && w11 * 0.0f == 0.0f) {  // uniform: finite weights, so a tap outside adds zero
#pragma unroll
            for (int k = 0; k < 4; k++) acc[k] += blk[k];
            return;
        }
        const int cx = X - q.ix - bx, cy = Y0 - q.iy - by;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            // covered: one of the two columns and one of the two rows in the block
            const bool in = (unsigned)cx <= (unsigned)g.bs && (unsigned)(cy + k) <= (unsigned)g.bs;
            if (in && (!far || inner[k])) acc[k] += blk[k];
        }
        if (!far) return;
#pragma unroll 1
        for (int k = 0; k < 4; k++) {
            if (!live[k] || inner[k]) continue;
            const float t = ad_border_pull(g, gp, X, Y0 + k, by >> g.bsl, bx >> g.bsl, q);
            if (k == 0) acc[0] += t;
            if (k == 1) acc[1] += t;
            if (k == 2) acc[2] += t;
            if (k == 3) acc[3] += t;
        }
    }
};

// Reference residual gradient: own node gradient plus the phase-signed
// bilinear transpose of every predictive sibling's gradient (pull form).  One
// wave64 takes a 16x16 tile of one reference plane, each lane four rows of
// one column.  The candidate blocks (those within the largest shift of the
// tile) are examined one per lane; the ones whose shifted taps land in the
// tile and that hold a non-zero gradient are walked in (sibling, block row,
// block column) order with their record in scalar registers, and every lane
// reads the five rows by two columns of source pixels its four taps need.
// A block left out adds exactly zero to every pixel of the tile.
//
// Bound by latency and issue (a tile's prologue and candidate test take about
// 300 instructions, a kept block 80 and five loads).  Staging the siblings'
// windows (tile plus the largest shift on every side) in LDS instead read 17
// values per pixel where the kept blocks hold about four, and two thirds of a
// tile's time went into waiting for them.  17x17 views of 512x512, 16
// rendered views (a quarter of the gradients non-zero): 3.77 -> 0.57 ms;
// 9x9 views of 256x256, three views: 0.288 -> 0.040 ms.  Four tiles per wave
// in sequence: 0.55 and 0.059 ms (too few waves on the small field).
__global__ void __launch_bounds__(256) k_ad_reference(LfGeom g, const int4* __restrict__ brec,
                                                      const AdFlags* __restrict__ flags, float* gres)
{
    const int plane = g.w * g.h;  // at most 2^28
    const int tiles_x = (g.w + AD_TILE - 1) / AD_TILE, tiles_y = (g.h + AD_TILE - 1) / AD_TILE;
    // 32-bit indices (the host bounds the tile count by 2^31 - 1)
    const int per_plane = tiles_x * tiles_y;
    const int n_tiles = 3 * g.n_refs * per_plane;
    // workgroup ids go round-robin over the 8 XCDs: each XCD takes a
    // contiguous range of tiles, so neighbouring tiles share its L2
    const int wg = (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
    const int T = __builtin_amdgcn_readfirstlane(wg * 4 + (int)(threadIdx.x >> 6));
    if (T >= n_tiles) return;  // uniform per wave
    const int lane = threadIdx.x & 63;
    const int reach = __builtin_amdgcn_readfirstlane((int)ceilf(fminf(flags->maxshift, (float)(g.w + g.h))) + 2);
    const int rp = T / per_plane, tt = T - rp * per_plane;
    const int c = rp / g.n_refs, r = rp - c * g.n_refs;
    int l = 0;
    while (l + 1 < g.H && r >= g.ref_base[l + 1]) l++;
    const int loc = r - g.ref_base[l], nar = g.na_l[l + 1], na = g.na_l[l];
    const int Bp = loc / nar, Br = 2 * Bp, Ar = 2 * (loc - Bp * nar);
    const int trow = tt / tiles_x;
    // siblings 1 (right), 2 (below) and 3: present or not, gradient plane, first record
    const bool h1 = Ar + 1 < na, h2 = Br + 1 < g.nb_l[l], h3 = h1 && h2;
    float* own = gres + ((int64_t)c * g.n_nodes + g.node_base[l] + Br * na + Ar) * plane;
    const float *gp1 = own + plane, *gp2 = own + (int64_t)na * plane, *gp3 = gp2 + plane;
    const int4* rec = brec + g.rec_base[c][l];
    const uint32_t r1 = (uint32_t)(pred_ordinal(na, Br, Ar + 1) * g.nblk), r2 = (uint32_t)(pred_ordinal(na, Br + 1, Ar) * g.nblk),
                   r3 = r2 + (uint32_t)g.nblk;  // the sibling below's right neighbour is the next node of its row
    const int ty0 = trow * AD_TILE, ty1 = min(ty0 + AD_TILE - 1, g.h - 1);
    const int cky0 = max(0, ty0 - reach) >> g.bsl, nky = min(g.h - 1, ty1 + reach) / g.bs - cky0 + 1;
    const int Y0 = ty0 + (lane >> 4) * 4;
    // shifts too far for the sets of outside positions, or NaN, which the
    // reach leaves out: a border pixel walks the source pixels of every tap
    // clamped onto it instead
    const bool far = reach > AD_FAR || __builtin_amdgcn_readfirstlane(flags->nan_shift);
    const int nv = (reach + AD_TILE - 1) / AD_TILE;
    const int tx0 = (tt - trow * tiles_x) * AD_TILE, tx1 = min(tx0 + AD_TILE - 1, g.w - 1);
    const int ckx0 = max(0, tx0 - reach) >> g.bsl, nkx = (min(g.w - 1, tx1 + reach) >> g.bsl) - ckx0 + 1;
    const int nk = nkx * nky;
    const int X = tx0 + (lane & 15);
    bool live[4], inner[4];
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 4; k++) {
        live[k] = X <= tx1 && Y0 + k <= ty1;
        inner[k] = X > 0 && X < g.w - 1 && Y0 + k > 0 && Y0 + k < g.h - 1;
    }
    bool touched = false;  // a tile that no block reaches is left as it is
    // A tile on the image border also takes the 16x16 sets of positions
    // outside the image next to it that taps can reach, and folds them
    // onto its border pixels (where the forward clamps those taps).
    const int vx0 = !far && tx0 == 0 ? -nv : 0, vx1 = !far && tx1 == g.w - 1 ? nv : 0;
    const int vy0 = !far && ty0 == 0 ? -nv : 0, vy1 = !far && ty1 == g.h - 1 ? nv : 0;
    for (int vy = vy0; vy <= vy1; vy++)
        for (int vx = vx0; vx <= vx1; vx++) {
            const int px0 = tx0 + vx * AD_TILE, py0 = ty0 + vy * AD_TILE;  // positions of this set
            const int PX = X + vx * AD_TILE, PY = Y0 + vy * AD_TILE;
            float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            bool some = false;
            for (int k0 = 0; k0 < 3 * nk; k0 += 64) {
                // one candidate block per lane, (sibling, row, column) order
                const int e = k0 + lane;
                const int sib = e >= 2 * nk ? 3 : (e >= nk ? 2 : 1), es = e - (sib - 1) * nk;
                const int ey = nk < (1 << 18) ? lf_small_div(es, nkx) : es / nkx;  // uniform choice
                const int kx = ckx0 + es - ey * nkx, ky = cky0 + ey;
                int4 v = make_int4(0, 0, 0, 0);
                if (e < 3 * nk && (sib == 1 ? h1 : (sib == 2 ? h2 : h3)))
                    v = rec[(sib == 1 ? r1 : (sib == 2 ? r2 : r3)) + (uint32_t)(ky * g.nbx + kx)];
                const AdRec d = ad_unpack(v);
                // taps of the block's pixels: [k bs + i, k bs + bs + i] per axis (far: clamped)
                int xlo = (kx << g.bsl) + d.ix, ylo = (ky << g.bsl) + d.iy, xhi = xlo + g.bs, yhi = ylo + g.bs;
                if (far) {
                    xlo = lf_clampi(xlo, 0, g.w - 1);
                    xhi = lf_clampi(xhi, 0, g.w - 1);
                    ylo = lf_clampi(ylo, 0, g.h - 1);
                    yhi = lf_clampi(yhi, 0, g.h - 1);
                }
                const bool keep = d.sg != 0 && xlo <= px0 + AD_TILE - 1 && xhi >= px0 && ylo <= py0 + AD_TILE - 1 &&
                                  yhi >= py0;
                uint64_t m = __ballot(keep);
                some |= m != 0;
                // two kept blocks at a time: the second's loads are in
                // flight while the first's are used
                while (m) {
                    const int src0 = __builtin_ctzll(m);
                    m &= m - 1;
                    const bool two = m != 0;  // uniform
                    const int src1 = two ? __builtin_ctzll(m) : src0;
                    m &= m - 1;
                    const int s0 = __builtin_amdgcn_readlane(sib, src0), s1 = __builtin_amdgcn_readlane(sib, src1);
                    const float* p0 = s0 == 1 ? gp1 : (s0 == 2 ? gp2 : gp3);
                    const float* p1 = s1 == 1 ? gp1 : (s1 == 2 ? gp2 : gp3);
                    AdTaps t0, t1;
                    t0.load(g, p0, v, kx, ky, src0, PX, PY);
                    if (two) t1.load(g, p1, v, kx, ky, src1, PX, PY);
                    t0.add(g, p0, far, live, inner, PX, PY, part);
                    if (two) t1.add(g, p1, far, live, inner, PX, PY, part);
                }
            }
            if (!some) continue;  // uniform
            touched = true;
            if (!far && (vx != 0 || vy != 0 || px0 + AD_TILE > g.w || py0 + AD_TILE > g.h)) {
                // positions left and right of the image onto its first and
                // last column, then those above and below onto its rows
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    float lo = PX < 0 ? part[k] : 0.0f, hi = PX >= g.w ? part[k] : 0.0f;
#pragma unroll
                    for (int o = 8; o >= 1; o >>= 1) {
                        lo += __shfl_xor(lo, o, 64);
                        hi += __shfl_xor(hi, o, 64);
                    }
                    part[k] = PX < 0 || PX >= g.w || vx != 0 ? 0.0f : part[k];
                    if (X == 0) part[k] += lo;
                    if (X == g.w - 1) part[k] += hi;
                }
                float lo = 0.0f, hi = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    lo += PY + k < 0 ? part[k] : 0.0f;
                    hi += PY + k >= g.h ? part[k] : 0.0f;
                    if (PY + k < 0 || PY + k >= g.h || vy != 0) part[k] = 0.0f;
                }
#pragma unroll
                for (int o = 16; o <= 32; o <<= 1) {
                    lo += __shfl_xor(lo, o, 64);
                    hi += __shfl_xor(hi, o, 64);
                }
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    if (Y0 + k == 0) part[k] += lo;
                    if (Y0 + k == g.h - 1) part[k] += hi;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; k++) acc[k] += part[k];
        }
    if (!touched) return;
#pragma unroll
    for (int k = 0; k < 4; k++)
        if (live[k]) own[(Y0 + k) * g.w + X] += acc[k];
}

// Predictive nodes of a tree as the shift pass numbers them: per channel,
// level H-1 first, raster order (the records' order); first[l] is the first
// node of level l.
struct AdPred {
    int total, first[LF_MAX_LEVELS];
};

// Shift gradients and block records.  A workgroup takes consecutive blocks of
// one predictive node, 2^LG lanes a block; each lane sums its pixels in
// order, then a fixed tree adds the lanes.  QUADS: a lane takes rows of four
// pixels (one 128-bit gradient load, five taps of each of two reference
// rows), so a 16x16 block is one wave64, an 8x8 block 16 lanes and a 4x4
// block four; with 16x16 blocks a wave takes AD_SHIFT_U blocks whose loads
// are in flight together.  Bound by the two passes over memory it cannot do
// without (every predictive gradient, every reference residual): 1.27 GB in
// 0.42 ms for 17x17 views of 512x512 (0.79 ms with one pixel per lane and
// load; 0.99 with five single loads per row of four).
#define AD_SHIFT_U 4
template <int LG, bool QUADS>
__global__ void __launch_bounds__(256) k_ad_shift(LfGeom g, LfPtrs p, AdPred pn, int groups, int n_wg,
                                                  const float* __restrict__ res, const float2* __restrict__ shift,
                                                  const float* __restrict__ gres_pred, float2* __restrict__ gshift,
                                                  int4* __restrict__ brec)
{
    constexpr int G = 1 << LG, U = LG == 6 ? AD_SHIFT_U : 1, PER = U * (256 / G);
    // one group of blocks a workgroup, except in launches of more than 2^22
    for (int wg = (int)blockIdx.x; wg < n_wg; wg += (int)gridDim.x) {
        // the node, scalar
        const int cn = wg / groups;
        const int c = cn / pn.total, np = cn - c * pn.total;
        int l = g.H - 1;
        while (l > 0 && np >= pn.first[l - 1]) l--;
        const int pord = np - pn.first[l], na = g.na_l[l], pair = na + na / 2;
        int B = 2 * (pord / pair), A;
        const int rem = pord % pair;
        if (rem < na / 2) {  // even rows hold the odd columns, odd rows every column
            A = 2 * rem + 1;
        } else {
            B += 1;
            A = rem - na / 2;
        }
        const int64_t plane = (int64_t)g.w * g.h;
        const float* R = res + ((int64_t)c * g.n_nodes + g.node_base[l] + (B & ~1) * na + (A & ~1)) * plane;
        const float* gp = gres_pred + ((int64_t)c * g.n_nodes + g.node_base[l] + B * na + A) * plane;
        const int64_t rec0 = g.rec_base[c][l] + (int64_t)pord * g.nblk;
        const uint32_t* code = p.mv + g.sig_word[c][l];
        const uint32_t j0 = (uint32_t)pord * (uint32_t)g.nblk;

        const int lane = threadIdx.x & (G - 1);
        const int sub = LG == 6 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : (int)(threadIdx.x >> LG);
        const int blk0 = (wg - cn * groups) * PER + sub * U;
        constexpr int N = QUADS ? 4 : 1;           // pixels per item
        const int rowl = g.bsl - (QUADS ? 2 : 0);  // log2 items per block row
        const int items = 1 << (g.bsl + rowl);
        AdRec d[U];
        float sx[U], sy[U];
        bool some[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int blk = min(blk0 + u, g.nblk - 1);  // past the end: the last block again, not stored
            const uint32_t j = j0 + (uint32_t)blk, cw = (code[j >> 4] >> (2u * (j & 15u))) & 3u;
            d[u] = ad_split(g, cw == 0u ? 1 : (cw == 1u ? -1 : 0), shift[rec0 + blk]);
            sx[u] = sy[u] = 0.0f;
            some[u] = false;
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int blk = min(blk0 + u, g.nblk - 1);
            const int ky = blk / g.nbx;
            const int by0 = ky << g.bsl, bx0 = (blk - ky * g.nbx) << g.bsl;
            const float fx = d[u].fx, fy = d[u].fy, gx = 1.0f - fx, gy = 1.0f - fy, sg = (float)d[u].sg;
            if (d[u].sg)
                for (int q = lane; q < items; q += G) {
                    const int y = by0 + (q >> rowl), x = bx0 + (q & ((1 << rowl) - 1)) * N;
                    float gv[N];
                    if (QUADS) {
                        const float4 t = *reinterpret_cast<const float4*>(gp + y * g.w + x);
                        gv[0] = t.x;
                        gv[N > 1 ? 1 : 0] = t.y;
                        gv[N > 2 ? 2 : 0] = t.z;
                        gv[N > 3 ? 3 : 0] = t.w;
                    } else {
                        gv[0] = gp[y * g.w + x];
                    }
                    const int ra = lf_clampi(y + d[u].iy, 0, g.h - 1) * g.w, rb = lf_clampi(y + d[u].iy + 1, 0, g.h - 1) * g.w;
                    float ta[N + 1], tb[N + 1];
                    const int xt = x + d[u].ix;
                    if (QUADS && xt >= 0 && xt + 4 < g.w) {
                        const ad_f4 a = *reinterpret_cast<const ad_f4*>(R + ra + xt), b = *reinterpret_cast<const ad_f4*>(R + rb + xt);
                        ta[N] = R[ra + xt + N];
                        tb[N] = R[rb + xt + N];
#pragma unroll
                        for (int t = 0; t < N; t++) {
                            ta[t] = a[t];
                            tb[t] = b[t];
                        }
                    } else {
#pragma unroll
                        for (int t = 0; t <= N; t++) {
                            const int xc = lf_clampi(xt + t, 0, g.w - 1);
                            ta[t] = R[ra + xc];
                            tb[t] = R[rb + xc];
                        }
                    }
#pragma unroll
                    for (int t = 0; t < N; t++) {
                        some[u] |= gv[t] != 0.0f;
                        const float v = sg * gv[t];
                        sx[u] = fmaf(v, gy * (ta[t + 1] - ta[t]) + fy * (tb[t + 1] - tb[t]), sx[u]);
                        sy[u] = fmaf(v, gx * (tb[t] - ta[t]) + fx * (tb[t + 1] - ta[t + 1]), sy[u]);
                    }
                }
        }
        uint64_t any[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            any[u] = __ballot(some[u]);
            if (LG < 6) any[u] = (any[u] >> (threadIdx.x & 63 & ~(G - 1))) & ((1ull << (G & 63)) - 1ull);
#pragma unroll
            for (int o = G / 2; o >= 1; o >>= 1) {
                sx[u] += __shfl_xor(sx[u], o, 64);
                sy[u] += __shfl_xor(sy[u], o, 64);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (lane == u && blk0 + u < g.nblk) {
                gshift[rec0 + blk0 + u] = make_float2(sx[u], sy[u]);
                // a block whose gradients are all zero adds zero to its reference
                // through finite weights: its record is empty
                AdRec e = d[u];
                if (!any[u] && e.fx * 0.0f == 0.0f && e.fy * 0.0f == 0.0f) e.sg = 0;
                brec[rec0 + blk0 + u] = ad_pack(e);
            }
    }
}

extern "C" lf_status lf_render_backward(const lf_handle* h, const float* d_residual, const float* d_shift,
                                        const float* d_cams, int32_t n_views, int32_t width, int32_t height,
                                        const float* d_grad_out, float* d_grad_residual, float* d_grad_shift,
                                        void* d_workspace, int64_t workspace_bytes, void* stream)
{
    if (!h || !d_residual || !d_shift || !d_cams || !d_grad_out || !d_grad_residual || !d_grad_shift || !d_workspace ||
        n_views < 1 || width < 1 || height < 1)
        return lf_fail(LF_EINVAL, "bad argument");
    if (lf_status cs = lf_require_full_chroma(h, "lf_render_backward")) return cs;
    const LfGeom& g = h->L.g;
    BwdLayout Bl;
    lf_status st = bwd_layout(h, n_views, width, height, &Bl);
    if (st != LF_OK) return st;
    if (workspace_bytes < Bl.total)
        return lf_fail(LF_ENOMEM, "workspace of %lld bytes, %lld needed", (long long)workspace_bytes, (long long)Bl.total);
    if (((uintptr_t)d_workspace) & 255) return lf_fail(LF_EINVAL, "workspace must be 256-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    uint8_t* W = (uint8_t*)d_workspace;
    AdFlags* flags = (AdFlags*)(W + Bl.o_max);
    float* parts = (float*)(W + Bl.o_parts);
    hipLaunchKernelGGL(k_ad_maxshift, dim3(AD_MAX_PARTS), dim3(256), 0, s, (const float2*)d_shift, h->L.n_rec, parts);
    hipLaunchKernelGGL(k_ad_maxparts, dim3(1), dim3(256), 0, s, parts, AD_MAX_PARTS, flags);
    AdAxes t;
    t.sep = (int*)(W + Bl.o_sep);
    t.flags = flags;
    t.all_general = !Bl.use_axes;
    // per light-field view and per record of a pixel; at 128 a record 1500
    // pinhole views of 64x64 over 17x17 of 256x256 took the tables, 4.52 ms
    // (2.79 by records)
    t.most = (uint64_t)(16 * (int64_t)g.na * g.nb + 64 * Bl.n_recs / ((int64_t)g.w * g.h));
    t.col = (float4*)(W + Bl.o_col);
    t.row = (float4*)(W + Bl.o_row);
    t.rx = (int2*)(W + Bl.o_rx);
    t.ry = (int2*)(W + Bl.o_ry);
    t.ra = (int2*)(W + Bl.o_ra);
    t.rb = (int2*)(W + Bl.o_rb);
    t.count = (int*)(W + Bl.o_count);
    t.list = (int*)(W + Bl.o_list);
    if (Bl.use_axes) {
        const int64_t items = n_views * ((int64_t)width + height + g.w + g.h + g.na + g.nb);
        hipLaunchKernelGGL(k_ad_axes, dim3((unsigned)std::min<int64_t>((items + 255) / 256, 1 << 20)), dim3(256), 0, s, g, d_cams, n_views, width,
                           height, t);
        hipLaunchKernelGGL(k_ad_lists, dim3((unsigned)((g.na * g.nb + 3) / 4)), dim3(256), 0, s, g, n_views, t);
    }
    AdSort srt;
    srt.kin = (uint32_t*)(W + Bl.o_kin);
    srt.kout = (uint32_t*)(W + Bl.o_kout);
    srt.vin = (uint32_t*)(W + Bl.o_vin);
    srt.vout = (uint32_t*)(W + Bl.o_vout);
    srt.hist = (uint32_t*)(W + Bl.o_hist);
    srt.n = Bl.n_recs;
    srt.per = ((Bl.n_recs / 4 + AD_SORT_WG - 1) / AD_SORT_WG) * 4;
    float4* rayf = (float4*)(W + Bl.o_rayf);
    uint32_t* start = (uint32_t*)(W + Bl.o_start);
    hipLaunchKernelGGL(k_ad_records, dim3(AD_SORT_WG), dim3(AD_SORT_T), 0, s, g, d_cams, n_views, width, height, t,
                       srt, rayf, start, Bl.n_samples);
    uint32_t *ki = srt.kin, *vi = srt.vin, *ko = srt.kout, *vo = srt.vout;
    for (int ps = 0; ps < Bl.passes; ps++) {
        if (ps > 0)
            hipLaunchKernelGGL(k_ad_sort_count, dim3(AD_SORT_WG), dim3(AD_SORT_T), 0, s, t, srt, ki,
                               8 * ps);
        hipLaunchKernelGGL(k_ad_sort_scatter, dim3(AD_SORT_WG), dim3(AD_SORT_T), 0, s, t, srt, ki, vi,
                           ko, vo, 8 * ps);
        std::swap(ki, ko);
        std::swap(vi, vo);
    }
    hipLaunchKernelGGL(k_ad_heads, dim3((unsigned)std::min<int64_t>((Bl.n_recs + 255) / 256, 8192)), dim3(256), 0, s,
                       t, ki, Bl.n_recs, Bl.n_samples, start);
    // level-0 gradients (every sample written) and up to two levels above
    const int64_t plane = (int64_t)g.w * g.h;
    AdGather ga{t, rayf, d_grad_out, ki, vi, start, Bl.n_recs, n_views, width, height};
    // Up to two levels above from a thread's registers, which gathers the
    // samples below (one pass, but up to 16 times fewer threads to gather with)
    // or reads their gradients back (two).  Waves of clusters of two levels, and
    // the call's time with one pass and with the samples by themselves (and a
    // pass a level): 102,400 (17x17 of 512x512), 24 views of 512x512
    // 1.67 and 2.15 ms; 25,600 (17x17 of 256x256), 16 views 527..690 and
    // 611..733 us; 9,216 (9x9 of 256x256), eight views of 256x256 (0.4 records
    // a sample) 161..190 and 189..203, 16 of 512x512 (3.2) 382..489 and
    // 317..382; 2,304 (9x9 of 128x128), two of 320x180 153 and 117; 256 (5x5 of
    // 64x64) 369 and 132.
    auto clusters_of = [&](int d) { return ((g.na + (1 << d) - 1) >> d) * ((g.nb + (1 << d) - 1) >> d); };
    auto gather = [&](int d, AdPass pass) {
        const int clusters = clusters_of(d);
        const int64_t wx = (plane + 255) / 256;
        // the launch that may find nothing to do is kept to 8,192 workgroups
        const int64_t wy = pass == AD_RECORD_LEAVES ? std::max<int64_t>(8192 / wx, 1) : 65535;
        hipLaunchKernelGGL(d == 0 ? k_ad_gather<0> : (d == 1 ? k_ad_gather<1> : k_ad_gather<2>),
                           dim3((unsigned)wx, (unsigned)std::min<int64_t>(clusters, wy)), dim3(256), 0, s, g, ga, clusters, pass,
                           d_grad_residual);
    };
    const int D = std::min(g.H - 1, 2);
    const int64_t waves = clusters_of(D) * plane / 64;
    const bool apart = waves < 4096 || (waves < 16384 && Bl.n_recs > 2 * Bl.n_samples);
    // Records take a chain of dependent loads each and are spread unevenly:
    // they want a thread a sample on larger fields too (17x17 of 256x256, two
    // projective views of 1280x720 2.20 and 1.92 ms; 5x5 of 64x64 34.3 and 7.5).
    const bool records_apart = waves < 32768 && 4 * Bl.n_recs > Bl.n_samples;
    if (D > 0 && (apart || records_apart)) {
        gather(0, apart ? AD_LEAVES : AD_RECORD_LEAVES);
        gather(D, apart ? AD_SUMS : AD_RECORD_SUMS);
    } else {
        gather(D, AD_WHOLE);
    }
    for (int l = D + 1; l < g.H; l++)
        hipLaunchKernelGGL(k_ad_tree, dim3(8192), dim3(256), 0, s, g, l, d_grad_residual);
    // the shift pass reads the predictive nodes' gradients, which the
    // reference pass leaves untouched, and writes the block records it pulls from
    int4* brec = (int4*)(W + Bl.o_brec);
    if (h->L.n_rec > 0) {
        // rows of four pixels are read as one 128-bit load: blocks of at least
        // 4x4 and a 16-byte aligned gradient buffer, else one pixel at a time
        const bool quads = g.bs >= 4 && !(((uintptr_t)d_grad_residual) & 15);
        const int lg = !quads ? 6 : (g.bs == 4 ? 2 : (g.bs == 8 ? 4 : 6));  // log2 lanes per block
        const int per_wg = (lg == 6 ? AD_SHIFT_U : 1) * (256 >> lg), groups = (g.nblk + per_wg - 1) / per_wg;
        AdPred pn = {};
        for (int l = g.H - 1; l >= 0; l--) {
            pn.first[l] = pn.total;
            pn.total += (g.nb_l[l] / 2) * g.na_l[l] + ((g.nb_l[l] + 1) / 2) * (g.na_l[l] / 2);
        }
        const auto kern = !quads    ? k_ad_shift<6, false>
                          : lg == 2 ? k_ad_shift<2, true>
                          : lg == 4 ? k_ad_shift<4, true>
                                    : k_ad_shift<6, true>;
        const int n_wg = 3 * pn.total * groups;
        hipLaunchKernelGGL(kern, dim3((unsigned)std::min(n_wg, 1 << 22)), dim3(256), 0, s, g, h->p, pn, groups, n_wg,
                           d_residual, (const float2*)d_shift, d_grad_residual, (float2*)d_grad_shift, brec);
    }
    const int64_t n_tiles = 3 * (int64_t)g.n_refs * ((g.w + AD_TILE - 1) / AD_TILE) * ((g.h + AD_TILE - 1) / AD_TILE);
    if (h->L.n_rec > 0)  // without predictive blocks the references keep their own gradients
        hipLaunchKernelGGL(k_ad_reference, dim3((unsigned)((n_tiles + 31) / 32 * 8)), dim3(256), 0, s, g,
                           (const int4*)brec, flags, d_grad_residual);
    return lf_check_launch("render_backward");
}
