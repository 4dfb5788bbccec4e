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
// Adjoint, deterministic and without atomics:
//  1. every ray emits one record per light-field view it blends, keyed by
//     the sample at the top-left of its 2x2 pixel footprint in that view
//     (ray * 4 + view corner), and its four blend fractions;
//  2. a stable radix sort groups the records by key, and a table gives the
//     first record of each key;
//  3. every sample gathers the records keyed at itself and at its left, upper
//     and upper-left neighbours (the footprints that cover it), in that order
//     and in ray order within each, forms each ray's blend weight from its
//     fractions and applies the colour transpose, writing the sample
//     gradients into the level-0 node planes;
//  4. node gradients are summed up the tree level by level in fixed order;
//  5. each block's shift gradient is a fixed-order reduction over its pixels,
//     and the block leaves a record: phase, split shift, and whether any of
//     its gradients is non-zero;
//  6. each reference residual pulls the phase-signed bilinear transpose of
//     its predictive siblings' gradients, from the recorded blocks.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>

#include "lf_internal.h"

#define AD_MAX_PARTS 1024  // partial maxima of the shift reduction
#define AD_TILE 16         // reference tile side of the pull kernel
#define AD_FAR 48          // reach up to which positions outside the image are folded (three tiles)

// n / d for 0 <= n <= 3072, 1 <= d <= 1024: the quotient of n + 1/2 is at
// least 1 / (2 d) from an integer, the rounded reciprocal and product are off
// by less than n 2^-22
__device__ __forceinline__ int lf_small_div(int n, int d)
{
    return (int)(((float)n + 0.5f) * __builtin_amdgcn_rcpf((float)d));
}

__device__ __forceinline__ float ad_lerp(float p, float q, float f) { return fmaf(f, q - p, p); }

// four (two) consecutive floats at any 4-byte aligned address, one load
typedef float ad_f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float ad_f2 __attribute__((ext_vector_type(2), aligned(4)));

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

// record index of predictive node (B, A) of level l, channel c, block blk
__device__ __forceinline__ int64_t ad_record(const LfGeom& g, int c, int l, int B, int A, int blk)
{
    return g.rec_base[c][l] + (int64_t)pred_ordinal(g.na_l[l], B, A) * g.nblk + blk;
}

// phase of record j of (channel c, level l): 2-bit codes, sixteen to a word
__device__ __forceinline__ int ad_phase_at(const LfGeom& g, const LfPtrs& p, int c, int l, uint32_t j)
{
    const uint32_t code = (p.mv[g.sig_word[c][l] + (j >> 4)] >> (2u * (j & 15u))) & 3u;
    return code == 0u ? 1 : (code == 1u ? -1 : 0);
}

__device__ __forceinline__ int ad_phase(const LfGeom& g, const LfPtrs& p, int c, int l, int B, int A, int blk)
{
    return ad_phase_at(g, p, c, l, (uint32_t)(pred_ordinal(g.na_l[l], B, A) * g.nblk + blk));
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

// bilinear sample of a real plane at (y + dy, x + dx), taps clamped
__device__ __forceinline__ float ad_bilerp(const float* __restrict__ R, int w, int h, int y, int x, float2 d)
{
    const float fdx = floorf(d.x), fdy = floorf(d.y);
    const float fx = d.x - fdx, fy = d.y - fdy;
    const int x0 = x + (int)fdx, y0 = y + (int)fdy;
    const int xa = lf_clampi(x0, 0, w - 1), xb = lf_clampi(x0 + 1, 0, w - 1);
    const int ya = lf_clampi(y0, 0, h - 1), yb = lf_clampi(y0 + 1, 0, h - 1);
    return ad_lerp(ad_lerp(R[ya * w + xa], R[ya * w + xb], fx), ad_lerp(R[yb * w + xa], R[yb * w + xb], fx), fy);
}

// Relaxed SRV values of node (B, A) of level l, channel c, at the pixels
// (ys[k >> 1], xs[k & 1]): the residual plus the phase-signed bilinear
// prediction; the block's phase and shift are read once per block.
__device__ inline void ad_srv_quad(const LfGeom& g, const LfPtrs& p, const float* __restrict__ res,
                                   const float2* __restrict__ shift, int c, int l, int B, int A, const int ys[2],
                                   const int xs[2], float v[4])
{
    const int64_t plane = (int64_t)g.w * g.h;
    const float* S = res + ((int64_t)c * g.n_nodes + g.node_base[l] + B * g.na_l[l] + A) * plane;
    const bool pred = (A | B) & 1;
    const float* R = res + ((int64_t)c * g.n_nodes + g.node_base[l] + (B & ~1) * g.na_l[l] + (A & ~1)) * plane;
    int blk0 = -1, sg = 0;
    float2 d = make_float2(0.0f, 0.0f);
#pragma unroll 1
    for (int k = 0; k < 4; k++) {
        const int y = ys[k >> 1], x = xs[k & 1];
        float sv = S[y * g.w + x];
        if (pred) {
            const int blk = (y / g.bs) * g.nbx + x / g.bs;
            if (blk != blk0) {
                sg = ad_phase(g, p, c, l, B, A, blk);
                if (sg) d = shift[ad_record(g, c, l, B, A, blk)];
                blk0 = blk;
            }
            if (sg) {
                const float q = ad_bilerp(R, g.w, g.h, y, x, d);
                sv += sg > 0 ? q : -q;
            }
        }
        v[k] = sv;
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

__global__ void __launch_bounds__(256) k_render_relaxed(LfGeom g, LfPtrs p, const float* __restrict__ res,
                                                        const float2* __restrict__ shift,
                                                        const float* __restrict__ cams, int nv, int wo, int ho,
                                                        float* __restrict__ out)
{
    const int64_t npix = (int64_t)wo * ho;
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= npix * nv) return;
    const int v = (int)(r / npix);
    const int64_t px = r - (int64_t)v * npix;
    const int j = (int)(px / wo), i = (int)(px % wo);
    const AdRay ry = ad_ray(g, cams + 18 * v, i, j);
    float Ys[16], Cos[16], Cgs[16];
    ad_ray_channel(g, p, res, shift, ry, 0, Ys);
    ad_ray_channel(g, p, res, shift, ry, 1, Cos);
    ad_ray_channel(g, p, res, shift, ry, 2, Cgs);
    float sm[16][3];
#pragma unroll
    for (int k = 0; k < 16; k++) {
        const float Y = Ys[k], Co = Cos[k], Cg = Cgs[k];
        sm[k][0] = Y + 0.5f * Co - 0.5f * Cg;
        sm[k][1] = Y + 0.5f * Cg;
        sm[k][2] = Y - 0.5f * Co - 0.5f * Cg;
    }
#pragma unroll
    for (int c = 0; c < 3; c++) {
        float vw[4];
#pragma unroll
        for (int q = 0; q < 4; q++)
            vw[q] = ad_lerp(ad_lerp(sm[4 * q][c], sm[4 * q + 1][c], ry.fs), ad_lerp(sm[4 * q + 2][c], sm[4 * q + 3][c], ry.fs),
                            ry.ft);
        out[((int64_t)v * 3 + c) * npix + px] =
            ad_lerp(ad_lerp(vw[0], vw[1], ry.fu), ad_lerp(vw[2], vw[3], ry.fu), ry.fv) * (1.0f / 255.0f);
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
    hipLaunchKernelGGL(k_render_relaxed, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       h->L.g, h->p, d_residual, (const float2*)d_shift, d_cams, n_views, width, height, d_out);
    return lf_check_launch("render_relaxed");
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------

struct BwdLayout {
    int64_t n_recs, n_samples;
    int end_bit;
    size_t sort_bytes;
    int64_t o_kin, o_kout, o_vin, o_vout, o_sort, o_start, o_max, o_parts, o_rayf, o_brec, total;
};

static int64_t al256(int64_t v) { return (v + 255) & ~(int64_t)255; }

static lf_status bwd_layout(const lf_handle* h, int nv, int wo, int ho, BwdLayout* B)
{
    const LfGeom& g = h->L.g;
    B->n_recs = (int64_t)nv * wo * ho * 4;
    B->n_samples = (int64_t)g.na * g.nb * g.w * g.h;
    // the record sort takes an int count: at most 2^31 - 1 records (2^29 - 1 rays per call)
    if (B->n_recs > 0x7FFFFFFFll) return lf_fail(LF_EINVAL, "too many rays for one backward call (at most 2^29 - 1)");
    if (B->n_samples >= 0xFFFFFFFFll) return lf_fail(LF_EINVAL, "too many light-field samples");
    // the reference pull indexes its 16x16 tiles with 32-bit integers
    if (3 * (int64_t)g.n_refs * ((g.w + AD_TILE - 1) / AD_TILE) * ((g.h + AD_TILE - 1) / AD_TILE) > 0x7FFFFFFFll)
        return lf_fail(LF_EINVAL, "too many reference tiles for the adjoint");
    int eb = 1;
    while (eb < 32 && ((int64_t)1 << eb) < B->n_samples) eb++;
    B->end_bit = eb;
    size_t sb = 0;
    if (hipcub::DeviceRadixSort::SortPairs(nullptr, sb, (uint32_t*)nullptr, (uint32_t*)nullptr, (uint32_t*)nullptr,
                                           (uint32_t*)nullptr, (int)B->n_recs, 0, eb) != hipSuccess)
        return lf_fail(LF_EDEVICE, "sort workspace query failed");
    B->sort_bytes = sb;
    const int64_t pb = al256(B->n_recs * 4);
    B->o_kin = 0;
    B->o_kout = B->o_kin + pb;
    B->o_vin = B->o_kout + pb;
    B->o_vout = B->o_vin + pb;
    B->o_sort = B->o_vout + pb;
    B->o_start = B->o_sort + al256((int64_t)sb);
    B->o_max = B->o_start + al256(B->n_samples * 4);
    B->o_parts = B->o_max + 256;
    B->o_rayf = B->o_parts + al256(AD_MAX_PARTS * 4);
    B->o_brec = B->o_rayf + al256(B->n_recs / 4 * 16);  // one float4 per ray
    B->total = B->o_brec + al256(h->L.n_rec * 16);         // one split shift per predictive block
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

__global__ void k_ad_records(LfGeom g, const float* __restrict__ cams, int nv, int wo, int ho,
                             uint32_t* __restrict__ keys, uint32_t* __restrict__ vals, float4* __restrict__ rayf)
{
    const int64_t npix = (int64_t)wo * ho;
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= npix * nv) return;
    const int v = (int)(r / npix);
    const int64_t px = r - (int64_t)v * npix;
    const AdRay ry = ad_ray(g, cams + 18 * v, (int)(px % wo), (int)(px / wo));
    rayf[r] = make_float4(ry.fu, ry.fv, ry.fs, ry.ft);  // the blend fractions, for the gather pass
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int b = (q & 2) ? ry.b1 : ry.b0, a = (q & 1) ? ry.a1 : ry.a0;
        keys[r * 4 + q] = (uint32_t)((((int64_t)b * g.na + a) * g.h + ry.y0) * g.w + ry.x0);
        vals[r * 4 + q] = (uint32_t)(r * 4 + q);
    }
}

__global__ void k_ad_nostart(uint32_t* __restrict__ start, int64_t n)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
        start[t] = 0xFFFFFFFFu;
}

// first record of every key present
__global__ void k_ad_heads(const uint32_t* __restrict__ keys, int64_t n, uint32_t* __restrict__ start)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t k = keys[i];
    if (i == 0 || keys[i - 1] != k) start[k] = (uint32_t)i;
}

// One thread per light-field sample ((b * na + a) * h + y) * w + x, which is
// also the offset of pixel (y, x) in the level-0 node planes of a channel, so
// the YCoCg sample gradients go straight into the residual gradient (channel
// stride cstride); samples no ray reaches get zero.  A record keyed at the
// footprint corner (y0, x0) reaches pixel corner (cy, cx) at (y0 + cy, x0 +
// cx), except along an axis of length 1, where both corners are pixel 0.
__global__ void k_ad_samples(const float4* __restrict__ rayf, int wo, int ho, const float* __restrict__ grad_out,
                             const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                             const uint32_t* __restrict__ start, int64_t n_recs, int64_t n_samples, int w, int h,
                             int64_t cstride, float* __restrict__ g0 /* level-0 planes of channel 0 */)
{
    const int64_t S = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (S >= n_samples) return;
    const int64_t npix = (int64_t)wo * ho;
    const int x = (int)(S % w), y = (int)((S / w) % h);
    float acc[3] = {0.0f, 0.0f, 0.0f};
    for (int cy = 0; cy < 2; cy++) {
        const int dy = h >= 2 ? cy : 0;
        if (y < dy) continue;
        for (int cx = 0; cx < 2; cx++) {
            const int dx = w >= 2 ? cx : 0;
            if (x < dx) continue;
            const uint32_t K = (uint32_t)(S - (int64_t)dy * w - dx);
            uint32_t j = start[K];
            if (j == 0xFFFFFFFFu) continue;
            for (; (int64_t)j < n_recs && keys[j] == K; j++) {
                const uint32_t val = vals[j];
                const int64_t ray = val >> 2;
                const int q = (int)(val & 3u);
                const int v = (int)(ray / npix);
                const int64_t px = ray - (int64_t)v * npix;
                const float4 f = rayf[ray];  // (fu, fv, fs, ft)
                const float wt = ((q & 2) ? f.y : 1.0f - f.y) * ((q & 1) ? f.x : 1.0f - f.x) *
                                 (cy ? f.w : 1.0f - f.w) * (cx ? f.z : 1.0f - f.z) * (1.0f / 255.0f);
#pragma unroll
                for (int c = 0; c < 3; c++) acc[c] = fmaf(wt, grad_out[((int64_t)v * 3 + c) * npix + px], acc[c]);
            }
        }
    }
    // colour transpose of R = Y + Co/2 - Cg/2, G = Y + Cg/2, B = Y - Co/2 - Cg/2
    g0[S] = acc[0] + acc[1] + acc[2];
    g0[cstride + S] = 0.5f * (acc[0] - acc[2]);
    g0[2 * cstride + S] = 0.5f * (acc[1] - acc[0] - acc[2]);
}

// node gradients of level l >= 1: the sum of its children's (level 0 holds
// the sample gradients themselves)
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

// largest |shift| component: AD_MAX_PARTS workgroups write partial maxima,
// then one workgroup reduces them (a maximum is exact in any order)
__global__ void k_ad_maxshift(const float2* __restrict__ shift, int64_t n, float* __restrict__ out)
{
    __shared__ float red[256];
    float m = 0.0f;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
        m = fmaxf(m, fmaxf(fabsf(shift[t].x), fabsf(shift[t].y)));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

__global__ void k_ad_maxparts(const float* __restrict__ parts, int n, float* __restrict__ out)
{
    __shared__ float red[256];
    float m = 0.0f;
    for (int t = threadIdx.x; t < n; t += blockDim.x) m = fmaxf(m, parts[t]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
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

// Phase and split shift of one predictive block: integer part (clamped to
// [-w-1, w] / [-h-1, h], which leaves every clamped tap where it was) and
// fractional part.
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
        d.ix = (int)fminf(fmaxf(fdx, (float)(-g.w - 1)), (float)g.w);
        d.iy = (int)fminf(fmaxf(fdy, (float)(-g.h - 1)), (float)g.h);
    }
    return d;
}

// What reference pixel (X, Y) pulls from one predictive block (row ky,
// column kx) with gradient plane gp: the bilinear weights of the block's taps
// that land on the pixel times the gradients of their pixels, phase-signed,
// added to acc.
template <class Get>
__device__ __forceinline__ float ad_block_pull(const LfGeom& g, Get get, int X, int Y, int ky, int kx, const AdRec& d,
                                               float acc)
{
    float blk_acc = 0.0f;
    const int bx0 = kx * g.bs, by0 = ky * g.bs;
    if (X > 0 && X < g.w - 1 && Y > 0 && Y < g.h - 1) {
        // away from the image border no tap is clamped: the tap (oy, ox)
        // landing on the pixel comes from source pixel (Y - iy - oy, X - ix - ox)
        // alone, when that pixel lies in the block
#pragma unroll
        for (int oy = 0; oy < 2; oy++) {
            const int ys = Y - d.iy - oy;
            const float wy = oy ? d.fy : 1.0f - d.fy;
#pragma unroll
            for (int ox = 0; ox < 2; ox++) {
                const int xs = X - d.ix - ox;
                if (ys >= by0 && ys < by0 + g.bs && xs >= bx0 && xs < bx0 + g.bs)
                    blk_acc = fmaf(wy * (ox ? d.fx : 1.0f - d.fx), get(ys, xs), blk_acc);
            }
        }
    } else {
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
                    for (int x = xlo; x <= xhi; x++) sum += get(y, x);
                blk_acc = fmaf(wxy, sum, blk_acc);
            }
        }
    }
    return acc + (d.sg > 0 ? blk_acc : -blk_acc);
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
#pragma unroll
        for (int t = 0; t < 5; t++) {
            const bool y = (unsigned)(ys + t - by) < (unsigned)g.bs;
            // both columns in one load: (xs - 1, xs), or (xs - 2, xs - 1) when
            // xs is past the block (a predictive plane is never the buffer's
            // first, so an element before it is still inside the buffer)
            const int at = y && (x0 || x1) ? first + t * g.w - (x0 ? 1 : 2) : 0;
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
            const float t = ad_block_pull(g, [&](int y, int x) { return gp[y * g.w + x]; }, X, Y0 + k, by >> g.bsl,
                                          bx >> g.bsl, q, 0.0f);
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
                                                      const float* __restrict__ maxshift, float* gres)
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
    const int reach = __builtin_amdgcn_readfirstlane((int)ceilf(fminf(maxshift[0], (float)(g.w + g.h))) + 2);
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
    // shifts too far for the sets of outside positions: a border pixel walks
    // the source pixels of every tap clamped onto it instead
    const bool far = reach > AD_FAR;
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
                const int ey = nk <= 1024 ? lf_small_div(es, nkx) : es / nkx;  // uniform choice
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
__global__ void __launch_bounds__(256) k_ad_shift(LfGeom g, LfPtrs p, AdPred pn, int groups,
                                                  const float* __restrict__ res, const float2* __restrict__ shift,
                                                  const float* __restrict__ gres_pred, float2* __restrict__ gshift,
                                                  int4* __restrict__ brec)
{
    constexpr int G = 1 << LG, U = LG == 6 ? AD_SHIFT_U : 1, PER = U * (256 / G);
    // the node, scalar
    const int cn = (int)blockIdx.x / groups;
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
    const int blk0 = ((int)blockIdx.x - cn * groups) * PER + sub * U;
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
    uint32_t *kin = (uint32_t*)(W + Bl.o_kin), *kout = (uint32_t*)(W + Bl.o_kout);
    uint32_t *vin = (uint32_t*)(W + Bl.o_vin), *vout = (uint32_t*)(W + Bl.o_vout);
    float* mxs = (float*)(W + Bl.o_max);
    float4* rayf = (float4*)(W + Bl.o_rayf);
    const int64_t rays = (int64_t)n_views * width * height;
    hipLaunchKernelGGL(k_ad_records, dim3((unsigned)((rays + 255) / 256)), dim3(256), 0, s, g, d_cams, n_views,
                       width, height, kin, vin, rayf);
    size_t sb = Bl.sort_bytes;
    if (hipcub::DeviceRadixSort::SortPairs(W + Bl.o_sort, sb, kin, kout, vin, vout, (int)Bl.n_recs, 0, Bl.end_bit, s) !=
        hipSuccess)
        return lf_fail(LF_EDEVICE, "radix sort failed");
    uint32_t* start = (uint32_t*)(W + Bl.o_start);
    hipLaunchKernelGGL(k_ad_nostart, dim3(4096), dim3(256), 0, s, start, Bl.n_samples);
    hipLaunchKernelGGL(k_ad_heads, dim3((unsigned)((Bl.n_recs + 255) / 256)), dim3(256), 0, s, kout, Bl.n_recs, start);
    // level-0 node planes of each channel, every sample written
    const int64_t plane = (int64_t)g.w * g.h, cstride = (int64_t)g.n_nodes * plane;
    float* g0 = d_grad_residual + (int64_t)g.node_base[0] * plane;
    hipLaunchKernelGGL(k_ad_samples, dim3((unsigned)((Bl.n_samples + 255) / 256)), dim3(256), 0, s, rayf, width, height,
                       d_grad_out, kout, vout, start, Bl.n_recs, Bl.n_samples, g.w, g.h, cstride, g0);
    for (int l = 1; l < g.H; l++)
        hipLaunchKernelGGL(k_ad_tree, dim3(8192), dim3(256), 0, s, g, l, d_grad_residual);
    float* parts = (float*)(W + Bl.o_parts);
    hipLaunchKernelGGL(k_ad_maxshift, dim3(AD_MAX_PARTS), dim3(256), 0, s, (const float2*)d_shift, h->L.n_rec, parts);
    hipLaunchKernelGGL(k_ad_maxparts, dim3(1), dim3(256), 0, s, parts, AD_MAX_PARTS, mxs);
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
        hipLaunchKernelGGL(kern, dim3((unsigned)(3 * pn.total * groups)), dim3(256), 0, s, g, h->p, pn, groups,
                           d_residual, (const float2*)d_shift, d_grad_residual, (float2*)d_grad_shift, brec);
    }
    const int64_t n_tiles = 3 * (int64_t)g.n_refs * ((g.w + AD_TILE - 1) / AD_TILE) * ((g.h + AD_TILE - 1) / AD_TILE);
    if (h->L.n_rec > 0)  // without predictive blocks the references keep their own gradients
        hipLaunchKernelGGL(k_ad_reference, dim3((unsigned)((n_tiles + 31) / 32 * 8)), dim3(256), 0, s, g,
                           (const int4*)brec, mxs, d_grad_residual);
    return lf_check_launch("render_backward");
}
