// Novel-view rendering fused with random-access decoding.
//
// Two kernels compute the same image bit for bit:
//  - k_render_rays: one thread per ray; each ray walks the tree paths of its
//    16 neighbouring samples (the simple reference path, and the fallback for
//    footprints beyond the staging budget);
//  - k_render_batch: a workgroup renders one screen tile for a group of
//    consecutive views.  It decodes the union footprint of those views once:
//    per-block descriptors (table entry, motion vector, reference plane) are
//    staged in LDS, every tree node above the leaf views that the footprint
//    reaches is decoded once per pixel (ancestor deduplication), and each
//    (view, pixel) sample is assembled once as RGBA8 in LDS.  The rays then
//    blend from LDS.
// Blending works on unscaled 8-bit values and scales by 1/255 at the end.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "lf_render_tile.h"

template <int RES>
__global__ void __launch_bounds__(256) k_render_rays(LfGeom g, LfPtrs p, const float* __restrict__ cams, int nv,
                                                     int wo, int ho, float* __restrict__ out, int lod)
{
    const int64_t npix = (int64_t)wo * ho;
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= npix * nv) return;
    const int v = (int)(r / npix);
    const int64_t px = r - (int64_t)v * npix;
    const int j = (int)(px / wo), i = (int)(px % wo);
    float o[3];
    lf_render_one<RES>(g, p, cams + 18 * v, i, j, o, lod);
#pragma unroll
    for (int c = 0; c < 3; c++) out[((int64_t)v * 3 + c) * npix + px] = o[c];
}

// 4:2:0 streams, one thread per ray (lf_render_one420).
__global__ void __launch_bounds__(256) k_render_rays420(LfGeom g, LfPtrs p, LfGeom gc, LfPtrs pc,
                                                        const float* __restrict__ cams, int nv, int wo, int ho,
                                                        float* __restrict__ out, int lod)
{
    const int64_t npix = (int64_t)wo * ho;
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= npix * nv) return;
    const int v = (int)(r / npix);
    const int64_t px = r - (int64_t)v * npix;
    const int j = (int)(px / wo), i = (int)(px % wo);
    float o[3];
    lf_render_one420(g, p, gc, pc, cams + 18 * v, i, j, o, lod);
#pragma unroll
    for (int c = 0; c < 3; c++) out[((int64_t)v * 3 + c) * npix + px] = o[c];
}

lf_status lf_launch_render_rays(const lf_handle* h, const float* d_cams, int nv, int wo, int ho, float* d_out,
                                hipStream_t s, int lod = 0)
{
    int64_t total = (int64_t)nv * wo * ho;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFF) return lf_fail(LF_EINVAL, "too many rays");
    if (h->L.chroma420)
        hipLaunchKernelGGL(k_render_rays420, dim3((unsigned)blocks), dim3(256), 0, s, h->L.g, h->p, h->L.gc, h->pc,
                           d_cams, nv, wo, ho, d_out, lod);
    else
        hipLaunchKernelGGL(h->L.sparse == LF_RES_CSR     ? k_render_rays<LF_RES_CSR>
                           : h->L.sparse == LF_RES_TILES ? k_render_rays<LF_RES_TILES>
                                                         : k_render_rays<LF_RES_DENSE>,
                           dim3((unsigned)blocks), dim3(256), 0, s, h->L.g, h->p, d_cams, nv, wo, ho, d_out, lod);
    return lf_check_launch("render_rays");
}

// C420: a 4:2:0 stream, chroma geometry gc, pc (unused otherwise).  LOD: the
// samples of a coarser tree level, g and gc cut off below it (grid unused
// otherwise).
template <bool SMALL_BLOCKS, bool C420, bool LOD, int RES, bool DIRECT = false>
__global__ void __launch_bounds__(NT, 3) k_render_batch(LfGeom g, LfPtrs p, LfGeom gc, LfPtrs pc,
                                                     const float* __restrict__ cams, int nv, int wo, int ho,
                                                     int tiles_x, int tiles_y, int chunk, int fpg, int64_t n_full,
                                                     int split, float* __restrict__ out, LodGrid grid)
{
    // A workgroup renders one screen tile for a chunk of consecutive views
    // (groups of fpg views, decoded values cached between the groups).
    // XCD-aware order: workgroup ids go round-robin over the 8 XCDs, so give
    // each XCD a contiguous range of (view chunk, tile) work: consecutive
    // views and neighbouring tiles share stream data in that XCD's L2.
    // The first n_full (chunk, tile) items go to one workgroup each; the
    // items after them, which would only part-fill the last round of
    // resident workgroups, are cut into `split` runs of views each.
    const int n_chunks = (nv + chunk - 1) / chunk;
    const int64_t n_work = (int64_t)tiles_x * tiles_y * n_chunks;
    const int64_t ga = (n_full + 7) / 8 * 8;  // workgroups of the whole items
    int64_t work;
    int part = 0;
    if ((int64_t)blockIdx.x < ga) {
        const int64_t per_xcd = ga / 8;
        work = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
        if (work >= n_full) return;  // uniform per workgroup
    } else {
        const int64_t b = blockIdx.x - ga, n_parts = (n_work - n_full) * split;
        const int64_t per_xcd = (n_parts + 7) / 8;
        const int64_t it = (b & 7) * per_xcd + (b >> 3);
        if (it >= n_parts) return;
        work = n_full + it / split;
        part = (int)(it % split);
    }
    TILE_LDS_DECL
    const int vc = (int)(work / ((int64_t)tiles_x * tiles_y));
    const int tt = (int)(work - (int64_t)vc * tiles_x * tiles_y);
    const int tyi = tt / tiles_x, txi = tt - tyi * tiles_x;
    const int c0 = vc * chunk, c1 = min(nv, c0 + chunk);
    int v0 = c0, nf = c1 - c0;
    if (work >= n_full) {
        const int per = (nf + split - 1) / split;
        v0 = c0 + part * per;
        nf = min(per, c1 - v0);
        if (nf <= 0) return;
    }
    lf_tile_views<false, SMALL_BLOCKS, C420, LOD, RES, DIRECT>(g, p, gc, pc, cams, v0, nf, fpg, wo, ho, txi, tyi, out, S, grid);
}

// Per-ray rendering of the (view, tile) pairs the batched kernel marked.
// Workgroup b checks pairs b, b + G, b + 2 G, ... of a grid of G, up to 3 NT of
// them at once (one per thread), compacts the marked ones and renders them one
// tile at a time.  G is a prime near the number of CUs (one workgroup is
// resident on each), so that marked rows, columns or views of tiles spread
// over all of them, and a launch that marks nothing costs few waves.  A ray is
// three threads in different waves, one per channel of its 16 samples: the
// chain of dependent loads of a channel bounds the pass, and marked tiles are
// often too few to fill the chip.  The channels meet in LDS and each thread
// blends one colour.  3 views of 157x750, far minified, 16x16 blocks: 558 ->
// 437 us for the call; 11 of 253x1032 2.37 -> 0.38 ms; 2 of 80x144 in 4:2:0
// 0.92 -> 0.44 ms (one thread a ray, a contiguous range a workgroup before).
// Calls of small blocks that mark most of some thousand tiles are up to a
// fifth slower than with one thread a ray in tile order: 37 views of 340x202
// on a path over 17x17 of 512x512 in 8x8 blocks 2.05 -> 2.34 ms, 65 of 137x139
// over 15x12 of 120x360 in 4x4 1.26 -> 1.51 (10 unrelated ones of 340x202 0.45
// -> 0.25).  Neighbouring tiles no longer run side by side.  Not better: a
// range of tiles per 251 workgroups (the first 2.08 to 2.25, the last 0.30 to
// 0.35 or 8 us more for every call), contiguous runs per XCD (2.19, others
// 1.3 times slower), one thread a ray where a workgroup holds three marked
// tiles (2.47).
template <bool C420, int RES>
__global__ void __launch_bounds__(3 * NT) k_render_fallback(LfGeom g, LfPtrs p, LfGeom gc, LfPtrs pc,
                                                            const float* __restrict__ cams, int nv, int wo, int ho,
                                                            int tiles_x, int tiles_y, float* __restrict__ out,
                                                            int lod)
{
    __shared__ int marked[3 * NT];
    __shared__ int wcount[3 * NT / 64];
    __shared__ int sample[3][16][NT];
    const int64_t n_pairs = (int64_t)nv * tiles_x * tiles_y;
    const int64_t npix = (int64_t)wo * ho;
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int c = wid / (NT / 64), t = (int)threadIdx.x - c * NT;
    for (int64_t base = blockIdx.x; base < n_pairs; base += (int64_t)3 * NT * gridDim.x) {
        const int64_t pr = base + (int64_t)threadIdx.x * gridDim.x;
        int mine = 0;
        if (pr < n_pairs) {
            const int v = (int)(pr / ((int64_t)tiles_x * tiles_y));
            const int tt = (int)(pr - (int64_t)v * tiles_x * tiles_y);
            const int tyi = tt / tiles_x, txi = tt - tyi * tiles_x;
            mine = __float_as_uint(out[(int64_t)v * 3 * npix + (int64_t)(tyi * TH) * wo + txi * TW]) == FALLBACK_MARK;
        }
        // compact the marked pairs in thread order
        const uint64_t bal = __ballot(mine);
        if (lane == 0) wcount[wid] = __popcll(bal);
        __syncthreads();
        int off = 0, total = 0;
        for (int w = 0; w < 3 * NT / 64; w++) {
            off += w < wid ? wcount[w] : 0;
            total += wcount[w];
        }
        if (mine) marked[off + __popcll(bal & ((1ull << lane) - 1ull))] = (int)threadIdx.x;
        __syncthreads();
        for (int k = 0; k < total; k++) {
            const int64_t q = base + (int64_t)marked[k] * gridDim.x;
            const int v = (int)(q / ((int64_t)tiles_x * tiles_y));
            const int tt = (int)(q - (int64_t)v * tiles_x * tiles_y);
            const int tyi = tt / tiles_x, txi = tt - tyi * tiles_x;
            const int i = txi * TW + t % TW, j = tyi * TH + t / TW;
            const bool in = i < wo && j < ho;
            Ray r;
            if (in) {
                r = lf_ray_setup(g, cams + 18 * v, i, j);
                if (C420) {
#pragma unroll 1
                    for (int m = 0; m < 16; m++) {
                        const int b = (m & 8) ? r.b1 : r.b0, a = (m & 4) ? r.a1 : r.a0;
                        const int y = (m & 2) ? r.y1 : r.y0, x = (m & 1) ? r.x1 : r.x0;
                        sample[c][m][t] = c == 0 ? lf_decode_channel(g, p, 0, b, a, y, x, lod)
                                                 : lf_chroma_up(gc, pc, c - 1, b, a, y, x, lod);
                    }
                } else {
                    int acc[16];
                    lf_ray_channel<RES>(g, p, r, c, lod, acc);
#pragma unroll
                    for (int m = 0; m < 16; m++) sample[c][m][t] = acc[m];
                }
            }
            __syncthreads();
            if (in) {
                const BlendW w = lf_blend_weights(r);
                float sm[16];
#pragma unroll
                for (int m = 0; m < 16; m++) {
                    int rgb[3];
                    lf_ycocg_to_rgb(sample[0][m][t], sample[1][m][t], sample[2][m][t], rgb[0], rgb[1], rgb[2]);
                    sm[m] = (float)(c == 0 ? rgb[0] : (c == 1 ? rgb[1] : rgb[2]));
                }
                out[((int64_t)v * 3 + c) * npix + (int64_t)j * wo + i] = lf_blend16(sm, w);
            }
            __syncthreads();  // the next tile rewrites the samples; marked[] and wcount[] are rewritten by the next round
        }
        __syncthreads();
    }
}

static int env_int(const char* name, int dflt, int lo, int hi)
{
    const char* e = getenv(name);
    int v = e ? atoi(e) : dflt;
    return v < lo ? lo : (v > hi ? hi : v);
}

// views per group (decoded together) and per chunk (one workgroup, values
// cached between its groups)
static int frames_per_group()
{
    static int v = env_int("HMLFC_VIEWS_PER_GROUP", 12, 1, FMAX);
    return v;
}
// views per chunk: HMLFC_VIEWS_PER_CHUNK if set, else chunks as long as
// possible while the launch still has about 2048 workgroups (balanced, at
// most FMAX views each)
static int frames_per_chunk(int nv, int tiles)
{
    static int v = env_int("HMLFC_VIEWS_PER_CHUNK", 0, 0, FMAX);
    if (v > 0) return v;
    int64_t n_chunks = std::min<int64_t>(nv, std::max<int64_t>(1, (2048 + tiles - 1) / std::max(tiles, 1)));
    n_chunks = std::max<int64_t>(n_chunks, (nv + FMAX - 1) / FMAX);
    return (int)((nv + n_chunks - 1) / n_chunks);
}

// runs each tail item of the batched launch is cut into
static int tail_split()
{
    static int v = env_int("HMLFC_TAIL_SPLIT", 2, 1, 8);
    return v;
}

// compute units of the current device (cached per device id)
static int device_cus()
{
    static int cus[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        cus[dev] = n;
    }
    return cus[dev];
}

extern "C" lf_status lf_get_render_config(int32_t n_views, int32_t width, int32_t height, int32_t* views_per_group,
                                          int32_t* views_per_chunk)
{
    if (n_views < 1 || width < 1 || height < 1) return lf_fail(LF_EINVAL, "bad argument");
    const int tiles = ((width + TW - 1) / TW) * ((height + TH - 1) / TH);
    if (views_per_group) *views_per_group = frames_per_group();
    if (views_per_chunk) *views_per_chunk = frames_per_chunk(n_views, tiles);
    return LF_OK;
}

// The geometry of tree levels lod .. H: level lod's nodes as the leaf views.
// Node, reference and motion indices keep their places in the stream.
static LfGeom lf_cut_geometry(const LfGeom& g, int lod)
{
    LfGeom c = g;
    c.H = g.H - lod;
    c.na = g.na_l[lod];
    c.nb = g.nb_l[lod];
    for (int l = 0; l <= c.H; l++) {
        c.na_l[l] = g.na_l[l + lod];
        c.nb_l[l] = g.nb_l[l + lod];
    }
    for (int l = 0; l < c.H; l++) {
        c.node_base[l] = g.node_base[l + lod];
        c.ref_base[l] = g.ref_base[l + lod];
        c.step[l] = g.step[l + lod];
        c.bias[l] = g.bias[l + lod];
        for (int ch = 0; ch < 3; ch++) {
            c.mv_word[ch][l] = g.mv_word[ch][l + lod];
            c.sig_word[ch][l] = g.sig_word[ch][l + lod];
            c.mv_mode[ch][l] = g.mv_mode[ch][l + lod];
            c.rec_base[ch][l] = g.rec_base[ch][l + lod];
        }
    }
    return c;
}

// lod: tree level the samples come from, 0 .. H - 1
lf_status lf_launch_render_batch(const lf_handle* h, const float* d_cams, int nv, int wo, int ho, float* d_out,
                                 hipStream_t s, int lod = 0)
{
    const int tx = (wo + TW - 1) / TW, ty = (ho + TH - 1) / TH;
    const int fpg = frames_per_group(), chunk = frames_per_chunk(nv, tx * ty);
    const int64_t n_work = (int64_t)tx * ty * ((nv + chunk - 1) / chunk);
    // Split the items past the last whole round of resident workgroups
    // (3 per CU) into runs of views, so the tail of the launch is spread
    // over more CUs; chunks too short to split keep one workgroup each.
    const int split = tail_split();
    const int64_t slots = 3 * (int64_t)device_cus();
    int64_t n_full = n_work;
    if (split > 1 && chunk >= 2 * split && n_work > slots && n_work % slots) n_full = n_work - n_work % slots;
    const int sp = n_full < n_work ? split : 1;
    const int64_t grid = (n_full + 7) / 8 * 8 + ((n_work - n_full) * sp + 7) / 8 * 8;
    if (grid > 0x7FFFFFFF) return lf_fail(LF_EINVAL, "too many tiles");
    const bool small = h->L.g.bs < 16, c420 = h->L.chroma420 != 0;
    const size_t lds = small ? LDS_DYN_BYTES_SB : LDS_DYN_BYTES;
    using BatchKernel = void (*)(LfGeom, LfPtrs, LfGeom, LfPtrs, const float*, int, int, int, int, int, int, int,
                                 int64_t, int, float*, LodGrid);
    const bool cut = lod > 0, tiles = h->L.sparse == LF_RES_TILES;
    // [small blocks][dense, coarser level, 4:2:0, 4:2:0 coarser level, block-sparse of any level, coarser level and
    // block-sparse coarser level of at most four views a chunk]
    constexpr int D = LF_RES_DENSE, T = LF_RES_TILES;
    static const BatchKernel kernels[2][7] = {
        {k_render_batch<false, false, false, D>, k_render_batch<false, false, true, D>, k_render_batch<false, true, false, D>,
         k_render_batch<false, true, true, D>, k_render_batch<false, false, true, T>,
         k_render_batch<false, false, true, D, true>, k_render_batch<false, false, true, T, true>},
        {k_render_batch<true, false, false, D>, k_render_batch<true, false, true, D>, k_render_batch<true, true, false, D>,
         k_render_batch<true, true, true, D>, k_render_batch<true, false, true, T>,
         k_render_batch<true, false, true, D, true>, k_render_batch<true, false, true, T, true>}};
    int kind = tiles ? 4 : 2 * c420 + cut;
    if (cut && !c420 && chunk <= 4) kind = tiles ? 6 : 5;
    const BatchKernel kern = kernels[small][kind];
    static bool attr_set[2][7] = {};
    if (lds > 65536 && !attr_set[small][kind]) {
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return lf_fail(LF_EDEVICE, "cannot reserve %zu bytes of LDS", lds);
        attr_set[small][kind] = true;
    }
    // a 4:4:4 stream passes its own geometry as the (unused) chroma geometry
    const LfGeom& gc = c420 ? h->L.gc : h->L.g;
    const LfPtrs& pc = c420 ? h->pc : h->p;
    const LfGeom gl = cut ? lf_cut_geometry(h->L.g, lod) : h->L.g, gcl = cut && c420 ? lf_cut_geometry(gc, lod) : gc;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NT), lds, s, gl, h->p, gcl, pc, d_cams, nv, wo, ho, tx, ty,
                       chunk, fpg, n_full, sp, d_out, LodGrid{h->L.g.na, h->L.g.nb, lod});
    // G of the per-ray pass: 256 workgroups more that find nothing cost 1.3 us,
    // so one on each CU does where few tiles are marked (16x16 blocks: one
    // 512x512 view 44.6 us, 46.0 with 509).  Smaller blocks mark more tiles,
    // whose costs differ: two views of 74x928, all marked, 131 us with 509, 200
    // with 251; 32 of 211x117 711 with 1021, 838 with 509.
    const int64_t pairs = (int64_t)tx * ty * nv;
    const int most = h->L.g.bs >= 16 ? 251 : (pairs <= 2048 ? 509 : 1021);
    const auto rest = c420 ? k_render_fallback<true, D> : (tiles ? k_render_fallback<false, T> : k_render_fallback<false, D>);
    hipLaunchKernelGGL(rest, dim3((unsigned)std::min<int64_t>(pairs, most)), dim3(3 * NT), 0, s, h->L.g, h->p, gc, pc,
                       d_cams, nv, wo, ho, tx, ty, d_out, lod);
    return lf_check_launch("render_batch");
}

// Whether the tile renderer takes a render from tree level `level`: it
// decodes quads of 4 pixels inside one block, on packed 16-bit lanes.  Dense
// handles: the load refuses leaf samples beyond the lanes' range, and settles
// the coarser levels' at once or not at all.  4:2:0 and block-sparse handles:
// taken when the load has settled the range of every level and of the motion
// vectors (nothing is refused there), or of a 4:2:0 handle's leaf views.  The root
// level is sixteen plain reads per ray: no tiles.  CSR handles search a row
// per tap: no tiles.  Nor do renders from the level below the root where its
// nodes are a single row or column, or, from level 2 on, where a workgroup
// would take fewer than five views: a ray's four views are often one node
// there, and where that is a reference a ray is a few reads, which the stages
// only beat shared among views.  Over 1x2 nodes two views of 986x429 44 us per
// ray and 84 through the tiles, 25 of 271x211 77 and 117; over 1x1 19 and 42.
// Over 8x8 nodes, 4x4 blocks, two of 986x429 from one point each 53 and 83
// (over 4x4 123 and 84), 16 of 512x512 on a path, eight a workgroup, 477 and
// 104 (over 2x2 to 8x8 nodes 306..523 and 73..105).  4:2:0 chroma is dearer
// per ray (342 us against 39).
static bool lf_tiles_apply(const lf_handle* h, int level, int nv, int wo, int ho)
{
    const LfLayout& L = h->L;
    if (L.g.bs < 4 || level >= L.g.H || L.sparse == LF_RES_CSR) return false;
    if (level > 0 && level + 1 == L.g.H && !L.chroma420) {
        if (L.g.na_l[level] == 1 || L.g.nb_l[level] == 1) return false;
        const int tiles = ((wo + TW - 1) / TW) * ((ho + TH - 1) / TH);
        if (level > 1 && std::min(frames_per_chunk(nv, tiles), nv) < 5) return false;
    }
    if (L.sparse || L.chroma420) return L.packed_levels || (level == 0 && L.packed_leaves);
    return level == 0 || L.packed_levels;
}

extern "C" lf_status lf_render_views(const lf_handle* h, const float* d_cams, int32_t n_views, int32_t width,
                                     int32_t height, float* d_out, void* stream)
{
    if (!h || n_views < 0 || width < 1 || height < 1) return lf_fail(LF_EINVAL, "bad argument");
    if (n_views == 0) return LF_OK;
    if (!d_cams || !d_out) return lf_fail(LF_EINVAL, "null buffer");
    if (lf_tiles_apply(h, 0, n_views, width, height)) return lf_launch_render_batch(h, d_cams, n_views, width, height, d_out, (hipStream_t)stream);
    return lf_launch_render_rays(h, d_cams, n_views, width, height, d_out, (hipStream_t)stream);
}

extern "C" lf_status lf_render_views_per_ray(const lf_handle* h, const float* d_cams, int32_t n_views, int32_t width,
                                             int32_t height, float* d_out, void* stream)
{
    if (!h || n_views < 0 || width < 1 || height < 1) return lf_fail(LF_EINVAL, "bad argument");
    if (n_views == 0) return LF_OK;
    if (!d_cams || !d_out) return lf_fail(LF_EINVAL, "null buffer");
    return lf_launch_render_rays(h, d_cams, n_views, width, height, d_out, (hipStream_t)stream);
}

extern "C" lf_status lf_render_views_lod(const lf_handle* h, int32_t level, const float* d_cams, int32_t n_views,
                                         int32_t width, int32_t height, float* d_out, void* stream)
{
    if (!h || n_views < 0 || width < 1 || height < 1 || level < 0 || level > h->L.g.H)
        return lf_fail(LF_EINVAL, "bad argument");
    if (n_views == 0) return LF_OK;
    if (!d_cams || !d_out) return lf_fail(LF_EINVAL, "null buffer");
    // 16 views of 512x512 at level 2 of 17x17x512x512: 0.098 ms through the
    // tiles, 1.09 ms one thread per ray
    if (lf_tiles_apply(h, level, n_views, width, height))
        return lf_launch_render_batch(h, d_cams, n_views, width, height, d_out, (hipStream_t)stream, level);
    return lf_launch_render_rays(h, d_cams, n_views, width, height, d_out, (hipStream_t)stream, level);
}
