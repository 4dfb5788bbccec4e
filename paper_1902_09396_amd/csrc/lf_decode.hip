// Random-access decoding of samples from dense handles (Decoding Procedure;
// Random Access for Interactive Rendering).
//
// A sample is the root plus one SRV per level, three channels: at four levels
// twelve block descriptors, payload windows and pairs of tap rows, each on a
// cache line of its own when requests are scattered.  Requests of many
// scattered samples are first ordered by the pixel block they fall in
// (counting sort in caller scratch), so that the samples of a block, whatever
// their view, meet the same lines in L2.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lf_internal.h"

#define DEC_KEYS 1024       // pixel blocks the requests are ordered by, at most
#define DEC_CHUNK 4096      // requests per workgroup of the ordering passes
#define DEC_L 2             // levels read together (more cost registers that hold waves: 66 us against 59 for 2^20 consecutive samples at 4)
#define DEC_T 1024          // threads of it
#define DEC_MAX (1 << 26)   // most requests ordered in one call (1 GiB of scratch)
#define DEC_SMALL 163840    // fewest unordered requests of a small field that keep the one-thread walk

// Words 2 e, 2 e + 1 of int16 elements from an even element on: 4-byte aligned.
typedef uint32_t lf_w2 __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t lf_w3 __attribute__((ext_vector_type(3), aligned(4)));

// Value i of a block from the three payload words of its group (bit o on);
// groups of at most 64 bits, else from the payload itself.  The digit of a
// group header is header / radix^k % radix, by multiplications that are exact
// for 8-bit (7-bit) headers.
__device__ __forceinline__ int dec_value(const uint32_t* __restrict__ block, uint32_t mode, uint32_t i, const lf_w3& w)
{
    const uint32_t fam = mode >> 5, b = mode & 31u;
    const uint32_t hb = fam == 0u ? 0u : (fam == 1u ? 8u : 7u);
    const uint32_t gs = fam == 0u ? 1u : (fam == 1u ? 5u : 3u);
    const uint32_t grp = fam == 0u ? i : __umulhi(i, fam == 1u ? 858993460u : 1431655766u);
    const uint32_t k = i - __umul24(grp, gs), gl = hb + gs * b;
    if (gl > 64u) return (int)lf_bise_get(block, (int)mode, i);
    const uint32_t o = __umul24(grp, gl) & 31u;
    const uint64_t X = ((uint64_t)__builtin_amdgcn_alignbit(w.z, w.y, o) << 32) | __builtin_amdgcn_alignbit(w.y, w.x, o);
    const uint32_t lo = (uint32_t)(X >> ((hb + __umul24(k, b)) & 63u)) & ((1u << b) - 1u);
    if (fam == 0u) return (int)lo;
    const uint32_t head = (uint32_t)X & ((1u << hb) - 1u);
    const uint32_t m3 = k == 0u ? 65536u : (k == 1u ? 21846u : (k == 2u ? 7282u : (k == 3u ? 2428u : 810u)));
    const uint32_t m5 = k == 0u ? 65536u : (k == 1u ? 13108u : 2622u);
    const uint32_t q = (head * (fam == 1u ? m3 : m5)) >> 16;
    const uint32_t digit = fam == 1u ? q - 3u * ((q * 21846u) >> 16) : q - 5u * ((q * 13108u) >> 16);
    return (int)((digit << b) | lo);
}

// First payload word of value i's group.
__device__ __forceinline__ uint32_t dec_word(uint32_t mode, uint32_t i)
{
    const uint32_t fam = mode >> 5, b = mode & 31u;
    const uint32_t grp = fam == 0u ? i : __umulhi(i, fam == 1u ? 858993460u : 1431655766u);
    return __umul24(grp, fam == 0u ? b : (fam == 1u ? 8u + 5u * b : 7u + 3u * b)) >> 5;
}

// One channel of the level-lod sample (B << lod, A << lod, y, x): the
// descriptors of DEC_L levels are read together, then their payload windows
// and tap rows together.  The same integers as lf_decode_channel.
__device__ __forceinline__ int dec_channel(const LfGeom& g, const LfPtrs& p, int c, int b, int a, int y, int x, int lod)
{
    const size_t plane = (size_t)g.w * g.h;
    int v = p.root[((size_t)(c * g.root_nb + (b >> g.H)) * g.root_na + (a >> g.H)) * plane + (size_t)(y * g.w + x)];
    const int blk = (y >> g.bsl) * g.nbx + (x >> g.bsl);
    const uint32_t i = (uint32_t)(((y & (g.bs - 1)) << g.bsl) | (x & (g.bs - 1)));
    const uint4* desc = p.desc + (size_t)c * g.n_nodes * g.nblk + blk;
    for (int l0 = lod; l0 < g.H; l0 += DEC_L) {
        uint4 d[DEC_L];
        lf_w3 w[DEC_L];
        lf_w2 ta[DEC_L], tb[DEC_L];
        uint32_t par[DEC_L];  // bits: odd start of rows a and b, column b beyond column a
#pragma unroll
        for (int q = 0; q < DEC_L; q++) {
            const int l = min(l0 + q, g.H - 1);  // past the top: the top level again, not added
            d[q] = desc[(size_t)(g.node_base[l] + (b >> l) * g.na_l[l] + (a >> l)) * g.nblk];
        }
#pragma unroll
        for (int q = 0; q < DEC_L; q++) {
            const uint32_t mode = d[q].z >> 24;
            const bool ref = mode == MODE_PLANE;
            w[q] = *reinterpret_cast<const lf_w3*>(p.payload + d[q].x + (ref ? 0u : dec_word(mode, i)));
            // a reference node's descriptor has a zero vector and no fraction:
            // its first tap is the sample
            const int X = 4 * x + (((int)(d[q].z << 20)) >> 20), Y = 4 * y + (((int)(d[q].z << 8)) >> 20);
            const int xa = lf_clampi(X >> 2, 0, g.w - 1), xb = lf_clampi((X >> 2) + 1, 0, g.w - 1);
            const int ya = lf_clampi(Y >> 2, 0, g.h - 1), yb = ref ? ya : lf_clampi((Y >> 2) + 1, 0, g.h - 1);
            const uint32_t ea = d[q].w + (uint32_t)(ya * g.w + xa), eb = d[q].w + (uint32_t)(yb * g.w + xa);
            ta[q] = *reinterpret_cast<const lf_w2*>(reinterpret_cast<const uint32_t*>(p.refs) + (ea >> 1));
            tb[q] = *reinterpret_cast<const lf_w2*>(reinterpret_cast<const uint32_t*>(p.refs) + (eb >> 1));
            par[q] = (ea & 1u) | ((eb & 1u) << 1) | (xb > xa ? 4u : 0u);
        }
#pragma unroll
        for (int q = 0; q < DEC_L; q++) {
            const uint32_t mode = d[q].z >> 24;
            const uint32_t ra = __builtin_amdgcn_alignbit(ta[q].y, ta[q].x, (par[q] & 1u) << 4);
            const uint32_t rb = __builtin_amdgcn_alignbit(tb[q].y, tb[q].x, (par[q] & 2u) << 3);
            const int t00 = (int)(int16_t)ra, t10 = (int)(int16_t)rb;
            int s = t00;
            if (mode != MODE_PLANE) {
                const int t01 = (par[q] & 4u) ? (int)ra >> 16 : t00, t11 = (par[q] & 4u) ? (int)rb >> 16 : t10;
                const int fx = (4 * x + (((int)(d[q].z << 20)) >> 20)) & 3, fy = (4 * y + (((int)(d[q].z << 8)) >> 20)) & 3;
                const int acc = (4 - fy) * ((4 - fx) * t00 + fx * t01) + fy * ((4 - fx) * t10 + fx * t11);
                const uint32_t code = d[q].y >> 29;
                const int pred = (acc + 8) >> 4;
                s = ((int)(int16_t)(d[q].y & 0xFFFFu) + dec_value(p.payload + d[q].x, mode, i, w[q])) *
                    (int)((d[q].y >> 16) & 0x1FFFu);
                s += code == 0u ? pred : (code == 1u ? -pred : 0);
            }
            if (l0 + q < g.H) v += s;
        }
    }
    return v;
}

// A request clamped to the level's grid: (B, A, y, x), and whether it was clamped.
__device__ __forceinline__ int4 dec_request(const LfGeom& g, int lod, int4 q, bool& clamped)
{
    const int4 r = make_int4(lf_clampi(q.x, 0, g.nb_l[lod] - 1), lf_clampi(q.y, 0, g.na_l[lod] - 1),
                             lf_clampi(q.z, 0, g.h - 1), lf_clampi(q.w, 0, g.w - 1));
    clamped = r.x != q.x || r.y != q.y || r.z != q.z || r.w != q.w;
    return r;
}

struct DecOrder {
    uint32_t* hist;   // [wgs][DEC_KEYS], then the counts of each key in the workgroups before
    uint32_t* total;  // [DEC_KEYS], then changes[wgs], then the flag "scattered"
    uint4* rec;       // [n] (request, B | A << 16, y | x << 16, 0) in order
    int wgs, shift, kx;
};

// Samples: one wave64 per channel of 64 samples, the channels meeting in LDS.
// ORDERED: in the order of o.rec if the requests were found scattered.
template <bool ORDERED>
__global__ void __launch_bounds__(192) k_decode_dense(LfGeom g, LfPtrs p, int lod, const int4* __restrict__ coords, int64_t n,
                                                      uint8_t* __restrict__ rgb, unsigned long long* __restrict__ clamps,
                                                      DecOrder o)
{
    __shared__ int vals[3][64];
    const int lane = threadIdx.x & 63, c = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool ordered = ORDERED && o.total[DEC_KEYS + o.wgs] != 0;
    // one run of 64 requests a workgroup; ordered: each XCD takes a contiguous
    // range of them, whose lines stay in its L2 (the launch has a multiple of 8
    // workgroups, at least one a run, and the last of a range may be past the end)
    const int64_t run = ordered ? (blockIdx.x & 7) * (int64_t)(gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    const int64_t k = run * 64 + lane;
    const bool in = k < n;
    int64_t at = k;
    if (in) {
        int4 r;
        if (ordered) {
            const uint4 q = o.rec[k];
            at = q.x;
            r = make_int4((int)(q.y & 0xFFFFu), (int)(q.y >> 16), (int)(q.z & 0xFFFFu), (int)(q.z >> 16));
        } else {
            bool clamped;
            r = dec_request(g, lod, coords[k], clamped);
            // counted by the ordering's first pass when there is one
            if (!ORDERED && c == 0) {
                const unsigned long long m = __ballot(clamped);
                if (m && lane == __ffsll((long long)m) - 1) atomicAdd(clamps, (unsigned long long)__popcll(m));
            }
        }
        vals[c][lane] = dec_channel(g, p, c, r.x << lod, r.y << lod, r.z, r.w, lod);
    }
    __syncthreads();
    if (c == 0 && in) {
        int R, G, B;
        lf_ycocg_to_rgb(vals[0][lane], vals[1][lane], vals[2][lane], R, G, B);
        rgb[3 * at] = (uint8_t)R;
        rgb[3 * at + 1] = (uint8_t)G;
        rgb[3 * at + 2] = (uint8_t)B;
    }
}

// ---- ordering: requests counted by pixel block, prefix sums, placed ----

__device__ __forceinline__ int dec_key(const DecOrder& o, const int4& r) { return (r.z >> o.shift) * o.kx + (r.w >> o.shift); }

__global__ void __launch_bounds__(DEC_T) k_dec_count(LfGeom g, int lod, const int4* __restrict__ coords, int64_t n,
                                                     unsigned long long* __restrict__ clamps, DecOrder o)
{
    __shared__ uint32_t h[DEC_KEYS];
    __shared__ uint32_t changes;
    for (int i = threadIdx.x; i < DEC_KEYS; i += DEC_T) h[i] = 0;
    if (threadIdx.x == 0) changes = 0;
    __syncthreads();
    for (int u = 0; u < DEC_CHUNK / DEC_T; u++) {
        const int64_t k = (int64_t)blockIdx.x * DEC_CHUNK + u * DEC_T + threadIdx.x;
        bool clamped = false;
        int key = -1;
        if (k < n) {
            key = dec_key(o, dec_request(g, lod, coords[k], clamped));
            atomicAdd(&h[key], 1u);
        }
        const int left = __shfl_up(key, 1, 64);
        const unsigned long long mc = __ballot(clamped), md = __ballot(key != left && (threadIdx.x & 63) != 0);
        if ((threadIdx.x & 63) == 0) {
            if (mc) atomicAdd(clamps, (unsigned long long)__popcll(mc));
            if (md) atomicAdd(&changes, (uint32_t)__popcll(md));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < DEC_KEYS; i += DEC_T) o.hist[(int64_t)blockIdx.x * DEC_KEYS + i] = h[i];
    if (threadIdx.x == 0) o.total[DEC_KEYS + blockIdx.x] = changes;
}

// 64 keys per workgroup: each key's counts become the counts in the
// workgroups before; 16 waves take a range of workgroups each.  Requests whose
// neighbours mostly share a block are left in their order.
__global__ void __launch_bounds__(1024) k_dec_prefix(int64_t n, DecOrder o)
{
    __shared__ uint32_t part[16][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, key = blockIdx.x * 64 + lane;
    const int per = (o.wgs + 15) / 16, w0 = min(wv * per, o.wgs), w1 = min(w0 + per, o.wgs);
    uint32_t sum = 0;
    for (int w = w0; w < w1; w++) sum += o.hist[(int64_t)w * DEC_KEYS + key];
    part[wv][lane] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (int q = 0; q < wv; q++) run += part[q][lane];
    for (int w = w0; w < w1; w++) {
        const uint32_t c = o.hist[(int64_t)w * DEC_KEYS + key];
        o.hist[(int64_t)w * DEC_KEYS + key] = run;
        run += c;
    }
    if (wv == 15) o.total[key] = run;
    if (blockIdx.x == 0) {
        uint32_t ch = 0;
        for (int w = threadIdx.x; w < o.wgs; w += 1024) ch += o.total[DEC_KEYS + w];
        __syncthreads();
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) ch += (uint32_t)__shfl_xor((int)ch, s, 64);
        if (lane == 0) part[0][wv] = ch;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint64_t all = 0;
            for (int q = 0; q < 16; q++) all += part[0][q];
            o.total[DEC_KEYS + o.wgs] = (int64_t)all * 4 > n;
        }
    }
}

__global__ void __launch_bounds__(DEC_T) k_dec_place(LfGeom g, int lod, const int4* __restrict__ coords, int64_t n, DecOrder o)
{
    if (!o.total[DEC_KEYS + o.wgs]) return;
    __shared__ uint32_t next[DEC_KEYS];
    __shared__ uint32_t wsum[DEC_T / 64];
    static_assert(DEC_KEYS == DEC_T, "one thread per key");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t mine = o.total[threadIdx.x];
    uint32_t inc = mine;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)inc, s, 64);
        if (lane >= s) inc += t;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    for (int q = 0; q < wv; q++) inc += wsum[q];
    next[threadIdx.x] = inc - mine + o.hist[(int64_t)blockIdx.x * DEC_KEYS + threadIdx.x];
    __syncthreads();
    for (int u = 0; u < DEC_CHUNK / DEC_T; u++) {
        const int64_t k = (int64_t)blockIdx.x * DEC_CHUNK + u * DEC_T + threadIdx.x;
        if (k >= n) break;
        bool clamped;
        const int4 r = dec_request(g, lod, coords[k], clamped);
        // the order inside a block is of no consequence: every request decodes for itself
        const uint32_t at = atomicAdd(&next[dec_key(o, r)], 1u);
        o.rec[at] = make_uint4((uint32_t)k, (uint32_t)r.x | ((uint32_t)r.y << 16), (uint32_t)r.z | ((uint32_t)r.w << 16), 0u);
    }
}

static int64_t al256(int64_t v) { return (v + 255) & ~(int64_t)255; }

static int64_t order_layout(const LfGeom& g, int64_t n, uint8_t* base, DecOrder* o)
{
    o->wgs = (int)((n + DEC_CHUNK - 1) / DEC_CHUNK);
    o->shift = 4;
    while ((int64_t)((g.w - 1) / (1 << o->shift) + 1) * ((g.h - 1) / (1 << o->shift) + 1) > DEC_KEYS) o->shift++;
    o->kx = (g.w - 1) / (1 << o->shift) + 1;
    int64_t at = 0;
    o->rec = (uint4*)(base + at);
    at += al256(n * 16);
    o->hist = (uint32_t*)(base + at);
    at += al256((int64_t)o->wgs * DEC_KEYS * 4);
    o->total = (uint32_t*)(base + at);
    at += al256((DEC_KEYS + o->wgs + 1) * 4);
    return at;
}

// Fields that L2 holds: requests are not ordered.
static bool dec_small_field(const LfGeom& g) { return (int64_t)g.na * g.nb * g.w * g.h < (1 << 22); }

// Whether k_decode_dense takes n unordered requests of a dense handle; more go
// to the one-thread walk, whose table and vectors are half the bytes of the
// descriptors: scattered over 17x17x512x512, 98,304 take 61 us here and 75
// there, 2^18 172 and 125.  Over 9x9x192x192, 163,840 take 57 and 56 in 4x4
// blocks, 42 and 56 in 16x16, 2^18 92 and 75, 67 and 66; consecutive ones 12
// and 21, 2^18 12 and 23.
bool lf_decode_unordered(const lf_handle* h, int64_t n)
{
    return n < (dec_small_field(h->L.g) ? DEC_SMALL : LF_DECODE_ORDER_MIN);
}

// Scratch that ordering n requests takes; 0 where requests are not ordered:
// few or more than 2^26 of them, and small fields, which L2 holds anyway.
// Over 17x17x512x512, scattered requests: 2^17 80 -> 50 us, 2^18 125 -> 75,
// 2^20 607 -> 237 (one thread per sample, unordered, before; the scattered
// walk fetches 31 cache lines a sample, 6.6 TB/s).  Consecutive ones, left in
// order: 2^18 34 -> 24 us, 2^20 87 -> 59.  The line: below it the three
// launches cost consecutive requests more than they had taken (98,304: 17.4
// us, 18.3 with them), and scattered ones run in 61 against 75 without.  Over
// fields of two or three levels, whose samples are cheaper, consecutive ones
// still pay for the launches there: 114,688 11..16 -> 20..22 us, 2^18 14..21 ->
// 20..22, even at 2^19; scattered 34..73 -> 25..56 and 48..143 -> 38..111.
int64_t lf_decode_scratch(const lf_handle* h, int64_t n)
{
    const LfGeom& g = h->L.g;
    if (h->L.sparse || h->L.chroma420 || n < LF_DECODE_ORDER_MIN || n > DEC_MAX) return 0;
    if (dec_small_field(g)) return 0;
    DecOrder o;
    return order_layout(g, n, nullptr, &o);
}

lf_status lf_launch_decode_dense(const lf_handle* h, int lod, const int32_t* d_coords, int64_t n, uint8_t* d_rgb,
                                 unsigned long long* clamps, void* d_scratch, hipStream_t s)
{
    const int64_t wgs = (n + 63) / 64;  // at most 2^20: n is at most DEC_MAX with scratch, below DEC_SMALL without
    const int4* coords = (const int4*)d_coords;
    DecOrder o = {};
    if (!d_scratch) {
        hipLaunchKernelGGL(k_decode_dense<false>, dim3((unsigned)wgs), dim3(192), 0, s, h->L.g, h->p, lod, coords, n, d_rgb,
                           clamps, o);
        return lf_check_launch("decode_pixels");
    }
    order_layout(h->L.g, n, (uint8_t*)d_scratch, &o);
    hipLaunchKernelGGL(k_dec_count, dim3((unsigned)o.wgs), dim3(DEC_T), 0, s, h->L.g, lod, coords, n, clamps, o);
    hipLaunchKernelGGL(k_dec_prefix, dim3(DEC_KEYS / 64), dim3(1024), 0, s, n, o);
    hipLaunchKernelGGL(k_dec_place, dim3((unsigned)o.wgs), dim3(DEC_T), 0, s, h->L.g, lod, coords, n, o);
    // a multiple of 8 workgroups: the XCD ranges cover all of them
    hipLaunchKernelGGL(k_decode_dense<true>, dim3((unsigned)((wgs + 7) / 8 * 8)), dim3(192), 0, s, h->L.g, h->p, lod, coords, n,
                       d_rgb, clamps, o);
    return lf_check_launch("decode_pixels");
}
