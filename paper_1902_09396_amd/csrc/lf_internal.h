// Host-side internals shared by the library's translation units.
#pragma once

#include <cstdarg>
#include <cstdint>

#include "../../include/hmlfc.h"
#include "lf_geom.h"

struct LfLayout {
    LfGeom g;
    uint64_t root_off, root_bytes, table_off, table_bytes, payload_off, payload_bytes, mv_off, mv_bytes;
    int64_t n_rec;        // motion records over all channels and levels
    int64_t stream_bytes;
    // per channel: sum over the levels of the largest SRV magnitude that the
    // block table allows
    int64_t srv_bound[3];
    // every motion vector fits the descriptors' 12 signed bits, by the sequences' widths
    int32_t packed_vectors;
    // set by the load: those bounds and the root keep every level's samples,
    // not the leaf views' alone, inside the range of the packed 16-bit decode
    int32_t packed_levels;
    // 4:2:0, set by the load: the leaf views' samples are, if not every level's
    int32_t packed_leaves;
    // arena offsets
    int64_t a_root, a_table, a_payload, a_mv, a_refs, a_desc, a_status, arena;
    // sparse reference residency (LF_LOAD_SPARSE_REFS): a_refs holds n_tiles
    // block tiles, a_slots the tile of every reference block; no descriptors
    int32_t sparse;  // reference residency: LF_RES_DENSE, LF_RES_TILES or LF_RES_CSR
    int64_t n_tiles, a_slots;
    // CSR residency: values (int16, at a_refs) and columns of at most
    // nnz_bound nonzero reference pixels, and row starts; nnz is the count
    // found at load
    int64_t nnz_bound, nnz, a_cols, a_rowptr;
    // 4:2:0 chroma (Co and Cg at half width and height): g is the luma
    // geometry (one channel) and gc the chroma geometry (two channels), each
    // with its own root, table, reference planes (at a_refs and a_refs_c)
    // and motion directories; no descriptors
    int32_t chroma420;
    LfGeom gc;
    int64_t a_refs_c;
};

struct lf_handle {
    LfLayout L;
    uint8_t* arena;
    LfPtrs p;   // every channel, or luma for 4:2:0
    LfPtrs pc;  // 4:2:0 chroma (Co, Cg)
};

// LF_EINVAL unless the handle's chroma planes are full size (calls built on
// one uniform plane geometry: the tile renderer, the relaxed model and its
// adjoint, footprint accounting, serving)
lf_status lf_require_full_chroma(const lf_handle* h, const char* what);

lf_status lf_fail(lf_status s, const char* fmt, ...);
lf_status lf_check_launch(const char* what);
lf_status lf_parse(const uint8_t* s, size_t n, LfLayout* L);

// A callable of one int, not owned and not copied to the heap.
class LfWork {
    const void* f;
    void (*call)(const void*, int);

public:
    template <class F>
    LfWork(const F& work) : f(&work), call([](const void* p, int k) { (*static_cast<const F*>(p))(k); })
    {
    }
    void operator()(int k) const { call(f, k); }
};

// work(0) .. work(parts - 1), each on a thread of its own while threads can be
// started (work(0) and the rest on the caller's); returns when all are done.
// work must not throw; nothing else is thrown.
void lf_parallel(int parts, LfWork work);

// Samples of level `lod` from a dense handle (lf_decode.hip); d_scratch: null,
// or lf_decode_scratch(h, n) > 0 bytes in which the requests are ordered first.
int64_t lf_decode_scratch(const lf_handle* h, int64_t n);
bool lf_decode_unordered(const lf_handle* h, int64_t n);
lf_status lf_launch_decode_dense(const lf_handle* h, int lod, const int32_t* d_coords, int64_t n, uint8_t* d_rgb,
                                 unsigned long long* clamps, void* d_scratch, hipStream_t s);

// Phase-shifted motion search (lf_search.hip) on device planes, for the
// device encoder: checks the sizes, enqueues k_mc_search on `stream`.
lf_status lf_search_launch(const int16_t* pred, const int16_t* ref, int64_t n_pred, int64_t n_ref, int w, int h,
                           int bs, int win, int subpel, int zero_phase, const int32_t* items, int64_t n, int32_t* out,
                           void* stream);
