// gfx950 kernels of the decoder.  Included once, by jpgd.hip.
//
// Launch geometry: every kernel runs kWG = 256 lanes (four wave64) per workgroup, except the
// inter-sequence kernel (one wave64).  A workgroup finds its image by bisection over the per-image
// first-workgroup fields of ImgDesc, so one launch covers a whole batch.
#pragma once
#include <hip/hip_runtime.h>

#include "jpgd_common.h"
#include "jpgd_idct.h"
#include "jpgd_lane.h"

namespace jpgd {

struct Params {
    const ImgDesc* img;
    ImgState* st;
    Status* status;
    const uint8_t* scans;
    uint8_t* stream;        // unstuffed streams, image i at img[i].stream_off
    uint32_t* tile_cnt;     // per unstuff tile: bytes removed in it (low half) and restart markers met in it (high
                            // half), then (in place, images of more than kSumMax tiles) bytes removed before it
    SInfo* sinfo;
    int4* grp_tot;          // per group of kWG subsequences: (units, dc0, dc1, dc2) totals
    int4* grp_pref;         // exclusive prefix of grp_tot inside the image
    uint32_t* bmap;         // interval-start bitmaps of images with restart intervals (ImgDesc::bmap_off)
    uint32_t* seq_rec;      // split synchronisation: per sequence 4 x kWG words, the records of all its lanes after their
                            // own subsequence (state, units, DC sums), handed from the first kernel to the second
    uint32_t* warm_x;       // per sequence: the state at its first subsequence's start that its records continue
                            // (packed like SInfo::x; 0xFFFFFFFF = none)
    const uint16_t* luts;
    const uint16_t* qts;
    int16_t* coef;
    uint8_t* pixels;
    uint32_t nimg;
    uint32_t logL;          // log2 of the subsequence size in bits
    uint32_t overlap;       // H: warm-up lanes in front of each sequence
    uint32_t seq_len;       // kWG - H: subsequences a sequence owns
    uint32_t tab_bytes;     // max bytes of any image's tables in LDS (stage_tables; a multiple of 16)
    uint32_t planar;        // pixel kernel: component planes (no upsampling, no colour conversion) instead of RGB
    uint32_t pix_per_wg;    // pixel kernel: runs of MCUs a workgroup takes one after the other
    uint32_t scale_log2;    // pixel kernel: output at 1/2^scale_log2 of the size (0..3)
    uint32_t handoff;       // intra-sequence kernel, split in two: chains left at which the first hands over (at most 64)
    uint32_t coop_max;      // intra-sequence kernel: with at most this many chains left, one wavefront per chain
    uint32_t tile_off;      // write kernel with the output gathered in LDS: where that lies and how many bytes it has
    uint32_t tile_bytes;
    uint32_t clear;         // the synchronisation kernels clear the coefficients (kClearAheadBytes), not the write kernel
    uint32_t fold;          // calls without restart intervals: the synchronisation kernels add up the group totals as they
                            // publish records, and k_group_totals only runs in further rounds
    uint32_t sync_waves;    // wavefronts per workgroup of that kernel: kWG / 64 that hold the lanes, the rest only take chains
    // A call with one image has the last up_wgs workgroups of its first kernel (k_unstuff_count, or k_unstuff_scatter<true>,
    // which leaves out the image states it writes itself) copy the call's parameter block (up_n16 16-byte words) from
    // pinned host memory into the workspace: that kernel does not need the block, all later ones do, and a kernel of
    // its own for the copy would cost a dispatch.  up_wgs = 0: nothing to copy.
    const uint4* up_src;
    uint4* up_dst;
    uint32_t up_n16;
    uint32_t up_wgs;
    // pixel kernel: where its first lane reports the outcome of the write kernel before anything else (pinned host
    // memory: flags, inter_changed, pending, .., ticket in word 15; null = somebody else reports) and this call's ticket
    uint32_t* verdict;
    uint32_t ticket;
    // A call with one image carries its descriptor in the kernel arguments: every workgroup of every kernel
    // starts by reading the descriptor, and when all of them ask memory for the same freshly written line
    // that read alone was measured at 1 to 11 microseconds per kernel.
    ImgDesc img0;
};

// A workgroup's image descriptor.  It is the same for every lane, but the compiler cannot see that (it merges
// the two sources into one load through a generic pointer and takes the result for lane-dependent), so what
// follows from it sits in vector registers and branches on it are taken with execution masks.
__device__ __forceinline__ ImgDesc image_desc(const Params& P, uint32_t ii) {
    if (P.nimg == 1u) return P.img0;
    return P.img[ii];
}

// Descriptors are written by nobody while a kernel runs that reads them.  Read through the constant address space
// they come by scalar loads, also behind a store, where the compiler otherwise reads lane by lane and takes the result
// for lane-dependent.
using ConstWords = const __attribute__((address_space(4))) uint32_t*;
__device__ __forceinline__ ConstWords const_words(const void* p) { return (ConstWords)(uintptr_t)p; }

// The same in scalar registers: what follows from the descriptor stays there and branches on it are scalar branches.
// Measured per kernel: pixels 9 %, write 2 % and unstuff_count 8 % faster with it; the two synchronisation kernels 2 to
// 4 % slower (their lane decoder is short of scalar registers, not of vector ones), so they keep the plain form.
__device__ __forceinline__ ImgDesc image_desc_uniform(const Params& P, uint32_t ii) {
    static_assert(sizeof(ImgDesc) % 4u == 0u, "descriptor is copied word by word");
    if (P.nimg == 1u) return P.img0;
    uint32_t w[sizeof(ImgDesc) / 4u];
    const ConstWords src = const_words(P.img + ii);
#pragma unroll
    for (uint32_t i = 0; i < sizeof(ImgDesc) / 4u; ++i) w[i] = src[i];
    ImgDesc d;
    __builtin_memcpy(&d, w, sizeof d);
    return d;
}

// ---- small helpers ------------------------------------------------------------------------------

// The image a workgroup belongs to; first_wg: the descriptor's word with the image's first workgroup.  (In the pixel
// kernel, whose first lane reports the verdict before this, every step of the search was a vector load and its wait: six
// trips to L2 for 48 images.)
__device__ __forceinline__ uint32_t find_image(const Params& P, uint32_t wg, const uint32_t ImgDesc::*first_wg) {
    uint32_t lo = 0, hi = P.nimg;  // last image whose first workgroup is <= wg
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (*const_words(&(P.img[mid].*first_wg)) <= wg) lo = mid; else hi = mid;
    }
    return lo;
}

// v plus the value some lanes further down (data-parallel moves between the lanes of a wavefront: no LDS round trip;
// lanes without a source add 0).  All 64 lanes must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v) {
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v = dpp_add<0x111, 0xF>(v);  // row_shr:1, :2, :4, :8 inside the rows of 16 lanes
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);  // row_bcast:15: rows 1 and 3 add the last lane of the row before them
    v = dpp_add<0x143, 0xC>(v);  // row_bcast:31: rows 2 and 3 add lane 31
    return v;
}

// exclusive prefix of v over the 256 lanes of the workgroup; *total gets the sum.  scratch: 8 words of LDS.
__device__ __forceinline__ uint32_t wg_excl_scan(uint32_t v, uint32_t* scratch, uint32_t* total) {
    uint32_t inc = wave_incl_scan(v);
    uint32_t wave = threadIdx.x >> 6;
    __syncthreads();  // scratch may still be read from a previous use
    if ((threadIdx.x & 63u) == 63u) scratch[wave] = inc;
    __syncthreads();
    uint32_t w0 = scratch[0], w1 = scratch[1], w2 = scratch[2], w3 = scratch[3];
    uint32_t before = wave == 0 ? 0u : wave == 1 ? w0 : wave == 2 ? w0 + w1 : w0 + w1 + w2;
    *total = w0 + w1 + w2 + w3;
    return before + inc - v;
}

// What the scan over s_info carries (paper, Algorithm 1: exclusive prefix sum on s_info.n; Section 4.2: prefix
// sum of the DC differences): data units, and the DC sums of the three components.  With restart intervals
// the DC sums are a segmented sum: a record whose subsequence holds the first symbol of an interval (flag)
// starts them afresh.  join(a, b) = a followed by b; it is associative, so the usual scans apply.
// (the sums are kept unsigned: only their low 16 bits are used and they may wrap on the way)
struct Seg {
    uint32_t units, flag;
    uint32_t d0, d1, d2;
};
__device__ __forceinline__ Seg seg_zero() { return Seg{0u, 0u, 0u, 0u, 0u}; }
__device__ __forceinline__ Seg seg_join(const Seg& a, const Seg& b) {
    Seg r;
    r.units = a.units + b.units;
    r.flag = a.flag | b.flag;
    r.d0 = b.flag ? b.d0 : a.d0 + b.d0;
    r.d1 = b.flag ? b.d1 : a.d1 + b.d1;
    r.d2 = b.flag ? b.d2 : a.d2 + b.d2;
    return r;
}
__device__ __forceinline__ uint32_t sx16(uint32_t v) { return (uint32_t)(int32_t)(int16_t)(v & 0xFFFFu); }
__device__ __forceinline__ Seg seg_of_record(const SInfo& r) {
    return Seg{rec_units(r.y), rec_restarted(r.y), sx16(r.z), sx16(r.z >> 16), sx16(r.w)};
}
// group totals travel as int4: units with the flag in bit 31, then the three sums
__device__ __forceinline__ int4 seg_pack(const Seg& s) { return make_int4((int)(s.units | (s.flag << 31)), (int)s.d0, (int)s.d1, (int)s.d2); }
__device__ __forceinline__ Seg seg_unpack(const int4& v) {
    return Seg{(uint32_t)v.x & 0x7FFFFFFFu, (uint32_t)v.x >> 31, (uint32_t)v.y, (uint32_t)v.z, (uint32_t)v.w};
}
__device__ __forceinline__ Seg seg_shfl_up(const Seg& v, int d) {
    Seg o;
    o.units = __shfl_up(v.units, d, 64); o.flag = __shfl_up(v.flag, d, 64);
    o.d0 = __shfl_up(v.d0, d, 64); o.d1 = __shfl_up(v.d1, d, 64); o.d2 = __shfl_up(v.d2, d, 64);
    return o;
}

// The join of records without interval starts is four plain sums, which the lanes pass on without LDS.
__device__ __forceinline__ Seg wave_incl_sums(const Seg& v) {
    return Seg{wave_incl_scan(v.units), 0u, wave_incl_scan(v.d0), wave_incl_scan(v.d1), wave_incl_scan(v.d2)};
}
__device__ __forceinline__ void put_sums(uint32_t* s4, const Seg& v) { s4[0] = v.units; s4[1] = v.d0; s4[2] = v.d1; s4[3] = v.d2; }
__device__ __forceinline__ Seg get_sums(const uint32_t* s4) { return Seg{s4[0], 0u, s4[1], s4[2], s4[3]}; }

// Group totals added up by the synchronisation kernels (Params::fold): the workgroup of tile lt, which runs before
// them, clears the total of group lt (a group of subsequences holds at least the bits of a tile, so an image has no
// more groups than tiles).
static_assert((uint64_t)kWG * kMinSubseqBits >= 8ull * kUnstuffTile, "every group's total is cleared by a tile of its own number");
__device__ __forceinline__ void clear_group_total(const Params& P, const ImgDesc& D, uint32_t lt) {
    if (P.fold && lt < D.ngrp_max && threadIdx.x < 4u) reinterpret_cast<uint32_t*>(P.grp_tot + D.grp0 + lt)[threadIdx.x] = 0u;
}
__device__ __forceinline__ void add_group_total(int4* tot, const Seg& s) {
    uint32_t* w = reinterpret_cast<uint32_t*>(tot);
    atomicAdd(w, s.units); atomicAdd(w + 1, s.d0); atomicAdd(w + 2, s.d1); atomicAdd(w + 3, s.d2);
}
__device__ __forceinline__ Seg seg_minus(const Seg& a, const Seg& b) {
    return Seg{a.units - b.units, 0u, a.d0 - b.d0, a.d1 - b.d1, a.d2 - b.d2};
}
// The records of a sequence are those of a decoder that entered it in the state `warm_x` holds for it (the
// state its workgroup's warm-up lanes arrived in, or the one an inter-sequence lane started from).  If the
// sequence before it now ends in another state - an inter-sequence lane rewrote its last record in the same
// round, after the lane of this boundary had looked - the states further on can still be right, and the write
// pass will find nothing wrong, but the counts and DC sums of the sequence's first records belong to the other
// entry state.  The boundaries inside group lg are looked at here (at most four: a sequence has at least 65
// subsequences), by the first four lanes of a kernel behind the inter-sequence kernel, and the host runs another
// round if one is found.
__device__ __forceinline__ void check_boundaries(const Params& P, const ImgDesc& D, uint32_t lg, uint32_t nsub) {
    if (nsub <= P.seq_len || threadIdx.x >= 4u) return;
    const uint32_t i0 = lg * (uint32_t)kWG;
    const uint32_t first = (i0 + P.seq_len - 1u) / P.seq_len;  // first sequence that starts in this group
    const uint32_t g = (first + threadIdx.x) * P.seq_len;
    if (g > 0u && g < nsub && g < i0 + (uint32_t)kWG &&
        P.warm_x[D.seq0 + first + threadIdx.x] != __atomic_load_n(&P.sinfo[D.sub0 + g - 1u].x, __ATOMIC_RELAXED))
        atomicOr(&P.status->pending, 1u);
}

// exclusive scan of v over the 256 lanes of the workgroup under seg_join; *total gets the join of all.
// scratch: 20 words of LDS.
__device__ __forceinline__ Seg wg_excl_segscan(Seg v, uint32_t* scratch, Seg* total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    Seg inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const Seg o = seg_shfl_up(inc, d);
        if (lane >= (uint32_t)d) inc = seg_join(o, inc);
    }
    __syncthreads();  // scratch may still be read from a previous use
    if (lane == 63u) {
        uint32_t* s5 = scratch + wave * 5u;
        s5[0] = inc.units; s5[1] = inc.flag; s5[2] = inc.d0; s5[3] = inc.d1; s5[4] = inc.d2;
    }
    __syncthreads();
    Seg carry = seg_zero(), all = seg_zero();
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) {
        const uint32_t* s5 = scratch + k * 5u;
        const Seg t = Seg{s5[0], s5[1], s5[2], s5[3], s5[4]};
        if (k < wave) carry = seg_join(carry, t);
        all = seg_join(all, t);
    }
    *total = all;
    Seg before = seg_shfl_up(inc, 1);
    if (lane == 0u) before = seg_zero();
    return seg_join(carry, before);
}

// The image's tables as the synchronisation kernels (sync_entry) or the write kernel (write_entry) read them, at the start of
// the dynamic LDS: DC tables, AC tables, subtables of the AC tables, subtables of the DC tables in any order.  dc_fill: a word of LDS, zero since the
// last barrier; all of it is complete after the next one.  What points into the tables (the rows, escapes) counts its bytes
// from the start of LDS: a lane then has its addresses without an addition.
using LdsBytes = const __attribute__((address_space(3))) uint8_t*;
using LdsWords = const __attribute__((address_space(3))) uint32_t*;
__device__ __forceinline__ uint32_t lds_at(const void* p) { return (uint32_t)(uintptr_t)(LdsBytes)p; }
__device__ __forceinline__ uint32_t lds_word(uint32_t at) { return *(LdsWords)(uintptr_t)at; }
typedef uint32_t lds_quad __attribute__((ext_vector_type(4)));
__device__ __forceinline__ SyncRow lds_row(uint32_t at) {
    const lds_quad q = *(const __attribute__((address_space(3))) lds_quad*)(uintptr_t)at;
    return SyncRow{q.x, q.y, q.z, q.w};
}
__device__ __forceinline__ uint32_t sync_ac_at(const ImgDesc& D) { return D.ndc * kSyncDcBytes; }
template <bool WRITE>
__device__ __forceinline__ void stage_tables(const Params& P, const ImgDesc& D, uint8_t* lds, uint32_t* dc_fill) {
    uint32_t* const tab = reinterpret_cast<uint32_t*>(lds);
    const uint16_t* luts = P.luts + D.lut_off;
    const uint8_t* pairs = reinterpret_cast<const uint8_t*>(luts + kMaxSlots * kLutEntries);
    const uint32_t nac = D.nslots - D.ndc;
    const uint32_t ac = sync_ac_at(D), l2 = ac + nac * kSyncAcBytes, lds0 = lds_at(lds);
    const uint32_t n0 = D.sub_words & 1023u, n1 = (D.sub_words >> 10) & 1023u, n2 = D.sub_words >> 20;
    static_assert(kMaxPairs == 3, "sub_words holds three counts");
    for (uint32_t k = threadIdx.x; k < nac * (uint32_t)(kLutL1 / 8); k += blockDim.x) {  // eight entries
        const uint32_t a = k / (uint32_t)(kLutL1 / 8), i = (k % (uint32_t)(kLutL1 / 8)) * 8u;
        const uint4 e = *reinterpret_cast<const uint4*>(luts + (D.ndc + a) * (uint32_t)kLutEntries + i);
        uint2 pb = make_uint2(0u, 0u);
        if (!WRITE) pb = *reinterpret_cast<const uint2*>(pairs + a * (uint32_t)kPairBytes + i);
        const uint32_t at = lds0 + l2 + (a > 0u ? n0 * 4u : 0u) + (a > 1u ? n1 * 4u : 0u);
        uint4* dst = reinterpret_cast<uint4*>(tab + (ac >> 2) + a * (uint32_t)kLutL1 + i);
        dst[0] = make_uint4(sync_ac_entry<WRITE>(0u, e.x & 0xFFFFu, pb.x & 255u, at), sync_ac_entry<WRITE>(1u, e.x >> 16, (pb.x >> 8) & 255u, at),
                            sync_ac_entry<WRITE>(0u, e.y & 0xFFFFu, (pb.x >> 16) & 255u, at), sync_ac_entry<WRITE>(1u, e.y >> 16, pb.x >> 24, at));
        dst[1] = make_uint4(sync_ac_entry<WRITE>(0u, e.z & 0xFFFFu, pb.y & 255u, at), sync_ac_entry<WRITE>(1u, e.z >> 16, (pb.y >> 8) & 255u, at),
                            sync_ac_entry<WRITE>(0u, e.w & 0xFFFFu, (pb.y >> 16) & 255u, at), sync_ac_entry<WRITE>(1u, e.w >> 16, pb.y >> 24, at));
    }
    for (uint32_t k = threadIdx.x; k < (n0 + n1 + n2) >> 1; k += blockDim.x) {  // two entries
        uint32_t j = 2u * k, a = 0u;
        if (j >= n0) { j -= n0; a = 1u; if (j >= n1) { j -= n1; a = 2u; } }
        const uint32_t e = *reinterpret_cast<const uint32_t*>(luts + (D.ndc + a) * (uint32_t)kLutEntries + (uint32_t)kLutL1 + j);
        reinterpret_cast<uint2*>(tab + (l2 >> 2))[k] = make_uint2(pass_entry<WRITE>(e & 0xFFFFu, false, 0u), pass_entry<WRITE>(e >> 16, false, 0u));
    }
    const uint32_t dc_sub = l2 + (n0 + n1 + n2) * 4u;
    for (uint32_t k = threadIdx.x; k < D.ndc << kSyncDcK; k += blockDim.x) {
        const uint16_t* lut = luts + (k >> kSyncDcK) * (uint32_t)kLutEntries;
        const uint32_t e = *reinterpret_cast<const uint32_t*>(lut + (k & ((1u << kSyncDcK) - 1u)) * 2u);
        const uint32_t a = e & 0xFFFFu, b = e >> 16, n = sync_dc_sub(a, b);
        if (n == 0xFFFFFFFFu) {
            tab[k] = sync_dc_direct<WRITE>(a);
        } else {
            const uint32_t at = dc_sub + atomicAdd(dc_fill, 8u << n);  // (a multiple of 8)
            for (uint32_t j = 0u; j < 2u << n; ++j) tab[(at >> 2) + j] = sync_dc_sub_entry<WRITE>(a, b, n, j, lut + kLutL1);
            tab[k] = sync_escape(n + 1u, lds0 + at);
        }
    }
}

// rows: 8 entries of LDS, complete after the next barrier
template <bool WRITE>
__device__ __forceinline__ void stage_rows(const ImgDesc& D, SyncRow* rows, uint32_t tab) {  // (rows, too, by their bytes of LDS)
    const uint32_t u = threadIdx.x, un = u + 1u == D.upm ? 0u : u + 1u;
    if (u >= D.upm) return;
    const uint32_t comp = (D.sched_comp >> (4u * u)) & 15u, comp_next = (D.sched_comp >> (4u * un)) & 15u;
    {
        rows[u] = SyncRow{tab + sync_ac_at(D) + (((D.sched_ac >> (4u * u)) & 15u) - D.ndc) * kSyncAcBytes,
                          tab + ((D.sched_dc >> (4u * un)) & 15u) * kSyncDcBytes,
                          WRITE ? (comp != comp_next ? 1u : 0u) : 1u << (15u * comp), lds_at(rows) + un * (uint32_t)sizeof(SyncRow)};
    }
}

// LDS copy of a stretch of the stream as big-endian 32-bit words.  No padding: lanes start a power of two
// apart and collide on a bank for their first reads only; after that they advance at their own pace.
__device__ __forceinline__ void stage_stream(const uint8_t* stream_img, uint32_t first_word, uint32_t nwords,
                                             uint32_t* strm) {
    // nwords is a multiple of 4 and first_word*4 a multiple of 16
    const uint4* src = reinterpret_cast<const uint4*>(stream_img + (size_t)first_word * 4u);
    uint4* dst = reinterpret_cast<uint4*>(strm);
    for (uint32_t k = threadIdx.x; k < nwords / 4u; k += blockDim.x) {
        uint4 v = src[k];
        v.x = __builtin_bswap32(v.x); v.y = __builtin_bswap32(v.y);
        v.z = __builtin_bswap32(v.z); v.w = __builtin_bswap32(v.w);
        dst[k] = v;
    }
}

// LDS copy of the part of an image's interval-start bitmap that covers stream words first_word .. +nwords;
// word k of the bitmap is then bm_s[k - (first_word >> 3)]
// Returns the OR of the words this lane copied: most workgroups of a scan with long intervals find no interval
// start at all in their stretch and can run the plain loops.
// With keep == false nothing is stored: the words are only looked at (subsequences of more than kBitmapLdsMaxL bits,
// whose kernels then read the few bitmap words they need from memory; see kBitmapLdsMaxL).
__device__ __forceinline__ uint32_t stage_bitmap(const uint32_t* bmap_img, uint32_t first_word, uint32_t nwords, uint32_t* bm_s,
                                                 bool keep) {
    const uint32_t k0 = first_word >> 3;
    const uint32_t n = ((first_word + nwords + 7u) >> 3) - k0 + 1u;
    uint32_t seen = 0u;
    for (uint32_t k = threadIdx.x; k < n; k += blockDim.x) {
        const uint32_t v = bmap_img[k0 + k];
        if (keep) bm_s[k] = v;
        seen |= v;
    }
    return seen;
}

__device__ __forceinline__ uint32_t pack_dc01(int64_t acc) {
    int32_t d0, d1, d2;
    dc_unpack(acc, d0, d1, d2);
    return ((uint32_t)d0 & 0xFFFFu) | ((uint32_t)d1 << 16);
}
__device__ __forceinline__ uint32_t pack_dc2(int64_t acc) {
    int32_t d0, d1, d2;
    dc_unpack(acc, d0, d1, d2);
    return (uint32_t)d2 & 0xFFFFu;
}

// ---- unstuffing (byte compaction) -----------------------------------------------------------------
// A 0x00 is dropped iff the byte before it is 0xFF: inside entropy-coded data a 0xFF is always followed by
// its stuffed 0x00 or, in a scan with restart intervals, by the second byte of a marker RST0..RST7; both
// bytes of such a marker are dropped too, and the byte that follows it is the first of an interval.  All
// decisions are local (one byte back, one byte ahead).

// Four bytes at a time: 0x80 in every byte of x that is zero (exact, no carry from byte to byte).
__device__ __forceinline__ uint32_t zero_bytes(uint32_t x) {
    return ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu);
}
// 0x80 in the first n bytes of word k of a lane's four
__device__ __forceinline__ uint32_t first_bytes(uint32_t n, uint32_t k) {
    const uint32_t m = n <= 4u * k ? 0u : min(n - 4u * k, 4u);
    return m == 4u ? 0x80808080u : 0x80808080u & ((1u << (8u * m)) - 1u);
}
__device__ __forceinline__ uint32_t count4(const uint32_t (&m)[4]) {
    return (uint32_t)(__popc(m[0]) + __popc(m[1]) + __popc(m[2]) + __popc(m[3]));
}

struct UnstuffLane {
    uint32_t bytes[4];  // 16 input bytes
    uint32_t drop[4];   // 0x80 in every byte that is not kept (bytes past the end among them)
    uint32_t mark[4];   // 0x80 in every byte that is the second of a restart marker
    uint32_t nvalid;    // bytes of this lane that exist
};

// pos is a multiple of 16.  A lane that holds any byte loads its whole 16-byte word (the input is readable up
// to the next multiple of 16); bytes past the end are masked out.  The bytes are looked at four at a time, beside
// the word that holds the byte before each of them: about 30 instructions for 16 bytes, where one byte after the
// other took 170 and filled three quarters of the chip's issue slots (66 MB: count 29.6 -> 17.9 us, 3.7 TB/s; scatter
// 53 -> 34 us, 3.9 TB/s).  No private array is indexed with a variable:
// the compiler would move such an array to LDS and read the dispatch packet for the workgroup's shape, and that
// packet lives in host memory -- measured at 2 to 11 microseconds per wavefront when a whole grid asks at once.
// All 64 lanes of the wavefront call this together.
__device__ __forceinline__ UnstuffLane unstuff_load(const uint8_t* scan, uint32_t n, uint32_t pos, bool restart) {
    UnstuffLane r;
    r.nvalid = pos >= n ? 0u : (n - pos < 16u ? n - pos : 16u);
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    uint32_t before = 0u;
    if (r.nvalid) {
        v = *reinterpret_cast<const uint4*>(scan + pos);
        if ((threadIdx.x & 63u) == 0u && pos > 0u) before = (uint32_t)scan[pos - 1u] << 24;
    }
    r.bytes[0] = v.x; r.bytes[1] = v.y; r.bytes[2] = v.z; r.bytes[3] = v.w;
    // the last word of the lane before (wave_shr:1); the first lane keeps what it loaded
    before = (uint32_t)__builtin_amdgcn_update_dpp((int)before, (int)v.w, 0x138, 0xF, 0xF, false);
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) {
        const uint32_t prev = __builtin_amdgcn_alignbyte(r.bytes[k], k ? r.bytes[k - 1u] : before, 3u);
        r.drop[k] = zero_bytes(r.bytes[k] | ~prev);  // 0x00 behind 0xFF
        r.mark[k] = 0u;
    }
    if (restart) {
        const uint32_t after = pos + 16u < n ? scan[pos + 16u] : 0u;
        const uint32_t nfollowed = pos + 16u < n ? 16u : (r.nvalid ? r.nvalid - 1u : 0u);  // bytes that have a next one
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t w = r.bytes[k];
            const uint32_t prev = __builtin_amdgcn_alignbyte(w, k ? r.bytes[k - 1u] : before, 3u);
            const uint32_t next = __builtin_amdgcn_alignbyte(k < 3u ? r.bytes[k + 1u] : after, w, 1u);
            r.mark[k] = zero_bytes(((w ^ 0xD0D0D0D0u) & 0xF8F8F8F8u) | ~prev) & first_bytes(r.nvalid, k);   // RSTm, second byte
            const uint32_t rst1 = zero_bytes(((next ^ 0xD0D0D0D0u) & 0xF8F8F8F8u) | ~w) & first_bytes(nfollowed, k);  // first byte
            r.drop[k] |= r.mark[k] | rst1;
        }
    }
    if (r.nvalid < 16u) {
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) r.drop[k] |= 0x80808080u & ~first_bytes(r.nvalid, k);
    }
    return r;
}

// The copy of the parameter block (one image per call only), by the last workgroups of the call's first kernel.
// WRITES_STATE: that kernel writes the image states, which lie between the block's status word and its descriptors, and
// they are left out of the copy.
template <bool WRITES_STATE>
__device__ __forceinline__ bool copy_parameters(const Params& P) {
    const uint32_t first = gridDim.x - P.up_wgs;
    if (blockIdx.x < first) return false;
    const uint4* const st0 = reinterpret_cast<const uint4*>(P.st);
    const uint4* const st1 = reinterpret_cast<const uint4*>(P.img);
    for (uint32_t k = (blockIdx.x - first) * kWG + threadIdx.x; k < P.up_n16; k += P.up_wgs * kWG)
        if (!WRITES_STATE || P.up_dst + k < st0 || P.up_dst + k >= st1) P.up_dst[k] = P.up_src[k];
    return true;
}

__global__ __launch_bounds__(kWG) void k_unstuff_count(Params P) {
    __shared__ uint32_t scratch[8];
    const uint32_t wg = blockIdx.x;
    if (copy_parameters<false>(P)) return;
    const uint32_t ii = find_image(P, wg, &ImgDesc::tile0);
    const ImgDesc D = image_desc_uniform(P, ii);
    const uint32_t lt = wg - D.tile0;
    const uint8_t* scan = P.scans + D.scan_off;
    const uint32_t pos = lt * (uint32_t)kUnstuffTile + threadIdx.x * 16u;
    const bool restart = D.restart != 0u;
    const UnstuffLane u = unstuff_load(scan, D.scan_bytes, pos, restart);
    if (restart) {
        // this tile's share of the interval-start bitmap is cleared here, the scatter kernel sets the bits;
        // the markers are counted so that the write pass can tell whether all intervals are there
        uint32_t* bm = P.bmap + D.bmap_off + lt * 128u;
        if (threadIdx.x < 128u) bm[threadIdx.x] = 0u;
        if (lt == D.ntiles - 1u && threadIdx.x < 128u) bm[128u + threadIdx.x] = 0u;
    }
    clear_group_total(P, D, lt);
    // bytes removed in the low half, markers in the high half: at most 4096 and 2048 in a tile
    uint32_t total;
    wg_excl_scan((u.nvalid + count4(u.drop) - 16u) | (count4(u.mark) << 16), scratch, &total);
    if (threadIdx.x == 0) P.tile_cnt[wg] = total;
}

// one workgroup per image: per-tile counts -> bytes removed before each tile; unstuffed length and
// number of subsequences of the image
__global__ __launch_bounds__(kWG) void k_unstuff_scan(Params P) {
    __shared__ uint32_t scratch[8];
    const uint32_t ii = blockIdx.x;
    const ImgDesc D = image_desc_uniform(P, ii);
    if (D.ntiles <= (uint32_t)kSumMax) return;  // (the scatter kernel sums the counts itself)
    // every lane takes a run of consecutive tiles: sum, one scan over the 256 sums, then the prefixes inside the run
    // (one pair of barriers in all; a loop of 256-tile scans was measured at 0.7 microseconds per step)
    uint32_t* cnt = P.tile_cnt + D.tile0;
    const uint32_t per = (D.ntiles + (uint32_t)kWG - 1u) / (uint32_t)kWG;
    const uint32_t k0 = min(threadIdx.x * per, D.ntiles), k1 = min(k0 + per, D.ntiles);
    uint32_t sum = 0u, msum = 0u;
#pragma unroll 8
    for (uint32_t k = k0; k < k1; ++k) {
        const uint32_t v = cnt[k];
        sum += v & 0xFFFFu;
        msum += v >> 16;
    }
    uint32_t carry, markers;
    wg_excl_scan(msum, scratch, &markers);
    uint32_t ex = wg_excl_scan(sum, scratch, &carry);
#pragma unroll 8
    for (uint32_t k = k0; k < k1; ++k) {
        const uint32_t v = cnt[k] & 0xFFFFu;
        cnt[k] = ex;
        ex += v;
    }
    if (threadIdx.x == 0) {
        uint32_t nbytes = D.scan_bytes - carry;
        P.st[ii].markers = markers;
        P.st[ii].nbytes = nbytes;
        uint32_t L = 1u << P.logL;
        P.st[ii].nsub = (uint32_t)(((uint64_t)nbytes * 8u + L - 1u) >> P.logL);
    }
}

// ALONE: the whole step in one kernel, for calls with one image of at most kAloneTiles tiles, without restart intervals:
// a workgroup counts the bytes removed in all tiles before its own itself.  It reads them once more for that, which
// for so few tiles takes less time than the kernel that would count them and the gap behind it.
template <bool ALONE>
__global__ __launch_bounds__(kWG) void k_unstuff_scatter(Params P) {
    __shared__ uint32_t scratch[16];
    __shared__ __attribute__((aligned(16))) uint8_t buf[kUnstuffTile + 32];
    const uint32_t wg = blockIdx.x;
    if (ALONE && copy_parameters<true>(P)) return;
    const uint32_t ii = find_image(P, wg, &ImgDesc::tile0);
    const ImgDesc D = image_desc_uniform(P, ii);
    const uint32_t lt = wg - D.tile0;
    const uint8_t* scan = P.scans + D.scan_off;
    uint8_t* out = P.stream + D.stream_off;
    const uint32_t pos = lt * (uint32_t)kUnstuffTile + threadIdx.x * 16u;
    // bytes removed before this tile: from the scan kernel, or, for images of up to kSumMax tiles, summed here
    const bool few_tiles = !ALONE && D.ntiles <= (uint32_t)kSumMax;
    uint32_t raw = 0u, more[kSumRun - 1] = {0u}, before = 0u, nbytes = 0u;
    if (ALONE) {
        clear_group_total(P, D, lt);
#pragma unroll 4
        for (uint32_t k = 0; k < lt; ++k) {  // (complete tiles: no byte is past the end)
            const uint32_t at = k * (uint32_t)kUnstuffTile + threadIdx.x * 16u;
            const uint4 v = *reinterpret_cast<const uint4*>(scan + at);
            const uint32_t b = at ? *reinterpret_cast<const uint32_t*>(scan + at - 4u) : 0u;
            const uint32_t drop[4] = {zero_bytes(v.x | ~__builtin_amdgcn_alignbyte(v.x, b, 3u)), zero_bytes(v.y | ~__builtin_amdgcn_alignbyte(v.y, v.x, 3u)),
                                      zero_bytes(v.z | ~__builtin_amdgcn_alignbyte(v.z, v.y, 3u)), zero_bytes(v.w | ~__builtin_amdgcn_alignbyte(v.w, v.z, 3u))};
            before += count4(drop);
        }
    } else if (few_tiles) {
        if (threadIdx.x < D.ntiles) raw = P.tile_cnt[D.tile0 + threadIdx.x];
        if (D.ntiles > (uint32_t)kWG) {
#pragma unroll
            for (uint32_t k = 1; k < (uint32_t)kSumRun; ++k)
                if (k * kWG + threadIdx.x < D.ntiles) more[k - 1u] = P.tile_cnt[D.tile0 + k * kWG + threadIdx.x];
        }
    } else {
        before = P.tile_cnt[wg];
        nbytes = P.st[ii].nbytes;
    }
    const UnstuffLane u = unstuff_load(scan, D.scan_bytes, pos, !ALONE && D.restart != 0u);
    const uint32_t kept = 16u - count4(u.drop);
    const uint32_t inc = wave_incl_scan(kept), wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 63u) scratch[wave] = inc;
    if (ALONE) {
        before = wave_incl_scan(before);
        if ((threadIdx.x & 63u) == 63u) scratch[8u + wave] = before;
    } else if (few_tiles) {
        uint32_t all = raw & 0xFFFFu, prior = threadIdx.x < lt ? raw & 0xFFFFu : 0u, marks = raw >> 16;
        if (D.ntiles > (uint32_t)kWG) {
#pragma unroll
            for (uint32_t k = 1; k < (uint32_t)kSumRun; ++k) {
                const uint32_t v = more[k - 1u] & 0xFFFFu;
                all += v;
                prior += k * kWG + threadIdx.x < lt ? v : 0u;
                marks += more[k - 1u] >> 16;
            }
        }
        all = wave_incl_scan(all);
        prior = wave_incl_scan(prior);
        marks = wave_incl_scan(marks);
        if ((threadIdx.x & 63u) == 63u) {
            scratch[4u + wave] = all;
            scratch[8u + wave] = prior;
            scratch[12u + wave] = marks;
        }
    }
    __syncthreads();
    const uint32_t w0 = scratch[0], w1 = scratch[1], w2 = scratch[2];
    const uint32_t T = w0 + w1 + w2 + scratch[3];
    const uint32_t off = (wave > 0u ? w0 : 0u) + (wave > 1u ? w1 : 0u) + (wave > 2u ? w2 : 0u) + inc - kept;
    if (ALONE) {
        before = scratch[8] + scratch[9] + scratch[10] + scratch[11];
        nbytes = lt * (uint32_t)kUnstuffTile - before + T;  // (of the last tile)
        if (lt == D.ntiles - 1u && threadIdx.x == 0u) {
            P.st[ii].markers = 0u;
            P.st[ii].nbytes = nbytes;
            P.st[ii].nsub = (uint32_t)(((uint64_t)nbytes * 8u + (1u << P.logL) - 1u) >> P.logL);
        }
    } else if (few_tiles) {
        before = scratch[8] + scratch[9] + scratch[10] + scratch[11];
        nbytes = D.scan_bytes - (scratch[4] + scratch[5] + scratch[6] + scratch[7]);
        if (lt == 0u && threadIdx.x == 0u) {
            P.st[ii].markers = scratch[12] + scratch[13] + scratch[14] + scratch[15];
            P.st[ii].nbytes = nbytes;
            P.st[ii].nsub = (uint32_t)(((uint64_t)nbytes * 8u + (1u << P.logL) - 1u) >> P.logL);
        }
    }
    // output position of this tile's first kept byte; in LDS the tile lies as far behind a multiple of 16
    const uint32_t o = lt * (uint32_t)kUnstuffTile - before;
    const uint32_t a = o & 15u;
    uint8_t* dst = buf + a + off;
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) {
        const uint32_t w = u.bytes[k], d = u.drop[k];
        if (d == 0u) {
            __builtin_memcpy(dst, &w, 4);
        } else {
            uint8_t* q = dst;
            if (!(d & 0x80u)) *q++ = (uint8_t)w;
            if (!(d & 0x8000u)) *q++ = (uint8_t)(w >> 8);
            if (!(d & 0x800000u)) *q++ = (uint8_t)(w >> 16);
            if (!(d & 0x80000000u)) *q = (uint8_t)(w >> 24);
        }
        dst += 4u - (uint32_t)__popc(d);
    }
    __syncthreads();
    // whole 16-byte words of the output; the first and the last one are shared with the neighbouring tiles
    uint8_t* base = out + (o - a);
    const uint32_t first16 = a ? 1u : 0u, last16 = (a + T) >> 4;
    for (uint32_t d = first16 + threadIdx.x; d < last16; d += kWG)
        reinterpret_cast<uint4*>(base)[d] = reinterpret_cast<const uint4*>(buf)[d];
    if (threadIdx.x < 32u) {
        const uint32_t at = threadIdx.x < 16u ? threadIdx.x : (last16 << 4) + (threadIdx.x & 15u);
        const bool mine = threadIdx.x < 16u ? (a != 0u && at >= a && at < a + T) : (at < a + T && (last16 != 0u || a == 0u));
        if (mine) base[at] = buf[at];
    }
    // the byte after a restart marker starts an interval: its position in the output goes into the bitmap
    if (!ALONE && D.restart) {
        uint32_t* bm = P.bmap + D.bmap_off;
        uint32_t at = o + off;
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            for (uint32_t m = u.mark[k]; m; m &= m - 1u) {
                const uint32_t below = (m & (0u - m)) - 1u;  // bits of the bytes in front of the marker's
                const uint32_t b = at + (uint32_t)__popc(~u.drop[k] & 0x80808080u & below);
                atomicOr(&bm[b >> 5], 1u << (b & 31u));
            }
            at += 4u - (uint32_t)__popc(u.drop[k]);
        }
    }
    // the last tile clears what lanes may read past the end: one subsequence plus 64 bytes
    if (lt == D.ntiles - 1u) {
        const uint32_t clear = (1u << (P.logL - 3u)) + 64u;
        for (uint32_t k = threadIdx.x; k < clear; k += kWG) out[nbytes + k] = 0u;
    }
}

// ---- one chain decoded by a whole wavefront -----------------------------------------------------------
// The last overflow rounds of a sequence have a handful of chains left, and a lane that decodes one step
// after the other spends over two hundred cycles on each.  So when few chains remain, each goes to a
// wavefront of its own: lane j looks up the symbol that WOULD start j bits into a window of 64, in every
// table of the image at once, and the chain is then followed through those 64 answers with scalar code (a
// readlane and a few scalar operations per symbol) until it leaves the window.  The synchronisation pass
// only needs (p, u, z), the count of completed units and the DC sums, so a symbol's value bits matter only for
// DC symbols.  Results are those of sync_span, symbol by symbol.
//
// What bounds it is the number of instructions and taken branches of a lone wavefront: a step of an AC symbol is four
// instructions, some 30 cycles, and everything else used to be four times that.  So the whole loop over the windows is
// assembly: the compiler's form of it set and tested flags around every exit, moved the next window's answers from
// register to register and spent six taken branches a window outside the walk.  Here a window costs 27 instructions and
// one taken branch, a unit's end and the DC symbol behind it 45 and three.  Each kind of data units, by their tables
// (ImgDesc::walk), has its own loop over AC symbols, so that nothing is selected per symbol.  Two kinds are the usual, and
// the walk of images with a third is a form of its own, which looks eight instructions longer at a window.
// Measured, window loop compiled around an assembly walk / this (kernels, us): second kernel of 15360x8640 848 / 705, 24
// images of 2047x1535 305 / 270, one 1600x1200 image 190 / 158, 256 images of 512x384 213 / 186, 1001x667 89 / 80; a round
// of 1024 bits with up to 23 chains on 16 wavefronts 28 000 / 19 800 cycles.  Three kinds of units in the lanes throughout / in
// the walk (calls, us, components with tables 0/0, 1/1 and 0/1): 4096x4096 302 / 239, six of them 687 / 613, one 1600x1200
// image 292 / 231, 24 of them 406 / 300; with two kinds 239, 611, 232 and 308.

// lane i < upm describes data unit i of the MCU (walk_unit)
__device__ __forceinline__ uint32_t coop_unit_word(const ImgDesc& D, uint32_t lane) {
    return lane < D.upm ? walk_unit(D.walk, D.sched_comp, D.upm, lane) : 0u;
}

// Where the tables of the kinds of units lie: bytes of LDS, the same in every lane.
struct CoopTables {
    uint32_t dc0, ac0, dc1, ac1, dc2, ac2;
    bool three;  // kinds; with fewer, kind 2 repeats kind 0 and is not looked at
};
__device__ __forceinline__ CoopTables coop_tables(const ImgDesc& D, uint32_t tab) {
    const uint32_t w = __builtin_amdgcn_readfirstlane(D.walk), ndc = __builtin_amdgcn_readfirstlane(D.ndc);
    return CoopTables{walk_dc(w, 0u, tab), walk_ac(w, 0u, ndc, tab), walk_dc(w, 1u, tab), walk_ac(w, 1u, ndc, tab),
                      walk_dc(w, 2u, tab), walk_ac(w, 2u, ndc, tab), ((w >> kWalkThree) & 1u) != 0u};
}

// What the walk's instructions take for granted of an entry (sync_entry), beside what the lanes do.
static_assert(kSyncStep == 0x7E1Fu && kSyncEsc == 0x8000u && kSyncDcK == 9u && kSyncAcK == 10u && kAdvEob == 63u);
constexpr uint32_t bit_field(uint32_t at, uint32_t bits) { return (bits << 16) | at; }  // operand of s_bfe

// p, u, z: state of the chain, the same in every lane, advanced until p >= limit (limit a multiple of 64; a subsequence is
// a whole number of 64-bit windows, and a chain enters it at most 31 bits behind its start, so no window is wasted).
// words: byte of LDS at which the stream's word with the window of bit p begins, big-endian words; the walk looks at 24
// bytes behind the last window.  All 64 lanes are active.
// S = window position j (bits 0..6, at most 63 + 31) and zig-zag index z (bits 9..15, at most 63 + 63); adding an entry
// advances both.  Bit 6 set: the window is behind us; bit 15: the data unit is complete; an escape sets bit 15 or carries
// out of it, and its step is taken back.  The answers for the next window and the words of the one after that are asked for
// before the chain is followed through this one.  At the first escape of a kind of units in a window all lanes follow up
// their own at once.  Every step moves on by at least one bit.
// dc_a holds the sums of components 0 and 1 (two 16-bit fields, the lower one's sign taken off the upper one), dc_b
// that of component 2.  (Sums that leave 16 bits come out otherwise than from the lanes' loop in the components behind; the
// sums of a chain that is in step do so only where DC values leave the range of 8-bit samples, and the 15-bit fields
// of the lanes do not hold those either.)
// THREE: the image has three kinds of units (a component with a pair of tables of its own).
template <bool THREE>
__device__ __forceinline__ void coop_span_kinds(uint32_t& p_io, uint32_t& u_io, uint32_t& z_io, uint32_t& nb_out, int64_t& dc_out,
                                                uint32_t limit, uint32_t words, uint32_t unit_word, uint32_t upm,
                                                const CoopTables& ct) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t p = __builtin_amdgcn_readfirstlane(p_io), u = __builtin_amdgcn_readfirstlane(u_io);
    const uint32_t ws = p & ~63u;
    uint32_t S = (p - ws) | (__builtin_amdgcn_readfirstlane(z_io) << 9);
    uint32_t left = (limit - ws) >> 6;  // windows; at least one
    uint32_t nb = 0u, dc_a = 0u, dc_b = 0u;
    uint32_t cur = __builtin_amdgcn_readlane(unit_word, u);
    // the lane's 32 bits start behind the first 1 to 32 bits of two words
    uint32_t at = words + ((lane + 31u) >> 5) * 4u - 4u;
    const uint32_t shift = 0u - lane;
    uint32_t d0, d1, a0, a1, c0, c1, peek, nd0, nd1, na0, na1, npeek, x0, x1;
    uint32_t t, t2, r, r2, v;
    uint64_t all;
// AC symbols of a unit of one kind, eight in a row; an escape, the end of the unit, else that of the window
#define JPGD_WALK_AC(LOOP, EVENT, ESCAPE, C)                                                               \
    LOOP ":\n"                                                                                             \
    ".rept 8\n"                                                                                            \
    "v_readlane_b32 %[t], " C ", %[S]\n"                                                                   \
    "s_add_u32 %[S], %[S], %[t]\n"                                                                         \
    "s_and_b32 %[t2], %[S], 0x18040\n"                                                                     \
    "s_cbranch_scc1 " EVENT "f\n"                                                                          \
    ".endr\n"                                                                                              \
    "s_branch " LOOP "b\n"                                                                                 \
    EVENT ":\n"                                                                                            \
    "s_bitcmp1_b32 %[t], 15\n"                                                                             \
    "s_cbranch_scc1 " ESCAPE "f\n"                                                                         \
    "s_bitcmp1_b32 %[S], 15\n"
// the escapes of one kind's AC table, followed up in every lane that holds one; the step is taken again with what they lead to
#define JPGD_WALK_ESCAPE(ESCAPE, LOOP, A, C, OTHER_A, OTHER_C)                                             \
    ESCAPE ":\n"                                                                                           \
    "s_sub_u32 %[S], %[S], %[t]\n"                                                                         \
    "v_cmp_gt_i32 vcc, 0, " A "\n"                                                                         \
    "s_and_saveexec_b64 %[all], vcc\n"                                                                     \
    "v_bfe_u32 " C ", " A ", 6, 3\n"                                                                       \
    "v_sub_u32 " OTHER_C ", 23, " C "\n"                                                                   \
    "v_bfe_u32 " C ", %[peek], " OTHER_C ", " C "\n"                                                       \
    "v_lshrrev_b32 " A ", 15, " A "\n"                                                                     \
    "v_and_b32 " A ", 0xfff8, " A "\n"                                                                     \
    "v_lshl_add_u32 " A ", " C ", 2, " A "\n"                                                              \
    "ds_read_b32 " A ", " A "\n"                                                                           \
    "s_waitcnt lgkmcnt(0)\n"                                                                               \
    "s_mov_b64 exec, %[all]\n"                                                                             \
    "v_and_b32 " C ", 0xfe1f, " A "\n"                                                                     \
    "v_and_b32 " OTHER_C ", 0xfe1f, " OTHER_A "\n"                                                         \
    "s_nop 1\n"                                                                                            \
    "s_branch " LOOP "b\n"
// THIRD(text): text where there is a third kind
#define JPGD_WALK(THIRD)                                                                                   \
    "s_waitcnt lgkmcnt(0)\n"                                                                               \
    "ds_read_b32 %[x0], %[at]\n"                                                                           \
    "ds_read_b32 %[x1], %[at] offset:4\n"                                                                  \
    "s_bitset1_b32 %[left], 31\n"                                                                          \
    "s_waitcnt lgkmcnt(0)\n"                                                                               \
    "s_branch 2f\n"                                                                                        \
    /* the next window's answers become this one's */                                                      \
    "1:\n"                                                                                                 \
    "s_waitcnt lgkmcnt(0)\n"                                                                               \
    "v_mov_b32 %[peek], %[npeek]\n"                                                                        \
    "v_mov_b32 %[d0], %[nd0]\n"                                                                            \
    "v_mov_b32 %[d1], %[nd1]\n"                                                                            \
    "v_mov_b32 %[a0], %[na0]\n"                                                                            \
    "v_mov_b32 %[a1], %[na1]\n"                                                                            \
    THIRD("v_mov_b32 %[d2], %[nd2]\n"                                                                      \
          "v_mov_b32 %[a2], %[na2]\n"                                                                      \
          "v_and_b32 %[c2], 0xfe1f, %[na2]\n")                                                             \
    "v_and_b32 %[c0], 0xfe1f, %[na0]\n"                                                                    \
    "v_and_b32 %[c1], 0xfe1f, %[na1]\n"                                                                    \
    /* ask for those of the window behind it, and for the words of the one after that */                   \
    "2:\n"                                                                                                 \
    "v_alignbit_b32 %[npeek], %[x0], %[x1], %[shift]\n"                                                    \
    "v_lshrrev_b32 %[x0], 23, %[npeek]\n"                                                                  \
    "v_lshrrev_b32 %[x1], 22, %[npeek]\n"                                                                  \
    "v_lshl_add_u32 %[nd0], %[x0], 2, %[bd0]\n"                                                            \
    "v_lshl_add_u32 %[nd1], %[x0], 2, %[bd1]\n"                                                            \
    "v_lshl_add_u32 %[na0], %[x1], 2, %[ba0]\n"                                                            \
    "v_lshl_add_u32 %[na1], %[x1], 2, %[ba1]\n"                                                            \
    "ds_read_b32 %[nd0], %[nd0]\n"                                                                         \
    "ds_read_b32 %[nd1], %[nd1]\n"                                                                         \
    "ds_read_b32 %[na0], %[na0]\n"                                                                         \
    "ds_read_b32 %[na1], %[na1]\n"                                                                         \
    THIRD("v_lshl_add_u32 %[nd2], %[x0], 2, %[bd2]\n"                                                      \
          "v_lshl_add_u32 %[na2], %[x1], 2, %[ba2]\n"                                                      \
          "ds_read_b32 %[nd2], %[nd2]\n"                                                                   \
          "ds_read_b32 %[na2], %[na2]\n")                                                                  \
    "ds_read_b32 %[x0], %[at] offset:8\n"                                                                  \
    "ds_read_b32 %[x1], %[at] offset:12\n"                                                                 \
    "v_add_u32 %[at], 8, %[at]\n"                                                                          \
    "s_bitcmp1_b32 %[left], 31\n"   /* (the first time round there is no window to walk through yet) */    \
    "s_cbranch_scc0 3f\n"                                                                                  \
    "s_bitset0_b32 %[left], 31\n"                                                                          \
    "s_branch 1b\n"                                                                                        \
    "3:\n"                                                                                                 \
    "s_cmp_lt_u32 %[S], 0x200\n"                                                                           \
    "s_cbranch_scc1 20f\n"                                                                                 \
    THIRD("s_bitcmp1_b32 %[cur], %[kind] + 1\n"                                                            \
          "s_cbranch_scc1 41f\n")                                                                          \
    "s_bitcmp1_b32 %[cur], %[kind]\n"                                                                      \
    "s_cbranch_scc1 31f\n"                                                                                 \
    JPGD_WALK_AC("21", "22", "27", "%[c0]")                                                                \
    "s_cbranch_scc0 29f\n"                                                                                 \
    /* unit complete */                                                                                    \
    "23:\n"                                                                                                \
    "s_add_u32 %[nb], %[nb], 1\n"                                                                          \
    "s_and_b32 %[S], %[S], 0x7f\n"                                                                         \
    "s_and_b32 %[t], %[cur], 15\n"                                                                         \
    "s_bitcmp1_b32 %[S], 6\n"                                                                              \
    "v_readlane_b32 %[cur], %[uw], %[t]\n"                                                                 \
    "s_cbranch_scc1 29f\n"                                                                                 \
    /* DC symbol at position S (its zig-zag index is 0): entry of the table, its value, the component's sum */ \
    "20:\n"                                                                                                \
    "v_readlane_b32 %[r], %[d0], %[S]\n"                                                                   \
    "v_readlane_b32 %[r2], %[d1], %[S]\n"                                                                  \
    "v_readlane_b32 %[v], %[peek], %[S]\n"                                                                 \
    "s_bitcmp1_b32 %[cur], %[kind]\n"                                                                      \
    "s_cselect_b32 %[r], %[r2], %[r]\n"                                                                    \
    THIRD("v_readlane_b32 %[r2], %[d2], %[S]\n"                                                            \
          "s_bitcmp1_b32 %[cur], %[kind] + 1\n"                                                            \
          "s_cselect_b32 %[r], %[r2], %[r]\n")                                                             \
    "s_bitcmp1_b32 %[r], 31\n"                                                                             \
    "s_cbranch_scc1 28f\n"                                                                                 \
    "24:\n"                                                                                                \
    "s_and_b32 %[t], %[r], 31\n"                                                                           \
    "s_bfe_u32 %[r2], %[r], %[f_size]\n"                                                                   \
    "s_sub_u32 %[t], 32, %[t]\n"                                                                           \
    "s_lshl_b32 %[t2], %[r2], 16\n"                                                                        \
    "s_or_b32 %[t], %[t], %[t2]\n"                                                                         \
    "s_bfe_i32 %[v], %[v], %[t]\n"        /* the value's bits, signed (none: 0) */                         \
    "s_ashr_i32 %[t], %[v], 31\n"                                                                          \
    "s_lshl_b32 %[t2], -1, %[r2]\n"                                                                        \
    "s_xor_b32 %[t], %[t], %[t2]\n"                                                                        \
    "s_add_i32 %[v], %[v], %[t]\n"                                                                         \
    "s_add_i32 %[v], %[v], 1\n"           /* the difference, as in symbol_value */                         \
    "s_bfe_u32 %[t], %[cur], %[f_shift]\n"                                                                 \
    "s_lshl_b32 %[v], %[v], %[t]\n"                                                                        \
    "s_bitcmp1_b32 %[cur], %[b_second]\n"                                                                  \
    "s_cselect_b32 %[t], %[v], 0\n"                                                                        \
    "s_cselect_b32 %[v], 0, %[v]\n"                                                                        \
    "s_add_u32 %[dcb], %[dcb], %[t]\n"                                                                     \
    "s_add_u32 %[dca], %[dca], %[v]\n"                                                                     \
    "s_and_b32 %[r], %[r], 0x7e1f\n"                                                                       \
    "s_add_u32 %[S], %[S], %[r]\n"        /* the index becomes 1 (2 where no codeword starts) */             \
    "s_bitcmp1_b32 %[S], 6\n"                                                                              \
    "s_cbranch_scc1 29f\n"                                                                                 \
    THIRD("s_bitcmp1_b32 %[cur], %[kind] + 1\n"                                                            \
          "s_cbranch_scc1 41f\n")                                                                          \
    "s_bitcmp1_b32 %[cur], %[kind]\n"                                                                      \
    "s_cbranch_scc0 21b\n"                                                                                 \
    JPGD_WALK_AC("31", "32", "37", "%[c1]")                                                                \
    "s_cbranch_scc1 23b\n"                                                                                 \
    /* the window ends */                                                                                  \
    "29:\n"                                                                                                \
    "s_sub_u32 %[S], %[S], 64\n"          /* the same position, seen from the next window */               \
    "s_sub_u32 %[left], %[left], 1\n"                                                                      \
    "s_cmp_lg_u32 %[left], 0\n"                                                                            \
    "s_cbranch_scc1 1b\n"                                                                                  \
    "s_branch 40f\n"                                                                                       \
    THIRD(JPGD_WALK_AC("41", "42", "47", "%[c2]")                                                          \
          "s_cbranch_scc1 23b\n"                                                                           \
          "s_branch 29b\n"                                                                                 \
          JPGD_WALK_ESCAPE("47", "41", "%[a2]", "%[c2]", "%[a0]", "%[c0]"))                                \
    JPGD_WALK_ESCAPE("27", "21", "%[a0]", "%[c0]", "%[a1]", "%[c1]")                                       \
    JPGD_WALK_ESCAPE("37", "31", "%[a1]", "%[c1]", "%[a0]", "%[c0]")                                       \
    /* an escape of a DC table */                                                                          \
    "28:\n"                                                                                                \
    "s_bfe_u32 %[t], %[r], %[f_n]\n"                                                                       \
    "s_sub_u32 %[t2], 23, %[t]\n"                                                                          \
    "s_lshl_b32 %[t], %[t], 16\n"                                                                          \
    "s_or_b32 %[t], %[t], %[t2]\n"                                                                         \
    "s_bfe_u32 %[t], %[v], %[t]\n"                                                                         \
    "s_lshl_b32 %[t], %[t], 2\n"                                                                           \
    "s_lshr_b32 %[r], %[r], 15\n"                                                                          \
    "s_and_b32 %[r], %[r], 0xfff8\n"                                                                       \
    "s_add_u32 %[t], %[t], %[r]\n"                                                                         \
    "v_mov_b32 %[c0], %[t]\n"                                                                              \
    "ds_read_b32 %[c0], %[c0]\n"                                                                           \
    "s_waitcnt lgkmcnt(0)\n"                                                                               \
    "v_readfirstlane_b32 %[r], %[c0]\n"                                                                    \
    "v_and_b32 %[c0], 0xfe1f, %[a0]\n"                                                                     \
    "s_branch 24b\n"                                                                                       \
    "40:\n"                                                                                                \
    "s_waitcnt lgkmcnt(0)\n"
#define JPGD_WALK_RESULTS                                                                                  \
    [S] "+&s"(S), [cur] "+&s"(cur), [left] "+&s"(left), [nb] "+&s"(nb), [dca] "+&s"(dc_a), [dcb] "+&s"(dc_b), [at] "+&v"(at), \
        [d0] "=&v"(d0), [d1] "=&v"(d1), [a0] "=&v"(a0), [a1] "=&v"(a1), [c0] "=&v"(c0), [c1] "=&v"(c1), [peek] "=&v"(peek), \
        [nd0] "=&v"(nd0), [nd1] "=&v"(nd1), [na0] "=&v"(na0), [na1] "=&v"(na1), [npeek] "=&v"(npeek), [x0] "=&v"(x0), \
        [x1] "=&v"(x1), [t] "=&s"(t), [t2] "=&s"(t2), [r] "=&s"(r), [r2] "=&s"(r2), [v] "=&s"(v), [all] "=&s"(all)
#define JPGD_WALK_INPUTS                                                                                   \
    [shift] "v"(shift), [uw] "v"(unit_word), [bd0] "s"(ct.dc0), [ba0] "s"(ct.ac0), [bd1] "s"(ct.dc1), [ba1] "s"(ct.ac1), \
        [kind] "i"(kUwKind), [f_size] "i"(bit_field(20u, 4u)), [f_shift] "i"(bit_field(kUwShift, 5u)),    \
        [b_second] "i"(kUwSecond), [f_n] "i"(bit_field(6u, 3u))
#define JPGD_NO_THIRD(text)
#define JPGD_THIRD(text) text
    if constexpr (THREE) {
        uint32_t d2, a2, c2, nd2, na2;
        asm volatile(JPGD_WALK(JPGD_THIRD)
                     : JPGD_WALK_RESULTS, [d2] "=&v"(d2), [a2] "=&v"(a2), [c2] "=&v"(c2), [nd2] "=&v"(nd2), [na2] "=&v"(na2)
                     : JPGD_WALK_INPUTS, [bd2] "s"(ct.dc2), [ba2] "s"(ct.ac2)
                     : "vcc", "scc", "memory");
    } else {
        asm volatile(JPGD_WALK(JPGD_NO_THIRD) : JPGD_WALK_RESULTS : JPGD_WALK_INPUTS : "vcc", "scc", "memory");
    }
#undef JPGD_WALK_AC
#undef JPGD_WALK_ESCAPE
#undef JPGD_WALK
#undef JPGD_WALK_RESULTS
#undef JPGD_WALK_INPUTS
#undef JPGD_NO_THIRD
#undef JPGD_THIRD
    p_io = limit + (S & 0x7Fu);
    z_io = S >> 9;
    const uint32_t next = cur & 15u;  // of the unit the chain is in now
    u_io = next == 0u ? upm - 1u : next - 1u;
    nb_out = nb;
    const int32_t s0 = (int32_t)(int16_t)(dc_a & 0xFFFFu), s1 = (int32_t)(dc_a - (uint32_t)s0) >> 16;
    dc_out = (int64_t)s0 + ((int64_t)s1 << 15) + ((int64_t)(int32_t)dc_b << 30);
}
__device__ __forceinline__ void coop_span_sync(uint32_t& p, uint32_t& u, uint32_t& z, uint32_t& nb, int64_t& dc, uint32_t limit,
                                               uint32_t words, uint32_t unit_word, uint32_t upm, const CoopTables& ct) {
    if (__builtin_expect(ct.three, false)) coop_span_kinds<true>(p, u, z, nb, dc, limit, words, unit_word, upm, ct);
    else coop_span_kinds<false>(p, u, z, nb, dc, limit, words, unit_word, upm, ct);
}

// The words the walk reads, for kernels that do not keep the stream in LDS: those from the window of bit p on, copied to `buf`
// (kCoopBufWords words, the wavefront's own) by the whole wavefront.  Returns what coop_span_sync calls words.  cursors of
// `fetch` from nwords on are not read.
constexpr uint32_t kCoopBufWords = kMaxSubseqBits / 32u + 16u;
template <class Fetch>
__device__ __forceinline__ uint32_t coop_words(uint32_t* buf, uint32_t p, uint32_t limit, uint32_t org_word, uint32_t nwords, Fetch fetch) {
    const uint32_t w0 = ((p & ~63u) >> 5) - org_word, n = ((limit - (p & ~63u)) >> 5) + 7u;
    for (uint32_t k = threadIdx.x & 63u; k < n; k += 64u) buf[1u + k] = w0 + k < nwords ? fetch(w0 + k) : 0u;
    return lds_at(buf + 1);
}

// sync_span as the kernels run it (jpgd_lane.h has the same in C++, which says what every value is; the host tests hold that
// one to the plain lanes, the GPU's records are compared with the oracle's).
// In assembly, because of what a wavefront on its own on a SIMD pays for (measured, cycles): a vector instruction 4, also
// behind the one it depends on; a mask from a compare to a select 8 more, if nothing else stands between them; a scalar
// instruction on a mask 16 more; a taken branch 20; a read from LDS 64.  The compiler's loop takes three scalar
// instructions on fresh masks a step (a second symbol or none, unit complete or escape, lanes that are done), stalls for
// two selects and branches once: 300 cycles for 46 vector instructions.  Here other work stands behind every compare,
// lanes that are done leave through v_cmpx, one branch serves two steps, and whether a second symbol may be taken is a
// threshold worked out in the step before.
// Measured against the compiler's loop: 15360x8640 head 622 -> 573 us and tail 705 -> 661, eight calls of 1600x1200 160 ->
// 149, 1001x753 83 -> 77, 3001x2003 with restart intervals 91 -> 89; a lane round of 4096x4096 (L = 1024) 33.5k -> 28.3k
// cycles.
// Rules for whoever moves an instruction, here, in write_span_device and in the walk above.  The compiler does not look into the
// block, and nothing but these makes the results right:
//  * between a vector compare (or v_addc, v_mad_i64) and a vector instruction that reads the mask it wrote, VCC or a pair of
//    scalar registers, stand two instructions, or s_nop 1: without them the old mask may be read.  Scalar instructions and
//    branches on such a mask wait by themselves;
//  * between a vector instruction and a v_readlane of the register it wrote stands one; a v_readlane's lane never comes from a
//    scalar register that a vector instruction wrote;
//  * an LDS or memory instruction's address and 8 bytes of data may be overwritten right behind it, what it loads may be read
//    only behind a wait.  LDS answers in order, so lgkmcnt(n) waits until all but the last n requests are answered: the
//    order entry, word, row (and the store, in the tile) is what the counts count.  What the surrounding code has still
//    outstanding makes them wait longer, never less.  Instructions with no lane on count like others;
//  * v56..v63 are the block's own (clobbers): rows arrive in v60..v63, behind the row's wait and before the next request for
//    one v60 and v61 are free; nothing may be outstanding to any register when the block ends.
// `ahead` is asked for when the window may have moved on and looked at a step later.  STAGED: big-endian words in LDS; else
// the stream in memory, bytes swapped when the word is used.
template <bool STAGED>
__device__ __forceinline__ void sync_span_device(SyncLane& l, uint32_t limit, int64_t& dcacc, const uint32_t* words) {
    const uint32_t stop = limit + kSyncBias, last_pair = stop - kSyncPairBits;
    uint32_t pos = sync_at(l);
    if (pos >= stop) return;
    uint32_t threshold = pos < last_pair ? kSyncEsc : 0u, peek = sync_peek(l);
    const uint32_t keep = kSyncStep, carry = kSyncEsc;
    uint32_t t0, t1, t2, t3, t4, t5;
    uint64_t ends, esc, done, all;
    if (!STAGED) l.ahead = __builtin_bswap32(l.ahead);
    const uint64_t base = (uint64_t)(uintptr_t)words;  // (the same in every lane)
    const uint32_t base_hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)), base_lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
    const uint64_t from = ((uint64_t)base_hi << 32) | base_lo;
#define JPGD_STEP(WAIT_ENTRY, WAIT_AHEAD, AHEAD, LOAD_AHEAD)                                              \
    WAIT_ENTRY                                                                                             \
    "v_add_u32_sdwa %[t0], %[S], %[e] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n" \
    "v_and_b32_sdwa %[t1], %[second], %[e] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n" \
    "v_cmp_lt_u32 vcc, %[t0], %[thr]\n"        /* one symbol completes nothing and is not late */          \
    "v_bfe_u32 %[t2], %[e], 20, 4\n"           /* value bits of a DC symbol */                             \
    "v_sub_u32 %[t3], 0, %[e]\n"                                                                           \
    "v_cndmask_b32 %[t1], 0, %[t1], vcc\n"                                                                 \
    "v_bfe_i32 %[t3], %[peek], %[t3], %[t2]\n" /* they, signed */                                          \
    "v_add_u32 %[t0], %[t0], %[t1]\n"                                                                      \
    "v_bfe_u32 %[t4], %[e], 6, 3\n"            /* escape: bits of the subtable's index */                  \
    "v_and_b32 %[t1], 32, %[t0]\n"             /* the window moves on by a word */                         \
    "v_cmp_lt_u32 %[ends], %[top], %[t0]\n"                                                                \
    "v_cmp_ne_u32 vcc, 0, %[t1]\n"                                                                         \
    "v_cmp_gt_i32 %[esc], 0, %[e]\n"                                                                       \
    "v_not_b32 %[t5], %[t0]\n"                                                                             \
    WAIT_AHEAD                                                                                             \
    "v_cndmask_b32 %[hi], %[hi], %[lo], vcc\n"                                                             \
    "v_cndmask_b32 %[lo], %[lo], " AHEAD ", vcc\n"                                                         \
    "v_alignbit_b32 %[peek], %[hi], %[lo], %[t5]\n"                                                        \
    "v_sub_u32 v59, 23, %[t4]\n"                                                                           \
    "s_waitcnt lgkmcnt(0)\n"                                                                               \
    "v_cndmask_b32 %[t5], 22, 23, %[ends]\n"                                                               \
    "v_cndmask_b32 v60, v60, v61, %[ends]\n"   /* table of the next symbol */                              \
    "v_lshrrev_b32 v61, 15, %[e]\n"                                                                        \
    "v_lshrrev_b32 %[t5], %[t5], %[peek]\n"                                                                \
    "v_bfe_u32 %[t4], %[peek], v59, %[t4]\n"                                                               \
    "v_and_b32 v61, 0xfff8, v61\n"                                                                         \
    "v_lshl_add_u32 v60, %[t5], 2, v60\n"                                                                  \
    "v_lshl_add_u32 v61, %[t4], 2, v61\n"                                                                  \
    "v_cndmask_b32 v60, v60, v61, %[esc]\n"                                                                \
    "ds_read_b32 %[e], v60\n"                                                                              \
    "v_add_u32 %[at], %[at], %[t1]\n"                                                                      \
    "s_andn2_b64 %[done], %[ends], %[esc]\n"                                                               \
    "v_lshrrev_b32 v60, 3, %[at]\n"                                                                        \
    LOAD_AHEAD                                                                                             \
    "v_cndmask_b32 %[row], %[row], v63, %[done]\n"                                                         \
    "v_cndmask_b32 %[t4], v62, 0, %[esc]\n"                                                                \
    "ds_read_b128 v[60:63], %[row]\n"                                                                      \
    "v_cndmask_b32 %[t5], %[keep], 31, %[done]\n"                                                          \
    "v_and_b32 %[S], %[t5], %[t0]\n"                                                                       \
    "v_addc_co_u32 %[nb], vcc, 0, %[nb], %[done]\n"                                                        \
    "v_lshlrev_b32 %[t2], %[t2], -1\n"                                                                     \
    "v_ashrrev_i32 %[t1], 31, %[t3]\n"                                                                     \
    "v_and_or_b32 %[pos], %[S], 31, %[at]\n"                                                               \
    "v_xor_b32 %[t2], %[t2], %[t1]\n"                                                                      \
    "v_cmp_lt_u32 vcc, %[pos], %[last]\n"                                                                  \
    "v_add3_u32 %[t3], %[t3], %[t2], 1\n"      /* a DC symbol's value, else 0 */                           \
    "v_mad_i64_i32 %[dc], %[done], %[t3], %[t4], %[dc]\n"                                                  \
    "v_cndmask_b32 %[thr], 0, %[carry], vcc\n"                                                             \
    "v_cmpx_lt_u32 vcc, %[pos], %[stop]\n"
#define JPGD_SPAN_OPERANDS                                                                                 \
    [S] "+&v"(l.S), [row] "+&v"(l.row), [e] "+&v"(l.e), [hi] "+&v"(l.hi), [lo] "+&v"(l.lo), [ahead] "+&v"(l.ahead), [at] "+&v"(l.at), \
        [nb] "+&v"(l.nb), [dc] "+&v"(dcacc), [pos] "+&v"(pos), [thr] "+&v"(threshold), [peek] "+&v"(peek), [t0] "=&v"(t0),   \
        [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [t4] "=&v"(t4), [t5] "=&v"(t5), [ends] "=&s"(ends), [esc] "=&s"(esc), \
        [done] "=&s"(done), [all] "=&s"(all)                                                               \
        : [stop] "v"(stop), [last] "v"(last_pair), [keep] "v"(keep), [carry] "v"(carry), [second] "s"(kSyncSecond), \
          [top] "s"(kSyncEsc - 1u)
#define JPGD_SPAN_CLOBBERS "vcc", "scc", "memory", "v59", "v60", "v61", "v62", "v63"
    static_assert(sizeof(SyncRow) == 16 && kSyncDcK == 9u && kSyncAcK == 10u);
    if constexpr (STAGED) {
        asm volatile(
            "s_mov_b64 %[all], exec\n"
            "ds_read_b128 v[60:63], %[row]\n"
            "1:\n"
            // in the order they were asked for: entry, word, row
            JPGD_STEP("s_waitcnt lgkmcnt(2)\n", "s_waitcnt lgkmcnt(1)\n", "%[ahead]", "ds_read_b32 %[ahead], v60\n")
            JPGD_STEP("s_waitcnt lgkmcnt(2)\n", "s_waitcnt lgkmcnt(1)\n", "%[ahead]", "ds_read_b32 %[ahead], v60\n")
            "s_cbranch_execnz 1b\n"
            "s_mov_b64 exec, %[all]\n"
            "s_waitcnt lgkmcnt(0)\n"
            : JPGD_SPAN_OPERANDS
            : JPGD_SPAN_CLOBBERS);
    } else {
        asm volatile(
            "s_mov_b64 %[all], exec\n"
            "ds_read_b128 v[60:63], %[row]\n"
            "1:\n"
            JPGD_STEP("s_waitcnt lgkmcnt(1)\n", "s_waitcnt vmcnt(0)\nv_perm_b32 %[ahead], %[ahead], %[ahead], %[swap]\n", "%[ahead]",
                      "global_load_dword %[ahead], v60, %[words]\n")
            JPGD_STEP("s_waitcnt lgkmcnt(1)\n", "s_waitcnt vmcnt(0)\nv_perm_b32 %[ahead], %[ahead], %[ahead], %[swap]\n", "%[ahead]",
                      "global_load_dword %[ahead], v60, %[words]\n")
            "s_cbranch_execnz 1b\n"
            "s_mov_b64 exec, %[all]\n"
            "s_waitcnt vmcnt(0) lgkmcnt(0)\n"
            "v_perm_b32 %[ahead], %[ahead], %[ahead], %[swap]\n"
            : JPGD_SPAN_OPERANDS, [words] "s"(from), [swap] "s"(0x00010203u)
            : JPGD_SPAN_CLOBBERS);
    }
#undef JPGD_STEP
#undef JPGD_SPAN_OPERANDS
#undef JPGD_SPAN_CLOBBERS
}

// write_span (jpgd_lane.h, which says what every value is) as the kernels run it in workgroups that see no start of a restart
// interval; in assembly for the reasons given at sync_span_device.  Entry and first predictor change places
// from one step to the next, so that neither has to be copied; lanes without a value are switched off for the store instead of
// branched around.  Kernel with the compiler's loop / with this one (us): batch of 256 87 / 68, 4096x4096 86 / 66, 15360x8640
// 368 / 320, 48 frames of 1920x1088 (bound by its stores) 158 / 149, 1920x1088 17 / 14, 256x256 gray 20 / 16.5.  A step takes
// some 400 cycles with a wavefront or two to a SIMD, 66 vector instructions.
// Memory: chunk_value, from `out` on, which is where slot0 goes.  A first loop runs until no lane is left in a chunk that it
// shares with the lane before; the second need not look for it.
// Tile: every value goes to its place in LDS on its own.  first: place of slot0 there, tile_n: slots there are room for.
// l.unit in, l.s, l.unit and l.seen out.
template <bool TILE>
__device__ __forceinline__ void write_span_device(WriteLane& l, uint32_t limit, uint32_t total_units, uint32_t slot0, uint32_t first,
                                                  uint32_t tile_n, const int16_t* out, WriteChunk& c) {
    const uint32_t stop = limit + kSyncBias;
    uint32_t pos = sync_at(l.s);
    if (pos >= stop || l.unit >= total_units) return;
    // slot of a symbol: the unit's first one, less one, from slot0 on (below zero in a unit that began before it), plus the
    // symbol's last zig-zag index plus one
    const uint32_t unit0 = l.unit;
    uint32_t unit = l.unit * 64u - slot0 - 1u;
    const uint32_t unit_end = min(total_units * 64u - slot0 - 1u, 0x7FFFFFFFu), unit_now = unit;
    const uint32_t keep = kSyncStep;
    uint32_t t0, t1, t2, t3, t4, t5, e2 = 0u, q0 = 0u;
    uint64_t ends, esc, done, other, run, all;
    const uint64_t base = (uint64_t)(uintptr_t)out;  // (the same in every lane)
    const uint32_t base_hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)), base_lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
    const uint64_t to = ((uint64_t)base_hi << 32) | base_lo;
    static_assert(sizeof(SyncRow) == 16 && kSyncDcK == 9u && kSyncAcK == 10u && kWriteValue == 0x40000000 && kWriteDc == 0x60000000);
#define JPGD_STEP(E, NEXT, P, PNEXT, W1, W2, W3, STORE)                                                    \
    "s_waitcnt lgkmcnt(" W1 ")\n"              /* the entry */                                             \
    "v_add_u32_sdwa %[t0], %[S], " E " dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n" \
    "v_bfe_u32 %[t2], " E ", 20, 4\n"                                                                      \
    "v_sub_u32 %[t3], 0, " E "\n"                                                                          \
    "v_and_b32 %[t1], 32, %[t0]\n"                                                                         \
    "v_bfe_i32 %[t3], %[peek], %[t3], %[t2]\n" /* value bits, signed */                                    \
    "v_cmp_ne_u32 vcc, 0, %[t1]\n"                                                                         \
    "v_cmp_lt_u32 %[ends], %[top], %[t0]\n"                                                                \
    "v_cmp_gt_i32 %[esc], 0, " E "\n"                                                                      \
    "v_not_b32 %[t5], %[t0]\n"                                                                             \
    "v_bfe_u32 %[t4], " E ", 6, 3\n"                                                                       \
    "s_waitcnt lgkmcnt(" W2 ")\n"              /* the word */                                              \
    "v_cndmask_b32 %[hi], %[hi], %[lo], vcc\n"                                                             \
    "v_cndmask_b32 %[lo], %[lo], %[ahead], vcc\n"                                                          \
    "v_alignbit_b32 %[peek], %[hi], %[lo], %[t5]\n"                                                        \
    "v_sub_u32 v59, 23, %[t4]\n"                                                                           \
    "s_waitcnt lgkmcnt(" W3 ")\n"              /* the row */                                               \
    "v_cndmask_b32 %[t5], 22, 23, %[ends]\n"                                                               \
    "v_cndmask_b32 v60, v60, v61, %[ends]\n"                                                               \
    "v_lshrrev_b32 v61, 15, " E "\n"                                                                       \
    "v_lshrrev_b32 %[t5], %[t5], %[peek]\n"                                                                \
    "v_bfe_u32 %[t4], %[peek], v59, %[t4]\n"                                                               \
    "v_and_b32 v61, 0xfff8, v61\n"                                                                         \
    "v_lshl_add_u32 v60, %[t5], 2, v60\n"                                                                  \
    "v_lshl_add_u32 v61, %[t4], 2, v61\n"                                                                  \
    "v_cndmask_b32 v60, v60, v61, %[esc]\n"                                                                \
    "ds_read_b32 " NEXT ", v60\n"                                                                          \
    "v_add_u32 %[at], %[at], %[t1]\n"                                                                      \
    "s_andn2_b64 %[done], %[ends], %[esc]\n"                                                               \
    "v_lshrrev_b32 v60, 3, %[at]\n"                                                                        \
    "ds_read_b32 %[ahead], v60\n"                                                                          \
    "v_cndmask_b32 %[row], %[row], v63, %[done]\n"                                                         \
    "v_cmp_ne_u32 %[other], 0, v62\n"                                                                      \
    "ds_read_b128 v[60:63], %[row]\n"                                                                      \
    "v_cndmask_b32 %[t5], %[keep], 31, %[done]\n"                                                          \
    "v_lshlrev_b32 %[t2], %[t2], -1\n"                                                                     \
    "v_ashrrev_i32 v59, 31, %[t3]\n"                                                                       \
    "v_and_b32 %[S], %[t5], %[t0]\n"                                                                       \
    "v_xor_b32 %[t2], %[t2], v59\n"                                                                        \
    "s_and_b64 %[other], %[other], %[done]\n" /* the next unit is another component's */                   \
    "v_cmp_le_i32 vcc, 0x60000000, " E "\n"   /* a DC value */                                             \
    "v_add3_u32 %[t3], %[t3], %[t2], 1\n"     /* the value */                                              \
    "v_lshrrev_b32 %[t5], 9, %[t0]\n"                                                                      \
    "v_add_u32 %[t4], " P ", %[t3]\n"                                                                      \
    "v_add_u32 %[t5], %[unit], %[t5]\n"       /* its slot */                                               \
    "v_cndmask_b32_sdwa v58, %[t3], %[t4], vcc dst_sel:WORD_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD\n" \
    "v_cndmask_b32 %[t4], " P ", %[t4], vcc\n"                                                             \
    "v_cndmask_b32 %[t1], 0, 64, %[done]\n"                                                                \
    "v_add_u32 %[unit], %[unit], %[t1]\n"                                                                  \
    "v_add_u32 %[t1], %[late], %[t0]\n"                                                                    \
    "v_cndmask_b32 " PNEXT ", %[t4], %[p1], %[other]\n"                                                    \
    "v_cndmask_b32 %[p1], %[p1], %[p2], %[other]\n"                                                        \
    "v_cndmask_b32 %[p2], %[p2], %[t4], %[other]\n"                                                        \
    "v_and_or_b32 %[seen], " E ", %[t1], %[seen]\n"                                                        \
    "v_and_or_b32 %[pos], %[S], 31, %[at]\n"                                                               \
    STORE(E)                                                                                               \
    "s_mov_b64 exec, %[run]\n"                                                                             \
    "v_cmpx_lt_i32 vcc, %[unit], %[unit_end]\n"                                                            \
    "v_cmpx_lt_u32 %[run], %[pos], %[stop]\n"
// (lanes that have no value are switched off)
#define JPGD_TO_TILE(E)                                                                                    \
    "v_lshl_add_u32 %[t1], %[t5], 1, %[first]\n"                                                           \
    "v_cmpx_le_i32 vcc, 0x40000000, " E "\n"                                                               \
    "v_cmpx_gt_u32 vcc, %[room], %[t5]\n"                                                                  \
    "v_cmpx_gt_u32 vcc, %[beyond], %[t0]\n"                                                                \
    "ds_write_b16 %[t1], v58\n"
// (done: lanes with a value, those among them that move on to another chunk store the one they leave, or keep it)
#define JPGD_CHUNK(E, FIRST)                                                                               \
    "v_cmpx_le_i32 vcc, 0x40000000, " E "\n"                                                               \
    "v_lshlrev_b32 %[t4], 4, %[t5]\n"                                                                      \
    "v_cmpx_gt_u32 %[done], %[beyond], %[t0]\n"                                                            \
    "v_mov_b32 v59, 0\n"                                                                                   \
    "v_and_b32 %[t5], -4, %[t5]\n"                                                                         \
    "v_lshlrev_b32 %[t1], 1, %[cur]\n"                                                                     \
    "v_lshlrev_b64 v[58:59], %[t4], v[58:59]\n"                                                            \
    "v_cmpx_ne_u32 %[other], %[t5], %[cur]\n"                                                              \
    FIRST                                                                                                  \
    "global_store_dwordx2 %[t1], v[56:57], %[to]\n"                                                        \
    "s_mov_b64 exec, %[other]\n"                                                                           \
    "v_mov_b32 %[cur], %[t5]\n"                                                                            \
    "v_mov_b32 v56, 0\n"                                                                                   \
    "v_mov_b32 v57, 0\n"                                                                                   \
    "s_mov_b64 exec, %[done]\n"                                                                            \
    "v_or_b32 v56, v56, v58\n"                                                                             \
    "v_or_b32 v57, v57, v59\n"
#define JPGD_TO_MEMORY(E) JPGD_CHUNK(E, "")
#define JPGD_TO_MEMORY_FIRST(E)                                                                            \
    JPGD_CHUNK(E, "v_cmp_ne_u32 vcc, %[cur], %[shared]\n"                                                  \
                  "s_nop 1\n"                                                                              \
                  "v_cndmask_b32 %[f0], v56, %[f0], vcc\n"                                                 \
                  "v_cndmask_b32 %[f1], v57, %[f1], vcc\n"                                                 \
                  "v_cmpx_ne_u32 vcc, %[cur], %[shared]\n")
#define JPGD_WRITE_OPERANDS                                                                                \
    [S] "+&v"(l.s.S), [row] "+&v"(l.s.row), [e] "+&v"(l.s.e), [e2] "+&v"(e2), [hi] "+&v"(l.s.hi), [lo] "+&v"(l.s.lo),     \
        [ahead] "+&v"(l.s.ahead), [at] "+&v"(l.s.at), [peek] "+&v"(l.peek), [unit] "+&v"(unit), [p0] "+&v"(l.p0),         \
        [q0] "+&v"(q0), [p1] "+&v"(l.p1), [p2] "+&v"(l.p2), [seen] "+&v"(l.seen), [pos] "+&v"(pos), [t0] "=&v"(t0),       \
        [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [t4] "=&v"(t4), [t5] "=&v"(t5), [ends] "=&s"(ends),               \
        [esc] "=&s"(esc), [done] "=&s"(done), [other] "=&s"(other), [run] "=&s"(run), [all] "=&s"(all)
#define JPGD_WRITE_INPUTS                                                                                  \
    [stop] "v"(stop), [keep] "v"(keep), [unit_end] "v"(unit_end), [top] "s"(kSyncEsc - 1u),           \
        [beyond] "s"(65u << 9), [late] "s"(kWriteNoCode + kWriteInside - (65u << 9))
#define JPGD_WRITE_CLOBBERS "vcc", "scc", "memory", "v58", "v59", "v60", "v61", "v62", "v63"
    if constexpr (TILE) {
        // in the order they were asked for: entry, word, row, and the store of the step before
        asm volatile(
            "s_mov_b64 %[all], exec\n"
            "s_mov_b64 %[run], exec\n"
            "ds_read_b128 v[60:63], %[row]\n"
            "s_waitcnt lgkmcnt(0)\n"
            "1:\n"
            JPGD_STEP("%[e]", "%[e2]", "%[p0]", "%[q0]", "3", "2", "1", JPGD_TO_TILE)
            JPGD_STEP("%[e2]", "%[e]", "%[q0]", "%[p0]", "3", "2", "1", JPGD_TO_TILE)
            "s_cbranch_execnz 1b\n"
            "s_mov_b64 exec, %[all]\n"
            "s_waitcnt lgkmcnt(0)\n"
            : JPGD_WRITE_OPERANDS
            : JPGD_WRITE_INPUTS, [first] "v"(first), [room] "v"(tile_n)
            : JPGD_WRITE_CLOBBERS);
    } else {
        uint32_t a0 = (uint32_t)c.acc, a1 = (uint32_t)(c.acc >> 32), f0 = (uint32_t)c.first, f1 = (uint32_t)(c.first >> 32);
        asm volatile(
            "s_mov_b64 %[all], exec\n"
            "s_mov_b64 %[run], exec\n"
            "v_mov_b32 v56, %[a0]\n"
            "v_mov_b32 v57, %[a1]\n"
            "ds_read_b128 v[60:63], %[row]\n"
            "1:\n"
            JPGD_STEP("%[e]", "%[e2]", "%[p0]", "%[q0]", "2", "1", "0", JPGD_TO_MEMORY_FIRST)
            JPGD_STEP("%[e2]", "%[e]", "%[q0]", "%[p0]", "2", "1", "0", JPGD_TO_MEMORY_FIRST)
            "v_cmp_eq_u32 vcc, %[cur], %[shared]\n"   /* (none where no lane is left) */
            "s_cbranch_vccnz 1b\n"
            "s_cbranch_execz 3f\n"
            "2:\n"
            JPGD_STEP("%[e]", "%[e2]", "%[p0]", "%[q0]", "2", "1", "0", JPGD_TO_MEMORY)
            JPGD_STEP("%[e2]", "%[e]", "%[q0]", "%[p0]", "2", "1", "0", JPGD_TO_MEMORY)
            "s_cbranch_execnz 2b\n"
            "3:\n"
            "s_mov_b64 exec, %[all]\n"
            "v_mov_b32 %[a0], v56\n"
            "v_mov_b32 %[a1], v57\n"
            "s_waitcnt lgkmcnt(0)\n"
            : JPGD_WRITE_OPERANDS, [cur] "+&v"(c.cur), [a0] "+&v"(a0), [a1] "+&v"(a1), [f0] "+&v"(f0), [f1] "+&v"(f1)
            : JPGD_WRITE_INPUTS, [to] "s"(to), [shared] "v"(c.shared)
            : JPGD_WRITE_CLOBBERS, "v56", "v57");
        c.acc = ((uint64_t)a1 << 32) | a0;
        c.first = ((uint64_t)f1 << 32) | f0;
    }
    l.unit = unit0 + ((unit - unit_now) >> 6);
#undef JPGD_STEP
#undef JPGD_TO_TILE
#undef JPGD_CHUNK
#undef JPGD_TO_MEMORY
#undef JPGD_TO_MEMORY_FIRST
#undef JPGD_WRITE_OPERANDS
#undef JPGD_WRITE_INPUTS
#undef JPGD_WRITE_CLOBBERS
}

// Part k of n of an image's coefficients is cleared by `lanes` lanes of a workgroup, this one being number `lane`.
__device__ __forceinline__ void clear_coefficients(const Params& P, const ImgDesc& D, uint32_t k, uint32_t n, uint32_t lane, uint32_t lanes) {
    const uint32_t u0 = (uint32_t)((uint64_t)D.total_units * k / n), u1 = (uint32_t)((uint64_t)D.total_units * (k + 1u) / n);
    uint4* out = reinterpret_cast<uint4*>(P.coef + D.coef_off + (size_t)u0 * 64u);
    const uint32_t n16 = (u1 - u0) * 8u;
    for (uint32_t j = lane; j < n16; j += lanes) out[j] = make_uint4(0u, 0u, 0u, 0u);
}

// ---- synchronisation, intra-sequence (paper, Algorithm 3, first loop) --------------------------------
// Workgroup w of an image covers the kWG subsequences base .. base+kWG-1, base = w*seq_len - overlap, and
// publishes the records of the last seq_len of them; the first `overlap` lanes only warm the chain up.

// The workgroup's stretch of the stream is copied to LDS first, but in the second kernel below.
// RST: the call has images with restart intervals.  Calls without get a kernel with none of that code in it (the
// intra-sequence kernel was measured 3 % slower on plain streams with it: registers and code layout).
// PHASE: kSyncAll = the whole of it in one kernel.  For calls with many more sequences than the chip holds at a time
// the work is split in two kernels.  kSyncHead is the same code up to the round in which at most P.handoff chains
// are still running; it leaves the records of all its lanes and the list of those chains in memory.  kSyncTail picks
// them up and runs the remaining rounds with the lanes reading the stream from memory (a handful of chains, each
// reading its words once).  The late rounds are chains of dependent symbols in a single wavefront or in one
// wavefront per chain, and what keeps the chip busy then is the number of sequences in flight: without the staged
// stream a workgroup needs a third of the LDS, and a CU holds eight of them instead of three.
constexpr int kSyncAll = 0, kSyncHead = 1, kSyncTail = 2;
constexpr uint32_t kHandWords = 4u * kWG;  // per sequence: 3 x kWG record words, the chains, in the last word their number
constexpr uint32_t kSyncFixedWords = 7u * kWG / 2u;  // of LDS: records and chains
constexpr uint32_t kSyncPadWords = 12u;   // behind the stream in LDS: what lanes, and the walk of a whole wavefront, look at
static_assert(kHandoff < kWG, "chains and their number in kWG words");
template <bool RST, int PHASE>
__device__ __forceinline__ void sync_intra_body(const Params& P) {
    constexpr bool STAGED = PHASE != kSyncTail;  // the second kernel reads the stream from memory
    static_assert(STAGED || !RST, "the second kernel has no room for a bitmap of interval starts");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    const uint32_t wg = blockIdx.x;
    const uint32_t ii = find_image(P, wg, &ImgDesc::seq0);
    const ImgDesc D = image_desc(P, ii);
    const uint32_t nsub = P.st[ii].nsub;
    const int32_t base = (int32_t)((wg - D.seq0) * P.seq_len) - (int32_t)P.overlap;
    if (base >= (int32_t)nsub || (int32_t)((wg - D.seq0) * P.seq_len) >= (int32_t)nsub) return;  // nothing owned

    // A record: the state after the subsequence (16 bits, pack_state), completed units (15 bits) and "an interval began"
    // (bit 31), the DC sums of components 0 and 1, that of component 2.
    static_assert(kMaxSubseqBits / 2u + 1u < 1u << 15, "a unit takes two symbols, of one bit at least; the first may have begun before the subsequence");
    uint32_t* rec = reinterpret_cast<uint32_t*>(lds_raw + P.tab_bytes);
    uint32_t* pdc01 = rec + kWG;
    uint16_t* pdc2 = reinterpret_cast<uint16_t*>(pdc01 + kWG);
    // chains on their way to another lane or wavefront: state before the target subsequence, target subsequence << 16
    uint32_t* mv = reinterpret_cast<uint32_t*>(pdc2 + kWG);
    static_assert(kSyncFixedWords == 2u * kWG + kWG / 2u + kWG, "what lies between the tables and the stream");
    uint32_t* strm = mv + kWG;
    __shared__ uint32_t scratch[8];

    const uint32_t L = 1u << P.logL, wps = L >> 5;  // words per subsequence
    const uint32_t first = base < 0 ? 0u : (uint32_t)base;
    const uint32_t t0 = (uint32_t)((int32_t)first - base);                  // first lane with a subsequence
    const uint32_t t1 = min((uint32_t)kWG, (uint32_t)((int32_t)nsub - base));  // one past the last such lane
    const uint32_t first_word = first * wps;
    const uint32_t nwords = (t1 - t0) * wps + 4u;
    __shared__ SyncRow rows_s[8];
    __shared__ uint32_t dc_fill;
    if (threadIdx.x == 0u) dc_fill = 0u;
    stage_rows<false>(D, rows_s, lds_at(lds_raw));
    __syncthreads();
    stage_tables<false>(P, D, lds_raw, &dc_fill);
    if (STAGED) stage_stream(P.stream + D.stream_off, first_word, nwords, strm);
    // scans with restart intervals: the bitmap of interval starts, for the bytes staged above
    uint32_t* bm_s = strm + kWG * wps + kSyncPadWords;
    const uint32_t bm_k0 = first_word >> 3;
    uint32_t seen = 0u;
    const bool bm_lds = (1u << P.logL) <= (uint32_t)kBitmapLdsMaxL;
    const uint32_t* bmap_img = P.bmap + D.bmap_off;
    if (RST && D.restart) seen = stage_bitmap(bmap_img, first_word, nwords, bm_s, bm_lds);
    auto bword = [&](uint32_t k) { return bm_lds ? bm_s[k - bm_k0] : bmap_img[k]; };
    bool restart = false;
    if (RST) restart = __syncthreads_or(seen != 0u) != 0;
    else __syncthreads();  // staged tables and stream are complete

    // The write pass only stores values that are not zero: the coefficients are cleared here, a sequence's share of them
    // by each workgroup (calls of moderate size, kClearAheadBytes): this kernel waits for chains of dependent symbols and leaves the memory idle, and the wavefronts
    // that are only here for single chains have nothing else to do yet.  Where the write pass cleared its own stretch, all
    // its workgroups did so first and waited for it: 24 images of 2047x1535 50 000 of 160 000 cycles a workgroup, batch of
    // 256 20 000 of 190 000, 4963x7013 gray 13 000 of 50 000.  (No barrier waits for these stores.)
    if (PHASE != kSyncTail && P.clear) {
        const uint32_t lanes0 = blockDim.x > (uint32_t)kWG ? (uint32_t)kWG : 0u;
        if (threadIdx.x >= lanes0)
            clear_coefficients(P, D, wg - D.seq0, (nsub + P.seq_len - 1u) / P.seq_len, threadIdx.x - lanes0, blockDim.x - lanes0);
    }

    const uint32_t* gwords = reinterpret_cast<const uint32_t*>(P.stream + D.stream_off) + first_word;
    // cursor = word index inside the workgroup's window
    auto fetch = [&](uint32_t c) { return STAGED ? strm[c] : __builtin_bswap32(gwords[c]); };
    // The lanes' bits count from the start of LDS, or of the stretch in memory: position in the image's stream plus org.
    const uint32_t org = (STAGED ? 8u * lds_at(strm) : 0u) - (first_word << 5);
    auto word = [&](uint32_t b) { return STAGED ? lds_word(b >> 3) : __builtin_bswap32(gwords[b >> 5]); };
    auto tab = [&](uint32_t k) { return lds_word(k); };
    const uint32_t row0 = lds_at(rows_s);
    auto rows = [&](uint32_t k) { return lds_row(k); };
    const uint32_t t = threadIdx.x;
    const bool valid = t >= t0 && t < t1;
    SyncLane l;
    l.nb = 0u;
    uint32_t* handed = P.seq_rec + (size_t)wg * kHandWords;
    bool active = false;
    uint32_t tt = t + 1u;
    uint32_t waves_used = kWG / 64u;
    // bit of the stream at which subsequence k of the workgroup starts
    auto start_of = [&](uint32_t k) { return (uint32_t)(base + (int32_t)k) << P.logL; };
    // chain and target as one word, and back
    auto state_of = [&](uint32_t end) { return pack_state(sync_pos(l) - org - end, (l.S >> 9) & 63u, (l.row - row0) / (uint32_t)sizeof(SyncRow)); };
    auto take_chain = [&](uint32_t m) {
        tt = m >> 16;
        sync_start(l, start_of(tt) + state_prel(m) + org, state_u(m), state_z(m), D.upm, row0, word, tab, rows);
    };
    auto span = [&](SyncLane& a, uint32_t to, int64_t& dc) { sync_span_device<STAGED>(a, to, dc, gwords); };
    auto decode_rst = [&](SyncLane& a, uint32_t limit, int64_t& dc, uint32_t& crossed) {
        sync_span_rst(a, limit + org, dc, crossed, org, [&](uint32_t p) { sync_start(a, p, 0u, 0u, D.upm, row0, word, tab, rows); },
                      [&](uint32_t to) { span(a, to, dc); }, bword);
    };
    auto decode = [&](SyncLane& a, uint32_t limit, int64_t& dc, uint32_t& crossed) {
        if (restart) decode_rst(a, limit, dc, crossed);
        else span(a, limit + org, dc);
    };
    auto put_record = [&](uint32_t k, uint32_t x, uint32_t units, uint32_t crossed, int64_t dc) {
        rec[k] = x | (units << 16) | (crossed << 31);
        pdc01[k] = pack_dc01(dc);
        pdc2[k] = (uint16_t)pack_dc2(dc);
    };
    if (PHASE == kSyncTail) {
        // the records the first kernel left, and the chains that were still running
        if (valid) {
            rec[t] = handed[t];
            pdc01[t] = handed[kWG + t];
            pdc2[t] = (uint16_t)handed[2 * kWG + t];
        }
        const uint32_t n = handed[4u * kWG - 1u];
        active = t < n;
        if (active) take_chain(handed[3u * kWG + t]);
        waves_used = (n + 63u) >> 6; if (waves_used == 0u) waves_used = 1u;
    } else if (valid) {
        const uint32_t limit = start_of(t + 1u);
        sync_start(l, start_of(t) + org, 0u, 0u, D.upm, row0, word, tab, rows);
        uint32_t crossed = 0u;
        int64_t dcacc = 0;
        decode(l, limit, dcacc, crossed);
        put_record(t, state_of(limit), l.nb, crossed, dcacc);
        active = t + 1u < t1;
    }
    // Overflow rounds: in round r the chain that started at subsequence c decodes subsequence c+r from its own
    // state and compares with the record left there one round earlier by the chain that started at c+1.
    // Chains drop out as they synchronise.  The chains still running are packed into the lowest lanes whenever
    // that frees a whole wavefront: a chain is (p, u, z, target), everything else is rebuilt from the staged
    // stream, so moving one costs two LDS words.  Between packings a round costs one barrier: the count of
    // running chains goes through one LDS word per wavefront, double-buffered by the parity of the round.
    // In a workgroup that sees restart intervals a chain may fall back to a single lane for a round (below): at most one chain per wavefront then, so that
    // such rounds never take longer than the packed ones they replace.
    const uint32_t coop_max = restart ? min(P.coop_max, P.sync_waves) : P.coop_max;
    uint32_t coop_n = 0u;
    for (uint32_t round = 0u;; ++round) {
        const uint64_t bal = __ballot(active);
        uint32_t* cnt = scratch + ((round & 1u) << 2);
        if ((t & 63u) == 0u && t < (uint32_t)kWG) cnt[t >> 6] = (uint32_t)__popcll(bal);
        __syncthreads();  // also orders the records written in the previous round before their readers
        const uint32_t c0 = cnt[0], c1 = cnt[1], c2 = cnt[2], c3 = cnt[3];
        const uint32_t now = c0 + c1 + c2 + c3;
        if (PHASE == kSyncHead && now <= P.handoff) {  // the rest is the second kernel's
            const uint32_t wave = t >> 6;
            const uint32_t before = wave == 0u ? 0u : wave == 1u ? c0 : wave == 2u ? c0 + c1 : c0 + c1 + c2;
            const uint32_t rank = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (active) handed[3u * kWG + rank] = state_of(start_of(tt)) | (tt << 16);
            if (t == 0u) handed[4u * kWG - 1u] = now;
            if (valid) {
                handed[t] = rec[t];
                handed[kWG + t] = pdc01[t];
                handed[2 * kWG + t] = pdc2[t];
            }
            return;
        }
        if (now == 0u) break;
        if (now <= coop_max) {  // few chains left: hand them to whole wavefronts (below)
            const uint32_t wave = t >> 6;
            const uint32_t before = wave == 0u ? 0u : wave == 1u ? c0 : wave == 2u ? c0 + c1 : c0 + c1 + c2;
            const uint32_t rank = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (active) mv[rank] = state_of(start_of(tt)) | (tt << 16);
            coop_n = now;
            __syncthreads();
            break;
        }
        if (((now + 63u) >> 6) < waves_used) {
            const uint32_t wave = t >> 6;
            const uint32_t before = wave == 0u ? 0u : wave == 1u ? c0 : wave == 2u ? c0 + c1 : c0 + c1 + c2;
            const uint32_t rank = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (active) mv[rank] = state_of(start_of(tt)) | (tt << 16);
            __syncthreads();
            active = t < now;
            if (active) take_chain(mv[t]);
            waves_used = (now + 63u) >> 6;
        }
        if (active) {
            l.nb = 0u;
            int64_t dcacc = 0;
            const uint32_t limit = start_of(tt + 1u);
            uint32_t crossed = 0u;
            decode(l, limit, dcacc, crossed);
            const uint32_t x = state_of(limit);
            const bool synced = x == (rec[tt] & 0xFFFFu);
            put_record(tt, x, l.nb, crossed, dcacc);
            ++tt;
            active = !synced && tt < t1;
        }
    }
    // The same rounds with one chain per wavefront.  The chains keep their slot k < coop_n in a list held twice
    // (read from one copy, written to the other, swapped every round; kCoopDone once a chain has
    // synchronised or reached the end of the sequence).  Every wavefront reads the whole list and takes the
    // running chains whose rank among them is its own number modulo the number of wavefronts (the four that hold
    // the lanes and the ones that are only here for this), so the work stays spread as chains drop out;
    // wavefront 0 carries the finished slots over.  One barrier per round.
    if (coop_n) {
        constexpr uint32_t kCoopDone = 0xFFFFFFFFu;
        // the compiler cannot know that these are the same in every lane (they come from the image descriptor and
        // the thread index); saying so keeps the chain's state in scalar registers
        const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63u;
        const uint32_t u_n = __builtin_amdgcn_readfirstlane(coop_n), u_t1 = __builtin_amdgcn_readfirstlane(t1);
        const uint32_t u_org = __builtin_amdgcn_readfirstlane(org);
        const uint32_t u_upm = __builtin_amdgcn_readfirstlane(D.upm);
        const CoopTables ct = coop_tables(D, lds_at(lds_raw));
        const uint32_t u_waves = P.sync_waves;  // a power of two
        const int32_t u_base = (int32_t)__builtin_amdgcn_readfirstlane((uint32_t)base);
        const uint32_t unit_word = coop_unit_word(D, lane);
        for (uint32_t par = 0u;; par ^= 1u) {
            const uint32_t rd = par << 6, wr = (par ^ 1u) << 6;
            const uint32_t mine = lane < u_n ? mv[rd + lane] : kCoopDone;
            const uint64_t running = __ballot(mine != kCoopDone);
            if (running == 0ull) break;
            if (wave == 0u && lane < u_n && mine == kCoopDone) mv[wr + lane] = kCoopDone;
            uint32_t rank = 0u;
            for (uint64_t m = running; m; m &= m - 1ull, ++rank) {
                if ((rank & (u_waves - 1u)) != wave) continue;
                const uint32_t k = (uint32_t)__ffsll((long long)m) - 1u;
                const uint32_t ms = __builtin_amdgcn_readfirstlane(mv[rd + k]);
                const uint32_t ctt = ms >> 16;
                uint32_t cu = state_u(ms), cz = state_z(ms), cnb = 0u;
                uint32_t cp = ((uint32_t)(u_base + (int32_t)ctt) << P.logL) + state_prel(ms);
                int64_t cdc = 0;
                const uint32_t limit = (uint32_t)(u_base + (int32_t)ctt + 1) << P.logL;
                // The wavefront's decoder does not know the rules of restart intervals.  A chain whose stretch holds
                // no interval start does not need them (sync_span_rst is sync_span then); one whose
                // stretch does is decoded by a single lane for this round.
                uint32_t crossed = 0u;
                uint32_t B = kNoBoundary;
                if (restart) B = __builtin_amdgcn_readfirstlane(next_boundary(cp, limit + 64u, bword));
                if (B == kNoBoundary) {
                    const uint32_t at = STAGED ? (u_org + (cp & ~63u)) >> 3 : coop_words(strm + wave * kCoopBufWords, cp, limit, first_word, nwords, fetch);
                    coop_span_sync(cp, cu, cz, cnb, cdc, limit, __builtin_amdgcn_readfirstlane(at), unit_word, u_upm, ct);
                } else {
                    if (lane == 0u) {
                        SyncLane cl;
                        cl.nb = 0u;
                        sync_start(cl, cp + org, cu, cz, D.upm, row0, word, tab, rows);
                        decode_rst(cl, limit, cdc, crossed);
                        cp = sync_pos(cl) - org; cu = (cl.row - row0) / (uint32_t)sizeof(SyncRow); cz = (cl.S >> 9) & 63u; cnb = cl.nb;
                    }
                    cp = __builtin_amdgcn_readfirstlane(cp);
                    cu = __builtin_amdgcn_readfirstlane(cu);
                    cz = __builtin_amdgcn_readfirstlane(cz);
                    cnb = __builtin_amdgcn_readfirstlane(cnb);
                    crossed = __builtin_amdgcn_readfirstlane(crossed);
                    const uint32_t dlo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)cdc);
                    const uint32_t dhi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)cdc >> 32));
                    cdc = (int64_t)(((uint64_t)dhi << 32) | (uint64_t)dlo);
                }
                const uint32_t x = pack_state(cp - limit, cz, cu);
                const bool synced = x == (rec[ctt] & 0xFFFFu);
                if (lane == 0u) {
                    put_record(ctt, x, cnb, crossed, cdc);
                    mv[wr + k] = (synced || ctt + 1u >= u_t1) ? kCoopDone : ((ctt + 1u) << 16) | x;
                }
            }
            __syncthreads();
        }
    }
    SInfo pub = {0u, 0u, 0u, 0u};
    const bool own = valid && t >= P.overlap;
    const uint32_t own_i = (uint32_t)(base + (int32_t)t);
    if (own) {
        pub.x = rec[t] & 0xFFFFu; pub.y = (rec[t] >> 16 & 0x7FFFu) | (rec[t] & 0x80000000u); pub.z = pdc01[t]; pub.w = pdc2[t];
        P.sinfo[D.sub0 + own_i] = pub;
    }
    // The sums of the published records go to the totals of the (at most two) groups they belong to.  A kernel of its
    // own that reads the records again for this costs every call 4.5 microseconds.
    if (!RST && t < (uint32_t)kWG) {
        const uint32_t g0 = ((wg - D.seq0) * P.seq_len) >> 8;
        static_assert(kWG == 256, "groups of 256 records");
        const Seg all = wave_incl_sums(seg_of_record(pub));
        const bool two = own && (own_i >> 8) != g0;
        const bool any_two = __ballot(two) != 0ull;
        Seg second = seg_zero();
        if (any_two) second = wave_incl_sums(two ? seg_of_record(pub) : seg_zero());
        if ((t & 63u) == 63u) {
            add_group_total(P.grp_tot + D.grp0 + g0, seg_minus(all, second));
            if (any_two) add_group_total(P.grp_tot + D.grp0 + g0 + 1u, second);
        }
    }
    // The published records continue the state the last warm-up lane ended in.  If the previous sequence ends
    // in that very state, the two sequences already form one chain and the inter-sequence kernel has nothing
    // to decode at this boundary.
    if (t == 0u) P.warm_x[wg] = (P.overlap > 0u && P.overlap - 1u >= t0) ? rec[P.overlap - 1u] & 0xFFFFu : 0xFFFFFFFFu;
}

template <bool RST>
__global__ __launch_bounds__(64 * kSyncWavesMax) void k_sync_intra(Params P) {
    sync_intra_body<RST, kSyncAll>(P);
}
// (calls with restart intervals are not split)
__global__ __launch_bounds__(kWG) void k_sync_head(Params P) {
    sync_intra_body<false, kSyncHead>(P);
}
__global__ __launch_bounds__(kWG) void k_sync_tail(Params P) {
    sync_intra_body<false, kSyncTail>(P);
}

// ---- synchronisation, inter-sequence (paper, Algorithm 3, second loop) ------------------------------
// One lane per sequence boundary: continue from the last record of sequence b into sequence b+1 until
// the state equals the recorded one or the sequence ends.  One wave64 per workgroup.

__global__ __launch_bounds__(64) void k_sync_inter(Params P) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    const uint32_t wg = blockIdx.x;
    const uint32_t ii = find_image(P, wg, &ImgDesc::bnd0);
    const ImgDesc D = image_desc(P, ii);
    const uint32_t nsub = P.st[ii].nsub;
    const uint32_t b = (wg - D.bnd0) * 64u + threadIdx.x;
    const uint64_t gfirst = (uint64_t)(b + 1u) * P.seq_len;
    SInfo* rec = P.sinfo + D.sub0;
    uint32_t* warm = P.warm_x + D.seq0 + b + 1u;  // of the sequence that starts at this boundary
    // nothing to do where the sequence behind the boundary already continues the state the one before ends in
    uint32_t g = 0u, x0 = 0u;
    bool work = false;
    // The state words of records at a boundary are read here while the lane of the boundary before may be rewriting
    // them (and read again by check_boundaries, in the write or the totals kernel, which opens another round if the two
    // did not agree): single 32-bit accesses, marked as such, with the rest of a record written before its state word.
    if (gfirst < nsub) {
        g = (uint32_t)gfirst;
        x0 = __atomic_load_n(&rec[g - 1u].x, __ATOMIC_RELAXED);
        work = *warm != x0;
    }
    if (!__syncthreads_or(work)) return;
    __shared__ SyncRow rows_s[8];
    __shared__ uint32_t dc_fill;
    if (threadIdx.x == 0u) dc_fill = 0u;
    stage_rows<false>(D, rows_s, lds_at(lds_raw));
    __syncthreads();
    stage_tables<false>(P, D, lds_raw, &dc_fill);
    __syncthreads();
    const uint32_t* words = reinterpret_cast<const uint32_t*>(P.stream + D.stream_off);
    auto fetch = [&](uint32_t w) { return __builtin_bswap32(words[w]); };
    auto word = [&](uint32_t b) { return __builtin_bswap32(words[b >> 5]); };
    auto tab = [&](uint32_t k) { return lds_word(k); };
    const uint32_t row0 = lds_at(rows_s);
    auto rows = [&](uint32_t k) { return lds_row(k); };
    // Usually a handful of boundaries in a whole image have something to decode, and the kernel lasts as long as
    // the slowest of them.  With few in this workgroup, each is walked by the whole wavefront, one after the other
    // (same results as the lane's loop below; the wavefront's decoder does not know restart intervals).
    const uint64_t workers = __ballot(work);
    if (!D.restart && __popcll(workers) <= kInterCoopMax) {
        const uint32_t lane = threadIdx.x;
        const uint32_t unit_word = coop_unit_word(D, lane);
        const uint32_t u_upm = __builtin_amdgcn_readfirstlane(D.upm);
        const CoopTables ct = coop_tables(D, lds_at(lds_raw));
        __shared__ uint32_t buf[kCoopBufWords];
        const uint32_t u_nsub = __builtin_amdgcn_readfirstlane(nsub);
        const uint32_t u_nwords = (u_nsub << (P.logL - 5u)) + 4u;
        for (uint64_t m = workers; m; m &= m - 1ull) {
            const uint32_t k = (uint32_t)__ffsll((long long)m) - 1u;
            uint32_t cg = __builtin_amdgcn_readlane(g, k);
            const uint32_t cx0 = __builtin_amdgcn_readlane(x0, k);
            const uint32_t cend = min(u_nsub, cg + P.seq_len);
            uint32_t cp = (cg << P.logL) + state_prel(cx0), cz = state_z(cx0), cu = state_u(cx0);
            bool first = true;
            for (;;) {
                uint32_t cnb = 0u;
                int64_t cdc = 0;
                const uint32_t limit = (cg + 1u) << P.logL;
                coop_span_sync(cp, cu, cz, cnb, cdc, limit, coop_words(buf, cp, limit, 0u, u_nwords, fetch), unit_word, u_upm, ct);
                const uint32_t x = pack_state(cp - limit, cz, cu);
                const bool synced = x == __atomic_load_n(&rec[cg].x, __ATOMIC_RELAXED);
                if (lane == 0u) {
                    if (first && !synced) atomicAdd(&P.status->inter_changed, 1u);
                    const SInfo now = {x, cnb, pack_dc01(cdc), pack_dc2(cdc)};
                    if (P.fold) add_group_total(P.grp_tot + D.grp0 + (cg >> 8), seg_minus(seg_of_record(now), seg_of_record(rec[cg])));
                    rec[cg].y = now.y;
                    rec[cg].z = now.z;
                    rec[cg].w = now.w;
                    __atomic_store_n(&rec[cg].x, x, __ATOMIC_RELAXED);
                }
                first = false;
                ++cg;
                if (synced || cg >= cend) break;
            }
        }
        if (work) *warm = x0;
        return;
    }
    if (!work) return;
    const uint32_t gend = min(nsub, g + P.seq_len);
    const uint32_t* bmap_img = P.bmap + D.bmap_off;
    auto bword = [&](uint32_t k) { return bmap_img[k]; };
    SyncLane l;
    sync_start(l, (g << P.logL) + state_prel(x0), state_u(x0), state_z(x0), D.upm, row0, word, tab, rows);
    bool first = true;
    for (;;) {
        l.nb = 0u;
        int64_t dcacc = 0;
        const uint32_t limit = (g + 1u) << P.logL;
        uint32_t crossed = 0u;
        auto span = [&](uint32_t to) { sync_span_device<false>(l, to, dcacc, words); };
        if (D.restart)
            sync_span_rst(l, limit, dcacc, crossed, 0u, [&](uint32_t p) { sync_start(l, p, 0u, 0u, D.upm, row0, word, tab, rows); }, span, bword);
        else span(limit);
        SInfo r;
        r.x = pack_state(sync_pos(l) - limit, (l.S >> 9) & 63u, (l.row - row0) / (uint32_t)sizeof(SyncRow));
        r.y = l.nb | (crossed << 31);
        r.z = pack_dc01(dcacc);
        r.w = pack_dc2(dcacc);
        const bool synced = r.x == __atomic_load_n(&rec[g].x, __ATOMIC_RELAXED);
        if (first && !synced) atomicAdd(&P.status->inter_changed, 1u);
        first = false;
        if (P.fold) add_group_total(P.grp_tot + D.grp0 + (g >> 8), seg_minus(seg_of_record(r), seg_of_record(rec[g])));
        rec[g].y = r.y;
        rec[g].z = r.z;
        rec[g].w = r.w;
        __atomic_store_n(&rec[g].x, r.x, __ATOMIC_RELAXED);
        ++g;
        if (synced || g >= gend) break;
    }
    *warm = x0;  // the sequence's records now continue this state
}

// ---- exclusive scan over s_info (paper, Algorithm 1: prefix sum on s_info.n) ---------------------------
// Level 1: totals of each group of kWG records.  Level 2: one workgroup per image scans the image's
// group totals.  Level 3 (inside the write kernel): scan within the group.

__global__ __launch_bounds__(kWG) void k_group_totals(Params P) {
    __shared__ uint32_t scratch[20];
    const uint32_t wg = blockIdx.x;
    const uint32_t ii = find_image(P, wg, &ImgDesc::grp0);
    const ImgDesc D = image_desc_uniform(P, ii);
    const uint32_t nsub = P.st[ii].nsub;
    const uint32_t i = (wg - D.grp0) * kWG + threadIdx.x;
    SInfo r = {0u, 0u, 0u, 0u};
    if (i < nsub) r = P.sinfo[D.sub0 + i];
    Seg tot;
    if (D.restart == 0u) {
        const Seg inc = wave_incl_sums(seg_of_record(r));
        if ((threadIdx.x & 63u) == 63u) put_sums(scratch + (threadIdx.x >> 6) * 4u, inc);
        __syncthreads();
        tot = seg_join(seg_join(get_sums(scratch), get_sums(scratch + 4)), seg_join(get_sums(scratch + 8), get_sums(scratch + 12)));
    } else {
        wg_excl_segscan(seg_of_record(r), scratch, &tot);
    }
    if (threadIdx.x == 0) P.grp_tot[wg] = seg_pack(tot);
    check_boundaries(P, D, wg - D.grp0, nsub);
}

// one workgroup per image: exclusive prefix of the group totals
__global__ __launch_bounds__(kWG) void k_group_scan(Params P) {
    __shared__ uint32_t scratch[20];
    const uint32_t ii = blockIdx.x;
    const ImgDesc D = image_desc_uniform(P, ii);
    if (D.ngrp_max <= (uint32_t)kSumMax) return;  // (the write kernel sums the totals itself)
    const uint32_t ngrp = (P.st[ii].nsub + kWG - 1u) / kWG;
    // as in k_unstuff_scan: a run of consecutive groups per lane, one scan over the 256 joined runs
    const int4* tot = P.grp_tot + D.grp0;
    int4* pref = P.grp_pref + D.grp0;
    const uint32_t per = (ngrp + (uint32_t)kWG - 1u) / (uint32_t)kWG;
    const uint32_t k0 = min(threadIdx.x * per, ngrp), k1 = min(k0 + per, ngrp);
    Seg run = seg_zero();
    for (uint32_t k = k0; k < k1; ++k) run = seg_join(run, seg_unpack(tot[k]));
    Seg all;
    Seg ex = wg_excl_segscan(run, scratch, &all);
    for (uint32_t k = k0; k < k1; ++k) {
        pref[k] = seg_pack(ex);
        ex = seg_join(ex, seg_unpack(tot[k]));
    }
}

// further rounds: what the write pass left from states that were not settled goes before it runs again
__global__ __launch_bounds__(kWG) void k_clear_coefficients(Params P) {
    const uint32_t ii = find_image(P, blockIdx.x, &ImgDesc::grp0);
    const ImgDesc D = image_desc_uniform(P, ii);
    clear_coefficients(P, D, blockIdx.x - D.grp0, D.ngrp_max, threadIdx.x, kWG);
}

// ---- write pass (paper, Algorithm 1 last loop; Algorithm 2 with write = true) ---------------------------

// TILE: calls of few workgroups and without restart intervals (kTileMaxGroups).  Where the coefficients a workgroup covers
// fit P.tile_bytes of LDS they are gathered there, value by value, and leave as full lines at the end: such a call
// waits for its slowest lane, and a lane that only stores into LDS takes a quarter fewer instructions per symbol;
// nothing is cleared in memory beforehand.
template <bool TILE>
__global__ __launch_bounds__(kWG) void k_write(Params P) {
    constexpr bool RST = !TILE;  // (a variant without the restart code, as for k_sync_intra, was measured 2 % slower)
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    __shared__ uint32_t scratch[36];
    const uint32_t wg = blockIdx.x;
    const uint32_t ii = find_image(P, wg, &ImgDesc::grp0);
    const ImgDesc D = image_desc_uniform(P, ii);
    const uint32_t nsub = P.st[ii].nsub;
    const uint32_t lg = wg - D.grp0;
    const uint32_t i0 = lg * kWG;
    if (i0 >= nsub) return;
    uint32_t* strm = reinterpret_cast<uint32_t*>(lds_raw + P.tab_bytes);

    const uint32_t L = 1u << P.logL, wps = L >> 5;
    const uint32_t nloc = min((uint32_t)kWG, nsub - i0);
    const uint32_t first_word = i0 * wps;
    const uint32_t nwords = nloc * wps + 4u;
    __shared__ SyncRow rows_s[8];
    __shared__ uint32_t dc_fill;
    if (threadIdx.x == 0u) dc_fill = 0u;
    stage_rows<true>(D, rows_s, lds_at(lds_raw));
    // the lane's record, its predecessor's state and the totals of the groups before this one are asked for
    // first: their way from memory overlaps the staging below
    const uint32_t t = threadIdx.x;
    const uint32_t i = i0 + t;
    const bool valid = t < nloc;
    const SInfo* rec = P.sinfo + D.sub0;
    SInfo mine = {0u, 0u, 0u, 0u};
    uint32_t xprev = 0u;
    if (valid) {
        mine = rec[i];
        if (i > 0u) xprev = rec[i - 1u].x;
    }
    const bool few_groups = D.ngrp_max <= (uint32_t)kSumMax;
    int4 before = make_int4(0, 0, 0, 0), more[kSumRun - 1];  // totals of a run of consecutive groups per lane
    const uint32_t per = (lg + (uint32_t)kWG - 1u) / (uint32_t)kWG;
    if (few_groups) {
        if (t * per < lg) before = P.grp_tot[D.grp0 + t * per];
        if (per > 1u) {
#pragma unroll
            for (uint32_t k = 1; k < (uint32_t)kSumRun; ++k) {
                more[k - 1u] = make_int4(0, 0, 0, 0);
                if (k < per && t * per + k < lg) more[k - 1u] = P.grp_tot[D.grp0 + t * per + k];
            }
        }
    } else {
        before = P.grp_pref[wg];
    }
    stage_stream(P.stream + D.stream_off, first_word, nwords, strm);
    __syncthreads();
    stage_tables<true>(P, D, lds_raw, &dc_fill);
    uint32_t* bm_s = strm + kWG * wps + 4u;
    const uint32_t bm_k0 = first_word >> 3;
    uint32_t seen = 0u;
    const bool bm_lds = (1u << P.logL) <= (uint32_t)kBitmapLdsMaxL;
    const uint32_t* bmap_img = P.bmap + D.bmap_off;
    if (RST && D.restart) seen = stage_bitmap(bmap_img, first_word, nwords, bm_s, bm_lds);
    auto bword = [&](uint32_t k) { return bm_lds ? bm_s[k - bm_k0] : bmap_img[k]; };
    bool restart = false;  // interval starts in this group's stretch of the stream?

    // position of this lane's first data unit and its DC predictors: exclusive scan inside the group
    // plus the group's prefix.  Both sums of a scan without restart intervals take lane-to-lane moves and the barrier
    // that ends the staging; the segmented join of the others takes four more barriers.  The states the group's first
    // subsequence starts from and its last one ends in travel the same way.
    Seg gp = seg_zero(), grp_tot = seg_zero(), ex = seg_zero(), run = seg_zero();
    const uint32_t wave = t >> 6;
    if (few_groups) {
        run = seg_unpack(before);
        if (per > 1u) {
#pragma unroll
            for (uint32_t k = 1; k < (uint32_t)kSumRun; ++k) run = seg_join(run, seg_unpack(more[k - 1u]));
        }
    }
    if (t == 0u) scratch[32] = xprev;
    if (t == nloc - 1u) scratch[33] = mine.x;
    if (D.restart == 0u) {
        const Seg inc = wave_incl_sums(seg_of_record(mine));
        const Seg bef = few_groups ? wave_incl_sums(run) : seg_zero();
        if ((t & 63u) == 63u) {
            put_sums(scratch + wave * 8u, inc);
            put_sums(scratch + wave * 8u + 4u, bef);
        }
        __syncthreads();
        Seg carry = seg_zero();
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const Seg s = get_sums(scratch + k * 8u);
            if (k < wave) carry = seg_join(carry, s);
            grp_tot = seg_join(grp_tot, s);
            gp = seg_join(gp, get_sums(scratch + k * 8u + 4u));
        }
        if (!few_groups) gp = seg_unpack(before);
        const Seg own = seg_of_record(mine);
        ex = seg_join(gp, carry);
        ex.units += inc.units - own.units;
        ex.d0 += inc.d0 - own.d0; ex.d1 += inc.d1 - own.d1; ex.d2 += inc.d2 - own.d2;
    } else {
        restart = __syncthreads_or(seen != 0u) != 0;
        if (few_groups) wg_excl_segscan(run, scratch, &gp);  // (zero, the identity of the join, where nothing is left)
        else gp = seg_unpack(before);
        ex = seg_join(gp, wg_excl_segscan(seg_of_record(mine), scratch, &grp_tot));
    }
    const uint32_t grp_units = grp_tot.units;
    uint32_t unit = ex.units;
    int32_t pred0 = (int32_t)ex.d0, pred1 = (int32_t)ex.d1, pred2 = (int32_t)ex.d2;

    // The group's slots: from where its first subsequence takes over (data unit and zig-zag index) to where the next
    // group's does; the last group goes on to the end of the image.  The ranges of the groups tile the image, and a lane
    // only stores inside its group's range.
    const uint64_t end_all = (uint64_t)D.total_units * 64u;
    const uint32_t x_in = scratch[32], x_out = scratch[33];
    uint64_t a = (uint64_t)gp.units * 64u + state_z(x_in);
    uint64_t b = i0 + nloc >= nsub ? end_all : ((uint64_t)gp.units + grp_units) * 64u + state_z(x_out);
    if (i0 == 0u) a = 0u;
    if (b > end_all) b = end_all;
    const uint64_t tile_a = a & ~(uint64_t)7u;  // first slot of the tile: a 16-byte word of the output
    const bool tiled = TILE && a < b && (b - tile_a) * 2u <= P.tile_bytes;
    uint4* const tile16 = reinterpret_cast<uint4*>(lds_raw + P.tile_off);
    const uint32_t tile_n = tiled ? (uint32_t)(b - tile_a) : 0u;  // slots
    if (tiled) {
        for (uint32_t k = t; k < (tile_n + 7u) >> 3; k += kWG) tile16[k] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    } else if (!P.clear) {
        if (a < b) {
            int16_t* c0 = P.coef + D.coef_off;
            uint64_t a8 = (a + 7u) & ~(uint64_t)7u;
            if (a8 > b) a8 = b;
            const uint64_t b8 = a8 + ((b - a8) & ~(uint64_t)7u);
            if (a + t < a8) c0[a + t] = 0;
            if (b8 + t < b) c0[b8 + t] = 0;
            uint4* body = reinterpret_cast<uint4*>(c0 + a8);
            const uint32_t n16 = (uint32_t)((b8 - a8) >> 3);
            const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
            for (uint32_t k = t; k < n16; k += kWG) body[k] = zero;
        }
        __syncthreads();  // the cleared range is in place
    }
    if (!tiled && !valid) return;

    // The lanes' bits: as in the synchronisation kernels.
    const uint32_t org = 8u * lds_at(strm) - (first_word << 5);
    auto word = [&](uint32_t b) { return lds_word(b >> 3); };
    auto tab = [&](uint32_t k) { return lds_word(k); };
    const uint32_t row0 = lds_at(rows_s);
    auto rows = [&](uint32_t k) { return lds_row(k); };
    int16_t* coef = P.coef + D.coef_off;
    // Slots are counted from the unit the group takes over in: none of its lanes starts before that.
    const uint32_t grp_slot = __builtin_amdgcn_readfirstlane(gp.units * 64u);
    int16_t* const grp_coef = coef + (size_t)grp_slot;
    WriteChunk chunk = chunk_start(unit * 64u + state_z(xprev) - grp_slot);
    auto store = [&](uint32_t k, uint32_t at, int16_t v) {
        chunk_value(chunk, k * 64u + at - grp_slot, v, [&](uint32_t slot, uint64_t a) { *reinterpret_cast<uint64_t*>(grp_coef + (size_t)slot) = a; });
    };
    WriteLane l;
    l.unit = unit;
    l.seen = 0u;
    const uint32_t u_in = state_u(xprev);
    write_predictors(l, (D.sched_comp >> (4u * u_in)) & 15u, (int32_t)(int16_t)pred0, (int32_t)(int16_t)pred1, (int32_t)(int16_t)pred2);
    auto start = [&]() { write_start(l, (i << P.logL) + state_prel(xprev) + org, u_in, state_z(xprev), D.upm, row0, word, tab, rows); };
    uint32_t flags = 0u;
    const uint32_t total = D.total_units;
    // unit modulo the 1, 3, 4 or 6 units of an MCU
    const uint32_t unit3 = (D.upm == 6u ? unit >> 1 : unit) % 3u;
    const uint32_t in_mcu = D.upm == 1u ? 0u : D.upm == 4u ? unit & 3u : D.upm == 3u ? unit3 : unit3 * 2u + (unit & 1u);
    if (unit < total && in_mcu != u_in) flags |= kStUnit;
    const uint32_t limit = (i + 1u) << P.logL;
    if (TILE && tiled) {
        if (valid && unit < total) {
            start();
            // (a damaged stream may leave the tile's range)
            write_span_device<true>(l, limit + org, total, (uint32_t)tile_a, lds_at(tile16), tile_n, nullptr, chunk);
        }
        __syncthreads();
        // the first and the last word are shared with the neighbouring workgroups
        const uint32_t lead = (uint32_t)(a - tile_a);
        uint4* out16 = reinterpret_cast<uint4*>(coef + tile_a);
        for (uint32_t k = (lead ? 1u : 0u) + t; k < tile_n >> 3; k += kWG) out16[k] = tile16[k];
        if (t < 16u) {
            const uint32_t slot = t < 8u ? t : (tile_n & ~7u) + (t & 7u);
            const bool mine = t < 8u ? (lead != 0u && slot >= lead && slot < tile_n) : (slot < tile_n && (tile_n >= 8u || lead == 0u));
            if (mine) coef[tile_a + slot] = reinterpret_cast<const int16_t*>(tile16)[slot];
        }
        if (!valid) return;
    } else if (unit < total) {
        start();
        if (restart) write_span_rst(l, limit + org, total, D.restart * D.upm, org, D.upm, row0, word, tab, rows, store, bword, &flags);
        else write_span_device<false>(l, limit + org, total, grp_slot, 0u, 0u, grp_coef, chunk);
    }
    // (in a workgroup with nothing to decode the lane stays where it was: behind the last unit)
    unit = l.unit;
    const uint32_t z_out = unit < total ? (l.s.S >> 9) & 63u : 0u;
    if (l.seen & kWriteBad) flags |= kStInvalid;
    if (!tiled) chunk_ends(chunk, [&](uint32_t slot, int16_t v) { grp_coef[slot] = v; });
    // all restart markers must have been there (the first lane of the image speaks for it)
    if (RST && D.restart && i == 0u && P.st[ii].markers != D.nint - 1u) flags |= kStInvalid;
    if (P.fold) check_boundaries(P, D, lg, nsub);
    // every lane checks the chain: unless the image is complete it must end in the recorded state
    if (unit < total) {
        const uint32_t p = sync_pos(l.s) - org;
        if (p < limit || pack_state(p - limit, z_out, (l.s.row - row0) / (uint32_t)sizeof(SyncRow)) != mine.x) flags |= kStMismatch;
        if (i == nsub - 1u) flags |= kStShort;
    }
    if (flags) atomicOr(&P.status->flags, flags);
}

// ---- pixels: de-zigzag, dequantise, 8x8 IDCT, level shift, chroma replication, YCbCr -> RGB -------------
// (paper, Section 4.3; the colour steps are not in the paper).  A workgroup takes runs of consecutive
// MCUs of one MCU row, kPixBlocks data units at most, transforms their columns in LDS and their rows on the way out, and
// writes the pixel rectangle they cover with row-contiguous stores.  Its rate depends on the wavefronts in flight: eight
// per SIMD with at most 64 registers (48 frames of 1920x1088 4:4:4, one run per workgroup: 307 us with 49 registers, 549
// with 93).

// Floats per data unit in LDS: 8 rows of 9 (one pad per row) and three more.  The phases ask for different strides (the
// columns for 72, under which 64 lanes meet 64 banks; the output loops, whose lanes hold the same row of neighbouring
// units, for an odd one), so it is a compromise, measured for 72 / 73 / 74 / 75 / 77: 48 frames of 1920x1088 4:4:4 223 /
// 228 / 224 / 219 / 228 us, batch of 256 63.9 / 68.0 / 66.4 / 64.6 / 70.0, 15360x8640 174 / 177 / 177 / 176 / 180.
constexpr int kBlkStride = 75;
__device__ __constant__ uint8_t c_zigzag[64] = JPGD_ZIGZAG_LITERAL;

// One row of a data unit behind the column pass: its eight samples, level shift applied.
__device__ __forceinline__ void row_samples(const float* b, float (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = b[e];
    v[0] += kLevelShiftDc;  // the level shift of +128 on all eight outputs, as one addition to the row's DC term
    idct8(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]);
}

// ONCE (pass_caches): the coefficients, read for the last time here, and the pixels pass by the caches' replacement order
// (non-temporal), so that they do not push each other out half used.  Measured on 48 frames of 1920x1088
// 4:4:4 (903 MB): 260 -> 225 us, 4.0 TB/s (reads alone 238, and the write pass of the next call slower; stores alone
// 265), the call 538 -> 488; 15360x8640 187 -> 177.  Gray and planar rows, eight bytes to a store, keep the ordinary
// ones (3001x2003 4:2:2 planes 13.8 / 14.6).
typedef uint32_t words4 __attribute__((ext_vector_type(4)));
typedef uint32_t words4_u __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t words2_u __attribute__((ext_vector_type(2), aligned(1)));
template <bool ONCE>
__device__ __forceinline__ uint4 load_coef(const uint4* p) {
    if constexpr (!ONCE) return *p;
    const words4 v = __builtin_nontemporal_load(reinterpret_cast<const words4*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// The first nbytes (at most 4 * NW) bytes of w.  Full groups leave as wide stores at any alignment.
template <int NW, bool ONCE>
__device__ __forceinline__ void put_bytes(uint8_t* dst, const uint32_t (&w)[NW], uint32_t nbytes) {
    if (nbytes == 4u * NW) {
        if constexpr (NW == 6 && ONCE) {
            __builtin_nontemporal_store(words4_u{w[0], w[1], w[2], w[3]}, reinterpret_cast<words4_u*>(dst));
            __builtin_nontemporal_store(words2_u{w[4], w[5]}, reinterpret_cast<words2_u*>(dst + 16));
        } else {
            __builtin_memcpy(dst, w, 4 * NW);
        }
        return;
    }
#pragma unroll
    for (uint32_t e = 0; e < 4u * NW; ++e)
        if (e < nbytes) dst[e] = (uint8_t)(w[e >> 2] >> (8u * (e & 3u)));
}

template <bool ONCE>
__global__ __launch_bounds__(kWG) void k_pixels(Params P) {
    __shared__ float blk[kPixBlocks * kBlkStride];
    __shared__ __attribute__((aligned(16))) float qf[3 * 64];
    uint32_t t = threadIdx.x;
    // The write kernel is complete when this kernel starts: its verdict goes to the waiting host from here, which
    // saves the dispatch of a kernel that would do nothing else.
    if (blockIdx.x == 0u && t == 0u && P.verdict) {
        volatile uint32_t* host = P.verdict;
        host[0] = P.status->flags;
        host[1] = P.status->inter_changed;
        host[2] = P.status->pending;
        __threadfence_system();
        host[15] = P.ticket;
    }
    // A lane always handles the same eighth of a data unit (256 is a multiple of 8): where its 8 coefficients
    // go inside the 8x9 tile is fixed, and is kept in registers.
    const uint32_t part = t & 7u;
    uint32_t zo[8];
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) {
        const uint32_t rc = c_zigzag[part * 8u + e];
        zo[e] = (rc >> 3) * 9u + (rc & 7u);
    }
    // A workgroup takes pix_per_wg runs of an image one after the other (Params::pix_per_wg).
    const uint32_t ii = find_image(P, blockIdx.x, &ImgDesc::pix_wg0);
    const ImgDesc D = image_desc_uniform(P, ii);
    const uint32_t upm = D.upm;
    const uint32_t M = (uint32_t)kPixBlocks / upm;
    const uint32_t first_run = (blockIdx.x - D.pix_wg0) * P.pix_per_wg;
    uint32_t left = min(P.pix_per_wg, D.pix_runs * D.mcus_y - first_run);
    uint32_t mrow = first_run / D.pix_runs, run = first_run % D.pix_runs;
    static_assert(kPixBlocks * 8 <= 2 * kWG, "two words of coefficients per lane");
    if (t < 3u * 64u) qf[t] = (float)P.qts[D.qt_off + t];
    __syncthreads();
    for (;;) {
    // (What is worked out from the lane's number inside the loop stays there: kept across it, it would take 30 more
    // registers, and a third of the wavefronts would have no place.)
    asm volatile("" : "+v"(t));
    const uint32_t m0 = run * M;
    const uint32_t nm = min(M, D.mcus_x - m0);
    const uint32_t nblk = nm * upm;
    // 8 coefficients (16 bytes) per lane and step
    uint4 raw0 = make_uint4(0u, 0u, 0u, 0u), raw1 = raw0;
    const uint4* coef = reinterpret_cast<const uint4*>(P.coef + D.coef_off + (size_t)((size_t)mrow * D.mcus_x + m0) * upm * 64u);
    if (t < nblk * 8u) raw0 = load_coef<ONCE>(coef + t);
    if (t + kWG < nblk * 8u) raw1 = load_coef<ONCE>(coef + t + kWG);

    // dequantise + de-zigzag
    auto place = [&](uint32_t j, const uint4& raw) {
        const uint32_t k = j >> 3;
        const uint32_t ku = upm == 1u ? 0u : (upm == 3u ? k % 3u : (upm == 4u ? (k & 3u) : k % 6u));
        const uint32_t comp = (D.sched_comp >> (ku * 4u)) & 15u;
        const float4 qa = *reinterpret_cast<const float4*>(qf + comp * 64u + part * 8u);
        const float4 qb = *reinterpret_cast<const float4*>(qf + comp * 64u + part * 8u + 4u);
        float* tile = blk + k * kBlkStride;
        tile[zo[0]] = (float)(int16_t)(raw.x) * qa.x;
        tile[zo[1]] = (float)((int32_t)raw.x >> 16) * qa.y;
        tile[zo[2]] = (float)(int16_t)(raw.y) * qa.z;
        tile[zo[3]] = (float)((int32_t)raw.y >> 16) * qa.w;
        tile[zo[4]] = (float)(int16_t)(raw.z) * qb.x;
        tile[zo[5]] = (float)((int32_t)raw.z >> 16) * qb.y;
        tile[zo[6]] = (float)(int16_t)(raw.w) * qb.z;
        tile[zo[7]] = (float)((int32_t)raw.w >> 16) * qb.w;
    };
    if (t < nblk * 8u) place(t, raw0);
    if (t + kWG < nblk * 8u) place(t + kWG, raw1);
    __syncthreads();
    // columns
    for (uint32_t j = t; j < nblk * 8u; j += kWG) {
        float* b = blk + (j >> 3) * kBlkStride + (j & 7u);
        float v0 = b[0], v1 = b[9], v2 = b[18], v3 = b[27], v4 = b[36], v5 = b[45], v6 = b[54], v7 = b[63];
        idct8(v0, v1, v2, v3, v4, v5, v6, v7);
        b[0] = v0; b[9] = v1; b[18] = v2; b[27] = v3; b[36] = v4; b[45] = v5; b[54] = v6; b[63] = v7;
    }
    __syncthreads();

    // Rows and output in one step: a lane transforms one row of a data unit and turns the eight samples into bytes,
    // without a way back through LDS.  Only the chroma rows of subsampled images, which several lanes need, are
    // transformed in place first.
    // (sampling factors are 1 or 2: shifts instead of divisions; the one division by a free number, the groups per
    // row, goes through a reciprocal that is exact for the few hundred items of a workgroup; all factors are far
    // under 2^24: the 24-bit multiply runs at full rate, the 32-bit one at a quarter)
    const uint32_t hs = D.hs, vs = D.vs, ncomp = D.ncomp;
    const uint32_t lhs = hs >> 1, lvs = vs >> 1;          // log2 of 1 or 2
    const uint32_t mcu_w = 8u * hs, mcu_h = 8u * vs, lmw = 3u + lhs;
    const uint32_t rows8 = nm * hs;                       // groups of 8 samples per luma row of the workgroup
    const float inv_rows8 = 1.0f / (float)rows8;
    uint8_t* pix = P.pixels + D.pix_off;
    const uint32_t x_base = m0 * mcu_w, y_base = mrow * mcu_h;
    auto pack8 = [](uint32_t (&w)[2], const float (&v)[8]) {
        w[0] = pack_u8(v[0], 0u, 0u); w[0] = pack_u8(v[1], 1u, w[0]); w[0] = pack_u8(v[2], 2u, w[0]); w[0] = pack_u8(v[3], 3u, w[0]);
        w[1] = pack_u8(v[4], 0u, 0u); w[1] = pack_u8(v[5], 1u, w[1]); w[1] = pack_u8(v[6], 2u, w[1]); w[1] = pack_u8(v[7], 3u, w[1]);
    };
    if (P.planar || ncomp == 1u) {
        // Gray, or the paper's own output (Section 3: one array per colour channel): every component at its own
        // resolution, rounded and clamped.  Luma plane first, then Cb, then Cr.
        for (uint32_t j = t; j < rows8 * mcu_h; j += kWG) {
            const uint32_t py = (uint32_t)(((float)j + 0.5f) * inv_rows8), px0 = (j - __umul24(py, rows8)) * 8u;
            const uint32_t gy = y_base + py, gx0 = x_base + px0;
            if (gy >= D.height || gx0 >= D.width) continue;
            const uint32_t m = px0 >> lmw, xin = px0 & (mcu_w - 1u);  // xin: 0, or 8 in the right half of a 16-wide MCU
            float v[8];
            row_samples(blk + __umul24(__umul24(m, upm) + __umul24(py >> 3, hs) + (xin >> 3), (uint32_t)kBlkStride) + (py & 7u) * 9u, v);
            uint32_t w[2];
            pack8(w, v);
            put_bytes<2, ONCE>(pix + (size_t)gy * D.width + gx0, w, min(8u, D.width - gx0));
        }
        if (ncomp == 3u) {
            const uint32_t cw = (D.width + hs - 1u) >> lhs, ch = (D.height + vs - 1u) >> lvs;  // chroma plane size
            uint8_t* cplane = pix + (size_t)D.width * D.height;
            const float inv_nm = 1.0f / (float)nm;
            for (uint32_t j = t; j < nm * 16u; j += kWG) {
                const uint32_t c = j >= nm * 8u ? 1u : 0u;
                const uint32_t r = j - c * nm * 8u;
                const uint32_t py = (uint32_t)(((float)r + 0.5f) * inv_nm), m = r - __umul24(py, nm);
                const uint32_t gy = mrow * 8u + py, gx0 = (m0 + m) * 8u;
                if (gy >= ch || gx0 >= cw) continue;
                float v[8];
                row_samples(blk + __umul24(__umul24(m, upm) + hs * vs + c, (uint32_t)kBlkStride) + py * 9u, v);
                uint32_t w[2];
                pack8(w, v);
                put_bytes<2, ONCE>(cplane + (size_t)c * cw * ch + (size_t)gy * cw + gx0, w, min(8u, cw - gx0));
            }
        }
    } else {
    // RGB: a lane produces the 24 bytes of eight horizontally adjacent pixels -- one row of a luma data unit.  The
    // colour terms of a chroma sample are computed once (a sample serves two of the pixels when chroma is subsampled
    // horizontally); each output sample then costs one addition and one conversion that also puts the byte in its place.
    const uint32_t row_bytes = D.width * 3u;  // a frame header holds the width in 16 bits
    // bytes in memory: R0 G0 B0 R1 | G1 B1 R2 G2 | B2 R3 G3 B3
    auto pack12 = [](uint32_t& wa, uint32_t& wb, uint32_t& wc, float y0, float y1, float y2, float y3,
                     const ChromaTerms& c0, const ChromaTerms& c1, const ChromaTerms& c2, const ChromaTerms& c3) {
        wa = pack_u8(y0 + c0.r, 0u, wa); wa = pack_u8(y0 + c0.g, 1u, wa); wa = pack_u8(y0 + c0.b, 2u, wa);
        wa = pack_u8(y1 + c1.r, 3u, wa); wb = pack_u8(y1 + c1.g, 0u, wb); wb = pack_u8(y1 + c1.b, 1u, wb);
        wb = pack_u8(y2 + c2.r, 2u, wb); wb = pack_u8(y2 + c2.g, 3u, wb); wc = pack_u8(y2 + c2.b, 0u, wc);
        wc = pack_u8(y3 + c3.r, 1u, wc); wc = pack_u8(y3 + c3.g, 2u, wc); wc = pack_u8(y3 + c3.b, 3u, wc);
    };
    if (hs * vs != 1u) {
        for (uint32_t j = t; j < nm * 16u; j += kWG) {  // j: MCU, Cb or Cr, row
            float* b = blk + __umul24(__umul24(j >> 4, upm) + hs * vs + ((j >> 3) & 1u), (uint32_t)kBlkStride) + (j & 7u) * 9u;
            float v[8];
            row_samples(b, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) b[e] = v[e];
        }
        __syncthreads();
    }
    for (uint32_t j = t; j < rows8 * mcu_h; j += kWG) {
        const uint32_t py = (uint32_t)(((float)j + 0.5f) * inv_rows8), px0 = (j - __umul24(py, rows8)) * 8u;
        const uint32_t gy = y_base + py, gx0 = x_base + px0;
        if (gy >= D.height || gx0 >= D.width) continue;
        const uint32_t m = px0 >> lmw, xin = px0 & (mcu_w - 1u);
        const uint32_t mu = __umul24(m, upm);
        float y[8];
        row_samples(blk + __umul24(mu + __umul24(py >> 3, hs) + (xin >> 3), (uint32_t)kBlkStride) + (py & 7u) * 9u, y);
        const float* cbb = blk + __umul24(mu + hs * vs, (uint32_t)kBlkStride) + (py >> lvs) * 9u + (xin >> lhs);
        const float* crb = cbb + kBlkStride;
        uint32_t w[6] = {0u, 0u, 0u, 0u, 0u, 0u};
        if (hs == 2u) {  // (the cases are written out so that none pays register moves for another)
            const ChromaTerms a = chroma_terms(cbb[0], crb[0]), b = chroma_terms(cbb[1], crb[1]);
            pack12(w[0], w[1], w[2], y[0], y[1], y[2], y[3], a, a, b, b);
            const ChromaTerms c = chroma_terms(cbb[2], crb[2]), d = chroma_terms(cbb[3], crb[3]);
            pack12(w[3], w[4], w[5], y[4], y[5], y[6], y[7], c, c, d, d);
        } else {
            float cb[8], cr[8];
            if (vs == 1u) {
                row_samples(cbb, cb);
                row_samples(crb, cr);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) { cb[e] = cbb[e]; cr[e] = crb[e]; }
            }
            {
                const ChromaTerms a = chroma_terms(cb[0], cr[0]), b = chroma_terms(cb[1], cr[1]);
                const ChromaTerms c = chroma_terms(cb[2], cr[2]), d = chroma_terms(cb[3], cr[3]);
                pack12(w[0], w[1], w[2], y[0], y[1], y[2], y[3], a, b, c, d);
            }
            {
                const ChromaTerms a = chroma_terms(cb[4], cr[4]), b = chroma_terms(cb[5], cr[5]);
                const ChromaTerms c = chroma_terms(cb[6], cr[6]), d = chroma_terms(cb[7], cr[7]);
                pack12(w[3], w[4], w[5], y[4], y[5], y[6], y[7], a, b, c, d);
            }
        }
        put_bytes<6, ONCE>(pix + (size_t)gy * row_bytes + __umul24(gx0, 3u), w, min(8u, D.width - gx0) * 3u);
    }
    }
    if (--left == 0u) break;
    if (++run == D.pix_runs) { run = 0u; ++mrow; }
    __syncthreads();  // the tiles are read no more
    }
}

// ---- pixels at reduced size ------------------------------------------------------------------------------
// Output at 1/2, 1/4 or 1/8 of the size straight from the coefficients: of every data unit only the N x N lowest
// frequencies are read, N = 4, 2, 1, and the N-point inverse transform is applied to them,
//   f(y,x) = 1/4 sum_{u<N} sum_{v<N} C(u) C(v) F(v,u) cos((2x+1) u pi/(2N)) cos((2y+1) v pi/(2N)),
// with the 8-point transform's factor, so that a unit holding only a DC term keeps its value.  Everything after
// that is as at full size: level shift, chroma replicated by the sampling factors, colour matrix, one rounding,
// crop to ceil(width / d) x ceil(height / d).  (The paper's decoder ends with the full-size transform, Section 4.3,
// and names it as the stage that now limits the decoder; this path reads the same coefficients and skips most of it.)

// c_basis*[x * N + u] = 1/2 C(u) cos((2x+1) u pi / (2N))
#define JPGD_BASIS4_LITERAL                                                                            \
    {0.35355339059327379f, 0.46193976625564337f, 0.35355339059327379f, 0.19134171618254489f,            \
     0.35355339059327379f, 0.19134171618254489f, -0.35355339059327379f, -0.46193976625564337f,          \
     0.35355339059327379f, -0.19134171618254489f, -0.35355339059327379f, 0.46193976625564337f,          \
     0.35355339059327379f, -0.46193976625564337f, 0.35355339059327379f, -0.19134171618254489f}
#define JPGD_BASIS2_LITERAL {0.35355339059327379f, 0.35355339059327379f, 0.35355339059327379f, -0.35355339059327379f}
// (the same values twice: as compile-time constants for sums whose position is unrolled, and in constant memory for
// the table a lane indexes with its row)
constexpr float c_basis4_host[16] = JPGD_BASIS4_LITERAL;
constexpr float c_basis2_host[4] = JPGD_BASIS2_LITERAL;
__device__ __constant__ float c_basis4[16] = {
    0.35355339059327379f, 0.46193976625564337f, 0.35355339059327379f, 0.19134171618254489f,
    0.35355339059327379f, 0.19134171618254489f, -0.35355339059327379f, -0.46193976625564337f,
    0.35355339059327379f, -0.19134171618254489f, -0.35355339059327379f, 0.46193976625564337f,
    0.35355339059327379f, -0.46193976625564337f, 0.35355339059327379f, -0.19134171618254489f};
__device__ __constant__ float c_basis2[4] = {0.35355339059327379f, 0.35355339059327379f,
                                             0.35355339059327379f, -0.35355339059327379f};

// natural (row-major) position -> zig-zag position: the inverse of the zig-zag literal, made at compile time
struct UnZigzag {
    uint8_t at[64];
    constexpr UnZigzag() : at{} {
        constexpr uint8_t zz[64] = JPGD_ZIGZAG_LITERAL;
        for (int i = 0; i < 64; ++i) at[zz[i]] = (uint8_t)i;
    }
};
__device__ __constant__ UnZigzag c_unzigzag = UnZigzag();

template <int N>
__global__ __launch_bounds__(kWG) void k_pixels_scaled(Params P) {
    constexpr uint32_t NN = N * N;
    constexpr uint32_t lN = N == 4 ? 2u : (N == 2 ? 1u : 0u);   // log2 N
    __shared__ float fin[kPixBlocksScaled * NN];   // dequantised low frequencies, [unit][v * N + u]
    __shared__ float smp[kPixBlocksScaled * NN];   // samples, level shift applied, [unit][y * N + x]
    __shared__ float bs[NN];
    const uint32_t wg = blockIdx.x;
    const uint32_t ii = find_image(P, wg, &ImgDesc::pix_wg0);
    const ImgDesc D = image_desc_uniform(P, ii);
    const uint32_t lw = wg - D.pix_wg0;
    const uint32_t mrow = lw / D.pix_runs, run = lw % D.pix_runs;
    const uint32_t upm = D.upm;
    const uint32_t M = (uint32_t)kPixBlocksScaled / upm;
    const uint32_t m0 = run * M;
    const uint32_t nm = min(M, D.mcus_x - m0);
    const uint32_t nblk = nm * upm;
    const uint32_t t = threadIdx.x;
    if (wg == 0u && t == 0u && P.verdict) {  // the verdict of the write kernel, as in k_pixels
        volatile uint32_t* host = P.verdict;
        host[0] = P.status->flags;
        host[1] = P.status->inter_changed;
        host[2] = P.status->pending;
        __threadfence_system();
        host[15] = P.ticket;
    }
    if (t < NN) bs[t] = N == 4 ? c_basis4[t] : (N == 2 ? c_basis2[t & 3u] : 0.35355339059327379f);
    // A lane always fetches the same frequency (256 is a multiple of N * N): its zig-zag position is looked up once.
    const uint32_t e = t & (NN - 1u);
    const uint32_t zpos = c_unzigzag.at[(e >> lN) * 8u + (e & (N - 1u))];
    const int16_t* coef = P.coef + D.coef_off + (size_t)((size_t)mrow * D.mcus_x + m0) * upm * 64u;
    const uint16_t* qt = P.qts + D.qt_off + zpos;
    const float q0 = (float)qt[0], q1 = (float)qt[64], q2 = (float)qt[128];
    for (uint32_t j = t; j < nblk * NN; j += kWG) {
        const uint32_t k = j >> (2u * lN);
        const uint32_t ku = upm == 1u ? 0u : (upm == 3u ? k % 3u : (upm == 4u ? (k & 3u) : k % 6u));
        const uint32_t comp = (D.sched_comp >> (ku * 4u)) & 15u;
        fin[j] = (float)coef[(size_t)k * 64u + zpos] * (comp == 0u ? q0 : (comp == 1u ? q1 : q2));
    }
    __syncthreads();
    // one lane per row of a unit's N x N samples: first the sum over the vertical frequencies for its row (weights
    // from the basis table in LDS, they depend on the row), then the N outputs (weights are constants)
    for (uint32_t j = t; j < nblk * N; j += kWG) {
        const uint32_t k = j >> lN, y = j & (N - 1u);
        const float* F = fin + k * NN;
        float g[N];
#pragma unroll
        for (uint32_t u = 0; u < (uint32_t)N; ++u) g[u] = 0.0f;
#pragma unroll
        for (uint32_t v = 0; v < (uint32_t)N; ++v) {
            const float w = bs[y * N + v];
#pragma unroll
            for (uint32_t u = 0; u < (uint32_t)N; ++u) g[u] = __builtin_fmaf(w, F[v * N + u], g[u]);
        }
#pragma unroll
        for (uint32_t x = 0; x < (uint32_t)N; ++x) {
            float acc = 128.0f;
#pragma unroll
            for (uint32_t u = 0; u < (uint32_t)N; ++u)
                acc = __builtin_fmaf(N == 4 ? c_basis4_host[x * 4u + u] : (N == 2 ? c_basis2_host[(x * 2u + u) & 3u] : 0.35355339059327379f), g[u], acc);
            smp[k * NN + y * N + x] = acc;
        }
    }
    __syncthreads();

    const uint32_t hs = D.hs, vs = D.vs, ncomp = D.ncomp;
    const uint32_t lhs = hs >> 1, lvs = vs >> 1;
    const uint32_t ls = 3u - lN;                                  // log2 of the scale denominator
    const uint32_t ow = (D.width + (1u << ls) - 1u) >> ls, oh = (D.height + (1u << ls) - 1u) >> ls;
    uint8_t* pix = P.pixels + D.pix_off;
    // sample (py, px) of the rectangle that component units [u0, u0 + ux * uy) of the workgroup's MCUs cover
    // (ux x uy units of N x N samples per MCU)
    auto sample = [&](uint32_t u0, uint32_t lux, uint32_t py, uint32_t px) {
        const uint32_t lmw = lN + lux;                            // log2 of the samples per MCU row
        const uint32_t m = px >> lmw, xin = px & ((1u << lmw) - 1u);
        const uint32_t unit = m * upm + u0 + ((py >> lN) << lux) + (xin >> lN);
        return smp[unit * NN + ((py & (N - 1u)) << lN) + (xin & (N - 1u))];
    };
    auto put = [&](uint8_t* dst, const uint32_t* w, uint32_t nbytes, bool words) {
        if (words) {
            for (uint32_t e = 0; e < nbytes / 4u; ++e) reinterpret_cast<uint32_t*>(dst)[e] = w[e];
        } else {
            for (uint32_t e = 0; e < nbytes; ++e) dst[e] = (uint8_t)(w[e >> 2] >> (8u * (e & 3u)));
        }
    };
    if (P.planar) {
        // component planes at reduced size, one after the other: plane c has ceil(plane_w / d) x ceil(plane_h / d) samples
        size_t plane_off = 0;
        for (uint32_t c = 0; c < ncomp; ++c) {
            const uint32_t lux = c == 0u ? lhs : 0u, luy = c == 0u ? lvs : 0u;
            const uint32_t u0 = c == 0u ? 0u : hs * vs + c - 1u;
            const uint32_t full_w = c == 0u ? D.width : (D.width + hs - 1u) >> lhs;
            const uint32_t full_h = c == 0u ? D.height : (D.height + vs - 1u) >> lvs;
            const uint32_t pw = (full_w + (1u << ls) - 1u) >> ls, ph = (full_h + (1u << ls) - 1u) >> ls;
            uint8_t* plane = pix + plane_off;
            plane_off += (size_t)pw * ph;
            const uint32_t region_w = nm << (lN + lux), region_h = 1u << (lN + luy);
            const uint32_t gpr = (region_w + 3u) >> 2;
            const uint32_t x_base = m0 << (lN + lux), y_base = mrow << (lN + luy);
            const bool words_ok = (pw & 3u) == 0u && (reinterpret_cast<size_t>(plane) & 3u) == 0u;
            for (uint32_t j = t; j < gpr * region_h; j += kWG) {
                const uint32_t py = j / gpr, px0 = (j - py * gpr) * 4u;
                const uint32_t gy = y_base + py, gx0 = x_base + px0;
                if (gy >= ph || gx0 >= pw) continue;
                const uint32_t cnt = min(4u, min(region_w - px0, pw - gx0));
                uint32_t w[1] = {0u};
                w[0] = pack_u8(sample(u0, lux, py, px0), 0u, w[0]);
                w[0] = pack_u8(sample(u0, lux, py, min(px0 + 1u, region_w - 1u)), 1u, w[0]);
                w[0] = pack_u8(sample(u0, lux, py, min(px0 + 2u, region_w - 1u)), 2u, w[0]);
                w[0] = pack_u8(sample(u0, lux, py, min(px0 + 3u, region_w - 1u)), 3u, w[0]);
                put(plane + (size_t)gy * pw + gx0, w, cnt, cnt == 4u && words_ok);
            }
        }
        return;
    }
    // gray or RGB: a lane produces four horizontally adjacent pixels
    const uint32_t region_w = nm << (lN + lhs), region_h = 1u << (lN + lvs);
    const uint32_t gpr = (region_w + 3u) >> 2;
    const uint32_t x_base = m0 << (lN + lhs), y_base = mrow << (lN + lvs);
    const uint32_t row_bytes = ow * ncomp;
    const bool words_ok = (row_bytes & 3u) == 0u && (reinterpret_cast<size_t>(pix) & 3u) == 0u;
    for (uint32_t j = t; j < gpr * region_h; j += kWG) {
        const uint32_t py = j / gpr, px0 = (j - py * gpr) * 4u;
        const uint32_t gy = y_base + py, gx0 = x_base + px0;
        if (gy >= oh || gx0 >= ow) continue;
        const uint32_t cnt = min(4u, min(region_w - px0, ow - gx0));
        uint32_t w[3] = {0u, 0u, 0u};
        float yv[4];
        ChromaTerms ct[4];
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) {
            const uint32_t px = min(px0 + e, region_w - 1u);
            yv[e] = sample(0u, lhs, py, px);
            if (ncomp == 3u) {
                const float cb = sample(hs * vs, 0u, py >> lvs, px >> lhs), cr = sample(hs * vs + 1u, 0u, py >> lvs, px >> lhs);
                ct[e] = chroma_terms(cb, cr);
            }
        }
        if (ncomp == 1u) {
            w[0] = pack_u8(yv[0], 0u, w[0]); w[0] = pack_u8(yv[1], 1u, w[0]);
            w[0] = pack_u8(yv[2], 2u, w[0]); w[0] = pack_u8(yv[3], 3u, w[0]);
        } else {
            // bytes in memory: R0 G0 B0 R1 | G1 B1 R2 G2 | B2 R3 G3 B3
            w[0] = pack_u8(yv[0] + ct[0].r, 0u, w[0]); w[0] = pack_u8(yv[0] + ct[0].g, 1u, w[0]); w[0] = pack_u8(yv[0] + ct[0].b, 2u, w[0]);
            w[0] = pack_u8(yv[1] + ct[1].r, 3u, w[0]); w[1] = pack_u8(yv[1] + ct[1].g, 0u, w[1]); w[1] = pack_u8(yv[1] + ct[1].b, 1u, w[1]);
            w[1] = pack_u8(yv[2] + ct[2].r, 2u, w[1]); w[1] = pack_u8(yv[2] + ct[2].g, 3u, w[1]); w[2] = pack_u8(yv[2] + ct[2].b, 0u, w[2]);
            w[2] = pack_u8(yv[3] + ct[3].r, 1u, w[2]); w[2] = pack_u8(yv[3] + ct[3].g, 2u, w[2]); w[2] = pack_u8(yv[3] + ct[3].b, 3u, w[2]);
        }
        put(pix + (size_t)gy * row_bytes + (size_t)gx0 * ncomp, w, cnt * ncomp, cnt == 4u && words_ok);
    }
}

}  // namespace jpgd
