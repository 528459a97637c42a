// Lossless stage, decoder: one wave per chunk; body -> LDS, every lane decodes one sub-block with a
// 4096-entry table, the packed rows are rebuilt in LDS and dequantized from there.  Compiled once per
// code width (-DKVC_BITS=2, 3, 4 or 8).  See kvc_huff.h.

#include "kvc_huff.h"

#ifndef KVC_BITS
#error "compile with -DKVC_BITS=2, 3, 4 or 8"
#endif

namespace kvc {

// ---- decoder ---------------------------------------------------------------------------------

typedef __attribute__((address_space(3))) const uint32_t *LdsWords;

struct BitReader {
    uint32_t hi, lo, ahead;      // the word being read, the next one, and the one after that, in flight
    uint32_t rest;               // low byte: bits of `hi` that are still to be read, 0..31 (the other bytes: anything)
    uint32_t next, last;         // where `ahead` comes from and the last readable word (LDS addresses)
};

__device__ __forceinline__ uint32_t lds_word(uint32_t at) { return *(LdsWords)at; }

// The stream starts at bit `bit` of the words behind the body's 64 bit counts; the body has `size` bytes.
__device__ __forceinline__ void reader_start(BitReader &br, const uint8_t *body, uint32_t bit, uint32_t size)
{
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const uint8_t *)body;
    br.last = base + size - 4;
    uint32_t at = base + 2 * kSubs + 4 * ((int)(bit - 1) >> 5);       // (bit 0: all of the word before the stream has been read)
    at = min(at, br.last);
    br.hi = lds_word(at);
    at = min(at + 4, br.last);
    br.lo = lds_word(at);
    br.next = min(at + 4, br.last);
    br.ahead = lds_word(br.next);
    br.rest = (0u - bit) & 31;
}

// Two symbols (24 bits at most).  A table entry is symbol << 8 | (256 - length): its low five bits shift the
// window by the length as they are, and added up they count `rest` down, so that no field is taken
// out of an entry before the symbols are collected.  The word that a refill brings in was requested a pair
// earlier, so the chain is two table look-ups, and a lane that needs no word asks for the same one again instead of
// branching.  15 vector operations per pair; a 64-bit window with a load in every refill took 21 and a third LDS
// round trip (decompress calls of 2^21 rows: 8 bits 449 -> 368 us, 4 bits 254 -> 247, half of the heads at 8 and half at
// 2 bits 370 -> 325; one layer of 32k tokens, 4 bits, 42.7 -> 41.2).
__device__ __forceinline__ void decode_pair(const uint16_t *lut, BitReader &br, uint32_t &e0, uint32_t &e1)
{
    const uint32_t window = __builtin_amdgcn_alignbit(br.hi, br.lo, br.rest);
    e0 = lut[window >> 20];
    e1 = lut[__builtin_amdgcn_alignbit(window, 0, e0) >> 20];
    const uint32_t rest = br.rest + e0 + e1, over = (rest >> 7) & 1;
    br.hi = over ? br.lo : br.hi;
    br.lo = over ? br.ahead : br.lo;
    br.rest = rest + (over << 5);
    br.next = min(br.next + (over << 2), br.last);
    br.ahead = lds_word(br.next);
}

template <int W> __device__ __forceinline__ void decode_half(uint32_t *sym, const uint16_t *lut, int half, BitReader &br)
{
#pragma unroll
    for (int k = 0; k < W / 2; ++k) {
        uint32_t e[4];
        decode_pair(lut, br, e[0], e[1]);
        decode_pair(lut, br, e[2], e[3]);
        const uint32_t low = __builtin_amdgcn_perm(e[1], e[0], 0x0c0c0501u), high = __builtin_amdgcn_perm(e[3], e[2], 0x0c0c0501u);
        sym[half * (W / 2) + k] = __builtin_amdgcn_perm(high, low, 0x05040100u);
    }
}

// metadata of the 32 rows starting at chunk row `r0`: K = the lane's 8 channels of that token
// block (two 16-byte loads), V = the lane's group in each of its 8 rows
__device__ __forceinline__ void load_meta_k(const QuantArgs &q, const ChunkPos &c, int r0, int col, u32x4 &m0, u32x4 &m1)
{
    const long long nb = (q.tokens + q.group - 1) / q.group;
    const u32x4 *m = (const u32x4 *)(q.meta + ((c.lh * nb + (c.row0 + r0) / q.group) * kDim + col * 8) * 4);
    m0 = m[0];
    m1 = m[1];
}

__device__ __forceinline__ void load_meta_v(const QuantArgs &q, const ChunkPos &c, int r0, uint32_t mv[8])
{
    const int lane = lane_id(), col = lane & 15, rsub = lane >> 4;
    const int ng = kDim / q.group, shift = q.group == 32 ? 2 : (q.group == 64 ? 3 : 4);
    const uint32_t *m = (const uint32_t *)q.meta + (c.lh * q.tokens + c.row0 + r0) * ng + (col >> shift);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = 4 * i + rsub;
        mv[i] = m[(r0 + r < c.rows ? r : 0) * ng];
    }
}

// Dequantize a decoded chunk from the wave's LDS region and store its rows; the metadata of a
// pass is in flight one pass ahead.  meta0 / meta1 (K) or metav (V): the first pass's metadata.
// first_anchor (delta transform): the first pass's anchor row.
template <int BITS, int DT, bool IS_V, bool DENSE, int TR>
__device__ __forceinline__ void dequant_chunk(const CoderArgs &a, const ChunkPos &c, uint8_t *lds, const u32x4 &meta0,
                                              const u32x4 &meta1, const uint32_t metav[8], const u32x4 &first_anchor,
                                              int first_blocks, bool &bad)
{
    using Dec = DecGeom<BITS>;
    const uint16_t *anchors = TR >= 2 ? head_anchors(a.q.anchors, c.lh, a.q.tokens, a.q.anchor_shift) : nullptr;
    constexpr bool one_anchor = TR == 2;
    u32x4 anchor = first_anchor, anchor_next = first_anchor;
    u32x4 mk0 = meta0, mk1 = meta1;
    uint32_t mv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) mv[i] = metav[i];
    // paged destination: the block-table entries of a pass are in flight one pass ahead as well
    const bool paged = !DENSE && a.q.x.block_table != nullptr && a.q.x.bt_wave;
    int blocks = first_blocks, blocks_next = first_blocks;
#pragma unroll 1
    for (int p = 0; p < kChunkRows / kPassRows; ++p) {
        if (p * kPassRows >= c.rows) break;
        float scale[8], zero[8];
        const bool clamp = IS_V ? v_meta_floats<BITS, DT>(mv, scale, zero) : k_meta_floats<BITS, DT>(mk0, mk1, scale, zero);
        if ((p + 1) * kPassRows < c.rows) {
            if (!IS_V) load_meta_k(a.q, c, (p + 1) * kPassRows, lane_octet(TR == 1), mk0, mk1);
            else load_meta_v(a.q, c, (p + 1) * kPassRows, mv);
            if (one_anchor) anchor_next = load_anchor(anchors, a.q.anchor_shift, c.row0 + (p + 1) * kPassRows);
            if (paged) blocks_next = pass_blocks(a.q.x, c.row0 + (p + 1) * kPassRows, c.row0 + c.rows);
        }
        PassFetch f;
        pass_fetch<BITS, DENSE, Dec::kLayout, TR == 1>(f, lds, a.q.x, c.head_off, c.row0 + p * kPassRows, c.rows - p * kPassRows, p * kPassRows,
                                              paged, blocks);
        dequant_pass<BITS, DT, IS_V, DENSE, TR>(f, scale, zero, clamp, a.q.x, c.head_off, c.row0 + p * kPassRows,
                                                c.rows - p * kPassRows, bad, anchors, TR == 3 ? anew(a.q.anchor_shift) : a.q.anchor_shift,
                                                one_anchor ? &anchor : nullptr);
        anchor = anchor_next;
        blocks = blocks_next;
    }
}

// TR: the inverse of stage T that the launch applies (see dequant_pass_rows).  One kernel per
// transform: in one kernel, every path pays for the registers of the most expensive one (the anchors
// of short runs, the rotation) with its fourth wave per SIMD.
// KV: the launch's tensor, K (0), V (1) or both (2: the batch holds items of either; without a transform).
template <int BITS, int DT, int KV, bool DENSE, int TR>
__global__ __launch_bounds__(ChunkGeom<BITS>::kDecWaves * 64) void decode_kernel(CoderBatch batch)
{
    using Geo = ChunkGeom<BITS>;
    using Dec = DecGeom<BITS>;
    constexpr int W = Geo::kWords, NW = Geo::kDecWaves;
    unsigned wg;
    // What the batch has for all items comes with the table of places, and an item's members in one trip.  Decompress calls without / with,
    // one layer of 1000 tokens, of 32k, 2^21 rows, seven requests of 2^17.6, fp16: 2 bits 16.4 / 16.1, 37.5 / 37.1, 216 / 216, 156.9 / 156.2 us; 3
    // bits 14.2 / 14.0, 34.4 / 34.1, 210 / 210, 155.9 / 155.4; 4 bits 19.6 / 19.4, 41.9 / 41.4, 247 / 246, 179 / 177; 8 bits 24.8 / 24.6, 73.4 / 72.9,
    // 359 / 359, 267.9 / 269.2; paged and bf16 layers as fp16 ones; half of the heads at 8 and half at 2 bits 311.5 / 312.0.
    int covered0 = batch.heads_covered[0], covered1 = batch.heads_covered[1], slots = batch.slots;
    int *status = batch.status;
    uint8_t *scratch = batch.ws;
    long long scratch_bytes = batch.ws_request;
    asm volatile("" ::"s"(covered0), "s"(covered1), "s"(slots), "s"(status), "s"(scratch), "s"(scratch_bytes));
    const CoderArgs a = coder_args<KV, true>(batch, place_item_of_many(batch.at, place_of_workgroup(batch.at), wg));
    const bool is_v = KV == 2 ? a.is_v != 0 : KV == 1;
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[NW * Dec::kLds];
    __shared__ uint16_t lut[4096];

    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();      // (kept per lane: as a scalar it costs this kernel its fourth wave per SIMD)
    long long chunk = (long long)wg * NW + wave;
    const bool live = chunk < a.chunks;
    if (!DENSE && live && a.q.head_minor) {
        // destination with the heads of a token next to each other: neighbouring waves take the same
        // rows of neighbouring heads, so that what they store together is contiguous
        const long long cph = (a.q.tokens + kChunkRows - 1) / kChunkRows;
        const long long t = chunk / a.q.heads, h = chunk - t * a.q.heads;
        const long long l = t / cph, cb = t - l * cph;
        chunk = (l * a.q.heads + h) * cph + cb;
    }
    uint8_t *lds = lds_all + wave * Dec::kLds;
    // Register headroom.  On this GPU a 64-bit shift whose count sits in the last VGPR of the
    // wave's allocation shifts by the lane number instead, now and then, once three or four such
    // waves share a SIMD (LLVM knows and avoids the fault for gfx90a only).  A build of this
    // kernel with a 64-bit window that needed exactly 112 registers kept a code length in v111 for `window <<= len`
    // and decoded the last two symbols of a sub-block wrongly in one wave of seven at full size.  The window has 32
    // bits now (decode_pair); 64-bit shifts are left in the addressing, by constants and scalars.
    // Naming a higher register keeps the allocation (128: still four waves per SIMD) above every
    // register the code touches; the build checks the assembly of all kernels for the pattern.
    if (BITS == 8) asm volatile("" ::: "v255");        // (the 8-bit kernel keeps more rows in registers: two waves per SIMD either way)
    else asm volatile("" ::: "v127");

    // Round trip 1: the chunk's two directory entries and the status word, with the decode
    // table right behind them.
    unsigned long long d0 = 0, d1 = 0;
    int st = 0;
    if (live) {
        const uint32_t *dir = (const uint32_t *)(a.payload + a.off_dir) + a.chunk_base + chunk;
        d0 = dir[0];
        d1 = dir[1];
        st = *a.q.status;
    }
    constexpr int LUTN = 512 / (NW * 64);
    u32x4 lutv[LUTN];
    {
        const u32x4 *src = (const u32x4 *)(a.ws.lut + 4096 * a.tab);
#pragma unroll
        for (int i = 0; i < LUTN; ++i) lutv[i] = src[tid + i * NW * 64];
    }
    ChunkPos c = chunk_pos(a.q, live ? chunk : 0);
    const uint32_t raw_bytes = (uint32_t)c.rows * Geo::kRowBytes;
    const unsigned long long size = (d1 - d0) * 16;
    bool ok = live && !(st & (KVC_DEV_BAD_HEADER | KVC_DEV_BAD_TABLE));
    if (ok && (d1 < d0 || size > raw_bytes || (long long)(a.off_bodies + d1 * 16) > a.capacity ||
               (size != raw_bytes && size < 2 * kSubs + 16))) {
        if (lane == 0) atomicOr(a.q.status, KVC_DEV_BAD_CHUNK);
        ok = false;
    }
    // Round trip 2: the body (into registers) and the metadata of the first pass.
    constexpr int NB = 2 * BITS;                       // 16-byte pieces per lane of a full raw chunk
    u32x4 bodyv[NB];
    u32x4 meta0 = {0, 0, 0, 0}, meta1 = {0, 0, 0, 0};
    uint32_t metav[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    u32x4 anchor0 = {0, 0, 0, 0};                      // delta transform: the first pass's anchor row
    int blocks0 = 0;                                   // paged destination: the first pass's block-table entries (pass_blocks)
    if (ok) {
        const uint8_t *body = a.payload + a.off_bodies + d0 * 16;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const uint32_t o = (k * 64 + lane) * 16;
            if (o < size) bodyv[k] = __builtin_nontemporal_load((const u32x4 *)(body + o));
        }
        if (!is_v) load_meta_k(a.q, c, 0, lane_octet(TR == 1), meta0, meta1);
        else load_meta_v(a.q, c, 0, metav);
        if (!DENSE && a.q.x.block_table != nullptr && a.q.x.bt_wave) blocks0 = pass_blocks(a.q.x, c.row0, c.row0 + c.rows);
        if (TR == 2)
            anchor0 = load_anchor(head_anchors(a.q.anchors, c.lh, a.q.tokens, a.q.anchor_shift), a.q.anchor_shift, c.row0);
    }
#pragma unroll
    for (int i = 0; i < LUTN; ++i) ((u32x4 *)lut)[tid + i * NW * 64] = lutv[i];
    __syncthreads();
    if (!ok) return;

    if (size == raw_bytes) {
        // stored raw: scatter the packed rows into the sub-block layout
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const uint32_t o = (k * 64 + lane) * 16;
            if (o < raw_bytes) {
                const uint32_t sub = o / Geo::kSubBytes, in = o - sub * Geo::kSubBytes;
                *(u32x4 *)Dec::piece_ptr(lds, sub, in / 16) = bodyv[k];
            }
        }
        wave_sync();
    } else {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const uint32_t o = (k * 64 + lane) * 16;
            if (o < size) *(u32x4 *)(lds + o) = bodyv[k];
        }
        wave_sync();
        const uint32_t bits = ((const uint16_t *)lds)[lane];
        const uint32_t incl = wave_inclusive_sum(bits);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (((2 * kSubs + 4 * ((total + 31) / 32) + 15) & ~15u) != size) {
            if (lane == 0) atomicOr(a.q.status, KVC_DEV_BAD_CHUNK);
            return;
        }
        const uint32_t start = incl - bits;
        BitReader br;
        reader_start(br, lds, start, (uint32_t)size);
        uint32_t sym[W];
#pragma unroll
        for (int k = 0; k < W; ++k) sym[k] = 0;
        const int have = min(max(c.rows - 2 * lane, 0), 2);
        if (have > 0) decode_half<W>(sym, lut, 0, br);
        if (have > 1) decode_half<W>(sym, lut, 1, br);
        wave_sync();                                   // all lanes are done reading the coded words
        {
#pragma unroll
            for (int q = 0; q < W / 4; ++q) {
                u32x4 v;
                v[0] = sym[4 * q]; v[1] = sym[4 * q + 1]; v[2] = sym[4 * q + 2]; v[3] = sym[4 * q + 3];
                *(u32x4 *)Dec::piece_ptr(lds, lane, q) = v;
            }
        }
        wave_sync();
    }

    // Dequantize the rows from LDS.  Until here the chunk's place is kept per lane (see `wave`).  In scalar registers from here on it leaves
    // the strided kernels with the transforms, and the fp16 ones for 3-bit K and V together, the vector registers of their fourth
    // wave per SIMD, once the anchor period of short runs is taken anew as well (which rows are anchors would otherwise be computed for
    // all passes and kept).  Registers and decompress calls, paged, without / with: 3 bits fp16, one layer of 32k tokens 131 / 128, 42.7 /
    // 38.7 us; 2^20 rows, runs of 8 tokens, fp16, 2 and 4 bits 142 / 128, 203 / 177 and 144 / 128, 225 / 196 us; runs of 32, 4 bits 133 / 128,
    // 155 / 149 us, 3 bits bf16 129 / 128, 142 / 132; the rotation (128 either way) 0.993 to 0.999 of the time; others up to 1.01, so they keep it per
    // lane.  (The view read where it lies, not copied, takes no registers either, but then a row's place in its block is
    // computed in every pass: 0.99 to 1.10 of the time.)
    if (!DENSE && BITS != 8 && (TR != 0 || (BITS == 3 && DT == DT_F16 && KV == 2))) {
        c.lh = uniform(c.lh);
        c.head_off = uniform(c.head_off);
        c.row0 = uniform(c.row0);
        c.rows = __builtin_amdgcn_readfirstlane(c.rows);
    }
    bool bad = false;
    if (is_v) dequant_chunk<BITS, DT, true, DENSE, TR>(a, c, lds, meta0, meta1, metav, anchor0, blocks0, bad);
    else dequant_chunk<BITS, DT, false, DENSE, TR>(a, c, lds, meta0, meta1, metav, anchor0, blocks0, bad);
    if (bad) atomicOr(a.q.status, KVC_DEV_BAD_BLOCK);
}

// ---- launchers ----------------------------------------------------------------------------------

// Runs of workgroups per XCD (place_of_workgroup) and LDS that nothing uses (as for the codec-free kernels: 14000 more leave three
// workgroups to a compute unit, 40000 two).  Decompress calls in us, as they were (a conversion per code, neither) / now:
//   dense    rows    2^18        2^19.6      2^20.6      2^21.6      2^22.6      2^23.3 (a launch per tensor)
//   2 bits   38.4 / 38.2   95 / 91   197 / 167   373 / 317   759 / 642   1080 / 1076
//   3 bits   35.5 / 35.5   94 / 91   180 / 165   390 / 313   773 / 636   1143 / 1121
//   4 bits   43.0 / 41.6  106 / 104  190 / 190   375 / 357   799 / 715   1206 / 1200
//   (2^21 rows, 4 bits: with run 64 249, 16 258, without 268; 3 bits with 14000 225, 40000 218; 8 bits, bound by the table
//   look-ups: without either 377, runs 384; 2^23.3 rows and more in one launch, run 64 for 16: +2 %)
//   paged    2 bits, 14000 below the large ones: 2^21 rows 239 / 231 (without 259), 2^23.3 1262 / 1220 (with it 1346); 3 bits
//   131 / 129, 757 / 730
//   launches that are resident at once or nearly gain nothing
struct DecodeShape {
    unsigned lds = 0;
    int run = 0;
};

// One shape for all groups and any number of requests lost calls against the former kernels; below the lines per group and
// number, former / one shape / now (ratios to the former, the worst of both types and the wider groups):
//   dense    3 bits, groups of 64 and 128, 2^20 rows 1 / 1.07 / 1.01, 2^22 1 / 1.05 / 0.99; several requests, groups of 32, 32 of 2^18.3
//            rows 1 / 1.03 / 0.98, 12 of 2^21 1 / 1.03 / 0.98, groups of 64, 8 of 2^20.8 1 / 1.08 / 1.00, 12 of 2^21 1 / 1.17 / 0.99
//            4 bits, groups of 64 and 128, 2^23.3 rows 1 / 1.05 / 1.02, 2^23.2 1 / 1.03 / 1.01 (2^25 1.20 with this shape: 1 / 1.00)
//            2 bits, groups of 32, 32 of 2^18.3 rows 1 / 1.04 / 1.00
//   paged    2 bits, groups of 64 and 128, 2^23.2 to 2^24 rows 1 / 1.07 to 1.10 / 0.99; groups of 32, 7 of 2^20.8 rows and 6 of 2^21 1 /
//            1.10 / 0.97, 32 of 2^18.3 1 / 1.07 / 0.97, 3 bits 1 / 1.04 / 1.00
// One paged request, 3 bits, groups of 32, K and V together, two workgroups per unit in place of three below 2^21.4 rows (three with
// arguments read where they are used, as the kernels were for a while / three / two, inputs in turn): 2^19.3 rows - / 90.3 / 89.9 us, 2^20
// 128.5 / 131.9 / 128.1, 2^21 242 / 255 / 241, 2^21.3 - / 324 / 299, 2^21.38 - / 324 / 318, 2^21.43 - / 332 / 333, 2^21.5 - / 361 / 381, 2^22 525 /
// 494 / 518, fp16 and bf16 alike.  (Calls repeated on one payload show two as the better one up to 2^23 rows.  Groups of 64 and 128
// lose 19 to 23 % by it.  2 bits had 126 and 233 us at 2^20 and 2^21 rows, now 128 and 246, at 2^22 554, now 495; no other shape is better.)
// Four requests of 2^20 rows (16 workgroups for every resident one) are better off as a single one is: 0.88 to 0.98.
template <int BITS> static DecodeShape decode_shape(unsigned wgs, bool both, bool dense, bool transform, int group, bool one)
{
    constexpr unsigned kResident = 4 * 256;
    const bool g32 = group == 32, large = !both && wgs >= 16 * kResident;
    if (transform || BITS == 8) return {};
    const bool several = !one && (wgs < 8 * kResident || wgs >= 24 * kResident);
    if (!dense) {
        if (BITS == 4 || wgs < 5 * kResident / 2) return {};
        if (BITS == 3 && g32 && both && one && wgs < 21 * kResident / 2) return {40000, 0};
        if (g32 && several) return {0, BITS == 3 ? 16 : 0};
        return {!large || (BITS == 2 && !g32 && one && wgs < 48 * kResident) ? 14000u : 0u, 0};
    }
    if (BITS < 4 && !g32 && one && wgs >= 2 * kResident && wgs < 3 * kResident)
        return BITS == 3 && wgs >= 5 * kResident / 2 ? DecodeShape{14000, 64} : DecodeShape{0, 16};
    if (wgs < 3 * kResident) return {};
    if (BITS < 4 && g32 && several) return {BITS == 3 ? 14000u : 0u, 16};
    if (BITS == 3 && group == 64 && several && wgs >= 24 * kResident) return {14000, 16};
    if (large && BITS == 4 && !g32 && one && wgs < 48 * kResident) return {14000, 64};
    if (large) return {BITS == 3 ? 14000u : 0u, 16};
    return {BITS == 2 || (BITS == 3 && !g32 && one) ? 14000u : BITS == 3 ? 40000u : 0u, 64};
}

template <int BITS, int DT, int KV> static int decode_launch(const CoderBatch &b, hipStream_t s)
{
    constexpr int NW = ChunkGeom<BITS>::kDecWaves;
    CoderBatch placed = b;
    unsigned need = 0;
    for (int i = 0; i < b.n; ++i) {
        placed.at.start[i] = need;
        need += (unsigned)((item_chunks(b, i) + NW - 1) / NW);
    }
    if (need == 0) return KVC_OK;
    const dim3 grid(need), block(NW * 64);
    const int tr = b.rotate ? 1 : !item_has_anchors(b.item[0]) ? 0 : b.anchor_shift >= 5 ? 2 : 3;
    const DecodeShape shape = decode_shape<BITS>(need, KV == 2, b.dense != 0, tr != 0, b.group[b.item[0].flags >> 7 & 1], b.n <= (KV == 2 ? 2 : 1));
    close_places(placed.at, b.n, need, shape.run);
#define KVC_DECODE(D, T) hipLaunchKernelGGL((decode_kernel<BITS, DT, KV, D, T>), grid, block, shape.lds, s, placed)
    if (KV == 2) {
        if (tr != 0) return KVC_ERR_UNSUPPORTED;
        if (b.dense) KVC_DECODE(true, 0); else KVC_DECODE(false, 0);
        return launched();
    }
    // (the transforms are not instantiated for both tensors together)
    constexpr int kRot = KV == 2 ? 0 : 1, kOne = KV == 2 ? 0 : 2, kShort = KV == 2 ? 0 : 3;
    if (b.dense) {
        if (tr == 0) KVC_DECODE(true, 0); else if (tr == 1) KVC_DECODE(true, kRot); else if (tr == 2) KVC_DECODE(true, kOne); else KVC_DECODE(true, kShort);
    } else {
        if (tr == 0) KVC_DECODE(false, 0); else if (tr == 1) KVC_DECODE(false, kRot); else if (tr == 2) KVC_DECODE(false, kOne); else KVC_DECODE(false, kShort);
    }
#undef KVC_DECODE
    return launched();
}

#define KVC_PASTE2(a, b) a##b
#define KVC_PASTE(a, b) KVC_PASTE2(a, b)

int KVC_PASTE(launch_decode_bits, KVC_BITS)(int kv, int dtype, const CoderBatch &a, hipStream_t s)
{
    switch (kv) {
    case 0: return dtype == DT_F16 ? decode_launch<KVC_BITS, DT_F16, 0>(a, s) : decode_launch<KVC_BITS, DT_BF16, 0>(a, s);
    case 1: return dtype == DT_F16 ? decode_launch<KVC_BITS, DT_F16, 1>(a, s) : decode_launch<KVC_BITS, DT_BF16, 1>(a, s);
    }
    return dtype == DT_F16 ? decode_launch<KVC_BITS, DT_F16, 2>(a, s) : decode_launch<KVC_BITS, DT_BF16, 2>(a, s);
}

}  // namespace kvc
