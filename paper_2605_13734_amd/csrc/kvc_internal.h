// Host-side declarations shared by the translation units of libkvc (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kvc_device.h"

namespace kvc {

// The stage T that a kernel has (XF): none, the delta transform, the rotation.  Every one has kernels of its own: what the plain
// ones do not use costs them registers (64 and 128 rows of K: 98 and 162 fp16 registers, 205 and 402 with both) and moves their
// loads, and the lanes of the rotation hold their rows in another order (lane_octet).
constexpr int kNoTransform = 0, kDelta = 1, kRotation = 2;

// Arguments of the codec-free quantize / dequantize kernels for one tensor of one request.
struct QuantArgs {
    TensorView x;               // source (compress) or destination (decompress)
    uint8_t *codes;             // section base inside the payload
    uint8_t *meta;              // metadata section base
    long long tokens;
    int heads;
    int group;                  // runtime copy of the group size
    int dense;                  // rows of a head are contiguous: stride_token == head_dim, no block table
    int head_minor;             // the heads of a token lie next to each other (stride_head < stride_token, as in a
                                // paged pool): neighbouring work units then take the same tokens of neighbouring heads
    int rotate;                 // stage T: rows are Hadamard-transformed on the way in / back on the way out
    // stage T, delta transform: the tensor's anchor rows inside the payload,
    // [layer * heads + head][ceil(tokens / period)][128] (null = transform off), period = 1 << anchor_shift
    uint16_t *anchors;
    int anchor_shift;
    // per-head bit widths (null = one width for all heads): the heads this launch covers, and for
    // every head the sum of the widths of the heads before it (its codes start at that many times
    // tokens * 16 bytes into the section)
    const int *head_list;
    const long long *bits_before;
    long long units_per_head;   // work units (one wave each) per (layer, head)
    long long total_units;
    int *status;                // device status word of the request
};

// Where the workgroups of a launch go: to the items of its batch, one item after the other.
template <int N> struct Places {
    unsigned start[N];          // first place of every item, the largest number for items that are not there
    unsigned run_end;           // places below are given out in runs (see place_of_workgroup); 0: none
    int run_shift;
};

// Closes the table behind item n - 1, `total` places in all.  run: a power of two, or 0.
template <int N> static inline void close_places(Places<N> &at, int n, unsigned total, int run)
{
    for (int i = n; i < N; ++i) at.start[i] = ~0u;
    at.run_shift = 0;
    while (run > 1 << at.run_shift) ++at.run_shift;
    at.run_end = run ? total & ~(8u * (unsigned)run - 1u) : 0;
}

// The workgroup's place.  The hardware deals workgroups to the eight XCDs in turn, so that without runs neighbouring
// pieces of a tensor go through eight L2s at a time.  With them every XCD gets 2^run_shift places in a row; the last,
// incomplete round stays as it is.  Which XCD a workgroup really runs on changes the speed only.  A kernel that just
// writes 5 GB, 32 KB per workgroup: 5.6 TB/s without runs, 6.6 with an eighth of the places each; what the kernels
// here gain is at launch_shape and decode_shape.
template <int N> __device__ __forceinline__ unsigned place_of_workgroup(const Places<N> &at)
{
    const unsigned id = blockIdx.x, in_round = (8u << at.run_shift) - 1u;
    const unsigned in_runs = (id & ~in_round) + ((id & 7u) << at.run_shift) + ((id & in_round) >> 3);
    return id < at.run_end ? in_runs : id;
}

// The item of a place, and the place's number among the item's (the same in all lanes).
template <int N> __device__ __forceinline__ int place_item(const Places<N> &at, unsigned place, unsigned &wg)
{
    int i = 0;
    while (i + 1 < N && place >= at.start[i + 1]) ++i;
    wg = place - at.start[i];
    return i;
}

// The same for the coder's many items: the first eight starts are read together and compared without branches, instead of one
// scalar load after the other at the start of every wave (one layer of 32k tokens, 4 bits, decompress call 44 -> 41.6 us; the codec-free
// compressions lose 3 % by it).  Launches with more items look up the eight and then the one of it (for all launches: 1 us of 41).
template <int N> __device__ __forceinline__ int place_item_of_many(const Places<N> &at, unsigned place, unsigned &wg)
{
    const auto one_of_eight = [&](const unsigned *start, int eight) {
        int item = eight;
        unsigned first = start[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) {
            const bool here = place >= start[k];
            item += here ? 1 : 0;
            first = here ? start[k] : first;
        }
        wg = place - first;
        return item;
    };
    unsigned s[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) s[k] = at.start[k];
    asm volatile("" : "+s"(s[0]), "+s"(s[1]), "+s"(s[2]), "+s"(s[3]), "+s"(s[4]), "+s"(s[5]), "+s"(s[6]), "+s"(s[7]), "+s"(s[8]));
    if (__builtin_expect(place < s[8], 1)) return one_of_eight(s, 0);
    int eight = 8;
#pragma unroll
    for (int k = 16; k < N; k += 8) eight += place >= at.start[k] ? 8 : 0;
    return one_of_eight(at.start + eight, eight);
}

// The same tensor (K or V) of several requests of a call in one launch, their workgroups one request
// after the other.
// All items take the same kernel (same plan; same layout class, see QuantArgs::dense).
constexpr int kQuantBatch = 12;     // (the argument block stays below 4 KB)
struct QuantBatch {
    QuantArgs item[kQuantBatch];
    Places<kQuantBatch> at;             // (set by the launcher)
    int n;
    int pace;                           // decompression: see launch_shape (set by the launcher)
};

// Geometry of one payload (all byte counts), shared by host code of compress / decompress.
struct Geometry {
    long long meta_k, meta_v, aux, codes_k, codes_v;
    long long aux_base;          // tables / directory part of the auxiliary section (before the anchors)
    long long code_tables;       // bytes of the coder's tables at the start of the auxiliary section (0, 512 or 2048)
    long long off_dir;           // the coder's directory
    long long off_widths, widths;    // the per-head width tables
    long long anchors_k, anchors_v, off_anchors_k, off_anchors_v;
    long long off_meta_k, off_meta_v, off_aux, off_codes_k, off_codes_v, total;
    long long chunks_k, chunks_v;
};

struct HeaderBytes { uint32_t w[32]; };

int launch_compress_tensor(int is_v, int bits, int group, int dtype, const QuantBatch &b, hipStream_t s);
int launch_decompress_tensor(int is_v, int bits, int group, int dtype, const QuantBatch &b, hipStream_t s);
// one translation unit per code width (kvc_quant.hip compiled with -DKVC_BITS=...)
#define KVC_DECLARE_QUANT(B)                                                                              \
    int launch_compress_bits##B(int is_v, int group, int dtype, const QuantBatch &b, hipStream_t s);     \
    int launch_decompress_bits##B(int is_v, int dtype, const QuantBatch &b, hipStream_t s);
KVC_DECLARE_QUANT(2) KVC_DECLARE_QUANT(3) KVC_DECLARE_QUANT(4) KVC_DECLARE_QUANT(8)
#undef KVC_DECLARE_QUANT
// Service work of one request before its tensors are compressed (see compress_prologue_kernel).
struct PrologueItem {
    uint32_t *payload;              // request payload base
    HeaderBytes header;
    long long pad_off[2];           // zero padding: byte offset inside the payload, 32-bit words
    int pad_words[2];
    const uint32_t *aux_src;        // device image of the width tables, copied to payload + aux_off
    long long aux_off, aux_words;
    uint32_t *zero;                 // coder scratch that starts from zero: candidate tables, ticket and scan state
    long long zero_words;
    unsigned long long *out_bytes;  // the request's size word
    unsigned long long total;
    int write_total;                // the size is known on the host (no coder, or an empty request)
    uint32_t *dir0;                 // empty request with the coder: the directory's only entry
    int *status;
};
constexpr int kPrologueBatch = 16;  // requests per launch (the argument block stays below 4 KB)
struct PrologueArgs {
    PrologueItem item[kPrologueBatch];
    int n;
};
static_assert(sizeof(PrologueArgs) <= 4000, "kernel arguments are limited to 4 KB");

// The request's status word and header, the zero padding between the parts of the payload, the width
// tables (copied from their device image), the coder's candidate tables, work-order counter and scan state, and whatever the
// host already knows of the result (the payload size without the coder; the closed directory of an empty
// request).  By `step` threads together, the calling one being number `first`.
__device__ __forceinline__ void write_prologue(const PrologueItem &it, long long first, long long step)
{
    if (first < 32) it.payload[first] = it.header.w[first];
    if (first == 32) *it.status = 0;
    if (first == 33 && it.write_total) *it.out_bytes = it.total;
    if (first == 34 && it.dir0) *it.dir0 = 0;
    for (int k = 0; k < 2; ++k)
        for (long long i = first; i < it.pad_words[k]; i += step) it.payload[it.pad_off[k] / 4 + i] = 0;
    for (long long i = first; i < it.aux_words; i += step) it.payload[it.aux_off / 4 + i] = it.aux_src[i];
    for (long long i = first; i < it.zero_words; i += step) it.zero[i] = 0;
}

// workgroups of 256 threads that share the zero fill of `words` words: 16 words per thread
static inline unsigned fill_slices(long long words)
{
    const long long n = (words + 4095) / 4096;
    return (unsigned)(n < 1 ? 1 : (n > 256 ? 256 : n));
}

// A small call without the coder in one launch (see compress_call_kernel): K and V of its requests in turn.
constexpr int kSmallRequests = 4;
struct SmallCompressArgs {
    QuantArgs item[2 * kSmallRequests];
    Places<2 * kSmallRequests> at;              // (set by the launcher)
    int n, requests;
    PrologueItem prologue[kSmallRequests];
};
struct SmallCheck {
    const uint32_t *payload;
    HeaderBytes expect;
};
struct SmallDecompressArgs {
    QuantArgs item[2 * kSmallRequests];
    Places<2 * kSmallRequests> at;
    int n, requests;
    SmallCheck check[kSmallRequests];
};
static_assert(sizeof(SmallCompressArgs) <= 4000 && sizeof(SmallDecompressArgs) <= 4000, "kernel arguments are limited to 4 KB");
int launch_compress_call(int bits, int group, int dtype, SmallCompressArgs &b, hipStream_t s);
int launch_decompress_call(int bits, int dtype, SmallDecompressArgs &b, hipStream_t s);
#define KVC_DECLARE_CALL(B)                                                                              \
    int launch_compress_call_bits##B(int group, int dtype, SmallCompressArgs &b, hipStream_t s);        \
    int launch_decompress_call_bits##B(int dtype, SmallDecompressArgs &b, hipStream_t s);
KVC_DECLARE_CALL(2) KVC_DECLARE_CALL(3) KVC_DECLARE_CALL(4) KVC_DECLARE_CALL(8)
#undef KVC_DECLARE_CALL

// Header (and width table) check of one request before it is decompressed.
struct CheckItem {
    const uint32_t *payload;
    HeaderBytes expect;
    const uint8_t *tables, *plan_tables;    // width tables in the payload and their device image
    long long table_bytes;
    int *status;
};
constexpr int kCheckBatch = 20;
struct CheckArgs {
    CheckItem item[kCheckBatch];
    int n;
};

int launch_compress_prologue(const PrologueArgs &a, hipStream_t s);
int launch_decompress_prologue(const CheckArgs &a, hipStream_t s);
int launch_fill_u32(uint32_t *dst, uint32_t value, long long n, hipStream_t s);

// ---- lossless stage (codec 1) -----------------------------------------------------------

// Code tables of a request: one per tensor, or with per-head widths one per tensor and width
// (slot 4 * is_v + index of the width in 2, 3, 4, 8).
constexpr int kTableSlots = 8;

// Chunks of a tensor (of a width of a tensor) that its code table is made from.
constexpr int kSampleChunks = 16;

// Per-request scratch inside the caller's workspace (device memory).
struct CoderScratch {
    uint16_t *sample;           // [slots][kSampleChunks][256] byte counts of the sample chunks
    uint16_t *lut;              // [kTableSlots][4096] decode table: symbol << 8 | (256 - length); while compressing, its end holds
                                // the candidates for the slots' code tables (CandidateTables)
    unsigned long long *state;  // scan state, one word per encode workgroup (in launch order)
    uint32_t *ticket;           // work-order counter, right behind `lut`
};

// The code tables of a slot for 0, 1, ... halvings of the sample's weights (see build_table).  They are built by workgroups of the
// launch that uses them, so every word says by itself whether it has been written: it starts from zero (the prologue's zero
// fill), and no entry is zero (a length is 1 or more).
constexpr int kCandidates = 11;
constexpr uint32_t kComplete = 1, kTooLong = 2;
struct CandidateTables {
    uint32_t state[32];                     // of every candidate (one line of memory for those who wait): kComplete, or kTooLong:
                                            // it exceeds the length limit and has no entries
    uint32_t entry[kCandidates][128];       // two per word: code | length << 12, by byte value
};
static_assert(sizeof(CandidateTables) <= 4096 * 2 && sizeof(CandidateTables) % 128 == 0, "fits the slot's decode table");

// slot 0 lies right in front of the ticket, the others in front of it: one range to fill with zeros
__host__ __device__ __forceinline__ CandidateTables *candidate_tables(uint32_t *ticket, int slot)
{
    return (CandidateTables *)ticket - (slot + 1);
}

// Chunks (= waves) per encoder workgroup, 8-bit chunks with twice the LDS: two.
// A workgroup reports its sizes when its slowest wave knows its own, so fewer chunks wait less for
// each other, and every workgroup costs a ticket and a state word (70B shape, 4 bits, half of the layers:
// eight 1325 us, four 1226, two 1600).
constexpr int enc_waves(int bits) { return bits == 8 ? 2 : 4; }

// Waves per SIMD the register allocation must leave room for: the variants that come close to 128 registers
// by themselves (2- to 4-bit codes, groups of 32, the dense layout or both tensors together; not the V
// kernels with the transforms for bf16 rows or 3-bit codes) are held to four; the others would spill, so
// they keep what they need.
// `transform`: the launch applies stage T.
constexpr int enc_min_waves(int bits, int group, int dtype, bool dense, bool is_v, bool transform)
{
    return bits != 8 && group == 32 && dense && !(is_v && transform && (dtype == DT_BF16 || bits == 3)) ? 4 : 1;
}

// One launch of the coder: a tensor, or with per-head widths the heads of one width of a tensor
// (q.head_list); the launches of a request follow each other in chunk order (K before V, widths
// ascending) and share the ticket counter and the scan state.
struct CoderArgs {
    QuantArgs q;                // tensor, meta, tokens, status ...
    uint8_t *payload;           // request payload base
    long long off_aux;          // the code tables (256 length bytes per slot)
    long long off_dir;          // the directory
    long long off_bodies;       // first chunk body (= K codes offset)
    long long capacity;         // payload bytes available
    long long chunks;           // chunks of this launch
    long long chunk_base;       // directory index of this launch's first chunk
    long long wg_base;          // scan-state index of this launch's first workgroup
    long long k_wgs;            // encode workgroups of all K launches
    long long total_wgs;        // encode workgroups of all launches of the request
    long long total_chunks;     // K and V together
    int is_v;
    int tab;                    // table slot of this launch
    int builders;               // workgroups of the request that build code tables: those with the first tickets (see build_table)
    int apart;                  // ... and have no chunks: tickets in front of the first chunk's (builders or 0)
    int slots;                  // table slots of the format (bits 31:8) and those in use (bits 7:0, a bit each)
    CoderScratch ws;
    unsigned long long *out_bytes;   // device: true payload size (written by the last workgroup)
};

// One launch of the encoder or decoder for the requests of a window (see request_window), the items' workgroups one
// after the other: a launch of every request (one tensor and width), or, where K and V share a launch, a
// K and a V item of every request.  All items have one width and take the same kernel.
// A launch costs a start and a tail of about 29 us with the encoder (4 bits, launches of 5000 to 9000 workgroups: 29 us + 0.031 a
// workgroup), so a batch holds as many requests as 4 KB of arguments allow: an item has what differs from request to request
// in 112 bytes, the batch what does not, and the kernels put CoderArgs together from both (coder_args).  32 requests of 512 to 2048
// tokens, 256 heads, 4 bits, in windows of twelve with CoderArgs for items / in one: 1356 / 1224 us.
struct CoderItem {
    uint16_t *base;             // TensorView
    long long stride_layer, stride_head, stride_token, stride_block;
    const int *block_table;
    uint8_t *payload;
    long long capacity;
    long long tokens;
    int num_phys_blocks;
    // inside the payload, of 16 bytes: the low words; four bits more of each are in `flags` (1 TB)
    uint32_t off_meta, off_aux, off_bodies, off_anchors;      // (off_anchors: 0 = no delta transform)
    uint32_t chunk_base, wg_base, k_wgs, total_wgs;
    uint32_t flags;             // bits 4:0 TensorView::bt_shift, 5 bt_wave, 6 QuantArgs::head_minor, 7 is_v, 10:8 tab, 15:11 number of the
                                // request behind the window's first, 19:16, 23:20, 27:24, 31:28 bits 35:32 of the places above
};
static_assert(sizeof(CoderItem) == 112, "what a batch of 32 has room for");
constexpr int kCoderBatch = 32;     // (the argument block stays below 4 KB, a request's number has five bits)
struct CoderBatch {
    CoderItem item[kCoderBatch];
    Places<kCoderBatch> at;             // (encoder, both tensors together: the items are the requests; set by the launcher)
    // The same for all items.  (Whole words only: a 16-bit member, indexed by the tensor, made the compiler take the address of
    // the word-sized ones apart into a base and an offset of two bytes too many and too few, and scalar loads drop the two lowest
    // bits of either, so that the V launches with width tables read half of each of two pointers.)
    // The window's first request's scratch (and its size), status and size words
    uint8_t *ws;
    long long ws_request;
    int *status;
    unsigned long long *out_bytes;
    const int *head_list[2];            // of K and of V, like the next two
    int heads_covered[2];               // heads of the launch
    int group[2];
    uint32_t ws_lut, ws_ticket, ws_state;       // places inside a request's scratch
    int heads, all_heads;               // KV heads of a layer, of all layers
    int dense, rotate, anchor_shift;
    int builders, apart, slots;
    int n;
    int waves;                          // encoder, both tensors together: chunks per workgroup
    unsigned front;                     // encoder: workgroups of every request in front of the items' places (the request's
                                        // first launch: CoderArgs::apart; others: none)
};

static inline bool item_has_anchors(const CoderItem &it) { return (it.off_anchors | (it.flags >> 28)) != 0; }

static inline long long item_chunks(const CoderBatch &b, int item)
{
    return b.heads_covered[(b.item[item].flags >> 7) & 1] * ((b.item[item].tokens + kChunkRows - 1) / kChunkRows);
}

// The k-th of an item's places inside the payload, in bytes; `low` is its low word.
__host__ __device__ __forceinline__ long long item_place(uint32_t low, uint32_t flags, int k)
{
    return (long long)((unsigned long long)((flags >> (16 + 4 * k)) & 15u) << 32 | low) << 4;
}

// KV: the launch's tensor, K (0), V (1) or both (2).  AT_ONCE: what a wave's first loads need of the item is requested together, not
// where it is used (decoder).
template <int KV, bool AT_ONCE = false> __device__ __forceinline__ CoderArgs coder_args(const CoderBatch &b, int item)
{
    CoderItem it = b.item[item];
    if (AT_ONCE)
        asm volatile("" ::"s"(it.payload), "s"(it.capacity), "s"(it.tokens), "s"(it.off_aux), "s"(it.off_bodies), "s"(it.chunk_base), "s"(it.flags));
    const bool is_v = KV == 2 ? ((it.flags >> 7) & 1) != 0 : KV == 1;
    CoderArgs a = {};
    a.q.x.base = it.base;
    a.q.x.stride_layer = it.stride_layer;
    a.q.x.stride_head = it.stride_head;
    a.q.x.stride_token = it.stride_token;
    a.q.x.stride_block = it.stride_block;
    a.q.x.block_table = it.block_table;
    a.q.x.bt_shift = it.flags & 31;
    a.q.x.num_phys_blocks = it.num_phys_blocks;
    a.q.x.bt_wave = (it.flags >> 5) & 1;
    a.q.meta = it.payload + item_place(it.off_meta, it.flags, 0);
    a.q.tokens = it.tokens;
    a.q.heads = b.heads;
    a.q.group = is_v ? b.group[1] : b.group[0];
    a.q.dense = b.dense;
    a.q.head_minor = (it.flags >> 6) & 1;
    a.q.rotate = b.rotate;
    a.q.anchors = it.off_anchors | (it.flags >> 28) ? (uint16_t *)(it.payload + item_place(it.off_anchors, it.flags, 3)) : nullptr;
    a.q.anchor_shift = b.anchor_shift;
    a.q.head_list = is_v ? b.head_list[1] : b.head_list[0];
    const int request = (int)((it.flags >> 11) & 31);
    a.q.status = b.status + request;
    a.payload = it.payload;
    a.off_aux = item_place(it.off_aux, it.flags, 1);
    a.off_dir = a.off_aux + 256 * (b.slots >> 8);
    a.off_bodies = item_place(it.off_bodies, it.flags, 2);
    a.capacity = it.capacity;
    const uint32_t per_head = (uint32_t)((unsigned long long)(it.tokens + kChunkRows - 1) / kChunkRows);     // (no request has 2^31 chunks)
    a.chunks = (uint32_t)(is_v ? b.heads_covered[1] : b.heads_covered[0]) * per_head;
    a.chunk_base = it.chunk_base;
    a.wg_base = it.wg_base;
    a.k_wgs = it.k_wgs;
    a.total_wgs = it.total_wgs;
    a.total_chunks = 2 * (uint32_t)b.all_heads * per_head;
    a.is_v = is_v;
    a.tab = (it.flags >> 8) & 7;
    a.builders = b.builders;
    a.apart = b.apart;
    a.slots = b.slots;
    uint8_t *ws = b.ws + request * b.ws_request;
    a.ws.sample = (uint16_t *)ws;
    a.ws.lut = (uint16_t *)(ws + b.ws_lut);
    a.ws.state = (unsigned long long *)(ws + b.ws_state);
    a.ws.ticket = (uint32_t *)(ws + b.ws_ticket);
    a.out_bytes = b.out_bytes + request;
    return a;
}

// The same number (in a scalar register), but one that the compiler knows nothing of.  What is put together from an item's number taken
// this way is put together there, and not kept in registers from an earlier part of the kernel; what depends on an anchor period taken
// this way is not computed in front of a loop for all its passes.
__device__ __forceinline__ int anew(int number)
{
    int n = __builtin_amdgcn_readfirstlane(number);
    asm volatile("" : "+s"(n));
    return n;
}
static_assert(sizeof(CoderBatch) <= 4000, "kernel arguments are limited to 4 KB");
static_assert(sizeof(QuantBatch) <= 4000, "kernel arguments are limited to 4 KB");

// Set-up of the requests of a call that is compressed with the coder: the prologue and the table samples
// of every request in one launch.
struct SetupTable {             // a table of the plan, the same for all requests
    const int *head_list;       // the heads it covers (null: all in their own order)
    int heads_covered, slot, is_v, bits, group;
    int anchor_shift;           // delta transform of this tensor (-1: none)
    int rotate;
};
struct SetupItem {
    PrologueItem prologue;
    TensorView x;               // the request's K
    uint16_t *v_base;           // and where V lies
    long long tokens;
    uint16_t *sample;           // CoderScratch::sample
};
constexpr int kSetupBatch = 8;  // requests per launch (the argument block stays below 4 KB)
struct SetupArgs {
    SetupItem item[kSetupBatch];
    SetupTable table[kTableSlots];
    int n, tables, heads;
};
static_assert(sizeof(SetupArgs) <= 4000, "kernel arguments are limited to 4 KB");

// Set-up of the requests of a call that is decompressed with the coder (see decode_setup_kernel).
struct DecodeSetupItem {
    const uint32_t *payload;
    HeaderBytes expect;
    long long off_aux;                      // the code tables' lengths inside the payload
    const uint8_t *tables, *plan_tables;    // width tables in the payload and their device image
    long long table_bytes;
    uint16_t *lut;
    int *status;
};
constexpr int kDecodeSetupBatch = 20;
struct DecodeSetupArgs {
    DecodeSetupItem item[kDecodeSetupBatch];
    uint32_t mask;                          // bit i = compare header word i
    int n, slots, slot_mask;
};
static_assert(sizeof(DecodeSetupArgs) <= 4000, "kernel arguments are limited to 4 KB");

int launch_setup(int dtype, const SetupArgs &a, hipStream_t s);
// kv: the tensor of the launch, K (0), V (1) or both (2: a K and a V item of every request in turn)
// resident: launch nothing, but say how many workgroups of the kernel the chip has at once (0: unknown)
int launch_encode_section(int kv, int bits, int group, int dtype, const CoderBatch &b, hipStream_t s, int *resident = nullptr);
int launch_decode_setup(const DecodeSetupArgs &a, hipStream_t s);
int launch_decode_section(int kv, int bits, int dtype, const CoderBatch &b, hipStream_t s);
// one translation unit per code width (kvc_huff_enc.hip / kvc_huff_dec.hip compiled with -DKVC_BITS=...)
#define KVC_DECLARE_CODER(B)                                                                  \
    int launch_encode_bits##B(int kv, int group, int dtype, const CoderBatch &b, hipStream_t s, int *resident); \
    int launch_decode_bits##B(int kv, int dtype, const CoderBatch &b, hipStream_t s);
KVC_DECLARE_CODER(2) KVC_DECLARE_CODER(3) KVC_DECLARE_CODER(4) KVC_DECLARE_CODER(8)
#undef KVC_DECLARE_CODER

}  // namespace kvc
