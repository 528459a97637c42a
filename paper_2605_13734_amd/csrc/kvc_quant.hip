// Codec-free kernels: quantize + pack (compress) and unpack + dequantize (decompress) one
// tensor of one request straight between the KV layout and the payload sections.
// One wave per work unit, four units per workgroup, no barriers.
//   K compress unit   = one token block of G rows x 128 channels (all 128 per-channel groups)
//   other units       = 32 token rows
// Stage Q of the pipeline (KVServe section 5.1); memory-bound, so no matrix cores.
// Compiled once per code width (-DKVC_BITS=2, 3, 4 or 8).

#include "kvc_quant.h"

#ifndef KVC_BITS
#error "compile with -DKVC_BITS=2, 3, 4 or 8"
#endif

namespace kvc {

// Waves per SIMD the register allocation must leave room for.  Left alone, the compiler gives the kernels for
// bf16 rows that are not dense 117 to 123 registers where 77 to 80 do: four waves instead of six (8-bit codes
// would spill below 82: five).  K token blocks of 64 and 128 rows need more, dense and fp16 rows are left
// alone.  Paged bf16, 32 layers of 16384 tokens, 4 bits, compress call with four and with six waves: with the
// rotation 678 and 619 us, with runs of 8 tokens 847 and 784, without a transform 487 and 471.
constexpr int min_waves(int bits, int rows, int dtype, bool dense)
{
    return dtype == DT_BF16 && !dense && rows == kPassRows ? (bits == 8 ? 5 : 6) : 1;
}

// ---- K: groups along tokens, one per channel ------------------------------------------------

// XF: see kNoTransform.  Sharing a kernel with the code of stage T doubles the registers of the plain path for token blocks
// of 64 and 128 rows.
// IN_CALL: a unit of compress_call_kernel.  There 8-bit bf16 loads stay where the compiler puts them: where all workgroups
// are resident, requesting them together loses 3 % (groups of 32, 2^16 and 2^17 rows 11.3 -> 11.6, 19.7 -> 20.5 us), and narrower
// ones are requested together for V as well (4 bits, 2^16 rows 10.8, K alone 11.0, both 10.5).  Dense rotated blocks of 128 rows at 8 bits
// stay as they are, too: from 2^21 rows on requesting them together is 3 % slower (below it was up to 9 % faster).
template <int BITS, int G, int DT, bool DENSE, int XF, bool IN_CALL = false>
__device__ __forceinline__ void compress_k_unit(const QuantArgs &a, unsigned wg, float *xch_all)
{
    UnitPos u;
    if (!unit_pos(a, wg, u)) return;
    constexpr int P = G / kPassRows;
    const long long row0 = u.blk * G;
    bool bad = false;
    u32x4 raw[P * 8];
#pragma unroll
    for (int p = 0; p < P; ++p) load_pass<DENSE, XF == kRotation>(a.x, u.head_off, row0 + p * kPassRows, a.tokens, raw + p * 8, bad);
    if (BITS < 8 || !(IN_CALL || (DENSE && XF == kRotation && P == 4))) rows_requested<DENSE, DT, XF, P>();
    if (XF == kRotation) rotate_rows<DT, P * 8, false>(raw);
    if (XF == kDelta && a.anchors)
        delta_rows<DT, DENSE, P * 8>(a.x, u.head_off, row0, a.tokens, a.anchor_shift,
                                     head_anchors(a.anchors, u.lh, a.tokens, a.anchor_shift), true, raw, bad);
    KParams kp;
    uint8_t *meta_block = a.meta + (u.lh * a.units_per_head + u.blk) * (kDim * 4);
    k_group_params<BITS, DT, P * 8, 16, XF == kRotation>(raw, (uint8_t *)(xch_all + wave_id() * kXchFloats), meta_block, kp);
    forget_unpacked<DT, P * 8>(raw);
    uint8_t *codes = head_codes<BITS>(a, u.lh) + row0 * (16 * BITS);
    const long long left = a.tokens - row0;
    k_emit<BITS, DT, P, false, XF == kRotation>(raw, kp, codes, left < G ? (int)left : G);
    report(a.status, bad);
}

template <int BITS, int G, int DT, bool DENSE, int XF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(min_waves(BITS, G, DT, DENSE))))
void compress_k_kernel(QuantBatch b)
{
    __shared__ __attribute__((aligned(16))) float xch_all[4 * kXchFloats];
    unsigned wg;
    const QuantArgs &a = b.item[place_item(b.at, place_of_workgroup(b.at), wg)];
    compress_k_unit<BITS, G, DT, DENSE, XF>(a, wg, xch_all);
}

// `refused()`: the request's payload does not fit the plan; asked once everything a unit reads is requested.
// XF: the inverse transform that it has.  PACED: with waits between the row stores (without a transform only).
template <int BITS, int DT, bool DENSE, int XF, bool PACED, class Refused>
__device__ __forceinline__ void decompress_k_unit(const QuantArgs &a, unsigned wg, int pace, Refused &&refused)
{
    UnitPos u;
    if (!unit_pos(a, wg, u)) return;
    const int col = lane_octet(XF == kRotation);
    const long long row0 = u.blk * kPassRows;
    const long long tb = row0 / a.group, nb = (a.tokens + a.group - 1) / a.group;
    const u32x4 *m = (const u32x4 *)(a.meta + ((u.lh * nb + tb) * kDim + col * 8) * 4);
    const u32x4 m0 = m[0], m1 = m[1];
    uint8_t *codes = head_codes<BITS>(a, u.lh) + row0 * (16 * BITS);
    const long long left = a.tokens - row0;
    const int rows = left < kPassRows ? (int)left : kPassRows;
    PassFetch f;
    pass_fetch<BITS, DENSE, 0, XF == kRotation>(f, codes, a.x, u.head_off, row0, rows);
    if (refused()) return;
    float scale[8], zero[8];
    const bool clamp = k_meta_floats<BITS, DT>(m0, m1, scale, zero);
    bool bad = false;
    const uint16_t *anchors = XF == kDelta ? head_anchors(a.anchors, u.lh, a.tokens, a.anchor_shift) : nullptr;
    if (XF == kRotation) dequant_pass<BITS, DT, false, DENSE, 1>(f, scale, zero, clamp, a.x, u.head_off, row0, rows, bad);
    else if (XF == kDelta && a.anchor_shift >= 5) dequant_pass<BITS, DT, false, DENSE, 2>(f, scale, zero, clamp, a.x, u.head_off, row0, rows, bad, anchors, a.anchor_shift);
    else if (XF == kDelta) dequant_pass<BITS, DT, false, DENSE, 3>(f, scale, zero, clamp, a.x, u.head_off, row0, rows, bad, anchors, a.anchor_shift);
    else dequant_pass<BITS, DT, false, DENSE, 0, PACED>(f, scale, zero, clamp, a.x, u.head_off, row0, rows, bad, nullptr, 0, nullptr, pace);
    report(a.status, bad);
}

template <int BITS, int DT, bool DENSE, int XF, bool PACED>
__global__ __launch_bounds__(256) void decompress_k_kernel(QuantBatch b)
{
    unsigned wg;
    const QuantArgs &a = b.item[place_item(b.at, place_of_workgroup(b.at), wg)];
    const int status = *a.status;
    decompress_k_unit<BITS, DT, DENSE, XF, PACED>(a, wg, b.pace, [&]() { return (status & KVC_DEV_BAD_HEADER) != 0; });
}

// ---- V: groups along channels, one set per token -----------------------------------------------

template <int BITS, int GV, int DT, bool DENSE, int XF, bool IN_CALL = false>
__device__ __forceinline__ void compress_v_unit(const QuantArgs &a, unsigned wg)
{
    UnitPos u;
    if (!unit_pos(a, wg, u)) return;
    constexpr int NG = kDim / GV;
    const long long row0 = u.blk * kPassRows;
    bool bad = false;
    u32x4 raw[8];
    load_pass<DENSE, XF == kRotation>(a.x, u.head_off, row0, a.tokens, raw, bad);
    if (BITS < 8 && IN_CALL) rows_requested<DENSE, DT, XF, 1>();
    if (XF == kRotation) rotate_rows<DT, 8, false>(raw);
    if (XF == kDelta && a.anchors)
        delta_rows<DT, DENSE, 8>(a.x, u.head_off, row0, a.tokens, a.anchor_shift,
                                 head_anchors(a.anchors, u.lh, a.tokens, a.anchor_shift), true, raw, bad);
    VParams vp;
    v_pass_params<BITS, GV, DT, XF == kRotation>(raw, vp);
    forget_unpacked<DT, 8>(raw);
    uint8_t *codes = head_codes<BITS>(a, u.lh) + row0 * (16 * BITS);
    uint32_t *meta = (uint32_t *)a.meta + (u.lh * a.tokens + row0) * NG;
    const long long left = a.tokens - row0;
    v_emit<BITS, GV, DT, false, XF == kRotation>(raw, vp, codes, left < kPassRows ? (int)left : kPassRows, meta);
    report(a.status, bad);
}

template <int BITS, int GV, int DT, bool DENSE, int XF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(min_waves(BITS, kPassRows, DT, DENSE))))
void compress_v_kernel(QuantBatch b)
{
    unsigned wg;
    const QuantArgs &a = b.item[place_item(b.at, place_of_workgroup(b.at), wg)];
    compress_v_unit<BITS, GV, DT, DENSE, XF>(a, wg);
}

template <int BITS, int DT, bool DENSE, int XF, bool PACED, class Refused>
__device__ __forceinline__ void decompress_v_unit(const QuantArgs &a, unsigned wg, int pace, Refused &&refused)
{
    UnitPos u;
    if (!unit_pos(a, wg, u)) return;
    const int lane = lane_id(), col = lane & 15, rsub = lane >> 4;
    const long long row0 = u.blk * kPassRows;
    const int lanes_shift = a.group == 32 ? 2 : (a.group == 64 ? 3 : 4), ng = kDim / a.group;
    const uint32_t *meta = (const uint32_t *)a.meta + (u.lh * a.tokens + row0) * ng + (col >> lanes_shift);
    const long long left = a.tokens - row0;
    const int rows = left < kPassRows ? (int)left : kPassRows;
    uint32_t mw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) mw[i] = meta[(4 * i + rsub < rows ? 4 * i + rsub : 0) * ng];
    uint8_t *codes = head_codes<BITS>(a, u.lh) + row0 * (16 * BITS);
    PassFetch f;
    pass_fetch<BITS, DENSE, 0, XF == kRotation>(f, codes, a.x, u.head_off, row0, rows);
    if (refused()) return;
    float scale[8], zero[8];
    const bool clamp = v_meta_floats<BITS, DT>(mw, scale, zero);
    bool bad = false;
    const uint16_t *anchors = XF == kDelta ? head_anchors(a.anchors, u.lh, a.tokens, a.anchor_shift) : nullptr;
    if (XF == kRotation) dequant_pass<BITS, DT, true, DENSE, 1>(f, scale, zero, clamp, a.x, u.head_off, row0, rows, bad);
    else if (XF == kDelta && a.anchor_shift >= 5) dequant_pass<BITS, DT, true, DENSE, 2>(f, scale, zero, clamp, a.x, u.head_off, row0, rows, bad, anchors, a.anchor_shift);
    else if (XF == kDelta) dequant_pass<BITS, DT, true, DENSE, 3>(f, scale, zero, clamp, a.x, u.head_off, row0, rows, bad, anchors, a.anchor_shift);
    else dequant_pass<BITS, DT, true, DENSE, 0, PACED>(f, scale, zero, clamp, a.x, u.head_off, row0, rows, bad, nullptr, 0, nullptr, pace);
    report(a.status, bad);
}

template <int BITS, int DT, bool DENSE, int XF, bool PACED>
__global__ __launch_bounds__(256) void decompress_v_kernel(QuantBatch b)
{
    unsigned wg;
    const QuantArgs &a = b.item[place_item(b.at, place_of_workgroup(b.at), wg)];
    const int status = *a.status;
    decompress_v_unit<BITS, DT, DENSE, XF, PACED>(a, wg, b.pace, [&]() { return (status & KVC_DEV_BAD_HEADER) != 0; });
}

// ---- a whole small call in one launch -------------------------------------------------------------

// Items 2r and 2r + 1 of the batch are K and V of request r; the first workgroups are the requests' prologues,
// which nothing in the launch waits for (the requests have no block table, so no unit has anything to
// report in the status word).  A call of 4 MB is launches and latency: prologue, K and V in turn were
// 1.6 + 5 + 4.8 us of kernels, 16 us per call; together 8.3.
template <int BITS, int G, int DT, bool DENSE>
__global__ __launch_bounds__(256) void compress_call_kernel(SmallCompressArgs b)
{
    __shared__ __attribute__((aligned(16))) float xch_all[4 * kXchFloats];
    if (blockIdx.x < (unsigned)b.requests) {
        write_prologue(b.prologue[blockIdx.x], threadIdx.x, 256);
        return;
    }
    unsigned wg;
    const int i = place_item(b.at, blockIdx.x, wg);
    if (i & 1) compress_v_unit<BITS, G, DT, DENSE, kNoTransform, true>(b.item[i], wg);
    else compress_k_unit<BITS, G, DT, DENSE, kNoTransform, true>(b.item[i], wg, xch_all);
}

// The same for decompression: every wave compares the header with the plan's for itself (its 128 bytes travel
// with the unit's own loads), the request's first workgroup writes the status word.
template <int BITS, int DT, bool DENSE>
__global__ __launch_bounds__(256) void decompress_call_kernel(SmallDecompressArgs b)
{
    const unsigned place = place_of_workgroup(b.at);
    const bool leads = place < (unsigned)b.requests;
    unsigned wg = 0;
    int i = place_item(b.at, place, wg);
    if (leads) i = 2 * (int)place;
    const SmallCheck &check = b.check[i >> 1];
    const int word = lane_id() & 31;
    const uint32_t got = check.payload[word];
    auto refused = [&]() { return __builtin_amdgcn_ballot_w64(got != check.expect.w[word]) != 0; };
    if (leads) {
        const bool bad = refused();
        if (threadIdx.x == 0) *b.item[i].status = bad ? KVC_DEV_BAD_HEADER : 0;
        return;
    }
    if (i & 1) decompress_v_unit<BITS, DT, DENSE, kNoTransform, false>(b.item[i], wg, 0, refused);
    else decompress_k_unit<BITS, DT, DENSE, kNoTransform, false>(b.item[i], wg, 0, refused);
}

// ---- launchers ----------------------------------------------------------------------------------

template <int BITS, int DT, bool DENSE, int XF> static int compress_bits_xf(int is_v, int group, const QuantBatch &b, hipStream_t s)
{
    const LaunchShape shape = launch_shape(b, true, is_v, BITS, group, DT);
    if (!is_v) {
        switch (group) {
        case 32: KVC_LAUNCH((compress_k_kernel<BITS, 32, DT, DENSE, XF>), b, shape, s);
        case 64: KVC_LAUNCH((compress_k_kernel<BITS, 64, DT, DENSE, XF>), b, shape, s);
        case 128: KVC_LAUNCH((compress_k_kernel<BITS, 128, DT, DENSE, XF>), b, shape, s);
        }
    } else {
        switch (group) {
        case 32: KVC_LAUNCH((compress_v_kernel<BITS, 32, DT, DENSE, XF>), b, shape, s);
        case 64: KVC_LAUNCH((compress_v_kernel<BITS, 64, DT, DENSE, XF>), b, shape, s);
        case 128: KVC_LAUNCH((compress_v_kernel<BITS, 128, DT, DENSE, XF>), b, shape, s);
        }
    }
    return KVC_ERR_UNSUPPORTED;
}

template <int BITS, int DT, bool DENSE> static int compress_bits_dt(int is_v, int group, const QuantBatch &b, hipStream_t s)
{
    const QuantArgs &a = b.item[0];
    if (a.rotate) return compress_bits_xf<BITS, DT, DENSE, kRotation>(is_v, group, b, s);
    if (a.anchors) return compress_bits_xf<BITS, DT, DENSE, kDelta>(is_v, group, b, s);
    return compress_bits_xf<BITS, DT, DENSE, kNoTransform>(is_v, group, b, s);
}

// Launches with a transform have kernels of their own, and paced ones, too: what the plain ones do not use costs them
// registers and moves their stores.
template <int BITS, int DT, bool DENSE> static int decompress_bits_dt(int is_v, const QuantBatch &b, hipStream_t s)
{
    const QuantArgs &a = b.item[0];
    const LaunchShape shape = launch_shape(b, false, is_v, BITS, 0, DT);
    if (a.rotate) {
        if (!is_v) KVC_LAUNCH((decompress_k_kernel<BITS, DT, DENSE, kRotation, false>), b, shape, s);
        KVC_LAUNCH((decompress_v_kernel<BITS, DT, DENSE, kRotation, false>), b, shape, s);
    }
    if (a.anchors) {
        if (!is_v) KVC_LAUNCH((decompress_k_kernel<BITS, DT, DENSE, kDelta, false>), b, shape, s);
        KVC_LAUNCH((decompress_v_kernel<BITS, DT, DENSE, kDelta, false>), b, shape, s);
    }
    if (shape.pace) {
        if (!is_v) KVC_LAUNCH((decompress_k_kernel<BITS, DT, DENSE, kNoTransform, true>), b, shape, s);
        KVC_LAUNCH((decompress_v_kernel<BITS, DT, DENSE, kNoTransform, true>), b, shape, s);
    }
    if (!is_v) KVC_LAUNCH((decompress_k_kernel<BITS, DT, DENSE, kNoTransform, false>), b, shape, s);
    KVC_LAUNCH((decompress_v_kernel<BITS, DT, DENSE, kNoTransform, false>), b, shape, s);
}

#define KVC_PASTE2(a, b) a##b
#define KVC_PASTE(a, b) KVC_PASTE2(a, b)

int KVC_PASTE(launch_compress_bits, KVC_BITS)(int is_v, int group, int dtype, const QuantBatch &b, hipStream_t s)
{
    if (b.item[0].dense)
        return dtype == DT_F16 ? compress_bits_dt<KVC_BITS, DT_F16, true>(is_v, group, b, s)
                               : compress_bits_dt<KVC_BITS, DT_BF16, true>(is_v, group, b, s);
    return dtype == DT_F16 ? compress_bits_dt<KVC_BITS, DT_F16, false>(is_v, group, b, s)
                           : compress_bits_dt<KVC_BITS, DT_BF16, false>(is_v, group, b, s);
}

int KVC_PASTE(launch_decompress_bits, KVC_BITS)(int is_v, int dtype, const QuantBatch &b, hipStream_t s)
{
    if (b.item[0].dense)
        return dtype == DT_F16 ? decompress_bits_dt<KVC_BITS, DT_F16, true>(is_v, b, s) : decompress_bits_dt<KVC_BITS, DT_BF16, true>(is_v, b, s);
    return dtype == DT_F16 ? decompress_bits_dt<KVC_BITS, DT_F16, false>(is_v, b, s) : decompress_bits_dt<KVC_BITS, DT_BF16, false>(is_v, b, s);
}

// units of four per workgroup behind the workgroups of the requests themselves
template <class Args> static unsigned place_call(Args &b, int run)
{
    unsigned total = (unsigned)b.requests;
    for (int i = 0; i < b.n; ++i) {
        b.at.start[i] = total;
        total += (unsigned)((b.item[i].total_units + 3) / 4);
    }
    close_places(b.at, b.n, total, run);
    return total;
}

// LDS that nothing uses and runs, as in launch_shape, for decompression calls; most compression calls gain nothing from the LDS (2^21
// rows, fp16, with 32000 bytes: 2 bits g64 210 and 210 us, 4 bits g64 227 and 229, 4 bits g32 230 and 224; bf16 231 and 233).
// Call times in us, without / with runs of 16:
//   4 bits g32  2^18 rows 27.2 26.6,  2^20 118 112;  bf16 27.4 26.8, 118 113;  2 bits g64  24.4 23.9, 91 87;  bf16 24.3 23.8, 92 85
//   3 bits g32  26.2 25.7, 96 94;  8 bits g32 level
constexpr LaunchShape kCallShape = {40000, 16};

template <int G> static void compress_call(int dtype, const SmallCompressArgs &b, unsigned wgs, hipStream_t s)
{
    // (bf16 rows requested together, groups of 32: 2^20 rows 2 bits 108 -> 103, 4 bits 116 -> 110 us with 32000, 2^20.55 158 -> 151, 178 ->
    // 162, which without was 174 before; 8 bits 2^20 level, 2^20.55 206 -> 199)
    const unsigned lds = G == 32 && dtype == DT_BF16 && b.item[0].dense && wgs >= (1u << 14) ? 32000 : 0;
#define KVC_CALL(DT, D) hipLaunchKernelGGL((compress_call_kernel<KVC_BITS, G, DT, D>), dim3(wgs), dim3(256), lds, s, b)
    if (b.item[0].dense) { if (dtype == DT_F16) KVC_CALL(DT_F16, true); else KVC_CALL(DT_BF16, true); }
    else if (dtype == DT_F16) KVC_CALL(DT_F16, false); else KVC_CALL(DT_BF16, false);
#undef KVC_CALL
}

int KVC_PASTE(launch_compress_call_bits, KVC_BITS)(int group, int dtype, SmallCompressArgs &b, hipStream_t s)
{
    const unsigned wgs = place_call(b, 0);
    if (group == 32) compress_call<32>(dtype, b, wgs, s);
    else if (group == 64) compress_call<64>(dtype, b, wgs, s);
    else compress_call<128>(dtype, b, wgs, s);
    return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_DEVICE;
}

int KVC_PASTE(launch_decompress_call_bits, KVC_BITS)(int dtype, SmallDecompressArgs &b, hipStream_t s)
{
    const unsigned wgs = place_call(b, kCallShape.run);
#define KVC_CALL(DT, D) hipLaunchKernelGGL((decompress_call_kernel<KVC_BITS, DT, D>), dim3(wgs), dim3(256), kCallShape.lds, s, b)
    if (b.item[0].dense) { if (dtype == DT_F16) KVC_CALL(DT_F16, true); else KVC_CALL(DT_BF16, true); }
    else if (dtype == DT_F16) KVC_CALL(DT_F16, false); else KVC_CALL(DT_BF16, false);
#undef KVC_CALL
    return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_DEVICE;
}

}  // namespace kvc
