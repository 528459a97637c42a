// Shared pieces of the codec-free kernels: work-unit addressing and the launch helper.
// One wave per work unit, four units per workgroup.
#pragma once

#include "kvc_internal.h"
#include "kvc_tile.h"
#include "../../include/kvc.h"

namespace kvc {

struct UnitPos {
    long long lh;        // layer * heads + head
    long long blk;       // unit index inside the head
    long long head_off;  // element offset of x[l][h][0][0]
};

__device__ __forceinline__ bool unit_pos(const QuantArgs &a, unsigned wg, UnitPos &u)
{
    long long unit = (long long)wg * 4 + wave_id();
    if (unit >= a.total_units) return false;
    if (a.head_minor) {
        // unit = (layer * units_per_head + block) * heads + head: the four waves of a workgroup read or
        // write the same token rows of four neighbouring heads, which are contiguous in memory
        const long long t = unit / a.heads;
        const long long l = t / a.units_per_head;
        u.blk = t - l * a.units_per_head;
        u.lh = l * a.heads + (unit - t * a.heads);
    } else {
        const long long slot = unit / a.units_per_head;
        u.lh = a.head_list ? a.head_list[slot] : slot;
        u.blk = unit - slot * a.units_per_head;
    }
    long long l = u.lh / a.heads, h = u.lh - l * a.heads;
    u.head_off = l * a.x.stride_layer + h * a.x.stride_head;
    return true;
}

// first code byte of head lh (width BITS) in its section
template <int BITS> __device__ __forceinline__ uint8_t *head_codes(const QuantArgs &a, long long lh)
{
    const long long widths = a.bits_before ? a.bits_before[lh] : lh * BITS;
    return a.codes + widths * a.tokens * 16;
}

__device__ __forceinline__ void report(int *status, bool bad)
{
    if (bad) atomicOr(status, KVC_DEV_BAD_BLOCK);
}

// workgroups of four units, item after item
static inline unsigned place_items(QuantBatch &b)
{
    unsigned at = 0;
    for (int i = 0; i < b.n; ++i) {
        b.start[i] = at;
        at += (unsigned)((b.item[i].total_units + 3) / 4);
    }
    b.start[b.n] = at;
    return at;
}

// Dynamic LDS that nothing uses: it bounds the workgroups of a compute unit, and with them the window of the
// tensor that the chip reads or writes at a time (a wave's rows are 8 KB), which memory takes better when it
// is small.  What pays was measured kernel by kernel (K and V apart; change of the call's time against no bound; 32
// layers of 16384 tokens and 94 x 4 heads of 24576, groups of 32, 64 and 128, fp16 and bf16), and the bound
// is off where it did not pay.  With 40000 bytes a unit takes four workgroups (three of a K compression, which has
// 4096 of its own; with 36000 four), with 32000 five (four).  Launches with a transform have none: its
// arithmetic needs the waves (rotation, 40000: compress +2 %, decompress +3 %).
//   decompress, dense    2 bits -1 to -7 % with 40000, 3 bits 0 to -2 %, 8 bits +1 to +2 %; 4 bits (the call) below 2^22
//                        rows -1 to -6 % (bf16 from 2^21.5: 0 to +3 %) with 40000, above up to +5 % with 40000 and -1 % with 32000;
//                        several requests in a launch, 2^21 rows and more: 4 bits 0 to +5 % with 40000, 3 bits -1 to
//                        +3 %, either 0 to -1 % with 32000
//   decompress, strided  with 40000: 4 bits 0 to -6 %, fp16 2 and 3 bits up to +4 %; from 2^19 rows bf16 2 bits 0 to
//                        -3 %, 8 bits -1 to -3 % (from 2^22: 0 to +1 %); from 2^21 bf16 3 bits +1 to -3 %; below these 0
//                        to +5 %
//   compress, dense      K, groups of 32: fp16 2 and 3 bits -1 to -4 % with 36000 (40000: -2 to +1 %), bf16 2 to 4 bits 0 to -1 % (+2
//                        to +6 %), fp16 4 bits and 8 bits -1 to -3 % with 40000; groups of 64 -1 to -3 % with 40000, of 128
//                        and V 0; below 2^20 rows, where the tensor is a few generations of workgroups, 0 to +2 %
//   compress, strided    K, groups of 32: fp16 4 bits and 8 bits -1 to -3 % with 32000, 2 and 3 bits and bf16 4 bits +2 to +7 %;
//                        V: fp16 0 to -2 % with 32000, bf16 0 to +2 %
static inline unsigned window_lds(const QuantBatch &b, bool compress, bool is_v, int bits, int group, int dtype)
{
    const QuantArgs &a = b.item[0];
    if (a.rotate || a.anchors) return 0;
    long long rows = 0;
    for (int i = 0; i < b.n; ++i) rows += b.item[i].total_units * (compress && !is_v ? group : kPassRows);
    if (!compress) {
        if (!a.dense) {
            if (bits == 8) return rows >= (1ll << 19) && rows < (1ll << 22) ? 40000 : 0;
            if (bits < 4) return dtype == DT_BF16 && rows >= (bits == 2 ? 1ll << 19 : 1ll << 21) ? 40000 : 0;
            return 40000;
        }
        if (bits == 8) return 0;
        const bool narrow = bits == 2 || rows < (1ll << 21) || (b.n == 1 && (bits == 3 || rows < (1ll << 22)));
        return narrow ? 40000 : 32000;
    }
    if (is_v) return !a.dense && dtype == DT_F16 ? 32000 : 0;
    const bool wide = bits == 8 || (bits == 4 && dtype == DT_F16);
    if (a.dense) return rows < (1ll << 20) ? 0 : group > 32 || wide ? 40000 : 36000;
    return group == 32 && wide ? 32000 : 0;
}

#define KVC_LAUNCH(kernel, batch, lds, s)                                                 \
    do {                                                                                  \
        QuantBatch placed_ = batch;                                                       \
        const unsigned wgs_ = place_items(placed_);                                       \
        if (wgs_ > 0) hipLaunchKernelGGL(kernel, dim3(wgs_), dim3(256), lds, s, placed_); \
        return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_DEVICE;                 \
    } while (0)

}  // namespace kvc
