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
static inline unsigned place_items(QuantBatch &b, int run)
{
    unsigned total = 0;
    for (int i = 0; i < b.n; ++i) {
        b.at.start[i] = total;
        total += (unsigned)((b.item[i].total_units + 3) / 4);
    }
    close_places(b.at, b.n, total, run);
    return total;
}

// How a launch is spread over the chip and over time.  Memory takes few, steady streams of stores better than many
// bursts, so the less arithmetic a kernel has, the more its time depends on these.
//
// lds: dynamic LDS that nothing uses.  It bounds the workgroups of a compute unit, and with them the window of the
// tensor that the chip reads or writes at a time (a wave's rows are 8 KB): with 80000 bytes two workgroups, 52000
// three, 40000 four (a K compression, which has 4096 of its own, three; with 36000 four), 32000 five.
// run: see place_of_workgroup.  pace: 64-cycle waits between the row stores of a unit.
// What pays was measured kernel by kernel, and each is off where it did not pay.  Launches with a transform have none
// (the arithmetic needs the waves: rotation, 40000: compress +2 %, decompress +3 %) but for large decompressions: rotation at 8 bits from 3 * 2^23
// rows (2^25 rows, as it was with one kernel for all transforms / without / with, dense 4743 4790 4710 us, paged 5177 5353 5050), dense differences
// from anchors 32 rows and more apart at 4 bits from 2^22 rows (2^23.3 rows bf16 1145 1163 1098, fp16 1163 1169 1130).
//
// Decompress calls in us, as they were (a conversion per code, holds of 0 to 40000) / now; groups of 32, 2 bits 64:
//            rows     2^21        2^21.6       2^22        2^22.6      2^23.2       2^23.3        2^23.9
//   dense    4 bits   229 / 226   343 / 336    456 / 440   732 / 670  1086 /  997   1158 / 1069   1757 / 1593
//            8 bits   274 / 273   408 / 405    548 / 530   886 / 844  1333 / 1241   1423 / 1331   2179 / 1949
//            3 bits   198 / 189   335 / 322    427 / 424   704 / 660   978 /  979   1041 / 1044   1610 / 1557
//            2 bits   183 / 173   290 / 251    413 / 409   656 / 634   923 /  935    982 / 1000   1547 / 1537
//       bf16 2 bits   182 / 174   291 / 253    420 / 405   665 / 632   960 /  937   1001 /  999   1590 / 1490
//   paged    4 bits   239 / 240   344 / 344    457 / 456   713 / 699  1141 / 1094   1280 / 1227   1869 / 1789
//       bf16 4 bits   247 / 241   365 / 346    485 / 461   758 / 702  1189 / 1085   1284 / 1222   1904 / 1785
//            8 bits   295 / 282   432 / 409    582 / 544   900 / 844  1393 / 1292   1515 / 1449   2224 / 2109
//            3 bits   200 / 200   352 / 334    465 / 443   718 / 680  1082 / 1031   1233 / 1188   1809 / 1734
//            2 bits   184 / 176   271 / 263    416 / 401   642 / 631   969 /  966   1094 / 1090   1606 / 1600
//       bf16 2 bits   184 / 176   271 / 264    430 / 414   655 / 640   981 /  950   1125 / 1090   1674 / 1601
//   What the neighbours of a choice cost: dense 3 bits 2^23.3 rows, 40000 for 80000 1073, no run 1085; dense fp16 2 bits 1013 with
//   run 16, 80000; paged 3 bits 32000 1264; a wait more or less 1 to 3 %, on dense rows 40 %.  Between 2^21 and 2^22.6 rows
//   dense 4 bits would gain another 3 % from 80000 (326 and 426 us).  Below 2^20 rows nothing but the runs of dense rows is
//   new.  With the cheaper arithmetic alone, the old holds and no runs: dense 2 bits 1000, paged 4 bits 1292.
// Wider groups have less metadata to read and send denser stores; several requests in a launch and large tensors differ too.
// One shape for all of them lost calls; as they were / one shape / now (dense 4 and 8 bits need no such lines: 4 to 10 % faster in all):
//              rows        2^21.6          2^22            2^23.2            2^23.3             2^25
//   paged    4 bits g32    353 346 347   483 479 479   1141 1073 1074   1278 1224 1230   4388 4512 4352
//                   g64    337 336 336   465 461 460   1056 1063 1035   1231 1196 1176   4230 4514 4243
//                   g128   331 333 333   456 453 451   1018 1050 1010   1205 1194 1162   4177 4531 4193
//       bf16 4 bits g128   342 332 332   470 455 456   1101 1040 1038   1237 1182 1181   4204 4537 4159
//            2 bits g64    265 298 264   420 418 418    939  948  948   1094 1084 1083   3730 3860 3718
//                   g128   270 300 268   416 417 417    931  947  947   1082 1075 1074   3680 3951 3686
//   dense    3 bits g64    308 317 311   420 427 425    949  953  962    999 1035 1010   3598 3378 3382
//                   g128   306 317 307   414 426 420    909  954  916    976 1036  985   3580 3377 3376
//       bf16 3 bits g128   314 314 311   426 423 423    921  946  922    995 1026  992   3629 3344 3350
//            2 bits g32    308 310 311   423 414 414    937  939  922   1004 1023 1009   3473 3437 3260
//                   g64    273 247 247   417 416 416    924  925  926    975  999 1000   3414 3411 3281   (2 % not recovered)
//   several  dense 3 bits, 8 of 2^20.8 rows g128 1477 1529 1470, 12 of 2^21 g32 2718 2720 2574; paged 4 bits, 8 of 2^20.8 rows g64 1511 1590 1506,
//            g128 1484 1575 1480, 2 bits bf16 g128 1433 1453 1339.  Dense 4 bits, 80000 from 6 * 2^20 rows: 7 of 2^20.8 rows 0.91 of
//            what it was, 12 of 2^21 0.90 (40000 0.96, 32000 0.98)
//   by head  (launches over some of the heads) paged bf16, half at 8 and half at 2 bits, 2^20.6 rows each 400 417 395
// Compression (32 layers of 16384 tokens and 94 x 4 heads of 24576, groups of 32, 64 and 128; change of the call by the hold):
//   dense    K, groups of 32: fp16 2 and 3 bits -1 to -4 % with 36000 (40000: -2 to +1 %), bf16 2 to 4 bits 0 to -1 % (+2
//            to +6 %), fp16 4 bits and 8 bits -1 to -3 % with 40000; groups of 64 -1 to -3 % with 40000, of 128
//            and V 0; below 2^20 rows, where the tensor is a few generations of workgroups, 0 to +2 %
//            in runs from 2^22 rows (2^23.3 rows without / with): 4 bits 1137 / 1090, 2 bits 1068 / 1023, 8 bits 1361 / 1307 (run
//            64; with 16 1336), bf16 4 bits 1138 / 1099, 2 bits 1071 / 1026; at 2^21 level
//   V and K at groups of 32 have few registers since the transforms have kernels of their own, and need a hold where their
//            registers were one: from 3 * 2^19 rows V 40000 (2^23.3 rows, 4 bits 1138 without, 1095 with; 2^21 rows 241, 227; bf16 2
//            bits groups of 64 217, 212), strided fp16 32000, bf16 24000 (2^21 rows paged 239, 232), V of any group (paged bf16 4 bits
//            g64 / g128, 2^23.2 rows 1078 / 1044 without, 1052 / 1014 with; 8 bits 32000 1309 / 1276, 1301 / 1266)
//   strided  K, groups of 32: fp16 4 bits and 8 bits -1 to -3 % with 32000, 2 and 3 bits and bf16 4 bits +2 to +7 %;
//            V: fp16 0 to -2 % with 32000, bf16 0 to +2 %; runs 0 to +3 %
struct LaunchShape {
    unsigned lds = 0;
    int run = 0;
    int pace = 0;
};

static inline LaunchShape dense_decompress_shape(int bits, bool f16, int group, long long rows, bool one)
{
    const bool g32 = group == 32;
    if (bits == 8) return {one && rows >= (1ll << 20) ? 80000u : 0u, 16};
    if (bits == 4) return {rows >= 6ll << 20 ? 80000u : rows < (1ll << 21) || (one && rows < (1ll << 22)) ? 40000u : 32000u, 16};
    if (!one) {
        if (rows < (1ll << 21)) return {40000, 16};
        if (rows < 3ll << 20) return {bits == 3 ? 32000u : 40000u, 16};
        if (g32) return {80000, 16};
        return {40000, f16 && bits == 2 && rows >= 6ll << 20 ? 8 : 16};
    }
    if (bits == 3 && !g32 && (f16 || group == 128) && rows >= 5ll << 19 && rows < 3ll << 23) return {40000, 0};
    if (bits == 2 && !g32 && f16 && rows >= 6ll << 20 && rows < 3ll << 23) return {40000, rows < 3ll << 22 ? 8 : 16};
    return {rows >= (1ll << 20) ? 80000u : 40000u, 16};
}

static inline LaunchShape paged_decompress_shape(int bits, bool f16, bool g32, long long rows, bool one, bool some_heads)
{
    if (bits == 4) {
        if (one && rows >= (1ll << 23)) return {52000, 0, rows < 3ll << 23 && (g32 || !f16) ? 1 : 0};
        return {40000, 0, rows < (1ll << 20) ? 0 : rows >= 5ll << 19 ? 4 : g32 ? 3 : 2};
    }
    if (rows < (1ll << 19)) return {};
    if (rows < (1ll << 20)) return {bits == 8 || (bits == 2 && !f16) ? 40000u : 0u};
    if (some_heads && bits != 3 && rows < 5ll << 19) return {40000};
    if (bits == 8) return {52000, 0, rows < (1ll << 21) ? 0 : 2};
    if (bits == 3) return rows < (1ll << 21) ? LaunchShape{32000, 16} : LaunchShape{40000, 0, f16 ? 0 : 1};
    if (rows < 5ll << 19) return {52000, 0, 2};
    if (!g32 && rows < 7ll << 19) return {40000};
    if (f16) {
        if (g32 && !one) return {40000, 16};
        return g32 || rows < 3ll << 23 ? LaunchShape{32000, 8, 2} : LaunchShape{40000};
    }
    if (!one) return {40000, 0, g32 ? 1 : 0};
    return {40000, 0, rows >= (g32 ? 7ll << 19 : 1ll << 23) ? 3 : 2};
}

static inline LaunchShape launch_shape(const QuantBatch &b, bool compress, bool is_v, int bits, int group, int dtype)
{
    const QuantArgs &a = b.item[0];
    long long rows = 0;
    for (int i = 0; i < b.n; ++i) rows += b.item[i].total_units * (compress && !is_v ? group : kPassRows);
    if (a.rotate) return {!compress && bits == 8 && rows >= 3ll << 23 ? a.dense ? 32000u : 40000u : 0u};
    if (a.anchors) return {!compress && bits == 4 && a.dense && a.anchor_shift >= 5 && rows >= (1ll << 22) ? 40000u : 0u};
    const bool f16 = dtype == DT_F16, one = b.n == 1;
    if (compress) {
        const bool wide = bits == 8 || (bits == 4 && f16), some = rows >= 3ll << 19;
        if (!a.dense) {
            if (is_v ? f16 : group == 32 && wide) return {32000};
            if (!is_v && group > 32) return {};
            return {!some ? 0u : f16 || (is_v && bits == 8) ? 32000u : 24000u};
        }
        const int run = rows < (1ll << 22) ? 0 : bits == 8 ? 64 : 16;
        if (is_v) return {some ? 40000u : 0u, run};
        return {rows < (1ll << 20) ? 0u : group > 32 || wide ? 40000u : 36000u, run};
    }
    const bool g32 = a.group == 32;
    return a.dense ? dense_decompress_shape(bits, f16, a.group, rows, one) : paged_decompress_shape(bits, f16, g32, rows, one, a.head_list != nullptr);
}

#define KVC_LAUNCH(kernel, batch, shape, s)                                                     \
    do {                                                                                        \
        QuantBatch placed_ = batch;                                                             \
        const LaunchShape shape_ = shape;                                                       \
        const unsigned wgs_ = place_items(placed_, shape_.run);                                 \
        placed_.pace = shape_.pace;                                                             \
        if (wgs_ > 0) hipLaunchKernelGGL(kernel, dim3(wgs_), dim3(256), shape_.lds, s, placed_); \
        return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_DEVICE;                       \
    } while (0)

}  // namespace kvc
