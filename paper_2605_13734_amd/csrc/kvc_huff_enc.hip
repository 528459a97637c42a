// Lossless stage, encoder: build the code tables, quantize + pack + Huffman-code one chunk per wave and place the body
// through a single-pass prefix sum over workgroups.  Compiled once per code width (-DKVC_BITS=2, 3,
// 4 or 8).  See kvc_huff.h for the format and the division of work, kvc_scan.h for
// the prefix sum, kvc_huff_build.h for the tables and kvc_huff_fetch.h for their way into LDS.

#include "kvc_huff_build.h"
#include "kvc_huff_fetch.h"

#include <atomic>

#ifndef KVC_BITS
#error "compile with -DKVC_BITS=2, 3, 4 or 8"
#endif

namespace kvc {

// ---- encoder ---------------------------------------------------------------------------------

// bit count of HALF (0 or 1) of the lane's sub-block
template <int W> __device__ __forceinline__ uint32_t half_bits(const uint32_t *sym, const EncTables &t, int half)
{
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < W / 2; ++k) {
        const uint32_t w = sym[half * (W / 2) + k];
#pragma unroll
        for (int b = 0; b < 4; ++b) bits += t.len[(w >> (8 * b)) & 255u];
    }
    return bits;
}

struct BitWriter {
    unsigned long long acc;
    uint32_t nbits;
    uint32_t *out;       // next word (LDS)
};

__device__ __forceinline__ void writer_start(BitWriter &bw, uint32_t *words, uint32_t bit)
{
    bw.acc = 0;
    bw.nbits = bit & 31;          // the leading bits of the first word belong to the previous stream
    bw.out = words + (bit >> 5);
}

__device__ __forceinline__ void put(BitWriter &bw, uint32_t e)
{
    const uint32_t len = e >> 12;
    bw.acc = (bw.acc << len) | (e & 0xfffu);
    bw.nbits += len;
}

__device__ __forceinline__ void flush(BitWriter &bw)
{
    if (bw.nbits >= 32) {
        atomicOr(bw.out, (uint32_t)(bw.acc >> (bw.nbits - 32)));
        ++bw.out;
        bw.nbits -= 32;
    }
}

__device__ __forceinline__ void writer_finish(BitWriter &bw)
{
    if (bw.nbits > 0) atomicOr(bw.out, (uint32_t)(bw.acc << (32 - bw.nbits)));
}

// Code the words [first, first + n) of the lane's sub-block.  Words of streams that share a
// boundary word are merged with LDS atomic OR (the region is zeroed beforehand).
template <int N> __device__ __forceinline__ void encode_words(const uint32_t *sym, const EncTables &t, BitWriter &bw)
{
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const uint32_t w = sym[k];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            put(bw, t.code[(w >> (8 * b)) & 255u]);
            if (b & 1) flush(bw);          // at most 24 new bits between checks
        }
    }
}

// Both halves of the sub-block as two independent streams (instruction-level parallelism).
template <int W> __device__ __forceinline__ void encode_two(const uint32_t *sym, const EncTables &t, BitWriter &b0, BitWriter &b1)
{
#pragma unroll
    for (int k = 0; k < W / 2; ++k) {
        const uint32_t w0 = sym[k], w1 = sym[W / 2 + k];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            put(b0, t.code[(w0 >> (8 * b)) & 255u]);
            put(b1, t.code[(w1 >> (8 * b)) & 255u]);
            if (b & 1) { flush(b0); flush(b1); }
        }
    }
}

// KV: the launch's tensor, K (0), V (1) or both (2: the items of the batch are then a K and a V launch of
// every request, one after the other).
template <int BITS, int G, int DT, int KV, bool DENSE, bool DELTA, int NW, bool ROTATION = false>
__global__ __launch_bounds__(NW * 64)
__attribute__((amdgpu_waves_per_eu(enc_min_waves(BITS, G, DT, DENSE || KV == 2, KV == 1, DELTA || ROTATION))))
void encode_kernel(CoderBatch batch)
{
    using Geo = ChunkGeom<BITS>;
    constexpr int W = Geo::kWords, XF = ROTATION ? kRotation : DELTA ? kDelta : kNoTransform;
    constexpr int kItems = KV == 2 ? 2 : 1;                      // items per request
    // the places of the workgroups that only build tables come first, so that those of all requests start early
    const unsigned front = (unsigned)batch.n * batch.front;
    unsigned wg = 0;
    const int item = kItems * (blockIdx.x < front ? (int)(blockIdx.x / batch.front) : place_item_of_many(batch.at, blockIdx.x - front, wg));
    const CoderArgs first = coder_args<KV>(batch, item);
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[NW * Geo::kLds];
    __shared__ EncTables enc;
    __shared__ uint32_t s_units[NW];
    __shared__ uint32_t s_ticket, s_sum, s_reported, s_table;
    __shared__ unsigned long long s_excl;

    const int tid = threadIdx.x, wave = wave_id(), lane = lane_id();
    if (tid == 0) {
        s_ticket = atomicAdd(first.ws.ticket, 1u);
        s_sum = s_reported = 0;
        s_excl = 0;
    }
    // The table, if it has been built already, in the time the ticket takes (both tensors in one launch: the workgroup's
    // number says which of them it most likely has, its ticket which it has).
    int second = KV == 2 && wg >= first.k_wgs ? 1 : 0, pick = -1;
    if (wave == 0) {
        const CoderArgs a = coder_args<KV>(batch, item + second);
        pick = fetch_table<true>(candidate_tables(a.ws.ticket, a.tab), enc);
        if (lane == 0) s_table = pick < 0 ? kNobody : kThere;
    }
    __syncthreads();
    // global order over table, K and V workgroups (the same in all lanes)
    const unsigned taken = (unsigned)__builtin_amdgcn_readfirstlane((int)s_ticket);
    if (taken < (unsigned)first.builders) {
        static_assert(sizeof(BuildLds) <= NW * Geo::kLds, "the construction uses the LDS of the chunks");
        build_table<NW * 64>(first, (int)taken, *(BuildLds *)lds_all);
        if (taken < (unsigned)first.apart) return;
        __syncthreads();
    }
    const long long ticket = (long long)(taken - (unsigned)first.apart);
    if (KV == 2 && second != (ticket >= first.k_wgs ? 1 : 0)) {
        second = 1 - second;
        __syncthreads();                                         // (no wave is left that may look at the other tensor's)
        if (tid == 0) s_table = kNobody;
        pick = -1;
        __syncthreads();
    }
    // From here on every part of the kernel takes its arguments anew.  (Kept from the start, they were more than the scalar registers hold:
    // nearly every encoder moved scalars to vector registers and back, and 3-bit dense K blocks of 64 bf16 rows with the delta transform lost
    // a wave per SIMD by it, 169 registers.  Compress call of 2^21 rows without / with: those 403 / 370 us; rotation, 4 bits, 359 / 347;
    // without a transform 1.00.  8-bit codes, two chunks per workgroup, feel the loads: one layer of 16k tokens 60.0 / 60.7.  Five waves
    // per SIMD for strided 2-bit K, 96 registers in place of 97, by a view read where it lies: 301 / 304.)
    const int mine_item = BITS == 8 ? item + second : anew(item + second);
    const CoderArgs a = coder_args<KV>(batch, mine_item);
    const auto args_again = [&](const CoderArgs &had, int i) { return BITS == 8 ? had : coder_args<KV>(batch, anew(i)); };
    const long long chunk = (ticket - a.wg_base) * NW + wave;
    const bool live = chunk < a.chunks;
    uint8_t *lds = lds_all + wave * Geo::kLds;
    // The first workgroup of the launch: its first wave becomes the scanner once its own chunk is done (a
    // workgroup of its own would hold the LDS of four chunks, and a launch that just fills the chip would
    // not fit).  What the launch before left is read before any size is reported: the scanner replaces it.
    const bool leads = ticket == first.wg_base;
    unsigned long long before = 0;
    if (leads) {
        before = *(const volatile unsigned long long *)scan_carry(a);
        asm volatile("" : "+v"(before));
    }

    // the wave's chunk size is known; the last wave of the workgroup to say so passes the sum on
    int last_to_report = 0;
    auto report_size = [&](uint32_t units) {
        if (lane != 0) return;
        s_units[wave] = units;
        atomicAdd(&s_sum, units);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (atomicAdd(&s_reported, 1u) != (uint32_t)NW - 1) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        const uint32_t sum = *(volatile uint32_t *)&s_sum;
        last_to_report = 1;
        const CoderArgs now = args_again(a, mine_item);
        __hip_atomic_store(&now.ws.state[ticket], kFlagSize | sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    uint32_t body_units = 0;      // body size in 16-byte units
    bool coded = false, coding = false;
    int rows = 0;
    uint32_t sym[W];
    if (live) {
        ChunkPos c = chunk_pos(a.q, chunk);
        rows = c.rows;
        bool bad = false;
        if (KV == 2 ? second != 0 : KV == 1) quantize_chunk<BITS, G, DT, true, DENSE, XF>(a.q, c, lds, bad);
        else quantize_chunk<BITS, G, DT, false, DENSE, XF>(a.q, c, lds, bad);
        if (bad) atomicOr(a.q.status, KVC_DEV_BAD_BLOCK);
        wave_sync();
        const CoderArgs now = args_again(a, mine_item);
        coding = wait_for_table(now, enc, &s_table, pick);
        // the table's lengths in the payload, unless the construction without halvings has written them already (by the wave that
        // brought the table)
        if (pick > 0 && ticket == now.wg_base)
            for (int k = lane; k < 256; k += 64) now.payload[now.off_aux + 256 * now.tab + k] = enc.len[k];
        load_sub<BITS>(lds, sym);
        const int have = coding ? min(max(rows - 2 * lane, 0), 2) : 0;        // valid rows of this sub-block
        uint32_t bits0 = 0, bits = 0;
        if (have > 0) bits0 = half_bits<W>(sym, enc, 0);
        bits = bits0;
        if (have > 1) bits += half_bits<W>(sym, enc, 1);
        const uint32_t incl = wave_inclusive_sum(bits);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        const uint32_t raw_bytes = (uint32_t)rows * Geo::kRowBytes;
        const uint32_t coded_bytes = (2 * kSubs + 4 * ((total + 31) / 32) + 15) & ~15u;
        coded = coded_bytes < raw_bytes;
        body_units = (coded ? coded_bytes : raw_bytes) / 16;
        // the size goes out before the code words are written
        report_size(body_units);
        if (coded) {
            wave_sync();                                          // every lane holds its symbols
            u32x4 zero = {0, 0, 0, 0};
            for (uint32_t o = lane * 16; o < coded_bytes; o += 64 * 16) *(u32x4 *)(lds + o) = zero;
            wave_sync();
            ((uint16_t *)lds)[lane] = (uint16_t)bits;
            const uint32_t start = incl - bits;
            uint32_t *words = (uint32_t *)(lds + 2 * kSubs);
            if (have > 1) {
                BitWriter b0, b1;
                writer_start(b0, words, start);
                writer_start(b1, words, start + bits0);
                encode_two<W>(sym, enc, b0, b1);
                writer_finish(b0);
                writer_finish(b1);
            } else if (have > 0) {
                BitWriter b0;
                writer_start(b0, words, start);
                encode_words<W / 2>(sym, enc, b0);
                writer_finish(b0);
            }
            wave_sync();
        }
    }
    if (!live) report_size(0);
    const CoderArgs out = args_again(a, mine_item);
    // The workgroup's prefix, left in its state word by the scanner once all its waves have reported.  The wave
    // that reported last polls for it, the others wait at an LDS word: four thousand waves polling memory would
    // slow the scanner down.  (The first workgroup of the launch, whose first wave is the scanner, knows its
    // prefix: the end of the launch before.)
    unsigned long long excl;
    if (leads) {
        excl = before;
        while (wave > 0 && __hip_atomic_load(&s_reported, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != (uint32_t)NW) __builtin_amdgcn_s_sleep(1);
    } else if (__builtin_amdgcn_readfirstlane(last_to_report)) {
        excl = wait_for_place(out, ticket);
        if (lane == 0) __hip_atomic_store(&s_excl, excl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
        // (the polling wave always ends: it finds the prefix or its spin limit)
        while (((excl = __hip_atomic_load(&s_excl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) >> 62) != 2) __builtin_amdgcn_s_sleep(1);
    }
    excl &= kValueMask;
    if (excl == kNoPlace || !coding) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");       // (the sizes of the other waves are older than the prefix)
    unsigned long long mine = excl;
    for (int w = 0; w < wave; ++w) mine += s_units[w];
    if (lane == 0) ((uint32_t *)(out.payload + out.off_dir))[out.chunk_base + chunk] = (uint32_t)mine;
    uint8_t *dst = out.payload + out.off_bodies + mine * 16;
    if ((long long)(out.off_bodies + (mine + body_units) * 16) > out.capacity) {
        // cannot happen: bodies never exceed raw size
    } else if (coded) {
        // (every store instruction covers whole lines of memory, but for the body's ends)
        const int skew = (int)((uintptr_t)dst & 127);
        for (int o = lane * 16 - skew; o < (int)(body_units * 16); o += 64 * 16)
            if (o >= 0) __builtin_nontemporal_store(*(const u32x4 *)(lds + o), (u32x4 *)(dst + o));
    } else {
        // raw chunk: each lane still holds its sub-block (2 rows) in registers
        const int have = min(max(rows - 2 * lane, 0), 2);
        u32x4 *p = (u32x4 *)(dst + lane * Geo::kSubBytes);
#pragma unroll
        for (int k = 0; k < W / 4; ++k)
            if (k * 2 < have * (W / 4)) {
                u32x4 v;
                v[0] = sym[4 * k]; v[1] = sym[4 * k + 1]; v[2] = sym[4 * k + 2]; v[3] = sym[4 * k + 3];
                p[k] = v;
            }
    }
    if (leads && wave == 0) {
        const CoderArgs scan = args_again(first, item);
        scan_sizes(scan, KV == 2 ? scan.total_wgs : scan.wg_base + (scan.chunks + NW - 1) / NW);
    }
}

// ---- launchers ----------------------------------------------------------------------------------

// LDS that nothing uses, for rotated K blocks of 64 rows: the kernel leaves room for three workgroups on a compute unit, and a
// launch of more than three and up to five per unit takes three and then one or two beside an idle rest.  With 40000
// bytes more they go two at a time (fp16, 880, 1024, 1136 and 1264 workgroups, compress call of 4 bits without / with: 153 143, 161
// 155, 190 185, 197 196 us; 3 bits 154 145, 161 155, 191 189, 199 201; bf16 5 % up to four per unit, level above).  8-bit codes
// have two workgroups by their LDS, groups of 128 by their registers, groups of 32 have four.
static unsigned encode_hold(int bits, int group, bool is_v, bool rotate, unsigned wgs)
{
    return rotate && !is_v && group == 64 && bits < 8 && wgs > 3 * 256 && wgs <= 5 * 256 ? 40000 : 0;
}

// Launches the kernel, or (with `resident`) says how many of its workgroups the chip has at once: asked once per kernel, where a launch
// has no LDS besides the kernel's own; 0 where there is no answer.
template <void (*KERNEL)(CoderBatch), int NW> static int encode_start(const CoderBatch &placed, unsigned wgs, unsigned lds, hipStream_t s, int *resident)
{
    if (resident) {
        static std::atomic<int> known{-1};
        int per_unit = lds == 0 ? known.load(std::memory_order_relaxed) : -1;
        if (per_unit < 0) {
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_unit, (const void *)KERNEL, NW * 64, lds) != hipSuccess) {
                (void)hipGetLastError();
                per_unit = 0;
            } else if (lds == 0) known.store(per_unit, std::memory_order_relaxed);
        }
        *resident = per_unit * 256;
        return KVC_OK;
    }
    hipLaunchKernelGGL(KERNEL, dim3(wgs), dim3(NW * 64), lds, s, placed);
    return launched();
}

template <int BITS, int G, int DT, int KV, int NW> static int encode_launch(const CoderBatch &b, hipStream_t s, int *resident)
{
    CoderBatch placed = b;
    if (KV == 2) placed.n = b.n / 2;                  // requests
    unsigned need = 0;
    for (int i = 0; i < placed.n; ++i) {
        placed.at.start[i] = need;
        need += KV == 2 ? b.item[2 * i].total_wgs : (unsigned)((item_chunks(b, i) + NW - 1) / NW);
    }
    close_places(placed.at, placed.n, need, 0);
    const unsigned front = placed.front * (unsigned)placed.n;
    if (resident) *resident = 0;
    if (front + need == 0) return KVC_OK;
    const unsigned lds = encode_hold(BITS, G, KV == 1, b.rotate != 0, need);
#define KVC_ENCODE(D, ...) return encode_start<encode_kernel<BITS, G, DT, KV, D, __VA_ARGS__>, NW>(placed, front + need, lds, s, resident)
    // the K kernels and the V kernels for groups of 32 channels have variants for launches without a
    // transform (its code costs the plain path registers); both tensors together run without one only
    constexpr bool kPlain = KV != 1 || G == 32;
    if (!b.rotate && !(item_has_anchors(b.item[0]) && kPlain)) {
        if (b.dense) KVC_ENCODE(true, !kPlain, NW); else KVC_ENCODE(false, !kPlain, NW);
    }
    if constexpr (KV != 2) {
        if (b.rotate) { if (b.dense) KVC_ENCODE(true, false, NW, true); else KVC_ENCODE(false, false, NW, true); }
        else if (b.dense) KVC_ENCODE(true, true, NW); else KVC_ENCODE(false, true, NW);
    }
    return KVC_ERR_UNSUPPORTED;
#undef KVC_ENCODE
}

// (the kernels for both tensors come with four and, where the registers allow, with eight chunks per
// workgroup, see shared_waves)
template <int BITS, int G, int DT, int KV> static int encode_waves(const CoderBatch &b, hipStream_t s, int *resident)
{
    if constexpr (KV == 2 && G == 32 && BITS != 8)
        if (b.waves == 8) return encode_launch<BITS, G, DT, KV, 8>(b, s, resident);
    return encode_launch<BITS, G, DT, KV, enc_waves(BITS)>(b, s, resident);
}

template <int DT, int KV> static int encode_g(int group, const CoderBatch &a, hipStream_t s, int *resident)
{
    switch (group) {
    case 32: return encode_waves<KVC_BITS, 32, DT, KV>(a, s, resident);
    case 64: return encode_waves<KVC_BITS, 64, DT, KV>(a, s, resident);
    case 128: return encode_waves<KVC_BITS, 128, DT, KV>(a, s, resident);
    }
    return KVC_ERR_UNSUPPORTED;
}

#define KVC_PASTE2(a, b) a##b
#define KVC_PASTE(a, b) KVC_PASTE2(a, b)

int KVC_PASTE(launch_encode_bits, KVC_BITS)(int kv, int group, int dtype, const CoderBatch &a, hipStream_t s, int *resident)
{
    switch (kv) {
    case 0: return dtype == DT_F16 ? encode_g<DT_F16, 0>(group, a, s, resident) : encode_g<DT_BF16, 0>(group, a, s, resident);
    case 1: return dtype == DT_F16 ? encode_g<DT_F16, 1>(group, a, s, resident) : encode_g<DT_BF16, 1>(group, a, s, resident);
    }
    return dtype == DT_F16 ? encode_g<DT_F16, 2>(group, a, s, resident) : encode_g<DT_BF16, 2>(group, a, s, resident);
}

}  // namespace kvc
