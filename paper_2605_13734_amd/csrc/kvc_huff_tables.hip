// Lossless stage, set-up kernels: the call's prologue and the table samples (byte counts of up to 16 chunks per section), and the
// decode tables.  See kvc_huff.h; the code construction is in kvc_huff_build.h, a part of the encoder.

#include "kvc_huff.h"

namespace kvc {

// ---- set-up of a call: prologues and table samples -------------------------------------------------

// Counts the bytes of the lane's packed codes of its 8 rows (tile row 4*i + rsub of the wave's pass, `rows` of
// the pass exist).  The width is a run-time value here: this is a few chunks per call, and one kernel for
// all widths, groups and both tensors lets one launch sample all of them.
template <int DT, bool IS_V>
__device__ __forceinline__ void count_rows(const u32x4 raw[8], const float zero[8], const float inv[8], int bits, int rows,
                                           uint32_t *hist)
{
    const int rsub = lane_id() >> 4;
    const float one = opaque_one(), qmax = (float)((1 << bits) - 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        uint32_t q[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float t = elem_minus<DT>(raw[i], e, zero[IS_V ? i : e], one) * inv[IS_V ? i : e];
            q[e] = (uint32_t)__builtin_rintf(__builtin_amdgcn_fmed3f(t, 0.0f, qmax));
        }
        if (4 * i + rsub >= rows) continue;
        if (bits == 8) {
#pragma unroll
            for (int e = 0; e < 8; ++e) atomicAdd(&hist[q[e] & 255u], 1u);
            continue;
        }
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) w |= q[e] << (bits * e);
        atomicAdd(&hist[w & 255u], 1u);
        atomicAdd(&hist[(w >> 8) & 255u], 1u);
        if (bits > 2) atomicAdd(&hist[(w >> 16) & 255u], 1u);
        if (bits > 3) atomicAdd(&hist[w >> 24], 1u);
    }
}

// The byte counts of sample chunk i of a table.  A wave takes 32 rows (one load round trip); the waves whose
// rows share K groups exchange their minima and maxima.
template <int DT>
__device__ __forceinline__ void sample_chunk(const SetupArgs &a, const SetupItem &it, const SetupTable &t, int i)
{
    __shared__ uint32_t hist[4][256];                          // one per wave
    __shared__ __attribute__((aligned(16))) float low[4][kDim], high[4][kDim];       // K: a wave's extremes per channel
    const int tid = threadIdx.x, wave = wave_id(), lane = lane_id(), col = lane & 15, rsub = lane >> 4;
#pragma unroll
    for (int w = 0; w < 4; ++w) hist[w][tid] = 0;
    __syncthreads();
    const long long cph = (it.tokens + kChunkRows - 1) / kChunkRows, n = t.heads_covered * cph;
    const long long chunk = (long long)i * n / kSampleChunks;
    if (n > 0 && (i == 0 || (long long)(i - 1) * n / kSampleChunks != chunk)) {      // each chunk is counted once
        const long long slot = chunk / cph, cb = chunk - slot * cph;
        const long long lh = t.head_list ? t.head_list[slot] : slot, l = lh / a.heads, h = lh - l * a.heads;
        const long long row0 = cb * kChunkRows + wave * kPassRows, head_off = l * it.x.stride_layer + h * it.x.stride_head;
        const long long left = it.tokens - row0;
        const int rows = left < kPassRows ? (int)left : kPassRows;      // (below 1 for a wave behind the end: it counts nothing)
        TensorView x = it.x;
        if (t.is_v) x.base = it.v_base;
        bool bad = false;                                       // (reported by the encoder, which reads the same rows)
        u32x4 raw[8];
        if (t.rotate) {
            load_pass<false, true>(x, head_off, row0, it.tokens, raw, bad);
            rotate_rows<DT, 8, true>(raw);
        } else {
            load_pass<false>(x, head_off, row0, it.tokens, raw, bad);
        }
        if (t.anchor_shift >= 0) delta_rows<DT, false, 8>(x, head_off, row0, it.tokens, t.anchor_shift, nullptr, false, raw, bad);
        const float qmax = (float)((1 << t.bits) - 1);
        const float c = t.bits == 2 ? 1.0f / 3 : t.bits == 3 ? 1.0f / 7 : t.bits == 4 ? 1.0f / 15 : 1.0f / 255;
        float zero[8], inv[8];
        if (!t.is_v) {
            float mn2[2], mx2[2];
            k_stats_own<DT, 8, false>(raw, mn2, mx2);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                low[wave][col * 8 + rsub * 2 + e] = mn2[e];
                high[wave][col * 8 + rsub * 2 + e] = mx2[e];
            }
            __syncthreads();                                    // (t and the chunk are the same for the whole workgroup)
            const int share = t.group / kPassRows, w0 = wave & ~(share - 1);
            float mn[8], mx[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                mn[e] = low[w0][col * 8 + e];
                mx[e] = high[w0][col * 8 + e];
            }
            for (int w = w0 + 1; w < w0 + share; ++w)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    mn[e] = fminf(mn[e], low[w][col * 8 + e]);
                    mx[e] = fmaxf(mx[e], high[w][col * 8 + e]);
                }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const GroupParams g = make_group<DT>(mn[e], mx[e], qmax, c);
                zero[e] = g.zero;
                inv[e] = g.inv;
            }
            count_rows<DT, false>(raw, zero, inv, t.bits, rows, hist[wave]);
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                float mn, mx;
                if (t.group == 32) v_row_minmax<32, DT>(raw[r], mn, mx);
                else if (t.group == 64) v_row_minmax<64, DT>(raw[r], mn, mx);
                else v_row_minmax<128, DT>(raw[r], mn, mx);
                const GroupParams g = make_group<DT>(mn, mx, qmax, c);
                zero[r] = g.zero;
                inv[r] = g.inv;
            }
            count_rows<DT, true>(raw, zero, inv, t.bits, rows, hist[wave]);
        }
    }
    __syncthreads();
    // (a chunk has at most 16384 bytes)
    it.sample[(t.slot * kSampleChunks + i) * 256 + tid] = (uint16_t)(hist[0][tid] + hist[1][tid] + hist[2][tid] + hist[3][tid]);
}

// Everything of a compress call with the coder that depends on nothing: grid = (kSampleChunks workgroups per
// table, then the slices of the zero fills; requests).  The sample leaves its counts chunk by chunk, so
// that no histogram has to be cleared first.  One request: 7 us, where a prologue, a K and a V sample in
// a launch each took 17 us.  The encoder builds the tables from the counts (kvc_huff_build.h).
template <int DT> __global__ __launch_bounds__(256) void setup_kernel(SetupArgs a)
{
    const SetupItem &it = a.item[blockIdx.y];
    const unsigned samples = (unsigned)a.tables * kSampleChunks;
    if (blockIdx.x >= samples) {
        write_prologue(it.prologue, (long long)(blockIdx.x - samples) * 256 + threadIdx.x, (long long)(gridDim.x - samples) * 256);
        return;
    }
    sample_chunk<DT>(a, it, a.table[blockIdx.x / kSampleChunks], (int)(blockIdx.x % kSampleChunks));
}

// ---- set-up of a decompress call with the coder ---------------------------------------------------

// grid = (table slots, requests), 512 threads: every workgroup turns the code lengths of its slot into the
// decode table (entry i describes the code word that is a prefix of the 12-bit string i); the first one
// also compares the header and the width tables with the plan's, checks the lengths of all slots (a
// complete prefix code each) and sets the request's status word.  It stays at one launch because
// nothing waits for the check here: a table is only used by kernels that look at the status first.
// (A header check and a table launch with one workgroup per slot that searched the lengths one by one: 4.6 + 13 us.)
__global__ __launch_bounds__(512) void decode_setup_kernel(DecodeSetupArgs a)
{
    const DecodeSetupItem &it = a.item[blockIdx.y];
    __shared__ __attribute__((aligned(16))) uint32_t block_count[16][4];     // symbols of each length in each block of 64 symbols
    __shared__ uint32_t kraft[kTableSlots];
    __shared__ int base[16];                           // from a left-aligned code of a length to its symbol's place
    __shared__ uint16_t by_len[256];                   // symbols by (length, symbol)
    const int sec = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    if (sec > 0 && !((a.slot_mask >> sec) & 1)) return;
    const uint8_t *lengths = (const uint8_t *)it.payload + it.off_aux;
    const int mylen = tid < 256 ? lengths[256 * sec + tid] : 0;
    if (sec == 0) {
        if (tid < kTableSlots) kraft[tid] = 0;
        int diff = tid < 32 && ((a.mask >> tid) & 1u) && it.payload[tid] != it.expect.w[tid];
        for (long long i = tid; i < it.table_bytes; i += 512) diff |= it.tables[i] != it.plan_tables[i];
        diff = __syncthreads_or(diff);
        for (int q = tid >> 8; q < a.slots; q += 2) {
            if (!((a.slot_mask >> q) & 1)) continue;
            const uint32_t l = lengths[256 * q + (tid & 255)];
            atomicAdd(&kraft[q], l >= 1 && l <= (uint32_t)kMaxLen ? 1u << (kMaxLen - l) : 1u << 20);
        }
        __syncthreads();
        if (tid == 0) {
            bool complete = true;
            for (int q = 0; q < a.slots; ++q) complete &= !((a.slot_mask >> q) & 1) || kraft[q] == 1u << kMaxLen;
            *it.status = diff ? KVC_DEV_BAD_HEADER : complete ? 0 : KVC_DEV_BAD_TABLE;
        }
        if (!((a.slot_mask >> sec) & 1)) return;
    }
    // canonical order: the first four waves hold one symbol per thread
    int within = 0;
    if (tid < 256) {
#pragma unroll
        for (int l = 1; l <= kMaxLen; ++l) {
            const unsigned long long same = __builtin_amdgcn_ballot_w64(mylen == l);
            if (lane == 0) block_count[l][wave] = (uint32_t)__builtin_popcountll(same);
            if (mylen == l) within = __builtin_popcountll(same & ((1ull << lane) - 1));
        }
    }
    __syncthreads();
    uint32_t limit[kMaxLen + 1];                       // end of the codes of a length, left aligned
    uint32_t first = 0, at = 0, mine = 0;
#pragma unroll
    for (int l = 1; l <= kMaxLen; ++l) {
        const u32x4 c = *(const u32x4 *)block_count[l];
        const uint32_t n = c[0] + c[1] + c[2] + c[3];
        if (mylen == l) mine = at + (wave > 0 ? c[0] : 0) + (wave > 1 ? c[1] : 0) + (wave > 2 ? c[2] : 0);
        if (tid == 0) base[l] = (int)at - (int)first;
        limit[l] = (first + n) << (kMaxLen - l);
        first = (first + n) << 1;
        at += n;
    }
    // (lengths that are no complete code leave a table that nothing uses; every index stays in range)
    if (tid < 256 && mylen >= 1 && mylen <= kMaxLen) by_len[(mine + within) & 255u] = (uint16_t)tid;
    __syncthreads();
    u32x4 out;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t i = (uint32_t)tid * 8 + k;
        int L = 1;
#pragma unroll
        for (int l = 1; l < kMaxLen; ++l) L += i >= limit[l] ? 1 : 0;
        const uint32_t e = (uint32_t)by_len[((int)(i >> (kMaxLen - L)) + base[L]) & 255] << 8 | (256u - (uint32_t)L);
        out[k >> 1] = (k & 1) ? out[k >> 1] | (e << 16) : e;
    }
    ((u32x4 *)(it.lut + 4096 * sec))[tid] = out;
}

// ---- launchers ----------------------------------------------------------------------------------

int launch_setup(int dtype, const SetupArgs &a, hipStream_t s)
{
    long long most = 1;
    for (int i = 0; i < a.n; ++i) {
        const PrologueItem &it = a.item[i].prologue;
        most = it.zero_words > most ? it.zero_words : most;
        most = it.aux_words > most ? it.aux_words : most;
    }
    const dim3 grid((unsigned)a.tables * kSampleChunks + fill_slices(most), (unsigned)a.n);
    if (dtype == DT_F16) hipLaunchKernelGGL(setup_kernel<DT_F16>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(setup_kernel<DT_BF16>, grid, dim3(256), 0, s, a);
    return launched();
}

int launch_decode_setup(const DecodeSetupArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(decode_setup_kernel, dim3((unsigned)a.slots, (unsigned)a.n), dim3(512), 0, s, a);
    return launched();
}

int launch_encode_section(int kv, int bits, int group, int dtype, const CoderBatch &a, hipStream_t s, int *resident)
{
    switch (bits) {
    case 2: return launch_encode_bits2(kv, group, dtype, a, s, resident);
    case 3: return launch_encode_bits3(kv, group, dtype, a, s, resident);
    case 4: return launch_encode_bits4(kv, group, dtype, a, s, resident);
    case 8: return launch_encode_bits8(kv, group, dtype, a, s, resident);
    }
    return KVC_ERR_UNSUPPORTED;
}

int launch_decode_section(int kv, int bits, int dtype, const CoderBatch &a, hipStream_t s)
{
    switch (bits) {
    case 2: return launch_decode_bits2(kv, dtype, a, s);
    case 3: return launch_decode_bits3(kv, dtype, a, s);
    case 4: return launch_decode_bits4(kv, dtype, a, s);
    case 8: return launch_decode_bits8(kv, dtype, a, s);
    }
    return KVC_ERR_UNSUPPORTED;
}

}  // namespace kvc
