// Lossless stage, set-up kernels: the call's prologue and the table samples (byte counts of up to 16 chunks per section),
// the code construction (Huffman lengths, canonical codes) and the decode tables.  See kvc_huff.h.

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
// a launch each took 17 us; with the build behind it for all requests of the call at once, the set-up
// of 32 requests takes 52 us instead of 134 us (four windows of two samples and a build).
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

// ---- code construction ----------------------------------------------------------------------------

constexpr uint32_t kNone = 1u << 28;           // a queue entry that does not exist: above every weight, and two of them still add up
constexpr int kWeightBits = 19;                // weights are below 2^19 (a table sample is at most 16 chunks of 16 KB)

struct BuildLds {
    uint32_t key[256];             // weight << 8 | symbol
    uint32_t sw[512];              // leaf weights by (weight, symbol): the first queue, then kNone
    uint32_t wi[512];              // weights of the joined nodes in order of creation, the second queue, then kNone
    uint16_t parent_leaf[256];     // by queue position: the joined node above the leaf
    uint16_t parent_int[256];      // by joined node: the joined node above it
};

// bits << 1, with a one at the bottom if a < b (both below 2^31): the sign of the difference is shifted in,
// without the wait states between a compare and the use of its mask
__device__ __forceinline__ uint32_t push_less(uint32_t bits, uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_alignbit(bits, a - b, 31);
}

// How many of the queue entries q[0], q[1], ... weigh less than `w`: N entries at once, STEP apart, per
// level.  The queues end in entries above every weight, and a round's counts are below 64, or at
// most 256 (`wide`), so no index needs a check.
template <int N, int STEP> __device__ __forceinline__ void search_level(const uint32_t *q, uint32_t w, int &below)
{
    uint32_t x[N], less = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = q[below + (i + 1) * STEP - 1];
#pragma unroll
    for (int i = 0; i < N; ++i) less = push_less(less, x[i], w);
    below += __builtin_popcount(less) * STEP;
}

// Huffman's algorithm over 256 symbols, always joining the two nodes with the smallest (weight, id):
// leaves have id = symbol, the k-th joined node has id 256 + k.  Leaves sorted by (weight, symbol)
// form one queue, joined nodes (created in non-decreasing weight order) the other.
//
// The joins are made in rounds by one wave.  With s the sum of the two smallest weights present, every
// node of weight <= s is joined before any node that does not exist yet: a later node weighs at least
// s and has a higher id.  So all nodes of weight <= s, merged from the two queues (a leaf before a joined
// node of the same weight), are joined pair by pair in that order; an odd one out waits for the next
// round.  The weights of a round span a factor of two, so a code takes about as many rounds as it
// has lengths (8 to 24), and a round is a search for every node's place in the other queue (two LDS
// round trips, eight ways each).  One join after the other, an LDS round trip each, this kernel
// took 37 us per call, 55 us for eight requests together; now 15.5 us for either, of which 11 rounds
// take 8 us and the sort 3 us (bound by the LDS reads of the keys).
__device__ __forceinline__ void join_rounds(BuildLds &s)
{
    const int lane = lane_id();
    int lo = 0, jo = 0, made = 0;              // leaves and joined nodes already used, joined nodes made
    for (int round = 0; round < 255 && made < 255; ++round) {      // (a round makes one join at least)
        const uint32_t *leaves = s.sw + lo, *joined = s.wi + jo;
        uint32_t wl = leaves[lane], wj = joined[lane];
        const uint32_t a0 = __builtin_amdgcn_readlane(wl, 0), a1 = __builtin_amdgcn_readlane(wl, 1);
        const uint32_t b0 = __builtin_amdgcn_readlane(wj, 0), b1 = __builtin_amdgcn_readlane(wj, 1);
        const uint32_t sum = min(min(a0 + a1, a0 + b0), b0 + b1);
        int nl = __builtin_popcountll(__builtin_amdgcn_ballot_w64(wl <= sum));      // nodes of weight <= sum in the two queues
        int ni = __builtin_popcountll(__builtin_amdgcn_ballot_w64(wj <= sum));
        const bool wide = nl == 64 || ni == 64;
        if (wide) {
#pragma unroll
            for (int first = 64; first < 256; first += 64) {
                nl += __builtin_popcountll(__builtin_amdgcn_ballot_w64(leaves[first + lane] <= sum));
                ni += __builtin_popcountll(__builtin_amdgcn_ballot_w64(joined[first + lane] <= sum));
            }
        }
        const int most = nl > ni ? nl : ni, used = (nl + ni) & ~1;
        bool leaf_left = false;
        for (int first = 0; first < most; first += 64) {
            const int e = first + lane;
            if (first > 0) {
                wl = leaves[e];
                wj = joined[e];
            }
            wl = e < nl ? wl : 0;              // (nothing weighs less: an idle lane's search stays at the front)
            wj = e < ni ? wj : 0;
            int below_l = 0, below_i = 0;      // joined nodes before the leaf; leaves before the joined node
            if (wide) {
                search_level<4, 64>(joined, wl, below_l);
                search_level<4, 64>(leaves, wj + 1, below_i);
            }
            if (most > 7) {
                search_level<7, 8>(joined, wl, below_l);
                search_level<7, 8>(leaves, wj + 1, below_i);
            }
            search_level<7, 1>(joined, wl, below_l);
            search_level<7, 1>(leaves, wj + 1, below_i);
            const int rank_l = e + below_l, rank_i = e + below_i;
            // the first of a pair finds its partner, the next node of the merged order, and makes the joined node
            // (a weight of `sum` or more, behind everything that this round looks for)
            const uint32_t after_l = min(leaves[e + 1], joined[below_l]), after_i = min(leaves[below_i], joined[e + 1]);
            if (e < nl && rank_l < used) {
                s.parent_leaf[lo + e] = (uint16_t)(made + (rank_l >> 1));
                if (!(rank_l & 1)) s.wi[made + (rank_l >> 1)] = wl + after_l;
            }
            if (e < ni && rank_i < used) {
                s.parent_int[jo + e] = (uint16_t)(made + (rank_i >> 1));
                if (!(rank_i & 1)) s.wi[made + (rank_i >> 1)] = wj + after_i;
            }
            leaf_left |= __builtin_amdgcn_ballot_w64(e < nl && rank_l >= used) != 0;
        }
        wave_sync();
        const int odd = (nl + ni) & 1;
        lo += nl - (odd && leaf_left ? 1 : 0);
        jo += ni - (odd && !leaf_left ? 1 : 0);
        made += used >> 1;
    }
}

// One construction of code lengths, by a workgroup of 256 threads with one symbol of weight w each:
// returns the symbol's length.
__device__ __forceinline__ int build_once(BuildLds &s, uint32_t w)
{
    const int tid = threadIdx.x;
    const uint32_t key = (w << 8) | (uint32_t)tid;
    s.key[tid] = key;
    s.wi[tid] = s.wi[256 + tid] = s.sw[256 + tid] = kNone;
    __syncthreads();
    // position of the thread's leaf among all leaves
    int pos = 0;
#pragma unroll 2
    for (int t = 0; t < 256; t += 32) {
        uint32_t less = 0;
#pragma unroll
        for (int i = 0; i < 32; i += 4) {
            const u32x4 k = *(const u32x4 *)(s.key + t + i);
            less = push_less(push_less(push_less(push_less(less, k[0], key), k[1], key), k[2], key), k[3], key);
        }
        pos += __builtin_popcount(less);
    }
    s.sw[pos] = w;
    __syncthreads();
    if (tid < 64) join_rounds(s);
    __syncthreads();
    int d = 1;
    for (int i = s.parent_leaf[pos]; i != 254 && d < 256; i = s.parent_int[i]) ++d;
    return d;
}

// The format's length limit: while the longest code exceeds kMaxLen all weights are halved (rounded
// up) and the construction is repeated.  k halvings turn a weight w into ceil(w / 2^k), so the
// constructions do not depend on each other: all of them run side by side, one workgroup each, every
// one that meets the limit leaves a complete table, and the encoder takes the one with the fewest
// halvings.  (Groups along 128 tokens or channels give strongly peaked codes that need
// five or six halvings.)
// Ten halvings are always enough: a code of 13 bits needs weights that add up to Fibonacci(15) = 610 or
// more (every weight being 1 or more), and a sample of 2^18 bytes plus one per symbol, halved ten times,
// adds up to less than (2^18 + 256) / 1024 + 256 = 513.
static_assert(kWeightBits >= 19 && (1 << 18) + 256 < (1 << kWeightBits), "sample weights");

__device__ __forceinline__ uint32_t halved(uint32_t w, int k) { return (w + ((1u << k) - 1u)) >> k; }

// grid = kCandidates workgroups of 256 threads (one symbol each) per table slot of the format.
__global__ __launch_bounds__(256) void build_tables_kernel(BuildArgs a)
{
    const BuildItem &it = a.item[blockIdx.y];
    const int sec = blockIdx.x / kCandidates, k = blockIdx.x - sec * kCandidates;
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    if (!((a.slot_mask >> sec) & 1)) {                 // a width the tensor does not use: an empty table
        if (k == 0) it.lengths[256 * sec + tid] = 0;
        return;
    }
    __shared__ __attribute__((aligned(16))) BuildLds s;
    __shared__ uint32_t block_count[4][16];            // symbols of each length in each block of 64 symbols
    uint32_t count = 0;
#pragma unroll
    for (int i = 0; i < kSampleChunks; ++i) count += it.sample[(sec * kSampleChunks + i) * 256 + tid];
    const int L = build_once(s, halved(min(count, 1u << 18) + 1, k));
    CandidateTables *out = candidate_tables(it.lut, sec);
    const int too_long = __syncthreads_or(L > kMaxLen);
    if (tid == 0) out->complete[k] = too_long ? 0 : 1;
    if (too_long) return;
    // canonical codes: first code of every length, and the symbol's place among the symbols of
    // its length (those of lower blocks, then the lower lanes of its own block)
    int within = 0;
#pragma unroll
    for (int l = 1; l <= kMaxLen; ++l) {
        const unsigned long long same = __builtin_amdgcn_ballot_w64(L == l);
        if (lane == 0) block_count[wave][l] = (uint32_t)__builtin_popcountll(same);
        if (L == l) within = __builtin_popcountll(same & ((1ull << lane) - 1));
    }
    __syncthreads();
    uint32_t next = 0, first = 0;
#pragma unroll
    for (int l = 1; l <= kMaxLen; ++l) {
        if (L == l) first = next;
        next = (next + block_count[0][l] + block_count[1][l] + block_count[2][l] + block_count[3][l]) << 1;
    }
    uint32_t rank = (uint32_t)within;
    for (int w = 0; w < wave; ++w) rank += block_count[w][L];
    out->entry[k][tid] = (uint16_t)((first + rank) | ((uint32_t)L << 12));
    // no halving is the usual pick (and the only one of an empty request); the encoder's first workgroup
    // writes the lengths of any other
    if (k == 0) it.lengths[256 * sec + tid] = (uint8_t)L;
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

int launch_build_tables(const BuildArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(build_tables_kernel, dim3((unsigned)(a.slots * kCandidates), (unsigned)a.n), dim3(256), 0, s, a);
    return launched();
}

int launch_decode_setup(const DecodeSetupArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(decode_setup_kernel, dim3((unsigned)a.slots, (unsigned)a.n), dim3(512), 0, s, a);
    return launched();
}

int launch_encode_section(int kv, int bits, int group, int dtype, const CoderBatch &a, hipStream_t s)
{
    switch (bits) {
    case 2: return launch_encode_bits2(kv, group, dtype, a, s);
    case 3: return launch_encode_bits3(kv, group, dtype, a, s);
    case 4: return launch_encode_bits4(kv, group, dtype, a, s);
    case 8: return launch_encode_bits8(kv, group, dtype, a, s);
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
