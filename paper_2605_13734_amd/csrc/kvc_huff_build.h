// Lossless stage, code construction: Huffman lengths and canonical codes from the samples that the set-up kernel
// counted.  A part of the encoder (kvc_huff_enc.hip): the workgroups with a request's first tickets build its code tables while
// the others load and quantize their chunks, which takes no table.  The construction is a chain of LDS round trips, 14 us whatever the
// size of the call; as a launch of its own it left the chip idle that long (compress call of one layer of 32k tokens, 8 heads,
// fp16, 4 bits: 66.1 us, so 56.2; of 1000 tokens 40 and 33; 32 requests of 512 to 2048 tokens and 256 heads 1365 and 1348; 80
// layers of 32k tokens 2300 and 2293).
#pragma once

#include "kvc_huff.h"

namespace kvc {

constexpr uint32_t kNone = 1u << 28;           // a queue entry that does not exist: above every weight, and two of them still add up
constexpr int kWeightBits = 19;                // weights are below 2^19 (a table sample is at most 16 chunks of 16 KB)

struct BuildLds {
    uint32_t key[256];             // weight << 8 | symbol
    uint32_t sw[512];              // leaf weights by (weight, symbol): the first queue, then kNone
    uint32_t wi[512];              // weights of the joined nodes in order of creation, the second queue, then kNone
    uint16_t parent_leaf[256];     // by queue position: the joined node above the leaf
    uint16_t parent_int[256];      // by joined node: the joined node above it
    uint32_t block_count[4][16];   // symbols of each length in each block of 64 symbols
    uint16_t entry[256];           // the finished table
    uint32_t too_long;             // a symbol has a code longer than the limit
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
// round trips, eight ways each).  One join after the other, an LDS round trip each, a construction
// took 37 us; now 14 us, of which 11 rounds take 8 us and the sort 3 us (bound by the LDS reads of the keys).
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

// One construction of code lengths, by a workgroup of THREADS threads with the symbols tid, tid + THREADS, ... of weight w each:
// d = the symbols' lengths.
template <int THREADS, int N> __device__ __forceinline__ void build_once(BuildLds &s, const uint32_t w[N], int d[N])
{
    const int tid = threadIdx.x;
    const bool mine = tid < 256;               // (the other threads of a large workgroup only keep its barriers)
    uint32_t key[N];
    int pos[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int sym = tid + i * THREADS;
        key[i] = (w[i] << 8) | (uint32_t)sym;
        pos[i] = 0;
        if (mine) {
            s.key[sym] = key[i];
            s.wi[sym] = s.wi[256 + sym] = s.sw[256 + sym] = kNone;
        }
    }
    if (tid == 0) s.too_long = 0;
    __syncthreads();
    // position of the threads' leaves among all leaves
    if (mine) {
#pragma unroll 2
        for (int t = 0; t < 256; t += 32) {
            uint32_t less[N] = {};
#pragma unroll
            for (int j = 0; j < 32; j += 4) {
                const u32x4 k = *(const u32x4 *)(s.key + t + j);
#pragma unroll
                for (int i = 0; i < N; ++i)
                    less[i] = push_less(push_less(push_less(push_less(less[i], k[0], key[i]), k[1], key[i]), k[2], key[i]), k[3], key[i]);
            }
#pragma unroll
            for (int i = 0; i < N; ++i) pos[i] += __builtin_popcount(less[i]);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) s.sw[pos[i]] = w[i];
    }
    __syncthreads();
    if (tid < 64) join_rounds(s);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        d[i] = 1;
        if (!mine) continue;
        for (int p = s.parent_leaf[pos[i]]; p != 254 && d[i] < 256; p = s.parent_int[p]) ++d[i];
    }
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

// Candidate `number` / tables of the (number % tables)-th table in use, by a workgroup of THREADS threads (the candidates
// without a halving, which are the usual picks, have the first tickets).  Its words go past the caches, each telling by itself that
// it is there, so nothing has to keep them in order.
template <int THREADS> __device__ __forceinline__ void build_table(const CoderArgs &a, int number, BuildLds &s)
{
    constexpr int N = THREADS >= 256 ? 1 : 256 / THREADS;
    const int tid = threadIdx.x, wave = wave_id(), lane = lane_id();
    const int tables = a.builders / kCandidates, k = number / tables;
    const bool mine = tid < 256;
    uint32_t in_use = (uint32_t)a.slots & 255u;
    int slot = __builtin_ctz(in_use);
    for (int i = number - k * tables; i > 0; --i) {
        in_use &= in_use - 1;
        slot = __builtin_ctz(in_use);
    }
    uint8_t *lengths = a.payload + a.off_aux;
    __builtin_amdgcn_s_setprio(3);             // (a chain of LDS round trips that everybody waits for, beside waves busy quantizing)
    if (number == 0)                           // a width the tensor does not use: an empty table
        for (int q = 0; q < a.slots >> 8; ++q)
            if (!((a.slots >> q) & 1))
                for (int i = tid; i < 256; i += THREADS) lengths[256 * q + i] = 0;
    uint32_t w[N];
    int L[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        uint32_t count = 0;
        if (mine) {
#pragma unroll
            for (int c = 0; c < kSampleChunks; ++c) count += a.ws.sample[(slot * kSampleChunks + c) * 256 + tid + i * THREADS];
        }
        w[i] = halved(min(count, 1u << 18) + 1, k);
    }
    build_once<THREADS, N>(s, w, L);
    // canonical codes: first code of every length, and the symbol's place among the symbols of
    // its length (those of lower blocks, then the lower lanes of its own block)
    int within[N];
    bool too_long = false;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        within[i] = 0;
        if (!mine) continue;                   // (whole waves)
        too_long |= L[i] > kMaxLen;
#pragma unroll
        for (int l = 1; l <= kMaxLen; ++l) {
            const unsigned long long same = __builtin_amdgcn_ballot_w64(L[i] == l);
            if (lane == 0) s.block_count[wave + i * (THREADS / 64)][l] = (uint32_t)__builtin_popcountll(same);
            if (L[i] == l) within[i] = __builtin_popcountll(same & ((1ull << lane) - 1));
        }
    }
    if (too_long) s.too_long = 1;
    __syncthreads();
    CandidateTables *out = candidate_tables(a.ws.ticket, slot);
    if (s.too_long) {
        if (tid == 0) __hip_atomic_store(&out->state[k], kTooLong, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_setprio(0);
        return;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (!mine) continue;
        uint32_t next = 0, first = 0;
#pragma unroll
        for (int l = 1; l <= kMaxLen; ++l) {
            if (L[i] == l) first = next;
            next = (next + s.block_count[0][l] + s.block_count[1][l] + s.block_count[2][l] + s.block_count[3][l]) << 1;
        }
        uint32_t rank = (uint32_t)within[i];
        for (int b = 0; b < wave + i * (THREADS / 64); ++b) rank += s.block_count[b][L[i]];
        s.entry[tid + i * THREADS] = (uint16_t)((first + rank) | ((uint32_t)L[i] << 12));
        // no halving is the usual pick (and the only one of an empty request); the encoder's first workgroup
        // writes the lengths of any other
        if (k == 0) lengths[256 * slot + tid + i * THREADS] = (uint8_t)L[i];
    }
    __syncthreads();
    if (tid < 128) __hip_atomic_store(&out->entry[k][tid], ((const uint32_t *)s.entry)[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0) __hip_atomic_store(&out->state[k], kComplete, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_setprio(0);
}

}  // namespace kvc
