// Lossless stage, encoder: a workgroup's code table, from memory to LDS once it has been built.  Used by the encoder
// (kvc_huff_enc.hip) and by the device self-test of its waits.
#pragma once

#include "kvc_scan.h"

namespace kvc {

// Encoder tables in LDS: code lengths as bytes, and code | length << 12 as 16-bit entries
// (narrow entries keep the hot byte values of a section in distinct banks).
struct __attribute__((aligned(8))) EncTables {
    uint8_t len[256];
    uint16_t code[256];
};

// two symbols of a code table (a word of CandidateTables)
__device__ __forceinline__ void put_entries(EncTables &t, int word, uint32_t e)
{
    ((uint32_t *)t.code)[word] = e;
    ((uint16_t *)t.len)[word] = (uint16_t)(((e >> 12) & 15u) | (e >> 28 << 8));
}

template <bool CACHED = false> __device__ __forceinline__ uint32_t table_word(const uint32_t *p)
{
    return CACHED ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
                  : __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The code table of the launch to LDS, by one wave, if it has been built: the candidate with the fewest halvings that meets the
// length limit.  Returns its number, or -1 while it is not there (the same in all lanes).  CACHED: the entries may come from L2, where
// they are for all but the first workgroups of an XCD; what L2 may have instead, zeros from before they were built, shows.
template <bool CACHED> __device__ __forceinline__ int fetch_table(const CandidateTables *tables, EncTables &t)
{
    const int lane = lane_id();
    const uint32_t state = lane < kCandidates ? table_word(&tables->state[lane]) : 0;
    const int pick = __builtin_ctzll(__builtin_amdgcn_ballot_w64(state != kTooLong));
    if (__builtin_amdgcn_readlane((int)state, pick) == 0) return -1;
    const uint32_t e0 = table_word<CACHED>(tables->entry[pick] + lane), e1 = table_word<CACHED>(tables->entry[pick] + 64 + lane);
    if (__builtin_amdgcn_ballot_w64(e0 == 0 || e1 == 0) != 0) return -1;
    put_entries(t, lane, e0);
    put_entries(t, 64 + lane, e1);
    return pick;
}

// The state of a workgroup's table in LDS.
constexpr uint32_t kNobody = 0, kFetching = 1, kThere = 2, kGivenUp = 3;

// Waits for the code table: the first wave of the workgroup to need it polls for it, the others wait at an LDS word (four
// thousand waves asking for the same lines of memory would take turns).  Returns whether it is there.
// The workgroups that build the tables have earlier tickets, so they are running, and they wait for nobody: the wait
// ends; it is bounded by `limit` looks all the same.
__device__ __forceinline__ bool wait_for_table(const CoderArgs &a, EncTables &t, uint32_t *state, int &pick, int limit = kSpinLimit)
{
    uint32_t now = kNobody;
    if (lane_id() == 0) now = atomicCAS(state, kNobody, kFetching);
    now = (uint32_t)__builtin_amdgcn_readfirstlane((int)now);
    if (now == kNobody) {
        const CandidateTables *tables = candidate_tables(a.ws.ticket, a.tab);
        now = kThere;
        for (int spins = 1; (pick = fetch_table<false>(tables, t)) < 0; ++spins) {
            if ((spins & (kSpinCheck - 1)) == 0 && (spins > limit || scan_failed(a))) {
                give_up(a);
                now = kGivenUp;
                break;
            }
            __builtin_amdgcn_s_sleep(4);
        }
        wave_sync();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane_id() == 0) __hip_atomic_store(state, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return now == kThere;
    }
    // (the fetching wave always ends: it finds the table or its limit)
    while ((now = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) == kFetching) __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    return now == kThere;
}

}  // namespace kvc
