// Lossless stage, encoder: the place of a workgroup's chunk bodies in the payload, a single-pass prefix
// sum over workgroups.  Used by the encoder (kvc_huff_enc.hip) and by the device self-test of its waits.
#pragma once

#include "kvc_huff.h"

namespace kvc {

// Scan state of an encode workgroup: 0, then (bits 63:62 = 1) the sum of its chunks' sizes, then (2) the
// sum of all sizes before it, both in 16-byte units.
constexpr unsigned long long kFlagSize = 1ull << 62, kFlagPrefix = 2ull << 62, kValueMask = (1ull << 40) - 1;
constexpr unsigned long long kNoPlace = kValueMask;      // in the carry word: a scan of this request gave up
constexpr int kScanWindows = 4;
constexpr int kScanCarry = 4;      // word of the ticket's block where the scan of one launch leaves its end to the next
constexpr int kSpinLimit = 1 << 20;
constexpr int kSpinCheck = 256;    // looks between two questions whether the wait is for somebody
constexpr long long kStartLimit = 1000000000;      // ticks of 10 ns: the longest wait for a workgroup to start

// One workgroup = kWaves chunks.  A chunk's body offset is the sum of all earlier bodies of the
// request (K chunks first, then V): a single-pass scan over one state word per workgroup, made by one
// wave per request, the scanner.  Workgroups take a ticket from a counter; as soon as the sizes of its
// chunks are known, before a code word is written, a workgroup leaves their sum in its state word; the
// scanner walks the words in ticket order and puts the prefix in their place; the waves of the
// workgroup, by then mostly done with the code words, pick it up.  The scanner is the first wave of the
// workgroup with the launch's first ticket.  A workgroup waits for the scanner and for workgroups with
// earlier tickets: all of them are running, so the wait ends; it is bounded by kSpinLimit all the same.
// The scanner waits for running workgroups too, but also for tickets that nobody has taken, for as long as
// other work keeps the rest of the launch off the chip: looks count only in the first kind of wait, the second
// ends after ten seconds (calls that overlap on one workspace may have taken each other's tickets).
// (Tickets are counted from behind those of the workgroups that only build code tables, kvc_huff_build.h.)
// Whoever gives up marks the request's carry word: everybody else who waits stops too, no later launch of the
// request places a body, and directory and header stay open.
// (Without a scanner every workgroup looked back over 64 predecessors for itself, after its barrier:
// hundreds of waves polling the same lines of memory.  70B shape, half of its layers, compress call: 1369 us
// with eight chunks per workgroup, now 1213; 2-bit codes / groups of 128 1370 -> 1135, 8 bits (a quarter of
// the layers) 1235 -> 1058.  With the bodies at fixed places, nothing to wait for, 1165.)

__device__ __forceinline__ unsigned long long *scan_carry(const CoderArgs &a)
{
    return (unsigned long long *)(a.ws.ticket + kScanCarry);      // units before this launch; units of K
}

__device__ __forceinline__ bool scan_failed(const CoderArgs &a)
{
    return __hip_atomic_load(scan_carry(a), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kNoPlace;
}

__device__ __forceinline__ void give_up(const CoderArgs &a)
{
    if (lane_id() != 0) return;
    __hip_atomic_store(scan_carry(a), kNoPlace, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    atomicOr(a.q.status, KVC_DEV_SCAN_TIMEOUT);
}

// The scan of one request's launch, whose last workgroup is `end` - 1; the last launch's scanner closes
// the directory and the header.  limit: looks without progress at a workgroup that is running; start_limit: ticks
// without progress for one that is not.
__device__ __forceinline__ void scan_sizes(const CoderArgs &a, long long end, int limit = kSpinLimit, long long start_limit = kStartLimit)
{
    const int lane = lane_id();
    unsigned long long *carry = scan_carry(a);
    unsigned long long prefix = carry[0], k_units = carry[1];
    if (prefix == kNoPlace) return;
    int spins = 0;
    bool nobody = false;               // the next ticket has not been taken
    long long since = 0;               // since when (0: it has, as far as known)
    __builtin_amdgcn_s_setprio(3);
    // kScanWindows windows of 64 workgroups per look (a look is a round trip to memory, and the scanner has to
    // keep up with all workgroups of the chip)
    for (long long next = a.wg_base; next < end;) {
        unsigned long long v[kScanWindows];
#pragma unroll
        for (int k = 0; k < kScanWindows; ++k) {
            const long long j = next + 64 * k + lane;
            v[k] = j < end ? __hip_atomic_load(&a.ws.state[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        }
        bool moved = false, open = true;
        const long long base = next;
#pragma unroll
        for (int k = 0; k < kScanWindows; ++k) {
            if (!open) continue;
            const unsigned long long known = __builtin_amdgcn_ballot_w64((v[k] >> 62) == 1);
            const int run = known == ~0ull ? 64 : __builtin_ctzll(~known);      // workgroups that have reported, up to the first gap
            open = run == 64;
            if (run == 0) continue;
            const uint32_t size = lane < run ? (uint32_t)v[k] : 0;               // (a workgroup's bodies are at most 8 * 1024 units)
            const uint32_t incl = wave_inclusive_sum(size);
            if (lane < run)
                __hip_atomic_store(&a.ws.state[base + 64 * k + lane], kFlagPrefix | (prefix + incl - size), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            const long long k_last = a.k_wgs - 1 - (base + 64 * k);              // the last K workgroup among these?
            if (k_last >= 0 && k_last < run) k_units = prefix + (uint32_t)__builtin_amdgcn_readlane((int)incl, (int)k_last);
            prefix += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            next += run;
            moved = true;
        }
        if (moved) {
            spins = 0;
            since = 0;
            nobody = false;
        } else if ((++spins & (kSpinCheck - 1)) == 0) {
            nobody = (unsigned)(next + a.apart) >= __hip_atomic_load(a.ws.ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (scan_failed(a)) return;
            if (nobody) {
                const long long now = wall_clock64();
                if (since == 0) since = now;
                if (now - since > start_limit) return give_up(a);
                spins = 0;
            } else if (spins > limit) return give_up(a);
        }
        if (nobody) __builtin_amdgcn_s_sleep(32);
    }
    if (lane != 0 || scan_failed(a)) return;
    carry[0] = prefix;
    carry[1] = k_units;
    if (end != a.total_wgs) return;
    ((uint32_t *)(a.payload + a.off_dir))[a.total_chunks] = (uint32_t)prefix;
    const unsigned long long total = (unsigned long long)a.off_bodies + prefix * 16;
    unsigned long long *h = (unsigned long long *)a.payload;
    h[5] = total;                                   // byte 40: total bytes
    h[13] = k_units * 16;                           // byte 104: K code bytes
    h[14] = (unsigned long long)a.off_bodies + k_units * 16;   // byte 112: V code offset
    h[15] = (prefix - k_units) * 16;                // byte 120: V code bytes
    *a.out_bytes = total;
}

// The prefix of the workgroup with this ticket, left in its state word by the scanner, or kNoPlace.
__device__ __forceinline__ unsigned long long wait_for_place(const CoderArgs &a, long long ticket, int limit = kSpinLimit)
{
    unsigned long long excl;
    int spins = 0;
    while (((excl = __hip_atomic_load(&a.ws.state[ticket], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 62) != 2) {
        if ((++spins & (kSpinCheck - 1)) == 0 && (spins > limit || scan_failed(a))) {
            give_up(a);
            return kFlagPrefix | kNoPlace;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return excl;
}

}  // namespace kvc
