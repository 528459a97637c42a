// Exhaustive device-side checks of the arithmetic shortcuts the quantizer kernels rely on.
// Each check counts, over the whole domain on which the kernels use a shortcut, the inputs for
// which it differs from the plain IEEE operation it stands for; all counts must be zero.
// The last count is for the waits of the encoder's prefix sum and of its code tables.
#include "kvc_huff_fetch.h"

namespace kvc {

__device__ __forceinline__ void count(unsigned long long *slot, unsigned long long bad)
{
    // one atomic per wave
    const unsigned long long m = __builtin_amdgcn_ballot_w64(bad != 0);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(((threadIdx.x & 63) ^ d) << 2, (int)(uint32_t)bad);
        bad += lo;
    }
    if (m != 0 && (threadIdx.x & 63) == 0) atomicAdd(slot, bad);
}

// range / (2^BITS - 1), limited to 65504 as the metadata stores it, for every non-negative float
// range including +infinity (max - min of two finite bfloat16 values can overflow).  fp16 input
// only reaches ranges up to 2 * 65504, where the limit never applies and the quotient itself is
// compared.
template <int BITS> __global__ __launch_bounds__(256) void selftest_div_kernel(unsigned long long *slot)
{
    constexpr float qmax = (float)((1 << BITS) - 1);
    const uint32_t last = 0x7f800000u;                     // +infinity
    unsigned long long bad = 0;
    for (unsigned long long u = blockIdx.x * 256ull + threadIdx.x; u <= last; u += gridDim.x * 256ull) {
        const float r = __uint_as_float((uint32_t)u);
        const float want = fminf(r / qmax, 65504.0f);      // correctly rounded division
        bad += __float_as_uint(fminf(rounded_f32(div_levels<BITS>(r)), 65504.0f)) != __float_as_uint(want);
    }
    count(slot, bad);
}

// 1 / s for every positive finite fp16 s
__global__ __launch_bounds__(256) void selftest_rcp_kernel(unsigned long long *slot)
{
    unsigned long long bad = 0;
    for (uint32_t h = blockIdx.x * 256u + threadIdx.x; h < 0x7c00u; h += gridDim.x * 256u) {
        if (h == 0) continue;
        const float s = f16_bits_to_f32(h);
        bad += __float_as_uint(rcp_f16_exact(s)) != __float_as_uint(1.0f / s);
    }
    count(slot, bad);
}

// x - zero for every pair of finite fp16 values (both halves of the packed register)
__global__ __launch_bounds__(256) void selftest_minus_kernel(unsigned long long *slot)
{
    unsigned long long bad = 0;
    const float one = opaque_one();
    const uint32_t zb = blockIdx.x;                        // one zero point per workgroup
    if ((zb & 0x7c00u) != 0x7c00u) {
        const float zero = f16_bits_to_f32(zb);
        for (uint32_t xb = threadIdx.x; xb < 0x10000u; xb += 256u) {
            if ((xb & 0x7c00u) == 0x7c00u) continue;
            const u32x4 r = {xb | (xb << 16), 0u, 0u, xb << 16};
            const float want = rounded_f32(f16_bits_to_f32(xb)) - zero;
            bad += __float_as_uint(elem_minus<DT_F16>(r, 0, zero, one)) != __float_as_uint(want);
            bad += __float_as_uint(elem_minus<DT_F16>(r, 1, zero, one)) != __float_as_uint(want);
            bad += __float_as_uint(elem_minus<DT_F16>(r, 7, zero, one)) != __float_as_uint(want);
        }
    }
    count(slot, bad);
}

// float -> byte conversion with insertion, for every float in [0, 255]: round to nearest even,
// placed in the selected byte, the other bytes kept
__global__ __launch_bounds__(256) void selftest_byte_kernel(unsigned long long *slot)
{
    const uint32_t last = 0x437f0000u;                     // 255.0f
    unsigned long long bad = 0;
    for (unsigned long long u = blockIdx.x * 256ull + threadIdx.x; u <= last; u += gridDim.x * 256ull) {
        const float t = __uint_as_float((uint32_t)u);
        const uint32_t want = (uint32_t)__builtin_rintf(t);
        const uint32_t keep = 0xa5c3961eu;
        bad += __builtin_amdgcn_cvt_pk_u8_f32(t, 0, keep) != ((keep & 0xffffff00u) | want);
        bad += __builtin_amdgcn_cvt_pk_u8_f32(t, 1, keep) != ((keep & 0xffff00ffu) | (want << 8));
        bad += __builtin_amdgcn_cvt_pk_u8_f32(t, 2, keep) != ((keep & 0xff00ffffu) | (want << 16));
        bad += __builtin_amdgcn_cvt_pk_u8_f32(t, 3, keep) != ((keep & 0x00ffffffu) | (want << 24));
    }
    count(slot, bad);
}

// ---- the waits of the encoder's prefix sum (kvc_scan.h), with a limit of about a millisecond ----------

constexpr int kScanTestLimit = 1024;
constexpr int kScanTestWgs = 3;                    // one K workgroup, two V workgroups, one wave each

static __device__ struct ScanTestMemory {
    unsigned long long state[8];
    uint32_t ticket[64];
    uint32_t payload[64];                          // header, then the directory
    unsigned long long out_bytes;
    int status;
} scan_test;

__device__ __forceinline__ CoderArgs scan_test_args()
{
    CoderArgs a = {};
    a.payload = (uint8_t *)scan_test.payload;
    a.off_dir = 128;
    a.off_bodies = 256;
    a.total_chunks = a.total_wgs = kScanTestWgs;
    a.k_wgs = 1;
    a.ws.state = scan_test.state;
    a.ws.ticket = scan_test.ticket;
    a.out_bytes = &scan_test.out_bytes;
    a.q.status = &scan_test.status;
    return a;
}

__device__ __forceinline__ unsigned long long scan_test_units(long long ticket) { return 5 + 10 * ticket; }

__global__ __launch_bounds__(64) void selftest_scan_start_kernel()
{
    uint32_t *words = (uint32_t *)&scan_test;
    for (unsigned i = threadIdx.x; i < sizeof scan_test / 4; i += 64) words[i] = 0;
}

// Waits (for a few seconds at most) until `ticket` is the next one, sleeps `naps` times 3 us, takes it and, unless
// `silent`, reports a size.
__device__ __forceinline__ bool scan_test_enter(const CoderArgs &a, unsigned ticket, int naps, bool silent)
{
    int spins = 0;
    while (__hip_atomic_load(a.ws.ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != ticket) {
        if (++spins > (1 << 20)) return false;
        __builtin_amdgcn_s_sleep(32);
    }
    for (int i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(127);
    if (lane_id() == 0) {
        atomicAdd(a.ws.ticket, 1u);
        if (!silent)
            __hip_atomic_store(&a.ws.state[ticket], kFlagSize | scan_test_units(ticket), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return true;
}

// The last ticket of a launch is taken 20 ms after the others, as when other work holds the chip: the scanner
// waits for it, however short its limit.
__global__ __launch_bounds__(64) void selftest_scan_late_kernel(unsigned long long *slot)
{
    const CoderArgs a = scan_test_args();
    const unsigned me = blockIdx.x;
    bool good = scan_test_enter(a, me, me == 2 ? 6000 : 0, false);
    if (good && me == 0) scan_sizes(a, kScanTestWgs, kScanTestLimit);
    else if (good) {
        unsigned long long before = 0;
        for (unsigned i = 0; i < me; ++i) before += scan_test_units(i);
        good = wait_for_place(a, me) == (kFlagPrefix | before);
    }
    if (!good && lane_id() == 0) atomicAdd(slot, 1ull);
}

// ... and closes directory and header as if nothing had happened.
__global__ __launch_bounds__(64) void selftest_scan_closed_kernel(unsigned long long *slot)
{
    if (threadIdx.x != 0) return;
    const unsigned long long k = scan_test_units(0), v = scan_test_units(1) + scan_test_units(2);
    const unsigned long long *h = (const unsigned long long *)scan_test.payload;
    const bool good = scan_test.status == 0 && scan_test.out_bytes == 256 + 16 * (k + v) && h[5] == 256 + 16 * (k + v) &&
                      h[13] == 16 * k && h[14] == 256 + 16 * k && h[15] == 16 * v && scan_test.payload[32 + kScanTestWgs] == k + v;
    if (!good) atomicAdd(slot, 1ull);
}

// A running workgroup that reports nothing: the scanner gives up, and the one that waits for its place, with the
// encoder's limit of about a second, stops soon after.
__global__ __launch_bounds__(64) void selftest_scan_silent_kernel(unsigned long long *slot)
{
    const CoderArgs a = scan_test_args();
    const unsigned me = blockIdx.x;
    bool good = scan_test_enter(a, me, 0, me == 1);
    const long long start = wall_clock64();                     // (100 MHz)
    if (good && me == 0) scan_sizes(a, kScanTestWgs, kScanTestLimit);
    else if (good && me == 2) good = wait_for_place(a, me) == (kFlagPrefix | kNoPlace);
    good = good && wall_clock64() - start < 5000000;            // 50 ms
    if (!good && lane_id() == 0) atomicAdd(slot, 1ull);
}

// The request's next launch, two more workgroups, places nothing and waits for nothing.
__global__ __launch_bounds__(64) void selftest_scan_after_kernel(unsigned long long *slot)
{
    CoderArgs a = scan_test_args();
    a.wg_base = kScanTestWgs;
    a.total_wgs = kScanTestWgs + 2;
    const unsigned me = kScanTestWgs + blockIdx.x;
    bool good = scan_test_enter(a, me, 0, false);
    const long long start = wall_clock64();
    if (good && me == kScanTestWgs) scan_sizes(a, a.total_wgs, kScanTestLimit);
    else if (good) good = wait_for_place(a, me) == (kFlagPrefix | kNoPlace);
    good = good && wall_clock64() - start < 5000000;
    if (!good && lane_id() == 0) atomicAdd(slot, 1ull);
}

// A workgroup that never starts: the scanner gives up after the time that it is given, 2 ms here.
__global__ __launch_bounds__(64) void selftest_scan_absent_kernel(unsigned long long *slot)
{
    const CoderArgs a = scan_test_args();
    bool good = scan_test_enter(a, 0, 0, false);
    const long long start = wall_clock64();
    if (good) scan_sizes(a, kScanTestWgs, kScanTestLimit, 200000);
    const long long took = wall_clock64() - start;
    good = good && took >= 200000 && took < 5000000;
    if (!good && lane_id() == 0) atomicAdd(slot, 1ull);
}

// Nothing has been closed and the request's status says so.
__global__ __launch_bounds__(64) void selftest_scan_open_kernel(unsigned long long *slot)
{
    if (threadIdx.x != 0) return;
    bool good = scan_test.status == KVC_DEV_SCAN_TIMEOUT && scan_test.out_bytes == 0;
    for (int i = 0; i < 64; ++i) good = good && scan_test.payload[i] == 0;
    if (!good) atomicAdd(slot, 1ull);
}

// ---- the wait for a code table (kvc_huff_fetch.h) ----------------------------------------------------

static __device__ struct __attribute__((aligned(128))) TableTestMemory {
    CandidateTables tables[1];                     // (right in front of the ticket)
    uint32_t ticket[64];
    int status;
} table_test;

__device__ __forceinline__ CoderArgs table_test_args()
{
    CoderArgs a = {};
    a.ws.ticket = table_test.ticket;
    a.q.status = &table_test.status;
    return a;
}

__device__ __forceinline__ uint32_t table_test_entry(int word) { return 0x30005000u | (uint32_t)(2 * word + 1) << 16 | (uint32_t)(2 * word); }

__global__ __launch_bounds__(256) void selftest_table_start_kernel()
{
    uint32_t *words = (uint32_t *)&table_test;
    for (unsigned i = threadIdx.x; i < sizeof table_test / 4; i += 256) words[i] = 0;
}

// Workgroup 0, four waves, waits for its table; workgroup 1 (where there is one) leaves it after `naps` times 3 us, the first
// candidate too long and one word of the second later than all others, and `short_of` words of it never.
// there: whether all four waves have to find it, or have to give up within 50 ms.
__global__ __launch_bounds__(256) void selftest_table_wait_kernel(unsigned long long *slot, int limit, int naps, int short_of, int there)
{
    const CoderArgs a = table_test_args();
    const int tid = threadIdx.x;
    CandidateTables *tables = candidate_tables(a.ws.ticket, 0);
    if (blockIdx.x == 1) {
        if (tid >= 64) return;
        for (int i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(127);
        if (tid == 0) {
            __hip_atomic_store(&tables->state[1], kComplete, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&tables->state[0], kTooLong, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        for (int w = tid; w < 127; w += 64) __hip_atomic_store(&tables->entry[1][w], table_test_entry(w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(127);
        if (tid == 0 && short_of == 0) __hip_atomic_store(&tables->entry[1][127], table_test_entry(127), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    __shared__ EncTables enc;
    __shared__ uint32_t state;
    if (tid == 0) state = kNobody;
    __syncthreads();
    const long long start = wall_clock64();                     // (100 MHz)
    int pick = -1;
    const bool found = wait_for_table(a, enc, &state, pick, limit);
    bool good = found == (there != 0) && (pick == -1 || (there && pick == 1));
    good = good && (there || wall_clock64() - start < 5000000);
    __syncthreads();
    if (there) {
        const uint32_t e = table_test_entry(tid >> 1) >> 16 * (tid & 1) & 0xffffu;
        good = good && enc.code[tid] == (uint16_t)e && enc.len[tid] == (uint8_t)(e >> 12);
    }
    if (__builtin_amdgcn_ballot_w64(!good) != 0 && lane_id() == 0) atomicAdd(slot, 1ull);
}

// The status word and the carry say that somebody gave up, or nothing.
__global__ __launch_bounds__(64) void selftest_table_end_kernel(unsigned long long *slot, int failed)
{
    if (threadIdx.x != 0) return;
    const bool good = table_test.status == (failed ? KVC_DEV_SCAN_TIMEOUT : 0) && scan_failed(table_test_args()) == (failed != 0);
    if (!good) atomicAdd(slot, 1ull);
}

} // namespace kvc

extern "C" int kvc_selftest(uint64_t *counts, void *stream)
{
    using namespace kvc;
    if (counts == nullptr) return KVC_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    unsigned long long *c = (unsigned long long *)counts;
    launch_fill_u32((uint32_t *)counts, 0u, 2 * KVC_SELFTEST_COUNTS, s);
    selftest_div_kernel<2><<<4096, 256, 0, s>>>(c + 0);
    selftest_div_kernel<3><<<4096, 256, 0, s>>>(c + 1);
    selftest_div_kernel<4><<<4096, 256, 0, s>>>(c + 2);
    selftest_div_kernel<8><<<4096, 256, 0, s>>>(c + 3);
    selftest_rcp_kernel<<<124, 256, 0, s>>>(c + 4);
    selftest_minus_kernel<<<65536, 256, 0, s>>>(c + 5);
    selftest_byte_kernel<<<4096, 256, 0, s>>>(c + 6);
    selftest_scan_start_kernel<<<1, 64, 0, s>>>();
    selftest_scan_late_kernel<<<kScanTestWgs, 64, 0, s>>>(c + 7);
    selftest_scan_closed_kernel<<<1, 64, 0, s>>>(c + 7);
    selftest_scan_start_kernel<<<1, 64, 0, s>>>();
    selftest_scan_silent_kernel<<<kScanTestWgs, 64, 0, s>>>(c + 7);
    selftest_scan_after_kernel<<<2, 64, 0, s>>>(c + 7);
    selftest_scan_open_kernel<<<1, 64, 0, s>>>(c + 7);
    selftest_scan_start_kernel<<<1, 64, 0, s>>>();
    selftest_scan_absent_kernel<<<1, 64, 0, s>>>(c + 7);
    selftest_scan_open_kernel<<<1, 64, 0, s>>>(c + 7);
    // a table that comes late, word by word; one that never does; one that stays a word short
    selftest_table_start_kernel<<<1, 256, 0, s>>>();
    selftest_table_wait_kernel<<<2, 256, 0, s>>>(c + 7, kSpinLimit, 600, 0, 1);
    selftest_table_end_kernel<<<1, 64, 0, s>>>(c + 7, 0);
    selftest_table_start_kernel<<<1, 256, 0, s>>>();
    selftest_table_wait_kernel<<<1, 256, 0, s>>>(c + 7, kScanTestLimit, 0, 0, 0);
    selftest_table_end_kernel<<<1, 64, 0, s>>>(c + 7, 1);
    selftest_table_start_kernel<<<1, 256, 0, s>>>();
    selftest_table_wait_kernel<<<2, 256, 0, s>>>(c + 7, kScanTestLimit, 0, 1, 0);
    selftest_table_end_kernel<<<1, 64, 0, s>>>(c + 7, 1);
    return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_DEVICE;
}
