// Exchange of hidden-state values between workgroups (device side): values that carry their own readiness, so that a consumer that
// sees it also has the value and a stale read is retried.  Either tagged slots of 64 bits (low word fp32 value, high word step tag, one
// 8-byte store publishes both), or stamped words, where a bit that the value leaves free holds a bit of the step count.
#pragma once
#include <hip/hip_runtime.h>

namespace l355 {

typedef unsigned long long u64;

__device__ __forceinline__ u64 pack_slot(float v, unsigned tag)
{
    return ((u64)tag << 32) | (u64)__float_as_uint(v);
}

// fp32 values of h published as one word, with one bit of the step count in the top exponent bit (clear in every |value| < 2).
constexpr unsigned kHStampBit = 0x40000000u;
// A published word without its stamp.  A NaN has bit 30 set itself and |h| <= 1 else: without that bit a (quiet) NaN is a pattern
// of at least 1.5, from which the addition carries into bit 30 again.  strip: kHStampBit, or 0 to take the word
// as it is.
__device__ __forceinline__ float unstamped(unsigned v, unsigned strip)
{
    const unsigned carried = (v & (kHStampBit - 1u)) + 0x00400000u;
    return __uint_as_float((v & ~strip) | (carried & strip));
}

// Pacing of a poll that would otherwise follow the wave's own publication at once.  A device-scope store takes about
// 0.3 us plus half a load round trip to become visible to the other XCDs; a poll round issued before that comes back
// without the value and the next round costs a whole further round trip (about 1 us with a few thousand slots polled by
// every workgroup).  Waiting `units` x 64 clocks first makes the first round the one that succeeds: the bare exchange of
// 3000 slots among 250 workgroups takes 1.83 us per round unpaced and 1.43 us with 10-12 units.  Where a kernel has work
// of its own between publication and poll (outputs, the next step's input products) that work is the pacing.
__device__ __forceinline__ void pace_poll(int units)
{
    for (int i = 0; i < units; ++i) __builtin_amdgcn_s_sleep(1);
}

// One polled slot array: n slots tagged `want` go to dst[0..n).  n = 0 switches the array off.
struct PollSrc {
    const u64* slots;
    float* dst;
    unsigned want;
    int n;
};

// Fetch the tagged values of up to two slot arrays into LDS.  The two arrays are treated as one index space
// so that all outstanding loads of a thread (up to four) are in flight together, whichever array they hit.
__device__ __forceinline__ void gather_tagged2(const PollSrc& A, const PollSrc& Bs, int tid, int nthreads,
                                               int* timeout_flag, unsigned spin_limit)
{
    constexpr int NF = 4;
    const int total = A.n + Bs.n;
    for (int e0 = tid; e0 < total; e0 += NF * nthreads) {
        u64 v[NF];
        unsigned spins = 0;
        bool ok;
        do {
            ok = true;
#pragma unroll
            for (int u = 0; u < NF; ++u) {
                const int e = e0 + u * nthreads;
                const bool second = e >= A.n;
                const u64* p = second ? (Bs.slots + (e - A.n)) : (A.slots + e);
                const unsigned want = second ? Bs.want : A.want;
                v[u] = (e < total) ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ((u64)want << 32);
                ok = ok && ((unsigned)(v[u] >> 32) == want);
            }
            if (!ok) {
                ++spins;
                if (spins > spin_limit) {
                    __hip_atomic_store(timeout_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                if ((spins & 63u) == 0 &&
                    __hip_atomic_load(timeout_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
                    break;
            }
        } while (!ok);
#pragma unroll
        for (int u = 0; u < NF; ++u) {
            const int e = e0 + u * nthreads;
            if (e < total) {
                if (e >= A.n) Bs.dst[e - A.n] = __uint_as_float((unsigned)v[u]);
                else A.dst[e] = __uint_as_float((unsigned)v[u]);
            }
        }
    }
}

__device__ __forceinline__ void gather_tagged(const u64* slots, int H, unsigned want, float* dst, int tid,
                                              int nthreads, int* timeout_flag, unsigned spin_limit)
{
    const PollSrc A{slots, dst, want, H}, none{nullptr, nullptr, 0u, 0};
    gather_tagged2(A, none, tid, nthreads, timeout_flag, spin_limit);
}
// ---- exchange inside one XCD -------------------------------------------------------------------------------------
// The compute units of an XCD share one L2.  A store at workgroup scope is written through the compute unit's vector
// cache into that L2 and stays there; an agent-scope load from any compute unit of the same XCD bypasses its vector
// cache and finds it in the L2.  For workgroups that all run on one XCD this hand-over measured 35-50 % faster than
// agent-scope stores, which travel to memory before anybody sees them (32 workgroups: 1.19 -> 0.78 us per round;
// 16: 1.71 -> 0.86 us).  A workgroup on another XCD would never see such a store, so a group uses it only after it has
// checked, in the launch itself, that its members do share an XCD.  (The loads stay at agent scope: polling loads at
// workgroup scope may be served by the compute unit's own cache and never see anything.)

// id of the XCD this wave runs on (hardware register XCC_ID, bits 3:0)
__device__ __forceinline__ unsigned xcc_id() { return __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)); }

// publish v at p for the other workgroups of the group
template <class T>
__device__ __forceinline__ void exchange_store(T* p, T v, bool same_xcd)
{
    if (same_xcd) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Agent-scope loads of 16 bytes (there is no atomic of that size; values that carry their own stamps need none: each is looked
// at by itself).  A buffer's base and the offset of a block are scalar, so an address takes one register, and a line is asked for once
// where two loads of 8 bytes ask twice.  Only the compiler's memory barrier in front keeps a load from being taken for an earlier
// one's.
// What is assumed of them: a naturally aligned word of 32 bits arrives whole, and one of 64 bits that was written by one store does
// too, as with the atomic loads of that size (persist_split.hip stamps one half of such a word only).  The instruction set promises no
// such thing of the halves of a 16-byte load; a store puts its word into a cache line at once, though, and a lane's sixteen bytes
// are one piece of a line.  Looked for with 16-byte loads against words being rewritten all the time, by device-scope stores and by stores inside an
// XCD: none torn among 2e10, 1.2e9 of them seen to have changed since the load before.  (A stamp in both halves: 1 to 4 % of a step.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t exchange_buffer(const void* base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);   // raw, 32-bit data format
}
// lane_bytes + 16 beyond the buffer's bytes reads zero; scalar_bytes is not checked: it stays inside for every lane_bytes used with it.
template <class T>
__device__ __forceinline__ T exchange_load16(__amdgpu_buffer_rsrc_t buffer, int lane_bytes, int scalar_bytes)
{
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(buffer, lane_bytes, scalar_bytes, 1 << 4 /* sc1 */));
}

// n 32-bit words (dst padded to whole groups of four) from `words`, an array that holds whole groups of four too, into LDS once
// every word's bit `bit` is as in `want`; values may be taken apart from their stamp by `value`.  NF groups of a thread are in flight
// together; groups beyond the array are not fetched (the buffer's bounds).  Bounded: *timeout_flag.
template <int NF, class Value>
__device__ __forceinline__ void gather_stamped(const unsigned* words, int n, unsigned bit, unsigned want, float* dst, int tid, int nthreads,
                                               int* timeout_flag, unsigned spin_limit, Value value)
{
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    const int n4 = (n + 3) >> 2;
    const __amdgpu_buffer_rsrc_t from = exchange_buffer(words, (unsigned)n4 * 16u);
    for (int e0 = 0; e0 < n4; e0 += NF * nthreads) {
        u32x4 v[NF];
        for (unsigned spins = 0;;) {
            asm volatile("" ::: "memory");                               // read anew in every round
#pragma unroll
            for (int u = 0; u < NF; ++u) v[u] = exchange_load16<u32x4>(from, (e0 + u * nthreads + tid) * 16, 0);   // (bounds: the lane's offset)
            __builtin_amdgcn_sched_barrier(0);                           // all on their way before the first is waited for
            unsigned differ = 0;
#pragma unroll
            for (int u = 0; u < NF; ++u) {
                const int left = n - 4 * (e0 + u * nthreads + tid);      // words from this group on
                const unsigned lo = (v[u].x ^ want) | (v[u].y ^ want), hi = (v[u].z ^ want) | (v[u].w ^ want);
                differ |= (left > 0 ? lo : 0u) | (left > 2 ? hi : 0u);   // (n is even)
            }
            if (!__builtin_amdgcn_ballot_w64((differ & bit) != 0u)) break;
            if (++spins > spin_limit) {
                __hip_atomic_store(timeout_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            if ((spins & 63u) == 0 && __hip_atomic_load(timeout_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
        }
#pragma unroll
        for (int u = 0; u < NF; ++u) {
            const int e = e0 + u * nthreads + tid;
            if (e < n4) reinterpret_cast<f32x4*>(dst)[e] = (f32x4){value(v[u].x), value(v[u].y), value(v[u].z), value(v[u].w)};
        }
    }
}

// ... with as many loads in flight as the array has for a thread, up to NF (loads beyond it cost their issue all the same)
template <int NF, class Value>
__device__ __forceinline__ void gather_stamped_all(const unsigned* words, int n, unsigned bit, unsigned want, float* dst, int tid, int nthreads,
                                                   int* timeout_flag, unsigned spin_limit, Value value)
{
    if (n <= 4 * nthreads) gather_stamped<1>(words, n, bit, want, dst, tid, nthreads, timeout_flag, spin_limit, value);
    else if (NF > 2 && n > 8 * nthreads) gather_stamped<NF>(words, n, bit, want, dst, tid, nthreads, timeout_flag, spin_limit, value);
    else gather_stamped<2>(words, n, bit, want, dst, tid, nthreads, timeout_flag, spin_limit, value);
}

// Do the `members` (<= 64) workgroups of this group all run on one XCD?  Every member publishes its XCD id in
// ids[me] (agent scope, tagged `tag`), polls the whole list and compares; all of them read the same list and so
// agree on the answer.  tmp: LDS, `members` floats, free for other use on return.  Called by the whole workgroup.
__device__ __forceinline__ bool group_shares_xcd(u64* ids, int members, int me, unsigned tag, float* tmp, int tid,
                                                 int nthreads, int* timeout_flag, unsigned spin_limit)
{
    if (tid == 0) __hip_atomic_store(ids + me, pack_slot((float)xcc_id(), tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    gather_tagged(ids, members, tag, tmp, tid, nthreads, timeout_flag, spin_limit);
    __syncthreads();
    bool same = true;
    const float first = tmp[0];
    for (int i = 1; i < members; ++i) same = same && (tmp[i] == first);
    __syncthreads();
    return same;
}

}  // namespace l355
