// Device-side pieces shared by the persistent kernels: work shares, bounded waits,
// the XCD-local hand-off of partial results.
#pragma once
#include "fused.h"

namespace ghd {

constexpr long long kWaitTicks = 2000000;   // bounded waits give up after 20 ms (100 MHz clock)

#define GLOBAL __attribute__((address_space(1)))

// a pointer to device memory, as such (a pointer read from memory is otherwise taken to point
// anywhere, and accessed with slower instructions)
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gp(T* p)
{
    return (__attribute__((address_space(1))) T*)p;
}

// keeps the compiler from moving memory operations, MFMAs or anything else across this point
// (a load ring only works if its loads are issued where they are written)
__device__ __forceinline__ void pin_order()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Kernels whose first loads must not wait for the argument block have what those need in their first twelve words,
// which the hardware puts into scalar registers (see LinHead), and the block behind them.
constexpr int kTailAt = 48;      // byte offset of FusedArgs in the kernel arguments
// FusedArgs as it lies in the kernel arguments.  The (empty) asm makes the pointer opaque:
// no read through it is moved ahead of this point.
typedef const __attribute__((address_space(4))) FusedArgs* ArgPtr;
__device__ __forceinline__ ArgPtr late_args()
{
    typedef const __attribute__((address_space(4))) char* kernarg_bytes;
    kernarg_bytes p = (kernarg_bytes)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p)::"memory");
    return (ArgPtr)(p + kTailAt);
}

struct Ctx {
    int j, G;            // logical workgroup index, number of workgroups
    char* lds;           // dynamic LDS
    int source[2];       // attention in one launch: see mask_source
    bool parents;        // ... whether that is parent[]
};

// What waits look with: a load at the scope of the counting atomics, past this compute unit's L1.  (A
// read-modify-write that changes nothing, atomicOr(p, 0), is compiled to the same load.)
__device__ __forceinline__ uint32_t ld_relaxed(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Partial results stay inside an XCD.  Workgroup i runs on the XCD of i % 8 (see arrive); an item
// - a block of a linear layer's tiles, a head - that several workgroups share is dealt to workgroups
// of one XCD, and its partial results go through that XCD's L2 with plain stores and loads: every
// wavefront waits for the acknowledgement of its own stores before the barrier after which thread 0
// bumps the item's counter, and a reader's first access to a slot line in a launch cannot hit in its
// L1.  No device-scope fence (a write-back and invalidate of a whole L2, about 4 us here) is needed
// anywhere inside a launch.

// Every wavefront calls this before the barrier that precedes a counter bump: it returns
// once the wavefront's own stores have been acknowledged by the L2, i.e. are visible to
// the other compute units of the XCD.  (The barrier alone orders the wavefronts of the
// workgroup, not their stores still on the way to the L2.)  s_waitcnt vmcnt(0).
__device__ __forceinline__ void wait_own_stores() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// a barrier that waits for this wavefront's own use of the LDS, but not for what it has requested (which
// __syncthreads() would, had any of it the LDS for its destination)
__device__ __forceinline__ void barrier_lds()
{
    pin_order();
    __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    pin_order();
}

// Invalidates this compute unit's vector L1 (workgroup-scope buffer_inv): loads that follow
// are served by the L2.
__device__ __forceinline__ void invalidate_l1() { asm volatile("buffer_inv sc0" ::: "memory"); }

// The workgroups that exchange something count themselves in on a line: arrivals in the low
// half of a word, the sum of the arrivals' XCD numbers in the high half.  Which XCD a
// dispatch begins with depends on the hardware queue (it goes round from there: workgroup i
// runs on XCD (i + offset) % 8) and may change from one launch of a call to the next, so nothing
// is assumed about it; what the exchange relies on is that the workgroups of one item share an XCD
// within a launch, and each of them sees that from the sum.  A line is used once per layer: two of
// its words take turns, and one workgroup of the launch that uses the one clears the other, which
// no launch but the next looks at (the set-up clears both).
__host__ __device__ constexpr uint32_t arrival_of(uint32_t xcd) { return 1u + (xcd << 16); }
__host__ __device__ constexpr bool all_from(uint32_t word, uint32_t xcd, uint32_t n) { return (word >> 16) == xcd * n; }
template <class Line>
__host__ __device__ __forceinline__ Line epoch_word(Line line, uint32_t epoch) { return line + (epoch & 1); }
static_assert(kRangeWgs / 8 * 7 < 0x10000, "at most an XCD's workgroups are summed up");

__device__ __forceinline__ uint32_t my_xcd() { return __builtin_amdgcn_s_getreg(20 | (31 << 11)) & 15u; }   // HW_REG_XCC_ID
__device__ __forceinline__ uint32_t arrive(uint32_t* p)      // returns the word with this arrival in it
{
    const uint32_t mine = arrival_of(my_xcd());
    return atomicAdd(p, mine) + mine;
}
// by one workgroup of the line's item, in the launch of `epoch`
__device__ __forceinline__ void clear_next(uint32_t* line, uint32_t epoch)
{
    __hip_atomic_store(epoch_word(line, epoch + 1), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Did all n arrivals summed up in `word` come from this workgroup's XCD?  If not, status 3.
__device__ __forceinline__ bool same_xcd(uint32_t* sync, uint32_t word, uint32_t n)
{
    if (all_from(word, my_xcd(), n)) return true;
    atomicCAS(sync + kSyncStatus, 0u, 3u);
    return false;
}

// Waits until the low half of p has come to `target`, then looks at the XCDs of the n arrivals
// summed up in the high half.  Gives up (and raises the status word to `code`) after kWaitTicks of
// wall-clock time, or within 64 looks of another workgroup's giving up, so that a launch that is not fully
// resident ends with an error instead of hanging.  One thread calls.  Returns false if what was
// waited for is not there, or not visible here.  `v` is what was seen of p already: who arrives last knows it from its
// own arrival, and everybody waits for that one (0.1 us of an attention call).
__device__ __forceinline__ bool bounded_wait(uint32_t* sync, uint32_t* p, uint32_t v, uint32_t target, uint32_t n,
                                             uint32_t code)
{
    if ((v & 0xffffu) < target) {
        // (whether another workgroup has given up is looked at now and then only: a second load in every turn, and
        // eight times the sleep, made the turns three times as long, and what is waited for is seen that much later)
        const long long t0 = wall_clock64();
        for (int turn = 1; ((v = ld_relaxed(p)) & 0xffffu) < target; ++turn) {
            if (wall_clock64() - t0 > kWaitTicks || (turn % 64 == 0 && ld_relaxed(sync + kSyncStatus) != 0)) {
                atomicCAS(sync + kSyncStatus, 0u, code);
                return false;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return same_xcd(sync, v, n);
}

// The status word is cleared for the calls that follow; what it held is kept in the sticky
// word (first failure wins), so that a caller who reads the status only now and then still
// learns of a call that gave up.  A workspace seen for the first time (no magic word) holds
// nothing meaningful.  One thread of a call's first launch.
__device__ __forceinline__ void carry_status(uint32_t* sync)
{
    const uint32_t st = sync[kSyncStatus], sticky = sync[kSyncSticky];
    const bool known = sync[kSyncMagic] == kSyncMagicValue;
    sync[kSyncSticky] = known ? (sticky ? sticky : st) : 0u;
    sync[kSyncMagic] = kSyncMagicValue;
    sync[kSyncStatus] = 0;
}

// Zeroes the sync block with BLOCKS workgroups of 256 threads, of which this is number `block`.
// (The sizes are constants: reading them from the dispatch packet delays the first store.)
template <int BLOCKS>
__device__ __forceinline__ void zero_sync(uint32_t* sync, int block)
{
    static_assert(kSyncMagic == 3 && kSyncWords % 4 == 0, "the status words are the first 16 bytes");
    typedef uint32_t word4 __attribute__((ext_vector_type(4)));
    constexpr int n = kSyncWords / 4;
#pragma unroll
    for (int i0 = 0; i0 < n; i0 += BLOCKS * 256) {
        const int i = i0 + block * 256 + (int)threadIdx.x;
        if (i > 0 && i < n) ((word4*)sync)[i] = (word4){0u, 0u, 0u, 0u};
    }
    if (block == 0 && threadIdx.x == 0) carry_status(sync);
}

}  // namespace ghd
