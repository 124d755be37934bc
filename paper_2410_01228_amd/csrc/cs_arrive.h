// "Last one merges": the workgroups that share a cut decode sequence or a cut prefill tile each
// leave a partial, announce it, and whoever finds all of them announced merges them.  That saves a merge
// kernel's launch, and where other workgroups still compute the merge itself; where neither weighs
// enough (the rules are beside the launch planning) a kernel merges and nothing is announced.
//
// Partials cross from one XCD's L2 to another's, so they are written through (store at agent scope:
// sc1) and read past the reader's caches (load at agent scope), and a wavefront waits for its stores
// to be acknowledged before the workgroup announces itself: no cache is written back or invalidated
// as a whole (agent-scope fences instead took 20 times as long on a grid of small workgroups).
//
// An announcement is a 64-bit word per partial, in scratch memory that nobody clears beforehand; it
// holds the launch's number (next_launch_number: never used twice in a process, starting at an
// arbitrary point, so whatever the memory held before is no announcement).  A workgroup stores its word, waits
// for the acknowledgement, and reads all of them: the one whose store came last sees every word.
// Two that see every word both merge, in the same order, and write the same bits.  Whoever merges sets the words to
// zero again, so a launch replayed from a graph (with the same number) starts clean.  (Counting
// arrivals with compare-and-swap at one word made 16 pieces that end together wait for each other's
// retries: 34 -> 39 us on a launch of 30 us.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cs {

typedef uint32_t a_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t a_u32x2 __attribute__((ext_vector_type(2)));

// A float from its bits.  (__builtin_bit_cast straight from a vector's element reads element 0.)
__device__ __forceinline__ float as_float(uint32_t bits) { return __builtin_bit_cast(float, bits); }

// Stores at agent scope, inline assembly: neither buffer stores through a Shared nor a bit cast of the
// value leave the register allocation of the tile loop in front of them as it is (two more hazard
// waits an iteration, 1% of the kernel).  Nothing but wait_stores() waits for them.
typedef float a_f32x4 __attribute__((ext_vector_type(4)));
typedef float a_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_shared4(float* p, a_f32x4 v) { asm volatile("global_store_dwordx4 %0, %1, off sc1" :: "v"(p), "v"(v) : "memory"); }
__device__ __forceinline__ void store_shared2(float* p, a_f32x2 v) { asm volatile("global_store_dwordx2 %0, %1, off sc1" :: "v"(p), "v"(v) : "memory"); }
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A window of memory for loads and stores at agent scope (cache policy 16: sc1); bytes: its extent
// from `base` on, beyond which loads return zero and stores are dropped.
struct Shared {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Shared(void* base, uint32_t bytes) : r(__builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000)) {}
    typedef uint32_t b2 __attribute__((vector_size(8)));           // the builtin's own vector type
    __device__ __forceinline__ a_u32x4 load4(uint32_t off) const { return __builtin_bit_cast(a_u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 16)); }
    __device__ __forceinline__ a_u32x2 load2(uint32_t off) const { return __builtin_bit_cast(a_u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 16)); }
    __device__ __forceinline__ void store2(a_u32x2 v, uint32_t off) const { __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(b2, v), r, off, 0, 16); }
};

// The words of the partials of one cut sequence or tile: `stride` bytes apart from byte `off` of `mem`
// on.  All of it is done by the 64 lanes of one wavefront.
struct Announcements {
    Shared mem;
    uint32_t off, stride, n;
    a_u32x2 word;
    __device__ __forceinline__ Announcements(const Shared& mem_, uint32_t off_, uint32_t stride_, uint32_t n_, uint64_t launch)
        : mem(mem_), off(off_), stride(stride_), n(n_), word{(uint32_t)launch, (uint32_t)(launch >> 32)} {}
    // Announces partial `me`; to be followed by wait_stores().  (Every wavefront of the workgroup
    // has waited for its partial's stores and passed a barrier before.)
    __device__ __forceinline__ void announce(uint32_t me) const {
        if ((threadIdx.x & 63) == 0) mem.store2(word, off + me * stride);
    }
    // Whether all partials are announced, `me` (if below n) taken for granted.
    __device__ __forceinline__ bool all_but(uint32_t me) const {
        bool all = true;
        for (uint32_t i0 = 0; i0 < n; i0 += 64) {
            const uint32_t i = min(i0 + (threadIdx.x & 63), n - 1);
            const a_u32x2 w = mem.load2(off + i * stride);
            all = all && ((w[0] == word[0] && w[1] == word[1]) || i == me);
        }
        return __all(all);
    }
    __device__ __forceinline__ bool all() const { return all_but(~0u); }
    __device__ __forceinline__ void clear() const {
        for (uint32_t i = threadIdx.x & 63; i < n; i += 64) mem.store2(a_u32x2{0u, 0u}, off + i * stride);
    }
};

}  // namespace cs
