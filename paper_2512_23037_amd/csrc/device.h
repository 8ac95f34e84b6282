// device.h -- device code shared by the sampler and the sign pass.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sampler.h"

namespace soft {

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).  MAD: each product from
// one v_mad_u64_u32 instead of a low and a high multiply.  Where Philox is the
// work it wins (the sign pass with a word per slot, 5 10^5 shots of the 42-qubit
// circuit: 1.39 -> 1.17 ms); the sampler is slower with it, for its registers.
template <bool MAD = false>
__device__ __forceinline__ void philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                         uint32_t k1, uint32_t &o0, uint32_t &o1, uint32_t &o2, uint32_t &o3) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t p0, p1;
        if (MAD) {
            asm("v_mad_u64_u32 %0, vcc, %1, %2, 0" : "=v"(p0) : "v"(c0), "s"(0xD2511F53u) : "vcc");
            asm("v_mad_u64_u32 %0, vcc, %1, %2, 0" : "=v"(p1) : "v"(c2), "s"(0xCD9E8D57u) : "vcc");
        } else {
            p0 = ((uint64_t)__umulhi(0xD2511F53u, c0) << 32) | (0xD2511F53u * c0);
            p1 = ((uint64_t)__umulhi(0xCD9E8D57u, c2) << 32) | (0xCD9E8D57u * c2);
        }
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32), lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    o0 = c0; o1 = c1; o2 = c2; o3 = c3;
}

// floor(x / d) for x < 16 d (a noise hit's Pauli code from its word): a
// binary search on exact integer compares instead of a 64-bit division.
__device__ __forceinline__ uint32_t quot16(uint64_t x, uint64_t d) {
    uint32_t m = 0;
#pragma unroll
    for (uint32_t b = 8; b != 0u; b >>= 1)
        if (x >= (uint64_t)(m + b) * d) m += b;
    return m;
}

// A launch's items [0, n) dealt out to its waves.  Wave w starts with item w,
// without a cursor, so a launch of at most one item a wave has no atomics;
// the rest come from eight cursors, wave w's being w mod 8 (of one-wave blocks,
// consecutive ones go to the eight XCDs in turn).  Atomics on one address
// follow each other every 16 ns: with one cursor for all, 25 000 items of four
// shots took 0.43 ms where the work in them took 0.14, and the 5120 waves of a
// small launch of the sampler spent 80 us finding that nothing was left.
// The next item of the wave (all lanes active); false when there is none.
// `started` is its state, false at first.
__device__ __forceinline__ bool take_item(unsigned long long *cursors, uint64_t n, uint32_t wave, uint32_t waves,
                                          uint32_t lane, bool &started, uint64_t &item) {
    if (!started) {
        started = true;
        item = wave;
        return item < n;
    }
    if (n <= waves) return false;
    const uint32_t id = wave % kQueueCursors;
    unsigned long long c = 0;
    if (lane == 0) c = atomicAdd(cursors + id * kCursorStride, 1ull);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)c);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(c >> 32));
    const uint32_t first = (waves - id + kQueueCursors - 1u) / kQueueCursors;  // items of this cursor that waves start with
    item = (first + (((uint64_t)hi << 32) | lo)) * kQueueCursors + id;
    return item < n;
}

}  // namespace soft
