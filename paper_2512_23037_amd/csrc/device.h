// device.h -- device code shared by the sampler and the sign pass.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sampler.h"

namespace soft {

// a ^ b ^ c in one instruction
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return (uint32_t)__builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The 64-bit product m x as (low, high) words.  MAD: from one v_mad_u64_u32
// instead of a low and a high multiply.  Where Philox is the work it wins (the
// sign pass with a word per slot, 5 10^5 shots of the 42-qubit circuit:
// 1.39 -> 1.17 ms); the sampler is slower with it, for its registers.  A block
// takes 222 cycles of a SIMD with it, 248 with two multiplies, 395 with three
// FP64 multiply-adds a product (exact when they round towards zero).
template <bool MAD> __device__ __forceinline__ void mul64(uint32_t m, uint32_t x, uint32_t &lo, uint32_t &hi) {
    if (MAD) {
        uint64_t p;
        asm("v_mad_u64_u32 %0, vcc, %1, %2, 0" : "=v"(p) : "v"(x), "s"(m) : "vcc");
        lo = (uint32_t)p;
        hi = (uint32_t)(p >> 32);
    } else {
        lo = m * x;
        hi = __umulhi(m, x);
    }
}

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u, kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

// Rounds FIRST .. 9 of Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) on
// the counter words c0..c3, in place.
template <bool MAD, int FIRST>
__device__ __forceinline__ void philox_rounds(uint32_t &c0, uint32_t &c1, uint32_t &c2, uint32_t &c3, uint32_t k0, uint32_t k1) {
    k0 += FIRST * kPhiloxW0;
    k1 += FIRST * kPhiloxW1;
#pragma unroll
    for (int r = FIRST; r < 10; ++r) {
        uint32_t lo0, hi0, lo1, hi1;
        mul64<MAD>(kPhiloxM0, c0, lo0, hi0);
        mul64<MAD>(kPhiloxM1, c2, lo1, hi1);
        c0 = xor3(hi1, c1, k0);
        c1 = lo1;
        c2 = xor3(hi0, c3, k1);
        c3 = lo0;
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
    }
}

template <bool MAD = false>
__device__ __forceinline__ void philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                         uint32_t k1, uint32_t &o0, uint32_t &o1, uint32_t &o2, uint32_t &o3) {
    philox_rounds<MAD, 0>(c0, c1, c2, c3, k0, k1);
    o0 = c0; o1 = c1; o2 = c2; o3 = c3;
}

// Philox blocks of one shot whose counters differ in the first word alone: the
// other words' part of the first two rounds, two of the twenty products.
struct PhiloxShot {
    uint32_t lo1, hi0, lo0;
    __device__ __forceinline__ void start(uint32_t c1, uint32_t c2, uint32_t k0) {
        uint32_t hi1;
        mul64<true>(kPhiloxM1, c2, lo1, hi1);
        mul64<true>(kPhiloxM0, xor3(hi1, c1, k0), lo0, hi0);
    }
    __device__ __forceinline__ void block(uint32_t c0, uint32_t c3, uint32_t k0, uint32_t k1, uint32_t &o0, uint32_t &o1,
                                          uint32_t &o2, uint32_t &o3) const {
        uint32_t l, h, l1, h1;
        mul64<true>(kPhiloxM0, c0, l, h);                     // round 0
        mul64<true>(kPhiloxM1, xor3(h, c3, k1), l1, h1);      // round 1
        o0 = xor3(h1, lo1, k0 + kPhiloxW0);
        o1 = l1;
        o2 = xor3(hi0, l, k1 + kPhiloxW1);
        o3 = lo0;
        philox_rounds<true, 2>(o0, o1, o2, o3, k0, k1);
    }
};

// floor(x / d) for x < 16 d (a noise hit's Pauli code from its word): a
// binary search on exact integer compares instead of a 64-bit division.
__device__ __forceinline__ uint32_t quot16(uint64_t x, uint64_t d) {
    uint32_t m = 0;
#pragma unroll
    for (uint32_t b = 8; b != 0u; b >>= 1)
        if (x >= (uint64_t)(m + b) * d) m += b;
    return m;
}

// The next of a launch's items [0, n) for this wave (queue.h, 2^shift() cursors,
// asked for where one is drawn from; all lanes active); false when there is
// none.  `started` is its state, false at first.
template <typename S>
__device__ __forceinline__ bool take_item(unsigned long long *cursors, uint64_t n, uint32_t wave, uint32_t waves,
                                          S shift, uint32_t lane, bool &started, uint64_t &item) {
    if (!started) {
        started = true;
        item = wave;
        return item < n;
    }
    if (n <= waves) return false;
    const uint32_t s = shift(), id = queue_cursor(wave, s);
    unsigned long long c = 0;
    if (lane == 0) c = atomicAdd(cursors + id * kCursorStride, 1ull);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)c);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(c >> 32));
    item = queue_item(id, ((uint64_t)hi << 32) | lo, waves, s);
    return item < n;
}

}  // namespace soft
