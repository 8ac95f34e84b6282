// queue.h -- how a launch's items are dealt out to its waves (host and device).
#pragma once
#include <stdint.h>

namespace soft {

// Wave w starts with item w, without a cursor, so a launch of at most one item
// a wave has no atomics; the rest come from one cursor or from eight, wave w's
// being w mod 8 (of one-wave blocks, consecutive ones go to the eight XCDs in
// turn).  Atomics on one address follow each other every 16 ns: with one cursor
// for all, 25 000 items of four shots took 0.43 ms where the work in them took
// 0.14, and the 5120 waves of a small launch of the sampler spent 80 us finding
// that nothing was left.  But a cursor's waves sit on two XCDs, and those whose
// cursor is dry do not help the others, so items that take long come from one.
// Below eight waves some of eight cursors would have no wave to draw from them.
constexpr uint32_t kQueueCursors = 8, kCursorStride = 16, kQueueWords = kQueueCursors * kCursorStride;

// log2 of a launch's cursors, where it may have eight.
constexpr uint32_t kQueueShift = 3;
static_assert(kQueueCursors == 1u << kQueueShift, "cursors");
constexpr uint32_t queue_shift(uint32_t waves) { return waves >= kQueueCursors ? kQueueShift : 0u; }

// The cursor that wave `wave` draws from, of 2^shift.
constexpr uint32_t queue_cursor(uint32_t wave, uint32_t shift) { return wave & ((1u << shift) - 1u); }

// The item of draw `c` (from 0) on cursor `id`: past the items of the cursor
// that waves start with.
constexpr uint64_t queue_item(uint32_t id, uint64_t c, uint32_t waves, uint32_t shift) {
    return ((((uint64_t)waves - id + (1u << shift) - 1u) >> shift) + c) << shift | id;
}

}  // namespace soft
