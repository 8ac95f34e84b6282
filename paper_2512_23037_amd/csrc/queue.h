// queue.h -- how a launch's items are dealt out to its waves (host and device).
#pragma once
#include <stdint.h>

namespace soft {

// Wave w starts with item w, without a cursor, so a launch of at most one item
// a wave has no atomics; the rest come from eight cursors, wave w's being
// w mod 8 (of one-wave blocks, consecutive ones go to the eight XCDs in turn).
// Atomics on one address follow each other every 16 ns: with one cursor for
// all, 25 000 items of four shots took 0.43 ms where the work in them took
// 0.14, and the 5120 waves of a small launch of the sampler spent 80 us finding
// that nothing was left.  Below eight waves some cursors would have no wave to
// draw from them: such a launch has one cursor.
constexpr uint32_t kQueueCursors = 8, kCursorStride = 16, kQueueWords = kQueueCursors * kCursorStride;

constexpr uint32_t queue_shift(uint32_t waves) { return waves >= kQueueCursors ? 3u : 0u; }
static_assert(kQueueCursors == 8u, "queue_shift");

// The cursor that wave `wave` draws from.
constexpr uint32_t queue_cursor(uint32_t wave, uint32_t waves) { return wave & ((1u << queue_shift(waves)) - 1u); }

// The item of draw `c` (from 0) on cursor `id`: past the items of the cursor
// that waves start with.
constexpr uint64_t queue_item(uint32_t id, uint64_t c, uint32_t waves) {
    const uint32_t s = queue_shift(waves);
    return ((((uint64_t)waves - id + (1u << s) - 1u) >> s) + c) << s | id;
}

}  // namespace soft
