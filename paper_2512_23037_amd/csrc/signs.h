// signs.h -- the sign program of an event list (see program.h).
#pragma once
#include <stdint.h>

#include <vector>

#include "compile.h"
#include "program.h"

namespace soft {

// Words of a vector: tests, then record words, then one word of observables.
struct SignLayout {
    uint32_t tests = 0, recs = 0;
    uint32_t out() const { return recs + 1u; }
};

struct SignProgram {
    bool on = false;
    SignLayout need;                          // what this list fills
    std::vector<SignTest> tests;              // one row more than tests: the end
    std::vector<std::vector<uint32_t>> mask;  // per row: record words and observables written by then
    std::vector<SignSlot> slots;
    std::vector<uint32_t> vecs;               // kSignVecs vectors per slot, each as long as `ref`
    std::vector<uint32_t> ref;                // noiseless values
    std::vector<uint32_t> coin_slot;          // measurement slots of the coins
    std::vector<std::vector<uint32_t>> coin;  // what a coin's 1 flips
    std::vector<SignPair> pairs;              // `vec` indexes pair_vecs
    std::vector<std::vector<uint32_t>> pair_vecs;
    std::vector<SignMeas> meas;
    bool complete = false;                    // the signs decide the whole list
    double ends = 0.0;                        // about the fraction of shots that a check ends by signs
    double breaks = 0.0;                      // about the T pairs that noise breaks per shot
};

// Signature vectors take at most this much: of a list here, of all lists of a
// context in its launch's layout (16 words a vector: 350 000 noise slots; the
// 42-qubit circuit has 2800).
constexpr uint64_t kMaxSignBytes = 128ull << 20;

// Build the sign program of the list P.  `on` stays false when the list has
// more tests, records, coins or noise slots than the tables hold, or a T pair
// whose two gates are not the same Pauli in the frame.  Throws std::bad_alloc.
void build_signs(const Program &P, SignProgram &out);

}  // namespace soft
