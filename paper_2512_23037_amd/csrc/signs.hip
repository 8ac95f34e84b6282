// signs.hip -- the sign pass: shots decided without their coefficients.
//
// One lane runs one shot on its variant's sign program (program.h): it draws
// the shot's noise hits in slot order, XORs each hit's signature into a vector
// of tests, record words and observables, and stops once no later slot can
// move the first set test.  What the coefficients decide (SGT_HAND) is left to
// the sampler kernel, which runs after this one on the pending shots.
//
// With gap sampling a shot is a few Philox blocks, table reads and XORs.  What
// bounds it is VALU issue with about half the lanes at work (a wave fills its
// lanes when half of them have ended: 50 of 64 busy in a step, fewer in the
// shots' ends and starts) and the reads' latency between: a step waits for its
// gaps, its slots and their signatures.  A launch of 10^7 shots of the 42-qubit
// circuit at p = 1e-3 takes 0.47 ms, 21 G shots/s (47.3 ms with the sampler
// kernel alone).  With a word per slot it is bound by the Philox blocks, 222
// cycles each of about 350 a step takes: 5 10^5 shots at p = 5e-4 (1.4 G words)
// take 0.91 ms (3.0 with the sampler kernel alone).
#include <hip/hip_runtime.h>

#include "device.h"
#include "program.h"
#include "sampler.h"

namespace soft {
namespace {

__device__ __forceinline__ uint32_t first32(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

// floor(mul w / (d1 + 1)) for mul = 3 or 15 and w <= d1: a hit's Pauli code.
// The quotient in single precision is off by less than 2^-17; 2^-10 below it,
// its floor is the result or one less, which an exact product tells.
__device__ __forceinline__ uint32_t part(uint32_t mul, uint32_t w, uint32_t d1) {
    const float f = (float)w * (float)mul * __builtin_amdgcn_rcpf((float)d1 + 1.0f);
    const uint32_t q = (uint32_t)fmaxf(f - 0.0009765625f, 0.0f) + 1u;
    return (uint64_t)q * d1 + q <= (uint64_t)mul * w ? q : q - 1u;
}

// Lanes that run one shot together.  With gap sampling a shot draws a few
// words: one lane each, 64 shots in flight.  With a word per slot a shot draws
// thousands: 16 lanes take 64 consecutive slots a step, so that a shot's chain
// of steps is short (one lane per shot left a launch of 500 000 shots waiting
// for single shots of 1329 steps) and a wave still holds four shots.
template <bool GAPS> constexpr uint32_t kLanes = GAPS ? 1u : 16u;

// Waves a SIMD holds by vector size, which the registers are set to.
constexpr int kSignWaves(int tests) { return tests <= 4 ? 5 : tests <= 8 ? 4 : 3; }

constexpr uint32_t kLeft = 0xFFFFFFFFu;

// Idle lanes take new shots once this many wait: a start costs about as much
// as a step of one-lane shots, whether one lane or all take it.  With a word
// per slot a step costs less than a start and a shot of n slots takes n / 64 of
// them: long shots fill one group at a time, short ones three.  us by ones, twos
// and threes: 524 slots 609, 510, 490; 861 298, 267, 264; 1125 422, 398, 401;
// 1970 599, 574, 619; 2397 542, 537, 591; 5314 883, 917, 1051.
template <bool GAPS> __device__ __forceinline__ uint32_t refill_at(uint32_t n_noise) {
    return GAPS ? 32u : n_noise >= 1536u ? 16u : 48u;
}

// One-lane shots stopped at a broken pair wait until this many do: settling
// takes longer than a step, however few lanes take part (4 10^6 shots of 42
// qubits at p = 1e-3: 237 us at once, 219 at 8, 218 at 12, 220 at 16, 225 at 32;
// 15 qubits 219, 202, 201, 199, 201).
constexpr uint32_t kSettle = 12;

// The launch's arguments, read again where they are used: everything outside
// the step is rare, and kept in scalar registers across it its pointers
// spilled (60 of them; the reloads hit the scalar cache).
typedef const __attribute__((address_space(4))) SignParams ConstParams;
typedef const __attribute__((address_space(4))) SignDesc ConstDesc;
typedef const __attribute__((address_space(4))) VariantDesc ConstVariant;
__device__ __forceinline__ ConstParams *args() {
    ConstParams *p = (ConstParams *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

template <int TW, int RO, bool GAPS>
__global__ void __launch_bounds__(kSignBlock) __attribute__((amdgpu_waves_per_eu(kSignWaves(TW), 8))) k_signs(SignParams P0) {
    constexpr int W = TW + RO, Q = W / 4;
    constexpr uint32_t GL = kLanes<GAPS>;
    static_assert(W % 4 == 0, "vectors are read four words at a time");
    __shared__ uint32_t hist[kMaxCheckpoints + 1];
    __shared__ uint32_t stops[32 * TW + 1];  // SignTest::stop of the variant's rows
    __shared__ uint64_t pair_rows[TW / 2 + 1];  // and which of them are SGT_PAIR
    const uint32_t lane = threadIdx.x, sub = lane % GL;
    const uint32_t key0 = (uint32_t)P0.seed, key1 = (uint32_t)(P0.seed >> 32);
    if (lane <= kMaxCheckpoints) hist[lane] = 0u;

    // The variant of the shots in flight: what the step reads of it, and the
    // shots' counts.
    uint32_t var = 0xFFFFFFFFu, n_noise = 0, n_tests = 0;
    float l2q = 0.0f;
    uint32_t refill = 1;
    const uint32_t *draws = nullptr;   // its gap table, or its thresholds
    const SignSlot *slots = nullptr;
    const uint4 *vecs = nullptr;       // its first slot's signatures
    uint32_t zero_vec = 0;             // the zero vector, from there
    uint32_t n_pass = 0, n_disc = 0, n_logical = 0, n_prefix = 0, n_broke = 0;
    uint64_t words = 0;  // of this lane
    auto desc = [&]() { return (ConstDesc *)args()->desc + var; };
    auto flush = [&]() {
        unsigned long long *row = args()->counters + ((size_t)var * args()->shards + (blockIdx.x & (args()->shards - 1u))) * C_COUNT;
        for (int o = 32; o >= 1; o >>= 1) words += __shfl_xor((unsigned long long)words, o, 64);
        const uint64_t v = lane == C_SHOTS ? n_pass + n_disc : lane == C_PASSED ? n_pass : lane == C_DISCARDED ? n_disc
                         : lane == C_LOGICAL ? n_logical : lane == C_NOISE ? words : lane == C_PREFIX ? n_prefix
                         : lane == C_RESTARTS ? n_broke : 0ull;
        if (v) atomicAdd(row + lane, (unsigned long long)v);
        if (lane <= kMaxCheckpoints) {
            if (hist[lane]) atomicAdd(row + C_CK0 + lane, (unsigned long long)hist[lane]);
            hist[lane] = 0u;
        }
        n_pass = n_disc = n_logical = n_prefix = n_broke = 0;
        words = 0;
    };

    // Run positions [cur, cur + rest) of this wave's chunk are still to start.
    uint64_t cur = 0;
    uint32_t rest = 0;
    bool started = false, dry = false;

    // ---- the lane's shot ----
    bool act = false;    // it has one
    bool stop = false;   // no slot below `limit` is undecided: to be settled
    uint64_t i = 0;
    uint32_t s_lo = 0, s_hi = 0;
    PhiloxShot stream0 = {0, 0, 0};  // a word per slot: the shot's noise words
    uint32_t x[W];
    uint32_t pos = 0;    // next word (GAPS) or noise slot (of the lane's group)
    uint32_t drawn = 0;  // GAPS: slots decided
    uint32_t next_s = 0, next_w = 0;  // GAPS: the candidate that stopped at `limit`, and its acceptance word
    bool held = false;                // GAPS: that candidate is still to be taken
    uint32_t row = 0;    // first set test, or n_tests
    uint32_t limit = 0;  // noise slots that can still move it
    uint32_t ck = 0;     // checkpoints before the first hit
    // Broken pairs not yet told apart: pair t's index in byte t of `pids`
    // (npend bytes used), and in nibble j of `gens` the pairs whose betas add
    // up to the j-th remaining index shift (0: none); the next measurement
    // that reads one of them (SignMeas `mrow`), its first test and its stop.
    uint32_t pids = 0, npend = 0, gens = 0, mrow = 0, mtest = 0, mstop = 0;
    bool broke = false;  // a pair of this shot was broken
#pragma unroll
    for (int w = 0; w < W; ++w) x[w] = 0u;
    auto add_to = [&](uint32_t (&v)[W], const uint4 *p) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint4 u = p[q];
            v[4 * q] ^= u.x;
            v[4 * q + 1] ^= u.y;
            v[4 * q + 2] ^= u.z;
            v[4 * q + 3] ^= u.w;
        }
    };
    auto find_first = [&]() {
        uint32_t t = n_tests;
#pragma unroll
        for (int w = TW - 1; w >= 0; --w)
            if (x[w]) t = 32u * w + (uint32_t)__builtin_ctz(x[w]);
        row = t;
        limit = stops[t];
        if (gens != 0u && t >= mtest) limit = mstop;
    };
    // The vectors whose sum is the signature of a hit at slot s, its Pauli from
    // the word w <= d1 (NZ_NONE: the zero vector twice).
    auto codes = [&](uint32_t s, uint32_t kind, uint32_t w, uint32_t d1, uint32_t &u, uint32_t &v) {
        const uint32_t code = part(kind == NZ_DEP2 ? 15u : 3u, w, d1) + 1u;
        const uint32_t a = kind == NZ_DEP2 ? code >> 2 : kind == NZ_DEP1 ? code : kind == NZ_ZERR ? 3u : kind == NZ_NONE ? 0u : 1u;
        const uint32_t b = kind == NZ_DEP2 ? code & 3u : 0u;
        const uint32_t v0 = kSignVecs * s - 1u;
        u = a ? v0 + a : zero_vec;
        v = b ? v0 + 3u + b : zero_vec;
    };
    auto sum_of = [&](uint32_t (&d)[W], uint32_t u, uint32_t v) {
        const uint4 *pa = vecs + (int64_t)(int32_t)u * Q, *pb = vecs + (int64_t)(int32_t)v * Q;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint4 ua = pa[q], ub = pb[q];
            d[4 * q] = ua.x ^ ub.x;
            d[4 * q + 1] = ua.y ^ ub.y;
            d[4 * q + 2] = ua.z ^ ub.z;
            d[4 * q + 3] = ua.w ^ ub.w;
        }
    };
    // GAPS: the gaps of two words: a gap is its table's #{j < lim : w < tb[j]}
    // (or more, past lim).  An estimate from the word's logarithm puts four
    // entries around it, which decide it unless they do not bracket it (then a
    // binary search).
    auto gaps_of = [&](uint32_t wa, uint32_t wb, uint32_t lim, uint32_t &ga, uint32_t &gb) {
        const uint32_t ws[2] = {wa, wb};
        uint32_t b[2], t[2][4], g[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float est = fminf(fmaxf((__log2f((float)ws[k] + 0.5f) - 32.0f) * l2q, 0.0f), (float)lim);
            b[k] = max((uint32_t)est, 2u) - 2u;
            __builtin_memcpy(t[k], draws + b[k], 16);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            uint32_t n = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) n += ws[k] < t[k][j] ? 1u : 0u;
            g[k] = b[k] + n;
            if ((n == 4u && b[k] + 4u < lim) || (n == 0u && b[k] != 0u)) {
                uint32_t lo = 0, hi = lim;  // ws[k] < draws[j] for j < lo, not for j >= hi (or past the slots)
                while (lo < hi) {
                    const uint32_t h = (lo + hi) >> 1;
                    if (ws[k] < draws[h]) lo = h + 1u;
                    else hi = h;
                }
                g[k] = lo;
            }
        }
        ga = g[0];
        gb = g[1];
    };

    // the index shift of a set of pending pairs
    auto shift_of = [&](const SignPair *pairs, uint32_t set) {
        uint64_t b = 0;
        for (uint32_t t = 0; t < npend; ++t)
            if ((set >> t) & 1u) b ^= pairs[(pids >> (8u * t)) & 255u].beta;
        return b;
    };
    // the next measurement that reads a remaining shift is k
    auto set_meas = [&](ConstParams *A, ConstDesc *D, uint32_t k) {
        mrow = k;
        mtest = 0xFFFFFFFFu;
        if (k < D->n_meas) {
            const SignMeas M = A->meas[D->meas_off + k];
            mtest = M.test;
            mstop = M.stop;
        }
    };
    // What happens where no slot below `limit` is undecided.  False when the
    // shot ends there (row kLeft: the sampler kernel runs it).
    auto settle = [&]() -> bool {
        ConstParams *A = args();
        ConstDesc *D = desc();
        const SignPair *pairs = A->pairs + D->pair_off;
        if (gens != 0u && row >= mtest) {
            const SignMeas M = A->meas[D->meas_off + mrow];
            if (M.rec == kNone) {
                row = kLeft;
                return false;
            }
            uint32_t c0, c1, c2, c3;
            philox10<true>(M.slot >> 2, s_lo, s_hi, 1u, key0, key1, c0, c1, c2, c3);
            const uint32_t q = M.slot & 3u;
            const uint32_t bit = (q == 0u ? c0 : q == 1u ? c1 : q == 2u ? c2 : c3) >> 31;
            uint32_t o = 0;  // its outcome on the entry that x follows
#pragma unroll
            for (int w = 0; w < RO - 1; ++w)
                if ((M.rec >> 5) == (uint32_t)w) o = (x[TW + w] >> (M.rec & 31u)) & 1u;
            if (!GAPS && M.flip < pos) {  // its record flip comes after, but x has it if it hit
                philox10<true>(M.flip >> 2, s_lo, s_hi, 0u, key0, key1, c0, c1, c2, c3);
                const uint32_t f = M.flip & 3u;
                o ^= (f == 0u ? c0 : f == 1u ? c1 : f == 2u ? c2 : c3) <= draws[M.flip] && slots[M.flip].kind == NZ_FLIP ? 1u : 0u;
            }
            // one shift that it reads is decided, the others lose it
            uint32_t pivot = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t set = (gens >> (4 * j)) & 15u;
                if (!(__popcll(M.gamma & shift_of(pairs, set)) & 1)) continue;
                gens ^= (pivot ? pivot : set) << (4 * j);
                if (!pivot) pivot = set;
            }
            if (o != bit)
                for (uint32_t t = 0; t < npend; ++t)
                    if ((pivot >> t) & 1u) add_to(x, A->vecs + (size_t)pairs[(pids >> (8u * t)) & 255u].vec * Q);
            if (gens == 0u) {
                pids = npend = 0u;
            } else {  // (a remaining shift may now be a sum of pairs')
                uint64_t b[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) b[j] = shift_of(pairs, (gens >> (4 * j)) & 15u);
                const SignMeas *meas = A->meas + D->meas_off;
                const uint32_t n = D->n_meas;
                uint32_t k = mrow + 1u;
                for (; k < n; ++k) {
                    const uint64_t g = meas[k].gamma;
                    if (g == ~0ull || ((__popcll(g & b[0]) | __popcll(g & b[1]) | __popcll(g & b[2]) | __popcll(g & b[3])) & 1)) break;
                }
                set_meas(A, D, k);
            }
            find_first();
            return true;
        }
        const SignTest T = A->tests[D->test_off + row];
        if (T.kind != SGT_PAIR) return false;
        broke = true;
        const SignPair S = pairs[T.pair];
        bool left = npend == 4u;
        for (uint32_t set = 1; set < (1u << npend); ++set) {  // dependent on the remaining shifts?
            uint32_t sum = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((set >> j) & 1u) sum ^= (gens >> (4 * j)) & 15u;
            left = left || shift_of(pairs, sum) == S.beta;
        }
        if (left) {
            row = kLeft;
            return false;
        }
#pragma unroll
        for (int w = 0; w < TW; ++w)
            if ((row >> 5) == (uint32_t)w) x[w] &= x[w] - 1u;  // the lowest set test
        // (what was pending is not read before this pair's end: it would have
        // been settled first)
        set_meas(A, D, gens ? min(mrow, S.meas) : S.meas);
        pids |= T.pair << (8u * npend);
        gens |= 1u << (5u * npend);  // nibble npend, pair npend
        ++npend;
        find_first();
        return true;
    };

    for (;;) {
        // ---- stopped shots are settled and end, idle lanes take new ones ----
        const uint64_t busy = __ballot(act && !stop);
        const uint32_t waiting = 64u - (uint32_t)__builtin_popcountll(dry ? busy | __ballot(!stop) : busy);
        if (waiting >= refill || busy == 0ull) {
            const bool open = stop && (!GAPS || (gens != 0u && row >= mtest) || ((pair_rows[row >> 6] >> (row & 63u)) & 1u));
            const bool do_settle = !GAPS || (uint32_t)__builtin_popcountll(__ballot(open)) >= kSettle || busy == 0ull;
            bool fin = stop && !open;
            if (open && do_settle) {
                bool on = settle();
                while (on && (GAPS ? next_s : pos) >= limit) on = settle();
                fin = !on;
                stop = false;
                held = on;
            }
            if (fin) stop = false;
            bool pass = false, disc = false, logical = false;
            if (fin) {
                ConstParams *A = args();
                ConstDesc *D = desc();
                act = false;
                const uint32_t r = D->test_off + (row == kLeft ? 0u : row);
                const SignTest T = A->tests[r];
                if (sub != 0u) {
                    // the group's first lane writes
                } else if (row == kLeft || T.kind == SGT_HAND) {
                    A->status[i] = kStatusPending;
                } else {
                    const uint32_t *mk = A->mask + (size_t)r * RO;
                    const uint32_t obs = x[W - 1] & mk[RO - 1];
                    pass = T.kind == SGT_NONE;
                    disc = !pass;
                    logical = pass && obs != 0u;
                    A->status[i] = pass ? (uint32_t)ST_PASSED : (uint32_t)ST_DISCARDED;
                    if (A->abort_op) A->abort_op[i] = T.src;
                    if (A->obs) A->obs[i] = obs;
                    if (A->outcomes) {
#pragma unroll
                        for (int w = 0; w < RO - 1; ++w)
                            if ((uint32_t)w < A->rec_words) A->outcomes[(uint64_t)w * A->n_shots + i] = x[TW + w] & mk[w];
                        // (a variant that this pass leaves to the sampler may have more words)
                        for (uint32_t w = RO - 1; w < A->rec_words; ++w) A->outcomes[(uint64_t)w * A->n_shots + i] = 0u;
                    }
                    words += GAPS ? pos : min(pos, n_noise);
                    atomicAdd(&hist[ck], 1u);
                }
            }
            n_pass += (uint32_t)__builtin_popcountll(__ballot(pass));
            n_disc += (uint32_t)__builtin_popcountll(__ballot(disc));
            n_logical += (uint32_t)__builtin_popcountll(__ballot(logical));
            n_broke += (uint32_t)__builtin_popcountll(__ballot((pass || disc) && broke));
            n_prefix += (uint32_t)__builtin_popcountll(__ballot((pass || disc) && ck != 0u && args()->prefix != 0u));

            const uint64_t idle = __ballot(!act);
            if (rest == 0u && !dry) {
                ConstParams *A = args();
                uint64_t got;
                // (more chunks than waves only where the grid fills the device: sign_params)
                dry = !take_item(A->next, (A->n_shots + A->chunk - 1u) / A->chunk, blockIdx.x, gridDim.x,
                                 []() { return kQueueShift; }, lane, started, got);
                if (!dry) {
                    cur = got * A->chunk;
                    rest = (uint32_t)min((uint64_t)A->chunk, A->n_shots - cur);
                }
            }
            if (dry && idle == ~0ull) break;
            if (rest != 0u && idle != 0ull) {
                ConstParams *A = args();
                const uint64_t shot = A->shot0 + cur;
                ConstVariant *V = (ConstVariant *)A->vars;
                bool ready = var != 0xFFFFFFFFu && shot < V[var].shot_end && (var == 0u || shot >= V[var - 1u].shot_end);
                if (!ready && idle == ~0ull) {  // another variant, once no lane runs the last one
                    if (var != 0xFFFFFFFFu) flush();
                    var = 0;
                    while (var + 1u < A->n_vars && V[var].shot_end <= shot) ++var;
                    var = first32(var);
                    ConstDesc *D = desc();
                    n_noise = V[var].n_noise;
                    n_tests = D->n_tests;
                    refill = refill_at<GAPS>(n_noise);
                    l2q = V[var].gap_l2q;
                    draws = GAPS ? A->gaps + V[var].gap_off : A->tm1 + V[var].tm1_off;
                    slots = A->slots + D->slot_off;
                    vecs = A->vecs + (size_t)D->vec_off * Q;
                    zero_vec = 0u - D->vec_off;
                    if (D->on)
                        for (uint32_t t0 = 0; t0 <= n_tests; t0 += 64u) {
                            const uint32_t t = min(t0 + lane, n_tests);
                            const SignTest T = A->tests[D->test_off + t];
                            stops[t] = T.stop;
                            const uint64_t m = __ballot(T.kind == SGT_PAIR);
                            if (lane == 0u) pair_rows[t0 >> 6] = m;
                        }
                    __syncthreads();  // (one wave: its LDS writes are done)
                    ready = true;
                }
                if (ready) {
                    ConstDesc *D = desc();
                    const uint64_t left = min((uint64_t)rest, V[var].shot_end - shot);
                    const uint32_t take = (uint32_t)min(left, (uint64_t)((uint32_t)__builtin_popcountll(idle) / GL));
                    const uint32_t rank = (uint32_t)__builtin_popcountll(idle & ((1ull << (lane - sub)) - 1ull)) / GL;
                    if (!act && rank < take) {
                        i = cur + rank;
                        if (!(D->on & (GAPS ? 1u : 2u))) {
                            if (sub == 0u) A->status[i] = kStatusPending;
                        } else {
                            act = true;
                            s_lo = (uint32_t)(A->shot0 + i);
                            s_hi = (uint32_t)((A->shot0 + i) >> 32);
                            if (!GAPS) stream0.start(s_lo, s_hi, key0);
#pragma unroll
                            for (int w = 0; w < W; ++w) x[w] = 0u;
                            add_to(x, A->vecs + (size_t)D->ref_vec * Q);
                            pos = drawn = 0u;
                            pids = npend = gens = 0u;
                            held = broke = false;
                            ck = D->ck_cnt;
                            uint32_t have = 0xFFFFFFFFu, c0 = 0, c1 = 0, c2 = 0, c3 = 0;
                            const uint32_t n_coins = D->n_coins;
                            for (uint32_t c = 0; c < n_coins; ++c) {
                                const uint2 cn = A->coins[D->coin_off + c];
                                if ((cn.x >> 2) != have) {
                                    have = cn.x >> 2;
                                    philox10<true>(have, s_lo, s_hi, 1u, key0, key1, c0, c1, c2, c3);
                                }
                                const uint32_t q = cn.x & 3u;
                                // outcome 1 iff (word + 1/2) 2^-32 >= 1/2
                                if ((q == 0u ? c0 : q == 1u ? c1 : q == 2u ? c2 : c3) >> 31)
                                    add_to(x, A->vecs + (size_t)cn.y * Q);
                            }
                            find_first();
                        }
                    }
                    cur += take;
                    rest -= take;
                }
            }
        }

        // ---- one step of every shot in flight: a Philox block a lane ----
        const bool run = act && !stop;
        uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;
        uint4 th;
        bool any = false;  // one of the lane's slots is hit
        if (run) {
            if (GAPS) philox10<true>(pos >> 2, s_lo, s_hi, 2u, key0, key1, w0, w1, w2, w3);
            else stream0.block((pos >> 2) + sub, 0u, key0, key1, w0, w1, w2, w3);
            if (GAPS) {
                // Two candidates a block (gap word, acceptance word); one that a
                // settled shot held back goes first.  Both are looked up before
                // the first is taken: the step waits for three reads in a row
                // (gap, slot, signatures), not six.
                const uint32_t lim = n_noise - drawn;
                uint32_t g1, g2;
                gaps_of(w0, w2, lim, g1, g2);
                const uint32_t s1 = held ? next_s : drawn + min(g1, lim), a1 = held ? next_w : w1;
                const bool two = !held || (pos & 2u);
                if (!held) pos += 2u;
                if (s1 >= limit) {
                    stop = true;
                    next_s = s1;
                    next_w = a1;
                } else {
                    held = false;
                    const uint32_t s2 = min(s1 + 1u + g2, n_noise), t2 = min(s2, n_noise - 1u);
                    const SignSlot sl1 = slots[s1], sl2 = slots[t2];
                    const bool hit1 = a1 <= sl1.acc1 && sl1.kind != NZ_NONE;
                    const bool hit2 = two && w3 <= sl2.acc1 && sl2.kind != NZ_NONE;
                    uint32_t u1, v1, u2, v2;
                    codes(s1, hit1 ? sl1.kind : (uint32_t)NZ_NONE, a1, sl1.acc1, u1, v1);
                    codes(t2, hit2 ? sl2.kind : (uint32_t)NZ_NONE, w3, sl2.acc1, u2, v2);
                    uint32_t d1[W], d2[W];
                    sum_of(d1, u1, v1);
                    sum_of(d2, u2, v2);
#pragma unroll
                    for (int w = 0; w < W; ++w) x[w] ^= d1[w];
                    if (hit1) ck = min(ck, sl1.ckpt);
                    drawn = s1 + 1u;
                    find_first();
                    if (two) {
                        pos += 2u;
                        if (s2 >= limit) {
                            stop = true;
                            next_s = s2;
                            next_w = w3;
                        } else {
#pragma unroll
                            for (int w = 0; w < W; ++w) x[w] ^= d2[w];
                            if (hit2) ck = min(ck, sl2.ckpt);
                            drawn = s2 + 1u;
                            find_first();
                        }
                    }
                }
            } else {
                // Signatures only reach forward, so hits past `limit` may be
                // taken too: they change nothing at or before test `row`.
                th = *reinterpret_cast<const uint4 *>(draws + pos + 4u * sub);
                any = (w0 <= th.x) | (w1 <= th.y) | (w2 <= th.z) | (w3 <= th.w);
            }
        }
        if (!GAPS) {
            if (__ballot(any) != 0ull) {
                // All lanes of a group take the group's hits, one after the
                // other (there is rarely a second): x needs no reduction.
                uint32_t m = any ? (w0 <= th.x ? 1u : 0u) | (w1 <= th.y ? 2u : 0u) | (w2 <= th.z ? 4u : 0u) | (w3 <= th.w ? 8u : 0u) : 0u;
                for (;;) {
                    const uint64_t hits = __ballot(m != 0u);
                    if (hits == 0ull) break;
                    const uint32_t group = (uint32_t)(hits >> (lane - sub)) & ((1u << GL) - 1u);
                    const uint32_t src = lane - sub + (uint32_t)__builtin_ctz(group | 0x10000u) % GL;
                    const uint32_t j = (uint32_t)__builtin_ctz(m | 8u);
                    const uint32_t s = (uint32_t)__shfl((int)(pos + 4u * sub + j), (int)src, 64);
                    const uint32_t w = (uint32_t)__shfl((int)(j == 0u ? w0 : j == 1u ? w1 : j == 2u ? w2 : w3), (int)src, 64);
                    if (lane == src) m &= m - 1u;
                    if (group != 0u && s < n_noise) {
                        const SignSlot sl = slots[s];
                        uint32_t u, v;
                        codes(s, sl.kind, w, sl.thr1, u, v);
                        add_to(x, vecs + (int64_t)(int32_t)u * Q);
                        add_to(x, vecs + (int64_t)(int32_t)v * Q);
                        if (sl.kind != NZ_NONE && s < limit) ck = min(ck, sl.ckpt);
                    }
                }
                if (run) find_first();
            }
            if (run) {
                pos += 4u * GL;
                stop = pos >= limit;
            }
        }
    }
    if (var != 0xFFFFFFFFu) flush();
}

template <int TW, int RO> const void *kernel_of(bool gaps) {
    return gaps ? (const void *)k_signs<TW, RO, true> : (const void *)k_signs<TW, RO, false>;
}
}  // namespace

const void *signs_kernel(uint32_t size, bool gaps) {
    switch (size) {
        case 0: return kernel_of<2, 2>(gaps);
        case 1: return kernel_of<4, 4>(gaps);
        case 2: return kernel_of<8, 8>(gaps);
        default: return kernel_of<16, 16>(gaps);
    }
}

hipError_t launch_signs(const SignParams &p, uint32_t size, bool gaps, dim3 grid, hipStream_t stream) {
    void *args[1] = {(void *)&p};
    return hipLaunchKernel(signs_kernel(size, gaps), grid, dim3(kSignBlock), args, 0, stream);
}

}  // namespace soft
