// soft_api.cpp -- the C ABI declared in include/soft.h.
//
// Host side of the sampler: owns the compiled circuit and its device copy,
// chooses the launch shape (fixed, default or autotuned), launches the
// reset, the sign pass and the sampler, and decodes kept final states for
// the readout calls.  No simulation arithmetic runs here; every shot is
// computed by the kernels in signs.hip and sampler.hip.
#include "soft.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "compile.h"
#include "devbuf.h"
#include "sampler.h"
#include "signs.h"

using namespace soft;

namespace {

thread_local std::string g_create_error;

struct Shape {
    uint32_t wpb = 0, bpc = 0, grab = 0;
    uint32_t gt = TM_LDS;  // tile placement: TM_LDS, TM_MEM or TM_SPLIT
    uint32_t lds_log2 = 0; // TM_SPLIT: log2 of the tile entries held in LDS
};

struct Variant {
    std::string text;
    NoiseModel noise;
    uint64_t shot_end = ~0ull;  // global shots [previous end, shot_end)
    Program prog;               // the full event list
    Program fast;               // the speculative list with DROP events (empty: none found)
    bool has_fast = false;
};

// counter rows, then the work cursors (on a cache line's start)
static_assert(kMaxVariants <= kCounterRows, "a row per variant");
constexpr size_t kCursorOff = ((size_t)kCounterRows * C_COUNT + kCursorStride - 1) / kCursorStride * kCursorStride;
constexpr size_t kCounterWords = kCursorOff + kCursorWords;
static_assert(kCounterWords * sizeof(unsigned long long) <= kScratchCounterBytes, "scratch counter area");

// Kept final states: at most this many shots, and at most kMaxKeepBytes of
// dense tiles (FP64 pairs) for them.
constexpr uint32_t kMaxKeep = 16384;
constexpr uint64_t kMaxKeepBytes = 4ull << 30;

// Autotuned launch shapes, shared by every context of the process: keyed by
// the device (architecture name and compute-unit count) and by what changes
// the timing of a circuit (its hash with the shot ranges, precision, pruning
// threshold, support cap, tile placement, noise draws, and whether the sign
// pass runs before the sampler: what is left to it then asks for other shapes).
typedef std::tuple<std::string, int, uint64_t, int, double, uint32_t, int, int, bool> TuneKey;
std::mutex g_tune_mu;
std::map<TuneKey, Shape> g_tuned;

struct HipMem {
    static int alloc(void **p, size_t bytes) { return (int)hipMalloc(p, bytes); }
    static int free(void *p) { return (int)hipFree(p); }
};

}  // namespace

struct soft_ctx {
    int device = 0;
    int num_cus = 0;
    int max_lds_block = 65536;
    std::string err;

    bool have_text = false;
    bool mixture = false;
    NoiseModel noise;            // model of a single loaded circuit
    std::vector<Variant> vars;   // the circuit, or the circuits of a mixture
    bool dirty = true;           // device tables must be rebuilt
    uint32_t kmax = 0, rec_words = 0;  // largest over the variants
    uint64_t hash = 0;           // of every variant and its shot range

    uint64_t seed = 0;
    const uint32_t *words_dev = nullptr;
    uint64_t words_n = 0;
    uint32_t words_noise = 0, words_meas = 0;
    int bits = 64;
    double tau = -1.0;
    uint32_t support_cap = 0;
    int tile_mode = 0;                        // 0 auto, 1 LDS, 2 device memory, 3 split
    uint32_t split_log2 = 0;                  // split: log2 of the LDS part asked for (0: default)
    bool speculate = true;                    // run speculative event lists where compiled
    bool shared_prefix = true;                // start shots at checkpoints of the noiseless trajectory
    bool defer_t = true;                      // skip deferrable T runs until an event needs their tile
    bool any_prefix = false;                  // some variant's lists have checkpoints
    int noise_mode = 0;                       // 0 a word per noise slot, 1 gap sampling
    Shape user;                               // explicit launch shape parts
    std::string arch;                         // gcnArchName of the device (autotune cache key)

    Buffers<HipMem> mem;
    DevBuf<Event> d_ev;
    DevBuf<NoiseLoc> d_nz;
    DevBuf<uint32_t> d_tm1, d_det, d_gap;
    DevBuf<BatchMember> d_bm;
    DevBuf<DiagInfo> d_diag;
    DevBuf<VariantDesc> d_vars;
    DevBuf<unsigned char> d_gtile;            // device-memory tiles
    DevBuf<unsigned char> d_prefix;           // checkpoint state slots (one per table entry)
    DevBuf<unsigned char> d_prefix_rec;       // those that recorded launches build in every replay
    DevBuf<Checkpoint> d_ckpt;                // checkpoint table
    uint32_t n_ckpt = 0;                      // its entries
    // What the states in d_prefix were built for (none: empty); a run that
    // asks for the same ones leaves the build out.
    std::vector<uint64_t> prefix_key;
    DevBuf<unsigned char> d_signs;            // the sign pass's tables, one after the other
    SignParams sign_tables = {};              // their places in it
    uint32_t sign_size = 0;                   // their vector size (kSignTestWords)
    uint32_t sign_on = 0;                     // some variant's shots are worth it: bit 0 gaps, bit 1 slots
    bool sign_few = false;                    // it leaves few shots to the sampler
    bool sign_whole = false;                  // it decides every variant's list to its end
    double sign_left = 1.0;                   // else about the share of shots that it leaves
    unsigned long long *d_counters = nullptr;  // kCounterRows rows of C_COUNT, then the work cursors
    const unsigned long long *last_counters = nullptr;  // counters of the last run
    uint32_t last_shards = 1, last_vars = 0;            // their rows per variant, and its variants
    double *d_phase = nullptr;                 // cos/sin of k pi/8, k = 0..15
    unsigned char *scratch = nullptr;          // this device's static scratch (soft_run_noalloc)

    uint64_t keep_lo = 0;
    uint32_t keep_n = 0;
    DevBuf<unsigned long long> d_keep_meta;
    DevBuf<double> d_keep_v;
    uint32_t keep_tile = 0;  // tile entries of the last run's keep buffer

    uint64_t trace_shot = 0;
    uint32_t trace_n = 0;
    DevBuf<unsigned long long> d_trace_meta;
    DevBuf<double> d_trace_v;
    uint32_t trace_tile = 0;

    uint64_t launches = 0;
    hipEvent_t done = nullptr;           // after the last launch, and its stream
    hipStream_t done_stream = nullptr;

    template <typename F> void each_table(F f) {
        f(d_ev), f(d_nz), f(d_tm1), f(d_det), f(d_gap), f(d_bm), f(d_diag), f(d_vars), f(d_ckpt), f(d_signs);
    }
    template <typename F> void each_buffer(F f) {
        each_table(f);
        f(d_gtile), f(d_prefix), f(d_prefix_rec), f(d_keep_meta), f(d_keep_v), f(d_trace_meta), f(d_trace_v);
    }

    bool ran = false;
    hipStream_t last_stream = nullptr;
    uint64_t last_shot0 = 0, last_n = 0;
    bool last_list = false;  // the last run sampled a shot list
    hipStream_t noalloc_stream = nullptr;  // of the last soft_run_noalloc that no capture recorded,
    bool noalloc_pending = false;          // not waited for since
};

namespace {

int fail(soft_ctx *c, int code, const std::string &msg) {
    if (c) c->err = msg;
    return code;
}

// No C++ exception crosses the C boundary: what a call cannot hold on the host
// is a capacity error (its text fits a string without allocation).
int no_memory(soft_ctx *c) {
    if (c) c->err = "no host memory";
    return SOFT_ECAPACITY;
}
#define SOFT_GUARD(ctx) catch (const std::bad_alloc &) { return no_memory(ctx); }

#define HIPCHK(ctx, expr)                                                                          \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess) return fail((ctx), SOFT_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

int alloc_rc(soft_ctx *c, int e) {
    return e ? fail(c, SOFT_EDEVICE, std::string("device memory: ") + hipGetErrorString((hipError_t)e)) : SOFT_OK;
}
template <typename T> int ensure(soft_ctx *c, DevBuf<T> &b, size_t n) { return alloc_rc(c, c->mem.ensure(b, n)); }
template <typename T> int renew(soft_ctx *c, DevBuf<T> &b, size_t n) { return alloc_rc(c, c->mem.renew(b, n)); }

// Whether a stream capture records the launches on `stream`.
bool capturing(hipStream_t stream) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &st) != hipSuccess) (void)hipGetLastError();  // (the launches report it)
    return st != hipStreamCaptureStatusNone;
}

// A recording holds the context's tables from here on, and of its other
// buffers those that these parameters name.
void mark_recorded(soft_ctx *c, const RunParams &rp) {
    c->each_table([](auto &b) { b.recorded = b.p != nullptr; });
    auto mark = [](auto &b, const void *p) { b.recorded = b.recorded || (p != nullptr && (const void *)b.p == p); };
    mark(c->d_gtile, rp.gtile);
    mark(c->d_prefix_rec, rp.prefix);
    mark(c->d_keep_meta, rp.keep_meta);
    mark(c->d_keep_v, rp.keep_v);
    mark(c->d_trace_meta, rp.trace_meta);
    mark(c->d_trace_v, rp.trace_v);
}

double tau_of(const soft_ctx *c) { return c->tau >= 0.0 ? c->tau : (c->bits == 32 ? 1e-6 : 1e-12); }

uint32_t tile_entries(const soft_ctx *c) { return 1u << c->kmax; }
uint32_t rec_words(const soft_ctx *c) { return c->rec_words; }
uint32_t entry_bytes(const soft_ctx *c) { return c->bits == 64 ? 16u : 8u; }
uint32_t tile_bytes(const soft_ctx *c) { return tile_entries(c) * entry_bytes(c); }
// Smallest LDS part of a split tile: the passes put up to 128 consecutive
// entries of one iteration on a wave's lanes, and the split keeps them in one
// place.
constexpr uint32_t kSplitMinLog2 = 7;
bool split_possible(const soft_ctx *c) { return c->kmax >= kSplitMinLog2 + 1u; }
// Tile bytes a wave keeps in LDS.
uint32_t lds_tile_bytes(const soft_ctx *c, const Shape &s) {
    if (s.gt == TM_MEM) return 0u;
    if (s.gt == TM_SPLIT) return (1u << s.lds_log2) * entry_bytes(c);
    return tile_bytes(c);
}
// Device-memory slab bytes per wave.
uint32_t slab_bytes(const soft_ctx *c, const Shape &s) { return tile_bytes(c) - lds_tile_bytes(c, s); }
// LDS bytes per wave: the tile or its LDS part, and the record.  A record of
// at most kRecSgpr words stays in scalar registers and takes no LDS.
uint32_t wave_bytes(const soft_ctx *c, const Shape &s) {
    const uint32_t recb = rec_words(c) > kRecSgpr ? (rec_words(c) * 4u + 15u) & ~15u : 0u;
    return std::max<uint32_t>(16u, ((lds_tile_bytes(c, s) + 15u) & ~15u) + recb);
}
// Bytes of one checkpoint slot: the state, the record words and a whole
// tile, 256-aligned.
uint32_t prefix_stride(const soft_ctx *c) {
    return (kCkptRecOff + ((rec_words(c) * 4u + 15u) & ~15u) + tile_bytes(c) + 255u) & ~255u;
}
bool use_prefix(const soft_ctx *c) { return c->shared_prefix && c->any_prefix; }

// The prefix build launch's parameters: item i = variant i / 2, list i & 1,
// no outputs, no kept states or trace, its own work cursor.
RunParams build_params(const RunParams &rp) {
    RunParams b = rp;
    b.prefix_build = 1;
    b.n_shots = 2ull * rp.n_vars;
    b.shot0 = 0;
    b.shot_list = nullptr;
    b.outcomes = nullptr;
    b.status = nullptr;
    b.abort_op = nullptr;
    b.obs = nullptr;
    b.keep_meta = nullptr;
    b.keep_v = nullptr;
    b.keep_n = 0;
    b.trace_meta = nullptr;
    b.trace_v = nullptr;
    b.trace_n = 0;
    b.grab = 1;
    b.queue_shift = 0;
    b.next = rp.next + kBuildCursor;
    return b;
}

// Default LDS part of a split tile: at most 8 KiB, below the whole tile.
uint32_t split_log2_default(const soft_ctx *c) {
    uint32_t L = c->kmax - 1u;
    while (L > kSplitMinLog2 && (1u << L) * entry_bytes(c) > 8192u) --L;
    return L;
}

// Wait for the last launch (each waits for the one before it); a
// soft_run_noalloc records no event, its stream is waited for.
void wait_done(soft_ctx *c) {
    if (c->done) (void)hipEventSynchronize(c->done);
    if (c->noalloc_pending) (void)hipStreamSynchronize(c->noalloc_stream);
    c->noalloc_pending = false;
}

int compile_into(soft_ctx *c, const std::string &text, const NoiseModel &nm, Program &out, bool speculate = false) {
    try {
        compile_circuit(text, nm, out, speculate);
    } catch (const CompileError &e) {
        return fail(c, e.line > 0 ? SOFT_EPARSE : SOFT_ECAPACITY,
                    e.line > 0 ? "line " + std::to_string(e.line) + ": " + e.msg : e.msg);
    } catch (const std::bad_alloc &) {
        return fail(c, SOFT_ECAPACITY, "out of host memory while compiling");
    }
    return SOFT_OK;
}

// Compile a variant's full event list and, when the circuit offers span
// truncations, its speculative list.
int compile_variant(soft_ctx *c, Variant &V) {
    int rc = compile_into(c, V.text, V.noise, V.prog);
    if (rc) return rc;
    V.has_fast = false;
    V.fast = Program();
    if ((rc = compile_into(c, V.text, V.noise, V.fast, true))) return rc;
    for (const Event &E : V.fast.events)
        if (E.kind == EV_DROP || (E.flags & EVF_DROP1)) V.has_fast = true;
    if (!V.has_fast) V.fast = Program();
    return SOFT_OK;
}

// A list is worth the sign pass when the signs decide it to its end, or when
// they end enough shots before the coefficients matter: the others are drawn
// twice.  Drawing by gaps costs little of a shot, a word per slot much of it.
// 10^5 shots of three circuits of T brackets and checks (36, 90 and 220 noise
// slots) whose coefficients are read at the end, time with the pass over time
// without, by the share of shots that a check ends: by gaps 1.02 to 1.03 at
// 0.016, 0.99 to 1.00 at 0.05, 0.95 at 0.14, 0.82 at 0.43; by slots 1.06 at
// 0.05, 1.03 to 1.11 at 0.15, 0.92 to 0.93 at 0.4.  (Checks that come first save
// the sampler nothing and lose 1 to 4% at any share.)
constexpr double kSignEndsGaps = 0.04, kSignEndsSlots = 0.25;

// Up to one broken T pair a shot, few shots break dependent ones or more than
// four at a time, which a complete list leaves to the sampler: of 6 10^4, 5
// 10^-5 on 15 qubits at 0.08 broken pairs a shot, 8 10^-4 at 0.4, 1.3 10^-3 at
// 0.8; none on 42 qubits up to 1.3.  Pairs on a span that is never empty are
// left whenever they break (one shot in 50 to 1000), and count here too: whole
// tiles then cost up to 1.7 times a split one's time or save up to 1.6 (spans
// 2^11 to 2^14, 10^5 and 10^6 shots, p = 10^-5 to 2 10^-3), by how many shots
// are left for a resident wave.
constexpr double kSignFewBreaks = 1.0;

// The sign pass's tables: every variant's sign program in the smallest common
// vector size.
int build_sign_tables(soft_ctx *c) {
    const size_t nv = c->vars.size();
    std::vector<SignProgram> sp(nv);
    c->sign_on = 0;
    c->sign_size = 0;
    c->sign_few = true;
    auto fits = [](const SignProgram &S, uint32_t k) {
        return S.need.tests <= kSignTestWords[k] && S.need.out() <= kSignOutWords[k];
    };
    // (a mixture often holds one circuit at several rates: only the
    // thresholds differ)
    auto same_vecs = [](const SignProgram &A, const SignProgram &B) {
        return A.on && A.need.tests == B.need.tests && A.vecs == B.vecs;
    };
    for (size_t v = 0; v < nv; ++v) {
        const Variant &V = c->vars[v];
        build_signs(V.has_fast ? V.fast : V.prog, sp[v]);
        SignProgram &S = sp[v];
        S.on = S.on && fits(S, 3u) && (S.complete || S.ends >= kSignEndsGaps);
        if (!S.on || !S.complete || S.breaks > kSignFewBreaks) c->sign_few = false;
        if (!S.on) continue;
        while (!fits(S, c->sign_size)) ++c->sign_size;
        c->sign_on = 1u;
    }
    if (!c->sign_on) return SOFT_OK;
    // variants past the tables' limit run without it
    uint64_t left = kMaxSignBytes;
    c->sign_on = 0;
    for (size_t v = 0; v < nv; ++v) {
        SignProgram &S = sp[v];
        if (!S.on) continue;
        const bool shared = v > 0 && same_vecs(sp[v - 1], S);
        const uint64_t bytes = shared ? 0u : S.slots.size() * kSignVecs * 4ull * (kSignTestWords[c->sign_size] + kSignOutWords[c->sign_size]);
        S.on = bytes <= left;
        if (!S.on) {
            c->sign_few = false;
            continue;
        }
        left -= bytes;
        c->sign_on |= 1u | ((S.complete || S.ends >= kSignEndsSlots) ? 2u : 0u);
    }
    if (!c->sign_on) return SOFT_OK;
    c->sign_whole = true;
    double left_shots = 0.0, all_shots = 0.0;
    for (size_t v = 0; v < nv; ++v) {
        const double n = (double)(c->vars[v].shot_end - (v ? c->vars[v - 1].shot_end : 0ull));
        const bool whole = sp[v].on && sp[v].complete;
        c->sign_whole = c->sign_whole && whole;
        all_shots += n;
        left_shots += whole ? 0.0 : sp[v].on ? n * (1.0 - sp[v].ends) : n;
    }
    c->sign_left = left_shots / all_shots;
    const uint32_t TW = kSignTestWords[c->sign_size], RO = kSignOutWords[c->sign_size], W = TW + RO;
    std::vector<SignDesc> desc(nv);
    std::vector<SignSlot> slot;
    std::vector<SignTest> test;
    std::vector<uint32_t> vec(W, 0u), mask;  // vector 0 is zero
    std::vector<uint2> coin;
    std::vector<SignPair> pair;
    std::vector<SignMeas> meas;
    std::memset(desc.data(), 0, nv * sizeof(SignDesc));
    // a program vector (tests, records, observables) in the launch's layout
    auto lay = [&](const uint32_t *x, const SignProgram &S, uint32_t *d) {
        for (uint32_t w = 0; w < S.need.tests; ++w) d[w] = x[w];
        for (uint32_t w = 0; w < S.need.recs; ++w) d[TW + w] = x[S.need.tests + w];
        d[W - 1u] = x[S.need.tests + S.need.recs];
    };
    for (size_t v = 0; v < nv; ++v) {
        const SignProgram &S = sp[v];
        SignDesc &D = desc[v];
        if (!S.on) continue;
        auto put = [&](const std::vector<uint32_t> &x) {
            const uint32_t at = (uint32_t)(vec.size() / W);
            vec.resize(vec.size() + W, 0u);
            lay(x.data(), S, &vec[(size_t)at * W]);
            return at;
        };
        D.on = 1u | ((S.complete || S.ends >= kSignEndsSlots) ? 2u : 0u);
        D.n_tests = (uint32_t)S.tests.size() - 1u;
        D.slot_off = (uint32_t)slot.size();
        D.test_off = (uint32_t)test.size();
        slot.insert(slot.end(), S.slots.begin(), S.slots.end());
        test.insert(test.end(), S.tests.begin(), S.tests.end());
        for (const auto &m : S.mask) {
            mask.resize(mask.size() + RO, 0u);
            uint32_t *d = &mask[mask.size() - RO];
            for (uint32_t w = 0; w < S.need.recs; ++w) d[w] = m[w];
            d[RO - 1u] = m.back();
        }
        D.ref_vec = put(S.ref);
        if (v > 0 && same_vecs(sp[v - 1], S)) {
            D.vec_off = desc[v - 1].vec_off;
        } else {
            D.vec_off = (uint32_t)(vec.size() / W);
            const size_t w0 = S.ref.size(), k = S.vecs.size() / w0;
            vec.resize(vec.size() + k * W, 0u);
            for (size_t i = 0; i < k; ++i) lay(&S.vecs[i * w0], S, &vec[(D.vec_off + i) * W]);
        }
        D.coin_off = (uint32_t)coin.size();
        D.n_coins = (uint32_t)S.coin.size();
        for (size_t i = 0; i < S.coin.size(); ++i) coin.push_back(make_uint2(S.coin_slot[i], put(S.coin[i])));
        D.pair_off = (uint32_t)pair.size();
        D.meas_off = (uint32_t)meas.size();
        D.n_meas = (uint32_t)S.meas.size();
        for (SignPair q : S.pairs) {
            q.vec = put(S.pair_vecs[q.vec]);
            pair.push_back(q);
        }
        meas.insert(meas.end(), S.meas.begin(), S.meas.end());
        const Program &P = c->vars[v].has_fast ? c->vars[v].fast : c->vars[v].prog;
        D.ck_cnt = (uint32_t)P.ckpts.size();
    }
    // one allocation and one copy
    std::vector<unsigned char> all;
    auto put = [&](const void *src, size_t bytes) {
        const size_t at = (all.size() + 255u) & ~(size_t)255u;
        all.resize(at + bytes);
        if (bytes) std::memcpy(&all[at], src, bytes);
        return at;
    };
    const size_t at[8] = {put(vec.data(), vec.size() * sizeof(uint32_t)), put(slot.data(), slot.size() * sizeof(SignSlot)),
                          put(test.data(), test.size() * sizeof(SignTest)), put(mask.data(), mask.size() * sizeof(uint32_t)),
                          put(coin.data(), coin.size() * sizeof(uint2)), put(desc.data(), nv * sizeof(SignDesc)),
                          put(pair.data(), pair.size() * sizeof(SignPair)), put(meas.data(), meas.size() * sizeof(SignMeas))};
    if (int rc = renew(c, c->d_signs, all.size())) return rc;
    HIPCHK(c, hipMemcpy(c->d_signs.p, all.data(), all.size(), hipMemcpyHostToDevice));
    SignParams &T = c->sign_tables;
    T.vecs = reinterpret_cast<const uint4 *>(c->d_signs.p + at[0]);
    T.slots = reinterpret_cast<const SignSlot *>(c->d_signs.p + at[1]);
    T.tests = reinterpret_cast<const SignTest *>(c->d_signs.p + at[2]);
    T.mask = reinterpret_cast<const uint32_t *>(c->d_signs.p + at[3]);
    T.coins = reinterpret_cast<const uint2 *>(c->d_signs.p + at[4]);
    T.desc = reinterpret_cast<const SignDesc *>(c->d_signs.p + at[5]);
    T.pairs = reinterpret_cast<const SignPair *>(c->d_signs.p + at[6]);
    T.meas = reinterpret_cast<const SignMeas *>(c->d_signs.p + at[7]);
    return SOFT_OK;
}

// The circuit runs without the sign pass too: where its tables find no memory,
// on the host or the device, it does.
void prepare_signs(soft_ctx *c) {
    int rc = SOFT_ECAPACITY;
    try {
        rc = build_sign_tables(c);
    } catch (const std::bad_alloc &) {
    }
    if (rc == SOFT_OK) return;
    (void)hipGetLastError();
    c->err.clear();
    c->sign_on = 0;
    c->sign_few = false;
}

// Upload the compiled variants as one set of tables: each variant's events,
// noise locations, thresholds, check pairs and run members are appended, and
// its references into the shared tables are rebased.
int prepare(soft_ctx *c) {
    if (!c->have_text) return fail(c, SOFT_ESTATE, "no circuit loaded");
    if (!c->dirty) return SOFT_OK;
    std::vector<Event> ev;
    std::vector<NoiseLoc> nz;
    std::vector<uint32_t> tm1, det, gap;
    std::vector<BatchMember> bm;
    std::vector<DiagInfo> dg;
    std::vector<VariantDesc> vd;
    std::vector<Checkpoint> ck;
    c->kmax = 0;
    c->rec_words = 0;
    uint64_t h = 1469598103934665603ULL;
    for (const Variant &V : c->vars) {
        const Program &P = V.prog;
        VariantDesc D;
        std::memset(&D, 0, sizeof(D));
        D.shot_end = V.shot_end;
        D.nz_off = (uint32_t)nz.size();
        D.tm1_off = (uint32_t)tm1.size();
        D.n_noise = P.n_noise;
        D.gap_off = (uint32_t)gap.size();
        D.gap_l2q = (P.gap_pmax > 0.0 && P.gap_pmax < 1.0) ? (float)(1.0 / std::log2(1.0 - P.gap_pmax)) : 0.0f;
        D.acc_one = P.noise.empty() ? 0u : 1u;
        for (const NoiseLoc &L : P.noise)
            if (L.acc != (1ull << 32)) D.acc_one = 0u;
        // each event list with its own check pairs and run members
        auto append = [&](const Program &Q) {
            const uint32_t off = (uint32_t)ev.size();
            const uint32_t det_base = (uint32_t)(det.size() / 2), bm_base = (uint32_t)bm.size();
            const uint32_t dg_base = (uint32_t)dg.size();
            for (Event E : Q.events) {
                E.det_off += det_base;
                if (E.flags & EVF_BATCH) E.boff += bm_base;
                if (E.kind == EV_DIAG) E.boff += dg_base;
                ev.push_back(E);
            }
            det.insert(det.end(), Q.det_pairs.begin(), Q.det_pairs.end());
            bm.insert(bm.end(), Q.batch.begin(), Q.batch.end());
            dg.insert(dg.end(), Q.diag.begin(), Q.diag.end());
            return off;
        };
        D.ev_off_full = append(P);
        D.ev_off = V.has_fast ? append(V.fast) : D.ev_off_full;
        // checkpoints of each list (one set when the variant has one list)
        D.ck_off_full = (uint32_t)ck.size();
        D.ck_cnt_full = (uint32_t)P.ckpts.size();
        ck.insert(ck.end(), P.ckpts.begin(), P.ckpts.end());
        D.ck_off = D.ck_off_full;
        D.ck_cnt = D.ck_cnt_full;
        if (V.has_fast) {
            D.ck_off = (uint32_t)ck.size();
            D.ck_cnt = (uint32_t)V.fast.ckpts.size();
            ck.insert(ck.end(), V.fast.ckpts.begin(), V.fast.ckpts.end());
        }
        nz.insert(nz.end(), P.noise.begin(), P.noise.end());
        tm1.insert(tm1.end(), P.noise_tm1.begin(), P.noise_tm1.end());
        gap.insert(gap.end(), P.gap.begin(), P.gap.end());
        gap.insert(gap.end(), 8u, 0u);  // the sign pass reads four entries from an estimate up to the end
        vd.push_back(D);
        c->kmax = std::max(c->kmax, P.kmax);
        c->rec_words = std::max(c->rec_words, (P.n_rec + 31u) / 32u);
        h = (h ^ P.hash) * 1099511628211ULL;
        h = (h ^ V.shot_end) * 1099511628211ULL;
    }
    c->hash = h;
    c->any_prefix = !ck.empty();
    c->n_ckpt = (uint32_t)ck.size();
    int rc;
    wait_done(c);  // its launches read the tables
    if ((rc = renew(c, c->d_ev, ev.size())) || (rc = renew(c, c->d_nz, std::max<size_t>(nz.size(), 1))) ||
        (rc = renew(c, c->d_tm1, tm1.size())) || (rc = renew(c, c->d_det, std::max<size_t>(det.size(), 2))) ||
        (rc = renew(c, c->d_bm, std::max<size_t>(bm.size(), 1))) || (rc = renew(c, c->d_vars, vd.size())) ||
        (rc = renew(c, c->d_diag, std::max<size_t>(dg.size(), 1))) ||
        (rc = renew(c, c->d_gap, std::max<size_t>(gap.size(), 1))) ||
        (rc = renew(c, c->d_ckpt, std::max<size_t>(ck.size(), 1))))
        return rc;
    if (!ck.empty()) HIPCHK(c, hipMemcpy(c->d_ckpt.p, ck.data(), ck.size() * sizeof(Checkpoint), hipMemcpyHostToDevice));
    if (!gap.empty()) HIPCHK(c, hipMemcpy(c->d_gap.p, gap.data(), gap.size() * sizeof(uint32_t), hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(c->d_ev.p, ev.data(), ev.size() * sizeof(Event), hipMemcpyHostToDevice));
    if (!nz.empty()) HIPCHK(c, hipMemcpy(c->d_nz.p, nz.data(), nz.size() * sizeof(NoiseLoc), hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(c->d_tm1.p, tm1.data(), tm1.size() * sizeof(uint32_t), hipMemcpyHostToDevice));
    if (!det.empty()) HIPCHK(c, hipMemcpy(c->d_det.p, det.data(), det.size() * sizeof(uint32_t), hipMemcpyHostToDevice));
    if (!bm.empty()) HIPCHK(c, hipMemcpy(c->d_bm.p, bm.data(), bm.size() * sizeof(BatchMember), hipMemcpyHostToDevice));
    if (!dg.empty()) HIPCHK(c, hipMemcpy(c->d_diag.p, dg.data(), dg.size() * sizeof(DiagInfo), hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(c->d_vars.p, vd.data(), vd.size() * sizeof(VariantDesc), hipMemcpyHostToDevice));
    prepare_signs(c);
    c->dirty = false;
    c->prefix_key.clear();
    return SOFT_OK;
}

// Largest LDS a CU offers to resident blocks (gfx950: 160 KiB).
constexpr uint32_t kLdsPerCu = 160u * 1024u;
constexpr uint32_t kMaxWavesPerCu = 32u;

// Untuned launch shape: as many resident waves per CU as the LDS tiles allow
// (at most 32), two waves per block when that still leaves >= 16 waves.
// Device-memory tiles are used when asked for, or (auto) when one wave's LDS
// tile does not fit in a block's LDS.
// Noise source of the next launch (explicit words use the per-slot form).
uint32_t noise_source(const soft_ctx *c) {
    return c->words_dev != nullptr ? NS_EXPLICIT : (c->noise_mode == 1 ? NS_GAPS : NS_SLOTS);
}

// Whether a launch runs the sign pass: its results stand on T pairs that
// cancel exactly and on checkpoints and deferred runs being allowed to skip
// their work, so every option that asks for that work keeps it (and a pruning
// threshold above rounding changes the states it would skip); kept states,
// traces, caps, shot lists (`list`) and explicit words need the sampler's own
// walk.
constexpr double kSignMaxTau = 1e-6;
bool use_signs(const soft_ctx *c, bool list) {
    const uint32_t bit = c->noise_mode == 1 ? 1u : 2u;
    return (c->sign_on & bit) && !list && !c->keep_n && !c->trace_n && !c->words_dev && !c->support_cap &&
           c->speculate && c->shared_prefix && c->defer_t && tau_of(c) <= kSignMaxTau;
}

// The placement asked for (soft_set_tile_memory), or (auto) LDS when one
// wave's tile fits in a block's LDS, else device memory.  A split needs a
// span of at least 2^8 entries; below that the tile is small and goes to LDS.
Shape placement(const soft_ctx *c, bool list) {
    Shape s;
    if (c->tile_mode == 2) {
        s.gt = TM_MEM;
    } else if (c->tile_mode == 3 && split_possible(c)) {
        s.gt = TM_SPLIT;
        s.lds_log2 = c->split_log2 ? std::min<uint32_t>(c->split_log2, c->kmax - 1u) : split_log2_default(c);
    } else if (c->tile_mode == 0) {
        // LDS up to 8 KiB a wave (20 waves a CU, the register-bound
        // occupancy), a split above that while the tile would fit a block's
        // LDS (its LDS part holds twice the waves or more), device memory for
        // tiles no block holds.  When the sign pass leaves few shots, waves in
        // flight do not count but each one's way through its list does: whole
        // tiles in LDS up to a block's (27 variants in FP64 343 -> 304 us, a
        // first call of the span-12 scan 1065 -> 850).
        Shape l;
        if (wave_bytes(c, l) > (uint32_t)c->max_lds_block) {
            s.gt = TM_MEM;
        } else if (c->sign_few && use_signs(c, list)) {
            s.gt = TM_LDS;
        } else if (tile_bytes(c) > 8192u && split_possible(c)) {
            s.gt = TM_SPLIT;
            s.lds_log2 = split_log2_default(c);
        }
    }
    return s;
}

// Resident waves per CU when the tile is not the limit (4 waves per SIMD).
constexpr uint32_t kMemTileWavesPerCu = 16u;

Shape default_shape(const soft_ctx *c, bool list) {
    Shape s = placement(c, list);
    const uint32_t wb = wave_bytes(c, s);
    const uint32_t cap = s.gt == TM_MEM ? kMemTileWavesPerCu : kMaxWavesPerCu;
    const uint32_t waves_cu = std::max<uint32_t>(1u, std::min<uint32_t>(cap, kLdsPerCu / wb));
    s.wpb = (waves_cu >= 16u && 2u * wb <= (uint32_t)c->max_lds_block) ? 2u : 1u;
    while (s.wpb > 1 && s.wpb * wb > (uint32_t)c->max_lds_block) s.wpb /= 2;
    s.bpc = std::max<uint32_t>(1u, waves_cu / s.wpb);
    // no more blocks than stay resident (registers can be the tighter limit)
    int res = 0;
    if (sampler_occupancy(c->bits == 64, noise_source(c), s.gt, (int)(64u * s.wpb), (size_t)s.wpb * wb,
                          &res) == hipSuccess && res > 0)
        s.bpc = std::min<uint32_t>(s.bpc, (uint32_t)res);
    else
        (void)hipGetLastError();
    s.grab = 16;
    return s;
}

TuneKey tune_key(const soft_ctx *c, bool list) {
    return TuneKey(c->arch, c->num_cus, c->hash, c->bits, tau_of(c), c->support_cap,
                   c->tile_mode | (int)(c->split_log2 << 8), c->noise_mode, use_signs(c, list));
}

Shape current_shape(const soft_ctx *c, bool list = false) {
    Shape s = default_shape(c, list);
    {
        std::lock_guard<std::mutex> lock(g_tune_mu);
        auto it = g_tuned.find(tune_key(c, list));
        if (it != g_tuned.end()) s = it->second;
    }
    if (c->tile_mode) {  // an explicit placement overrides a tuned one
        const Shape p = placement(c, list);
        if (p.gt != s.gt || (p.gt == TM_SPLIT && c->split_log2)) {
            s.gt = p.gt;
            s.lds_log2 = p.lds_log2;
        }
    }
    if (c->user.wpb) s.wpb = c->user.wpb;
    if (c->user.bpc) s.bpc = c->user.bpc;
    if (c->user.grab) s.grab = c->user.grab;
    return s;
}

int check_shape(soft_ctx *c, const Shape &s) {
    if (s.gt == TM_SPLIT && (s.lds_log2 < kSplitMinLog2 || s.lds_log2 >= c->kmax))
        return fail(c, SOFT_EINVAL, "split tile: LDS part out of range");
    const uint64_t lds = (uint64_t)s.wpb * wave_bytes(c, s);
    if (s.wpb < 1 || s.wpb > 4) return fail(c, SOFT_EINVAL, "waves_per_block must be 1..4");
    if (lds > (uint64_t)c->max_lds_block)
        return fail(c, SOFT_ECAPACITY, "coefficient tile needs " + std::to_string(lds) + " bytes of LDS per block; the device allows " +
                                           std::to_string(c->max_lds_block) + " (span dimension " + std::to_string(c->kmax) + ")");
    if (s.bpc < 1 || s.grab < 1 || s.grab > 64) return fail(c, SOFT_EINVAL, "blocks_per_cu must be >= 1 and grab in 1..64");
    return SOFT_OK;
}

// Blocks of a launch: the resident blocks of the shape, at most one per
// `wpb` shots.
uint64_t grid_blocks(const soft_ctx *c, const Shape &s, uint64_t n_shots) {
    const uint64_t blocks_needed = (n_shots + s.wpb - 1) / s.wpb;
    return std::min<uint64_t>((uint64_t)c->num_cus * s.bpc, std::max<uint64_t>(blocks_needed, 1));
}

// Blocks of the prefix build: one item a wave, so that it needs no cursors and
// may run before they are reset.
uint32_t build_blocks(const Shape &s, const RunParams &rp) { return (2u * rp.n_vars + s.wpb - 1u) / s.wpb; }

// LDS layout of a wave's slot (tile unless in device memory, record words
// past kRecSgpr).
void set_wave_layout(const soft_ctx *c, const Shape &s, RunParams &rp) {
    rp.wave_bytes = wave_bytes(c, s);
    rp.rec_off = (s.gt != TM_MEM && rec_words(c) > kRecSgpr) ? ((lds_tile_bytes(c, s) + 15u) & ~15u) : 0u;
    rp.gtile = nullptr;
    rp.tile_mode = s.gt;
    rp.lds_entries = s.gt == TM_SPLIT ? (1u << s.lds_log2) : 0u;
}

// The sign pass's arguments and grid (waves), after rp's outputs, counters and
// cursors are set.
uint32_t sign_params(const soft_ctx *c, const RunParams &rp, SignParams &sp) {
    sp = c->sign_tables;
    sp.vars = rp.vars;
    sp.tm1 = rp.tm1;
    sp.gaps = rp.gaps;
    sp.outcomes = rp.outcomes;
    sp.status = rp.status;
    sp.abort_op = rp.abort_op;
    sp.obs = rp.obs;
    sp.counters = rp.counters;
    sp.shards = rp.shards;
    sp.next = rp.next + kSignCursor;
    sp.seed = rp.seed;
    sp.shot0 = rp.shot0;
    sp.n_shots = rp.n_shots;
    sp.n_vars = rp.n_vars;
    sp.rec_words = rp.rec_words;
    sp.prefix = rp.prefix ? 1u : 0u;
    // no more waves than stay resident: the chunks are dealt out evenly
    const uint64_t most = (uint64_t)c->num_cus * kSignWavesPerCu[c->sign_size];
    // Whole waves of shots (64 with gap sampling, 4 with a word per slot).
    // With gaps a shot takes a step or two: a wave waits for its chunks, and
    // lanes past a chunk's end for the next one, so it gets its share at once,
    // up to four waves of shots (2 10^6 shots of 27 variants: 225 us, 254 in
    // chunks of one; 10^7 of 42 qubits: 502, and 521 in chunks of 13).  A word
    // per slot makes shots long and uneven: eight chunks a wave (5 10^5 shots:
    // 927 us, 969 with four, 1057 with two).
    const bool gaps = rp.noise_mode == 1u;
    const uint64_t held = gaps ? 64u : 4u, share = rp.n_shots / (most * held);
    sp.chunk = (uint32_t)(held * std::max<uint64_t>(1u, gaps ? std::min<uint64_t>(4u, share) : std::min<uint64_t>(16u, share / 8u)));
    // (the kernel draws from eight cursors where the chunks outnumber its waves)
    static_assert(kSignWavesPerCu[3] >= kQueueCursors, "a wave on every cursor");
    return (uint32_t)std::min<uint64_t>(most, (rp.n_shots + sp.chunk - 1u) / sp.chunk);
}

// Positions a wave of the sampler takes at a time.  A launch of a few shots a
// wave deals them out evenly (16 at a time, 256 shots ran on 16 waves); a
// larger one leaves at least four groups a wave to even out their lengths, up
// to the shape's.  After the sign pass few positions are left to run: whole
// reads of 64 statuses, about four groups a wave, since each group is an
// atomic (10^7 shots in groups of 64 took 1.9 ms to find none left).  Where it
// leaves nearly none, about two groups of whole reads of 256 (42 qubits, 10^7:
// 471 us a run, 483 with four groups; 10^6 FP64 120 and 128; 15 qubits 10^6
// 516 and 538).
// Where the pass does not decide whole lists many shots are left: groups as
// without it, by the shots left in them (5 10^4 shots of injected T gates after
// a check that 60% of them fail, 1.38 -> 0.87 ms; 2 10^5 of 8 qubits, of which
// 94% end, 177 -> 144 us: a wave's share in one group waited for the longest).
uint32_t group_size(const soft_ctx *c, const Shape &s, uint64_t grid, uint64_t n_shots, bool signs) {
    if (c->user.grab) return c->user.grab;
    const uint64_t waves = grid * s.wpb, each = (n_shots + waves - 1u) / waves;
    if (signs && !c->sign_whole && each >= 4u) {
        const double left = std::max(c->sign_left, 1e-3);  // (at least about one of them in a group)
        const double n = std::max((double)(each / 4u), std::min((double)each, 1.0 / left));
        return (uint32_t)std::min(1024.0, std::min(n, s.grab / left));
    }
    if (signs && each > 64u) {
        const uint64_t n = c->sign_few ? (each / 2u + 255u) / 256u * 256u : (each / 4u + 63u) / 64u * 64u;
        return (uint32_t)std::min<uint64_t>(1024u, n);
    }
    if (signs) return (uint32_t)each;
    return (uint32_t)(each < 4u ? each : std::min<uint64_t>(s.grab, each / 4u));
}

// Cursors of the sampler's queue.  Without the sign pass a shot takes long, and
// groups of eight or more (32 shots a wave) come from one cursor, which keeps
// every wave at work to the end: span-12 lists in circuit order 16.2 -> 15.3 ms
// (2.4 10^5 shots), 42 qubits in device-memory tiles 29.6 -> 27.8 (10^6), 15
// qubits with kept states 1.58 -> 1.56 (6.6 10^5), 8 qubits the same.  Below
// that its atomics count: 15 qubits 0.28 -> 0.34 ms at 15 shots a wave, 8
// qubits 0.23 -> 0.29.
constexpr uint32_t kOneCursorGroup = 8;
uint32_t cursor_shift(const RunParams &rp, uint64_t waves, bool signs) {
    return !signs && rp.grab >= kOneCursorGroup ? 0u : queue_shift((uint32_t)std::min<uint64_t>(waves, kQueueCursors));
}

// The launches of a run, one after the other on `stream`: the checkpoint build
// where its states are not there yet, the reset, the sign pass where it runs,
// the sampler.  A stream takes them 7 us faster than as one graph of kernel
// nodes with new arguments (4096 shots of 42 qubits: 36.7 against 43.2 us a
// call, 10^6: 130.6 against 138.4).
int launch(soft_ctx *c, RunParams rp, const Shape &s, uint64_t n_shots, hipStream_t stream) {
    const uint32_t wb = wave_bytes(c, s);
    const size_t lds = (size_t)s.wpb * wb;
    const uint64_t grid = grid_blocks(c, s, n_shots);
    const dim3 g((uint32_t)grid), b(64u * s.wpb);
    set_wave_layout(c, s, rp);
    const bool captured = capturing(stream);
    if (s.gt != TM_LDS) {  // one slab per wave of the grid (the build's or the sampler's)
        int rc = ensure(c, c->d_gtile, std::max<size_t>(grid, build_blocks(s, rp)) * s.wpb * slab_bytes(c, s));
        if (rc) return rc;
        rp.gtile = c->d_gtile.p;
    }
    // Shared-prefix slots, filled by the build launch before the sampler.  The
    // states depend on the loaded tables and on what this key holds, so they
    // stay for the runs that follow: one wave walks a whole list for them
    // (85 to 265 us, with the sign pass most of a launch of 10^5 shots).  Runs
    // of a context are in stream order, or ordered by the caller.  A recorded
    // launch has slots of its own and builds its states in every replay.
    const bool pfx = use_prefix(c);
    bool build = false;
    std::vector<uint64_t> pkey;
    rp.prefix = nullptr;
    rp.prefix_stride = 0;
    if (pfx) {
        const size_t bytes = (size_t)c->n_ckpt * prefix_stride(c);
        if (captured && c->d_prefix_rec.n < bytes && c->d_prefix.n >= bytes) {
            // (a capture may forbid allocation: it takes the slots that are there)
            if (int rc = alloc_rc(c, c->mem.drop(c->d_prefix_rec))) return rc;
            std::swap(c->d_prefix, c->d_prefix_rec);
            c->prefix_key.clear();
        }
        DevBuf<unsigned char> &slots = captured ? c->d_prefix_rec : c->d_prefix;
        if (int rc = ensure(c, slots, bytes)) return rc;
        rp.prefix = slots.p;
        rp.prefix_stride = prefix_stride(c);
        const double tau = tau_of(c);
        uint64_t tb;
        std::memcpy(&tb, &tau, sizeof(tb));
        pkey = {(uint64_t)(uintptr_t)slots.p, (uint64_t)c->bits, tb, rp.support_cap};
        build = captured || pkey != c->prefix_key;
    }
    if (captured) mark_recorded(c, rp);
    const bool sgn = use_signs(c, rp.shot_list != nullptr);
    rp.grab = group_size(c, s, grid, n_shots, sgn);
    rp.queue_shift = cursor_shift(rp, grid * s.wpb, sgn);
    // another stream than the last launch's: after it, for the states it built
    if (!captured && c->done && stream != c->done_stream) HIPCHK(c, hipStreamWaitEvent(stream, c->done, 0));
    if (build) {
        if (!captured) c->prefix_key.clear();
        HIPCHK(c, launch_prefix_build(build_params(rp), c->bits == 64, dim3(build_blocks(s, rp)), b, lds, stream));
    }
    HIPCHK(c, launch_reset(rp.counters, rp.n_vars * rp.shards * (uint32_t)C_COUNT, rp.next, stream));
    if (sgn) {
        rp.signs = 1;
        SignParams sp;
        const uint32_t sgrid = sign_params(c, rp, sp);
        HIPCHK(c, launch_signs(sp, c->sign_size, rp.noise_mode == 1u, dim3(sgrid), stream));
    }
    HIPCHK(c, launch_sampler(rp, c->bits == 64, g, b, lds, stream));
    ++c->launches;
    if (captured) return SOFT_OK;
    if (build) c->prefix_key = pkey;
    if (!c->done) HIPCHK(c, hipEventCreateWithFlags(&c->done, hipEventDisableTiming));
    HIPCHK(c, hipEventRecord(c->done, stream));
    c->done_stream = stream;
    return SOFT_OK;
}

// Counter rows per variant.
uint32_t shards(const soft_ctx *c) {
    uint32_t s = kMaxShards;
    while (s * c->vars.size() > kCounterRows) s /= 2u;
    return s;
}

int make_params(soft_ctx *c, uint64_t shot0, uint64_t n_shots, uint32_t *outcomes, uint32_t *status, uint32_t *abort_op,
                uint32_t *obs, RunParams &rp) {
    std::memset(&rp, 0, sizeof(rp));
    rp.ev = c->d_ev.p;
    rp.nz = c->d_nz.p;
    rp.tm1 = c->d_tm1.p;
    rp.det = c->d_det.p;
    rp.bm = c->d_bm.p;
    rp.diag = c->d_diag.p;
    rp.ckpts = c->d_ckpt.p;
    rp.defer = c->defer_t ? 1u : 0u;
    rp.speculate = c->speculate ? 1u : 0u;
    rp.gaps = c->d_gap.p;
    rp.noise_mode = (uint32_t)c->noise_mode;
    rp.vars = c->d_vars.p;
    rp.n_vars = (uint32_t)c->vars.size();
    rp.words = c->words_dev;
    rp.phase_tab = c->d_phase;
    rp.word_stride = (uint64_t)c->vars[0].prog.n_noise + c->vars[0].prog.n_meas;
    rp.outcomes = outcomes;
    rp.status = status;
    rp.abort_op = abort_op;
    rp.obs = obs;
    rp.counters = c->d_counters;
    rp.next = c->d_counters + kCursorOff;
    rp.shards = shards(c);
    rp.seed = c->seed;
    rp.shot0 = shot0;
    rp.n_shots = n_shots;
    rp.rec_words = rec_words(c);
    rp.support_cap = c->support_cap ? c->support_cap : 0xFFFFFFFFu;
    rp.tile_entries = tile_entries(c);
    rp.tile_bytes = tile_bytes(c);
    const double t = tau_of(c);
    rp.tau2 = t * t;
    rp.grab = 1;
    if (c->keep_n) {
        const uint32_t te = tile_entries(c);
        if ((uint64_t)c->keep_n * te * 16u > kMaxKeepBytes)
            return fail(c, SOFT_ECAPACITY, "kept states would take more than 4 GiB (" + std::to_string(c->keep_n) +
                                               " shots of 2^" + std::to_string(c->kmax) + " entries); keep fewer shots");
        int rc;
        if ((rc = ensure(c, c->d_keep_meta, (size_t)c->keep_n * KM_COUNT)) ||
            (rc = ensure(c, c->d_keep_v, (size_t)c->keep_n * te * 2)))
            return rc;
        rp.keep_meta = c->d_keep_meta.p;
        rp.keep_v = c->d_keep_v.p;
        rp.keep_lo = c->keep_lo;
        rp.keep_n = c->keep_n;
        c->keep_tile = te;
    }
    if (c->trace_n) {
        const uint32_t te = tile_entries(c);
        int rc;
        if ((rc = ensure(c, c->d_trace_meta, (size_t)c->trace_n * KM_COUNT)) ||
            (rc = ensure(c, c->d_trace_v, (size_t)c->trace_n * te * 2)))
            return rc;
        rp.trace_meta = c->d_trace_meta.p;
        rp.trace_v = c->d_trace_v.p;
        rp.trace_shot = c->trace_shot;
        rp.trace_n = c->trace_n;
        c->trace_tile = te;
    }
    return SOFT_OK;
}

// (`vars`: other shot ranges than the loaded ones)
int run_impl(soft_ctx *c, uint64_t shot0, uint64_t n_shots, uint32_t *outcomes, uint32_t *status, uint32_t *abort_op,
             uint32_t *obs, hipStream_t stream, const Shape &s, const uint64_t *shot_list = nullptr,
             const VariantDesc *vars = nullptr) {
    RunParams rp;
    int rc = make_params(c, shot0, n_shots, outcomes, status, abort_op, obs, rp);
    if (rc) return rc;
    if (vars) rp.vars = vars;
    rp.grab = s.grab;
    rp.shot_list = shot_list;
    if (c->trace_n)  // mark every trace step unwritten
        HIPCHK(c, launch_clear(c->d_trace_meta.p, (uint64_t)c->trace_n * KM_COUNT, stream));
    if ((rc = launch(c, rp, s, n_shots, stream))) return rc;
    c->ran = true;
    c->last_counters = c->d_counters;
    c->last_shards = rp.shards;
    c->last_vars = rp.n_vars;
    c->last_stream = stream;
    c->last_shot0 = shot0;
    c->last_n = n_shots;
    c->last_list = shot_list != nullptr;
    return SOFT_OK;
}

// The event list that produced a dumped state.
const Program &program_of(const soft_ctx *c, const std::vector<unsigned long long> &meta) {
    const Variant &V = c->vars[meta[KM_VAR]];
    return (meta[KM_PROG] || !V.has_fast) ? V.prog : V.fast;
}

// Frame (x/z bits and span basis) in which a dumped state is expressed.
const Frame *frame_of(soft_ctx *c, const std::vector<unsigned long long> &meta, int &rc) {
    const uint64_t v = meta[KM_VAR], term = meta[KM_TERM_EV];
    if (v >= c->vars.size()) {
        rc = fail(c, SOFT_EDEVICE, "corrupt dumped state");
        return nullptr;
    }
    const Program &P = program_of(c, meta);
    if (term >= P.events.size()) {
        rc = fail(c, SOFT_EDEVICE, "corrupt dumped state");
        return nullptr;
    }
    return meta[KM_AFTER] ? &P.after[term] : &P.before[term];
}

const Frame *kept_frame(soft_ctx *c, uint64_t shot, std::vector<unsigned long long> &meta, std::vector<double> &tile, int &rc) {
    rc = SOFT_OK;
    if (!c->ran) { rc = fail(c, SOFT_ESTATE, "no run yet"); return nullptr; }
    if (!c->keep_n || shot < c->keep_lo || shot - c->keep_lo >= c->keep_n ||
        (!c->last_list && (shot < c->last_shot0 || shot - c->last_shot0 >= c->last_n))) {
        rc = fail(c, SOFT_EINVAL, "shot was not kept by the last run (see soft_set_keep)");
        return nullptr;
    }
    hipError_t e = hipStreamSynchronize(c->last_stream);
    if (e != hipSuccess) { rc = fail(c, SOFT_EDEVICE, std::string("hipStreamSynchronize: ") + hipGetErrorString(e)); return nullptr; }
    const uint64_t kk = shot - c->keep_lo;
    meta.resize(KM_COUNT);
    tile.resize((size_t)c->keep_tile * 2);
    e = hipMemcpy(meta.data(), c->d_keep_meta.p + kk * KM_COUNT, KM_COUNT * sizeof(unsigned long long), hipMemcpyDeviceToHost);
    if (e == hipSuccess)
        e = hipMemcpy(tile.data(), c->d_keep_v.p + kk * (uint64_t)c->keep_tile * 2, tile.size() * sizeof(double), hipMemcpyDeviceToHost);
    if (e != hipSuccess) { rc = fail(c, SOFT_EDEVICE, std::string("hipMemcpy: ") + hipGetErrorString(e)); return nullptr; }
    return frame_of(c, meta, rc);
}

// Coefficients of a dumped state: alpha(j) = a ^ sum_t j_t b_t over the
// frame's span basis; entries below the pruning threshold are left out.
int decode_coeffs(soft_ctx *c, const Frame &f, const std::vector<unsigned long long> &meta,
                  const std::vector<double> &tile, uint64_t *alpha, double *re, double *im, uint32_t cap,
                  uint32_t *count) {
    const uint32_t k = (uint32_t)meta[KM_K];
    if (k != f.basis.size() || (1ull << k) * 2 > tile.size())
        return fail(c, SOFT_EDEVICE, "dumped state does not match the compiled frame");
    const uint64_t a = meta[KM_A];
    const uint32_t cnt = 1u << k;
    double n2 = 0.0;
    for (uint32_t j = 0; j < cnt; ++j) n2 += tile[2 * j] * tile[2 * j] + tile[2 * j + 1] * tile[2 * j + 1];
    const double t = tau_of(c);
    std::vector<std::pair<uint64_t, uint32_t>> keep;
    for (uint32_t j = 0; j < cnt; ++j) {
        const double q = tile[2 * j] * tile[2 * j] + tile[2 * j + 1] * tile[2 * j + 1];
        if (q == 0.0 || q < t * t * n2) continue;
        uint64_t al = a;
        for (uint32_t b = 0; b < k; ++b)
            if ((j >> b) & 1u) al ^= f.basis[b];
        keep.push_back({al, j});
    }
    std::sort(keep.begin(), keep.end());
    *count = (uint32_t)keep.size();
    for (uint32_t i = 0; i < keep.size() && i < cap; ++i) {
        if (alpha) alpha[i] = keep[i].first;
        if (re) re[i] = tile[2 * keep[i].second];
        if (im) im[i] = tile[2 * keep[i].second + 1];
    }
    return SOFT_OK;
}

// Tableau rows of a dumped state: x/z from the frame, signs from the shot.
void decode_tableau(const Frame &f, const std::vector<unsigned long long> &meta, uint64_t *x,
                    uint64_t *z, uint8_t *r) {
    const int n = (int)f.xd.size();
    for (int i = 0; i < n; ++i) {
        uint64_t xd = 0, zd = 0, xs = 0, zs = 0;
        for (int q = 0; q < n; ++q) {
            xd |= ((f.xd[q] >> i) & 1ull) << q;
            zd |= ((f.zd[q] >> i) & 1ull) << q;
            xs |= ((f.xs[q] >> i) & 1ull) << q;
            zs |= ((f.zs[q] >> i) & 1ull) << q;
        }
        if (x) { x[i] = xd; x[n + i] = xs; }
        if (z) { z[i] = zd; z[n + i] = zs; }
        if (r) {
            r[i] = (uint8_t)((meta[KM_RD] >> i) & 1ull);
            r[n + i] = (uint8_t)((meta[KM_RS] >> i) & 1ull);
        }
    }
}

// Candidate shapes of a launch: the default first, then a grid of shapes per
// tile placement (in automatic mode LDS when it fits, device memory, and splits
// whose LDS part is 1/2, 1/4 or 1/8 of the tile).
std::vector<Shape> shape_candidates(const soft_ctx *c, bool list) {
    std::vector<Shape> cands;
    cands.push_back(default_shape(c, list));
    const uint32_t wpbs[3] = {1, 2, 4};
    // (after the sign pass the groups follow from the launch: group_size)
    std::vector<uint32_t> grabs = {16, 64};
    if (use_signs(c, list)) grabs.resize(1);
    std::vector<Shape> places;
    if (c->tile_mode != 0) {
        places.push_back(placement(c, list));
        if (places[0].gt == TM_SPLIT && !c->split_log2)  // other LDS parts of the split
            for (uint32_t d = 1; d <= 3; ++d) {
                Shape p = places[0];
                p.lds_log2 = c->kmax - d;
                if (p.lds_log2 >= kSplitMinLog2 && p.lds_log2 != places[0].lds_log2) places.push_back(p);
            }
    } else {
        const Shape lds_p;  // the whole tile in LDS, when a block holds it
        if (wave_bytes(c, lds_p) <= (uint32_t)c->max_lds_block) places.push_back(lds_p);
        Shape m;
        m.gt = TM_MEM;
        places.push_back(m);
        for (uint32_t d = 1; d <= 3 && split_possible(c); ++d) {
            Shape p;
            p.gt = TM_SPLIT;
            p.lds_log2 = c->kmax - d;
            if (p.lds_log2 >= kSplitMinLog2) places.push_back(p);
        }
    }
    for (const Shape &place : places) {
        const uint32_t wb = wave_bytes(c, place);
        for (uint32_t wpb : wpbs) {
            if (wpb * wb > (uint32_t)c->max_lds_block) continue;
            const uint32_t cap = place.gt == TM_MEM ? kMemTileWavesPerCu : kMaxWavesPerCu;
            const uint32_t occ = std::max<uint32_t>(1u, std::min<uint32_t>(kLdsPerCu / (wpb * wb), cap / wpb));
            std::vector<uint32_t> bpcs;
            for (uint32_t d : {4u, 2u, 1u}) {
                uint32_t v = std::max<uint32_t>(1u, occ / d);
                if (std::find(bpcs.begin(), bpcs.end(), v) == bpcs.end()) bpcs.push_back(v);
            }
            for (uint32_t bpc : bpcs)
                for (uint32_t grab : grabs) {
                    Shape sh = place;
                    sh.wpb = wpb;
                    sh.bpc = bpc;
                    sh.grab = grab;
                    cands.push_back(sh);
                }
        }
    }
    return cands;
}

// What a tuning holds while it runs; given back at its end.
struct TuneScope {
    soft_ctx *c;
    uint32_t keep_n;
    uint32_t *status = nullptr;
    uint64_t *list = nullptr;
    VariantDesc *vars = nullptr;
    hipEvent_t t0 = nullptr, t1 = nullptr;
    hipStream_t st;
    TuneScope(soft_ctx *c_, hipStream_t st_) : c(c_), keep_n(c_->keep_n), st(st_) { c->keep_n = 0; }
    ~TuneScope() {
        c->keep_n = keep_n;
        (void)hipStreamSynchronize(st);
        if (t0) (void)hipEventDestroy(t0);
        if (t1) (void)hipEventDestroy(t1);
        if (status) (void)hipFree(status);
        if (list) (void)hipFree(list);
        if (vars) (void)hipFree(vars);
    }
};

// After the sign pass a launch is short, and what is left to the sampler a
// small part of it: a shape replaces the default only where it is faster by
// more than the runs of one shape differ (0.1 to 0.7%).
constexpr float kTuneGain = 0.98f;

}  // namespace

extern "C" {

int soft_create(soft_ctx **out, int hip_device) {
    if (!out) return SOFT_EINVAL;
    *out = nullptr;
    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess || hip_device < 0 || hip_device >= ndev) {
        g_create_error = e != hipSuccess ? std::string("hipGetDeviceCount: ") + hipGetErrorString(e) : "no such HIP device";
        return e != hipSuccess ? SOFT_EDEVICE : SOFT_EINVAL;
    }
    soft_ctx *c = new (std::nothrow) soft_ctx();
    if (!c) { g_create_error = "out of host memory"; return SOFT_ECAPACITY; }
    c->device = hip_device;
    auto bad = [&](hipError_t err, const char *what) {
        g_create_error = std::string(what) + ": " + hipGetErrorString(err);
        soft_destroy(c);
        return SOFT_EDEVICE;
    };
    if ((e = hipSetDevice(hip_device)) != hipSuccess) return bad(e, "hipSetDevice");
    if ((e = hipDeviceGetAttribute(&c->num_cus, hipDeviceAttributeMultiprocessorCount, hip_device)) != hipSuccess)
        return bad(e, "hipDeviceGetAttribute");
    int lds = 0;
    if ((e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, hip_device)) != hipSuccess)
        return bad(e, "hipDeviceGetAttribute");
    c->max_lds_block = lds;
    {
        hipDeviceProp_t prop;
        if ((e = hipGetDeviceProperties(&prop, hip_device)) != hipSuccess) return bad(e, "hipGetDeviceProperties");
        c->arch = prop.gcnArchName;
    }
    if (sampler_set_lds_limit(lds) != hipSuccess) {
        (void)hipGetLastError();
        c->max_lds_block = std::min(lds, 65536);
    }
    if ((e = hipMalloc((void **)&c->d_counters, kCounterWords * sizeof(unsigned long long))) != hipSuccess)
        return bad(e, "hipMalloc");
    if ((e = hipMemset(c->d_counters, 0, kCounterWords * sizeof(unsigned long long))) != hipSuccess) return bad(e, "hipMemset");
    // the static scratch of soft_run_noalloc: its device address on this GPU
    if ((e = scratch_address(hip_device, &c->scratch)) != hipSuccess) return bad(e, "hipGetSymbolAddress(scratch)");
    {
        double tab[32];
        for (int q = 0; q < 16; ++q) {
            tab[q] = std::cos(M_PI * q / 8.0);
            tab[16 + q] = std::sin(M_PI * q / 8.0);
        }
        if ((e = hipMalloc((void **)&c->d_phase, sizeof(tab))) != hipSuccess) return bad(e, "hipMalloc");
        if ((e = hipMemcpy(c->d_phase, tab, sizeof(tab), hipMemcpyHostToDevice)) != hipSuccess) return bad(e, "hipMemcpy");
    }
    *out = c;
    return SOFT_OK;
}

void soft_destroy(soft_ctx *c) {
    if (!c) return;
    (void)hipSetDevice(c->device);
    if (c->ran && c->last_stream) (void)hipStreamSynchronize(c->last_stream);
    wait_done(c);
    c->each_buffer([c](auto &b) { c->mem.release(b); });
    c->mem.release_aside();
    if (c->d_counters) (void)hipFree(c->d_counters);
    if (c->d_phase) (void)hipFree(c->d_phase);
    if (c->done) (void)hipEventDestroy(c->done);
    delete c;
}

const char *soft_last_error(const soft_ctx *c) { return c ? c->err.c_str() : g_create_error.c_str(); }

int soft_load_circuit(soft_ctx *c, const char *text, size_t len) try {
    if (!c || (!text && len)) return fail(c, SOFT_EINVAL, "null argument");
    Variant V;
    V.text.assign(text ? text : "", len);
    V.noise = c->noise;
    int rc = compile_variant(c, V);
    if (rc) return rc;
    c->vars.clear();
    c->vars.push_back(std::move(V));
    c->have_text = true;
    c->mixture = false;
    c->dirty = true;
    (void)hipSetDevice(c->device);
    return prepare(c);
} SOFT_GUARD(c)

int soft_load_noise(soft_ctx *c, const soft_noise *m) try {
    if (!c || !m) return fail(c, SOFT_EINVAL, "null argument");
    if (c->mixture) return fail(c, SOFT_ESTATE, "a mixture carries one noise model per variant; load it again instead");
    NoiseModel nm;
    nm.p1 = m->p1;
    nm.p2 = m->p2;
    nm.p_idle = m->p_idle;
    nm.p_meas = m->p_meas;
    nm.p_reset = m->p_reset;
    nm.p_mpp = m->p_mpp;
    const double ps[6] = {nm.p1, nm.p2, nm.p_idle, nm.p_meas, nm.p_reset, nm.p_mpp};
    for (double p : ps)
        if (!(p >= 0.0 && p <= 1.0)) return fail(c, SOFT_EINVAL, "noise probability out of [0,1]");
    if (c->have_text) {
        Variant V;
        V.text = c->vars[0].text;
        V.noise = nm;
        int rc = compile_variant(c, V);
        if (rc) return rc;
        c->vars[0] = std::move(V);
        c->dirty = true;
    }
    c->noise = nm;
    if (!c->have_text) return SOFT_OK;
    (void)hipSetDevice(c->device);
    return prepare(c);
} SOFT_GUARD(c)

int soft_load_mixture(soft_ctx *c, uint32_t n_variants, const char *const *texts, const size_t *lens,
                      const soft_noise *models, const uint64_t *shot_ends) try {
    if (!c || !texts || !lens || !models || !shot_ends) return fail(c, SOFT_EINVAL, "null argument");
    if (n_variants < 1 || n_variants > kMaxVariants)
        return fail(c, SOFT_EINVAL, "n_variants must be in 1.." + std::to_string(kMaxVariants));
    std::vector<Variant> vs(n_variants);
    for (uint32_t v = 0; v < n_variants; ++v) {
        if (!texts[v] && lens[v]) return fail(c, SOFT_EINVAL, "null circuit text");
        if (shot_ends[v] == 0 || (v > 0 && shot_ends[v] <= shot_ends[v - 1]))
            return fail(c, SOFT_EINVAL, "shot_ends must be positive and strictly increasing");
        const soft_noise &m = models[v];
        NoiseModel nm;
        nm.p1 = m.p1;
        nm.p2 = m.p2;
        nm.p_idle = m.p_idle;
        nm.p_meas = m.p_meas;
        nm.p_reset = m.p_reset;
        nm.p_mpp = m.p_mpp;
        vs[v].text.assign(texts[v] ? texts[v] : "", lens[v]);
        vs[v].noise = nm;
        vs[v].shot_end = shot_ends[v];
        int rc = compile_variant(c, vs[v]);
        if (rc) return fail(c, rc, "variant " + std::to_string(v) + ": " + c->err);
    }
    c->vars = std::move(vs);
    c->have_text = true;
    c->mixture = true;
    c->dirty = true;
    (void)hipSetDevice(c->device);
    return prepare(c);
} SOFT_GUARD(c)

int soft_set_rng(soft_ctx *c, uint64_t seed) {
    if (!c) return SOFT_EINVAL;
    c->seed = seed;
    return SOFT_OK;
}

int soft_set_uniforms(soft_ctx *c, const uint32_t *words_dev, uint64_t n_shots, uint32_t noise_slots, uint32_t meas_slots) {
    if (!c) return SOFT_EINVAL;
    if (!words_dev) {
        c->words_dev = nullptr;
        c->words_n = 0;
        return SOFT_OK;
    }
    if (((uintptr_t)words_dev & 3u) != 0) return fail(c, SOFT_EINVAL, "words_dev must be 4-byte aligned");
    c->words_dev = words_dev;
    c->words_n = n_shots;
    c->words_noise = noise_slots;
    c->words_meas = meas_slots;
    return SOFT_OK;
}

int soft_set_precision(soft_ctx *c, int bits) {
    if (!c) return SOFT_EINVAL;
    if (bits != 32 && bits != 64) return fail(c, SOFT_EINVAL, "coeff_bits must be 32 or 64");
    c->bits = bits;
    return SOFT_OK;
}

int soft_set_prune(soft_ctx *c, double tau) {
    if (!c) return SOFT_EINVAL;
    if (std::isnan(tau) || tau >= 1.0) return fail(c, SOFT_EINVAL, "tau must be < 1");
    c->tau = tau < 0.0 ? -1.0 : tau;
    return SOFT_OK;
}

int soft_set_caps(soft_ctx *c, uint32_t support_cap, uint32_t wpb, uint32_t bpc, uint32_t grab) {
    if (!c) return SOFT_EINVAL;
    if (wpb > 4) return fail(c, SOFT_EINVAL, "waves_per_block must be <= 4");
    if (bpc > kMaxWavesPerCu) return fail(c, SOFT_EINVAL, "blocks_per_cu must be <= 32");
    if (grab > 64) return fail(c, SOFT_EINVAL, "grab must be <= 64");
    c->support_cap = support_cap;
    c->user.wpb = wpb;
    c->user.bpc = bpc;
    c->user.grab = grab;
    return SOFT_OK;
}

int soft_set_speculation(soft_ctx *c, int on) {
    if (!c) return SOFT_EINVAL;
    c->speculate = on != 0;
    return SOFT_OK;
}

int soft_set_shared_prefix(soft_ctx *c, int on) {
    if (!c) return SOFT_EINVAL;
    c->shared_prefix = on != 0;
    return SOFT_OK;
}

int soft_set_deferred_t(soft_ctx *c, int on) {
    if (!c) return SOFT_EINVAL;
    c->defer_t = on != 0;
    return SOFT_OK;
}

int soft_set_noise_mode(soft_ctx *c, int mode) {
    if (!c) return SOFT_EINVAL;
    if (mode < 0 || mode > 1) return fail(c, SOFT_EINVAL, "noise mode must be 0 (a word per slot) or 1 (gap sampling)");
    c->noise_mode = mode;
    return SOFT_OK;
}

int soft_set_tile_memory(soft_ctx *c, int mode) {
    if (!c) return SOFT_EINVAL;
    const int base = mode & 0xff, L = mode >> 8;
    if (mode < 0 || base > 3 || (base != 3 && L != 0) || (L != 0 && (L < (int)kSplitMinLog2 || L > 19)))
        return fail(c, SOFT_EINVAL, "tile memory mode must be 0 (auto), 1 (LDS), 2 (device memory), 3 (split) or "
                                    "256 L + 3 (split with 2^L entries in LDS, 7 <= L <= 19)");
    c->tile_mode = base;
    c->split_log2 = (uint32_t)L;
    return SOFT_OK;
}

int soft_set_keep(soft_ctx *c, uint64_t shot_lo, uint32_t count) {
    if (!c) return SOFT_EINVAL;
    if (count > kMaxKeep) return fail(c, SOFT_ECAPACITY, "at most " + std::to_string(kMaxKeep) + " kept shots");
    c->keep_lo = shot_lo;
    c->keep_n = count;
    return SOFT_OK;
}

int soft_run(soft_ctx *c, uint64_t shot0, uint64_t n_shots, uint32_t *outcomes, uint32_t *status, uint32_t *abort_op,
             uint32_t *obs, void *hip_stream) try {
    if (!c) return SOFT_EINVAL;
    if (!status && n_shots) return fail(c, SOFT_EINVAL, "status_dev is required");
    HIPCHK(c, hipSetDevice(c->device));
    int rc = prepare(c);
    if (rc) return rc;
    if (c->words_dev) {
        if (c->mixture) return fail(c, SOFT_EUNSUPPORTED, "explicit words are for a single circuit, not a mixture");
        const Program &P = c->vars[0].prog;
        if (c->words_noise != P.n_noise || c->words_meas != P.n_meas)
            return fail(c, SOFT_EINVAL, "explicit words: expected " + std::to_string(P.n_noise) + " noise and " +
                                            std::to_string(P.n_meas) + " measurement slots per shot");
        if (n_shots > c->words_n) return fail(c, SOFT_EINVAL, "explicit words: fewer rows than shots");
    }
    if (shot0 + n_shots < shot0 || shot0 + n_shots > c->vars.back().shot_end)
        return fail(c, SOFT_EINVAL, "shots beyond the last variant's range");
    if (n_shots == 0) return SOFT_OK;
    Shape s = current_shape(c);
    if ((rc = check_shape(c, s))) return rc;
    return run_impl(c, shot0, n_shots, outcomes, status, abort_op, obs, (hipStream_t)hip_stream, s);
} SOFT_GUARD(c)

int soft_run_noalloc(soft_ctx *c, uint64_t shot0, uint64_t n_shots, uint32_t *outcomes, uint32_t *status,
                     uint32_t *abort_op, uint32_t *obs, void *hip_stream) try {
    if (!c) return SOFT_EINVAL;
    if (!status && n_shots) return fail(c, SOFT_EINVAL, "status_dev is required");
    HIPCHK(c, hipSetDevice(c->device));
    if (!c->have_text) return fail(c, SOFT_ESTATE, "no circuit loaded");
    if (c->dirty)  // the soft_load_* calls upload the tables; this stays only after a failed upload
        return fail(c, SOFT_ESTATE, "the circuit's device tables are not uploaded (the last soft_load_* failed)");
    if (c->keep_n || c->trace_n)
        return fail(c, SOFT_EUNSUPPORTED, "kept states and traces use buffers the library allocates; turn them off "
                                          "(soft_set_keep(ctx, 0, 0), soft_set_trace(ctx, 0, 0)) for soft_run_noalloc");
    if (c->words_dev) {
        if (c->mixture) return fail(c, SOFT_EUNSUPPORTED, "explicit words are for a single circuit, not a mixture");
        const Program &P = c->vars[0].prog;
        if (c->words_noise != P.n_noise || c->words_meas != P.n_meas)
            return fail(c, SOFT_EINVAL, "explicit words: expected " + std::to_string(P.n_noise) + " noise and " +
                                            std::to_string(P.n_meas) + " measurement slots per shot");
        if (n_shots > c->words_n) return fail(c, SOFT_EINVAL, "explicit words: fewer rows than shots");
    }
    if (shot0 + n_shots < shot0 || shot0 + n_shots > c->vars.back().shot_end)
        return fail(c, SOFT_EINVAL, "shots beyond the last variant's range");
    if (n_shots == 0) return SOFT_OK;
    Shape s = current_shape(c);
    int rc = check_shape(c, s);
    if (rc) return rc;
    RunParams rp;
    if ((rc = make_params(c, shot0, n_shots, outcomes, status, abort_op, obs, rp))) return rc;
    rp.grab = s.grab;
    set_wave_layout(c, s, rp);
    // counters and cursor, then (device-memory tiles) one slab per wave, all
    // in this device's static scratch; with slabs the grid shrinks to what
    // the scratch holds (the kernel is persistent, so fewer waves take more
    // shots each)
    rp.counters = reinterpret_cast<unsigned long long *>(c->scratch);
    rp.next = rp.counters + kCursorOff;
    // shared-prefix slots when they fit their part of the scratch (without
    // them every shot runs from the start: the same results)
    const bool pfx = use_prefix(c) && (uint64_t)c->n_ckpt * prefix_stride(c) <= kScratchPrefixBytes;
    rp.prefix = pfx ? c->scratch + kScratchCounterBytes : nullptr;
    rp.prefix_stride = pfx ? prefix_stride(c) : 0u;
    uint64_t grid = grid_blocks(c, s, n_shots);
    if (s.gt != TM_LDS) {
        const uint64_t slab = (uint64_t)s.wpb * slab_bytes(c, s);
        const uint64_t fit = kScratchTileBytes / slab;
        if (fit == 0)
            return fail(c, SOFT_ECAPACITY, "device-memory tiles of one block need " + std::to_string(slab) +
                                               " bytes; soft_run_noalloc's scratch holds " +
                                               std::to_string(kScratchTileBytes) + " (span dimension " +
                                               std::to_string(c->kmax) + ")");
        grid = std::min<uint64_t>(grid, fit);
        rp.gtile = c->scratch + kScratchCounterBytes + kScratchPrefixBytes;
    }
    const hipStream_t stream = (hipStream_t)hip_stream;
    if (capturing(stream)) {
        mark_recorded(c, rp);
    } else {
        c->noalloc_stream = stream;
        c->noalloc_pending = true;
    }
    HIPCHK(c, launch_reset(rp.counters, rp.n_vars * rp.shards * (uint32_t)C_COUNT, rp.next, stream));
    if (pfx)
        HIPCHK(c, launch_prefix_build(build_params(rp), c->bits == 64,
                                 dim3((uint32_t)std::min<uint64_t>(grid, (2ull * rp.n_vars + s.wpb - 1) / s.wpb)),
                                 dim3(64u * s.wpb), (size_t)s.wpb * wave_bytes(c, s), stream));
    const bool sgn = use_signs(c, rp.shot_list != nullptr);
    rp.grab = group_size(c, s, grid, n_shots, sgn);
    rp.queue_shift = cursor_shift(rp, grid * s.wpb, sgn);
    if (sgn) {
        rp.signs = 1;
        SignParams sp;
        const uint32_t sgrid = sign_params(c, rp, sp);
        HIPCHK(c, launch_signs(sp, c->sign_size, rp.noise_mode == 1u, dim3(sgrid), stream));
    }
    HIPCHK(c, launch_sampler(rp, c->bits == 64, dim3((uint32_t)grid), dim3(64u * s.wpb),
                             (size_t)s.wpb * wave_bytes(c, s), stream));
    c->ran = true;
    c->last_counters = rp.counters;
    c->last_shards = rp.shards;
    c->last_vars = rp.n_vars;
    c->last_stream = stream;
    c->last_shot0 = shot0;
    c->last_n = n_shots;
    c->last_list = false;
    return SOFT_OK;
} SOFT_GUARD(c)

namespace {
// Sum of the last run's counters over its variants [v0, v1) (maximum for the
// norm deviation).  A load since then changes neither that run's variants nor
// where its rows lie; variants that it did not have counted nothing.
int read_rows(soft_ctx *c, uint32_t v0, uint32_t v1, soft_counters *out) {
    if (!c->ran) return fail(c, SOFT_ESTATE, "no run yet");
    HIPCHK(c, hipSetDevice(c->device));
    HIPCHK(c, hipStreamSynchronize(c->last_stream));
    const uint32_t k = c->last_shards;
    v1 = std::min(v1, c->last_vars);
    v0 = std::min(v0, v1);
    std::vector<unsigned long long> h((size_t)(v1 - v0) * k * C_COUNT);
    if (!h.empty())
        HIPCHK(c, hipMemcpy(h.data(), c->last_counters + (size_t)v0 * k * C_COUNT, h.size() * sizeof(unsigned long long),
                            hipMemcpyDeviceToHost));
    std::memset(out, 0, sizeof(*out));
    double dev = 0.0;
    for (uint32_t v = 0; v < (v1 - v0) * k; ++v) {
        const unsigned long long *r = h.data() + (size_t)v * C_COUNT;
        out->shots += r[C_SHOTS];
        out->passed += r[C_PASSED];
        out->discarded += r[C_DISCARDED];
        out->overflow += r[C_OVERFLOW];
        out->numeric += r[C_NUMERIC];
        out->logical_errors += r[C_LOGICAL];
        out->entries_t += r[C_ENTRIES_T];
        out->entries_m += r[C_ENTRIES_M];
        out->noise_slots += r[C_NOISE];
        out->events += r[C_EVENTS];
        out->restarts += r[C_RESTARTS];
        out->prefix_shots += r[C_PREFIX];
        out->redo_shots += r[C_REDO];
        for (int b = 0; b < 16; ++b) out->support_hist[b] += r[C_HIST0 + b];
        double d;
        std::memcpy(&d, &r[C_NORMDEV_BITS], sizeof(double));
        dev = std::max(dev, d);
    }
    out->max_norm_dev = dev;
    return SOFT_OK;
}
}  // namespace

int soft_run_list(soft_ctx *c, const uint64_t *shots_dev, uint64_t n_shots, uint32_t *outcomes, uint32_t *status,
                  uint32_t *abort_op, uint32_t *obs, void *hip_stream) try {
    if (!c) return SOFT_EINVAL;
    if (!status && n_shots) return fail(c, SOFT_EINVAL, "status_dev is required");
    if (!shots_dev && n_shots) return fail(c, SOFT_EINVAL, "shots_dev is required");
    if (((uintptr_t)shots_dev & 7u) != 0) return fail(c, SOFT_EINVAL, "shots_dev must be 8-byte aligned");
    HIPCHK(c, hipSetDevice(c->device));
    int rc = prepare(c);
    if (rc) return rc;
    if (c->words_dev) return fail(c, SOFT_EUNSUPPORTED, "explicit words are for soft_run");
    if (n_shots == 0) return SOFT_OK;
    Shape s = current_shape(c, true);
    if ((rc = check_shape(c, s))) return rc;
    return run_impl(c, 0, n_shots, outcomes, status, abort_op, obs, (hipStream_t)hip_stream, s, shots_dev);
} SOFT_GUARD(c)

int soft_read_counters(soft_ctx *c, soft_counters *out) try {
    if (!c || !out) return fail(c, SOFT_EINVAL, "null argument");
    return read_rows(c, 0, c->last_vars, out);
} SOFT_GUARD(c)

int soft_read_variant_counters(soft_ctx *c, uint32_t variant, soft_counters *out) try {
    if (!c || !out) return fail(c, SOFT_EINVAL, "null argument");
    if (variant >= c->vars.size()) return fail(c, SOFT_EINVAL, "no such variant");
    return read_rows(c, variant, variant + 1, out);
} SOFT_GUARD(c)

int soft_read_coeffs(soft_ctx *c, uint64_t shot, uint64_t *alpha, double *re, double *im, uint32_t cap, uint32_t *count) try {
    if (!c || !count) return fail(c, SOFT_EINVAL, "null argument");
    HIPCHK(c, hipSetDevice(c->device));
    std::vector<unsigned long long> meta;
    std::vector<double> tile;
    int rc;
    const Frame *f = kept_frame(c, shot, meta, tile, rc);
    if (!f) return rc;
    return decode_coeffs(c, *f, meta, tile, alpha, re, im, cap, count);
} SOFT_GUARD(c)

int soft_read_tableau(soft_ctx *c, uint64_t shot, uint64_t *x, uint64_t *z, uint8_t *r) try {
    if (!c) return SOFT_EINVAL;
    HIPCHK(c, hipSetDevice(c->device));
    std::vector<unsigned long long> meta;
    std::vector<double> tile;
    int rc;
    const Frame *f = kept_frame(c, shot, meta, tile, rc);
    if (!f) return rc;
    decode_tableau(*f, meta, x, z, r);
    return SOFT_OK;
} SOFT_GUARD(c)

int soft_set_trace(soft_ctx *c, uint64_t shot, uint32_t steps) {
    if (!c) return SOFT_EINVAL;
    if (steps > 65536) return fail(c, SOFT_ECAPACITY, "at most 65536 traced steps");
    c->trace_shot = shot;
    c->trace_n = steps;
    return SOFT_OK;
}

int soft_read_trace(soft_ctx *c, uint32_t step, uint64_t info[6], uint64_t *x, uint64_t *z, uint8_t *r,
                    uint64_t *alpha, double *re, double *im, uint32_t cap, uint32_t *count) try {
    if (!c || !info) return fail(c, SOFT_EINVAL, "null argument");
    if (!c->ran || !c->trace_n || !c->trace_tile) return fail(c, SOFT_ESTATE, "no traced run");
    if (step >= c->trace_n) return fail(c, SOFT_EINVAL, "step beyond the traced range");
    HIPCHK(c, hipSetDevice(c->device));
    HIPCHK(c, hipStreamSynchronize(c->last_stream));
    std::vector<unsigned long long> meta(KM_COUNT);
    std::vector<double> tile((size_t)c->trace_tile * 2);
    HIPCHK(c, hipMemcpy(meta.data(), c->d_trace_meta.p + (uint64_t)step * KM_COUNT, KM_COUNT * sizeof(unsigned long long),
                        hipMemcpyDeviceToHost));
    for (int i = 0; i < 6; ++i) info[i] = 0;
    if (count) *count = 0;
    if (meta[KM_VALID] != kStateValid) return SOFT_OK;
    HIPCHK(c, hipMemcpy(tile.data(), c->d_trace_v.p + (uint64_t)step * c->trace_tile * 2, tile.size() * sizeof(double),
                        hipMemcpyDeviceToHost));
    int rc = SOFT_OK;
    const Frame *f = frame_of(c, meta, rc);
    if (!f) return rc;
    const Event &E = program_of(c, meta).events[meta[KM_TERM_EV]];
    info[0] = 1;
    info[1] = (meta[KM_STATUS] != ST_PASSED && meta[KM_ABORT] != 0xFFFFFFFFull) ? meta[KM_ABORT] : E.src;
    info[2] = meta[KM_STATUS];
    info[3] = meta[KM_K];
    info[4] = meta[KM_NRM2];
    info[5] = (meta[KM_STATUS] != ST_PASSED || E.kind == EV_END) ? 1 : 0;
    decode_tableau(*f, meta, x, z, r);
    uint32_t cnt = 0;
    rc = decode_coeffs(c, *f, meta, tile, alpha, re, im, cap, &cnt);
    if (count) *count = cnt;
    return rc;
} SOFT_GUARD(c)

namespace {
void program_info(const Program &P, uint64_t info[8]) {
    info[0] = (uint64_t)P.n;
    info[1] = P.n_rec;
    info[2] = P.n_noise;
    info[3] = P.n_meas;
    info[4] = P.n_obs;
    info[5] = P.events.size();
    info[6] = P.kmax;
    info[7] = (P.n_rec + 31u) / 32u;
}
}  // namespace

int soft_circuit_info(soft_ctx *c, uint64_t info[8]) try {
    if (!c || !info) return fail(c, SOFT_EINVAL, "null argument");
    (void)hipSetDevice(c->device);
    int rc = prepare(c);
    if (rc) return rc;
    for (int i = 0; i < 8; ++i) info[i] = 0;
    for (const Variant &V : c->vars) {
        uint64_t vi[8];
        program_info(V.prog, vi);
        for (int i = 0; i < 8; ++i) info[i] = std::max(info[i], vi[i]);
    }
    return SOFT_OK;
} SOFT_GUARD(c)

int soft_variant_info(soft_ctx *c, uint32_t variant, uint64_t info[8]) try {
    if (!c || !info) return fail(c, SOFT_EINVAL, "null argument");
    if (!c->have_text) return fail(c, SOFT_ESTATE, "no circuit loaded");
    if (variant >= c->vars.size()) return fail(c, SOFT_EINVAL, "no such variant");
    program_info(c->vars[variant].prog, info);
    return SOFT_OK;
} SOFT_GUARD(c)

int soft_graph_info(soft_ctx *c, uint64_t out[2]) {
    if (!c || !out) return fail(c, SOFT_EINVAL, "null argument");
    out[0] = 0;
    out[1] = c->launches;
    return SOFT_OK;
}

int soft_launch_shape(soft_ctx *c, uint32_t out[5]) try {
    if (!c || !out) return fail(c, SOFT_EINVAL, "null argument");
    (void)hipSetDevice(c->device);
    int rc = prepare(c);
    if (rc) return rc;
    Shape s = current_shape(c);
    out[0] = s.wpb;
    out[1] = s.bpc;
    out[2] = s.grab;
    out[3] = wave_bytes(c, s);
    out[4] = s.gt;
    return SOFT_OK;
} SOFT_GUARD(c)

int soft_autotune(soft_ctx *c, uint64_t sample_shots, void *hip_stream) try {
    if (!c) return SOFT_EINVAL;
    if (sample_shots == 0) return fail(c, SOFT_EINVAL, "sample_shots must be > 0");
    HIPCHK(c, hipSetDevice(c->device));
    int rc = prepare(c);
    if (rc) return rc;
    if (c->words_dev) return fail(c, SOFT_ESTATE, "autotune runs on Philox draws; clear explicit uniforms first");
    hipStream_t st = (hipStream_t)hip_stream;
    TuneScope T(c, st);
    // The sample: the first shots of each variant's range, sample_shots in all,
    // as one shot list so that every timing is a single launch.  Runs that take
    // the sign pass, which lists do not, are timed with the variants' ranges
    // shortened to the same numbers of shots.
    std::vector<uint64_t> list;
    std::vector<uint64_t> ends;
    {
        const uint64_t per = std::max<uint64_t>(1, sample_shots / c->vars.size());
        uint64_t lo = 0;
        for (const Variant &V : c->vars) {
            const uint64_t n = std::min<uint64_t>(per, V.shot_end - lo);
            for (uint64_t i = 0; i < n; ++i) list.push_back(lo + i);
            ends.push_back(list.size());
            lo = V.shot_end;
        }
    }
    const size_t nv = c->vars.size();
    HIPCHK(c, hipMalloc((void **)&T.status, list.size() * sizeof(uint32_t)));
    HIPCHK(c, hipMalloc((void **)&T.list, list.size() * sizeof(uint64_t)));
    HIPCHK(c, hipMemcpy(T.list, list.data(), list.size() * sizeof(uint64_t), hipMemcpyHostToDevice));
    {
        std::vector<VariantDesc> vd(nv);
        HIPCHK(c, hipMemcpy(vd.data(), c->d_vars.p, nv * sizeof(VariantDesc), hipMemcpyDeviceToHost));
        for (size_t v = 0; v < nv; ++v) vd[v].shot_end = ends[v];
        HIPCHK(c, hipMalloc((void **)&T.vars, nv * sizeof(VariantDesc)));
        HIPCHK(c, hipMemcpy(T.vars, vd.data(), nv * sizeof(VariantDesc), hipMemcpyHostToDevice));
    }
    HIPCHK(c, hipEventCreate(&T.t0));
    HIPCHK(c, hipEventCreate(&T.t1));
    auto sample_pass = [&](const Shape &s, bool by_list) {
        return by_list ? run_impl(c, 0, list.size(), nullptr, T.status, nullptr, nullptr, st, s, T.list)
                       : run_impl(c, 0, list.size(), nullptr, T.status, nullptr, nullptr, st, s, nullptr, T.vars);
    };
    // Each candidate is run once untimed and twice timed; the faster timing
    // counts, so one noisy launch cannot pick a worse shape than the default.
    auto tune = [&](bool by_list) {
        const std::vector<Shape> cands = shape_candidates(c, by_list);
        Shape best = cands[0];
        float best_ms = 1e30f;
        for (size_t i = 0; i < cands.size(); ++i) {
            const Shape &sh = cands[i];
            if (check_shape(c, sh) != SOFT_OK) continue;
            int e = sample_pass(sh, by_list);  // untimed: caches
            float ms = 1e30f;
            for (int rep = 0; rep < 2 && !e; ++rep) {
                float t = 0.0f;
                HIPCHK(c, hipEventRecord(T.t0, st));
                if ((e = sample_pass(sh, by_list))) break;
                HIPCHK(c, hipEventRecord(T.t1, st));
                HIPCHK(c, hipEventSynchronize(T.t1));
                HIPCHK(c, hipEventElapsedTime(&t, T.t0, T.t1));
                ms = std::min(ms, t);
            }
            if (e) return e;
            if (ms < best_ms) {
                best_ms = i == 0 && !by_list ? kTuneGain * ms : ms;
                best = sh;
            }
        }
        std::lock_guard<std::mutex> lock(g_tune_mu);
        g_tuned[tune_key(c, by_list)] = best;
        return (int)SOFT_OK;
    };
    if ((rc = tune(true))) return rc;
    if (use_signs(c, false) && (rc = tune(false))) return rc;
    c->ran = false;  // counters of the last sample run are not a user run
    return SOFT_OK;
} SOFT_GUARD(c)

}  // extern "C"
