// signs.cpp -- the sign program of an event list (program.h).
//
// Two passes over the list.  Forward, on the noiseless shot's signs: the
// reference values, the tests in list order and what each one's shot has
// written.  Backward: for every sign bit (d_i, s_i, and bit i of the offset a)
// the vector of everything that flipping it now changes later, so a noise
// slot's signature is the XOR over the rows its Pauli anticommutes with.
#include "signs.h"

#include <algorithm>
#include <cmath>

namespace soft {
namespace {

// Limits of the tables (the kernel's largest vector) and of the coins a shot
// draws up front.
constexpr uint32_t kMaxTestWords = 16, kMaxOutWords = 16, kMaxCoins = 256;

typedef std::vector<uint32_t> Vec;

inline uint32_t par64(uint64_t w) { return (uint32_t)__builtin_parityll(w); }

void add(uint32_t *a, const uint32_t *b, size_t n) {
    for (size_t i = 0; i < n; ++i) a[i] ^= b[i];
}
void add(Vec &a, const Vec &b) { add(a.data(), b.data(), a.size()); }
void flip(Vec &a, uint32_t bit) { a[bit >> 5] ^= 1u << (bit & 31u); }

// The signs' rows as vectors: what flipping row i changes from here on.
struct Rows {
    std::vector<Vec> D, S, A;
    Rows(uint32_t w) : D(64, Vec(w)), S(64, Vec(w)), A(64, Vec(w)) {}
    void sum(uint32_t *v, uint64_t d, uint64_t s) const {
        for (; d; d &= d - 1) add(v, D[__builtin_ctzll(d)].data(), D[0].size());
        for (; s; s &= s - 1) add(v, S[__builtin_ctzll(s)].data(), S[0].size());
    }
    void sum(Vec &v, uint64_t d, uint64_t s) const { sum(v.data(), d, s); }
    // a value read as parity(rD & beta) ^ parity(rS & gamma), and with
    // `entry` parity(a & gamma), changes v
    void read(uint64_t beta, uint64_t gamma, bool entry, const Vec &v) {
        for (; beta; beta &= beta - 1) add(D[__builtin_ctzll(beta)], v);
        for (; gamma; gamma &= gamma - 1) {
            add(S[__builtin_ctzll(gamma)], v);
            if (entry) add(A[__builtin_ctzll(gamma)], v);
        }
    }
};

// The list's events that read no coefficient: all up to the first random
// measurement other than a coin, or a condition that is no XOR of record bits.
bool stops(const Event &E) {
    return E.kind == EV_M_CUT || E.kind == EV_M_MERGE ||
           (E.kind == EV_FEEDBACK && (E.flags & EVF_AND));
}

struct Test {
    uint32_t ev;
    int pair;  // index of the T pair, or -1 (a check, or the stop)
};

}  // namespace

void build_signs(const Program &P, SignProgram &out) {
    out = SignProgram();
    const uint32_t n = (uint32_t)P.events.size();
    uint32_t last = 0;  // the event the signs stop at
    while (last < n && P.events[last].kind != EV_END && !stops(P.events[last])) ++last;
    if (last >= n) return;
    // past the limits nothing below is worth its time: a list has a test mask
    // of all record words for each of its tests
    const uint32_t rw = (P.n_rec + 31u) / 32u;
    if (rw + 1u > kMaxOutWords) return;
    out.complete = P.events[last].kind == EV_END;
    std::vector<uint32_t> flip_of(P.n_rec, kNone);  // the noise slot that flips a record
    for (uint32_t s = 0; s < P.n_noise; ++s) {
        const NoiseLoc &L = P.noise[s];
        if (L.kind != NZ_FLIP) continue;
        if (flip_of[L.rec] != kNone) return;  // (a record has one)
        flip_of[L.rec] = s;
    }
    auto is_t = [](const Event &E) { return E.kind == EV_T_PHASE || E.kind == EV_T_DOUBLE || E.kind == EV_T_BFLY; };

    // ---- pairs by closing event ----
    std::vector<int> closes(n, -1);
    for (size_t i = 0; i < P.pairs.size(); ++i) {
        const TPair &T = P.pairs[i];
        if (T.close >= last) continue;
        const Event &o = P.events[T.open], &c = P.events[T.close];
        if (o.beta != c.beta || o.gamma != c.gamma || ((o.cexp ^ c.cexp) & 1u)) return;
        // a pair diagonal on a single entry is a global phase
        if (o.beta == 0 && T.k0 == 0) continue;
        closes[T.close] = (int)i;
    }

    // ---- forward: the tests, and the noiseless values ----
    uint64_t rD = 0, rS = 0, a = 0;
    std::vector<uint32_t> rec(P.n_rec, 0);
    std::vector<uint32_t> sign_of(n, 0);  // T events: quarter turns of c
    std::vector<Test> tests;
    std::vector<uint32_t> ref_bits;       // of the tests
    std::vector<Vec> mask;
    Vec written(rw + 1u, 0u);             // records and observables so far
    uint32_t obs = 0, ne = 0;
    auto parity = [&](const Event &E) {
        uint32_t v = E.expect;
        for (uint32_t t = 0; t < E.det_cnt; ++t) {
            const uint32_t w = P.det_pairs[2u * (E.det_off + t)];
            for (uint32_t m = P.det_pairs[2u * (E.det_off + t) + 1u]; m; m &= m - 1u)
                v ^= rec[32u * w + (uint32_t)__builtin_ctz(m)];
        }
        return v & 1u;
    };
    auto add_test = [&](uint32_t e, int pair, uint32_t ref, uint32_t kind, uint32_t src) {
        tests.push_back(Test{e, pair});
        ref_bits.push_back(ref);
        mask.push_back(written);
        out.tests.push_back(SignTest{P.events[e].noise_end, src, kind, 0u});
    };
    // A pair can be followed by signs when the bracket started and ends on one
    // entry: its closing layer leaves an empty span.
    auto follows = [&](const TPair &T) {
        if (T.k0 != 0 || P.events[T.close].beta == 0 || out.pairs.size() >= kMaxSignPairs) return false;
        uint32_t e = T.close;
        while (e < last && (is_t(P.events[e]) || P.events[e].kind == EV_DROP)) ++e;
        return P.before[e].basis.empty();
    };
    for (uint32_t e = 0; e <= last; ++e) {
        const Event &E = P.events[e];
        if (E.noise_end < ne) return;  // (slots come in list order)
        ne = E.noise_end;
        if (tests.size() > 32u * kMaxTestWords || out.coin_slot.size() > kMaxCoins) return;
        if (e == last) {
            if (!out.complete) add_test(e, -1, 1u, SGT_HAND, 0u);
            break;
        }
        rD ^= E.cliffD;
        rS ^= E.cliffS;
        const uint32_t sga = par64((rD & E.beta) ^ ((rS ^ a) & E.gamma));
        switch (E.kind) {
            case EV_T_PHASE: case EV_T_DOUBLE: case EV_T_BFLY:
                // (the gate's own sign: what `a` adds is the entry's)
                sign_of[e] = (E.cexp + 2u * par64((rD & E.beta) ^ (rS & E.gamma))) & 3u;
                if (closes[e] >= 0) {
                    const TPair &T = P.pairs[closes[e]];
                    const bool f = follows(T);
                    add_test(e, closes[e], sign_of[e] != sign_of[T.open], f ? SGT_PAIR : SGT_HAND, 0u);
                    if (f) {
                        out.tests.back().pair = (uint32_t)out.pairs.size();
                        out.pairs.push_back(SignPair{E.beta, (uint32_t)out.pairs.size(), (uint32_t)out.meas.size()});
                    }
                }
                break;
            case EV_M_DET: case EV_M_SPLIT: {
                uint32_t bit = (E.cexp == 2u ? 1u : 0u) ^ sga;
                if (E.kind == EV_M_SPLIT || E.gamma) {
                    const bool ok = E.kind == EV_M_DET && (E.flags & EVF_RECORD);
                    out.meas.push_back(SignMeas{E.kind == EV_M_DET ? E.gamma : ~0ull, E.noise_end, (uint32_t)tests.size(),
                                                E.mslot, ok ? E.rec : kNone, ok ? flip_of[E.rec] : kNone, 0u});
                }
                if (E.kind == EV_M_SPLIT) {
                    bit = 0u;  // the coin's 0; its 1 is one more vector
                    const uint32_t p = E.pbit;
                    const uint64_t b = (rS >> p) & 1ull;
                    rD ^= (b ? E.AD : 0ull) ^ E.PhD;
                    rS ^= (b ? E.AS : 0ull) ^ E.PhS;
                    rD = (rD & ~(1ull << p)) | (b << p);
                    rS = (rS & ~(1ull << p)) | ((uint64_t)(bit ^ E.psign) << p);
                    if ((a >> p) & 1ull) a ^= E.beta;
                    out.coin_slot.push_back(E.mslot);
                }
                if (E.flags & EVF_RECORD) {
                    rec[E.rec] ^= bit;
                    written[E.rec >> 5] |= 1u << (E.rec & 31u);
                }
                if ((E.flags & EVF_RESET) && bit) {
                    rD ^= E.xD;
                    rS ^= E.xS;
                }
                if (E.flags & EVF_CHECK) add_test(e, -1, parity(E), SGT_CHECK, E.chk_src);
                break;
            }
            case EV_DETECTOR: add_test(e, -1, parity(E), SGT_CHECK, E.src); break;
            case EV_OBSERVABLE:
                obs |= parity(E) << E.rec;
                written[rw] |= 1u << E.rec;
                break;
            case EV_FEEDBACK:
                if (parity(E)) {
                    rD ^= E.xD;
                    rS ^= E.xS;
                }
                break;
            default: break;  // T, DROP and diagonal gates leave the signs alone
        }
    }
    for (SignPair &S : out.pairs)  // so far: the first measurement after the pair
        while (S.meas < out.meas.size() && out.meas[S.meas].gamma != ~0ull && !par64(out.meas[S.meas].gamma & S.beta))
            ++S.meas;
    const uint32_t nt = (uint32_t)tests.size(), tw = (nt + 31u) / 32u;
    if (tw > kMaxTestWords || out.coin_slot.size() > kMaxCoins) return;
    if ((uint64_t)P.n_noise * kSignVecs * (tw + rw + 1u) * sizeof(uint32_t) > kMaxSignBytes) return;
    out.tests.push_back(SignTest{P.n_noise, 0xFFFFFFFFu, SGT_NONE, 0u});
    mask.push_back(written);
    out.mask.swap(mask);
    out.need.tests = tw;
    out.need.recs = rw;
    // bit positions: tests, records, observables
    const uint32_t R0 = 32u * tw, O0 = R0 + 32u * rw, W = tw + rw + 1u;
    out.ref.assign(W, 0u);
    for (uint32_t t = 0; t < nt; ++t)
        if (ref_bits[t]) flip(out.ref, t);
    for (uint32_t r = 0; r < P.n_rec; ++r)
        if (rec[r]) flip(out.ref, R0 + r);
    out.ref[W - 1u] = obs;

    // ---- backward: what each row, record bit and noise slot changes ----
    Rows F(W);
    std::vector<Vec> RS(P.n_rec, Vec(W));
    for (uint32_t r = 0; r < P.n_rec; ++r) flip(RS[r], R0 + r);
    out.slots.assign(P.n_noise, SignSlot{NZ_NONE, 0u, 0u, 0u});
    out.vecs.assign((size_t)P.n_noise * kSignVecs * W, 0u);
    auto to_records = [&](const Event &E, const Vec &v) {
        for (uint32_t t = 0; t < E.det_cnt; ++t) {
            const uint32_t w = P.det_pairs[2u * (E.det_off + t)];
            for (uint32_t m = P.det_pairs[2u * (E.det_off + t) + 1u]; m; m &= m - 1u)
                add(RS[32u * w + (uint32_t)__builtin_ctz(m)], v);
        }
    };
    auto unit = [&](uint32_t bit) {
        Vec v(W);
        flip(v, bit);
        return v;
    };
    std::vector<Vec> open_at(n);  // opening T events: tests that read their sign
    out.coin.assign(out.coin_slot.size(), Vec());
    out.pair_vecs.assign(out.pairs.size(), Vec());
    uint32_t t = nt, c = (uint32_t)out.coin_slot.size();
    for (uint32_t e = last + 1u; e-- > 0;) {
        const Event &E = P.events[e];
        if (e == last) {
            if (!out.complete) --t;  // the stop: always set, nothing flips it
        } else {
            switch (E.kind) {
                case EV_T_PHASE: case EV_T_DOUBLE: case EV_T_BFLY:
                    if (closes[e] >= 0) {
                        const Vec v = unit(--t);
                        if (out.tests[t].kind == SGT_PAIR) {
                            Vec &u = out.pair_vecs[out.tests[t].pair];
                            u.assign(W, 0u);
                            for (uint64_t b = E.beta; b; b &= b - 1) add(u, F.A[__builtin_ctzll(b)]);
                        }
                        F.read(E.beta, E.gamma, false, v);
                        open_at[P.pairs[closes[e]].open] = v;
                    }
                    if (!open_at[e].empty()) F.read(E.beta, E.gamma, false, open_at[e]);
                    break;
                case EV_M_DET: case EV_M_SPLIT: {
                    if (E.flags & EVF_CHECK) to_records(E, unit(--t));
                    Vec v(W);  // what the outcome changes
                    if (E.flags & EVF_RECORD) add(v, RS[E.rec]);
                    if (E.flags & EVF_RESET) F.sum(v, E.xD, E.xS);
                    if (E.kind == EV_M_DET) {
                        F.read(E.beta, E.gamma, true, v);
                        break;
                    }
                    // d_p <- s_p (absorbed by the rows AD, AS), s_p <- the
                    // coin, a <- a ^ beta when bit p of a is set
                    const uint32_t p = E.pbit;
                    add(v, F.S[p]);
                    out.coin[--c] = v;
                    Vec sp(W), ap(W);
                    F.sum(sp, E.AD, E.AS);
                    add(sp, F.D[p]);
                    for (uint64_t b = E.beta & ~(1ull << p); b; b &= b - 1) add(ap, F.A[__builtin_ctzll(b)]);
                    F.D[p].assign(W, 0u);
                    F.S[p] = sp;
                    F.A[p] = ap;
                    break;
                }
                case EV_DETECTOR: to_records(E, unit(--t)); break;
                case EV_OBSERVABLE: to_records(E, unit(O0 + E.rec)); break;
                case EV_FEEDBACK: {
                    Vec v(W);
                    F.sum(v, E.xD, E.xS);
                    to_records(E, v);
                    break;
                }
                default: break;
            }
        }
        // the slots between the event before and this one
        for (uint32_t s = e ? P.events[e - 1u].noise_end : 0u; s < E.noise_end; ++s) {
            const NoiseLoc &L = P.noise[s];
            SignSlot &Q = out.slots[s];
            Q.kind = L.kind;
            Q.thr1 = L.thr ? (uint32_t)(L.thr - 1ull) : 0u;
            Q.acc1 = L.acc ? (uint32_t)(L.acc - 1ull) : 0u;
            if (L.kind == NZ_NONE) continue;
            uint32_t *g = &out.vecs[(size_t)s * kSignVecs * W];
            if (L.kind == NZ_FLIP) {
                add(g, RS[L.rec].data(), W);
                continue;
            }
            for (uint32_t q = 0; q < (L.kind == NZ_DEP2 ? 2u : 1u); ++q, g += 3u * W) {
                const uint64_t *m = L.masks + 4u * q;
                F.sum(g, m[0], m[1]);
                F.sum(g + 2u * W, m[2], m[3]);
                add(g + W, g, W);
                add(g + W, g + 2u * W, W);
            }
        }
    }

    // checkpoints that precede each slot
    for (uint32_t s = 0; s < P.n_noise; ++s)
        for (const Checkpoint &k : P.ckpts) out.slots[s].ckpt += k.nz <= s ? 1u : 0u;

    // ---- how many shots a check ends: hits whose signature has a check, and
    // coins (independent ones halve the shots that go on) ----
    Vec checks(W), pairs(W);
    bool any = false;
    for (uint32_t i = 0; i < nt; ++i) {
        if (out.tests[i].kind == SGT_CHECK) {
            flip(checks, i);
            any = any || ((out.ref[i >> 5] >> (i & 31u)) & 1u);
        } else if (tests[i].pair >= 0) {
            flip(pairs, i);
        }
    }
    double lam = 0.0;
    for (uint32_t s = 0; s < P.n_noise; ++s) {
        const uint32_t kind = out.slots[s].kind;
        if (kind == NZ_NONE) continue;
        const uint32_t *g = &out.vecs[(size_t)s * kSignVecs * W];
        uint32_t bad = 0, broken = 0, all = 1;
        auto count = [&](uint32_t a, uint32_t b) {  // Paulis 1..3 (0: none) on the two qubits
            uint32_t c = 0, p = 0;
            for (uint32_t i = 0; i < tw; ++i) {
                const uint32_t v = (a ? g[(a - 1u) * W + i] : 0u) ^ (b ? g[(2u + b) * W + i] : 0u);
                c |= v & checks[i];
                p |= v & pairs[i];
            }
            bad += c ? 1u : 0u;
            broken += p ? 1u : 0u;
        };
        if (kind == NZ_DEP1) {
            all = 3;
            for (uint32_t a = 1; a < 4u; ++a) count(a, 0u);
        } else if (kind == NZ_DEP2) {
            all = 15;
            for (uint32_t i = 1; i < 16u; ++i) count(i >> 2, i & 3u);
        } else {
            count(kind == NZ_ZERR ? 3u : 1u, 0u);
        }
        lam -= std::log1p(-std::min(P.noise_p[s] * bad / all, 1.0 - 1e-12));
        out.breaks += P.noise_p[s] * broken / all;
    }
    std::vector<Vec> ech;
    for (Vec v : out.coin) {
        for (size_t i = 0; i < W; ++i) v[i] &= checks[i];
        for (const Vec &r : ech) {
            size_t w = W;
            while (w-- > 0 && !r[w]) {}
            if (v[w] & (1u << (31 - __builtin_clz(r[w])))) add(v, r);
        }
        if (std::any_of(v.begin(), v.end(), [](uint32_t x) { return x != 0u; })) ech.push_back(v);
    }
    out.ends = any ? 1.0 : 1.0 - std::exp(-lam - std::log(2.0) * (double)ech.size());
    out.on = true;
}

}  // namespace soft
