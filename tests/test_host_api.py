"""The host side of the C ABI (soft_api.cpp) on the CPU, against a device that
is host memory: kernels are recorded instead of run, device allocations are
heap blocks under AddressSanitizer.  What it shows is about lifetimes, ranges,
routes and errors: that the addresses a recorded launch holds stay allocated and
unchanged, that reads stay within the counters, which launches a call makes, and
that a failing allocation is an error code.
"""
from __future__ import annotations

import os
import subprocess

import pytest

import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_23037_amd", "csrc")

DRIVER = r"""
#include <hip/hip_runtime.h>
#include "sampler.h"
#include "soft.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <map>
#include <new>
#include <sstream>
#include <string>
#include <vector>
using namespace soft;

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)
#define OK(x) do { int rc_ = (x); if (rc_) { std::printf("line %d: %s = %d: %s\n", __LINE__, #x, rc_, soft_last_error(g_ctx)); std::exit(1); } } while (0)

static soft_ctx *g_ctx = nullptr;

// ---- host allocations that fail on demand ----
static long g_new_left = -1;  // allocations until they fail (-1: never)
static void *take(size_t n) {
    if (g_new_left == 0) throw std::bad_alloc();
    if (g_new_left > 0) --g_new_left;
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(size_t n) { return take(n); }
void *operator new[](size_t n) { return take(n); }
void *operator new(size_t n, const std::nothrow_t &) noexcept { return std::malloc(n ? n : 1); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete[](void *p, size_t) noexcept { std::free(p); }
void operator delete(void *p, const std::nothrow_t &) noexcept { std::free(p); }

// ---- the device ----
struct Block { size_t n; };
static std::map<void *, size_t> g_live;
static bool g_capture = false, g_log = true;
static int g_clock = 0;
struct Launch {
    char what;  // r reset, b build, g signs, s sampler, c clear
    RunParams p;
    SignParams sp;
    uint32_t grid, block;
    int events;  // event records before it
    bool captured;
};
static std::vector<Launch> g_launches;
static int g_syncs = 0;
template <typename... A> static void log(char what, const RunParams *p, const SignParams *sp, dim3 g, dim3 b) {
    if (!g_log) return;
    const long left = g_new_left;
    g_new_left = -1;
    Launch L;
    std::memset((void *)&L, 0, sizeof(L));
    L.what = what;
    if (p) L.p = *p;
    if (sp) L.sp = *sp;
    L.grid = g.x;
    L.block = b.x;
    L.events = g_clock;
    L.captured = g_capture;
    g_launches.push_back(L);
    g_new_left = left;
}
extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { std::memset((void *)p, 0, sizeof(*p)); std::strcpy(p->gcnArchName, "gfx950"); return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
    if (g_capture) return hipErrorStreamCaptureUnsupported;
    const long left = g_new_left;
    g_new_left = -1;
    *p = std::malloc(n);
    g_live[*p] = n;
    g_new_left = left;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (p && !g_live.erase(p)) { std::printf("free of unknown memory\n"); std::exit(1); }
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { if (g_capture) { std::printf("memset recorded\n"); std::exit(1); } std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++g_syncs; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)std::malloc(8); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { ++g_clock; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
// each timing takes g_step times the one before it
static float g_ms = 1.0f, g_step = 1.001f;
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = g_ms *= g_step; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "hip error"; }
}
namespace soft {
hipError_t launch_reset(unsigned long long *c, uint32_t n, unsigned long long *next, hipStream_t) {
    RunParams p;
    std::memset((void *)&p, 0, sizeof(p));
    p.counters = c;
    p.next = next;
    log('r', &p, nullptr, dim3(1), dim3(1));
    if (!g_capture) std::memset(c, 0, n * 8ull);
    return hipSuccess;
}
hipError_t launch_clear(unsigned long long *c, uint64_t n, hipStream_t) {
    RunParams p;
    std::memset((void *)&p, 0, sizeof(p));
    p.counters = c;
    log('c', &p, nullptr, dim3(1), dim3(1));
    if (!g_capture) std::memset(c, 0, n * 8ull);
    return hipSuccess;
}
hipError_t launch_sampler(const RunParams &p, bool, dim3 g, dim3 b, size_t, hipStream_t) {
    log('s', &p, nullptr, g, b);
    if (!g_capture)  // every row counts one shot
        for (uint32_t r = 0; r < p.n_vars * p.shards; ++r) p.counters[(size_t)r * C_COUNT + C_SHOTS] += 1;
    return hipSuccess;
}
hipError_t launch_prefix_build(const RunParams &p, bool, dim3 g, dim3 b, size_t, hipStream_t) { log('b', &p, nullptr, g, b); return hipSuccess; }
hipError_t launch_signs(const SignParams &p, uint32_t, bool, dim3 g, hipStream_t) { log('g', nullptr, &p, g, dim3(64)); return hipSuccess; }
bool sampler_lean(const RunParams &p) { return !p.keep_n && !p.trace_n && p.support_cap == 0xFFFFFFFFu && !p.shot_list && !p.words; }
hipError_t sampler_occupancy(bool, uint32_t, uint32_t, int block, size_t lds, int *n) {
    *n = (int)std::min<size_t>(20u / (block / 64), 160u * 1024u / std::max<size_t>(lds, 1));
    return hipSuccess;
}
hipError_t sampler_set_lds_limit(int) { return hipSuccess; }
static unsigned char g_scratch[kScratchBytes];
hipError_t scratch_address(int, unsigned char **p) { *p = g_scratch; return hipSuccess; }
}

// Every device address of the recorded launches still holds what it held.
static std::map<const void *, unsigned char> g_held;
static void hold(const void *p) { if (p) g_held[p] = *(const volatile unsigned char *)p; }
static size_t replay(bool record) {
    size_t n = 0;
    for (const Launch &L : g_launches) {
        if (!L.captured) continue;
        ++n;
        const RunParams &p = L.p;
        const SignParams &s = L.sp;
        // tables: allocated and not rewritten; work buffers: allocated
        const void *tables[] = {p.ev, p.nz, p.tm1, p.det, p.bm, p.diag, p.ckpts, p.gaps, p.vars, s.desc, s.vars, s.vecs,
                                s.slots, s.tests, s.mask, s.coins, s.pairs, s.meas, s.tm1, s.gaps};
        for (const void *t : tables) {
            if (!t) continue;
            if (record) hold(t);
            CHECK(*(const volatile unsigned char *)t == g_held[t]);
        }
        void *work[] = {p.gtile, p.prefix, p.keep_meta, p.keep_v, p.trace_meta, p.trace_v, p.counters, p.next, s.counters};
        for (void *w : work)
            if (w) *(volatile unsigned char *)w = *(volatile unsigned char *)w;
        if (p.prefix && p.prefix_stride) *(volatile unsigned char *)(p.prefix + p.prefix_stride - 1) = 1;
    }
    return n;
}
static std::string read(const char *f) { std::ifstream i(f); std::stringstream s; s << i.rdbuf(); return s.str(); }
static std::string kinds(size_t from = 0) {
    std::string k;
    for (size_t i = from; i < g_launches.size(); ++i) k += g_launches[i].what;
    return k;
}

int main(int argc, char **argv) {
    const std::string what = argv[1], big = read(argv[2]), small = read(argv[3]);
    const soft_noise nm = {1e-3, 1e-3, 1e-3, 1e-3, 1e-3, 1e-3};
    soft_ctx *c = nullptr;
    OK(soft_create(&c, 0));
    g_ctx = c;
    std::vector<uint32_t> st(4096);
    OK(soft_load_noise(c, &nm));
    auto load = [&](const std::string &t) { OK(soft_load_circuit(c, t.c_str(), t.size())); };
    auto mixture = [&](uint32_t n) {
        const long left_for_the_call = g_new_left;
        g_new_left = -1;
        std::vector<const char *> t(n, small.c_str());
        std::vector<size_t> l(n, small.size());
        std::vector<soft_noise> m(n, nm);
        std::vector<uint64_t> e;
        for (uint32_t v = 0; v < n; ++v) e.push_back(100 * (v + 1));
        g_new_left = left_for_the_call;
        return soft_load_mixture(c, n, t.data(), l.data(), m.data(), e.data());
    };
    if (what == "capture") {
        const bool noalloc = std::string(argv[4]) == "noalloc";
        const int tiles = std::atoi(argv[5]);
        load(big);
        OK(soft_set_precision(c, 32));
        OK(soft_set_noise_mode(c, 1));
        OK(soft_set_tile_memory(c, tiles));
        auto run = [&](uint64_t n) { OK(soft_run(c, 0, n, nullptr, st.data(), nullptr, nullptr, nullptr)); };
        if (tiles == 2) {
            // a buffer that a recording names stays beside the larger one, one
            // that none does is freed
            run(100);
            g_capture = true;
            if (noalloc) OK(soft_run_noalloc(c, 0, 100, nullptr, st.data(), nullptr, nullptr, nullptr));
            else run(100);
            g_capture = false;
            if (!noalloc) run(100);  // (eager checkpoint slots again)
            const size_t blocks = g_live.size();
            run(1000000);
            CHECK(g_live.size() == blocks + (noalloc ? 0 : 1));
            run(3000000);
            CHECK(g_live.size() == blocks + (noalloc ? 0 : 1));
            g_launches.clear();
        }
        auto record = [&](uint64_t n) {
            run(n);
            g_capture = true;
            if (noalloc) OK(soft_run_noalloc(c, 0, n, nullptr, st.data(), nullptr, nullptr, nullptr));
            else run(n);
            g_capture = false;
            CHECK(replay(true) > 0);
        };
        record(100);
        OK(soft_set_precision(c, 64));
        run(1000000);
        CHECK(replay(false));
        record(200);
        run(1000000);
        replay(false);
        for (const std::string *t : {&small, &big, &small}) {
            load(*t);
            run(500000);
            replay(false);
        }
        OK(mixture(20));
        if (!noalloc) OK(soft_set_keep(c, 0, 50));
        run(1000);
        record(1000);
        if (!noalloc) OK(soft_set_keep(c, 0, 500));
        run(1000);
        replay(false);
        load(big);
        run(1000);
        replay(false);
        // states stay between runs that no capture records
        g_launches.clear();
        OK(soft_set_keep(c, 0, 0));
        run(1000);
        run(1000);
        CHECK(kinds().find('b') == std::string::npos);
    } else if (what == "counters") {
        const uint32_t rows_of[] = {1, 64, 3, 27};
        for (uint32_t ran : rows_of) {
            if (ran == 1) load(small);
            else OK(mixture(ran));
            OK(soft_run(c, 0, 100, nullptr, st.data(), nullptr, nullptr, nullptr));
            soft_counters k;
            OK(soft_read_counters(c, &k));
            const uint64_t all = k.shots;
            CHECK(all > 0 && all % ran == 0);
            for (uint32_t now : rows_of) {
                if (now == 1) load(small);
                else OK(mixture(now));
                OK(soft_read_counters(c, &k));
                CHECK(k.shots == all);
                for (uint32_t v = 0; v < now; ++v) {
                    OK(soft_read_variant_counters(c, v, &k));
                    CHECK(k.shots == (v < ran ? all / ran : 0));
                }
                CHECK(soft_read_variant_counters(c, now, &k) == SOFT_EINVAL);
            }
        }
    } else if (what == "memory") {
        // every host allocation of a call fails once: an error code, and the
        // context goes on
        g_log = false;
        auto each = [&](auto call) {
            long k = 0;
            for (;; k += k < 200 ? 1 : k / 17) {
                g_new_left = k;
                const int rc = call();
                const bool done = g_new_left > 0;
                g_new_left = -1;
                CHECK(rc == SOFT_OK || rc == SOFT_ECAPACITY);
                if (done) {
                    CHECK(rc == SOFT_OK);
                    break;
                }
            }
            return k;
        };
        CHECK(each([&]() { return soft_load_circuit(c, small.c_str(), small.size()); }) > 100);
        CHECK(each([&]() { return soft_load_noise(c, &nm); }) > 100);
        each([&]() { return mixture(3); });
        load(small);
        each([&]() { return soft_run(c, 0, 1000, nullptr, st.data(), nullptr, nullptr, nullptr); });
        each([&]() { return soft_run_noalloc(c, 0, 1000, nullptr, st.data(), nullptr, nullptr, nullptr); });
        soft_counters k;
        each([&]() { return soft_read_counters(c, &k); });
        uint32_t shape[5];
        each([&]() { return soft_launch_shape(c, shape); });
        g_log = true;
        load(small);
        OK(soft_run(c, 0, 1000, nullptr, st.data(), nullptr, nullptr, nullptr));
        CHECK(kinds() == "brgs");
    }
    else if (what == "autotune") {
        // runs that take the sign pass are tuned with it, over the variants'
        // first shots, and keep a shape of their own
        OK(soft_set_noise_mode(c, 1));
        OK(soft_set_precision(c, 64));
        const bool single = std::atoi(argv[4]) == 1;
        if (single) load(big);
        else OK(mixture(8));
        auto shape = [&](bool list) {  // grid, waves a block, tile placement of a run
            g_launches.clear();
            std::vector<uint64_t> which(800);
            for (size_t i = 0; i < which.size(); ++i) which[i] = i;
            if (list) OK(soft_run_list(c, which.data(), 800, nullptr, st.data(), nullptr, nullptr, nullptr));
            else OK(soft_run(c, 0, 800, nullptr, st.data(), nullptr, nullptr, nullptr));
            const Launch &L = g_launches.back();
            CHECK(L.what == 's' && (kinds().find('g') != std::string::npos) != list);
            CHECK((L.p.shot_list != nullptr) == list);
            return std::vector<uint32_t>{L.grid, L.block, L.p.tile_mode, L.p.lds_entries};
        };
        const auto run0 = shape(false), list0 = shape(true);
        // timings that get slower: the default stays, for each route
        g_launches.clear();
        OK(soft_autotune(c, 800, nullptr));
        size_t with = 0, without = 0;
        std::vector<uint32_t> first;
        for (size_t i = 0; i < g_launches.size(); ++i) {
            const Launch &L = g_launches[i];
            if (L.what != 's') continue;
            const bool signs = g_launches[i - 1].what == 'g';
            CHECK(signs == (L.p.shot_list == nullptr) && signs == (L.p.signs != 0));
            if (signs && first.empty()) first = {L.grid, L.block, L.p.tile_mode, L.p.lds_entries};
            (signs ? with : without)++;
            CHECK(L.p.n_shots == 800);
            if (signs && !single) {
                CHECK(g_launches[i - 1].sp.vars == L.p.vars);
            }
        }
        CHECK(with >= 30 && without >= 30 && first == run0);
        CHECK(shape(false) == run0 && shape(true) == list0);
        // a gain within the noise of a timing: the default stays where the pass runs
        g_step = 0.99995f;
        OK(soft_autotune(c, 800, nullptr));
        CHECK(shape(false) == run0 && shape(true) != list0);
        // timings that get faster: the last candidate of each route
        g_step = 0.99f;
        g_ms = 1.0f;
        OK(soft_autotune(c, 800, nullptr));
        const auto run1 = shape(false), list1 = shape(true);
        CHECK(run1 != run0 && list1 != list0);
        // kept states leave the pass out: the shape of the other route
        OK(soft_set_keep(c, 0, 4));
        OK(soft_run(c, 0, 800, nullptr, st.data(), nullptr, nullptr, nullptr));
        const Launch &L = g_launches.back();
        CHECK((std::vector<uint32_t>{L.grid, L.block, L.p.tile_mode, L.p.lds_entries}) == list1);
        OK(soft_set_keep(c, 0, 0));
        CHECK(shape(false) == run1);
    }
    soft_destroy(c);
    CHECK(g_live.empty());
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    (d / "host.cpp").write_text(DRIVER)
    flags = ["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
             "-I", CSRC, "-I", os.path.join(ROOT, "include")]
    procs = []
    for src in [str(d / "host.cpp")] + [os.path.join(CSRC, f) for f in ("soft_api.cpp", "signs.cpp", "compile.cpp")]:
        obj = str(d / (os.path.basename(src) + ".o"))
        procs.append((subprocess.Popen(flags + ["-c", src, "-o", obj], stderr=subprocess.PIPE, text=True), obj))
    for p, _ in procs:
        err = p.communicate()[1]
        assert p.returncode == 0, err[-2000:]
    subprocess.run(["g++", "-fsanitize=address", "-o", str(d / "host")] + [o for _, o in procs], check=True)
    (d / "big.txt").write_text(workloads.config("cultivation_42q", seed=1).text)
    (d / "small.txt").write_text(workloads.config("cultivation_15q", seed=1).text)
    return d


def go(d, *args):
    out = subprocess.run([str(d / "host"), args[0], str(d / "big.txt"), str(d / "small.txt")] + list(args[1:]),
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stdout[-1500:] + out.stderr[-3000:]
    return out.stdout


@pytest.mark.parametrize("tiles", ["0", "2", "3"])
@pytest.mark.parametrize("how", ["run", "noalloc"])
def test_recorded_addresses_stay(driver, how, tiles):
    go(driver, "capture", how, tiles)


def test_counter_reads_stay_in_the_last_runs_rows(driver):
    go(driver, "counters")


@pytest.mark.parametrize("single", ["0", "1"])
def test_autotune_times_the_routes_that_runs_take(driver, single):
    go(driver, "autotune", single)


def test_failing_host_allocations(driver):
    go(driver, "memory")
