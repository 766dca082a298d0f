// The batched runtime's host code on a stand-in for the HIP runtime, under the
// address and undefined-behaviour sanitizers and without a GPU (built by
// tests/test_host_runtime.py).  Device memory is host memory of exactly the
// size asked for, so every access beyond an allocation and every use after its
// release is caught; streams run their work at once, or record it while
// capturing, and graphs replay it.  A grouped launch touches what its kernel
// would: the block map, the films' arguments, the ends of their buffers.  The
// rules of captures are checked: no allocation, copy or synchronisation while a
// capture is open, every branch joined, no wait for an event of another
// capture, no launch of a graph that was destroyed.
#include "../../paper_1102_3069_amd/csrc/batch.hip"

#include <stdlib.h>

#include <functional>
#include <map>
#include <set>

#define REQUIRE(cond)                                                          \
    do {                                                                       \
        if (!(cond)) {                                                         \
            fprintf(stderr, "%s:%d: %s\n", __FILE__, __LINE__, #cond);         \
            abort();                                                           \
        }                                                                      \
    } while (0)

namespace sim {
using Work = std::function<void()>;
struct Capture {
    std::vector<Work> work;
    hipStream_t origin;
    std::set<hipStream_t> streams, unjoined;   // in this capture; with work that no wait has joined yet
};
struct Event {
    Capture* cap = nullptr;      // capture it was last recorded in (nullptr: none)
    bool recorded = false;
    std::set<hipStream_t> covers;
};
std::map<hipStream_t, Capture*> streams;       // live streams and what they capture into
std::map<hipEvent_t, Event> events;
std::set<Capture*> graphs, execs;
std::set<void*> dev;
Capture* open_capture = nullptr;
long long launches = 0, replays = 0;

void enqueue(hipStream_t s, Work w) {
    auto it = streams.find(s);
    REQUIRE(it != streams.end());
    ++launches;
    if (it->second) {
        it->second->work.push_back(w);
        if (s != it->second->origin) it->second->unjoined.insert(s);
    } else {
        w();
    }
}
void no_capture() { REQUIRE(open_capture == nullptr); }
}  // namespace sim

// ---- the HIP calls of the batched runtime -------------------------------------
extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMalloc(void** p, size_t n) {
    sim::no_capture();
    *p = malloc(n);
    memset(*p, 0xa5, n);
    sim::dev.insert(*p);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    sim::no_capture();
    REQUIRE(sim::dev.erase(p) == 1);
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    sim::no_capture();
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    sim::no_capture();
    REQUIRE(sim::streams.count(st));
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
    sim::no_capture();
    REQUIRE(sim::streams.count(st));
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)malloc(1);
    sim::streams[*s] = nullptr;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    REQUIRE(sim::streams.count(s) && !sim::streams[s]);
    sim::streams.erase(s);
    free((void*)s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    sim::no_capture();
    REQUIRE(sim::streams.count(s));
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = (hipEvent_t)malloc(1);
    sim::events[*e] = {};
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    REQUIRE(sim::events.erase(e) == 1);
    free((void*)e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    REQUIRE(sim::events.count(e) && sim::streams.count(s));
    sim::Event& ev = sim::events[e];
    ev.recorded = true;
    ev.cap = sim::streams[s];
    ev.covers = {s};
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    REQUIRE(sim::events.count(e) && sim::streams.count(s));
    sim::Event& ev = sim::events[e];
    REQUIRE(ev.recorded);
    if (ev.cap) {
        REQUIRE(ev.cap == sim::open_capture);               // not of a capture that has ended
        REQUIRE(!sim::streams[s] || sim::streams[s] == ev.cap);
        sim::streams[s] = ev.cap;                           // the waiting stream joins the capture
        ev.cap->streams.insert(s);
        for (hipStream_t c : ev.covers) ev.cap->unjoined.erase(c);
        if (s != ev.cap->origin) ev.cap->unjoined.insert(s);
    } else {
        REQUIRE(!sim::streams[s]);
    }
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    sim::no_capture();
    REQUIRE(sim::events.count(e) && sim::events[e].recorded && !sim::events[e].cap);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    REQUIRE(sim::events.count(a) && sim::events.count(b));
    *ms = 1.f + 0.001f * (float)(sim::launches % 7);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    sim::no_capture();
    REQUIRE(sim::streams.count(s) && !sim::streams[s]);
    sim::open_capture = new sim::Capture;
    sim::open_capture->origin = s;
    sim::open_capture->streams = {s};
    sim::streams[s] = sim::open_capture;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
    sim::Capture* c = sim::open_capture;
    REQUIRE(c && c->origin == s && c->unjoined.empty());
    for (hipStream_t t : c->streams) sim::streams[t] = nullptr;
    sim::open_capture = nullptr;
    sim::graphs.insert(c);
    *g = (hipGraph_t)c;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    sim::no_capture();
    sim::Capture* c = (sim::Capture*)g;
    REQUIRE(sim::graphs.count(c));
    sim::Capture* e = new sim::Capture(*c);
    sim::execs.insert(e);
    *x = (hipGraphExec_t)e;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
    REQUIRE(sim::graphs.erase((sim::Capture*)g) == 1);
    delete (sim::Capture*)g;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
    REQUIRE(sim::execs.erase((sim::Capture*)x) == 1);
    delete (sim::Capture*)x;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
    sim::no_capture();
    REQUIRE(sim::execs.count((sim::Capture*)x) && sim::streams.count(s));
    ++sim::replays;
    for (auto& w : ((sim::Capture*)x)->work) w();
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
}

// ---- the kernels' launchers ----------------------------------------------------
namespace {
volatile unsigned char sink;
template <typename T>
void touch(const T* p, size_t n) {          // first and last byte of n elements
    if (!p) return;
    sink = ((const unsigned char*)p)[0];
    sink = ((const unsigned char*)(p + n))[-1];
}
void touch_ref(const BufRef& r, size_t n) {
    touch(r.p[0], n);
    touch(r.p[1], n);
}
void touch_state(const Grid& g, const float2* S, const float2* twx, const DevState* st) {
    touch(S, (size_t)3 * g.nrows * g.nkxp);
    touch(twx, g.Px);
    touch(st, 1);
}
}  // namespace

namespace llg {
hipError_t launch_row_fwd_group(int Px, int var, const FilmRow* films, const int2* map, int nblocks, hipStream_t s) {
    REQUIRE(nblocks > 0 && fast2d_row_ok(Px, var));
    const int per = fast2d_row_rows_per_block(Px, var);
    sim::enqueue(s, [=] {
        for (int b = 0; b < nblocks; ++b) {
            const FilmRow& f = films[map[b].x];
            REQUIRE(f.g.Px == Px && map[b].y * per < f.g.nrows);
            touch_state(f.g, f.S, f.twx, f.st);
            const size_t n = (size_t)3 * f.g.ncells;
            touch_ref(f.fa.m_in, n);
            touch_ref(f.fa.m0, n);
            touch_ref(f.fa.k1, n);
            touch_ref(f.fa.m_out, n);
        }
    });
    return hipSuccess;
}
hipError_t launch_row_inv_group(int Px, int var, const FilmRow* films, const int2* map, int nblocks, hipStream_t s) {
    REQUIRE(nblocks > 0 && fast2d_row_ok(Px, var));
    const int per = fast2d_row_rows_per_block(Px, var);
    sim::enqueue(s, [=] {
        for (int b = 0; b < nblocks; ++b) {
            const FilmRow& f = films[map[b].x];
            REQUIRE(f.g.Px == Px && map[b].y * per < f.g.nrows && f.sa.nk <= kMaxK);
            touch_state(f.g, f.S, f.twx, f.st);
            const size_t n = (size_t)3 * f.g.ncells;
            touch_ref(f.sa.m_in, n);
            touch_ref(f.sa.m0, n);
            touch_ref(f.sa.m_out, n);
            touch_ref(f.sa.k_out, n);
            for (int j = 0; j + 1 < f.sa.nk; ++j) touch_ref(f.sa.kprev[j], n);
        }
    });
    return hipSuccess;
}
hipError_t launch_col_group(int L, int var, const FilmCol* films, const int2* map, int nblocks, hipStream_t s) {
    REQUIRE(nblocks > 0 && fast2d_col_ok(L, 1, var));
    sim::enqueue(s, [=] {
        for (int b = 0; b < nblocks; ++b) {
            const FilmCol& f = films[map[b].x];
            REQUIRE(f.a.Py == 2 * L && map[b].y < fast2d_col_blocks(L, var, f.a.nkx));
            touch(f.a.S, (size_t)3 * f.a.ny * f.a.nkxp);
            touch(f.a.K, (size_t)4 * f.a.nkx_full * (L + 1));
            touch(f.a.tw, f.a.Py);
            touch(f.st, 1);
        }
    });
    return hipSuccess;
}
// every third attempt of a film is rejected; films finish at their own pace
hipError_t launch_ctrl_dp45_group(DevState* st, int n, hipStream_t s) {
    sim::enqueue(s, [=] {
        for (int i = 0; i < n; ++i) {
            DevState& h = st[i];
            if (h.done) continue;
            const long long a = h.nattempt++;
            const bool ok = a % 3 != 2;
            if (a < h.log_cap && h.log) h.log[a] = llg_attempt{h.dt, 0.5f, ok};
            h.nevals += 6;
            if (!ok) { ++h.nrej; continue; }
            h.t += h.dt;
            h.cur ^= 1;
            ++h.step;
            ++h.nsteps;
            h.dt_next = 1e-14 * (1 + i % 17);
            if (h.clipped) { h.t = h.t_end; h.done = 1; }
            const double rem = h.t_end - h.t;
            h.clipped = h.dt_next >= rem;
            h.dt = h.clipped ? rem : h.dt_next;
        }
    });
    return hipSuccess;
}
hipError_t launch_ctrl_fixed_group(DevState* st, int n, int evals, hipStream_t s) {
    sim::enqueue(s, [=] {
        for (int i = 0; i < n; ++i) { st[i].t += st[i].dt; st[i].cur ^= 1; ++st[i].step; ++st[i].nsteps; st[i].nevals += evals; }
    });
    return hipSuccess;
}
hipError_t launch_normalize_check(float* m, int ncells, int* bad, hipStream_t s) {
    sim::enqueue(s, [=] { touch(m, (size_t)3 * ncells); touch(bad, 1); });
    return hipSuccess;
}
hipError_t build_kernel_spectrum(const Grid& g, const TensorGeom&, float* K, double* resid, hipStream_t) {
    touch(K, (size_t)4 * g.nkx * (g.Py / 2 + 1));
    *resid = 0.0;
    return hipSuccess;
}
}  // namespace llg

namespace {
void ok(llg_batch* b, llg_status rc) {
    if (rc != LLG_OK) {
        fprintf(stderr, "status %d: %s\n", (int)rc, llg_batch_last_error(b));
        abort();
    }
}
llg_batch* make(int films, int seed, std::vector<std::vector<float>>& m) {
    m.assign(films, {});
    std::vector<llg_film_desc> d(films);
    for (int i = 0; i < films; ++i) {
        llg_film_desc& f = d[i];
        f = {};
        f.nx = 20 + (i * 37 + seed * 11) % 130;
        f.ny = 18 + (i * 53 + seed * 7) % 170;
        f.dx = f.dy = 4e-9; f.dz = 3e-9;
        f.Ms = 8e5; f.Aex = 1.3e-11; f.alpha = 0.1; f.Ku = 0; f.u[0] = 1;
        m[i].assign((size_t)3 * f.nx * f.ny, 0.f);
        for (int c = 0; c < f.nx * f.ny; ++c) m[i][c] = 1.f;
        f.m0 = m[i].data();
    }
    llg_batch* b = nullptr;
    ok(b, llg_batch_create(0, d.data(), films, &b));
    return b;
}
}  // namespace

int main() {
    constexpr int N = 64;
    // three objects alive, their states set anew and run to t_end again and
    // again: films drop out, the maps and graphs are rebuilt mid-run
    std::vector<std::vector<float>> m[3];
    llg_batch* b[3];
    for (int k = 0; k < 3; ++k) b[k] = make(N, k, m[k]);
    std::vector<llg_stats> st(N);
    std::vector<llg_attempt> att(1000);
    for (int round = 0; round < 40; ++round)
        for (int k = 0; k < 3; ++k) {
            for (int i = 0; i < N; ++i) ok(b[k], llg_batch_set_m(b[k], i, m[k][i].data(), LLG_HOST));
            ok(b[k], llg_batch_run(b[k], 5e-13, 1e-5, 1e-14, 0, round % 2 ? st.data() : nullptr));
            for (int i = 0; i < N; i += 9) {
                ok(b[k], llg_batch_get_m(b[k], i, m[k][i].data(), LLG_HOST));
                int64_t n = 0;
                ok(b[k], llg_batch_get_attempts(b[k], i, att.data(), (int64_t)att.size(), &n));
                REQUIRE(n > 0);
            }
            if (round % 2) for (int i = 0; i < N; ++i) REQUIRE(st[i].done && st[i].t == 5e-13);
            // and what a caller mixes in
            if (round % 5 == 1) ok(b[k], llg_batch_step(b[k], round % 2 ? LLG_RK4 : LLG_HEUN, 1e-14, 3));
            if (round % 7 == 2) ok(b[k], llg_batch_run(b[k], 9e-13, 1e-5, 0.0, 5, st.data()));
            if (round == 11) ok(b[k], llg_batch_autotune(b[k], 2, nullptr, 0, nullptr));
            if (round == 17 + k) {
                llg_batch_destroy(b[k]);
                b[k] = make(N, k + 3, m[k]);
            }
        }
    for (int k = 0; k < 3; ++k) llg_batch_destroy(b[k]);
    REQUIRE(sim::dev.empty() && sim::streams.empty() && sim::events.empty() && sim::graphs.empty() && sim::execs.empty());
    printf("batch ok (%lld launches, %lld replays)\n", sim::launches, sim::replays);
    return 0;
}
