// Host-side check of libplse's sessions on a stand-in for the HIP runtime
// (tests/test_host_sessions.py builds and runs it; no GPU).  The stand-in runs
// no kernel.  It keeps what a real device would have: which launches, copies
// and graph replays of a stream are still running, what an event stands for,
// which streams take part in a capture, and checks
//   - that every stream, event and graph used is alive, and none is left over;
//   - that no stream or graph is destroyed while work of it runs;
//   - that no stream of a capture is destroyed before the events recorded in it
//     (the runtime looks such an event's stream up by address when the event
//     goes, and addresses are used again);
//   - that nothing runs in a workspace once a call that hands it back returned;
//   - launch shapes: blocks, threads, dynamic LDS.
// Argument blocks are real: workspaces are host memory.
//
//   host_sessions_check SCENARIO  (prints "ok")
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "../include/plse.h"
#include "../paper_2103_10453_amd/csrc/kernels.h"

namespace {

using Ops = std::set<long>;

struct Launch {
    std::string kernel;
    dim3 grid, block;
    size_t lds;
    std::vector<const void *> blocks;  // argument blocks of the listed instances
};
struct Stream {
    Ops pend;
    Stream *origin = nullptr;  // of the capture it takes part in
};
struct Graph {
    std::vector<Launch> nodes;
};
struct Exec {
    std::vector<Launch> nodes;
    Ops ops;
};
struct Event {
    Ops snap;
    Stream *captured = nullptr;  // recorded in a capture, on this stream
    bool recorded = false;
};

std::recursive_mutex mu;
std::set<Stream *> streams;
std::set<Event *> events;
std::set<Exec *> execs;
std::map<Stream *, Graph *> capturing;  // by origin
std::set<Stream *> was_captured;        // live streams that took part in a capture
Stream null_stream;
Ops running;
long next_op = 1;
std::vector<Launch> log_;
// (filled by the library's own constructors, before this program's)
std::map<const void *, std::string> &kernel_names() {
    static std::map<const void *, std::string> m;
    return m;
}
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t s;
};
std::vector<Config> configs;
int bad = 0;
size_t lds_limit = 163840;       // per block
bool refuse_lds = false;         // hipFuncSetAttribute fails
long fail_at = 0, calls = 0;     // fail the fail_at-th fallible call
hipError_t last_error = hipSuccess;

void complain(const std::string &what) {
    if (bad++ < 10) std::fprintf(stderr, "violation: %s\n", what.c_str());
}
bool injected() {
    if (++calls != fail_at) return false;
    last_error = hipErrorOutOfMemory;
    return true;
}
Stream *of(hipStream_t s) {
    if (!s) return &null_stream;
    Stream *p = reinterpret_cast<Stream *>(s);
    if (!streams.count(p)) {
        complain("stream used after its destruction");
        return &null_stream;
    }
    return p;
}
Event *of(hipEvent_t e) {
    Event *p = reinterpret_cast<Event *>(e);
    if (!events.count(p)) {
        complain("event used after its destruction");
        std::abort();
    }
    return p;
}
bool any_running(const Ops &o) {
    for (long q : o)
        if (running.count(q)) return true;
    return false;
}
void complete(Ops &o) {
    for (long q : o) running.erase(q);
    o.clear();
}
void add_op(Stream *s, Exec *x = nullptr) {
    const long q = next_op++;
    running.insert(q);
    s->pend.insert(q);
    if (x) x->ops.insert(q);
}

}  // namespace

extern "C" {

hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    configs.push_back({g, b, lds, s});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    *g = configs.back().grid, *b = configs.back().block;
    *lds = configs.back().lds, *s = configs.back().s;
    configs.pop_back();
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) {
    static void *x;
    return &x;
}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
    kernel_names()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}

hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) {
    return refuse_lds ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) {
    std::memset(a, 0, sizeof(*a));
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t lds) {
    *n = lds ? (int)std::min<size_t>(16, 163840 / lds) : 8;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static void *mem = mmap(nullptr, PLSE_NOALLOC_BYTES, PROT_READ | PROT_WRITE,
                            MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    *p = mem;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::free(p);
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (injected()) return hipErrorOutOfMemory;
    Stream *p = new Stream();
    streams.insert(p);
    *s = reinterpret_cast<hipStream_t>(p);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    Stream *p = of(s);
    if (any_running(p->pend)) complain("stream destroyed while its work runs");
    if (p->origin) complain("stream destroyed during its capture");
    for (Event *e : events)
        if (e->captured == p) complain("stream of a capture destroyed before an event of it");
    streams.erase(p);
    delete p;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (of(s)->origin) complain("stream waited for during its capture");
    complete(of(s)->pend);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (injected()) return hipErrorOutOfMemory;
    Stream *p = of(s);
    Event *v = of(e);
    if (v->captured) {
        if (!v->captured->origin) complain("event of an ended capture waited for");
        if (p->origin && p->origin != v->captured->origin) complain("two captures joined");
        p->origin = v->captured->origin;
    }
    p->pend.insert(v->snap.begin(), v->snap.end());
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    Stream *p = of(s);
    p->origin = p;
    capturing[p] = new Graph();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    Stream *p = of(s);
    *g = reinterpret_cast<hipGraph_t>(capturing[p]);
    capturing.erase(p);
    for (Stream *q : streams)
        if (q->origin == p) q->origin = nullptr;
    return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (injected()) return hipErrorOutOfMemory;
    Event *p = new Event();
    events.insert(p);
    *e = reinterpret_cast<hipEvent_t>(p);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    Event *p = of(e);
    events.erase(p);
    delete p;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (injected()) return hipErrorOutOfMemory;
    Stream *p = of(s);
    Event *v = of(e);
    v->recorded = true;
    v->snap = p->pend;
    v->captured = p->origin ? p : nullptr;
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (of(e)->captured) complain("event of a capture queried");
    complete(of(e)->snap);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return hipEventQuery(e); }
hipError_t hipEventElapsedTime(float *t, hipEvent_t a, hipEvent_t b) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    for (hipEvent_t e : {a, b})
        if (!of(e)->recorded || of(e)->captured || any_running(of(e)->snap))
            complain("time of an event that has not passed");
    *t = 1.0f;
    return hipSuccess;
}

hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (injected()) return hipErrorOutOfMemory;
    Exec *p = new Exec();
    p->nodes = reinterpret_cast<Graph *>(g)->nodes;
    execs.insert(p);
    *x = reinterpret_cast<hipGraphExec_t>(p);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
    delete reinterpret_cast<Graph *>(g);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (injected()) return hipErrorOutOfMemory;
    Exec *p = reinterpret_cast<Exec *>(x);
    if (!execs.count(p)) {
        complain("graph launched after its destruction");
        return hipErrorInvalidValue;
    }
    log_.insert(log_.end(), p->nodes.begin(), p->nodes.end());
    add_op(of(s), p);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    Exec *p = reinterpret_cast<Exec *>(x);
    if (!execs.erase(p)) {
        complain("graph destroyed twice");
        return hipErrorInvalidValue;
    }
    if (any_running(p->ops)) complain("graph destroyed while it runs");
    delete p;
    return hipSuccess;
}

hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t q) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (injected()) return hipErrorOutOfMemory;
    std::memcpy(d, s, n);
    add_op(of(q));
    (void)k;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (injected()) return hipErrorOutOfMemory;
    Stream *p = of(s);
    const std::string &name = kernel_names()[f];
    Launch l{name, g, b, lds, {}};
    if (name.find("ArgList") != std::string::npos) {
        const plse::ArgList &L = *static_cast<const plse::ArgList *>(args[0]);
        const unsigned listed = name.find("persistent") != std::string::npos ? 0 : g.y;
        for (unsigned i = 0; i < listed; ++i) l.blocks.push_back(L.p[i]);
    }
    if (!g.x || !g.y || !b.x || b.x > 1024 || lds > lds_limit)
        complain("launch of " + l.kernel + ": " + std::to_string(g.x) + " x " +
                 std::to_string(b.x) + ", " + std::to_string(lds) + " bytes of LDS");
    if (p->origin)
        capturing[p->origin]->nodes.push_back(l);
    else {
        log_.push_back(l);
        add_op(p);
    }
    return hipSuccess;
}

}  // extern "C"

namespace {

#define NEED(x)                                                              \
    do {                                                                     \
        if (!(x)) {                                                          \
            std::fprintf(stderr, "line %d: %s\n", __LINE__, #x);             \
            ++bad;                                                           \
        }                                                                    \
    } while (0)

// An instance: cyclic square of order n with about (1 - keep) of its cells
// emptied, and a workspace for populations of p.
struct Inst {
    int n;
    plse_handle h = nullptr;
    void *ws = MAP_FAILED;
    size_t bytes = 0;
    std::vector<int8_t> out;
    Inst(int n_, int keep_percent, int p, uint32_t seed) : n(n_), out((size_t)n_ * n_) {
        std::vector<int8_t> g((size_t)n * n);
        uint32_t x = seed * 2654435761u + 1u;
        for (int i = 0; i < n; ++i)
            for (int j = 0; j < n; ++j) {
                x = x * 1664525u + 1013904223u;
                g[(size_t)i * n + j] = (int)((x >> 8) % 100) < keep_percent ? (int8_t)((i + j) % n + 1) : 0;
            }
        NEED(plse_create(n, g.data(), &h) == PLSE_OK);
        if (p) attach(p);
    }
    void attach(int p) {
        NEED(plse_workspace_bytes(h, p, &bytes) == PLSE_OK);
        ws = mmap(nullptr, bytes, PROT_READ | PROT_WRITE,
                  MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        NEED(ws != MAP_FAILED);
        NEED(plse_attach_workspace(h, ws, bytes) == PLSE_OK);
    }
    ~Inst() {
        plse_destroy(h);
        if (ws != MAP_FAILED) munmap(ws, bytes);
    }
};

// Mixed orders: several launch shapes, so several groups of searches.
struct Batch {
    std::vector<Inst *> in;
    std::vector<plse_handle> hs;
    std::vector<uint64_t> seeds;
    std::vector<int8_t *> grids;
    std::vector<int32_t> filled;
    explicit Batch(int p) {
        const int orders[] = {6, 12, 20, 33, 45, 60, 70, 12};
        for (int k = 0; k < 8; ++k) {
            in.push_back(new Inst(orders[k], 40 + 5 * k, p, k));
            NEED(plse_set_param(in[k]->h, "max_generations", 6) == PLSE_OK);
            if (k == 7) NEED(plse_set_param(in[k]->h, "variant", 1) == PLSE_OK);
            hs.push_back(in[k]->h);
            seeds.push_back(77 + k);
            grids.push_back(in[k]->out.data());
        }
        filled.resize(8);
    }
    int solve(int p, int G) {
        return plse_solve_batch(hs.data(), 8, p, G, seeds.data(), nullptr, grids.data(),
                                filled.data());
    }
    ~Batch() {
        for (Inst *i : in) delete i;
    }
};

void nothing_left(const char *where) {
    if (!streams.empty() || !events.empty() || !execs.empty() || !running.empty()) {
        std::fprintf(stderr, "%s: %zu streams, %zu events, %zu graphs, %zu operations left\n", where,
                     streams.size(), events.size(), execs.size(), running.size());
        ++bad;
    }
}

// Repeated batches, whole and in parts, below and above the populations whose
// distances start beside the searches.
void batch() {
    for (int p : {8, 130, 200}) {
        Batch b(p);
        for (int rep = 0; rep < 3; ++rep) {
            NEED(b.solve(p, 2) == PLSE_OK);
            nothing_left("batch");
        }
        plse_batch s = nullptr;
        NEED(plse_batch_begin(b.hs.data(), 8, p, b.seeds.data(), nullptr, &s) == PLSE_OK);
        NEED(plse_batch_step(s, 2, nullptr) == PLSE_OK);
        NEED(plse_batch_step(s, 1, nullptr) == PLSE_OK);
        NEED(plse_batch_end(s, nullptr, b.grids.data(), b.filled.data()) == PLSE_OK);
        nothing_left("batch in parts");
    }
}

// Single solves: by graphs, staged, without allocation, resumed, served.
void single() {
    for (int p : {5, 64, 130}) {
        Inst a(20, 50, p, 3);
        int32_t f = 0;
        NEED(plse_solve(a.h, p, 3, 1, nullptr, a.out.data(), &f) == PLSE_OK);
        nothing_left("solve");
        NEED(plse_set_param(a.h, "stage_timing", 1) == PLSE_OK);
        NEED(plse_solve(a.h, p, 3, 1, nullptr, a.out.data(), &f) == PLSE_OK);
        nothing_left("staged");
        NEED(plse_set_param(a.h, "stage_timing", 0) == PLSE_OK);
        size_t need = 0;
        NEED(plse_solve_noalloc(a.h, p, 3, 1, nullptr, a.out.data(), &f, &need) == PLSE_OK);
        nothing_left("no allocation");
        NEED(plse_begin(a.h, p, 1, nullptr) == PLSE_OK);
        NEED(plse_step(a.h, 1, nullptr) == PLSE_OK);
        size_t bytes = 0;
        NEED(plse_checkpoint(a.h, nullptr, nullptr, 0, &bytes) == PLSE_OK);
        std::vector<uint8_t> img(bytes);
        NEED(plse_checkpoint(a.h, nullptr, img.data(), bytes, &bytes) == PLSE_OK);
        NEED(plse_end(a.h, nullptr, a.out.data(), &f) == PLSE_OK);
        NEED(plse_resume(a.h, p, nullptr, img.data(), bytes) == PLSE_OK);
        NEED(plse_step(a.h, 1, nullptr) == PLSE_OK);
        NEED(plse_end(a.h, nullptr, a.out.data(), &f) == PLSE_OK);
        nothing_left("resumed");
    }
}

// Each unit of distances is computed once a generation: those that start beside
// the searches and the rest do not overlap, and miss none.
void units() {
    const int sizes[] = {2, 3, 5, 32, 63, 64, 65, 100, 127, 128, 129, 200, 255, 256, 257, 400,
                         4095, 4096, 4097, 4160, 4225};
    for (int p : sizes) {
        Inst a(6, 50, p, 3);
        int32_t f = 0;
        log_.clear();
        NEED(plse_solve(a.h, p, 1, 1, nullptr, a.out.data(), &f) == PLSE_OK);
        const int m = 2 * p;
        std::vector<int> once;
        int pairs_rows = 0;
        for (const Launch &l : log_) {
            if (l.kernel.find("pack_kernel") != std::string::npos)
                pairs_rows += static_cast<const plse::PackArgs *>(l.blocks[0])->m;
            if (l.kernel.find("dist_kernel") == std::string::npos) continue;
            const plse::DistArgs &d = *static_cast<const plse::DistArgs *>(l.blocks[0]);
            const size_t all = (size_t)plse::dist_units((m + plse::kDistCols - 1) / plse::kDistCols,
                                                        plse::kDistShort);
            if (once.empty()) once.assign(all, 0);  // short units are the most there are
            NEED(d.unit0 >= 0 && d.unit1 <= (int)all && (long)l.grid.x * 4 >= d.unit1 - d.unit0);
            for (int u = d.unit0; u < d.unit1; ++u) ++once[u];
        }
        NEED(!once.empty());
        const int rows = m <= 8192 ? plse::kDistShort : plse::kDistTall;
        const long all = plse::dist_units((m + plse::kDistCols - 1) / plse::kDistCols, rows);
        long twice = 0, missed = 0;
        for (long u = 0; u < all; ++u) twice += once[u] > 1, missed += once[u] == 0;
        if (twice || missed || pairs_rows != m) {
            std::fprintf(stderr, "p = %d: %ld of %ld units twice, %ld missed, %d of %d rows packed\n", p,
                         twice, all, missed, pairs_rows, m);
            ++bad;
        }
        nothing_left("units");
    }
}

// The k-th runtime call of a solve fails, for every k: the call reports it,
// nothing of it runs on or is left over, and the next call knows nothing of it.
void errors() {
    const int p = 130;
    Batch b(p);
    Inst a(20, 50, p, 3);
    int32_t f = 0;
    size_t need = 0;
    std::vector<uint8_t> img;
    NEED(plse_begin(a.h, p, 1, nullptr) == PLSE_OK);
    NEED(plse_checkpoint(a.h, nullptr, nullptr, 0, &need) == PLSE_OK);
    img.resize(need);
    NEED(plse_checkpoint(a.h, nullptr, img.data(), need, &need) == PLSE_OK);
    NEED(plse_end(a.h, nullptr, a.out.data(), &f) == PLSE_OK);
    for (int kind = 0; kind < 4; ++kind) {
        bool through = false;
        for (long k = 1; !through && k < 5000; ++k) {
            complete(null_stream.pend);
            calls = 0;
            fail_at = k;
            int rc = PLSE_OK;
            switch (kind) {
                case 0: rc = plse_solve(a.h, p, 2, 1, nullptr, a.out.data(), &f); break;
                case 1: rc = plse_solve_noalloc(a.h, p, 2, 1, nullptr, a.out.data(), &f, &need); break;
                case 2: rc = b.solve(p, 2); break;
                default: rc = plse_resume(a.h, p, nullptr, img.data(), img.size());
            }
            through = calls < k;
            fail_at = 0;
            if (kind == 3 && !rc) NEED(plse_end(a.h, nullptr, a.out.data(), &f) == PLSE_OK);
            const std::string at = "kind " + std::to_string(kind) + ", call " + std::to_string(k);
            if ((rc == PLSE_E_HIP) == through) complain(at + ": status " + std::to_string(rc));
            nothing_left(at.c_str());
            if (bad > 10) return;
        }
        NEED(through);
    }
}

// Where the runtime refuses more than 64 KiB of dynamic LDS, every launch stays
// within: populations up to the largest whose distances fit a device.
void lds64() {
    refuse_lds = true;
    lds_limit = 65536;
    for (int p : {2, 64, 2048, 3584, 4096, 5000, 8192, 12000, 16384, 32768})
        for (int hook : {0, 1}) {
            Inst a(6, 50, p, 3);
            int32_t f = 0;
            NEED(plse_set_param(a.h, "select_global_sort", hook) == PLSE_OK);
            const int before = bad;
            NEED(plse_solve(a.h, p, 1, 1, nullptr, a.out.data(), &f) == PLSE_OK);
            if (bad != before) std::fprintf(stderr, "  population %d, hook %d\n", p, hook);
            nothing_left("64 KiB");
        }
}

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "batch") batch();
    else if (what == "single") single();
    else if (what == "units") units();
    else if (what == "errors") errors();
    else if (what == "lds64") lds64();
    else return std::fprintf(stderr, "no scenario %s\n", what.c_str()), 2;
    if (!bad) std::puts("ok");
    return bad ? 1 : 0;
}
