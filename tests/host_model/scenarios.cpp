// Scenarios of the simulation contexts on the modelled device, one per run:
// scenarios <name>.  Prints what differs and exits with 1, or exits with 0.
#include <atomic>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <thread>
#include <vector>

#include "lbm.h"
#include "lbm_host.hpp"
#include "model.hpp"

using namespace lbm;

namespace {

int wrong = 0;
void expect(bool ok, const std::string& what)
{
    if (!ok) std::printf("wrong: %s\n", what.c_str()), ++wrong;
}
void expect_count(const void* p, long t, const std::string& what)
{
    expect(count_at(p) == t, what + ": " + std::to_string(count_at(p)) + " instead of " + std::to_string(t));
}

constexpr int NX = 64, NY = 32, NZ = 8;
const int SCHEMES[] = {S_LPTL, S_NPTL, S_PUSH, S_NPOL, S_NSOL, S_AA};
const char* const NAMES[] = {"LPTL", "NPTL", "PUSH", "NPOL", "NSOL", "AA"};

struct Sim {
    Stream* stream = new Stream();
    lbm_ctx* c = nullptr;
    float* out = nullptr;
    explicit Sim(int scheme, int64_t nx = NX, int64_t ny = NY)
    {
        const std::vector<uint8_t> flags(nx * ny, 0);
        lbm_grid g{nx, ny, scheme, 0, 0, 0, 0};
        lbm_bc bc{};
        bc.x_axis = bc.y_axis = LBM_CLOSED;
        bc.rho0 = 1.0;
        status = lbm_create(&g, flags.data(), 0.8, &bc, stream, &c);
        (void)hipMalloc(&out, 1024);
    }
    ~Sim()
    {
        lbm_destroy(c);
        (void)hipFree(out);
        delete stream;
    }
    lbm_status status;
    // the state's update count, by a readout
    long count()
    {
        expect(lbm_macros(c, out, nullptr, 1) == LBM_OK, "macros");
        return count_at(out);
    }
};
struct Sim3 {
    Stream* stream = new Stream();
    lbm3_ctx* c = nullptr;
    float* out = nullptr;
    explicit Sim3(int scheme)
    {
        const std::vector<uint8_t> flags(NX * NY * NZ, 0);
        lbm3_grid g{NX, NY, NZ, scheme, 0, 0, 0, 0};
        lbm3_bc bc{};
        bc.x_axis = bc.y_axis = bc.z_axis = LBM_CLOSED;
        bc.rho0 = 1.0;
        status = lbm3_create(&g, flags.data(), 0.8, &bc, stream, &c);
        (void)hipMalloc(&out, 1024);
    }
    ~Sim3()
    {
        lbm3_destroy(c);
        (void)hipFree(out);
        delete stream;
    }
    lbm_status status;
    long count()
    {
        expect(lbm3_macros(c, out, nullptr, 1) == LBM_OK, "macros");
        return count_at(out);
    }
};

Graph capture(Stream* s, const std::function<void()>& call)
{
    Graph g;
    s->capture = &g;
    call();
    s->capture = nullptr;
    return g;
}
void replay(const Graph& g)
{
    for (const Work& w : g.work) w();
}

void each_scheme(const std::function<void(int, const std::string&)>& run)
{
    for (int s : SCHEMES)
        for (int tile : {0, 1}) {
            plan = FusedPlan{8, tile, 64};
            run(s, std::string(NAMES[s]) + (tile ? " tile " : " strip "));
        }
}

// A captured readout reports, and a captured load replaces, the state that
// eager updates have moved on since.
void captured_readout()
{
    each_scheme([](int scheme, const std::string& name) {
        Sim a(scheme);
        float* got = nullptr;
        double* d = nullptr;
        (void)hipMalloc(&got, 4096);
        (void)hipMalloc(&d, 64);
        lbm_step(a.c, 36);
        const Graph g = capture(a.stream, [&] {
            lbm_macros(a.c, got, got + 64, 1);
            lbm_get_populations(a.c, got + 128, 1);
            lbm_diag_noalloc(a.c, nullptr, 0, d);
        });
        long t = 36;
        for (int n : {2, 8, 12, 34, 100}) {
            lbm_step(a.c, n);
            replay(g);
            t += n;
            for (int k : {0, 64, 128}) expect_count(got + k, t, name + "readout after " + std::to_string(n));
            expect_count(d, t, name + "diagnostics after " + std::to_string(n));
            expect(a.count() == t, name + "state");
        }
    });
}

void captured_load()
{
    each_scheme([](int scheme, const std::string& name) {
        Sim a(scheme);
        float* f = nullptr;
        (void)hipMalloc(&f, 4096);
        set_count(f, 1000);
        lbm_step(a.c, 36);
        const Graph g = capture(a.stream, [&] { lbm_set_state(a.c, f, 1); });
        for (int n : {2, 8, 12, 34}) {
            const long t = a.count();
            lbm_step(a.c, n);
            expect(a.count() == t + n, name + "updates before a replay");
            replay(g);
            expect(a.count() == 1000, name + "load after " + std::to_string(n));
            lbm_step(a.c, 6);
            expect(a.count() == 1006, name + "updates after a load");
        }
    });
}

// Eager updates between a capture and its first replay, and a capture that is
// never replayed.
void eager_before_replay()
{
    each_scheme([](int scheme, const std::string& name) {
        for (bool replayed : {true, false}) {
            Sim a(scheme);
            lbm_step(a.c, 36);
            const Graph g = capture(a.stream, [&] { lbm_step(a.c, 2); });
            lbm_step(a.c, 2);
            long t = 38;
            expect(a.count() == t, name + "updates before the first replay");
            for (int n : {32, 2, 40}) {
                if (replayed) replay(g), t += 2;
                lbm_step(a.c, n);
                t += n;
                expect(a.count() == t, name + "updates after a replay");
            }
        }
    });
}

void captured_3d()
{
    for (int scheme : {S_NPTL, S_AA}) {
        serves3 = true;
        Sim3 a(scheme);
        float *got = nullptr, *f = nullptr;
        (void)hipMalloc(&got, 4096);
        (void)hipMalloc(&f, 4096);
        set_count(f, 1000);
        lbm3_step(a.c, 6);
        const Graph read = capture(a.stream, [&] {
            lbm3_macros(a.c, got, got + 64, 1);
            lbm3_get_populations(a.c, got + 128, 1);
        });
        const Graph load = capture(a.stream, [&] { lbm3_set_state(a.c, f, 1); });
        long t = 6;
        for (int n : {2, 6, 4}) {
            lbm3_step(a.c, n);
            t += n;
            replay(read);
            for (int k : {0, 64, 128}) expect_count(got + k, t, "D3Q19 readout");
            replay(load);
            t = 1000;
            expect(a.count() == t, "D3Q19 load");
        }
    }
}

// After a captured call bundles of single updates are replayed as cached graphs
// again, none that was made before it, and none while the stream is captured.
void graphs_after_capture()
{
    for (int scheme : SCHEMES) {
        plan = FusedPlan{4, 1, 0};
        const std::string name = NAMES[scheme];
        Sim a(scheme);
        lbm_set_bundle(a.c, 24);
        lbm_step(a.c, 24); // six launches: a graph
        expect(dev.graph_launches > 0, name + ": graph before");
        const Graph g = capture(a.stream, [&] {
            const int before = dev.graph_launches;
            expect(lbm_step(a.c, 48) == LBM_OK && dev.graph_launches == before, name + ": no graph while captured");
        });
        expect(g.work.size() >= 48, name + ": single updates captured");
        long t = 24;
        for (int k = 0; k < 4; ++k) {
            const int graphs = dev.graph_launches, singles = dev.singles, fused = dev.fused;
            lbm_step(a.c, 72);
            expect(dev.graph_launches == graphs + 3, name + ": graphs after");
            expect(dev.singles == singles + 72 && dev.fused == fused, name + ": single updates after");
            t += 72;
            expect(a.count() == t, name + ": state");
            replay(g);
            t += 48;
            expect(a.count() == t, name + ": state after a replay");
        }
    }
}

// Calls of one update of NPOL and NSOL: in place where the plan says so, but
// not right after launches of several updates.
void calls_of_one_update()
{
    for (int scheme : {S_NPOL, S_NSOL})
        for (bool own : {true, false}) {
            plan = FusedPlan{8, 0, 64, own};
            Sim a(scheme);
            long t = 0;
            auto step = [&](int n, bool in_place) {
                const int before = dev.singles;
                lbm_step(a.c, n);
                t += n;
                expect((dev.singles > before) == in_place, NAMES[scheme] + std::string(" route of update ") + std::to_string(t));
                expect(a.count() == t, NAMES[scheme] + std::string(" state"));
            };
            for (int k = 0; k < 3; ++k) {
                step(1, own && k == 0);
                step(1, own);
                step(1, own);
                step(10, false);
            }
        }
}

// Host readouts of a simulation while another device is the current one: the
// first through the pinned chunks, and later ones.
void readout_from_another_device()
{
    for (int first : {0, 1}) {
        plan = FusedPlan{8, 1, 0};
        (void)hipSetDevice(0);
        Sim a(S_NPTL, 1024, 600); // rho alone goes through the chunks
        std::vector<float> f(9 * 1024 * 600, 7.0f);
        expect(lbm_set_state(a.c, f.data(), 0) == LBM_OK, "load");
        for (int k = 0; k < 3; ++k) {
            (void)hipSetDevice(k == 0 ? first : 1 - first);
            expect(lbm_macros(a.c, f.data(), nullptr, 0) == LBM_OK, "readout with another device current");
            expect(f[0] == 7.0f, "its values");
            expect(lbm_get_populations(a.c, f.data(), 0) == LBM_OK, "populations with another device current");
        }
        int now = 0;
        (void)hipGetDevice(&now);
        expect(now == 1 - first, "the current device stays");
        (void)hipSetDevice(0);
    }
}

// Served requests of few nodes run single updates, more of them several per
// launch, and a request may see both.
void served_by_load()
{
    Stream* stream = new Stream();
    lbm_server* s = nullptr;
    expect(lbm_server_create(1 << 28, 4, 10, 0, 0, stream, &s) == LBM_OK, "server");
    const std::vector<uint8_t> flags(1000 * 400, 0);
    lbm_bc bc{};
    bc.x_axis = bc.y_axis = LBM_CLOSED;
    bc.rho0 = 1.0;
    uint64_t id[2];
    lbm_grid small{100, 100, S_NPTL, 0, 0, 0, 0}, large{1000, 400, S_NPTL, 0, 0, 0, 0};
    lbm_server_submit(s, &small, flags.data(), 0.8, &bc, 35, &id[0]);
    lbm_server_run_bundle(s);
    expect(dev.singles == 10 && dev.fused == 0, "a small request alone");
    lbm_server_submit(s, &large, flags.data(), 0.8, &bc, 12, &id[1]);
    lbm_server_run_bundle(s);
    lbm_server_run_bundle(s);
    expect(dev.singles == 10 && dev.fused == 6, "beside a large one");
    lbm_server_run_bundle(s);
    expect(dev.singles == 20 && dev.fused == 6, "alone again");
    lbm_server_run_bundle(s);
    int32_t status[2], n = 0;
    expect(lbm_server_poll(s, id, status, 2, &n) == LBM_OK && n == 2, "both finished");
    lbm_server_destroy(s);
    delete stream;
}

// A served request that needs single updates finds its bundles captured.
void served_single_updates()
{
    Stream* stream = new Stream();
    lbm_server* s = nullptr;
    expect(lbm_server_create(1 << 24, 4, 10, 0, 0, stream, &s) == LBM_OK, "server");
    const std::vector<uint8_t> flags(NX * NY, 0);
    lbm_grid g{NX, NY, S_NPTL, 0, 0, 0, 0};
    lbm_bc bc{};
    bc.x_axis = LBM_NEUMANN_OUTFLOW;
    bc.y_axis = LBM_CLOSED;
    bc.rho0 = 1.0;
    uint64_t id = 0;
    expect(lbm_server_submit(s, &g, flags.data(), 0.8, &bc, 25, &id) == LBM_OK, "request");
    const int before = dev.captures;
    for (int k = 0; k < 4; ++k) expect(lbm_server_run_bundle(s) == LBM_OK, "bundle");
    expect(dev.singles == 30 && dev.fused == 0, "launches of three bundles, not " + std::to_string(dev.singles));
    expect(dev.captures == before, std::to_string(dev.captures - before) + " captures in the serving loop");
    int32_t status[2], n = 0;
    uint64_t ids[2];
    expect(lbm_server_poll(s, ids, status, 2, &n) == LBM_OK && n == 1 && ids[0] == id, "finished");
    lbm_server_destroy(s);
    delete stream;
}

// Memory held for several updates per launch goes back when an allocation
// fails, but nothing that a captured call refers to.
void given_back()
{
    double d[5];
    for (int scheme : {S_NPTL, S_AA})
        for (bool several : {true, false})
            for (int captured : {0, 1, 2}) { // nothing, an update and a readout, a load
                if (scheme == S_AA && !several && captured == 2) continue; // allocates, which a capture refuses
                serves3 = several;
                Sim3 a(scheme);
                const std::string name = std::string("D3Q19 ") + NAMES[scheme] + " captured " + std::to_string(captured);
                float* f = nullptr;
                (void)hipMalloc(&f, 4096);
                set_count(f, 1000);
                lbm3_step(a.c, 4);
                const Graph g = capture(a.stream, [&] {
                    if (captured == 1) lbm3_step(a.c, 2), lbm3_macros(a.c, f + 64, nullptr, 1);
                    if (captured == 2) lbm3_set_state(a.c, f, 1);
                });
                const size_t before = dev.free_bytes;
                dev.largest = 0;
                expect(lbm3_diag(a.c, d) == LBM_ENOMEM, name + ": diagnostics without memory");
                dev.largest = SIZE_MAX;
                if (!captured) expect(dev.free_bytes > before, name + ": memory goes back");
                replay(g);
                const long t = captured == 2 ? 1000 : captured ? 6 : 4;
                expect(a.count() == t, name + ": state");
                lbm3_step(a.c, 6);
                expect(a.count() == t + 6, name + ": updates after");
                expect(lbm3_diag(a.c, d) == LBM_OK, name + ": diagnostics");
            }
    for (int scheme : {S_NPOL, S_NSOL, S_AA})
        for (int captured : {0, 1, 2}) {
            plan = FusedPlan{8, 0, 64};
            Sim a(scheme);
            const std::string name = std::string(NAMES[scheme]) + " captured " + std::to_string(captured);
            float* f = nullptr;
            (void)hipMalloc(&f, 4096);
            set_count(f, 1000);
            lbm_step(a.c, 8);
            const Graph g = capture(a.stream, [&] {
                if (captured == 1) lbm_step(a.c, 2), lbm_macros(a.c, f + 64, nullptr, 1);
                if (captured == 2) lbm_set_state(a.c, f, 1);
            });
            const size_t before = dev.free_bytes;
            dev.largest = 0;
            expect(lbm_diag(a.c, d) == LBM_ENOMEM, name + ": diagnostics without memory");
            dev.largest = SIZE_MAX;
            if (captured < 2) expect(dev.free_bytes > before, name + ": memory goes back");
            replay(g);
            const long t = captured == 2 ? 1000 : captured ? 10 : 8;
            expect(a.count() == t, name + ": state");
            lbm_step(a.c, 6);
            expect(a.count() == t + 6, name + ": updates after");
            expect(lbm_diag(a.c, d) == LBM_OK, name + ": diagnostics");
        }
}

// A simulation whose allocation fails gets the memory that others hold only to
// be faster; they go on in place.
void given_back_to_others()
{
    const size_t all = dev.free_bytes;
    for (int scheme : {S_NPOL, S_NSOL, S_AA})
        for (int n : {8, 16}) { // the state in the second lattice, in the first
            plan = FusedPlan{8, 0, 64};
            serves3 = true;
            Sim a(scheme);
            Sim3 b(S_AA), b2(S_NPTL);
            lbm_step(a.c, n);
            lbm3_step(b.c, 6);
            lbm3_step(b2.c, 6);
            const size_t before = dev.free_bytes;
            dev.free_bytes = 0; // others use the rest of the device
            {
                Sim more(S_NPTL, 32, 16);
                expect(more.status == LBM_OK, std::string("a simulation beside ") + NAMES[scheme]);
                lbm_step(more.c, 40);
                expect(more.count() == 40, "its state");
            }
            expect(dev.free_bytes > 0, "memory went back");
            dev.free_bytes += before;
            const int fused = dev.fused;
            lbm_step(a.c, 16);
            lbm3_step(b.c, 4);
            lbm3_step(b2.c, 4);
            expect(dev.fused == fused, "single updates from then on");
            expect(a.count() == n + 16, std::string(NAMES[scheme]) + ": state afterwards");
            expect(b.count() == 10 && b2.count() == 10, "D3Q19: state afterwards");
        }
    expect(dev.free_bytes == all, "all memory freed");
}

// Spare memory of all simulations together is bounded, and only taken while
// enough stays free.
void spare_memory_is_bounded()
{
    plan = FusedPlan{8, 0, 64};
    auto fused = [](Sim& a) {
        const int before = dev.fused;
        lbm_step(a.c, 16);
        return dev.fused > before;
    };
    size_t one; // spare bytes of one simulation
    {
        size_t f = dev.free_bytes;
        Sim a(S_AA), b(S_NPTL);
        lbm_info ia, ib;
        lbm_get_info(a.c, &ia), lbm_get_info(b.c, &ib);
        expect(ia.device_bytes == ib.device_bytes, "two lattices each");
        expect(fused(a), "several updates per launch");
        one = (f - dev.free_bytes) / 5;
    }
    dev.total = 32 * 10 * one;
    dev.free_bytes = dev.total;
    {
        std::vector<Sim*> sims;
        int with = 0;
        for (int k = 0; k < 20; ++k) {
            sims.push_back(new Sim(S_AA));
            expect(sims.back()->status == LBM_OK, "creation");
            with += fused(*sims.back());
        }
        expect(with > 3 && with < 20, "a bounded number of second lattices, not " + std::to_string(with));
        for (Sim* s : sims) delete s;
        expect(dev.free_bytes == dev.total, "all memory freed");
    }
    {
        Sim a(S_AA);
        expect(fused(a), "room again");
    }
    dev.free_bytes = dev.total / 20;
    {
        Sim a(S_AA);
        expect(a.status == LBM_OK && !fused(a) && a.count() == 16, "in place while little is free");
    }
}

// Simulations come, run and go on four threads while a fifth asks for their
// spare memory again and again.
void given_back_across_threads()
{
    plan = FusedPlan{8, 0, 64};
    serves3 = true;
    std::atomic<bool> stop{false};
    std::atomic<int> bad{0};
    std::vector<std::thread> th;
    for (int k = 0; k < 4; ++k)
        th.emplace_back([&, k] {
            while (!stop) {
                Sim a(k % 2 ? S_AA : S_NPOL);
                Sim3 b(S_AA);
                long t = 0;
                for (int i = 0; i < 20; ++i) {
                    lbm_step(a.c, 8 + 2 * i);
                    lbm3_step(b.c, 8 + 2 * i);
                    t += 8 + 2 * i;
                    bad += a.count() != t || b.count() != t;
                }
            }
        });
    for (int i = 0; i < 300; ++i) {
        void* p;
        expect(device_alloc(&p, (size_t)1 << 50, nullptr) != hipSuccess, "more than there is");
        std::this_thread::yield();
    }
    stop = true;
    for (std::thread& t : th) t.join();
    expect(!bad, "states");
}

const std::map<std::string, void (*)()> SCENARIOS = {
    {"captured_readout", captured_readout},
    {"captured_load", captured_load},
    {"eager_before_replay", eager_before_replay},
    {"captured_3d", captured_3d},
    {"graphs_after_capture", graphs_after_capture},
    {"readout_from_another_device", readout_from_another_device},
    {"served_by_load", served_by_load},
    {"served_single_updates", served_single_updates},
    {"calls_of_one_update", calls_of_one_update},
    {"given_back", given_back},
    {"given_back_to_others", given_back_to_others},
    {"given_back_across_threads", given_back_across_threads},
    {"spare_memory_is_bounded", spare_memory_is_bounded},
};

} // namespace

int main(int argc, char** argv)
{
    const auto it = argc == 2 ? SCENARIOS.find(argv[1]) : SCENARIOS.end();
    if (it == SCENARIOS.end()) {
        for (const auto& s : SCENARIOS) std::printf("%s\n", s.first.c_str());
        return argc == 1 ? 0 : 2;
    }
    it->second();
    expect(dev.faults == 0, std::to_string(dev.faults) + " accesses to memory that is not allocated");
    return wrong ? 1 : 0;
}
