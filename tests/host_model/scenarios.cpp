// Scenarios of the simulation contexts on the modelled device, one per run:
// scenarios <name>.  Prints what differs and exits with 1, or exits with 0.
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "lbm.h"
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

const std::map<std::string, void (*)()> SCENARIOS = {
    {"captured_readout", captured_readout},
    {"captured_load", captured_load},
    {"eager_before_replay", eager_before_replay},
    {"captured_3d", captured_3d},
    {"given_back", given_back},
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
