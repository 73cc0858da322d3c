// CPU check of the host runtime (runtime.cpp) over a HIP runtime whose memory is host memory
// (fake_hip.h): under every budget that admits a sequence of calls, each launch stays inside live
// allocations.  The argument names the scenario.  Built with sanitizers by tests/test_runtime_memory.py.
#include <cmath>
#include <cstdio>
#include <fstream>
#include <functional>
#include <random>
#include <thread>

#include "fake_hip.h"
#include "nao.h"

#define CHECK(cond)                                                                             \
    do {                                                                                        \
        if (!(cond)) {                                                                          \
            std::fprintf(stderr, "CHECK failed at %s:%d: %s\n", __FILE__, __LINE__, #cond);      \
            std::exit(1);                                                                       \
        }                                                                                       \
    } while (0)

namespace {

// Atoms on a line of cubes of 2.2 Angstrom, 14 or 28 functions each, random points around every atom.
struct Structure {
    std::vector<double> axyz, rmin, rcut, samples, xyz, w;
    std::vector<int32_t> spc, shell_ptr{0}, shell_l, shell_rad;
    nao_basis_desc d{};
    int64_t nb = 0, np = 0;
    Structure(int nx, int ny, int nz, double cutoff, int points_per_atom, int max_l, unsigned seed)
    {
        std::mt19937_64 rng(seed);
        std::normal_distribution<double> g(0.0, 0.8);
        for (int x = 0; x < nx; ++x)
            for (int y = 0; y < ny; ++y)
                for (int z = 0; z < nz; ++z) {
                    const double at[3] = {2.2 * x, 2.2 * y, 2.2 * z};
                    for (double q : at) axyz.push_back(q);
                    spc.push_back(0);
                    for (int k = 0; k < points_per_atom; ++k)
                        for (double q : at) xyz.push_back(q + g(rng));
                }
        const int nk = 8;
        int nf = 0;
        for (int l : {0, 0, 1, 1, 2, 3})
            if (l <= max_l) {
                shell_l.push_back(l);
                shell_rad.push_back((int32_t)rmin.size());
                rmin.push_back(1e-3);
                rcut.push_back(cutoff);
                for (int k = 0; k < nk; ++k) samples.push_back(k + 1 < nk ? 1.0 : 0.0);
                nf += 2 * l + 1;
            }
        shell_ptr.push_back((int32_t)shell_l.size());
        np = (int64_t)xyz.size() / 3;
        w.assign(np, 0.5);
        nb = nf * (int64_t)spc.size();
        d.n_atoms = (int64_t)spc.size();
        d.atom_xyz = axyz.data();
        d.atom_species = spc.data();
        d.n_species = 1;
        d.species_shell_ptr = shell_ptr.data();
        d.shell_l = shell_l.data();
        d.shell_radial = shell_rad.data();
        d.n_radial = (int32_t)rmin.size();
        d.n_knots = nk;
        d.radial_rmin = rmin.data();
        d.radial_rcut = rcut.data();
        d.radial_samples = samples.data();
    }
};

template <typename T> T* device(int64_t n)
{
    void* p = nullptr;
    CHECK(hipMalloc(&p, sizeof(T) * n) == hipSuccess);
    return static_cast<T*>(p);
}

// The caller's device buffers of a structure (not part of any context's budget).
struct Buffers {
    double *D, *Q, *H, *n, *gn, *v, *a, *F;
    explicit Buffers(const Structure& s)
        : D(device<double>(s.nb * s.nb)), Q(device<double>(s.nb * s.nb)), H(device<double>(s.nb * s.nb)), n(device<double>(s.np)),
          gn(device<double>(3 * s.np)), v(device<double>(s.np)), a(device<double>(3 * s.np)), F(device<double>(3 * s.d.n_atoms))
    {
    }
    ~Buffers()
    {
        for (double* p : {D, Q, H, n, gn, v, a, F}) CHECK(hipFree(p) == hipSuccess);
    }
};

bool no_faults(const char* where)
{
    for (const auto& f : fake::faults) std::fprintf(stderr, "%s: %s\n", where, f.c_str());
    return fake::faults.empty();
}

nao_status build(nao_ctx c, const Structure& s, nao_system* out) { return nao_build_batches(c, &s.d, s.np, s.xyz.data(), s.w.data(), 200, out); }

// true when the call was accepted; a refusal for want of memory is the only other outcome
bool took(nao_status st)
{
    if (st != NAO_OK && st != NAO_ERR_BUDGET && st != NAO_ERR_OUT_OF_MEMORY) std::fprintf(stderr, "status %d\n", (int)st);
    CHECK(st == NAO_OK || st == NAO_ERR_BUDGET || st == NAO_ERR_OUT_OF_MEMORY);
    return st == NAO_OK;
}

// Every operation with device arrays; the number that was accepted.
int operations(nao_system s, const Buffers& b, nao_precision p)
{
    int k = 0;
    k += took(nao_update_density(s, b.D, NAO_MEM_DEVICE, p, b.n, NAO_MEM_DEVICE, nullptr));
    k += took(nao_integrate_h(s, b.v, NAO_MEM_DEVICE, p, b.H, NAO_MEM_DEVICE));
    if (p <= NAO_FP32) {
        k += took(nao_update_density_gradient(s, b.D, NAO_MEM_DEVICE, p, b.n, b.gn, NAO_MEM_DEVICE));
        k += took(nao_integrate_h_gga(s, b.v, b.a, NAO_MEM_DEVICE, p, b.H, NAO_MEM_DEVICE));
        k += took(nao_integrate_h_ks(s, b.v, b.a, NAO_MEM_DEVICE, p, b.H, NAO_MEM_DEVICE));
        k += took(nao_pulay_forces(s, b.D, b.Q, b.v, NAO_MEM_DEVICE, p, b.F, NAO_MEM_DEVICE));
    }
    return k;
}

// `sequence` runs on a context of the given budget and returns how many of its calls were accepted.
// Over budgets from `lo` (nothing fits) to beyond what it takes at most: no launch out of range.
struct Sweep {
    std::vector<size_t> budget;
    std::vector<int> accepted, clusters;
};
Sweep sweep(const std::function<int(nao_ctx)>& sequence, int steps)
{
    auto once = [&](size_t budget, size_t* used, int* clusters) {
        nao_ctx c = nullptr;
        CHECK(nao_ctx_create(0, nullptr, budget, &c) == NAO_OK);
        fake::cluster_launches = 0;
        const int k = sequence(c);
        if (clusters) *clusters = fake::cluster_launches;
        if (used) CHECK(nao_ctx_memory(c, used, nullptr) == NAO_OK);
        nao_ctx_destroy(c);
        return k;
    };
    size_t most = 0;
    Sweep r;
    (void)once(0, &most, nullptr);
    CHECK(no_faults("without a budget"));
    most += most / 4;
    for (int k = 0; k <= steps; ++k) {
        const size_t b = most / 8 + (most - most / 8) * k / steps;
        int clusters = 0;
        r.accepted.push_back(once(b, nullptr, &clusters));
        r.budget.push_back(b);
        r.clusters.push_back(clusters);
        if (!no_faults("under a budget")) {
            std::fprintf(stderr, "budget %zu of %zu, %d calls accepted\n", b, most, r.accepted.back());
            std::exit(1);
        }
    }
    return r;
}

// An earlier system of the context needs more scratch than a later one, whose clusters need still
// more: a refused growth must leave the scratch that the earlier one has.
void scratch()
{
    const Structure A(9, 5, 3, 5.0, 75, 3, 1), B(8, 5, 3, 5.0, 75, 3, 2);
    const Buffers a(A), b(B);
    const Sweep r = sweep(
        [&](nao_ctx c) {
            nao_system sa = nullptr, sb = nullptr;
            int k = 0;
            if (!took(build(c, A, &sa))) return 0;
            if (took(build(c, B, &sb))) k += 1 + operations(sb, b, NAO_FP64);
            k += operations(sa, a, NAO_FP64) + operations(sa, a, NAO_FP32);
            if (sb) k += operations(sb, b, NAO_BF16X6);
            if (sb) nao_system_destroy(sb);
            nao_system_destroy(sa);
            return k;
        },
        60);
    CHECK(r.clusters.back() > 0);
}

// The last allocations of a build are the ones that the clusters want larger (w v, the segment
// table): budgets and device limits a little below what the build takes.
void arrays()
{
    const Structure A(8, 5, 3, 5.0, 75, 3, 2);
    const Buffers a(A);
    nao_ctx c = nullptr;
    nao_system s = nullptr;
    CHECK(nao_ctx_create(0, nullptr, 0, &c) == NAO_OK);
    const size_t before = fake::device_used;
    CHECK(build(c, A, &s) == NAO_OK);
    size_t used = 0;
    CHECK(nao_ctx_memory(c, &used, nullptr) == NAO_OK);
    const size_t device = fake::device_used - before;
    nao_system_destroy(s);
    nao_ctx_destroy(c);
    int built = 0, refused = 0;
    for (int k = 0; k <= 240; ++k) {
        const size_t less = (size_t)(k / 2) * 1024;
        CHECK(nao_ctx_create(0, nullptr, k & 1 ? used - less : 0, &c) == NAO_OK);
        fake::device_limit = k & 1 ? 0 : fake::device_used + device - less;
        s = nullptr;
        if (took(build(c, A, &s))) {
            ++built;
            operations(s, a, NAO_FP64);
            operations(s, a, NAO_BF16X3);
            nao_system_destroy(s);
        } else {
            ++refused;
        }
        fake::device_limit = 0;
        nao_ctx_destroy(c);
        CHECK(no_faults(k & 1 ? "under a budget" : "under a device limit"));
    }
    CHECK(built > 0);
    std::printf("%d builds, %d refused\n", built, refused);
}

// Other groups or tiles refused for want of device memory: the system keeps working over the groups it
// had, or, where not even those come back, refuses its operations.
void regroup()
{
    const Structure A(8, 5, 3, 5.0, 75, 3, 2);
    const Buffers a(A);
    int refused = 0, lost = 0;
    for (int k = 0; k <= 60; ++k) {
        nao_ctx c = nullptr;
        nao_system s = nullptr;
        CHECK(nao_ctx_create(0, nullptr, 0, &c) == NAO_OK);
        const size_t before = fake::device_used;
        CHECK(build(c, A, &s) == NAO_OK);
        operations(s, a, NAO_FP64);
        fake::device_limit = before + (fake::device_used - before) * k / 60;
        refused += !took(nao_system_set_group_max(s, 64));
        refused += !took(nao_system_set_h_tile(s, 128));
        fake::device_limit = 0;
        if (nao_integrate_h(s, a.v, NAO_MEM_DEVICE, NAO_FP64, a.H, NAO_MEM_DEVICE) == NAO_ERR_INTERNAL) {
            ++lost;
            CHECK(nao_update_density(s, a.D, NAO_MEM_DEVICE, NAO_FP64, a.n, NAO_MEM_DEVICE, nullptr) == NAO_ERR_INTERNAL);
            CHECK(nao_system_set_group_max(s, 128) == NAO_OK);  // memory is there again
        }
        CHECK(operations(s, a, NAO_FP64) == 6 && operations(s, a, NAO_FP32) == 6);
        nao_system_destroy(s);
        nao_ctx_destroy(c);
        CHECK(no_faults("after a refused change"));
    }
    std::printf("%d changes refused, %d systems lost\n", refused, lost);
    CHECK(refused > 0);
}

// Clusters are a faster form and no more: what is accepted at some budget is accepted at every larger
// one, and the smallest budgets that take a Hamiltonian take it over the units.
void budget()
{
    const Structure A(8, 5, 3, 5.0, 75, 3, 2), B(6, 4, 3, 5.0, 60, 3, 3);
    const Buffers a(A), b(B);
    std::vector<double> D(A.nb * A.nb), H(A.nb * A.nb), n(A.np), v(A.np);
    struct Call {
        const char* name;
        bool hamiltonian;
        std::function<nao_status(nao_system)> f;
    };
    nao_ctx ctx = nullptr;
    const Call calls[] = {
        {"H", true, [&](nao_system s) { return nao_integrate_h(s, a.v, NAO_MEM_DEVICE, NAO_FP64, a.H, NAO_MEM_DEVICE); }},
        {"H host", true, [&](nao_system s) { return nao_integrate_h(s, v.data(), NAO_MEM_HOST, NAO_FP32, H.data(), NAO_MEM_HOST); }},
        {"density host", false, [&](nao_system s) { return nao_update_density(s, D.data(), NAO_MEM_HOST, NAO_FP64, n.data(), NAO_MEM_HOST, nullptr); }},
        {"gradient", false, [&](nao_system s) { return nao_update_density_gradient(s, a.D, NAO_MEM_DEVICE, NAO_FP64, a.n, a.gn, NAO_MEM_DEVICE); }},
        {"GGA", true, [&](nao_system s) { return nao_integrate_h_gga(s, a.v, a.a, NAO_MEM_DEVICE, NAO_FP64, a.H, NAO_MEM_DEVICE); }},
        {"KS", true, [&](nao_system s) { return nao_integrate_h_ks(s, a.v, nullptr, NAO_MEM_DEVICE, NAO_FP64, a.H, NAO_MEM_DEVICE); }},
        {"forces", false, [&](nao_system s) { return nao_pulay_forces(s, a.D, a.Q, a.v, NAO_MEM_DEVICE, NAO_FP64, a.F, NAO_MEM_DEVICE); }},
        {"resident", false, [&](nao_system s) { return nao_system_set_resident_basis(s, 1); }},
        {"second system", false, [&](nao_system) {
             nao_system t = nullptr;
             const nao_status st = build(ctx, B, &t);
             if (st == NAO_OK) nao_system_destroy(t);
             return st;
         }},
        {"run_many", true, [&](nao_system s) {
             const nao_work w[] = {{s, 0, a.v, a.H, nullptr}, {s, 1, a.D, a.n, nullptr}};
             return nao_run_many(ctx, w, 2, NAO_FP64, nullptr, 0);
         }},
        {"captured run_many", true, [&](nao_system s) {
             const nao_work w[] = {{s, 0, a.v, a.H, nullptr}, {s, 1, a.D, a.n, nullptr}};
             for (int k = 0; k < 2; ++k)
                 if (const nao_status st = nao_run_many(ctx, w, 2, NAO_FP64, nullptr, NAO_RUN_CAPTURE_GRAPH)) return st;
             return NAO_OK;
         }},
    };
    for (const Call& q : calls) {
        auto once = [&](size_t limit, size_t* used, int* clusters) {
            CHECK(nao_ctx_create(0, nullptr, limit, &ctx) == NAO_OK);
            nao_system s = nullptr;
            bool ok = false;
            fake::cluster_launches = 0;
            if (took(build(ctx, A, &s))) {
                ok = took(q.f(s));
                operations(s, a, NAO_FP64);  // whatever the call did: in range
                nao_system_destroy(s);
            }
            if (clusters) *clusters = fake::cluster_launches;
            if (used) CHECK(nao_ctx_memory(ctx, used, nullptr) == NAO_OK);
            nao_ctx_destroy(ctx);
            CHECK(no_faults(q.name));
            return ok;
        };
        size_t most = 0;
        CHECK(once(0, &most, nullptr));
        most *= 2;
        int accepted = 0, over_units = 0, over_clusters = 0;
        const int steps = 40;
        for (int k = 0; k <= steps; ++k) {
            int clusters = 0;
            const bool ok = once(most / 16 + (most - most / 16) / steps * k, nullptr, &clusters);
            if (accepted && !ok) {
                std::fprintf(stderr, "%s: accepted at budget step %d, refused at %d\n", q.name, k - 1, k);
                std::exit(1);
            }
            accepted += ok;
            if (ok && q.hamiltonian) (clusters ? over_clusters : over_units) += 1;
        }
        std::printf("%s: %d of %d budgets accept, %d with clusters\n", q.name, accepted, steps + 1, over_clusters);
        CHECK(accepted > 0 && accepted <= steps);
        if (q.hamiltonian) CHECK(over_units > 0 && over_clusters > 0);
    }
}

// What a server does: one thread builds and releases systems of a context whose budget is tight, so
// that clusters are given back, while another runs a system of it through a context of its own.
void serve()
{
    const Structure A(8, 5, 3, 5.0, 75, 3, 2), B(8, 5, 3, 5.0, 60, 3, 3);
    const Buffers a(A);
    nao_ctx home = nullptr, slot = nullptr;
    nao_system s = nullptr, t = nullptr;
    CHECK(nao_ctx_create(0, nullptr, 0, &home) == NAO_OK);
    CHECK(build(home, A, &s) == NAO_OK);
    size_t one = 0;
    CHECK(nao_ctx_memory(home, &one, nullptr) == NAO_OK);
    nao_system_destroy(s);
    nao_ctx_destroy(home);
    int all = 0, clustered = 0;
    for (int k = 0; k < 24; ++k) {
        CHECK(nao_ctx_create(0, nullptr, one / 2 + one * k / 32, &home) == NAO_OK);
        if (!took(build(home, A, &s))) {
            nao_ctx_destroy(home);
            continue;
        }
        CHECK(nao_ctx_create(0, nullptr, 0, &slot) == NAO_OK);
        fake::cluster_launches = 0;
        std::atomic<bool> stop{false};
        std::atomic<int> runs{0};
        std::thread builder([&]() {
            while (runs < 2) std::this_thread::yield();
            for (int j = 0; j < 3; ++j)
                if (took(build(home, B, &t))) nao_system_destroy(t);
            stop = true;
        });
        while (!stop || runs < 4) {
            const nao_work w[] = {{s, 1, a.D, a.n, nullptr}, {s, 0, a.v, a.H, nullptr}};
            CHECK(nao_run_many(slot, w, 2, NAO_FP64, nullptr, 0) == NAO_OK);
            CHECK(nao_ctx_synchronize(slot) == NAO_OK);  // retires the plan
            ++runs;
        }
        builder.join();
        CHECK(no_faults("run beside builds"));
        all += runs;
        clustered += fake::cluster_launches;
        nao_ctx_destroy(slot);
        nao_system_destroy(s);
        nao_ctx_destroy(home);
        CHECK(no_faults("at the end"));
    }
    std::printf("%d runs, %d with clusters\n", all, clustered);
    CHECK(clustered > 0 && clustered < all);
}

// A choice cached by the kernels of an earlier version (no version in its key) is not taken.
void tune(const char* path)
{
    const Structure A(3, 2, 2, 5.0, 40, 2, 4);
    const Buffers a(A);
    setenv("NAO_TUNE_CACHE", path, 1);
    nao_ctx c = nullptr;
    nao_system s = nullptr;
    CHECK(nao_ctx_create(0, nullptr, 0, &c) == NAO_OK && build(c, A, &s) == NAO_OK);
    int32_t tile = 0, groups = 0;
    double ms = 0.0;
    auto run = [&](uint32_t flags) {
        CHECK(nao_system_autotune(s, NAO_FP64, a.v, a.D, NAO_MEM_DEVICE, flags, &tile, &groups, &ms) == NAO_OK);
        return ms >= 0.0;  // timed, not taken from the file
    };
    CHECK(run(NAO_TUNE_FORCE) && !run(0));
    std::ifstream in(path);
    std::string line, key;
    while (std::getline(in, line))
        if (line.find("fp64") != std::string::npos) key = line.substr(line.find('"') + 1, line.rfind('"') - line.find('"') - 1);
    CHECK(!key.empty());
    const size_t v = key.find("/k");
    if (v != std::string::npos) key.erase(v, key.find('/', v + 1) - v);
    std::ofstream(path) << "{\n  \"" << key << "\": [128, 128]\n}\n";
    CHECK(run(0) && tile == 64 && groups == 256);
    CHECK(!run(0) && tile == 64);  // the new choice joined the file
    nao_system_destroy(s);
    nao_ctx_destroy(c);
    CHECK(no_faults("autotune"));
}

}  // namespace

int main(int argc, char** argv)
{
    setenv("NAO_SCRATCH_MB", "512", 1);
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "scratch") scratch();
    else if (what == "arrays") arrays();
    else if (what == "regroup") regroup();
    else if (what == "budget") budget();
    else if (what == "serve") serve();
    else if (what == "tune") tune(argc > 2 ? argv[2] : "/tmp/nao_tune_check.json");
    else return 2;
    std::printf("%s: all ok\n", what.c_str());
    return 0;
}
