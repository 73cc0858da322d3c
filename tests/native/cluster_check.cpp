// Host check of the Hamiltonian clusters (plan.cpp make_clusters): every unit is in exactly one
// cluster, in order; rows are the units' points rounded up to 16 and stay within the limit unless
// one unit exceeds it; a cluster's atoms are the union of its units', each once, ordered by the
// points of the batches they reach and, in the second list, ascending; columns are contiguous; the
// element limit holds.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>

#include "plan.h"

using namespace nao;

static void expect(bool ok, const char* what)
{
    if (!ok) {
        std::printf("FAILED: %s\n", what);
        std::exit(1);
    }
}

static void check(uint32_t seed, int n_atoms, int n_points, double box, int32_t group_max, int32_t max_rows, int64_t max_elems)
{
    std::mt19937 rng(seed);
    std::uniform_real_distribution<double> U(0.0, box);
    HostBasis b;
    b.n_atoms = n_atoms;
    b.n_species = 2;
    const int32_t nfn[2] = {5, 14};
    b.atom_first.assign(1, 0);
    for (int a = 0; a < n_atoms; ++a) {
        for (int d = 0; d < 3; ++d) b.atom_xyz.push_back(U(rng));
        b.atom_species.push_back(a % 2);
        b.atom_rcut.push_back(a % 2 ? 3.0 : 2.0);
        b.atom_first.push_back(b.atom_first.back() + nfn[a % 2]);
    }
    b.n_basis = b.atom_first.back();
    std::vector<double> xyz;
    for (int p = 0; p < 3 * n_points; ++p) xyz.push_back(U(rng));
    std::vector<int64_t> perm, bptr, aptr, cnt;
    std::vector<int32_t> atoms, uat, ucol, cat, ccol, aat, acol;
    octree_batches(xyz.data(), n_points, 96, perm, bptr);
    relevant_atoms(b, xyz.data(), perm, bptr, aptr, atoms);
    std::vector<Unit> units;
    make_groups(b, bptr, aptr, atoms, group_max, units, uat, ucol);
    std::vector<Cluster> cl;
    make_clusters(b, bptr, aptr, atoms, units, uat, max_rows, 64, max_elems, cl, cat, ccol, aat, acol);
    int64_t next = 0;
    int joined = 0;
    for (const Cluster& c : cl) {
        expect(c.unit_begin == next && c.unit_count >= 1, "units in order, each once");
        next += c.unit_count;
        joined += c.unit_count > 1;
        std::set<int32_t> want;
        std::vector<int64_t> reach(n_atoms, 0);
        int64_t rows = 0;
        for (int k = c.unit_begin; k < c.unit_begin + c.unit_count; ++k) {
            rows += (units[k].n_points + 15) / 16 * 16;
            want.insert(uat.begin() + units[k].atom_begin, uat.begin() + units[k].atom_begin + units[k].n_atoms);
            for (size_t q = 0; q + 1 < bptr.size(); ++q) {
                const int64_t p0 = std::max(bptr[q], units[k].point_begin);
                const int64_t p1 = std::min(bptr[q + 1], units[k].point_begin + units[k].n_points);
                if (p0 < p1)
                    for (int64_t t = aptr[q]; t < aptr[q + 1]; ++t) reach[atoms[t]] += p1 - p0;
            }
        }
        expect(rows == c.n_rows && rows % 16 == 0, "rows");
        expect(c.unit_count == 1 || rows <= max_rows, "row limit");
        expect(c.unit_count == 1 || rows * ((c.m + 63) / 64 * 64) <= max_elems, "element limit");
        expect((int)want.size() == c.n_atoms, "union size");
        int32_t col = 0;
        std::set<int32_t> asc(want);
        auto it = asc.begin();
        for (int t = 0; t < c.n_atoms; ++t, ++it) {
            expect(aat[c.atom_begin + t] == *it && acol[c.atom_begin + t] == col, "ascending order");
            col += nfn[*it % 2];
        }
        expect(col == c.m, "ascending columns");
        col = 0;
        for (int t = 0; t < c.n_atoms; ++t) {
            const int32_t a = cat[c.atom_begin + t];
            expect(want.erase(a) == 1, "union member, once");
            expect(ccol[c.atom_begin + t] == col, "contiguous columns");
            col += nfn[a % 2];
            expect(t == 0 || reach[cat[c.atom_begin + t - 1]] >= reach[a], "ordered by reach");
        }
        expect(col == c.m, "columns");
    }
    expect(next == (int64_t)units.size(), "all units");
    expect(max_rows < 64 || max_elems < 1000 || units.size() < 2 || joined > 0, "some units were joined");
}

int main()
{
    check(1, 12, 4000, 6.0, 256, 960, 1 << 28);
    check(2, 12, 4000, 6.0, 256, 512, 1 << 28);
    check(3, 30, 9000, 14.0, 128, 960, 1 << 28);   // points out of reach between units
    check(4, 12, 4000, 6.0, 256, 960, 60000);      // the element limit cuts clusters short
    check(5, 12, 4000, 6.0, 16, 16, 1 << 28);      // nothing to join
    check(6, 1, 40, 2.0, 256, 960, 1 << 28);       // one atom, few points
    check(7, 3, 0, 2.0, 256, 960, 1 << 28);        // no points
    std::printf("cluster check: all ok\n");
    return 0;
}
