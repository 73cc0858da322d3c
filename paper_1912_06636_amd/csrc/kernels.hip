// HIP kernels for gfx950 (CDNA4): basis evaluation, the two batch contractions on FP64
// MFMA, and the small elementwise / reduction / mirror kernels around them.
//
// Data layout (device memory):
//   - points, weights and w*v in batch order (structure of arrays, FP64);
//   - basis values of an execution unit: [n_points][ld] FP64, point-major, ld a multiple of
//     the 64-wide basis tile, padding columns zero;
//   - D and H dense row-major [N_b][N_b] FP64; n in the caller's point order.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include <hip/hip_runtime.h>

#include "devtypes.h"

namespace nao {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// Pointers into device memory read from the segment tables are generic to the compiler;
// casting them to the global address space makes it emit global (not flat) loads, stores and
// atomics, which are counted by vmcnt only and do not hold up waits for LDS results.
template <typename T> using gp = __attribute__((address_space(1))) T*;
template <typename T> __device__ inline gp<T> gptr(T* p) { return (gp<T>)p; }
__device__ inline void gadd(gp<double> p, double v)
{
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------------------------------
// helpers

template <typename F>
__device__ inline int find_segment(const DevSeg* segs, int n_segs, int64_t b, F prefix_of)
{
    int lo = 0, hi = n_segs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (prefix_of(segs[mid]) <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Workgroup ids are dealt round-robin to the 8 XCDs (each with its own L2).  Items are dealt to
// the XCDs in runs of 2^lg consecutive ones: virtual index v in [0, xcd_span) maps to item
// ((v / 8 / 2^lg) * 8 + v % 8) * 2^lg + (v / 8) % 2^lg, so that the tiles of one execution unit
// mostly share one L2 while every XCD sees units from the whole range.  (One contiguous eighth of
// the list per XCD left CUs idle 31 % of the density launches of a 100-atom block and 38 % of
// the basis launches: eighths at the rim of a structure hold shorter lists.)  Items >= total are
// skipped.
constexpr int N_XCD = 8;
__host__ __device__ inline int64_t xcd_span(int64_t total, int lg)
{
    const int64_t run = (int64_t)N_XCD << lg;
    return (total + run - 1) / run * run;
}
__device__ inline int64_t xcd_item(int64_t v, int lg)
{
    const int64_t q = v / N_XCD;
    return ((((q >> lg) * N_XCD) + v % N_XCD) << lg) + (q & ((1 << lg) - 1));
}
// Runs of at most 2^most items, shorter ones where the launch would otherwise have fewer than
// eight runs per XCD to even out.
static int xcd_run(int64_t total, int most)
{
    int lg = 0;
    while (lg < most && total >> (lg + 7) > 0) ++lg;
    return lg;
}
constexpr int HRUN = 5;  // tile pairs (28 of a unit with 7 tiles): 16 to 64 measure alike, 512 a few percent slower
constexpr int NRUN = 4;  // column tiles (7 to 11 of a unit): runs of 4 cost the 375-atom slab 4 %, 64 gain nothing
constexpr int FRUN = 2;  // of the FP32 forces, whose workgroups hold a CU alone: runs of 4 or 8 measure alike,
                         // 16 cost a 64-atom slab on a small grid 10 % (3.46 against 3.13 ms)

// Lane-uniform values kept in scalar registers: FP64 and FP32 MFMA do not issue beside vector
// instructions (measured: 69 and 31 cycles per MFMA alone, about 3 more for every vector
// instruction between them), so what is uniform is computed by the scalar unit.
__device__ inline int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline int64_t uni(int64_t x)
{
    const uint32_t lo = (uint32_t)uni((int)(uint32_t)x), hi = (uint32_t)uni((int)(uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <typename T> __device__ inline T* uni(T* p) { return reinterpret_cast<T*>(uni((int64_t)(uintptr_t)p)); }

// (dx*dx + dy*dy) + dz*dz without contraction: the same arithmetic that decides relevance.
__device__ inline double dist2_exact(double dx, double dy, double dz)
{
#pragma clang fp contract(off)
    const double xx = dx * dx;
    const double yy = dy * dy;
    const double zz = dz * dz;
    return (xx + yy) + zz;
}

// Real orthonormal spherical harmonics of degree L (<= 3) of a unit vector, m = -L..L, into
// Y[0 .. 2L]; Y_11 ~ +x.
template <int L>
__device__ inline void ylm_l(double x, double y, double z, double* Y)
{
    if constexpr (L == 0) {
        Y[0] = 0.28209479177387814;  // 1 / (2 sqrt(pi))
    } else if constexpr (L == 1) {
        const double c1 = 0.48860251190291992;  // sqrt(3 / (4 pi))
        Y[0] = c1 * y;
        Y[1] = c1 * z;
        Y[2] = c1 * x;
    } else if constexpr (L == 2) {
        const double c2a = 1.0925484305920792;   // sqrt(15 / pi) / 2
        const double c2b = 0.31539156525252005;  // sqrt(5 / pi) / 4
        const double c2c = 0.54627421529603959;  // sqrt(15 / pi) / 4
        Y[0] = c2a * x * y;
        Y[1] = c2a * y * z;
        Y[2] = c2b * (3.0 * z * z - 1.0);
        Y[3] = c2a * x * z;
        Y[4] = c2c * (x * x - y * y);
    } else {
        const double c3a = 0.59004358992664352;  // sqrt(35 / (2 pi)) / 4
        const double c3b = 2.8906114426405538;   // sqrt(105 / pi) / 2
        const double c3c = 0.45704579946446572;  // sqrt(21 / (2 pi)) / 4
        const double c3d = 0.37317633259011546;  // sqrt(7 / pi) / 4
        const double c3e = 1.4453057213202769;   // sqrt(105 / pi) / 4
        Y[0] = c3a * y * (3.0 * x * x - y * y);
        Y[1] = c3b * x * y * z;
        Y[2] = c3c * y * (5.0 * z * z - 1.0);
        Y[3] = c3d * (5.0 * z * z * z - 3.0 * z);
        Y[4] = c3c * x * (5.0 * z * z - 1.0);
        Y[5] = c3e * z * (x * x - y * y);
        Y[6] = c3a * x * (x * x - 3.0 * y * y);
    }
}

// Partial derivatives of the harmonic polynomials of ylm_l (index lm = l^2 + l + m) with respect to
// the three components of the unit vector, taken as independent variables.
__device__ inline void ylm_grad_one(int lm, double x, double y, double z, double* g)
{
    const double c1 = 0.48860251190291992, c2a = 1.0925484305920792, c2b = 0.31539156525252005;
    const double c2c = 0.54627421529603959, c3a = 0.59004358992664352, c3b = 2.8906114426405538;
    const double c3c = 0.45704579946446572, c3d = 0.37317633259011546, c3e = 1.4453057213202769;
    double gx = 0.0, gy = 0.0, gz = 0.0;
    switch (lm) {
    case 1: gy = c1; break;
    case 2: gz = c1; break;
    case 3: gx = c1; break;
    case 4: gx = c2a * y; gy = c2a * x; break;
    case 5: gy = c2a * z; gz = c2a * y; break;
    case 6: gz = 6.0 * c2b * z; break;
    case 7: gx = c2a * z; gz = c2a * x; break;
    case 8: gx = 2.0 * c2c * x; gy = -2.0 * c2c * y; break;
    case 9: gx = 6.0 * c3a * x * y; gy = 3.0 * c3a * (x * x - y * y); break;
    case 10: gx = c3b * y * z; gy = c3b * x * z; gz = c3b * x * y; break;
    case 11: gy = c3c * (5.0 * z * z - 1.0); gz = 10.0 * c3c * y * z; break;
    case 12: gz = c3d * (15.0 * z * z - 3.0); break;
    case 13: gx = c3c * (5.0 * z * z - 1.0); gz = 10.0 * c3c * x * z; break;
    case 14: gx = 2.0 * c3e * x * z; gy = -2.0 * c3e * y * z; gz = c3e * (x * x - y * y); break;
    case 15: gx = 3.0 * c3a * (x * x - y * y); gy = -6.0 * c3a * x * y; break;
    default: break;
    }
    g[0] = gx;
    g[1] = gy;
    g[2] = gz;
}

// ------------------------------------------------------------------------------------------
// Basis evaluation
constexpr int BASIS_ATOMS = 192;   // atoms of a unit staged in LDS
constexpr int BASIS_SHELLS = 128;  // shells of a system staged in LDS
// work items per unit (point slices): rows staged, pairs, and pairs with gradients
constexpr int BASIS_SLICES = 2, BASIS_SLICES_PAIRS = 4, BASIS_SLICES_PLANES = 8;
// waves of a workgroup, as many as its registers allow a CU
constexpr int basis_waves(int extra)
{
    return extra == EXTRA_NONE ? 16 : extra == EXTRA_GRAD ? 12 : 8;
}
constexpr int BASIS_LDS = 160 * 1024, BASIS_STATIC = 13312;  // LDS of a CU, and the kernel's static arrays
// The lines of launch_basis' rule
constexpr double BASIS_ROWS_PAIRS = 4096, BASIS_ROWS_PAIRS_GRAD = 1536;  // atoms of all units together
constexpr double BASIS_ROWS_FEW_ATOMS = 6, BASIS_ROWS_PAIRS_FEW = 2816;  // atoms per unit, and of all then (gradients)
constexpr double BASIS_ROWS_BYTES = 96, BASIS_ROWS_BYTES_GRAD = 64;  // bytes per atom and plane
constexpr double BASIS_ROWS_GLOBAL_FN = 12;    // functions per atom, spline table in global memory
constexpr double BASIS_PLANES_FN = 8;          // functions per atom, eight slices

// N consecutive values of one lane, 16 bytes per store (values are only aligned to their own size).
template <int N, typename T> __device__ inline void store_run(gp<T> dst, const T* v)
{
    constexpr int V = 16 / (int)sizeof(T);
    typedef T vec __attribute__((ext_vector_type(V)));
    typedef vec uvec __attribute__((aligned(sizeof(T))));
    typedef T two __attribute__((ext_vector_type(2)));
    typedef two utwo __attribute__((aligned(sizeof(T))));
    int k = 0;
#pragma unroll
    for (; k + V <= N; k += V) {
        vec x;
#pragma unroll
        for (int j = 0; j < V; ++j) x[j] = v[k + j];
        *reinterpret_cast<gp<uvec>>(dst + k) = x;
    }
    if (V == 4 && k + 2 <= N) {
        *reinterpret_cast<gp<utwo>>(dst + k) = two{v[k], v[k + 1]};
        k += 2;
    }
    if (k < N) dst[k] = v[k];
}

// Basis values of execution units: `slices` workgroups per unit, each taking a contiguous slice of the
// unit's points.  The unit's atoms (position, cutoff, species, first column) and the system's shell
// tables (l, radial function and its parameters) are staged in LDS first, so that a pair's chain of
// table lookups stays on chip; a unit or system larger than the staging arrays reads them from global
// memory instead.  Two ways to the rows of the block, in kernels of their own (ROWS; in one kernel they
// cost each other registers, up to 5 % of the pairs' time):
//   rows_staged: the values go to LDS first, in the place that they have in the row, and leave in full
//   64-byte segments.  A lane that stores its own pair's values makes an L2 request of 12 to 22 bytes
//   out of every 16-byte store, and the L2s, not HBM, bound the launch (100-atom block, FP64, a value
//   and three gradients: 9.7 ms at 2.9 TB/s; staged 5.1 ms at 5.4 TB/s, a fill writes 6.4).  One plane at
//   a time, a wave's LDS being 64 pairs of one plane, which recomputes the radial functions per plane
//   (8 % VALU before, the arithmetic is not what bounds).  Values alone: 3.9 to 3.0 ms (FP64, 14
//   functions per atom), 7.0 to 4.4 ms (slab of 100, FP32, 28 functions).
//   pairs: every lane stores its own.  Less work per value where the runs are short, see launch_basis.
template <typename T, bool SPLINE_LDS, int EX, bool ROWS>
__global__ __launch_bounds__(64 * basis_waves(EX), basis_waves(EX) / 4) void basis_kernel(const DevSeg* __restrict__ segs, int n_segs,
                                                                                           int64_t total, int lg, int slices, int spline_lds, int run)
{
    extern __shared__ __align__(16) double lds_spline[];  // spline table, then four rows of run values per wave
    __shared__ double s_atom[BASIS_ATOMS][4];  // x, y, z, (largest cutoff)^2
    __shared__ int32_t s_aspc[BASIS_ATOMS][2];  // species, first column in the unit
    __shared__ double s_par[BASIS_SHELLS][4];  // rmin, rcut^2, 1/Delta, ln rmin of the shell's radial
    __shared__ int32_t s_shell[BASIS_SHELLS];  // l + 4 (same radial grid as the shell before) + 8 radial function
    __shared__ int32_t s_shptr[BASIS_SHELLS + 1];
    const int tid = threadIdx.x;
    const DevSys* table_of = nullptr;  // the system whose spline table is in LDS
    for (int64_t v_ = blockIdx.x; v_ < xcd_span(total, lg); v_ += gridDim.x) {
        const int64_t bi = xcd_item(v_, lg);
        if (bi >= total) continue;
        // item = (unit, slice): consecutive items split one unit's points
        const int64_t b = bi / slices;
        const int slice = (int)(bi - b * slices);
        __syncthreads();  // the previous item may still read LDS
        const int s = find_segment(segs, n_segs, b, [](const DevSeg& g) { return g.unit_prefix; });
        const DevSeg& sg = segs[s];
        const DevUnit u = sg.units[sg.unit_begin + (b - sg.unit_prefix)];
        const int row0 = (int)(((int64_t)u.n_points * slice) / slices);
        const int row1 = (int)(((int64_t)u.n_points * (slice + 1)) / slices);
        if (row1 <= row0) continue;
        const DevSys* S = sg.sys;
        const int nk = S->n_knots;
        const int na = u.n_atoms, n_sp = S->n_species, n_sh = S->n_shells;
        gp<const double> spl = gptr(S->spline);
        gp<const int32_t> uat = gptr(sg.unit_atoms) + u.atom_begin;
        gp<const int32_t> ucol = gptr(sg.unit_cols) + u.atom_begin;
        gp<const double> axyz = gptr(S->atom_xyzr);
        gp<const int32_t> aspecies = gptr(S->atom_species);
        gp<const int32_t> shell_ptr = gptr(S->species_shell_ptr);
        gp<const int32_t> shell_l = gptr(S->shell_l);
        gp<const int32_t> shell_rad = gptr(S->shell_radial);
        gp<const double> rpar = gptr(S->radial_par);
        const bool staged = na <= BASIS_ATOMS && n_sh <= BASIS_SHELLS && n_sp <= BASIS_SHELLS;  // uniform
        // the table is staged once per workgroup and system (the grid is capped, so that a
        // workgroup takes many items)
        const bool restage = SPLINE_LDS && S != table_of;  // uniform
        if (restage) {
            const int nsp = S->n_radial * nk * 2;
            for (int i = tid; i < nsp; i += blockDim.x) lds_spline[i] = spl[i];
            table_of = S;
        }
        if (staged) {
            for (int ai = tid; ai < na; ai += blockDim.x) {
                const int atom = uat[ai];
#pragma unroll
                for (int k = 0; k < 4; ++k) s_atom[ai][k] = axyz[4 * (int64_t)atom + k];
                s_aspc[ai][0] = aspecies[atom];
                s_aspc[ai][1] = ucol[ai];
            }
            for (int j = tid; j < n_sh; j += blockDim.x) {
                const int rr = shell_rad[j], r0 = shell_rad[max(j - 1, 0)];
                const bool same = rpar[4 * rr] == rpar[4 * r0] && rpar[4 * rr + 2] == rpar[4 * r0 + 2] && rpar[4 * rr + 3] == rpar[4 * r0 + 3];
                s_shell[j] = shell_l[j] + 4 * same + 8 * rr;
#pragma unroll
                for (int k = 0; k < 4; ++k) s_par[j][k] = rpar[4 * rr + k];
            }
            for (int k = tid; k <= n_sp; k += blockDim.x) s_shptr[k] = shell_ptr[k];
        }
        if (restage || staged) __syncthreads();
        gp<T> __restrict__ out = gptr(static_cast<T*>(sg.phi) + u.out_offset);
        // EX = EXTRA_GRAD: the gradient, a plane of values per component; EX = EXTRA_GGA_L: L =
        // (w v / 2) phi + (w a) . grad phi; EX = EXTRA_KS_L: L = (w v / 2) phi - (w / 4) lap phi
        // (+ (w a) . grad phi when the segment has a field); EX = EXTRA_GRAD_H: the gradient, and
        // w h_KS phi = (w v) phi - (w / 2) lap phi (hphi).  All planes are laid out as the values are.
        constexpr bool LAPL = EX == EXTRA_GRAD_H;
        constexpr bool GRAD = EX == EXTRA_GRAD || LAPL, GGA = EX == EXTRA_GGA_L, KS = EX == EXTRA_KS_L;
        const bool field = GGA || (KS && sg.wa != nullptr);  // uniform
        constexpr int NP = 1 + (GRAD ? 3 : EX != EXTRA_NONE) + LAPL;  // planes: values, gradient or L, h phi
        auto plane = [&](int k) {
            return k == 0 ? out : gptr(static_cast<T*>(k == 4 ? sg.hphi : sg.gphi) + (k == 4 ? 0 : (k - 1) * sg.plane) + u.out_offset);
        };
        const int64_t npairs = (int64_t)(row1 - row0) * na;
        const double tmax = (double)(nk - 1);

        // One (point, atom) pair: what its shells share
        struct Pair {
            double d2, r, ir, lnr, x, y, z;
            double hwv, wax, way, waz, qw;
            bool near;
        };
        auto pair_at = [&](int64_t p, double ax, double ay, double az, double arc2) {
            Pair q{};
            const double dx = gptr(S->px)[p] - ax, dy = gptr(S->py)[p] - ay, dz = gptr(S->pz)[p] - az;
            q.d2 = dist2_exact(dx, dy, dz);
            q.near = q.d2 < arc2;  // else every value of the pair is zero, whatever w v is at the point
            // (read for every pair: behind the test the reads would start later, 193 against 205 us)
            if (GGA || KS) q.hwv = 0.5 * gptr(sg.wv)[p];
            if (field) {
                gp<const double> wa = gptr(sg.wa) + 3 * p;
                q.wax = wa[0], q.way = wa[1], q.waz = wa[2];
            }
            if (KS) q.qw = 0.25 * gptr(S->pw)[p];
            if (LAPL) {
                q.hwv = gptr(sg.wv)[p];
                q.qw = 0.5 * gptr(S->pw)[p];
            }
            if (!q.near) q.hwv = q.wax = q.way = q.waz = 0.0;
            q.z = 1.0;
            if (q.near) {
                q.r = sqrt(q.d2);
                if (q.r > 0.0) {
                    q.ir = 1.0 / q.r;
                    q.x = dx * q.ir;
                    q.y = dy * q.ir;
                    q.z = dz * q.ir;
                    q.lnr = log(q.r);
                }
            }
            return q;
        };
        // phi = R Y, grad phi = R'(r) u Y + (R / r) (G - u (u . G)) with G = dY/du (zero where the
        // function is cut off or r <= rmin), lap phi = lap Y
        struct Radial {
            double R, dR, Rr, lap;
        };
        // place on a radial grid: knots k and k + 1 with weights v and w
        struct Knot {
            int k;
            double v, w;
        };
        auto knot_of = [&](const Pair& q, double rmin, double idel, double lnmin) {
            double t = q.r > rmin ? (q.lnr - lnmin) * idel : 0.0;
            t = fmin(fmax(t, 0.0), tmax);
            Knot g;
            g.k = min((int)t, nk - 2);
            g.w = t - (double)g.k;
            g.v = 1.0 - g.w;
            return g;
        };
        auto radial_of = [&](const Pair& q, const Knot& g, int l, int rr, double rmin, double rc2, double idel) {
            Radial f{};
            if (q.near && q.d2 < rc2) {
                const double w = g.w, v = g.v;
                // (y_k, M_k / 6, y_{k+1}, M_{k+1} / 6), 32 contiguous bytes
                const int ci = (rr * nk + g.k) * 2;
                double ya, pa, yb, pb;
                if (SPLINE_LDS) {
                    ya = lds_spline[ci], pa = lds_spline[ci + 1], yb = lds_spline[ci + 2], pb = lds_spline[ci + 3];
                } else {
                    gp<const double> c = spl + ((int64_t)rr * nk + g.k) * 2;
                    ya = c[0], pa = c[1], yb = c[2], pb = c[3];
                }
                f.R = v * (ya + (v * v - 1.0) * pa) + w * (yb + (w * w - 1.0) * pb);
                if (EX != EXTRA_NONE && q.r > rmin) {
                    // dR/dr = dR/dt dt/dr with dt/dr = 1 / (r Delta); the clamped part r <= rmin is constant
                    const double dS = (yb - ya) - (3.0 * v * v - 1.0) * pa + (3.0 * w * w - 1.0) * pb;  // dR/dt
                    f.dR = dS * idel * q.ir;
                    f.Rr = f.R * q.ir;
                    // lap phi = (S''/Delta^2 + S'/Delta - l(l+1) S) Y / r^2 in the spline variable
                    const double d2S = 6.0 * (v * pa + w * pb);  // d2R/dt2
                    if (KS || LAPL) f.lap = ((d2S * idel + dS) * idel - (double)(l * (l + 1)) * f.R) * q.ir * q.ir;
                }
            }
            return f;
        };
        // the 2 L + 1 values of plane P of a shell
        auto shell_values = [&](auto which, auto deg, const Pair& q, const Radial& f, T* val) {
            constexpr int P = decltype(which)::value, L = decltype(deg)::value, NF = 2 * L + 1;
            // harmonics and their derivatives per shell: left to itself the compiler takes those of
            // all degrees out of the loop over the shells, some 60 values that then spill
            double x = q.x, y = q.y, z = q.z;
            asm volatile("" : "+v"(x), "+v"(y), "+v"(z));
            double Y[NF];
            ylm_l<L>(x, y, z, Y);
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                if constexpr (P == 0) {
                    val[i] = T(f.R * Y[i]);
                } else if constexpr (P == 4) {
                    val[i] = T(q.hwv * (f.R * Y[i]) - q.qw * (f.lap * Y[i]));
                } else {
                    double g[3] = {};
                    if (GRAD || field) {
                        double gv[3];
                        ylm_grad_one(L * L + i, x, y, z, gv);
                        const double ug = (x * gv[0] + y * gv[1]) + z * gv[2];
                        g[0] = f.dR * x * Y[i] + f.Rr * (gv[0] - x * ug);
                        g[1] = f.dR * y * Y[i] + f.Rr * (gv[1] - y * ug);
                        g[2] = f.dR * z * Y[i] + f.Rr * (gv[2] - z * ug);
                    }
                    if constexpr (GRAD) val[i] = T(g[P - 1]);
                    else val[i] = T((q.hwv * (f.R * Y[i]) - q.qw * (f.lap * Y[i])) + ((q.wax * g[0] + q.way * g[1]) + q.waz * g[2]));
                }
            }
        };
        // planes 0 .. NP - 1, h phi being plane 4
        auto each_plane = [&](auto&& fn) {
            fn(std::integral_constant<int, 0>{});
            if constexpr (NP > 1) fn(std::integral_constant<int, 1>{});
            if constexpr (NP > 3) fn(std::integral_constant<int, 2>{});
            if constexpr (NP > 3) fn(std::integral_constant<int, 3>{});
            if constexpr (NP > 4) fn(std::integral_constant<int, 4>{});
        };
        auto by_degree = [&](int l, auto&& fn) {
            switch (l) {
            case 0: fn(std::integral_constant<int, 0>{}); break;
            case 1: fn(std::integral_constant<int, 1>{}); break;
            case 2: fn(std::integral_constant<int, 2>{}); break;
            default: fn(std::integral_constant<int, 3>{}); break;
            }
        };
        // Threads over pairs, each storing its own values (units or systems past the staging arrays,
        // and functions per atom past the row stage)
        auto pairs = [&](auto on_chip) {
            constexpr bool ST = decltype(on_chip)::value;
            for (int64_t e = tid; e < npairs; e += blockDim.x) {
                const int pq = (int)e / na;
                const int ai = (int)e - pq * na;
                const int pl = row0 + pq;
                const int atom = ST ? 0 : uat[ai];
                gp<const double> xyzr = axyz + 4 * (int64_t)atom;
                const Pair q = ST ? pair_at(u.point_begin + pl, s_atom[ai][0], s_atom[ai][1], s_atom[ai][2], s_atom[ai][3])
                                  : pair_at(u.point_begin + pl, xyzr[0], xyzr[1], xyzr[2], xyzr[3]);
                const int sp = ST ? s_aspc[ai][0] : aspecies[atom];
                const int sh0 = ST ? s_shptr[sp] : shell_ptr[sp];
                const int sh1 = ST ? s_shptr[sp + 1] : shell_ptr[sp + 1];
                int64_t at = (int64_t)pl * u.ld + (ST ? s_aspc[ai][1] : ucol[ai]);
                for (int j = sh0; j < sh1; ++j) {
                    const int l = ST ? s_shell[j] & 3 : shell_l[j];
                    const int rr = ST ? s_shell[j] >> 3 : shell_rad[j];
                    const double rmin = ST ? s_par[j][0] : rpar[4 * rr], rc2 = ST ? s_par[j][1] : rpar[4 * rr + 1];
                    const double idel = ST ? s_par[j][2] : rpar[4 * rr + 2], lnmin = ST ? s_par[j][3] : rpar[4 * rr + 3];
                    const Radial f = radial_of(q, knot_of(q, rmin, idel, lnmin), l, rr, rmin, rc2, idel);
                    by_degree(l, [&](auto deg) {
                        constexpr int NF = 2 * decltype(deg)::value + 1;
                        each_plane([&](auto which) {
                            T val[NF];
                            shell_values(which, deg, q, f, val);
                            store_run<NF>(plane(decltype(which)::value) + at, val);
                        });
                        at += NF;
                    });
                }
            }
        };
        // A wave takes 16 neighbouring atoms of four points, plane by plane: every lane puts the values of
        // its pair where they belong in the run of columns that the atoms have in each row, and the runs
        // are copied out by 16 bytes per lane from 64-byte boundaries.  Where the unit's atoms split evenly
        // into parts of 12 or fewer the wave takes such a part of five or more points: 16 left 11 of 16
        // lanes idle with five atoms (6-atom slab, FP64, a value and three gradients: 400 to 264 us; 45
        // atoms: 4.6 to 4.0 ms).
        auto rows_staged = [&]() {
            constexpr int V = 16 / (int)sizeof(T), SEG = 64 / (int)sizeof(T);
            typedef T vec __attribute__((ext_vector_type(V)));
            const int lane = tid & 63, wave = uni(tid >> 6), waves = (int)blockDim.x >> 6;
            T* win = reinterpret_cast<T*>(lds_spline + spline_lds) + wave * 4 * run;
            const int parts = (na + 15) >> 4, even = (na + parts - 1) / max(parts, 1), per = even <= 12 ? max(even, 1) : 16;
            // a row of the window: `per` atoms from up to a segment on (run is that of 16)
            const int wrow = ((run - SEG) / 16 * per + V - 1) / V * V + SEG, R = min(64 / per, 4 * run / wrow);
            const int rl = lane / per, al = lane - rl * per;
            const int tasks = (row1 - row0 + R - 1) / R * parts;
            for (int task = wave; task < tasks; task += waves) {
                const int part = task % parts, rowb = row0 + R * (task / parts);
                const int c0 = uni(s_aspc[per * part][1]), c1 = part + 1 < parts ? uni(s_aspc[per * part + per][1]) : u.m;
                const int ai = per * part + al;
                const bool mine = ai < na && rl < R && rowb + rl < row1;
                const int pl = min(rowb + rl, row1 - 1), aj = min(ai, na - 1);
                const Pair q = pair_at(u.point_begin + pl, s_atom[aj][0], s_atom[aj][1], s_atom[aj][2], s_atom[aj][3]);
                const int sp = s_aspc[aj][0];
                const bool any = __any(mine && q.near);  // else zeros throughout
                const int sh0 = s_shptr[sp], sh1 = mine && any ? s_shptr[sp + 1] : sh0;
                each_plane([&](auto which) {
                    gp<T> dst = plane(decltype(which)::value) + (int64_t)rowb * u.ld + c0;
                    // values by which a row's run starts past a 64-byte boundary
                    auto past = [&](int r) { return (int)(reinterpret_cast<uintptr_t>(dst + (int64_t)r * u.ld) / sizeof(T)) & (SEG - 1); };
                    T* at = win + rl * wrow + past(rl) + (s_aspc[aj][1] - c0);
                    Knot g{};
                    for (int j = sh0; j < sh1; ++j) {
                        const int sh = s_shell[j], l = sh & 3;
                        if (j == sh0 || !(sh & 4)) g = knot_of(q, s_par[j][0], s_par[j][2], s_par[j][3]);
                        const Radial f = radial_of(q, g, l, sh >> 3, s_par[j][0], s_par[j][1], s_par[j][2]);
                        by_degree(l, [&](auto deg) {
                            constexpr int NF = 2 * decltype(deg)::value + 1;
                            T val[NF];
                            shell_values(which, deg, q, f, val);
#pragma unroll
                            for (int i = 0; i < NF; ++i) at[i] = val[i];
                            at += NF;
                        });
                    }
                    // the wave's own LDS writes are performed before its later reads (in order)
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    const int n_rows = min(R, row1 - rowb);
                    // row r by `step` lanes, the first of them at its value i0
                    auto copy_row = [&](int r, int i0, int step) {
                        const int b0 = past(r), b1 = b0 + c1 - c0;
                        const T* src = win + r * wrow;
                        gp<T> to = dst + (int64_t)r * u.ld - b0;
                        for (int i = i0; i < b1; i += step) {
                            vec x = *reinterpret_cast<const vec*>(src + i);
                            if (!any) x = vec(T(0));
                            if (i >= b0 && i + V <= b1) {
                                *reinterpret_cast<gp<vec>>(to + i) = x;
                            } else {
#pragma unroll
                                for (int k = 0; k < V; ++k)
                                    if (i + k >= b0 && i + k < b1) to[i + k] = x[k];
                            }
                        }
                    };
                    if (R <= 4) {
                        for (int r = 0; r < n_rows; ++r) copy_row(r, lane * V, 64 * V);
                    } else {  // short runs: 2, 4, ... rows at a time
                        int lg = 2;
                        while (lg < 6 && V << lg < c1 - c0 + SEG - V) ++lg;
                        for (int r = lane >> lg; r < n_rows; r += 64 >> lg) copy_row(r, (lane & ((1 << lg) - 1)) * V, V << lg);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                });
            }
        };
        if constexpr (ROWS) {
            if (staged) rows_staged();
            else pairs(std::false_type{});
        } else {
            if (staged) pairs(std::true_type{});
            else pairs(std::false_type{});
        }
        if (slice == slices - 1 && u.n_rows > u.n_points) {  // padding rows of a cluster's unit
            const int64_t z0 = (int64_t)u.n_points * u.ld, z1 = (int64_t)u.n_rows * u.ld;
            for (int64_t q = z0 + tid; q < z1; q += blockDim.x) each_plane([&](auto which) { plane(decltype(which)::value)[q] = T(0); });
        }
        const int pad = u.ld - u.m;
        if (pad > 0) {
            const int64_t ne = (int64_t)(row1 - row0) * pad;
            for (int64_t q = tid; q < ne; q += blockDim.x) {
                const int64_t pl = row0 + q / pad;
                const int64_t at = pl * u.ld + u.m + (q - (pl - row0) * pad);
                each_plane([&](auto which) { plane(decltype(which)::value)[at] = T(0); });
            }
        }
    }
}

static unsigned grid_for(int64_t n, int lg, int64_t max_grid)
{
    const int64_t span = xcd_span(n, lg);
    if (max_grid > 0) {
        const int64_t cap = std::max<int64_t>(N_XCD, max_grid / N_XCD * N_XCD);
        if (span > cap) return (unsigned)cap;
    }
    return (unsigned)span;
}

hipError_t launch_basis(const DevSeg* segs_dev, int n_segs, int64_t n_units, int spline_lds, const BasisShape& shape,
                        bool fp32_out, hipStream_t st, int64_t max_grid, int extra)
{
    if (n_units <= 0 || n_segs <= 0) return hipSuccess;
    if (n_units > 0x7ffffff0 / BASIS_SLICES_PAIRS || spline_lds < 0 || spline_lds > MAX_SPLINE_LDS || shape.max_fn < 0)
        return hipErrorInvalidValue;
    if (extra != EXTRA_NONE && extra != EXTRA_GRAD && extra != EXTRA_GGA_L && extra != EXTRA_KS_L &&
        extra != EXTRA_GRAD_H)
        return hipErrorInvalidValue;
    static std::atomic<int> n_cu{0};
    if (n_cu.load() == 0) {
        int dev = 0, cu = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cu > 0)
            n_cu.store(cu);
    }
    const int cus = std::max(1, n_cu.load());
    // Rows are staged where the LDS left by the spline table holds those of four waves or more, and
    // where their longer way pays (all figures FP64 unless said; rows against pairs, us):
    //   - not in launches of little work, counted by the atoms of all units.  Values: 5 atoms and 28
    //     functions each, 510 units (2,500 atoms) 66 against 46; 8 atoms, 472 units (3,700) 54 against
    //     58; 10 atoms, 590 units (5,600) 68 against 73; 14 atoms 114 against 136.  L: 3,700 121 against
    //     112, 10,700 266 against 258, 45-atom slab 2.5 ms against 4.0.  Gradients gain earlier: 1,100
    //     atoms 84 against 64, 1,700 88 against 116, 2,300 189 against 207, 3,700 163 against 227; units
    //     of 5 atoms later: 1,900 188 against 172, 2,500 187 against 140, 3,000 264 against 319;
    //   - not for short runs: 5 functions per atom 100 against 63, 9.5 of them 0.28 ms against 0.25; 14
    //     FP32 ones 0.77 against 0.72.  Gradients: 5 functions 115 against 72, 9.5 0.80 ms against 1.37;
    //     14 FP32 ones 402 against 299;
    //   - with the table in global memory and 14 functions per atom FP32 gradients gain all the same:
    //     36 radial functions, 60 atoms, 2.9 ms against 4.2;
    //   - not for L in FP32, two planes with the arithmetic of four (2.3 ms against 2.0).
    // Pairs with gradients store a plane at a time.  Where four slices of every unit are more than run
    // at once, eight leave a shorter last round (4 atoms 72 to 63, FP32 594 to 526 for 9.5 functions per
    // atom; where they all run at once 27 against 31 with eight), but not for 5 functions (139 against 150).
    const int size = fp32_out ? sizeof(float) : sizeof(double), most = basis_waves(extra);
    const int64_t table = 8 * (int64_t)spline_lds, room = BASIS_LDS - BASIS_STATIC - table;
    const int64_t run = 16 * (int64_t)shape.max_fn + 64 / size;
    const int fit = (int)std::min<int64_t>(most, room / (4 * run * size));
    const bool grad = extra == EXTRA_GRAD || extra == EXTRA_GRAD_H;
    const double pairs = n_units * shape.mean_atoms, bytes = shape.mean_fn * size;
    const double least = !grad ? BASIS_ROWS_PAIRS : shape.mean_atoms < BASIS_ROWS_FEW_ATOMS ? BASIS_ROWS_PAIRS_FEW : BASIS_ROWS_PAIRS_GRAD;
    const bool rows = fit >= 4 && pairs >= least &&
                      (bytes >= (grad ? BASIS_ROWS_BYTES_GRAD : BASIS_ROWS_BYTES) || (grad && table == 0 && shape.mean_fn >= BASIS_ROWS_GLOBAL_FN)) &&
                      !(fp32_out && (extra == EXTRA_GGA_L || extra == EXTRA_KS_L));
    const int64_t at_once = cus * std::max<int64_t>(1, std::min<int64_t>(most / 4, BASIS_LDS / (table + BASIS_STATIC)));
    const bool fine = grad && shape.mean_fn >= BASIS_PLANES_FN && n_units * BASIS_SLICES_PAIRS > at_once &&
                      n_units <= 0x7ffffff0 / BASIS_SLICES_PLANES;
    const int waves = rows ? fit : 4, slices = rows ? BASIS_SLICES : fine ? BASIS_SLICES_PLANES : BASIS_SLICES_PAIRS;
    const int64_t n_items = n_units * slices;
    const size_t lds = (size_t)(table + (rows ? waves * 4 * run * size : 0));
    // as many workgroups as fit the chip at once (LDS and registers): each takes many items and
    // stages its spline table once
    if (max_grid <= 0)
        max_grid = cus * std::max<int64_t>(1, std::min<int64_t>(most / waves, BASIS_LDS / ((int64_t)lds + BASIS_STATIC)));
    const dim3 g(grid_for(n_items, 2, max_grid)), b(64 * waves);
    const bool staged = spline_lds > 0;
    // dynamic LDS above 64 KiB must be allowed per kernel, once per device
    static std::atomic<uint64_t> attrs_set{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attrs_set.load() & bit)) {
#define NAO_BASIS_FNS(TT, EE)                                                                                     \
    reinterpret_cast<const void*>(&basis_kernel<TT, true, EE, true>), reinterpret_cast<const void*>(&basis_kernel<TT, false, EE, true>), \
        reinterpret_cast<const void*>(&basis_kernel<TT, true, EE, false>), reinterpret_cast<const void*>(&basis_kernel<TT, false, EE, false>)
#define NAO_BASIS_TYPE(TT)                                                                                        \
    NAO_BASIS_FNS(TT, EXTRA_NONE), NAO_BASIS_FNS(TT, EXTRA_GRAD), NAO_BASIS_FNS(TT, EXTRA_GGA_L),                 \
        NAO_BASIS_FNS(TT, EXTRA_KS_L), NAO_BASIS_FNS(TT, EXTRA_GRAD_H)
        const void* fns[] = {NAO_BASIS_TYPE(float), NAO_BASIS_TYPE(double)};
#undef NAO_BASIS_TYPE
#undef NAO_BASIS_FNS
        for (const void* f : fns) {
            const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, BASIS_LDS - BASIS_STATIC);
            if (e != hipSuccess) return e;
        }
        attrs_set.fetch_or(bit);
    }
#define NAO_BASIS_ROWS(TT, SS, EE)                                                                                \
    do {                                                                                                          \
        if (rows) hipLaunchKernelGGL((basis_kernel<TT, SS, EE, true>), g, b, lds, st, segs_dev, n_segs, n_items, 2, slices, spline_lds, (int)run); \
        else hipLaunchKernelGGL((basis_kernel<TT, SS, EE, false>), g, b, lds, st, segs_dev, n_segs, n_items, 2, slices, spline_lds, 0); \
    } while (0)
#define NAO_BASIS_LAUNCH(TT, EE)                                                                                  \
    do {                                                                                                          \
        if (staged) NAO_BASIS_ROWS(TT, true, EE);                                                                 \
        else NAO_BASIS_ROWS(TT, false, EE);                                                                       \
    } while (0)
#define NAO_BASIS_EXTRA(TT)                                           \
    do {                                                              \
        if (extra == EXTRA_GRAD) NAO_BASIS_LAUNCH(TT, EXTRA_GRAD);    \
        else if (extra == EXTRA_GGA_L) NAO_BASIS_LAUNCH(TT, EXTRA_GGA_L); \
        else if (extra == EXTRA_KS_L) NAO_BASIS_LAUNCH(TT, EXTRA_KS_L); \
        else if (extra == EXTRA_GRAD_H) NAO_BASIS_LAUNCH(TT, EXTRA_GRAD_H); \
        else NAO_BASIS_LAUNCH(TT, EXTRA_NONE);                        \
    } while (0)
    if (fp32_out) NAO_BASIS_EXTRA(float);
    else NAO_BASIS_EXTRA(double);
#undef NAO_BASIS_EXTRA
#undef NAO_BASIS_LAUNCH
#undef NAO_BASIS_ROWS
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Contractions with one value per lane per operand: FP64 (v_mfma_f64_16x16x4f64) and FP32
// (v_mfma_f32_16x16x4f32).  Operand layouts of both: A lane l holds A[l%16][l/16], B lane l
// holds B[l/16][l%16].  The result register r of lane l is D[l/16 + 4r][l%16] for FP64 and
// D[4(l/16) + r][l%16] for FP32 (measured on gfx950).

// Sum over the 16 lanes of each DPP row (lanes 16 r .. 16 r + 15), every lane receiving the sum:
// quad swaps (xor 1, xor 2), then the half-row and row mirrors pair the quads.
template <int CTRL>
__device__ inline double dpp_move(double x)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ inline double row_sum16(double v)
{
    v += dpp_move<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_move<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_move<0x141>(v);  // row_half_mirror
    v += dpp_move<0x140>(v);  // row_mirror
    return v;
}

template <typename T> struct Mma;
template <> struct Mma<double> {
    typedef d4 acc_t;
    static __device__ inline acc_t zero() { return d4{0.0, 0.0, 0.0, 0.0}; }
    static __device__ inline acc_t op(double a, double b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lk, int r) { return lk + 4 * r; }
};
template <> struct Mma<float> {
    typedef f4 acc_t;
    static __device__ inline acc_t zero() { return f4{0.f, 0.f, 0.f, 0.f}; }
    static __device__ inline acc_t op(float a, float b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lk, int r) { return 4 * lk + r; }
};

// ------------------------------------------------------------------------------------------
// Parts shared by the tile kernels of H below.

// A raw buffer over [p, p + bytes): loads beyond its end return zeros.
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void* p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}
// One wave load from a buffer straight into LDS, 16 or 4 bytes per lane to dst + lane * 16 or 4.
__device__ inline void load16_to_lds(__amdgpu_buffer_rsrc_t r, void* dst, int voffset, int soffset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, voffset, soffset, 0, 0);
}
__device__ inline void load4_to_lds(__amdgpu_buffer_rsrc_t r, void* dst, int voffset, int soffset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 4, voffset, soffset, 0, 0);
}
// One FP64 or FP32 value per lane from a buffer.
template <typename T> __device__ inline T load_value(__amdgpu_buffer_rsrc_t r, int voffset)
{
    if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voffset, 0, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voffset, 0, 0));
}
// Wait until at most N of this wave's vector loads are outstanding and its LDS reads are done.
template <int N> __device__ inline void wait_loads() { __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4)); }

// Hamiltonian, per work item one 64x64 tile pair (I <= J) of a unit:
//   TWO = false: H[I, J] += (w v Phi[:, I])^T Phi[:, J];
//   TWO = true:  H[I, J] += Phi_I^T L_J + L_I^T Phi_J, with L written by the basis launch (a vector
//                field or the kinetic term).
// K = the unit's points in chunks of KC, held in an S-stage ring in LDS that is filled by direct
// buffer loads (16 bytes per lane, rows beyond the unit's last point read as zeros).  Four waves,
// each a strip of 16 rows by 64 columns as four 16x16 MFMA blocks.
//
// Bound: the matrix pipes, which share their issue slots with the vector instructions, so the loop
// has next to none: uniform addresses are scalar, LDS addresses are per-lane constants plus
// immediate stage offsets (the ring is unrolled), and w v costs one multiplication per four MFMAs.
// unit_mask holds, per 16 columns, which 16-point chunks of the unit any of their functions
// reaches: chunks that reach only one of the two tiles are not loaded, and 16x16 blocks that a
// chunk cannot change skip its MFMAs (they would add zeros).  The strip of a wave rotates with the
// item, so that the blocks below the diagonal, left out, do not idle the same SIMD in every item.
// Measured, kernel alone, against the form with register math in its loop (6.7 vector instructions
// per MFMA): 100-atom block FP64 7.45 -> 6.5 ms, 375-atom slab 113 -> 98 ms; with L 12.6 -> 10.0 ms.
// Two stages and four workgroups per CU measure 2 % faster than three and three.
template <typename T, int KC, int S, bool TWO>
__global__ __launch_bounds__(256, TWO ? 3 : 4) void h_tiles(const DevSeg* __restrict__ segs, int n_segs, int64_t total, int lg)
{
    typedef Mma<T> M;
    constexpr int NOP = TWO ? 4 : 2;                    // tiles of a stage: Phi_I, Phi_J, then L_I, L_J
    constexpr int ROWB = TILE * (int)sizeof(T);         // bytes of a tile row
    constexpr int TILEB = KC * ROWB, STAGEB = NOP * TILEB;
    constexpr int SPR = ROWB / 16;                      // 16-byte slots per row
    constexpr int RPL = 64 / SPR;                       // rows per wave load
    constexpr int LOADS = KC / RPL / 4;                 // wave loads per tile, wave and chunk
    static_assert(LOADS >= 1 && (KC == 8 || KC == 16) && (S == 2 || S == 3), "chunk geometry");
    constexpr int WV = S * STAGEB, FN = WV + (TWO ? 0 : MAX_CLUSTER_ROWS * 8);
    __shared__ __align__(16) unsigned char lds[FN + 2 * TILE * 4];  // ring | w v | row and column indices
    const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    const int lr = lane & 15, lk = lane >> 4;
    // FP32 rows are half a bank period long: odd rows have their 64-byte halves swapped, so that the
    // two rows a read of 32 lanes touches fall in distinct banks
    const int swz = sizeof(T) == 4 ? (lk & 1) * 64 : 0;
    for (int64_t v_ = blockIdx.x; v_ < xcd_span(total, lg); v_ += gridDim.x) {
        const int64_t b = xcd_item(v_, lg);
        if (b >= total) continue;
        const int s = find_segment(segs, n_segs, b, [](const DevSeg& g) { return g.item_prefix; });
        const DevSeg& sg = segs[s];
        const HItem it = static_cast<const HItem*>(sg.items)[sg.item_begin + (b - sg.item_prefix)];
        const int ti = uni((int)it.ti), tj = uni((int)it.tj);
        const DevUnit* up = sg.item_units + uni(it.unit);
        const int np = uni(up->n_rows), ld = uni(up->ld), m = uni(up->m);
        const int64_t out_offset = uni(up->out_offset), row_begin = uni(up->row_begin);
        const int64_t fn_begin = uni(up->fn_begin), mask_begin = uni(up->mask_begin);
        uint64_t sub_first = sizeof(T) == 4 ? (uint64_t)uni((int64_t)up->sub_first) : 0;
        const uint64_t* mI = sg.unit_mask + mask_begin + 4 * ti;
        const uint64_t* mJ = sg.unit_mask + mask_begin + 4 * tj;
        uint64_t any_i = 0, any_j = 0, mj[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            any_i |= (uint64_t)uni((int64_t)mI[q]);
            any_j |= mj[q] = (uint64_t)uni((int64_t)mJ[q]);
        }
        uint64_t todo = any_i & any_j;  // 16-row chunks both tiles reach
        if (todo == 0) continue;        // none
        const bool diag = ti == tj;
        const int strip = (wave + tj) & 3;
        const uint64_t ma = (uint64_t)uni((int64_t)mI[strip]);
        uint64_t mm[4];  // chunks that change this wave's block jb (none below the diagonal)
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) mm[jb] = diag && jb < strip ? 0 : ma & mj[jb];
        const uint64_t m_any = mm[0] | mm[1] | mm[2] | mm[3];

        const char* phi = static_cast<const char*>(sg.phi) + out_offset * (int)sizeof(T);
        const char* lv = TWO ? static_cast<const char*>(sg.gphi) + out_offset * (int)sizeof(T) : nullptr;
        const int ldb = ld * (int)sizeof(T);
        const int I0b = ti * ROWB, J0b = tj * ROWB;
        // every wave must be done reading the previous item's LDS
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (!TWO) {  // w v of the rows, zeros beyond the last one
            const __amdgpu_buffer_rsrc_t r = buffer_of(sg.wv + row_begin, np * 8);
            for (int q = wave; 32 * q < np; q += 4) load4_to_lds(r, lds + WV + q * 256, 4 * lane + q * 256, 0);
        }
        if (wave < 2)  // global indices of the tile's rows and columns
            load4_to_lds(buffer_of(sg.unit_fn + fn_begin, m * 4), lds + FN + wave * TILE * 4,
                           4 * ((wave ? tj : ti) * TILE + lane), 0);
        int voff[LOADS];  // this lane's 16 bytes of every wave load, within a chunk's rows
#pragma unroll
        for (int q = 0; q < LOADS; ++q) {
            const int row = (wave * LOADS + q) * RPL + lane / SPR;
            voff[q] = row * ldb + (((lane % SPR) * 16) ^ (sizeof(T) == 4 ? (row & 1) * 64 : 0));
        }
        // a chunk of 16 rows is taken in steps of KC: step h of chunk c
        constexpr int STEPS = 16 / KC;
        auto issue = [&](int c, int h, int stg) {
            const int row = c * 16 + h * KC;
            const int64_t o = (int64_t)row * ldb;
            const int bytes = max(0, np - row) * ldb;
#pragma unroll
            for (int op = 0; op < NOP; ++op) {
                if ((op & 1) && diag) continue;
                const __amdgpu_buffer_rsrc_t r = buffer_of((op < 2 ? phi : lv) + o, bytes);
#pragma unroll
                for (int q = 0; q < LOADS; ++q)
                    load16_to_lds(r, lds + stg * STAGEB + op * TILEB + (wave * LOADS + q) * 1024, voff[q], op & 1 ? J0b : I0b);
            }
        };
        // per-lane LDS offsets of the operands: row lk of a stage's tiles
        const int a_off = lk * ROWB + ((strip * 16 * (int)sizeof(T)) ^ swz) + lr * (int)sizeof(T);
        const int b_tile = diag ? 0 : TILEB;
        int b_off[2];
        b_off[0] = b_tile + lk * ROWB + swz + lr * (int)sizeof(T);
        b_off[1] = b_tile + lk * ROWB + ((16 * (int)sizeof(T)) ^ swz) + lr * (int)sizeof(T);

        typename M::acc_t acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = M::zero();
        // FP32: the sums of a unit move to FP64 when the next one starts
        d4 acc64[sizeof(T) == 4 ? 4 : 1] = {};
        auto flush = [&]() {
            if constexpr (sizeof(T) == 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc64[j][r] += (double)acc[j][r];
                    acc[j] = M::zero();
                }
        };
        auto compute = [&](int c, int h, int stg) {
            if (__builtin_expect(!((m_any >> c) & 1), 0)) return;
            if (sizeof(T) == 4) {
                const uint64_t past = sub_first & ((2ull << c) - 1);
                if (past) {
                    flush();
                    sub_first &= ~past;
                }
            }
            constexpr int KK = KC / 4;
            const unsigned char* base = lds + stg * STAGEB;
            T a[KK], bv[4][KK], a2[TWO ? KK : 1], b2[TWO ? 4 : 1][KK];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const T x = *reinterpret_cast<const T*>(base + a_off + kk * 4 * ROWB);
                if (TWO) a[kk] = x, a2[kk] = *reinterpret_cast<const T*>(base + a_off + 2 * TILEB + kk * 4 * ROWB);
                else a[kk] = T((double)x * *reinterpret_cast<const double*>(lds + WV + lk * 8 + (c * 16 + h * KC + kk * 4) * 8));
#pragma unroll
                for (int jb = 0; jb < 4; ++jb) {
                    const unsigned char* q = base + b_off[jb & 1] + (jb & 2) * 16 * (int)sizeof(T) + kk * 4 * ROWB;
                    // the factors of Phi_I are L_J, those of L_I are Phi_J
                    bv[jb][kk] = *reinterpret_cast<const T*>(q + (TWO ? 2 * TILEB : 0));
                    if (TWO) b2[jb][kk] = *reinterpret_cast<const T*>(q);
                }
            }
            // block by block, four dependent MFMAs each: the other waves of the SIMD fill their
            // latency, and the accumulators stay where they are on every path
#pragma unroll
            for (int jb = 0; jb < 4; ++jb)
                if (__builtin_expect((mm[jb] >> c) & 1, 1))
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) {
                        acc[jb] = M::op(a[kk], bv[jb][kk], acc[jb]);
                        if (TWO) acc[jb] = M::op(a2[kk], b2[jb][kk], acc[jb]);
                    }
        };
        uint64_t ahead = todo;
        int ah = 0, th = 0;  // steps of the chunks at the front of ahead and todo
        auto issue_next = [&](int stg) {
            issue(__builtin_ctzll(ahead), ah, stg);
            if (++ah == STEPS) {
                ah = 0;
                ahead &= ahead - 1;
            }
        };
#pragma unroll
        for (int k = 0; k < S - 1; ++k)
            if (ahead) issue_next(k);
        // per step: its loads (every wave's) have landed and every wave is done with the stage that
        // is refilled next
        while (todo) {
#pragma unroll
            for (int stg = 0; stg < S; ++stg) {
                const int c = __builtin_ctzll(todo), h = th;
                if (++th == STEPS) {
                    th = 0;
                    todo &= todo - 1;
                }
                if (S == 2 || todo == 0) wait_loads<0>();
                else if (diag) wait_loads<LOADS * NOP / 2>();
                else wait_loads<LOADS * NOP>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (__builtin_expect(ahead != 0, 1)) issue_next((stg + S - 1) % S);
                compute(c, h, stg);
                if (todo == 0) break;
            }
        }
        if (m_any == 0) continue;
        // pairs of a cluster's columns are not ordered by their global indices, so a pair's sum may
        // go above or below the diagonal of H; the mirror adds the two
        const int32_t* gi = reinterpret_cast<const int32_t*>(lds + FN);
        gp<double> __restrict__ H = gptr(sg.H);
        const int64_t ldh = sg.ld;
        const int row0 = strip * 16, I0 = ti * TILE, J0 = tj * TILE;
        gp<double> Hr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) Hr[r] = H + (int64_t)gi[row0 + M::row(lk, r)] * ldh;
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            if (!mm[jb]) continue;  // no chunk reaches this block
            const int32_t gj = gi[TILE + jb * 16 + lr];
            const bool whole = I0 + row0 + 16 <= m && J0 + jb * 16 + 16 <= m && !(diag && jb == strip);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = row0 + M::row(lk, r), col = jb * 16 + lr;
                if (whole || (I0 + row < m && J0 + col < m && (!diag || row <= col))) gadd(Hr[r] + gj, sizeof(T) == 4 ? acc64[sizeof(T) == 4 ? jb : 0][r] + (double)acc[jb][r] : (double)acc[jb][r]);
            }
        }
    }
}

// Hamiltonian with 128x128 tile pairs: eight waves, each a 32x64 block (2x4 MFMA blocks), so
// that every staged basis value feeds twice as many MFMAs as in the 64-wide kernel.  Chunks
// of 16 points, double-buffered as above.
constexpr int WTILE = 128;

template <typename T>
__global__ __launch_bounds__(512) void h_kernel_wide(const DevSeg* __restrict__ segs, int n_segs, int64_t total, int lg)
{
    typedef Mma<T> M;
    __shared__ T As[2][KCHUNK][WTILE + 2];
    __shared__ T Bs[2][KCHUNK][WTILE + 2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave >> 1, wc = wave & 1;  // rows 32 wr .. 32 wr + 31, columns 64 wc .. 64 wc + 63
    const int lr = lane & 15, lk = lane >> 4;
    for (int64_t v_ = blockIdx.x; v_ < xcd_span(total, lg); v_ += gridDim.x) {
        const int64_t b = xcd_item(v_, lg);
        if (b >= total) continue;
        const int s = find_segment(segs, n_segs, b, [](const DevSeg& g) { return g.item_prefix; });
        const DevSeg& sg = segs[s];
        const HItem it = static_cast<const HItem*>(sg.items)[sg.item_begin + (b - sg.item_prefix)];
        const DevUnit u = sg.item_units[it.unit];
        gp<const T> __restrict__ phi = gptr(static_cast<const T*>(sg.phi) + u.out_offset);
        gp<const double> __restrict__ wv = gptr(sg.wv + u.point_begin);
        const int np = u.n_points, ld = u.ld;
        const int I0 = it.ti * WTILE, J0 = it.tj * WTILE;
        const int n_chunks = (np + KCHUNK - 1) / KCHUNK;

        if (np <= 0) continue;
        T ra[4], rb[4];
        double rw[4];
        auto fetch = [&](int c) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = tid + 512 * q;
                const int pc = min(c * KCHUNK + (e >> 7), np - 1), col = e & 127;
                gp<const T> rowp = phi + (int64_t)pc * ld;
                ra[q] = rowp[I0 + col];
                rb[q] = rowp[J0 + col];
                rw[q] = wv[pc];
            }
        };
        auto stash = [&](int c, int buf) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = tid + 512 * q;
                const bool ok = c * KCHUNK + (e >> 7) < np;
                As[buf][e >> 7][e & 127] = ok ? T((double)ra[q] * rw[q]) : T(0);
                Bs[buf][e >> 7][e & 127] = ok ? rb[q] : T(0);
            }
        };
        gp<const int32_t> __restrict__ fn = gptr(sg.unit_fn + u.fn_begin);
        int32_t gI[2][4], gJ[4];
#pragma unroll
        for (int ib = 0; ib < 2; ++ib)
#pragma unroll
            for (int r = 0; r < 4; ++r) gI[ib][r] = fn[min(I0 + wr * 32 + ib * 16 + M::row(lk, r), u.m - 1)];
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) gJ[jb] = fn[min(J0 + wc * 64 + jb * 16 + lr, u.m - 1)];

        typename M::acc_t acc[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = M::zero();
        fetch(0);
        stash(0, 0);
        __syncthreads();
        for (int c = 0; c < n_chunks; ++c) {
            const int buf = c & 1;
            if (c + 1 < n_chunks) fetch(c + 1);
#pragma unroll
            for (int kk = 0; kk < KCHUNK / 4; ++kk) {
                const int kr = kk * 4 + lk;
                T a[2], bq[4];
#pragma unroll
                for (int i = 0; i < 2; ++i) a[i] = As[buf][kr][wr * 32 + i * 16 + lr];
#pragma unroll
                for (int j = 0; j < 4; ++j) bq[j] = Bs[buf][kr][wc * 64 + j * 16 + lr];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][j] = M::op(a[i], bq[j], acc[i][j]);
            }
            if (c + 1 < n_chunks) stash(c + 1, buf ^ 1);
            __syncthreads();
        }

        gp<double> __restrict__ H = gptr(sg.H);
        const int64_t ldh = sg.ld;
        const bool diag = it.ti == it.tj;
#pragma unroll
        for (int ib = 0; ib < 2; ++ib)
#pragma unroll
            for (int jb = 0; jb < 4; ++jb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = wr * 32 + ib * 16 + M::row(lk, r);
                    const int col = wc * 64 + jb * 16 + lr;
                    const int ci = I0 + row, cj = J0 + col;
                    if (ci < u.m && cj < u.m && (!diag || row <= col))
                        gadd(H + (int64_t)gI[ib][r] * ldh + gJ[jb], (double)acc[ib][jb][r]);
                }
    }
}

// Density, its gradient and the local Pulay forces: per work item up to 128 rows (8 row blocks) of an
// execution unit and one 64-wide column tile J,
//   NK_DENSITY:  T[:, J] = sum over the list up to J of Phi D[:, J],  n_p += sum_{j in J} T_pj Phi_pj
//                (every pair of tiles once, doubled; the diagonal tile once);
//   NK_GRADIENT: T[:, J] = Phi D[:, J] over the whole list, and four row dots, n and
//                grad n = 2 T . grad Phi;
//   NK_FORCE:    M[:, J] = (w h_KS Phi) D[:, J] - diag(w) Phi Q[:, J] over the whole list, and column
//                sums f_j += sum_p grad phi_pj M_pj into fb[N_b][3].
// Only upper triangles of D and Q are read: rows i of D for tiles I < J, columns of D (rows j of the
// matrix) for I > J, and the diagonal tile element by element.
//
// K = the list in steps of KC functions through two LDS stages filled by direct loads: 128 x KC
// basis values (rows of 64 bytes, their 16-byte slots XOR-swizzled by row so that reads meet distinct
// banks) and KC x 64 values of D (16 bytes per lane and two matrix rows per wave load where the
// tile's columns come in neighbouring pairs, else 4 bytes and half a row; right of the diagonal rows
// of the tile).  Four waves, a 16-column block each, with D as the first
// MFMA operand, so that a lane's results belong to one point and the row dots are sums within a lane
// and over four lanes.
//
// Bound: the matrix pipes; as in h_tiles there are next to no vector instructions in the loop.  Four
// workgroups of four waves share a CU, so that three compute while one starts, ends or waits at a
// barrier.  unit_mask leaves out the MFMAs of row blocks that either side does not reach, and the
// FP64 density contracts the diagonal tile's upper triangle alone (its diagonal halved, everything
// doubled at the end); FP32 keeps the order and the rounding of full diagonal tiles.
// Measured, kernel alone, against sixteen waves per 256 rows with staging through registers (4.9 vector
// instructions per MFMA): FP64 density 7.9 -> 5.5 ms (100-atom block), 117 -> 83 ms (375-atom slab),
// FP32 13.3 -> 8.8 ms (100-atom slab), gradient 16.0 -> 12.7 ms, forces 33 -> 26 ms.  Eight waves per
// 256 rows took 6.6 ms, loads of D by 4 bytes alone 6.4, a third stage gains nothing.
enum NKind { NK_DENSITY = 0, NK_GRADIENT = 1, NK_FORCE = 2 };
constexpr int NWIN = 512;   // functions whose indices and masks are in LDS at a time
template <typename T, int KIND>
__global__ __launch_bounds__(256, 4) void n_tiles(const DevSeg* __restrict__ segs, int n_segs, int64_t total, int lg)
{
    typedef Mma<T> M;
    constexpr bool F64 = sizeof(T) == 8;
    constexpr bool FULL = KIND != NK_DENSITY, TRI = F64 && !FULL;
    constexpr int KC = 64 / (int)sizeof(T);             // functions per step: 8 (FP64), 16 (FP32)
    constexpr int KR = KC / 4;                          // D rows per wave and step
    constexpr int AB = NTILE_ROWS * 64, BB = KC * TILE * 8, STAGEB = AB + BB;
    constexpr int FN = 2 * STAGEB, MK = FN + NWIN * 4;
    __shared__ __align__(16) unsigned char lds[MK + 64 * 4];  // (the masks' wave load fills 64 entries)
    typedef T slot_t __attribute__((ext_vector_type(16 / sizeof(T))));
    typedef double d2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    const int lr = lane & 15, lk = lane >> 4;
    for (int64_t v_ = blockIdx.x; v_ < xcd_span(total, lg); v_ += gridDim.x) {
        const int64_t b = xcd_item(v_, lg);
        if (b >= total) continue;
        const int s = find_segment(segs, n_segs, b, [](const DevSeg& g) { return g.item_prefix; });
        const DevSeg& sg = segs[s];
        const NTile* it = static_cast<const NTile*>(sg.items) + (sg.item_begin + (b - sg.item_prefix));
        const int tj = uni(it->tj), np = uni(it->n_rows), ld = uni(it->ld), m = uni(it->m), rb0 = uni(it->row_block);
        const int64_t out_offset = uni(it->out_offset), point_begin = uni(it->point_begin);
        const int64_t fn_begin = uni(it->fn_begin), mask_begin = uni(it->mask_begin);
        const int64_t ldd = uni(sg.ld);
        const uint64_t* mp = sg.unit_mask + mask_begin;
        const int J0 = tj * TILE, cb = (wave + tj) & 3;
        uint32_t any_j = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) any_j |= (uint32_t)uni((int)mp[4 * tj + q]);
        const uint32_t own = (1u << ((np + 15) / 16)) - 1;  // the item's row blocks
        any_j = (any_j >> rb0) & own;
        if (any_j == 0) continue;
        const uint32_t col_rows = ((uint32_t)uni((int)mp[4 * tj + cb]) >> rb0) & own;  // row blocks this wave's columns reach
        const int32_t* fn = sg.unit_fn + fn_begin;
        const int ldb = ld * (int)sizeof(T);
        // D by 16 bytes per lane, a wave load for two of its rows: the tile's columns have to come in
        // pairs of neighbours (atoms with an even number of functions) and D to lie within 32-bit offsets
        const int ldd8 = (int)(ldd * 8);
        const int cp = J0 + 2 * (lane & 31), gp0 = fn[min(cp, m - 1)], gp1 = fn[min(cp + 1, m - 1)];
        const bool pairs = ldd <= D_OFFSET_MAX_BASIS && __all(cp + 1 >= m || gp1 == gp0 + 1);
        // else by 4 bytes per lane, half of a row per wave load: columns J0 + 32 q + lane / 2
        int voff_d[2];
        int64_t row_j[FULL || !F64 ? 2 : 1];  // byte offsets of those columns' own rows (diagonal tile)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int g = fn[min(J0 + 32 * q + (lane >> 1), m - 1)];
            voff_d[q] = g * 8 + 4 * (lane & 1);
            if (FULL || !F64) row_j[q] = ((int64_t)g * ldd) * 8 + 4 * (lane & 1);
        }
        // right of the diagonal a wave load takes rows j of D, 64 / (2 KC) of them
        constexpr int JPL = 32 / KC, NLOW = FULL ? 2 * KR : 1;
        int64_t low_j[NLOW];
        int low_k[NLOW];
        if (FULL)
#pragma unroll
            for (int q = 0; q < NLOW; ++q) {
                const int j = (wave * 2 * KR + q) * JPL + lane / (2 * KC), d = lane % (2 * KC);
                low_j[q] = ((int64_t)fn[min(J0 + j, m - 1)] * ldd) * 8 + 4 * (d & 1);
                low_k[q] = 2 * ((d >> 2) ^ (F64 ? (j >> 1) & 3 : j & 7)) + ((d >> 1) & 1);
            }
        int voff_a[2];  // row blocks wave and wave + 4
#pragma unroll
        for (int q = 0; q < 2; ++q)
            voff_a[q] = ((wave + 4 * q) * 16 + (lane >> 2)) * ldb + (((lane & 3) ^ ((lane >> 3) & 3)) * 16);
        // per-lane LDS offsets: rows lr of this wave's row blocks, D columns cb * 16 + lr
        const int a_sw = (lr >> 1) & 3;
        const int a_off = lr * 64 + (F64 ? (lk ^ a_sw) * 16 : lk * 4);
        const int b_col = cb * 16 + lr;
        const int b_up = AB + (F64 ? 2 * lk : lk) * 512 + b_col * 8;
        const int b_low = AB + b_col * (KC * 8) + (F64 ? (lk ^ ((b_col >> 1) & 3)) * 16 : 0);

        typename M::acc_t acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = M::zero();

        // acc += A[:, list] mat[list, J] over the functions k < K (A: rows of ldb bytes)
        auto contract = [&](const T* A, const double* mat, int K) {
            const char* a_base = reinterpret_cast<const char*>(A);
            const char* d_base = reinterpret_cast<const char*>(mat);
            for (int w0 = 0; w0 < K; w0 += NWIN) {
                const int k_end = min(K, w0 + NWIN);
                __builtin_amdgcn_s_waitcnt(0xC07F);  // every wave is done with the LDS of the step before
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                const __amdgpu_buffer_rsrc_t rf = buffer_of(fn, m * 4);  // past the list: its last function
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    load4_to_lds(rf, lds + FN + q * 1024 + wave * 256, min(w0 + q * 256 + wave * 64 + lane, m - 1) * 4, 0);
                if (wave == 0)
                    load4_to_lds(buffer_of(mp, ld / 16 * 8), lds + MK, (w0 / 16 + (lane & 31)) * 8, 0);
                wait_loads<0>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                const int32_t* fnw = reinterpret_cast<const int32_t*>(lds + FN) - w0;
                const uint32_t* mkw = reinterpret_cast<const uint32_t*>(lds + MK) - w0 / 16;
                const __amdgpu_buffer_rsrc_t ra = buffer_of(a_base, np * ldb);
                const __amdgpu_buffer_rsrc_t rd = buffer_of(d_base, (int)(uint32_t)(pairs ? ldd * ldd8 : 0));
                // list indices and mask of the step that is issued next, read a step ahead: this
                // wave's D rows are KR wave .. KR wave + KR - 1 of the step's, two per wave load
                int nx_k[KR / 2], nx_low[NLOW];
                uint32_t nx_m;
                auto peek = [&](int k0) {
                    nx_m = mkw[k0 >> 4];
#pragma unroll
                    for (int t = 0; t < KR / 2; ++t) nx_k[t] = fnw[k0 + KR * wave + 2 * t + (lane >> 5)];
                    if (FULL)
#pragma unroll
                        for (int q = 0; q < NLOW; ++q) nx_low[q] = fnw[k0 + low_k[q]];
                };
                auto tile_diag = [&](int k0) { return (k0 >> 6) == tj; };
                auto tile_low = [&](int k0) { return FULL && (k0 >> 6) > tj; };
                uint32_t mk[2];  // masks of the steps in the two stages
                auto issue = [&](int k0, int stg) {
                    unsigned char* st = lds + stg * STAGEB;
                    mk[stg] = (uint32_t)uni((int)nx_m) >> rb0;
                    // rows past the last one lie past the buffer's end by their voffset alone
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        load16_to_lds(ra, st + (wave + 4 * q) * 1024, voff_a[q], k0 * (int)sizeof(T));
                    unsigned char* bt = st + AB + KR * wave * 512;
                    if (tile_low(k0)) {
#pragma unroll
                        for (int q = 0; q < NLOW; ++q) {
                            const char* src = d_base + (low_j[q] + (int64_t)nx_low[q] * 8);
                            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                             (__attribute__((address_space(3))) void*)(st + AB + (wave * 2 * KR + q) * 256),
                                                             4, 0, 0);
                        }
                    } else if (pairs && (TRI || !tile_diag(k0))) {
#pragma unroll
                        for (int t = 0; t < KR / 2; ++t) load16_to_lds(rd, bt + t * 1024, (int)d_offset(nx_k[t], ldd, gp0), 0);
                    } else {
#pragma unroll
                        for (int t = 0; t < KR; ++t) {
                            const int gk = __builtin_amdgcn_readlane(nx_k[t / 2], 32 * (t & 1));
                            const char* row = d_base + (int64_t)gk * ldd * 8;
                            const __amdgpu_buffer_rsrc_t r = buffer_of(row, ldd8);
#pragma unroll
                            for (int q = 0; q < 2; ++q) {
                                unsigned char* dst = bt + t * 512 + q * 256;
                                if (!TRI && tile_diag(k0)) {  // below the diagonal: the transposed element
                                    const bool below = k0 + KR * wave + t > J0 + 32 * q + (lane >> 1);
                                    const char* src = below ? d_base + (row_j[FULL || !F64 ? q : 0] + (int64_t)gk * 8) : row + voff_d[q];
                                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                                     (__attribute__((address_space(3))) void*)dst, 4, 0, 0);
                                } else {
                                    load4_to_lds(r, dst, voff_d[q], 0);
                                }
                            }
                        }
                    }
                };
                // one step: its operands are read, the next step is issued while they come, and then the
                // MFMAs run
                auto step = [&](int k0, int stg, int ki) {
                    const uint32_t act = mk[stg] & col_rows;
                    const bool at_diag = tile_diag(k0), low = tile_low(k0);
                    const int kb = (k0 >> 4) & 3;  // 16-function block within its tile
                    const unsigned char* st = lds + stg * STAGEB;
                    auto next = [&]() {
                        if (ki >= k_end) return;
                        issue(ki, stg ^ 1);
                        peek(ki + KC);
                    };
                    if constexpr (F64) {
                        slot_t a[8];
                        double b0, b1;
                        if (low) {
                            const d2 x = *reinterpret_cast<const d2*>(st + b_low);
                            b0 = x[0], b1 = x[1];
                        } else {
                            b0 = *reinterpret_cast<const double*>(st + b_up);
                            b1 = *reinterpret_cast<const double*>(st + b_up + 512);
                        }
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            if (!FULL) a[q] = *reinterpret_cast<const slot_t*>(st + a_off + q * 1024);
                        next();
                        if (!act || (TRI && at_diag && kb > cb)) return;
                        if (TRI && at_diag && kb == cb) {
                            const int k = (k0 & 15) + 2 * lk;
                            b0 = k < lr ? b0 : k == lr ? 0.5 * b0 : 0.0;
                            b1 = k + 1 < lr ? b1 : k + 1 == lr ? 0.5 * b1 : 0.0;
                        }
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            if ((act >> q) & 1) {
                                if (FULL) a[q] = *reinterpret_cast<const slot_t*>(st + a_off + q * 1024);  // fewer registers
                                acc[q] = M::op(b0, a[q][0], acc[q]);
                                acc[q] = M::op(b1, a[q][1], acc[q]);
                            }
                    } else {
                        double bd[4];
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) {
                            const int k = kk * 4 + lk;
                            bd[kk] = low ? *reinterpret_cast<const double*>(st + b_low + (((k >> 1) ^ (b_col & 7)) * 16) + (k & 1) * 8)
                                         : *reinterpret_cast<const double*>(st + b_up + kk * 2048);
                        }
                        next();
                        if (KIND == NK_DENSITY && k0 == J0)  // the tiles before the diagonal count twice
#pragma unroll
                            for (int q = 0; q < 8; ++q) acc[q] += acc[q];
                        if (!act) return;
                        T bv[4];
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) bv[kk] = T(bd[kk]);
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            if ((act >> q) & 1) {
                                T a[4];
#pragma unroll
                                for (int kk = 0; kk < 4; ++kk)
                                    a[kk] = *reinterpret_cast<const T*>(st + a_off + q * 1024 + ((kk ^ a_sw) * 16));
#pragma unroll
                                for (int kk = 0; kk < 4; ++kk) acc[q] = M::op(bv[kk], a[kk], acc[q]);
                            }
                    }
                };
                peek(w0);
                issue(w0, 0);
                peek(w0 + KC);
                int kc = w0;
                while (kc < k_end) {
#pragma unroll
                    for (int stg = 0; stg < 2; ++stg) {
                        wait_loads<0>();
                        __builtin_amdgcn_s_barrier();
                        asm volatile("" ::: "memory");
                        step(kc, stg, kc + KC);
                        kc += KC;
                        if (kc >= k_end) break;
                    }
                }
            }
        };

        const T* phi = static_cast<const T*>(sg.phi) + out_offset;
        if constexpr (KIND == NK_FORCE) {
            contract(phi, sg.Q, m);
            gp<const double> pw = gptr(sg.sys->pw + point_begin);
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] *= -pw[min(q * 16 + lr, np - 1)];
            contract(static_cast<const T*>(sg.hphi) + out_offset, sg.D, m);
        } else {
            contract(phi, sg.D, FULL ? m : min(J0 + TILE, m));
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();  // the ring is free
        asm volatile("" ::: "memory");
        // acc[q][r] belongs to row 16 q + lr and column J0 + 16 cb + row(lk, r)
        double* red = reinterpret_cast<double*>(lds);
        const int c0 = J0 + cb * 16;
        // columns past the list (the last one's values of D, not zeros, were loaded for them)
        if (c0 + 16 > m)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (c0 + M::row(lk, r) >= m)
#pragma unroll
                    for (int q = 0; q < 8; ++q) acc[q][r] = T(0);
        constexpr int SZ = (int)sizeof(T);
        const int voff_e = lr * ldb + c0 * SZ;  // row lr of a row block, first column of this wave
        if constexpr (KIND == NK_FORCE) {
            const char* g = static_cast<const char*>(sg.gphi) + out_offset * SZ;
            double f[4][3] = {};
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int rb = q;
                if (!((col_rows >> rb) & 1)) continue;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const __amdgpu_buffer_rsrc_t rg = buffer_of(g + k * sg.plane * SZ + (int64_t)rb * 16 * ldb, max(0, np - rb * 16) * ldb);
#pragma unroll
                    for (int r = 0; r < 4; ++r) f[r][k] += (double)acc[q][r] * (double)load_value<T>(rg, voff_e + M::row(lk, r) * SZ);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double x = row_sum16(f[r][k]);
                    if (lr == 0) red[k * TILE + cb * 16 + M::row(lk, r)] = x;
                }
            __syncthreads();
            const int k = threadIdx.x / TILE, col = threadIdx.x % TILE;
            if (k < 3 && J0 + col < m)
                gadd(gptr(sg.fb) + 3 * (v_ % FORCE_COPIES * ldd + fn[J0 + col]) + k, red[k * TILE + col]);
        } else {
            constexpr int NQ = KIND == NK_GRADIENT ? 4 : 1;
            const char* ph = reinterpret_cast<const char*>(phi);
            const char* g = KIND == NK_GRADIENT ? static_cast<const char*>(sg.gphi) + out_offset * SZ : nullptr;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int rb = q, p = rb * 16 + lr;
                double dot[NQ] = {};
                if ((col_rows >> rb) & 1) {
                    const int rows = max(0, np - rb * 16);
                    const __amdgpu_buffer_rsrc_t rp = buffer_of(ph + (int64_t)rb * 16 * ldb, rows * ldb);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        dot[0] += (double)acc[q][r] * (double)load_value<T>(rp, voff_e + M::row(lk, r) * SZ);
                    if constexpr (KIND == NK_GRADIENT) {
#pragma unroll
                        for (int k = 1; k < NQ; ++k) {
                            const __amdgpu_buffer_rsrc_t rg = buffer_of(g + (k - 1) * sg.plane * SZ + (int64_t)rb * 16 * ldb, rows * ldb);
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                dot[k] += (double)acc[q][r] * (double)load_value<T>(rg, voff_e + M::row(lk, r) * SZ);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < NQ; ++k) {
                        dot[k] += __shfl_xor(dot[k], 16);
                        dot[k] += __shfl_xor(dot[k], 32);
                    }
                }
#pragma unroll
                for (int k = 0; k < NQ; ++k)
                    if (lk == 0) red[(k * 4 + cb) * NTILE_ROWS + p] = dot[k];
            }
            __syncthreads();
            const int p = threadIdx.x;
            if (p < np) {
                const int32_t pc = gptr(sg.sys->perm)[point_begin + p];
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    const double* x = red + k * 4 * NTILE_ROWS + p;
                    const double v = (x[0] + x[NTILE_ROWS]) + (x[2 * NTILE_ROWS] + x[3 * NTILE_ROWS]);
                    if (k == 0) gadd(gptr(sg.n) + pc, TRI ? 2.0 * v : v);
                    else gadd(gptr(sg.gn) + 3 * (int64_t)pc + k - 1, 2.0 * v);
                }
            }
        }
    }
}

// Local Pulay forces in FP32: as n_tiles NK_FORCE with every -w phi rounded to FP32 before the
// second product (direct loads cannot scale what they stage, so basis values and D go through
// registers: rows padded to 17 values, double-buffered chunks of 16 functions, the next chunk
// prefetched while the MFMAs of the current one run).  Sixteen waves: wave w owns column block w % 4
// and row blocks w / 4 + 4 q.
__global__ __launch_bounds__(1024) void n_force_f32(const DevSeg* __restrict__ segs, int n_segs, int64_t total, int lg)
{
    typedef float T;
    typedef Mma<T> M;
    constexpr int KC = 16, NT = 1024, RB = 4, RS = 4;
    constexpr int NA = MAX_UNIT_POINTS * KC / NT;  // basis values per thread per chunk
    __shared__ T As[2][MAX_UNIT_POINTS][KC + 1];
    __shared__ T Bs[2][KC][TILE + 2];
    __shared__ double red[3][RS][TILE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cb = wave & 3, rh = wave >> 2;  // column block; row blocks rh, rh + RS, ...
    const int lr = lane & 15, lk = lane >> 4;
    for (int64_t v_ = blockIdx.x; v_ < xcd_span(total, lg); v_ += gridDim.x) {
        const int64_t b = xcd_item(v_, lg);
        if (b >= total) continue;
        const int s = find_segment(segs, n_segs, b, [](const DevSeg& g) { return g.item_prefix; });
        const DevSeg& sg = segs[s];
        const NItem it = static_cast<const NItem*>(sg.items)[sg.item_begin + (b - sg.item_prefix)];
        const DevUnit u = sg.item_units[it.unit];
        gp<const T> __restrict__ phi = gptr(static_cast<const T*>(sg.phi) + u.out_offset);
        gp<const T> __restrict__ hphi = gptr(static_cast<const T*>(sg.hphi) + u.out_offset);
        gp<const int32_t> __restrict__ fn = gptr(sg.unit_fn + u.fn_begin);
        const int64_t ldd = sg.ld;
        const int np = u.n_points, ld = u.ld, m = u.m;
        if (np <= 0 || m <= 0) continue;
        const int P = (np + 15) >> 4;
        const int J0 = it.tj * TILE;
        // chunks 0 .. half - 1 run the list against D, half .. 2 half - 1 against Q
        const int half = (m + KC - 1) / KC, n_chunks = 2 * half;
        auto col0 = [&](int c) { return KC * (c >= half ? c - half : c); };
        const int cjd = J0 + (tid & (TILE - 1));  // this thread's D column in every chunk
        const int64_t gjd = fn[min(cjd, m - 1)];
        // F = row blocks staged per wave's share (RB, or RB / 2 for at most 128 points)
        auto run = [&](auto rows_staged) {
            constexpr int F = decltype(rows_staged)::value;
            constexpr int NAR = NA * F / RB;
            T pa[NAR];
            double pd;
            int32_t gcur, gnxt;
            auto load_idx = [&](int c) { return fn[min(col0(c) + (tid >> 6), m - 1)]; };
            double sw[NAR];  // -w of this thread's staged rows, for the Q pass
            gp<const double> pw = gptr(sg.sys->pw + u.point_begin);
#pragma unroll
            for (int q = 0; q < NAR; ++q) sw[q] = -pw[min((tid + NT * q) / KC, np - 1)];
            auto fetch = [&](int c) {
#pragma unroll
                for (int q = 0; q < NAR; ++q) {
                    const int e = tid + NT * q;
                    const int64_t el = (int64_t)min(e / KC, np - 1) * ld + col0(c) + (e % KC);
                    pa[q] = c < half ? hphi[el] : phi[el];
                }
                gp<const double> src = gptr(c >= half ? sg.Q : sg.D);
                const bool lower = col0(c) + (tid >> 6) > cjd;  // only the upper triangle is read
                pd = src[lower ? gjd * ldd + gcur : (int64_t)gcur * ldd + gjd];
                gnxt = load_idx(c + 1);
            };
            auto stash = [&](int c, int buf) {
                gcur = gnxt;
#pragma unroll
                for (int q = 0; q < NAR; ++q) {
                    const int e = tid + NT * q;
                    const T x = c >= half ? T((double)pa[q] * sw[q]) : pa[q];
                    As[buf][e / KC][e % KC] = (e / KC) < np ? x : T(0);
                }
                Bs[buf][tid >> 6][tid & 63] = col0(c) + (tid >> 6) < m && cjd < m ? T(pd) : T(0);
            };
            M::acc_t acc[F];
#pragma unroll
            for (int i = 0; i < F; ++i) acc[i] = M::zero();
            gcur = load_idx(0);
            fetch(0);
            stash(0, 0);
            __syncthreads();
            for (int c = 0; c < n_chunks; ++c) {
                const int buf = c & 1;
                if (c + 1 < n_chunks) fetch(c + 1);
#pragma unroll
                for (int kk = 0; kk < KC / 4; ++kk) {
                    const T bv = Bs[buf][kk * 4 + lk][cb * 16 + lr];
#pragma unroll
                    for (int q = 0; q < F; ++q) acc[q] = M::op(As[buf][(RS * q + rh) * 16 + lr][kk * 4 + lk], bv, acc[q]);
                }
                if (c + 1 < n_chunks) stash(c + 1, buf ^ 1);
                __syncthreads();
            }
            // f_j += sum_p grad phi_pj M_pj: this wave's rows, then the lanes of one column
            const int cj = J0 + cb * 16 + lr;
            gp<const T> gph = gptr(static_cast<const T*>(sg.gphi) + u.out_offset);
            double f[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < F; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int p = (RS * q + rh) * 16 + M::row(lk, r);
                    const int64_t e = (int64_t)min(p, np - 1) * ld + cj;
                    const double a = p < np && cj < m ? (double)acc[q][r] : 0.0;
#pragma unroll
                    for (int k = 0; k < 3; ++k) f[k] += a * (double)gph[k * sg.plane + e];
                }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                double v = f[k];
                v += __shfl_xor(v, 16);
                v += __shfl_xor(v, 32);
                if (lk == 0) red[k][rh][cb * 16 + lr] = v;
            }
        };
        if (P > RB / 2 * RS) run(std::integral_constant<int, RB>{});
        else run(std::integral_constant<int, RB / 2>{});
        __syncthreads();
        if (tid < 3 * TILE) {
            const int k = tid / TILE, col = tid % TILE;
            if (J0 + col < m)
                gadd(gptr(sg.fb) + 3 * (v_ % FORCE_COPIES * ldd + fn[J0 + col]) + k,
                     (red[k][0][col] + red[k][1][col]) + (red[k][2][col] + red[k][3][col]));
        }
        __syncthreads();  // red is rewritten by the next item
    }
}

// ------------------------------------------------------------------------------------------
// Reduced-precision contractions.  Basis values arrive as FP32 (rounded from the FP64
// evaluation); w*v and D are rounded from FP64 when staged.  Per-tile results are flushed
// into FP64 accumulators and reach H and n through FP64 atomics.


// Split of two FP32 values into NS bf16 parts each: x ~ x0 + x1 (+ x2), each part the rounding to
// nearest of what the previous parts leave.  part[s]: the two values' part s, packed.
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
template <int NS>
__device__ inline void split_bf16(float x, float y, uint32_t* part)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x, y}, bf2));
        part[s] = h;
        x -= __builtin_bit_cast(float, h << 16);
        y -= __builtin_bit_cast(float, h & 0xffff0000u);
    }
}

// Products kept: parts (s, t) with s + t <= NS - 1 (3 terms for NS = 2, 6 terms for NS = 3).
template <int NS>
__device__ inline f4 mfma_split(const bf8* a, const bf8* b, f4 acc)
{
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int t = 0; t < NS; ++t)
            if (s + t <= NS - 1) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[t], acc, 0, 0, 0);
    return acc;
}

constexpr int BK = 32;  // K per bf16 MFMA step
// LDS rows are 64 bytes, their four 16-byte slots permuted by row (no bank conflicts, no padding):
// first of the elements 8 g .. 8 g + 7 of a row
__device__ inline int bf16_slot(int row, int g) { return 8 * (g ^ ((row >> 1) & 3)); }

// Hamiltonian, split-BF16 MFMA (v_mfma_f32_16x16x32_bf16): per item one 64x64 tile pair of a unit or
// a cluster, in chunks of 32 points of one unit, four waves of 32x32.  LDS holds
// [buffer][part][column][point] so that every lane reads its 8 consecutive points as one 16-byte
// vector; the next chunk's FP32 basis values and w v are prefetched while the MFMAs of the current
// one run and are split into bf16 parts at the stash.  The FP32 sums move into FP64 after every
// chunk, so that a cluster's sums are those of its units and reach H by a half to a quarter of the
// atomics; chunks that one of the tiles does not reach are left out.  FP64 atomics into the upper
// triangle of H.  The splitting binds it (8 vector and 6 scalar instructions beside every MFMA), then the atomics: three
// workgroups per CU, two values per conversion, scalar row addresses and w v; 64-atom block, three
// parts, units alone 3.03 ms before and 2.81 after (MFMA busy 15 %), over clusters 2.10 (23 %).
template <int NS>
__global__ __launch_bounds__(256, 3) void h_kernel_bf16(const DevSeg* __restrict__ segs, int n_segs, int64_t total, int lg)
{
    constexpr int NQ = BK * TILE / 256;  // values per thread per chunk and operand
    __shared__ __attribute__((aligned(16))) __bf16 As[2][NS][TILE][BK];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][NS][TILE][BK];
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1;
    const int lr = lane & 15, lk = lane >> 4;
    for (int64_t v_ = blockIdx.x; v_ < xcd_span(total, lg); v_ += gridDim.x) {
        const int64_t b = xcd_item(v_, lg);
        if (b >= total) continue;
        const int s = find_segment(segs, n_segs, b, [](const DevSeg& g) { return g.item_prefix; });
        const DevSeg& sg = segs[s];
        const HItem it = static_cast<const HItem*>(sg.items)[sg.item_begin + (b - sg.item_prefix)];
        const DevUnit& u = sg.item_units[uni(it.unit)];
        const int ld = uni(u.ld), m = uni(u.m), n_sub = uni(u.sub_count);
        const DevUnit* sub = sg.units + uni(u.sub_begin);
        const int64_t row_begin = uni(u.row_begin);
        gp<const float> __restrict__ phi = gptr(static_cast<const float*>(sg.phi) + uni(u.out_offset));
        gp<const double> __restrict__ wv = gptr(sg.wv + row_begin);
        const int ti = uni((int)it.ti), tj = uni((int)it.tj), I0 = ti * TILE, J0 = tj * TILE;
        const uint64_t* mI = sg.unit_mask + uni(u.mask_begin) + 4 * ti;
        const uint64_t* mJ = sg.unit_mask + uni(u.mask_begin) + 4 * tj;
        uint64_t any_i = 0, any_j = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            any_i |= (uint64_t)uni((int64_t)mI[q]);
            any_j |= (uint64_t)uni((int64_t)mJ[q]);
        }
        const uint64_t todo = any_i & any_j;  // 16-row chunks both tiles reach
        if (todo == 0) continue;
        // the next chunk: rows p .. p + 31 of the np rows that unit k has from row r0 on
        int k, r0, np, p;
        auto unit_at = [&]() {
            r0 = (int)(uni(sub[k].row_begin) - row_begin);
            np = uni(sub[k].n_points);
            p = 0;
        };
        auto seek = [&]() {  // to one that both tiles reach, or k = n_sub
            while (k < n_sub && (p >= np || !((todo >> ((r0 + p) >> 4)) & 3))) {
                if (p < np) p += BK;
                else if (++k < n_sub) unit_at();
            }
        };

        // this thread's column of both operands and its NQ = 8 consecutive points of a chunk, so
        // that every part is stashed as one 16-byte run of a column (loads: a wave reads 64
        // consecutive columns of one point)
        static_assert(NQ == 8, "eight points per thread");
        const int col = lane, p0 = NQ * wave;  // the points are the wave's: scalar addresses and w v
        float ra[NQ], rb[NQ];
        double rw[NQ];
        // points past the unit's last: w v = 0 makes their products zero
        auto fetch = [&]() {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int pc = min(p + p0 + q, np - 1);
                gp<const float> rowp = phi + (int64_t)(r0 + pc) * ld;
                ra[q] = rowp[I0 + col];
                rb[q] = rowp[J0 + col];
                rw[q] = p + p0 + q < np ? wv[r0 + pc] : 0.0;
            }
            p += BK;
            seek();
        };
        auto stash = [&](int buf) {
            u4 pa[NS], pb[NS];
#pragma unroll
            for (int q = 0; q < NQ; q += 2) {
                uint32_t xa[NS], xb[NS];
                split_bf16<NS>((float)((double)ra[q] * rw[q]), (float)((double)ra[q + 1] * rw[q + 1]), xa);
                split_bf16<NS>(rb[q], rb[q + 1], xb);
#pragma unroll
                for (int t = 0; t < NS; ++t) {
                    pa[t][q / 2] = xa[t];
                    pb[t][q / 2] = xb[t];
                }
            }
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                *reinterpret_cast<u4*>(&As[buf][t][col][bf16_slot(col, wave)]) = pa[t];
                *reinterpret_cast<u4*>(&Bs[buf][t][col][bf16_slot(col, wave)]) = pb[t];
            }
        };
        gp<const int32_t> __restrict__ fn = gptr(sg.unit_fn + uni(u.fn_begin));
        int32_t gI[2][4], gJ[2];
#pragma unroll
        for (int ib = 0; ib < 2; ++ib) {
#pragma unroll
            for (int r = 0; r < 4; ++r) gI[ib][r] = fn[min(I0 + wr * 32 + ib * 16 + lk * 4 + r, m - 1)];
            gJ[ib] = fn[min(J0 + wc * 32 + ib * 16 + lr, m - 1)];
        }

        d4 acc64[2][2] = {};
        auto k_loop = [&](auto with_mfma) {
            k = 0;
            unit_at();
            seek();
            if (k >= n_sub) return;
            fetch();
            stash(0);
            __syncthreads();
            for (int buf = 0;; buf ^= 1) {
                const bool more = k < n_sub;
                if (more) fetch();
                if (decltype(with_mfma)::value) {
                    bf8 a0[NS], a1[NS], b0[NS], b1[NS];
#pragma unroll
                    for (int t = 0; t < NS; ++t) {
                        const int sl = bf16_slot(lr, lk);
                        a0[t] = *reinterpret_cast<const bf8*>(&As[buf][t][wr * 32 + lr][sl]);
                        a1[t] = *reinterpret_cast<const bf8*>(&As[buf][t][wr * 32 + 16 + lr][sl]);
                        b0[t] = *reinterpret_cast<const bf8*>(&Bs[buf][t][wc * 32 + lr][sl]);
                        b1[t] = *reinterpret_cast<const bf8*>(&Bs[buf][t][wc * 32 + 16 + lr][sl]);
                    }
                    // every chunk of 32 points: its FP32 sums move into FP64
                    const f4 zero{0.f, 0.f, 0.f, 0.f};
                    const f4 x[2][2] = {{mfma_split<NS>(a0, b0, zero), mfma_split<NS>(a0, b1, zero)},
                                        {mfma_split<NS>(a1, b0, zero), mfma_split<NS>(a1, b1, zero)}};
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
#pragma unroll
                            for (int r = 0; r < 4; ++r) acc64[i][j][r] += (double)x[i][j][r];
                }
                if (more) stash(buf ^ 1);
                __syncthreads();
                if (!more) break;
            }
        };
        const bool diag = ti == tj;
        if (diag && wr > wc) {  // the strictly lower quarter of a diagonal tile pair only stages data
            k_loop(std::false_type{});
            continue;
        }
        k_loop(std::true_type{});
        gp<double> __restrict__ H = gptr(sg.H);
        const int64_t ldh = sg.ld;
#pragma unroll
        for (int ib = 0; ib < 2; ++ib)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = wr * 32 + ib * 16 + lk * 4 + r, col = wc * 32 + jb * 16 + lr;
                    const int ci = I0 + row, cj = J0 + col;
                    if (ci < m && cj < m && (!diag || row <= col))
                        gadd(H + (int64_t)gI[ib][r] * ldh + gJ[jb], acc64[ib][jb][r]);
                }
    }
}

// Density, split-BF16 MFMA: per item (NTile) one 64-wide column tile J of up to 128 rows of a unit,
// K = 32 functions per chunk; eight waves, wave w takes column block w % 4 and row blocks w / 4 + 2 q.
// A (points x functions) in LDS as [part][point][function], B (functions x columns) as
// [part][column][function], two buffers.  The FP32 sums move into FP64 after every 64-function tile;
// the row dot and the sums over tiles and units are FP64.
// Bound by the splitting and the wait at the barrier of every chunk (one workgroup of 256 rows: MFMA
// busy 18 %, VALU 39 %), so that two workgroups of 128 rows share a CU.  64-atom block, three parts:
// 4.4 ms with parts stored by 2 bytes to one padded buffer, 2.35 by 16 bytes to two with permuted
// slots, 2.22 with 128 rows.
template <int NS>
__global__ __launch_bounds__(512, 4) void n_kernel_bf16(const DevSeg* __restrict__ segs, int n_segs, int64_t total, int lg)
{
    constexpr int RB = 4, RS = 2;
    constexpr int CPT = TILE / BK;  // chunks per tile (2)
    __shared__ __attribute__((aligned(16))) __bf16 As[2][NS][NTILE_ROWS][BK];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][NS][TILE][BK];
    __shared__ double red[4][NTILE_ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int cb = wave & 3, rh = wave >> 2;
    const int lr = lane & 15, lk = lane >> 4;
    for (int64_t v_ = blockIdx.x; v_ < xcd_span(total, lg); v_ += gridDim.x) {
        const int64_t b = xcd_item(v_, lg);
        if (b >= total) continue;
        const int s = find_segment(segs, n_segs, b, [](const DevSeg& g) { return g.item_prefix; });
        const DevSeg& sg = segs[s];
        const NTile* it = static_cast<const NTile*>(sg.items) + (sg.item_begin + (b - sg.item_prefix));
        const int tj = uni(it->tj), np = uni(it->n_rows), ld = uni(it->ld), m = uni(it->m);
        const int64_t out_offset = uni(it->out_offset), point_begin = uni(it->point_begin);
        gp<const float> __restrict__ phi = gptr(static_cast<const float*>(sg.phi) + out_offset);
        gp<const int32_t> __restrict__ fn = gptr(sg.unit_fn + uni(it->fn_begin));
        gp<const double> __restrict__ D = gptr(sg.D);
        const int64_t ldd = uni(sg.ld);
        const int P = (np + 15) >> 4;
        const int J0 = tj * TILE, n_chunks = (tj + 1) * CPT;  // chunk c covers functions 32 c .. 32 c + 31
        // staged by this thread: functions 8 (tid % 4) .. of row tid / 4, and functions 4 wave ..
        // 4 wave + 3 of column tid % 64
        const int ar = tid >> 2, ag = tid & 3;
        const bool stages_a = wave < P;  // wave-uniform: 16 rows per wave
        gp<const float> a_row = phi + (int64_t)min(ar, np - 1) * ld + 8 * ag;
        const int cjd = J0 + lane;
        const int64_t gjd = fn[min(cjd, m - 1)];
        f4 pa[2];
        double pd[4];
        int32_t gcur[4], gnxt[4];
        auto load_idx = [&](int c, int32_t* g) {
#pragma unroll
            for (int q = 0; q < 4; ++q) g[q] = uni(fn[min(BK * c + 4 * wave + q, m - 1)]);
        };
        auto fetch = [&](int c) {
            if (stages_a) {
                pa[0] = *reinterpret_cast<gp<const f4>>(a_row + BK * c);
                pa[1] = *reinterpret_cast<gp<const f4>>(a_row + BK * c + 4);
            }
            const bool diag = c / CPT == tj;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool lower = diag && BK * c + 4 * wave + q > cjd;
                pd[q] = D[lower ? gjd * ldd + gcur[q] : (int64_t)gcur[q] * ldd + gjd];
            }
            load_idx(c + 1, gnxt);
        };
        auto stash = [&](int c, int buf) {
#pragma unroll
            for (int q = 0; q < 4; ++q) gcur[q] = gnxt[q];
            if (stages_a) {
                u4 part[NS];
#pragma unroll
                for (int k = 0; k < 8; k += 2) {
                    uint32_t x[NS];
                    split_bf16<NS>(ar < np ? pa[k >> 2][k & 3] : 0.f, ar < np ? pa[k >> 2][(k & 3) + 1] : 0.f, x);
#pragma unroll
                    for (int t = 0; t < NS; ++t) part[t][k / 2] = x[t];
                }
#pragma unroll
                for (int t = 0; t < NS; ++t) *reinterpret_cast<u4*>(&As[buf][t][ar][bf16_slot(ar, ag)]) = part[t];
            }
            typedef uint32_t u2 __attribute__((ext_vector_type(2)));
            u2 part[NS];
            const bool diag = c / CPT == tj;
            float d[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) d[q] = BK * c + 4 * wave + q < m && cjd < m ? (float)(diag ? pd[q] : 2.0 * pd[q]) : 0.f;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                uint32_t x[NS];
                split_bf16<NS>(d[2 * q], d[2 * q + 1], x);
#pragma unroll
                for (int t = 0; t < NS; ++t) part[t][q] = x[t];
            }
#pragma unroll
            for (int t = 0; t < NS; ++t)
                *reinterpret_cast<u2*>(&Bs[buf][t][lane][bf16_slot(lane, wave >> 1) + 4 * (wave & 1)]) = part[t];
        };

        f4 acc[RB];
        d4 acc64[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            acc[q] = f4{0.f, 0.f, 0.f, 0.f};
            acc64[q] = d4{0.0, 0.0, 0.0, 0.0};
        }
        load_idx(0, gcur);
        fetch(0);
        stash(0, 0);
        __syncthreads();
        for (int c = 0; c < n_chunks; ++c) {
            const int buf = c & 1;
            if (c + 1 < n_chunks) fetch(c + 1);
            bf8 bv[NS];
#pragma unroll
            for (int t = 0; t < NS; ++t) bv[t] = *reinterpret_cast<const bf8*>(&Bs[buf][t][cb * 16 + lr][bf16_slot(lr, lk)]);
#pragma unroll
            for (int q = 0; q < RB; ++q)
                if (RS * q + rh < P) {
                    bf8 av[NS];
#pragma unroll
                    for (int t = 0; t < NS; ++t)
                        av[t] = *reinterpret_cast<const bf8*>(&As[buf][t][(RS * q + rh) * 16 + lr][bf16_slot(lr, lk)]);
                    acc[q] = mfma_split<NS>(av, bv, acc[q]);
                }
            if (c % CPT == CPT - 1) {  // end of a 64-function tile
#pragma unroll
                for (int q = 0; q < RB; ++q)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        acc64[q][r] += (double)acc[q][r];
                        acc[q][r] = 0.f;
                    }
            }
            if (c + 1 < n_chunks) stash(c + 1, buf ^ 1);
            __syncthreads();
        }
        const int cj = J0 + cb * 16 + lr;
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const int pblk = RS * q + rh;
            if (pblk < P) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int p = pblk * 16 + lk * 4 + r;
                    const double f = (double)phi[(int64_t)min(p, np - 1) * ld + cj];
                    const double v = row_sum16((p < np && cj < m) ? acc64[q][r] * f : 0.0);
                    if (lr == 0) red[cb][p] = v;
                }
            }
        }
        __syncthreads();
        if (tid < np) {
            const double v = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
            gadd(gptr(sg.n) + gptr(sg.sys->perm)[point_begin + tid], v);
        }
        __syncthreads();  // red is rewritten by the next item
    }
}

hipError_t launch_h(Mode mode, const DevSeg* segs_dev, int n_segs, int64_t n_items, hipStream_t st,
                    int64_t max_grid, int h_tile)
{
    if (h_tile == WTILE && (mode == MODE_FP64 || mode == MODE_FP32)) {
        if (n_items <= 0 || n_segs <= 0) return hipSuccess;
        if (n_items > 0x7ffffff0) return hipErrorInvalidValue;
        const int lg = xcd_run(n_items, HRUN);
        const dim3 g(grid_for(n_items, lg, max_grid)), b(512);
        if (mode == MODE_FP64) hipLaunchKernelGGL(h_kernel_wide<double>, g, b, 0, st, segs_dev, n_segs, n_items, lg);
        else hipLaunchKernelGGL(h_kernel_wide<float>, g, b, 0, st, segs_dev, n_segs, n_items, lg);
        return hipGetLastError();
    }
    if (h_tile != TILE) return hipErrorInvalidValue;
    if (n_items <= 0 || n_segs <= 0) return hipSuccess;
    if (n_items > 0x7ffffff0) return hipErrorInvalidValue;
    const int lg = xcd_run(n_items, HRUN);
    const dim3 g(grid_for(n_items, lg, max_grid)), b(256);
    switch (mode) {
    case MODE_FP64: hipLaunchKernelGGL((h_tiles<double, 16, 2, false>), g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_FP32: hipLaunchKernelGGL((h_tiles<float, 16, 2, false>), g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_BF16X3: hipLaunchKernelGGL(h_kernel_bf16<2>, g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_BF16X6: hipLaunchKernelGGL(h_kernel_bf16<3>, g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_n(Mode mode, const DevSeg* segs_dev, int n_segs, int64_t n_items, hipStream_t st,
                    int64_t max_grid)
{
    if (n_items <= 0 || n_segs <= 0) return hipSuccess;
    if (n_items > 0x7ffffff0) return hipErrorInvalidValue;
    const int lg = xcd_run(n_items, NRUN);
    const dim3 g(grid_for(n_items, lg, max_grid)), b(512);
    switch (mode) {
    case MODE_FP64: hipLaunchKernelGGL((n_tiles<double, NK_DENSITY>), g, dim3(256), 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_FP32: hipLaunchKernelGGL((n_tiles<float, NK_DENSITY>), g, dim3(256), 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_BF16X3: hipLaunchKernelGGL(n_kernel_bf16<2>, g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_BF16X6: hipLaunchKernelGGL(n_kernel_bf16<3>, g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_n_grad(Mode mode, const DevSeg* segs_dev, int n_segs, int64_t n_items, hipStream_t st)
{
    if (n_items <= 0 || n_segs <= 0) return hipSuccess;
    if (n_items > 0x7ffffff0) return hipErrorInvalidValue;
    const int lg = xcd_run(n_items, NRUN);
    const dim3 g(grid_for(n_items, lg, 0)), b(256);
    switch (mode) {
    case MODE_FP64: hipLaunchKernelGGL((n_tiles<double, NK_GRADIENT>), g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_FP32: hipLaunchKernelGGL((n_tiles<float, NK_GRADIENT>), g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_n_force(Mode mode, const DevSeg* segs_dev, int n_segs, int64_t n_items, hipStream_t st)
{
    if (n_items <= 0 || n_segs <= 0) return hipSuccess;
    if (n_items > 0x7ffffff0) return hipErrorInvalidValue;
    const int lg = xcd_run(n_items, mode == MODE_FP32 ? FRUN : NRUN);
    const dim3 g(grid_for(n_items, lg, 0)), b(1024);
    switch (mode) {
    case MODE_FP64: hipLaunchKernelGGL((n_tiles<double, NK_FORCE>), g, dim3(256), 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_FP32: hipLaunchKernelGGL(n_force_f32, g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_h_gga(Mode mode, const DevSeg* segs_dev, int n_segs, int64_t n_items, hipStream_t st)
{
    if (n_items <= 0 || n_segs <= 0) return hipSuccess;
    if (n_items > 0x7ffffff0) return hipErrorInvalidValue;
    const int lg = xcd_run(n_items, HRUN);
    const dim3 g(grid_for(n_items, lg, 0)), b(256);
    switch (mode) {
    case MODE_FP64: hipLaunchKernelGGL((h_tiles<double, 8, 3, true>), g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    case MODE_FP32: hipLaunchKernelGGL((h_tiles<float, 16, 3, true>), g, b, 0, st, segs_dev, n_segs, n_items, lg); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// small kernels

__global__ void fill_kernel(double* __restrict__ p, int64_t n, double value)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

// One wave per atom: the copies' sums of its functions, then over the lanes.
__global__ __launch_bounds__(64) void force_atoms_kernel(const double* __restrict__ fb, const int64_t* __restrict__ atom_first,
                                                         int64_t n_basis, double* __restrict__ F)
{
    const int64_t a = blockIdx.x, j0 = atom_first[a], nf = atom_first[a + 1] - j0;
    double v[3] = {};
    for (int64_t e = threadIdx.x; e < FORCE_COPIES * nf; e += 64) {
        const double* f = fb + 3 * (e % FORCE_COPIES * n_basis + j0 + e / FORCE_COPIES);
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] += f[k];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) v[k] += __shfl_xor(v[k], m);
        if (threadIdx.x == 0) F[3 * a + k] = 2.0 * v[k];
    }
}

hipError_t launch_force_atoms(const double* fb, const int64_t* atom_first, int64_t n_atoms, int64_t n_basis, double* F,
                              hipStream_t st)
{
    if (n_atoms <= 0) return hipSuccess;
    if (n_atoms > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(force_atoms_kernel, dim3((unsigned)n_atoms), dim3(64), 0, st, fb, atom_first, n_basis, F);
    return hipGetLastError();
}

// Reach of the units' functions (DevSeg::unit_mask): per 16 columns of a unit or cluster, bit c is
// set when some point of rows 16 c .. 16 c + 15 lies within the largest cutoff of an atom that owns
// one of the columns; padding columns give no bits.  Geometry alone decides, so the masks are made
// once per set of units.  One wave per unit or cluster, a thread per 16 columns.
__global__ __launch_bounds__(64) void unit_mask_kernel(const DevSys* __restrict__ S, const DevUnit* __restrict__ units,
                                                       const DevUnit* __restrict__ subs,
                                                       const int32_t* __restrict__ unit_atoms,
                                                       const int32_t* __restrict__ unit_cols, int64_t n_units,
                                                       uint64_t* __restrict__ mask)
{
    for (int64_t k = blockIdx.x; k < n_units; k += gridDim.x) {
        const DevUnit u = units[k];
        const int32_t* at = unit_atoms + u.atom_begin;
        const int32_t* col = unit_cols + u.atom_begin;
        for (int blk = threadIdx.x; blk < u.ld / 16; blk += 64) {
            uint64_t bits = 0;
            if (blk * 16 < u.m) {
                int lo = 0, hi = u.n_atoms - 1;  // the atom that owns column 16 blk
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (col[mid] <= blk * 16) lo = mid; else hi = mid - 1;
                }
                for (int q = lo; q < u.n_atoms && col[q] < blk * 16 + 16; ++q) {
                    const double* A = S->atom_xyzr + 4 * (int64_t)at[q];
                    const double ax = A[0], ay = A[1], az = A[2], rc2 = A[3];
                    for (int t = u.sub_begin; t < u.sub_begin + u.sub_count; ++t) {
                        const int64_t p0 = subs[t].point_begin, r0 = subs[t].row_begin - u.row_begin;
                        for (int p = 0; p < subs[t].n_points; ++p)
                            if (dist2_exact(S->px[p0 + p] - ax, S->py[p0 + p] - ay, S->pz[p0 + p] - az) < rc2)
                                bits |= 1ull << ((r0 + p) >> 4);
                    }
                }
            }
            mask[u.mask_begin + blk] = bits;
        }
    }
}

hipError_t launch_unit_masks(const DevSys* sys, const DevUnit* units, const DevUnit* subs, const int32_t* unit_atoms,
                             const int32_t* unit_cols, int64_t n_units, uint64_t* mask, hipStream_t st)
{
    if (n_units <= 0) return hipSuccess;
    hipLaunchKernelGGL(unit_mask_kernel, dim3((unsigned)std::min<int64_t>(n_units, 1 << 20)), dim3(64), 0, st, sys, units,
                       subs, unit_atoms, unit_cols, n_units, mask);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void wv_rows_kernel(const DevUnit* __restrict__ subs, int64_t n_subs,
                                                      const double* __restrict__ pw, const int32_t* __restrict__ perm,
                                                      const double* __restrict__ v, double* __restrict__ wv)
{
    for (int64_t k = blockIdx.x; k < n_subs; k += gridDim.x) {
        const int64_t p0 = subs[k].point_begin, r0 = subs[k].row_begin;
        const int np = subs[k].n_points, nr = subs[k].n_rows;
        for (int r = threadIdx.x; r < nr; r += blockDim.x) wv[r0 + r] = r < np ? pw[p0 + r] * v[perm[p0 + r]] : 0.0;
    }
}

hipError_t launch_wv_rows(const DevUnit* subs, int64_t n_subs, const double* pw, const int32_t* perm, const double* v_caller,
                          double* wv, hipStream_t st)
{
    if (n_subs <= 0) return hipSuccess;
    hipLaunchKernelGGL(wv_rows_kernel, dim3((unsigned)std::min<int64_t>(n_subs, 65536)), dim3(256), 0, st, subs, n_subs, pw,
                       perm, v_caller, wv);
    return hipGetLastError();
}

hipError_t launch_fill(double* p, int64_t n, double value, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, n, value);
    return hipGetLastError();
}

__global__ void wv_kernel(const double* __restrict__ pw, const int32_t* __restrict__ perm,
                          const double* __restrict__ v, double* __restrict__ wv, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        wv[i] = pw[i] * v[perm[i]];
}

hipError_t launch_wv(const double* pw, const int32_t* perm, const double* v_caller, double* wv,
                     int64_t n_points, hipStream_t st)
{
    if (n_points <= 0) return hipSuccess;
    int64_t blocks = (n_points + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(wv_kernel, dim3((unsigned)blocks), dim3(256), 0, st, pw, perm, v_caller, wv, n_points);
    return hipGetLastError();
}

__global__ void wa_kernel(const double* __restrict__ pw, const int32_t* __restrict__ perm,
                          const double* __restrict__ a, double* __restrict__ wa, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 3 * n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = i / 3;
        wa[i] = pw[p] * a[3 * (int64_t)perm[p] + (i - 3 * p)];
    }
}

hipError_t launch_wa(const double* pw, const int32_t* perm, const double* a_caller, double* wa, int64_t n_points,
                     hipStream_t st)
{
    if (n_points <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((3 * n_points + 255) / 256, 65536);
    hipLaunchKernelGGL(wa_kernel, dim3((unsigned)blocks), dim3(256), 0, st, pw, perm, a_caller, wa, n_points);
    return hipGetLastError();
}

// H[i][j] = H[j][i] = H[i][j] + H[j][i] for i < j, through 32x32 LDS tiles (coalesced on both
// sides): the contractions add a pair's sums to either of the two.
__global__ __launch_bounds__(256) void mirror_kernel(double* __restrict__ H, int64_t n)
{
    __shared__ double up[32][33], lo[32][33];
    const int64_t bi = blockIdx.y, bj = blockIdx.x;
    if (bi > bj) return;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
    for (int r = ty; r < 32; r += 8) {
        const int64_t i = bi * 32 + r, j = bj * 32 + tx, k = bj * 32 + r, l = bi * 32 + tx;
        up[r][tx] = (i < n && j < n) ? H[i * n + j] : 0.0;
        lo[r][tx] = (k < n && l < n) ? H[k * n + l] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int64_t i = bi * 32 + r, j = bj * 32 + tx, k = bj * 32 + r, l = bi * 32 + tx;
        if (i < n && j < n && i < j) H[i * n + j] = up[r][tx] + lo[tx][r];
        if (k < n && l < n && k > l) H[k * n + l] = up[tx][r] + lo[r][tx];
    }
}

hipError_t launch_mirror(double* H, int64_t n, hipStream_t st)
{
    if (n <= 1) return hipSuccess;
    const int64_t nt = (n + 31) / 32;
    if (nt > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(mirror_kernel, dim3((unsigned)nt, (unsigned)nt), dim3(256), 0, st, H, n);
    return hipGetLastError();
}

// N_e = sum_p w_p n_p: per-block partial sums, then one block adds them in a fixed order.
__global__ __launch_bounds__(256) void wsum_partial_kernel(const double* __restrict__ pw, const int32_t* __restrict__ perm,
                                                           const double* __restrict__ n, int64_t np,
                                                           double* __restrict__ partial)
{
    __shared__ double s[256];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < np; i += (int64_t)gridDim.x * blockDim.x)
        acc += pw[i] * n[perm[i]];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = s[0];
}

__global__ __launch_bounds__(256) void wsum_final_kernel(const double* __restrict__ partial, int nb, double* out)
{
    __shared__ double s[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nb; i += blockDim.x) acc += partial[i];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = s[0];
}

hipError_t launch_weighted_sum(const double* pw, const int32_t* perm, const double* n_caller,
                               int64_t n_points, double* partial, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(wsum_partial_kernel, dim3(WSUM_BLOCKS), dim3(256), 0, st, pw, perm, n_caller, n_points,
                       partial);
    hipLaunchKernelGGL(wsum_final_kernel, dim3(1), dim3(256), 0, st, partial, WSUM_BLOCKS, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Scratch of the allocation-free Hamiltonian call.  Every GPU that loads this code object holds
// its own copy of the array until the process ends.  In host code `scratch` names a host-side
// stand-in, not device memory: the device address is looked up once per device and kept in
// g_noalloc_ptr, and only that address is ever handed to kernels or copies.
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[NOALLOC_MAX_DEVICES] = {};
}  // namespace

hipError_t noalloc_scratch_init(int device)
{
    if (device < 0 || device >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    if (g_noalloc_ptr[device]) return hipSuccess;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;  // the caller makes `device` current first
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_noalloc_ptr[device] = ptr;
    return hipSuccess;
}

void* noalloc_scratch(int device)
{
    if (device < 0 || device >= NOALLOC_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    return g_noalloc_ptr[device];
}

}  // namespace nao
