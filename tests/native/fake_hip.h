// A HIP runtime and the kernel launchers of devtypes.h on the host, for checks of runtime.cpp
// without a GPU: device memory is host memory whose live ranges are known, and every launcher
// checks the ranges that its kernel would read or write against them.  A violation is recorded in
// fake::faults.  Captured launches are checked again whenever their graph is launched.
#pragma once

#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "devtypes.h"

namespace fake {

std::recursive_mutex mu;
std::map<uintptr_t, size_t> live;
std::vector<std::string> faults;
size_t device_limit = 0;          // bytes that hipMalloc gives out at most (0 = no limit)
size_t device_used = 0;
std::atomic<int> launches{0};      // contraction launches
std::atomic<int> cluster_launches{0};  // ... of them over clusters
std::vector<std::function<void()>>* capturing = nullptr;

inline void fault(const std::string& m)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (faults.size() < 100) faults.push_back(m);
}

// [p, p + bytes) must lie in one live allocation
inline bool range(const void* p, int64_t bytes, const char* what)
{
    if (bytes == 0) return true;
    std::lock_guard<std::recursive_mutex> lk(mu);
    const uintptr_t a = (uintptr_t)p;
    auto it = live.upper_bound(a);
    if (bytes > 0 && it != live.begin()) {
        --it;
        if (a + (size_t)bytes <= it->first + it->second) return true;
    }
    fault(std::string(what) + ": " + std::to_string(bytes) + " B are not in one allocation");
    return false;
}

inline hipError_t run(std::function<void()> f)
{
    if (capturing) capturing->push_back(std::move(f));
    else f();
    return hipSuccess;
}

using namespace nao;

inline bool system_ok(const DevSeg& g)
{
    if (!range(g.sys, sizeof(DevSys), "system")) return false;
    const DevSys& S = *g.sys;
    return range(S.px, S.n_points * 8, "px") && range(S.pw, S.n_points * 8, "pw") && range(S.perm, S.n_points * 4, "perm");
}

// rows of a unit or cluster and its lists, as a contraction reads them
inline bool unit_rows(const DevSeg& g, const DevUnit& u, size_t esz, const char* what)
{
    return range(static_cast<const char*>(g.phi) + u.out_offset * esz, (int64_t)u.n_rows * u.ld * esz, what) &&
           range(g.unit_fn + u.fn_begin, u.m * 4, "function list") &&
           range(g.unit_mask + u.mask_begin, u.ld / 16 * 8, "masks");
}

inline void check_basis(const DevSeg* segs, int n, bool f32, int extra)
{
    const size_t esz = f32 ? 4 : 8;
    if (!range(segs, n * sizeof(DevSeg), "basis segments")) return;
    for (int s = 0; s < n; ++s) {
        const DevSeg g = segs[s];
        if (!system_ok(g) || !range(g.units + g.unit_begin, g.unit_count * sizeof(DevUnit), "basis units")) return;
        for (int64_t k = 0; k < g.unit_count; ++k) {
            const DevUnit& u = g.units[g.unit_begin + k];
            const int64_t bytes = (int64_t)u.n_rows * u.ld * esz;
            if (!range(static_cast<char*>(g.phi) + u.out_offset * esz, bytes, "basis values")) return;
            if (!range(g.unit_atoms + u.atom_begin, u.n_atoms * 4, "atoms") || !range(g.unit_cols + u.atom_begin, u.n_atoms * 4, "columns")) return;
            const bool grad = extra == EXTRA_GRAD || extra == EXTRA_GRAD_H;
            for (int p = 0; p < (grad ? 3 : extra != EXTRA_NONE); ++p)
                if (!range(static_cast<char*>(g.gphi) + (p * g.plane + u.out_offset) * esz, bytes, "extra values")) return;
            if (extra == EXTRA_GRAD_H && !range(static_cast<char*>(g.hphi) + u.out_offset * esz, bytes, "h values")) return;
            if (extra > EXTRA_GRAD && !range(g.wv + u.point_begin, u.n_points * 8, "w v of the basis launch")) return;
            if (g.wa && !range(g.wa + 3 * u.point_begin, u.n_points * 24, "w a")) return;
        }
    }
}

inline void check_h(const DevSeg* segs, int n, bool f32, bool two)
{
    const size_t esz = f32 ? 4 : 8;
    if (!range(segs, n * sizeof(DevSeg), "Hamiltonian segments")) return;
    ++launches;
    for (int s = 0; s < n; ++s) {
        const DevSeg g = segs[s];
        if (g.item_units != g.units) ++cluster_launches;
        if (!system_ok(g) || !range(static_cast<const HItem*>(g.items) + g.item_begin, g.item_count * sizeof(HItem), "tile pairs")) return;
        if (!range(g.H, g.ld * g.ld * 8, "H")) return;
        for (int64_t k = 0; k < g.item_count; ++k) {
            const DevUnit* u = g.item_units + static_cast<const HItem*>(g.items)[g.item_begin + k].unit;
            if (!range(u, sizeof(DevUnit), "unit of a tile pair") || !unit_rows(g, *u, esz, "values of a tile pair")) return;
            if (!two && !range(g.wv + u->row_begin, u->n_rows * 8, "w v of a tile pair")) return;
            if (two && !range(static_cast<char*>(g.gphi) + u->out_offset * esz, (int64_t)u->n_rows * u->ld * esz, "L of a tile pair")) return;
        }
    }
}

inline void check_n(const DevSeg* segs, int n, bool f32, int planes, bool force)
{
    const size_t esz = f32 ? 4 : 8;
    if (!range(segs, n * sizeof(DevSeg), "density segments")) return;
    ++launches;
    for (int s = 0; s < n; ++s) {
        const DevSeg g = segs[s];
        if (!system_ok(g) || !range(g.D, g.ld * g.ld * 8, "D")) return;
        if (force ? !range(g.fb, FORCE_COPIES * g.ld * 24, "force sums") || !range(g.Q, g.ld * g.ld * 8, "Q") : !range(g.n, g.sys->n_points * 8, "n")) return;
        if (planes == 3 && !force && !range(g.gn, g.sys->n_points * 24, "grad n")) return;
        if (force && f32) {
            if (!range(static_cast<const NItem*>(g.items) + g.item_begin, g.item_count * sizeof(NItem), "column tiles")) return;
            for (int64_t k = 0; k < g.item_count; ++k) {
                const DevUnit& u = g.item_units[static_cast<const NItem*>(g.items)[g.item_begin + k].unit];
                const int64_t bytes = (int64_t)u.n_rows * u.ld * esz;
                if (!unit_rows(g, u, esz, "values of a column tile") || !range(static_cast<char*>(g.hphi) + u.out_offset * esz, bytes, "h values of a tile")) return;
                for (int p = 0; p < 3; ++p)
                    if (!range(static_cast<char*>(g.gphi) + (p * g.plane + u.out_offset) * esz, bytes, "gradients of a tile")) return;
            }
            continue;
        }
        if (!range(static_cast<const NTile*>(g.items) + g.item_begin, g.item_count * sizeof(NTile), "column tiles")) return;
        for (int64_t k = 0; k < g.item_count; ++k) {
            const NTile& t = static_cast<const NTile*>(g.items)[g.item_begin + k];
            const int64_t bytes = (int64_t)t.n_rows * t.ld * esz;
            if (!range(static_cast<char*>(g.phi) + t.out_offset * esz, bytes, "values of a column tile") ||
                !range(g.unit_fn + t.fn_begin, t.m * 4, "function list") || !range(g.unit_mask + t.mask_begin, t.ld / 16 * 8, "masks")) return;
            for (int p = 0; p < planes; ++p)
                if (!range(static_cast<char*>(g.gphi) + (p * g.plane + t.out_offset) * esz, bytes, "gradients of a tile")) return;
            if (force && !range(static_cast<char*>(g.hphi) + t.out_offset * esz, bytes, "h values of a tile")) return;
        }
    }
}

}  // namespace fake

// ------------------------------------------------------------------------------ launchers
namespace nao {

hipError_t launch_basis(const DevSeg* s, int n, int64_t, int, const BasisShape&, bool f32, hipStream_t, int64_t, int extra)
{
    return fake::run([=] { fake::check_basis(s, n, f32, extra); });
}
hipError_t launch_h(Mode m, const DevSeg* s, int n, int64_t, hipStream_t, int64_t, int)
{
    return fake::run([=] { fake::check_h(s, n, m != MODE_FP64, false); });
}
hipError_t launch_h_gga(Mode m, const DevSeg* s, int n, int64_t, hipStream_t)
{
    return fake::run([=] { fake::check_h(s, n, m != MODE_FP64, true); });
}
hipError_t launch_n(Mode m, const DevSeg* s, int n, int64_t, hipStream_t, int64_t)
{
    return fake::run([=] { fake::check_n(s, n, m != MODE_FP64, 0, false); });
}
hipError_t launch_n_grad(Mode m, const DevSeg* s, int n, int64_t, hipStream_t)
{
    return fake::run([=] { fake::check_n(s, n, m != MODE_FP64, 3, false); });
}
hipError_t launch_n_force(Mode m, const DevSeg* s, int n, int64_t, hipStream_t)
{
    return fake::run([=] { fake::check_n(s, n, m != MODE_FP64, 3, true); });
}
hipError_t launch_force_atoms(const double* fb, const int64_t* first, int64_t n, int64_t nb, double* F, hipStream_t)
{
    return fake::run([=] {
        if (fake::range(first, (n + 1) * 8, "atom_first")) fake::range(fb, FORCE_COPIES * first[n] * 24, "force sums");
        fake::range(F, 24 * n, "F");
    });
}
hipError_t launch_wa(const double* pw, const int32_t* perm, const double* a, double* wa, int64_t n, hipStream_t)
{
    return fake::run([=] {
        fake::range(pw, 8 * n, "pw") && fake::range(perm, 4 * n, "perm") && fake::range(a, 24 * n, "a") && fake::range(wa, 24 * n, "w a written");
    });
}
hipError_t launch_wv(const double* pw, const int32_t* perm, const double* v, double* wv, int64_t n, hipStream_t)
{
    return fake::run([=] {
        fake::range(pw, 8 * n, "pw") && fake::range(perm, 4 * n, "perm") && fake::range(v, 8 * n, "v") && fake::range(wv, 8 * n, "w v written");
    });
}
hipError_t launch_wv_rows(const DevUnit* subs, int64_t n, const double* pw, const int32_t*, const double* v, double* wv, hipStream_t)
{
    return fake::run([=] {
        if (!fake::range(subs, n * sizeof(DevUnit), "units of w v rows")) return;
        for (int64_t k = 0; k < n; ++k)
            if (!fake::range(pw + subs[k].point_begin, 8 * subs[k].n_points, "pw of w v rows") ||
                !fake::range(wv + subs[k].row_begin, 8 * subs[k].n_rows, "w v rows written"))
                return;
        fake::range(v, 8, "v");
    });
}
hipError_t launch_unit_masks(const DevSys* sys, const DevUnit* units, const DevUnit* subs, const int32_t* atoms, const int32_t* cols,
                             int64_t n, uint64_t* mask, hipStream_t)
{
    return fake::run([=] {
        if (!fake::range(sys, sizeof(DevSys), "system") || !fake::range(units, n * sizeof(DevUnit), "units of masks")) return;
        for (int64_t k = 0; k < n; ++k) {
            const DevUnit& u = units[k];
            if (!fake::range(subs + u.sub_begin, u.sub_count * sizeof(DevUnit), "parts of masks") ||
                !fake::range(atoms + u.atom_begin, u.n_atoms * 4, "atoms of masks") || !fake::range(cols + u.atom_begin, u.n_atoms * 4, "columns of masks") ||
                !fake::range(mask + u.mask_begin, u.ld / 16 * 8, "masks written"))
                return;
        }
    });
}
hipError_t launch_fill(double* p, int64_t n, double, hipStream_t)
{
    return fake::run([=] { fake::range(p, 8 * n, "fill"); });
}
hipError_t launch_mirror(double* H, int64_t n, hipStream_t)
{
    return fake::run([=] { fake::range(H, 8 * n * n, "mirror"); });
}
hipError_t launch_weighted_sum(const double* pw, const int32_t*, const double* nc, int64_t n, double* partial, double* out, hipStream_t)
{
    return fake::run([=] {
        fake::range(pw, 8 * n, "pw"), fake::range(nc, 8 * n, "n"), fake::range(partial, 8 * WSUM_BLOCKS, "partials"), fake::range(out, 8, "N_e");
    });
}
void* noalloc_scratch(int)
{
    static void* p = nullptr;
    std::lock_guard<std::recursive_mutex> lk(fake::mu);
    if (!p) {
        p = std::malloc(NOALLOC_SCRATCH_BYTES);
        fake::live[(uintptr_t)p] = NOALLOC_SCRATCH_BYTES;
    }
    return p;
}
hipError_t noalloc_scratch_init(int) { return hipSuccess; }

}  // namespace nao

// ----------------------------------------------------------------------------------- runtime
extern "C" {

hipError_t hipMalloc(void** p, size_t n)
{
    std::lock_guard<std::recursive_mutex> lk(fake::mu);
    *p = nullptr;
    if (fake::device_limit && fake::device_used + n > fake::device_limit) return hipErrorOutOfMemory;
    *p = std::malloc(n ? n : 1);
    if (!*p) return hipErrorOutOfMemory;
    fake::live[(uintptr_t)*p] = n;
    fake::device_used += n;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    std::lock_guard<std::recursive_mutex> lk(fake::mu);
    if (!p) return hipSuccess;
    auto it = fake::live.find((uintptr_t)p);
    if (it == fake::live.end()) return fake::fault("hipFree of memory that is not live"), hipErrorInvalidValue;
    fake::device_used -= it->second;
    fake::live.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t)
{
    bool ok = true;
    if (k == hipMemcpyHostToDevice || k == hipMemcpyDeviceToDevice) ok = fake::range(d, n, "copy to the device") && ok;
    if (k == hipMemcpyDeviceToHost || k == hipMemcpyDeviceToDevice) ok = fake::range(s, n, "copy from the device") && ok;
    if (ok && n) std::memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950:fake");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)std::malloc(1), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free((void*)e), hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { return *t = 1.0f, hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)std::malloc(1), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free((void*)s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    fake::capturing = new std::vector<std::function<void()>>();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    *g = reinterpret_cast<hipGraph_t>(fake::capturing);
    fake::capturing = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t)
{
    return *e = reinterpret_cast<hipGraphExec_t>(g), hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t)
{
    for (auto& f : *reinterpret_cast<std::vector<std::function<void()>>*>(e)) f();
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return delete reinterpret_cast<std::vector<std::function<void()>>*>(g), hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"
