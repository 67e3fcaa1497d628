// A context's set-up and first uses on a device that is not there: api.cpp and eig1d.cpp with the HIP calls and the
// launch functions replaced by stand-ins that keep an account of the memory, of which arrays have been filled, and of
// work that was queued and not waited for, and that fail at a chosen call.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "helm_internal.h"

using namespace helm;

namespace {

std::map<char *, size_t> live;       // allocations
std::set<const void *> filled;       // arrays with contents, by their address
size_t live_bytes = 0, copied = 0;
long calls = 0, fail_at = 0;         // device calls; the one that fails (0: none)
int queued = 0;                      // launches since the last wait for the stream
int bad = 0;
std::string at;

bool fails() { return ++calls == fail_at; }
void complain(const char *what) {
    ++bad;
    std::printf("%s: %s\n", at.c_str(), what);
}
bool inside(const void *p) {
    auto it = live.upper_bound((char *)p);
    if (it == live.begin()) return false;
    --it;
    return (char *)p < it->first + it->second;
}
void need(const void *p, const char *what) {
    if (!p || !inside(p)) complain((std::string(what) + " is no allocated array").c_str());
    else if (!filled.count(p)) complain((std::string(what) + " was never filled").c_str());
}
hipError_t launch(std::initializer_list<const void *> in = {}, std::initializer_list<const void *> out = {}, const char *what = "an input") {
    if (fails()) return hipErrorLaunchFailure;
    for (const void *p : in) need(p, what);
    for (const void *p : out)
        if (p) filled.insert(p);
    ++queued;
    return hipSuccess;
}

}  // namespace

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    if (fails()) return hipErrorOutOfMemory;
    *p = std::malloc(n ? n : 1);
    live[(char *)*p] = n;
    live_bytes += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    auto it = live.find((char *)p);
    if (it == live.end()) { complain("free of what was not allocated"); return hipErrorInvalidValue; }
    for (auto f = filled.lower_bound(p); f != filled.end() && (char *)*f < (char *)p + it->second;) f = filled.erase(f);
    live_bytes -= it->second;
    live.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    if (fails()) return hipErrorUnknown;
    std::memcpy(d, s, n);
    copied += n;
    // one copy fills every array of its range: they begin at multiples of 256 bytes
    for (size_t o = 0; o < n; o += 256) filled.insert((char *)d + o);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *, size_t n, hipMemcpyKind, hipStream_t) {
    if (fails()) return hipErrorUnknown;
    if (!inside(d)) { complain("copy to what was not allocated"); return hipErrorInvalidValue; }
    std::memset(d, 0, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    if (fails()) return hipErrorUnknown;
    queued = 0;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { queued = 0; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
}

namespace helm {
int tri_chunks(int nz) { return (nz + 7) / 8; }
int dots_blocks(long long n) { return (int)((n + 255) / 256); }
int ring_max_n() { return 832; }
int ring_rowgroups() { return 8; }
void stencil_split(StencilParams *const *ps, int n) { for (int i = 0; i < n; ++i) { ps[i]->zchunk = 1; ps[i]->zchunks = ps[i]->nz; } }
hipError_t launch_derived_fields(const double *, int, double *k2, double4 *fld, const StencilParams &, double, hipStream_t) { return launch({}, {k2, fld}); }
hipError_t launch_derived_fields_c(const double2 *, int, double *k2, double *k2i, double4 *fld, double4 *fldi, const StencilParams &, double, hipStream_t) { return launch({}, {k2, k2i, fld, fldi}); }
hipError_t launch_rhs(const StencilParams &, const double2 *, const double *k2, const double4 *, double, double2 *, hipStream_t) { return launch({k2}); }
hipError_t launch_matvec(const StencilParams &, const double2 *, const double *k2, const double4 *, const double2 *, double2 *, hipStream_t) { return launch({k2}); }
hipError_t launch_matvec(const StencilParams &, const float2 *, const double *k2, const double4 *, const double2 *, double2 *, hipStream_t) { return launch({k2}); }
hipError_t launch_dots(const double2 *, long long, int, const double2 *, long long, double2 *part, int, double2 *red, double2 *, hipStream_t) {
    if (!part || !inside(part) || !red || !inside(red)) complain("a reduction without its arrays");
    return launch();
}
hipError_t launch_lincomb(double2 *, const double2 *, double2, const double2 *, long long, int, const double2 *, long long, hipStream_t) { return launch(); }
hipError_t launch_lincomb(double2 *, const double2 *, double2, const float2 *, long long, int, const double2 *, long long, hipStream_t) { return launch(); }
hipError_t launch_lincomb_cgs(double2 *, const double2 *, long long, int, const double2 *, long long, double, hipStream_t) { return launch(); }
hipError_t launch_to_c64(const double2 *, float2 *, long long, hipStream_t) { return launch(); }
hipError_t launch_fill_zero(double2 *, long long, hipStream_t) { return launch(); }
hipError_t launch_fold_expand(const FoldBlocks &f, hipStream_t) {
    if (fails()) return hipErrorLaunchFailure;
    for (int i = 0; i < f.n; ++i) {
        need(f.b[i].src, "a compact block");
        filled.insert(f.b[i].d64);
        filled.insert(f.b[i].d32);
    }
    ++queued;
    return hipSuccess;
}
hipError_t launch_dense_forms(const double2 *s, double2 *p, double2 *t, int, hipStream_t) { return launch({s}, {p, t}, "a matrix"); }
hipError_t launch_dense_forms(const double2 *s, float2 *p, float2 *t, int, hipStream_t) { return launch({s}, {p, t}, "a matrix"); }
hipError_t launch_tri_pivots(const double2 *dx, const double2 *dy, int, int, int, double, double, double, double2, double2 *p, float2 *p32, hipStream_t, double) { return launch({dx, dy}, {p, p32}, "an eigenvalue table"); }
#define FOLD(name, TD, TM, TC) \
    hipError_t name(int, const FoldDesc &, const TD *, const TM *Ms, const TM *Ma, TC *, hipStream_t, int, bool) { return launch({Ms, Ma}, {}, "a transform block"); }
FOLD(launch_fold_z64, double2, double2, double2)
FOLD(launch_fold_z32, float2, float2, float2)
FOLD(launch_fold_z32_in64, double2, float2, float2)
FOLD(launch_fold_z32_out64, float2, float2, double2)
hipError_t launch_tridiag_chunk_z64(const double2 *, double2 *, const double2 *piv, const double2 *dx, const double2 *dy, int, int, int, double, double, double, double2, double, hipStream_t, double) { return launch({piv, dx, dy}, {}, "a z-solve table"); }
hipError_t launch_tridiag_chunk_z32(const float2 *, float2 *, const float2 *piv, const double2 *dx, const double2 *dy, int, int, int, double, double, double, double2, double, hipStream_t, double) { return launch({piv, dx, dy}, {}, "a z-solve table"); }
hipError_t launch_sym_divide_z64(double2 *, const double *tx, const double *ty, const double *tz, int, int, int, const SymParams &, hipStream_t) { return launch({tx, ty, tz}, {}, "a symbol table"); }
hipError_t launch_sym_divide_z32(float2 *, const double *tx, const double *ty, const double *tz, int, int, int, const SymParams &, hipStream_t) { return launch({tx, ty, tz}, {}, "a symbol table"); }
#define RING(S, CT)                                                                                                        \
    hipError_t launch_ring_inverse_##S(const CT *, CT *, const CT *a, const CT *b, const CT *c, const CT *d, int, int, int, int, CT *, CT *, CT *, hipStream_t) { return launch({a, b, c, d}, {}, "a face matrix"); } \
    hipError_t launch_ring_forward_##S(const CT *, const CT *, const CT *, const CT *, const CT *, double, CT *, const CT *a, const CT *b, double2, double2, double2, double2, int, int, int, CT *, CT *, hipStream_t) { return launch({a, b}, {}, "a face matrix"); }
RING(z64, double2)
RING(z32, float2)
}  // namespace helm

namespace {

constexpr int NX = 20, NY = 17, NZ = 12;
std::vector<double> k2((NX + 4) * (NY + 4) * (NZ + 4), 1.0);
char vec_y[16], vec_z[16];            // never read: the kernels are stand-ins

helm_status setup(helm_ctx **c, int kind = HELM_BC_ABC2) {
    const double h[3] = {0.05, 0.05, 0.05};
    return helm_setup(c, helm_grid{NX, NY, NZ}, h, k2.data(), 2, 4, helm_bc{kind, 3.0}, nullptr);
}

// everything that set-up queues is done when it returns: a batch works on a stream of its own
void check_setup_waits() {
    at = "set-up";
    helm_ctx *c = nullptr;
    if (setup(&c) != HELM_OK) complain("failed");
    if (queued) complain("returned with queued work on its stream");
    helm_destroy(c);
}

// every device call of a set-up or a first use fails once: the call reports it, and the next one does what was not done
void check_faults() {
    helm_ctx *c = nullptr;
    fail_at = 0, calls = 0;
    if (setup(&c) != HELM_OK) complain("set-up failed");
    const long of_setup = calls;
    helm_destroy(c);
    for (long k = 1; k <= of_setup; ++k) {
        at = "set-up, call " + std::to_string(k);
        calls = 0, fail_at = k;
        if (setup(&c) == HELM_OK || c) complain("not reported");
        if (!live.empty()) complain("memory not given back");
    }
    for (int bc : {HELM_BC_ABC2, HELM_BC_ABC3})
        for (int kind : {HELM_PREC_EIGT, HELM_PREC_PFFT, HELM_PREC_FFT2, HELM_PREC_FFT4})
            for (int fp32 = 0; fp32 < 2; ++fp32)
                for (long k = 1, of_use = 1; k <= of_use; ++k) {
                    at = "closure " + std::to_string(bc) + ", kind " + std::to_string(kind) + ", fp32 " + std::to_string(fp32) + ", call " + std::to_string(k);
                    fail_at = 0;
                    if (setup(&c, bc) != HELM_OK) complain("set-up failed");
                    calls = 0;
                    if (k == 1) {                              // how many calls the first use makes
                        if (helm_precond_apply(c, vec_y, vec_z, kind, fp32) != HELM_OK) complain("first use failed");
                        of_use = calls;
                        helm_destroy(c);
                        setup(&c, bc);
                        calls = 0;
                    }
                    fail_at = k;
                    if (helm_precond_apply(c, vec_y, vec_z, kind, fp32) == HELM_OK) complain("not reported");
                    fail_at = 0;
                    if (helm_precond_apply(c, vec_y, vec_z, kind, fp32) != HELM_OK) complain("next use failed");
                    helm_destroy(c);
                }
    // the work of helm_scale_guess: its vector, partials and reduced values on the device and the latter on the host
    for (long k = 1; k <= 4; ++k) {
        at = "scaled guess, call " + std::to_string(k);
        fail_at = 0;
        if (setup(&c) != HELM_OK) complain("set-up failed");
        calls = 0, fail_at = k;
        const helm_status st = helm_scale_guess(c, vec_y, vec_z, nullptr, nullptr);
        if (st == HELM_OK) complain("not reported");
        fail_at = 0;
        (void)helm_scale_guess(c, vec_y, vec_z, nullptr, nullptr);
        helm_destroy(c);
    }
}

// the FP32 form of the face corrections is made from the FP64 one on the device: only the sine matrices go up again
void check_uploads() {
    at = "first FP32 use of PFFT";
    helm_ctx *c = nullptr;
    if (setup(&c) != HELM_OK) complain("set-up failed");
    if (helm_precond_apply(c, vec_y, vec_z, HELM_PREC_PFFT, 0) != HELM_OK) complain("failed");
    copied = 0;
    if (helm_precond_apply(c, vec_y, vec_z, HELM_PREC_PFFT, 1) != HELM_OK) complain("failed");
    if (copied > sizeof(float2) * (NX * NX + NY * NY) + 256) complain("uploads the eigenvector matrices once more");
    helm_destroy(c);
}

// a small context is small: next to 100 bytes per unknown, its transform blocks and tables stay below half a megabyte, and
// below one with the sine transforms'
void check_memory() {
    at = "memory of a small context";
    helm_ctx *c = nullptr;
    if (setup(&c) != HELM_OK) complain("set-up failed");
    const size_t vectors = (size_t)100 * NX * NY * NZ;
    if (live_bytes > vectors + (512u << 10)) complain("set-up takes more than half a megabyte");
    if (helm_precond_apply(c, vec_y, vec_z, HELM_PREC_FFT2, 0) != HELM_OK) complain("failed");
    if (live_bytes > vectors + (1u << 20)) complain("the sine transforms take more than half a megabyte");
    helm_destroy(c);
}

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "waits") check_setup_waits();
    else if (what == "faults") check_faults();
    else if (what == "uploads") check_uploads();
    else if (what == "memory") check_memory();
    else return 2;
    if (!live.empty()) { at = "end"; complain("memory not given back"); }
    std::printf(bad ? "%d faults\n" : "ok\n", bad);
    return bad != 0;
}
