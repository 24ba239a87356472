// The plans' host logic (sde_api.cpp) on a host without a GPU: the HIP runtime
// and the kernel launchers are stand-ins that record what they are asked for
// and can be told to fail.  Exits non-zero when a check fails.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>

#include "inputs.hpp"
#include "sde.h"
#include "sde_internal.hpp"

static int failures = 0;
static size_t last_reset = 0;         // voxel words cleared by the last reset
static int fail_transport = 0;        // fail the next launches of the transport
static int instantiated = 0;          // graphs
static int launched = 0;
static bool capturing = false;
static sde::KParams last_params;

static void check(const char* what, bool ok) {
    std::printf("%-66s %s\n", what, ok ? "ok" : "FAILED");
    if (!ok) ++failures;
}

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    *p = std::calloc(1, n ? n : 1);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreate(hipStream_t* s) {
    *s = reinterpret_cast<hipStream_t>(8);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    capturing = true;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    capturing = false;
    *g = reinterpret_cast<hipGraph_t>(8);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    ++instantiated;
    *e = reinterpret_cast<hipGraphExec_t>(8);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
    ++launched;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = reinterpret_cast<hipEvent_t>(8);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 0.0f;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorNotSupported; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
// what a translation unit with a device variable registers at start-up
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}

namespace sde {
hipError_t launch_pack_phantom(const uint8_t*, const float*, uint2*, size_t, int, unsigned int*,
                               unsigned int* rho_max, hipStream_t) {
    const float one = 1.0f;
    std::memcpy(rho_max, &one, sizeof one);
    return hipSuccess;
}
hipError_t launch_reset(unsigned long long*, size_t n, unsigned long long*, unsigned long long*,
                        hipStream_t) {
    last_reset = n;
    return hipSuccess;
}
hipError_t launch_transport(const KParams& p, int, int, size_t, hipStream_t) {
    last_params = p;
    if (fail_transport > 0) {
        --fail_transport;
        return hipErrorLaunchFailure;
    }
    return hipSuccess;
}
hipError_t launch_convert(unsigned long long*, int, const uint2*, size_t, double, double, double*,
                          unsigned long long*, hipStream_t) { return hipSuccess; }
hipError_t launch_gamma(const double*, const double*, int, int, int, int, double, double, double,
                        double, double, double, double, int, int, unsigned long long*, unsigned*,
                        unsigned, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_zero_u64(unsigned long long*, int, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_max(const double*, size_t, unsigned long long*, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_sbm_polar(const float*, const float*, const float*, int, float*, float*,
                            hipStream_t) { return hipErrorNotSupported; }
hipError_t transport_kernel_attributes(size_t) { return hipSuccess; }
hipError_t launch_philox_words(unsigned long long, const unsigned long long*, const unsigned*,
                               const unsigned*, int, uint4*, hipStream_t) {
    return hipErrorNotSupported;
}
}  // namespace sde

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    const Bundle b = Bundle::read(argv[1]);
    Inputs in(b);
    check("tables", sde_init_materials(in.mats.data(), 1, &in.params, nullptr) == SDE_OK);

    const int n = 40;
    const size_t nvox = (size_t)n * n * n;
    uint8_t* mat = (uint8_t*)std::calloc(nvox, 1);
    float* rho = (float*)std::calloc(nvox, sizeof(float));
    double* dose = (double*)std::calloc(nvox, sizeof(double));
    sde_spot spot{100.0, 0.0, 0.0, 0.0, 0.1, 1e6, 1000};
    sde_beam beam{1, &spot};
    sde_phantom ph{n, n, n, 0.1, 0.1, 0.1, {-2.0, -2.0, 0.0}, mat, rho};
    sde_plan* p = nullptr;

    // the launch of a caller who names none: a tile around the beam, and one
    // inside the phantom wherever the beam is or the phantom is said to be
    check("plan", sde_plan_create(&beam, &ph, 0, 1, nullptr, &p) == SDE_OK);
    check("plan executes", sde_plan_execute(p, dose, 0) == SDE_OK);
    check("a tile around the beam",
          last_params.tile_nx > 0 && last_params.tile_x0 <= 20 &&
              last_params.tile_x0 + last_params.tile_nx > 20);
    sde_plan_destroy(p);
    const double inf = std::numeric_limits<double>::infinity(), nan = std::nan("");
    for (const double o : {nan, inf, -inf, 1e300, -1e300})
        for (int a = 0; a < 3; ++a) {
            sde_phantom q = ph;
            q.origin_cm[a] = o;
            p = nullptr;
            const int rc = sde_plan_create(&beam, &q, 0, 1, nullptr, &p);
            char what[80];
            std::snprintf(what, sizeof what, "origin %g on axis %d", o, a);
            check(what, rc == SDE_OK);
            sde_plan_destroy(p);
        }
    // tally replicas: an execution clears the first one; after one that failed
    // half-way the next clears all of them, and no later one does
    sde_launch L{};
    L.tally_replicas = 4;
    for (const int graph : {0, 1}) {
        std::printf("graph %d\n", graph);
        p = nullptr;
        check("plan", sde_plan_create(&beam, &ph, 0, 1, &L, &p) == SDE_OK);
        check("executes", sde_plan_execute(p, dose, graph) == SDE_OK && last_reset == nvox);
        fail_transport = 1;
        check("an execution fails", sde_plan_execute(p, dose, 0) != SDE_OK);
        last_reset = 0;
        check("the next clears every replica",
              sde_plan_execute(p, dose, graph) == SDE_OK && last_reset == 4 * nvox);
        check("the one after the first alone",
              sde_plan_execute(p, dose, graph) == SDE_OK && last_reset == nvox);
        const int made = instantiated, ran = launched;
        check("and goes on", sde_plan_execute(p, dose, graph) == SDE_OK &&
                                 sde_plan_execute(p, dose, 1 - graph) == SDE_OK &&
                                 last_reset == nvox);
        check("with the graph it has", graph ? instantiated == made && launched == ran + 1
                                             : instantiated <= made + 1);
        sde_plan_destroy(p);
    }
    // recording runs nothing: one that fails leaves the replicas as they were
    p = nullptr;
    check("plan", sde_plan_create(&beam, &ph, 0, 1, &L, &p) == SDE_OK);
    fail_transport = 1;
    check("recording fails", sde_plan_execute(p, dose, 1) != SDE_OK);
    check("the next execution clears the first replica",
          sde_plan_execute(p, dose, 0) == SDE_OK && last_reset == nvox);
    fail_transport = 1;
    check("an execution fails", sde_plan_execute(p, dose, 0) != SDE_OK);
    // a caller's own recording of an execution clears all, and so does the next
    capturing = true;
    check("recorded by the caller",
          sde_plan_execute(p, dose, 0) == SDE_OK && last_reset == 4 * nvox);
    capturing = false;
    last_reset = 0;
    check("and run", sde_plan_execute(p, dose, 0) == SDE_OK && last_reset == 4 * nvox);
    check("then the first alone", sde_plan_execute(p, dose, 0) == SDE_OK && last_reset == nvox);
    sde_plan_destroy(p);
    std::printf("done: %d failures\n", failures);
    return failures ? 1 : 0;
}
