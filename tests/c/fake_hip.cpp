// A GPU runtime made of host memory, loaded in front of the HIP library so
// that the host side of libpsweep.so runs on a machine without a GPU.  Device
// memory is host memory, copies happen at once, and a kernel launch is a line
// of a log: which kernel, and for the sweeps what the tables it was given say
// (the job's size, sources, output map, plane table, and whether every item
// lies inside the job).  The preparation is played as far as the log needs it:
// it marks each job's plane table with its settings and clears the counters.
// Test infrastructure only; never part of libpsweep.so.
#include <dlfcn.h>
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <string>
#include <vector>

#include "../../paper_1809_06132_amd/csrc/psweep_internal.h"

using namespace psw;

namespace {

std::string g_log;
int g_cu = 256, g_resident = 4;

void line(const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_log += buf;
    g_log += '\n';
}

const void *named(const char *symbol) {
    void *f = dlsym(RTLD_DEFAULT, symbol);
    return f ? reinterpret_cast<const void *(*)()>(f)() : nullptr;
}

const KernelEntry *sweep_kernel(const void *fn) {
    static const char *const tables[] = {"psw_kernels_grid",  "psw_kernels_extra",  "psw_kernels_small",
                                         "psw_kernels_grid8", "psw_kernels_f32img", "psw_kernels_persistent"};
    for (const char *t : tables) {
        auto *get = reinterpret_cast<int (*)(const KernelEntry **)>(dlsym(RTLD_DEFAULT, t));
        const KernelEntry *e = nullptr;
        const int n = get ? get(&e) : 0;
        for (int i = 0; i < n; ++i)
            if (e[i].fn == fn) return e + i;
    }
    return nullptr;
}

// 0 <= item < tiles x chunks of the job, and the job one of the run's
bool inside(const JobDev &J, int item) {
    const int chunks = J.nch_f + J.nch_g > 1 ? J.nch_f + J.nch_g : 1;
    return item >= 0 && item < J.tiles_x * J.tiles_y * chunks;
}

void job_line(const char *form, const KernelEntry &e, const JobDev &J, long items, bool ok) {
    line("%s w=%d h=%d src=%d window=%d tile=%dx%d chunks=%d items=%ld index=%llu plane0=%g inside=%d store=%d", form, J.w, J.h,
         J.n_src, J.window, e.rows, e.waves, J.nch_f + J.nch_g > 1 ? J.nch_f + J.nch_g : 1, items,
         (unsigned long long)(uintptr_t)J.index, J.theta ? (double)J.theta[0] : -1.0, ok ? 1 : 0, e.store);
}

int g_prep_jobs = 0;   // of the last preparation: the jobs that its run has

}  // namespace

extern "C" {

const char *fake_hip_log() { return g_log.c_str(); }
void fake_hip_clear() { g_log.clear(); }
void fake_hip_device(int cu, int resident) { g_cu = cu; g_resident = resident; }

hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3, void **args, size_t, hipStream_t) {
    if (fn == named("psw_prep_kernel")) {
        const SetupDev *su = *static_cast<SetupDev **>(args[2]);
        int *counters = *static_cast<int **>(args[3]);
        const int n = *static_cast<int *>(args[4]);
        for (unsigned z = 0; su && z < grid.z; ++z) su[z].theta[0] = (float)(su[z].near_m + 100.0 * su[z].t[0][0]);
        for (int i = 0; i < n; ++i) counters[i] = 0;
        g_prep_jobs = (int)grid.z;
        line("prep jobs=%u setup=%d", grid.z, su ? 1 : 0);
        return hipSuccess;
    }
    if (const KernelEntry *e = sweep_kernel(fn)) {
        const JobDev *jobs = *static_cast<JobDev **>(args[0]);
        if (!e->persistent) {
            bool ok = true;
            for (unsigned b = 0; b < grid.x; ++b) ok = ok && inside(*jobs, jobs->order[b]);
            job_line("grid", *e, *jobs, (long)grid.x, ok);
            return hipSuccess;
        }
        const int32_t *q = *static_cast<int32_t **>(args[1]);
        std::vector<long> items(kMaxJobs, 0);
        std::vector<char> ok(kMaxJobs, 1);
        for (int i = 0; i < q[kQueues]; ++i) {
            const uint32_t it = (uint32_t)q[kQueueHead + i];
            const int j = (int)(it >> kItemBits);
            ++items[j];
            if (j >= g_prep_jobs || !inside(jobs[j], (int)(it & ((1u << kItemBits) - 1)))) ok[j] = 0;
        }
        for (int j = 0; j < g_prep_jobs; ++j) job_line("queues", *e, jobs[j], items[j], ok[j] != 0);
        return hipSuccess;
    }
    line("other grid=%u", grid.x);
    return hipSuccess;
}

hipError_t hipGetSymbolAddress(void **p, const void *) {
    static void *mem = aligned_alloc(256, kStaticScratchBytes);
    *p = mem;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); line("upload"); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    line("upload");
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = g_cu;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = g_resident; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { *g = (hipGraph_t)malloc(1); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *x = (hipGraphExec_t)malloc(1);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { free(x); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { free(g); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { line("graph"); return hipSuccess; }

}  // extern "C"
