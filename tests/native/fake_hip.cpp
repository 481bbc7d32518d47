// A HIP runtime without a GPU for host-side tests: loaded into the global
// scope before the library, it answers the library's runtime calls from host
// memory and logs what would have run, one line per event: "launch <kernel>
// <grid x> <grid y>" (plain launches and each kernel node of a graph launch),
// "instantiate", "alloc".  No kernel runs.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

std::string g_log;
int g_fail_instantiate = 0;  // the next so many instantiations fail
long g_graphs = 0;           // graphs and executables that are not destroyed
std::map<const void *, std::string> g_kernels;
std::map<const void *, void *> g_vars;

struct Config {
    dim3 grid, block;
    size_t shmem;
    hipStream_t stream;
} g_config;

struct Node {
    void *func;
    dim3 grid;
};

void log_launch(const void *func, dim3 grid) {
    g_log += "launch " + g_kernels[func] + " " + std::to_string(grid.x) + " " +
             std::to_string(grid.y) + "\n";
}

hipError_t allocate(void **p, size_t bytes) {
    g_log += "alloc\n";
    *p = std::calloc(1, bytes ? bytes : 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}

}  // namespace

struct ihipGraph {
    std::vector<Node *> nodes;
};
struct hipGraphExec {
    std::vector<Node *> nodes;
    std::vector<Node> params;
};

extern "C" {

const char *fake_log() { return g_log.c_str(); }
void fake_clear() { g_log.clear(); }
void fake_fail_instantiate(int n) { g_fail_instantiate = n; }
long fake_graphs() { return g_graphs; }

void **__hipRegisterFatBinary(const void *) {
    static void *module = nullptr;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
    g_kernels[host] = name;
}
void __hipRegisterVar(void **, void *host, char *, char *, int, size_t size, int, int) {
    g_vars[host] = std::calloc(1, size);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
    g_config = Config{grid, block, shmem, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *stream) {
    *grid = g_config.grid;
    *block = g_config.block;
    *shmem = g_config.shmem;
    *stream = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *func, dim3 grid, dim3, void **, size_t, hipStream_t) {
    log_launch(func, grid);
    return hipSuccess;
}

hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t *p, int) {
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *symbol) {
    return *p = g_vars[symbol], hipSuccess;
}

hipError_t hipMalloc(void **p, size_t bytes) { return allocate(p, bytes); }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { return allocate(p, bytes); }
hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
    return std::memset(d, v, n), hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t *e) {
    return *e = reinterpret_cast<hipEvent_t>(std::malloc(1)), hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    return *s = hipStreamCaptureStatusNone, hipSuccess;
}

hipError_t hipGraphCreate(hipGraph_t *g, unsigned) {
    ++g_graphs;
    return *g = new ihipGraph, hipSuccess;
}
hipError_t hipGraphAddKernelNode(hipGraphNode_t *n, hipGraph_t g, const hipGraphNode_t *, size_t,
                                 const hipKernelNodeParams *p) {
    g->nodes.push_back(new Node{p->func, p->gridDim});
    *n = reinterpret_cast<hipGraphNode_t>(g->nodes.back());
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
    g_log += "instantiate\n";
    if (g_fail_instantiate > 0) return --g_fail_instantiate, hipErrorOutOfMemory;
    ++g_graphs;
    *e = new hipGraphExec;
    for (Node *n : g->nodes) {
        (*e)->nodes.push_back(n);
        (*e)->params.push_back(*n);
    }
    return hipSuccess;
}
hipError_t hipGraphExecKernelNodeSetParams(hipGraphExec_t e, hipGraphNode_t n,
                                           const hipKernelNodeParams *p) {
    for (size_t k = 0; k < e->nodes.size(); ++k)
        if (reinterpret_cast<hipGraphNode_t>(e->nodes[k]) == n) {
            e->params[k] = Node{p->func, p->gridDim};
            return hipSuccess;
        }
    return hipErrorInvalidValue;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
    if (!e) return hipErrorInvalidValue;
    for (const Node &n : e->params) log_launch(n.func, n.grid);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    --g_graphs;
    return delete e, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
    for (Node *n : g->nodes) delete n;
    --g_graphs;
    return delete g, hipSuccess;
}

}  // extern "C"
