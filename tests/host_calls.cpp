// Runs calls of libswarm.so on a stand-in for the HIP runtime that keeps device memory on the host and executes nothing, and
// prints what the library asked of it: kernel launches by name, event records and waits, the status of each call.
// The symbols below are found ahead of the real runtime's, which the library is linked against.  No GPU is touched.
//   host_calls run      n d bits H batch graph count       swarm_run_sequential; batch 0: diagonal objective, else least squares
//   host_calls interact n d bits H batch graph             swarm_interact(0, a neighbour)
//   host_calls steps    n d bits H batch graph             swarm_local_steps(all)
//   host_calls rounds   n d bits H fail count              `count` rounds of one pair; the launch numbered `fail` fails (0: none)
//   host_calls two      n d bits H batch graph             the same of one swarm, then of a second one that is set up after it
//   host_calls mlp      n in hid out batch H nodes         swarm_local_steps(0 .. nodes - 1) of perceptrons, bf16x3 arithmetic
//   host_calls mlp_fp32 n in hid out batch H nodes         the same in float32
//   host_calls mlp_room n in hid out batch H nodes room    as mlp, with `room` bytes of device memory left for the arithmetic; and
//                                                          device memory with the objective, the arithmetic, and back in float32
// In the environment, for the least-squares objective: GROUPS_PER_UNIT, workgroups that fit one of 256 compute units (else the
// runtime cannot tell), ROOM, bytes of device memory left for it, and INPLACE, where the steps update the models themselves.
// graph: complete, ring (two neighbours), path, star, or hubsK (nodes 0..K-1 joined to all others).
#include <cxxabi.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "swarm.h"

namespace {
struct Dim3 { uint32_t x, y, z; };
bool logging = false;
int launches = 0, fail_at = 0, last_error = 0;
size_t in_use = 0, memory = ~(size_t)0;                            // device memory
const char *setting(const char *name) { return std::getenv(name); }
std::map<void *, size_t> &allocations() { static std::map<void *, size_t> a; return a; }
struct Call { Dim3 grid, block; size_t shared; void *stream; } pushed;
std::map<const void *, std::string> &kernels() { static std::map<const void *, std::string> k; return k; }
int event_number(const void *e) { return (int)(intptr_t)e; }
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    int status;
    char *text = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    std::string plain = status == 0 ? text : name;
    std::free(text);
    if (plain.rfind("void ", 0) == 0) plain.erase(0, 5);
    kernels()[host] = plain.substr(plain.find("swarm::") + 7, plain.find('(') - plain.find("swarm::") - 7);
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream) { pushed = Call{grid, block, shared, stream}; return 0; }
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream) {
    *grid = pushed.grid; *block = pushed.block; *shared = pushed.shared; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *kernel, Dim3 grid, Dim3 block, void **, size_t shared, void *) {
    if (!logging) return 0;
    std::printf("launch %s grid %u %u block %u shared %zu\n", kernels()[kernel].c_str(), grid.x, grid.y, block.x, shared);
    if (++launches == fail_at) last_error = 1;
    return last_error;
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int) { return "stand-in error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *value, int, int) { *value = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *groups, const void *, int, size_t) {
    if (!setting("GROUPS_PER_UNIT")) { last_error = 1; return 1; }
    *groups = std::atoi(setting("GROUPS_PER_UNIT"));
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(n ? n : 1, 1); return *p ? 0 : 2; }
int hipHostFree(void *p) { std::free(p); return 0; }
int hipMalloc(void **p, size_t n) {
    if (n > memory - in_use || hipHostMalloc(p, n, 0)) { last_error = 2; return 2; }
    in_use += allocations()[*p] = n;
    return 0;
}
int hipFree(void *p) {
    in_use -= allocations()[p];
    allocations().erase(p);
    return hipHostFree(p);
}
int hipHostGetDevicePointer(void **d, void *p, unsigned) { *d = p; return 0; }
int hipMemset(void *, int, size_t) { return 0; }
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipMemcpy(void *, const void *, size_t, int) { return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) {
    if (logging) std::printf("copy\n");
    return 0;
}
int hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, int, void *) { return 0; }
int hipGetSymbolAddress(void **p, const void *) { static char symbol[64]; *p = symbol; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = (void *)1; return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { static intptr_t next = 0; *e = (void *)++next; return 0; }
int hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0.f; return 0; }
int hipEventRecord(void *e, void *) { if (logging) std::printf("record %d\n", event_number(e)); return 0; }
int hipDeviceSynchronize() { if (logging) std::printf("wait for all\n"); return 0; }
int hipStreamIsCapturing(void *, int *capturing) { *capturing = 0; return 0; }
int hipStreamWaitEvent(void *, void *e, unsigned) { if (logging) std::printf("stream waits %d\n", event_number(e)); return 0; }
int hipEventSynchronize(void *e) { if (logging) std::printf("wait %d\n", event_number(e)); return 0; }
}

namespace {
std::vector<uint32_t> edges_of(const std::string &graph, uint32_t n) {
    std::vector<uint32_t> e;
    const uint32_t hubs = graph == "star" ? 1 : graph.rfind("hubs", 0) == 0 ? (uint32_t)std::atoi(graph.c_str() + 4) : 0;
    for (uint32_t u = 0; u < n; ++u)
        for (uint32_t v = u + 1; v < n; ++v) {
            const bool next = v == u + 1, around = u == 0 && v == n - 1 && n > 2;
            if (graph == "complete" || (graph == "path" && next) || (graph == "ring" && (next || around)) ||
                (hubs && u < hubs && v >= hubs)) {
                e.push_back(u);
                e.push_back(v);
            }
        }
    return e;
}
}  // namespace

static int perceptrons(char **argv, uint32_t arithmetic, const char *room) {
    uint32_t v[7];                                                  // n, in, hid, out, batch, H, nodes
    for (int k = 0; k < 7; ++k) v[k] = (uint32_t)std::strtoul(argv[2 + k], nullptr, 10);
    const std::vector<uint32_t> edges = edges_of("ring", v[0]);
    swarm_config c{};
    c.n = v[0];
    c.d = (uint64_t)v[2] * v[1] + v[2] + (uint64_t)v[3] * v[2] + v[3];
    c.bits = 8;
    c.H = v[5];
    c.edges = edges.data();
    c.n_edges = (uint32_t)(edges.size() / 2);
    c.eps = 0.5f;
    c.lr = 0.1f;
    c.seed = 1;
    swarm_t h = nullptr;
    const float *data = reinterpret_cast<const float *>(64);        // the host never reads them
    if (swarm_init(&c, nullptr, nullptr, &h) != SWARM_OK) { std::printf("init: %s\n", swarm_last_error(nullptr)); return 1; }
    swarm_status rc = swarm_set_objective_mlp(h, v[1], v[2], v[3], data, data, 0.5f, v[4]);
    const size_t objective = in_use;
    if (room) memory = in_use + std::strtoull(room, nullptr, 10);
    if (rc == SWARM_OK) rc = swarm_set_mlp_arithmetic(h, arithmetic);
    const size_t chosen = in_use;
    memory = ~(size_t)0;
    if (rc != SWARM_OK) { std::printf("objective: %s\nstatus %d\n", swarm_last_error(h), rc); swarm_destroy(h); return 0; }
    std::vector<uint32_t> nodes(v[6]);
    for (uint32_t k = 0; k < v[6]; ++k) nodes[k] = k;
    logging = true;
    rc = v[6] < v[0] ? swarm_local_steps(h, nodes.data(), v[6]) : swarm_local_steps(h, nullptr, 0);
    logging = false;
    std::printf("status %d\n", rc);
    if (room) {
        rc = swarm_set_mlp_arithmetic(h, SWARM_MLP_FP32);
        std::printf("memory %zu %zu %zu\nstatus %d\n", objective, chosen, in_use, rc);
    }
    swarm_destroy(h);
    return 0;
}

int main(int argc, char **argv) {
    if (argc < 8) return 2;
    const std::string call = argv[1];
    if (call == "mlp") return argc < 9 ? 2 : perceptrons(argv, SWARM_MLP_BF16X3, nullptr);
    if (call == "mlp_room") return argc < 10 ? 2 : perceptrons(argv, SWARM_MLP_BF16X3, argv[9]);
    if (call == "mlp_fp32") return argc < 9 ? 2 : perceptrons(argv, SWARM_MLP_FP32, nullptr);
    const uint32_t batch = call == "rounds" ? 0u : (uint32_t)std::atoi(argv[6]);
    const std::string graph = call == "rounds" ? "complete" : argv[7];
    swarm_config c{};
    c.n = (uint32_t)std::atoi(argv[2]);
    c.d = std::strtoull(argv[3], nullptr, 10);
    c.bits = (uint32_t)std::atoi(argv[4]);
    c.H = (uint32_t)std::atoi(argv[5]);
    const std::vector<uint32_t> edges = edges_of(graph, c.n);
    c.edges = edges.data();
    c.n_edges = (uint32_t)(edges.size() / 2);
    c.eps = 0.5f;
    c.lr = 0.1f;
    c.seed = 1;
    c.apply_mode = setting("INPLACE") ? SWARM_APPLY_INPLACE : SWARM_APPLY_DEFERRED;
    swarm_t h = nullptr;
    const float *data = reinterpret_cast<const float *>(64);        // objective data: the host never reads them
    if (swarm_init(&c, nullptr, nullptr, &h) != SWARM_OK) { std::printf("init: %s\n", swarm_last_error(nullptr)); return 1; }
    if (setting("ROOM")) memory = in_use + std::strtoull(setting("ROOM"), nullptr, 10);
    swarm_status rc = batch ? swarm_set_objective_lsq(h, data, data, 64, batch) : swarm_set_objective_diag(h, data, data, 0.1f);
    if (rc != SWARM_OK) { std::printf("objective: %s\n", swarm_last_error(h)); return 1; }
    memory = ~(size_t)0;
    float *snapshots = nullptr;
    if (c.apply_mode == SWARM_APPLY_DEFERRED) swarm_models_ptr(h, SWARM_MODELS_SNAP, &snapshots);      // created ahead of the log
    logging = true;
    if (call == "run") {
        uint32_t reported = 0;
        rc = swarm_run_sequential(h, (uint32_t)std::atoi(argv[8]), nullptr, &reported);
        std::printf("reported %u\n", reported);
    } else if (call == "interact") {
        rc = swarm_interact(h, edges[0], edges[1]);
    } else if (call == "steps") {
        rc = swarm_local_steps(h, nullptr, 0);
    } else if (call == "two") {
        swarm_t second = nullptr;
        rc = swarm_local_steps(h, nullptr, 0);
        if (rc == SWARM_OK) rc = swarm_init(&c, nullptr, nullptr, &second);
        if (rc == SWARM_OK) rc = swarm_set_objective_lsq(second, data, data, 64, batch);
        if (rc == SWARM_OK) rc = swarm_local_steps(second, nullptr, 0);
        if (rc == SWARM_OK) rc = swarm_local_steps(h, nullptr, 0);
        swarm_destroy(second);
        if (rc == SWARM_OK) rc = swarm_local_steps(h, nullptr, 0);
    } else if (call == "rounds") {
        fail_at = std::atoi(argv[6]);
        const uint32_t pair[2] = {0, 1};
        for (int r = 0; r < std::atoi(argv[7]); ++r) {
            rc = swarm_round_fused(h, pair, 1, nullptr);
            std::printf("status %d\n", rc);
        }
    } else {
        return 2;
    }
    logging = false;
    std::printf("status %d\n", rc);
    swarm_destroy(h);
    return 0;
}
