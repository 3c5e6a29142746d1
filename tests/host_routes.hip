// The library's host side on the CPU: sigattn_api.hip compiled for the host alone, with a HIP runtime that launches nothing and
// keeps what it was asked to launch.
#include "sigattn_api.hip"

#include <cstring>
#include <map>
#include <string>
#include <vector>

struct Launch {
    char kernel[128];
    int grid, block, lds;
    int B, N, N_str, in_order, groups;       // of the (first) parameters; of a one-pass launch B, L_q, L_k, group, 0
    const void *q;
    const void *part, *plan, *flags;         // one pass: its places in the workspace
};

static std::map<const void *, std::string> names;
static std::vector<Launch> launches;
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } config;
static void *module_handle;

extern "C" {
void **__hipRegisterFatBinary(const void *) { return &module_handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names[host] = name; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) { config = {grid, block, lds, stream}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
    *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int *device) { *device = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **address, const void *) { *address = reinterpret_cast<void *>(4096); return hipSuccess; }
hipError_t hipLaunchKernel(const void *host, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t) {
    Launch l{};
    const std::string &name = names[host];
    strncpy(l.kernel, name.c_str(), sizeof l.kernel - 1);
    l.grid = (int)grid.x; l.block = (int)block.x; l.lds = (int)lds;
    if (name.find("onepass") != std::string::npos) {
        const onepass::Params &p = *static_cast<const onepass::Params *>(args[0]);
        l.B = p.B; l.N = p.L_q; l.N_str = p.L_k; l.in_order = p.group; l.q = p.q;
        l.part = p.part; l.plan = p.plan; l.flags = p.flags;
    } else if (name.find("db_reduce") == std::string::npos) {
        const Params &p = *static_cast<const Params *>(args[0]);
        l.B = p.B; l.N = p.N; l.N_str = p.N_str; l.in_order = p.in_order; l.groups = p.groups; l.q = p.q;
    }
    launches.push_back(l);
    return hipSuccess;
}

int routes_take(Launch *out, int most) {     // the launches since the last call
    const int n = (int)launches.size();
    for (int i = 0; i < n && i < most; ++i) out[i] = launches[i];
    launches.clear();
    return n;
}
}
