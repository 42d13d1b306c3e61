// Runs calls of include/irbe.h without a GPU and prints what each asks of the HIP
// runtime: this program defines the runtime functions that libirbe.so imports, so
// that the library's references bind here. "Device" memory is host memory, copies
// are made, kernels are not run.
//
//   hip_record <libirbe.so> <command>...
//
// Commands (each prints "= <command> <status>" and, before it, one line per runtime
// call made meanwhile):
//   create:key=value,...   a handle (n, box, rcore, rshell, p, types, hint, skin, fp64, stencil, entries)
//   set | lj | charge      irbe_set_system; irbe_update_parameters with LJ tables, with charges
//   build | forces | backward | sync
//   counts                 prints the row capacities of IRBE_DBG_COUNTS
//   capture=0|1            the stream reports that it is being captured
//   overflow=core,shell,words,err   what the list checks read back from now on
//   fail=k                 the (k + 1)-th allocation from now on fails, once (-1: none)
#include <dlfcn.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "irbe.h"

namespace {
struct Dim3 {
    uint32_t x, y, z;
};
std::map<const void*, std::string> names;
std::map<char*, size_t> blocks;
struct Config {
    Dim3 grid, block;
    size_t lds;
    void* stream;
} pending;
int capturing = 0;
long fail_in = -1;
int32_t check[4] = {0, 0, 0, 0};  // error word and maxima that a 16-byte read-back returns
char symbol[64];

bool inside(const void* p)
{
    auto it = blocks.upper_bound((char*)p);
    if (it == blocks.begin()) return false;
    --it;
    return (char*)p < it->first + it->second;
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*)
{
    static void* m;
    return &m;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* s)
{
    pending = {g, b, lds, s};
    return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** s)
{
    *g = pending.grid;
    *b = pending.block;
    *lds = pending.lds;
    *s = pending.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void**, size_t lds, void*)
{
    printf("launch %s %u %u %u %u %zu\n", names[f].c_str(), g.x, g.y, g.z, b.x, lds);
    return 0;
}
int hipMalloc(void** p, size_t bytes)
{
    if (fail_in >= 0 && fail_in-- == 0) {
        *p = nullptr;
        printf("malloc %zu failed\n", bytes);
        return 2;  // hipErrorOutOfMemory
    }
    *p = calloc(bytes, 1);
    blocks[(char*)*p] = bytes;
    printf("malloc %zu\n", bytes);
    return 0;
}
int hipFree(void* p)
{
    blocks.erase((char*)p);
    free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t bytes, unsigned)
{
    *p = calloc(bytes, 1);
    return 0;
}
int hipHostFree(void* p)
{
    free(p);
    return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int, void*)
{
    printf("copy %s %zu\n", inside(src) ? (inside(dst) ? "d2d" : "d2h") : "h2d", bytes);
    memcpy(dst, src, bytes);
    if (bytes == sizeof(check) && inside(src) && !inside(dst)) memcpy(dst, check, bytes);
    return 0;
}
int hipMemcpy(void* dst, const void* src, size_t bytes, int)
{
    printf("copy wait %zu\n", bytes);
    memcpy(dst, src, bytes);
    return 0;
}
int hipMemsetAsync(void* p, int v, size_t bytes, void*)
{
    printf("memset %zu\n", bytes);
    memset(p, v, bytes);
    return 0;
}
int hipStreamSynchronize(void*)
{
    printf("wait\n");
    return capturing ? 900 : 0;  // hipErrorStreamCaptureUnsupported
}
int hipStreamIsCapturing(void*, int* s)
{
    *s = capturing;
    return 0;
}
int hipEventCreate(void** e)
{
    *e = malloc(1);
    return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e)
{
    free(e);
    return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventQuery(void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*)
{
    *ms = 0;
    return 0;
}
int hipGetDevice(int* d)
{
    *d = 0;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int)
{
    *v = 256;
    return 0;
}
int hipGetSymbolAddress(void** p, const void*)
{
    *p = symbol;
    return 0;
}
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "error"; }
}

int main(int argc, char** argv)
{
    if (argc < 3) return 2;
    void* lib = dlopen(argv[1], RTLD_NOW);
    if (!lib) {
        fprintf(stderr, "%s\n", dlerror());
        return 2;
    }
#define FN(name) auto* const f_##name = (decltype(&name))dlsym(lib, #name)
    FN(irbe_create);
    FN(irbe_set_system);
    FN(irbe_update_parameters);
    FN(irbe_build_lists);
    FN(irbe_compute_forces);
    FN(irbe_compute_forces_backward);
    FN(irbe_get_debug);
    FN(irbe_sync);
    irbe_handle h = nullptr;
    int64_t n = 0;
    int types = 1;
    // the caller's device arrays, of the larger element size
    std::vector<int32_t> type, mol;
    std::vector<double> q, pos, out, sigma, eps;
    for (int a = 2; a < argc; ++a) {
        const std::string cmd = argv[a];
        const std::string name = cmd.substr(0, cmd.find_first_of(":="));
        int st = 0;
        if (name == "create") {
            std::map<std::string, double> v{{"n", 1000}, {"box", 3}, {"rcore", 0.5}, {"rshell", 1.2}, {"p", 10},
                                            {"types", 1}, {"hint", 0}, {"skin", 0}, {"fp64", 0}, {"stencil", 0},
                                            {"entries", 0}, {"mol", 0}};
            std::string rest = cmd.size() > 7 ? cmd.substr(7) : "";
            while (!rest.empty()) {
                const size_t c = rest.find(','), e = rest.find('=');
                v[rest.substr(0, e)] = atof(rest.substr(e + 1, c == std::string::npos ? c : c - e - 1).c_str());
                rest = c == std::string::npos ? "" : rest.substr(c + 1);
            }
            n = (int64_t)v["n"];
            types = (int)v["types"];
            type.assign(n, 0);
            mol.assign(n, -1);
            if (v["mol"] > 0)
                for (int64_t i = 0; i < n; ++i) mol[i] = (int32_t)(i / (int64_t)v["mol"]);
            q.assign(n, 0);
            pos.assign(3 * n, 0);
            out.assign(3 * n, 0);
            sigma.assign(types * types, 0.3);
            eps.assign(types * types, 0.5);
            irbe_config c{};
            c.abi_version = IRBE_ABI_VERSION;
            c.precision = v["fp64"] != 0 ? IRBE_FP64 : IRBE_MIXED_FP32;
            c.n_atoms = n;
            c.box_length = v["box"];
            c.ewald_beta = 3.0 / v["rcore"] * 0.5;
            c.coulomb_k = 1.0;
            c.r_core = v["rcore"];
            c.r_shell = v["rshell"];
            c.p_shell = (int32_t)v["p"];
            c.p_kspace = 8;
            c.n_types = types;
            c.shell_source = v["stencil"] != 0 ? IRBE_SHELL_STENCIL : IRBE_SHELL_LIST;
            c.capacity_hint = v["hint"];
            c.skin = v["skin"];
            c.shell_entries = (int32_t)v["entries"];
            st = f_irbe_create(&c, nullptr, &h);
            // the caller's arrays count as device memory
            for (auto* p : {&q, &pos, &out}) blocks[(char*)p->data()] = p->size() * sizeof(double);
            for (auto* p : {&type, &mol}) blocks[(char*)p->data()] = p->size() * sizeof(int32_t);
        } else if (name == "set") {
            st = f_irbe_set_system(h, type.data(), q.data(), mol.data(), sigma.data(), eps.data());
        } else if (name == "lj") {
            st = f_irbe_update_parameters(h, nullptr, sigma.data(), eps.data());
        } else if (name == "charge") {
            st = f_irbe_update_parameters(h, q.data(), nullptr, nullptr);
        } else if (name == "build") {
            st = f_irbe_build_lists(h, pos.data(), 0);
        } else if (name == "forces") {
            st = f_irbe_compute_forces(h, pos.data(), 0, out.data(), 0, nullptr);
        } else if (name == "backward") {
            st = f_irbe_compute_forces_backward(h, pos.data(), 0, out.data(), out.data(), nullptr, nullptr);
        } else if (name == "sync") {
            st = f_irbe_sync(h);
        } else if (name == "counts") {
            int64_t v[4] = {0, 0, 0, 0}, w = 0;
            st = f_irbe_get_debug(h, IRBE_DBG_COUNTS, v, 4, &w);
            printf("capacities %lld %lld\n", (long long)v[2], (long long)v[3]);
        } else if (name == "capture") {
            capturing = atoi(cmd.c_str() + 8);
        } else if (name == "fail") {
            fail_in = atol(cmd.c_str() + 5);
        } else if (name == "overflow") {
            if (sscanf(cmd.c_str(), "overflow=%d,%d,%d,%d", &check[1], &check[2], &check[3], &check[0]) != 4) return 2;
        } else {
            return 2;
        }
        printf("= %s %d\n", cmd.c_str(), st);
    }
    return 0;
}
