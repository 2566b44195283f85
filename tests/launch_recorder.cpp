// A stand-in for the HIP runtime under libee on a machine without a GPU: kernel launches are recorded, not run.  Loaded before the
// library with its symbols visible (tests/host_launches.py).  Allocations are host memory, so that the small tables the
// library keeps are written somewhere; everything else the library is given is an address it never touches on the host.
// Built with g++: the few prototypes that libee calls, as the HIP runtime's C interface has them.
#include <cxxabi.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

struct dim3 { uint32_t x, y, z; };
struct Config { dim3 grid, block; size_t shared; void* stream; };
struct Launch { std::string name; dim3 grid, block; std::vector<int64_t> args; };

static std::map<const void*, std::string> g_names;      // host stub -> demangled kernel
static std::vector<Config> g_configs;
static std::vector<Launch> g_launches;
static char g_symbol[64];

// types of the parameters, as the demangled name gives them
static std::vector<std::string> params(const std::string& name) {
    std::vector<std::string> out;
    size_t at = std::string::npos;
    int depth = 0;
    for (size_t i = 0; i < name.size(); ++i) {
        const char c = name[i];
        if (c == '<') ++depth;
        if (c == '>') --depth;
        if (depth) continue;
        if (c == '(') at = i + 1;
        else if ((c == ',' || c == ')') && at != std::string::npos) {
            while (name[at] == ' ') ++at;
            out.push_back(name.substr(at, i - at));
            at = i + 1;
        }
    }
    return out;
}

extern "C" {

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    int status = 0;
    char* d = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    g_names[fn] = status == 0 ? d : name;
    free(d);
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
    g_configs.push_back(Config{grid, block, shared, stream});
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
    const Config c = g_configs.back();
    g_configs.pop_back();
    *grid = c.grid; *block = c.block; *shared = c.shared; *stream = c.stream;
    return 0;
}
int hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t, void*) {
    Launch l{g_names[fn], grid, block, {}};
    size_t k = 0;
    for (const std::string& t : params(l.name)) {         // a number, a pointer, or the first eight bytes of a structure
        int64_t v = 0;
        if (t == "int") { int32_t i; memcpy(&i, args[k], 4); v = i; }
        else if (t == "float" || t == "unsigned int") { uint32_t u; memcpy(&u, args[k], 4); v = u; }
        else memcpy(&v, args[k], 8);
        l.args.push_back(v);
        ++k;
    }
    g_launches.push_back(l);
    return 0;
}
int hipMalloc(void** p, size_t n) { *p = calloc(1, n); return *p ? 0 : 2; }
int hipFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipMemset(void* d, int v, size_t n) { memset(d, v, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "recorded"; }
int hipGetSymbolAddress(void** p, const void*) { *p = g_symbol; return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipEventCreate(void**) { return 1; }
int hipEventRecord(void*, void*) { return 1; }
int hipEventSynchronize(void*) { return 1; }
int hipEventElapsedTime(float*, void*, void*) { return 1; }

// ------------------------------------------------------------------ what was launched
void rec_clear() { g_launches.clear(); }
int rec_count() { return (int)g_launches.size(); }
const char* rec_name(int i) { return g_launches[i].name.c_str(); }
void rec_dims(int i, uint32_t* out) {
    const Launch& l = g_launches[i];
    const uint32_t v[6] = {l.grid.x, l.grid.y, l.grid.z, l.block.x, l.block.y, l.block.z};
    memcpy(out, v, sizeof v);
}
int rec_args(int i, int64_t* out, int most) {
    const Launch& l = g_launches[i];
    const int n = (int)l.args.size() < most ? (int)l.args.size() : most;
    memcpy(out, l.args.data(), n * sizeof(int64_t));
    return n;
}
}
