// Stands in for the few HIP runtime calls that libtcuscan.so makes when it enqueues work, and writes down every kernel
// launch instead of making it (tests/launch_recorder.py compiles this file with g++ and puts it in front of the runtime
// in a process of its own).  Which kernel a call takes, and what runs in front of it, is decided on the host: with this it can
// be tested without a GPU.
#include <cxxabi.h>

#include <cstdlib>
#include <map>
#include <string>

struct Dim3 { unsigned x, y, z; };
struct FlatArgs {                                            // as in tcuscan.hip
    const void *offsets, *first_rows;
    unsigned expect, check_rows, stream, stride;
};

static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
static std::string g_launches;

extern "C" {

void **__hipRegisterFatBinary(const void *)
{
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    int status = 0;
    char *plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    names()[host] = status == 0 && plain ? plain : name;
    std::free(plain);
}

int hipLaunchKernel(const void *kernel, Dim3 grid, Dim3 block, void **args, size_t, void *)
{
    const auto it = names().find(kernel);
    const std::string name = it == names().end() ? "?" : it->second;
    const unsigned stride = name.find("seg_flat") == std::string::npos ? 0u : ((const FlatArgs *)args[1])->stride;
    g_launches += std::to_string(grid.x) + " " + std::to_string(block.x) + " " + std::to_string(stride) + " " + name + "\n";
    return 0;
}
int hipStreamIsCapturing(void *, int *status) { *status = 0; return 0; }
int hipGetLastError(void) { return 0; }

const char *shim_launches(void) { return g_launches.c_str(); }
void shim_clear(void) { g_launches.clear(); }

}
