// Stands in for the HIP runtime calls that libplora makes, so that a test on the CPU sees every launch of a call: preloaded in
// front of the runtime, it takes the launches down (kernel, workgroups, dynamic LDS, and how much of that the kernel was allowed
// before) and runs nothing.  Device pointers are never followed on the host.
#include <cstddef>
#include <cstdint>
#include <map>
#include <string>
#include <vector>

struct Dim { uint32_t x, y, z; };
struct Launch { std::string kernel; Dim grid; size_t lds, allowed; };

static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static std::map<const void *, size_t> &allowed() { static std::map<const void *, size_t> m; return m; }
static std::vector<Launch> &launches() { static std::vector<Launch> v; return v; }
static Dim g_grid, g_block;
static size_t g_lds;
static void *g_stream;
static void *g_fatbin;
alignas(256) static char g_symbol[256];

extern "C" {
void **__hipRegisterFatBinary(const void *) { return &g_fatbin; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream)
{
    g_grid = grid; g_block = block; g_lds = lds; g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream)
{
    *grid = g_grid; *block = g_block; *lds = g_lds; *stream = g_stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim grid, Dim, void **, size_t lds, void *)
{
    launches().push_back(Launch{names()[f], grid, lds, allowed()[f]});
    return 0;
}
int hipFuncSetAttribute(const void *f, int, int value) { allowed()[f] = (size_t)value; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }        // the compute units of an MI355X
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = g_symbol; return 0; }

void recorder_clear() { launches().clear(); }
int recorder_count() { return (int)launches().size(); }
const char *recorder_kernel(int i) { return launches()[i].kernel.c_str(); }
uint64_t recorder_workgroups(int i) { const Dim &g = launches()[i].grid; return (uint64_t)g.x * g.y * g.z; }
uint64_t recorder_lds(int i) { return launches()[i].lds; }
uint64_t recorder_allowed(int i) { return launches()[i].allowed; }
}
