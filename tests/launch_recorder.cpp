// Stand-ins for the entry points of the HIP runtime and of rocBLAS that the library calls: launches and products are written down
// instead of run, so the library's host code (which path a call takes, on which stream, with which operands) can be tested without a GPU.
// Loaded before the library, with its symbols global.
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <unistd.h>

#include <map>
#include <mutex>
#include <string>
#include <vector>

struct dim3 { uint32_t x, y, z; };

static std::mutex g_mutex;
static std::map<const void *, std::string> g_names;   // host stub -> kernel
static std::vector<std::string> g_log;                // one line per launch or product, tabs between its fields
static thread_local struct { dim3 grid, block; size_t lds; void *stream; } g_config;
static int g_units = 256;

static void put(const std::string &line)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_log.push_back(line);
}

extern "C" {

void recorder_reset() { std::lock_guard<std::mutex> lock(g_mutex); g_log.clear(); }
int recorder_count() { return (int)g_log.size(); }
const char *recorder_line(int i) { return g_log[i].c_str(); }
int recorder_built_count() { return (int)g_names.size(); }   // kernels of the library
const char *recorder_built(int i) { auto it = g_names.begin(); std::advance(it, i); return it->second.c_str(); }
void recorder_compute_units(int n) { g_units = n; }

void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *stub, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *)
{
    g_names[stub] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream)
{
    g_config = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream)
{
    *grid = g_config.grid, *block = g_config.block, *lds = g_config.lds, *stream = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void *stub, dim3 grid, dim3 block, void **, size_t lds, void *stream)
{
    char at[160];
    snprintf(at, sizeof at, "\t%u %u %u\t%u\t%zu\t%llu", grid.x, grid.y, grid.z, block.x * block.y * block.z, lds, (unsigned long long)(uintptr_t)stream);
    put("kernel\t" + g_names[stub] + at);
    return 0;
}
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int *value, int, int) { *value = g_units; return 0; }   // (the library asks for the number of compute units only)
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "recorded"; }
int hipGetSymbolAddress(void **address, const void *) { *address = (void *)((uintptr_t)1 << 44); return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *blocks, const void *, int, size_t) { *blocks = 1; return 0; }

// rocBLAS: a product goes to the stream that its handle has when the product is enqueued, some time after the call began
struct Handle { void *volatile stream; };
int rocblas_create_handle(Handle **h) { *h = new Handle{nullptr}; return 0; }
int rocblas_set_stream(Handle *h, void *stream) { h->stream = stream; return 0; }
static int product(Handle *h, int ta, int tb, int m, int n, int k, const void *a, int lda, int64_t sa, const void *b, int ldb, int64_t sb,
                   const void *c, int ldc, int64_t sc, int batch, int type)
{
    usleep(20);
    char line[512];
    snprintf(line, sizeof line, "product\t%d %d\t%d %d %d\t%llu %d %lld\t%llu %d %lld\t%llu %d %lld\t%d\t%d\t%llu", ta, tb, m, n, k,
             (unsigned long long)(uintptr_t)a, lda, (long long)sa, (unsigned long long)(uintptr_t)b, ldb, (long long)sb,
             (unsigned long long)(uintptr_t)c, ldc, (long long)sc, batch, type, (unsigned long long)(uintptr_t)h->stream);
    put(line);
    return 0;
}
int rocblas_gemm_strided_batched_ex(Handle *h, int ta, int tb, int m, int n, int k, const void *, const void *a, int a_type, int lda, int64_t sa,
                                    const void *b, int, int ldb, int64_t sb, const void *, const void *c, int, int ldc, int64_t sc, void *, int,
                                    int, int64_t, int batch, int, int, int32_t, uint32_t)
{
    return product(h, ta, tb, m, n, k, a, lda, sa, b, ldb, sb, c, ldc, sc, batch, a_type);
}
int rocblas_gemm_ex(Handle *h, int ta, int tb, int m, int n, int k, const void *, const void *a, int a_type, int lda, const void *b, int, int ldb,
                    const void *, const void *c, int, int ldc, void *, int, int, int, int, int32_t, uint32_t)
{
    return product(h, ta, tb, m, n, k, a, lda, 0, b, ldb, 0, c, ldc, 0, 1, a_type);
}

}  // extern "C"
