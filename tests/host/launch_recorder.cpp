// Preloaded in front of the HIP runtime on a machine without a GPU: every kernel launch of the process goes to a callback (the
// kernel's symbol and its arguments) that says whether it succeeds, and nothing is launched.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

static int (*g_callback)(const char *kernel, void **args) = nullptr;
static thread_local hipError_t g_last = hipSuccess;

extern "C" {
void recorder_set_callback(int (*callback)(const char *, void **)) { g_callback = callback; }

// (the runtime's own pair wants a device)
static thread_local dim3 g_grid, g_block;
static thread_local size_t g_lds;
static thread_local hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream)
{
    g_grid = grid; g_block = block; g_lds = lds; g_stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream)
{
    *grid = g_grid; *block = g_block; *lds = g_lds; *stream = g_stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *function, dim3, dim3, void **args, size_t, hipStream_t)
{
    Dl_info info{};
    dladdr(function, &info);
    const hipError_t e = g_callback && g_callback(info.dli_sname ? info.dli_sname : "?", args) ? hipErrorLaunchFailure : hipSuccess;
    if (e != hipSuccess) g_last = e;
    return e;
}

hipError_t hipGetLastError(void)
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
}
