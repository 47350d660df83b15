// A HIP runtime that launches nothing and writes down what it was asked to launch: which kernel, how many
// workgroups of how many lanes, and the arguments that say which elements they take.  The library's launchers
// are compiled for the host only and linked against it, so every rule by which they choose a shape runs here,
// at any range, without a GPU and without memory behind the pointers.  Test infrastructure only.
//
// As the HIP runtime does, hipLaunchKernel refuses an empty launch and one of 2^32 work items or more.
#include <hip/hip_runtime.h>

#include <cxxabi.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "gs_internal.h"

struct Launch {
    char kernel[128];
    uint64_t grid, block;
    uint64_t stream;
    uint64_t lds;            // bytes of LDS asked for beyond what the kernel itself declares
    int64_t begin, end;      // the elements it is given
    int64_t extra;           // the last integer argument: cuts, span, or the folds' number of partials
    int64_t keep_from;
    uint64_t partials, out;  // where partials are written (or, folding, read) and where the result goes
    int32_t status;
};

// built on first use: the kernels register themselves before this file's own objects are constructed
static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> n;
    return n;
}
static std::vector<Launch> g_launches;
static std::vector<uint64_t> g_mask_queries;
static int g_stream_cus = 256;
static hipError_t g_last = hipSuccess;

static std::string kernel_name(const char *mangled)
{
    int st = 0;
    char *d = abi::__cxa_demangle(mangled, nullptr, nullptr, &st);
    std::string s = st == 0 && d ? d : mangled;
    free(d);
    const size_t at = s.find("gs::k_");
    const size_t args = s.find('(', at);
    return at == std::string::npos ? s : s.substr(at + 4, args - at - 4);
}

extern "C" {

extern const char __hip_fatbin[16] = {0};
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names()[host] = kernel_name(name);
}

static dim3 g_grid, g_block;
static size_t g_shared;
static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    g_grid = grid;
    g_block = block;
    g_shared = shared;
    g_stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    *grid = g_grid;
    *block = g_block;
    *shared = g_shared;
    *stream = g_stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t shared, hipStream_t stream)
{
    Launch l;
    memset(&l, 0, sizeof l);
    const std::string &name = names()[fn];
    strncpy(l.kernel, name.c_str(), sizeof l.kernel - 1);
    l.grid = grid.x;
    l.block = block.x;
    l.stream = reinterpret_cast<uint64_t>(stream);
    l.lds = shared;
    const uint64_t items = (uint64_t)grid.x * block.x;
    l.status = items == 0 || items >= (1ull << 32) || block.x > 1024 ? hipErrorInvalidConfiguration : hipSuccess;
    auto arg = [&](int i) { return args[i]; };
    auto is = [&](const char *p) { return name.compare(0, strlen(p), p) == 0; };
    auto addr = [](const void *p) { return reinterpret_cast<uint64_t>(p); };
    if (is("k_accum_adamw")) {
        const gs::StepArgs &a = *static_cast<gs::StepArgs *>(arg(0));
        l.begin = a.begin;
        l.end = a.end;
        l.keep_from = a.end;
        if (is("k_accum_adamw_spec")) {
            l.partials = addr(*static_cast<double **>(arg(1)));
            l.extra = *static_cast<int *>(arg(2));
        } else {
            l.extra = *static_cast<int *>(arg(1));
        }
    } else if (is("k_grad_sqnorm") || is("k_grad_accum_sqnorm")) {
        const gs::SqnormArgs &a = *static_cast<gs::SqnormArgs *>(arg(0));
        l.begin = a.begin;
        l.end = a.end;
        l.keep_from = a.keep_from;
        l.partials = addr(a.partials);
        l.out = addr(a.out);
        l.extra = *static_cast<int *>(arg(1));
    } else if (is("k_accum_add")) {
        const gs::AccumAddArgs &a = *static_cast<gs::AccumAddArgs *>(arg(0));
        l.begin = a.begin;
        l.end = a.end;
        l.keep_from = a.keep_from;
        l.partials = addr(a.partials);
        l.extra = *static_cast<int *>(arg(1));
    } else if (is("k_acc_sqnorm")) {
        l.begin = *static_cast<int64_t *>(arg(1));
        l.end = *static_cast<int64_t *>(arg(2));
        l.keep_from = *static_cast<int64_t *>(arg(3));
        l.partials = l.out = addr(*static_cast<double **>(arg(4)));
        l.extra = *static_cast<int *>(arg(6));
    } else {                                     // the two folds
        l.partials = addr(*static_cast<double **>(arg(0)));
        l.extra = *static_cast<int *>(arg(1));
        l.out = addr(*static_cast<double **>(arg(2)));
    }
    g_launches.push_back(l);
    if (l.status != hipSuccess) g_last = hipErrorInvalidConfiguration;
    return (hipError_t)l.status;
}

hipError_t hipGetLastError()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "refused by the recorder"; }
hipError_t hipGetDevice(int *dev)
{
    *dev = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t, int)
{
    *value = 256;
    return hipSuccess;
}
hipError_t hipExtStreamGetCUMask(hipStream_t stream, uint32_t words, uint32_t *mask)
{
    g_mask_queries.push_back(reinterpret_cast<uint64_t>(stream));
    for (uint32_t w = 0; w < words; ++w) {
        const int left = g_stream_cus - (int)w * 32;
        mask[w] = left >= 32 ? 0xffffffffu : left > 0 ? (1u << left) - 1 : 0u;
    }
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **ptr, const void *)
{
    *ptr = reinterpret_cast<void *>((uintptr_t)1 << 60);
    return hipSuccess;
}
hipError_t hipExtStreamCreateWithCUMask(hipStream_t *, uint32_t, const uint32_t *) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipErrorNotSupported; }
hipError_t hipHostMalloc(void **, size_t, unsigned) { return hipErrorNotSupported; }
hipError_t hipHostFree(void *) { return hipErrorNotSupported; }

// ---- what the tests call -----------------------------------------------------------------
// CUs that every stream but the null stream is said to be confined to (256: none)
void rec_reset(int stream_cus)
{
    g_launches.clear();
    g_mask_queries.clear();
    g_stream_cus = stream_cus;
    g_last = hipSuccess;
}
int rec_count() { return (int)g_launches.size(); }
void rec_get(int i, Launch *out) { *out = g_launches[i]; }
int rec_mask_queries() { return (int)g_mask_queries.size(); }
uint64_t rec_mask_query(int i) { return g_mask_queries[i]; }
int rec_kernels(char *out, int cap)              // the names of all kernels in the library, one a line
{
    std::string s;
    for (const auto &n : names()) s += n.second + "\n";
    strncpy(out, s.c_str(), cap);
    return (int)s.size();
}
// the step of the in-place host context: states in host memory
int rec_step_on_host_memory(int k, int64_t begin, int64_t end, void *stream)
{
    gs::StepArgs A;
    memset(&A, 0, sizeof A);
    A.k = k;
    A.begin = begin;
    A.end = end;
    A.over_link = true;
    return gs::launch_accum_adamw(A, static_cast<hipStream_t>(stream));
}
}
