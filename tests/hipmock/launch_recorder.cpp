// A HIP runtime that launches nothing and writes down what it was asked to launch: which kernel, how many
// workgroups of how many lanes, and the arguments that say which elements they take and where the arrays lie.  Each
// kernel's arguments are read as its own parameter list has them, so what is checked is what the kernel would get.  The
// library's launchers are compiled for the host only and linked against it, so every rule by which they choose a shape runs
// here, at any range, without a GPU and without memory behind the pointers.  Test infrastructure only.
//
// As the HIP runtime does, hipLaunchKernel refuses an empty launch and one of 2^32 work items or more.
#include <hip/hip_runtime.h>

#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "gs_internal.h"

struct Launch {
    char kernel[512];        // with its template arguments and its parameter list
    uint64_t grid, block;
    uint64_t stream;
    uint64_t lds;            // bytes of LDS asked for beyond what the kernel itself declares
    int64_t begin, end;      // the elements it is given
    int64_t extra;           // cuts, span, or the folds' number of partials
    int64_t keep_from;       // elements from here on are kept in the cache; of the gradient norms' launches -1:
    int64_t keep_block;      // workgroups from here on (of all others -1)
    uint64_t partials, out;  // where partials are written (or, folding, read) and where the result goes
    uint64_t states[6];      // p, m, v in and out
    uint64_t w, acc, sqnorm; // the step's weights, the fp32 sum, the norm a step clips by (null: it does not)
    uint64_t streams[GS_MAX_K];
    gs::StepConsts c;
    float max_norm;
    int32_t k;               // how many of those are read
    int32_t accumulate;      // onto what `out` holds
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
static bool g_capturing;
static hipError_t g_last = hipSuccess;

static std::string kernel_name(const char *mangled)
{
    int st = 0;
    char *d = abi::__cxa_demangle(mangled, nullptr, nullptr, &st);
    std::string s = st == 0 && d ? d : mangled;
    free(d);
    const size_t at = s.find("gs::k_");
    return at == std::string::npos ? s : s.substr(at + 4);
}

// The arguments of one launch, read in order; each by the type that the kernel's parameter has.
struct Args {
    void **at;
    template <typename T>
    const T &next()
    {
        return *static_cast<const T *>(*at++);
    }
    uint64_t address() { return next<uint64_t>(); }
};

static uint64_t addr(const void *p) { return reinterpret_cast<uint64_t>(p); }

static void streams_of(Launch &l, const uint16_t *const *g, int k)
{
    l.k = k;
    for (int j = 0; j < k; ++j) l.streams[j] = addr(g[j]);
}

static void step_args(Launch &l, const gs::StepArgs &a)
{
    const void *const states[6] = {a.p, a.m, a.v, a.po, a.mo, a.vo};
    l.begin = a.begin;
    l.end = l.keep_from = a.end;
    for (int i = 0; i < 6; ++i) l.states[i] = addr(states[i]);
    l.w = addr(a.w);
    l.acc = addr(a.acc);
    l.sqnorm = a.max_norm > 0.0f ? addr(a.d_sqnorm) : 0;
    l.c = a.c;
    l.max_norm = a.max_norm;
    if (!a.acc) streams_of(l, a.gt.g, a.k);
}

// a step whose arrays are given by their distances from p
template <int K>
static void near_args(Launch &l, Args a)
{
    l.begin = a.next<int64_t>();
    l.extra = a.next<int>();
    const uint32_t packed = a.next<uint32_t>();
    l.end = l.keep_from = l.begin + packed % GS_NEAR_CLIP_BIT;
    const uint64_t p = a.address(), sqnorm = a.address();
    const auto at = [&](int distance) { return p + ((int64_t)distance << (packed & GS_NEAR_UNIT_BIT ? 8 : 4)); };
    l.states[0] = l.states[3] = p;
    l.states[1] = l.states[4] = at(a.next<int>());
    l.states[2] = l.states[5] = at(a.next<int>());
    l.k = K;
    int g[8];
    for (int j = 0; j < 4; ++j) g[j] = a.next<int>();
    const gs::NearRest<K> &rest = a.next<gs::NearRest<K>>();
    for (int j = 4; j < 8; ++j) g[j] = rest.g[j - 4];
    for (int j = 0; j < K; ++j) l.streams[j] = at(g[j]);
    l.w = at(rest.w);
    l.sqnorm = packed & GS_NEAR_CLIP_BIT ? sqnorm : 0;
    l.c = rest.c;
    l.max_norm = rest.max_norm;
}

template <int STREAMS>
static void table(Launch &l, Args &a)
{
    const gs::GradTableOf<STREAMS> &gt = a.next<gs::GradTableOf<STREAMS>>();
    streams_of(l, gt.g, a.next<int>());
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
    l.keep_from = l.keep_block = -1;
    auto is = [&](const char *p) { return name.compare(0, strlen(p), p) == 0; };
    auto has = [&](const char *p) { return name.find(p) != std::string::npos; };
    auto takes = [&](const char *parameters) {
        if (has(parameters)) return;
        fprintf(stderr, "the recorder does not know how to read %s\n", name.c_str());
        abort();
    };
    Args a{args};
    if (is("k_accum_adamw_spec")) {
        takes("(gs::StepArgs, double*, int)");
        step_args(l, a.next<gs::StepArgs>());
        l.partials = a.address();
        l.extra = a.next<int>();
    } else if (is("k_accum_adamw") && has("(gs::StepArgs, int)")) {
        step_args(l, a.next<gs::StepArgs>());
        l.extra = a.next<int>();
    } else if (is("k_accum_adamw")) {
        takes("(long, int, unsigned int, float*, double const*, int, int, int, int, int, int, gs::NearRest<");
        if (has("NearRest<1>")) near_args<1>(l, a);
        else if (has("NearRest<2>")) near_args<2>(l, a);
        else if (has("NearRest<3>")) near_args<3>(l, a);
        else if (has("NearRest<4>")) near_args<4>(l, a);
        else if (has("NearRest<5>")) near_args<5>(l, a);
        else if (has("NearRest<6>")) near_args<6>(l, a);
        else if (has("NearRest<7>")) near_args<7>(l, a);
        else takes("NearRest<8>"), near_args<8>(l, a);
    } else if (is("k_grad_sqnorm") || is("k_grad_accum_sqnorm")) {
        const bool staged = is("k_grad_accum_sqnorm"), by_table = has("GradTableOf");
        takes(staged ? "(long, int, int, long, float*, gs::GradTableOf<" : by_table ? "(long, int, int, long, gs::GradTableOf<"
                     : "(long, int, int, long, unsigned short const*, unsigned short const*, unsigned short const*, unsigned short const*, "
                       "double*, double*, int)");
        if (by_table) takes(staged ? ">, int, double*)" : ">, int, int, double*, double*)");
        l.begin = a.next<int64_t>();
        l.extra = a.next<int>();
        l.keep_block = a.next<int>();
        l.end = a.next<int64_t>();
        if (staged) l.acc = a.address();
        if (has("GradTableOf<8>")) table<8>(l, a);
        else if (has("GradTableOf<16>")) table<16>(l, a);
        else if (has("GradTableOf<32>")) table<32>(l, a);
        else {
            l.k = atoi(name.c_str() + strlen("k_grad_sqnorm<"));       // up to four, by the kernel's number of streams
            for (int j = 0; j < 4; ++j) {
                const uint64_t g = a.address();
                if (j < l.k) l.streams[j] = g;
            }
        }
        if (!staged && by_table) l.accumulate = a.next<int>();
        l.partials = a.address();
        if (!staged) l.out = a.address();
        if (!by_table) l.accumulate = a.next<int>();
    } else if (is("k_accum_add")) {
        takes("(gs::AccumAddArgs, int)");
        const gs::AccumAddArgs &A = a.next<gs::AccumAddArgs>();
        l.begin = A.begin;
        l.end = A.end;
        l.keep_from = A.keep_from;
        l.partials = addr(A.partials);
        l.acc = addr(A.acc);
        streams_of(l, &A.g, 1);
        l.extra = a.next<int>();
    } else if (is("k_acc_sqnorm")) {
        takes("(float const*, long, long, long, double*, int, int)");
        l.acc = a.address();
        l.begin = a.next<int64_t>();
        l.end = a.next<int64_t>();
        l.keep_from = a.next<int64_t>();
        l.partials = l.out = a.address();
        l.accumulate = a.next<int>();
        l.extra = a.next<int>();
    } else {                                     // the two folds
        takes(is("k_sqnorm_finalize") ? "(double const*, int, double*, int)" : "k_sqnorm_fold_slices(double const*, int, double*)");
        l.partials = a.address();
        l.extra = a.next<int>();
        l.out = a.address();
        if (is("k_sqnorm_finalize")) l.accumulate = a.next<int>();
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
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *status)
{
    *status = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
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
// CUs that every stream but the null stream is said to be confined to (256: none), and whether it is being captured
void rec_reset(int stream_cus, int capturing)
{
    g_capturing = capturing;
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
