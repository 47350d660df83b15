// gs_internal.h -- types shared by the library's own translation units (not installed).
#ifndef GS_INTERNAL_H
#define GS_INTERNAL_H

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "gs.h"

// limits of the step's shapes (step_shape and launch_accum_adamw_spec say why they lie there)
#define GS_LATENCY_MAX (1 << 19)      // elements up to which every load is in flight at once
#define GS_LATENCY_THROUGH_STEP 12000 // what each stream takes off that line for steps of 5 to 15 streams that write through
#define GS_RESIDENT_MAX (1 << 21)     // elements up to which 4 per lane keep all waves resident together
#define GS_LATE_MIN 960000            // elements above which a step of one generation of waves reads its arguments late;
#define GS_LATE_MIN_STEP 140000       // the line lies that much higher for each stream below 7
#define GS_LATE_MAX_MANY 1400000      // and up to which it does with 8 streams and more
#define GS_FULL_MAX 7000000           // elements up to which a CU holds as many workgroups as it can
#define GS_FULL_ODD_MAX (1 << 24)     // the same line for 9 to 23 streams that are no multiple of 8
#define GS_DEEP_MAX (1 << 25)         // elements up to which multiples of 8 streams have 8 loads in flight
#define GS_DEEP_ODD_MAX (1 << 26)     // the same line for 9 to 19 streams that are no multiple of 8
#define GS_NEAR_MAX 1200000           // elements up to which a step's arrays are given by distances; with all loads in flight only up to
#define GS_NEAR_LATENCY_MAX 430000    // this many with one and eight streams, with two to seven
#define GS_NEAR_THROUGH_MAX 330000    // up to this line less
#define GS_NEAR_THROUGH_STEP 9000     // this for each of them
#define GS_NEAR_FULL_MAX 5000000      // and above 2^21 up to this many again
#define GS_NEAR_CLIP_BIT (1u << 23)   // such a step: whether the norm clips and the distances' unit, above its number of elements
#define GS_NEAR_UNIT_BIT (1u << 24)
#define GS_SERIAL_MAX_K 7             // "few streams"
#define GS_LINK_WAVES 22              // of a step on host memory in flight on a die with up to 8 of its CUs
#define GS_LINK_WAVES_WIDE 64         // and with more of them
#define GS_LDS_GRANULES 128           // a CU's 160 KB of LDS are handed out in this many pieces
#define GS_LDS_GRANULE_BYTES 1280
#define GS_SPEC_FEW_MAX 7000000       // speculative pass: elements up to which everything is in flight
#define GS_SPEC_RUN_LONG (1 << 28)    // small workspace: elements from which a CU holds one workgroup fewer for the runs of tiles
#define GS_SPEC_RUN_MAX (1 << 29)     // and up to which they are of small tiles (up to 2 streams: the line before)
#define GS_KEEP_BYTES ((int64_t)256 << 20)  // of a re-read stream: left in the memory-side cache (keep_from)
#define GS_KEEP_FEW_MIN 1300000       // elements from which the norm of two and three streams leaves its lines there,
#define GS_KEEP_MANY_MIN (3 << 18)    // and of four and more (the other passes: above GS_RESIDENT_MAX)
#define GS_FINAL_BLOCK 1024           // threads of the partial-folding kernels
#define GS_FINAL_SLICES 128           // workgroups of the first folding stage for large partial counts
#define GS_FINAL_DIRECT_MAX 8192      // up to this many partials are folded by one workgroup directly
#define GS_PARTIAL_ELEMS 256          // elements per norm partial in the shapes that leave most of them
#define GS_SQNORM_MAX_BLOCKS 262144   // upper bound on block partials => workspace size (2 MB)
// limits of the staged norm's and the adding kernel's shapes (launch_staged_norm, launch_accum_add)
#define GS_STAGED_WIDE_MAX (1 << 22)  // elements up to which a workgroup takes 4096 of them
#define GS_STAGED_WIDE_MANY_MAX (1 << 20)  // the same for more than 16 streams
#define GS_STAGED_WIDE_AGAIN_MIN 4500000   // and, up to 16 streams on all CUs, from this length
#define GS_STAGED_WIDE_AGAIN_MAX 10000000  // to this one
#define GS_STAGED_PAIR_MIN (1 << 25)  // elements from which, with 8 streams or more, a lane takes 2 of them
#define GS_STAGED_KEEP_MAX_K 16       // streams up to which the end of the sum is left in the memory-side cache
#define GS_ADD_SMALL_MAX (1 << 22)    // without the norm: elements up to which both loads are in flight together
#define GS_ADD_FIRST_256_MAX 900000   // first micro-batch: elements up to which workgroups have 256 lanes
#define GS_ADD_FIRST_128_MAX (1 << 25) // and, above 2^21, 128
#define GS_ADD_WIDE_MAX (1 << 23)     // with the norm: elements up to which a workgroup takes 4096 of them unless the sum stays in the cache,
#define GS_ADD_KEEP_MIN (1 << 22)     // which after a later micro-batch it does from here on (after the first from the line before)
// limits of the norm's shapes (launch_grad_norm)
#define GS_NORM_SMALL_MAX (1 << 22)   // up to 4 streams: elements up to which workgroups are kept small
#define GS_NORM_256_MAX (3 << 18)     // from 5 streams on: elements up to which workgroups have 256 lanes
#define GS_NORM_512_MAX 5500000       // and up to which one of 512 lanes reads one tile; above that two, with 5 to 7 streams
#define GS_NORM_1024_MAX (1 << 25)    // up to this line with 1024 lanes
#define GS_NORM_RUN8_MIN (1 << 23)    // one stream: elements from which a workgroup reads eight tiles instead of four,
#define GS_NORM_RUN8_MAX (3 << 24)    // and up to which it does on all CUs
#define GS_NORM_LONG_MIN (1 << 29)    // elements from which a workgroup reads four tiles instead of two (one stream: eight instead of four)
#define GS_ACC_NORM_LONG_MIN (1 << 27)  // the same line of the fp32 norm (eight tiles)
#define GS_ONE_MAX_LOADS 65536        // from 5 streams on: elements times streams up to which that workgroup takes more than one tile
#define GS_ONE_MAX_LOADS_CAPTURED 40960  // and in a captured norm
#define GS_ONE_BLOCK 1024             // threads of the norm in a single workgroup
#define GS_BUDGET_RUN_MIN 49152       // elements per CU of a confined stream from which the norms take shapes of their own

namespace gs {

// Per-step constants, formed on the host in double and rounded to float once.
struct StepConsts {
    float beta1, beta2, omb1, omb2, eps, step_size, rsbc2, decay;
};

template <int STREAMS> struct GradTableOf {
    const uint16_t *g[STREAMS];
};
typedef GradTableOf<GS_MAX_K> GradTable;

struct StepArgs {
    int64_t begin, end;
    const float *p, *m, *v;   // states in
    float *po, *mo, *vo;      // states out (the same arrays for the in-place entry points)
    uint16_t *w;
    GradTable gt;
    int k;
    StepConsts c;
    float max_norm;
    const double *d_sqnorm;
    const float *acc;   // non-null: staged fp32 gradient sum replaces the k bf16 streams
    bool over_link;     // the states are host memory, reached over PCIe
};

// what a step whose arrays are given by their distances from p takes as a block (K: a kernel for each number of streams)
template <int K> struct NearRest {
    int g[4];           // streams 4 to 7
    int w;
    float max_norm;
    StepConsts c;
};

struct SqnormArgs {
    int64_t begin, end;
    GradTable gt;
    int k;
    double *partials;
    float *acc;         // non-null: also write the fp32 gradient sum here
    int64_t keep_from;  // elements from here on are left in the memory-side cache
    double *out;        // norm in a single workgroup: the result, added to if accumulate is set
    int accumulate;
};

struct AccumAddArgs {
    float *acc;
    const uint16_t *g;
    int64_t begin, end;
    double *partials;   // used only when a norm is asked for
    int64_t keep_from;  // elements of acc from here on are left in the memory-side cache
};

hipError_t launch_accum_adamw(const StepArgs &A, hipStream_t stream);
hipError_t launch_accum_adamw_spec(const StepArgs &A, double *partials, size_t workspace_bytes, double *d_out,
                                   int accumulate, hipStream_t stream);
hipError_t launch_grad_sqnorm(const SqnormArgs &A, size_t workspace_bytes, double *d_out, int accumulate,
                              hipStream_t stream);

// d_out == nullptr: no norm (then the workspace is not touched)
hipError_t launch_accum_add(const AccumAddArgs &A, int first, size_t workspace_bytes, double *d_out, int accumulate,
                            hipStream_t stream);

// squared norm of a finished fp32 buffer over [begin,end)
hipError_t launch_acc_sqnorm(const float *acc, int64_t begin, int64_t end, double *partials, size_t workspace_bytes,
                             double *d_out, int accumulate, hipStream_t stream);

// host side (gs_api.hip)
gs_status validate_hparams(const gs_adamw_hparams *hp);
gs_status validate_grads(const uint16_t *const *grads, int k);
StepConsts make_consts(const gs_adamw_hparams &hp);
gs_status hip_fail(hipError_t e, const char *what);

}  // namespace gs
#endif
