// Internal to the library: the context every entry point takes, shared by
// its translation units (orloj.hip: kernels and scoring entry points;
// sched.hip: the host scheduling runtime).  Not part of the C ABI.
#ifndef ORLOJ_CTX_INTERNAL_H
#define ORLOJ_CTX_INTERNAL_H

#include <hip/hip_runtime_api.h>
#include <stdarg.h>
#include <stdio.h>

#include "../../include/orloj.h"

// A scratch block of a context, grown on demand.
struct orloj_block {
    void* p;
    size_t bytes;
};

struct orloj_ctx {
    int device;
    int n_cu;        // compute units of the device
    hipStream_t stream;
    int* d_err;      // device status word (data error bits)
    float* d_fill;   // stand-in table entries: 16 zeros, 16 ones
    // Scratch.  A block's growth frees the old one, which a captured graph may
    // still name, so each use has a block that only its own larger calls grow.
    orloj_block work;  // the affine scorer's sums (emax_kernel, turned_esum_kernel)
    orloj_block drop;  // iterate_kernel's split drop phase
    // laws_mix_kernel's powers, for as many bins as it takes, so that it is
    // allocated once and never grown.  Never used under capture: a
    // graph may be replayed beside this context's own laws.
    orloj_block mix;
    float* noalloc_scratch;   // this device's fixed scratch array (NULL: unavailable)
    hipError_t noalloc_err;   // why it is unavailable
    char msg[512];
};

// Record a failure message on the context and return `code`.
static inline int orloj_ctx_fail(orloj_ctx* ctx, int code, const char* fmt, ...)
    __attribute__((format(printf, 3, 4)));
static inline int orloj_ctx_fail(orloj_ctx* ctx, int code, const char* fmt, ...) {
    if (ctx) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(ctx->msg, sizeof ctx->msg, fmt, ap);
        va_end(ap);
    }
    return code;
}

// One scheduling round's scoring and selection (sched.hip): the outputs of
// orloj_score_candidates (triangle prefixes) followed by orloj_select_batch,
// bit for bit.
// d_done (mapped host memory, or NULL): each select workgroup g writes
// `round` to d_done[g] once its writes are visible to the host;
// *n_groups receives the number of select workgroups.
__attribute__((visibility("hidden"))) int orloj_internal_score_select(
    orloj_ctx* ctx, const orloj_grid* grid, const float* d_ccdf, const int32_t* d_support,
    const orloj_queues* queues, double b_expo_per_ms, const int64_t* d_cand_off,
    const int64_t* d_prob_off, float* d_finish_prob, double* d_expected_finish,
    float* d_expected_latency_ms, float* d_score, int32_t* d_sel_n, int32_t* d_sel_bs,
    float* d_sel_score, int32_t* d_done, int32_t round, int* n_groups);

#endif
