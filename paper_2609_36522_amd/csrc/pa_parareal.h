// Internal declarations of the cached Parareal sampler (kernels in k_parareal.hip).
#pragma once

#include "pa_device.h"

namespace pa {

// Device control block of one Parareal handle.
struct alignas(64) PrCtrl {
    int32_t done;       // converged (Eq. (2) on every boundary) or B iterations done
    int32_t iters;      // completed iterations
    int32_t nonfinite;  // sticky: a boundary residual was NaN/Inf
    int32_t pad;
};

enum PrMode : int32_t { PR_INIT = 0, PR_FINE = 1, PR_COARSE = 2, PR_COPY = 3 };
enum PrKernel : int32_t { PRK_RESET, PRK_TEST, PRK_FINE, PRK_COARSE, PRK_CHECK };

// Which request, if any, Parareal block n makes in this launch (uniform per block).
__device__ __forceinline__ bool pr_request(const PrArgs& a, int n, int* t) {
    if (a.mode == PR_FINE) {
        *t = n * a.L + a.j;
        return n >= a.k;
    }
    *t = n * a.L;
    return n == a.n;
}

// Outcome of block n's request at timestep t with Eq. (4) deviation dev (NaN without an entry),
// for the step kernel of the request, the counters and the trace. One thread per block.
__device__ __forceinline__ void pr_publish(const Dev& d, const PrArgs& a, int n, int t, bool hit, double dev) {
    Ctrl* c = d.ctrl + n;
    c->m = hit ? 0 : 1;
    c->miss_idx[0] = t;
    c->newest = t;
    c->done = 0;
    c->slot_miss[0] = hit ? 0 : 1;
    if (hit) c->hits += 1;
    else c->nfe += 1;
    if (d.trace_pr) {
        pa_request_trace_t* r = d.trace_pr + a.rec + (a.mode == PR_FINE ? n - a.k : 0);
        r->iteration = a.mode == PR_INIT ? -1 : a.k;
        r->phase = a.mode;
        r->t = t;
        r->block = n;
        r->hit = hit ? 1 : 0;
        r->dev = dev;
    }
}

hipError_t launch_pr(const Dev& d, const PrArgs& a, int kernel, hipStream_t st);
int pr_chunks(int D);

}  // namespace pa
