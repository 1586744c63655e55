// Internal declarations shared by the host library and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "paraanya.h"

namespace pa {

// Device-resident control block of one sample. Every per-sweep decision lives here, so
// the host can enqueue sweeps without reading anything back.
struct alignas(256) Ctrl {
    int32_t s;          // window start: states 0..s are final
    int32_t e;          // window end: drift points s..e-1, updated states s+1..e
    int32_t newest;     // highest computed state; a state above it reads as X[newest]
    int32_t m;          // misses of the current sweep
    int32_t done;       // s >= T
    int32_t nonfinite;  // sticky: a residual was NaN/Inf
    int32_t c;          // leading converged count of the last sweep
    int32_t sweep;      // completed sweeps since reset
    int64_t nfe;
    int64_t hits;
    int64_t revisits;       // window slots whose timestep holds a cache entry
    int64_t revisits_below; // ... with Eq. (4) deviation below Dev::revisit_thr
    int32_t miss_idx[PA_MAX_WINDOW];  // ascending miss timesteps
    uint8_t slot_miss[PA_MAX_WINDOW]; // per window slot j: 1 if t = s + j is a miss
    uint8_t slot_rank[PA_MAX_WINDOW]; // per miss slot j: its position in miss_idx
    int32_t ended;      // Dev::sweep_id of the launch that set done; 0 before
};

// The control-block fields the window slide reads, as they were before it (the fused sweep's
// Picard kernel leaves this snapshot for the slide that the next network kernel computes).
struct SlidePre {
    int32_t s, e, newest, sweep, nonfinite;
    int32_t pending;    // a slide of this state is outstanding (0 right after reset)
    int64_t nfe, hits, revisits, revisits_below;
};

// Where a network launch left the fresh outputs of the misses.
enum EpsMode : int32_t {
    EPS_SPLIT = 0,      // one partial output per half of 512 units, in Ep
    EPS_WHOLE = 1,      // whole outputs, in Eh
    EPS_FINE = 2        // one partial output per 64 units, in Ep by list entry
};
constexpr int kFineGroups = 8;  // 64-unit partial outputs per half

struct PrCtrl;

// The requests a Parareal launch serves (see pa_parareal.h).
struct PrArgs {
    int32_t mode;       // PrMode
    int32_t L;          // fine steps per block
    int32_t k;          // iteration (fine: blocks n >= k are active)
    int32_t j;          // fine step within the block
    int32_t n;          // block of a coarse request or copy
    int32_t rec;        // trace record index of the launch's first request
    int32_t nchunk;     // partial sums per boundary and per request
    PrCtrl* pc;
};

// Geometry and device buffers handed to every kernel launcher. Per-sample buffers are
// stacked along a leading sample index n < N.
struct Dev {
    int32_t N;                 // samples
    int32_t T, P, D;
    int32_t C, Himg, Wimg;
    int32_t ntok, hidden;      // patch-MLP only
    double delta, tol;
    double revisit_thr;        // threshold of the revisit counters
    float* X;                  // [N][T+1][D] trajectories
    float* Xh;                 // [N][T][D]   cached inputs
    float* Eh;                 // [N][T][D]   cached outputs
    uint8_t* valid;            // [N][T]
    const float* noise;        // [N][T][D]   pre-sampled step noise z (eta > 0), else null
    double* coef;              // [T][3]      (alpha_i, b_i, sigma_i) in fp64
    float* lin_c;              // [T]         linear network coefficients (or null)
    double* part_res;          // [N][P][picard_blocks] fp64 partial sums of Eq. (2) residuals
    double* part_dev;          // [N][P][picard_blocks] fp64 partial sums of Eq. (4) deviations
                               // (both twice with fused_linear, by sweep parity)
    Ctrl* ctrl;                // [N]
    SlidePre* pre;             // [N] pre-slide snapshots (fused sweep; [2][N] with fused_linear)
    int32_t fused_slide;       // 1: the network kernel computes the slide (N = 1), no k_slide
    int32_t fused_linear;      // 1: the Picard kernel of a linear network computes the last
                               // sweep's slide itself if it is outstanding, no k_slide
    int32_t sweep_id;          // of the sweep enqueued last: never 0, odd and even in turn
    uint64_t* progress;        // [N] host-mapped words: sweeps << 32 | done << 31 | nonfinite << 30 | s
    uint64_t* counters;        // [N][4] host-mapped final counters (epoch << 40 | value) or null
    uint32_t epoch;            // sample epoch of the counter words (24 bits, set at reset)
    pa_sweep_trace_t* trace;   // [N][T] or null
    // patch-MLP weights in device layouts
    const __bf16* w1t;         // [hidden][16]     (transposed W1)
    const __bf16* w2f;         // W2^T fragment-major: [hidden/32][hidden/16][64 lanes][8]
    const __bf16* w3p;         // [hidden/32][2][64][8] lane-permuted W3 fragments
    float* temb;               // [T][hidden]      e_j = temb(t_j) Wt
    float* Ep;                 // partial outputs of the misses: [nsplit][N][P][D] per half, or
                               // [hidden / 64][fine_rows][D] per 64 units of a list entry
    int32_t nsplit;            // halves of the output units (partials summed by k_picard)
    int32_t* eps_mode;         // [1 + N] set by each network launch: where the fresh outputs are
                               // (EpsMode), then each sample's first entry in the list of
                               // misses; null = always EPS_SPLIT
    int32_t whole_ok;          // whole outputs may be written into Eh
    int32_t fine_rows;         // list entries whose partial outputs per 64 units fit Ep (EPS_FINE)
    int32_t picard_blocks;
    int32_t mlp_grid;
    // Parareal sampler only (k_parareal.hip)
    double* pr_dev;                    // [B][chunks] partial sums of the Eq. (4) deviation of each
                                       // block's next request, left by the kernel that wrote its
                                       // input; null: k_pr_test computes the deviations
    PrArgs pr;                         // requests whose hit tests the network launch computes
    float* Gc;                         // [B][D] stored coarse values G_n
    double* pr_coef;                   // [B][2] coarse step (ac_n, bc_n)
    pa_request_trace_t* trace_pr;      // request records or null
    float* trace_eps;                  // [records][D] fresh outputs of the misses, or null
    double* trace_res;                 // [B][B+1] boundary residuals per iteration, or null
    // Solver kernels only
    double* part_rows;                 // [N][picard_blocks][2P] part_res and part_dev with a Picard
                                       // block's partials in a row, for the sweeps that k_slide
                                       // of several samples ends (part_res and part_dev are then
                                       // null), or null
};

// Kernel launchers (all asynchronous on `st`).
hipError_t launch_reset(const Dev& d, hipStream_t st);
// start/stop: optional events attached to the kernel's dispatch (null = untimed).
hipError_t launch_slide(const Dev& d, hipStream_t st, hipEvent_t start, hipEvent_t stop);
// The slide outstanding after a fused sweep, from the Picard kernel's snapshot (no-op if none).
hipError_t launch_slide_pending(const Dev& d, hipStream_t st);
// Largest fp64 partial-sum volume per sample the network kernel reduces redundantly per block.
constexpr size_t kFusedSlideMaxBytes = 256 * 1024;
// The same for the Picard kernel of a linear network, its longest window and the most blocks of a
// launch (two per CU). Sample with a slide launch per sweep -> without (D, T, window, samples):
// 256, 10, 4, 1 63 -> 46 us; 2220, 50, 17, 5 90 -> 75; 4096, 100, 32, 1 95 -> 85; 4096, 100, 32, 8
// (512 blocks) 111 -> 100. More blocks repeat the slide more than they save: 4096, 100, 32, 32
// (2048 blocks) 156 -> 190, 16384, 100, 8, 8 (2048) 254 -> 265.
constexpr size_t kFusedLinearMaxBytes = 32 * 1024;
constexpr int kFusedLinearMaxWindow = 64;
constexpr long long kFusedLinearMaxBlocks = 512;
// pending: the last sweep's slide is outstanding (fused_linear: the kernel computes it).
hipError_t launch_picard(const Dev& d, hipStream_t st, int linear, hipEvent_t start, hipEvent_t stop, int pending);
// single: the launch evaluates at most one latent.
hipError_t launch_eps_mlp(const Dev& d, hipStream_t st, hipEvent_t start, hipEvent_t stop, int single = 0);
// List entries up to which a launch may take items that leave partial outputs per 64 units.
int mlp_fine_rows(int hidden, int ntok, int grid);
// Rearranges the patch-MLP weights ([in][out] bf16 bit patterns, device) into the network
// kernel's layouts: w1t [H][16], w2f (W2^T fragments, halved), w3p (lane-permuted W3
// fragments, halved).
hipError_t launch_pack_weights(const uint16_t* w1, const uint16_t* w2, const uint16_t* w3, int H,
                               __bf16* w1t, __bf16* w2f, __bf16* w3p, hipStream_t st);
hipError_t launch_temb_table(const Dev& d, const double* t_values_dev, const __bf16* wt_dev,
                             int temb_dim, hipStream_t st);
int picard_blocks(int D, int P);
int mlp_supported(int hidden);
int mlp_tokens_per_item();
int mlp_splits(int hidden);
int mlp_grid_size(int device_cus);

}  // namespace pa
