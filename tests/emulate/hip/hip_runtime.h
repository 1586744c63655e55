// Host stand-in for the device language the kernels of csrc/*.hip use, so that a test can run them
// on the CPU in an order of its choosing: a block is an OS thread, its lanes are fibers of that
// thread (64 to a wave, a wave runs until all of its lanes wait), shared memory is the thread's.
// Matrix and buffer instructions are not there: a launch that reaches one ends the program.
//
// The order: waves of a block in turn, blocks of a launch in turn. With emu::hook set, block
// hook.block stops before its hook.step-th run of a wave, the launch's block 0 runs from its start
// to its end, and then the stopped block goes on: what a block sees that shares the chip with a
// faster one. emu::uneven counts barriers that a lane of the block did not reach because it had
// left the kernel already.
#pragma once
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <functional>
#include <thread>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static thread_local

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
struct alignas(16) double4 { double x, y, z, w; };
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline double4 make_double4(double x, double y, double z, double w) { return {x, y, z, w}; }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }

typedef void* hipStream_t;
typedef void* hipEvent_t;
enum hipError_t { hipSuccess, hipErrorInvalidValue };
inline hipError_t hipGetLastError() { return hipSuccess; }

namespace emu {

enum State { READY, WAVE_OP, BARRIER, LEFT };
constexpr size_t kStack = 256 * 1024;

struct Lane {
    ucontext_t ctx;
    State state = READY;
    int op = 0;                     // which wave operation, and its operand
    uint64_t value = 0;
};

struct Block {
    std::vector<Lane> lanes;
    ucontext_t sched;
    int current = 0;
    std::function<void()> kernel;
    std::vector<uint64_t> seen;     // operands of the wave's last operation
};

struct Hook {
    int block = -1, step = 0;
    bool reached = false;
};

inline Hook hook;
inline int uneven = 0;
inline thread_local Block* self = nullptr;
inline thread_local dim3 thread_idx, block_idx, block_dim, grid_dim;

[[noreturn]] inline void die(const char* what) {
    fprintf(stderr, "emulated kernel: %s (block %u, lane %u)\n", what, block_idx.x, thread_idx.x);
    abort();
}

inline void wait(State s) {
    Block* b = self;
    Lane& l = b->lanes[b->current];
    l.state = s;
    swapcontext(&l.ctx, &b->sched);
}

// All lanes of the wave that have not left give a value; each returns to the values of all 64.
inline const uint64_t* exchange(int op, uint64_t v) {
    Lane& l = self->lanes[self->current];
    l.op = op;
    l.value = v;
    wait(WAVE_OP);
    return &self->seen[self->current / 64 * 64];
}

inline void lane_main() {
    Block* b = self;
    b->kernel();
    b->lanes[b->current].state = LEFT;
    swapcontext(&b->lanes[b->current].ctx, &b->sched);
}

inline void run_block(const std::function<void()>& kernel, dim3 grid, dim3 block, unsigned bx, unsigned by,
                      const std::function<void()>& at_step, int step) {
    std::thread([&] {
        Block b;
        const int n = (int)block.x;
        b.lanes.resize(n);
        b.seen.assign((n + 63) / 64 * 64, 0);
        b.kernel = kernel;
        self = &b;
        block_idx = dim3(bx, by);
        block_dim = block;
        grid_dim = grid;
        char* stacks = (char*)mmap(nullptr, n * kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        if (stacks == MAP_FAILED) die("no memory for the stacks");
        for (int i = 0; i < n; ++i) {
            ucontext_t& c = b.lanes[i].ctx;
            getcontext(&c);
            c.uc_stack.ss_sp = stacks + i * kStack;
            c.uc_stack.ss_size = kStack;
            c.uc_link = nullptr;
            makecontext(&c, lane_main, 0);
        }
        for (int runs = 0;;) {
            bool ran = false;
            for (int w = 0; w < n; w += 64) {
                const int end = w + 64 < n ? w + 64 : n;
                for (bool more = true; more;) {
                    more = false;
                    bool ready = false;
                    for (int i = w; i < end; ++i) ready = ready || b.lanes[i].state == READY;
                    if (!ready) break;
                    if (at_step && runs == step) at_step();
                    ++runs;
                    ran = true;
                    int ops = 0, barriers = 0, op = -1;
                    for (int i = w; i < end; ++i) {
                        if (b.lanes[i].state == READY) {
                            b.current = i;
                            thread_idx = dim3(i);
                            swapcontext(&b.sched, &b.lanes[i].ctx);
                        }
                        const Lane& l = b.lanes[i];
                        if (l.state == WAVE_OP) {
                            if (op >= 0 && op != l.op) die("lanes of a wave at different operations");
                            op = l.op;
                            ++ops;
                        }
                        barriers += l.state == BARRIER;
                    }
                    if (ops && barriers) die("lanes of a wave at an operation and at a barrier");
                    if (ops) {
                        for (int i = w; i < end; ++i) b.seen[i] = b.lanes[i].state == WAVE_OP ? b.lanes[i].value : 0;
                        for (int i = w; i < end; ++i)
                            if (b.lanes[i].state == WAVE_OP) b.lanes[i].state = READY;
                        more = true;
                    }
                }
            }
            int left = 0;
            for (const Lane& l : b.lanes) left += l.state == LEFT;
            if (left == n) break;
            if (!ran) die("no lane can run");
            if (left) ++uneven;             // the hardware's barrier would go on without them
            for (Lane& l : b.lanes)
                if (l.state == BARRIER) l.state = READY;
        }
        munmap(stacks, n * kStack);
    }).join();
}

inline void launch(const std::function<void()>& kernel, dim3 grid, dim3 block) {
    for (unsigned y = 0; y < grid.y; ++y) {
        bool first_done = false;
        const std::function<void()> none, first = [&, y] {
            run_block(kernel, grid, block, 0, y, none, 0);
            first_done = true;
            hook.reached = true;
        };
        const bool hooked = hook.block > 0 && hook.block < (int)grid.x;
        if (hooked) run_block(kernel, grid, block, hook.block, y, first, hook.step);
        for (unsigned x = 0; x < grid.x; ++x) {
            if (hooked && ((int)x == hook.block || (x == 0 && first_done))) continue;
            run_block(kernel, grid, block, x, y, none, 0);
        }
    }
}

template <class T>
inline T shuffle(T v, int src) {
    uint64_t bits = 0;
    memcpy(&bits, &v, sizeof v);
    const uint64_t* all = exchange(1, bits);
    T r;
    memcpy(&r, &all[src], sizeof r);
    return r;
}

}  // namespace emu

#define threadIdx emu::thread_idx
#define blockIdx emu::block_idx
#define blockDim emu::block_dim
#define gridDim emu::grid_dim
#define __syncthreads() emu::wait(emu::BARRIER)

template <class T>
inline T __shfl_xor(T v, int off, int width) {
    const int lane = threadIdx.x & 63, s = lane ^ off;
    return emu::shuffle(v, s / width == lane / width ? s : lane);
}
template <class T>
inline T __shfl_up(T v, int off, int width) {
    const int lane = threadIdx.x & 63;
    return emu::shuffle(v, lane % width >= off ? lane - off : lane);
}
inline unsigned long long __ballot(int p) {
    const uint64_t* all = emu::exchange(2, p != 0);
    unsigned long long m = 0;
    for (int i = 0; i < 64; ++i) m |= (unsigned long long)(all[i] & 1) << i;
    return m;
}
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __ffsll(long long v) { return __builtin_ffsll(v); }

#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define __hip_atomic_store(p, v, order, scope) (void)(*(p) = (v))
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_s_setprio(x) ((void)0)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, x, y, z) (emu::die("matrix instruction"), (c))
typedef int __amdgpu_buffer_rsrc_t;
#define __builtin_amdgcn_make_buffer_rsrc(p, s, n, f) 0
typedef unsigned emu_u32x4 __attribute__((ext_vector_type(4)));
#define __builtin_amdgcn_raw_buffer_load_b128(r, v, s, a) (emu::die("buffer load"), emu_u32x4{})

#define hipLaunchKernelGGL(k, grid, block, lds, st, ...) \
    ((void)(st), emu::launch([&] { k(__VA_ARGS__); }, grid, block))
#define hipExtLaunchKernelGGL(k, grid, block, lds, st, e0, e1, flags, ...) \
    ((void)(st), (void)(e0), (void)(e1), emu::launch([&] { k(__VA_ARGS__); }, grid, block))
