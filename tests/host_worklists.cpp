// Runs the kernel build_worklists (csrc/worklists.h, the source the library is built from) on the CPU: 1024 threads
// as coroutines, each run from one barrier or wavefront operation to the next, the wavefronts and the lanes in an
// order that the caller chooses.  Between two barriers nothing orders the wavefronts of a workgroup, so the lists
// must be the same for every order.
//   stdin: order (0 ascending, 1 descending), E, L, rt_cap, d, f, then the E + 1 segment offsets
//   stdout: header, row tiles, token-contraction items
#include <ucontext.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(n)
#define __shared__ static
using std::max;
using std::min;
struct int4 { int x, y, z, w; };
static int4 make_int4(int x, int y, int z, int w) { return int4{x, y, z, w}; }

constexpr int kThreads = 1024;
enum Wait { RUN, BARRIER, SCAN, XOR, DONE };
struct Thread {
    ucontext_t ctx;
    std::vector<char> stack;
    Wait wait = RUN;
    int value = 0, arg = 0;
};
static Thread g_thread[kThreads];
static ucontext_t g_main;
static struct { int x; } threadIdx;

static int wait_for(Wait w, int value, int arg) {
    const int me = threadIdx.x;
    g_thread[me].wait = w; g_thread[me].value = value; g_thread[me].arg = arg;
    swapcontext(&g_thread[me].ctx, &g_main);
    return g_thread[me].value;
}
static void __syncthreads() { wait_for(BARRIER, 0, 0); }
static int wave_scan_incl(int v) { return wait_for(SCAN, v, 0); }
static int __shfl_xor(int v, int mask) { return wait_for(XOR, v, mask); }

#include "../paper_2411_01288_amd/csrc/worklists.h"

static struct { const int32_t* offsets; int E, L; int32_t* wl; int rt_cap, d, f; } g_arg;
static void body() {
    build_worklists(g_arg.offsets, g_arg.E, g_arg.L, g_arg.wl, g_arg.rt_cap, g_arg.d, g_arg.f);
    wait_for(DONE, 0, 0);
}

// one wavefront up to the barrier or the end
static void run_wave(int wave, bool descending) {
    Thread* lanes = g_thread + 64 * wave;
    for (;;) {
        for (int i = 0; i < 64; ++i) {
            const int l = descending ? 63 - i : i;
            if (lanes[l].wait != RUN) continue;
            threadIdx.x = 64 * wave + l;
            swapcontext(&g_main, &lanes[l].ctx);
        }
        const Wait w = lanes[0].wait;
        for (int l = 1; l < 64; ++l)
            if (lanes[l].wait != w) { std::fprintf(stderr, "wavefront %d diverges\n", wave); std::exit(2); }
        if (w == BARRIER || w == DONE) return;
        int in[64], sum = 0;
        for (int l = 0; l < 64; ++l) in[l] = lanes[l].value;
        for (int l = 0; l < 64; ++l) {
            sum += in[l];
            lanes[l].value = w == SCAN ? sum : in[l ^ lanes[l].arg];
            lanes[l].wait = RUN;
        }
    }
}

int main() {
    int order;
    if (std::scanf("%d %d %d %d %d %d", &order, &g_arg.E, &g_arg.L, &g_arg.rt_cap, &g_arg.d, &g_arg.f) != 6) return 1;
    std::vector<int32_t> offsets(g_arg.E + 1);
    for (int32_t& o : offsets)
        if (std::scanf("%d", &o) != 1) return 1;
    const int items = offsets.back() / g_arg.L + g_arg.E;
    std::vector<int32_t> wl(kWlHeader + 4 * (size_t)(g_arg.rt_cap + items), -9);
    g_arg.offsets = offsets.data(); g_arg.wl = wl.data();
    for (Thread& t : g_thread) {
        t.stack.resize(32768);
        getcontext(&t.ctx);
        t.ctx.uc_stack.ss_sp = t.stack.data(); t.ctx.uc_stack.ss_size = t.stack.size(); t.ctx.uc_link = nullptr;
        makecontext(&t.ctx, body, 0);
    }
    for (bool done = false; !done;) {
        for (int i = 0; i < kThreads / 64; ++i) run_wave(order ? kThreads / 64 - 1 - i : i, order != 0);
        done = g_thread[0].wait == DONE;
        for (Thread& t : g_thread) {
            if ((t.wait == DONE) != done) { std::fprintf(stderr, "wavefronts disagree on a barrier\n"); return 2; }
            if (!done) t.wait = RUN;
        }
    }
    for (int32_t v : wl) std::printf("%d\n", v);
}
