// The work lists of the 256x256 contraction kernels.  Without HIP headers of its own, so that a host program with
// stand-ins for the few device functions it uses can run the kernel too.
#pragma once
#include "segments.h"

// 256x256 tiles take theirs from work lists: with one workgroup per CU nothing hides the look-up, two scalar
// loads are the shortest, and the launch that builds the lists (once per forward call; the backward pass reads the same
// ones, they are part of what the forward pass leaves in the workspace) is small beside theirs.
//   header (kWlHeader ints): number of row tiles, of token-contraction items; then 1 or 0: the fused backward
//       grid of the second / first linear layer starts with its token contraction (see gemm_bf16_pair)
//   row tiles, then items, four ints each:  expert, first perm row, end perm row, partial buffer
enum WlHeader { WL_TILES = 0, WL_ITEMS, WL_ORDER2, WL_ORDER1 };
constexpr int kWlHeader = 8;

static __global__ __launch_bounds__(1024) void build_worklists(const int32_t* __restrict__ offsets, int E, int L,
                                                               int32_t* __restrict__ wl, int rt_cap, int d, int f) {
    constexpr int NQ = 3;                      // row tiles, items, partial buffers
    __shared__ int s_end[NQ][1024];            // inclusive sums over the experts
    __shared__ int s_off[1025];
    __shared__ int s_wave[NQ + 1][16];
    const int e = threadIdx.x, lane = e & 63, wave = e >> 6;
    int n = 0, b = 0;
    if (e < E) { b = offsets[e]; n = offsets[e + 1] - b; }
    const int nc = chunk_count(n, L);
    int v[NQ] = {wave_scan_incl(ceil_div(n, 256)), wave_scan_incl(nc), wave_scan_incl(nc > 1 ? nc : 0)};
    int longest = n / max(nc, 1);
    // (one writer per entry: nothing orders thread E, which has no expert, behind thread E - 1)
    if (e < E) s_off[e] = b;
    if (e == E - 1) s_off[E] = b + n;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) longest = max(longest, __shfl_xor(longest, off));
    if (lane == 63) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) s_wave[q][wave] = v[q];
        s_wave[NQ][wave] = longest;
    }
    __syncthreads();
    for (int w = 0; w < wave; ++w)
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] += s_wave[q][w];
#pragma unroll
    for (int q = 0; q < NQ; ++q) s_end[q][e] = v[q];
    __syncthreads();
    // the expert that holds number i: the first one whose inclusive sum exceeds i
    auto find = [&](int q, int i) {
        int lo = 0, hi = E - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_end[q][mid] > i) hi = mid; else lo = mid + 1;
        }
        return lo;
    };
    int4* tiles = reinterpret_cast<int4*>(wl + kWlHeader);
    int4* items = tiles + rt_cap;
    for (int i = e; i < s_end[0][E - 1]; i += 1024) {
        const int x = find(0, i);
        const int r0 = s_off[x] + (i - (x > 0 ? s_end[0][x - 1] : 0)) * 256;
        tiles[i] = make_int4(x, r0, min(s_off[x + 1], r0 + 256), -1);
    }
    for (int i = e; i < s_end[1][E - 1]; i += 1024) {
        const int x = find(1, i);
        const int first = x > 0 ? s_end[1][x - 1] : 0, c = i - first;
        const int chunks = s_end[1][x] - first, rows = s_off[x + 1] - s_off[x];
        const int slot = chunks > 1 ? (x > 0 ? s_end[2][x - 1] : 0) + c : -1;
        items[i] = make_int4(x, s_off[x] + chunk_start(rows, chunks, c), s_off[x] + chunk_start(rows, chunks, c + 1), slot);
    }
    if (e == 0) {
        // the longest token-contraction item, in rows; a fused backward grid starts with the token
        // contraction when that item runs at least eight times as long as a tile of the row GEMM it
        // shares the grid with (K = d for the second layer's, K = f for the first layer's)
        for (int w = 1; w < 16; ++w) longest = max(longest, s_wave[NQ][w]);
        wl[WL_TILES] = s_end[0][E - 1]; wl[WL_ITEMS] = s_end[1][E - 1];
        wl[WL_ORDER2] = longest >= 8 * d ? 1 : 0;
        wl[WL_ORDER1] = longest >= 8 * f ? 1 : 0;
    }
}
