// How expert segments are cut: plain arithmetic, without HIP headers, so that host programs can include it too.
#pragma once

__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// How a token contraction cuts an expert's n rows: into as many chunks as keep them below 9/8 L (a second chunk
// for a few rows would cost two partial tiles written and read back), equal up to the 64-row blocks they start on.
// Measured, backward launches in us with equal chunks below L / 9/8 L / 3/2 L: 4096 x 384 x 1536 top-2 of 8 experts (1024
// rows each, L = 1024) 93.9 / 83.9 / 83.9; 3001 x 320 x 448 top-3 of 17 under Zipf routing 50.4 / 50.3 / 53.3; 32768 x 768 x
// 3072 under Zipf routing the same within 0.3 %.  The first is the shape that tells L from 9/8 L, because L is its average
// expert's rows: about half of its experts lie just above L.  The line moves that step to where few experts lie.
__device__ __forceinline__ int chunk_count(int n, int L) { return n > 0 ? max(1, (n - L / 8 - 1) / L + 1) : 0; }
__device__ __forceinline__ int chunk_start(int n, int nc, int c) {
    const int q = n / nc;
    return c >= nc ? n : (c * q + min(c, n - nc * q)) & ~63;
}
