// fp32 path: the same dataflow as the 16-bit MFMA path (App. B Table 5 rows 1-10 on the re-index
// vector) on the fp32 matrix instructions, for workloads where products must stay in fp32.
//
// What bounds it: v_mfma_f32_16x16x4_f32 runs at 256 FLOP per clock and CU (157 TFLOP/s on the chip), a
// sixteenth of the bf16 rate and twice what plain FMAs reach without the packed forms, so unlike in the
// 16-bit path a 64x64 tile already asks LDS and L2 for a small part of what they deliver (16 B per clock
// and CU from L2).  The tiles are therefore small (64x64, or 32x32 where those are too few for 256 CUs),
// several workgroups share a CU and hide each other's latencies, and any size and any (dword) alignment of
// rows is taken: 16-byte loads where a block is whole, element by element where a tile meets an edge.
// Measured at 8192 rows, d = 384, f = 1536, 8 experts (9.7 GFLOP a contraction), against 16x16 tiles of plain
// FMAs: fc1 601 -> 114 us, fc2 631 -> 112, the two backward layers 1249 -> 203 and 1303 -> 199: 85 to 97
// TFLOP/s, where a loop of nothing but these instructions reaches 136 to 145.  The rest is the uneven last
// round of tiles and, in fc1 and dgrad2, tanhf.
#include <type_traits>

#include "common.h"

namespace {

enum Op { F32_FC1 = 0, F32_FC2, F32_DGRAD2, F32_DGRAD1, F32_WGRAD2, F32_WGRAD1 };

struct TileArgs {
    const float* A;        // row GEMM: [rows][K] (tokens for FC1, else perm positions); token contraction: [rows][M]
    const float* B;        // row GEMM: weights [E][..]; token contraction: [A][N] perm order
    const float* bias;     // FC1, FC2: [E][N]
    const float* pre_in;   // DGRAD2: saved pre-activations [A][N]
    float* out0;           // row GEMM: [A][N]; token contraction: [E][M][N]
    float* kpart;          // token contraction: partial tiles [slot][M][N] of experts cut into chunks
    float* out1;           // FC1: h
    float* colpart;        // DGRAD2: column sums of its output per (row tile, wave row)
    const int32_t* perm;
    const int32_t* offsets;
    int K, N, M, E, k, act;
    int chunk_len;         // token contraction: rows per chunk that are aimed at (see chunk_count)
};

__device__ __forceinline__ float gelu_f(float u) {
    return 0.5f * u * (1.f + tanhf(HEXA_GELU_C * (u + HEXA_GELU_A * u * u * u)));
}
__device__ __forceinline__ float gelu_grad_f(float u) {
    const float th = tanhf(HEXA_GELU_C * (u + HEXA_GELU_A * u * u * u));
    return 0.5f * (1.f + th) +
           0.5f * u * (1.f - th * th) * HEXA_GELU_C * (1.f + 3.f * HEXA_GELU_A * u * u);
}

// F and F' for the three activations (accurate library functions: this is the 1e-5 path)
__device__ __forceinline__ float act_f(float u, int act) {
    if (act == HEXA_ACT_RELU) return u > 0.f ? u : 0.f;
    if (act == HEXA_ACT_SILU) return u / (1.f + expf(-u));
    return gelu_f(u);
}
__device__ __forceinline__ float act_grad_f(float u, int act) {
    if (act == HEXA_ACT_RELU) return u > 0.f ? 1.f : 0.f;
    if (act == HEXA_ACT_SILU) {
        const float sg = 1.f / (1.f + expf(-u));
        return sg * (1.f + u * (1.f - sg));
    }
    return gelu_grad_f(u);
}

// One operand's share of a K-block: R rows (or columns) x BK contraction elements, 256 threads, NC chunks of
// four floats each.  K-contiguous operands lie in LDS as [row][BK + 4], K-strided ones as [k][R + 4], both as
// in memory.  The four extra floats make a row pitch of 4 mod 16 words: the 16 rows (128-bit reads) and the
// four k-rows (32-bit reads) that a fragment read touches at once fall on different banks.
template <bool KS, int R, int BK>
struct Operand {
    static constexpr int CPR = (KS ? R : BK) / 4;      // chunks per image row
    static constexpr int STEP = 256 / CPR;             // image rows from a thread's chunk to its next one
    static constexpr int NC = R * BK / 4 / 256;
    static constexpr int PITCH = (KS ? R : BK) + 4;
    static constexpr int FLOATS = (KS ? BK : R) * PITCH;
    static_assert(PITCH % 16 == 4 && NC >= 1 && NC * STEP == (KS ? BK : R), "unsupported block shape");

    __device__ static __forceinline__ int row() { return (int)threadIdx.x / CPR; }
    __device__ static __forceinline__ int col() { return 4 * ((int)threadIdx.x % CPR); }
    __device__ static __forceinline__ void put(float* s, const f32x4 (&r)[NC]) {
#pragma unroll
        for (int i = 0; i < NC; ++i) *reinterpret_cast<f32x4*>(s + (row() + STEP * i) * PITCH + col()) = r[i];
    }
    // The four contraction elements 16 h + 4 grp + 0..3 of row (column) `base + l16`.
    __device__ static __forceinline__ f32x4 frag(const float* s, int base, int h, int l16, int grp) {
        if constexpr (!KS) return *reinterpret_cast<const f32x4*>(s + (base + l16) * PITCH + 16 * h + 4 * grp);
        f32x4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = s[(16 * h + 4 * grp + q) * PITCH + base + l16];
        return v;
    }
};

// LDS of a tile class: two buffers (one multiplied, one filled) of both operands.
template <int FM, int BK>
constexpr int tile_floats() {
    constexpr int kc = Operand<false, 32 * FM, BK>::FLOATS, ks = Operand<true, 32 * FM, BK>::FLOATS;
    return 4 * (kc > ks ? kc : ks);
}

// One tile of contraction OP: BM x BM outputs (BM = 32 FM), four wavefronts as 2 x 2, FM x FM blocks of
// v_mfma_f32_16x16x4_f32 each.  ESMM (Sec. 3.1 item 1; App. B Alg. 2) for the row GEMMs, whose rows are
// one expert's segment; ESTMM (item 3; Alg. 4) for the token contractions.
template <int FM, int BK, int OP>
__device__ __forceinline__ void f32_tile(const TileArgs& a, const int item, float* smem) {
    constexpr int BM = 32 * FM;
    constexpr bool TOKENS = OP == F32_WGRAD2 || OP == F32_WGRAD1;
    constexpr bool B_KS = TOKENS || OP == F32_FC1 || OP == F32_FC2;
    using OA = Operand<TOKENS, BM, BK>;
    using OB = Operand<B_KS, BM, BK>;
    constexpr int BUF = tile_floats<FM, BK>() / 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, grp = lane >> 4;

    // ---- which tile: an XCD takes a contiguous eighth of the row GEMM's tiles (column tiles fastest), or an
    // eighth of every chunk's tiles of a token contraction, so that its L2 holds what they share
    const int tn = ceil_div(a.N, BM);
    int e, m0, n0, rows, K, kbeg = 0, row_tile = 0;
    float* tok_out = nullptr;
    if constexpr (!TOKENS) {
        const int tiles = seg_tiles_total_wave(a.offsets, a.E, BM) * tn;
        const int per = ceil_div(tiles, kXcds), loc = item / kXcds;
        const int t = item % kXcds * per + loc;
        if (loc >= per || t >= tiles) return;
        row_tile = t / tn;
        const SegTile s = seg_tile_find_wave(a.offsets, a.E, BM, row_tile);
        e = s.e; m0 = s.row0; rows = s.rows; n0 = (t - row_tile * tn) * BM; K = a.K;
    } else {
        int t;
        const int i = token_item_of(item, ceil_div(a.M, BM) * tn, t);
        if (i < 0) return;
        const ChunkItem c = chunk_find_wave(a.offsets, a.E, a.chunk_len, i);
        if (c.e < 0) return;
        e = c.e; kbeg = c.beg; K = c.end - c.beg;
        m0 = (t / tn) * BM; n0 = (t % tn) * BM; rows = min(BM, a.M - m0);
        tok_out = c.slot >= 0 ? a.kpart + (size_t)c.slot * a.M * a.N : a.out0 + (size_t)e * a.M * a.N;
    }
    const int nk = ceil_div(K, BK);

    // ---- operand loads of block k0 (a thread's NC chunks); a chunk is masked where the block is not whole
    const int ar = OA::row(), ac = OA::col(), br = OB::row(), bc = OB::col();
    const float* ap[TOKENS ? 1 : OA::NC];
    const float* bp[B_KS ? 1 : OB::NC];
    if constexpr (!TOKENS) {
#pragma unroll
        for (int i = 0; i < OA::NC; ++i) {   // rows past the segment repeat its last one (their results are not stored)
            const int p = m0 + min(ar + OA::STEP * i, rows - 1);
            ap[i] = a.A + (size_t)(OP == F32_FC1 ? a.perm[p] / a.k : p) * a.K + ac;
        }
    } else {
        ap[0] = a.A + (OP == F32_WGRAD1 ? 0 : (size_t)(kbeg + ar) * a.M) + m0 + ac;
    }
    if constexpr (TOKENS) bp[0] = a.B + (size_t)(kbeg + br) * a.N + n0 + bc;
    else if constexpr (B_KS) bp[0] = a.B + ((size_t)e * a.K + br) * a.N + n0 + bc;
    else {
#pragma unroll
        for (int i = 0; i < OB::NC; ++i)
            bp[i] = a.B + ((size_t)e * a.N + min(n0 + br + OB::STEP * i, a.N - 1)) * a.K + bc;
    }
    int prow[OA::NC] = {};    // WGRAD1: perm entries of the block that is loaded next
    auto load_perm = [&](int k0) __attribute__((always_inline)) {
        if constexpr (OP == F32_WGRAD1) {
#pragma unroll
            for (int i = 0; i < OA::NC; ++i) prow[i] = a.perm[kbeg + min(k0 + ar + OA::STEP * i, K - 1)];
        }
    };
    // loads block k0 (WGRAD1: and the perm entries of the block behind it, ahead of the data, so that waiting
    // for them does not wait for the data)
    auto load = [&](auto whole, int k0, f32x4 (&va)[OA::NC], f32x4 (&vb)[OB::NC]) __attribute__((always_inline)) {
        const float* p[OA::NC];
#pragma unroll
        for (int i = 0; i < OA::NC; ++i) {
            if constexpr (OP == F32_WGRAD1) p[i] = ap[0] + (size_t)(prow[i] / a.k) * a.M;
            else if constexpr (TOKENS) p[i] = ap[0] + (size_t)(k0 + OA::STEP * i) * a.M;
            else p[i] = ap[i] + k0;
        }
        load_perm(k0 + BK);
#pragma unroll
        for (int i = 0; i < OA::NC; ++i) {
            if constexpr (decltype(whole)::value) va[i] = *reinterpret_cast<const f32x4u*>(p[i]);
            else va[i] = load4(p[i], TOKENS ? (k0 + ar + OA::STEP * i < K ? a.M - m0 - ac : 0) : K - k0 - ac);
        }
#pragma unroll
        for (int i = 0; i < OB::NC; ++i) {
            const float* q = B_KS ? bp[0] + (size_t)(k0 + OB::STEP * i) * a.N : bp[B_KS ? 0 : i] + k0;
            if constexpr (decltype(whole)::value) vb[i] = *reinterpret_cast<const f32x4u*>(q);
            else vb[i] = load4(q, B_KS ? (k0 + br + OB::STEP * i < K ? a.N - n0 - bc : 0) : K - k0 - bc);
        }
    };
    // blocks that need no masking: none in a tile at an edge of the output
    const bool inner = (!TOKENS || m0 + BM <= a.M) && (!B_KS || n0 + BM <= a.N);
    const int nwhole = inner ? K / BK : 0;

    f32x4 acc[FM][FM];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Block j + 2 is on its way to registers and block j + 1 already there while block j is multiplied.
    f32x4 va0[OA::NC], vb0[OB::NC], va1[OA::NC], vb1[OB::NC];
    constexpr std::true_type WHOLE;
    constexpr std::false_type MASKED;
    if (nk > 0) {
        load_perm(0);
        load(MASKED, 0, va0, vb0);
        if (nk > 1) load(MASKED, BK, va1, vb1);
        OA::put(smem, va0);
        OB::put(smem + BUF, vb0);
    }
    __syncthreads();
    // multiplies block j; f: registers for block j + 2, n: block j + 1
    auto block = [&](auto whole, int j, f32x4 (&vaf)[OA::NC], f32x4 (&vbf)[OB::NC], f32x4 (&van)[OA::NC], f32x4 (&vbn)[OB::NC])
                     __attribute__((always_inline)) {
        const float* sa = smem + (j & 1) * 2 * BUF;
        const float* sb = sa + BUF;
        if (decltype(whole)::value || j + 2 < nk) load(whole, (j + 2) * BK, vaf, vbf);
#pragma unroll
        for (int h = 0; h < BK / 16; ++h) {
            f32x4 fa[FM], fb[FM];
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                fb[i] = OB::frag(sb, 16 * (wn * FM + i), h, l16, grp);
                fa[i] = OA::frag(sa, 16 * (wm * FM + i), h, l16, grp);
            }
            // B first: the block comes out transposed, a lane holds row l16 and four consecutive columns
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int jj = 0; jj < FM; ++jj)
                        acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[jj][q], fa[i][q], acc[i][jj], 0, 0, 0);
        }
        if (decltype(whole)::value || j + 1 < nk) {
            float* s = smem + ((j + 1) & 1) * 2 * BUF;   // last read in block j - 1, before the barrier behind it
            OA::put(s, van);
            OB::put(s + BUF, vbn);
        }
        __syncthreads();
    };
    int j = 0;
    for (; j + 3 < nwhole; j += 2) {   // two loops, so that the compiler can count the loads in flight in the first
        block(WHOLE, j, va0, vb0, va1, vb1);
        block(WHOLE, j + 1, va1, vb1, va0, vb0);
    }
    for (; j < nk; j += 2) {
        block(MASKED, j, va0, vb0, va1, vb1);
        if (j + 1 < nk) block(MASKED, j + 1, va1, vb1, va0, vb0);
    }

    // ---- epilogue
    float* out = TOKENS ? tok_out : a.out0;
#pragma unroll
    for (int jj = 0; jj < FM; ++jj) {
        const int n = n0 + 16 * (wn * FM + jj) + 4 * grp, nv = a.N - n;
        f32x4 bias = {0.f, 0.f, 0.f, 0.f}, cs = {0.f, 0.f, 0.f, 0.f};
        if constexpr (OP == F32_FC1 || OP == F32_FC2) bias = load4(a.bias + (size_t)e * a.N + n, nv);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int m = 16 * (wm * FM + i) + l16;
            if (m < rows && nv > 0) {
                const size_t oi = (size_t)(m0 + m) * a.N + n;
                f32x4 v = acc[i][jj] + bias;
                if constexpr (OP == F32_DGRAD2) {
                    const f32x4 u = load4(a.pre_in + oi, nv);
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] *= act_grad_f(u[r], a.act);
                    cs += v;
                }
                store4(out + oi, v, nv);
                if constexpr (OP == F32_FC1) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = act_f(v[r], a.act);
                    store4(a.out1 + oi, v, nv);
                }
            }
        }
        if constexpr (OP == F32_DGRAD2) {   // bias gradient (ESS, Table 5 row 8): this wave row's share of the column sums
#pragma unroll
            for (int r = 0; r < 4; ++r) cs[r] = row_sum16(cs[r]);
            if (l16 == 0) store4(a.colpart + (size_t)(2 * row_tile + wm) * a.N + n, cs, nv);
        }
    }
}

template <int FM, int BK, int OP>
__global__ __launch_bounds__(256) void f32_gemm(TileArgs a) {
    __shared__ __align__(16) float smem[tile_floats<FM, BK>()];
    f32_tile<FM, BK, OP>(a, (int)blockIdx.x, smem);
}

// Input gradient (OPA, slots [0, items_a)) and weight gradient (OPB) of one linear layer in one grid: neither
// needs the other's result, and the tail of one fills with tiles of the other.
template <int FM, int BK, int OPA, int OPB>
__global__ __launch_bounds__(256) void f32_gemm_pair(TileArgs ra, TileArgs rb, int items_a) {
    __shared__ __align__(16) float smem[tile_floats<FM, BK>()];
    const int item = (int)blockIdx.x;
    if (item < items_a) f32_tile<FM, BK, OPA>(ra, item, smem);
    else f32_tile<FM, BK, OPB>(rb, item - items_a, smem);
}

int row_items(const MoeDims& D, int bm, int N) {
    return kXcds * ceil_div((D.A / bm + D.E) * ceil_div(N, bm), kXcds);
}
int token_items(const MoeDims& D, int bm) {
    return kXcds * ceil_div(ceil_div(D.d, bm) * ceil_div(D.f, bm), kXcds) * (D.A / f32_chunk_len(D) + D.E);
}

// Which class a launch takes: 64x64 tiles fetch half as much per FLOP, 32x32 tiles are four times as many and
// waste less at the ends of segments.  The line is where a row GEMM has 700 of the larger tiles, not quite three
// per CU; measured on both sides (us, 64x64 / 32x32), d = 384, f = 1536, 8 experts, top-2: fc1 113 / 142 at
// 4096 tokens (3264 tiles), 46 / 45 at 1024 (960 tiles); fc2 at 1024 tokens (240 tiles) 46 / 43; d = 64,
// f = 256, 4 experts at 256 tokens (32 tiles): fc1 9.6 / 6.5.
bool small_rows(const MoeDims& D, int N) {
    return (long long)(D.A / 64 + D.E) * ceil_div(N, 64) < 700;
}

template <int FM, int BK, int OP>
void rows_launch(const MoeDims& D, const TileArgs& a, hipStream_t st, const char* label) {
    ProfScope ps(st, label);
    hipLaunchKernelGGL((f32_gemm<FM, BK, OP>), dim3(row_items(D, 32 * FM, a.N)), dim3(256), 0, st, a);
}
template <int FM, int BK, int OPA, int OPB>
void pair_launch(const MoeDims& D, const TileArgs& ra, const TileArgs& rb, hipStream_t st, const char* label) {
    ProfScope ps(st, label);
    const int items_a = row_items(D, 32 * FM, ra.N), items_b = token_items(D, 32 * FM);
    hipLaunchKernelGGL((f32_gemm_pair<FM, BK, OPA, OPB>), dim3(items_a + items_b), dim3(256), 0, st, ra, rb, items_a);
}

}  // namespace

// Rows per chunk of the token contractions: what makes four workgroups per CU of chunks and tiles, at least 256 (a
// chunk costs a partial d x f tile written and read back).
int f32_chunk_len(const MoeDims& D) {
    const long long tiles = (long long)ceil_div(D.d, 64) * ceil_div(D.f, 64);
    long long L = ((long long)D.A * tiles / 1024 + 63) / 64 * 64;
    if (L < 256) L = 256;
    return (int)(L < 0x7fffffc0 ? L : 0x7fffffc0);
}
void f32_tile_classes(const MoeDims& D, int (&tile)[4]) {
    tile[0] = tile[2] = small_rows(D, D.f) ? 32 : 64;
    tile[1] = tile[3] = small_rows(D, D.d) ? 32 : 64;
}
int f32_dgrad2_row_tile(const MoeDims& D) { return small_rows(D, D.f) ? 32 : 64; }

hipError_t launch_f32_fwd(const MoeDims& D, const float* x, const float* W1, const float* b1,
                          const float* W2, const float* b2, const hexa_moe_idx& idx,
                          const MoeWorkspace& ws, hipStream_t st) {
    TileArgs a{};
    a.offsets = idx.offsets; a.perm = idx.perm; a.k = D.k; a.E = D.E; a.act = D.act;
    // fc1: pre = x W1 + b1, h = F(pre)
    a.A = x; a.B = W1; a.bias = b1; a.out0 = (float*)ws.pre; a.out1 = (float*)ws.h; a.K = D.d; a.N = D.f;
    if (small_rows(D, a.N)) rows_launch<1, 64, F32_FC1>(D, a, st, "fc1");
    else rows_launch<2, 32, F32_FC1>(D, a, st, "fc1");
    // fc2: o = h W2 + b2
    a.A = (const float*)ws.h; a.B = W2; a.bias = b2; a.out0 = (float*)ws.o; a.out1 = nullptr; a.K = D.f; a.N = D.d;
    if (small_rows(D, a.N)) rows_launch<1, 64, F32_FC2>(D, a, st, "fc2");
    else rows_launch<2, 32, F32_FC2>(D, a, st, "fc2");
    return hipGetLastError();
}

hipError_t launch_f32_bwd(const MoeDims& D, const float* x, const float* W1, const float* W2,
                          const hexa_moe_idx& idx, const MoeWorkspace& ws, float* dW1, float* dW2,
                          hipStream_t st) {
    TileArgs g{};
    g.offsets = idx.offsets; g.perm = idx.perm; g.k = D.k; g.E = D.E; g.act = D.act; g.chunk_len = f32_chunk_len(D);
    // 2nd linear layer: dpre = (do W2^T) * F'(pre)  and  dW2[e] = h^T do
    TileArgs r = g, t = g;
    r.A = (const float*)ws.dout; r.B = W2; r.pre_in = (const float*)ws.pre; r.out0 = (float*)ws.dpre;
    r.colpart = ws.colpart1; r.K = D.d; r.N = D.f;
    t.A = (const float*)ws.h; t.B = (const float*)ws.dout; t.out0 = dW2; t.kpart = ws.kpart2; t.M = D.f; t.N = D.d;
    if (small_rows(D, r.N)) pair_launch<1, 64, F32_DGRAD2, F32_WGRAD2>(D, r, t, st, "bwd_fc2");
    else pair_launch<2, 32, F32_DGRAD2, F32_WGRAD2>(D, r, t, st, "bwd_fc2");
    // 1st linear layer: dxp = dpre W1^T  and  dW1[e] = x[perm/k]^T dpre
    r = g; t = g;
    r.A = (const float*)ws.dpre; r.B = W1; r.out0 = (float*)ws.dxp; r.K = D.f; r.N = D.d;
    t.A = x; t.B = (const float*)ws.dpre; t.out0 = dW1; t.kpart = ws.kpart1; t.M = D.d; t.N = D.f;
    if (small_rows(D, r.N)) pair_launch<1, 64, F32_DGRAD1, F32_WGRAD1>(D, r, t, st, "bwd_fc1");
    else pair_launch<2, 32, F32_DGRAD1, F32_WGRAD1>(D, r, t, st, "bwd_fc1");
    return hipGetLastError();
}
