// fp32 path: the same dataflow as the 16-bit MFMA path (App. B Table 5 rows 1-10 on the re-index
// vector), for workloads whose products and sums must be fp32.  Any size and any (dword) alignment of rows is taken:
// 16-byte range-checked loads, element-by-element stores where a tile meets an edge; tiles are small (64x64, 128x64 for long
// contractions, or 32x32 where those are too few for 256 CUs) and several workgroups share a CU and hide each other's latencies.
//
// 32x32 tiles run on v_mfma_f32_16x16x4_f32: 256 FLOP per clock and CU (157 TFLOP/s on the chip), a sixteenth of the bf16
// rate.  Larger tiles run on the bf16 instruction with every operand split into three bf16 numbers that add up to it (see split2;
// the method of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations",
// 2019): six products instead of one, at sixteen times the rate.  What bounds them is no longer the matrix pipe (27 to 31 % busy) but
// everything around it in turn: splitting, LDS (33 to 39 %), two barriers a step.
// Measured at 8192 rows, d = 384, f = 1536, 8 experts (9.7 GFLOP a contraction), against the fp32 instruction on the same tiles:
// fc1 110 -> 94 us, fc2 108 -> 91, the two backward layers 199 -> 167 and 192 -> 163.  Errors against fp64, that shape's step: y 8.0e-7 ->
// 1.7e-7, dx 8.0e-7 -> 1.7e-7, dW1 6.8e-7 -> 1.5e-7, db1 3.8e-7 -> 1.4e-7; at other lengths see split2, multiply_split and kSplitFrom.  Tried
// and not kept: all fragments read at once (three workgroups per CU, 12 % slower), two LDS buffers with the split between the products
// (12 % slower), 64x128 tiles (fc2 3 % faster, fc1 20 % slower).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

enum Op { F32_FC1 = 0, F32_FC2, F32_DGRAD2, F32_DGRAD1, F32_WGRAD2, F32_WGRAD1 };

struct TileArgs {
    const float* A;        // row GEMM: [rows][K] (tokens for FC1, else perm positions); token contraction: [rows][M]
    const float* B;        // row GEMM: weights [E][..]; token contraction: [A][N] perm order
    const float* bias;     // FC1, FC2: [E][N]
    const float* pre_in;   // DGRAD2: the saved F'(pre) [A][N]
    float* out0;           // row GEMM: [A][N]; token contraction: [E][M][N]
    float* kpart;          // token contraction: partial tiles [slot][M][N] of experts cut into chunks
    float* out1;           // FC1: h
    float* colpart;        // DGRAD2: column sums of its output per (row tile, wave row)
    const int32_t* perm;
    const int32_t* offsets;
    int K, N, M, E, k, act;
    int T;                 // rows of x
    int far;               // some operand has more than 4 GB
    int chunk_len;         // token contraction: rows per chunk that are aimed at (see chunk_count)
};

// h = F(u) and g = F'(u); the forward pass saves g for the backward pass in the place of u, the same bytes.
// GELU: with t = sqrt(2/pi) (u + 0.044715 u^3) and s = 1 / (1 + exp(-2 t)) it is tanh t = 2 s - 1, so h = u s and
// g = s + u s (1 - s) 2C (1 + 3 A u^2).  Of s and 1 - s the larger is r = 1 / (1 + e), e = exp(-2 |t|), the smaller e r: nothing is subtracted from a
// number near itself.  What x = 2 |t| log2(e) and 1 + e lose in rounding is put back, and the reciprocal refined.  About 25 instructions for both, where
// tanhf takes twice that for one (8192 rows, 384 x 1536 of 8: bwd_fc2 170 -> 158 us, fc1 as before).  Below 2^-90 the smaller is 0:
// such numbers only have to be multiplied on the slow way (see split2).
__device__ __forceinline__ void act_both(float u, int act, float& h, float& g) {
    if (act == HEXA_ACT_RELU) {
        h = u > 0.f ? u : 0.f;
        g = u > 0.f ? 1.f : 0.f;
        return;
    }
    if (act == HEXA_ACT_SILU) {
        const float s = 1.f / (1.f + expf(-u));
        h = u / (1.f + expf(-u));
        g = s * (1.f + u * (1.f - s));
        return;
    }
    constexpr double C = 0.79788456080286535588, L = 1.44269504088896340736;
    constexpr float k1 = (float)(2 * C * L), k3 = (float)(2 * C * L * 0.044715);
    const float u2 = u * u, w = fabsf(u), p = fmaf(k3, u2, k1), x = w * p;
    float e = x > 90.f ? 0.f : __builtin_amdgcn_exp2f(-x);
    e = fmaf(-0.69314718f * e, x > 90.f ? 0.f : fmaf(w, p, -x), e);
    const float d = 1.f + e, r0 = __builtin_amdgcn_rcpf(d);
    const float r = fmaf(fmaf(d - 1.f - e, r0, fmaf(-d, r0, 1.f)), r0, r0), er = e * r;
    const float s = u > 0.f ? r : er;
    h = u * s;
    // (from |u| = 1.8e19 on u^2 is infinite and the smaller of s and 1 - s 0: their product is 0)
    g = s + h * (u > 0.f ? er : r) * (x > 90.f ? 0.f : fmaf((float)(6 * C * 0.044715), u2, (float)(2 * C)));
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

// ---- three bf16 planes ----
// a = a1 + a2 + a3: a rounded to bf16, what is left rounded to bf16, and what is left then: 8 + 8 + 8 bits of mantissa, so exactly a but
// for bits below 2^-133, the smallest number of bf16 (that is, for |a| >= 2^-109).  a b is the six products a1 b1, a1 b2, a2 b1,
// a2 b2, a1 b3, a3 b1; the other three are 2^-24 of it at most (a2 is 2^-8 of a at most, a3 2^-17), 7e-9 in the root mean square, and of
// either sign.  (Planes cut off instead of rounded: 2^-21 and always towards zero; sums of a single product were off by 4.2e-7 at
// most and 6.9e-8 in the root mean square, now 9.7e-8 and 2.6e-8, the fp32 instruction 6.0e-8 and 2.5e-8.)  Products of bf16 are exact, sums are fp32.
// `lost` collects what is left for the third plane: a tile in which a bit of any operand has no place (the lower half of that is not zero)
// is multiplied again on the fp32 instruction.  Sums of 512 products with operands of 1e-36 are off by 4e-7 that way, by 5e-5 in planes.  The
// collecting takes 1 % (a step of 4096 x 384 x 1536 of 8 520 -> 527 us); a launch of such tiles only takes both times (bwd_fc2 there 172 -> 322).
struct Planes { uint32_t w[3]; };   // of two values, or of their negatives
template <bool NEG>
__device__ __forceinline__ Planes split2(float a, float b, uint32_t& lost) {
    Planes p;
    if constexpr (NEG) {
        asm("v_cvt_pk_bf16_f32 %0, -%1, -%2" : "=v"(p.w[0]) : "v"(a), "v"(b));   // (the compiler negates in instructions of their own)
        a = -a;
        b = -b;
    } else {
        p.w[0] = pack_bf2(a, b);
    }
    a -= __uint_as_float(p.w[0] << 16);
    b -= __uint_as_float(p.w[0] & 0xffff0000u);
    p.w[1] = pack_bf2(a, b);
    a -= __uint_as_float(p.w[1] << 16);
    b -= __uint_as_float(p.w[1] & 0xffff0000u);
    p.w[2] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);   // the upper halves
    // (in assembly: the compiler would keep all remainders of a step and combine them at its end)
    asm("v_or3_b32 %0, %0, %1, %2" : "+v"(lost) : "v"(a), "v"(b));
    return p;
}

// One operand's share of a K-step of the split path: R rows (or columns) x 32 contraction elements, 256 threads, NC loads
// of four floats each.  LDS holds each plane as [8 elements of k][row][16 bytes], row r at r ^ chunk, whatever the operand's
// order in memory: a 128-bit fragment read touches 16 rows of one chunk (256 consecutive bytes, permuted), and the
// 64-bit stores of a wavefront spread over all banks.
template <bool KS, int R>
struct SplitOperand {
    static constexpr int NC = R / 32;
    static constexpr int KT = KS ? NC : 4;             // consecutive k of a thread
    static constexpr int GROUPS = 32 / KT;             // threads along k
    static constexpr int STEP = KS ? 1 : 256 / GROUPS; // k-rows (KS) or rows from a thread's load to its next one
    static constexpr int PLANE = R * 64;               // bytes
    static_assert(R == 64, "two loads per thread");

    __device__ static __forceinline__ int group() { return (int)threadIdx.x % GROUPS; }
    // first row and column (in memory order, within the block) of the thread's loads
    __device__ static __forceinline__ int row() { return KS ? KT * group() : (int)threadIdx.x / GROUPS; }
    __device__ static __forceinline__ int col() { return KS ? 4 * ((int)threadIdx.x / GROUPS) : 4 * group(); }
    // stores the planes of v, or of -v
    template <bool NEG>
    __device__ static __forceinline__ void put(uint8_t* s, const f32x4 (&v)[NC], uint32_t& lost) {
        const int k = KT * group(), chunk = k / 8, byte = k % 8 * 2;
        auto at = [&](int r) __attribute__((always_inline)) { return s + (chunk * R + (r ^ chunk)) * 16 + byte; };
        if constexpr (KS) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const Planes p = split2<NEG>(v[0][i], v[1][i], lost);
#pragma unroll
                for (int q = 0; q < 3; ++q) *reinterpret_cast<uint32_t*>(at(col() + i) + q * PLANE) = p.w[q];
            }
        } else {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const Planes lo = split2<NEG>(v[i][0], v[i][1], lost), hi = split2<NEG>(v[i][2], v[i][3], lost);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<uint2*>(at(row() + STEP * i) + q * PLANE) = make_uint2(lo.w[q], hi.w[q]);
            }
        }
    }
    // the contraction elements 8 grp + 0..7 of row (column) `base + l16`, plane q
    __device__ static __forceinline__ bf16x8 frag(const uint8_t* s, int q, int base, int l16, int grp) {
        return *reinterpret_cast<const bf16x8*>(s + q * PLANE + (grp * R + ((base + l16) ^ grp)) * 16);
    }
};

// Where a tile lies: expert, first row and column of the output, valid rows, length of the contraction, first perm row (token
// contraction), number of the row tile (row GEMM).
struct TilePlace { int e, m0, n0, rows, K, kbeg, row_tile; };

// p / k for 0 <= p < 2^31 by a product: with 2^(s-1) < k <= 2^s and m = floor(2^(31+s) / k) + 1 it is 2 p m / 2^(32+s), as m k exceeds 2^(31+s)
// by 2^s at most.
struct DivideBy {
    uint32_t m, s;
    __device__ __forceinline__ explicit DivideBy(uint32_t k) : s(k > 1 ? 32 - __builtin_clz(k - 1) : 0) { m = (uint32_t)((1ull << (31 + s)) / k + 1); }
    __device__ __forceinline__ uint32_t operator()(uint32_t p) const { return __umulhi(2 * p, m) >> s; }
};

// A tensor's floats from p on; what is read behind them is zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t floats_at(const float* p, size_t floats) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)(uint32_t)(floats * 4), 0x00020000);
}
// First of the four columns that a thread at `col` of a K-strided block fetches: the last ones at the edge (what lies past it is the next row's
// and the results of those columns are not stored; at most three floats are read past the end of a row).
__device__ __forceinline__ uint32_t edge_column(int n0, int col, int N) { return (uint32_t)(n0 + min(col, (N - n0 - 1) / 4 * 4)) * 4u; }

// Of the four columns from there, the last ones at the edge: zeros where they lie past it.
template <int NC>
__device__ __forceinline__ void clear_edge(f32x4 (&v)[NC], int n0, int col, int N) {
    const int valid = N - n0 - min(col, (N - n0 - 1) / 4 * 4);
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int q = 1; q < 4; ++q) v[i][q] = q < valid ? v[i][q] : 0.f;
}

// What both ways of multiplying share: the loads of K-block k0 (a thread's NC chunks of four floats per operand; OA, OB:
// Operand or SplitOperand), range-checked by buffer resources, so that no edge of a tensor takes a branch: k-rows past the end of a K-strided
// operand are zeros, and the last elements of a K-contiguous one are cleared where the last block is not whole.  (Masked element by element
// at edges and in the first and last blocks of every tile, a step of 1001 x 90 x 362 of 5, top-2, took 58.4 us; so 51.7.)  For operands
// of up to 4 GB (TileArgs::far: larger ones, FarLoader).
template <int BM, int BN, int BK, int OP, typename OA, typename OB, bool SPLIT>
struct BlockLoader {
    static constexpr bool TOKENS = OP == F32_WGRAD2 || OP == F32_WGRAD1, GATHER = OP == F32_WGRAD1;
    static constexpr bool B_KS = TOKENS || OP == F32_FC1 || OP == F32_FC2;
    const TileArgs& a;
    const TilePlace& t;
    const int ar, ac, br, bc;
    const DivideBy token;
    __amdgpu_buffer_rsrc_t ra, rb;
    uint32_t ao[TOKENS ? 1 : OA::NC], bo[B_KS ? 1 : OB::NC];   // K-strided: one, the rest is in the scalar offset
    int prow[OA::NC] = {};    // WGRAD1: perm entries of the block that is loaded next
    int nwhole;               // blocks that need no masking

    __device__ __forceinline__ BlockLoader(const TileArgs& a_, const TilePlace& t_)
        : a(a_), t(t_), ar(OA::row()), ac(OA::col()), br(OB::row()), bc(OB::col()), token((uint32_t)a_.k), nwhole(SPLIT && (ragged_a() || ragged_b()) ? 0 : t_.K / BK) {
        if constexpr (TOKENS) rb = floats_at(a.B + (size_t)t.kbeg * a.N, (size_t)t.K * a.N);
        else rb = floats_at(a.B + (size_t)t.e * a.K * a.N, (size_t)a.K * a.N);
        if constexpr (B_KS) {
            bo[0] = (uint32_t)br * (uint32_t)a.N * 4u + edge_column(t.n0, bc, a.N);
        } else {
#pragma unroll
            for (int i = 0; i < OB::NC; ++i) bo[i] = ((uint32_t)min(t.n0 + br + OB::STEP * i, a.N - 1) * (uint32_t)a.K + (uint32_t)bc) * 4u;
        }
        if constexpr (TOKENS) {
            ra = GATHER ? floats_at(a.A, (size_t)a.T * a.M) : floats_at(a.A + (size_t)t.kbeg * a.M, (size_t)t.K * a.M);
            ao[0] = (GATHER ? 0u : (uint32_t)ar * (uint32_t)a.M * 4u) + edge_column(t.m0, ac, a.M);
        } else {
            ra = OP == F32_FC1 ? floats_at(a.A, (size_t)a.T * a.K) : floats_at(a.A + (size_t)t.m0 * a.K, (size_t)t.rows * a.K);
#pragma unroll
            for (int i = 0; i < OA::NC; ++i) {   // rows past the segment repeat its last one (their results are not stored)
                const int r = min(ar + OA::STEP * i, t.rows - 1);
                ao[i] = ((OP == F32_FC1 ? token((uint32_t)a.perm[t.m0 + r]) : (uint32_t)r) * (uint32_t)a.K + (uint32_t)ac) * 4u;
            }
        }
    }
    __device__ __forceinline__ bool ragged_a() const { return TOKENS && t.m0 + BM > a.M && a.M % 4; }
    __device__ __forceinline__ bool ragged_b() const { return B_KS && t.n0 + BN > a.N && a.N % 4; }
    // What a block holds past the edge of the output is the next row's (weights of other columns, another expert's token): no part of what
    // decides how this tile is multiplied (see split2), so zeros before it is split.
    __device__ __forceinline__ void clear(f32x4 (&va)[OA::NC], f32x4 (&vb)[OB::NC]) {
        if (ragged_a()) clear_edge(va, t.m0, ac, a.M);
        if (ragged_b()) clear_edge(vb, t.n0, bc, a.N);
    }
    __device__ __forceinline__ void load_perm(int k0) {
        if constexpr (GATHER) {
#pragma unroll
            for (int i = 0; i < OA::NC; ++i) prow[i] = a.perm[t.kbeg + min(k0 + ar + OA::STEP * i, t.K - 1)];
        }
    }
    // loads block k0 (WGRAD1: and the perm entries of the block behind it, ahead of the data, so that waiting
    // for them does not wait for the data)
    template <bool WHOLE>
    __device__ __forceinline__ void load(int k0, f32x4 (&va)[OA::NC], f32x4 (&vb)[OB::NC]) {
        auto get = [](__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) __attribute__((always_inline)) {
            return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)v, (int)s, 0));
        };
        uint32_t o[OA::NC];
#pragma unroll
        for (int i = 0; i < OA::NC; ++i) {
            o[i] = ao[TOKENS ? 0 : i];
            if constexpr (GATHER) {
                o[i] += token((uint32_t)prow[i]) * (uint32_t)a.M * 4u;
                if (!WHOLE && k0 + ar + OA::STEP * i >= t.K) o[i] = 0xfffffff0u;   // behind any range
            }
        }
        load_perm(k0 + BK);
#pragma unroll
        for (int i = 0; i < OA::NC; ++i)
            va[i] = get(ra, o[i], GATHER ? 0u : TOKENS ? (uint32_t)(k0 + OA::STEP * i) * (uint32_t)a.M * 4u : (uint32_t)k0 * 4u);
#pragma unroll
        for (int i = 0; i < OB::NC; ++i)
            vb[i] = get(rb, bo[B_KS ? 0 : i], B_KS ? (uint32_t)(k0 + OB::STEP * i) * (uint32_t)a.N * 4u : (uint32_t)k0 * 4u);
        if (!WHOLE && k0 + BK > t.K) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (!TOKENS)
#pragma unroll
                    for (int i = 0; i < OA::NC; ++i) va[i][q] = k0 + ac + q < t.K ? va[i][q] : 0.f;
                if constexpr (!B_KS)
#pragma unroll
                    for (int i = 0; i < OB::NC; ++i) vb[i][q] = k0 + bc + q < t.K ? vb[i][q] : 0.f;
            }
        }
    }
};

// The same for operands of any size: 64-bit addresses, masked where the block is not whole.
template <int BM, int BN, int BK, int OP, typename OA, typename OB>
struct FarLoader {
    static constexpr bool TOKENS = OP == F32_WGRAD2 || OP == F32_WGRAD1;
    static constexpr bool B_KS = TOKENS || OP == F32_FC1 || OP == F32_FC2;
    const TileArgs& a;
    const TilePlace& t;
    const int ar, ac, br, bc;
    const float* ap[TOKENS ? 1 : OA::NC];
    const float* bp[B_KS ? 1 : OB::NC];
    int prow[OA::NC] = {};    // WGRAD1: perm entries of the block that is loaded next
    int nwhole;               // blocks that need no masking: none in a tile at an edge of the output

    __device__ __forceinline__ FarLoader(const TileArgs& a_, const TilePlace& t_)
        : a(a_), t(t_), ar(OA::row()), ac(OA::col()), br(OB::row()), bc(OB::col()) {
        if constexpr (!TOKENS) {
#pragma unroll
            for (int i = 0; i < OA::NC; ++i) {   // rows past the segment repeat its last one (their results are not stored)
                const int p = t.m0 + min(ar + OA::STEP * i, t.rows - 1);
                ap[i] = a.A + (size_t)(OP == F32_FC1 ? a.perm[p] / a.k : p) * a.K + ac;
            }
        } else {
            ap[0] = a.A + (OP == F32_WGRAD1 ? 0 : (size_t)(t.kbeg + ar) * a.M) + t.m0 + ac;
        }
        if constexpr (TOKENS) bp[0] = a.B + (size_t)(t.kbeg + br) * a.N + t.n0 + bc;
        else if constexpr (B_KS) bp[0] = a.B + ((size_t)t.e * a.K + br) * a.N + t.n0 + bc;
        else {
#pragma unroll
            for (int i = 0; i < OB::NC; ++i)
                bp[i] = a.B + ((size_t)t.e * a.N + min(t.n0 + br + OB::STEP * i, a.N - 1)) * a.K + bc;
        }
        const bool inner = (!TOKENS || t.m0 + BM <= a.M) && (!B_KS || t.n0 + BN <= a.N);
        nwhole = inner ? t.K / BK : 0;
    }
    __device__ __forceinline__ void clear(f32x4 (&)[OA::NC], f32x4 (&)[OB::NC]) {}   // (the masks leave none)
    __device__ __forceinline__ void load_perm(int k0) {
        if constexpr (OP == F32_WGRAD1) {
#pragma unroll
            for (int i = 0; i < OA::NC; ++i) prow[i] = a.perm[t.kbeg + min(k0 + ar + OA::STEP * i, t.K - 1)];
        }
    }
    // loads block k0 (WGRAD1: and the perm entries of the block behind it, ahead of the data, so that waiting
    // for them does not wait for the data)
    template <bool WHOLE>
    __device__ __forceinline__ void load(int k0, f32x4 (&va)[OA::NC], f32x4 (&vb)[OB::NC]) {
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
            if constexpr (WHOLE) va[i] = *reinterpret_cast<const f32x4u*>(p[i]);
            else va[i] = load4(p[i], TOKENS ? (k0 + ar + OA::STEP * i < t.K ? a.M - t.m0 - ac : 0) : t.K - k0 - ac);
        }
#pragma unroll
        for (int i = 0; i < OB::NC; ++i) {
            const float* q = B_KS ? bp[0] + (size_t)(k0 + OB::STEP * i) * a.N : bp[B_KS ? 0 : i] + k0;
            if constexpr (WHOLE) vb[i] = *reinterpret_cast<const f32x4u*>(q);
            else vb[i] = load4(q, B_KS ? (k0 + br + OB::STEP * i < t.K ? a.N - t.n0 - bc : 0) : t.K - k0 - bc);
        }
    }
};

// A tile is 32 FM x 32 FN, four wavefronts as 2 x 2, FM x FN blocks each: 32x32, 64x64, 128x64.
constexpr int frag_cols(int fm) { return fm == 4 ? 2 : fm; }

// acc += the tile's contraction on v_mfma_f32_16x16x4_f32; two LDS buffers of both operands, one multiplied, one filled.
template <int R, int BK>
constexpr int f32_image() { return Operand<false, R, BK>::FLOATS > Operand<true, R, BK>::FLOATS ? Operand<false, R, BK>::FLOATS : Operand<true, R, BK>::FLOATS; }
template <int FM, int BK>
constexpr int f32_floats() { return 2 * (f32_image<32 * FM, BK>() + f32_image<32 * frag_cols(FM), BK>()); }
template <int FM, int BK, int OP, bool FAR>
__device__ __forceinline__ void multiply_f32(const TileArgs& a, const TilePlace& t, float* smem, f32x4 (&acc)[FM][frag_cols(FM)]) {
    constexpr int BM = 32 * FM, FN = frag_cols(FM), BN = 32 * FN;
    constexpr bool TOKENS = OP == F32_WGRAD2 || OP == F32_WGRAD1;
    constexpr bool B_KS = TOKENS || OP == F32_FC1 || OP == F32_FC2;
    using OA = Operand<TOKENS, BM, BK>;
    using OB = Operand<B_KS, BN, BK>;
    constexpr int A_BUF = OA::FLOATS, PAIR = OA::FLOATS + OB::FLOATS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, grp = lane >> 4;
    const int nk = ceil_div(t.K, BK);
    typename std::conditional<FAR, FarLoader<BM, BN, BK, OP, OA, OB>, BlockLoader<BM, BN, BK, OP, OA, OB, false>>::type in(a, t);
    // Block j + 2 is on its way to registers and block j + 1 already there while block j is multiplied.
    f32x4 va0[OA::NC], vb0[OB::NC], va1[OA::NC], vb1[OB::NC];
    if (nk > 0) {
        in.load_perm(0);
        in.template load<false>(0, va0, vb0);
        if (nk > 1) in.template load<false>(BK, va1, vb1);
        OA::put(smem, va0);
        OB::put(smem + A_BUF, vb0);
    }
    __syncthreads();
    // multiplies block j; f: registers for block j + 2, n: block j + 1
    auto block = [&](auto whole, int j, f32x4 (&vaf)[OA::NC], f32x4 (&vbf)[OB::NC], f32x4 (&van)[OA::NC], f32x4 (&vbn)[OB::NC])
                     __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value;
        const float* sa = smem + (j & 1) * PAIR;
        const float* sb = sa + A_BUF;
        if (WHOLE || j + 2 < nk) in.template load<WHOLE>((j + 2) * BK, vaf, vbf);
#pragma unroll
        for (int h = 0; h < BK / 16; ++h) {
            f32x4 fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < FN; ++i) fb[i] = OB::frag(sb, 16 * (wn * FN + i), h, l16, grp);
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[i] = OA::frag(sa, 16 * (wm * FM + i), h, l16, grp);
            // B first: the block comes out transposed, a lane holds row l16 and four consecutive columns
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int jj = 0; jj < FN; ++jj)
                        acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[jj][q], fa[i][q], acc[i][jj], 0, 0, 0);
        }
        if (WHOLE || j + 1 < nk) {
            float* s = smem + ((j + 1) & 1) * PAIR;   // last read in block j - 1, before the barrier behind it
            OA::put(s, van);
            OB::put(s + A_BUF, vbn);
        }
        __syncthreads();
    };
    int j = 0;
    for (; j + 3 < in.nwhole; j += 2) {   // two loops, so that the compiler can count the loads in flight in the first
        block(std::true_type{}, j, va0, vb0, va1, vb1);
        block(std::true_type{}, j + 1, va1, vb1, va0, vb0);
    }
    for (; j < nk; j += 2) {
        block(std::false_type{}, j, va0, vb0, va1, vb1);
        if (j + 1 < nk) block(std::false_type{}, j + 1, va1, vb1, va0, vb0);
    }
}

// The same on v_mfma_f32_16x16x32_bf16 with both operands in three planes; one LDS buffer, the next K-step in registers.
// The products of the first planes are added up from zero in every step and then to the accumulator, so that a step rounds once where the
// sums meet; the small ones are added up apart over all steps, and to the accumulator at the end.  The matrix instruction itself
// cuts what lies below its largest product off downwards, which is little of that but adds up in sums over very many results, so every other
// step multiplies by -A and is subtracted (db1 over 300000 rows of 512 products: 3.0e-7 to one side -> 0.5e-7; errors of 4.8e-7, of 6.5e-7
// on the fp32 instruction).
// Steps and signs are the same in every tile: a row's result does not depend on its place in the batch.  lost: see split2.
// Errors are below the fp32 instruction's but where a long contraction has a single product that is not zero (2.6e-8 against 2.5e-8 in the
// root mean square; of two 2.2e-8 against 2.6e-8, of 16 1.3e-8 against 2.8e-8 of their sizes).  (All but a3 b3 of the nine products: a step of
// 4096 x 384 x 1536 of 8 541 -> 584 us.  The small products added up with the large ones in every step: the same time, of two 3.1e-8.)
// Contractions of one K-step run on the fp32 instruction: the planes gain them nothing (fc1 at 8192 tokens x 8, 16, 24, 32 x 2048 of 8,
// top-2, us: 77, 80, 86, 87 that way, 83, 87, 86, 88 in planes; a step of 200000 x 4 x 4 of 4 284 -> 275), and the dropped products show
// where few are summed (rms error of 1, 2, 4, 8 products 2.5e-8, 2.6e-8, 2.7e-8, 2.7e-8 of their sizes' sum, 6.9e-8, 5.7e-8, 4.5e-8, 3.4e-8 in planes).
constexpr int kSplitFrom = 33;
template <int FM>
constexpr int split_bytes() { return 3 * 64 * 64 * FM; }
template <int FM, int OP, bool FAR>
__device__ __forceinline__ void multiply_split(const TileArgs& a, const TilePlace& t, uint8_t* smem, f32x4 (&acc)[FM][FM], uint32_t& lost) {
    constexpr int BM = 32 * FM, BK = 32;
    constexpr bool TOKENS = OP == F32_WGRAD2 || OP == F32_WGRAD1;
    constexpr bool B_KS = TOKENS || OP == F32_FC1 || OP == F32_FC2;
    using OA = SplitOperand<TOKENS, BM>;
    using OB = SplitOperand<B_KS, BM>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, grp = lane >> 4;
    uint8_t* const sb = smem + 3 * OA::PLANE;
    const int nk = ceil_div(t.K, BK);
    typename std::conditional<FAR, FarLoader<BM, BM, BK, OP, OA, OB>, BlockLoader<BM, BM, BK, OP, OA, OB, true>>::type in(a, t);
    // Block j + 1 is on its way to registers while block j is multiplied.
    f32x4 va[OA::NC], vb[OB::NC];
    if (nk > 0) {
        in.load_perm(0);
        in.template load<false>(0, va, vb);
    }
    f32x4 low[FM][FM];    // the small products of all steps
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int jj = 0; jj < FM; ++jj) low[i][jj] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](auto whole, auto odd, int j) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value, ODD = decltype(odd)::value;
        if constexpr (!WHOLE) in.clear(va, vb);
        OA::template put<ODD>(smem, va, lost);
        OB::template put<false>(sb, vb, lost);
        __syncthreads();
        if (WHOLE || j + 1 < nk) in.template load<WHOLE>((j + 1) * BK, va, vb);
        __builtin_amdgcn_sched_barrier(0);   // (the compiler would put the loads behind the products)
        if (j > 0) {     // the small products have the sign of the step's.  (As a branch: spills none of the step's registers)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int jj = 0; jj < FM; ++jj) low[i][jj] = -low[i][jj];
        }
        bf16x8 a1[FM], b1[FM], a2[FM], b2[FM], a3[FM], b3[FM];
        auto read_a = [&](int q, bf16x8 (&f)[FM]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < FM; ++i) f[i] = OA::frag(smem, q, 16 * (wm * FM + i), l16, grp);
        };
        auto read_b = [&](int q, bf16x8 (&f)[FM]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < FM; ++i) f[i] = OB::frag(sb, q, 16 * (wn * FM + i), l16, grp);
        };
        // B first: the block comes out transposed, a lane holds row l16 and four consecutive columns
        auto product = [&](const bf16x8 (&fa)[FM], const bf16x8 (&fb)[FM]) __attribute__((always_inline)) {
#pragma unroll
            for (int jj = 0; jj < FM; ++jj)
#pragma unroll
                for (int i = 0; i < FM; ++i) low[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[jj], fa[i], low[i][jj], 0, 0, 0);
        };
        // planes are read as they are needed (all at once they take the registers of a fourth workgroup on the CU)
        read_a(2, a3); read_b(0, b1);
        __builtin_amdgcn_sched_barrier(0);
        read_a(1, a2);
        product(a3, b1);
        __builtin_amdgcn_sched_barrier(0);
        read_b(1, b2);
        product(a2, b1);
        __builtin_amdgcn_sched_barrier(0);
        read_a(0, a1);
        product(a2, b2);
        __builtin_amdgcn_sched_barrier(0);
        read_b(2, b3);
        product(a1, b2);
        __builtin_amdgcn_sched_barrier(0);
        product(a1, b3);
#pragma unroll
        for (int jj = 0; jj < FM; ++jj)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                if (i == 0) __builtin_amdgcn_sched_barrier(0);   // (two at a time: registers)
                const f32x4 hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b1[jj], a1[i], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                acc[i][jj] = ODD ? acc[i][jj] - hi : acc[i][jj] + hi;
            }
        __syncthreads();
    };
    constexpr std::true_type YES;
    constexpr std::false_type NO;
    int j = 0;
    for (; j + 2 < in.nwhole; j += 2) {
        step(YES, NO, j);
        step(YES, YES, j + 1);
    }
    for (; j < nk; j += 2) {
        step(NO, NO, j);
        if (j + 1 < nk) step(NO, YES, j + 1);
    }
    // low has the sign of the last step
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int jj = 0; jj < FM; ++jj) acc[i][jj] = nk & 1 ? acc[i][jj] + low[i][jj] : acc[i][jj] - low[i][jj];
}

// ---- 128x64 tiles ----
// The same products and sums on 128x64 tiles, 64x32 outputs per wavefront, two workgroups per CU: three quarters of the splitting, of the fragment
// reads and of the loads per product.  The work of a K-step is laid out by hand: behind each of a wavefront's 48 matrix instructions stand
// a fragment read of this step, a piece of the splitting of the next step's operands, the stores of its planes, a load, the additions of the large
// products.  Two LDS buffers, one barrier a step, two steps of operands on their way to registers.
// What a wavefront does with its cycles (counters, fc2 / bwd_fc1 at 8192 rows, 384 x 1536 of 8 experts): it issues in 47 / 43 % (vector and matrix instructions 32 / 29), waits
// to issue in 30 / 31, for loads, LDS and the barrier in 23 / 26, two to a SIMD at most and 1.15 / 1.58 on average; the matrix pipe is busy in 30 / 35 % of
// the launch.  fc2's 432 tiles are less than one round of 512.  Tried and not kept: v_dot2_f32_bf16, which takes a plane off in one instruction instead
// of two (the same time); 128x128 tiles, one workgroup per CU (fc1 there 94 -> 116 us: nothing runs under a tile's start and
// epilogue, 13 us; with four wavefronts of 64x64, 142).
// (a, b), or their negatives, as a bf16 pair; what is left of them, or of their negatives, is left in a and b.
template <bool NEG>
__device__ __forceinline__ uint32_t split_off(float& a, float& b) {
    uint32_t w;
    if constexpr (NEG) {
        asm("v_cvt_pk_bf16_f32 %0, -%1, -%2" : "=v"(w) : "v"(a), "v"(b));
        a = -a;
        b = -b;
    } else {
        w = pack_bf2(a, b);
    }
    a -= __uint_as_float(w << 16);
    b -= __uint_as_float(w & 0xffff0000u);
    return w;
}

// One operand's share of a K-step, R rows (or columns) x 32 contraction elements, 256 threads: a thread has N = R / 32 times four consecutive k, of
// rows row, row + 32, ... (K contiguous: N loads of four floats), or of N consecutive columns (K strided: four loads of N floats).  Neighbouring
// threads have rows or columns four apart, which spreads their 64-bit stores over all banks.  All loads are range-checked by the buffer resource:
// k-rows past the end are zeros (or masked), and so are columns past the edge; at most three floats past the end of a row are read.  LDS holds the planes as in SplitOperand, twice.  (A key of more than two bits would put rows that are read in the same cycle, of
// different chunks, on the same banks: fragment reads took twice as long.)
template <bool KS, bool GATHER, int R>
struct WideOperand {
    static constexpr int N = R / 32, NL = KS ? 4 : N, W = KS ? N : 4;
    static constexpr int PLANE = R * 64, BUFFER = 3 * PLANE;
    static constexpr int PIECES = 7 * N;
    typedef float load_t __attribute__((ext_vector_type(W)));
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t voff[KS && !GATHER ? 1 : NL];
    uint32_t pitch = 0;         // bytes of a k-row
    uint8_t* put_at[KS ? N : 1];
    const uint8_t* frag_at;
    load_t v[2][NL];            // blocks j + 1 and j + 2

    const int tid;              // threadIdx.x
    __device__ __forceinline__ explicit WideOperand(int t) : tid(t) {}
    __device__ __forceinline__ int group() const { return tid & 7; }
    __device__ __forceinline__ int line() const { return tid >> 3; }
    __device__ __forceinline__ int row() const { return (line() & 3) << 2 | (line() >> 2 & 3) | (line() & 16); }
    // a thread's columns of a K-strided operand, the last ones at the edge
    __device__ __forceinline__ uint32_t column(int n0, int n) const { return (uint32_t)(n0 + min(W * line(), (n - n0 - 1) / W * W)) * 4u; }
    __device__ __forceinline__ void resource(const float* p, size_t floats) {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)(uint32_t)(floats * 4), 0x00020000);
    }
    // base: first row or column of the wavefront's fragments
    __device__ __forceinline__ void place(uint8_t* s, int base) {
        const int chunk = group() >> 1, l16 = tid & 15, grp = tid >> 4 & 3;
#pragma unroll
        for (int i = 0; i < (KS ? N : 1); ++i)
            put_at[i] = s + (chunk * R + ((KS ? N * line() + i : row()) ^ chunk)) * 16 + (group() & 1) * 8;
        frag_at = s + (grp * R + base + (l16 ^ grp)) * 16;
    }
    __device__ __forceinline__ bf16x8 frag(int buf, int q, int i) const {
        return *reinterpret_cast<const bf16x8*>(frag_at + buf * BUFFER + q * PLANE + i * 256);
    }
    __device__ __forceinline__ void load(int set, int i, int k0) {
        const uint32_t o = KS && !GATHER ? voff[0] : voff[i];
        const uint32_t s = KS ? GATHER ? 0u : (uint32_t)(k0 + i) * pitch : (uint32_t)k0 * 4u;
        if constexpr (W == 4) v[set][i] = __builtin_bit_cast(load_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)o, (int)s, 0));
        else v[set][i] = __builtin_bit_cast(load_t, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)o, (int)s, 0));
    }
    // zeros for k >= K of block k0 (K contiguous)
    __device__ __forceinline__ void mask(int set, int k0, int K) {
        if constexpr (!KS) {
#pragma unroll
            for (int i = 0; i < NL; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (k0 + 4 * group() + q >= K) v[set][i][q] = 0.f;
        }
    }
    // zeros for columns past the edge (see BlockLoader::clear)
    static __device__ __forceinline__ bool ragged(int n0, int n) { return KS && n0 + R > n && n % W; }
    __device__ __forceinline__ void clear(int set, int n0, int n) {
        if constexpr (KS) {
            int at = W * line();
            asm volatile("" : "+v"(at));   // (computed again in every step: registers)
            const int valid = n - n0 - min(at, (n - n0 - 1) / W * W);
#pragma unroll
            for (int i = 0; i < NL; ++i)
#pragma unroll
                for (int q = 1; q < W; ++q)
                    if (q >= valid) v[set][i][q] = 0.f;
        }
    }
    // Piece P of splitting a set into the planes of buffer `set`: P / 7 is the row (K contiguous) or column (K strided), whose
    // four values are two pairs, taken in turn.
    float x[4];
    uint32_t w[2][3];
    template <bool NEG, int set, int P>
    __device__ __forceinline__ void piece(uint32_t& lost) {
        constexpr int i = P / 7, s = P % 7, h = s % 2;
        if constexpr (s < 4) {
            if constexpr (s < 2) {
                x[2 * h] = v[set][KS ? 2 * h : i][KS ? i : 2 * h];
                x[2 * h + 1] = v[set][KS ? 2 * h + 1 : i][KS ? i : 2 * h + 1];
            }
            w[h][s / 2] = split_off<NEG && s < 2>(x[2 * h], x[2 * h + 1]);
        } else if constexpr (s < 6) {
            w[h][2] = __builtin_amdgcn_perm(__float_as_uint(x[2 * h + 1]), __float_as_uint(x[2 * h]), 0x07060302u);
            lost |= __float_as_uint(x[2 * h]) | __float_as_uint(x[2 * h + 1]);
        } else {
#pragma unroll
            for (int q = 0; q < 3; ++q)
                *reinterpret_cast<uint2*>(put_at[KS ? i : 0] + set * BUFFER + q * PLANE + (KS ? 0 : i * 512)) = make_uint2(w[0][q], w[1][q]);
        }
    }
};

// f(0), f(1), ... as compile-time constants
template <typename F, int... I>
__device__ __forceinline__ void for_each_of(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
// (in assembly: the compiler would move sums between register files)
__device__ __forceinline__ void small_product(f32x4& c, bf16x8 fb, bf16x8 fa) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(fb), "v"(fa));
}
// (its user leaves four matrix instructions between)
__device__ __forceinline__ void large_product(f32x4& c, bf16x8 fb, bf16x8 fa) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(fb), "v"(fa));
}

constexpr int kWideLds = 2 * 3 * 64 * (128 + 64);   // two buffers of three planes of both operands
// RAGGED: the tile holds columns past the edge of a K-strided operand, which are cleared (see BlockLoader::clear)
template <int OP>
__device__ __forceinline__ bool wide_ragged(const TileArgs& a, const TilePlace& t) {
    constexpr bool TOKENS = OP == F32_WGRAD2 || OP == F32_WGRAD1;
    return WideOperand<TOKENS, false, 128>::ragged(t.m0, a.M) || WideOperand<TOKENS || OP == F32_FC2, false, 64>::ragged(t.n0, a.N);
}
template <int OP, bool RAGGED>
__device__ __forceinline__ void multiply_wide(const TileArgs& a, const TilePlace& t, uint8_t* smem, f32x4 (&acc)[4][2], uint32_t& lost) {
    static_assert(OP != F32_FC1, "fc1 takes no wide tiles");
    constexpr bool TOKENS = OP == F32_WGRAD2 || OP == F32_WGRAD1, GATHER = OP == F32_WGRAD1;
    constexpr bool A_KS = TOKENS, B_KS = TOKENS || OP == F32_FC2;
    int tid = (int)threadIdx.x;
    if constexpr (RAGGED) asm volatile("" : "+v"(tid));   // (the compiler would compute ahead for both variants together, and spill)
    const int wave = tid >> 6, nk = ceil_div(t.K, 32);    // at least two steps
    WideOperand<A_KS, GATHER, 128> oa(tid);
    WideOperand<B_KS, false, 64> ob(tid);
    oa.place(smem, (wave >> 1) * 64);
    ob.place(smem + 2 * oa.BUFFER, (wave & 1) * 32);
    const int group = oa.group(), row = oa.row();
    const DivideBy token((uint32_t)a.k);
    // WGRAD1: perm entries of the block whose offsets are computed next (past the end: zeros; see perm_end)
    __amdgpu_buffer_rsrc_t perm_rsrc;
    if constexpr (GATHER) perm_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.perm + t.kbeg), 0, t.K * 4, 0x00020000);
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 pv;
    const uint32_t col = oa.column(t.m0, a.M);
    auto perm_load = [&](int kb) __attribute__((always_inline)) {
        if constexpr (GATHER) pv = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(perm_rsrc, 16 * group, 128 * min(kb, nk - 1), 0));
    };
    auto perm_take = [&](int i) __attribute__((always_inline)) {
        if constexpr (GATHER) oa.voff[i] = token(pv[i]) * oa.pitch + col;
    };
    // block kb's rows past the end of the chunk: behind any range, so zeros
    auto perm_end = [&](int kb) __attribute__((always_inline)) {
        if constexpr (GATHER)
            if (kb + 1 >= nk && t.K % 32) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (32 * (nk - 1) + 4 * group + i >= t.K) oa.voff[i] = 0xfffffff0u;
            }
    };
    if constexpr (B_KS) {
        ob.pitch = (uint32_t)a.N * 4u;
        if constexpr (TOKENS) ob.resource(a.B + (size_t)t.kbeg * a.N, (size_t)t.K * a.N);
        else ob.resource(a.B + (size_t)t.e * a.K * a.N, (size_t)a.K * a.N);
        ob.voff[0] = (uint32_t)(4 * group) * ob.pitch + ob.column(t.n0, a.N);
    } else {
        ob.resource(a.B + (size_t)t.e * a.K * a.N, (size_t)a.K * a.N);
#pragma unroll
        for (int i = 0; i < 2; ++i) ob.voff[i] = (uint32_t)min(t.n0 + row + 32 * i, a.N - 1) * (uint32_t)a.K * 4u + 16u * group;
    }
    if constexpr (TOKENS) {
        oa.pitch = (uint32_t)a.M * 4u;
        if constexpr (GATHER) {
            oa.resource(a.A, (size_t)a.T * a.M);
        } else {
            oa.resource(a.A + (size_t)t.kbeg * a.M, (size_t)t.K * a.M);
            oa.voff[0] = (uint32_t)(4 * group) * oa.pitch + col;
        }
    } else {
        oa.resource(a.A + (size_t)t.m0 * a.K, (size_t)t.rows * a.K);
#pragma unroll
        for (int i = 0; i < 4; ++i)      // rows past the segment repeat its last one (their results are not stored)
            oa.voff[i] = (uint32_t)min(row + 32 * i, t.rows - 1) * (uint32_t)a.K * 4u + 16u * group;
    }
    auto take_and_load = [&](int set, int kb) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ob.NL; ++i) ob.load(set, i, 32 * min(kb, nk - 1));
#pragma unroll
        for (int i = 0; i < oa.NL; ++i) perm_take(i);
        perm_end(kb);
#pragma unroll
        for (int i = 0; i < oa.NL; ++i) oa.load(set, i, 32 * min(kb, nk - 1));
        perm_load(kb + 1);
    };
    perm_load(0);
    take_and_load(0, 0);
    take_and_load(1, 1);
    auto clear = [&](int set) __attribute__((always_inline)) {
        if constexpr (RAGGED) {
            oa.clear(set, t.m0, a.M);
            ob.clear(set, t.n0, a.N);
        }
    };
    clear(0);
    for_each_of([&](auto p) __attribute__((always_inline)) { oa.template piece<false, 0, decltype(p)::value>(lost); }, std::make_integer_sequence<int, oa.PIECES>{});
    for_each_of([&](auto p) __attribute__((always_inline)) { ob.template piece<false, 0, decltype(p)::value>(lost); }, std::make_integer_sequence<int, ob.PIECES>{});
    take_and_load(0, 2);
    __syncthreads();
    bf16x8 a1[4], a2[4], a3[4], b1[2], b2[2], b3[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) a3[i] = oa.frag(0, 2, i);
#pragma unroll
    for (int i = 0; i < 2; ++i) b1[i] = ob.frag(0, 0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) perm_take(i);
    perm_end(3);
    perm_load(4);
    f32x4 low[2][4][2];    // the small products of the even and of the odd steps, which have signs of their own
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) low[p][i][jj] = f32x4{0.f, 0.f, 0.f, 0.f};
    // multiplies block j, splits block j + 1, loads block j + 3
    auto step = [&](auto odd, int j) __attribute__((always_inline)) {
        constexpr bool ODD = decltype(odd)::value;
        constexpr int cur = ODD, nxt = !ODD;
        const int kb = min(j + 3, nk - 1);
        // (FC2: what A holds there is of the tile's own rows, and meets zeros.  The last step splits the last block once more)
        if constexpr (!A_KS && !B_KS) {
            if (j + 2 >= nk && t.K % 32) {
                oa.mask(nxt, 32 * (nk - 1), t.K);
                ob.mask(nxt, 32 * (nk - 1), t.K);
            }
        }
        clear(nxt);
        f32x4 hi[6];
        __builtin_amdgcn_sched_barrier(0);
        for_each_of([&](auto slot) __attribute__((always_inline)) {
            constexpr int m = decltype(slot)::value, prod = m / 8, r = m % 8, jj = r / 4, i = jj % 2 ? 3 - r % 4 : r % 4;
            if constexpr (prod == 0) small_product(low[cur][i][jj], b1[jj], a3[i]);
            else if constexpr (prod == 1) small_product(low[cur][i][jj], b1[jj], a2[i]);
            else if constexpr (prod == 2) small_product(low[cur][i][jj], b2[jj], a2[i]);
            else if constexpr (prod == 3) small_product(low[cur][i][jj], b2[jj], a1[i]);
            else if constexpr (prod == 4) large_product(hi[r % 6], b1[jj], a1[i]);
            else small_product(low[cur][i][jj], b3[jj], a1[i]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (m < 4) a2[m] = oa.frag(cur, 1, m);
            else if constexpr (m >= 6 && m < 10 && m % 2 == 0) b2[(m - 6) / 2] = ob.frag(cur, 1, (m - 6) / 2);
            else if constexpr (m >= 10 && m < 18 && m % 2 == 0) a1[(m - 10) / 2] = oa.frag(cur, 0, (m - 10) / 2);
            else if constexpr (m >= 18 && m < 22 && m % 2 == 0) b3[(m - 18) / 2] = ob.frag(cur, 2, (m - 18) / 2);
            if constexpr (m < oa.PIECES) oa.template piece<!ODD, nxt, m>(lost);
            else if constexpr (m < oa.PIECES + ob.PIECES) ob.template piece<false, nxt, m - oa.PIECES>(lost);
            // the loads of block j + 3, one at a time, into what has been split: a row of them fills the address queue, and the wavefront waits
            constexpr int la = A_KS ? m - 28 : m % 7 == 3 ? m / 7 : -1, lb = B_KS ? m - 42 : m == 31 ? 0 : m == 38 ? 1 : -1;
            if constexpr (la >= 0 && la < oa.NL) oa.load(nxt, la, 32 * kb);
            if constexpr (lb >= 0 && lb < ob.NL) ob.load(nxt, lb, 32 * kb);
            if constexpr (m >= 37 && m < 45) {     // the large products of five instructions ago
                constexpr int r5 = m - 37, j5 = r5 / 4, i5 = j5 % 2 ? 3 - r5 % 4 : r5 % 4;
                acc[i5][j5] = ODD ? acc[i5][j5] - hi[r5 % 6] : acc[i5][j5] + hi[r5 % 6];
            }
            if constexpr (GATHER) {
                if constexpr (m >= 34 && m < 38) perm_take(m - 34);
                if constexpr (m == 38) {
                    perm_end(j + 4);
                    perm_load(j + 5);
                }
            }
            if constexpr (m == 41) __syncthreads();
            if constexpr (m >= 42 && m < 46) a3[m - 42] = oa.frag(nxt, 2, m - 42);
            if constexpr (m == 42 || m == 45) b1[(m - 42) / 3] = ob.frag(nxt, 0, (m - 42) / 3);
            __builtin_amdgcn_sched_barrier(0);
        }, std::make_integer_sequence<int, 48>{});
    };
    int j = 0;
    for (;;) {
        step(std::false_type{}, j);
        if (++j >= nk) break;
        step(std::true_type{}, j);
        if (++j >= nk) break;
    }
    // (the compiler does not count the wait states that the results of the assembly's instructions need)
    asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            asm volatile("" : "+v"(low[0][i][jj]), "+v"(low[1][i][jj]));
            acc[i][jj] += low[0][i][jj] - low[1][i][jj];
        }
}

// One tile of contraction OP: 32 FM x 32 frag_cols(FM) outputs.  ESMM (Sec. 3.1 item 1; App. B Alg. 2) for
// the row GEMMs, whose rows are one expert's segment; ESTMM (item 3; Alg. 4) for the token contractions.
// BK: K-block of the fp32 instructions.
template <int FM, int BK, bool SPLIT>
constexpr int tile_bytes() {
    constexpr int f = 4 * f32_floats<FM, BK>(), s = FM == 4 ? kWideLds : SPLIT ? split_bytes<FM>() : 0;
    return f > s ? f : s;
}
// (what exceeds 64 KB is the launch's to ask for)
template <int FM, int BK, bool SPLIT>
__device__ __forceinline__ uint8_t* tile_lds() {
    if constexpr (tile_bytes<FM, BK, SPLIT>() > 65536) {
        extern __shared__ __align__(16) uint8_t dynamic_lds[];
        return dynamic_lds;
    } else {
        __shared__ __align__(16) uint8_t lds[tile_bytes<FM, BK, SPLIT>()];
        return lds;
    }
}
template <int FM, int BK, bool SPLIT>
constexpr int dynamic_bytes() { return tile_bytes<FM, BK, SPLIT>() > 65536 ? tile_bytes<FM, BK, SPLIT>() : 0; }
template <int FM, int BK, bool SPLIT, int OP, bool FAR>
__device__ __forceinline__ void f32_tile_of(const TileArgs& a, const int item, uint8_t* smem) {
    constexpr int BM = 32 * FM, FN = frag_cols(FM), BN = 32 * FN;
    constexpr bool TOKENS = OP == F32_WGRAD2 || OP == F32_WGRAD1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, grp = lane >> 4;

    // ---- which tile: an XCD takes a contiguous eighth of the row GEMM's tiles (column tiles fastest), or an
    // eighth of every chunk's tiles of a token contraction, so that its L2 holds what they share
    const int tn = ceil_div(a.N, BN);
    TilePlace t{};
    float* tok_out = nullptr;
    if constexpr (!TOKENS) {
        const int tiles = seg_tiles_total_wave(a.offsets, a.E, BM) * tn;
        const int per = ceil_div(tiles, kXcds), loc = item / kXcds;
        const int i = item % kXcds * per + loc;
        if (loc >= per || i >= tiles) return;
        t.row_tile = i / tn;
        const SegTile s = seg_tile_find_wave(a.offsets, a.E, BM, t.row_tile);
        t.e = s.e; t.m0 = s.row0; t.rows = s.rows; t.n0 = (i - t.row_tile * tn) * BN; t.K = a.K;
    } else {
        int tile;
        const int i = token_item_of(item, ceil_div(a.M, BM) * tn, tile);
        if (i < 0) return;
        const ChunkItem c = chunk_find_wave(a.offsets, a.E, a.chunk_len, i);
        if (c.e < 0) return;
        t.e = c.e; t.kbeg = c.beg; t.K = c.end - c.beg;
        t.m0 = (tile / tn) * BM; t.n0 = (tile % tn) * BN; t.rows = min(BM, a.M - t.m0);
        tok_out = c.slot >= 0 ? a.kpart + (size_t)c.slot * a.M * a.N : a.out0 + (size_t)t.e * a.M * a.N;
    }

    f32x4 acc[FM][FN];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    bool plain = true;
    if constexpr (SPLIT) if (t.K >= kSplitFrom) {
        uint32_t lost = 0;
        if constexpr (FM == 4) {
            if (!wide_ragged<OP>(a, t)) multiply_wide<OP, false>(a, t, smem, acc, lost);
            else multiply_wide<OP, true>(a, t, smem, acc, lost);
        }
        else multiply_split<FM, OP, FAR>(a, t, smem, acc, lost);
        // An infinity has no planes (inf - inf is NaN): a tile whose sums are not all finite is multiplied again on the fp32
        // instruction, too.
        float z = 0.f;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) z = fmaf(acc[i][j][r], 0.f, z);
        plain = __syncthreads_or(z != z || (lost & 0xffffu) != 0) != 0;
        if (plain) clear();
    }
    if (plain) multiply_f32<FM, BK, OP, FAR>(a, t, reinterpret_cast<float*>(smem), acc);

    // ---- epilogue
    float* out = TOKENS ? tok_out : a.out0;
#pragma unroll
    for (int jj = 0; jj < FN; ++jj) {
        const int n = t.n0 + 16 * (wn * FN + jj) + 4 * grp, nv = a.N - n;
        f32x4 bias = {0.f, 0.f, 0.f, 0.f}, cs = {0.f, 0.f, 0.f, 0.f};
        if constexpr (OP == F32_FC1 || OP == F32_FC2) bias = load4(a.bias + (size_t)t.e * a.N + n, nv);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int m = 16 * (wm * FM + i) + l16;
            if (m < t.rows && nv > 0) {
                const size_t oi = (size_t)(t.m0 + m) * a.N + n;
                f32x4 v = acc[i][jj] + bias;
                if constexpr (OP == F32_DGRAD2) {
                    const f32x4 u = load4(a.pre_in + oi, nv);
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] *= u[r];
                    cs += v;
                }
                if constexpr (OP == F32_FC1) {
                    f32x4 h;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float hr, gr;
                        act_both(v[r], a.act, hr, gr);
                        h[r] = hr; v[r] = gr;
                    }
                    store4(a.out1 + oi, h, nv);
                }
                store4(out + oi, v, nv);
            }
        }
        if constexpr (OP == F32_DGRAD2) {   // bias gradient (ESS, Table 5 row 8): this wave row's share of the column sums
#pragma unroll
            for (int r = 0; r < 4; ++r) cs[r] = row_sum16(cs[r]);
            if (l16 == 0) store4(a.colpart + (size_t)(2 * t.row_tile + wm) * a.N + n, cs, nv);
        }
    }
}

template <int FM, int BK, bool SPLIT, int OP>
__device__ __forceinline__ void f32_tile(const TileArgs& a, const int item, uint8_t* smem) {
    if constexpr (FM == 4) f32_tile_of<FM, BK, SPLIT, OP, false>(a, item, smem);   // (not for larger operands)
    else if (a.far) f32_tile_of<FM, BK, SPLIT, OP, true>(a, item, smem);
    else f32_tile_of<FM, BK, SPLIT, OP, false>(a, item, smem);
}
template <int FM, int BK, bool SPLIT, int OP>
__global__ __launch_bounds__(256, FM == 4 ? 2 : SPLIT ? 4 : 1) void f32_gemm(TileArgs a) {
    uint8_t* const smem = tile_lds<FM, BK, SPLIT>();
    f32_tile<FM, BK, SPLIT, OP>(a, (int)blockIdx.x, smem);
}

// Input gradient (OPA) and weight gradient (OPB) of one linear layer in one grid: neither needs the other's result, and
// the tail of one fills with tiles of the other.  Workgroups start in order; the one with the longer tiles comes first
// (b_first: OPB in slots [0, items), else OPA).
template <int FM, int BK, bool SPLIT, int OPA, int OPB>
__global__ __launch_bounds__(256, FM == 4 ? 2 : SPLIT ? 4 : 1) void f32_gemm_pair(TileArgs ra, TileArgs rb, int items, int b_first) {
    uint8_t* const smem = tile_lds<FM, BK, SPLIT>();
    const int item = (int)blockIdx.x, local = item < items ? item : item - items;
    if ((item < items) != (b_first != 0)) f32_tile<FM, BK, SPLIT, OPA>(ra, local, smem);
    else f32_tile<FM, BK, SPLIT, OPB>(rb, local, smem);
}

int tile_cols(int bm) { return bm < 64 ? bm : 64; }
int row_items(const MoeDims& D, int bm, int N) {
    return kXcds * ceil_div((D.A / bm + D.E) * ceil_div(N, tile_cols(bm)), kXcds);
}
// M x N: an expert's weight gradient
int token_items(const MoeDims& D, int bm, int M, int N) {
    return kXcds * ceil_div(ceil_div(M, bm) * ceil_div(N, tile_cols(bm)), kXcds) * (D.A / f32_chunk_len(D) + D.E);
}

// Which class a launch takes: 64x64 tiles fetch half as much per FLOP and multiply in planes, 32x32 tiles are four times as many and
// waste less at the ends of segments.  The line is where a row GEMM has 700 of the larger tiles, not quite three
// per CU; measured on both sides (us, 64x64 / 32x32), d = 384, f = 1536, 8 experts, top-2: fc1 91 / 107 at 4096 tokens
// (3264 tiles), 34 / 34 at 1024 (960), 24 / 23 at 512 (576), 23 / 17 at 256 (384); fc2 89 / 97 at 4096 (816), 54 / 56 at 2048 (432),
// 43 / 35 at 1024 (240).  A backward grid takes its row GEMM's class; by itself it would take 64x64 tiles earlier (bwd_fc1 at 2048
// tokens 91 / 106) and for the narrowest layers not at all (bwd_fc2 at 100000 x 4 x 4 of 4, 1566 tiles, 36 / 24).
bool small_rows(const MoeDims& D, int N) {
    return (long long)(D.A / 64 + D.E) * ceil_div(N, 64) < 700;
}

// K-blocks of 32x32 tiles: 64 means half as many barriers, 32 half of LDS, eight workgroups on a CU instead of four, which is worth
// more once there are tiles for them.  Measured, us, 64 / 32: bwd_fc2 at 1001 x 90 x 362 of 5 (1140 tiles) 18.3 / 13.9, bwd_fc1 at 512
// x 512 x 2048 of 16 110 / 85, fc2 at 8192 x 256 x 301 of 2 (2064) 25.7 / 22.8; fc2 at 1024 x 384 x 1536 of 8 (864) 38.5 / 39.5.
bool short_blocks(int tiles) { return tiles > 4 * 256; }

// Whether a tile's operands (x, an expert's weights, a chunk's or a tile's rows) lie beyond what 32-bit byte offsets reach.
bool far_operands(const MoeDims& D) {
    constexpr long long most = 0xffff0000LL;
    const long long chunk = 9LL * f32_chunk_len(D) / 8 + 256, wider = D.d > D.f ? D.d : D.f;
    return 4LL * D.T * D.d > most || 4LL * D.d * D.f + 256 * wider > most || 4 * chunk * wider > most;
}
// Planes on 128x64 tiles, two workgroups per CU, or on 64x64, four.  Wide tiles split and fetch less per product, and that is worth more the
// longer the contraction; against it stand the rows that an expert's last tile pads (64 on average instead of 32) and a start and an epilogue that
// are hidden under one other workgroup's K loop instead of three.  So the line lies at the length K and, for the padding, at the
// rows per expert n: 1024, or 512 where K is 1536.  Measured on both sides, us, 64x64 / 128x64 (tokens = rows, d x f of experts):
//   fc2 (K = f): 8192 rows, 384 x 1536 of 8 (n = 1024) 92 / 86, 8192 x 640 x 640 of 4 62 / 59, 4096 x 768 x 3072 of 8 (n = 512) 176 / 160, 4096 x 1024 x
//     1024 of 8 (n = 512) 83 / 85, 4096 x 1024 x 2048 of 16 (n = 256) 165 / 168, 3000 x 768 x 768 of 64 (n = 47) 52 / 79; one column of tiles,
//     whose A nothing else reads: 300000 x 64 x 600 of 4 263 / 270.
//   bwd_fc1 (K = f) at the same: 164 / 151, 117 / 114, 310 / 302, 147 / 146, 298 / 310, 117 / 158.
//   bwd_fc2 (K = d, long epilogue: from 1024): 4096 rows of 4, 1536 x 1536 302 / 285, 2048 x 2048 511 / 489, 8192 x 1024 x 2048 of 8 521 / 493; 8192 x
//     640 x 640 of 4 112 / 114, 5000 top-2 x 600 x 1000 of 9 206 / 213, 4096 x 768 x 3072 of 8 306 / 306.
//   fc1 (K = d, epilogue longer yet): 4096 top-2 x 576 x 2304 of 8 186 / 193, 4096 x 1024 x 1024 of 8 90 / 94, 8192 x 1024 x 2048 of 8 271 / 269, 4096 x 2048 x 2048 of
//     4 274 / 267, 2048 x 4096 x 1024 of 4 184 / 182: stays on 64x64.
// A backward grid's token contraction takes the same tiles: its chunks have to be as long, and its M must not pad much on 128 rows (bwd_fc1 at 300000 x 64 x
// 600 of 4 508 / 729, at 16384 x 576 x 576 of 2 180 / 184).
constexpr int kWideFrom = 576;
bool wide_rows(const MoeDims& D, int K) {
    const int n = D.A / std::min(D.E, D.A);
    return n >= (K >= 1536 ? 512 : 1024) && K >= kWideFrom && !far_operands(D);
}
bool wide_tokens(const MoeDims& D, int M) {
    const int half = ceil_div(M, 64), padded = 2 * ceil_div(M, 128);
    return f32_chunk_len(D) >= 512 && 16 * (padded - half) <= half;
}
// what the launches run on.  32: fp32 instruction, 64: planes, 128: planes on wide tiles
int fc1_class(const MoeDims& D) { return small_rows(D, D.f) ? 32 : 64; }
int fc2_class(const MoeDims& D) { return small_rows(D, D.d) ? 32 : wide_rows(D, D.f) && D.d > 64 ? 128 : 64; }
int bwd_fc2_class(const MoeDims& D) { return small_rows(D, D.f) ? 32 : D.d >= 1024 && wide_rows(D, D.d) && wide_tokens(D, D.f) ? 128 : 64; }
int bwd_fc1_class(const MoeDims& D) { return small_rows(D, D.d) ? 32 : wide_rows(D, D.f) && wide_tokens(D, D.d) ? 128 : 64; }

template <int FM, int BK, bool SPLIT, int OP>
void rows_launch_as(int grid, const TileArgs& a, hipStream_t st) {
    hipLaunchKernelGGL((f32_gemm<FM, BK, SPLIT, OP>), dim3(grid), dim3(256), (dynamic_bytes<FM, BK, SPLIT>()), st, a);
}
template <int OP>
void rows_launch(const MoeDims& D, int c, const TileArgs& a, hipStream_t st, const char* label) {
    const int grid = row_items(D, c, a.N);
    ProfScope ps(st, label);
    if constexpr (OP == F32_FC2)
        if (c == 128) return rows_launch_as<4, 16, true, OP>(grid, a, st);
    if (c == 64) rows_launch_as<2, 16, true, OP>(grid, a, st);
    else if (short_blocks(grid)) rows_launch_as<1, 32, false, OP>(grid, a, st);
    else rows_launch_as<1, 64, false, OP>(grid, a, st);
}
template <int FM, int BK, bool SPLIT, int OPA, int OPB>
void pair_launch_as(int grid, const TileArgs& ra, const TileArgs& rb, int items, bool b_first, hipStream_t st) {
    hipLaunchKernelGGL((f32_gemm_pair<FM, BK, SPLIT, OPA, OPB>), dim3(grid), dim3(256), (dynamic_bytes<FM, BK, SPLIT>()), st, ra, rb, items,
                       (int)b_first);
}
template <int OPA, int OPB>
void pair_launch(const MoeDims& D, int c, const TileArgs& ra, const TileArgs& rb, hipStream_t st, const char* label) {
    const int items_a = row_items(D, c, ra.N), items_b = token_items(D, c, rb.M, rb.N), grid = items_a + items_b;
    // rows of a token contraction's tile on average (the host does not know the routing), against K of a row GEMM's.  bwd_fc2 at
    // 4096 x 384 x 1536 of 8 (1024 against 384): row GEMM first 195 us, token contraction first 191 (on a machine 2 % slower)
    const long long rows = D.A / (D.E < D.A ? D.E : D.A), chunk = f32_chunk_len(D);
    const bool b_first = (rows < chunk ? rows : chunk) > ra.K;
    const int items = b_first ? items_b : items_a;
    ProfScope ps(st, label);
    if (c == 128) pair_launch_as<4, 16, true, OPA, OPB>(grid, ra, rb, items, b_first, st);
    else if (c == 64) pair_launch_as<2, 16, true, OPA, OPB>(grid, ra, rb, items, b_first, st);
    else if (short_blocks(grid)) pair_launch_as<1, 32, false, OPA, OPB>(grid, ra, rb, items, b_first, st);
    else pair_launch_as<1, 64, false, OPA, OPB>(grid, ra, rb, items, b_first, st);
}

template <typename KERNEL>
hipError_t allow_wide(KERNEL* kern) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, dynamic_bytes<4, 16, true>());
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
// (32 or 64: what a tile is multiplied with; wide tiles: see f32_wide)
void f32_tile_classes(const MoeDims& D, int (&tile)[4]) {
    tile[0] = tile[2] = small_rows(D, D.f) ? 32 : 64;
    tile[1] = tile[3] = small_rows(D, D.d) ? 32 : 64;
}
void f32_wide(const MoeDims& D, bool (&wide)[4]) {
    wide[0] = false;
    wide[1] = fc2_class(D) == 128;
    wide[2] = bwd_fc2_class(D) == 128;
    wide[3] = bwd_fc1_class(D) == 128;
}
int f32_dgrad2_row_tile(const MoeDims& D) { return bwd_fc2_class(D); }
hipError_t f32_device_init() {
    hipError_t e = allow_wide(f32_gemm<4, 16, true, F32_FC2>);
    if (e == hipSuccess) e = allow_wide(f32_gemm_pair<4, 16, true, F32_DGRAD2, F32_WGRAD2>);
    if (e == hipSuccess) e = allow_wide(f32_gemm_pair<4, 16, true, F32_DGRAD1, F32_WGRAD1>);
    return e;
}

hipError_t launch_f32_fwd(const MoeDims& D, const float* x, const float* W1, const float* b1,
                          const float* W2, const float* b2, const hexa_moe_idx& idx,
                          const MoeWorkspace& ws, hipStream_t st) {
    TileArgs a{};
    a.offsets = idx.offsets; a.perm = idx.perm; a.k = D.k; a.E = D.E; a.act = D.act; a.T = D.T; a.far = far_operands(D);
    // fc1: pre = x W1 + b1, h = F(pre), F'(pre)
    a.A = x; a.B = W1; a.bias = b1; a.out0 = (float*)ws.pre; a.out1 = (float*)ws.h; a.K = D.d; a.N = D.f;
    rows_launch<F32_FC1>(D, fc1_class(D), a, st, "fc1");
    // fc2: o = h W2 + b2
    a.A = (const float*)ws.h; a.B = W2; a.bias = b2; a.out0 = (float*)ws.o; a.out1 = nullptr; a.K = D.f; a.N = D.d;
    rows_launch<F32_FC2>(D, fc2_class(D), a, st, "fc2");
    return hipGetLastError();
}

hipError_t launch_f32_bwd(const MoeDims& D, const float* x, const float* W1, const float* W2,
                          const hexa_moe_idx& idx, const MoeWorkspace& ws, float* dW1, float* dW2,
                          hipStream_t st) {
    TileArgs g{};
    g.offsets = idx.offsets; g.perm = idx.perm; g.k = D.k; g.E = D.E; g.act = D.act; g.T = D.T; g.far = far_operands(D); g.chunk_len = f32_chunk_len(D);
    // 2nd linear layer: dpre = (do W2^T) * F'(pre)  and  dW2[e] = h^T do
    TileArgs r = g, t = g;
    r.A = (const float*)ws.dout; r.B = W2; r.pre_in = (const float*)ws.pre; r.out0 = (float*)ws.dpre;
    r.colpart = ws.colpart1; r.K = D.d; r.N = D.f;
    t.A = (const float*)ws.h; t.B = (const float*)ws.dout; t.out0 = dW2; t.kpart = ws.kpart2; t.M = D.f; t.N = D.d;
    pair_launch<F32_DGRAD2, F32_WGRAD2>(D, bwd_fc2_class(D), r, t, st, "bwd_fc2");
    // 1st linear layer: dxp = dpre W1^T  and  dW1[e] = x[perm/k]^T dpre
    r = g; t = g;
    r.A = (const float*)ws.dpre; r.B = W1; r.out0 = (float*)ws.dxp; r.K = D.f; r.N = D.d;
    t.A = x; t.B = (const float*)ws.dpre; t.out0 = dW1; t.kpart = ws.kpart1; t.M = D.d; t.N = D.f;
    pair_launch<F32_DGRAD1, F32_WGRAD1>(D, bwd_fc1_class(D), r, t, st, "bwd_fc1");
    return hipGetLastError();
}
