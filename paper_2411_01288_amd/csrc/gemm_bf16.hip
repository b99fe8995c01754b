// bf16 MFMA contractions of the expert-specific MoE layer (HEXA-MoE Sec. 3.1; App. B Table 5).
//
// Six contractions share one tile routine (forward: one grid each; backward: the input-gradient
// and weight-gradient contractions of a linear layer share a grid):
//   row GEMMs  (ESMM, App. B Alg. 2): rows are one expert segment of the re-index vector
//       FC1     pre = x[perm/k] W1[e] + b1[e],  h = F(pre), g = F'(pre) saved        K = d, N = f
//       FC2     o   = h W2[e] + b2[e]   (stored as bf16)                 K = f, N = d
//       DGRAD2  dpre = (do W2[e]^T) * g                              K = d, N = f
//       DGRAD1  dxp = dpre W1[e]^T      (stored as bf16)                 K = f, N = d
//   token contractions (ESTMM, App. B Alg. 4): the sum runs over one expert's rows
//       WGRAD2  dW2[e] = h^T do                                      M = f, N = d
//       WGRAD1  dW1[e] = x[perm/k]^T dpre  (token rows gathered)      M = d, N = f
//
// What is kept from the paper: rows of a tile all belong to one expert, so a tile needs one
// expert's weights; rows are addressed through the re-index vector, so nothing is padded to a
// capacity and nothing is dropped.  What is not: the 16x16x16 warp tiles, the per-expert serial
// loop of Alg. 4 and the padded (-1) re-index vector.  Here a workgroup owns a 256x256 or (small
// problems) a 128x128 tile, each 64-lane wavefront a grid of 16x16x32 bf16 MFMA blocks, operands go from
// global memory straight into LDS (no registers in between) as [row][64 k] with a 16-byte XOR
// swizzle (conflict-free 128-bit reads); operands whose contraction index is the slow one in
// memory (weights in the forward GEMMs, both operands of the token contractions) keep their
// memory layout in LDS and are transposed by the LDS read instruction; segments are tiled
// individually (ragged tails are masked, not padded), long segments of the token contractions
// are split into chunks whose partial tiles are reduced in a fixed order, and workgroup ids are
// remapped so that the 32 CUs of one XCD work on neighbouring tiles.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "deal.h"
#include "worklists.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vector: stays in registers
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kNumCUs = kXcds * kCusPerXcd;
constexpr int BK = 64;            // contraction elements per block of the K loop (one 128-byte line per row)
constexpr int NSLOT = 5;          // LDS ring: five slots (of the larger tile), each holds one operand's share of a block

// (OP_FC2P: a share of FC2's contraction, unrounded, the first one with the bias; see choose_fc2_shares)
enum Op { OP_FC1 = 0, OP_FC2, OP_DGRAD2, OP_DGRAD1, OP_WGRAD2, OP_WGRAD1, OP_FC2P };

struct GemmArgs {
    const bf16_t* A;      // row GEMM: [rows][K] (rows = tokens when gather, else perm positions)
                          // token contraction: [A][M] perm order
    const bf16_t* B;      // row GEMM: weights [E][..]; token contraction: [A][N] perm order
    const int32_t* perm;  // FC1 gather
    const uint32_t* rowoff;  // WGRAD1 gather: byte offsets of the token rows, written by the backward prologue
    const int32_t* offsets;
    const bf16_t* bias;   // [E][N] (FC1, FC2, FC2P)
    const bf16_t* pre_in; // DGRAD2: the saved GELU'(pre)
    void* out0;
    void* out1;
    float* kpart;         // split-K slots [slot][M][N]
    float* colpart;       // DGRAD2: per (row tile, wave row) column sums of dpre [2*tiles][N]
    int topk, E, K, N, M;
    int a_rows;           // FC1, WGRAD1: rows of the gathered operand (tokens T); FC2P: rows of the output
    int chunk_len;        // token contraction: tokens per work item that are aimed at (see chunk_count)
    int share;            // FC2P: number of this share of K, and 64-k blocks per share
    int share_blocks;
    int streamed;         // 128x128 tiles of a forward pass: large weights, less than a tile of rows per expert (see RowTiles)
    int token_first;      // 256x256 tiles of a backward grid: see token_first()
    const int32_t* lists; // 256x256 tiles: the work lists (see build_worklists)
    int rt_cap;           // their capacity in row tiles
};

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// s = 1 / (1 + exp(-2 t)),  t = sqrt(2/pi) (u + 0.044715 u^3):  tanh(t) = 2 s - 1, GELU(u) = u s.
// exp(-2 t) = 2^(u (k1 + k3 u^2)) with -log2(e) folded into the two constants.
// h = GELU(u) = u s and g = GELU'(u) = s + u s (1 - s) 2C (1 + 3 A u^2) from one s: eight
// full-rate operations and two transcendental ones
// (App. B Table 5 rows 2 and 7 need both; the forward epilogue has u in registers, so it saves g
// for the backward pass instead of u itself: same bytes, and the backward epilogue is one multiply).
__device__ __forceinline__ void gelu_both(float u, float& h, float& g) {
    constexpr float k1 = -2.f * HEXA_GELU_C * 1.4426950408889634f;
    constexpr float k3 = k1 * HEXA_GELU_A;
    const float u2 = u * u;
    const float s = fast_rcp(1.f + fast_exp2(u * (k1 + k3 * u2)));
    h = u * s;
    const float q = 2.f * HEXA_GELU_C + 6.f * HEXA_GELU_C * HEXA_GELU_A * u2;
    g = s + (h - h * s) * q;
}

// The same pair for the other activations: ReLU (derivative 0 at 0) and SiLU u s(u), s = 1/(1+e^-u),
// with derivative s (1 + u (1 - s)).
template <int ACT>
__device__ __forceinline__ void act_both(float u, float& h, float& g) {
    if constexpr (ACT == HEXA_ACT_RELU) {
        h = u > 0.f ? u : 0.f;
        g = u > 0.f ? 1.f : 0.f;
    } else if constexpr (ACT == HEXA_ACT_SILU) {
        const float sg = fast_rcp(1.f + fast_exp2(-1.4426950408889634f * u));
        h = u * sg;
        g = sg * (1.f + u * (1.f - sg));
    } else {
        gelu_both(u, h, g);
    }
}

// LDS image of a K-contiguous operand: row r = BK*2 = 128 bytes = CPRK chunks of 16 bytes (8 bf16
// along k); chunk c of row r sits at position c ^ key(r).  gfx950's LDS serves 128-bit reads 16 lanes
// (256 bytes, 64 banks) per clock; a 16x16x32 fragment read has 16 consecutive lanes on 16
// consecutive rows with one chunk index.  Two consecutive 128-byte rows fill the 256 bytes of bank
// space, so rows r, r+2, ..., r+14 must sit on eight different chunk positions:
// key(r) = (r >> 1) & 7.
constexpr int CPRK = BK * 2 / 16;                 // chunks per row
constexpr int ROWB = BK * 2;                      // bytes per row
static_assert(BK == 64, "the K loop and the swizzle are written for 64-element blocks");
__device__ __forceinline__ uint32_t lds_swz(int row) { return (uint32_t)((row >> 1) & 7); }

// ---------------------------------------------------------------------------------------------
// Operand staging: global -> LDS without passing through registers.
//
// gfx950 can write a 16-byte-per-lane buffer load straight into LDS ("buffer_load_dwordx4 ... lds"):
// the 64 lanes of one instruction fill 1024 consecutive LDS bytes in lane order, each lane
// fetching from its own global address.  LDS stores from registers run at ~64 B/clk/CU on this
// part, half of what a 256x256 tile needs at the MFMA rate, and cost 128 VGPRs per stage; the
// direct path costs neither.  Because the LDS position of a lane is fixed, the bank swizzle is
// applied on the global side: a lane fetches the chunk that belongs at its position.
//
// Reads past the byte range of the buffer resource return zero, which masks ragged row tails and
// the K tail of the token contractions for free.
// ---------------------------------------------------------------------------------------------
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef i32x4 rsrc_t;   // raw buffer resource: base[47:0], stride 0, byte range, gfx9 data format word
typedef __attribute__((address_space(3))) void* lds_void_t;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    // all four words are wave-uniform; say so, the staging instruction wants them in SGPRs
    const uint64_t b = (uint64_t)base;
    return rsrc_t{__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)b),
                  __builtin_amdgcn_readfirstlane((int32_t)((uint32_t)(b >> 32) & 0xffffu)),
                  __builtin_amdgcn_readfirstlane((int32_t)bytes), 0x00020000};
}
// one instruction: lane l's 16 bytes at (voff + soff) land at lds + 16*l; lds is wave-uniform.
// Written as inline assembly on purpose: the compiler then neither tracks these loads in vmcnt nor
// assumes that every later LDS read may alias them (which made it wait for the whole stage in
// front of each fragment read).  The kernel counts its own requests and waits explicitly (one
// "s_waitcnt vmcnt(n)" in front of the barrier that publishes a block, n = the requests that may
// still be in flight); the only other vector-memory loads inside the K loop are the row-offset
// loads of the gathered token contraction, inline assembly too and counted with them.  M0 carries
// the LDS address (one wait state before the load reads it).
__device__ __forceinline__ void dtl16(rsrc_t r, uint8_t* lds, uint32_t voff, uint32_t soff) {
    const uint32_t lds_addr = __builtin_amdgcn_readfirstlane(
        (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)lds);
    soff = __builtin_amdgcn_readfirstlane(soff);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(r), "s"(soff)
                 : "memory", "m0");
}

// The same in two parts for the K loop, where the instructions of a staging request are spread over
// two issue slots: the LDS address (an integer byte address, wave-uniform) goes into M0 in one slot,
// the load follows in the next one (an MFMA in between provides the wait state).  Nothing else in the
// K loop uses M0.
__device__ __forceinline__ void dtl_m0(uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0" : : "s"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory", "m0");
}
__device__ __forceinline__ void dtl_load(rsrc_t r, uint32_t voff, uint32_t soff) {
    asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds"
                 :
                 : "v"(voff), "s"(r), "s"(__builtin_amdgcn_readfirstlane(soff))
                 : "memory");
}

// A 16-byte-per-lane store to (voff + soff) of a buffer resource.  The hardware fetches the data of a
// store of more than 8 bytes over the cycles behind its issue: a vector instruction that overwrites one of
// its data registers within two wait states changes what is stored.  The compiler leaves that gap only
// where the scalar offset is no register, which is not enough on gfx950: with two wavefronts on a SIMD the
// first word of a 16-byte chunk was lost here and there.  So the gap is part of the statement.
__device__ __forceinline__ void buf_store16(u32x4 data, rsrc_t r, int voff, int soff) {
    asm volatile("buffer_store_dwordx4 %0, %1, %2, %3 offen\n\ts_nop 1"
                 :
                 : "v"(data), "v"(voff), "s"(r), "s"(__builtin_amdgcn_readfirstlane(soff))
                 : "memory");
}

// K-contiguous operand (R rows x BK k, ROWB bytes per row in memory order along k).
// Instruction q (= wave + NW*i) fills RPQ = 1024/ROWB rows: lane l -> row RPQ*q + l/CPRK,
// position l%CPRK.
template <int R, int NW, bool GATHER>
struct StageKC {
    static constexpr int RPQ = 1024 / ROWB;      // rows per instruction
    static constexpr int CPR = CPRK;             // lanes per row
    static_assert(RPQ == 8, "one look-up per lane and staged row");
    static constexpr int NI = R / RPQ / NW;      // instructions per wave and stage
    static_assert(R % (RPQ * NW) == 0 && (RPQ * NW) % 16 == 0, "unsupported staging shape");
    // byte offset of (row, chunk) from the resource base: one per instruction when the rows are
    // gathered; otherwise instruction i is RPQ*NW*i rows further down, which goes into the scalar
    // offset
    struct Lane { uint32_t voff[GATHER ? NI : 1]; };
    // chunk this lane must fetch: its position XOR the swizzle key of its row (the key has period
    // 16 rows and RPQ*NW is a multiple of 16, so it is the same for every instruction of a wave)
    __device__ static __forceinline__ int lane_chunk(int wave, int lane) {
        return (lane % CPRK) ^ (int)lds_swz(RPQ * wave + lane / CPRK);
    }
    __device__ static __forceinline__ int lane_row(int wave, int lane, int i) {
        return RPQ * (wave + NW * i) + lane / CPRK;
    }
    // instruction i of this wave: set-up (LDS address of its 1 KB piece of the slot at lds_slot) and load
    __device__ static __forceinline__ void prep(uint32_t lds_slot, int wave, int i) {
        dtl_m0(lds_slot + (uint32_t)(wave + NW * i) * 1024u);
    }
    __device__ static __forceinline__ void load(rsrc_t r, uint32_t soff, uint32_t row_bytes, const Lane& ln, int i) {
        if constexpr (GATHER) dtl_load(r, ln.voff[i], soff);
        else dtl_load(r, ln.voff[0], soff + (uint32_t)(RPQ * NW * i) * row_bytes);
    }
};

// K-strided operand (BK k-rows x R columns, a k-row is R*2 contiguous bytes in memory).
// LDS image: k-row k at k*R*2, 16-byte chunk c (8 columns) at position c ^ ks_key(k).
// It is read with ds_read_b64_tr_b16, which hands each lane four k-values of one column; a
// 32-lane half of such a read touches k-rows {8a + j, 8(a+1) + j : j < 4}, 32 bytes (16 columns) of
// each, and the key puts those eight pieces on the eight 32-byte slots of the bank space.
// Instruction q fills k-rows RPI*q .. RPI*q + RPI-1 (RPI = 512 / R rows of R*2 bytes).
__device__ __forceinline__ int ks_key(int k) { return ((k & 3) << 2) | (((k >> 3) & 1) << 1); }

template <int R, int NW>
struct StageKS {
    static constexpr int RB = R * 2;            // bytes per k-row
    static constexpr int CPR = RB / 16;         // chunks per k-row
    static constexpr int RPI = 1024 / RB;       // k-rows per instruction
    static constexpr int NI = BK / RPI / NW;    // instructions per wave and block
    static constexpr int STEP = RPI * NW;       // k-rows from one instruction of a wave to its next one
    static_assert(RPI >= 1 && (BK / RPI) % NW == 0 && (STEP == 8 || STEP == 16) && CPR >= 16, "unsupported staging shape");
    // instruction i of a wave covers k-rows RPI*wave + kin + STEP i: (k & 3) is the same for all i and
    // ((k >> 3) & 1) too (STEP 16) or i & 1 (STEP 8), so a lane needs one offset or two (even and odd i)
    static constexpr int NV = STEP == 8 ? 2 : 1;
    struct Lane { uint32_t voff[NV]; };
    // (row_bytes = 0 when the k-rows are gathered: the row part of the offset then comes from a table)
    __device__ static __forceinline__ Lane lane_init(int wave, int lane, uint32_t row_bytes, int col0) {
        const int kin = lane / CPR;                          // k-row inside the instruction
        const int k = (RPI * wave + kin);                    // k-row of instruction i = 0  (< STEP)
        Lane ln;
#pragma unroll
        for (int odd = 0; odd < NV; ++odd) {
            const int c = (lane % CPR) ^ ks_key(k + 8 * odd);
            ln.voff[odd] = (uint32_t)k * row_bytes + (uint32_t)(col0 + 8 * c) * 2u;
        }
        return ln;
    }
    // gathered k-rows: instruction i fetches the rows whose byte offsets are roff[i] (per lane)
    __device__ static __forceinline__ void load_gathered(rsrc_t r, const uint32_t (&roff)[NI], const Lane& ln, int i) {
        dtl_load(r, roff[i] + ln.voff[i % NV], 0u);
    }
    __device__ static __forceinline__ void prep(uint32_t lds_slot, int wave, int i) {
        dtl_m0(lds_slot + (uint32_t)(wave + NW * i) * 1024u);
    }
    __device__ static __forceinline__ void load(rsrc_t r, uint32_t soff, uint32_t ld_bytes, const Lane& ln, int i) {
        dtl_load(r, ln.voff[i % NV], soff + (uint32_t)(STEP * i) * ld_bytes);
    }
};

// ---------------------------------------------------------------------------------------------
// Work decomposition
// ---------------------------------------------------------------------------------------------

// Which tile a workgroup works on follows from the segment offsets alone.  Rows are cut into tiles numbered
// expert-major (tiles never straddle experts; experts without rows have none); the items of a token contraction
// are numbered expert-major, then chunk (see chunk_count), with the number of the partial-tile
// buffer of an expert that was cut into several chunks (-1: one chunk, its tile goes straight to the output).
//
// 256x256 tiles take theirs from the work lists of worklists.h.

// 128x128 tiles are found by every wavefront for itself: a lane takes EPL consecutive experts, a scan over the
// lanes numbers their tiles, and all offsets arrive in one memory latency.  It costs a workgroup a few hundred
// instructions that the CU's second workgroup hides, and saves the launch that would build a list (5 us of a
// 70 us decode step; used for 256x256 tiles too it cost their contractions 1 to 3 %).
// What takes a division per expert (into how many chunks one is cut, and how long they are) is only asked where some expert is cut
// or long enough: with 16 experts per lane the divisions took every workgroup, also those without a tile, several us (bwd_fc2 of 49
// tokens, 64 x 3392 of 292, top-2: 217 -> 94 us; of 5261 tokens, 768 x 2496 of 126 342 -> 300).  With one expert per lane a division costs
// no more than the question whether it is needed.
template <int EPL>
struct ExpertLanes {
    int b[EPL + 1];                            // segment starts of this lane's experts, and the end of the last
    int most = 0;                              // rows of the largest of them
    __device__ __forceinline__ ExpertLanes(const int32_t* __restrict__ offsets, int E) {
        const int e0 = (int)(threadIdx.x & 63) * EPL;
#pragma unroll
        for (int q = 0; q <= EPL; ++q) b[q] = offsets[min(e0 + q, E)];
#pragma unroll
        for (int q = 0; q < EPL; ++q) most = max(most, b[q + 1] - b[q]);
    }
    __device__ __forceinline__ int total() const { return __builtin_amdgcn_readlane(b[EPL], 63); }   // rows of all experts
    // whether any expert makes several chunks (see chunk_count)
    __device__ __forceinline__ bool any_cut(int len) const { return __any(most - len / 8 > len) != 0; }
    // pieces of an expert of n rows: row tiles of `len` rows, or (CHUNKS) token-contraction items
    template <bool CHUNKS>
    __device__ static __forceinline__ int count(int n, int len, bool cut) {
        return CHUNKS ? cut ? chunk_count(n, len) : n > 0 : ceil_div(n, len);
    }
    // their number: inclusive scan over the lanes
    template <bool CHUNKS>
    __device__ __forceinline__ int pieces(int len, bool cut, int& mine) const {
        mine = 0;
        if (EPL > 1 && CHUNKS && !cut) {
#pragma unroll
            for (int q = 0; q < EPL; ++q) mine += count<CHUNKS>(b[q + 1] - b[q], len, false);
        } else {
#pragma unroll
            for (int q = 0; q < EPL; ++q) mine += count<CHUNKS>(b[q + 1] - b[q], len, true);
        }
        return wave_scan_incl(mine);
    }
    // whether the longest token-contraction item has `rows` rows or more
    __device__ __forceinline__ bool any_long(int len, bool cut, int rows) const {
        if (EPL > 1 ? __any(most >= rows) == 0 || !cut : !cut) return __any(most >= rows) != 0;
        int longest = 0;
#pragma unroll
        for (int q = 0; q < EPL; ++q) longest = max(longest, (b[q + 1] - b[q]) / max(chunk_count(b[q + 1] - b[q], len), 1));
        return __any(longest >= rows) != 0;
    }
    // piece number i (wave-uniform, below the total): expert, first row, end row, and (CHUNKS) the number of partial
    // buffers of the experts in front that have several pieces plus the piece's own (-1: the expert's only one)
    template <bool CHUNKS, bool CUT>
    __device__ __forceinline__ ChunkItem find(int i, int len, int incl, int mine) const {
        int slots = 0, slot = 0;
        if constexpr (CHUNKS && CUT) {
#pragma unroll
            for (int q = 0; q < EPL; ++q) {
                const int n = count<true>(b[q + 1] - b[q], len, true);
                slots += n > 1 ? n : 0;
            }
            slot = wave_scan_incl(slots) - slots;
        }
        int at = incl - mine;
        ChunkItem r{0, 0, 0, -1};
#pragma unroll
        for (int q = 0; q < EPL; ++q) {
            const int rows = b[q + 1] - b[q], n = count<CHUNKS>(rows, len, CUT), c = i - at;
            if (c >= 0 && c < n) {
                r.e = (int)(threadIdx.x & 63) * EPL + q;
                if constexpr (CHUNKS && !CUT) {
                    r.beg = b[q];
                    r.end = b[q + 1];
                } else {
                    r.beg = b[q] + (CHUNKS ? chunk_start(rows, n, c) : c * len);
                    r.end = CHUNKS ? b[q] + chunk_start(rows, n, c + 1) : min(b[q + 1], r.beg + len);
                    r.slot = n > 1 ? slot + c : -1;
                }
            }
            at += n;
            slot += n > 1 ? n : 0;
        }
        const int src = __ffsll((long long)__ballot(incl > i)) - 1;
        return ChunkItem{__builtin_amdgcn_readlane(r.e, src), __builtin_amdgcn_readlane(r.beg, src),
                         __builtin_amdgcn_readlane(r.end, src), __builtin_amdgcn_readlane(r.slot, src)};
    }
};

__device__ __forceinline__ ChunkItem list_entry(const int32_t* p) {
    const i32x4 v = *reinterpret_cast<const i32x4*>(p);
    return ChunkItem{v.x, v.y, v.z, v.w};
}

// A workgroup's tile: its segment rows (row GEMM: those of the row tile; token contraction: those that are summed over),
// and its place in the output.
struct Tile { ChunkItem it; int tile_m, tile_n; };

// A row GEMM on its own.  False: no tile.
template <int EPL, int BM, int BN>
__device__ __forceinline__ bool pick_rows_wave(const GemmArgs& g, int x, int loc, Tile& t) {
    const ExpertLanes<EPL> s(g.offsets, g.E);
    int mine;
    const int incl = s.template pieces<false>(BM, false, mine);
    const RowTiles<BM> rows(__builtin_amdgcn_readlane(incl, 63), ceil_div(g.N, BN), g.streamed != 0);
    if (loc >= rows.count(x)) return false;
    rows.tile(x, loc, t.tile_m, t.tile_n);
    t.it = s.template find<false, false>(t.tile_m, BM, incl, mine);
    return true;
}
template <int BM, int BN>
__device__ __forceinline__ bool pick_rows_small(const GemmArgs& g, int x, int loc, Tile& t) {
    return g.E <= 64 ? pick_rows_wave<1, BM, BN>(g, x, loc, t)
           : g.E <= 256 ? pick_rows_wave<4, BM, BN>(g, x, loc, t) : pick_rows_wave<16, BM, BN>(g, x, loc, t);
}
__device__ __forceinline__ bool pick_rows_big(const GemmArgs& g, int x, int loc, Tile& t, int& quarter) {
    const RowTiles<256> rows(g.lists[WL_TILES], ceil_div(g.N, 256), false);
    if (!tile_or_quarter(rows, x, loc, quarter)) return false;
    rows.tile(x, loc, t.tile_m, t.tile_n);
    t.it = list_entry(g.lists + kWlHeader + 4 * t.tile_m);
    return true;
}

// Row GEMM ga and token contraction gb in one grid.  0: no tile, 1: one of ga, 2: one of gb.  Workgroups start roughly
// in order, so the contraction with the longer tiles should come first.  256x256 tiles: the row GEMM, but the token
// contraction when routing is so skewed that one expert's chunk runs many times longer than a row-GEMM tile, eight times
// or more (with Zipf routing at C5's shape the largest expert's tiles run 1582 K-blocks against 32 or 128), or in a launch of a
// few rounds (token_first()).  128x128 tiles, of which a launch has a round or two: whichever has the longer ones on average, but the
// token contraction where its longest are twice as long (4096 x 384 x 1536 of 8, bwd_fc2: 38 -> 33 us; 3001 x 320 x 448 of 17 under
// Zipf routing, the step: 81.0 -> 80.1; by the longest item alone, 1146 x 576 x 2304 of 20 under Zipf routing, bwd_fc2: 48 -> 53).
__device__ __forceinline__ int pair_order(int na, int nb, bool b_first, int& loc) {
    const bool is_b = b_first ? loc < nb : loc >= na;
    if (is_b && !b_first) loc -= na;
    if (!is_b && b_first) loc -= nb;
    return is_b ? 2 : 1;
}
template <int EPL, int BM>
__device__ __forceinline__ int pick_pair_wave(const GemmArgs& ga, const GemmArgs& gb, int x, int loc, Tile& t) {
    const ExpertLanes<EPL> s(ga.offsets, ga.E);
    const bool cut = s.any_cut(gb.chunk_len);
    int rmine, cmine;
    const int rincl = s.template pieces<false>(BM, false, rmine), cincl = s.template pieces<true>(gb.chunk_len, cut, cmine);
    const RowTiles<BM> rows(__builtin_amdgcn_readlane(rincl, 63), ceil_div(ga.N, BM), false);
    const int tm = ceil_div(gb.M, BM), tn = ceil_div(gb.N, BM);
    const TokenTiles tok{tm * tn};
    const int items = __builtin_amdgcn_readlane(cincl, 63);
    // (the second: more than K rows on average, rounded down)
    const bool b_first = s.any_long(gb.chunk_len, cut, 2 * ga.K) || (long long)s.total() >= (ga.K + 1LL) * items;
    const int na = rows.count(x), nb = tok.count(x, items);
    if (loc >= na + nb) return 0;
    const int which = pair_order(na, nb, b_first, loc);
    if (which == 1) {
        rows.tile(x, loc, t.tile_m, t.tile_n);
        t.it = s.template find<false, false>(t.tile_m, BM, rincl, rmine);
    } else {
        int tile;
        const int i = tok.find(x, loc, tile);
        t.it = cut ? s.template find<true, true>(i, gb.chunk_len, cincl, cmine) : s.template find<true, false>(i, gb.chunk_len, cincl, cmine);
        grouped_tile<group_rows(BM)>(tile, tm, tn, t.tile_m, t.tile_n);
    }
    return which;
}
template <int BM>
__device__ __forceinline__ int pick_pair(const GemmArgs& ga, const GemmArgs& gb, int order, int x, int loc, Tile& t) {
    if constexpr (BM == 256) {
        const RowTiles<BM> rows(ga.lists[WL_TILES], ceil_div(ga.N, BM), false);
        const int tm = ceil_div(gb.M, BM), tn = ceil_div(gb.N, BM);
        const TokenTiles tok{tm * tn};
        const int na = rows.count(x), nb = tok.count(x, ga.lists[WL_ITEMS]);
        if (loc >= na + nb) return 0;
        const int which = pair_order(na, nb, ga.lists[order] != 0 || ga.token_first != 0, loc);
        if (which == 1) {
            rows.tile(x, loc, t.tile_m, t.tile_n);
            t.it = list_entry(ga.lists + kWlHeader + 4 * t.tile_m);
        } else {
            int tile;
            t.it = list_entry(ga.lists + kWlHeader + 4 * (ga.rt_cap + tok.find(x, loc, tile)));
            grouped_tile<group_rows(BM)>(tile, tm, tn, t.tile_m, t.tile_n);
        }
        return which;
    } else {
        return ga.E <= 64 ? pick_pair_wave<1, BM>(ga, gb, x, loc, t)
               : ga.E <= 256 ? pick_pair_wave<4, BM>(ga, gb, x, loc, t) : pick_pair_wave<16, BM>(ga, gb, x, loc, t);
    }
}

// ---------------------------------------------------------------------------------------------
// The kernel
// ---------------------------------------------------------------------------------------------
// One tile of contraction OP.
template <int BM, int BN, int WM, int WN, int OP, int ACT, bool F16, int DEPTH = 2>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, const Tile& t) {
    constexpr int NT = WM * WN * 64;
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / 16, FN = TN / 16;   // 16x16 MFMA blocks per wave tile
    constexpr bool TOKENS = (OP == OP_WGRAD2 || OP == OP_WGRAD1);
    constexpr bool B_KS = TOKENS || OP == OP_FC1 || OP == OP_FC2 || OP == OP_FC2P;
    constexpr bool A_GK = (OP == OP_WGRAD1);   // operand A's k-rows (tokens) are gathered rows of x
    constexpr int SLOT = (BM > BN ? BM : BN) * ROWB;   // bytes of one ring slot (one operand, one block)
    constexpr int SPS = BK / 32;              // k-substeps (one MFMA k = 32 each) per block
    static_assert(TM % 16 == 0 && TN % 16 == 0, "wave tile must be a multiple of 16x16");

    extern __shared__ __align__(1024) uint8_t smem[];   // the slot ring; reused by the epilogue

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int l16 = lane & 15, grp = lane >> 4;   // MFMA lane coordinates

    const int e = t.it.e, n0 = t.tile_n * BN;
    const int m0 = TOKENS ? t.tile_m * BM : t.it.beg;
    const int mvalid = TOKENS ? min(BM, g.M - m0) : t.it.end - t.it.beg;
    const int row_tile = t.tile_m;    // row GEMMs: number of this row tile over all segments
    int nk = g.K / BK;                // 64-element blocks of the contraction
    int kbeg = 0, kend = 0;           // token contraction: perm rows of this item; FC2P: first block of K
    float* tok_out = nullptr;         // token contraction: where the tile goes
    if constexpr (TOKENS) {
        kbeg = t.it.beg; kend = t.it.end;
        nk = ceil_div(kend - kbeg, BK);
        tok_out = (t.it.slot >= 0) ? g.kpart + (size_t)t.it.slot * g.M * g.N
                                   : reinterpret_cast<float*>(g.out0) + (size_t)e * g.M * g.N;
    }
    if constexpr (OP == OP_FC2P) {
        kbeg = g.share * g.share_blocks;            // (in blocks)
        nk = min(g.share_blocks, nk - kbeg);
    }
    const int nvalid = min(BN, g.N - n0);

    // ---- staging set-up -----------------------------------------------------------------------
    constexpr int NW = WM * WN;
    using SA = typename std::conditional<TOKENS, StageKS<BM, NW>, StageKC<BM, NW, OP == OP_FC1>>::type;
    using SB = typename std::conditional<B_KS, StageKS<BN, NW>, StageKC<BN, NW, false>>::type;
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    typename SA::Lane lna;
    typename SB::Lane lnb;
    rsrc_t ra, rb;
    uint32_t a_step, b_step;      // bytes one K-step advances each operand
    uint32_t a_ld = 0, b_ld = 0;  // row pitch in bytes of the K-strided operands
    if constexpr (!TOKENS) {
        // FC1 gathers token rows of x through the re-index vector; the other row GEMMs read
        // perm-ordered rows, and rows past the segment fall outside the resource (zeros)
        if constexpr (OP == OP_FC1) ra = make_rsrc(g.A, (uint32_t)g.a_rows * (uint32_t)g.K * 2u);
        else ra = make_rsrc(g.A + (size_t)m0 * g.K + kbeg * BK, (uint32_t)mvalid * (uint32_t)g.K * 2u - (uint32_t)(kbeg * BK) * 2u);
        a_step = BK * 2;
        const uint32_t ca = (uint32_t)SA::lane_chunk(uwave, lane) * 16u;
        if constexpr (OP == OP_FC1) {
            // a wavefront stages 8 NI rows: each lane looks up one (an eight-fold look-up with as many divisions
            // sits in front of every tile's first request) and hands it to the eight lanes that fetch it
            const int mine = SA::lane_row(uwave, lane % 8 * SA::CPR, lane / 8 % SA::NI);
            // (rows past the segment point behind the last row of x: the range check makes them zeros without a fetch)
            const uint32_t row = (uint32_t)(mine < mvalid ? g.perm[m0 + mine] / g.topk : g.a_rows) * (uint32_t)g.K * 2u;
#pragma unroll
            for (int i = 0; i < SA::NI; ++i) lna.voff[i] = (uint32_t)__shfl((int)row, 8 * i + lane / SA::CPR) + ca;
        } else {
            lna.voff[0] = (uint32_t)SA::lane_row(uwave, lane, 0) * (uint32_t)g.K * 2u + ca;
        }
        if constexpr (B_KS) {  // W[e][K][N]
            b_ld = (uint32_t)g.N * 2u;
            rb = make_rsrc(g.B + ((size_t)e * g.K + kbeg * BK) * g.N, (uint32_t)(g.K - kbeg * BK) * b_ld);
            b_step = BK * b_ld;
            lnb = SB::lane_init(uwave, lane, b_ld, n0);
        } else {               // W[e][N][K]: rows past N fall outside the resource
            rb = make_rsrc(g.B + ((size_t)e * g.N + n0) * g.K, (uint32_t)nvalid * (uint32_t)g.K * 2u);
            b_step = BK * 2;
            const uint32_t cb = (uint32_t)SB::lane_chunk(uwave, lane) * 16u;
            lnb.voff[0] = (uint32_t)SB::lane_row(uwave, lane, 0) * (uint32_t)g.K * 2u + cb;
        }
    } else {
        // both operands are [tokens][features] in perm order; tokens past this item's range fall
        // outside the resources
        // (WGRAD1: operand A is x itself, [tokens][M]; the row of perm position p comes from the
        // offset table, whose entries past a segment's end point behind the last row of x)
        a_ld = (uint32_t)g.M * 2u; b_ld = (uint32_t)g.N * 2u;
        if constexpr (A_GK) ra = make_rsrc(g.A, (uint32_t)g.a_rows * a_ld);
        else ra = make_rsrc(g.A + (size_t)kbeg * g.M, (uint32_t)(kend - kbeg) * a_ld);
        rb = make_rsrc(g.B + (size_t)kbeg * g.N, (uint32_t)(kend - kbeg) * b_ld);
        a_step = BK * a_ld; b_step = BK * b_ld;
        if constexpr (TOKENS) {
            lna = SA::lane_init(uwave, lane, A_GK ? 0u : a_ld, m0);
            lnb = SB::lane_init(uwave, lane, b_ld, n0);
        }
    }
    // staging instruction i_ of operand A / B for block kt_ into the ring slot at LDS byte address
    // slot_: set-up part (M0) and load part
    const uint32_t smem0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)smem;
    const uint32_t a_row = TOKENS ? a_ld : (uint32_t)g.K * 2u, b_row = B_KS ? b_ld : (uint32_t)g.K * 2u;
#define PREP_A(slot_, i_) SA::prep((slot_), uwave, i_)
#define PREP_B(slot_, i_) SB::prep((slot_), uwave, i_)
#define LOAD_A(kt_, i_)                                                                          \
    do {                                                                                         \
        if constexpr (A_GK) SA::load_gathered(ra, rcur, lna, i_);                                \
        else SA::load(ra, (kt_) * a_step, a_row, lna, i_);                                       \
    } while (0)
#define LOAD_B(kt_, i_) SB::load(rb, (kt_) * b_step, b_row, lnb, i_)

    // The bias values this lane adds in the epilogue (block j: columns j*16 + 4*grp + 0..3 of the
    // wave tile), fetched before the K loop: loaded in the epilogue they would be re-read after every
    // band's stores (which may alias them as far as the compiler knows), each time with the full
    // memory latency and nothing to hide it behind.  These plain loads are older than every staging
    // request, so the staging waits, which count from the youngest request back, cover them.
    u32x2 biasv[FN];
    if constexpr (OP == OP_FC1 || OP == OP_FC2 || OP == OP_FC2P) {
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int gc = min(n0 + wn * TN + j * 16 + 4 * grp, g.N - 4);   // masked columns read a valid bias
            biasv[j] = *reinterpret_cast<const u32x2*>(g.bias + (size_t)e * g.N + gc);
            if (OP == OP_FC2P && g.share > 0) biasv[j] = u32x2{0, 0};
        }
    }

    // ---- per-lane fragment addresses -----------------------------------------------------------
    // A 16x16x32 MFMA operand fragment: lane (l16, grp) holds k = 8*grp + 0..7 of row (or column) l16
    // of its 16-wide block.
    // K-contiguous image: one 128-bit read of row (block row + l16), chunk (4*sub + grp) ^ key(l16)
    // (wave-tile and block rows are multiples of 16, so key(row) = key(l16)).
    // K-strided image: two transposing 64-bit reads per fragment.  In a group of 16 lanes, lane s
    // addresses k-row (s >> 2) and columns 4*(s & 3).., and receives column s of the block's 16,
    // k-rows 0..3; group grp reads k-rows 32*sub + 8*grp + 4*half + 0..3 (see StageKS).
    constexpr int A_RB = BM * 2, B_RB = BN * 2;  // LDS k-row pitch of the K-strided images
    // KC: aoff[sub] = byte offset of this lane's chunk in block row 0.
    // KS: one lane constant a_l0: k-row part | within-chunk byte | (chunk of block 0 ^ key) << 4.
    // Block q's chunk index differs from block 0's in the bits of 2q only (the wave tile's first chunk is a
    // multiple of the 2 FM or 2 FN chunks of a wave tile), so its offset is a_l0 ^ (q << 5); the k-row of (substep, half) is an immediate.
    uint32_t aoff[SPS], boff[SPS];
    uint32_t a_l0 = 0, b_l0 = 0;
    {
        const int krel = l16 >> 2, pair = (l16 & 3) >> 1, half8 = (l16 & 1) * 8;
        const int key = ks_key(8 * grp + krel);  // the key of every k-row this lane reads
        static_assert(A_RB % 256 == 0 && B_RB % 256 == 0 && TM % 64 == 0 && TN % 64 == 0 && TM / 8 >= 2 * FM && TN / 8 >= 2 * FN,
                      "bit fields of the K-strided fragment offset");
        if constexpr (TOKENS) {
            a_l0 = (uint32_t)((8 * grp + krel) * A_RB + half8 + ((((wm * TM) / 8 + pair) ^ key) << 4));
        } else {
#pragma unroll
            for (int sb = 0; sb < SPS; ++sb)
                aoff[sb] = (uint32_t)((wm * TM + l16) * ROWB) + (uint32_t)(((4 * sb + grp) ^ lds_swz(l16)) << 4);
        }
        if constexpr (B_KS) {
            b_l0 = (uint32_t)((8 * grp + krel) * B_RB + half8 + ((((wn * TN) / 8 + pair) ^ key) << 4));
        } else {
#pragma unroll
            for (int sb = 0; sb < SPS; ++sb)
                boff[sb] = (uint32_t)((wn * TN + l16) * ROWB) + (uint32_t)(((4 * sb + grp) ^ lds_swz(l16)) << 4);
        }
    }

    // two fragment sets: one is multiplied while the other one is being read (a read never targets
    // registers an MFMA in flight may still be reading)
    bf16x8 fa0[FM], fb0[FN], fa1[FM], fb1[FN];
#define FENCE() __builtin_amdgcn_sched_barrier(0)
#define TR_READ(p_) __builtin_bit_cast(s16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p_)))
#define TR_JOIN(lo_, p_) __builtin_bit_cast(bf16x8, __builtin_shufflevector((lo_), TR_READ(p_), 0, 1, 2, 3, 4, 5, 6, 7))
    // The MFMAs of a substep run B-fragment-major (MFMA m: B fragment m / FM, the A fragments up and down in turn),
    // so the next substep needs B fragment 0 and every A fragment first: its LDS reads are numbered
    // B0, A0 .. A(FM-1), B1 .. B(FN-1); a K-strided fragment takes two reads (k-rows +0..3 and
    // +4..7), a K-contiguous one takes one.
    constexpr int RA = TOKENS ? 2 : 1, RBn = B_KS ? 2 : 1;
    constexpr int NRD = FM * RA + FN * RBn;
    s16x4 trt;   // first half of the K-strided fragment being read
#define READ_A(fa, ab_, s_, q_, h_)                                                              \
    do {                                                                                         \
        if constexpr (TOKENS) {                                                                  \
            const uint8_t* p_ = (ab_) + (a_l0 ^ (uint32_t)((q_) << 5)) + (32 * (s_) + 4 * (h_)) * A_RB; \
            if ((h_) == 0) trt = TR_READ(p_);                                                    \
            else fa[q_] = TR_JOIN(trt, p_);                                                      \
        } else {                                                                                 \
            fa[q_] = *reinterpret_cast<const bf16x8*>((ab_) + aoff[s_] + (q_) * 16 * ROWB);       \
        }                                                                                        \
    } while (0)
#define READ_B(fb, bb_, s_, q_, h_)                                                              \
    do {                                                                                         \
        if constexpr (B_KS) {                                                                    \
            const uint8_t* p_ = (bb_) + (b_l0 ^ (uint32_t)((q_) << 5)) + (32 * (s_) + 4 * (h_)) * B_RB; \
            if ((h_) == 0) trt = TR_READ(p_);                                                    \
            else fb[q_] = TR_JOIN(trt, p_);                                                      \
        } else {                                                                                 \
            fb[q_] = *reinterpret_cast<const bf16x8*>((bb_) + boff[s_] + (q_) * 16 * ROWB);       \
        }                                                                                        \
    } while (0)
    // read number r_ of k-substep s_ from the slots at ab_ (A image) and bb_ (B image)
#define READ_ONE(fa, fb, ab_, bb_, s_, r_)                                                       \
    do {                                                                                         \
        if ((r_) < RBn) READ_B(fb, bb_, s_, 0, (r_));                                            \
        else if ((r_) < RBn + FM * RA) READ_A(fa, ab_, s_, ((r_) - RBn) / RA, ((r_) - RBn) % RA); \
        else if ((r_) < NRD) READ_B(fb, bb_, s_, 1 + ((r_) - RBn - FM * RA) / RBn, ((r_) - RBn - FM * RA) % RBn); \
    } while (0)

    constexpr int NM = FM * FN;   // MFMAs per k-substep and wave
    // Read r goes into memory slot (RSPAN * r) / NRD: the reads end a quarter substep before the
    // substep does, because the wave waits for all of them at the block barrier and at the loop head
    // (where the compiler merges its counters), and an LDS read issued just before would be waited
    // for in full.
    constexpr int RSPAN = NM * 3 / 4;
    static_assert((FM == 8 && FN == 8 && NRD <= RSPAN) || (FM == 4 && FN == 4 && NRD <= 2 * RSPAN), "issue slots");
    static_assert(SPS == 2, "the schedule below is written for two k-substeps per block");
    constexpr int NIA = SA::NI, NIB = SB::NI;    // staging instructions per wave, operand and block
    static_assert(NIA == NIB && NM % NIA == 0 && NM / NIA >= 4, "one staging request per NM / NIA MFMAs");
    constexpr int SGAP = NM / NIA;               // MFMAs per staging request
    constexpr int SLOTS = 2 * DEPTH + 1;         // of the LDS ring
    constexpr int AHEAD = (DEPTH - 2) * (NIA + NIB) + NIA;   // requests behind those of the next block
    static_assert(DEPTH == 2 || !A_GK, "row offsets are loaded for two blocks ahead");
    // A 16-cycle MFMA leaves the wave three more issue cycles, so no memory slot may hold more than
    // three instructions: fragment reads are spread evenly over the first three quarters, staging request o sits in the slots
    // SGAP o + 1 (M0 set-up) and SGAP o + 3 (load; the MFMA in between is the wait state M0 needs).
    // Operand A's requests go into substep 0, operand B's follow the block barrier in substep 1:
    // every wave has waited for its own fragment reads of the slot that is refilled (lgkmcnt) before
    // that barrier.
#define STAGE_AT(m_, PREP_, LOAD_, slot_, kt_)                                                   \
    do {                                                                                         \
        if ((m_) % SGAP == 1) PREP_(slot_, (m_) / SGAP);                                         \
        if ((m_) % SGAP == 3) LOAD_(kt_, (m_) / SGAP);                                           \
    } while (0)
    // The MFMA gets the B fragment as its first and the A fragment as its second operand (both
    // have the same lane layout), so each 16x16 block comes out transposed: a lane then holds ONE
    // block row (l16) and the 4 consecutive block columns 4*grp + 0..3, which the epilogue stores
    // as 8- or 16-byte vectors.  (16x16x32 rather than 32x32x16: the same FLOP per cycle, but the
    // accumulator traffic per FLOP is half, and under the part's power limit the clock settles
    // higher.)
    // One k-substep: NM MFMAs on fragment set (fa, fb); after MFMA m, memory slot m is issued
    // (at most one fragment read for the next substep or one half of a staging request), so the
    // LDS and vector-memory queues are fed a little at a time while the matrix pipe stays busy:
    // one wavefront per SIMD (256x256 tiles) has nobody else to hide a burst behind.
    // A fragments run up and down in turn, so that successive MFMAs always share one operand: fewer operand bits
    // toggle, which the power limit turns into clock (registers-only loop: both operands new every time 1.96, one held
    // for eight 2.05, up and down 2.07 PFLOP/s; steps at 32768 x 768 x 3072 of 16 experts, 16384 x 1024 x 4096 fp16 of 32, 65536 x
    // 1024 x 4096 of 32: -0.3, -0.4, -0.5 %).
#define SUBSTEP(fa, fb, READ_, EXTRA_)                                                           \
    do {                                                                                         \
        _Pragma("unroll") for (int m = 0; m < NM; ++m) {                                         \
            const int ia = m / FM % 2 ? FM - 1 - m % FM : m % FM;                                \
            if constexpr (F16)                                                                   \
                asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0"                            \
                             : "+a"(acc[ia][m / FM]) : "v"(fb[m / FM]), "v"(fa[ia]));            \
            else                                                                                 \
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"                           \
                             : "+a"(acc[ia][m / FM]) : "v"(fb[m / FM]), "v"(fa[ia]));            \
            FENCE();                                                                             \
            _Pragma("unroll") for (int r = 0; r < NRD; ++r)                                      \
                if ((RSPAN * r) / NRD == m) { READ_; }                                           \
            EXTRA_;                                                                              \
            FENCE();                                                                             \
        }                                                                                        \
    } while (0)
    static_assert((DEPTH - 1) * (NIA + NIB) <= 63 && AHEAD <= 63, "vmcnt is a 6-bit counter");

    // The K loop runs in blocks of BK = 64 (two k-substeps): a row of a K-contiguous operand is
    // then one whole 128-byte line per block, and the texture-address path, which pays per line
    // touched, moves twice the bytes it would with 32-k stages.  One block of one operand (32 KB
    // of a 256-wide tile, 16 KB of a 128-wide one) is a ring slot; the 2 DEPTH + 1 slots (DEPTH = 2: five, all or half of the
    // 160 KB LDS) hold, in request order,
    //     A(j) B(j) | A(j+1) B(j+1) A(j+2)       block j being multiplied | requested ahead
    // i.e. half-block h (A(j): h = 2j, B(j): h = 2j+1) lives in slot h % SLOTS.
    // During block j: substep 0 requests A(j+DEPTH) into the slot B(j-1) left; before substep 1 the
    // wave waits until only what was requested behind B(j+1) is outstanding (so A(j+1), B(j+1) are complete) and the
    // barrier publishes them; every fragment read of block j has completed by then, so substep 1
    // requests B(j+DEPTH) into A(j)'s slot while it reads the first fragments of block j+1.  Past the
    // last block the requests re-fetch the last block into slots nobody reads, which keeps the
    // loop body free of branches.
    // DEPTH 2 gives a request half a block to a block to arrive: enough for 256x256 tiles and for two workgroups per CU, but a
    // 128x128 tile alone on its CU multiplies a block in 512 cycles and waited for half of its time (1480 to 1780 cycles a
    // block out of HBM); with all of LDS to itself it looks four blocks ahead (900 to 1300).
    // nk >= 1: K is at least one block in the row GEMMs, and a token-contraction item holds at least
    // one row.  The K loop is bottom-tested for that reason: with a zero-trip path the accumulators
    // of the two paths meet behind the loop, and the register allocator shuffles them there.
    const int klast = nk - 1;
    // WGRAD1: the byte offsets in x of the RO token rows this lane fetches per K-block, eight with 256x256
    // tiles, four with 128x128 (instruction i of a wave covers the block's rows STEP i + RPI wave + lane / CPR
    // of StageKS; the table stores a block's 64 offsets transposed, so those RO are consecutive).  rcur holds the offsets of the
    // block requested next (block j + 2 during block j); those of the block after it are loaded at
    // the head of block j and taken over at the wait in its middle, which covers them because they
    // are older than operand A's requests of that block.  The loads are inline assembly like the
    // staging requests (own counting of vmcnt).  Their results are tied to the wait statement, so
    // nothing can read them in front of it, and they do not live across the loop's back edge, where
    // the compiler would copy them (before they have arrived).
    constexpr int RO = SA::NI;         // row offsets per lane and block
    uint32_t rcur[RO] = {};
    const uint32_t* rbase = nullptr;   // this item's first table entry (wave-uniform)
    uint32_t rl_off = 0;               // this lane's entries of a block
    if constexpr (A_GK) rl_off = (uint32_t)(RO * (SA::RPI * uwave + lane / SA::CPR)) * 4u;
    auto roff_request = [&](int kt, u32x4& lo, u32x4& hi) __attribute__((always_inline)) {
        const uint32_t* p_ = rbase + (size_t)64 * kt;   // scalar base + lane offset: no vector arithmetic per block
        if constexpr (RO == 8)
            asm volatile("global_load_dwordx4 %0, %2, %3\n\tglobal_load_dwordx4 %1, %2, %3 offset:16"
                         : "=&v"(lo), "=&v"(hi) : "v"(rl_off), "s"(p_) : "memory");
        else
            asm volatile("global_load_dwordx4 %0, %1, %2" : "=&v"(lo) : "v"(rl_off), "s"(p_) : "memory");
    };
#define ROFF_TAKE(to_, lo_, hi_)                                                                  \
    do {                                                                                          \
        _Pragma("unroll") for (int q_ = 0; q_ < RO; ++q_) to_[q_] = q_ < 4 ? (lo_)[q_] : (hi_)[q_ - 4]; \
    } while (0)
    {
        u32x4 r_lo[3] = {}, r_hi[3] = {};
        if constexpr (A_GK) {
            rbase = g.rowoff + (size_t)kbeg + (size_t)64 * e;
#pragma unroll
            for (int b = 0; b < 3; ++b) roff_request(min(b, klast), r_lo[b], r_hi[b]);
            asm volatile("s_waitcnt vmcnt(0)"
                         : "+v"(r_lo[0]), "+v"(r_hi[0]), "+v"(r_lo[1]), "+v"(r_hi[1]), "+v"(r_lo[2]), "+v"(r_hi[2]) : : "memory");
        }
#pragma unroll
        for (int b = 0; b < DEPTH; ++b) {
            const uint32_t kb = (uint32_t)min(b, klast);
            if constexpr (A_GK) ROFF_TAKE(rcur, r_lo[b % 3], r_hi[b % 3]);
            _Pragma("unroll") for (int o = 0; o < NIA; ++o) { PREP_A(smem0 + 2 * b * SLOT, o); asm volatile("s_nop 0"); LOAD_A(kb, o); }
            _Pragma("unroll") for (int o = 0; o < NIB; ++o) { PREP_B(smem0 + (2 * b + 1) * SLOT, o); asm volatile("s_nop 0"); LOAD_B(kb, o); }
        }
        if constexpr (A_GK) ROFF_TAKE(rcur, r_lo[2], r_hi[2]);
    }
    // The accumulators are cleared here, between the first requests and the wait for them: claimed
    // in their accumulation registers by the empty statements (which keep their place among the
    // other volatile statements), the writes run while the first block is on its way instead of
    // after it has arrived.
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int jj = 0; jj < FN; ++jj) {
            acc[i][jj] = f32x4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+a"(acc[i][jj]));
        }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DEPTH - 1) * (NIA + NIB)) : "memory");
    __syncthreads();
    int sa = 0, sb = 1;                           // slots of A(j), B(j)
    int j = 0;
    if constexpr (!TOKENS) {
        // A wave whose rows all lie past the segment's end (the lower half of a tail tile with
        // at most BM / 2 rows) has nothing to multiply: it keeps its share of the staging requests and
        // the barriers, and skips the fragment reads, the MFMAs and the epilogue.  The time of the
        // tile is the other waves'; what is saved is energy, which is what this part runs short of.
        if (__builtin_amdgcn_readfirstlane(mvalid - wm * TM) <= 0) {
            do {
                const int sa1 = sa + 2 >= SLOTS ? sa + 2 - SLOTS : sa + 2;
                const int sb1 = sb + 2 >= SLOTS ? sb + 2 - SLOTS : sb + 2;
                const int sa2 = sa + 2 * DEPTH >= SLOTS ? sa + 2 * DEPTH - SLOTS : sa + 2 * DEPTH;
                const uint32_t a2 = smem0 + (uint32_t)(sa2 * SLOT), b2 = smem0 + (uint32_t)(sa * SLOT);
                const uint32_t kreq = (uint32_t)min(j + DEPTH, klast);
                _Pragma("unroll") for (int o = 0; o < NIA; ++o) { PREP_A(a2, o); asm volatile("s_nop 0"); LOAD_A(kreq, o); }
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AHEAD) : "memory");
                __syncthreads();
                _Pragma("unroll") for (int o = 0; o < NIB; ++o) { PREP_B(b2, o); asm volatile("s_nop 0"); LOAD_B(kreq, o); }
                sa = sa1; sb = sb1;
            } while (++j < nk);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();   // the barrier in front of the other waves' epilogue
            if constexpr (OP == OP_DGRAD2) {   // this wave's column-sum partials: no rows, zeros
                const int col = wn * TN + 2 * lane;
                if (2 * lane < TN && col < nvalid)
                    *reinterpret_cast<float2*>(g.colpart + (size_t)(row_tile * WM + wm) * (size_t)g.N + n0 + col) =
                        make_float2(0.f, 0.f);
            }
            return;
        }
    }
    _Pragma("unroll") for (int r = 0; r < NRD; ++r) READ_ONE(fa0, fb0, smem, smem + SLOT, 0, r);

    do {
        uint8_t* abase = smem + sa * SLOT;
        uint8_t* bbase = smem + sb * SLOT;
        const int sa1 = sa + 2 >= SLOTS ? sa + 2 - SLOTS : sa + 2;
        const int sb1 = sb + 2 >= SLOTS ? sb + 2 - SLOTS : sb + 2;
        const int sa2 = sa + 2 * DEPTH >= SLOTS ? sa + 2 * DEPTH - SLOTS : sa + 2 * DEPTH;
        uint8_t* anext = smem + sa1 * SLOT;
        uint8_t* bnext = smem + sb1 * SLOT;
        const uint32_t a2 = smem0 + (uint32_t)(sa2 * SLOT);   // A(j+2): the slot of B(j-1)
        const uint32_t b2 = smem0 + (uint32_t)(sa * SLOT);    // B(j+2): the slot of A(j)
        const uint32_t kreq = (uint32_t)min(j + DEPTH, klast);
        u32x4 rn_lo = {}, rn_hi = {};
        uint32_t rnx[RO];   // the same values once they have arrived
        if constexpr (A_GK) roff_request(min(j + 3, klast), rn_lo, rn_hi);
        FENCE();
        SUBSTEP(fa0, fb0, READ_ONE(fa1, fb1, abase, bbase, 1, r), STAGE_AT(m, PREP_A, LOAD_A, a2, kreq));
        if constexpr (A_GK) {
            asm volatile("s_waitcnt vmcnt(%2)" : "+v"(rn_lo), "+v"(rn_hi) : "n"(AHEAD) : "memory");
            ROFF_TAKE(rnx, rn_lo, rn_hi);
        } else {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AHEAD) : "memory");
        }
        __syncthreads();
        FENCE();
        // (WGRAD1 takes the new row offsets over one register per eighth of the substep, each copy in
        // an issue slot of its own: left to the compiler, the copies sit in a row at the
        // loop's back edge, two MFMAs' worth of issue cycles)
#define TAKE_AT(m_)                                                                               \
    do {                                                                                          \
        if constexpr (A_GK) {                                                                     \
            if ((m_) % SGAP == (SGAP == 8 ? 5 : 2))                                                \
                asm volatile("v_mov_b32 %0, %1" : "=v"(rcur[(m_) / SGAP]) : "v"(rnx[(m_) / SGAP])); \
        }                                                                                         \
    } while (0)
        SUBSTEP(fa1, fb1, READ_ONE(fa0, fb0, anext, bnext, 0, r), STAGE_AT(m, PREP_B, LOAD_B, b2, kreq); TAKE_AT(m));
#undef TAKE_AT
        sa = sa1; sb = sb1;
    } while (++j < nk);
    // no staging write may still be in flight when the workgroup gives its LDS back
    // (the MFMAs are inline assembly, so the compiler does not count the wait states their results
    // need before the epilogue reads the accumulators: 16 idle cycles cover the 4-pass MFMA)
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 7\n\ts_nop 7" ::: "memory");
    // pin every accumulator to its accumulation register at the loop exit (keeps the register
    // allocator from shuffling them between the loop and the epilogue)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int jj = 0; jj < FN; ++jj) asm volatile("" : "+a"(acc[i][jj]));
#undef STAGE_AT
#undef ROFF_TAKE
#undef SUBSTEP
#undef READ_ONE
#undef READ_A
#undef READ_B
#undef TR_JOIN
#undef TR_READ
#undef FENCE
#undef PREP_A
#undef PREP_B
#undef LOAD_A
#undef LOAD_B

    // ---- epilogue ------------------------------------------------------------------------------
    // In block (i, j) a lane holds row i*16 + l16 and the four columns j*16 + 4*grp + 0..3.  Stored
    // from there, a wave instruction would touch 16 rows with 8 or 16 bytes each.  Instead each
    // wave turns one 16-row band (i) at a time through its own part of the (now idle) ring:
    // vectors are written at [row][chunk ^ row] (16-byte chunks, so both directions are
    // conflict-free), read back with a lane per 16-byte chunk of a row, and leave as full 256- or
    // 512-byte row segments.  DGRAD2's saved activation derivatives come in the same way, staged
    // one band ahead.
    __syncthreads();   // every wave is done reading fragments
    {
        uint8_t* wreg = smem + uwave * (TN * 256);
        constexpr bool OUT_F32 = TOKENS || OP == OP_FC2P;   // weight gradients, partial sums; every other output is 16-bit
        constexpr int ESZ = OUT_F32 ? 4 : 2;
        constexpr int RPB = TN * ESZ;                 // bytes per staged row (TN columns)
        constexpr int CPRO = RPB / 16;                // 16-byte chunks per staged row
        constexpr int BAND = 16;                      // rows per band = rows of an MFMA block
        constexpr int H_OFF = BAND * RPB;             // FC1: second output of a band, behind the first
        constexpr int G_OFF = 2 * BAND * TN * 4, G_BUF = BAND * TN * 2;   // DGRAD2: two bands of saved derivatives
        static_assert(TN == 128 || TN == 64, "epilogue staging is laid out for 128- and 64-column wave tiles");
        static_assert(NW * TN * 256 <= NSLOT * SLOT && G_OFF + 2 * G_BUF <= TN * 256, "epilogue staging exceeds the ring");
        const size_t ldo = (size_t)g.N;
        const int wrow0 = wm * TM, wcol0 = wn * TN;
        // DGRAD2: stage the saved F'(pre)[band][TN cols] (16-bit, G_CPR chunks a row, chunk ^ (row % G_CPR))
        // with direct loads; instruction t covers rows G_RPI*t .. G_RPI*t + G_RPI-1
        constexpr int G_CPR = TN / 8, G_RPI = 64 / G_CPR;
        constexpr int GI = BAND / G_RPI;              // staging instructions per band
        rsrc_t rp;
        uint32_t pre_voff = 0;
        if constexpr (OP == OP_DGRAD2) {
            rp = make_rsrc(g.pre_in + (size_t)m0 * ldo, (uint32_t)mvalid * (uint32_t)ldo * 2u);
            pre_voff = (uint32_t)((wrow0 + lane / G_CPR) * (int)ldo + n0 + wcol0) * 2u;
        }
        auto stage_pre = [&](int band, int buf) {
            if constexpr (OP == OP_DGRAD2) {
#pragma unroll
                for (int t = 0; t < GI; ++t) {
                    const int row = G_RPI * t + lane / G_CPR;
                    const int c = (lane % G_CPR) ^ (row % G_CPR);
                    dtl16(rp, wreg + G_OFF + buf * G_BUF + t * 1024,
                          pre_voff + (uint32_t)((band * BAND + G_RPI * t) * (int)ldo + c * 8) * 2u, 0u);
                }
            }
        };
        // Output window of this wave: a buffer resource from (first row, first column) of the wave
        // tile to the end of its last valid row, so stores to rows past the segment are dropped by
        // the range check; a lane whose 16-byte chunk lies past the last valid column gets an
        // offset outside any window.  Instruction t of a band stores rows RPI_O*t + lane/CPRO; the
        // chunk a lane holds there is (lane % CPRO) ^ (row % CPRO) = c0 ^ (RPI_O*t % CPRO) (RPI_O*t has
        // no bit in common with lane/CPRO), so the per-lane offsets of the NST instructions are the
        // same for every band and the band's row offset is a scalar.
        constexpr int RPI_O = 1024 / RPB;            // rows per store instruction
        constexpr int NST = BAND / RPI_O;            // store instructions per band and output
        const int mv_w = min(TM, mvalid - wrow0), nv_w = min(TN, nvalid - wcol0);
        const int obytes = (mv_w > 0 && nv_w > 0) ? ((mv_w - 1) * (int)ldo + nv_w) * ESZ : 0;
        const size_t o0 = ((size_t)(m0 + wrow0) * ldo + (size_t)(n0 + wcol0)) * ESZ;
        uint8_t* obase0 = TOKENS ? reinterpret_cast<uint8_t*>(tok_out) : reinterpret_cast<uint8_t*>(g.out0);
        const rsrc_t ro0 = make_rsrc(obase0 + o0, (uint32_t)obytes);
        rsrc_t ro1 = ro0;
        if constexpr (OP == OP_FC1) ro1 = make_rsrc(reinterpret_cast<uint8_t*>(g.out1) + o0, (uint32_t)obytes);
        const int ldo_b = __builtin_amdgcn_readfirstlane((int)ldo * ESZ);   // bytes per output row
        int ovoff[NST];
        {
            const int q = lane / CPRO, c0 = (lane % CPRO) ^ (q % CPRO);
#pragma unroll
            for (int t = 0; t < NST; ++t) {
                const int c = c0 ^ (RPI_O * t % CPRO);
                ovoff[t] = c * 16 < nv_w * ESZ ? q * (int)ldo * ESZ + c * 16 : (int)0x80000000;
            }
        }
        stage_pre(0, 0);
        float cs0 = 0.f, cs1 = 0.f;   // DGRAD2: sums of columns 2*lane, 2*lane+1 over this wave's rows (ESS, Table 5 row 8)
        // The bands run as a two-stage pipeline over two LDS band buffers: the reads that fetch band
        // i-1 back from LDS are issued before the arithmetic of band i and their results are stored
        // (and, DGRAD2, added up) after it, so neither the write-to-read turn-around of LDS nor the
        // latency of the reads is waited for.  LDS executes a wave's instructions in order, so the
        // writes of band i+1 cannot overtake the reads of band i-1 from the same buffer.
        constexpr int BAND_BYTES = BAND * RPB;
        constexpr int BUF_STRIDE = (OP == OP_FC1 ? 2 : 1) * BAND_BYTES;   // FC1 stages two outputs per band
        static_assert(H_OFF == BAND_BYTES && 2 * BUF_STRIDE <= G_OFF, "band buffers overlap");
        u32x4 d0[NST], d1[OP == OP_FC1 ? NST : 1];
        // DGRAD2: with 128 columns a lane adds up two columns over all rows of a band, with 64 columns the
        // two half waves take every other row
        constexpr int CS_STEP = 128 / TN;
        uint32_t cw[OP == OP_DGRAD2 ? BAND / CS_STEP : 1];
        const int cs_row = lane / (TN / 2), cs_l = lane % (TN / 2);
        auto band_reads = [&](int buf) __attribute__((always_inline)) {
            uint8_t* wb = wreg + buf * BUF_STRIDE;
#pragma unroll
            for (int t = 0; t < NST; ++t) {
                d0[t] = *reinterpret_cast<const u32x4*>(wb + t * 1024 + lane * 16);
                if constexpr (OP == OP_FC1) d1[t] = *reinterpret_cast<const u32x4*>(wb + H_OFF + t * 1024 + lane * 16);
            }
            if constexpr (OP == OP_DGRAD2) {
                // bias-gradient partial: the band holds the rounded dpre values the weight gradient
                // will read; rows past the segment and columns past N are exact zeros
#pragma unroll
                for (int q = 0; q < BAND / CS_STEP; ++q) {
                    const int row = CS_STEP * q + cs_row;
                    cw[q] = *reinterpret_cast<const uint32_t*>(
                        wb + row * RPB + (((cs_l >> 2) ^ (row % CPRO)) << 4) + (cs_l & 3) * 4);
                }
            }
        };
        auto band_store_one = [&](int i, int t) __attribute__((always_inline)) {
            const int soff = (i * BAND + RPI_O * t) * ldo_b;
            buf_store16(d0[t], ro0, ovoff[t], soff);
            if constexpr (OP == OP_FC1) buf_store16(d1[t], ro1, ovoff[t], soff);
        };
        auto band_stores = [&](int i, bool with_stores) __attribute__((always_inline)) {
            if (with_stores) {
#pragma unroll
                for (int t = 0; t < NST; ++t) band_store_one(i, t);
            }
            if constexpr (OP == OP_DGRAD2) {
#pragma unroll
                for (int q = 0; q < BAND / CS_STEP; ++q) {
                    float c0, c1;
                    unpack2<F16>(cw[q], c0, c1);
                    cs0 += c0; cs1 += c1;
                }
            }
        };
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            uint8_t* wb = wreg + (i & 1) * BUF_STRIDE;
            if (i > 0) band_reads((i - 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (OP == OP_DGRAD2) {
                // the next band's derivatives are requested before this band's are awaited; the
                // counter also holds stores of earlier bands, which are older than both
                if (i + 1 < FM) stage_pre(i + 1, (i + 1) & 1);
                if (i + 1 < FM) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(GI) : "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            // -- registers -> LDS band
            // (the band's accumulators are claimed in their accumulation registers at this point:
            // otherwise the register allocator permutes and copies a few hundred of them ahead of
            // the first band)
#pragma unroll
            for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j]));
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int col = j * 16 + 4 * grp;                  // column inside the wave tile
                f32x4 v = acc[i][j];
                if constexpr (OP == OP_FC1 || OP == OP_FC2 || OP == OP_FC2P) {
                    const u32x2 bb = biasv[j];
                    float b0, b1, b2, b3;
                    unpack2<F16>(bb.x, b0, b1); unpack2<F16>(bb.y, b2, b3);
                    v[0] += b0; v[1] += b1; v[2] += b2; v[3] += b3;
                }
                if constexpr (OP == OP_FC2P) {
                    const int c = col >> 2;
                    *reinterpret_cast<f32x4*>(wb + l16 * RPB + ((c ^ (l16 % CPRO)) << 4)) = v;
                } else if constexpr (OUT_F32) {
                    // straight from the accumulation registers (an LDS store may take its data from
                    // them; through ordinary registers it is 256 more copies per wave and tile)
                    const int c = col >> 2;
                    const uint32_t la = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)(wb + l16 * RPB + ((c ^ (l16 % CPRO)) << 4));
                    asm volatile("ds_write_b128 %0, %1" : : "v"(la), "a"(acc[i][j]) : "memory");
                } else {
                    const int c = col >> 3;
                    const uint32_t off = (uint32_t)(l16 * RPB + ((c ^ (l16 % CPRO)) << 4) + (grp & 1) * 8);
                    if constexpr (OP == OP_FC1) {
                        float hh[4], gg[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) act_both<ACT>(v[r], hh[r], gg[r]);
                        u32x2 pz, hz;
                        pz.x = pack2<F16>(gg[0], gg[1]); pz.y = pack2<F16>(gg[2], gg[3]);
                        hz.x = pack2<F16>(hh[0], hh[1]); hz.y = pack2<F16>(hh[2], hh[3]);
                        *reinterpret_cast<u32x2*>(wb + off) = pz;
                        *reinterpret_cast<u32x2*>(wb + H_OFF + off) = hz;
                    } else if constexpr (OP == OP_FC2 || OP == OP_DGRAD1) {
                        u32x2 z;
                        z.x = pack2<F16>(v[0], v[1]); z.y = pack2<F16>(v[2], v[3]);
                        *reinterpret_cast<u32x2*>(wb + off) = z;
                    } else {   // DGRAD2
                        const u32x2 pp = *reinterpret_cast<const u32x2*>(wreg + G_OFF + (i & 1) * G_BUF + off);
                        float p0, p1, p2, p3;
                        unpack2<F16>(pp.x, p0, p1); unpack2<F16>(pp.y, p2, p3);
                        u32x2 d;
                        d.x = pack2<F16>(v[0] * p0, v[1] * p1);
                        d.y = pack2<F16>(v[2] * p2, v[3] * p3);
                        *reinterpret_cast<u32x2*>(wb + off) = d;
                    }
                }
                // the previous band's stores go out one at a time between the blocks of this band's
                // arithmetic: issued in a row behind it they fill the address queue of the texture
                // unit and the wave waits (5 % of fc1's cycles)
                if (i > 0 && j % (FN / NST) == FN / NST - 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    band_store_one(i - 1, j / (FN / NST));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (i > 0) band_stores(i - 1, false);   // (DGRAD2: the previous band's column sums)
        }
        band_reads((FM - 1) & 1);
        band_stores(FM - 1, true);
        if constexpr (OP == OP_DGRAD2) {
            const int col = wcol0 + 2 * cs_l;
            if constexpr (CS_STEP == 2) { cs0 += __shfl_xor(cs0, 32); cs1 += __shfl_xor(cs1, 32); }
            if (cs_row == 0 && col < nvalid)
                *reinterpret_cast<float2*>(g.colpart + (size_t)(row_tile * WM + wm) * ldo + n0 + col) =
                    make_float2(cs0, cs1);
        }
    }
}

template <int BM, int BN, int WM, int WN, int OP, int ACT = HEXA_ACT_GELU_TANH, bool F16 = false>
__global__ __launch_bounds__(WM * WN * 64, BM == 256 ? 1 : 2) void gemm_bf16(GemmArgs g) {
    if constexpr (OP == OP_FC2P) {
        g.share = (int)blockIdx.y;
        g.out0 = reinterpret_cast<float*>(g.out0) + (size_t)g.share * g.a_rows * g.N;
    }
    Tile t;
    const int x = (int)blockIdx.x % kXcds, loc = (int)blockIdx.x / kXcds;
    if constexpr (BM == 256) {
        int quarter;
        if (!pick_rows_big(g, x, loc, t, quarter)) return;
        if (quarter >= 0) {        // (products and sums in the same order as in a whole tile)
            t.it.beg += 128 * (quarter >> 1);
            t.it.end = min(t.it.end, t.it.beg + 128);
            t.tile_n = 2 * t.tile_n + (quarter & 1);
            if (t.it.beg < t.it.end && t.tile_n * 128 < g.N) gemm_tile<128, 128, WM, WN, OP, ACT, F16, 4>(g, t);
            return;
        }
    } else if (!pick_rows_small<BM, BN>(g, x, loc, t)) return;
    gemm_tile<BM, BN, WM, WN, OP, ACT, F16>(g, t);
}

// Two independent contractions in one grid (the paper's fused backward kernel, Sec. 3.2 "Fused
// Kernel in Backward Propagation": the input gradient and the weight gradient of one linear layer
// do not depend on each other), so the tail of one fills with tiles of the other.
template <int BM, int BN, int WM, int WN, int OPA, int OPB, bool F16 = false>
__global__ __launch_bounds__(WM * WN * 64, BM == 256 ? 1 : 2) void gemm_bf16_pair(GemmArgs ga, GemmArgs gb) {
    Tile t;
    const int which = pick_pair<BM>(ga, gb, OPA == OP_DGRAD2 ? WL_ORDER2 : WL_ORDER1, (int)blockIdx.x % kXcds,
                                    (int)blockIdx.x / kXcds, t);
    if (which == 2) gemm_tile<BM, BN, WM, WN, OPB, HEXA_ACT_GELU_TANH, F16>(gb, t);
    else if (which == 1) gemm_tile<BM, BN, WM, WN, OPA, HEXA_ACT_GELU_TANH, F16>(ga, t);
}


// A row GEMM of a forward pass with few rows per expert, as in a decode step: what it takes is reading the weights once, which is bound by the bytes that are
// on their way.  32x128 tiles; each wavefront takes every fourth 32-k step of the tile's contraction by itself, from memory to registers without
// LDS or barriers, four steps on their way (8 KB each; eight wavefronts on a CU, 256 KB): a lane loads 16 bytes, 8 columns, of 8 k-rows and transposes
// the 8x8 block with 32 v_perm into the operands of matrix instruction c = 0 .. 7, for columns c, 8 + c, ...; token rows come straight in operand
// order.  The four wavefronts' sums meet in LDS, in order.
// The columns are 16-byte chunks (N is a multiple of 64); past the edge a lane repeats the last one.  Token rows past the segment are zeros.
constexpr int kThinRows = 32, kThinCols = 128, kThinDepth = 4;
template <int OP, int ACT = HEXA_ACT_GELU_TANH, bool F16 = false>
__global__ __launch_bounds__(256, 2) void gemm_bf16_thin(GemmArgs g) {
    static_assert(OP == OP_FC1 || OP == OP_FC2 || OP == OP_FC2P, "weights [K][N]");
    constexpr int PITCH = kThinCols + 4;
    __shared__ __align__(16) float sums[4][16][PITCH];
    if constexpr (OP == OP_FC2P) {
        g.share = (int)blockIdx.y;
        g.out0 = reinterpret_cast<float*>(g.out0) + (size_t)g.share * g.a_rows * g.N;
    }
    Tile t;
    if (!pick_rows_small<kThinRows, kThinCols>(g, (int)blockIdx.x % kXcds, (int)blockIdx.x / kXcds, t)) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l16 = lane & 15, grp = lane >> 4;
    const int e = t.it.e, m0 = t.it.beg, rows = t.it.end - m0, n0 = t.tile_n * kThinCols, cols = min(kThinCols, g.N - n0);
    const int first = OP == OP_FC2P ? 2 * g.share * g.share_blocks : 0;
    const int steps = OP == OP_FC2P ? min(2 * g.share_blocks, g.K / 32 - first) : g.K / 32;
    const int n = (steps - wave + 3) / 4;        // this wavefront's: first + wave, + 4, ...

    const uint32_t nb = (uint32_t)g.N * 2u, kb = (uint32_t)g.K * 2u;
    auto resource = [](const bf16_t* p, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, (int)bytes, 0x00020000); };
    const __amdgpu_buffer_rsrc_t rw = resource(g.B + (size_t)e * g.K * g.N, (uint32_t)g.K * nb);
    const uint32_t wv = (uint32_t)(8 * grp) * nb + (uint32_t)(n0 + min(8 * l16, cols - 8)) * 2u;
    const __amdgpu_buffer_rsrc_t ra = OP == OP_FC1 ? resource(g.A, (uint32_t)g.a_rows * kb) : resource(g.A + (size_t)m0 * g.K, (uint32_t)rows * kb);
    uint32_t av[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = 16 * h + l16;
        const uint32_t row = OP != OP_FC1 ? (uint32_t)r : (uint32_t)(r < rows ? g.perm[m0 + r] / g.topk : g.a_rows);
        av[h] = row * kb + 16u * grp;
    }
    u32x4 w[kThinDepth][8], a[kThinDepth][2];
    auto load = [&](int s, int i) __attribute__((always_inline)) {
        // past the end: the last step again for A, no weights (behind the range)
        const uint32_t k0 = 32u * (uint32_t)(first + wave + 4 * min(i, n - 1)), k0w = i < n ? k0 : (uint32_t)g.K;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            w[s][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)wv, (int)((k0w + q) * nb), 0));
#pragma unroll
        for (int h = 0; h < 2; ++h)
            a[s][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)av[h], (int)(k0 * 2u), 0));
    };
    f32x4 acc[2][8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[h][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            u32x4 b;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                b[p] = __builtin_amdgcn_perm(w[s][2 * p + 1][c / 2], w[s][2 * p][c / 2], c % 2 ? 0x07060302u : 0x05040100u);
            // (weights first: a lane then holds row l16 and columns 8 (4 grp + r) + c, r = 0 .. 3)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if constexpr (F16) acc[h][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, b), __builtin_bit_cast(f16x8, a[s][h]), acc[h][c], 0, 0, 0);
                else acc[h][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b), __builtin_bit_cast(bf16x8, a[s][h]), acc[h][c], 0, 0, 0);
            }
        }
    };
    if (n > 0) {
#pragma unroll
        for (int s = 0; s < kThinDepth; ++s) load(s, s);
        int i = 0;
        for (; i + kThinDepth <= n; i += kThinDepth) {
#pragma unroll
            for (int s = 0; s < kThinDepth; ++s) {
                multiply(s);
                load(s, i + s + kThinDepth);
            }
        }
#pragma unroll
        for (int s = 0; s < kThinDepth - 1; ++s)
            if (i + s < n) multiply(s);
    }

    // ---- the four wavefronts' sums, 16 rows at a time: a thread adds up 8 columns of one row
    const int row = (int)threadIdx.x / 16, col = (int)threadIdx.x % 16 * 8;
    u32x4 bias = {0, 0, 0, 0};
    if ((OP != OP_FC2P || g.share == 0) && col < cols) bias = *reinterpret_cast<const u32x4*>(g.bias + (size_t)e * g.N + n0 + col);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (16 * h >= rows) break;
        if (h) __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c4 = 0; c4 < 2; ++c4)
                *reinterpret_cast<f32x4*>(&sums[wave][l16][8 * (4 * grp + r) + 4 * c4]) =
                    f32x4{acc[h][4 * c4][r], acc[h][4 * c4 + 1][r], acc[h][4 * c4 + 2][r], acc[h][4 * c4 + 3][r]};
        __syncthreads();
        if (16 * h + row >= rows || col >= cols) continue;
        float v[8];
#pragma unroll
        for (int c4 = 0; c4 < 2; ++c4) {
            f32x4 s = *reinterpret_cast<const f32x4*>(&sums[0][row][col + 4 * c4]);
#pragma unroll
            for (int q = 1; q < 4; ++q) s += *reinterpret_cast<const f32x4*>(&sums[q][row][col + 4 * c4]);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float b0, b1;
                unpack2<F16>(bias[2 * c4 + q], b0, b1);
                v[4 * c4 + 2 * q] = s[2 * q] + b0;
                v[4 * c4 + 2 * q + 1] = s[2 * q + 1] + b1;
            }
        }
        const size_t o = (size_t)(m0 + 16 * h + row) * g.N + n0 + col;
        if constexpr (OP == OP_FC2P) {
            float* out = reinterpret_cast<float*>(g.out0) + o;
            *reinterpret_cast<f32x4*>(out) = f32x4{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<f32x4*>(out + 4) = f32x4{v[4], v[5], v[6], v[7]};
        } else {
            u32x4 z, z1;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (OP == OP_FC1) {
                    float h0, g0, h1, g1;
                    act_both<ACT>(v[2 * q], h0, g0);
                    act_both<ACT>(v[2 * q + 1], h1, g1);
                    z[q] = pack2<F16>(g0, g1);
                    z1[q] = pack2<F16>(h0, h1);
                } else {
                    z[q] = pack2<F16>(v[2 * q], v[2 * q + 1]);
                }
            }
            *reinterpret_cast<u32x4*>(reinterpret_cast<bf16_t*>(g.out0) + o) = z;
            if constexpr (OP == OP_FC1) *reinterpret_cast<u32x4*>(reinterpret_cast<bf16_t*>(g.out1) + o) = z1;
        }
    }
}
template <int OP, int ACT = HEXA_ACT_GELU_TANH, bool F16 = false>
void launch_thin(const MoeDims& D, const GemmArgs& g, hipStream_t st, const char* label, int shares = 1) {
    ProfScope ps(st, label);
    auto kern = gemm_bf16_thin<OP, ACT, F16>;
    const int grid = kXcds * RowTiles<kThinRows>::most(D.A / kThinRows + std::min(D.E, D.A), ceil_div(g.N, kThinCols));
    hipLaunchKernelGGL(kern, dim3(grid, shares), dim3(256), 0, st, g);
}

template <int BM, int BN, int WM, int WN, int OP, int ACT = HEXA_ACT_GELU_TANH, bool F16 = false>
void launch_rows(const MoeDims& D, const GemmArgs& g, hipStream_t st, const char* label, int shares = 1) {
    ProfScope ps(st, label);
    auto kern = gemm_bf16<BM, BN, WM, WN, OP, ACT, F16>;
    constexpr int lds = NSLOT * (BM > BN ? BM : BN) * ROWB;
    const int tm_max = D.A / BM + D.E;
    const int grid = kXcds * (RowTiles<BM>::most(tm_max, ceil_div(g.N, BN)) + (BM == 256 ? 3 * kQuartersUpTo : 0));
    hipLaunchKernelGGL(kern, dim3(grid, shares), dim3(WM * WN * 64), lds, st, g);
}

// Row GEMM OPA and token contraction OPB of one linear layer's backward in one grid.
template <int BM, int BN, int WM, int WN, int OPA, int OPB, bool F16 = false>
void launch_pair(const MoeDims& D, const GemmArgs& ga, const GemmArgs& gb, hipStream_t st, const char* label) {
    auto kern = gemm_bf16_pair<BM, BN, WM, WN, OPA, OPB, F16>;
    constexpr int lds = NSLOT * (BM > BN ? BM : BN) * ROWB;
    const int tm_max = D.A / BM + D.E;
    const TokenTiles tok{ceil_div(gb.M, BM) * ceil_div(gb.N, BN)};
    const int per_xcd = RowTiles<BM>::most(tm_max, ceil_div(ga.N, BN)) + tok.most(D.A / gb.chunk_len + D.E);
    ProfScope ps(st, label);
    hipLaunchKernelGGL(kern, dim3(kXcds * per_xcd), dim3(WM * WN * 64), lds, st, ga, gb);
}

// Two tile classes.  256x256: one workgroup per CU (all of LDS, 512 registers per lane), the cheaper one
// per FLOP (a 128x128 tile fetches and reads twice the bytes per FLOP), which wins once its tiles fill the
// chip.  128x128: two workgroups per CU (half of LDS, 256 registers), four times as many tiles, so it wins
// where 256x256 tiles are too few for 256 CUs or mostly padding.
constexpr int BIG = 256, SMALL = 128;

// Which class a launch takes: the one with the shorter estimated time.  A tile takes a start-up and epilogue
// time plus a time per 64-k block; a launch takes its tiles' summed time over the slots of the chip plus a
// share of its longest tile for the uneven end, and never less than its longest tile.  The four numbers of a
// class are fitted to 120 launches (30 shapes: 256 to 65536 tokens, d 64 to 2048, f 256 to 8192, 4 to 64
// experts, both classes measured): with them the slower class is picked by 1 % of a launch's time on average
// and by 14 % at most (a skewed 32768 x 256 x 1024 case); always taking 256x256 tiles costs 16 % on average
// and up to a factor of 2.2.  As a prediction of a launch's time it is rough, and it knows no whole rounds of tiles: of 30
// traced launches (profiles/pass_kernel_times.md) it gives the 256x256 ones 0.90 to 1.06 of their time, the 128x128
// ones 1.1 to 2.3 (block_us is that of two workgroups side by side on a CU, and a small grid leaves one).  Measured on both sides of the line, 256x256 against 128x128, in us:
// d = 384, f = 1536, 8 experts, top-2: fc2 32.4 / 16.5 at 4096 tokens, 72 / 59 at 16384; d = 768, f = 3072,
// 16 experts: fc2 78 / 54 at 2048 tokens, 77 / 71 at 4096, 95 / 115 at 8192, 164 / 205 at 16384.
struct ClassCost { double slots, start_us, block_us, tail; };
constexpr ClassCost kCostBig{256, 15.1, 1.22, 0.87}, kCostSmall{512, 7.3, 1.31, 0.54};

struct Work { double tiles, blocks; };   // tiles of a contraction, 64-k blocks per tile

inline double launch_us(const ClassCost& c, std::initializer_list<Work> parts) {
    double sum = 0, longest = 0;
    for (const Work& w : parts) {
        const double t = c.start_us + c.block_us * w.blocks;
        sum += w.tiles * t;
        longest = std::max(longest, t);
    }
    return std::max(longest, sum / c.slots + c.tail * longest);
}

// Row tiles of height bm the experts' segments are expected to make (the host does not know the routing):
// rows spread over the experts that can have any, half a tile of padding each.
inline double expected_row_tiles(const MoeDims& D, int bm) {
    const double e = D.E < D.A ? D.E : D.A, rows = D.A / e;
    return rows > bm / 2 ? e * std::max(1.0, rows / bm + 0.5) : e;
}
inline Work row_work(const MoeDims& D, int bm, int K, int N) {
    return {expected_row_tiles(D, bm) * ceil_div(N, bm), K / 64.0};
}
inline Work token_work(const MoeDims& D, int bm) {
    const double rows = D.A / (double)(D.E < D.A ? D.E : D.A), chunk = wgrad_chunk_len(D);
    return {D.E * std::max(1.0, rows / chunk) * ceil_div(D.d, bm) * ceil_div(D.f, bm), std::min(rows, chunk) / 64.0};
}
inline bool small_rows(const MoeDims& D, int K, int N) {
    return launch_us(kCostSmall, {row_work(D, SMALL, K, N)}) < launch_us(kCostBig, {row_work(D, BIG, K, N)});
}
inline bool small_pair(const MoeDims& D, int K, int N) {
    return launch_us(kCostSmall, {row_work(D, SMALL, K, N), token_work(D, SMALL)}) <
           launch_us(kCostBig, {row_work(D, BIG, K, N), token_work(D, BIG)});
}
// A backward grid of 256x256 tiles of a few rounds: with the shorter row-GEMM tiles first, the token contraction's fill the
// last rounds unevenly (us, row GEMM / token contraction first: 118378 x 384 x 1536 of 2, bwd_fc1 385 / 347; 39567 x 320 x 256 of 9,
// bwd_fc2 150 / 89; 9655 x 832 x 1280 of 4, bwd_fc1 198 / 170).  In a launch of many rounds the row GEMM first is 0.2 to 1 % faster
// (steps at 32768 x 768 x 3072 of 16 and 65536 x 1024 x 4096 of 32).  The line: four times the longer tile.
inline bool token_first(const MoeDims& D, int K, int N) {
    const Work r = row_work(D, BIG, K, N), t = token_work(D, BIG);
    const double tr = kCostBig.start_us + kCostBig.block_us * r.blocks, tt = kCostBig.start_us + kCostBig.block_us * t.blocks;
    return tt > tr && r.tiles * tr + t.tiles * tt < 4.0 * kCostBig.slots * tt;
}
// Weights that are read once and do not fit the Infinity Cache (256 MB): see RowTiles.  For the forward pass (fc1 / fc2 in us, an eighth
// of all tiles per XCD -> streamed: 64 tokens, 2048 x 8192 of 64 350 / 248 -> 327 / 243; 1000, 1024 x 4096 of 64 195 / 108 -> 166 / 115; 2000, 2048 x 2048
// of 64 191 / 132 -> 159 / 107; 300, 1536 x 6144 of 24 155 / 100 -> 153 / 101).  In the backward pass the weight gradients, which share the
// grid, lose to it where there are few rows: bwd_fc2 of the first 796 -> 842, of 8 tokens at 2048 x 8192 of 16 218 -> 228, of the second 326 -> 318.
inline bool streamed(const MoeDims& D) {
    return (long long)D.A < (long long)SMALL * D.E && (double)D.E * D.d * D.f * 2.0 > 256e6;
}
inline bool small_fc1(const MoeDims& D) { return small_rows(D, D.d, D.f); }
inline bool small_fc2(const MoeDims& D) { return small_rows(D, D.f, D.d); }
inline bool small_bwd2(const MoeDims& D) { return small_pair(D, D.d, D.f); }
inline bool small_bwd1(const MoeDims& D) { return small_pair(D, D.f, D.d); }

// Which forward launches take the thin tiles: with more rows, experts have several of them, which fetch the weights again (16 rows per expert, 512
// tokens, 2048 x 8192 of 64, top-2, us, 128x128 / thin: fc1 411 / 432, fc2 389 / 399; 300, 1536 x 6144 of 24 (12.5) 101 / 97, 97 / 121; 16 tokens, 1536 x 6144 of 2, one tile
// each 19.6 / 13.9, 45.7 / 18.0).  Under skewed routing some experts have more than 32 rows at fewer on average, which sets the other line, rows in all.
// Measured on both sides under the benchmark's "bias" routing, Zipf (exponent 1.2), three quarters of the tokens on four experts, all tokens
// on the first ones, us, 128x128 / thin:
//   fc1: 32 tokens, 1024 x 4096 of 4 16 / 12, 16 / 13, 16 / 12, 15 / 12; 192, 1024 x 4096 of 32 56 / 53, 31 / 30, 48 / 41, 15 / 13; 64, 2048 x 8192 of 64,
//     top-2 275 / 258, 111 / 103, 148 / 146, 32 / 25; 128 there 322 / 309, 132 / 126, 212 / 204, 33 / 37; 384, 512 x 2048 of 64 35 / 32, 13 / 15, 31 / 27, 12 / 10;
//     192 there, top-2, at 2048 x 8192 357 / 346, 140 / 148, 253 / 258, 33 / 45; 1500, 512 x 1024 of 256 61 / 53, 14 / 17, 45 / 42, 13 / 16.  (Where the tiles are one
//     round either way: 8, 2048 x 8192 of 8 44 / 45, 33 / 25, 41 / 44, 21 / 14.)
//   fc2 + combine, up to 1024 tiles: 16, 768 x 3072 of 16, top-2 (96 tiles) 26 / 23, 20 / 19, 23 / 20, 18 / 16; 32, 1024 x 4096 of 16,
//     top-2 (128) 34 / 37, 32 / 30, 33 / 33, 22 / 21; 24, 1024 x 4096 of 24, top-2 (192) 47 / 40, 31 / 29, 31 / 30, 21 / 21; 64, 1024 x 4096 of 32 (256) 52 / 47, 30 / 30, 34 / 36,
//     22 / 18; 48 there, top-3 60 / 62, 47 / 47, 52 / 49, 23 / 24; 13, 1216 x 4864 of 41, top-4 (410) 92 / 75, 50 / 50, 51 / 51, 41 / 27; 8, 2048 x 8192 of 64, top-4 (512) 139 / 134, 91 / 92,
//     88 / 88, 47 / 45; 40, 1088 x 1280 of 108, top-2 (720) 36 / 36, 23 / 20, 29 / 26, 21 / 18; 96, 1024 x 4096 of 96, top-2 (768) 123 / 116, 51 / 50, 77 / 71, 28 / 27; 64, 2048 x 8192 of
//     64, top-2 (1024) 250 / 260, 115 / 115, 163 / 157, 61 / 44; 48, 2048 x 1024 of 64, top-4 (1024) 55 / 56, 32 / 35, 35 / 41, 20 / 21.
// (K + 64 rows of weights have to fit the 32-bit offsets of requests past the end.)
constexpr int kThinUpTo = 6, kThinMostRows = 192, kThinFc2Tiles = 1024;
inline bool thin_fc1(const MoeDims& D) {
    const double wider = D.d > D.f ? D.d : D.f, other = D.d > D.f ? D.f : D.d;
    return (D.A <= kThinRows || (D.A <= kThinMostRows && D.A <= (long long)kThinUpTo * std::min(D.E, D.A))) &&
           (wider * other + 64 * wider) * 2 < 4294967296.0;
}
inline long long thin_fc2_tiles(const MoeDims& D) { return (long long)std::min(D.E, D.A) * ceil_div(D.d, kThinCols); }
inline bool thin_fc2(const MoeDims& D) { return thin_fc1(D) && thin_fc2_tiles(D) <= kThinFc2Tiles; }
// Shares of K for FC2 on thin tiles: what makes four workgroups per CU, so that half of the experts fill the chip, two at least (one, with 1024 tiles: 64
// tokens, 2048 x 8192 of 64, top-2 258, under Zipf 127, with two 260, 115), at least three 64-k blocks each.
// At most 7: of eight, all workgroups start at the same offset of a power of two, where f is one (fc2 + combine in us at 8 / 7 / 6 / 5 shares: 8 tokens, 2048
// x 8192 of 8 48 / 45 / 46 / 45; 32, 1024 x 4096 of 16, top-2 38 / 37 / 36 / 37; 32 there of 4 19 / 18 / 17 / 17; 20, 1280 x 5120 of 12 33 / 33 / 33 / 35; 24, 1536 x 6144 of 8, top-2
// 41 / 41 / 44 / 41).  Two workgroups per CU / four: 24 tokens, 1024 x 4096 of 24, top-2 48 / 40, under Zipf 41 / 29; 12, 2048 x 8192 of 12 69 / 59; 16, 768 x 3072 of
// 16, top-2 24 / 23.
inline int thin_fc2_shares(const MoeDims& D) {
    return std::max(1, std::min({7, std::max(2, 4 * kNumCUs / (int)thin_fc2_tiles(D)), D.f / BK / 3}));
}

// FC2 in shares of K: with few rows its tiles are few and long (K = d_ff), so a decode step leaves most CUs idle.
// The workgroups of a share write unrounded sums, combine_split adds them up in order; that traffic and the
// number of shares are weighed by the same estimate.  It was checked against 1, 2, 4 and 8 shares on 13 shapes of
// 1 to 4096 tokens: never more than 10 % behind the best of them for fc2 + combine, 2 % on average.  Measured,
// fc2 + combine in us at 1 / 2 / 4 / 8 shares: 16 tokens, d = 768, f = 3072, 16 experts, top-2: 35 / 25 / 22 / 26;
// 64 tokens, 2048 x 8192 x 64: 287 / 251 / 257 / 263; 1024 tokens, 512 x 2048 x 8: 28 / 28 / 25 / 31; 2048 tokens,
// 768 x 3072 x 16: 47 / 56 / 62 / 83 (one share is taken).
int choose_fc2_shares(const MoeDims& D) {
    if (thin_fc2(D)) return thin_fc2_shares(D);
    if (!small_fc2(D)) return 1;
    const int blocks = D.f / BK;
    int best = 1;
    double best_us = 0;
    for (int s = 1; s <= 8 && s <= blocks; ++s) {
        Work w = row_work(D, SMALL, D.f, D.d);
        w.tiles *= s;
        w.blocks = ceil_div(blocks, s);
        double us = launch_us(kCostSmall, {w});
        if (s > 1) us += s + (double)s * D.A * D.d * 8.0 / 4e6;   // written and read back at 4 TB/s
        if (s == 1 || us < best_us) { best = s; best_us = us; }
    }
    return best;
}

}  // namespace

// (rounded so that every share has at least one block)
int fc2_share_blocks(const MoeDims& D) { return ceil_div(D.f / BK, choose_fc2_shares(D)); }
int fc2_shares(const MoeDims& D) { return ceil_div(D.f / BK, fc2_share_blocks(D)); }

// Every contraction kernel needs more dynamic shared memory than a kernel may use before its attribute
// has been raised, once per device.
template <int B, typename K>
static hipError_t allow_lds(K kern) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, NSLOT * B * ROWB);
}
template <int B, bool F16>
static hipError_t device_init_class() {
    hipError_t e = allow_lds<B>(gemm_bf16<B, B, 2, 2, OP_FC1, HEXA_ACT_GELU_TANH, F16>);
    if (e == hipSuccess) e = allow_lds<B>(gemm_bf16<B, B, 2, 2, OP_FC1, HEXA_ACT_RELU, F16>);
    if (e == hipSuccess) e = allow_lds<B>(gemm_bf16<B, B, 2, 2, OP_FC1, HEXA_ACT_SILU, F16>);
    if (e == hipSuccess) e = allow_lds<B>(gemm_bf16<B, B, 2, 2, OP_FC2, HEXA_ACT_GELU_TANH, F16>);
    if constexpr (B == SMALL) {
        if (e == hipSuccess) e = allow_lds<B>(gemm_bf16<B, B, 2, 2, OP_FC2P, HEXA_ACT_GELU_TANH, F16>);
    }
    if (e == hipSuccess) e = allow_lds<B>(gemm_bf16_pair<B, B, 2, 2, OP_DGRAD2, OP_WGRAD2, F16>);
    if (e == hipSuccess) e = allow_lds<B>(gemm_bf16_pair<B, B, 2, 2, OP_DGRAD1, OP_WGRAD1, F16>);
    return e;
}
hipError_t gemm_bf16_device_init() {
    hipError_t e = device_init_class<BIG, false>();
    if (e == hipSuccess) e = device_init_class<BIG, true>();
    if (e == hipSuccess) e = device_init_class<SMALL, false>();
    if (e == hipSuccess) e = device_init_class<SMALL, true>();
    return e;
}

void gemm_thin(const MoeDims& D, bool (&thin)[2]) {
    thin[0] = thin_fc1(D);
    thin[1] = thin_fc2(D);
}
void gemm_tile_classes(const MoeDims& D, int (&tile)[4]) {
    const bool small[4] = {small_fc1(D), small_fc2(D), small_bwd2(D), small_bwd1(D)};
    for (int i = 0; i < 4; ++i) tile[i] = small[i] ? SMALL : BIG;
}

// Row-tile height of the DGRAD2 column-sum partials (for the finisher).
int gemm_dgrad2_row_tile(const MoeDims& D) { return small_bwd2(D) ? SMALL : BIG; }
int gemm_rowoff_step(const MoeDims& D) { return small_bwd1(D) ? StageKS<SMALL, 4>::STEP : StageKS<BIG, 4>::STEP; }

// Tokens per split-K chunk of the token contractions: an expert is cut only when its rows alone
// would give every CU a tile's worth of work for longer than the whole contraction takes on
// average (chunk = the rows that make one tile per CU of the chip: A * tiles / CUs).  Shorter chunks
// balance no better, because the grid is shared with the row GEMM of the same layer, whose tiles
// fill the gaps, and every extra chunk costs a partial d x f tile written and read back (measured:
// a quarter of this length made C3 5.6 %, C4 1.9 % and C5 under Zipf routing 0.5 % slower; half
// as many chunks again made C3 and C4 slower).
int wgrad_chunk_len(const MoeDims& D) {
    const long long tmn = (long long)ceil_div(D.d, BIG) * ceil_div(D.f, BIG);
    long long L = (long long)D.A * tmn / kNumCUs;
    L = (L + 63) / 64 * 64;
    if (L < 1024) L = 1024;
    // one item's rows (less than 2 L) are addressed with 32-bit byte offsets: 2 L * max(d, f) * 2 < 2^32
    const long long cap = (0xffffffffLL / (4LL * (D.d > D.f ? D.d : D.f))) / 64 * 64;
    if (L > cap) L = cap;
    return (int)L;
}

// Capacity of the work lists: row tiles, token-contraction items.
static size_t worklist_rt_cap(const MoeDims& D) { return (size_t)(D.A / BIG + D.E); }
size_t gemm_worklist_ints(const MoeDims& D) {
    return kWlHeader + 4 * (worklist_rt_cap(D) + (size_t)(D.A / wgrad_chunk_len(D) + D.E));
}
static void use_lists(const MoeDims& D, const MoeWorkspace& ws, GemmArgs& g) {
    g.lists = ws.worklist;
    g.rt_cap = (int)worklist_rt_cap(D);
}

template <int B, bool F16>
static void launch_fc1(const MoeDims& D, const GemmArgs& g, hipStream_t st) {
    if (D.act == HEXA_ACT_RELU) launch_rows<B, B, 2, 2, OP_FC1, HEXA_ACT_RELU, F16>(D, g, st, "fc1");
    else if (D.act == HEXA_ACT_SILU) launch_rows<B, B, 2, 2, OP_FC1, HEXA_ACT_SILU, F16>(D, g, st, "fc1");
    else launch_rows<B, B, 2, 2, OP_FC1, HEXA_ACT_GELU_TANH, F16>(D, g, st, "fc1");
}

template <bool F16>
static void launch_thin_fc1(const MoeDims& D, const GemmArgs& g, hipStream_t st) {
    if (D.act == HEXA_ACT_RELU) launch_thin<OP_FC1, HEXA_ACT_RELU, F16>(D, g, st, "fc1");
    else if (D.act == HEXA_ACT_SILU) launch_thin<OP_FC1, HEXA_ACT_SILU, F16>(D, g, st, "fc1");
    else launch_thin<OP_FC1, HEXA_ACT_GELU_TANH, F16>(D, g, st, "fc1");
}

template <bool F16>
static hipError_t fwd_impl(const MoeDims& D, const bf16_t* x, const bf16_t* W1, const bf16_t* b1,
                           const bf16_t* W2, const bf16_t* b2, const hexa_moe_idx& idx,
                           const MoeWorkspace& ws, hipStream_t st) {
    GemmArgs g{};
    g.offsets = idx.offsets; g.perm = idx.perm; g.topk = D.k; g.E = D.E;
    g.streamed = streamed(D);
    use_lists(D, ws, g);
    // the backward pass that may follow reads the lists too
    if (!(small_fc1(D) && small_fc2(D) && small_bwd2(D) && small_bwd1(D))) {
        ProfScope ps(st, "worklists");
        hipLaunchKernelGGL(build_worklists, dim3(1), dim3(1024), 0, st, idx.offsets, D.E, wgrad_chunk_len(D),
                           ws.worklist, g.rt_cap, D.d, D.f);
    }
    g.A = x; g.a_rows = D.T; g.B = W1; g.bias = b1; g.out0 = ws.pre; g.out1 = ws.h; g.K = D.d; g.N = D.f;
    if (thin_fc1(D)) launch_thin_fc1<F16>(D, g, st);
    else if (small_fc1(D)) launch_fc1<SMALL, F16>(D, g, st);
    else launch_fc1<BIG, F16>(D, g, st);
    g.A = (const bf16_t*)ws.h; g.B = W2; g.bias = b2; g.out0 = ws.o; g.out1 = nullptr; g.K = D.f; g.N = D.d;
    if (fc2_shares(D) > 1) {
        g.out0 = ws.fc2part; g.a_rows = D.A; g.share_blocks = fc2_share_blocks(D);
        if (thin_fc2(D)) launch_thin<OP_FC2P, HEXA_ACT_GELU_TANH, F16>(D, g, st, "fc2", fc2_shares(D));
        else launch_rows<SMALL, SMALL, 2, 2, OP_FC2P, HEXA_ACT_GELU_TANH, F16>(D, g, st, "fc2", fc2_shares(D));
    } else if (thin_fc2(D)) launch_thin<OP_FC2, HEXA_ACT_GELU_TANH, F16>(D, g, st, "fc2");
    else if (small_fc2(D)) launch_rows<SMALL, SMALL, 2, 2, OP_FC2, HEXA_ACT_GELU_TANH, F16>(D, g, st, "fc2");
    else launch_rows<BIG, BIG, 2, 2, OP_FC2, HEXA_ACT_GELU_TANH, F16>(D, g, st, "fc2");
    return hipGetLastError();
}

template <bool F16>
static hipError_t bwd_impl(const MoeDims& D, const bf16_t* x, const bf16_t* W1, const bf16_t* W2,
                           const hexa_moe_idx& idx, const MoeWorkspace& ws, float* dW1, float* dW2,
                           hipStream_t st) {
    const bool small2 = small_bwd2(D), small1 = small_bwd1(D);
    GemmArgs g{};
    g.offsets = idx.offsets; g.perm = idx.perm; g.topk = D.k; g.E = D.E;
    use_lists(D, ws, g);
    g.chunk_len = wgrad_chunk_len(D);
    // 2nd linear layer: dpre = (do W2^T) * F'(pre)  and  dW2[e] = h^T do
    GemmArgs r = g, t = g;
    r.A = (const bf16_t*)ws.dout; r.B = W2; r.pre_in = (const bf16_t*)ws.pre; r.out0 = ws.dpre;
    r.colpart = ws.colpart1; r.K = D.d; r.N = D.f; r.token_first = token_first(D, r.K, r.N);
    t.A = (const bf16_t*)ws.h; t.B = (const bf16_t*)ws.dout; t.out0 = dW2; t.kpart = ws.kpart2; t.M = D.f; t.N = D.d;
    if (small2) launch_pair<SMALL, SMALL, 2, 2, OP_DGRAD2, OP_WGRAD2, F16>(D, r, t, st, "bwd_fc2");
    else launch_pair<BIG, BIG, 2, 2, OP_DGRAD2, OP_WGRAD2, F16>(D, r, t, st, "bwd_fc2");
    // 1st linear layer: dxp = dpre W1^T  and  dW1[e] = x[perm/k]^T dpre
    r = g; t = g;
    r.A = (const bf16_t*)ws.dpre; r.B = W1; r.out0 = ws.dxp; r.K = D.f; r.N = D.d; r.token_first = token_first(D, r.K, r.N);
    t.A = x; t.a_rows = D.T; t.rowoff = ws.rowoff;
    t.B = (const bf16_t*)ws.dpre; t.out0 = dW1; t.kpart = ws.kpart1; t.M = D.d; t.N = D.f;
    if (small1) launch_pair<SMALL, SMALL, 2, 2, OP_DGRAD1, OP_WGRAD1, F16>(D, r, t, st, "bwd_fc1");
    else launch_pair<BIG, BIG, 2, 2, OP_DGRAD1, OP_WGRAD1, F16>(D, r, t, st, "bwd_fc1");
    return hipGetLastError();
}

// The 16-bit paths: all pointers are raw 16-bit storage, bf16 or (f16 = true) IEEE fp16.
hipError_t launch_bf16_fwd(const MoeDims& D, const bf16_t* x, const bf16_t* W1, const bf16_t* b1,
                           const bf16_t* W2, const bf16_t* b2, const hexa_moe_idx& idx,
                           const MoeWorkspace& ws, hipStream_t st, bool f16) {
    return f16 ? fwd_impl<true>(D, x, W1, b1, W2, b2, idx, ws, st)
               : fwd_impl<false>(D, x, W1, b1, W2, b2, idx, ws, st);
}

hipError_t launch_bf16_bwd(const MoeDims& D, const bf16_t* x, const bf16_t* W1, const bf16_t* W2,
                           const hexa_moe_idx& idx, const MoeWorkspace& ws, float* dW1, float* dW2,
                           hipStream_t st, bool f16) {
    return f16 ? bwd_impl<true>(D, x, W1, W2, idx, ws, dW1, dW2, st)
               : bwd_impl<false>(D, x, W1, W2, idx, ws, dW1, dW2, st);
}
