// Shared device helpers and the internal launcher interface of libhexa_moe.
// gfx950 (CDNA4) only: 64-wide wavefronts, bf16 / fp16 MFMA, 160 KB LDS per CU.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/hexa_moe.h"
#include "segments.h"

typedef uint16_t bf16_t;  // raw bfloat16 bits

// two floats -> two bf16 (round to nearest even) in one word: a single v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf2(float lo, float hi) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

typedef _Float16 f16_t;   // IEEE binary16

// two floats -> two fp16 (round to nearest even) in one word
__device__ __forceinline__ uint32_t pack_h2(float lo, float hi) {
    typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));
}
// one word of two 16-bit values -> two floats
template <bool F16>
__device__ __forceinline__ void unpack2(uint32_t w, float& lo, float& hi) {
    if constexpr (F16) {
        typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
        const f16x2_t h = __builtin_bit_cast(f16x2_t, w);
        lo = (float)h[0]; hi = (float)h[1];
    } else {
        lo = __uint_as_float(w << 16); hi = __uint_as_float(w & 0xffff0000u);
    }
}
template <bool F16>
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    if constexpr (F16) return pack_h2(lo, hi);
    else return pack_bf2(lo, hi);
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// GELU, tanh form (the activation F between the two MLPs; App. B Table 5 rows 2, 7).
#define HEXA_GELU_C 0.7978845608028654f
#define HEXA_GELU_A 0.044715f

// A segment tile: `rows` (<= BM) consecutive rows of perm order that all belong
// to expert `e`, starting at perm position `row0`.
struct SegTile { int e, row0, rows; };

// Look-ups over the expert segments by a whole wavefront (all 64 lanes active), an expert per lane: a scan over
// the lanes instead of a walk over the experts, whose loads a workgroup would wait for one after the other.
// Inclusive scan over the 64 lanes with the data-parallel moves of the vector unit (within rows of 16, then
// lane 15 of rows 0 and 2 into the row behind, then lane 31 into the upper half).
__device__ __forceinline__ int wave_scan_incl(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}
// Number of BM-row tiles over the first E expert segments (each segment tiled on its own, so no tile straddles
// two experts and none is padded to a capacity).
__device__ __forceinline__ int seg_tiles_total_wave(const int32_t* __restrict__ offsets, int E, int BM) {
    const int lane = threadIdx.x & 63;
    int v = 0;
    for (int e = lane; e < E; e += 64) v += ceil_div(offsets[e + 1] - offsets[e], BM);
    return __builtin_amdgcn_readlane(wave_scan_incl(v), 63);
}

// Map tile number `tile` (0-based over all segments, expert-major; wave-uniform) to its segment tile.
// Returns e = -1 when `tile` is past the last one.
__device__ __forceinline__ SegTile seg_tile_find_wave(const int32_t* __restrict__ offsets, int E, int BM,
                                                      int tile) {
    const int lane = threadIdx.x & 63;
    int acc = 0;
    for (int e0 = 0; e0 < E; e0 += 64) {
        const int e = e0 + lane;
        const int b = e < E ? offsets[e] : 0, n = e < E ? offsets[e + 1] - b : 0;
        const int nt = ceil_div(n, BM);
        const int end = acc + wave_scan_incl(nt);
        const uint64_t hit = __ballot(end > tile);
        if (hit) {
            const int src = __ffsll((long long)hit) - 1;
            const int r0 = (tile - (__builtin_amdgcn_readlane(end, src) - __builtin_amdgcn_readlane(nt, src))) * BM;
            return SegTile{e0 + src, __builtin_amdgcn_readlane(b, src) + r0,
                           min(BM, __builtin_amdgcn_readlane(n, src) - r0)};
        }
        acc = __builtin_amdgcn_readlane(end, 63);
    }
    return SegTile{-1, 0, 0};
}

// Token-contraction item number `item` (expert-major, then chunks): expert, perm rows
// [beg, end) and, for an expert of several chunks, the number of its partial-tile buffer (-1 otherwise).
// e = -1 past the last item; experts without rows have none.
struct ChunkItem { int e, beg, end, slot; };
__device__ __forceinline__ ChunkItem chunk_find_wave(const int32_t* __restrict__ offsets, int E, int L, int item) {
    const int lane = threadIdx.x & 63;
    int acc = 0, sacc = 0;
    for (int e0 = 0; e0 < E; e0 += 64) {
        const int e = e0 + lane;
        const int b = e < E ? offsets[e] : 0, n = e < E ? offsets[e + 1] - b : 0;
        const int nc = chunk_count(n, L), ns = nc > 1 ? nc : 0;
        const int end = acc + wave_scan_incl(nc), send = sacc + wave_scan_incl(ns);
        const uint64_t hit = __ballot(end > item);
        if (hit) {
            const int src = __ffsll((long long)hit) - 1;
            const int chunks = __builtin_amdgcn_readlane(nc, src);
            const int c = item - (__builtin_amdgcn_readlane(end, src) - chunks);
            const int beg = __builtin_amdgcn_readlane(b, src), rows = __builtin_amdgcn_readlane(n, src);
            const int slots = __builtin_amdgcn_readlane(ns, src);
            return ChunkItem{e0 + src, beg + chunk_start(rows, chunks, c), beg + chunk_start(rows, chunks, c + 1),
                             slots ? __builtin_amdgcn_readlane(send, src) - slots + c : -1};
        }
        acc = __builtin_amdgcn_readlane(end, 63);
        sacc = __builtin_amdgcn_readlane(send, 63);
    }
    return ChunkItem{-1, 0, 0, -1};
}

// Slot `slot` of a token contraction whose items have `tiles` output tiles each: the item, and the tile, one of an
// eighth of the item's tiles (neighbouring ones) per XCD; -1: none.  Where the tiles are no multiple of eight, which XCDs
// take one more goes round from item to item.  (The fp32 path's deal; the 16-bit path's, in deal.h, leaves no slots without a tile.)
__device__ __forceinline__ int token_item_of(int slot, int tiles, int& tile) {
    const int per = ceil_div(tiles, kXcds), loc = slot / kXcds;
    const int item = loc / per;
    const int x = (slot + item) % kXcds;
    const int first = x * tiles / kXcds, end = (x + 1) * tiles / kXcds;
    tile = first + loc - item * per;
    return tile < end ? item : -1;
}

// ---- four consecutive floats of a row of any length (dword-aligned) ----
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
// the first `nv` exist (the others read as zero and are not touched)
__device__ __forceinline__ f32x4 load4(const float* p, int nv) {
    if (nv >= 4) return *reinterpret_cast<const f32x4u*>(p);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (nv > 0) v[0] = p[0];
    if (nv > 1) v[1] = p[1];
    if (nv > 2) v[2] = p[2];
    return v;
}
__device__ __forceinline__ void store4(float* p, f32x4 v, int nv) {
    if (nv >= 4) { *reinterpret_cast<f32x4u*>(p) = v; return; }
    if (nv > 0) p[0] = v[0];
    if (nv > 1) p[1] = v[1];
    if (nv > 2) p[2] = v[2];
}
// sum over the 16 lanes of a DPP row (every lane gets it)
__device__ __forceinline__ float row_sum16(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));   // row_ror:8
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));
    return v;
}

// ---- optional per-kernel timing (off unless hexa_moe_profile_enable(1); bench_support.hip) ----
// A ProfScope brackets one kernel launch with two HIP events on the launch stream.
void prof_begin(hipStream_t st, const char* label);
void prof_end(hipStream_t st, const char* label);
struct ProfScope {
    hipStream_t st;
    const char* label;
    ProfScope(hipStream_t s, const char* l) : st(s), label(l) { prof_begin(s, l); }
    ~ProfScope() { prof_end(st, label); }
};

// ---- internal launchers (one per translation unit), all asynchronous on `st` ----
struct MoeDims { int T, d, f, E, k, A, act; };

// Host-side validation of a shape (sizes, dtype, activation, the size rules of the 16-bit path);
// fills D on HEXA_OK.  Touches no device.
hexa_status hexa_check_shape(const hexa_moe_shape* s, MoeDims* D);

constexpr int kMaxDevices = 64;   // per-device state of the library is kept in arrays of this length

// Sets the launch attributes of every contraction kernel (160 or 80 KB of dynamic LDS) on the current
// device.  Called once per device by the entry points, outside any stream capture.
hipError_t gemm_bf16_device_init();
hipError_t f32_device_init();   // 72 KB

// saved + staging regions inside the caller's workspace (device pointers)
struct MoeWorkspace {
    void* pre;      // [A,f] elem   F'(pre), perm order                 (saved by fwd)
    void* h;        // [A,f] elem   activations, perm order            (saved by fwd)
    void* o;        // [A,d] elem   per-assignment expert outputs      (saved by fwd)
    float* fc2part; // [shares,A,d] f32 unrounded sums of a split FC2 (16-bit path, few rows; fwd staging)
    void* dout;     // [A,d] elem   gate * dY gathered to perm order   (bwd staging)
    void* dpre;     // [A,f] elem                                       (bwd staging)
    void* dxp;      // [A,d] elem   per-assignment input gradients     (bwd staging)
    uint32_t* rowoff; // [A + 64 E]  byte offsets in x of the token rows, in the order WGRAD1 fetches them (16-bit path; bwd staging)
    float* colpart1; // [rows, f] f32 partial column sums for db1         (bwd staging)
    float* colpart2; // [rows, d] f32 partial column sums for db2         (bwd staging)
    float* kpart1;  // [slots, d, f] f32 partial dW1 tiles of experts cut into chunks   (bwd staging)
    float* kpart2;  // [slots, f, d] f32 partial dW2 tiles
    int32_t* worklist; // tiles and items of the 256x256 contraction kernels (saved by fwd, read by bwd)
    size_t total_bytes;
};

// tile sizes of the launches fc1, fc2, bwd_fc2, bwd_fc1
void gemm_tile_classes(const MoeDims& D, int (&tile)[4]);
void gemm_thin(const MoeDims& D, bool (&thin)[2]);  // whether fc1 and fc2 take 32x128 tiles instead
void f32_tile_classes(const MoeDims& D, int (&tile)[4]);
void f32_wide(const MoeDims& D, bool (&wide)[4]);   // which of them take 128x64 tiles
int gemm_dgrad2_row_tile(const MoeDims& D);   // rows of a DGRAD2 tile of the 16-bit path
int f32_dgrad2_row_tile(const MoeDims& D);    // rows of a DGRAD2 tile of the fp32 path
constexpr int kColpartRows = 2;               // DGRAD2 writes this many column-sum partial rows per row tile
int wgrad_chunk_len(const MoeDims& D);        // tokens per split-K chunk of the 16-bit path (host policy)
int f32_chunk_len(const MoeDims& D);          // ... of the fp32 path
// The most partial-tile buffers that any routing needs.  An expert of L + L/8 + 1 rows is the smallest that is cut, into
// two chunks, and every L rows more are one chunk more (see chunk_count): as many experts as possible that are just
// cut, and the rows left over on one of them.
inline size_t split_slots(const MoeDims& D, int L) {
    const long long cut = (long long)L + L / 8 + 1;
    const long long n = D.A / cut < D.E ? D.A / cut : D.E;
    return n > 0 ? (size_t)(2 * n + (D.A - n * cut) / L) : 0;
}
size_t gemm_worklist_ints(const MoeDims& D);  // int32 entries of MoeWorkspace::worklist
int fc2_shares(const MoeDims& D);             // shares of K in which the 16-bit path runs FC2 (1: unsplit)
int gemm_rowoff_step(const MoeDims& D);       // layout of MoeWorkspace::rowoff that the launch of this shape reads
size_t prologue_partial_rows(const MoeDims& D);   // rows of MoeWorkspace::colpart2
int64_t prologue_blocks(const MoeDims& D, bool rowoff, bool dgate);   // workgroups: tiles, then side jobs

hipError_t launch_index(const MoeDims& D, const int32_t* topk_idx, hexa_moe_idx out, void* scratch,
                        hipStream_t st);
size_t index_scratch_bytes(const MoeDims& D);
void index_chunks(const MoeDims& D, int64_t* ids, int64_t* chunks);   // ids per workgroup, workgroups
hipError_t launch_padded_index(const MoeDims& D, const hexa_moe_idx& idx, int blk, long long cap,
                               int32_t* v, int32_t* idx_, hipStream_t st);

template <typename T>
hipError_t launch_combine_y(const MoeDims& D, const T* o, const int32_t* inv, const float* gate,
                            T* y, hipStream_t st);
// the same from the partial sums of an FC2 in `shares` shares of K, which it also finishes: o = round(sum)
template <typename T>
hipError_t launch_combine_split(const MoeDims& D, const float* part, int shares, const int32_t* inv,
                                const float* gate, T* o, T* y, hipStream_t st);
// dout_p = gate_a dY_t, dgate_a = <dY_t, o_p>, for a = perm[p], and partial column sums of gate_a dY_t for db2
// (ESS) in ws.colpart2; 16-bit types: also the row-offset table of WGRAD1
template <typename T>
hipError_t launch_bwd_prologue(const MoeDims& D, const T* dY, const float* gate, const hexa_moe_idx& idx,
                               const MoeWorkspace& ws, float* dgate, hipStream_t st);
// dx_t = sum over the k slots of dxp; db1, db2 from their partial rows; dW1, dW2 of the experts that were cut into
// chunks of L rows, and zeros for experts without rows
template <typename T>
hipError_t launch_bwd_finish(const MoeDims& D, const hexa_moe_idx& idx, const MoeWorkspace& ws, int dgrad2_row_tile,
                             int L, T* dx, float* dW1, float* db1, float* dW2, float* db2, hipStream_t st);

// fp32 path (fp32 matrix instructions, or bf16 ones on operands in three parts)
hipError_t launch_f32_fwd(const MoeDims& D, const float* x, const float* W1, const float* b1,
                          const float* W2, const float* b2, const hexa_moe_idx& idx,
                          const MoeWorkspace& ws, hipStream_t st);
hipError_t launch_f32_bwd(const MoeDims& D, const float* x, const float* W1, const float* W2,
                          const hexa_moe_idx& idx, const MoeWorkspace& ws, float* dW1, float* dW2,
                          hipStream_t st);

// 16-bit MFMA path: pointers are raw 16-bit storage, bf16 or (f16 = true) IEEE fp16
hipError_t launch_bf16_fwd(const MoeDims& D, const bf16_t* x, const bf16_t* W1, const bf16_t* b1,
                           const bf16_t* W2, const bf16_t* b2, const hexa_moe_idx& idx,
                           const MoeWorkspace& ws, hipStream_t st, bool f16);
hipError_t launch_bf16_bwd(const MoeDims& D, const bf16_t* x, const bf16_t* W1, const bf16_t* W2,
                           const hexa_moe_idx& idx, const MoeWorkspace& ws, float* dW1, float* dW2,
                           hipStream_t st, bool f16);
