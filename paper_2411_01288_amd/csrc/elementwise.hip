// Bandwidth-bound steps around the contractions:
//   combine_rows   y_t  = sum_j gate[t,j] * o[inv[t*k+j]]          (top-k sum of App. B Table 5 row 3,
//                                                                    done as a gather in fixed slot order
//                                                                    instead of the paper's atomicAdd)
//   bwd_prologue   do_p = gate_a * dY_t  (a = perm[p]) ; dgate_a = <dY_t, o_p> ; db2 partials ; WGRAD1's row offsets
//   bwd_finish     dx_t = sum_j dxp[inv[t*k+j]] (Table 5 row 10, sum over the k slots) ; second stage of the
//                  bias gradients (ESS, Sec. 3.1 item 2; App. B Alg. 3) ; second stage of split weight gradients
#include "common.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Vec;   // access to 4 floats or 8 16-bit values of a row, `nv` of which exist
template <> struct Vec<float> {
    static constexpr int N = 4;      // (rows of any length: dword-aligned)
    typedef f32x4 Raw;               // a chunk as loaded
    __device__ static Raw load_raw(const float* p, int nv) { return load4(p, nv); }
    __device__ static void unpack(const Raw& q, float (&v)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = q[i];
    }
    __device__ static void store(float* p, const float (&v)[4], int nv) {
        store4(p, f32x4{v[0], v[1], v[2], v[3]}, nv);
    }
};
// (16-bit rows are multiples of 64 elements: a chunk exists whole or not at all)
template <> struct Vec<bf16_t> {
    static constexpr int N = 8;
    typedef u32x4 Raw;
    __device__ static Raw load_raw(const bf16_t* p, int) { return *reinterpret_cast<const u32x4*>(p); }
    __device__ static void unpack(const Raw& q, float (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) unpack2<false>(q[i], v[2 * i], v[2 * i + 1]);
    }
    __device__ static Raw pack(const float (&v)[8]) {
        return Raw{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
    }
    __device__ static void store(bf16_t* p, const float (&v)[8], int) { *reinterpret_cast<Raw*>(p) = pack(v); }
};
template <> struct Vec<f16_t> {
    static constexpr int N = 8;
    typedef u32x4 Raw;
    __device__ static Raw load_raw(const f16_t* p, int) { return *reinterpret_cast<const u32x4*>(p); }
    __device__ static void unpack(const Raw& q, float (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) unpack2<true>(q[i], v[2 * i], v[2 * i + 1]);
    }
    __device__ static Raw pack(const float (&v)[8]) {
        return Raw{pack_h2(v[0], v[1]), pack_h2(v[2], v[3]), pack_h2(v[4], v[5]), pack_h2(v[6], v[7])};
    }
    __device__ static void store(f16_t* p, const float (&v)[8], int) { *reinterpret_cast<Raw*>(p) = pack(v); }
};

// One thread per VN consecutive columns of one token; workgroup `block` of the combination.  The rows of two
// slots are fetched together (their positions are loads themselves); the sum runs in slot order.
template <typename T>
__device__ __forceinline__ void combine_block(uint32_t block, int T_, int d, int k, const T* __restrict__ src,
                                              const int32_t* __restrict__ inv,
                                              const float* __restrict__ gate,  // NULL: plain sum
                                              T* __restrict__ dst) {
    constexpr int VN = Vec<T>::N;
    const uint32_t per_row = (uint32_t)ceil_div(d, VN);
    const uint32_t gid = block * 256u + threadIdx.x;   // (a grid has less than 2^32 threads)
    const uint32_t t = gid / per_row;
    if (t >= (uint32_t)T_) return;
    const int c = (int)(gid - t * per_row) * VN;
    float acc[VN];
#pragma unroll
    for (int i = 0; i < VN; ++i) acc[i] = 0.f;
    for (int j = 0; j < k; j += 2) {
        const size_t a = (size_t)t * k + j;
        const bool two = j + 1 < k;
        const int p0 = inv[a], p1 = two ? inv[a + 1] : -1;   // -1: a dropped assignment
        const float g0 = gate ? gate[a] : 1.f, g1 = gate && two ? gate[a + 1] : 1.f;
        typename Vec<T>::Raw q0{}, q1{};
        if (p0 >= 0) q0 = Vec<T>::load_raw(src + (size_t)p0 * d + c, d - c);
        if (p1 >= 0) q1 = Vec<T>::load_raw(src + (size_t)p1 * d + c, d - c);
        float v0[VN], v1[VN];
        Vec<T>::unpack(q0, v0);
        Vec<T>::unpack(q1, v1);
        if (p0 >= 0) {
#pragma unroll
            for (int q = 0; q < VN; ++q) acc[q] += g0 * v0[q];
        }
        if (p1 >= 0) {
#pragma unroll
            for (int q = 0; q < VN; ++q) acc[q] += g1 * v1[q];
        }
    }
    Vec<T>::store(dst + (size_t)t * d + c, acc, d - c);
}

template <typename T>
inline uint32_t combine_blocks(const MoeDims& D) {
    return (uint32_t)(((long long)D.T * ceil_div(D.d, Vec<T>::N) + 255) / 256);
}

template <typename T>
__global__ __launch_bounds__(256) void combine_rows(int T_, int d, int k, const T* __restrict__ src,
                                                    const int32_t* __restrict__ inv,
                                                    const float* __restrict__ gate, T* __restrict__ dst) {
    combine_block<T>(blockIdx.x, T_, d, k, src, inv, gate, dst);
}

// The same for an FC2 that ran in shares of K: adds the shares' sums in order, rounds, stores the expert outputs o
// that the backward pass reads, and combines the rounded values.
template <typename T>
__global__ __launch_bounds__(256) void combine_split(int T_, int d, int k, int shares, size_t share_elems,
                                                     const float* __restrict__ part,
                                                     const int32_t* __restrict__ inv, const float* __restrict__ gate,
                                                     T* __restrict__ o, T* __restrict__ y) {
    constexpr int VN = Vec<T>::N;
    const uint32_t per_row = (uint32_t)(d / VN);
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
    const uint32_t t = gid / per_row;
    if (t >= (uint32_t)T_) return;
    const int c = (int)(gid - t * per_row) * VN;
    float acc[VN];
#pragma unroll
    for (int i = 0; i < VN; ++i) acc[i] = 0.f;
    for (int j = 0; j < k; ++j) {
        const size_t a = (size_t)t * k + j;
        const int p = inv[a];
        if (p < 0) continue;   // dropped assignment
        const float g = gate[a];
        const float* src = part + (size_t)p * d + c;
        float v[VN];
#pragma unroll
        for (int i = 0; i < VN; ++i) v[i] = 0.f;
        for (int s0 = 0; s0 < shares; s0 += 4) {
            f32x4 q[4][VN / 4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < VN / 4; ++h) {
                    q[u][h] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (s0 + u < shares) q[u][h] = *reinterpret_cast<const f32x4*>(src + (s0 + u) * share_elems + 4 * h);
                }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < VN; ++i) v[i] += q[u][i / 4][i % 4];
        }
        const typename Vec<T>::Raw r = Vec<T>::pack(v);
        *reinterpret_cast<typename Vec<T>::Raw*>(o + (size_t)p * d + c) = r;
        Vec<T>::unpack(r, v);
#pragma unroll
        for (int i = 0; i < VN; ++i) acc[i] += g * v[i];
    }
    Vec<T>::store(y + (size_t)t * d + c, acc, VN);
}

// ---------------------------------------------------------------------------------------------
// Backward prologue: dout, dgate and the fc2 bias gradient's partial sums in one pass over dY and o (ESS,
// Sec. 3.1 item 2; Table 5 row 4), plus two small jobs in workgroups of their own.
// ---------------------------------------------------------------------------------------------
struct PrologueArgs {
    const void* dY; const void* o; void* dout;
    const int32_t* perm; const int32_t* offsets; const int32_t* inv;
    const float* gate;
    float* dgate;          // or NULL
    float* partial;        // [tiles][d] column sums of a tile's rows
    uint32_t* rowoff;      // row-offset table (16-bit types), or NULL
    int A, d, k, E, T;
    int tile_rows;         // rows per workgroup, a power of two, 16 ... 128
    int tile_blocks;       // workgroups [0, tile_blocks) are tiles, the others side jobs
    int step;              // layout of the row-offset table
};

// Zero gate gradients of dropped assignments, and the row-offset table of the gathered token contraction
// (WGRAD1 reads x[perm[p] / k] for perm position p; ESTMM, App. B Alg. 4, takes its tokens through the
// re-index vector the same way).  In the table, expert e's part starts at entry offsets[e] + 64 e and is cut
// into blocks of 64 rows (the K-blocks of the contraction; a chunk starts on a block boundary); inside a
// block, entry (64/step) j + i belongs to row step i + j, the transposed order in which a lane of the
// contraction's staging instructions needs them.  An entry is the byte offset of the token's row in x;
// entries past the segment's end hold an offset behind the last row of x, which the buffer range check turns
// into zeros.
__device__ __forceinline__ void prologue_side_jobs(const PrologueArgs& a, int block) {
    const uint32_t g = (uint32_t)block * 256u + threadIdx.x;   // (A + 64 E may pass 2^31)
    if (a.dgate && g < (uint32_t)a.A && a.inv[g] < 0) a.dgate[g] = 0.f;
    if (!a.rowoff || g >= (uint32_t)a.A + 64u * (uint32_t)a.E) return;
    int lo = 0, hi = a.E - 1;                       // the last expert whose part starts at or before g
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((uint32_t)a.offsets[mid] + 64u * (uint32_t)mid <= g) lo = mid; else hi = mid - 1;
    }
    const int b = a.offsets[lo], n = a.offsets[lo + 1] - b;
    const int local = (int)(g - ((uint32_t)b + 64u * (uint32_t)lo));
    const int s = local & 63;
    const int per = 64 / a.step;
    const int r = (local & ~63) + a.step * (s % per) + s / per;
    const uint32_t row_bytes = (uint32_t)a.d * 2u;
    a.rowoff[g] = (uint32_t)(r < n ? a.perm[b + r] / a.k : a.T) * row_bytes;
}

// One workgroup per segment tile.  A group of G lanes (a whole wavefront, or 16 lanes where rows are short)
// takes a row at a time, NS chunks of VN columns per lane, and the tile's rows go round over the wavefronts:
// the column sums of do = gate * dY (unrounded) stay in a lane's registers, <dY_t, o_p> is a sum over the
// group, and the four wavefronts' column sums meet in LDS, added in wavefront order.  Which assignment a row is, its
// token and its gate are looked up for all rows of a wavefront at once, so that the only chain of latencies per
// tile is offsets -> perm -> gate -> rows.  Workgroups past the last tile zero the rows past the last segment
// (they exist only when expert ids were dropped).
template <typename T, int NS, int G>
__global__ __launch_bounds__(256) void bwd_prologue_tiles(PrologueArgs a) {
    constexpr int VN = Vec<T>::N;
    constexpr int NG = 64 / G;                 // rows per wavefront at a time
    constexpr int COLS = NS * G * VN;          // columns per sweep
    constexpr int U = NS >= 4 ? 2 : 4;         // rows in flight per group
    __shared__ __align__(16) float part[4][COLS];
    if ((int)blockIdx.x >= a.tile_blocks) return prologue_side_jobs(a, (int)blockIdx.x - a.tile_blocks);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gl = lane % G, gr = lane / G;
    const T* dY = (const T*)a.dY;
    const T* o = (const T*)a.o;
    T* dout = (T*)a.dout;
    const SegTile s = seg_tile_find_wave(a.offsets, a.E, a.tile_rows, blockIdx.x);
    if (s.e < 0) {
        const int ntiles = seg_tiles_total_wave(a.offsets, a.E, a.tile_rows);
        const long long r0 = (long long)a.offsets[a.E] + (long long)((int)blockIdx.x - ntiles) * a.tile_rows;
        float z[VN];
#pragma unroll
        for (int q = 0; q < VN; ++q) z[q] = 0.f;
        for (long long r = r0; r < r0 + a.tile_rows && r < a.A; ++r)
            for (int c = tid * VN; c < a.d; c += 256 * VN) Vec<T>::store(dout + (size_t)r * a.d + c, z, a.d - c);
        return;
    }
    // row number n of this wavefront is row 4 NG (n / NG) + NG wave + n % NG of the tile; lane n looks it up
    const int my_row = 4 * NG * (lane / NG) + NG * wave + lane % NG;
    const int as = my_row < s.rows ? a.perm[s.row0 + my_row] : 0;
    const float gs = a.gate[as];
    const int ts = as / a.k;
    const int trips = ceil_div(max(0, s.rows - NG * wave), 4 * NG);   // rows of this wavefront's first group
    for (int c0 = 0; c0 < a.d; c0 += COLS) {
        float cs[NS][VN];
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int q = 0; q < VN; ++q) cs[i][q] = 0.f;
        for (int i0 = 0; i0 < trips; i0 += U) {
            typename Vec<T>::Raw v[U][NS], ov[U][NS];
            int asg[U], row[U];
            float g[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int n = (i0 + u) * NG + gr;    // (at most 63 for a row that exists)
                int t;
                if constexpr (G == 64) {
                    t = __builtin_amdgcn_readlane(ts, n & 63);
                    asg[u] = __builtin_amdgcn_readlane(as, n & 63);
                    g[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gs), n & 63));
                } else {
                    t = __shfl(ts, n & 63);
                    asg[u] = __shfl(as, n & 63);
                    g[u] = __shfl(gs, n & 63);
                }
                const int r = 4 * NG * (i0 + u) + NG * wave + gr;
                row[u] = r < s.rows ? s.row0 + r : -1;
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    const int c = c0 + (i * G + gl) * VN;
                    v[u][i] = ov[u][i] = typename Vec<T>::Raw{};
                    if (row[u] >= 0 && c < a.d) {
                        v[u][i] = Vec<T>::load_raw(dY + (size_t)t * a.d + c, a.d - c);
                        ov[u][i] = Vec<T>::load_raw(o + (size_t)row[u] * a.d + c, a.d - c);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float dot = 0.f;
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    const int c = c0 + (i * G + gl) * VN;
                    float y[VN], x[VN], w[VN];
                    Vec<T>::unpack(v[u][i], y);
                    Vec<T>::unpack(ov[u][i], x);
#pragma unroll
                    for (int q = 0; q < VN; ++q) {
                        dot += y[q] * x[q];
                        w[q] = g[u] * y[q];
                    }
                    if (row[u] >= 0 && c < a.d) {
#pragma unroll
                        for (int q = 0; q < VN; ++q) cs[i][q] += w[q];
                        Vec<T>::store(dout + (size_t)row[u] * a.d + c, w, a.d - c);
                    }
                }
                if (a.dgate) {
                    dot = row_sum16(dot);
                    if constexpr (G == 64) { dot += __shfl_xor(dot, 16); dot += __shfl_xor(dot, 32); }
                    if (gl == 0 && row[u] >= 0) a.dgate[asg[u]] = c0 == 0 ? dot : a.dgate[asg[u]] + dot;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int q = 0; q < VN; ++q) {
                if constexpr (G == 16) { cs[i][q] += __shfl_xor(cs[i][q], 16); cs[i][q] += __shfl_xor(cs[i][q], 32); }
                if (gr == 0) part[wave][(i * G + gl) * VN + q] = cs[i][q];
            }
        __syncthreads();
        for (int c = 4 * tid; c < COLS && c0 + c < a.d; c += 1024) {
            f32x4 sum = *reinterpret_cast<const f32x4*>(&part[0][c]);
#pragma unroll
            for (int w = 1; w < 4; ++w) sum += *reinterpret_cast<const f32x4*>(&part[w][c]);
            store4(a.partial + (size_t)blockIdx.x * a.d + c0 + c, sum, a.d - c0 - c);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// Backward finish: everything that is left once the contractions are done, in one launch.
// ---------------------------------------------------------------------------------------------
struct ColsumJob { const float* partial; float* out; int ncols, bm, parts; };   // `parts` partial rows per bm-row tile
struct SplitJob { const float* kpart; float* out; };
struct FinishArgs {
    const void* dxp; void* dx;
    const int32_t* inv; const int32_t* offsets;
    ColsumJob cols[2];
    SplitJob split[2];
    int T, d, k, E, L;
    unsigned long long mn;       // elements of one expert's weight gradient
    uint32_t cols_end[2];        // workgroups [0, cols_end[0]) are the first column sum, ...
    uint32_t split_blocks;       // then split_blocks for each weight gradient, then the combination
};

// out[e][c] = sum of the expert's partial rows (exact 0 for an empty expert).  The expert's tiles (tile height
// bm, `parts` partial rows per tile) hold rows first*parts .. (first+nt)*parts - 1 of `partial`.  A workgroup is
// 64 columns x 16 slices (a lane owns four columns): slice s adds up a contiguous share of the rows in order, and
// the slice sums are added in slice order, so the result does not depend on scheduling.
__device__ __forceinline__ void colsum_block(const ColsumJob& j, uint32_t block, const int32_t* __restrict__ offsets,
                                             f32x4 (&part)[16][16]) {
    const uint32_t cb = (uint32_t)ceil_div(j.ncols, 64);
    const int e = (int)(block / cb), c0 = (int)(block - e * cb) * 64;
    const int slice = threadIdx.x >> 4, l = threadIdx.x & 15;
    const int c = c0 + 4 * l, nv = j.ncols - c;
    const int first = seg_tiles_total_wave(offsets, e, j.bm);
    const int nrows = ceil_div(offsets[e + 1] - offsets[e], j.bm) * j.parts;
    const int per = ceil_div(nrows, 16);
    const int r0 = min(nrows, slice * per), r1 = min(nrows, r0 + per);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const float* src = j.partial + (size_t)first * j.parts * j.ncols + c;
    for (int i = r0; i < r1; i += 4) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = load4(src + (size_t)(i + u) * j.ncols, i + u < r1 ? nv : 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += v[u];
    }
    part[slice][l] = acc;
    __syncthreads();
    if (slice == 0) {
        for (int q = 1; q < 16; ++q) acc += part[q][l];
        store4(j.out + (size_t)e * j.ncols + c, acc, nv);
    }
}

// Second stage of the split token contraction, plus exact zeros for experts without tokens:
// out[e] = sum_c kpart[slot_e + c] in chunk order when the expert was cut into several chunks (see chunk_count); untouched
// when it had exactly one (the contraction wrote it directly).  The work is cut into pieces of 4096 elements,
// which the workgroups of this job take in turn.
__device__ __forceinline__ void split_block(const SplitJob& j, uint32_t block, uint32_t nblocks,
                                            const int32_t* __restrict__ offsets, int E, int L, size_t mn) {
    const int lane = threadIdx.x & 63;
    const uint32_t pieces = (uint32_t)((mn + 4095) / 4096);
    // a wavefront walks the experts 64 at a time; `before` and `slot` count those in front
    uint32_t before = 0;
    int slot0 = 0;
    for (int e0 = 0; e0 < E; e0 += 64) {
        const int e = e0 + lane;
        const int n = e < E ? offsets[e + 1] - offsets[e] : 0;
        const int nc = chunk_count(n, L), ns = nc > 1 ? nc : 0;
        const int send = wave_scan_incl(ns);
        uint64_t todo = __ballot(e < E && nc != 1);
        for (; todo; todo &= todo - 1, ++before) {
            const int src = __ffsll((long long)todo) - 1;
            const int nch = __builtin_amdgcn_readlane(nc, src);
            const int slot = slot0 + __builtin_amdgcn_readlane(send, src) - nch;
            // the pieces of this expert are numbers before * pieces ... of the whole job
            const unsigned long long base = (unsigned long long)before * pieces;
            uint32_t i = (uint32_t)((block + nblocks - base % nblocks) % nblocks);
            for (; i < pieces; i += nblocks) {
                const size_t at = (size_t)i * 4096 + 4 * threadIdx.x;
                f32x4 s[4];
                int nv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    s[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                    const size_t p = at + 1024 * u;
                    nv[u] = p < mn ? (int)(mn - p < 4 ? mn - p : 4) : 0;
                }
                for (int c = 0; c < nch; ++c) {
                    const float* src_c = j.kpart + (size_t)(slot + c) * mn + at;
                    f32x4 v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = load4(src_c + 1024 * u, nv[u]);
#pragma unroll
                    for (int u = 0; u < 4; ++u) s[u] += v[u];
                }
                float* dst = j.out + (size_t)(e0 + src) * mn + at;
#pragma unroll
                for (int u = 0; u < 4; ++u) store4(dst + 1024 * u, s[u], nv[u]);
            }
        }
        slot0 += __builtin_amdgcn_readlane(send, 63);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void bwd_finish(FinishArgs a) {
    __shared__ f32x4 part[16][16];
    uint32_t b = blockIdx.x;
    if (b < a.cols_end[0]) return colsum_block(a.cols[0], b, a.offsets, part);
    if (b < a.cols_end[1]) return colsum_block(a.cols[1], b - a.cols_end[0], a.offsets, part);
    b -= a.cols_end[1];
    if (b < a.split_blocks) return split_block(a.split[0], b, a.split_blocks, a.offsets, a.E, a.L, (size_t)a.mn);
    b -= a.split_blocks;
    if (b < a.split_blocks) return split_block(a.split[1], b, a.split_blocks, a.offsets, a.E, a.L, (size_t)a.mn);
    b -= a.split_blocks;
    combine_block<T>(b, a.T, a.d, a.k, (const T*)a.dxp, a.inv, nullptr, (T*)a.dx);
}

// Rows per workgroup of the backward prologue: 128 when that still gives 1024 workgroups, fewer (down to 16, four
// per wavefront) on small problems.
int prologue_tile_rows(const MoeDims& D) {
    int r = 128;
    while (r > 16 && D.A / r < 1024) r >>= 1;
    return r;
}

template <typename T, int NS, int G>
void prologue_launch(const PrologueArgs& a, int blocks, hipStream_t st) {
    hipLaunchKernelGGL((bwd_prologue_tiles<T, NS, G>), dim3(blocks), dim3(256), 0, st, a);
}

}  // namespace

size_t prologue_partial_rows(const MoeDims& D) { return (size_t)(D.A / prologue_tile_rows(D) + D.E + 1); }
int64_t prologue_blocks(const MoeDims& D, bool rowoff, bool dgate) {
    const int64_t side = rowoff ? (int64_t)D.A + 64 * D.E : dgate ? D.A : 0;
    return (int64_t)prologue_partial_rows(D) + (side + 255) / 256;
}

template <typename T>
hipError_t launch_combine_y(const MoeDims& D, const T* o, const int32_t* inv, const float* gate,
                            T* y, hipStream_t st) {
    ProfScope ps(st, "combine_y");
    hipLaunchKernelGGL(combine_rows<T>, dim3(combine_blocks<T>(D)), dim3(256), 0, st, D.T, D.d, D.k, o, inv, gate, y);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_combine_split(const MoeDims& D, const float* part, int shares, const int32_t* inv,
                                const float* gate, T* o, T* y, hipStream_t st) {
    ProfScope ps(st, "combine_y");
    hipLaunchKernelGGL(combine_split<T>, dim3(combine_blocks<T>(D)), dim3(256), 0, st, D.T, D.d, D.k, shares,
                       (size_t)D.A * D.d, part, inv, gate, o, y);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_bwd_prologue(const MoeDims& D, const T* dY, const float* gate, const hexa_moe_idx& idx,
                               const MoeWorkspace& ws, float* dgate, hipStream_t st) {
    constexpr int VN = Vec<T>::N;
    PrologueArgs a{};
    a.dY = dY; a.o = ws.o; a.dout = ws.dout;
    a.perm = idx.perm; a.offsets = idx.offsets; a.inv = idx.inv; a.gate = gate; a.dgate = dgate;
    a.partial = ws.colpart2; a.rowoff = ws.rowoff;
    a.A = D.A; a.d = D.d; a.k = D.k; a.E = D.E; a.T = D.T;
    a.tile_rows = prologue_tile_rows(D);
    a.tile_blocks = (int)prologue_partial_rows(D);
    a.step = a.rowoff ? gemm_rowoff_step(D) : 64;
    const int blocks = (int)prologue_blocks(D, a.rowoff != nullptr, dgate != nullptr);
    ProfScope ps(st, "bwd_prologue");
    if (D.d <= 16 * VN) prologue_launch<T, 1, 16>(a, blocks, st);
    else if (D.d <= 64 * VN) prologue_launch<T, 1, 64>(a, blocks, st);
    else if (D.d <= 128 * VN) prologue_launch<T, 2, 64>(a, blocks, st);
    else prologue_launch<T, 4, 64>(a, blocks, st);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_bwd_finish(const MoeDims& D, const hexa_moe_idx& idx, const MoeWorkspace& ws, int dgrad2_row_tile,
                             int L, T* dx, float* dW1, float* db1, float* dW2, float* db2, hipStream_t st) {
    FinishArgs a{};
    a.dxp = ws.dxp; a.dx = dx; a.inv = idx.inv; a.offsets = idx.offsets;
    a.T = D.T; a.d = D.d; a.k = D.k; a.E = D.E; a.L = L;
    a.mn = (unsigned long long)D.d * D.f;
    a.cols[0] = ColsumJob{ws.colpart1, db1, D.f, dgrad2_row_tile, kColpartRows};
    a.cols[1] = ColsumJob{ws.colpart2, db2, D.d, prologue_tile_rows(D), 1};
    a.split[0] = SplitJob{ws.kpart2, dW2};
    a.split[1] = SplitJob{ws.kpart1, dW1};
    a.cols_end[0] = (uint32_t)D.E * ceil_div(D.f, 64);
    a.cols_end[1] = a.cols_end[0] + (uint32_t)D.E * ceil_div(D.d, 64);
    const unsigned long long pieces = (a.mn + 4095) / 4096 * D.E;
    a.split_blocks = (uint32_t)(pieces < 1024 ? pieces : 1024);
    ProfScope ps(st, "bwd_finish");
    hipLaunchKernelGGL(bwd_finish<T>, dim3(a.cols_end[1] + 2 * a.split_blocks + combine_blocks<T>(D)), dim3(256), 0, st, a);
    return hipGetLastError();
}

#define INSTANTIATE(T)                                                                              \
    template hipError_t launch_combine_y<T>(const MoeDims&, const T*, const int32_t*,              \
                                            const float*, T*, hipStream_t);                        \
    template hipError_t launch_bwd_prologue<T>(const MoeDims&, const T*, const float*,             \
                                               const hexa_moe_idx&, const MoeWorkspace&, float*,   \
                                               hipStream_t);                                       \
    template hipError_t launch_bwd_finish<T>(const MoeDims&, const hexa_moe_idx&, const MoeWorkspace&, int, int, T*, \
                                             float*, float*, float*, float*, hipStream_t);
template hipError_t launch_combine_split<bf16_t>(const MoeDims&, const float*, int, const int32_t*, const float*, bf16_t*, bf16_t*,
                                                 hipStream_t);
template hipError_t launch_combine_split<f16_t>(const MoeDims&, const float*, int, const int32_t*, const float*, f16_t*, f16_t*,
                                                 hipStream_t);
INSTANTIATE(float)
INSTANTIATE(bf16_t)
INSTANTIATE(f16_t)
