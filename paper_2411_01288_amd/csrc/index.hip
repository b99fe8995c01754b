// Re-index build (HEXA-MoE Sec. 3.2; App. B Alg. 1), redesigned for CDNA4.
//
// The paper scatters token ids with one global atomicAdd per token, which makes
// the order inside an expert's segment depend on scheduling.  Here the result is
// the unique stable counting sort of the flat assignment ids, built without any
// order-dependent atomic.  A workgroup owns a contiguous chunk of ids, each of its
// wavefronts a contiguous run of the chunk:
//   1. index_count    (more than one chunk) histograms a chunk (integer adds
//                     commute, so the counts are exact);
//   2. index_scatter  every workgroup adds up the chunks' histograms for itself:
//                     totals (-> offsets) and the share in front of its own chunk;
//                     it counts its wavefronts' runs, which gives each wavefront
//                     its first output position per expert, and re-reads its ids
//                     64 at a time: the rank of an id among equal experts in its
//                     row comes from one ballot per bit of the expert id, rows are
//                     chained through a per-wavefront LDS cursor.
// Bound by launches and by the chain of latencies inside them, not by bytes (3 MB at
// 262144 ids), hence as few launches as possible.
// Segments carry no padding: tiles are cut per segment by the consumers.
#include "common.h"

#include <mutex>

namespace {

// Chunks: one up to kOneChunk ids (a single workgroup, a single launch), else at most kMaxChunks.
constexpr int kOneChunk = 8192;
constexpr int kMaxChunks = 128;

constexpr int kLongChunk = 4096;   // ids from which on the kernels for long chunks are used

struct IndexPlan { int waves, chunk, nchunks; };   // wavefronts per workgroup, ids per chunk

IndexPlan plan_for(const MoeDims& D) {
    IndexPlan p;
    p.waves = D.E <= 512 ? 16 : 8;   // (a wavefront's histogram is E words of LDS)
    const long long unit = 64 * p.waves;
    const long long want = D.A <= kOneChunk ? D.A : ((long long)D.A + kMaxChunks - 1) / kMaxChunks;
    const long long chunk = (want + unit - 1) / unit * unit;
    p.chunk = (int)chunk;
    p.nchunks = (int)((D.A + chunk - 1) / chunk);
    return p;
}

constexpr int kRows = 8;   // rows of 64 ids that a wavefront loads together

// Counts a wavefront's next n rows (at most kRows; ids of -1: none) in an LDS histogram.  Additions to one address are
// made one after the other, so rows of equal ids, the usual ones where routing has collapsed or there is one expert,
// are a single addition.  Only where chunks are long (LONG): index build in us, 2000000 ids on one of 16 experts
// 44 -> 21, 8000000 on one of 64 308 -> 132, one expert 144 -> 52, spread evenly over 64 170 -> 143 (loads of eight rows
// at once in index_count); with a row or two per wavefront the longer code costs more than it saves (9003 ids: 1 us).
__device__ __forceinline__ void count_rows(int32_t* hist, const int (&e)[kRows], int n, int E) {
    const int e0 = __builtin_amdgcn_readfirstlane(e[0]);
    if (__all(e[0] == e0)) {
        bool same = true;
#pragma unroll
        for (int u = 1; u < kRows; ++u) same = same && (u >= n || e[u] == e0);
        if (__all(same)) {
            if ((unsigned)e0 < (unsigned)E && (threadIdx.x & 63) == 0) atomicAdd(&hist[e0], 64 * min(n, kRows));
            return;
        }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u)
        if ((unsigned)e[u] < (unsigned)E) atomicAdd(&hist[e[u]], 1);
}

template <bool LONG>
__global__ __launch_bounds__(1024) void index_count(const int32_t* __restrict__ idx, int A, int E,
                                                    int chunk, int32_t* __restrict__ hist) {
    extern __shared__ int32_t lh[];  // [E]
    for (int i = threadIdx.x; i < E; i += blockDim.x) lh[i] = 0;
    __syncthreads();
    const long long a0 = (long long)blockIdx.x * chunk;
    if constexpr (LONG) {
        const int rows = chunk / 64, waves = blockDim.x / 64, lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
        for (int r0 = wave; r0 < rows; r0 += kRows * waves) {   // rows go round over the wavefronts
            int e[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const int r = r0 + u * waves;
                const long long a = a0 + (long long)r * 64 + lane;
                e[u] = r < rows && a < A ? idx[a] : -1;
            }
            count_rows(lh, e, ceil_div(rows - r0, waves), E);
        }
    } else {
        for (int i = threadIdx.x; i < chunk; i += blockDim.x) {
            const long long a = a0 + i;
            const int e = a < A ? idx[a] : -1;
            if ((unsigned)e < (unsigned)E) atomicAdd(&lh[e], 1);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < E; i += blockDim.x) hist[(size_t)blockIdx.x * E + i] = lh[i];
}

// LDS: [waves][E] run counts, then first output positions; [E] totals, then offsets; [E] ids of earlier chunks
template <int WAVES, bool LONG>
__global__ __launch_bounds__(64 * WAVES) void index_scatter(const int32_t* __restrict__ idx, int A, int E, int bits,
                                                            int chunk, int nchunks,
                                                            const int32_t* __restrict__ hist,
                                                            int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ offsets,
                                                            int32_t* __restrict__ perm,
                                                            int32_t* __restrict__ inv) {
    constexpr int NT = 64 * WAVES;
    constexpr int B = kRows;              // rows of 64 ids whose loads are issued together
    extern __shared__ int32_t lds[];
    __shared__ int32_t s_valid;
    int32_t* run = lds;
    int32_t* tot = lds + WAVES * E;
    int32_t* before = tot + E;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (int i = t; i < (WAVES + 2) * E; i += NT) lds[i] = 0;
    __syncthreads();
    const int rows = chunk / NT;          // rows per wavefront
    const long long a0 = (long long)blockIdx.x * chunk + (long long)wave * rows * 64 + lane;
    auto load_rows = [&](int r0, int (&e)[B]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const long long a = a0 + (long long)(r0 + u) * 64;
            e[u] = r0 + u < rows && a < A ? idx[a] : -1;
        }
    };
    for (int r0 = 0; r0 < rows; r0 += B) {
        int e[B];
        load_rows(r0, e);
        if constexpr (LONG) {
            count_rows(run + wave * E, e, rows - r0, E);
        } else {
#pragma unroll
            for (int u = 0; u < B; ++u)
                if ((unsigned)e[u] < (unsigned)E) atomicAdd(&run[wave * E + e[u]], 1);
        }
    }
    // totals and the share of the chunks in front of this one (integer sums: exact in any order)
    if (nchunks > 1) {
        const int G = max(1, NT / E), cpg = ceil_div(nchunks, G);
        for (int i = t; i < G * E; i += NT) {
            const int e = i % E, c0 = i / E * cpg, c1 = min(nchunks, c0 + cpg);
            int s = 0, f = 0;
            for (int c = c0; c < c1; c += B) {
                int v[B];
#pragma unroll
                for (int u = 0; u < B; ++u) v[u] = c + u < c1 ? hist[(size_t)(c + u) * E + e] : 0;
#pragma unroll
                for (int u = 0; u < B; ++u) { s += v[u]; f += c + u < (int)blockIdx.x ? v[u] : 0; }
            }
            atomicAdd(&tot[e], s);
            atomicAdd(&before[e], f);
        }
    }
    __syncthreads();
    if (nchunks == 1) {
        for (int e = t; e < E; e += NT) {
            int s = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s += run[w * E + e];
            tot[e] = s;
        }
        __syncthreads();
    }
    if (wave == 0) {
        int acc = 0;
        for (int e0 = 0; e0 < E; e0 += 64) {
            const int e = e0 + lane;
            const int n = e < E ? tot[e] : 0;
            const int end = acc + wave_scan_incl(n);
            if (e < E) {
                tot[e] = end - n;
                if (blockIdx.x == 0) { counts[e] = n; offsets[e] = end - n; }
            }
            acc = __builtin_amdgcn_readlane(end, 63);
        }
        if (lane == 0) {
            s_valid = acc;
            if (blockIdx.x == 0) offsets[E] = acc;
        }
    }
    __syncthreads();
    for (int e = t; e < E; e += NT) {
        int pos = tot[e] + before[e];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const int n = run[w * E + e];
            run[w * E + e] = pos;
            pos += n;
        }
    }
    __syncthreads();
    const int n_valid = s_valid;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    volatile int32_t* cursor = run + wave * E;
    for (int r0 = 0; r0 < rows; r0 += B) {
        int e[B];
        load_rows(r0, e);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (r0 + u >= rows) break;
            const long long a = a0 + (long long)(r0 + u) * 64;
            const bool valid = (unsigned)e[u] < (unsigned)E;
            uint64_t same = __ballot(valid);          // lanes with this lane's expert
            for (int q = 0; q < bits; ++q) {
                const uint64_t m = __ballot((e[u] >> q) & 1);
                same &= (e[u] >> q) & 1 ? m : ~m;
            }
            const int rank = __popcll(same & lt_mask), cnt = __popcll(same);
            int b = 0;
            if (valid) b = cursor[e[u]];
            __builtin_amdgcn_wave_barrier();
            if (valid) {
                const int pos = b + rank;
                perm[pos] = (int)a;
                inv[a] = pos;
                if (rank == cnt - 1) cursor[e[u]] = b + cnt;
            } else if (a < A) {
                inv[a] = -1;  // dropped: expert id outside [0, E)
            }
            if (a < A && a >= n_valid) perm[a] = -1;  // tail left empty by dropped ids
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// The paper's padded form of the index (App. B Alg. 1; Sec. 3.2), derived from the unpadded one:
// expert e's sub-vector starts at idx_[e] = sum over e' < e of ceil(n_e' / blk) * blk and holds its
// perm entries followed by -1 up to the next multiple of blk; entries past idx_[E] are -1 too.
// Two launches: the padded starts (one workgroup, E <= 1024 threads), then one thread per entry
// of v, which finds its expert by bisection over the padded starts.
__global__ __launch_bounds__(1024) void padded_starts(const int32_t* __restrict__ offsets, int E, int blk,
                                                      int32_t* __restrict__ idx_) {
    __shared__ int s[1024];
    const int e = threadIdx.x;
    const int n = e < E ? offsets[e + 1] - offsets[e] : 0;
    const int padded = ceil_div(n, blk) * blk;
    s[e] = padded;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {     // inclusive scan
        const int v = e >= off ? s[e - off] : 0;
        __syncthreads();
        s[e] += v;
        __syncthreads();
    }
    if (e < E) idx_[e + 1] = s[e];
    if (e == 0) idx_[0] = 0;
}

__global__ __launch_bounds__(256) void padded_fill(const int32_t* __restrict__ offsets,
                                                   const int32_t* __restrict__ perm,
                                                   const int32_t* __restrict__ idx_, int E, long long cap,
                                                   int32_t* __restrict__ v) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= cap) return;
    int out = -1;
    if (i < idx_[E]) {
        int lo = 0, hi = E;                         // largest e with idx_[e] <= i
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (idx_[mid] <= i) lo = mid; else hi = mid;
        }
        const int r = (int)(i - idx_[lo]);
        if (r < offsets[lo + 1] - offsets[lo]) out = perm[offsets[lo] + r];
    }
    v[i] = out;
}

}  // namespace

hipError_t launch_padded_index(const MoeDims& D, const hexa_moe_idx& idx, int blk, long long cap,
                               int32_t* v, int32_t* idx_, hipStream_t st) {
    ProfScope ps(st, "padded_index");
    hipLaunchKernelGGL(padded_starts, dim3(1), dim3(1024), 0, st, idx.offsets, D.E, blk, idx_);
    hipLaunchKernelGGL(padded_fill, dim3((unsigned)((cap + 255) / 256)), dim3(256), 0, st, idx.offsets,
                       idx.perm, idx_, D.E, cap, v);
    return hipGetLastError();
}

void index_chunks(const MoeDims& D, int64_t* ids, int64_t* chunks) {
    const IndexPlan p = plan_for(D);
    *ids = p.chunk; *chunks = p.nchunks;
}

// What the interface asks for: a word per expert and run of 64 ids (at most 1024 runs).  The chunks need no more.
size_t index_scratch_bytes(const MoeDims& D) {
    const long long per = ((long long)D.A + 64 * 1024 - 1) / (64 * 1024) * 64;
    return align_up((size_t)(((long long)D.A + per - 1) / per) * D.E * sizeof(int32_t), 256);
}

hipError_t launch_index(const MoeDims& D, const int32_t* topk_idx, hexa_moe_idx out, void* scratch,
                        hipStream_t st) {
    const IndexPlan p = plan_for(D);
    int32_t* hist = (int32_t*)scratch;
    int bits = 0;
    while ((1 << bits) < D.E) ++bits;
    const bool lng = p.nchunks > 1 && p.chunk >= kLongChunk;
    if (p.nchunks > 1) {
        ProfScope ps(st, "index_count");
        hipLaunchKernelGGL(lng ? index_count<true> : index_count<false>, dim3(p.nchunks), dim3(1024),
                           D.E * sizeof(int32_t), st, topk_idx, D.A, D.E, p.chunk, hist);
    }
    ProfScope ps(st, "index_scatter");
    const size_t lds = (size_t)(p.waves + 2) * D.E * sizeof(int32_t);
    const auto kern = p.waves == 16 ? (lng ? index_scatter<16, true> : index_scatter<16, false>)
                                    : (lng ? index_scatter<8, true> : index_scatter<8, false>);
    hipLaunchKernelGGL(kern, dim3(p.nchunks), dim3(64 * p.waves), lds, st, topk_idx, D.A, D.E, bits, p.chunk,
                       p.nchunks, hist, out.counts, out.offsets, out.perm, out.inv);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// hexa_moe_index_static: the same one or two launches with the chunk histogram in a fixed array of
// device memory that belongs to the library, for callers that cannot allocate (no hipMalloc under
// stream capture, tight serving loops).  Nothing here allocates or frees.
// ---------------------------------------------------------------------------------------------
namespace {

// One copy per GPU, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; kernels get the address that call returns.
static __device__ __align__(256) unsigned char scratch[HEXA_INDEX_STATIC_SCRATCH_BYTES];

std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU, looked up on first use

// The address of this device's copy of the array (the device must be current).
hipError_t static_scratch(void** out) {
    int d = -1;
    hipError_t e = hipGetDevice(&d);
    if (e != hipSuccess) return e;
    if (d < 0 || d >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[d]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[d] = p;
    }
    *out = g_scratch_ptr[d];
    return hipSuccess;
}

}  // namespace

extern "C" hexa_status hexa_moe_index_static(const hexa_moe_shape* shape, const int32_t* topk_idx,
                                             hexa_moe_idx out, void* stream) {
    MoeDims D;
    const hexa_status s = hexa_check_shape(shape, &D);
    if (s != HEXA_OK) return s;
    if (!topk_idx || !out.counts || !out.offsets || !out.perm || !out.inv) return HEXA_ERR_NULL;
    if (index_scratch_bytes(D) > (size_t)HEXA_INDEX_STATIC_SCRATCH_BYTES) return HEXA_ERR_WORKSPACE;
    void* ptr = nullptr;
    if (static_scratch(&ptr) != hipSuccess) return HEXA_ERR_DEVICE;
    // index_count overwrites every histogram entry that index_scatter reads (a single chunk reads none), so what an
    // earlier call left in the array needs no clearing
    return launch_index(D, topk_idx, out, ptr, (hipStream_t)stream) == hipSuccess ? HEXA_OK : HEXA_ERR_DEVICE;
}
