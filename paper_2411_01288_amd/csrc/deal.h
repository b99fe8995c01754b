// Which tiles of the 16-bit contractions a workgroup works on: plain arithmetic, without HIP headers, so that host programs
// can include it too.
#pragma once
#include "segments.h"

constexpr int group_rows(int bm) { return 1024 / bm; }   // row tiles per L2-sharing group: 1024 rows' worth
constexpr int kSplitBelow = 128; // row GEMMs with fewer groups share out the last ngroups % 8 groups among the XCDs

// Tiles in order: groups of GM row tiles x all column tiles, row tile fastest inside a group.
template <int GM>
__device__ __forceinline__ void grouped_tile(int local, int tm, int tn, int& tile_m, int& tile_n) {
    const int per_group = GM * tn;
    const int group = local / per_group;
    const int first = group * GM;
    const int gsz = min(GM, tm - first);
    const int in = local - group * per_group;
    tile_m = first + in % gsz;
    tile_n = in / gsz;
}

// Workgroup i runs on XCD i % 8, as number i / 8 of that XCD, and the XCDs fill up in this order: so an XCD's
// tiles are numbered without gaps, and workgroups without a tile (the grid is sized for the worst routing) come last.
// With such workgroups in between, the ones behind them find places taken: 492 tiles of two per CU took two rounds
// instead of one (bwd_fc1 at 4096 x 384 x 1536 of 8 experts, 33 -> 26 us).

// The tiles of a row GEMM, tm x tn.  256x256 tiles: groups dealt round-robin to the XCDs, so the 8 XCDs work on
// neighbouring row tiles (mostly one expert) at any time; what is left after rounds of eight groups is shared out tile by tile,
// every XCD taking neighbouring ones, so that no XCD is a whole group behind the others at the end; with many
// groups (kSplitBelow) all are dealt whole (an XCD's CUs finish their tiles one tile-time apart either way, and whole
// groups keep their L2 locality).  128x128 and 32x128 tiles are for smaller problems: an eighth of all tiles in a row per XCD.  Or,
// where experts have less than a tile of rows and their weights are read once and come from HBM (`streamed`), every group cut in eight, so that the
// whole chip reads whole rows of eight experts' weights at a time.  Both ways, in us: 64 tokens, 2048 x 8192 x 64, a
// serving pass 519 / 504 streamed; steps at 3001 x 320 x 448 of 17 80.3 / 86.6, 4096 x 384 x 1536 of 8 143 / 152.
template <int BM>
struct RowTiles {
    static constexpr int GM = group_rows(BM);
    static_assert(BM == 256 || GM % kXcds == 0, "a group in eight equal parts");
    int tm, tn, per_group, dealt;   // the first `dealt` tiles go out by group
    __device__ __forceinline__ RowTiles(int tm_, int tn_, bool streamed) : tm(tm_), tn(tn_), per_group(GM * tn_) {
        const int total = tm * tn;
        if (BM != 256) dealt = streamed ? total / per_group * per_group : 0;
        else dealt = ceil_div(tm, GM) >= kSplitBelow ? total : total / (kXcds * per_group) * (kXcds * per_group);
    }
    // tiles of XCD x among the dealt ones, and how many the XCDs in front of it (first) and it itself (n) have of the others
    __device__ __forceinline__ int dealt_to(int x) const {
        if (BM != 256) return dealt / kXcds;
        const int round = kXcds * per_group, r = dealt / round;
        return r * per_group + min(max(dealt - r * round - x * per_group, 0), per_group);
    }
    __device__ __forceinline__ void shared(int x, int& first, int& n) const {
        const int left = tm * tn - dealt, q = left / kXcds, m = left % kXcds;
        first = x * q + min(x, m);
        n = q + (x < m ? 1 : 0);
    }
    __device__ __forceinline__ int count(int x) const {
        int first, n;
        shared(x, first, n);
        return dealt_to(x) + n;
    }
    // tile number loc (< count) of XCD x
    __device__ __forceinline__ void tile(int x, int loc, int& tile_m, int& tile_n) const {
        const int mine = dealt_to(x);
        int lin, n;
        if (loc < mine) {
            const int part = BM != 256 ? per_group / kXcds : per_group;
            lin = loc + (loc / part * (kXcds - 1) + x) * part;
        } else {
            shared(x, lin, n);
            lin += dealt + loc - mine;
        }
        grouped_tile<GM>(lin, tm, tn, tile_m, tile_n);
    }
    // the most that any XCD can have with at most tm_max row tiles
    static int most(int tm_max, int tn) {
        const int even = ceil_div(tm_max * tn, kXcds), ngroups = ceil_div(tm_max, GM);
        const int whole = BM == 256 && ngroups >= kSplitBelow ? ceil_div(ngroups, kXcds) * GM * tn : 0;
        return even > whole ? even : whole;
    }
};

// The last round of 256x256 tiles, one per CU, leaves most of an XCD's 32 CUs idle for a whole tile where few are left:
// up to kQuartersUpTo of them are cut into four 128x128 tiles each, which have the CU to themselves too and take 0.33 to 0.4
// of the time.  Two full rounds of quarters do not win (16 tiles per XCD, 3720 tokens, 960 x 3840 of 4, fc2: 86 -> 91 us).  fc2 of a serving
// pass of 8192 tokens, 1024 x 4096 of 32 (324 tiles, 256 a round): 184 -> 151 us; in a step at 16384 x 1024 x 4096 of 32 279 -> 267, 32768 x 768 x 3072
// of 16 303 -> 283, 65536 x 1024 x 4096 of 32 462 -> 423.
constexpr int kCusPerXcd = 32, kQuartersUpTo = 12;

// What workgroup number loc of XCD x works on: tile number loc of the XCD (changed to it), all of it (quarter -1) or the quarter
// with these rows (quarter / 2) and columns (quarter % 2).  False: nothing.
__device__ __forceinline__ bool tile_or_quarter(const RowTiles<256>& rows, int x, int& loc, int& quarter) {
    const int n = rows.count(x), rest = n % kCusPerXcd, whole = rest <= kQuartersUpTo ? n - rest : n;
    quarter = -1;
    if (loc >= whole) {
        quarter = (loc - whole) % 4;
        loc = whole + (loc - whole) / 4;
    }
    return loc < n;
}

// The tiles of a token contraction: every (expert, chunk) item is a set of `tiles` tiles over the same tokens.  Each
// XCD takes an eighth of every item's tiles (neighbouring ones), so the XCDs stay balanced however uneven the
// experts are, and the whole chip streams the same token rows at a time.  Where the tiles are no multiple of eight,
// which XCDs take one more goes round from item to item (36 tiles as 5 5 5 5 5 5 5 1 for every item left the last XCD idle:
// the backward contractions of 32768 x 768 x 3072 under Zipf routing 632 + 548 -> 615 + 529 us).
struct TokenTiles {
    int tiles;
    __device__ __forceinline__ int share(int x, int item, int& first) const {
        const int s = (x + item) % kXcds;
        first = s * tiles / kXcds;
        return (s + 1) * tiles / kXcds - first;
    }
    // tiles of XCD x among the first `items` items (eight items in a row give every XCD `tiles`)
    __device__ __forceinline__ int count(int x, int items) const {
        int n = items / kXcds * tiles, first;
        for (int i = 0; i < items % kXcds; ++i) n += share(x, i, first);
        return n;
    }
    // tile number loc of XCD x: its item, and its number in there
    __device__ __forceinline__ int find(int x, int loc, int& tile) const {
        int item = loc / tiles * kXcds, rest = loc % tiles;
        for (;; ++item) {                      // (at most eight rounds: rest < tiles)
            int first;
            const int n = share(x, item, first);
            if (rest < n) {
                tile = first + rest;
                return item;
            }
            rest -= n;
        }
    }
    // at least what any XCD can have with at most `items` items
    int most(int items) const {
        const int rest = items % kXcds * ceil_div(tiles, kXcds);
        return items / kXcds * tiles + (rest < tiles ? rest : tiles);
    }
};
