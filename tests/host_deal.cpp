// The deal of tiles to XCDs (csrc/deal.h) on the CPU.
//   argv: rows BM TM TN TM_MAX STREAMED   the tiles of a row GEMM
//         tokens TILES ITEMS CAP          those of a token contraction
//         quarters TM TN TM_MAX           256x256 tiles, some in quarters: 5 * tile for a whole one, 5 * tile + 1 + quarter
//   stdout: per XCD, the tiles in order (row * TN + column, or item * TILES + tile); then the grid's size per XCD
#include <cstdio>
#include <cstdlib>
#include <cstring>

#define __host__
#define __device__
#define __forceinline__ inline
#include <algorithm>
using std::max;
using std::min;
#include "../paper_2411_01288_amd/csrc/deal.h"

template <int BM>
static void rows(int tm, int tn, int tm_max, bool streamed) {
    const RowTiles<BM> r(tm, tn, streamed);
    for (int x = 0; x < kXcds; ++x) {
        for (int loc = 0; loc < r.count(x); ++loc) {
            int m, n;
            r.tile(x, loc, m, n);
            std::printf("%d ", m >= 0 && m < tm && n >= 0 && n < tn ? m * tn + n : -1);
        }
        std::printf("\n");
    }
    std::printf("%d\n", RowTiles<BM>::most(tm_max, tn));
}

static void quarters(int tm, int tn, int tm_max) {
    const RowTiles<256> r(tm, tn, false);
    for (int x = 0; x < kXcds; ++x) {
        for (int slot = 0; slot < RowTiles<256>::most(tm_max, tn) + 3 * kQuartersUpTo; ++slot) {
            int loc = slot, m, n, quarter;
            if (!tile_or_quarter(r, x, loc, quarter)) continue;
            r.tile(x, loc, m, n);
            std::printf("%d ", 5 * (m * tn + n) + 1 + quarter);
        }
        std::printf("\n");
    }
    std::printf("0\n");
}

int main(int argc, char** argv) {
    if (argc < 5) return 2;
    auto arg = [&](int i) { return std::atoi(argv[i]); };
    if (!std::strcmp(argv[1], "rows")) {
        if (argc != 7) return 2;
        if (arg(2) == 256) rows<256>(arg(3), arg(4), arg(5), arg(6) != 0);
        else if (arg(2) == 128) rows<128>(arg(3), arg(4), arg(5), arg(6) != 0);
        else if (arg(2) != 32) return 2;
        else rows<32>(arg(3), arg(4), arg(5), arg(6) != 0);
        return 0;
    }
    if (!std::strcmp(argv[1], "quarters")) {
        quarters(arg(2), arg(3), arg(4));
        return 0;
    }
    const TokenTiles t{arg(2)};
    for (int x = 0; x < kXcds; ++x) {
        for (int loc = 0; loc < t.count(x, arg(3)); ++loc) {
            int tile;
            const int item = t.find(x, loc, tile);
            std::printf("%d ", tile >= 0 && tile < t.tiles ? item * t.tiles + tile : -1);
        }
        std::printf("\n");
    }
    std::printf("%d\n", t.most(arg(4)));
    return 0;
}
