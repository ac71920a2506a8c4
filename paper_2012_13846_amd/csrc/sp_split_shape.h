// How gather_split_kernel (sp_conv_split.hip) cuts a layer: slices, channel tiles, rows of a tile and links of a step.  Host
// arithmetic without another header of this library, so that a test on the CPU can check it.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace sp {

// Slices of cc contraction channels, tiles of cot destination channels.
struct SplitShape {
    int cc, nsl, cot, ny;
};

// The cut with the least padding.
inline SplitShape split_shape(int cc, int co) {
    SplitShape t{};
    int best = 1 << 30;
    for (int c : {64, 32}) {
        const int n = (cc + c - 1) / c, cost = n * c + 8 * (n - 1);
        if (cost < best) {
            best = cost;
            t.cc = c;
            t.nsl = n;
        }
    }
    best = 1 << 30;
    for (int c : {128, 64, 48, 32}) {
        const int n = (co + c - 1) / c, cost = n * c + 8 * (n - 1);
        if (cost < best) {
            best = cost;
            t.cot = c;
            t.ny = n;
        }
    }
    return t;
}
inline size_t split_copy_bytes(const SplitShape& t, int kvol) { return (size_t)kvol * t.nsl * t.cc * t.ny * t.cot * 6; }

// Dynamic LDS of a workgroup of nw = cot / 16 wavefronts: accumulator rows of 16 nw + 4 floats, a spare one for links that do not
// exist; two steps' rows as three bf16 pieces; their accumulator offsets; a descriptor per step.
constexpr int split_lds(int cc, int nw, int g, int halves, int kvol) {
    const int links = 16 * g;
    return (halves * 32 + 1) * (16 * nw + 4) * 4 + 2 * links * cc * 6 + 2 * links * 4 + kvol * ((halves * 32 + links - 1) / links) * 8;
}
constexpr int kSplitLdsMost = 163840 - 256;

// Wavefronts of a SIMD that find registers.
constexpr int split_simd_waves(int cc, int nw, int g) { return cc == 32 ? 4 : nw == 4 && g == 2 ? 3 : 2; }

// Rows of a tile (in halves of 32) and links of a step (in blocks of 16).
struct SplitTile {
    int halves, g;
};

// More rows are fewer reads of an offset's weights, as long as its links in a tile fit one step, and fuller blocks; fewer let more
// workgroups share a CU and fill its last round better.  A tile costs, for every offset with mu links in it, its steps (their weights are
// read again in each; as much as 6 blocks, 7.4 with rows for 48 links) and its blocks of 16, each 0.7 more than mu alone would fill, and
// little for its rows.  The tiles of the fullest CU add up (some of the last round's start early), and a round of those that share
// it takes `hide` / wavefronts of a tile more, which more wavefronts hide.  Of equals the lower one, since surfaces fill tall tiles unevenly
// (1.5 % a half; 32 -> 64 none above 128 rows: on 0.1 M rows of objects, per 28, H = 2 .. 7: 58, 53, 53, 54, 62, 67), and 20 % on tall tiles
// of several steps an offset that all start together: nothing balances heavy ones that meet on a CU (64 -> 64, 86 k rows of
// objects, per 27, two tiles a CU: H = 6 90 us, H = 3 66).
// Steps of 48 links save weights where an offset has more than 32 in a tile, and their rows take registers: 64 -> 64 has two such
// workgroups on a CU against three.  Tiles of 128 channels lose no workgroup by them, but time where few links fill the step, and gain
// from about 64 links of an offset in 128 rows (per) on: 96 k rows, per 89, 128 -> 128 467 / 431 us, 64 -> 128 241 / 225; per 12 0.83 times as fast.
// Over 1571 launches (objects, spheres, rooms in sampling order, random clouds, full cubes; K = 2, 3, 5, strides 1 and 2; 14 k to 0.6 M rows,
// per 5 to 120) this takes 1.7 % longer than the best of all heights and both steps (32 -> 128 5 %: no steps of 48), tiles of 128 rows (64
// where those were fewer than 128) with steps of 32 or 48 by per 18 %, a rule that counted an offset's weights once a tile 2.6 %.
// H = halves of 32 rows, us, steps of 32 / 48:
//   64 -> 64     0.61 M rows of objects, per 39, H = 2 .. 6: 486, 425, 476, 464, 451 / 638, 489, 441, 628, 624
//                0.14 M, per 38: 121, 109, 125, 119, 131 / 152, 121, 116, 160, 157;   96 k, random, per 89: 150, 150, 151, 182, 142 / 140, 146, 140, 225, 170
//                0.16 M, per 19: 118, 95, 94, 91, 86;   0.6 M, random, per 14, H = 3 .. 6: 348, 311, 268, 250
//   80 -> 48     75 k, per 39, H = 2 .. 5, steps of 48: 128, 113, 111, 127      48 -> 48   96 k, per 30, H = 3 .. 7: 84, 89, 91, 79, 112
//   64 -> 128    96 k, per 30, H = 2 .. 7: 158, 137, 135, 135, 139, 135 / 186, 146, 142, 141, 146, 138;   random, per 16, H = 3 .. 7: 115, 94, 98, 78, 80
//   128 -> 128   0.16 M, per 19, H = 2 .. 7: 432, 328, 291, 271, 254, 263        32 -> 64   96 k, per 30, H = 2 .. 7: 59, 50, 51, 68, 58, 64
inline SplitTile split_tile(const SplitShape& t, int64_t n_rows, int kvol, int64_t links) {
    const int nw = t.cot / 16;
    const double per = std::max(1.0, (double)links * 128.0 / ((double)n_rows * kvol));
    const int g0 = nw == 3 ? 3 : 2, g1 = t.cc == 64 && (nw == 4 || (nw == 8 && per >= 64.0)) ? 3 : g0;
    const double hide = nw >= 4 ? 8.5 : 14.0;
    const int most = t.cc == 32 && nw == 4 ? 4 : 7;
    SplitTile best{0, 0};
    double least = 0.0;
    for (int g = g0; g <= g1; ++g) {
        const int fit = std::max(1, 4 * split_simd_waves(t.cc, nw, g) / nw), step = 16 * g;
        for (int h = 2; h <= most; ++h) {
            const int lds = split_lds(t.cc, nw, g, h, kvol), there = std::max(1, std::min(fit, 163840 / (lds + 1024)));
            if (lds > kSplitLdsMost) break;
            const int64_t tiles = (n_rows + h * 32 - 1) / (h * 32) * t.ny, fullest = (tiles + 255) / 256;
            const double mu = per * h / 4.0, some = std::min(1.0, mu);
            const double steps = std::min(std::max(some, mu / step + 0.7), (double)((h * 32 + step - 1) / step));
            const double blocks = std::min(std::max(some, mu / 16.0 + 0.7), 2.0 * h);
            const double one = (double)t.nsl * kvol * ((g == 2 ? 6.0 : 7.4) * steps + blocks) + h;
            const double cu = std::max(1.0, 0.7 * (double)fullest + 0.3 * ((double)tiles / 256.0 + 0.5)), share = cu / there;
            const double rounds = share > 2.0 ? share : 0.7 * (double)((fullest + there - 1) / there) + 0.3 * std::max(1.0, share);
            const double uneven = g == 2 && nw < 8 && h >= 5 && mu > 32.0 && fullest <= there ? 1.2 : 1.0;
            const double cost = one * (cu + hide / nw * rounds) * (1.0 + 0.015 * h) * uneven;
            if (best.g == 0 || cost < least) {
                least = cost;
                best = SplitTile{h, g};
            }
        }
    }
    return best;
}

}  // namespace sp
