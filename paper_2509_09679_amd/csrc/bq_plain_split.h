// How the backward pass of n = 256 .. 8192 splits a batch on a flagged plan (plain C++: the tests compile it for the host).
#pragma once

#include <cstdint>

namespace bq {

// Tiles of rows_per_tile rows of one head, dealt in turn to `parts` workgroups, each of which adds its tiles' sums to a slice of its own.
struct PlainSplit {
    int rows_per_tile;
    int64_t tiles;
    int parts;
};

// s: the split of the kernel for any n, up to 512 workgroups of 256 threads.  Here a workgroup has 1024 threads and a compute unit to
// itself, so tiles grow to 4096 elements (n = 2048 and 4096: 8192) where there are more of them than units, and 256 workgroups take
// them (20000 fp16 rows of 512: 359 -> 235 us).  The float32 sums stay as exact: a tile adds up in double and rounds once, and half as
// many slices hold at most half as many sums of tiles.  Tiles of one row round nothing but their products, so they grow only
// where a slice adds up more than four.  Error of dtheta against 64 bits, the kernel for any n / with 256 slices of float32 sums / this:
// 20000 float32 rows of 4096 2.26e-7 / 2.40e-7 / 2.11e-7, 100000 fp16 rows 3.53e-7 / 3.96e-7 / 3.04e-7, 1500 float32 rows of 2048
// 1.77e-7 / 1.78e-7 / 1.77e-7.
inline PlainSplit grown_split(PlainSplit s, int64_t rows, int n, int heads)
{
    const int64_t most = n < 2048 ? 4096 : 8192, enough = s.parts > 256 ? 256 : s.parts;
    PlainSplit g = s;
    if (s.rows_per_tile == 1 && s.tiles <= 4 * (int64_t)s.parts) return g;
    while (g.tiles > enough && (int64_t)g.rows_per_tile * 2 * n <= most) {
        g.rows_per_tile *= 2;
        g.tiles = (rows + g.rows_per_tile - 1) / g.rows_per_tile * heads;
    }
    if (g.rows_per_tile > s.rows_per_tile) {
        if (g.parts > 256) g.parts = 256;
        if (g.parts > g.tiles) g.parts = (int)g.tiles;
    }
    return g;
}

}  // namespace bq
