// How many workgroups the quantisers of n = 256 .. 4096 run (plain C++: the tests compile it for the host).
#pragma once

#include <cstdint>

namespace bq {

struct QuantiserCall {
    bool stores_rows, counts, big, f32;  // fake-quantised rows are stored, bins are counted, groups above 128 channels, float32 rows
};

// Time of `heads * per_head` workgroups of 1 / per_head of `rows` rows each, in a twentieth of a row of two workgroups of one
// compute unit.  512 fit at a time, two per unit; a lone one runs 1.4 times as fast as one of two, so what is left after the whole
// rounds of 512 costs 14 / 20 of a round if it fits one per unit.  Before its first row a workgroup reads its tables, from many
// heads: as long as 8 16-bit rows take where codes are stored, 12 where rows are, 4 with groups above 128 channels, whose rows take
// longer; 12 float32 rows, fewer of which are in flight.
inline int64_t quantiser_cost(int64_t rows, int64_t heads, int64_t per_head, QuantiserCall c)
{
    const int64_t workgroups = heads * per_head, full = workgroups / 512, rest = workgroups % 512;
    const int64_t tables = c.f32 ? 12 : c.big ? 4 : c.stores_rows || c.counts ? 12 : 8;
    return ((rows + per_head - 1) / per_head + tables) * (20 * full + (rest == 0 ? 0 : rest <= 256 ? 14 : 20));
}

// Workgroups per head for `rows` rows of 4096 elements per head.
//
// One head: two workgroups per compute unit, the two that fit, from the batch on that gives each a few rows; below, one, which
// reads half as many tables (213 KB each).  One / two per unit / 1280 workgroups: 1777 fp16 rows of 4096, INT4 11.4 / 11.5 / 17.2 us,
// 700 rows 7.2 / 8.3 / 10.3, 4000 rows 19.8 / 18.2 / 22.5, 65536 rows 225 / 185 / 189; float32 rows 2000 13.5 / 13.9 / 19.5, 16000
// 64.6 / 61.0 / 68.2; 2000 blocks of n = 512 .. 2048 12.7 / 11.7 / 17.2.  The lines cross between 800 and 2000 rows.  A call that counts
// bins ends with one atomic per bin and workgroup, and its lines cross later: 2000 rows 25.8 / 28.1 / 43.5, 4000 33.7 / 33.9 / 50.9,
// 16000 80.0 / 69.8 / 89.5.  Batches of 1.5 GB and more run 1 to 5 % faster in 1280 workgroups, which drift out of step (two
// per unit / 1280: 262144 fp16 rows, INT2 674 / 664, fake-quantised 870 / 852; 131072 float32 rows 482 / 459; half as many rows
// -2 to +1.5 %), unless their groups are large (910 / 922).
//
// Head counts that leave an eighth or more of those places empty, because workgroups come in multiples of the heads: the count of least
// cost.  2^28 elements in 300 heads, fp16 INT4: 271 us with one per head, 230 two, 206 three, 203 four; 171 heads 338, 237 (two),
// 254, 213, 206 (five); 2^24 elements in 300 heads 28.6, 31.9, 37.1, 43.7.
inline int64_t quantiser_workgroups_per_head(int64_t rows, int64_t heads, QuantiserCall c)
{
    const int64_t blocks = rows * heads, few = c.counts ? 3072 : 1280, vast = ((int64_t)3 << 29) / (4096 * (c.f32 ? 4 : 2));
    const int64_t target = blocks <= few ? 256 : c.big || blocks < vast ? 512 : 1280;
    int64_t best = target / heads > 0 ? target / heads : 1;
    if (heads > 1 && heads * best < target - target / 8) {
        best = 1;
        for (int64_t p = 2; p * heads <= 1280 && p <= rows; ++p)
            if (quantiser_cost(rows, heads, p, c) < quantiser_cost(rows, heads, best, c)) best = p;
    }
    return best < rows ? best : rows;
}

}  // namespace bq
