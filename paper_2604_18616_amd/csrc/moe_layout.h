// Row tiles of the grouped FP8 products: how an expert's rows are cut, and which of the two cuts a call takes.  Plain
// integer arithmetic, shared by the kernels, the host side and the host test.
#pragma once

#define MOE_HD __host__ __device__ constexpr

// Row tiles of an expert with cnt rows: tiles of bm rows and a remainder.  An expert with one full tile and
// at most 32 rows more gets a single tile of up to bm + 32 rows (one more 32-row MFMA block instead of a
// second copy of every weight tile: 13 % on the whole call where experts have about bm rows).  With two or
// more full tiles the remainder stays a tile of its own: measured, the short tiles then cost little (their
// weights are L2 hits) and fill the last round of workgroups, which equal long tiles leave mostly idle.
MOE_HD int moe_row_tiles(int cnt, int bm) {
    const int n = cnt / bm, r = cnt - n * bm;
    return (n == 1 && r <= 32) ? 1 : n + (r > 0 ? 1 : 0);
}

// Few rows per expert, also if every slot were local: the call runs on the kernel whose workgroups share a CU by twos, with bm = 32:
// every tile has up to 32 rows.  The host chooses and does not know the routing: a favoured expert's weights are copied once for
// every 32 of its rows, by neighbouring workgroups, the second time from L2.
MOE_HD bool moe_few(int T, int E, int KTOP) {
    const long long slots = T <= 32 ? 12 : T <= 64 ? 4 : 0;      // per expert
    return (long long)T * KTOP <= slots * E;
}

// bm = 0: an expert with up to 160 rows gets one tile, more rows the fewest tiles of at most 256, cut evenly at multiples of
// 32.  Never more tiles than bm = 128 makes.
MOE_HD int moe_tiles(int cnt, int bm) {
    if (bm == 32) return (cnt + 31) / 32;
    if (bm != 0) return moe_row_tiles(cnt, bm);
    return cnt <= 160 ? (cnt > 0 ? 1 : 0) : (cnt + 255) / 256;
}
// First row of tile j of the n = moe_tiles(cnt, bm) of an expert; j = n gives its number of rows.
MOE_HD int moe_tile_begin(int cnt, int n, int j, int bm) {
    const int at = bm != 0 ? j * bm : (int)((unsigned)j * ((unsigned)(cnt + 31) / 32) / (unsigned)n) * 32;
    return j >= n || at > cnt ? cnt : at;
}

// Estimated time of a product, in hundredths of a microsecond: `rows` routed rows in `tiles` row tiles, `cols` column tiles,
// `stages` 128-deep stages; `down`: its column tiles are halved where the whole ones would fill half the chip at most.
// A stage of a workgroup, a round of 256 workgroups and a last round that does not fill the chip are charged what makes the
// choice below agree with the times it was fitted to, not what they take one by one: a stage 0.51 us + 0.17 per 32 rows of its
// tile with all 256 CUs at it, 0.48 + 0.19 in a round of a few workgroups, four fifths of either on half a column tile; every
// round 6.3 us + 1.15 per 32 rows.
MOE_HD int moe_product_time(int rows, int tiles, int cols, int stages, bool down) {
    int alone = 48 + 19 * rows / (32 * tiles), full = 51 + 17 * rows / (32 * tiles), wgs = tiles * cols;
    if (down && wgs <= 128) { wgs *= 2; alone = alone * 4 / 5; full = full * 4 / 5; }
    const int rounds = wgs / 256, rest = wgs % 256, share = full * rest / 256;
    const int last = rest == 0 ? 0 : share > alone ? share : alone;
    return stages * (rounds * full + last) + (rounds + (rest > 0 ? 1 : 0)) * (630 + 115 * rows / (32 * tiles));
}

// The cut a call takes when the caller leaves it open: bm = 0, whose larger tiles copy a third less from L2 per product, or
// bm = 128, whose larger number fills the chip where the large ones would leave CUs idle or start another round.
// Gate/up + down, us, tiles of 128 rows against up to 256, same rows on every expert: 8 experts of 1024 x 512, 256 rows
// 23 / 33, 2000 rows 57 / 51; 4 of 4096 x 1408, 200 rows 50 / 63, 700 rows 105 / 87; 12 of 2944 x 1152, 256 rows 64 / 74,
// 300 rows 88 / 73; 8 of 4096 x 14336, 200 rows 454 / 400, 400 rows 832 / 616; 32 of 7168 x 2048, 256 rows 493 / 434.  With the
// same rows on every expert, 36 configurations of 8 layers, the choice is the better one within 3 %.  It sees the mean of the rows
// only: over 176 even and uneven routings of the layers it cost 0.6 % in the mean, most where a few experts have many times the
// rows of the others (8688 tokens on 32 of 7168 x 2048: 696, against 611 with 128 rows).
MOE_HD int moe_choose(int rows, int tiles128, int tiles256, int H, int I) {
    if (tiles128 == tiles256) return 0;
    const int small = moe_product_time(rows, tiles128, I / 128, H / 128, false) + moe_product_time(rows, tiles128, (H + 255) / 256, I / 128, true);
    const int large = moe_product_time(rows, tiles256, I / 128, H / 128, false) + moe_product_time(rows, tiles256, (H + 255) / 256, I / 128, true);
    return small < large ? 128 : 0;
}
