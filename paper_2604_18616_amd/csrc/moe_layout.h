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

// bm = 0: an expert with up to 160 rows gets one tile, more rows the fewest tiles of at most 256, cut evenly at multiples of
// 32.  Never more tiles than bm = 128 makes.
MOE_HD int moe_tiles(int cnt, int bm) {
    if (bm != 0) return moe_row_tiles(cnt, bm);
    return cnt <= 160 ? (cnt > 0 ? 1 : 0) : (cnt + 255) / 256;
}
// First row of tile j of the n = moe_tiles(cnt, bm) of an expert; j = n gives its number of rows.
MOE_HD int moe_tile_begin(int cnt, int n, int j, int bm) {
    const int at = bm != 0 ? j * bm : (int)((long long)j * ((cnt + 31) / 32) / n) * 32;
    return j >= n || at > cnt ? cnt : at;
}

// Estimated time of a product, in hundredths of a microsecond: `rows` routed rows in `tiles` row tiles, `cols` column tiles,
// `stages` 128-deep stages; `down`: its column tiles are halved where the whole ones would fill half the chip at most.
// Measured: a stage of a workgroup takes 0.22 us + 0.17 per 32 rows of its tile while its CU's share of L2 is no limit,
// 0.30 + 0.25 with all 256 CUs at it, four fifths of that on half a column tile; launch, start and end 3 us + 0.8 per 32
// rows, in every round of workgroups.  (The mean tile is charged half a block of 32 rows for its remainder.)
MOE_HD int moe_product_time(int rows, int tiles, int cols, int stages, bool down) {
    int alone = 30 + 17 * rows / (32 * tiles), full = 42 + 25 * rows / (32 * tiles), wgs = tiles * cols;
    if (down && wgs <= 128) { wgs *= 2; alone = alone * 4 / 5; full = full * 4 / 5; }
    const int rounds = wgs / 256, rest = wgs % 256, share = full * rest / 256;
    const int last = rest == 0 ? 0 : share > alone ? share : alone;
    return stages * (rounds * full + last) + (rounds + (rest > 0 ? 1 : 0)) * (340 + 80 * rows / (32 * tiles));
}

// The cut a call takes when the caller leaves it open: bm = 0, whose larger tiles copy a third less from L2 per product, or
// bm = 128, whose larger number fills the chip where the large ones would leave CUs idle or start another round.
// Gate/up + down, us, tiles of 128 rows against up to 256, same rows on every expert: 8 experts of 1024 x 512, 256 rows
// 21.7 / 34.2, 2000 rows 59.3 / 50.9; 4 of 4096 x 1408, 200 rows 48.9 / 74.9, 700 rows 106 / 90; 12 of 2944 x 1152, 200 rows
// 62.3 / 68.9, 300 rows 85.7 / 78.1; 8 of 4096 x 14336, 256 rows 471 / 520, 400 rows 841 / 712; 32 of 7168 x 2048, 256 rows
// 520 / 480.  Of 156 measured configurations one came out more than 3 % slower than with tiles of 128 rows (64 of 2048 x 1408,
// 256 +- 16 rows: 267 / 275).  A last round of a few workgroups is where the estimate errs: 12 of 2944 x 1152, 250 +- 15 rows:
// 79 / 90, and it takes the larger tiles.
MOE_HD int moe_choose(int rows, int tiles128, int tiles256, int H, int I) {
    if (tiles128 == tiles256) return 0;
    const int small = moe_product_time(rows, tiles128, I / 128, H / 128, false) + moe_product_time(rows, tiles128, (H + 255) / 256, I / 128, true);
    const int large = moe_product_time(rows, tiles256, I / 128, H / 128, false) + moe_product_time(rows, tiles256, (H + 255) / 256, I / 128, true);
    return small < large ? 128 : 0;
}
