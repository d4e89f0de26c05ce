// Host-side check of the expert layer's row tiles (csrc/moe_layout.h), compiled with g++ by tests/test_layout_host.py: every
// cut of every row count is a partition the kernel can run, the two cuts of a call fit the tables sized for 128-row tiles,
// and the choice between them is the faster one at the sizes both were measured at.
#include <cstdio>
#define __host__
#define __device__
#include "../../paper_2604_18616_amd/csrc/moe_layout.h"

static int failures = 0;
#define CHECK(cond, ...) do { if (!(cond) && ++failures < 20) { printf(__VA_ARGS__); printf("\n"); } } while (0)

static void check_cuts() {
    const int bms[] = {0, 32, 64, 128};
    for (int bm : bms)
        for (int cnt = 0; cnt <= 1 << 20; cnt += cnt < 20000 ? 1 : 4093) {
            const int n = moe_tiles(cnt, bm), most = bm == 32 ? 32 : bm ? bm + 32 : 256;
            CHECK((n == 0) == (cnt == 0), "bm %d, %d rows: %d tiles", bm, cnt, n);
            CHECK(bm != 0 || n <= moe_tiles(cnt, 128), "%d rows: %d tiles, more than of 128 rows", cnt, n);
            for (int j = 0; j < n; ++j) {
                const int begin = moe_tile_begin(cnt, n, j, bm), end = moe_tile_begin(cnt, n, j + 1, bm);
                CHECK(begin % 32 == 0 && end > begin && end - begin <= most, "bm %d, %d rows: tile %d is %d .. %d", bm, cnt, j, begin, end);
                CHECK(j > 0 || begin == 0, "bm %d, %d rows: starts at %d", bm, cnt, begin);
            }
            CHECK(n == 0 || moe_tile_begin(cnt, n, n, bm) == cnt, "bm %d, %d rows: ends at %d", bm, cnt, moe_tile_begin(cnt, n, n, bm));
        }
    CHECK((1 << 20) / 128 + 256 < 1 << 15, "two tile counts share an int");
}

// Calls of few tokens: however the slots fall on the experts, even all on one, there are at most slots / 32 + E tiles, whose
// records fit the table for slots / 64 + E and the 512 bytes behind it.
static void check_few() {
    CHECK(moe_few(32, 8, 3) && !moe_few(33, 8, 3) && !moe_few(32, 8, 4) && moe_few(64, 64, 4) && !moe_few(65, 64, 4) && !moe_few(64, 63, 4), "lines");
    unsigned seed = 1;
    for (int T = 1; T <= 64; ++T)
        for (int k = 1; k <= 16; ++k)
            for (int E = 1; E <= 256; E += E < 16 ? 1 : 24) {
                if (!moe_few(T, E, k)) continue;
                CHECK(((T * k + 31) / 32 - (T * k + 63) / 64) * 16 <= 512, "%d tokens x %d on %d experts: records", T, k, E);
                for (int form = 0; form < 4; ++form) {                 // all on one; 33 each as far as they go; 1 each; random
                    int left = T * k, tiles = 0;
                    for (int e = 0; e < E && left > 0; ++e) {
                        seed = seed * 1664525u + 1013904223u;
                        int n = form == 0 ? left : form == 1 ? 33 : form == 2 ? 1 : (int)((seed >> 16) % 70);
                        if (n > left || (form != 2 && e == E - 1)) n = left;
                        left -= n;
                        tiles += moe_tiles(n, 32);
                    }
                    CHECK(tiles <= (T * k + 31) / 32 + E, "%d tokens x %d on %d experts: %d tiles", T, k, E, tiles);
                }
            }
}

static void check_choice() {
    // E experts with `rows` rows each; us of the two products with tiles of 128 rows and of up to 256, as the kernels are now.
    // Either cut will do where the times are within 3 %, what two runs may differ by
    struct { int H, I, E, rows; double t128, t256; } const measured[] = {
        {1024, 512, 8, 175, 22.8, 26.5}, {1024, 512, 8, 256, 22.8, 33.1}, {1024, 512, 8, 400, 23.8, 30.3}, {1024, 512, 8, 512, 24.0, 34.1},
        {1024, 512, 8, 700, 27.3, 34.4}, {1024, 512, 8, 1000, 29.5, 36.8}, {1024, 512, 8, 1400, 49.7, 43.4}, {1024, 512, 8, 2000, 57.4, 50.8},
        {4096, 1408, 4, 200, 49.7, 63.3}, {4096, 1408, 4, 300, 54.3, 55.2}, {4096, 1408, 4, 500, 59.6, 77.3}, {4096, 1408, 4, 700, 104.8, 87.2},
        {4096, 1408, 4, 1000, 116.8, 99.1}, {2944, 1152, 12, 200, 63.5, 64.6}, {2944, 1152, 12, 256, 63.5, 73.7}, {2944, 1152, 12, 300, 87.6, 72.7},
        {2944, 1152, 12, 400, 107.0, 91.3}, {2944, 1152, 12, 600, 135.6, 127.3}, {4096, 14336, 8, 200, 454.1, 399.7},
        {4096, 14336, 8, 256, 443.8, 451.6}, {4096, 14336, 8, 400, 832.2, 615.5}, {4096, 14336, 8, 600, 1062.5, 931.9},
        {2048, 1408, 64, 170, 232.7, 183.6}, {2048, 1408, 64, 200, 240.9, 198.1}, {2048, 1408, 64, 256, 245.6, 215.7},
        {2048, 1408, 64, 400, 435.1, 330.3}, {2048, 768, 128, 200, 292.3, 239.6}, {2048, 768, 128, 256, 299.7, 265.8},
        {2048, 768, 128, 400, 530.1, 398.1}, {5120, 1536, 16, 200, 165.1, 139.3}, {5120, 1536, 16, 256, 171.3, 154.6},
        {5120, 1536, 16, 400, 258.8, 227.8}, {7168, 2048, 32, 180, 470.9, 367.9}, {7168, 2048, 32, 256, 493.4, 433.6},
        {7168, 2048, 32, 300, 647.3, 558.7}, {7168, 2048, 32, 400, 877.5, 660.4}};
    for (const auto& m : measured) {
        const int bm = moe_choose(m.E * m.rows, m.E * moe_tiles(m.rows, 128), m.E * moe_tiles(m.rows, 0), m.H, m.I);
        CHECK((bm ? m.t128 : m.t256) <= 1.03 * (m.t128 < m.t256 ? m.t128 : m.t256), "%d experts of %d x %d, %d rows: bm %d, measured %.1f / %.1f us",
              m.E, m.H, m.I, m.rows, bm, m.t128, m.t256);
    }
    // the largest sums that the estimate can meet stay inside an int and positive
    const int tiles = (1 << 20) / 128 + 256;
    CHECK(moe_product_time(1 << 20, tiles, 128, 128, false) > 0 && moe_product_time(1 << 20, tiles / 2, 128, 128, true) > 0, "overflow");
    CHECK(moe_choose(1, 1, 1, 128, 128) == 0, "one row");
}

int main() {
    check_cuts();
    check_few();
    check_choice();
    if (failures) { printf("%d moe layout check(s) FAILED\n", failures); return 1; }
    printf("moe layout checks passed\n");
    return 0;
}
