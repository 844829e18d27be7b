// Host-side check of the rules that choose a launch's shape (tm_internal.h), at the points where both sides were
// measured.  Built for the host only and run on the CPU by tests/test_launch_rules.py; prints "ALL OK".
#include <cstdio>

#include "../paper_1610_02370_amd/csrc/tm_api_internal.h"
#include "../paper_1610_02370_amd/csrc/tm_internal.h"

using namespace tmsap;

static int failures = 0;
static void expect(const char* what, int got, int want) {
    if (got == want) return;
    std::printf("FAIL: %s: %d, expected %d\n", what, got, want);
    ++failures;
}

int main() {
    // systems per workgroup: unsplit where the blocks fill the device ...
    expect("FP64 4^3x2 blocks, 864, 6 systems", sap_sys_tile(864, 6, 128, true, false), 6);
    expect("FP64 3^3x4 blocks, 864, 12 systems", sap_sys_tile(864, 12, 128, true, false), 12);
    expect("BF16 8x4^3 blocks, 864, 6 systems", sap_sys_tile(864, 6, 512, false, false), 6);
    expect("BF16 8x4^3 blocks, 864, 12 systems", sap_sys_tile(864, 12, 512, false, false), 12);
    expect("FP32 4^4 blocks, 20736, 12 systems", sap_sys_tile(20736, 12, 256, false, false), 12);
    // ... and split where they do not
    expect("FP32 4^4 blocks, 128, 12 systems", sap_sys_tile(128, 12, 256, false, false), 3);
    expect("FP32 8x4^3 blocks, 128, 6 systems", sap_sys_tile(128, 6, 512, false, false), 3);
    expect("FP64 2^4 blocks, 8, 2 systems", sap_sys_tile(8, 2, 64, true, false), 1);
    // every system once, whatever the shape
    for (long long blocks = 1; blocks < 5000; blocks = blocks * 3 / 2 + 1)
        for (int nsys = 1; nsys <= kMaxSys; ++nsys)
            for (int nt = 64; nt <= 1024; nt += 64)
                for (int k = 0; k < 4; ++k) {
                    const int tile = sap_sys_tile(blocks, nsys, nt, k & 1, k & 2);
                    if (tile < 1 || tile > nsys) expect("tile in 1..nsys", tile, nsys);
                }
    // the tuner times all systems in one workgroup too, whatever the launch would choose, and no tile twice
    for (int nsys = 1; nsys <= kMaxSys; ++nsys) {
        const std::vector<int> tiles = tune_tiles(nsys);
        expect("first tile", tiles.front(), nsys);
        for (size_t k = 1; k < tiles.size(); ++k)
            if (tiles[k] >= tiles[k - 1] || tiles[k] < 1) expect("tiles fall", tiles[k], tiles[k - 1] - 1);
    }
    expect("tiles of 12 systems", (int)tune_tiles(12).size(), 5);
    if (failures) return 1;
    std::printf("ALL OK\n");
    return 0;
}
