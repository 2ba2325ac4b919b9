// Host check of the tile numbering (amr_tiles.h): for frames of many shapes every super-tile of the frame has one
// place in the launch order, places beyond lie outside the frame, the order holds no more places than the
// slack allows (or is row by row), and launch slices hold every block.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "amr_tiles.h"

using namespace amr;

static void check(bool ok, const char *what, long x, long y) {
    if (ok) return;
    std::fprintf(stderr, "%s: %ld x %ld tiles\n", what, x, y);
    std::exit(1);
}

static void frame(int64_t tx, int64_t ty, int slack) {
    const int64_t w = (tx + 3) / 4, h = (ty + 3) / 4;
    const Cover c = cover_of(tx, ty, slack);
    check(c.n >= w * h && (c.sq == 0 ? c.n == w * h : 2 * c.n <= slack * w * h), "places", tx, ty);
    std::vector<char> seen((size_t)(w * h), 0);
    const uint32_t end = (uint32_t)((c.n + 7) / 8 * 8 + 4096);
    for (uint32_t i = 0; i < end; i++) {
        const SuperTile s = super_tile(c.sq, c.nx, i);
        check(s.x >= 0 && s.y >= 0 && (i < c.n || s.y >= h), "place beyond the order", tx, ty);
        if (s.x >= w || s.y >= h) continue;
        check(!seen[(size_t)(s.y * w + s.x)], "place taken twice", tx, ty);
        seen[(size_t)(s.y * w + s.x)] = 1;
    }
    for (char v : seen) check(v, "place missing", tx, ty);
}

int main() {
    for (int slack : {kLaunchSlack, kQueueSlack}) {
        for (int64_t ty = 1; ty <= 70; ty++)
            for (int64_t tx = 1; tx <= 140; tx++) frame(tx, ty, slack);
        for (int64_t a : {1, 2, 5, 16, 33, 127, 128, 129, 255, 256, 257, 1000, 4096})
            for (int64_t b : {1, 3, 4, 64, 129, 512, 513}) {
                frame(a, b, slack);
                frame(b, a, slack);
            }
        frame(4096, 4096, slack);
        for (int k = 0; k <= 10; k++) {          // a square of a power of two is one Morton curve, as it was
            const Cover c = cover_of((int64_t)4 << k, (int64_t)4 << k, slack);
            check(c.sq == k && c.nx == 1, "square", 4 << k, 4 << k);
        }
    }
    for (int64_t n = 8; n < (int64_t)1 << 31; n = n * 3 / 8 * 8 + 8) {
        const Slices l = slices_of(n);
        check((int64_t)l.x * l.z >= n && (int64_t)l.x * (l.z - 1) < n && l.x % 8 == 0 && (int64_t)l.x * 64 < (int64_t)1 << 32,
              "slices", (long)n, 0);
    }
    std::puts("ok");
}
