// Rules by which a launch is chosen from sizes alone: plain host C++, so that
// they can be checked over extents that no test could run.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace raysh {

// Launch shapes selectable per call (the autotuner's search space).
struct TileShape {
    int cx, cy;      // rays per lane along x and y
    int share;       // r^2 values sharing one reciprocal (FP64 path)
    int star_tile;   // FP64: consecutive stars among them (the rest are the lane's
                     // neighbouring rays); FP32-bulk: stars staged in LDS per pass
};

// A one-dimensional grid that HIP launches: fewer than 2^32 threads.
inline bool grid_fits(int64_t blocks, int threads) { return blocks <= (((int64_t)1 << 32) - 1) / threads; }

// Forms of the one-pass FP64 kernel in which the waves of a workgroup share a
// tile of 8 cx x 8 cy rays (waves_fp64_kernel): cx, cy, share, star_tile, waves.
#define RAYSH_FP64_WAVES(X) \
    X(8, 4, 16, 1, 4)       \
    X(4, 4, 16, 1, 8)       \
    X(4, 2, 8, 1, 16)       \
    X(2, 2, 4, 1, 16)

inline int64_t tiles_of(int64_t nx, int64_t ny, int w, int h) { return ((nx + w - 1) / w) * ((ny + h - 1) / h); }

// Time of the busiest compute unit, in instructions of a lane (64 lanes a
// cycle), of a launch whose workgroups each take a tile of w x h rays and
// `once` besides the star sum.  A ray and star take 6 instructions, a lane's
// column and row one and two (shared by its rays), a reciprocal four with its
// tree, and a mass per ray half of one.  A unit takes whole tiles, and the
// last of them runs partly alone (0.15 of a tile: 2048^2 rays and 10000 stars
// take 8.63 ms in 2 tiles a unit and 8.03 in 8, 4096^2 rays and 16384 stars
// 52.7 in 8 and 51.8 in 32); a unit with one wave a SIMD for all its tiles
// issues 0.8 times as fast.
inline double busiest_unit(int64_t nx, int64_t ny, int64_t n_stars, const TileShape &t, int w, int h, int waves,
                           double once, int n_cu) {
    const int64_t mine = (tiles_of(nx, ny, w, h) + n_cu - 1) / n_cu;
    const double v = 6.0 + 1.0 / t.cy + 2.0 / t.cx + 4.0 / t.share + (t.star_tile > 1 ? 0.5 : 0.0);
    const double last = mine * waves >= 8 ? 0.15 : 0.25;
    return ((double)mine + last) * (double)n_stars * w * h * v + (double)mine * once;
}

// A tile's epilogue, in the same unit: 16 us for 8192 rays, about 4 for each
// shape of waves_fp64_kernel (1000^2 rays and 10 stars: 21 us in one such
// tile a unit, 11.6 in two of 2048 rays, 41 in eight of 512).
constexpr double kOncePerTile = 2.4e6, kOnceShared = 6.5e5;

// One pass in the fastest form for the lattice: `t` (the shape for lattices
// that fill the device many times over: -1) or the waves of a workgroup sharing
// a tile (the form's place in RAYSH_FP64_WAVES), whichever keeps the busiest
// compute unit busy least and can be launched.  The forms add a ray's stars in
// runs, t in one, as the batch kernel does, so a form has to save a twentieth:
// lattices that fill the device have the rounding of their batch and of their
// bands (4096^2 rays and 20000 stars would save 2 %).  Measured (us, t and the
// form chosen): 100 stars and 1000^2 rays 64 -> 31, 1000 and 500^2 458 -> 62,
// 1000 and 250^2 457 -> 25, 3000 and 100^2 1343 -> 58, 10000 and 2048^2 8630 ->
// 8030; 1000 and 8192^2 stay with t (12.70 ms against 12.91, its epilogue
// being cheaper a ray).
inline int waves_form(int64_t nx, int64_t ny, int64_t n_stars, const TileShape &t, int n_cu) {
    if (n_cu < 1) n_cu = 1;
    double best = 0.95 * busiest_unit(nx, ny, n_stars, t, 16 * t.cx, 16 * t.cy, 4, kOncePerTile, n_cu);
    int form = -1, i = 0;
#define RAYSH_CASE(CX, CY, S, NS, W)                                                                      \
    if (grid_fits(tiles_of(nx, ny, 8 * CX, 8 * CY), 64 * W)) {                                            \
        const double cost =                                                                               \
            busiest_unit(nx, ny, n_stars, TileShape{CX, CY, S, NS}, 8 * CX, 8 * CY, W, kOnceShared, n_cu); \
        if (cost < best) {                                                                                \
            best = cost;                                                                                  \
            form = i;                                                                                     \
        }                                                                                                 \
    }                                                                                                     \
    ++i;
    RAYSH_FP64_WAVES(RAYSH_CASE)
#undef RAYSH_CASE
    return form;
}

// Ray tiles of a lattice block in the expansion mode (shoot_expansion.hip):
// 4096 rays, w x h = 64 / 2^skew x 64 * 2^skew.
struct TileGrid {
    int skew, w, h;
    int64_t tiles_x, tiles_y;
};
constexpr int kTileRays = 4096, kMaxSkew = 2;   // |skew|

// The skew nearest to half the logarithm of dx / dy, so that the sides differ
// by a factor of sqrt(2) at most (|skew| <= kMaxSkew): near lists, and with them
// the stars summed directly, grow as the square of the tile's radius.  But no
// side of twice the lattice's length or more: on a lattice of a few rows a
// taller tile holds fewer rays, and there are more tiles (2^20 x 1 rays, 3000
// stars, dx = 16 dy: 592 us in tiles of 64 x 64, 2245 in 16 x 256).
inline TileGrid expansion_tiles(int64_t nx, int64_t ny, double dx, double dy) {
    TileGrid g;
    const double k = std::round(0.5 * std::log2(dx / dy));
    g.skew = k >= kMaxSkew ? kMaxSkew : k <= -kMaxSkew ? -kMaxSkew : (int)k;   // (dx / dy may be 0 or infinite)
    while (g.skew > 0 && ny <= 32 << g.skew) --g.skew;
    while (g.skew < 0 && nx <= 32 << -g.skew) ++g.skew;
    g.w = g.skew >= 0 ? 64 >> g.skew : 64 << -g.skew;
    g.h = kTileRays / g.w;
    g.tiles_x = (nx + g.w - 1) / g.w;
    g.tiles_y = (ny + g.h - 1) / g.h;
    return g;
}

// Workgroups of smooth_rows_slide_kernel (256 outputs of 4 rows each) and of
// disk_prefix_kernel (one, and one for every 4 rows).  Both take a wave per
// row however short the row is, so a map of few columns and 2^26 rows or more
// exceeds the grid, where a thread per output does not.
inline int64_t smooth_row_blocks(int wx, int ny) { return ((wx + (int64_t)255) / 256) * ((ny + (int64_t)3) / 4); }
inline int64_t disk_prefix_blocks(int ny) { return 1 + (ny + (int64_t)3) / 4; }

// Whether prefix sums pay for a disk's map.  Its about 0.79 (2 rx + 1)(2 ry + 1)
// counts a pixel are read in 0.9 us each on a 2048^2 map and, as one thread's
// chain of loads, in no less than 0.08 us on a small one; 2 (2 ry + 1) prefix
// sums take 1.6 us each (0.05), and their making 15 us and 4 besides.
// Directly and with them: radius 3 and 4 on 2048^2 60 us and 62, 80 and 59;
// radius 4 and 5.5 on 1024^2 20.5 and 24.5, 32 and 26; radius 8.5 on 256^2 21.5
// and 16.5; radius 25 on 2048^2 1770 and 200; a disk one pixel wide and any
// height never.
inline bool disk_by_prefix(int rx, int ry, int64_t pixels) {
    const double maps = (double)pixels / (2048.0 * 2048.0), rows = 2.0 * ry + 1.0, cols = 2.0 * rx + 1.0;
    const double direct = 0.79 * cols * rows * std::max(0.9 * maps, 0.08);
    const double prefix = 2.0 * rows * std::max(1.6 * maps, 0.05) + 15.0 * maps + 4.0;
    return prefix < direct;
}

}  // namespace raysh
