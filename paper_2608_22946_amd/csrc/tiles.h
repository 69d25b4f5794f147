// Tiles of the stencil launches and the bound on their number.  Host code without HIP: the launches
// and the size of the fused norm's partials come from the same counts.
#pragma once

#include <algorithm>

namespace helm {

constexpr int kTileX = 62;      // output nodes per wavefront along x (64 lanes, 1-node halo each side)
constexpr int kWavesY = 4;      // wavefronts (rows y) per workgroup

inline int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }

// Tiles of one stencil launch: a wavefront covers a tile of columns, its rows and a chunk of tz
// planes; a block holds four wavefronts that follow each other.
//   Edge tiles hold both x-PML strips: `strip` output columns at each end of a row, strip + 2 lanes
//   each, and as many rows as fill the wavefront (strip 30, 14 or 6: 1, 2 or 4 rows).  Every
//   other tile is then free of x stretching (inner tiles of 62 columns from column `strip` on).
//   Rows in the tensor form cost about twice those in the shell form, so the strip is the one with
//   the least work a plane of rows (row_cost): on 89 columns with a 4-cell PML 14-column strips
//   take 2 units a row where 30-column ones take 3 (4h level of a 352^3 grid: apply 9.6 -> 8.4 us, J2 11.4 -> 10.6 us).
//   Without a strip that fits (no edge tiles) the columns are cut into tiles of 62 as they come.
//   The last edge block may have rows for fewer than `rows` groups; the groups without rows get no inner
//   blocks (launched and left at once, they put a second block on some compute units of a thin
//   level: A_h on 400 x 24 x 36 cells in FP64 at depth 8 took 12.1 us with them and takes 9.7, J2 13.9 and 10.6).
// Where the tiling allows, the inner tiles of rows between the y-PML strips may run as a launch of
// their own (PART 1), which compiles to fewer registers, and the rest (PART 2) before it;
// PART 0 covers everything.  A fused norm spans both launches through block_offset / total_blocks.
struct TileMap {
    int strip, rows;       // edge tiles: output columns at each end (0: none), rows a wavefront
    int nxi;               // inner x tiles
    int nyt;               // groups of four rows (a block of inner tiles each)
    int neb;               // blocks of edge tiles a chunk of planes (`rows` groups each)
    int yt_lo, nyi;        // groups of four rows of the inner launch: yt_lo .. yt_lo + nyi - 1
    int tz;
    int block_offset;      // index of this launch's first block among all blocks of the call
    int total_blocks;      // blocks over all launches of the call
    int stream;            // 1: the result is stored past the caches (stream_result)
};

constexpr int kStrips[] = {30, 14, 6};

// tiles of an nx x ny x nz level with the given strips (0: none)
inline TileMap tile_counts(int nx, int ny, int nz, int strip, int tz) {
    TileMap M = {};
    M.tz = tz;
    M.strip = strip;
    M.rows = strip ? 64 / (2 * (strip + 2)) : 1;
    M.nxi = ceil_div(nx + 1 - 2 * strip, kTileX);
    M.nyt = ceil_div(ny + 1, kWavesY);
    M.neb = strip ? ceil_div(M.nyt, M.rows) : 0;
    M.total_blocks = (M.neb + M.nyt * M.nxi) * ceil_div(nz + 1, tz);
    return M;
}

// work a row: inner tiles count one, tiles in the tensor form two; columns lox .. hix are free of stretching
inline double row_cost(int nx, int lox, int hix, int strip) {
    if (strip == 0) {
        int cost = 0;
        for (int x0 = 0; x0 <= nx; x0 += kTileX)
            cost += std::max(1, x0) >= lox && std::min(x0 + kTileX - 1, nx - 1) <= hix ? 1 : 2;
        return cost;
    }
    return ceil_div(nx + 1 - 2 * strip, kTileX) + 2.0 * (2 * (strip + 2)) / 64;
}

inline TileMap make_tiles(int nx, int ny, int nz, int lox, int hix, int tz) {
    int best_strip = 0;
    double best = row_cost(nx, lox, hix, 0);
    for (int strip : kStrips) {
        if (nx < 2 * strip || lox < 1 || lox > strip || hix < nx - strip) continue;
        const double c = row_cost(nx, lox, hix, strip);
        if (c < best) best = c, best_strip = strip;
    }
    return tile_counts(nx, ny, nz, best_strip, tz);
}

// Upper bound of make_tiles' total_blocks over every width of the PML and every depth from tz on: the
// number of partials a fused norm may write.  Taken over the tilings themselves.
inline int stencil_blocks(int nx, int ny, int nz, int tz) {
    int most = tile_counts(nx, ny, nz, 0, tz).total_blocks;
    for (int strip : kStrips)
        if (nx >= 2 * strip) most = std::max(most, tile_counts(nx, ny, nz, strip, tz).total_blocks);
    return most;
}

// Tiles of the fused residual + restriction: x tiles of 60 columns (30 coarse ones), no edge tiles, chunks of
// `depth` coarse planes.
inline TileMap restrict_tiles(int nx, int ny, int nz, int depth) {
    TileMap M = {};
    M.rows = 1;
    M.nxi = std::max(1, ceil_div((nx >> 1) - 1, 30));
    M.nyt = ceil_div(ny + 1, kWavesY);
    M.tz = depth;
    M.total_blocks = M.nxi * M.nyt * ceil_div(nz >> 1, depth);
    return M;
}
// Their depth where the caller fixes none: the least rounds of 512 blocks (two a compute unit) times the fine
// planes of a march, 2 depth + 1 and about four for its start.  Over twenty grids of 32^3 to 352^3 in
// FP32 and FP64 this took 1% longer than the best depth on average and 7% at most.  Half the depth timed for
// the apply, which was used before, moves with that kernel: 19.2 to 20.1 us instead of 17.1 on 84^3 in FP64,
// 31.1 instead of 26.6 on 200 x 72 x 104, 17.8 instead of 14.0 on 64^3.
inline int restrict_depth(int nx, int ny, int nz, int slots) {
    int best = 1;
    long long least = -1;
    for (int d = 1; d <= 32 && d <= std::max(1, nz >> 1); ++d) {
        const long long blocks = (long long)restrict_tiles(nx, ny, nz, d).total_blocks * slots;
        const long long cost = (blocks + 511) / 512 * (2 * d + 5);
        if (least < 0 || cost < least) least = cost, best = d;
    }
    return best;
}

// Whether an apply or a residual on its own stores its result past the caches (non-temporal).  Inside the
// nested maps the next kernel reads the result, and such stores make them slower (S_h at 176^3 260 -> 297 us).  A call
// on its own that fits in the last-level cache (256 MB) leaves its operands there instead: B_h in FP32 at
// 176^3 37.5 -> 29 us, A_2h of a 352^3 grid 37.5 -> 28.6, in FP64 at 144^3 39 -> 30.  Larger calls keep nothing
// (256^3: 112 -> 117 us) and small ones nothing that matters (32^3: 3% slower).
inline bool stream_result(long long bytes) { return bytes >= (16ll << 20) && bytes <= (256ll << 20); }

// Rows and weight nodes that a wavefront reads.  A march goes past the grid on purpose (the last edge
// tile's rows lie up to three beyond ny, the fused restriction starts at plane -1): the indices that
// it loads with are clamped to 0 .. n, and a row is formed with its weights inside the boundary only.
constexpr int clamp_node(int a, int n) { return a < 0 ? 0 : (a > n ? n : a); }
struct MarchRows {
    int m, c, p;   // rows y - 1, y, y + 1
};
constexpr MarchRows march_rows(int y, int ny) {
    return {clamp_node(y - 1, ny), clamp_node(y, ny), clamp_node(y + 1, ny)};
}

}  // namespace helm
