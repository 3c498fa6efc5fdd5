// Which 3D kernel a step takes: a rule on sizes, types and modes.  No HIP
// here, so it also builds with a plain host compiler (a test evaluates it).
#pragma once

#include <stdint.h>

namespace fdk {

constexpr int kShortTX = 64, kShortTY = 16;   // the short kernel's tile: 16 lanes of 4 cells x 16 rows

// Cells of an x-y plane as whole tiles of tx by ty cover it.
inline int64_t covered(int64_t nx, int64_t ny, int64_t tx, int64_t ty)
{
    return (nx + tx - 1) / tx * tx * ((ny + ty - 1) / ty * ty);
}

// The short kernel's planes per block (0: the streaming kernel) and whether
// its accesses bypass the caches.
struct ShortPlan {
    int zc;
    bool stream;
};

// tx, ty: the streaming kernel's tile on this grid.
//
// Up to 22 M padded cells an FP32 grid's fields (12 B per cell) fit the 256 MB
// Infinity Cache and the short kernel is the faster one on every measured
// grid that its 16-row tiles fit (256^3 49-51 us against 50-54, 64 x 512^2 48
// against 51, 128 x 512^2 102 against 96, 64^3 5.0 against 8.2), with 2 planes
// per block below 12 M cells and 4 above (100 x 200 x 300 23.0 / 23.8 us, 201 x
// 333 x 289 61.5 / 58).  Where the tiles reach past the last row they cover
// more than the streaming kernel's 8-row tiles and idle threads still take
// their place: 5% more is outweighed; more than that only if all blocks run in
// one round (100 x 8 x 1000, 800 blocks: a gradient 399 us against 485; 1500 x
// 8 x 300, 3750 blocks: 20.1 us against 16.1), or nearly so with up to 18% (100
// x 65 x 1000, 4000 blocks: a gradient 1634 us against 1767; 100 x 49 x 4000,
// 6300 blocks: 81 us against 67).  Share of rows in use and blocks at which it
// lost: 1/2 and 2000 0.77, 3/4 and 1600 0.90, 5/6 and 4725 0.90 (time of the
// streaming kernel over its own).
//
// Beyond 22 M cells, with accesses that bypass the caches, it stays ahead for
// the adjoint step (384^3 239 against 260 us, 512^3 560 against 562), tiles
// permitting as above, and for the forward step where the streaming tiles are
// mostly padding: nx <= 64 in 128-wide tiles at every size (1024 x 1024 x 64
// 176 against 267 us), 4/3 of the width up to 200 M cells (913 x 912 x 192
// 482 against 529; 1519 x 1519 x 130 1456 against 1397), 6/5 up to 50 M (300^3
// 87 against 94; 577 x 577 x 300 359 against 320).
//
// With 16-bit fields it pays up to 3 M padded cells (BF16, streaming / short:
// 48^3 9.7 / 6.4 us, 66 x 480 x 49 16.9 / 10.0, 96 x 120 x 152 14.3 / 11.8; with
// tiles past the last row 100 x 8 x 1000 11.7 / 8.7, 1000 x 4 x 500 16.9 /
// 21.9); the streaming kernel's fewer, longer blocks read the magnitude words
// and fold a maximum less often, and larger grids keep it.
inline ShortPlan short_plan(int64_t nz, int64_t ny, int64_t nx, int64_t px, bool f32, bool adjoint, int64_t tx,
                            int64_t ty)
{
    const int64_t cells = px * ny * nz;
    const int64_t own = covered(px, ny, kShortTX, kShortTY), other = covered(nx, ny, tx, ty);
    if (cells <= (f32 ? 22000000 : 3000000)) {
        const int zc = cells <= (f32 ? 12000000 : 1000000) ? 2 : 4;
        const int64_t blocks = own / (kShortTX * kShortTY) * ((nz + zc - 1) / zc);
        const bool fits = 100 * own <= 105 * other || blocks <= 1024 || (100 * own <= 118 * other && blocks <= 4096);
        return {fits ? zc : 0, false};
    }
    if (!f32) return {0, false};
    const bool pays = adjoint ? 100 * own <= 105 * other
                              : 100 * other >= 190 * own || (100 * other >= 125 * own && cells <= 200000000) ||
                                    (100 * other >= 115 * own && cells <= 50000000);
    return {pays ? 4 : 0, true};
}

}  // namespace fdk
