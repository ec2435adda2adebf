// How a lattice, or the lattices of a batch, take a time step: in two launches
// or in one, and the shape of the one.  A rule on sizes, storage precision and
// compute units, applied once when a domain or batch is made.
#pragma once

#include "lbboil.h"

#include "lbb_step.hpp"

#include <algorithm>
#include <cstdint>
#include <vector>

namespace {

struct StepDims {
    int nx, ny;
};

// How lattices step: two launches (height 0), or one in tiles or marching
// strips of `height` rows, or one in the LB tiles of isothermal lattices.
struct StepForm {
    int height = 0;
    bool march = false;
    bool lb = false;
};

// ---- the one-launch step (k_step, k_march) ----
//
// Where tiles (k_step) are taken.  They recompute a halo of five rows and
// columns, so they pay while a step is bound by launch and phase latencies,
// not by the work itself: when tiles of some height fit the compute units in
// one round.  Timed on graph replays, one launch against two (us per step):
// 128x64 FP64 7.1 against 13.1, 301x77 FP32 6.6 against 12.1, 600x151 FP32 8.5
// against 12.6, 511x257 FP64 10.9 against 15.4, 512x256 FP32 8.9 against 12.7,
// 1024x512 FP32 20.2 against 22.7.  One block more than compute units costs a
// second round (600x151: 18.3 with 912 blocks, 14.6 with 612, 9.2 with 228),
// and a block alone on a compute unit cannot hide its loads under another's
// arithmetic (2048x1024: 77 against 64).
//
// The tile height is the smallest that fits one round, but at least 4: lower
// tiles only add halo (128x64: 7.0-7.1 for heights 1 to 4; 256x128 FP64 8.1
// with 3 and 7.9 with 4; 600x151 9.2 with 8, 10.1 with 13, 12.6 with 22).
//
// Where marching strips (k_march) are taken: from the size on at which strips
// of march_min rows fill every wave slot.  The height is then the smallest
// that still fits one round, up to kMarchMax, where more rows no longer pay
// (4096x2048 FP32: 205, 202, 202 us with 26, 32, 53 rows; two launches 275).
// Below, too few rows a wave leave too much halo: 2048x1024 FP32 61 us either
// way with 14 rows, 1024x512 36 against 22 with 8; FP64 gains earlier, since its
// two launches are slower: 1500x700 51 against 59 with 11 rows.  Heights are 2
// modulo 3: with the ten rows of the halo whole turns of the kernel's loop.
constexpr int kStepMinHeight = 4;
constexpr int kMarchWaves = 4;  // waves of a block
constexpr int kMarchMax = 53;
constexpr int march_min(int precision) { return precision == LBB_FP64 ? 11 : 17; }
// Every wave adds up the mass partials of its lattice's blocks before its first
// row, so that work would grow with the square of the lattice: higher strips
// keep the partials of a lattice below this (ms per step FP32, two launches /
// strips of 53 rows / higher ones: 8192x24576, 17632 partials, 6.58 / 4.96 /
// 4.98; 8192x65536, 17.3 / 16.3 / 14.2; 8192x131000, 34.0 / 41.6 / 29.5).
constexpr int kMarchMaxPartials = 8192;
constexpr int kMarchMinNy = 32;     // rows a strip's halo may wrap around once
constexpr int kMarchMaxNx = 8192;   // its one block for the heat flux walks the bottom rows
// region rows a block of 16 waves has room for: four rows a wave in FP32,
// three in FP64 (whose planes take twice the LDS)
constexpr int step_max_rows(int precision) { return precision == LBB_FP64 ? 48 : 64; }

// Blocks of a lattice (without the one for its bookkeeping).
int64_t step_blocks(const StepDims &l, const StepForm &f)
{
    if (!f.height) return 0;
    const int width = f.lb ? lbb::TXA : lbb::TXF;
    const int64_t tiles = (int64_t)((l.nx + width - 1) / width) * ((l.ny + f.height - 1) / f.height);
    return f.march ? (tiles + kMarchWaves - 1) / kMarchWaves : tiles;
}

// Isothermal lattices step in one launch of k_lb (ONE, default tiles) where
// every block can add up the mass partials of the tiles with few loads a
// thread: up to 2048 rows of tile columns, four of which make a tile.  Eleven
// 160x60 FP64 lattices: 7.3 us per step against 11.1 with the temperature
// launch, which only reduces.  Tuned shapes do not matter to it: 248x512 FP64
// 7.2 us, against 9.8 in two launches of the fastest shapes.
constexpr int kOneMaxRows = 2048;

// One block of a lattice samples the heat flux of its bottom row in every
// step, a chunk of TXB columns a wave; on wide lattices of few rows it is the
// last to end.  Isothermal (four waves; us per step, one launch / two): 1000x120
// FP64 7.5 / 10.4, 1500x80 9.4 / 10.5 (a step with its flush 14.4 / 13.6),
// 2000x60 11.4 / 11.1, 8000x15 34 / 12.  Tiles (16 waves): 3400x16 FP32
// 7.7 / 11.3, 5000x100 21.0 / 22.6, 6800x8 FP64 14.3 / 12.0, 13700x4 24.4 / 13.4,
// but 13700x38 29.3 / 37.1: tall tiles take longer than the sample.
constexpr int kOneMaxChunks = 28;
constexpr int kTileMaxChunks = 96, kTileLongRows = 32;
constexpr int heat_flux_chunks(int nx) { return (nx + lbb::TXB - 1) / lbb::TXB; }

// Form of the step of lattices that step together.
StepForm step_form(const std::vector<StepDims> &ls, int precision, int mode, int ncu)
{
    StepForm f;
    if (mode == LBB_ISOTHERMAL) {
        for (const StepDims &l : ls)
            if ((int64_t)((l.nx + lbb::TXA - 1) / lbb::TXA) * l.ny > kOneMaxRows ||
                heat_flux_chunks(l.nx) > kOneMaxChunks)
                return f;
        f.height = lbb::kShapeA[0].ty;
        f.lb = true;
        return f;
    }
    if (mode != LBB_COUPLED) return f;
    auto blocks = [&](const StepForm &g) {
        int64_t n = 0;
        for (const StepDims &l : ls) n += step_blocks(l, g) + 1;
        return n;
    };
    bool wide = false;
    for (const StepDims &l : ls) wide = wide || (heat_flux_chunks(l.nx) > kTileMaxChunks && l.ny < kTileLongRows);
    for (f.height = kStepMinHeight; f.height + 2 * lbb::HF <= step_max_rows(precision); ++f.height)
        if (blocks(f) <= ncu) return wide ? StepForm{} : f;
    f = StepForm{march_min(precision), true};
    const int64_t slots = (int64_t)ncu * (precision == LBB_FP64 ? 2 : 3);  // blocks resident at once
    for (const StepDims &l : ls)
        if (l.ny < kMarchMinNy || l.nx > kMarchMaxNx) return StepForm{};
    if (blocks(f) <= slots) return StepForm{};
    while (f.height < kMarchMax && blocks(f) > slots) f.height += 3;
    for (const StepDims &l : ls)
        while (step_blocks(l, f) > kMarchMaxPartials) f.height += 3;
    return f;
}

// Most blocks any form gives a lattice alone or in a batch (a batch's tiles
// and strips are no lower than a lattice's own).
int64_t step_max_blocks(const StepDims &l, int precision, int mode, int ncu)
{
    const StepForm own = step_form({l}, precision, mode, ncu);
    return std::max(own.march ? 0 : step_blocks(l, own), step_blocks(l, StepForm{march_min(precision), true}));
}

}  // namespace
