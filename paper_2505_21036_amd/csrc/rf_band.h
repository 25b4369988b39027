// What the lists of the banded patterns and the table of the position-major order say, by arithmetic, for workgroups that
// split a block's keys and would wait for both before their first tile: the same on the host and on the device.
#pragma once
#include "rf_internal.h"
#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define RF_BAND_BOTH __host__ __device__ __forceinline__
#else
#define RF_BAND_BOTH inline
#endif

namespace rf {

// The tiles that a block of rows visits under a band of radius r over groups of consecutive rows, as build_plan lists them:
// one run of tiles with keys of groups within reach, then those with text keys; a block with text rows visits all.
struct BandTiles {
    int run, run_tiles;    // the run's first tile, and how many they are
    int text;              // first of the other tiles
    int tiles;             // in all
    int all_from, all_to;  // every row of the block keeps the video keys all_from .. all_to - 1
    RF_BAND_BOTH BandTiles() {}
    RF_BAND_BOTH BandTiles(int q0, int block, int group, int r, int N, int Nv) {
        const int q1 = q0 + block < N ? q0 + block : N, last = (q1 < Nv ? q1 : Nv) - 1, nKT = (N + kTileK - 1) / kTileK;
        const bool has_video = q0 < Nv, has_text = q1 > Nv;
        const int lo = q0 / group, hi = last / group;
        all_from = has_video ? (hi - r) * group : 0;
        all_to = has_video ? (lo + r + 1) * group : Nv;
        const int reach = (hi + r + 1) * group;
        run = has_text || lo < r ? 0 : (lo - r) * group / kTileK;
        const int end = has_text ? nKT : ((reach < Nv ? reach : Nv) + kTileK - 1) / kTileK;
        const int first_text = N > Nv ? Nv / kTileK : nKT;
        run_tiles = end - run;
        text = end > first_text ? end : first_text;
        tiles = run_tiles + nKT - text;
    }
    // entry t of the list
    RF_BAND_BOTH int entry(int t, int N, int Nv) const {
        const int tile = t < run_tiles ? run + t : text + t - run_tiles, k0 = tile * kTileK, k1 = k0 + kTileK;
        const bool all = k0 >= Nv || (k0 >= all_from && (k1 < Nv ? k1 : Nv) <= all_to), tail = k1 > N, mixed = k1 > Nv && k0 < Nv;
        return tile | (!all || tail ? RF_PLAN_PARTIAL : 0) | (tail || (mixed && !all) ? kTileBoundary : 0);
    }
};

// Tensor row of row n of the position-major order (the plan's pm_token): T rows a position, HW tokens a frame.  n is below 2^24
// and exact as a float; its product with 1 / T is less than one off, and so the quotient at most one.
RF_BAND_BOTH int position_major_row(int n, int T, int HW, int Nv, int video_shift, int text_shift) {
    int at = static_cast<int>(static_cast<float>(n) * (1.f / static_cast<float>(T))), frame = n - at * T;
    const int off = (frame >= T ? 1 : 0) - (frame < 0 ? 1 : 0);
    at += off;
    frame -= off * T;
    return n < Nv ? frame * HW + at + video_shift : n + text_shift;
}

}  // namespace rf
