// What the kernels of the filter gradient share (wgrad.hip, wgrad_split.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "plan.hpp"

namespace dwm {

struct WgradArgs {
    int K, Kp, T, tblocks;       // filters, filters rounded up to whole output tiles, tiles, blocks of 64 tiles
    int dm_rows, vblock_rows;    // rows of one dM block / one V block
    int n_planes, n_tiles;
    int splits, chunks_per_split;
    long long split_floats;      // floats of one split's partial dU
    int tile0[kMaxPlanes + 1];   // first output tile of each plane
    int nlt[kMaxPlanes];         // l tiles of each plane (64 wide; wgrad_split.hip: 128)
    int vrow[kMaxPlanes];        // first V row of each plane
    int poff64[kMaxPlanes];      // offset of the plane's dU[Kp][lstride] inside a split, in units of 64 floats
    int lreal[kMaxPlanes];       // rows of each plane that are not padding
    // The plane's dM: which of the n_dm written ones, whether negated (bit 8), its pattern (bits 16..23, see
    // DevPlaneEntry::coef).  A^T's columns are y0, y0+y1, y0-y1, -y1 or fewer for every piece length, so that at most 16 of
    // up to 81 planes differ by more than sign.
    int dmp[kMaxPlanes];
    int n_dm;
    int lstride[kMaxPlanes];     // floats between consecutive filters k of the plane's dU
};

struct DyShape {
    int T, K, Kp, TH, TW, OH, OW, dm_rows;
};

// wgrad_split.hip: A dY A^T split three ways, and the GEMM over the tiles on the bfloat16 matrix cores
constexpr int kWsplitTile = 128;  // filters and rows of its output tile
dwm_status_t launch_wgrad_split(const WgradArgs& a, const DyShape& ds, const PlaneTable& dm_table, const float* dy,
                                const float* V, unsigned char* dm, float* partial, hipStream_t stream);

}  // namespace dwm
