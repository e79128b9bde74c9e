// The data update of LM-SPDHG by image tile (lm_tiles.hip): the back
// projection of a subset's dual increments is binned by 8x8x8-voxel tile
// once, at plan creation, so that each update accumulates every tile in LDS
// without global atomics and applies the z / zbar / primal step to the
// tile's voxels in the same kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "lm_device.hpp"
#include "lm_segs.hpp"

namespace lmk {

// Per-plan state of the tile path; `on` false: the per-event path runs.
struct TilePlan {
  bool on = false;
  TileGeom tg{};
  int maxp = 0;                  // plane bound of every event (setup_ray's clamp)
  long long *seg_off = nullptr;  // [nsub * ntiles + 1] first entry of seg of (subset, tile), all subsets in a row
  unsigned *seg = nullptr;       // events (relative to the subset's first) of every tile, by subset and tile
  int *order = nullptr;          // tiles by decreasing load (launch order of phase 2)
  SegRay *rays = nullptr;        // rays and back projected values of the subset being updated
  float *cf = nullptr;
  TofTab tt{};                   // layout of the tabulated TOF weights
  float4 *tab = nullptr;         // the table (nullptr: erfc, or no TOF)
  size_t bytes = 0;              // device bytes of the above
};

bool tiles_supported(const GeomDev &g);

// Upper bound of the device bytes the tile path of a plan of n events in
// nsub subsets holds (segments, offsets, launch order, the rays and values of
// the largest subset) plus its temporaries at creation; 0 when the geometry
// does not qualify.  Each event has at most one segment per tile
// that its corners reach on 8 consecutive planes.
size_t tile_bytes_bound(const GeomDev &g, long long n, int nsub);

// Builds the segment lists of every subset of the plan's stored events
// (subset i at rec[off[i] .. off[i+1])).  Device memory that the plan keeps
// is allocated stream-ordered and appended to `owned` (the plan frees it);
// temporaries are freed before returning.  Returns LM_OK with tp.on ==
// false when the geometry does not qualify or the segments do not fit (the
// per-event path then runs), an error code for a failed HIP call.
// Synchronous.
int build_tiles(const GeomDev &g, const int4 *rec, const std::vector<int> &off, TilePlan &tp,
                std::vector<void *> &owned, hipStream_t st);

// Phase 1 of a data update of the subset stored at positions [o, o + n):
// forward projection, dual prox, and the subset's rays and back projected
// values.
int launch_tile_fwd(const GeomDev &g, const TilePlan &tp, const float *x, const int4 *rec, const float *S,
                    const float *mu, float *cdual, long long o, long long n, hipStream_t st);
// Phase 2: back projection of these by tile; dz_out != NULL writes dz (every voxel of
// the layout) instead of the z / zbar / primal step.
int launch_tile_back(const GeomDev &g, const TilePlan &tp, int subset, float *z, float *x, const float *T,
                     float *zbar, float *dz_out, float inv_p, bool fuse, hipStream_t st);

}  // namespace lmk
