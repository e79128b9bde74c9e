// Back projection by image tile: the pieces shared by the data update of a
// plan (lm_tiles.hip) and the back projection of a caller's list
// (lm_back_tiles.hip).
//
// A tile is 8x8x8 or 16x16x16 voxels (TE voxels per edge).  A segment is the
// part of an event's samples that lies on TE consecutive planes along the
// event's dominant axis (planes TE c .. TE c + TE - 1) and reaches one tile.
// Segments are listed per tile, and a workgroup accumulates a tile's
// segments in LDS.
//
// The accumulators are doubles: gfx950 adds doubles into LDS natively
// (ds_add_f64, 9 clocks per wavefront and CU without bank conflicts) while
// its ds_add_f32 takes 193 clocks, and the double sums round less than the
// float sums of the per-event atomics.  A lane owns one (segment, plane)
// sample and adds its four bilinear corners, so 64 / TE segments go through
// a wavefront at a time.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lm_device.hpp"

namespace lmk {

// Tiles of TE voxels per edge over an image (of a single slice: the tile's
// other slices stay empty).
struct TileGeom {
  int ntx, nty, ntz, ntiles;
};

// A ray as the lanes of the segment kernels read it (32 bytes): plane range
// and axis, integer parts of the interpolation coordinates, the float
// coefficients of Ray.  The value of the event's samples (L times the
// back projected value) travels in a list of its own.
struct __align__(16) SegRay {
  int4 a;    // {m0 | nplanes << 10 | axis << 20, I1 & 0xffff | I2 << 16, F1, V1}
  float4 b;  // {F2, V2, C, B}
};
static_assert(sizeof(SegRay) == 32, "two records per 64-byte sector");

// Images whose rays fit the record: planes and sizes up to 512 (the
// library's largest image) and integer parts of at most n + 3 planes of the
// steepest ray, max h / min h voxels per plane, in 16 bits.
constexpr double kMaxVoxelRatio = 1024.0;

__device__ __forceinline__ SegRay pack_seg_ray(const Ray &r) {
  SegRay s;
  s.a = make_int4(r.m0 | (r.nplanes << 10) | (r.a << 20), (r.I1 & 0xffff) | (int)((unsigned)r.I2 << 16),
                  __float_as_int(r.F1), __float_as_int(r.V1));
  s.b = make_float4(r.F2, r.V2, r.C, r.B);
  return s;
}
__device__ __forceinline__ SegRay empty_seg_ray() {
  SegRay s;
  s.a = make_int4(0, 0, 0, 0);
  s.b = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  return s;
}
__device__ __forceinline__ int seg_m0(const SegRay &s) { return s.a.x & 1023; }
__device__ __forceinline__ int seg_np(const SegRay &s) { return (s.a.x >> 10) & 1023; }
__device__ __forceinline__ int seg_axis(const SegRay &s) { return s.a.x >> 20; }
__device__ __forceinline__ int seg_i1(const SegRay &s) { return (int)(short)(s.a.y & 0xffff); }
__device__ __forceinline__ int seg_i2(const SegRay &s) { return s.a.y >> 16; }

// Calls f(tile) for every tile that a corner of a sample of the ray on planes
// [TE ta, TE ta + TE - 1] can reach, for every ta the ray visits.  The coordinate
// of a sample, fmaf(j, V, F), is monotonic in j, so its range over a chunk
// of planes is that of the chunk's end samples.
template <int TE, class F>
__device__ __forceinline__ void for_each_segment(const GeomDev &g, const SegRay &s, const TileGeom &tg, F f) {
  const int np = seg_np(s);
  if (np <= 0) return;
  const int a = seg_axis(s), m0 = seg_m0(s), i1 = seg_i1(s), i2 = seg_i2(s);
  const float F1 = __int_as_float(s.a.z), V1 = __int_as_float(s.a.w), F2 = s.b.x, V2 = s.b.y;
  const int n1 = a == 0 ? g.n[1] : g.n[0], n2 = a == 2 ? g.n[1] : g.n[2];
  const int last = m0 + np - 1;
  for (int ta = m0 / TE; ta <= last / TE; ++ta) {
    const int jlo = max(0, ta * TE - m0), jhi = min(np - 1, ta * TE + TE - 1 - m0);
    const float u1a = fmaf((float)jlo, V1, F1), u1b = fmaf((float)jhi, V1, F1);
    const float u2a = fmaf((float)jlo, V2, F2), u2b = fmaf((float)jhi, V2, F2);
    const int f1a = i1 + (int)floorf(u1a), f1b = i1 + (int)floorf(u1b);
    const int f2a = i2 + (int)floorf(u2a), f2b = i2 + (int)floorf(u2b);
    const int lo1 = max(min(f1a, f1b), 0), hi1 = min(max(f1a, f1b) + 1, n1 - 1);
    const int lo2 = max(min(f2a, f2b), 0), hi2 = min(max(f2a, f2b) + 1, n2 - 1);
    if (lo1 > hi1 || lo2 > hi2) continue;
    for (int t1 = lo1 / TE; t1 <= hi1 / TE; ++t1)
      for (int t2 = lo2 / TE; t2 <= hi2 / TE; ++t2) {
        const int tx = a == 0 ? ta : t1;
        const int ty = a == 0 ? t1 : (a == 1 ? ta : t2);
        const int tz = a == 2 ? ta : t2;
        f((tz * tg.nty + ty) * tg.ntx + tx);
      }
  }
}

// The accumulators of a tile of TE voxels per edge (8 or 16), with a margin
// of one voxel on every side that takes the corners of its samples that
// belong to a neighbour (and is thrown away): voxel (i, j, k) of the tile at
// (i + 1) + Y (j + 1) + Z (k + 1).  Y and Z are odd, so the planes of a
// segment, 1, Y or Z doubles apart, are on different LDS banks.
template <int TE>
struct AccShape {
  static constexpr int Y = TE + 3, Z = Y * (TE + 2) + 1;
  static constexpr int size = Z * (TE + 2);
  static_assert(Y % 2 == 1 && Z % 2 == 1, "odd strides");
};

__device__ __forceinline__ void lds_add(char *p, float v) {
  __hip_atomic_fetch_add((double *)p, (double)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// What a lane (plane p of the segments' TE planes) needs of its workgroup's
// tile: the tile's origin (ox, oy, oz) and, per axis, origin + p and the
// accumulator offset (bytes) of plane p, the margin included.
template <int TE>
struct TileLane {
  int ox, oy, oz;
  int px, py, pz;
  float ax, ay, az;
};
template <int TE>
__device__ __forceinline__ TileLane<TE> tile_lane(int ox, int oy, int oz, int p) {
  using S = AccShape<TE>;
  TileLane<TE> t;
  t.ox = ox;
  t.oy = oy;
  t.oz = oz;
  t.px = ox + p;
  t.py = oy + p;
  t.pz = oz + p;
  constexpr int margin = 1 + S::Y + S::Z;
  t.ax = 8.0f * (float)(p + margin);
  t.ay = 8.0f * (float)(p * S::Y + margin);
  t.az = 8.0f * (float)(p * S::Z + margin);
  return t;
}

// Adds the sample of ray s on the lane's plane, with event value val, where
// `on`.  A value that is not finite reaches the corners of the samples inside
// the TOF window (also corners of weight 0).  The corner's place in the
// accumulators is computed in float (whole numbers below 2^24, exact): the
// voxel coordinates are floats already and an integer product takes four
// times as long.
template <int TM, int TE>
__device__ __forceinline__ void add_sample(const GeomDev &g, const TileLane<TE> &t, const SegRay &s, float val,
                                           bool on, float D, const TofTab &tu, const float4 *tab, char *acc) {
  using S = AccShape<TE>;
  const int a = seg_axis(s);
  const bool x_dom = a == 0, z_dom = a == 2;
  const int j = sel3(a, t.px, t.py, t.pz) - seg_m0(s);
  const float fj = (float)j;
  const float u1 = fmaf(fj, __int_as_float(s.a.w), __int_as_float(s.a.z)), u2 = fmaf(fj, s.b.y, s.b.x);
  const float fl1 = floorf(u1), fl2 = floorf(u2);
  const float f1 = u1 - fl1, f2 = u2 - fl2;
  // corner 0 relative to the tile
  const float l1 = (float)(seg_i1(s) - sel3(a, t.oy, t.ox, t.ox)) + fl1;
  const float l2 = (float)(seg_i2(s) - sel3(a, t.oz, t.oz, t.oy)) + fl2;
  const float tc = TM != kTofNone ? fmaf(-fj, s.b.w, s.b.z) : 0.0f;
  // on the ray, in the window, and a corner in the tile
  if (on && (unsigned)j < (unsigned)seg_np(s) && (TM != kTofTable || fabsf(tc) < tu.te) && l1 >= -1.0f &&
      l1 < (float)TE && l2 >= -1.0f && l2 < (float)TE) {
    float v = val;
    if constexpr (TM == kTofTable) v *= tof_weight_tab(tu, tab, tc);
    if constexpr (TM == kTofErfc) {
      const float vh = fmaf(0.5f, D, tc), w = tof_weight(vh, vh - D, g.vclip, g.inv_norm);
      v = w != 0.0f ? val * w : 0.0f;
    }
    const float d1 = x_dom ? 8.0f * S::Y : 8.0f, d2 = z_dom ? 8.0f * S::Y : 8.0f * S::Z;
    const int at = (int)fmaf(l1, d1, fmaf(l2, d2, sel3(a, t.ax, t.ay, t.az)));
    const int s1 = x_dom ? 8 * S::Y : 8, s2 = z_dom ? 8 * S::Y : 8 * S::Z;
    const float g1 = 1.0f - f1, vg = v * (1.0f - f2), vf = v * f2;
    char *q = acc + at;
    lds_add(q, vg * g1);
    lds_add(q + s1, vg * f1);
    lds_add(q + s2, vf * g1);
    lds_add(q + (s1 + s2), vf * f1);
  }
}

// Adds the segments seg[0 .. cnt) (event numbers into rays and val) of the
// workgroup's tile: a wavefront takes 64 / TE segments at a time, one per
// group of TE lanes (lane = plane), wavefront wv of nw the wv-th group of
// them and every nw-th after.  A segment's number is loaded two steps and its
// ray one step before they are used, in that order, so that waiting for a
// number leaves the rays in flight; two steps per turn of the loop, so that
// no register is copied (a copy would wait for the loads).  cnt is at most
// kMaxSegments, whose byte offsets and those of the loads ahead fit 32 bits.
constexpr int kMaxSegments = 1 << 29;
template <int TM, int TE>
__device__ __forceinline__ void add_segments(const GeomDev &g, const TileLane<TE> &t, const unsigned *__restrict__ seg,
                                             int cnt, const SegRay *__restrict__ rays,
                                             const float *__restrict__ val, float D, const TofTab &tu,
                                             const float4 *tab, double *acc, int wv, int nw, int lane) {
  constexpr int kSegs = 64 / TE;
  const int k0 = kSegs * wv, sub = lane / TE, step = kSegs * nw;
  if (k0 >= cnt) return;
  // numbers past the end are clamped to the last one; their samples are not added
  const unsigned lim = 4u * (unsigned)(cnt - 1);
  auto num = [&](unsigned byte) { return *(const unsigned *)((const char *)seg + min(byte, lim)); };
  auto ray = [&](unsigned e) {
    SegRay r;
    r.a = rays[e].a;
    r.b = rays[e].b;
    return r;
  };
  unsigned byte = 4u * (unsigned)(k0 + sub);
  const unsigned bstep = 4u * (unsigned)step;
  unsigned eA = num(byte), eB = num(byte + bstep);
  SegRay rA = ray(eA);
  float vA = val[eA];
  for (int k = k0; k < cnt; k += 2 * step, byte += 2 * bstep) {
    eA = num(byte + 2 * bstep);
    const SegRay rB = ray(eB);
    const float vB = val[eB];
    add_sample<TM, TE>(g, t, rA, vA, byte <= lim, D, tu, tab, (char *)acc);
    eB = num(byte + 3 * bstep);
    rA = ray(eA);
    vA = val[eA];
    add_sample<TM, TE>(g, t, rB, vB, byte + bstep <= lim, D, tu, tab, (char *)acc);
  }
}

bool segs_supported(const GeomDev &g);
TileGeom tile_geom(const int n[3], int te);
// Upper bound of the segments (tiles of edge te) of one event that visits at
// most maxp planes; slack: voxels for the corners of float32 coordinates that
// round across a voxel's edge (1 is enough).
long long segs_per_event(const GeomDev &g, int maxp, int te, int slack);

// Back projection of a caller's list (ev, or a plan's records rec when ev is
// NULL) by tile, img += P^T v in the layout of g (lm_back_tiles.hip), in
// batches whose temporaries take at most `room` bytes.  queued is false, with
// nothing enqueued, when the list is too short, the image does not qualify or
// the temporaries do not fit.
// room of back_tiles_min_bytes is enough.
size_t back_tiles_min_bytes(const GeomDev &g, long long n);
int launch_back_tiles(const GeomDev &g, const float *v, const int16_t *ev, const int4 *rec, long long n, float *img,
                      size_t room, hipStream_t st, bool &queued);

}  // namespace lmk
