// Back projection of an event list by image tile.
//
// The per-event kernel adds every sample with float atomics, which gfx950
// executes beyond the L2 at about 2e10 requests/s: ~50 requests per event,
// 2.5 ms per 1e6 events whatever the image.  Here a batch of events is first
// binned by 16x16x16-voxel tile on the GPU: a count and a placement pass
// with per-workgroup histograms in LDS (one global atomic per workgroup and
// tile instead of one per segment) write, per tile, the numbers of the
// events that reach it; then workgroups accumulate part of a tile's list in
// LDS and add the tile to the image, one atomic request per 16 voxels.
//
// 1e7 events on 200x200x96: 25.2 -> 3.2 ms (counting 0.37, placing 0.50,
// accumulating 2.5 under the profiler); 4 x 1e6 events on 128x128x48 with a TOF window of 43
// planes 6.5 -> 1.3 ms; 1e5 events without TOF on 121x127x47 0.64 -> 0.13 ms.
// The accumulation is bound by its LDS adds (the LDS is busy 74 % of its time)
// and by the rays and values of its segments, which come from beyond the L2 at
// 5.6 to 6.3 TB/s; the placement by its scattered 4-byte stores.  Tiles of 8
// voxels per edge took 3.2 ms to accumulate and 1.7 ms to place the 1e7
// events: an event has 14 segments in those, 6 in tiles of 16.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "lm_host.hpp"
#include "lm_segs.hpp"

using namespace lmk;

namespace {

constexpr int kTL = 16;           // tile edge of the list path
constexpr int kBinBlock = 512;   // threads of the binning kernels
constexpr int kItemMin = 256, kItemMax = 2048;  // segments of a tile per work item
constexpr int kBackBlock = 512;
constexpr int kBackGrid = 256 * 3;  // work items are strided over this many workgroups

__global__ __launch_bounds__(256) void k_zero_u32(unsigned *p, long long n) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) p[i] = 0u;
}

// Adds an event to the image by one lane: the per-event projector's samples
// and conditions (corners of weight 0 add nothing).
__device__ void scatter_event(const GeomDev &g, const Ray &r, float c, float *img) {
  for (int j = 0; j < r.nplanes; ++j) {
    const Sample s = sample_at(g, r, j, g.tof_on);
    const float cs = c * s.w;
    for (int q = 0; q < 4; ++q) {
      float wc;
      const int ix = corner(g, r, s, q, wc);
      if (cs != 0.0f && ix >= 0 && wc != 0.0f) atomicAdd(img + ix, cs * wc);
    }
  }
}

// Rays, sample values and tile totals of a batch.  An event that is out of
// range, has value zero or misses the image gets an empty ray, and so does
// one whose value is not finite, which is added to the image here (the tile
// kernel adds all four corners of a sample, also those of weight 0).
__global__ __launch_bounds__(kBinBlock) void k_list_count(GeomDev g, TileGeom tg, int maxp, const int16_t *ev,
                                                          const int4 *rec, const float *__restrict__ v, int n,
                                                          int chunk, SegRay *__restrict__ rays,
                                                          float *__restrict__ val, unsigned *tot,
                                                          unsigned *__restrict__ base, float *img) {
  extern __shared__ unsigned h[];
  for (int t = threadIdx.x; t < tg.ntiles; t += kBinBlock) h[t] = 0u;
  __syncthreads();
  const int e1 = min(n, ((int)blockIdx.x + 1) * chunk);
  for (int e = blockIdx.x * chunk + threadIdx.x; e < e1; e += kBinBlock) {
    int id1 = 0, id2 = 0, k = 0;
    const float ve = v[e];
    bool ok = ve != 0.0f;
    if (ev) {
      ok = ok && decode_event(g, ev + 5 * (long long)e, id1, id2, k);
    } else {
      const int4 r = rec[e];
      id1 = r.x;
      id2 = r.y;
      k = r.z;
    }
    SegRay s = empty_seg_ray();
    float c = 0.0f;
    if (ok) {
      const Ray r = setup_ray(g, id1, id2, k, W_BIN, maxp);
      c = r.L * ve;
      if (fabsf(c) < INFINITY) s = pack_seg_ray(r);
      else scatter_event(g, r, c, img);
    }
    rays[e] = s;
    val[e] = c;
    for_each_segment<kTL>(g, s, tg, [&](int t) { atomicAdd(&h[t], 1u); });
  }
  __syncthreads();
  // the workgroup's place within each tile is what the tile's count was
  base += (long long)tg.ntiles * blockIdx.x;
  for (int t = threadIdx.x; t < tg.ntiles; t += kBinBlock)
    if (h[t]) base[t] = atomicAdd(tot + t, h[t]);
}

// First segment of every tile (off, ntiles + 1 entries) and the work items:
// item i takes the segments of tile items[i].x from items[i].y on, at most
// nitems[1] of them; nitems[0] = the number of items.  The size of an item
// leaves a few items per workgroup of the accumulating kernel's grid where
// the list is long enough, between kItemMin (its tile must still be cleared
// and added) and kItemMax segments.  One workgroup.
__global__ __launch_bounds__(1024) void k_list_items(const unsigned *__restrict__ tot, int ntiles, unsigned *off,
                                                     uint2 *items, unsigned *nitems) {
  __shared__ unsigned sc[1024], si[1024];
  const int t = threadIdx.x;
  const int per = (ntiles + 1023) / 1024;
  const int a = min(ntiles, t * per), b = min(ntiles, a + per);
  unsigned c = 0;
  for (int i = a; i < b; ++i) c += tot[i];
  sc[t] = c;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const unsigned ac = t >= o ? sc[t - o] : 0u;
    __syncthreads();
    sc[t] += ac;
    __syncthreads();
  }
  const unsigned total = sc[1023];
  const unsigned size = min(max(total / (4u * kBackGrid), (unsigned)kItemMin), (unsigned)kItemMax);
  unsigned m = 0;
  for (int i = a; i < b; ++i) m += (tot[i] + size - 1) / size;
  si[t] = m;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const unsigned ai = t >= o ? si[t - o] : 0u;
    __syncthreads();
    si[t] += ai;
    __syncthreads();
  }
  unsigned rc = sc[t] - c, ri = si[t] - m;
  for (int i = a; i < b; ++i) {
    off[i] = rc;
    for (unsigned s = 0; s < tot[i]; s += size) items[ri++] = make_uint2((unsigned)i, rc + s);
    rc += tot[i];
  }
  if (t == 1023) {
    off[ntiles] = total;
    nitems[0] = si[1023];
    nitems[1] = size;
  }
}

// Lists the events of every tile: seg[off[t] ..] of tile t, each workgroup
// in the range that it reserved when counting (tiles that it did not count
// have none, and are not met here).
__global__ __launch_bounds__(kBinBlock) void k_list_place(GeomDev g, TileGeom tg, const SegRay *__restrict__ rays,
                                                          int n, int chunk, const unsigned *__restrict__ off,
                                                          const unsigned *__restrict__ base,
                                                          unsigned *__restrict__ seg) {
  extern __shared__ unsigned h[];
  base += (long long)tg.ntiles * blockIdx.x;
  for (int t = threadIdx.x; t < tg.ntiles; t += kBinBlock) h[t] = off[t] + base[t];
  __syncthreads();
  const int e0 = blockIdx.x * chunk, e1 = min(n, e0 + chunk);
  for (int e = e0 + threadIdx.x; e < e1; e += kBinBlock)
    for_each_segment<kTL>(g, rays[e], tg, [&](int t) { seg[atomicAdd(&h[t], 1u)] = (unsigned)e; });
}

// Accumulates the work items and adds them to the image.
template <int TM>
__global__ __launch_bounds__(kBackBlock) void k_list_back(GeomDev g, TileGeom tg, const unsigned *__restrict__ off,
                                                          const uint2 *__restrict__ items,
                                                          const unsigned *__restrict__ nitems,
                                                          const unsigned *__restrict__ seg,
                                                          const SegRay *__restrict__ rays,
                                                          const float *__restrict__ val, TofTab tt,
                                                          const float4 *__restrict__ tab, float *img) {
  using S = AccShape<kTL>;
  __shared__ double acc[S::size];
  extern __shared__ float4 stab[];
  const unsigned ni = nitems[0];
  if (blockIdx.x >= ni) return;
  if constexpr (TM == kTofTable)
    for (int i = threadIdx.x; i < tof_tab_size(tt); i += kBackBlock) stab[i] = tab[i];
  const TofTab tu = tof_tab_uniform(tt);
  const float D = tof_bin_width(g);
  const int lane = threadIdx.x & 63;
  for (unsigned it = blockIdx.x; it < ni; it += gridDim.x) {
    const uint2 w = items[it];
    const int cnt = (int)min(off[w.x + 1] - w.y, nitems[1]);
    const int tile = (int)w.x, ox = tile % tg.ntx * kTL, oy = (tile / tg.ntx) % tg.nty * kTL,
              oz = tile / (tg.ntx * tg.nty) * kTL;
    for (int i = threadIdx.x; i < S::size; i += kBackBlock) acc[i] = 0.0;
    __syncthreads();
    add_segments<TM, kTL>(g, tile_lane<kTL>(ox, oy, oz, lane % kTL), seg + w.y, cnt, rays, val, D, tu, stab, acc,
                          threadIdx.x >> 6, kBackBlock / 64, lane);
    __syncthreads();
    // voxels in brick order: 16 consecutive threads on one 64-byte sector
    constexpr int kB = kTL / 4;  // bricks per edge
    for (int q = threadIdx.x; q < kTL * kTL * kTL; q += kBackBlock) {
      const int b = q >> 6;
      const int i = (b % kB) * 4 + (q & 3), j = (b / kB % kB) * 4 + ((q >> 2) & 3), k = b / (kB * kB) * 4 + ((q >> 4) & 3);
      const float d = (float)acc[(i + 1) + S::Y * (j + 1) + S::Z * (k + 1)];
      if (d != 0.0f && ox + i < g.n[0] && oy + j < g.n[1] && oz + k < g.n[2])
        atomicAdd(img + vidx(g.lay, ox + i, oy + j, oz + k), d);
    }
    __syncthreads();
  }
}

}  // namespace

namespace lmk {

TileGeom tile_geom(const int n[3], int te) {
  TileGeom t;
  t.ntx = (n[0] + te - 1) / te;
  t.nty = (n[1] + te - 1) / te;
  t.ntz = (n[2] + te - 1) / te;
  t.ntiles = t.ntx * t.nty * t.ntz;
  return t;
}

bool segs_supported(const GeomDev &g) {
  if (g.lay.sx != 2 || g.lay.sy != 2) return false;
  const double hmin = std::min(g.h[0], std::min(g.h[1], g.h[2])), hmax = std::max(g.h[0], std::max(g.h[1], g.h[2]));
  return hmax <= kMaxVoxelRatio * hmin;
}

long long segs_per_event(const GeomDev &g, int maxp, int te, int slack) {
  // chunks of te planes along axis a, and tiles a chunk can reach along axis
  // b: the corners span at most ceil((te - 1) h_a / h_b) + 2 voxels and the
  // slack (and at most the axis)
  long long most = 1;
  for (int a = 0; a < 3; ++a) {
    long long m = (std::min(maxp, g.n[a]) + te - 2) / te + 1;
    for (int b = 0; b < 3; ++b) {
      if (b == a) continue;
      const long long span = (long long)std::ceil((te - 1) * g.h[a] / g.h[b] - 1e-9) + 2 + slack;
      m *= std::min<long long>((span + te - 2) / te + 1, (g.n[b] + te - 1) / te);
    }
    most = std::max(most, m);
  }
  return most;
}

// Lists of at least this many events go by tile: its calls, the binning and
// the clearing and adding of the tiles cost 60 to 80 us whatever the list.  The
// per-event kernel takes 1.2 to 3.4 us per 1000 events with TOF and 2.4 to 10
// without, by grid, so it spends that on 2e4 to 6e4 events with TOF and 6e3
// to 3e4 without.  33000 events, per event / by tile: 128x128x1 with TOF 81 /
// 72, without 103 / 68; 64x64x16 of a small scanner 52 / 70 (the worst grid
// measured), 99 / 70; 200x200x96 124 / 95, 287 / 118.
constexpr long long kMinListEvents = 1 << 15;
// Tiles of an image: the histogram of a binning workgroup, 4 bytes per tile,
// is in LDS.
constexpr int kMaxListTiles = 36 << 10;
// Bytes of the segment numbers of a batch; longer lists go in batches.
constexpr long long kListSegBytes = 1LL << 30;

// Events of a binning workgroup: enough workgroups to fill the chip, few
// enough that their histograms (cleared, added and kept per workgroup) stay a
// small part.
static int bin_chunk(long long batch) {
  return (int)std::min<long long>(4096, ((batch + 1023) / 1024 + kBinBlock - 1) / kBinBlock * kBinBlock);
}

namespace {
// The temporaries of a batch, with a table of ntab intervals.
struct BackArrays {
  SegRay *rays;
  uint2 *item;
  unsigned *seg, *tot, *off, *nitems, *base;
  float *val;
  float4 *tab = nullptr;
  lmh::Slab slab;
  BackArrays(long long batch, long long pe, int ntiles, int ntab) {
    const int chunk = bin_chunk(batch);
    slab.add(&rays, batch);
    slab.add(&item, batch * pe / kItemMin + ntiles);
    slab.add(&seg, batch * pe);
    slab.add(&val, batch);
    slab.add(&tot, ntiles);
    slab.add(&off, ntiles + 1);
    slab.add(&nitems, 2);
    slab.add(&base, (batch + chunk - 1) / chunk * ntiles);
    if (ntab) slab.add(&tab, ntab);
  }
  BackArrays(const BackArrays &) = delete;  // the slab holds the addresses of the others
  BackArrays &operator=(const BackArrays &) = delete;
};

// A list's way by tile; batch 0: per event.
struct BackShape {
  TileGeom tg;
  int maxp;
  long long pe, batch;
  TofTab tt{};
  int ntab;
  BackShape(const GeomDev &g, long long n)
      : tg(tile_geom(g.n, kTL)), maxp(lmh::max_planes(g, W_BIN)), ntab(tof_table_size(g, tt)) {
    pe = segs_per_event(g, maxp, kTL, 1);  // the batch's list is allocated by it
    batch = std::min(std::min(n, 1LL << 30), kListSegBytes / (4 * pe));
    // very unequal voxel sides: too many tiles per event to plan for
    if (batch < kMinListEvents || tg.ntiles > kMaxListTiles || !segs_supported(g)) batch = 0;
  }
  size_t bytes(long long events) const { return BackArrays(events, pe, tg.ntiles, ntab).slab.bytes(); }
};
}  // namespace

size_t back_tiles_min_bytes(const GeomDev &g, long long n) {
  const BackShape s(g, n);
  return s.batch ? s.bytes(kMinListEvents) : 0;
}

int launch_back_tiles(const GeomDev &g, const float *v, const int16_t *ev, const int4 *rec, long long n, float *img,
                      size_t room, hipStream_t st, bool &queued) {
  queued = false;
  const BackShape shape(g, n);
  long long batch = shape.batch;
  if (room != SIZE_MAX && batch) {
    while (batch > kMinListEvents && shape.bytes(batch) > room)
      batch = std::max(kMinListEvents, batch - batch / 16);
    if (shape.bytes(batch) > room) batch = 0;
  }
  if (!batch) return LM_OK;
  {  // equal batches
    const long long count = (n + batch - 1) / batch;
    batch = (n + count - 1) / count;
  }
  const TileGeom tg = shape.tg;
  const int maxp = shape.maxp, chunk = bin_chunk(batch);
  BackArrays a(batch, shape.pe, tg.ntiles, shape.ntab);
  void *tmp = nullptr;
  {
    const hipError_t e = a.slab.alloc(st, &tmp);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      return LM_OK;  // the per-event path needs no temporaries
    }
    LM_TRY_HIP(e);
  }
  const int rc = shape.ntab ? fill_tof_table(g, shape.tt, a.tab, st) : LM_OK;
  const size_t lds = (size_t)tg.ntiles * sizeof(unsigned), tlds = shape.ntab * sizeof(float4);
  hipError_t e = hipSuccess;
  for (long long o = 0; rc == LM_OK && e == hipSuccess && o < n; o += batch) {
    const int m = (int)std::min(batch, n - o);
    const unsigned nb = (unsigned)((m + chunk - 1) / chunk);
    const int16_t *evo = ev ? ev + 5 * o : nullptr;
    const int4 *reco = ev ? nullptr : rec + o;
    hipLaunchKernelGGL(k_zero_u32, dim3(std::min(64, (tg.ntiles + 255) / 256)), dim3(256), 0, st, a.tot,
                       (long long)tg.ntiles);
    hipLaunchKernelGGL(k_list_count, dim3(nb), dim3(kBinBlock), lds, st, g, tg, maxp, evo, reco, v + o, m, chunk,
                       a.rays, a.val, a.tot, a.base, img);
    hipLaunchKernelGGL(k_list_items, dim3(1), dim3(1024), 0, st, a.tot, tg.ntiles, a.off, a.item, a.nitems);
    hipLaunchKernelGGL(k_list_place, dim3(nb), dim3(kBinBlock), lds, st, g, tg, a.rays, m, chunk, a.off, a.base,
                       a.seg);
#define LM_LB(TM_)                                                                                                \
  hipLaunchKernelGGL((k_list_back<TM_>), dim3(kBackGrid), dim3(kBackBlock), tlds, st, g, tg, a.off, a.item,       \
                     a.nitems, a.seg, a.rays, a.val, shape.tt, a.tab, img)
    if (!g.tof_on) LM_LB(kTofNone);
    else if (a.tab) LM_LB(kTofTable);
    else LM_LB(kTofErfc);
#undef LM_LB
    e = hipGetLastError();
  }
  (void)hipFreeAsync(tmp, st);  // a release error has no caller to go to
  if (rc != LM_OK) return rc;
  LM_TRY_HIP(e);
  queued = true;
  return LM_OK;
}

}  // namespace lmk
