// The data update of LM-SPDHG (Algorithm 2, data-subset branch: forward
// projection, dual prox of Eq. proxD, back projection of the dual
// increments, z / zbar step) by image tile, for 3D plans.
//
// The per-event kernel (k_data_update) adds each event's back projection
// into dz with FP32 atomics.  On gfx950 those atomics are executed beyond
// the L2 at about 2e10 requests/s, one request per 64-byte sector that the
// lanes of an instruction share: ~47 requests per event, most of a data
// update's time.  Here the subsets are fixed when the plan is created, so
// the back projection of every subset is binned once by 8x8x8-voxel tile
// (2x2x2 bricks): per tile, the numbers of the subset's events that reach
// it.  An update then runs in two kernels:
//
//   phase 1, per event (8 lanes per event, as the forward projector):
//     q = (P x)_e + s_e, the dual prox, c = 1 - y updated; it leaves the
//     event's ray (32 bytes) and its back projected value cf = L dy / mu;
//   phase 2, one workgroup per tile: the tile's events are accumulated in
//     LDS (lm_segs.hpp: 8 segments at a time in a wavefront, a lane per
//     sample, native double additions), and the tile's voxels, loaded at
//     the start, take the z / zbar step and the fused primal step of the
//     next update.  No global atomics, and dz never goes to memory.
//
// A subset of 44.6e3 events on 200x200x96 has 0.62e6 segments.  Phase 1
// used to write each segment's 8 sample values (a 64-byte record) for phase
// 2 to read: 40 MB written and read back per update, and the loop over an
// event's segments was more than half of phase 1's instructions.  Computing
// the samples again in phase 2 costs it some 40 instructions per 8 segments.
//
// The per-sample arithmetic (coordinates, bilinear weights, TOF weights) is
// that of the forward projection, so P^T is the transpose of P up to the
// order of the additions.  Tiles are launched hottest first (most segments
// over all subsets), so the long ones do not trail at the end of a launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "lm_device.hpp"
#include "lm_host.hpp"
#include "lm_tiles.hpp"

using namespace lmk;

namespace {

constexpr int kTE = 8;                 // tile edge, voxels
constexpr int kLanes1 = 8;             // lanes per event in phase 1
constexpr int kBlock1 = 256;
// The tile path runs when the largest subset has at least this many events
// per tile: a workgroup's fixed cost (clearing its accumulators, the latency
// of its first segments and of its voxels) must be shared by enough
// segments.
constexpr long long kMinEventsPerTile = 4;
constexpr int kBinBlock = 512;         // threads of the binning kernels
constexpr int kBinChunk = 4096;        // events of a binning workgroup
// Tiles that a binning workgroup counts: its histogram, 4 bytes per tile, is
// in LDS.  Images of more tiles are binned in ranges of tiles, by a workgroup
// each, which walk the same events: a plan of 400x400x128 (40000 tiles, two
// ranges) and 1.6e6 events in 8 subsets takes 7 ms to create and 214 us per
// data update, per event 3 ms and 410 us.
constexpr int kHistTiles = 36 << 10;

// Planes an event may visit: the segment lists' bound per event grows with
// them, to 1 KB on a grid of 200 planes without TOF, more than the per-event
// path's plan holds altogether.
constexpr int kMaxTilePlanes = 114;

// Images of fewer tiles run phase 2 with 512 threads per tile instead of 256,
// so that its workgroups fill the chip.
constexpr int kWideTiles = 4096;

// The events of binning workgroup (blockIdx.x, subset blockIdx.y): positions
// [a, b) of the stored list.
__device__ __forceinline__ void bin_range(const long long *sub, long long &a, long long &b) {
  a = sub[blockIdx.y] + (long long)blockIdx.x * kBinChunk;
  b = min(sub[blockIdx.y + 1], a + kBinChunk);
}

// The tiles of binning workgroup (blockIdx.z): t0 and the number of them.
__device__ __forceinline__ int tile_range(const TileGeom &tg, int &t0) {
  t0 = blockIdx.z * kHistTiles;
  return min(tg.ntiles - t0, kHistTiles);
}

// cnt[subset ntiles + tile] = the segments of the subset in the tile.  One
// LDS histogram per workgroup and one global atomic per workgroup and tile.
__global__ __launch_bounds__(kBinBlock) void k_tile_count(GeomDev g, TileGeom tg, int maxp,
                                                          const int4 *__restrict__ rec, const long long *sub,
                                                          unsigned *cnt) {
  extern __shared__ unsigned h[];
  long long a, b;
  bin_range(sub, a, b);
  if (a >= b) return;
  int t0;
  const int nt = tile_range(tg, t0);
  for (int t = threadIdx.x; t < nt; t += kBinBlock) h[t] = 0u;
  __syncthreads();
  for (long long e = a + threadIdx.x; e < b; e += kBinBlock) {
    const int4 rc = rec[e];
    const SegRay s = pack_seg_ray(setup_ray(g, rc.x, rc.y, rc.z, W_BIN, maxp));
    for_each_segment<kTE>(g, s, tg, [&](int t) {
      if ((unsigned)(t - t0) < (unsigned)nt) atomicAdd(&h[t - t0], 1u);
    });
  }
  __syncthreads();
  unsigned *c = cnt + (long long)blockIdx.y * tg.ntiles + t0;
  for (int t = threadIdx.x; t < nt; t += kBinBlock)
    if (h[t]) atomicAdd(c + t, h[t]);
}

// Lists the events of every (subset, tile), as positions relative to the
// subset's first event: seg[off[subset ntiles + tile] ..], each workgroup in
// a range of its own (reserved with one atomic on fill; the order inside a
// tile is not fixed).  The two passes over the events set their rays up
// twice: cheaper than keeping 32 bytes per event for it.
__global__ __launch_bounds__(kBinBlock) void k_tile_place(GeomDev g, TileGeom tg, int maxp,
                                                          const int4 *__restrict__ rec, const long long *sub,
                                                          const long long *__restrict__ off, unsigned *fill,
                                                          unsigned *__restrict__ seg) {
  extern __shared__ unsigned h[];
  long long a, b;
  bin_range(sub, a, b);
  if (a >= b) return;
  int t0;
  const int nt = tile_range(tg, t0);
  for (int t = threadIdx.x; t < nt; t += kBinBlock) h[t] = 0u;
  __syncthreads();
  const long long first = off[(long long)blockIdx.y * tg.ntiles], s0 = sub[blockIdx.y];
  unsigned *sg = seg + first;  // a subset's segments: below 2^32
  for (int pass = 0; pass < 2; ++pass) {
    for (long long e = a + threadIdx.x; e < b; e += kBinBlock) {
      const int4 rc = rec[e];
      const SegRay s = pack_seg_ray(setup_ray(g, rc.x, rc.y, rc.z, W_BIN, maxp));
      for_each_segment<kTE>(g, s, tg, [&](int t) {
        if ((unsigned)(t - t0) >= (unsigned)nt) return;
        const unsigned at = atomicAdd(&h[t - t0], 1u);
        if (pass == 1) sg[at] = (unsigned)(e - s0);
      });
    }
    __syncthreads();
    if (pass == 0) {
      const long long *o = off + (long long)blockIdx.y * tg.ntiles + t0;
      unsigned *f = fill + (long long)blockIdx.y * tg.ntiles + t0;
      for (int t = threadIdx.x; t < nt; t += kBinBlock)
        if (h[t]) h[t] = (unsigned)(o[t] - first) + atomicAdd(f + t, h[t]);
      __syncthreads();
    }
  }
}

// first[i] = the first segment of subset i (i = 0 .. nsub; the last one is
// the number of segments).
__global__ __launch_bounds__(256) void k_subset_first(const long long *__restrict__ off, int ntiles, int nsub,
                                                      long long *first) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i <= nsub) first[i] = off[(long long)i * ntiles];
}

// load[t] = segments of tile t over all subsets.
__global__ __launch_bounds__(256) void k_tile_load(const unsigned *__restrict__ cnt, int ntiles, int nsub,
                                                   unsigned long long *load) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= ntiles) return;
  unsigned long long s = 0;
  for (int i = 0; i < nsub; ++i) s += cnt[(long long)i * ntiles + t];
  load[t] = s;
}

// Exclusive prefix sum of cnt[0 .. n) into off[0 .. n] (64-bit); one block
// of 1024 threads, each summing a contiguous segment.
__global__ __launch_bounds__(1024) void k_scan64(const unsigned long long *cnt, long long n, long long *off) {
  __shared__ long long part[1024];
  const int t = threadIdx.x;
  const long long seg = (n + 1023) / 1024;
  const long long a = min(n, t * seg), b = min(n, a + seg);
  long long sum = 0;
  for (long long i = a; i < b; ++i) sum += cnt[i];
  part[t] = sum;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const long long add = t >= o ? part[t - o] : 0;
    __syncthreads();
    part[t] += add;
    __syncthreads();
  }
  long long run = part[t] - sum;
  for (long long i = a; i < b; ++i) {
    off[i] = run;
    run += cnt[i];
  }
  if (t == 1023) off[n] = part[1023];
}

// Exclusive prefix sum of a long list in three launches: sums of blocks of
// kScanB entries, their prefix (k_scan64), then the prefix inside each block.
constexpr int kScanB = 1024;

__global__ __launch_bounds__(kScanB) void k_block_sums(const unsigned *in, long long n,
                                                      unsigned long long *bsum) {
  __shared__ unsigned long long red[kScanB];
  const long long i = (long long)blockIdx.x * kScanB + threadIdx.x;
  red[threadIdx.x] = i < n ? in[i] : 0ull;
  __syncthreads();
  for (int o = kScanB / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(kScanB) void k_block_scan(const unsigned *in, long long n, const long long *boff,
                                                       unsigned long long *out) {
  __shared__ unsigned long long s[kScanB];
  const int t = threadIdx.x;
  const long long i = (long long)blockIdx.x * kScanB + t;
  const unsigned v = i < n ? in[i] : 0u;
  s[t] = v;
  __syncthreads();
  for (int o = 1; o < kScanB; o <<= 1) {  // inclusive scan
    const unsigned long long add = t >= o ? s[t - o] : 0ull;
    __syncthreads();
    s[t] += add;
    __syncthreads();
  }
  if (i < n) out[i] = (unsigned long long)boff[blockIdx.x] + s[t] - v;
  if (i == n - 1) out[n] = (unsigned long long)boff[blockIdx.x] + s[t];
}

// Phase 1: per event (8 lanes), the forward projection and the dual prox
// (the cancellation-free form of k_data_update); leaves the event's ray and
// cf = L dy / mu (0 where nothing is back projected) for phase 2.  The
// double-precision set-up of a wavefront's 8 rays runs in its lanes 0 .. 7
// and reaches the others through LDS.
//
// Bound by the L1's look-ups, about 1.4 lanes per clock and CU when the four
// corners of a sample lie on lines of their own (12 us of the 21 us that a
// subset of 44.6e3 events takes on 200x200x96; keeping the rays, without the
// set-up here, took 20.4 us).
template <int TM>
__global__ __launch_bounds__(kBlock1) void k_tile_fwd(GeomDev g, int maxp, const float *__restrict__ x,
                                                      const int4 *__restrict__ rec, const float *__restrict__ S,
                                                      const float *__restrict__ mu, float *__restrict__ cdual,
                                                      long long n, SegRay *__restrict__ rays, float *__restrict__ cf,
                                                      TofTab tt, const float4 *__restrict__ tab) {
  constexpr int kEv = kBlock1 / kLanes1;  // events per block
  __shared__ SegRay lray[kEv];
  __shared__ float2 lls[kEv];  // {L, s}
  extern __shared__ float4 stab[];
  const long long e_first = (long long)blockIdx.x * kEv;
  const int lane = threadIdx.x % kLanes1;
  const long long e = e_first + threadIdx.x / kLanes1;
  const float Se = e < n ? S[e] : 0.0f;  // loaded while the ray is set up
  const int wl = threadIdx.x & 63, we = (threadIdx.x >> 6) * 8;
  if (wl < 8 && e_first + we + wl < n) {
    const int4 rc = rec[e_first + we + wl];
    const Ray r = setup_ray(g, rc.x, rc.y, rc.z, W_BIN, maxp);
    const SegRay s = pack_seg_ray(r);
    rays[e_first + we + wl] = s;
    lray[we + wl] = s;
    lls[we + wl] = make_float2(r.L, __int_as_float(rc.w));
  }
  if constexpr (TM == kTofTable)
    for (int i = threadIdx.x; i < tof_tab_size(tt); i += kBlock1) stab[i] = tab[i];
  __syncthreads();
  if (e >= n) return;
  const SegRay r = lray[threadIdx.x / kLanes1];
  const float2 ls = lls[threadIdx.x / kLanes1];
  float acc = 0.0f;
  const int np = Se != 0.0f ? seg_np(r) : 0;  // step 0: the LOR misses the image, the prox leaves y unchanged
  if (np > 0) {
    const int a = seg_axis(r), m0 = seg_m0(r), i1 = seg_i1(r), i2 = seg_i2(r);
    const int b1 = (a == 0) ? 1 : 0, b2 = (a == 2) ? 1 : 2;
    const int n1 = sel3(b1, g.n[0], g.n[1], g.n[2]), n2 = sel3(b2, g.n[0], g.n[1], g.n[2]);
    const AxisTerm ta = axis_term(g.lay, a), t1 = axis_term(g.lay, b1), t2 = axis_term(g.lay, b2);
    const float F1 = __int_as_float(r.a.z), V1 = __int_as_float(r.a.w);
    const TofTab tu = tof_tab_uniform(tt);
    const float D = tof_bin_width(g);
    const ImageBuf img = image_buf(x, g.lay);
    // lanes from the brick boundary at or below the first plane; plane term
    // of the lane's plane, advanced by 8 planes (two bricks) per step
    int j = lane - (m0 & ta.mask & kMaxBrickOffset);
    int fa = axis_index(ta, m0 + j);
    const int fa_step = (kLanes1 >> ta.s) * ta.bs;
    for (; j < np; j += kLanes1, fa += fa_step) {
      const float fj = (float)j;
      const float u1 = fmaf(fj, V1, F1), u2 = fmaf(fj, r.b.y, r.b.x);
      const float fl1 = floorf(u1), fl2 = floorf(u2);
      // the loads first: the TOF weight's arithmetic runs while they are in
      // flight; corners outside the image read as zero
      const float v = gather_terms(img, t1, t2, n1, n2, fa, i1 + (int)fl1, i2 + (int)fl2, u1 - fl1, u2 - fl2);
      float w = 1.0f;
      if constexpr (TM != kTofNone) {
        const float tc = fmaf(-fj, r.b.w, r.b.z);
        if constexpr (TM == kTofTable) {
          w = tof_weight_tab(tu, stab, tc);
        } else {
          const float vh = fmaf(0.5f, D, tc);
          w = tof_weight(vh, vh - D, g.vclip, g.inv_norm);
        }
      }
      // the planes of the brick before the ray's first add nothing, whatever
      // value they hold
      acc = fmaf(w, j >= 0 ? v : 0.0f, acc);
    }
  }
  acc = group_sum<kLanes1>(acc);
  if (lane != 0) return;
  float back = 0.0f;
  if (Se != 0.0f) {
    const float c = cdual[e], me = mu[e];
    const float q = fmaf(ls.x, acc, ls.y);
    const float sq = Se * q;
    const float t = sq - c;
    const float rt = sqrtf(fmaf(t, t, 4.0f * Se * me));
    const float dy = 2.0f * Se * fmaf(q, c, -me) / (sq + c + rt);
    cdual[e] = c - dy;
    if (dy != 0.0f) back = ls.x * (dy / me);
  }
  cf[e] = back;
}

// V consecutive floats of an image, read or written as one access.
template <int V>
struct __align__(4 * V) Vox {
  float v[V];
};

// Phase 2: one workgroup of NT threads per tile; seg the numbers of the
// subset's events of every tile, off the subset's per-tile ranges of seg,
// rays and cf from phase 1.
template <int TM, int NT>
__global__ __launch_bounds__(NT) void k_tile_back(GeomDev g, TileGeom tg, const int *__restrict__ order,
                                                  const long long *__restrict__ off,
                                                  const unsigned *__restrict__ seg, const SegRay *__restrict__ rays,
                                                  const float *__restrict__ cf, TofTab tt,
                                                  const float4 *__restrict__ tab, float *__restrict__ z,
                                                  float *__restrict__ x, const float *__restrict__ T,
                                                  float *__restrict__ zbar, float *__restrict__ dz_out, float inv_p,
                                                  int fuse) {
  constexpr int V = kTE * kTE * kTE / NT;  // voxels of the tile per thread, a part of a brick's row along x
  static_assert(V * NT == kTE * kTE * kTE && V <= 4, "threads cover the tile");
  using A = AccShape<kTE>;
  __shared__ __align__(16) double acc[A::size];
  extern __shared__ float4 stab[];
  const int tile = order[blockIdx.x];
  const int tx = tile % tg.ntx, ty = (tile / tg.ntx) % tg.nty, tz = tile / (tg.ntx * tg.nty);
  const long long s0 = off[tile];
  const int cnt = (int)(off[tile + 1] - s0);
  // the thread's voxels (threads in the plan's brick order); their image
  // values are loaded now and used at the end
  const Layout &L = g.lay;
  const int v0 = V * threadIdx.x, b = v0 >> 6;
  const int bi = tx * 2 + (b & 1), bj = ty * 2 + ((b >> 1) & 1), bk = tz * 2 + (b >> 2);
  const bool mine_vox = bi < L.nbx && bj < L.nby && bk < L.nbz;
  const long long gi = ((((long long)bk * L.nby + bj) * L.nbx + bi) << 6) | (v0 & 63);
  Vox<V> xv{}, zv{}, Tv{};
  if (mine_vox && !dz_out) {
    zv = *(const Vox<V> *)(z + gi);
    if (fuse) {
      xv = *(const Vox<V> *)(x + gi);
      Tv = *(const Vox<V> *)(T + gi);
    }
  }
  static_assert(A::size % 2 == 0, "cleared two at a time");
  for (int i = threadIdx.x; i < A::size / 2; i += NT) ((double2 *)acc)[i] = make_double2(0.0, 0.0);
  if constexpr (TM == kTofTable)
    for (int i = threadIdx.x; i < tof_tab_size(tt); i += NT) stab[i] = tab[i];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  add_segments<TM, kTE>(g, tile_lane<kTE>(tx * kTE, ty * kTE, tz * kTE, lane % kTE), seg + s0, cnt, rays, cf,
                        tof_bin_width(g), tof_tab_uniform(tt), stab, acc, threadIdx.x >> 6, NT / 64, lane);
  __syncthreads();
  if (!mine_vox) return;
  const int i = (b & 1) * 4 + (v0 & 3), j = ((b >> 1) & 1) * 4 + ((v0 >> 2) & 3), k = (b >> 2) * 4 + ((v0 >> 4) & 3);
  const double *d0 = acc + (i + 1) + A::Y * (j + 1) + A::Z * (k + 1);
  // voxels of the row inside the image (padding voxels get nothing)
  const int row = (ty * kTE + j < g.n[1] && tz * kTE + k < g.n[2]) ? g.n[0] - (tx * kTE + i) : 0;
  Vox<V> d, zb;
#pragma unroll
  for (int q = 0; q < V; ++q) d.v[q] = q < row ? (float)d0[q] : 0.0f;
  if (dz_out) {
    *(Vox<V> *)(dz_out + gi) = d;
    return;
  }
#pragma unroll
  for (int q = 0; q < V; ++q) {
    zv.v[q] += d.v[q];
    zb.v[q] = fmaf(d.v[q], inv_p, zv.v[q]);
    xv.v[q] = fmaxf(0.0f, fmaf(-Tv.v[q], zb.v[q], xv.v[q]));
  }
  *(Vox<V> *)(z + gi) = zv;
  if (fuse)
    *(Vox<V> *)(x + gi) = xv;
  else
    *(Vox<V> *)(zbar + gi) = zb;
}

inline unsigned blocks(long long n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

namespace lmk {

// 3D plans (4x4x4 bricks) whose rays fit the record and the planned lists.
bool tiles_supported(const GeomDev &g) {
  if (g.n[2] < 2 || g.lay.sx != 2 || g.lay.sy != 2 || g.lay.sz != 2) return false;
  return segs_supported(g) && lmh::max_planes(g, W_BIN) <= kMaxTilePlanes;
}

size_t tile_bytes_bound(const GeomDev &g, long long n, int nsub) {
  if (!tiles_supported(g) || n <= 0) return 0;
  const TileGeom tg = tile_geom(g.n, kTE);
  const long long nmax = (n + nsub - 1) / nsub;
  if (nmax < kMinEventsPerTile * tg.ntiles) return 0;
  const long long per_event = segs_per_event(g, lmh::max_planes(g, W_BIN), kTE, 0);
  const long long nbin = (long long)nsub * tg.ntiles, nblk = (nbin + kScanB - 1) / kScanB;
  using lmh::Slab;
  const size_t kept = Slab::padded<unsigned>(n * per_event) + Slab::padded<long long>(nbin + 1) +
                      Slab::padded<int>(tg.ntiles) + Slab::padded<SegRay>(nmax) + Slab::padded<float>(nmax) +
                      Slab::padded<float4>(kTofTabMax);
  const size_t temporary = Slab::padded<unsigned>(nbin) + Slab::padded<unsigned long long>(tg.ntiles) +
                           Slab::padded<long long>(nblk) + Slab::padded<long long>(nblk + 1) +
                           2 * Slab::padded<long long>(nsub + 1);
  return kept + temporary;
}

int build_tiles(const GeomDev &g, const int4 *rec, const std::vector<int> &off, TilePlan &tp,
                std::vector<void *> &owned, hipStream_t st) {
  tp = TilePlan{};
  if (!tiles_supported(g)) return LM_OK;
  const int nsub = (int)off.size() - 1;
  const long long N = off.back();
  if (N == 0) return LM_OK;
  const TileGeom tg = tile_geom(g.n, kTE);
  long long nlargest = 0;
  for (int i = 0; i < nsub; ++i) nlargest = std::max<long long>(nlargest, off[i + 1] - off[i]);
  if (nlargest < kMinEventsPerTile * tg.ntiles) return LM_OK;
  const int maxp = lmh::max_planes(g, W_BIN);
  const long long nbin = (long long)nsub * tg.ntiles;
  const long long nblk = (nbin + kScanB - 1) / kScanB;
  // temporaries: counts per (subset, tile), their block sums, tile loads, the
  // subsets' first positions and segments
  unsigned *cnt = nullptr;
  unsigned long long *bsum = nullptr;
  long long *boff = nullptr, *sub = nullptr, *first = nullptr;
  unsigned long long *load = nullptr;
  // kept by the plan
  long long *soff = nullptr;
  unsigned *seg = nullptr;
  int *ord = nullptr;
  SegRay *rays = nullptr;
  float *cf = nullptr;
  void *tmp = nullptr, *kept = nullptr;  // allocations of the temporaries and of what is kept beside soff
  auto drop = [&](bool keep_error) {
    for (void *q : {tmp, (void *)soff, kept})
      if (q) (void)hipFreeAsync(q, st);
    if (!keep_error) (void)hipGetLastError();
  };
  lmh::Slab temporaries;
  temporaries.add(&cnt, nbin);
  temporaries.add(&bsum, nblk);
  temporaries.add(&boff, nblk + 1);
  temporaries.add(&load, tg.ntiles);
  temporaries.add(&sub, nsub + 1);
  temporaries.add(&first, nsub + 1);
  hipError_t e = temporaries.alloc(st, &tmp);
  if (e == hipSuccess && (e = hipMallocAsync((void **)&soff, (nbin + 1) * sizeof(long long), st)) != hipSuccess)
    soff = nullptr;
  if (e != hipSuccess) {
    drop(false);
    return LM_OK;  // no room: the per-event path
  }
  auto fail = [&](hipError_t he) {
    drop(true);
    lmh::set_error("tile binning: %s", hipGetErrorString(he));
    return LM_EHIP;
  };
  // the host copy stays alive until the synchronisation below
  const std::vector<long long> hsub(off.begin(), off.end());
  if ((e = hipMemcpyAsync(sub, hsub.data(), (nsub + 1) * sizeof(long long), hipMemcpyHostToDevice, st)) !=
          hipSuccess ||
      (e = hipMemsetAsync(cnt, 0, nbin * sizeof(unsigned), st)) != hipSuccess)
    return fail(e);
  const size_t lds = (size_t)std::min(tg.ntiles, kHistTiles) * sizeof(unsigned);
  const unsigned ranges = blocks(tg.ntiles, kHistTiles);
  // subsets in groups of at most 2^15 (the grid's y extent)
  constexpr int kGroup = 1 << 15;
  const unsigned bx = blocks(nlargest, kBinChunk);
  for (int i = 0; i < nsub; i += kGroup)
    hipLaunchKernelGGL(k_tile_count, dim3(bx, std::min(kGroup, nsub - i), ranges), dim3(kBinBlock), lds, st, g, tg, maxp, rec,
                       sub + i, cnt + (long long)i * tg.ntiles);
  hipLaunchKernelGGL(k_tile_load, dim3(blocks(tg.ntiles, 256)), dim3(256), 0, st, cnt, tg.ntiles, nsub, load);
  hipLaunchKernelGGL(k_block_sums, dim3((unsigned)nblk), dim3(kScanB), 0, st, cnt, nbin, bsum);
  hipLaunchKernelGGL(k_scan64, dim3(1), dim3(1024), 0, st, bsum, nblk, boff);
  hipLaunchKernelGGL(k_block_scan, dim3((unsigned)nblk), dim3(kScanB), 0, st, cnt, nbin, boff,
                     (unsigned long long *)soff);
  hipLaunchKernelGGL(k_subset_first, dim3(blocks(nsub + 1, 256)), dim3(256), 0, st, soff, tg.ntiles, nsub, first);
  if ((e = hipGetLastError()) != hipSuccess) return fail(e);
  // the tiles' loads (launch order) and the subsets' first segments
  std::vector<unsigned long long> hload(tg.ntiles);
  std::vector<long long> hoff(nsub + 1);
  if ((e = hipMemcpyAsync(hload.data(), load, tg.ntiles * sizeof(unsigned long long), hipMemcpyDeviceToHost, st)) !=
          hipSuccess ||
      (e = hipMemcpyAsync(hoff.data(), first, (nsub + 1) * sizeof(long long), hipMemcpyDeviceToHost, st)) !=
          hipSuccess)
    return fail(e);
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return fail(e);
  const long long total = hoff[nsub];
  for (int i = 0; i < nsub; ++i)
    if (hoff[i + 1] - hoff[i] >= (1LL << 32)) {
      drop(false);
      return LM_OK;  // a subset's segments are numbered in 32 bits
    }
  std::vector<int> order(tg.ntiles);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return hload[a] > hload[b]; });
  if (hload[order[0]] > (unsigned long long)kMaxSegments) {
    drop(false);
    return LM_OK;  // so many events on an image of a few tiles
  }
  lmh::Slab lists;
  lists.add(&seg, total);
  lists.add(&ord, tg.ntiles);
  lists.add(&rays, nlargest);
  lists.add(&cf, nlargest);
  e = lists.alloc(st, &kept);
  if (e != hipSuccess) {
    drop(false);
    return LM_OK;  // no room for the segments: the per-event path
  }
  if ((e = hipMemcpyAsync(ord, order.data(), tg.ntiles * sizeof(int), hipMemcpyHostToDevice, st)) != hipSuccess ||
      (e = hipMemsetAsync(cnt, 0, nbin * sizeof(unsigned), st)) != hipSuccess)
    return fail(e);
  for (int i = 0; i < nsub; i += kGroup)
    hipLaunchKernelGGL(k_tile_place, dim3(bx, std::min(kGroup, nsub - i), ranges), dim3(kBinBlock), lds, st, g, tg, maxp, rec,
                       sub + i, soff + (long long)i * tg.ntiles, cnt + (long long)i * tg.ntiles, seg);
  if ((e = hipGetLastError()) != hipSuccess) return fail(e);
  // the host order vector dies with this call
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return fail(e);
  (void)hipFreeAsync(tmp, st);
  for (void *q : {(void *)soff, kept}) owned.push_back(q);
  // TOF weights from a table where the geometry has one
  TofTab tt{};
  float4 *tab = nullptr;
  if (int rc = build_tof_table(g, tt, &tab, st)) return rc;
  if (tab) owned.push_back(tab);
  tp.tt = tt;
  tp.tab = tab;
  tp.on = true;
  tp.tg = tg;
  tp.seg_off = soff;
  tp.seg = seg;
  tp.order = ord;
  tp.maxp = maxp;
  tp.rays = rays;
  tp.cf = cf;
  tp.bytes = (size_t)(nbin + 1) * sizeof(long long) + lists.bytes() + (tab ? tof_tab_size(tt) * sizeof(float4) : 0);
  return LM_OK;
}

// The TOF weights of a plan's kernels and the LDS of their table.
static TofMode tof_mode(const GeomDev &g, const TilePlan &tp) {
  return !g.tof_on ? kTofNone : (tp.tab ? kTofTable : kTofErfc);
}
static size_t tab_lds(const TilePlan &tp) { return tp.tab ? (size_t)tof_tab_size(tp.tt) * sizeof(float4) : 0; }

int launch_tile_fwd(const GeomDev &g, const TilePlan &tp, const float *x, const int4 *rec, const float *S,
                    const float *mu, float *cdual, long long o, long long n, hipStream_t st) {
  if (n == 0) return LM_OK;
#define LM_TF(TM_)                                                                                                  \
  hipLaunchKernelGGL((k_tile_fwd<TM_>), dim3(blocks(n, kBlock1 / kLanes1)), dim3(kBlock1), tab_lds(tp), st, g,      \
                     tp.maxp, x, rec + o, S + o, mu + o, cdual + o, n, tp.rays, tp.cf, tp.tt, tp.tab)
  switch (tof_mode(g, tp)) {
    case kTofNone: LM_TF(kTofNone); break;
    case kTofErfc: LM_TF(kTofErfc); break;
    case kTofTable: LM_TF(kTofTable); break;
  }
#undef LM_TF
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

int launch_tile_back(const GeomDev &g, const TilePlan &tp, int subset, float *z, float *x, const float *T,
                     float *zbar, float *dz_out, float inv_p, bool fuse, hipStream_t st) {
  const long long *off = tp.seg_off + (long long)subset * tp.tg.ntiles;
  const bool wide = tp.tg.ntiles < kWideTiles;
#define LM_TB(TM_, NT_)                                                                                             \
  hipLaunchKernelGGL((k_tile_back<TM_, NT_>), dim3(tp.tg.ntiles), dim3(NT_), tab_lds(tp), st, g, tp.tg, tp.order,   \
                     off, tp.seg, tp.rays, tp.cf, tp.tt, tp.tab, z, x, T, zbar, dz_out, inv_p, fuse ? 1 : 0)
#define LM_TBW(TM_)            \
  do {                         \
    if (wide) LM_TB(TM_, 512); \
    else LM_TB(TM_, 256);      \
  } while (0)
  switch (tof_mode(g, tp)) {
    case kTofNone: LM_TBW(kTofNone); break;
    case kTofErfc: LM_TBW(kTofErfc); break;
    case kTofTable: LM_TBW(kTofTable); break;
  }
#undef LM_TBW
#undef LM_TB
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

}  // namespace lmk
