// Listmode TOF Joseph projector kernels for gfx950 and their C ABI entry
// points: lm_fwd, lm_back, lm_sens, lm_validate_events, plus the fused
// subset update of LM-SPDHG used by the plan code.
//
// The forward operator is the paper's listmode operator (Eq. lmop): one
// row of the TOF system matrix per event.  The fused update evaluates, for
// every event of a subset, the forward value, the dual prox (Eq. proxD with
// d = mu_e) and back-projects the scaled dual increment (the data-subset
// branch of Algorithm 2) in a single pass, so the samples of the forward pass are reused
// from registers by the back projection.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "lm_device.hpp"
#include "lm_host.hpp"
#include "lm_image.hpp"
#include "lm_order.hpp"
#include "lm_segs.hpp"

using namespace lmk;

namespace {

constexpr int kBlock = 256;

// Event sources: the caller's int16[5] records, the plan's int4 records,
// or the caller's records in a given order (out[order[e]] for the e-th).
// kXcdOrder: the blocks of a launch take the list in eight contiguous
// parts, one per XCD (blocks are dealt to the XCDs round robin), so that
// the events of a part share that XCD's L2.
struct CallerEvents {
  static constexpr bool kXcdOrder = false;
  const int16_t *ev;
  CallerEvents offset(long long o) const { return CallerEvents{ev + 5 * o}; }
  __device__ __forceinline__ bool get(const GeomDev &g, long long e, int &id1, int &id2, int &k) const {
    return decode_event(g, ev + 5 * e, id1, id2, k);
  }
  __device__ __forceinline__ long long slot(long long e) const { return e; }
};
struct PlanEvents {
  static constexpr bool kXcdOrder = false;
  const int4 *rec;
  PlanEvents offset(long long o) const { return PlanEvents{rec + o}; }
  __device__ __forceinline__ bool get(const GeomDev &, long long e, int &id1, int &id2, int &k) const {
    const int4 r = rec[e];
    id1 = r.x;
    id2 = r.y;
    k = r.z;
    return true;
  }
  __device__ __forceinline__ long long slot(long long e) const { return e; }
};
// The caller's events in spatial order.
struct OrderedEvents {
  static constexpr bool kXcdOrder = false;
  const OrderedEvent *rec;
  OrderedEvents offset(long long o) const { return OrderedEvents{rec + o}; }
  __device__ __forceinline__ bool get(const GeomDev &g, long long e, int &id1, int &id2, int &k) const {
    const OrderedEvent o = rec[e];
    return decode_event(g, o.ev, id1, id2, k);
  }
  __device__ __forceinline__ long long slot(long long e) const { return e; }
};
struct SortedEvents {
  static constexpr bool kXcdOrder = true;
  const int16_t *ev;
  const unsigned *order;
  SortedEvents offset(long long o) const { return SortedEvents{ev, order + o}; }
  __device__ __forceinline__ bool get(const GeomDev &g, long long e, int &id1, int &id2, int &k) const {
    return decode_event(g, ev + 5 * (long long)order[e], id1, id2, k);
  }
  __device__ __forceinline__ long long slot(long long e) const { return order[e]; }
};

// Events per launch of the forward projector (2^19 blocks of 64 events per
// wavefront).
constexpr long long kFwdLaunch = 1LL << 27;

// Forward projection.  A wavefront takes EPW consecutive events of the
// source: lane e < EPW first sets up the ray of event e (the
// double-precision set-up runs once per event rather than once per lane of
// a group) and stores it in LDS; then, in rounds, each group of LPE lanes
// walks the planes of one event (lane l of the group from the brick boundary
// at or below the first plane, every LPE-th plane), and lane e of the
// wavefront collects event e's sum for one store per lane.
//
// Bound on long lists by the L1's look-ups: the corners of a wavefront's 64
// samples lie on lines of their own, which the L1 serves at 1.4 lanes per
// clock and CU, the rate this kernel reaches (2.7 ms for 1e7 events on
// 200x200x96).  Tabulated TOF weights, 40 of 130 instructions per sample
// fewer, took 3.0 ms.  PAIRS: x is a pair image, which halves the look-ups
// of rays along x or y, but not the lines that it misses in the L2: 3.2 ms
// in list order, 1.75 in spatial order (2.0 with the ordering), bound by
// instruction issue.
template <class Src, bool TOF, int LPE, int EPW, bool PAIRS>
__global__ __launch_bounds__(kBlock) void k_fwd(GeomDev g, const int *skip, const float *__restrict__ x, Src src,
                                                long long n, float *__restrict__ out) {
  constexpr int kGroups = 64 / LPE, kRounds = EPW / kGroups, kPerBlock = EPW * (kBlock / 64);
  static_assert(kRounds * kGroups == EPW && EPW <= 64, "whole rounds");
  __shared__ RayPack rays[kPerBlock];
  if (skip && *skip) return;  // the list went to the path by line
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  long long blk = blockIdx.x;
  if constexpr (Src::kXcdOrder) {  // gridDim.x is a multiple of 8
    const long long per = gridDim.x / 8;
    blk = (blk % 8) * per + blk / 8;
  }
  const long long e0 = blk * kPerBlock + wv * EPW, e = e0 + lane;
  if (e0 >= n) return;  // the whole wavefront is past the end
  RayPack *wrays = rays + wv * EPW;
  if (lane < EPW) {
    // every field defined on every path: lanes past the end and invalid
    // events store an empty ray, and only valid events reach the set-up
    // (which reads the crystal table at the decoded ids)
    RayPack pk = empty_ray();
    int id1 = 0, id2 = 0, k = 0;
    if (e < n && src.get(g, e, id1, id2, k)) pk = pack_ray(setup_ray(g, id1, id2, k, W_BIN, 1 << 20));
    wrays[lane] = pk;
  }
  // LDS operations of one wavefront complete in order; the fences keep the
  // compiler from moving the reads above the writes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const float D = tof_bin_width(g);
  const int gl = lane % LPE, grp = lane / LPE;
  float mine = 0.0f;
  for (int round = 0; round < kRounds; ++round) {
    const RayPack pk = wrays[kGroups * round + grp];
    float acc = 0.0f;
    if constexpr (PAIRS) {
      const bool along_z = __any(pk.p.y > 0 && pk.p.z == 2);
      if (pk.p.y > 0) {
        if (!along_z) acc = fwd_walk<TOF, LPE, kPairs>(g, x, pk, D, gl);
        else acc = fwd_walk<TOF, LPE, kPairsAnyAxis>(g, x, pk, D, gl);
      }
    } else {
      if (pk.p.y > 0) acc = fwd_walk<TOF, LPE>(g, x, pk, D, gl);
    }
    acc = group_sum<LPE>(acc);
    // lanes kGroups round .. take the sums of the groups
    const float got = __shfl(acc, LPE * (lane % kGroups));
    if (lane / kGroups == round) mine = got;
  }
  if (lane < EPW && e < n) out[src.slot(e)] = __int_as_float(wrays[lane].q.w) * mine;
}

// Per-wavefront LDS staging of the interleaved scatter (4 wavefronts per
// block, 4 corners x 64 lanes each).
struct Stage {
  int idx[kBlock / 64][256];
  float val[kBlock / 64][256];
};

// Back projection of a short list: one event per wavefront, the scatter of
// every 64 planes interleaved over corners; the grid strides over the list.
template <class Src>
__global__ __launch_bounds__(kBlock) void k_back(GeomDev g, const float *__restrict__ v, Src src, long long n,
                                                 float *img) {
  __shared__ Stage st;
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  const long long stride = (long long)gridDim.x * (kBlock / 64);
  for (long long e = (long long)blockIdx.x * (kBlock / 64) + wv; e < n; e += stride) {
    const float ve = v[e];
    if (ve == 0.0f) continue;
    int id1, id2, k;
    if (!src.get(g, e, id1, id2, k)) continue;
    const Ray r = setup_ray(g, id1, id2, k, W_BIN, 1 << 20);
    const float c = r.L * ve;
    const int off = brick_offset(g.lay, r);
    for (int j0 = -off; j0 < r.nplanes; j0 += 64) {
      const int j = j0 + lane;
      Sample s = sample_at(g, r, j, g.tof_on);
      const float cs = (j >= 0 && j < r.nplanes) ? c * s.w : 0.0f;
      scatter_interleaved(g, img, r, s, cs, lane, st.idx[wv], st.val[wv]);
    }
  }
}

// Sensitivity: every unordered pair (id1 < id2) of crystals, weight summed
// over all TOF bins, one pair per wavefront, the grid striding over the
// pairs; nothing when *skip is non-zero (the pairs went to the line path).
__global__ __launch_bounds__(kBlock) void k_sens(GeomDev g, const int *skip, long long npairs, float *img) {
  __shared__ Stage st;
  if (skip && *skip) return;
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  const long long nd = g.n_det;
  const long long stride = (long long)gridDim.x * (kBlock / 64);
  for (long long p = (long long)blockIdx.x * (kBlock / 64) + wv; p < npairs; p += stride) {
    // row i holds pairs (i, i+1..nd-1); first index of row i is i*nd - i(i+1)/2
    const double b = 2.0 * nd - 1.0;
    long long i = (long long)floor((b - sqrt(b * b - 8.0 * (double)p)) * 0.5);
    auto first = [&](long long r) { return r * nd - r * (r + 1) / 2; };
    if (i < 0) i = 0;
    while (i > 0 && first(i) > p) --i;
    while (i + 1 < nd && first(i + 1) <= p) ++i;
    const long long jdx = i + 1 + (p - first(i));
    const Ray r = setup_ray(g, (int)i, (int)jdx, 0, W_SUM, 1 << 20);
    const int off = brick_offset(g.lay, r);
    for (int j0 = -off; j0 < r.nplanes; j0 += 64) {
      const int j = j0 + lane;
      Sample s = sample_at(g, r, j, g.tof_on);
      const float cs = (j >= 0 && j < r.nplanes) ? r.L * s.w : 0.0f;
      scatter_interleaved(g, img, r, s, cs, lane, st.idx[wv], st.val[wv]);
    }
  }
}

// Fused subset update (the data-subset branch of Algorithm 2) for the events
// of one subset, stored contiguously in the plan's order, one event per
// wavefront:
//   q = (P x)_e + s_e;  y+ = prox(y_e + S_e q) with d = mu_e;
//   dz += P^T((y+ - y_e)/mu_e);  y_e = y+.
// The dual is kept as its complement c = 1 - y (y tends to 1 on LORs with
// large expected counts, where 1 - y would cancel), and the increment is
// evaluated in the cancellation-free form
//   y+ - y = 2 S (q c - mu) / (S q + c + sqrt((S q - c)^2 + 4 S mu)),
// algebraically identical to Eq. proxD minus y; c+ = c - (y+ - y).  The
// samples of the forward pass stay in registers for the back projection.
template <int JMAX>
__global__ __launch_bounds__(kBlock) void k_data_update(GeomDev g, const float *__restrict__ x,
                                                        const int4 *__restrict__ rec,
                                                        const float *__restrict__ S,
                                                        const float *__restrict__ mu,
                                                        float *__restrict__ cdual, float *dz, long long n) {
  __shared__ Stage st;
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  const long long e = (long long)blockIdx.x * (kBlock / 64) + wv;
  if (e >= n) return;
  const int4 rc = rec[e];
  const float Se = S[e];
  if (Se == 0.0f) return;  // LOR misses the image: the prox leaves y unchanged
  const Ray r = setup_ray(g, rc.x, rc.y, rc.z, W_BIN, JMAX * 64 - kMaxBrickOffset);
  const int off = brick_offset(g.lay, r);
  Sample cache[JMAX];
  float acc = 0.0f;
#pragma unroll
  for (int jj = 0; jj < JMAX; ++jj) {
    const int j = lane + jj * 64 - off;
    cache[jj] = sample_at(g, r, j, g.tof_on);
    if (j >= 0 && j < r.nplanes) {
      acc = fmaf(cache[jj].w, gather(g, x, r, cache[jj]), acc);
    } else {
      cache[jj].w = 0.0f;
    }
  }
  acc = group_sum<64>(acc);
  const float q = fmaf(r.L, acc, __int_as_float(rc.w));
  const float c = cdual[e], me = mu[e];
  const float sq = Se * q;
  const float t = sq - c;
  const float rt = sqrtf(fmaf(t, t, 4.0f * Se * me));
  const float dy = 2.0f * Se * fmaf(q, c, -me) / (sq + c + rt);
  if (lane == 0) cdual[e] = c - dy;
  if (dy == 0.0f) return;
  const float cf = r.L * (dy / me);
#pragma unroll
  for (int jj = 0; jj < JMAX; ++jj) {
    if (jj * 64 - off < r.nplanes) {
      const float cs = (cache[jj].w != 0.0f) ? cf * cache[jj].w : 0.0f;
      scatter_interleaved(g, dz, r, cache[jj], cs, lane, st.idx[wv], st.val[wv]);
    }
  }
}

// Counts events with an out-of-range crystal, ring or TOF index.
__global__ void k_validate(GeomDev g, const int16_t *ev, long long n, unsigned long long *bad) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  int id1, id2, k;
  const bool ok = (e >= n) || decode_event(g, ev + 5 * e, id1, id2, k);
  const unsigned long long m = __ballot(!ok);
  if ((threadIdx.x % 64) == 0 && m) atomicAdd(bad, (unsigned long long)__popcll(m));
}


inline unsigned blocks_for(long long n, int lpe) {
  const long long per = kBlock / lpe;
  return (unsigned)((n + per - 1) / per);
}

// A launch covers at most 2^22 blocks (2^30 work-items): the total number
// of work-items of one dispatch must stay below 2^32.  Larger inputs are
// processed in consecutive launches on the same stream.
constexpr long long kMaxBlocks = 1LL << 22;
inline long long chunk_items(int lpe) { return kMaxBlocks * (kBlock / lpe); }

}  // namespace

// --------------------------------------------------------------------------
// geometry and launch policy

namespace lmh {

int make_geom(const lm_geom *G, lmk::GeomDev *o) {
  LM_REQUIRE(G != nullptr, LM_EINVAL, "lm_geom is NULL");
  LM_REQUIRE(G->det != nullptr, LM_EINVAL, "lm_geom.det is NULL");
  LM_REQUIRE(G->n_cry > 0 && G->n_ring > 0, LM_EINVAL, "n_cry and n_ring must be positive");
  LM_REQUIRE((long long)G->n_cry * G->n_ring < (1LL << 30), LM_EINVAL, "too many crystals");
  for (int a = 0; a < 3; ++a) {
    LM_REQUIRE(G->n[a] >= 1 && G->n[a] <= kMaxDim, LM_EINVAL, "image size n[%d]=%d outside 1..%d", a,
               G->n[a], kMaxDim);
    LM_REQUIRE(G->h[a] > 0.0 && std::isfinite(G->h[a]), LM_EINVAL, "voxel size h[%d] must be > 0", a);
  }
  LM_REQUIRE(G->n_tof >= 1 && (G->n_tof % 2) == 1 && G->n_tof < 32767, LM_EINVAL,
             "n_tof must be odd and positive");
  if (G->tof_on) {
    LM_REQUIRE(G->tof_bin > 0.0 && G->tof_fwhm > 0.0 && G->tof_nsigma > 0.0, LM_EINVAL,
               "TOF bin, FWHM and truncation must be positive");
  }
  o->det = G->det;
  o->n_cry = G->n_cry;
  o->n_ring = G->n_ring;
  o->n_det = G->n_cry * G->n_ring;
  for (int a = 0; a < 3; ++a) {
    o->n[a] = G->n[a];
    o->h[a] = G->h[a];
    o->c0[a] = -0.5 * (G->n[a] - 1) * G->h[a];
  }
  o->lay = lmh::row_major(G->n);
  o->n_tof = G->n_tof;
  o->kmax = (G->n_tof - 1) / 2;
  o->tof_on = G->tof_on ? 1 : 0;
  const double sigma = G->tof_fwhm / (2.0 * std::sqrt(2.0 * std::log(2.0)));
  o->tof_bin = G->tof_bin;
  o->inv_sr2 = G->tof_on ? 1.0 / (sigma * std::sqrt(2.0)) : 0.0;
  o->half_win = G->tof_on ? G->tof_nsigma * sigma + 0.5 * G->tof_bin : 0.0;
  o->vclip = (float)(G->tof_nsigma / std::sqrt(2.0));
  o->inv_norm = (float)(1.0 / (2.0 * std::erf(G->tof_nsigma / std::sqrt(2.0))));
  return LM_OK;
}

int max_planes(const lmk::GeomDev &g, int mode) {
  const int nmax = std::max(g.n[0], std::max(g.n[1], g.n[2]));
  if (!g.tof_on || mode == lmk::W_SUM) return nmax;
  const double hmin = std::min(g.h[0], std::min(g.h[1], g.h[2]));
  // the LOR advances at least h_a along t per plane; +3 covers the margins
  const long long b = (long long)std::ceil(2.0 * g.half_win / hmin) + 3;
  return (int)std::min<long long>(b, nmax);
}


}  // namespace lmh

// --------------------------------------------------------------------------
// launchers

namespace lmk {

template <class Src, int LPE, int EPW, bool PAIRS>
static int fwd_launch(const GeomDev &g, const float *x, Src src, long long n, float *out, hipStream_t st,
                      const int *skip) {
  constexpr int kPerBlock = EPW * (kBlock / 64);
  for (long long o = 0; o < n; o += kFwdLaunch) {
    const long long m = std::min(kFwdLaunch, n - o);
    unsigned nb = (unsigned)((m + kPerBlock - 1) / kPerBlock);
    if (Src::kXcdOrder) nb = (nb + 7) / 8 * 8;
    // sorted sources write out[order[e]]: out is the whole list's
    float *o_out = Src::kXcdOrder ? out : out + o;
    if (g.tof_on)
      hipLaunchKernelGGL((k_fwd<Src, true, LPE, EPW, PAIRS>), dim3(nb), dim3(kBlock), 0, st, g, skip, x, src.offset(o), m,
                         o_out);
    else
      hipLaunchKernelGGL((k_fwd<Src, false, LPE, EPW, PAIRS>), dim3(nb), dim3(kBlock), 0, st, g, skip, x, src.offset(o), m,
                         o_out);
    LM_TRY_HIP(hipGetLastError());
  }
  return LM_OK;
}

// The split of a list over wavefronts: 64 events per wavefront share the
// set-up's instructions best, but a shorter list leaves the chip idle (a
// wavefront then walks its events one after the other); below 2^14 events
// half a wavefront takes each event, which shortens the chain of its
// samples.  3571 events of the single-slice problem: 41 -> 6.4 us in the
// kernel.
template <class Src, bool PAIRS = false>
static int fwd_impl(const GeomDev &g, const float *x, Src src, long long n, float *out, hipStream_t st,
                    const int *skip = nullptr) {
  if (n == 0) return LM_OK;
  if (Src::kXcdOrder || n >= (1 << 19)) return fwd_launch<Src, 8, 64, PAIRS>(g, x, src, n, out, st, skip);
  if (n >= (1 << 16)) return fwd_launch<Src, 8, 16, PAIRS>(g, x, src, n, out, st, skip);
  if (n >= (1 << 14)) return fwd_launch<Src, 8, 8, PAIRS>(g, x, src, n, out, st, skip);
  return fwd_launch<Src, 32, 2, PAIRS>(g, x, src, n, out, st, skip);
}

// Grid of the grid-stride scattering kernels: enough wavefronts to fill the
// chip, few enough that a launch whose work went to another path costs next
// to nothing (65536 blocks that return at once took 15 us, 4096 take 2).
constexpr long long kStrideBlocks = 1LL << 12;

template <class Src>
static int back_impl(const GeomDev &g, const float *v, Src src, long long n, float *img, hipStream_t st) {
  const long long nb = std::min<long long>(kStrideBlocks, blocks_for(n, 64));
  hipLaunchKernelGGL((k_back<Src>), dim3((unsigned)nb), dim3(kBlock), 0, st, g, v, src, n, img);
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

// A device flag (one int), allocated and freed stream-ordered.
struct DevFlag {
  int *p = nullptr;
  hipStream_t st = nullptr;
  int alloc(hipStream_t s) {
    st = s;
    const hipError_t e = hipMallocAsync((void **)&p, sizeof(int), s);
    if (e != hipSuccess) {
      p = nullptr;
      lmh::set_error("flag temporary: %s", hipGetErrorString(e));
      return LM_ENOMEM;
    }
    return LM_OK;
  }
  ~DevFlag() {
    if (p) (void)hipFreeAsync(p, st);  // a release error has no caller to go to
  }
};

int launch_fwd(const GeomDev &g, const float *x, const int16_t *ev, long long n, float *out, hipStream_t st) {
  return fwd_impl(g, x, CallerEvents{ev}, n, out, st);
}
// By tile, or per event where the list is short or the tile path does not
// apply.
static int back_any(const GeomDev &g, const float *v, const int16_t *ev, const int4 *rec, long long n, float *img,
                    size_t room, hipStream_t st) {
  if (n == 0) return LM_OK;
  bool queued = false;
  if (int rc = launch_back_tiles(g, v, ev, rec, n, img, room, st, queued)) return rc;
  if (queued) return LM_OK;
  return ev ? back_impl(g, v, CallerEvents{ev}, n, img, st) : back_impl(g, v, PlanEvents{rec}, n, img, st);
}
int launch_back(const GeomDev &g, const float *v, const int16_t *ev, long long n, float *img, hipStream_t st) {
  return back_any(g, v, ev, nullptr, n, img, SIZE_MAX, st);
}
int launch_fwd_rec(const GeomDev &g, const float *x, const int4 *rec, long long n, float *out, hipStream_t st) {
  return fwd_impl(g, x, PlanEvents{rec}, n, out, st);
}
int launch_back_rec(const GeomDev &g, const float *v, const int4 *rec, long long n, float *img, size_t room,
                    hipStream_t st) {
  return back_any(g, v, nullptr, rec, n, img, room, st);
}

int launch_sens(const GeomDev &g, float *img, hipStream_t st) {
  const long long nd = g.n_det;
  const long long npairs = nd * (nd - 1) / 2;
  const long long nb = std::min<long long>(kStrideBlocks, blocks_for(npairs, 64));
  if (!lines_possible(g)) {
    hipLaunchKernelGGL(k_sens, dim3((unsigned)nb), dim3(kBlock), 0, st, g, nullptr, npairs, img);
    LM_TRY_HIP(hipGetLastError());
    return LM_OK;
  }
  DevFlag cyl;
  if (int rc = cyl.alloc(st)) return rc;
  if (int rc = launch_cylindrical(g, cyl.p, st)) return rc;
  if (int rc = launch_sens_lines(g, cyl.p, img, st)) return rc;
  hipLaunchKernelGGL(k_sens, dim3((unsigned)nb), dim3(kBlock), 0, st, g, cyl.p, npairs, img);
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

int launch_data_update(const GeomDev &g, const float *x, const int4 *rec, const float *S, const float *mu,
                       float *cdual, float *dz, long long n, hipStream_t st) {
  if (n == 0) return LM_OK;
  // the lanes of an event start up to kMaxBrickOffset planes before its
  // first plane
  const int planes = lmh::max_planes(g, W_BIN) + kMaxBrickOffset;
  const int jneed = (planes + 63) / 64;
#define LM_DU(J_)                                                                                       \
  if (jneed <= J_) {                                                                                    \
    for (long long o = 0; o < n; o += chunk_items(64)) {                                                \
      const long long m = std::min(chunk_items(64), n - o);                                             \
      hipLaunchKernelGGL((k_data_update<J_>), dim3(blocks_for(m, 64)), dim3(kBlock), 0, st, g, x, rec + o, \
                         S + o, mu + o, cdual + o, dz, m);                                              \
      LM_TRY_HIP(hipGetLastError());                                                                    \
    }                                                                                                   \
    return LM_OK;                                                                                       \
  }
  LM_DU(1) LM_DU(2) LM_DU(3) LM_DU(4) LM_DU(6) LM_DU(9)
#undef LM_DU
  lmh::set_error("no update kernel for %d planes per event", planes);
  return LM_EINVAL;
}

}  // namespace lmk

// --------------------------------------------------------------------------
// Scratch of lm_fwd_noalloc: the bricked copy of the caller's image lives in
// a file-scope device array (64 MiB on every device the library runs on,
// held until the process ends) instead of a stream-ordered allocation.  In
// host code `scratch` names a host-side stand-in, not device memory: kernels
// get the address that hipGetSymbolAddress returns for the device.

constexpr long long kNoAllocScratchFloats = 1LL << 24;
static __device__ __align__(256) float scratch[kNoAllocScratchFloats];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (which must be the
// device of `st`), looked up once per device with that device current.
int noalloc_scratch(hipStream_t st, float **out) {
  int dev = -1;
  LM_TRY_HIP(hipGetDevice(&dev));
  LM_REQUIRE(dev >= 0 && dev < kMaxDevices, LM_EINVAL, "device %d beyond the %d the library serves", dev,
             kMaxDevices);
  if (st != nullptr) {
    hipDevice_t sdev = -1;
    LM_TRY_HIP(hipStreamGetDevice(st, &sdev));
    LM_REQUIRE(sdev == dev, LM_EINVAL, "stream of device %d, but device %d is current", (int)sdev, dev);
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void *ptr = nullptr;
    LM_TRY_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = static_cast<float *>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return LM_OK;
}

}  // namespace

// Short lists work on the caller's row-major image: the bricked copy costs
// its allocation and release, two or three launches and a pass over the image
// each way, which a list earns back by its samples (events x planes).  Back
// projection earns it back sooner, as its atomics share fewer sectors of a
// row-major image, the later the larger the image, and later with TOF, where
// part of the planes counted have no weight.  Wall time per call (emissions of a
// phantom), row-major / bricked, in us:
//   forward, TOF: 32000 events 14 / 32 (128x128x48), 27 / 35 (200x200x96);
//     no TOF: 16000 events 17 / 34, 51 / 45; 32000 29 / 37, 72 / 57
//   back, TOF: 8000 events 26 / 38 (128x128x1), 29 / 32 (128x128x48), 43 / 61
//     (200x200x96); 12000 38 / 40, 42 / 38, 62 / 72; 20000 60 / 53, 67 / 57, 104 / 98
//     no TOF: 4000 events 24 / 38, 42 / 38, 64 / 72; 6000 36 / 38, 61 / 54, 99 / 95;
//     8000 46 / 38, 80 / 63, 123 / 104
static bool short_list(const GeomDev &g, long long n, long long samples) {
  return n < (1 << 15) && n * lmh::max_planes(g, W_BIN) <= samples;
}
constexpr long long kShortFwd = 1LL << 22;
static long long short_back(const GeomDev &g) {
  return g.tof_on ? 850000 + lmh::nvox_of(g.n) / 6 : 650000 + lmh::nvox_of(g.n) / 8;
}

// Lists projected from the pair image (twice the memory), and in spatial
// order (which costs some 60 us and 20 ns per event).  Without the order pairs
// pay while the L2 of an XCD holds a good part of them, beyond that only with
// it.  Wall time per call in us, bricks / pairs / pairs in order (672 crystals
// x 96 rings, emissions of a phantom; TOF: 90 planes per event):
//   128x128x48, TOF      1e5  53 / 51 / 106    1e6  231 / 190 / 242     8e6  1380 / 1086 / 1209
//   128x128x48, no TOF   1e5  85 / 62 / 112    1e6  536 / 337 / 335     8e6  3815 / 2375 / 1832
//   160x160x64, TOF      1e5  64 / 53 / 111    1e6  280 / 224 / 272     8e6  1724 / 1290 / 1466
//   200x200x96, TOF      3e5  135 / 126 / 172  1e6  331 / 351 / 316     8e6  2154 / 2571 / 1689
//   200x200x96, no TOF   3e5  359 / 370 / 411  1e6  1119 / 1174 / 1024  8e6  9002 / 9299 / 5615
//   300x300x96, TOF      3e5  234 / 287 / 234  1e6  653 / 680 / 578     8e6  4738 / 4420 / 2403
constexpr long long kPairsAlone = 16LL << 20;  // bytes
static long long pair_bytes(const GeomDev &g) { return 8LL * g.n[0] * g.n[1] * (g.n[2] + 1); }
static bool order_pays(const GeomDev &g, long long n) {
  return g.n[2] > 1 && order_possible(g) && n >= (1 << 19) && pair_bytes(g) > (g.tof_on ? kPairsAlone : 4LL << 20) &&
         n * lmh::max_planes(g, W_BIN) >= 16 * lmh::nvox_of(g.n);
}
static bool pairs_pay(const GeomDev &g, long long n) {
  return g.n[2] > 1 && pair_bytes(g) <= kPairsAlone && n * lmh::max_planes(g, W_BIN) >= 4 * lmh::nvox_of(g.n);
}

// Forward projection from a pair image in spatial order, in equal pieces of
// up to 2^26 events (equal, so that each is projected like a long list);
// queued is false, with nothing enqueued, without room for the order.
constexpr long long kOrderPiece = 1LL << 26;
static int fwd_ordered(const GeomDev &g, const float *pairs, const int16_t *ev, long long n, float *out,
                       hipStream_t st, bool &queued) {
  const long long pieces = (n + kOrderPiece - 1) / kOrderPiece, piece = (n + pieces - 1) / pieces;
  EventOrder o;
  lmh::Slab arrays;
  lmk::add_order(arrays, piece, o);
  void *tmp = nullptr;
  const hipError_t e = arrays.alloc(st, &tmp);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    return LM_OK;
  }
  LM_TRY_HIP(e);
  int rc = LM_OK;
  for (long long a = 0; rc == LM_OK && a < n; a += piece) {
    const long long m = std::min(piece, n - a);
    rc = lmk::launch_order(g, ev + 5 * a, m, o, st);
    if (rc == LM_OK) rc = fwd_impl<OrderedEvents, true>(g, pairs, OrderedEvents{o.rec}, m, o.val, st);
    if (rc == LM_OK) rc = lmk::launch_order_back(o, m, out + a, st);
  }
  (void)hipFreeAsync(tmp, st);  // a release error has no caller to go to
  queued = true;
  return rc;
}

// --------------------------------------------------------------------------
// C ABI

extern "C" {

int lm_fwd(const lm_geom *G, const float *x, const int16_t *ev, int64_t n, float *out, void *stream) {
  lmh::clear_error();
  GeomDev g;
  if (int rc = lmh::make_geom(G, &g)) return rc;
  LM_REQUIRE(n >= 0, LM_EINVAL, "negative event count");
  LM_REQUIRE(n == 0 || (x && ev && out), LM_EINVAL, "NULL array");
  if (n == 0) return LM_OK;
  hipStream_t st = lmh::as_stream(stream);
  if (short_list(g, n, kShortFwd)) return launch_fwd(g, x, ev, n, out, st);
  // a long list without TOF, or of a single slice, is sorted by transaxial
  // crystal pair and projected line by line on a cylindrical scanner, else
  // per event in the sorted order (so that the events of a line share cache
  // lines); with TOF the spatial order is faster at any length (128 crystals x
  // 16 rings on 200x200x96, 8e6 events: 2190 us by line, 1703 in order)
  unsigned *order = nullptr, *off = nullptr;
  if (!g.tof_on || g.n[2] == 1)
    if (int rc = lmk::sort_events_by_line(g, ev, n, &order, &off, st)) return rc;
  lmh::BrickImage b;
  const bool ordered = !order && order_pays(g, n);
  if (ordered || (!order && pairs_pay(g, n))) {
    if (int rc = b.alloc_pairs(g, st)) return rc;
    if (b.p) {
      if (int rc = lmk::launch_to_pairs(g.n, g.lay, x, b.p, st)) return rc;
      bool queued = false;
      if (ordered)
        if (int rc = fwd_ordered(g, b.p, ev, n, out, st, queued)) return rc;
      if (queued) return LM_OK;
      return fwd_impl<CallerEvents, true>(g, b.p, CallerEvents{ev}, n, out, st);
    }
  }
  int rc = b.alloc(g, st);
  if (rc == LM_OK) rc = lmk::launch_to_layout(g.n, g.lay, 1, x, b.p, st);
  if (!order) return rc ? rc : launch_fwd(g, b.p, ev, n, out, st);
  if (rc == LM_OK) {
    DevFlag cyl;
    bool queued = false;
    if (lines_possible(g)) {
      rc = cyl.alloc(st);
      if (rc == LM_OK) rc = launch_cylindrical(g, cyl.p, st);
      if (rc == LM_OK) rc = launch_fwd_lines(g, cyl.p, b.p, ev, order, off, n, out, st, queued);
    }
    if (rc == LM_OK) rc = fwd_impl(g, b.p, SortedEvents{ev, order}, n, out, st, queued ? cyl.p : nullptr);
  }
  (void)hipFreeAsync(order, st);  // release errors have no caller to go to
  (void)hipFreeAsync(off, st);
  return rc;
}

int lm_fwd_noalloc(const lm_geom *G, const float *x, const int16_t *ev, int64_t n, float *out, void *stream) {
  lmh::clear_error();
  GeomDev g;
  if (int rc = lmh::make_geom(G, &g)) return rc;
  LM_REQUIRE(n >= 0, LM_EINVAL, "negative event count");
  LM_REQUIRE(n == 0 || (x && ev && out), LM_EINVAL, "NULL array");
  g.lay = lmh::brick_layout(g.n);
  const long long need = layout_size(g.lay);
  LM_REQUIRE(need <= kNoAllocScratchFloats, LM_EINVAL,
             "the image takes %lld floats in brick layout, beyond the %lld of lm_fwd_noalloc's scratch", need,
             kNoAllocScratchFloats);
  if (n == 0) return LM_OK;
  hipStream_t st = lmh::as_stream(stream);
  float *scr = nullptr;
  if (int rc = noalloc_scratch(st, &scr)) return rc;
  if (int rc = lmk::launch_to_layout(g.n, g.lay, 1, x, scr, st)) return rc;
  return launch_fwd(g, scr, ev, n, out, st);
}

int lm_back(const lm_geom *G, const float *v, const int16_t *ev, int64_t n, float *img, void *stream) {
  lmh::clear_error();
  GeomDev g;
  if (int rc = lmh::make_geom(G, &g)) return rc;
  LM_REQUIRE(n >= 0, LM_EINVAL, "negative event count");
  LM_REQUIRE(n == 0 || (v && ev && img), LM_EINVAL, "NULL array");
  if (n == 0) return LM_OK;
  hipStream_t st = lmh::as_stream(stream);
  if (short_list(g, n, short_back(g))) return launch_back(g, v, ev, n, img, st);
  lmh::BrickImage b;
  if (int rc = b.alloc(g, st)) return rc;
  if (int rc = lmk::launch_to_layout(g.n, g.lay, 1, img, b.p, st)) return rc;
  if (int rc = launch_back(g, v, ev, n, b.p, st)) return rc;
  return lmk::launch_from_layout(g.n, g.lay, 1, b.p, img, st);
}

int lm_sens(const lm_geom *G, float *img, void *stream) {
  lmh::clear_error();
  GeomDev g;
  if (int rc = lmh::make_geom(G, &g)) return rc;
  LM_REQUIRE(img != nullptr, LM_EINVAL, "NULL image");
  hipStream_t st = lmh::as_stream(stream);
  lmh::BrickImage b;
  if (int rc = b.alloc(g, st)) return rc;
  if (int rc = lmk::launch_to_layout(g.n, g.lay, 1, img, b.p, st)) return rc;
  if (int rc = launch_sens(g, b.p, st)) return rc;
  return lmk::launch_from_layout(g.n, g.lay, 1, b.p, img, st);
}

int lm_validate_events(const lm_geom *G, const int16_t *ev, int64_t n, int64_t *n_bad, void *stream) {
  lmh::clear_error();
  GeomDev g;
  if (int rc = lmh::make_geom(G, &g)) return rc;
  LM_REQUIRE(n >= 0 && n_bad != nullptr, LM_EINVAL, "bad arguments");
  *n_bad = 0;
  if (n == 0) return LM_OK;
  LM_REQUIRE(ev != nullptr, LM_EINVAL, "NULL events");
  hipStream_t st = lmh::as_stream(stream);
  unsigned long long *d = nullptr;
  LM_TRY_HIP(hipMallocAsync((void **)&d, sizeof(unsigned long long), st));
  hipError_t e = hipMemsetAsync(d, 0, sizeof(unsigned long long), st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_validate, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g, ev, (long long)n, d);
    e = hipGetLastError();
  }
  unsigned long long h = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&h, d, sizeof(h), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  (void)hipFreeAsync(d, st);
  LM_TRY_HIP(e);
  *n_bad = (int64_t)h;
  return LM_OK;
}

}  // extern "C"
