// Event lists in spatial order for the forward projection.
//
// Events in list order touch the whole image at any time, which the L2 of an
// XCD (4 MB) does not hold: k_fwd on 1e7 events and the pair image of
// 200x200x96 then waits for 1.9e8 lines from beyond the L2 (3.2 ms).  Here
// the events are binned by the part of the image that they cross, in two
// passes with per-workgroup histograms in LDS, projected bin after bin, and
// their results put back in list order.  With TOF a bin is the region that
// holds the centre of the event's window (an eighth of the image per axis);
// without, a strip of lines of like direction, distance from the axis and
// height.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "lm_host.hpp"
#include "lm_order.hpp"

using namespace lmk;

namespace {

constexpr int kBlock = 1024;
// Workgroups of the binning: one per CU, whose open lines (one per bin) then
// stay in the L2 until they are full.
constexpr int kRows = 256;
constexpr int kRegions = 8;      // per axis, at most
constexpr int kBins = kRegions * kRegions * kRegions + 1;  // the last: events that are out of range

// Bins per axis and the scale from positions to them.
struct Regions {
  int n[3];
  float scale[3], first[3];  // region = (position - first) * scale
  float radius;              // without TOF: of the lines that meet the image
};

// Crystal positions as the order takes them: the transaxial ones of ring 0
// and the heights of crystal 0 of every ring, in LDS.  On a scanner that is no
// cylinder they are wrong, which costs locality only; so the bin is
// computed in float.
constexpr int kTable = 7 << 10;  // floats
struct Crystals {
  const float *xy, *z;
};
__device__ __forceinline__ Crystals load_crystals(const GeomDev &g, float *lds) {
  for (int c = threadIdx.x; c < 2 * g.n_cry; c += kBlock) lds[c] = g.det[3 * (c >> 1) + (c & 1)];
  for (int r = threadIdx.x; r < g.n_ring; r += kBlock) lds[2 * g.n_cry + r] = g.det[3 * ((long long)g.n_cry * r) + 2];
  return {lds, lds + 2 * g.n_cry};
}

template <bool TOF>
__device__ __forceinline__ int bin_of(const GeomDev &g, const Regions &r, const Crystals &cr, int c1, int r1, int c2,
                                      int r2, int k) {
  const float ax = cr.xy[2 * c1], ay = cr.xy[2 * c1 + 1], az = cr.z[r1];
  const float dx = cr.xy[2 * c2] - ax, dy = cr.xy[2 * c2 + 1] - ay, dz = cr.z[r2] - az;
  float u[3];
  if constexpr (TOF) {
    const float lam = 0.5f + (float)k * (float)g.tof_bin * rsqrtf(fmaxf(dx * dx + dy * dy + dz * dz, 1e-12f));
    u[0] = fmaf(lam, dx, ax) - r.first[0];
    u[1] = fmaf(lam, dy, ay) - r.first[1];
    u[2] = fmaf(lam, dz, az) - r.first[2];
  } else {
    // direction in [0, 2) (of the line, either way), signed distance, middle height
    const float inv = rsqrtf(fmaxf(dx * dx + dy * dy, 1e-12f));
    const float s = dy < 0.0f ? -inv : inv;
    u[0] = 1.0f - dx * s;
    u[1] = (dx * ay - dy * ax) * s + r.radius;
    u[2] = fmaf(0.5f, dz, az) - r.first[2];
  }
  int bin = 0;
#pragma unroll
  for (int c = 2; c >= 0; --c) bin = bin * r.n[c] + (int)fminf(fmaxf(u[c] * r.scale[c], 0.0f), (float)(r.n[c] - 1));
  return bin;
}

// Bins of the events and the workgroup's counts; base: where the workgroup's
// events begin within each bin.
template <bool TOF>
__global__ __launch_bounds__(kBlock) void k_order_count(GeomDev g, Regions r, const int16_t *__restrict__ ev, int n,
                                                        int chunk, uint16_t *__restrict__ bins, unsigned *total,
                                                        unsigned *__restrict__ base) {
  __shared__ unsigned h[kBins];
  __shared__ float table[kTable];
  for (int t = threadIdx.x; t < kBins; t += kBlock) h[t] = 0u;
  const Crystals cr = load_crystals(g, table);
  __syncthreads();
  const int e0 = blockIdx.x * chunk, e1 = min(n, e0 + chunk);
#pragma unroll 4
  for (int e = e0 + threadIdx.x; e < e1; e += kBlock) {
    const int16_t *p = ev + 5 * (long long)e;
    int id1, id2, k, bin = kBins - 1;
    if (decode_event(g, p, id1, id2, k)) bin = bin_of<TOF>(g, r, cr, p[0], p[1], p[2], p[3], k);
    bins[e] = (uint16_t)bin;
    atomicAdd(&h[bin], 1u);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kBins; t += kBlock)
    if (h[t]) base[(long long)blockIdx.x * kBins + t] = atomicAdd(total + t, h[t]);
}

// total: counts -> first event of every bin.  One workgroup.
__global__ __launch_bounds__(kBlock) void k_order_scan(unsigned *total) {
  static_assert(kBins <= kBlock, "one bin per thread");
  __shared__ unsigned s[kBlock];
  const int t = threadIdx.x;
  const unsigned v = t < kBins ? total[t] : 0u;
  s[t] = v;
  __syncthreads();
  for (int o = 1; o < kBlock; o <<= 1) {
    const unsigned add = t >= o ? s[t - o] : 0u;
    __syncthreads();
    s[t] += add;
    __syncthreads();
  }
  if (t < kBins) total[t] = s[t] - v;
}

// The events in order, and every event's place in it.
__global__ __launch_bounds__(kBlock) void k_order_place(const int16_t *__restrict__ ev, int n, int chunk,
                                                        const uint16_t *__restrict__ bins,
                                                        const unsigned *__restrict__ first,
                                                        const unsigned *__restrict__ base,
                                                        OrderedEvent *__restrict__ rec, unsigned *__restrict__ place) {
  __shared__ unsigned h[kBins];
  // bins that the workgroup did not count hold no base and are not used
  for (int t = threadIdx.x; t < kBins; t += kBlock) h[t] = first[t] + base[(long long)blockIdx.x * kBins + t];
  __syncthreads();
  const int e0 = blockIdx.x * chunk, e1 = min(n, e0 + chunk);
#pragma unroll 4
  for (int e = e0 + threadIdx.x; e < e1; e += kBlock) {
    const int16_t *p = ev + 5 * (long long)e;
    OrderedEvent o;
    for (int c = 0; c < 5; ++c) o.ev[c] = p[c];
    o.ev[5] = 0;
    const unsigned at = atomicAdd(&h[bins[e]], 1u);
    rec[at] = o;
    place[e] = at;
  }
}

// out[e] = in[place[e]]: a workgroup's events lie in runs, one per bin, whose
// lines it reads through the L2.
__global__ __launch_bounds__(kBlock) void k_order_back(const float *__restrict__ in,
                                                       const unsigned *__restrict__ place, int n, int chunk,
                                                       float *__restrict__ out) {
  const int e0 = blockIdx.x * chunk, e1 = min(n, e0 + chunk);
#pragma unroll 4
  for (int e = e0 + threadIdx.x; e < e1; e += kBlock) out[e] = in[place[e]];
}

__global__ __launch_bounds__(256) void k_zero(unsigned *p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

}  // namespace

namespace lmk {

// Events of a workgroup: whole rounds of its threads.
static int order_chunk(long long n) { return (int)((n + kRows * kBlock - 1) / (kRows * kBlock)) * kBlock; }
static unsigned order_blocks(long long n) { return (unsigned)((n + order_chunk(n) - 1) / order_chunk(n)); }

bool order_possible(const GeomDev &g) { return 2LL * g.n_cry + g.n_ring <= kTable; }

void add_order(lmh::Slab &arrays, long long n, EventOrder &o) {
  arrays.add(&o.rec, n);
  arrays.add(&o.val, n);
  arrays.add(&o.place, n);
  arrays.add(&o.bins, n);
  arrays.add(&o.total, kBins);
  arrays.add(&o.base, kRows * kBins);
}

int launch_order(const GeomDev &g, const int16_t *ev, long long n, const EventOrder &o, hipStream_t st) {
  Regions r;
  double diag2 = 0.0;
  for (int a = 0; a < 3; ++a) {
    const int edge = std::max((g.n[a] + kRegions - 1) / kRegions, 4);
    r.n[a] = (g.n[a] + edge - 1) / edge;
    r.scale[a] = (float)(1.0 / (edge * g.h[a]));
    r.first[a] = (float)(g.c0[a] - 0.5 * g.h[a]);
    if (a < 2) diag2 += 0.25 * (g.n[a] * g.h[a]) * (g.n[a] * g.h[a]);
  }
  r.radius = (float)std::sqrt(diag2);
  if (!g.tof_on) {
    r.n[0] = r.n[1] = kRegions;
    r.scale[0] = 0.5f * kRegions;
    r.scale[1] = 0.5f * kRegions / r.radius;
  }
  const unsigned nb = order_blocks(n);
  const int chunk = order_chunk(n);
  hipLaunchKernelGGL(k_zero, dim3((kBins + 255) / 256), dim3(256), 0, st, o.total, kBins);
  if (g.tof_on)
    hipLaunchKernelGGL((k_order_count<true>), dim3(nb), dim3(kBlock), 0, st, g, r, ev, (int)n, chunk, o.bins, o.total,
                       o.base);
  else
    hipLaunchKernelGGL((k_order_count<false>), dim3(nb), dim3(kBlock), 0, st, g, r, ev, (int)n, chunk, o.bins, o.total,
                       o.base);
  hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(kBlock), 0, st, o.total);
  hipLaunchKernelGGL(k_order_place, dim3(nb), dim3(kBlock), 0, st, ev, (int)n, chunk, o.bins, o.total, o.base, o.rec,
                     o.place);
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

int launch_order_back(const EventOrder &o, long long n, float *out, hipStream_t st) {
  hipLaunchKernelGGL(k_order_back, dim3(order_blocks(n)), dim3(kBlock), 0, st, o.val, o.place, (int)n,
                     order_chunk(n), out);
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

}  // namespace lmk
