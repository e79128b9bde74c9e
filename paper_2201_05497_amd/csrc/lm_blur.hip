// Image-space resolution model (Section 1: the forward model includes
// limited spatial resolution): P = G B with B a separable Gaussian
// convolution, zero outside the image, so that B is symmetric and the back
// projection applies the same B after G^T.  Radii up to kFusedRadius: all
// axes in one pass over the plan's bricked images, by box in LDS.  Beyond:
// one pass per blurred axis; each voxel reads 2 r + 1 neighbours along the
// axis (L2 hits, all loads in flight at once) and writes one value.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "lm_blur.hpp"
#include "lm_host.hpp"
#include "lm_layout32.hpp"

namespace {

constexpr int kBlock = 256;

inline unsigned grid_for(long long n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// The blur along one axis at the voxel of layout position p with
// coordinate c0 along that axis (n voxels): the sum over t = -R..R, in that
// order, of w[t + R] x(c0 + t), taps outside the image skipped.  The 2R + 1
// loads (at clamped, always valid positions) are all issued before the
// first product, so a wavefront waits for memory once per voxel, not once
// per tap.
template <int R>
__device__ __forceinline__ float blur_at(const float *__restrict__ in, const lmk::AxisTerm &ta, unsigned p, int c0,
                                         int n, const lmk::BlurAxis &taps) {
  const int base = (int)p - lmk::axis_index(ta, c0);
  float v[2 * R + 1];
#pragma unroll
  for (int t = -R; t <= R; ++t) v[t + R] = in[base + lmk::axis_index(ta, min(max(c0 + t, 0), n - 1))];
  float acc = 0.0f;
#pragma unroll
  for (int t = -R; t <= R; ++t)
    if (c0 + t >= 0 && c0 + t < n) acc = fmaf(taps.w[t + R], v[t + R], acc);
  return acc;
}

// out = blur of `in` along `axis` with radius R (= taps.r).
template <int R>
__global__ __launch_bounds__(kBlock) void k_blur_axis(const float *__restrict__ in, float *__restrict__ out,
                                                      lmk::Layout L, int nx, int ny, int nz, long long ne, int axis,
                                                      lmk::BlurAxis taps) {
  const unsigned p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= ne) return;
  int c[3];
  lmk::vpos32(L, p, c[0], c[1], c[2]);
  if (c[0] >= nx || c[1] >= ny || c[2] >= nz) return;  // padding
  const int n = axis == 0 ? nx : axis == 1 ? ny : nz;
  out[p] = blur_at<R>(in, lmk::axis_term(L, axis), p, c[axis], n, taps);
}

// The last blur pass of a data update's back projection fused with the z
// step: d = (blur along `axis` of src)_p, z += d, zbar = z + d inv_p,
// fuse ? x = max(0, x - T zbar) : store zbar, and dz = 0 for the next
// update's atomics (dz is not read by this pass: src is a temporary).
template <int R>
__global__ __launch_bounds__(kBlock) void k_blur_axis_dual(const float *__restrict__ src, float *__restrict__ dz,
                                                           float *__restrict__ z, float *__restrict__ x,
                                                           const float *__restrict__ T, float *__restrict__ zbar,
                                                           float inv_p, int fuse, lmk::Layout L, int nx, int ny,
                                                           int nz, long long ne, int axis, lmk::BlurAxis taps) {
  const unsigned p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= ne) return;
  int c[3];
  lmk::vpos32(L, p, c[0], c[1], c[2]);
  if (c[0] >= nx || c[1] >= ny || c[2] >= nz) return;  // padding (stays zero)
  const int n = axis == 0 ? nx : axis == 1 ? ny : nz;
  const float d = blur_at<R>(src, lmk::axis_term(L, axis), p, c[axis], n, taps);
  const float zn = z[p] + d;
  const float zb = fmaf(d, inv_p, zn);
  z[p] = zn;
  if (fuse)
    x[p] = fmaxf(0.0f, fmaf(-T[p], zb, x[p]));
  else
    zbar[p] = zb;
  dz[p] = 0.0f;
}

__global__ __launch_bounds__(kBlock) void k_clear(float *__restrict__ p, long long n) {
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

// What the last pass over a voxel does with its blurred value.
struct StoreImage {
  float *out;
  struct Pre {};
  __device__ __forceinline__ Pre pre(unsigned) const { return {}; }
  __device__ __forceinline__ void operator()(unsigned p, float d, const Pre &) const { out[p] = d; }
};
// the z step: z += d, zbar = z + d inv_p, fuse ? x = max(0, x - T zbar) : store zbar
struct DualStep {
  float *z, *x;
  const float *T;
  float *zbar;
  float inv_p;
  int fuse;
  struct Pre {
    float z, x, T;
  };
  __device__ __forceinline__ Pre pre(unsigned p) const { return {z[p], fuse ? x[p] : 0.0f, fuse ? T[p] : 0.0f}; }
  __device__ __forceinline__ void operator()(unsigned p, float d, const Pre &v) const {
    const float zn = v.z + d, zb = fmaf(d, inv_p, zn);
    z[p] = zn;
    if (fuse) x[p] = fmaxf(0.0f, fmaf(-v.T, zb, v.x));
    else zbar[p] = zb;
  }
};

// `N` consecutive outputs along an axis of radius r <= R whose cells are
// `stride` floats apart: out[k] = sum over t = -r..r of w[t + r] v[k + t],
// in that order, with `first` the cell R below output 0.
template <int R, int N>
__device__ __forceinline__ void blur_run(const float *first, int stride, const float *w, int r, float (&out)[N]) {
  float v[N + 2 * R];
#pragma unroll
  for (int c = 0; c < N + 2 * R; ++c)
    if (c >= R - r && c < N + R + r) v[c] = first[c * stride];
#pragma unroll
  for (int k = 0; k < N; ++k) out[k] = 0.0f;
#pragma unroll
  for (int t = -R; t <= R; ++t)
    if (t >= -r && t <= r) {
      const float wt = w[t + r];
#pragma unroll
      for (int k = 0; k < N; ++k) out[k] = fmaf(wt, v[k + t + R], out[k]);
    }
}

// Blur along all axes (radii up to R, along z up to RZ) of a TX x TY x TZ
// tile per workgroup: the tile with its ring is read into LDS (zero outside the
// image: a skipped tap), blurred along x, y and z between LDS buffers in
// runs that read each cell once, and handed to `store`.  The values and their
// order are those of the passes per axis.  Bound by instruction issue and
// the reads of the ring, which the L2 holds where neighbouring tiles run on
// one XCD (contiguous runs of tiles per XCD).  A thread reads a column of the
// box, so that what depends on the plane is uniform; row strides are odd, or
// odd multiples of 8, so that a wavefront's LDS accesses spread over the
// banks.
template <int R, int RZ, int TX, int TY, int TZ, class Store>
__global__ __launch_bounds__(kBlock) void k_blur_box(const float *__restrict__ in, lmk::Layout L, int nx, int ny,
                                                     int nz, lmk::Blur b, Store store) {
  constexpr int NZ = TX * TY * TZ / kBlock;  // outputs per thread
  static_assert(NZ >= 1 && TZ % NZ == 0 && TX % 4 == 0 && TY % 4 == 0 && TX * TY * TZ == NZ * kBlock, "tile");
  constexpr int bx = TX + 2 * R, by = TY + 2 * R, bz = TZ + 2 * RZ;  // the box
  constexpr int sa = bx | 1, sb = TX * (by | 1), sc = TX * TY + 8;
  __shared__ __attribute__((aligned(16))) float B[bz * sb];
  __shared__ float A[bz * (by * sa > sc ? by * sa : sc)];
  float *C = A;
  const int rx = b.ax[0].r, ry = b.ax[1].r, rz = b.ax[2].r;
  const int t = threadIdx.x;
  int blk = blockIdx.x;
  const int full = (int)gridDim.x & ~7;
  if (blk < full) blk = (blk & 7) * (full >> 3) + (blk >> 3);
  const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
  const int x0 = blk % ntx * TX, y0 = blk / ntx % nty * TY, z0 = blk / (ntx * nty) * TZ;
#pragma unroll
  for (int e = t; e < bx * by; e += kBlock) {
    const int ix = e % bx, iy = e / bx, i = x0 - R + ix, j = y0 - R + iy;
    const bool ok = (unsigned)i < (unsigned)nx && (unsigned)j < (unsigned)ny;
    const int ij = ok ? lmk::vidx(L, i, j, 0) : 0;
    float v[bz];
#pragma unroll
    for (int k = 0; k < bz; ++k) {
      const int z = z0 - RZ + k;
      v[k] = ok && (unsigned)z < (unsigned)nz ? in[ij + lmk::vidx(L, 0, 0, z)] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < bz; ++k) A[(k * by + iy) * sa + ix] = v[k];
  }
  // this thread's outputs: column (ti, tj), planes tk .. tk + NZ - 1; lanes
  // 0..15 are one 4x4 slab of a brick
  const int col = t % (TX * TY), tk = t / (TX * TY) * NZ;
  const int slab = col >> 4, ti = (slab % (TX / 4)) * 4 + (col & 3), tj = slab / (TX / 4) * 4 + ((col >> 2) & 3);
  const bool own = x0 + ti < nx && y0 + tj < ny;
  unsigned at[NZ];
  typename Store::Pre pre[NZ];
#pragma unroll
  for (int k = 0; k < NZ; ++k) {
    const bool ok = own && z0 + tk + k < nz;
    at[k] = ok ? (unsigned)lmk::vidx(L, x0 + ti, y0 + tj, z0 + tk + k) : ~0u;
    if (ok) pre[k] = store.pre(at[k]);
  }
  __syncthreads();
  for (int e = t; e < by * bz * (TX / 4); e += kBlock) {
    const int h = e % (TX / 4), row = e / (TX / 4), iy = row % by, iz = row / by;
    float o[4];
    blur_run<R, 4>(A + row * sa + 4 * h, 1, b.ax[0].w, rx, o);
    *(float4 *)(B + iz * sb + iy * TX + 4 * h) = make_float4(o[0], o[1], o[2], o[3]);
  }
  __syncthreads();
  for (int e = t; e < TX * bz * (TY / 4); e += kBlock) {
    const int ix = e % TX, h = e / TX % (TY / 4), iz = e / (TX * (TY / 4));
    float o[4];
    blur_run<R, 4>(B + iz * sb + 4 * h * TX + ix, TX, b.ax[1].w, ry, o);
#pragma unroll
    for (int k = 0; k < 4; ++k) C[iz * sc + (4 * h + k) * TX + ix] = o[k];
  }
  __syncthreads();
  float o[NZ];
  blur_run<RZ, NZ>(C + tk * sc + tj * TX + ti, sc, b.ax[2].w, rz, o);
#pragma unroll
  for (int k = 0; k < NZ; ++k)
    if (at[k] != ~0u) store(at[k], o[k], pre[k]);
}

// One pass where every radius is at most kFusedRadius: beyond, the ring
// outgrows LDS and its reads.  A data update of 2000 events, two blurs, on
// 128x128x48 / 200x200x96: radius 2, 39.3 -> 26.7 / 105 -> 66.8 us; radius 4,
// 45.6 -> 32.3 / 139 -> 90.9 us (one blur of 128x128x48 at radius 2: 15.2 -> 7.9
// us).
constexpr int kFusedRadius = 4;

bool fused_blur_ok(const lmk::Blur &b) {
  return std::max({b.ax[0].r, b.ax[1].r, b.ax[2].r}) <= kFusedRadius;
}

template <int R, int RZ, int TX, int TY, int TZ, class Store>
int launch_box_tile(const float *in, const lmk::Layout &L, const int n[3], const lmk::Blur &b, const Store &store,
                    hipStream_t st) {
  const long long nb = (long long)((n[0] + TX - 1) / TX) * ((n[1] + TY - 1) / TY) * ((n[2] + TZ - 1) / TZ);
  hipLaunchKernelGGL((k_blur_box<R, RZ, TX, TY, TZ, Store>), dim3((unsigned)nb), dim3(kBlock), 0, st, in, L, n[0],
                     n[1], n[2], b, store);
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

template <int R, class Store>
int launch_box_radius(const float *in, const lmk::Layout &L, const int n[3], const lmk::Blur &b, const Store &store,
                      hipStream_t st) {
  return n[2] == 1 ? launch_box_tile<R, 0, 16, 16, 1>(in, L, n, b, store, st)
                   : launch_box_tile<R, R, 8, 8, 8>(in, L, n, b, store, st);
}

template <class Store>
int launch_box(const float *in, const lmk::Layout &L, const int n[3], lmk::Blur b, const Store &store,
               hipStream_t st) {
  for (lmk::BlurAxis &ax : b.ax)
    if (ax.r == 0) ax.w[0] = 1.0f;  // an axis left alone
  lmk::BlurAxis &az = b.ax[2];
  if (n[2] == 1) {  // one slice: only the middle tap along z meets the image
    az.w[0] = az.w[az.r];
    az.r = 0;
  }
  switch (std::max({b.ax[0].r, b.ax[1].r, az.r})) {
    case 0:
    case 1:
    case 2: return launch_box_radius<2>(in, L, n, b, store, st);
    case 3: return launch_box_radius<3>(in, L, n, b, store, st);
    default: return launch_box_radius<kFusedRadius>(in, L, n, b, store, st);
  }
}

// The kernels of radius taps.r (0..kMaxBlurRadius).
#define LM_BLUR_RADII(M) \
  M(0) M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15) M(16)
static_assert(lmk::kMaxBlurRadius == 16, "one kernel per radius up to kMaxBlurRadius");

int launch_axis(const float *in, float *out, const lmk::Layout &L, const int n[3], long long ne, int axis,
                const lmk::BlurAxis &taps, hipStream_t st) {
  switch (taps.r) {
#define LM_CASE(R_)                                                                                              \
  case R_:                                                                                                       \
    hipLaunchKernelGGL((k_blur_axis<R_>), dim3(grid_for(ne)), dim3(kBlock), 0, st, in, out, L, n[0], n[1], n[2], \
                       ne, axis, taps);                                                                          \
    break;
    LM_BLUR_RADII(LM_CASE)
#undef LM_CASE
    default:
      lmh::set_error("blur radius %d outside 0..%d", taps.r, lmk::kMaxBlurRadius);
      return LM_EINVAL;
  }
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

int launch_axis_dual(const float *src, float *dz, float *z, float *x, const float *T, float *zbar, float inv_p,
                     bool fuse, const lmk::Layout &L, const int n[3], long long ne, int axis,
                     const lmk::BlurAxis &taps, hipStream_t st) {
  switch (taps.r) {
#define LM_CASE(R_)                                                                                              \
  case R_:                                                                                                       \
    hipLaunchKernelGGL((k_blur_axis_dual<R_>), dim3(grid_for(ne)), dim3(kBlock), 0, st, src, dz, z, x, T, zbar,  \
                       inv_p, fuse ? 1 : 0, L, n[0], n[1], n[2], ne, axis, taps);                                \
    break;
    LM_BLUR_RADII(LM_CASE)
#undef LM_CASE
    default:
      lmh::set_error("blur radius %d outside 0..%d", taps.r, lmk::kMaxBlurRadius);
      return LM_EINVAL;
  }
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

}  // namespace

namespace lmk {

int make_blur(const double fwhm[3], Blur *b) {
  b->on = false;
  for (int a = 0; a < 3; ++a) {
    BlurAxis &ax = b->ax[a];
    ax.r = 0;
    for (float &w : ax.w) w = 0.0f;
    const double f = fwhm[a];
    LM_REQUIRE(f >= 0.0 && std::isfinite(f), LM_EINVAL, "FWHM along axis %d must be finite and >= 0", a);
    if (f == 0.0) continue;
    const double sig = f / (2.0 * std::sqrt(2.0 * std::log(2.0)));
    const int r = (int)std::ceil(3.0 * sig);
    LM_REQUIRE(r <= kMaxBlurRadius, LM_EINVAL, "FWHM %.3g voxels along axis %d exceeds the largest supported (%d taps)",
               f, a, 2 * kMaxBlurRadius + 1);
    double w[2 * kMaxBlurRadius + 1], sum = 0.0;
    for (int t = -r; t <= r; ++t) sum += (w[t + r] = std::exp(-(double)t * t / (2.0 * sig * sig)));
    for (int t = -r; t <= r; ++t) ax.w[t + r] = (float)(w[t + r] / sum);
    ax.r = r;
    b->on = true;
  }
  return LM_OK;
}

int launch_blur(const int n[3], const Layout &L, long long ne, const Blur &b, const float *in, float *out, float *t1,
                float *t2, hipStream_t st) {
  int axes[3], na = 0;
  for (int a = 0; a < 3; ++a)
    if (b.ax[a].r > 0) axes[na++] = a;
  if (na == 0) {
    LM_TRY_HIP(hipMemcpyAsync(out, in, (size_t)ne * sizeof(float), hipMemcpyDeviceToDevice, st));
    return LM_OK;
  }
  if (fused_blur_ok(b)) return launch_box(in, L, n, b, StoreImage{out}, st);
  const float *src = in;
  for (int k = 0; k < na; ++k) {
    float *dst = k + 1 == na ? out : (k % 2 == 0 ? t1 : t2);
    if (int rc = launch_axis(src, dst, L, n, ne, axes[k], b.ax[axes[k]], st)) return rc;
    src = dst;
  }
  return LM_OK;
}

int launch_blur_dual_image(const int n[3], const Layout &L, long long ne, const Blur &b, float *dz, float *t1,
                           float *t2, float *z, float *x, const float *T, float *zbar, float inv_p, bool fuse,
                           bool clear, hipStream_t st) {
  int axes[3], na = 0;
  for (int a = 0; a < 3; ++a)
    if (b.ax[a].r > 0) axes[na++] = a;
  LM_REQUIRE(na > 0, LM_EINVAL, "no blurred axis");
  if (fused_blur_ok(b)) {
    if (int rc = launch_box(dz, L, n, b, DualStep{z, x, T, zbar, inv_p, fuse ? 1 : 0}, st)) return rc;
    if (clear) {
      hipLaunchKernelGGL(k_clear, dim3(grid_for(ne)), dim3(kBlock), 0, st, dz, ne);
      LM_TRY_HIP(hipGetLastError());
    }
    return LM_OK;
  }
  // all passes but the last; with one blurred axis that pass goes to t1
  // and the fused pass applies the identity (it must not read dz)
  const float *src = dz;
  const int plain = na == 1 ? 1 : na - 1;
  for (int k = 0; k < plain; ++k) {
    float *dst = k % 2 == 0 ? t1 : t2;
    if (int rc = launch_axis(src, dst, L, n, ne, axes[k], b.ax[axes[k]], st)) return rc;
    src = dst;
  }
  BlurAxis last{};
  int axis = 0;
  if (na == 1) {
    last.r = 0;
    last.w[0] = 1.0f;
  } else {
    axis = axes[na - 1];
    last = b.ax[axis];
  }
  return launch_axis_dual(src, dz, z, x, T, zbar, inv_p, fuse, L, n, ne, axis, last, st);
}

}  // namespace lmk
