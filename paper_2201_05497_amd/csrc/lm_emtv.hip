// Listmode EM-TV (Algorithm 3 of the paper), the warm start of LM-SPDHG:
// per subset an EM step z = x n / g P_i^T (1 / (P_i x + s_i)), the weights
// w = g / (beta x), and the weighted TV denoising
//   x+ = argmin_{u >= 0} sum_j w_j / 2 (u_j - z_j)^2 + ||K u||_{2,1}
// solved by the accelerated primal-dual algorithm of Chambolle & Pock (J.
// Math. Imaging Vis. 40, 2011, Algorithm 2).
//
// The EM step reuses the projector pair (bricked image, the events of the
// subset stored contiguously).  The denoising works on row-major images:
// each of its iterations is one pass marching along z (the dual step: forward
// differences of ubar, projection onto the unit balls; and the primal step:
// adjoint stencil, weighted prox, extrapolation), bound by the bandwidth of
// HBM and of the memory-side cache.  The step sizes of all
// iterations are computed on the device from the smallest finite weight,
// so a call never waits for the device.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "lm_host.hpp"
#include "lm_image.hpp"

namespace {

using lmk::GeomDev;

constexpr int kBlock = 256;
constexpr unsigned kInfBits = 0x7f800000u;  // +inf as float bits
constexpr long long kMaxGrid = 1LL << 20;   // grid-stride loops beyond this

inline unsigned grid_for(long long n) {
  return (unsigned)std::min<long long>((n + kBlock - 1) / kBlock, kMaxGrid);
}

// Subset i = {e : e mod n = i} stored contiguously: subset i starts at
// i (N div n) + min(i, N mod n) and holds its events in list order.
__host__ __device__ inline long long subset_start(long long N, int nsub, int i) {
  const long long r = N % nsub;
  return (long long)i * (N / nsub) + (i < r ? i : r);
}

__global__ __launch_bounds__(kBlock) void k_subset_order(const int16_t *__restrict__ ev, const float *__restrict__ s,
                                                         long long N, int nsub, int16_t *__restrict__ ev_out,
                                                         float *__restrict__ s_out) {
  for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < N; e += (long long)gridDim.x * kBlock) {
    const int i = (int)(e % nsub);
    const long long d = subset_start(N, nsub, i) + e / nsub;
#pragma unroll
    for (int c = 0; c < 5; ++c) ev_out[5 * d + c] = ev[5 * e + c];
    s_out[d] = s[e];
  }
}

// EM quotient, in place: q_e <- 1 / (q_e + s_e), 0 where q_e + s_e <= 0.
__global__ __launch_bounds__(kBlock) void k_em_quotient(float *__restrict__ q, const float *__restrict__ s,
                                                        long long m) {
  for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < m; e += (long long)gridDim.x * kBlock) {
    const float d = q[e] + s[e];
    q[e] = d > 0.0f ? 1.0f / d : 0.0f;
  }
}

__global__ void k_fill_u32(unsigned *__restrict__ p, long long n, unsigned v) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = v;
}

// The dual variable of the denoising, one image per component.
struct Dual {
  float *q[3];
};

// EM image z = x n bp / g (0 where g = 0), x <- z; bp is in layout L.  With
// beta > 0 also the weights w = g / (beta x) (inf where x = 0), the start of
// the denoising (u = ubar = z, with u in x) and the smallest weight of each
// block in part[blockIdx.x] (as float bits: non-negative floats order like
// their bits).
__global__ __launch_bounds__(kBlock) void k_em_image(float *__restrict__ x, const float *__restrict__ bp,
                                                     lmk::Layout L, int nx, int ny, const float *__restrict__ g,
                                                     long long nv, float nsub, float beta, float *__restrict__ z,
                                                     float *__restrict__ w, float *__restrict__ ubar,
                                                     unsigned *__restrict__ part) {
  __shared__ unsigned red[kBlock / 64];
  unsigned lo = kInfBits;
  for (long long j = (long long)blockIdx.x * kBlock + threadIdx.x; j < nv; j += (long long)gridDim.x * kBlock) {
    const float xj = x[j], gj = g[j];
    const unsigned row = (unsigned)j / (unsigned)nx, k = row / (unsigned)ny;
    const float b = bp[lmk::vidx(L, (int)((unsigned)j - row * nx), (int)(row - k * ny), (int)k)];
    const float zj = gj > 0.0f ? xj * nsub * b / gj : 0.0f;
    x[j] = zj;
    if (beta > 0.0f) {
      const float wj = xj > 0.0f ? gj / (beta * xj) : INFINITY;
      z[j] = zj;
      w[j] = wj;
      ubar[j] = zj;
      lo = min(lo, __float_as_uint(wj));
    }
  }
  if (beta <= 0.0f) return;
  for (int o = 32; o > 0; o >>= 1) lo = min(lo, (unsigned)__shfl_xor((int)lo, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lo;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kBlock / 64; ++i) lo = min(lo, red[i]);
    part[blockIdx.x] = lo;
  }
}

// Step sizes of the accelerated iterations: tau_0 = sigma_0 = 1/||K||,
// theta_k = 1 / sqrt(1 + 2 gam tau_k), tau_{k+1} = theta_k tau_k,
// sigma_{k+1} = sigma_k / theta_k, with gam the smallest finite weight
// (0 if every weight is infinite or the smallest is 0), reduced here from
// the npart block minima.  One block.
constexpr int kSchedBlock = 1024;
__global__ __launch_bounds__(kSchedBlock) void k_pd_schedule(const unsigned *__restrict__ part, int npart,
                                                             double tau0, int iters, float4 *__restrict__ sched) {
  __shared__ unsigned red[kSchedBlock / 64];
  unsigned lo = kInfBits;
#pragma unroll 4
  for (int i = threadIdx.x; i < npart; i += kSchedBlock) lo = min(lo, part[i]);
  for (int o = 32; o > 0; o >>= 1) lo = min(lo, (unsigned)__shfl_xor((int)lo, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lo;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int i = 1; i < kSchedBlock / 64; ++i) lo = min(lo, red[i]);
  const double gam = lo < kInfBits ? (double)__uint_as_float(lo) : 0.0;
  double tau = tau0, sigma = tau0;
  for (int k = 0; k < iters; ++k) {
    const double theta = 1.0 / sqrt(1.0 + 2.0 * gam * tau);
    sched[k] = make_float4((float)tau, (float)sigma, (float)theta, 0.0f);
    tau *= theta;
    sigma /= theta;
  }
}

// One iteration of the denoising, marching along z:
//   q+ = projection of q + sigma_k K ubar onto the unit ball of each voxel
//        (K = forward differences, zero in the last layer),
//   v = u - tau_k K^T q+,  u+ = max(0, (v + tau_k w z) / (1 + tau_k w)) (z
//        where w = inf),  ubar+ = u+ + theta_k (u+ - u).
// A block owns a column of 64 x 4 voxels (rows of 256 bytes) and a run of CZ
// planes.  K^T q+ needs q+ at the three lower neighbours: the thread's own
// value of the plane below (z), LDS (x, y), or the dual step of the column's
// left and front faces, which threads 0 .. 67 repeat; the plane below the
// run is computed first.  Planes k and k + 1 of ubar with a one-voxel ring
// are in LDS, plane k + 2 in registers; q, u, z and w of the next plane are
// loaded a step ahead.  ubar and q are read from one set of images and written to
// another (neighbouring blocks read them); u is the thread's own.
//
// 48 bytes per voxel, where a dual and a primal pass took 60 (q went to
// memory and back between them): 200x200x96, 48.8 -> 34.8 us, 5.3 TB/s, which is
// what a copy of this size reaches.  Columns are dealt so that each XCD works
// on a contiguous run: the lines of the ring and the faces, as many as the
// column's own, are then in its L2 (in the launch order of the blocks 54.6 us).
constexpr int kPX = 64, kPY = 4;  // the column

template <int CZ>
__global__ __launch_bounds__(kBlock) void k_pd_march(const float *__restrict__ ubar, Dual q, Dual qo, float *u,
                                                     const float *__restrict__ z, const float *__restrict__ w,
                                                     float *__restrict__ ubar_out, int nx, int ny, int nz,
                                                     const float4 *__restrict__ sched, int it) {
  static_assert(kPX * kPY == kBlock, "one thread per voxel of a plane");
  constexpr int RX = kPX + 2, RY = kPY + 2;        // box of ubar with its ring
  constexpr int kRing = RX * RY - kBlock, kFace = kPX + kPY;
  __shared__ float ub[2][RX * RY];
  __shared__ float s0[kPY][kPX + 1], s1[kPY + 1][kPX];
  const int t = threadIdx.x, ti = t % kPX, tj = t / kPX;
  const int ntx = (nx + kPX - 1) / kPX, nty = (ny + kPY - 1) / kPY;
  int blk = blockIdx.x;
  const int full = (int)gridDim.x & ~7;
  if (blk < full) blk = (blk & 7) * (full >> 3) + (blk >> 3);
  const int x0 = blk % ntx * kPX, y0 = blk / ntx % nty * kPY;
  const int kz0 = blk / (ntx * nty) * CZ, kz1 = min(nz, kz0 + CZ);
  const int i = x0 + ti, j = y0 + tj;
  const bool own = i < nx && j < ny;
  // images have at most 512^3 voxels: 32-bit indices
  const unsigned nxy = (unsigned)nx * ny;
  const unsigned at = own ? (unsigned)j * nx + i : 0u;
  const int ob = (ti + 1) + RX * (tj + 1);
  // ring cell of thread t < kRing: front row, back row, left and right columns
  int rb = 0;
  unsigned r_at = 0;
  bool r_ok = false;
  if (t < kRing) {
    int bx, by;
    if (t < RX) { bx = t; by = 0; }
    else if (t < 2 * RX) { bx = t - RX; by = RY - 1; }
    else { bx = (t - 2 * RX) & 1 ? RX - 1 : 0; by = 1 + (t - 2 * RX) / 2; }
    rb = bx + RX * by;
    const int gi = x0 - 1 + bx, gj = y0 - 1 + by;
    r_ok = gi >= 0 && gi < nx && gj >= 0 && gj < ny;
    r_at = r_ok ? (unsigned)gj * nx + gi : 0u;
  }
  // face voxel of thread t < kFace: left column (component 0), front row (1)
  int fb = 0, fi = 0, fj = 0;
  unsigned f_at = 0;
  bool f_ok = false;
  if (t < kFace) {
    const int bx = t < kPY ? 0 : t - kPY + 1, by = t < kPY ? t + 1 : 0;
    fb = bx + RX * by;
    fi = x0 - 1 + bx;
    fj = y0 - 1 + by;
    f_ok = fi >= 0 && fi < nx && fj >= 0 && fj < ny;
    f_at = f_ok ? (unsigned)fj * nx + fi : 0u;
  }
  const float4 st = sched[it];
  const float tau = st.x, sigma = st.y, theta = st.z;
  auto own_at = [&](int k) { return own && k < nz ? ubar[at + (unsigned)k * nxy] : 0.0f; };
  auto ring_at = [&](int k) { return r_ok && k < nz ? ubar[r_at + (unsigned)k * nxy] : 0.0f; };
  // the dual step at box position b of voxel (vi, vj, k): planes k and k + 1 of ubar in lo and up
  auto dual = [&](const float *lo, float upv, int b, int vi, int vj, int k, const float (&qv)[3], float (&qn)[3]) {
    const float c = lo[b];
    const float gx = vi + 1 < nx ? lo[b + 1] - c : 0.0f;
    const float gy = vj + 1 < ny ? lo[b + RX] - c : 0.0f;
    const float gz = k + 1 < nz ? upv - c : 0.0f;
    const float a0 = fmaf(sigma, gx, qv[0]), a1 = fmaf(sigma, gy, qv[1]), a2 = fmaf(sigma, gz, qv[2]);
    const float r = 1.0f / fmaxf(1.0f, sqrtf(a0 * a0 + a1 * a1 + a2 * a2));
    qn[0] = a0 * r;
    qn[1] = a1 * r;
    qn[2] = a2 * r;
  };
  auto load_q = [&](bool ok, unsigned p, float (&v)[3]) {
    for (int c = 0; c < 3; ++c) v[c] = ok && it > 0 ? q.q[c][p] : 0.0f;  // q = 0 at the start
  };
  float below = 0.0f;  // q+ along z of the plane below
  if (kz0 > 0) {
    const int k = kz0 - 1;
    ub[0][ob] = own_at(k);
    if (t < kRing) ub[0][rb] = ring_at(k);
    const float up = own_at(kz0);
    float qv[3], qn[3];
    load_q(own, at + (unsigned)k * nxy, qv);
    __syncthreads();
    dual(ub[0], up, ob, i, j, k, qv, qn);
    below = qn[2];
    __syncthreads();
  }
  ub[0][ob] = own_at(kz0);
  ub[1][ob] = own_at(kz0 + 1);
  if (t < kRing) {
    ub[0][rb] = ring_at(kz0);
    ub[1][rb] = ring_at(kz0 + 1);
  }
  float po = own_at(kz0 + 2), pr = ring_at(kz0 + 2);
  float qv[3], fq[3], uv = 0.0f, zv = 0.0f, wv = 0.0f;
  {
    const unsigned p = at + (unsigned)kz0 * nxy;
    load_q(own, p, qv);
    load_q(f_ok, f_at + (unsigned)kz0 * nxy, fq);
    if (own) {
      uv = u[p];
      zv = z[p];
      wv = w[p];
    }
  }
  __syncthreads();
  int lo = 0;  // LDS buffer of plane k
  for (int k = kz0; k < kz1; ++k, lo ^= 1) {
    // loads of the next step
    const float no = own_at(k + 3), nr = ring_at(k + 3);
    const bool more = k + 1 < kz1;
    const unsigned pn = at + (unsigned)(k + 1) * nxy;
    float nq[3], nfq[3], nu = 0.0f, nzv = 0.0f, nw = 0.0f;
    load_q(own && more, pn, nq);
    load_q(f_ok && more, f_at + (unsigned)(k + 1) * nxy, nfq);
    if (own && more) {
      nu = u[pn];
      nzv = z[pn];
      nw = w[pn];
    }
    const float *pl = ub[lo], *pu = ub[lo ^ 1];
    const unsigned p = at + (unsigned)k * nxy;
    float qn[3];
    dual(pl, pu[ob], ob, i, j, k, qv, qn);
    s0[tj][ti + 1] = qn[0];
    s1[tj + 1][ti] = qn[1];
    if (own)
      for (int c = 0; c < 3; ++c) qo.q[c][p] = qn[c];
    if (t < kFace) {
      float fn[3] = {0.0f, 0.0f, 0.0f};
      if (f_ok) dual(pl, pu[fb], fb, fi, fj, k, fq, fn);
      if (t < kPY) s0[t][0] = fn[0];
      else s1[0][t - kPY] = fn[1];
    }
    __syncthreads();
    // plane k + 2 takes the buffer of plane k
    ub[lo][ob] = po;
    if (t < kRing) ub[lo][rb] = pr;
    po = no;
    pr = nr;
    if (own) {
      float kt = 0.0f;
      if (i > 0) kt += s0[tj][ti];
      if (i + 1 < nx) kt -= qn[0];
      if (j > 0) kt += s1[tj][ti];
      if (j + 1 < ny) kt -= qn[1];
      if (k > 0) kt += below;
      if (k + 1 < nz) kt -= qn[2];
      float un;
      if (isinf(wv)) {
        un = zv;
      } else {
        const float v = fmaf(-tau, kt, uv);
        const float tw = tau * wv;
        un = fmaxf(0.0f, fmaf(tw, zv, v) / (1.0f + tw));
      }
      u[p] = un;
      ubar_out[p] = fmaf(theta, un - uv, un);
    }
    below = qn[2];
    for (int c = 0; c < 3; ++c) {
      qv[c] = nq[c];
      fq[c] = nfq[c];
    }
    uv = nu;
    zv = nzv;
    wv = nw;
    __syncthreads();
  }
}

// An iteration's launch: runs of 16 planes where that leaves three blocks per
// CU and more (200x200x96: 34.8 us, runs of 8 35.9, of 32 45.9), of 4 on
// smaller images (each run repeats the dual step of the plane below it).
int launch_pd(const float *ubar, const Dual &q, const Dual &qo, float *u, const float *z, const float *w,
              float *ubar_out, const int n[3], const float4 *sched, int it, hipStream_t st) {
  const long long cols = (long long)((n[0] + kPX - 1) / kPX) * ((n[1] + kPY - 1) / kPY);
  auto runs = [&](int cz) { return cols * ((n[2] + cz - 1) / cz); };
  if (runs(16) >= 768)
    hipLaunchKernelGGL((k_pd_march<16>), dim3((unsigned)runs(16)), dim3(kBlock), 0, st, ubar, q, qo, u, z, w,
                       ubar_out, n[0], n[1], n[2], sched, it);
  else
    hipLaunchKernelGGL((k_pd_march<4>), dim3((unsigned)runs(4)), dim3(kBlock), 0, st, ubar, q, qo, u, z, w, ubar_out,
                       n[0], n[1], n[2], sched, it);
  LM_TRY_HIP(hipGetLastError());
  return LM_OK;
}

// Stream-ordered device temporaries of one call, freed (stream-ordered)
// when the call returns.
struct Temps {
  hipStream_t st;
  void *p = nullptr;
  explicit Temps(hipStream_t s) : st(s) {}
  int get(lmh::Slab &arrays) {
    const hipError_t e = arrays.alloc(st, &p);
    if (e == hipSuccess) return LM_OK;
    lmh::set_error("lm_emtv temporaries of %zu bytes: %s", arrays.bytes(), hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? LM_ENOMEM : LM_EHIP;
  }
  ~Temps() {
    if (p) (void)hipFreeAsync(p, st);  // a release error has no caller to go to
  }
};

// Largest singular value of K (forward differences with a zero last layer
// along each axis): sqrt(sum_a 4 sin^2(pi (N_a - 1) / (2 N_a))).
double knorm(const int n[3]) {
  double s = 0.0;
  for (int a = 0; a < 3; ++a) {
    const double t = std::sin(M_PI * (n[a] - 1) / (2.0 * n[a]));
    s += 4.0 * t * t;
  }
  return std::sqrt(s);
}

}  // namespace

extern "C" {

int lm_emtv(const lm_geom *G, const int16_t *ev, const float *s, int64_t n, int32_t n_subsets, int32_t n_iter,
            const float *g, float beta, int32_t denoise_iter, float *x, void *stream) {
  lmh::clear_error();
  GeomDev gd;
  if (int rc = lmh::make_geom(G, &gd)) return rc;
  LM_REQUIRE(n >= 0, LM_EINVAL, "negative event count");
  LM_REQUIRE(n_subsets >= 1, LM_EINVAL, "n_subsets must be >= 1");
  LM_REQUIRE(n_iter >= 0 && denoise_iter >= 0, LM_EINVAL, "negative iteration count");
  LM_REQUIRE(beta >= 0.0f && std::isfinite(beta), LM_EINVAL, "beta must be finite and >= 0");
  LM_REQUIRE(g && x, LM_EINVAL, "NULL image");
  LM_REQUIRE(n == 0 || (ev && s), LM_EINVAL, "NULL event list");
  if (n_iter == 0) return LM_OK;
  hipStream_t st = lmh::as_stream(stream);
  const long long nv = lmh::nvox_of(gd.n);
  GeomDev gb = gd;
  gb.lay = lmh::brick_layout(gd.n);
  const long long nb = lmk::layout_size(gb.lay);
  const long long m_max = (n + n_subsets - 1) / n_subsets;
  const bool denoise = beta > 0.0f;
  const int iters = denoise ? denoise_iter : 0;

  Temps t(st);
  int16_t *evs = nullptr;
  float *ss = nullptr, *qe = nullptr, *xb = nullptr, *bpb = nullptr;
  float *z = nullptr, *w = nullptr, *u = nullptr, *ubar = nullptr, *ubar2 = nullptr, *q3 = nullptr;
  float4 *sched = nullptr;
  unsigned *part = nullptr;
  Dual qa{}, qb{};
  const unsigned img_grid = grid_for(nv);
  lmh::Slab arrays;
  arrays.add(&evs, 5 * n);
  arrays.add(&ss, n);
  arrays.add(&qe, m_max);
  for (float **q : {&xb, &bpb}) arrays.add(q, nb);
  if (denoise) {
    for (float **q : {&z, &w, &u, &ubar, &ubar2}) arrays.add(q, nv);
    arrays.add(&q3, 3 * nv);
    arrays.add(&part, img_grid);
    arrays.add(&sched, iters);
  }
  if (int rc = t.get(arrays)) return rc;
  if (denoise) {
    // the second set of ubar and q: images that are free while the denoising
    // runs (its u lives in x)
    qa = Dual{{q3, q3 + nv, q3 + 2 * nv}};
    qb = Dual{{xb, bpb, u}};
  }
  if (n > 0) {
    hipLaunchKernelGGL(k_subset_order, dim3(grid_for(n)), dim3(kBlock), 0, st, ev, s, (long long)n, (int)n_subsets,
                       evs, ss);
    LM_TRY_HIP(hipGetLastError());
  }
  const double tau0 = 1.0 / knorm(gd.n);
  for (int it = 0; it < n_iter; ++it) {
    for (int i = 0; i < n_subsets; ++i) {
      const long long o = subset_start(n, n_subsets, i);
      const long long m = subset_start(n, n_subsets, i + 1) - o;
      // EM step: bp = P_i^T (1 / (P_i x + s_i)) on the bricked image
      hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nb)), dim3(kBlock), 0, st, (unsigned *)bpb, nb, 0u);
      LM_TRY_HIP(hipGetLastError());
      if (m > 0) {
        if (int rc = lmk::launch_to_layout(gd.n, gb.lay, 1, x, xb, st)) return rc;
        if (int rc = lmk::launch_fwd(gb, xb, evs + 5 * o, m, qe, st)) return rc;
        hipLaunchKernelGGL(k_em_quotient, dim3(grid_for(m)), dim3(kBlock), 0, st, qe, ss + o, m);
        LM_TRY_HIP(hipGetLastError());
        if (int rc = lmk::launch_back(gb, qe, evs + 5 * o, m, bpb, st)) return rc;
      }
      hipLaunchKernelGGL(k_em_image, dim3(img_grid), dim3(kBlock), 0, st, x, bpb, gb.lay, gd.n[0], gd.n[1], g, nv,
                         (float)n_subsets, beta, z, w, ubar, part);
      LM_TRY_HIP(hipGetLastError());
      if (iters == 0) continue;
      hipLaunchKernelGGL(k_pd_schedule, dim3(1), dim3(kSchedBlock), 0, st, part, (int)img_grid, tau0, iters, sched);
      LM_TRY_HIP(hipGetLastError());
      float *ua = ubar, *ub = ubar2;
      for (int k = 0; k < iters; ++k) {
        if (int rc = launch_pd(ua, k % 2 ? qb : qa, k % 2 ? qa : qb, x, z, w, ub, gd.n, sched, k, st)) return rc;
        std::swap(ua, ub);
      }
    }
  }
  return LM_OK;
}

}  // extern "C"
