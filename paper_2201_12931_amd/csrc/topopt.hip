// Density filter (weights of Eqs. 4-5) and the optimality-criteria update
// (Eqs. 8-9) on the GPU.
//
// Filter: rho~_e = sum_i w_ei x_i / sum_i w_ei over in-domain elements i with
// w_ei = max(0, r - |c_e - c_i|).  The weight sum is recomputed per element
// (it only depends on how the stencil is cut by the domain), so no array of
// weight sums is stored.  The adjoint is g_x = H (g / Hs) (H is symmetric).
//
// OC: x_new(lambda) = clamp(x B^eta, max(0, x - m), min(1, x + m)) with
// B = -dc / (lambda dv).  Because x B^eta = s_e lambda^(-eta) with
// s_e = x_e (-dc_e / dv_e)^eta, one pass over the elements evaluates the volume
// dv^T x_new(lambda) (the filtered volume is linear in x) for kOcProbes values
// of lambda at once, and one small launch narrows the bracket by that factor; the
// number of passes is known beforehand, so the host waits only at the end.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "hexmg_impl.h"

namespace hexmg {

namespace {

// In-plane distance classes of a filter of half-width R: the distinct di^2 +
// dj^2 with |di|, |dj| <= R, ascending.
template <int R>
struct FilterClasses {
  static constexpr int n = R == 1 ? 3 : (R == 2 ? 6 : 10);
  static constexpr int d2(int c) {
    constexpr int v[10] = {0, 1, 2, 4, 5, 8, 9, 10, 13, 18};
    return v[c];
  }
  static constexpr int of(int d) {
    int c = 0;
    while (d2(c) != d) ++c;
    return c;
  }
};
constexpr int kFilterMaxR = 3, kFilterMaxClasses = 10;
// Weights by plane distance and in-plane class, w[dk][c] = rmin - sqrt(dk^2 +
// d2(c)); the first n[dk] classes have a positive one (the others take no part).
struct FilterWeights {
  double w[kFilterMaxR + 1][kFilterMaxClasses];
  int n[kFilterMaxR + 1];
};

// out[dk] = sum of w[dk][c] S[c] over the classes that take part at dk
template <int R>
__device__ inline void class_products(const FilterWeights& fw, const double (&S)[FilterClasses<R>::n],
                                      double (&out)[R + 1]) {
#pragma unroll
  for (int dk = 0; dk <= R; ++dk) {
    double t = 0.0;
#pragma unroll
    for (int c = 0; c < FilterClasses<R>::n; ++c)
      if (c < fw.n[dk]) t += fw.w[dk][c] * S[c];  // uniform: a class without weight may hold anything
    out[dk] = t;
  }
}
// Weight sums of element column (i, j) by plane distance: the in-domain offsets
// of each class, counted and weighted.
template <int R>
__device__ inline void column_weights(const FilterWeights& fw, int i, int j, int nx, int ny, double (&P)[R + 1]) {
  using C = FilterClasses<R>;
  double N[C::n];
#pragma unroll
  for (int c = 0; c < C::n; ++c) N[c] = 0.0;
#pragma unroll
  for (int dj = -R; dj <= R; ++dj)
#pragma unroll
    for (int di = -R; di <= R; ++di)
      N[C::of(di * di + dj * dj)] += (i + di >= 0 && i + di < nx && j + dj >= 0 && j + dj < ny) ? 1.0 : 0.0;
  class_products<R>(fw, N, P);
}
// Hs of the element at height k of a column with weight sums P.
template <int R>
__device__ inline double weight_sum(const double (&P)[R + 1], int k, int nz) {
  double ws = P[0];
#pragma unroll
  for (int d = 1; d <= R; ++d) ws += (k - d >= 0 ? P[d] : 0.0) + (k + d < nz ? P[d] : 0.0);
  return ws;
}

// The filters for half-widths 1..3 (rmin <= 4).  A block of 32 x 8 element
// columns marches through zchunk planes; each plane of its tile, with a halo of
// R, is staged in LDS once (double-buffered; the next plane's loads are in
// flight meanwhile), so an input is read from memory once per tile instead of
// once per neighbour.  Offsets at the same distance share a weight: a thread
// sums the (2R+1)^2 values around its column by distance class, forms the
// plane's contribution at each plane distance from the class sums (the two
// sides dk and -dk share it) and adds it to the 2R+1 outputs in flight.  That
// is 25 LDS reads and about 50 operations per element for R = 2 instead of
// 125 loads, square roots and products, and leaves the pass bound by the LDS
// reads and its traffic: forward, adjoint and sensitivity filter of 256x128x128
// at rmin 3 take 0.120 ms together (1.96 TB/s of their 7 vectors) where one
// thread per element over its neighbours, each weight a square root, took
// 1.65 ms.
// MODE 0: out = (H in) / Hs;  2: out = H (in / Hs);  3 (sensitivity filter,
// Eq. 3): out = (H (x in)) / (max(gamma, x) Hs).
template <int MODE, int R>
__global__ __launch_bounds__(256) void k_filter_tile(int nx, int ny, int nz, int zchunk, FilterWeights fw,
                                                     double gamma, const double* __restrict__ x,
                                                     const double* __restrict__ in, double* __restrict__ out) {
  using C = FilterClasses<R>;
  constexpr int TX = 32, TY = 8, SX = TX + 2 * R, SY = TY + 2 * R, NS = (SX * SY + 255) / 256;
  __shared__ double tile[2][SY][SX];
  const int tx = threadIdx.x & (TX - 1), ty = threadIdx.x / TX;
  const int i0 = blockIdx.x * TX, j0 = blockIdx.y * TY;
  const int k0 = blockIdx.z * zchunk, k1 = min(k0 + zchunk, nz);
  const int i = i0 + tx, j = j0 + ty;
  const long long plane = (long long)nx * ny;
  // the columns this thread stages: tile slot, offset in a plane (-1: outside)
  int so[NS];
  double Ps[MODE == 2 ? NS : 1][R + 1];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int e = threadIdx.x + 256 * s;
    const int ii = i0 - R + e % SX, jj = j0 - R + e / SX;
    so[s] = (e < SX * SY && ii >= 0 && ii < nx && jj >= 0 && jj < ny) ? ii + nx * jj : -1;
    if (MODE == 2) column_weights<R>(fw, ii, jj, nx, ny, Ps[MODE == 2 ? s : 0]);
  }
  auto load = [&](int kk, double (&v)[NS]) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const bool on = so[s] >= 0 && kk >= 0 && kk < nz && kk < k1 + R;
      const long long o = on ? so[s] + plane * kk : 0;
      v[s] = on ? in[o] : 0.0;
      if (MODE == 3) v[s] = on ? x[o] * v[s] : 0.0;
      if (MODE == 2) v[s] = on ? v[s] / weight_sum<R>(Ps[MODE == 2 ? s : 0], kk, nz) : 0.0;
    }
  };
  double P[R + 1];
  if (MODE != 2) column_weights<R>(fw, i, j, nx, ny, P);
  double acc[2 * R + 1];  // outputs kk - R .. kk + R
#pragma unroll
  for (int t = 0; t <= 2 * R; ++t) acc[t] = 0.0;
  double v[NS];
  load(k0 - R, v);
  for (int kk = k0 - R; kk < k1 + R; ++kk) {
    double(*buf)[SX] = tile[(kk - k0 + R) & 1];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int e = threadIdx.x + 256 * s;
      if (e < SX * SY) buf[e / SX][e % SX] = v[s];
    }
    __syncthreads();  // the other buffer's readers passed the previous barrier's plane
    load(kk + 1, v);
    double S[C::n];
#pragma unroll
    for (int c = 0; c < C::n; ++c) S[c] = 0.0;
#pragma unroll
    for (int dj = -R; dj <= R; ++dj)
#pragma unroll
      for (int di = -R; di <= R; ++di) S[C::of(di * di + dj * dj)] += buf[ty + R + dj][tx + R + di];
    double con[R + 1];
    class_products<R>(fw, S, con);
#pragma unroll
    for (int t = 0; t <= 2 * R; ++t) acc[t] += con[t < R ? R - t : t - R];
    const int k = kk - R;
    if (k >= k0 && i < nx && j < ny) {
      const long long me = i + nx * j + plane * k;
      if (MODE == 2)
        out[me] = acc[0];
      else if (MODE == 0)
        out[me] = acc[0] / weight_sum<R>(P, k, nz);
      else
        out[me] = acc[0] / (fmax(gamma, x[me]) * weight_sum<R>(P, k, nz));
    }
#pragma unroll
    for (int t = 0; t < 2 * R; ++t) acc[t] = acc[t + 1];
    acc[2 * R] = 0.0;
  }
}

// The filters for any half-width, one thread per element over its neighbours.
// The launchers take it above half-width kFilterMaxR, where the tiled form's
// unrolled classes and weights outgrow the registers (half-width 3 already
// spills scalars), and for half-width 0.
// MODE 0: out = (H in) / Hs;  1: out = in / Hs;  2: out = H in.
template <int MODE>
__global__ void k_filter(int nx, int ny, int nz, double rmin, int R, const double* __restrict__ in,
                         double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y, k = blockIdx.z;
  if (i >= nx) return;
  const long long me = i + (long long)nx * (j + (long long)ny * k);
  double s = 0.0, ws = 0.0;
  for (int dk = -R; dk <= R; ++dk) {
    const int kk = k + dk;
    if (kk < 0 || kk >= nz) continue;
    for (int dj = -R; dj <= R; ++dj) {
      const int jj = j + dj;
      if (jj < 0 || jj >= ny) continue;
      for (int di = -R; di <= R; ++di) {
        const int ii = i + di;
        if (ii < 0 || ii >= nx) continue;
        const double w = rmin - sqrt((double)(di * di + dj * dj + dk * dk));
        if (w <= 0.0) continue;
        ws += w;
        if (MODE != 1) s += w * in[ii + (long long)nx * (jj + (long long)ny * kk)];
      }
    }
  }
  if (MODE == 0)
    out[me] = s / ws;
  else if (MODE == 1)
    out[me] = in[me] / ws;
  else
    out[me] = s;
}

// Sensitivity filter (Eq. 3): out_e = (sum_i w_ei x_i dc_i) / (max(gamma, x_e) sum_i w_ei)
__global__ void k_sens_filter(int nx, int ny, int nz, double rmin, int R, double gamma, const double* __restrict__ x,
                              const double* __restrict__ dc, double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y, k = blockIdx.z;
  if (i >= nx) return;
  const long long me = i + (long long)nx * (j + (long long)ny * k);
  double s = 0.0, ws = 0.0;
  for (int dk = -R; dk <= R; ++dk) {
    const int kk = k + dk;
    if (kk < 0 || kk >= nz) continue;
    for (int dj = -R; dj <= R; ++dj) {
      const int jj = j + dj;
      if (jj < 0 || jj >= ny) continue;
      for (int di = -R; di <= R; ++di) {
        const int ii = i + di;
        if (ii < 0 || ii >= nx) continue;
        const double w = rmin - sqrt((double)(di * di + dj * dj + dk * dk));
        if (w <= 0.0) continue;
        const long long o = ii + (long long)nx * (jj + (long long)ny * kk);
        ws += w;
        s += w * x[o] * dc[o];
      }
    }
  }
  out[me] = s / (fmax(gamma, x[me]) * ws);
}

// Self-weight: f = f_ext - (g / 8) sum_{e adjacent} rho_e along z (each of an
// element's eight nodes takes an eighth of its weight).  f_ext may be null.
__global__ void k_gravity_load(Level L, const double* __restrict__ rho, double g, const double* __restrict__ f_ext,
                               double* __restrict__ f) {
  const int n = blockIdx.x * kBlock + threadIdx.x;
  if (n >= L.nn) return;
  const int i = n % L.nxn, t = n / L.nxn, j = t % L.nyn, k = t / L.nyn;
  double s = 0.0;
  for (int a = 0; a < 8; ++a) {
    const int ei = i - (a & 1), ej = j - ((a >> 1) & 1), ek = k - (a >> 2);
    if (ei < 0 || ei >= L.nx || ej < 0 || ej >= L.ny || ek < 0 || ek >= L.nz) continue;
    s += rho[ei + L.nx * (ej + L.ny * ek)];
  }
  const long long b = 3ll * n;
  f[b] = f_ext ? f_ext[b] : 0.0;
  f[b + 1] = f_ext ? f_ext[b + 1] : 0.0;
  f[b + 2] = (f_ext ? f_ext[b + 2] : 0.0) - 0.125 * g * s;
}

// dc_e += coef * sum of u_z over the element's nodes (coef = 2 w (-g / 8))
__global__ void k_gravity_sensitivity(Level L, const double* __restrict__ u, double coef, double* __restrict__ dc) {
  const int e = blockIdx.x * kBlock + threadIdx.x;
  if (e >= L.ne) return;
  const int i = e % L.nx, t = e / L.nx, j = t % L.ny, k = t / L.ny;
  double s = 0.0;
  for (int a = 0; a < 8; ++a) {
    const int m = (i + (a & 1)) + L.nxn * ((j + ((a >> 1) & 1)) + L.nyn * (k + (a >> 2)));
    s += u[3ll * m + 2];
  }
  dc[e] += coef * s;
}

// passive elements: 1 = solid (x = 1), 2 = void (x = 0); others unchanged
__global__ void k_apply_passive(long long n, const uint8_t* __restrict__ passive, double* __restrict__ x) {
  const long long e = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n) return;
  const int p = passive[e];
  if (p == 1) x[e] = 1.0;
  else if (p == 2) x[e] = 0.0;
}

// x B^eta of Eqs. 8-9 without the multiplier: s_e = x_e (-dc_e / dv_e)^eta.  The
// usual eta = 1/2 by the square root (of the same value range: 0 at B <= 0 or NaN).
__device__ inline double oc_factor(double xe, double dce, double ve, double eta) {
  double B = -dce / ve;
  B = B > 0.0 ? B : 0.0;
  return xe * (eta == 0.5 ? sqrt(B) : pow(B, eta));
}
// The bracket [lo, hi] of log lambda and its kOcProbes interior points.
__device__ inline double oc_point(double lo, double hi, int p) { return lo + (hi - lo) * (p + 1) / (kOcProbes + 1); }

// Volume at the kOcProbes points of the bracket in st: partial[block][p] =
// sum_e dv_e x_new_e(lambda_p).  The block's sums over its 64 lanes are taken for
// all points at once: in each of five exchanges a lane hands half of its points to its
// partner and keeps the other half, so 32 exchanges do what 32 separate sums do
// in 192.  One pass at 256x128x128 takes 33 us (100 MB read, beside the square root, the
// division and 32 products, clamps and sums per element in binary64), 72 with pow
// for the square root; at 120x56x40 8.6 us (10.9 with one element per thread).
// SQRT: eta = 1/2, without pow's registers (94 instead of 149).
template <bool SQRT>
__global__ __launch_bounds__(kBlock) void k_oc_probe(long long n, const double* __restrict__ x,
                                                     const double* __restrict__ dc, const double* __restrict__ dv,
                                                     double eta, double move, const OcState* __restrict__ st,
                                                     double* __restrict__ partials) {
  static_assert(kOcProbes == 32, "five halvings over the 64 lanes");
  __shared__ double part[kBlock / 64][kOcProbes], lam_pow[kOcProbes];
  if (threadIdx.x < kOcProbes) lam_pow[threadIdx.x] = exp(-eta * oc_point(st->lo, st->hi, threadIdx.x));
  __syncthreads();
  double acc[kOcProbes], lp[kOcProbes];
#pragma unroll
  for (int p = 0; p < kOcProbes; ++p) {
    acc[p] = 0.0;
    // the same in every lane: kept in scalar registers
    const unsigned long long b = (unsigned long long)__double_as_longlong(lam_pow[p]);
    lp[p] = __longlong_as_double(((long long)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
                                 (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b));
  }
  // the next element is requested before this one's 32 points are evaluated
  const long long step = (long long)gridDim.x * kBlock;
  long long e = (long long)blockIdx.x * kBlock + threadIdx.x;
  double xe = 0.0, ve = 0.0, de = 0.0;
  if (e < n) {
    xe = x[e];
    ve = dv[e];
    de = dc[e];
  }
  while (e < n) {
    e += step;
    double xnext = 0.0, vnext = 0.0, dnext = 0.0;
    if (e < n) {
      xnext = x[e];
      vnext = dv[e];
      dnext = dc[e];
    }
    if (ve != 0.0) {  // else outside the volume constraint (passive)
      const double se = oc_factor(xe, de, ve, SQRT ? 0.5 : eta);
      const double lo = fmax(0.0, xe - move), hi = fmin(1.0, xe + move);
#pragma unroll
      for (int p = 0; p < kOcProbes; ++p) acc[p] += ve * fmin(hi, fmax(lo, se * lp[p]));
    }
    xe = xnext;
    ve = vnext;
    de = dnext;
  }
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int h = kOcProbes / 2, m = 32; h >= 1; h >>= 1, m >>= 1) {
    const bool up = lane & m;  // keeps the upper half of its points
#pragma unroll
    for (int p = 0; p < h; ++p) {
      const double give = up ? acc[p] : acc[p + h];
      acc[p] = (up ? acc[p + h] : acc[p]) + __shfl_xor(give, m, 64);
    }
  }
  acc[0] += __shfl_xor(acc[0], 1, 64);
  if (!(lane & 1)) part[w][lane >> 1] = acc[0];  // point: the lane bits 32, 16, ..., 2, highest first
  __syncthreads();
  if (threadIdx.x < kOcProbes) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kBlock / 64; ++q) s += part[q][threadIdx.x];
    partials[(long long)blockIdx.x * kOcProbes + threadIdx.x] = s;
  }
}

// One block of 1024 threads (3 to 6 us; one thread per point took 25, and the host's wait
// for the volumes of every pass another 15): the volumes from the nb partials per point (32
// threads per point, a fixed order), then the bracket narrowed to the points between which
// the volume falls to volfrac.  A non-finite volume at the first point stops the
// update (st->bad).
__global__ __launch_bounds__(1024) void k_oc_narrow(const double* __restrict__ partials, int nb, double volfrac,
                                                    OcState* __restrict__ st) {
  __shared__ double part[32][kOcProbes];
  const int p = threadIdx.x & (kOcProbes - 1), q = threadIdx.x / kOcProbes;
  double s = 0.0;
#pragma unroll 8
  for (int b = q; b < nb; b += 32) s += partials[(long long)b * kOcProbes + p];
  part[q][p] = s;
  __syncthreads();
  if (threadIdx.x >= kOcProbes) return;
  s = 0.0;
#pragma unroll
  for (int r = 0; r < 32; ++r) s += part[r][threadIdx.x];
  const double lo = st->lo, hi = st->hi;
  // points above volfrac up to the first that is not
  const unsigned above = (unsigned)__ballot(s > volfrac);
  const int k = above == 0xffffffffu ? kOcProbes : __ffs(~above) - 1;
  if (threadIdx.x == 0) {
    if (!(fabs(s) < INFINITY)) st->bad = 1.0;
    st->lo = k > 0 ? oc_point(lo, hi, k - 1) : lo;
    st->hi = k < kOcProbes ? oc_point(lo, hi, k) : hi;
  }
}

__global__ void k_oc_start(OcState* __restrict__ st, double lo, double hi) {
  st->lo = lo;
  st->hi = hi;
  st->bad = 0.0;
}

// Number of design elements (passive == 0) per block: count[b].
__global__ __launch_bounds__(kBlock) void k_count_design(long long n, const uint8_t* __restrict__ passive,
                                                         int* __restrict__ count) {
  __shared__ int part[kBlock / 64];
  int c = 0;
  for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < n; e += (long long)gridDim.x * kBlock)
    c += passive[e] == 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
#pragma unroll
    for (int q = 0; q < kBlock / 64; ++q) t += part[q];
    count[blockIdx.x] = t;
  }
}

// dv_e = [passive_e == 0] / (number of design elements); every block sums the
// kReduceBlocks counts itself.
__global__ __launch_bounds__(kBlock) void k_volume_weights(long long n, const uint8_t* __restrict__ passive,
                                                           const int* __restrict__ count, double* __restrict__ dv) {
  __shared__ long long tot;
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int b = 0; b < kReduceBlocks; ++b) t += count[b];
    tot = t;
  }
  __syncthreads();
  const double w = tot > 0 ? 1.0 / (double)tot : 0.0;
  for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < n; e += (long long)gridDim.x * kBlock)
    dv[e] = passive[e] == 0 ? w : 0.0;
}

// x_new at the multiplier in the middle of the bracket, one grid-stride pass; each
// block also writes the largest |x_new - x| and the partial sum of dv x_new over
// its elements to partials[2 b], partials[2 b + 1].
__global__ __launch_bounds__(kBlock) void k_oc_apply(long long n, const double* __restrict__ x,
                                                     const double* __restrict__ dc, const double* __restrict__ dv,
                                                     double eta, double move, const OcState* __restrict__ st,
                                                     double* __restrict__ xn, double* __restrict__ partials) {
  if (st->bad != 0.0) return;
  __shared__ double part[kBlock / 64][2];
  const double lam_pow = exp(-eta * (0.5 * (st->lo + st->hi)));
  double ch = 0.0, vol = 0.0;
  for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < n; e += (long long)gridDim.x * kBlock) {
    const double xe = x[e], ve = dv[e];
    double y = xe;  // outside the volume constraint: left to the caller (passive)
    if (ve != 0.0) {
      const double se = oc_factor(xe, dc[e], ve, eta);
      y = fmin(fmin(1.0, xe + move), fmax(fmax(0.0, xe - move), se * lam_pow));
    }
    xn[e] = y;
    ch = fmax(ch, fabs(y - xe));
    vol += ve * y;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    ch = fmax(ch, __shfl_down(ch, off, 64));
    vol += __shfl_down(vol, off, 64);
  }
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    part[w][0] = ch;
    part[w][1] = vol;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double c = 0.0, v = 0.0;
#pragma unroll
    for (int q = 0; q < kBlock / 64; ++q) {
      c = fmax(c, part[q][0]);
      v += part[q][1];
    }
    partials[2ll * blockIdx.x] = c;
    partials[2ll * blockIdx.x + 1] = v;
  }
}

// One block of kBlock threads: the largest change, dv . x_new (a fixed order) and
// the multiplier into st.
__global__ __launch_bounds__(kBlock) void k_oc_finish(const double* __restrict__ partials, int nb,
                                                      OcState* __restrict__ st) {
  __shared__ double part[kBlock / 64][2];
  double c = 0.0, v = 0.0;
  for (int b = threadIdx.x; b < nb; b += kBlock) {
    c = fmax(c, partials[2 * b]);
    v += partials[2 * b + 1];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    c = fmax(c, __shfl_down(c, off, 64));
    v += __shfl_down(v, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    part[threadIdx.x >> 6][0] = c;
    part[threadIdx.x >> 6][1] = v;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  c = v = 0.0;
#pragma unroll
  for (int q = 0; q < kBlock / 64; ++q) {
    c = fmax(c, part[q][0]);
    v += part[q][1];
  }
  st->change = c;
  st->volume = v;
  st->lambda = exp(0.5 * (st->lo + st->hi));
}

}  // namespace

namespace {
// The tiled filter of half-width R = 1..kFilterMaxR; false where the general
// kernel is to be taken (other half-widths; launch grids past the y and z
// limits, which it refuses).  zchunk: enough blocks for four per compute unit
// (1024), at most 32 planes, so that a block repeats 2R of its planes at the
// most where there are blocks to spare, and at least 4.
template <int MODE>
bool launch_filter_tile(int nx, int ny, int nz, double rmin, double gamma, const double* x, const double* in,
                        double* out, hipStream_t s) {
  const int R = (int)std::ceil(rmin) - 1;
  if (R < 1 || R > kFilterMaxR || ny > 65535 || nz > 65535) return false;
  FilterWeights fw{};
  const int ncls = R == 1 ? FilterClasses<1>::n : (R == 2 ? FilterClasses<2>::n : FilterClasses<3>::n);
  for (int dk = 0; dk <= R; ++dk)
    for (int c = 0; c < ncls; ++c) {
      fw.w[dk][c] = rmin - std::sqrt((double)(dk * dk + FilterClasses<kFilterMaxR>::d2(c)));
      if (fw.w[dk][c] > 0.0) fw.n[dk] = c + 1;
    }
  const long long tiles = (long long)((nx + 31) / 32) * ((ny + 7) / 8);
  const int zchunk = (int)std::max(4ll, std::min(32ll, nz * tiles / 1024));
  const dim3 grid((nx + 31) / 32, (ny + 7) / 8, (nz + zchunk - 1) / zchunk);
  if (R == 1)
    k_filter_tile<MODE, 1><<<grid, 256, 0, s>>>(nx, ny, nz, zchunk, fw, gamma, x, in, out);
  else if (R == 2)
    k_filter_tile<MODE, 2><<<grid, 256, 0, s>>>(nx, ny, nz, zchunk, fw, gamma, x, in, out);
  else
    k_filter_tile<MODE, 3><<<grid, 256, 0, s>>>(nx, ny, nz, zchunk, fw, gamma, x, in, out);
  return true;
}
}  // namespace

void launch_filter(int nx, int ny, int nz, double rmin, int adjoint, const double* in, double* out, double* tmp,
                   hipStream_t s) {
  if (adjoint ? launch_filter_tile<2>(nx, ny, nz, rmin, 0.0, nullptr, in, out, s)
              : launch_filter_tile<0>(nx, ny, nz, rmin, 0.0, nullptr, in, out, s))
    return;
  const int R = (int)std::ceil(rmin) - 1;
  const int bx = 64;
  dim3 grid((nx + bx - 1) / bx, ny, nz);
  if (adjoint) {
    k_filter<1><<<grid, bx, 0, s>>>(nx, ny, nz, rmin, R, in, tmp);
    k_filter<2><<<grid, bx, 0, s>>>(nx, ny, nz, rmin, R, tmp, out);
  } else {
    k_filter<0><<<grid, bx, 0, s>>>(nx, ny, nz, rmin, R, in, out);
  }
}

// Scratch of the adjoint filter for callers that cannot allocate: in / Hs for
// up to kFilterScratchElems elements.  Each device holds its own copy for the
// life of the process; its device address is looked up once per device (the
// array's name is a host-side stand-in and is never passed to a kernel).
__device__ __align__(256) double scratch[kFilterScratchElems];

int filter_scratch_ptr(double** ptr) {
  static std::mutex mu;
  static std::vector<double*> addr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  std::lock_guard<std::mutex> lock(mu);
  if ((int)addr.size() <= dev) addr.resize(dev + 1, nullptr);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    addr[dev] = static_cast<double*>(p);
  }
  *ptr = addr[dev];
  return 0;
}

void launch_sens_filter(int nx, int ny, int nz, double rmin, double gamma, const double* x, const double* dc,
                        double* out, hipStream_t s) {
  if (launch_filter_tile<3>(nx, ny, nz, rmin, gamma, x, dc, out, s)) return;
  const int R = (int)std::ceil(rmin) - 1;
  const int bx = 64;
  k_sens_filter<<<dim3((nx + bx - 1) / bx, ny, nz), bx, 0, s>>>(nx, ny, nz, rmin, R, gamma, x, dc, out);
}

void launch_gravity_load(const Level& L, const double* rho, double g, const double* f_ext, double* f,
                         hipStream_t s) {
  k_gravity_load<<<(L.nn + kBlock - 1) / kBlock, kBlock, 0, s>>>(L, rho, g, f_ext, f);
}

void launch_gravity_sensitivity(const Level& L, const double* u, double coef, double* dc, hipStream_t s) {
  k_gravity_sensitivity<<<(L.ne + kBlock - 1) / kBlock, kBlock, 0, s>>>(L, u, coef, dc);
}

void launch_apply_passive(long long n, const uint8_t* passive, double* x, hipStream_t s) {
  k_apply_passive<<<(int)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(n, passive, x);
}

void launch_volume_weights(long long n, const uint8_t* passive, int* count, double* dv, hipStream_t s) {
  k_count_design<<<kReduceBlocks, kBlock, 0, s>>>(n, passive, count);
  k_volume_weights<<<kReduceBlocks, kBlock, 0, s>>>(n, passive, count, dv);
}

void launch_oc_update(long long n, const double* x, const double* dc, const double* dv, double volfrac, double eta,
                      double move, double lo, double hi, int passes, double* xn, double* partials, OcState* st,
                      hipStream_t s) {
  const int nb = (int)std::min<long long>(kReduceBlocks, (n + kBlock - 1) / kBlock);
  // a probe's thread takes four elements or more: its 32 sums over the block, and
  // their partials in the next launch, cost more than an element
  const int np = (int)std::min<long long>(kReduceBlocks, (n + 4 * kBlock - 1) / (4 * kBlock));
  k_oc_start<<<1, 1, 0, s>>>(st, lo, hi);
  for (int k = 0; k < passes; ++k) {
    if (eta == 0.5)
      k_oc_probe<true><<<np, kBlock, 0, s>>>(n, x, dc, dv, eta, move, st, partials);
    else
      k_oc_probe<false><<<np, kBlock, 0, s>>>(n, x, dc, dv, eta, move, st, partials);
    k_oc_narrow<<<1, 1024, 0, s>>>(partials, np, volfrac, st);
  }
  k_oc_apply<<<nb, kBlock, 0, s>>>(n, x, dc, dv, eta, move, st, xn, partials);
  k_oc_finish<<<1, kBlock, 0, s>>>(partials, nb, st);
}

}  // namespace hexmg
