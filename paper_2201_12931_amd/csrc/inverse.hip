// Exact inverse of the dense coarsest operator (SPD, binary64), which the
// V-cycle applies as a product (Alg. 3 solves the coarsest grid directly).
//
// Block sweeps.  Sweeping the pivot block K of a symmetric matrix replaces
//   A_KK <- -D,  A_IK <- A_IK D,  A_IJ <- A_IJ - A_IK D A_KJ,   D = A_KK^-1,
// and keeps it symmetric; swept over every pivot block it is -A^-1.  The
// diagonal blocks met on the way are SPD, so no pivoting is needed.  Only the
// 64x64 tiles (I, J) with I >= J are kept, so a step does half the tiles of a
// Gauss-Jordan step on the full matrix.
//
// The operator couples tiles up to wb apart, and sweeping pivots from the top
// fills only the tiles up to row K + wb (from the bottom: down to row K - wb).  So
// while K' - K > wb a step sweeps two pivots, K from the top and K' from the
// bottom: A_KK' is still zero, and D of the two together is block diagonal.  It
// leaves alone what neither reaches.  The wb + 1 pivots at most that are left between
// them, and then the last two tiles' pivots, are swept one to a step on all tiles.
//
// Why the last two tiles wait: the pivot swept last is the whole structure condensed onto
// its block, the softest and least accurate one.  Ending between the two fronts cost
// digits on slender grids, whose blocks are whole rows of nodes along the length: the
// inverse was 37 times (20x1x2 elements), 26 (24x1x2) and 4 times (20x2x2) as far from
// the exact one as in the natural order (geometric means over 12 to 14 densities, with the
// 64 terms of an update added one by one); ending at the last tiles, as the natural order
// does, and summing the terms on their own, 0.86, 1.4 and 1.2 times, and 0.78 over
// 213 designs on 16 grid shapes.  It costs one step at most.
//
// A step on few tiles is bound by its serial chain (launch, one round of loads, two
// 64^3 products at the binary64 matrix rate, the next pivot tile's inverse: 18 us, the
// inverse 8 of them), one on many by the products.  Measured, pack to unpack: 675
// unknowns (wb = 3) 158 us in 8 steps, 1911 (5) 401 us in 19, 2304 (7) 521 us in 23; in order
// on all tiles 205, 714 and 885 us in 11, 30 and 36 steps (and 290, 1960 and 2200 us as a
// full Gauss-Jordan whose tiles took three rounds of loads).
//
// Layouts.  v_mfma_f64_16x16x4f64: lane l holds the left operand's (row l%16, k
// l/16), the right operand's (k l/16, column l%16), and of the result, value v,
// (row 4v + l/16, column l%16).  The result's layout is that of a right operand
// with k = 4v + l/16, so X = D A_KJ feeds y -= A_IK X from the registers it was
// formed in.  Storage follows:
//   tiles (result order):   T[w][t][v][l]  = element (16t + 4v + l/16, 16w + l%16),
//   pivot columns and pivot inverses (operand order): P[r][ks][l] = element
//     (16r + l%16, 4ks + l/16); the same order serves as left operand and, transposed, as
//     right operand,
// so every load of a wave is contiguous and conflict-free in LDS.
#include <algorithm>

#include "hexmg_impl.h"

namespace hexmg {

namespace {

constexpr int kTile = kGJBlock * kGJBlock;  // elements of a tile
constexpr int kLastPivots = 2;  // tiles whose pivots are swept after all others
typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

// index of the tile (I, J), I >= J, in the packed lower triangle
__host__ __device__ inline long long tri(int I, int J) { return ((long long)I * (I + 1) / 2 + J) * kTile; }

// Inverse of a symmetric positive 2x2 block.  1/det from the hardware reciprocal
// r: with e = 1 - det r, 1/det = r (1 + e + e^2) up to e^3 (below 2^-60), applied
// to the products with r, which do not wait for it -- the shortest chain here.
__device__ inline void inv2(double a00, double a01, double a11, double (&q)[3]) {
  const double det = a00 * a11 - a01 * a01;
  const double r = __builtin_amdgcn_rcp(det);
  const double e = fma(-det, r, 1.0);
  const double e2 = fma(e, e, e);
  const double t00 = a11 * r, t01 = -a01 * r, t11 = a00 * r;
  q[0] = fma(t00, e2, t00);
  q[1] = fma(t01, e2, t01);
  q[2] = fma(t11, e2, t11);
}

// z = P^-1 x for a symmetric positive 4x4 block P, by the Schur complement of its
// leading 2x2 block: forward and back substitution run beside the inverses, so
// only what follows the second reciprocal adds to the chain.
__device__ inline void solve4(const double (&p)[4][4], const double (&x)[4], double (&z)[4]) {
  double ai[3], si[3];
  inv2(p[0][0], p[0][1], p[1][1], ai);
  // X = A^-1 B, u = A^-1 x_top
  const double x00 = ai[0] * p[0][2] + ai[1] * p[1][2], x01 = ai[0] * p[0][3] + ai[1] * p[1][3];
  const double x10 = ai[1] * p[0][2] + ai[2] * p[1][2], x11 = ai[1] * p[0][3] + ai[2] * p[1][3];
  const double u0 = ai[0] * x[0] + ai[1] * x[1], u1 = ai[1] * x[0] + ai[2] * x[1];
  inv2(fma(-p[1][2], x10, fma(-p[0][2], x00, p[2][2])), fma(-p[1][2], x11, fma(-p[0][2], x01, p[2][3])),
       fma(-p[1][3], x11, fma(-p[0][3], x01, p[3][3])), si);
  const double w0 = fma(-p[1][2], u1, fma(-p[0][2], u0, x[2])), w1 = fma(-p[1][3], u1, fma(-p[0][3], u0, x[3]));
  z[2] = fma(si[0], w0, si[1] * w1);
  z[3] = fma(si[1], w0, si[2] * w1);
  z[0] = fma(-x01, z[3], fma(-x00, z[2], u0));
  z[1] = fma(-x11, z[3], fma(-x10, z[2], u1));
}

struct InverseLds {
  double row[2][4][256];  // by parity and wave: the tile of the pivot row in its column block
  double Q[256];
  double pr[2][16][4];    // 4x4 pivot rows, by parity and column
};

// Inverse of the SPD 64x64 tile y (result order: wave w holds the column block w),
// written to D in operand order: sweeps of four 16x16 pivot blocks s.
//   Q = M_ss^-1      one element per thread, by sweeps of four 4x4 pivots (solve4):
//                    a_ij <- a_ij - c_i P^-1 x_j, with x_j = e_j for a pivot column j and c_i = e_i
//                    for a pivot row i;
//   W_J = Q M_sJ     wave J: its own tile y[s] is the right operand;
//   M_IJ -= M_Is W_J, the left operand M_Is = M_sI^T being wave I's y[s] as it lies in LDS;
//   M_sJ <- W_J, M_Is <- M_Is Q (wave s), M_ss <- -Q.
// Each 16-wide step takes six barriers and about 2.5 us; the serial 4x4 chain (two
// reciprocals, about 20 dependent operations) is what bounds it.
__device__ inline void invert_tile(InverseLds& lds, d4 (&y)[4], double* __restrict__ D) {
  static_assert(kGJBlock == 64 && kBlock == 256, "four waves, 16x16 pivot blocks");
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  const int ti = t >> 4, tj = t & 15;  // element of the 16x16 pivot block
  // y[i] holds block row (s + i) % 4: the pivot row is always y[0], and the code
  // stays one loop body (unrolled, its fetches are the longer part)
#pragma unroll 1
  for (int s = 0; s < 4; ++s) {
    double(*row)[256] = lds.row[s & 1];
#pragma unroll
    for (int v = 0; v < 4; ++v) row[w][v * 64 + l] = y[0][v];
    __syncthreads();
    double a = row[s][t];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int kb = 4 * m, hy = ti - kb, hx = tj - kb;
      const bool rowk = hy >= 0 && hy < 4, colk = hx >= 0 && hx < 4;
      double(*pr)[4] = lds.pr[m & 1];
      if (rowk) pr[tj][hy] = a;
      __syncthreads();
      double pk[4][4], x[4], c[4], z[4];
#pragma unroll
      for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int g = 0; g < 4; ++g) pk[h][g] = pr[kb + g][h];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        x[g] = colk ? (hx == g ? 1.0 : 0.0) : pr[tj][g];
        c[g] = rowk ? (hy == g ? 1.0 : 0.0) : pr[ti][g];
      }
      solve4(pk, x, z);
      const double d = fma(c[1], z[1], c[0] * z[0]) + fma(c[3], z[3], c[2] * z[2]);
      a = rowk != colk ? d : (rowk ? -d : a - d);
    }
    lds.Q[t] = -a;
    __syncthreads();
    double Q[4];
    d4 W = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int v = 0; v < 4; ++v) Q[v] = lds.Q[v * 64 + l];
    if (w != s) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) W = __builtin_amdgcn_mfma_f64_16x16x4f64(Q[ks], y[0][ks], W, 0, 0, 0);
    } else {  // M_Is Q: the product below with -Q for W and nothing to subtract from
#pragma unroll
      for (int v = 0; v < 4; ++v) W[v] = -Q[v];
#pragma unroll
      for (int i = 1; i < 4; ++i) y[i] = d4{0.0, 0.0, 0.0, 0.0};
    }
    d4 z[3];  // summed on their own, as in sweep_tile
#pragma unroll
    for (int i = 0; i < 3; ++i) z[i] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < 3; ++i)
        z[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(row[(s + i + 1) & 3][ks * 64 + l], W[ks], z[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 3; ++i) y[i] = y[i + 1] - z[i];
    y[3] = W;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v) D[w * 1024 + (4 * r + v) * 64 + l] = -y[r][v];
}

// The pivots of a step: K[0] from the top and K[1] from the bottom; or K[0] alone
// (K[1] = -1), which then reaches every tile.  Both -1: no step.
struct Pivots {
  int K[2];
  __host__ __device__ int of(int side) const { return side ? K[1] : K[0]; }
};
// Whether a pivot of side 0 or 1 changes row (or column) block I.
__device__ inline bool reaches(const Pivots& p, int side, int wb, int I) {
  const int K = p.of(side);
  return K >= 0 && (p.K[1] < 0 || (side == 0 ? I <= K + wb : I >= K - wb));
}

// What the next step (pivots q) reads of a tile after its last change: tiles of a
// pivot column K go to its panel P (operand order; of a tile (K, J) its transpose),
// a pivot tile's inverse to D.  Panels and inverses of side 1 follow those of side 0.
__device__ inline void hand_over(InverseLds& s, const Pivots& q, int nt, int I, int J, d4 (&y)[4],
                                 double* __restrict__ P, double* __restrict__ D) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {  // at most one side is this tile's pivot
    const int K = q.of(side);
    if (K < 0) continue;  // uniform per block, as is what follows
    double* Ps = P + (long long)side * nt * kTile;
    if (I == K && J == K) {
      invert_tile(s, y, D + side * kTile);
      return;
    }
    if (I == K) {
      double* p = Ps + (long long)J * kTile + w * 1024 + l;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) p[(4 * t + v) * 64] = y[t][v];
    } else if (J == K) {
      double* p = Ps + (long long)I * kTile + (4 * w + ((l >> 2) & 3)) * 64 + (l & 3) * 16 + (l >> 4);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) p[t * 1024 + 4 * v] = y[t][v];
    }
  }
}

// The lower triangle of the row-major A (n x n) as tiles, padded by the identity
// to whole tiles; the panels and pivot inverses of the first step (q).  One block per tile.
__global__ __launch_bounds__(kBlock) void k_sweep_pack(int n, int nt, Pivots q, const double* __restrict__ A,
                                                       double* __restrict__ T, double* __restrict__ P,
                                                       double* __restrict__ D) {
  __shared__ InverseLds lds;
  int I = 0;
  const int b = blockIdx.x;
  while ((I + 1) * (I + 2) / 2 <= b) ++I;
  const int J = b - I * (I + 1) / 2;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  d4 y[4];
  double* tile = T + tri(I, J) + w * 1024 + l;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = I * kGJBlock + 16 * t + 4 * v + (l >> 4), j = J * kGJBlock + 16 * w + (l & 15);
      y[t][v] = (i < n && j < n) ? A[(long long)i * n + j] : (i == j ? 1.0 : 0.0);
    }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) tile[(4 * t + v) * 64] = y[t][v];
  hand_over(lds, q, nt, I, J, y, P, D);
}

struct SweepOperands {
  double op[2][kTile];  // D and A_IK in operand order
};

// The change of the tile (I, J), I >= J, by the pivot K: y <- y - A_IK D A_KJ, or
// (I = K or J = K) y <- its new value.  P: the pivot column's panel.
__device__ __forceinline__ void sweep_tile(SweepOperands& lds, int K, int I, int J, const double* __restrict__ P,
                                           const double* __restrict__ D, d4 (&y)[4]) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (I == K && J == K) {  // -D: row-major position (r, c) of the symmetric D in operand order
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) y[t][v] = -D[w * 1024 + (4 * t + v) * 64 + l];
    return;
  }
  // every global load is issued before the first use
  constexpr int kPairs = kTile / kBlock / 2;
  const d2 *gd = (const d2*)D + threadIdx.x, *gi = (const d2*)(P + (long long)I * kTile) + threadIdx.x;
  const double* gj = (J == K ? D : P + (long long)J * kTile) + w * 1024 + l;
  d2 vd[kPairs], vi[kPairs];
  double r[16];  // A_KJ (columns 16w..16w+15), or D where J = K
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) r[ks] = gj[ks * 64];
  if (J != K) {
#pragma unroll
    for (int m = 0; m < kPairs; ++m) vd[m] = gd[m * kBlock];
  }
  if (I != K) {
#pragma unroll
    for (int m = 0; m < kPairs; ++m) vi[m] = gi[m * kBlock];
  }
  if (I == K || J == K) {
#pragma unroll
    for (int t = 0; t < 4; ++t) y[t] = d4{0.0, 0.0, 0.0, 0.0};
  }
  if (J != K) {
#pragma unroll
    for (int m = 0; m < kPairs; ++m) ((d2*)lds.op[0])[threadIdx.x + m * kBlock] = vd[m];
  }
  if (I != K) {
#pragma unroll
    for (int m = 0; m < kPairs; ++m) ((d2*)lds.op[1])[threadIdx.x + m * kBlock] = vi[m];
  }
  __syncthreads();
  d4 x[4];  // X = D A_KJ, or -D where J = K
  if (J == K) {
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) x[ks >> 2][ks & 3] = -r[ks];
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t) x[t] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        x[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(lds.op[0][t * 1024 + ks * 64 + l], r[ks], x[t], 0, 0, 0);
  }
  if (I == K) {
#pragma unroll
    for (int t = 0; t < 4; ++t) y[t] = x[t];
  } else {
    // the 64 terms are summed on their own: added one by one to an element much larger than
    // they are, each would round at its size
    d4 z[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) z[t] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        z[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(lds.op[1][t * 1024 + ks * 64 + l], x[ks >> 2][ks & 3], z[t], 0, 0,
                                                    0);
#pragma unroll
    for (int t = 0; t < 4; ++t) y[t] -= z[t];
  }
}

// Sweep of the pivots p, one block per tile (I, J), I >= J, in place (a tile is
// read and written by its own block only; the pivot columns are read from the
// panels P that the previous step left), and what the next step (pivots q) reads
// of the tiles that it reaches.  The first blocks take the next pivot tiles: their
// inverses are the serial part of the step (every other block needs them in the next
// one) and so start first and run beside the other tiles.
__global__ __launch_bounds__(kBlock) void k_sweep_step(int nt, int wb, Pivots p, Pivots q, double* __restrict__ T,
                                                       const double* __restrict__ P, const double* __restrict__ D,
                                                       double* __restrict__ Pn, double* __restrict__ Dn) {
  __shared__ union Lds {
    SweepOperands op;
    InverseLds inv;
    __device__ Lds() {}
  } lds;
  int b = blockIdx.x;
  if (q.K[0] >= 0) {  // the next pivot tiles' places in row order, the first of them before the second
    const int p0 = q.K[0] * (q.K[0] + 3) / 2, p1 = q.K[1] >= 0 ? q.K[1] * (q.K[1] + 3) / 2 : -1;
    if (b == 0) {
      b = p0;
    } else if (p1 < 0) {
      b = b <= p0 ? b - 1 : b;
    } else if (b == 1) {
      b = p1;
    } else {
      b = b - 2 < p0 ? b - 2 : (b - 1 < p1 ? b - 1 : b);
    }
  }
  int I = (int)((sqrtf(8.0f * (float)b + 1.0f) - 1.0f) * 0.5f);
  while ((I + 1) * (I + 2) / 2 <= b) ++I;
  while (I * (I + 1) / 2 > b) --I;
  const int J = b - I * (I + 1) / 2;
  bool change = false, hand = false;  // uniform per block
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    change = change || (reaches(p, side, wb, I) && reaches(p, side, wb, J));
    hand = hand || ((I == q.of(side) || J == q.of(side)) && reaches(q, side, wb, I) && reaches(q, side, wb, J));
  }
  if (!change && !hand) return;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  double* tile = T + tri(I, J) + w * 1024 + l;
  d4 y[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) y[t][v] = tile[(4 * t + v) * 64];
  bool used = false;
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {
    if (!(reaches(p, side, wb, I) && reaches(p, side, wb, J))) continue;
    if (used) __syncthreads();  // the operands' readers are done with the LDS
    sweep_tile(lds.op, p.of(side), I, J, P + (long long)side * nt * kTile, D + side * kTile, y);
    used = true;
  }
  if (change) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) tile[(4 * t + v) * 64] = y[t][v];
  }
  if (hand) {
    if (used && I == J) __syncthreads();  // as above, before a pivot tile's inverse
    hand_over(lds.inv, q, nt, I, J, y, Pn, Dn);
  }
}

// The inverse, row-major and exactly symmetric, from the swept tiles: B = -T, the
// upper triangle mirrored through LDS.  One block per tile.
__global__ __launch_bounds__(kBlock) void k_sweep_unpack(int n, const double* __restrict__ T,
                                                         double* __restrict__ B) {
  __shared__ double m[kGJBlock][kGJBlock + 1];
  int I = 0;
  const int b = blockIdx.x;
  while ((I + 1) * (I + 2) / 2 <= b) ++I;
  const int J = b - I * (I + 1) / 2;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double* tile = T + tri(I, J) + w * 1024 + l;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) m[16 * t + 4 * v + (l >> 4)][16 * w + (l & 15)] = -tile[(4 * t + v) * 64];
  __syncthreads();
  const int i0 = I * kGJBlock, j0 = J * kGJBlock;
#pragma unroll
  for (int p = 0; p < kGJBlock / 4; ++p) {
    const int r = 4 * p + w;  // rows of the tile, then rows of its mirror image
    if (i0 + r < n && j0 + l < n) B[(long long)(i0 + r) * n + j0 + l] = (I != J || l <= r) ? m[r][l] : m[l][r];
    if (I != J && j0 + r < n && i0 + l < n) B[(long long)(j0 + r) * n + i0 + l] = m[l][r];
  }
}

}  // namespace

size_t spd_inverse_scratch(int n) {
  const long long nt = (n + kGJBlock - 1) / kGJBlock;
  return (size_t)(tri((int)nt, 0) + 2 * (2 * nt + 2) * kTile);
}

void launch_spd_inverse(int n, int band, double* A, double* scratch, hipStream_t s) {
  const int nt = (n + kGJBlock - 1) / kGJBlock, tiles = nt * (nt + 1) / 2;
  const int wb = (band + kGJBlock - 1) / kGJBlock;
  double* T = scratch;
  double* P[2] = {T + tri(nt, 0), T + tri(nt, 0) + 2ll * nt * kTile};  // by parity, then side
  double* D[2] = {P[1] + 2ll * nt * kTile, P[1] + (2ll * nt + 2) * kTile};
  // pivots lo and hi while they are not coupled, then what is left between them in
  // order, then the last tiles
  int lo = 0, rest = std::max(nt - kLastPivots, 0), hi = rest - 1;
  auto next = [&]() -> Pivots {
    if (lo <= hi) return Pivots{{lo, hi - lo > wb ? hi : -1}};
    return Pivots{{rest < nt ? rest : -1, -1}};
  };
  Pivots p = next();
  k_sweep_pack<<<tiles, kBlock, 0, s>>>(n, nt, p, A, T, P[0], D[0]);
  for (int k = 0; p.K[0] >= 0; ++k) {
    if (lo <= hi) {
      ++lo;
      if (p.K[1] >= 0) --hi;
    } else {
      ++rest;
    }
    const Pivots q = next();
    k_sweep_step<<<tiles, kBlock, 0, s>>>(nt, wb, p, q, T, P[k & 1], D[k & 1], P[(k + 1) & 1], D[(k + 1) & 1]);
    p = q;
  }
  k_sweep_unpack<<<tiles, kBlock, 0, s>>>(n, T, A);
}

}  // namespace hexmg
