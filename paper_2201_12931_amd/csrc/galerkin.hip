// Galerkin coarse operators (Eq. 23): A_{l+1} = P~^T A_l P~ + (I - M_{l+1}),
// P~ = M_l P M_{l+1}, as an alternative to the re-discretized coarse levels.
//
// A Galerkin level is stored as its 27-point block stencil, of which the operator's
// symmetry needs half: for node n and the neighbour offsets o = (dz+1)*9 +
// (dy+1)*3 + (dx+1) >= 13 (the centre and the 13 that follow it), the 3x3 block
// A(3n+ci, 3(n+o)+cj) at S[(9*(o-13) + 3*ci + cj) * nn + n] (coefficient-major, so
// a wave reading one coefficient of 64 consecutive nodes is coalesced).  The
// block of an offset o < 13 is the transpose of what node n+o holds at 26-o.  The
// stencil already holds the supports: zero rows and columns at fixed DOFs and
// a unit diagonal there, so applying it needs no masking.
//
// Level 1 is built from the matrix-free level 0.  Every fine element lies in
// one coarse element and is one of its eight children c, so
//   P~^T (M K M) P~ = sum over coarse elements of sum_c E_c G_c,
// G_c = P_c^T K0 P_c (24x24, constant, computed on the host), except where a
// child touches a fixed fine DOF: there the masked product is formed on the
// fly (the nodes concerned are listed once per grid).  Deeper levels take the
// triple product of the stencils, axis by axis.
//
// Storage of the binary32 V-cycle's stencils: binary32, or 16 bits per
// coefficient (half the bytes of the HBM-bound stencil sweep).  bfloat16 keeps
// binary32's exponent range; binary16 keeps 3 more significand bits but not the
// range (the coefficients span Emin..E0 times 2^l), so each stored 3x3 block is
// scaled by a power of two of its own that brings the largest magnitude in it
// into [2^14, 2^15), and the sweep applies 2^-s to the products with the block.  (One
// power per node is not enough: a block is read by both nodes that it couples, and
// under the scale of a stiff node its blocks towards a soft one -- the soft one's
// largest -- lie in binary16's subnormals: off by 1.6e-3 of the soft node's largest
// coefficient at Emin / E0 = 1e-9, by 0.45 at 1e-12, against 5e-4 by block.)  Both are
// rounded to nearest from the binary64 stencil (bfloat16 through binary32).
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include <utility>

#include "hexmg_impl.h"
#include "node_ops.h"

namespace hexmg {

namespace {

__device__ inline int off_dx(int o) { return o % 3 - 1; }
__device__ inline int off_dy(int o) { return (o / 3) % 3 - 1; }
__device__ inline int off_dz(int o) { return o / 9 - 1; }

// 1-D trilinear weight of coarse corner a (0/1) at fine offset t (0..2) inside a coarse element
__device__ inline double wt(int t, int a) {
  return a == 0 ? (t == 0 ? 1.0 : (t == 1 ? 0.5 : 0.0)) : (t == 2 ? 1.0 : (t == 1 ? 0.5 : 0.0));
}

// Writes the 3x3 block (m, m + o), o >= 13, with the coarse supports applied.
__device__ inline void store_block(const Level& C, int m, int m2, int o, const double (&blk)[9], double* S64,
                                   float* S32) {
  const int mk = C.mask[m], mk2 = m2 >= 0 ? C.mask[m2] : 7;
#pragma unroll
  for (int ci = 0; ci < 3; ++ci)
#pragma unroll
    for (int cj = 0; cj < 3; ++cj) {
      double v = (((mk >> ci) & 1) || ((mk2 >> cj) & 1)) ? 0.0 : blk[3 * ci + cj];
      if (o == 13 && ci == cj && ((mk >> ci) & 1)) v = 1.0;
      const long long idx = (long long)(9 * (o - 13) + 3 * ci + cj) * C.nn + m;
      S64[idx] = v;
      if (S32) S32[idx] = (float)v;  // absent when the binary32 V-cycle reads 16-bit coefficients
    }
}

// Level-1 nodes with a fixed fine DOF in their support: flag[m], and their list
// (in any order; *count of them, zeroed by the caller).
__global__ void k_galerkin_flag(Level F, Level C, uint8_t* __restrict__ flag, int* __restrict__ list,
                                int* __restrict__ count) {
  const int m = blockIdx.x * kBlock + threadIdx.x;
  if (m >= C.nn) return;
  int I, J, K, fixed = 0;
  node_coords(C, m, I, J, K);
  for (int dz = -2; dz <= 2; ++dz)
    for (int dy = -2; dy <= 2; ++dy)
      for (int dx = -2; dx <= 2; ++dx) {
        const int i = 2 * I + dx, j = 2 * J + dy, k = 2 * K + dz;
        if (i >= 0 && i < F.nxn && j >= 0 && j < F.nyn && k >= 0 && k < F.nzn) fixed |= F.mask[i + F.nxn * (j + F.nyn * k)];
      }
  flag[m] = fixed != 0;
  if (fixed) list[atomicAdd(count, 1)] = m;
}

// Element pairs (a, b = a + offset) of the stored offsets before o.
constexpr int pairs_before(int o) {
  int n = 0;
  for (int p = 13; p < o; ++p)
    n += (2 - (p % 3 == 1 ? 0 : 1)) * (2 - ((p / 3) % 3 == 1 ? 0 : 1)) * (2 - (p / 9 == 1 ? 0 : 1));
  return n;
}
typedef const __attribute__((address_space(4))) double* ConstPtr;  // read by scalar loads
// The block (m, m + O) from the 4x4x4 fine moduli around m.
template <int O>
__device__ __forceinline__ void first_block(const Level& C, const double (&Ee)[4][4][4], ConstPtr& Gp, int m,
                                            int I, int J, int K, double* S64, float* S32) {
  constexpr int dx = O % 3 - 1, dy = (O / 3) % 3 - 1, dz = O / 9 - 1;
  double blk[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  int pair = pairs_before(O);
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int ax = a & 1, ay = (a >> 1) & 1, az = a >> 2;
    if (ax + dx < 0 || ax + dx > 1 || ay + dy < 0 || ay + dy > 1 || az + dz < 0 || az + dz > 1) continue;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      // 36 coefficients at a time: hoisted, they would spill the scalar registers
      if ((c & 3) == 0)
        asm volatile("" : "+s"(Gp), "+v"(blk[0]), "+v"(blk[1]), "+v"(blk[2]), "+v"(blk[3]), "+v"(blk[4]), "+v"(blk[5]),
                     "+v"(blk[6]), "+v"(blk[7]), "+v"(blk[8]));
      const double e = Ee[2 - 2 * az + (c >> 2)][2 - 2 * ay + ((c >> 1) & 1)][2 - 2 * ax + (c & 1)];
#pragma unroll
      for (int q = 0; q < 9; ++q) blk[q] += e * Gp[(pair * 8 + c) * 9 + q];
    }
    ++pair;
  }
  const int I2 = I + dx, J2 = J + dy, K2 = K + dz;
  const bool in = I2 >= 0 && I2 < C.nxn && J2 >= 0 && J2 < C.nyn && K2 < C.nzn;
  store_block(C, m, in ? I2 + C.nxn * (J2 + C.nyn * K2) : -1, O, blk, S64, S32);
}
template <int... O>
__device__ __forceinline__ void first_blocks(std::integer_sequence<int, O...>, const Level& C,
                                             const double (&Ee)[4][4][4], ConstPtr& Gp, int m, int I, int J, int K,
                                             double* S64, float* S32) {
  (first_block<13 + O>(C, Ee, Gp, m, I, J, K, S64, S32), ...);
}

// The level-1 stencil at the nodes without fixed fine DOFs around them, one thread
// per node: its 4x4x4 fine moduli are read once, and every block is a sum over
// the coarse elements that hold both nodes (corners a, b of one of them) and
// their eight children, blk += E_c G_c[a, b].  Gp holds G_c by (a, b, c) in the
// order the unrolled loops take it (uniform indices: scalar loads).  2592
// multiply-adds per node, below the time of writing 126 coefficients in two
// precisions, which bounds the pass.  Level 1 of 256x128x128: 0.27 ms, and 0.14
// ms for the 8450 nodes listed next to the supports (2.3 ms together as one
// thread per block that read its moduli and supports child by child).
__global__ __launch_bounds__(kBlock) void k_galerkin_first(Level F, Level C, const double* __restrict__ E,
                                                           const double* Gp, const uint8_t* __restrict__ flag,
                                                           double* __restrict__ S64, float* __restrict__ S32) {
  const int m = blockIdx.x * kBlock + threadIdx.x;
  if (m >= C.nn || flag[m]) return;
  int I, J, K;
  node_coords(C, m, I, J, K);
  double Ee[4][4][4];
#pragma unroll
  for (int z = 0; z < 4; ++z)
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int i = 2 * I - 2 + x, j = 2 * J - 2 + y, k = 2 * K - 2 + z;
        const bool in = i >= 0 && i < F.nx && j >= 0 && j < F.ny && k >= 0 && k < F.nz;
        const double e = E[in ? i + F.nx * (j + F.ny * k) : 0];
        Ee[z][y][x] = in ? e : 0.0;
      }
  ConstPtr gp = (ConstPtr)Gp;
  first_blocks(std::make_integer_sequence<int, 14>(), C, Ee, gp, m, I, J, K, S64, S32);
}

// The same at the nodes listed by k_galerkin_flag: grid (ceil(count / 64), 14).  Each
// wave of a block takes the coarse element on one side of its 64 nodes (bits of side: above
// the node along x, y, z), the eight are summed in that order: a chain an eighth as long
// as a thread that walks its elements one after the other.  Two blocks to a compute unit (the
// second launch bound) are worth the registers that they spill: 8450 nodes in 0.14
// ms, 0.21 with one block and 0.23 with a thread per block of the stencil.
__global__ __launch_bounds__(512, 4) void k_galerkin_first_masked(Level F, Level C, const double* __restrict__ E,
                                                               const double* __restrict__ G,
                                                               const double* __restrict__ Ke,
                                                               const int* __restrict__ list, int count,
                                                               double* __restrict__ S64, float* __restrict__ S32) {
  __shared__ double part[8][9][64];
  const int lane = threadIdx.x & 63, side = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = blockIdx.x * 64 + lane, o = 13 + blockIdx.y;
  const int m = t < count ? list[t] : 0;
  int I, J, K;
  node_coords(C, m, I, J, K);
  const int I2 = I + off_dx(o), J2 = J + off_dy(o), K2 = K + off_dz(o);
  double blk[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  const bool in = I2 >= 0 && I2 < C.nxn && J2 >= 0 && J2 < C.nyn && K2 >= 0 && K2 < C.nzn;
  const int m2 = in ? I2 + C.nxn * (J2 + C.nyn * K2) : -1;
  const int EI = I - 1 + (side & 1), EJ = J - 1 + ((side >> 1) & 1), EK = K - 1 + (side >> 2);
  // an element of the grid that holds both nodes
  if (t < count && in && EI >= 0 && EI < C.nx && EJ >= 0 && EJ < C.ny && EK >= 0 && EK < C.nz && I2 >= EI &&
      I2 <= EI + 1 && J2 >= EJ && J2 <= EJ + 1 && K2 >= EK && K2 <= EK + 1) {
    // the corners of m and m2 in the coarse element, the same for the whole wave
    const int ax = 1 - (side & 1), ay = 1 - ((side >> 1) & 1), az = 1 - (side >> 2);
    const int bx = ax + off_dx(o), by = ay + off_dy(o), bz = az + off_dz(o);
    const int a = ax + 2 * ay + 4 * az, b = bx + 2 * by + 4 * bz;
    // the coarse element's 27 fine nodes' supports (bit q of fixed[d]: component d
    // of node q) and its eight moduli, requested together
    unsigned fixed[3] = {0, 0, 0};
#pragma unroll
    for (int q = 0; q < 27; ++q) {
      const unsigned mk = F.mask[(2 * EI + q % 3) + F.nxn * ((2 * EJ + (q / 3) % 3) + F.nyn * (2 * EK + q / 9))];
#pragma unroll
      for (int d = 0; d < 3; ++d) fixed[d] |= ((mk >> d) & 1u) << q;
    }
    double Ee[8];
#pragma unroll
    for (int c = 0; c < 8; ++c)
      Ee[c] = E[(2 * EI + (c & 1)) + F.nx * ((2 * EJ + ((c >> 1) & 1)) + F.ny * (2 * EK + (c >> 2)))];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int cx = c & 1, cy = (c >> 1) & 1, cz = c >> 2;
      const int n0 = cx + 3 * cy + 9 * cz;  // the child's first node; its nodes: n0 + {0, 1, 3, 4, 9, 10, 12, 13}
      if (!(((fixed[0] | fixed[1] | fixed[2]) >> n0) & 0x361bu)) {
        const double* Gc = G + c * 576 + (3 * a) * 24 + 3 * b;
#pragma unroll
        for (int ci = 0; ci < 3; ++ci)
#pragma unroll
          for (int cj = 0; cj < 3; ++cj) blk[3 * ci + cj] += Ee[c] * Gc[ci * 24 + cj];
      } else {  // masked child: P_c^T (M K0 M) P_c restricted to corners a, b
        for (int p = 0; p < 8; ++p) {
          const int px = p & 1, py = (p >> 1) & 1, pz = p >> 2;
          const double wa = wt(cx + px, ax) * wt(cy + py, ay) * wt(cz + pz, az);
          if (wa == 0.0) continue;
          const int np = n0 + px + 3 * py + 9 * pz;
          for (int q = 0; q < 8; ++q) {
            const int qx = q & 1, qy = (q >> 1) & 1, qz = q >> 2;
            const double wb = wt(cx + qx, bx) * wt(cy + qy, by) * wt(cz + qz, bz);
            if (wb == 0.0) continue;
            const int nq = n0 + qx + 3 * qy + 9 * qz;
            const double w = Ee[c] * wa * wb;
#pragma unroll
            for (int ci = 0; ci < 3; ++ci)
#pragma unroll
              for (int cj = 0; cj < 3; ++cj)
                blk[3 * ci + cj] += (((fixed[ci] >> np) | (fixed[cj] >> nq)) & 1u)
                                        ? 0.0
                                        : w * Ke[(3 * p + ci) * 24 + 3 * q + cj];
          }
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 9; ++q) part[side][q][lane] = blk[q];
  __syncthreads();
  if (side > 0 || t >= count) return;
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    double v = part[0][q][lane];
#pragma unroll
    for (int e = 1; e < 8; ++e) v += part[e][q][lane];
    blk[q] = v;
  }
  store_block(C, m, m2, o, blk, S64, S32);
}

// Coefficient (ci, cj) at offset o of node i from the stored half: 0 where i + o
// lies outside the grid (out).
__device__ inline double half_coef(const Level& F, const double* __restrict__ S, int i, int o, int ci, int cj,
                                   bool in) {
  const int step = off_dx(o) + F.nxn * (off_dy(o) + F.nyn * off_dz(o));
  const long long at = o >= 13 ? (long long)(9 * (o - 13) + 3 * ci + cj) * F.nn + i
                               : (long long)(9 * (13 - o) + 3 * cj + ci) * F.nn + (in ? i + step : i);
  const double v = S[at];
  return in ? v : 0.0;
}

// The next level's stencil, P~^T A_f P~ from the fine one, one thread per coarse
// node and component pair (ci, cj): grid (ceil(C.nn / 64), 9).  Per axis a fine
// row i (at distance -1, 0, 1 from the coarse node, weight 1/2, 1, 1/2) and its
// neighbour i + t contribute to the coarse offsets whose support holds i + t; the
// three axes are combined one inside the other, so a fine coefficient costs
// 13/9 multiply-adds on the x axis and a ninth of that on the next instead of
// one per coarse offset.  The fine diagonal's ones at fixed DOFs take no part.
// Level 2 of 256x128x128 takes 0.46 ms (3.7 ms as one thread per block of the
// stencil, every coarse offset summing its own products), levels 3 to 5 0.07 ms
// together (2.5 ms); the loads of the fine stencil, each made by the 27/8 coarse
// nodes it reaches, bound it.
__device__ inline constexpr double axis_weight(int i, int t, int c) {  // row i, neighbour i + t, coarse offset c
  const int e = i + t - 2 * c;                                         // distance of i + t from the coarse node c
  return (i ? 0.5 : 1.0) * (e == 0 ? 1.0 : (e == 1 || e == -1 ? 0.5 : 0.0));
}
__global__ __launch_bounds__(64) void k_galerkin_coarsen(Level F, Level C, const double* __restrict__ Sf,
                                                         double* __restrict__ S64, float* __restrict__ S32) {
  const int m = blockIdx.x * 64 + threadIdx.x;
  const int ci = blockIdx.y / 3, cj = blockIdx.y % 3;
  if (m >= C.nn) return;
  int I, J, K;
  node_coords(C, m, I, J, K);
  const int fx = 2 * I, fy = 2 * J, fz = 2 * K;
  double acc[2][3][3];  // coarse offsets (0 or 1, -1..1, -1..1)
#pragma unroll
  for (int q = 0; q < 18; ++q) acc[q / 9][(q / 3) % 3][q % 3] = 0.0;
#pragma unroll 1
  for (int zq = 1; zq < 9; ++zq) {  // (iz, tz); (-1, -1) reaches offset -1 only
    const int iz = zq / 3 - 1, tz = zq % 3 - 1;
    const bool zin = fz + iz >= 0 && fz + iz < F.nzn, zin2 = fz + iz + tz >= 0 && fz + iz + tz < F.nzn;
    if (!zin || !zin2) continue;
    double ay[3][3];
#pragma unroll
    for (int q = 0; q < 9; ++q) ay[q / 3][q % 3] = 0.0;
#pragma unroll 1
    for (int iy = -1; iy <= 1; ++iy) {
      if (fy + iy < 0 || fy + iy >= F.nyn) continue;
#pragma unroll
      for (int ty = -1; ty <= 1; ++ty) {
        const bool yin2 = fy + iy + ty >= 0 && fy + iy + ty < F.nyn;
        double v[9];
#pragma unroll
        for (int xq = 0; xq < 9; ++xq) {
          const int ix = xq / 3 - 1, tx = xq % 3 - 1;
          const bool xin = fx + ix >= 0 && fx + ix < F.nxn;
          const bool in = xin && yin2 && fx + ix + tx >= 0 && fx + ix + tx < F.nxn;
          const int i = (xin ? fx + ix : fx) + F.nxn * ((fy + iy) + F.nyn * (fz + iz));
          const int o = (tz + 1) * 9 + (ty + 1) * 3 + tx + 1;
          v[xq] = half_coef(F, Sf, i, o, ci, cj, in);
          if (tx == 0 && ty == 0)  // a fixed DOF's unit diagonal
            v[xq] = (tz == 0 && ci == cj && ((F.mask[i] >> ci) & 1)) ? 0.0 : v[xq];
        }
        double ax[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int xq = 0; xq < 9; ++xq)
#pragma unroll
          for (int c = -1; c <= 1; ++c) {
            const double wgt = axis_weight(xq / 3 - 1, xq % 3 - 1, c);
            if (wgt != 0.0) ax[c + 1] += wgt * v[xq];
          }
#pragma unroll
        for (int c = -1; c <= 1; ++c) {
          const double wgt = axis_weight(iy, ty, c);
#pragma unroll
          for (int q = 0; q < 3; ++q) ay[c + 1][q] += wgt * ax[q];
        }
      }
    }
#pragma unroll
    for (int c = 0; c <= 1; ++c) {
      const double wgt = axis_weight(iz, tz, c);
#pragma unroll
      for (int q = 0; q < 9; ++q) acc[c][q / 3][q % 3] += wgt * ay[q / 3][q % 3];
    }
  }
  const int mk = C.mask[m];
#pragma unroll
  for (int o = 13; o < 27; ++o) {
    const int dx = off_dx(o), dy = off_dy(o), dz = off_dz(o);
    const int I2 = I + dx, J2 = J + dy, K2 = K + dz;
    const bool in = I2 >= 0 && I2 < C.nxn && J2 >= 0 && J2 < C.nyn && K2 < C.nzn;
    const int mk2 = in ? C.mask[I2 + C.nxn * (J2 + C.nyn * K2)] : 7;
    double v = (((mk >> ci) & 1) || ((mk2 >> cj) & 1)) ? 0.0 : acc[dz][dy + 1][dx + 1];
    if (o == 13 && ci == cj && ((mk >> ci) & 1)) v = 1.0;
    const long long idx = (long long)(9 * (o - 13) + 3 * ci + cj) * C.nn + m;
    S64[idx] = v;
    if (S32) S32[idx] = (float)v;
  }
}

// One node's stored binary64 coefficients to 16 bits: bfloat16 (STORE ==
// HEXMG_STENCIL_BF16) or binary16, block b of node n scaled by
// 2^sexp[b * nn + n] (HEXMG_STENCIL_F16).
template <int STORE>
__global__ void k_stencil_to16(Level L, const double* __restrict__ S64, uint16_t* __restrict__ S16,
                               int8_t* __restrict__ sexp) {
  const int n = blockIdx.x * kBlock + threadIdx.x;
  if (n >= L.nn) return;
  if (STORE == HEXMG_STENCIL_BF16) {
    for (int q = 0; q < kStencilCoefs; ++q) {
      const long long idx = (long long)q * L.nn + n;
      S16[idx] = __bfloat16_as_ushort(__float2bfloat16((float)S64[idx]));
    }
    return;
  }
  for (int b = 0; b < kStencilBlocks; ++b) {
    double v[9], amax = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      v[q] = S64[(long long)(9 * b + q) * L.nn + n];
      amax = fmax(amax, fabs(v[q]));
    }
    int e = 0;
    if (amax > 0.0) (void)frexp(amax, &e);  // amax in [2^(e-1), 2^e)
    const int sc = min(max(15 - e, -126), 126);  // amax * 2^sc in [2^14, 2^15)
    sexp[(long long)b * L.nn + n] = (int8_t)sc;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const _Float16 h = (_Float16)ldexp(v[q], sc);
      S16[(long long)(9 * b + q) * L.nn + n] = __builtin_bit_cast(uint16_t, h);
    }
  }
}

__device__ inline float stencil_coef(const float* S, long long i) { return S[i]; }
__device__ inline double stencil_coef(const double* S, long long i) { return S[i]; }

// 16-bit coefficients (bfloat16 or binary16, by storage type tag)
struct Bf16Tag {};
struct F16Tag {};
template <typename Tag>
struct Stored16 {
  const uint16_t* p;
};
__device__ inline float stencil_coef(Stored16<Bf16Tag> S, long long i) {
  return __uint_as_float((unsigned)S.p[i] << 16);
}
__device__ inline float stencil_coef(Stored16<F16Tag> S, long long i) {
  return __half2float(__ushort_as_half(S.p[i]));
}

// The 2^-e of a binary16 block (|e| <= 126).
__device__ inline float block_scale(int e) { return __int_as_float((127 - e) << 23); }

// y = A u from the stencil (MODE as the element kernels: 0 A u, 1 Jacobi
// sweep, 2 residual).  A block takes 64 nodes; its wave W the offsets W, W + 4,
// ..., so that a thread asks for all its coefficients (63 at the most) and
// neighbour values at once and waits on memory once -- on the small levels that
// is the whole cost --, and the four waves' sums meet in LDS.  A stored
// coefficient is read by both nodes it couples, the second time from the L2: the
// blocks of a plane go to the XCDs in bands (xcd_band_block), which keeps the planes
// in between within each XCD's L2.  The sweep on a large level is bound by the
// bytes of the stored half: 78 us on level 1 of 256x128x128 in binary32 (120 us
// with the whole stencil stored, one thread per node), and the levels under 10^4
// nodes take 4.7 us (16.6 us).  SP: the coefficient array (T*, or
// Stored16<tag> for the 16-bit storages); sexp: the binary16 blocks' scale exponents
// (null otherwise).
template <typename T, typename SP, bool SCALED, int W>
__device__ __forceinline__ void stencil_wave(const Level& L, SP S, const int8_t* __restrict__ sexp,
                                             const T* __restrict__ u, int n, int i, int j, int k, T (&a)[3]) {
  constexpr int kMine = (27 - W + 3) / 4;
  T v[kMine][3], cf[kMine][9];
  T sc[kMine];
#pragma unroll
  for (int t = 0; t < kMine; ++t) {
    const int o = W + 4 * t, dx = o % 3 - 1, dy = (o / 3) % 3 - 1, dz = o / 9 - 1;
    const bool in = i + dx >= 0 && i + dx < L.nxn && j + dy >= 0 && j + dy < L.nyn && k + dz >= 0 && k + dz < L.nzn;
    const int m = in ? n + dx + L.nxn * (dy + L.nyn * dz) : n;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const T x = u[3ll * m + c];
      v[t][c] = in ? x : T(0);
    }
    // own rows, or the transposed block of the neighbour
#pragma unroll
    for (int q = 0; q < 9; ++q)
      cf[t][q] = o >= 13 ? stencil_coef(S, (long long)(9 * (o - 13) + q) * L.nn + n)
                         : stencil_coef(S, (long long)(9 * (13 - o) + 3 * (q % 3) + q / 3) * L.nn + m);
    if constexpr (SCALED)
      sc[t] = block_scale(sexp[o >= 13 ? (long long)(o - 13) * L.nn + n : (long long)(13 - o) * L.nn + m]);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) a[c] = T(0);
#pragma unroll
  for (int t = 0; t < kMine; ++t)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const T p = cf[t][3 * c] * v[t][0] + cf[t][3 * c + 1] * v[t][1] + cf[t][3 * c + 2] * v[t][2];
      a[c] += SCALED ? sc[t] * p : p;
    }
}

template <typename T, typename SP, int MODE, bool SCALED>
__global__ __launch_bounds__(kBlock) void k_stencil(Level L, SP S, const int8_t* __restrict__ sexp,
                                                    const T* __restrict__ u, const T* __restrict__ f,
                                                    const T* __restrict__ wdinv, T* __restrict__ y,
                                                    const int* __restrict__ act, int slab) {
  static_assert(kBlock == 256, "four waves share 64 nodes");
  if (act && !act[blockIdx.y]) return;
  __shared__ T part[4][3][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int node = xcd_band_block(slab) * 64 + lane;
  const int n = min(node, L.nn - 1);
  const long long off = 3ll * L.nn * blockIdx.y;
  u += off;
  y += off;
  if (MODE != kApply) f += off;
  int i, j, k;
  node_coords(L, n, i, j, k);
  // the epilogue's inputs of component w (waves 0..2)
  const long long b = 3ll * n + (w < 3 ? w : 0);
  T ub = T(0), fb = T(0), wb = T(0);
  if (MODE == kSmooth) {
    ub = u[b];
    wb = wdinv[b];
  }
  if (MODE != kApply) fb = f[b];
  T a[3];
  if (w == 0)
    stencil_wave<T, SP, SCALED, 0>(L, S, sexp, u, n, i, j, k, a);
  else if (w == 1)
    stencil_wave<T, SP, SCALED, 1>(L, S, sexp, u, n, i, j, k, a);
  else if (w == 2)
    stencil_wave<T, SP, SCALED, 2>(L, S, sexp, u, n, i, j, k, a);
  else
    stencil_wave<T, SP, SCALED, 3>(L, S, sexp, u, n, i, j, k, a);
#pragma unroll
  for (int c = 0; c < 3; ++c) part[w][c][lane] = a[c];
  __syncthreads();
  if (w == 3 || node >= L.nn) return;
  const T Au = (part[0][w][lane] + part[1][w][lane]) + (part[2][w][lane] + part[3][w][lane]);
  y[b] = MODE == kApply ? Au : (MODE == kSmooth ? ub + wb * (fb - Au) : fb - Au);
}

__global__ void k_stencil_diag(Level L, const double* __restrict__ S, double* __restrict__ wd64,
                               float* __restrict__ wd32) {
  const int n = blockIdx.x * kBlock + threadIdx.x;
  if (n >= L.nn) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double w = L.omega / S[(long long)(4 * c) * L.nn + n];
    if (wd64) wd64[3ll * n + c] = w;  // either output may be absent
    if (wd32) wd32[3ll * n + c] = (float)w;
  }
}

// grid (ceil(N / kBlock), N): dense operator entry (r, c) from the stencil
__global__ void k_dense_from_stencil(Level C, const double* __restrict__ S, double* __restrict__ A) {
  const int N = 3 * C.nn;
  const int c = blockIdx.x * kBlock + threadIdx.x, r = blockIdx.y;
  if (c >= N) return;
  const int m = r / 3, ci = r % 3, m2 = c / 3, cj = c % 3;
  int I, J, K, I2, J2, K2;
  node_coords(C, m, I, J, K);
  node_coords(C, m2, I2, J2, K2);
  const int dx = I2 - I, dy = J2 - J, dz = K2 - K;
  double v = 0.0;
  if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1) {
    const int o = (dz + 1) * 9 + (dy + 1) * 3 + (dx + 1);
    v = o >= 13 ? S[(long long)(9 * (o - 13) + 3 * ci + cj) * C.nn + m]
                : S[(long long)(9 * (13 - o) + 3 * cj + ci) * C.nn + m2];
  }
  A[(long long)r * N + c] = v;
}

inline int blocks_for(long long n) { return (int)((n + kBlock - 1) / kBlock); }

}  // namespace

int galerkin_flag(const Level& F, const Level& C, uint8_t* flag, int* list, int* count, hipStream_t s) {
  int n = 0;
  const int zero = 0;
  if (hipMemcpyAsync(count, &zero, sizeof(int), hipMemcpyHostToDevice, s) != hipSuccess) return -1;
  k_galerkin_flag<<<blocks_for(C.nn), kBlock, 0, s>>>(F, C, flag, list, count);
  if (hipMemcpyAsync(&n, count, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return -1;
  return n;
}

void launch_galerkin_first(const Level& F, const Level& C, const double* E, const double* G, const double* Ke,
                           const uint8_t* flag, const int* list, int count, double* S64, float* S32, hipStream_t s) {
  k_galerkin_first<<<blocks_for(C.nn), kBlock, 0, s>>>(F, C, E, G + 8 * 576, flag, S64, S32);
  if (count > 0)
    k_galerkin_first_masked<<<dim3((count + 63) / 64, 14), 512, 0, s>>>(F, C, E, G, Ke, list, count, S64, S32);
}

void launch_galerkin_coarsen(const Level& F, const Level& C, const double* Sf, double* S64, float* S32,
                             hipStream_t s) {
  k_galerkin_coarsen<<<dim3((C.nn + 63) / 64, 9), 64, 0, s>>>(F, C, Sf, S64, S32);
}

namespace {
template <typename T, typename SP, bool SCALED = false>
void launch_stencil_sp(int mode, const Level& L, SP S, const int8_t* sexp, const T* u, const T* f, const T* wd,
                       T* y, int nrhs, const int* act, hipStream_t s, const LaunchTimer& t) {
  const dim3 g((L.nn + 63) / 64, nrhs);
  const int slab = band_slab(((long long)L.nxn * L.nyn + 63) / 64);  // the blocks of one plane
  if (mode == kApply)
    launch_timed(k_stencil<T, SP, kApply, SCALED>, g, dim3(kBlock), s, t, L, S, sexp, u, f, wd, y, act, slab);
  else if (mode == kSmooth)
    launch_timed(k_stencil<T, SP, kSmooth, SCALED>, g, dim3(kBlock), s, t, L, S, sexp, u, f, wd, y, act, slab);
  else
    launch_timed(k_stencil<T, SP, kResidual, SCALED>, g, dim3(kBlock), s, t, L, S, sexp, u, f, wd, y, act, slab);
}
}  // namespace

template <typename T>
void launch_stencil(int mode, const Level& L, const T* S, const T* u, const T* f, const T* wd, T* y, int nrhs,
                    const int* act, hipStream_t s, const LaunchTimer& t) {
  launch_stencil_sp<T, const T*>(mode, L, S, nullptr, u, f, wd, y, nrhs, act, s, t);
}

void launch_stencil16(int store, int mode, const Level& L, const uint16_t* S16, const int8_t* sexp, const float* u,
                      const float* f, const float* wd, float* y, int nrhs, const int* act, hipStream_t s,
                      const LaunchTimer& t) {
  if (store == HEXMG_STENCIL_BF16)
    launch_stencil_sp<float, Stored16<Bf16Tag>>(mode, L, Stored16<Bf16Tag>{S16}, nullptr, u, f, wd, y, nrhs, act,
                                                 s, t);
  else
    launch_stencil_sp<float, Stored16<F16Tag>, true>(mode, L, Stored16<F16Tag>{S16}, sexp, u, f, wd, y, nrhs, act, s, t);
}

void launch_stencil_to16(int store, const Level& L, const double* S64, uint16_t* S16, int8_t* sexp,
                         hipStream_t s) {
  if (store == HEXMG_STENCIL_BF16)
    k_stencil_to16<HEXMG_STENCIL_BF16><<<blocks_for(L.nn), kBlock, 0, s>>>(L, S64, S16, sexp);
  else
    k_stencil_to16<HEXMG_STENCIL_F16><<<blocks_for(L.nn), kBlock, 0, s>>>(L, S64, S16, sexp);
}
template void launch_stencil<double>(int, const Level&, const double*, const double*, const double*, const double*,
                                     double*, int, const int*, hipStream_t, const LaunchTimer&);
template void launch_stencil<float>(int, const Level&, const float*, const float*, const float*, const float*,
                                    float*, int, const int*, hipStream_t, const LaunchTimer&);

void launch_stencil_diag(const Level& L, const double* S, double* wd64, float* wd32, hipStream_t s) {
  k_stencil_diag<<<blocks_for(L.nn), kBlock, 0, s>>>(L, S, wd64, wd32);
}

void launch_dense_from_stencil(const Level& C, const double* S, double* A, hipStream_t s) {
  const int N = 3 * C.nn;
  k_dense_from_stencil<<<dim3(blocks_for(N), N), kBlock, 0, s>>>(C, S, A);
}

// G_c = P_c^T K0 P_c for the eight children c of a coarse element (host):
// G[c][(3a+ci)*24 + 3b+cj], a, b the coarse corners; after them (at 8 * 576) the
// blocks [a, b] of every offset b - a >= 0 as k_galerkin_first takes them,
// [offset, a][c][3ci+cj].
void galerkin_child_matrices(const double* Ke, double* G) {
  auto w1 = [](int t, int a) { return a == 0 ? (t == 0 ? 1.0 : (t == 1 ? 0.5 : 0.0)) : (t == 2 ? 1.0 : (t == 1 ? 0.5 : 0.0)); };
  for (int c = 0; c < 8; ++c) {
    const int cx = c & 1, cy = (c >> 1) & 1, cz = c >> 2;
    double P[8][8];  // P[p][a]: weight of coarse corner a at fine corner p of child c
    for (int p = 0; p < 8; ++p)
      for (int a = 0; a < 8; ++a)
        P[p][a] = w1(cx + (p & 1), a & 1) * w1(cy + ((p >> 1) & 1), (a >> 1) & 1) * w1(cz + (p >> 2), a >> 2);
    for (int a = 0; a < 8; ++a)
      for (int b = 0; b < 8; ++b)
        for (int ci = 0; ci < 3; ++ci)
          for (int cj = 0; cj < 3; ++cj) {
            double s = 0.0;
            for (int p = 0; p < 8; ++p) {
              if (P[p][a] == 0.0) continue;
              for (int q = 0; q < 8; ++q) s += P[p][a] * P[q][b] * Ke[(3 * p + ci) * 24 + 3 * q + cj];
            }
            G[c * 576 + (3 * a + ci) * 24 + 3 * b + cj] = s;
          }
  }
  double* Gp = G + 8 * 576;
  for (int o = 13; o < 27; ++o)
    for (int a = 0; a < 8; ++a) {
      const int bx = (a & 1) + o % 3 - 1, by = ((a >> 1) & 1) + (o / 3) % 3 - 1, bz = (a >> 2) + o / 9 - 1;
      if (bx < 0 || bx > 1 || by < 0 || by > 1 || bz < 0 || bz > 1) continue;
      const int b = bx + 2 * by + 4 * bz;
      for (int c = 0; c < 8; ++c)
        for (int q = 0; q < 9; ++q) *Gp++ = G[c * 576 + (3 * a + q / 3) * 24 + 3 * b + q % 3];
    }
}

}  // namespace hexmg
