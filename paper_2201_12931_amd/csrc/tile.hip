// V-cycle steps of the small levels (Alg. 3), several to a launch.
//
// On a level of a few thousand nodes every step is one launch whose 3.4 us are
// mostly its start, so the three launches on the way down (a sweep, the
// residual, the restriction) and the three on the way up (the prolongation, two
// sweeps) each become one: a block computes its few nodes' results from a tile in LDS
// with the halo that the chain of steps needs, repeating its neighbours' work
// (a sweep is formed 7.7 times on the way down, 4.5 times on the way up), which
// costs less than the launches.  What bounds them is one block's chain: loads 1.2 us,
// each product 1 to 2 us, 7.2 us down and 7.5 us up in all, so the products of a node are
// split over two to eight threads.  17x9x9 and 9x5x5 nodes under 32x16x16: a V-cycle in
// binary64 takes 48 us, 57 step by step.  Two pre- and two post-sweeps; the first
// pre-sweep from zero is omega/D f.
//
// The product at a node gathers its eight elements' rows of K0 from the tile: the
// rows hold ten distinct values (an entry depends on which axes its nodes differ
// in, with the sign of their derivatives), kept in scalar registers, and apply to the
// differences of u from the node's own value.
#include "hexmg_impl.h"

namespace hexmg {

namespace {

constexpr int kTx = 4, kTy = 4, kTz = 2;  // fine nodes of a tile (coarse: half of each)
constexpr int kTileBlock = 512;

// What the elements on the sides [Z0, Z1) along z and [Y0, Y1) along y (0: below the
// node, 1: above) contribute to K u at a node, from values in LDS: u (three planes
// of us entries) around entry c with row and plane strides sy, sz; moduli Em
// around entry e (the element on the lower side of every axis) with strides esy, esz.
template <typename T, int Z0, int Z1, int Y0, int Y1>
__device__ __forceinline__ void tile_product(const K0Coef<T>& k, const T* u, int us, int c, int sy, int sz, const T* Em,
                                             int e, int esy, int esz, T (&Ku)[3]) {
  T v[3][3][3][3];  // [z][y][x][component]
#pragma unroll
  for (int z = Z0; z < Z1 + 1; ++z)
#pragma unroll
    for (int y = Y0; y < Y1 + 1; ++y)
#pragma unroll
      for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int q = 0; q < 3; ++q) v[z][y][x][q] = u[q * us + c + (x - 1) + (y - 1) * sy + (z - 1) * sz];
  // the rows of K0 sum to zero: products of the differences from the node itself, which
  // do not cancel where u is smooth (binary32 V-cycles of a body force: 0.99 of the step
  // launches' distance from the oracle's, 1.39 on the values themselves; same time)
#pragma unroll
  for (int z = Z0; z < Z1 + 1; ++z)
#pragma unroll
    for (int y = Y0; y < Y1 + 1; ++y)
#pragma unroll
      for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          if (z != 1 || y != 1 || x != 1) v[z][y][x][q] -= v[1][1][1][q];
  T acc[2][3] = {{T(0), T(0), T(0)}, {T(0), T(0), T(0)}};
#pragma unroll
  for (int ez = Z0; ez < Z1; ++ez)
#pragma unroll
    for (int ey = Y0; ey < Y1; ++ey)
#pragma unroll
      for (int ex = 0; ex < 2; ++ex) {
        const int a[3] = {1 - ex, 1 - ey, 1 - ez};  // the node's corner of this element
        const T E = Em[e + ex + ey * esy + ez * esz];
        T s[3] = {T(0), T(0), T(0)};
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const int bb[3] = {b & 1, (b >> 1) & 1, b >> 2};
          if (bb[0] == a[0] && bb[1] == a[1] && bb[2] == a[2]) continue;  // the node itself
          const T(&w)[3] = v[ez + bb[2]][ey + bb[1]][ex + bb[0]];
#pragma unroll
          for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              if (i == j) {
                const int differ = (a[(i + 1) % 3] != bb[(i + 1) % 3]) + (a[(i + 2) % 3] != bb[(i + 2) % 3]);
                s[i] += k.d[a[i] != bb[i]][differ] * w[j];
              } else {
                const int o = 3 - i - j;  // the third axis
                const bool pos = (a[i] != 0) == (bb[j] != 0), same = pos == ((a[j] != 0) == (bb[i] != 0));
                const T kk = same ? k.p[a[o] != bb[o]] : k.m[a[o] != bb[o]];
                if (pos)
                  s[i] += kk * w[j];
                else
                  s[i] -= kk * w[j];
              }
            }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) acc[ex][i] += E * s[i];
      }
#pragma unroll
  for (int i = 0; i < 3; ++i) Ku[i] = acc[0][i] + acc[1][i];
}

// Way down, tile (bx, by, bz) of the level: u (the two pre-sweeps' result) at the
// tile's kTx x kTy x kTz nodes, and at the coarse nodes under them f_c = M_c P^T (f - A u) and
// (wdc non-null) the coarse level's first sweep.
// Coordinates below are relative to the tile's first node.
template <typename T>
__device__ __forceinline__ void tile_down(const TileDownTask<T>& t, const K0Coef<T>& k0, int bx, int by, int bz,
                                          int rhs) {
  const Level& F = t.F;
  if (t.act && !t.act[rhs]) return;
  // regions: first sweep and f (halo 3), second sweep (2 below, 1 above each further one), residual (1)
  constexpr int AX = kTx + 5, AY = kTy + 5, AZ = kTz + 5, NA = AX * AY * AZ;  // from -3
  constexpr int BX = kTx + 3, BY = kTy + 3, BZ = kTz + 3, NB = BX * BY * BZ;  // from -2
  constexpr int CX = kTx + 1, CY = kTy + 1, CZ = kTz + 1, NC = CX * CY * CZ;  // from -1
  constexpr int EX = kTx + 4, EY = kTy + 4, EZ = kTz + 4, NE = EX * EY * EZ;  // elements, from -3
  static_assert(NB <= 256 && NC <= 128 && kTileBlock == 512, "a node's product by 2 or 4 threads in one round");
  __shared__ T f[3 * NA], u1[3 * NA], u2[3 * NB], Em[NE], wd[NB], half[2][3 * NB], r[4][3 * NC];
  __shared__ unsigned char mk[NB];
  const int tid = threadIdx.x;
  const int x0 = bx * kTx, y0 = by * kTy, z0 = bz * kTz;
  const long long off = 3ll * F.nn * rhs;
  // every input of the tile is requested before the first use
  constexpr int RA = (NA + kTileBlock - 1) / kTileBlock, RE = (NE + kTileBlock - 1) / kTileBlock;
  T fv[RA][3], wv[RA], ev[RE];
#pragma unroll
  for (int p = 0; p < RA; ++p) {
    const int n = tid + p * kTileBlock;
    const int i = x0 - 3 + n % AX, j = y0 - 3 + (n / AX) % AY, k = z0 - 3 + n / (AX * AY);
    const bool in = n < NA && i >= 0 && i < F.nxn && j >= 0 && j < F.nyn && k >= 0 && k < F.nzn;
    const int g = in ? i + F.nxn * (j + F.nyn * k) : 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) fv[p][c] = in ? t.f[off + 3ll * g + c] : T(0);
    wv[p] = in ? t.wd[g] : T(0);
  }
#pragma unroll
  for (int p = 0; p < RE; ++p) {
    const int n = tid + p * kTileBlock;
    const int i = x0 - 3 + n % EX, j = y0 - 3 + (n / EX) % EY, k = z0 - 3 + n / (EX * EY);
    const bool in = n < NE && i >= 0 && i < F.nx && j >= 0 && j < F.ny && k >= 0 && k < F.nz;
    ev[p] = in ? t.E[i + F.nx * (j + F.ny * k)] : T(0);
  }
  // second-sweep node of this thread: two threads (halves of the block) per node
  const int nb = tid & 255, bxn = nb % BX, byn = (nb / BX) % BY, bzn = nb / (BX * BY);
  int m = 0;
  {
    const int i = x0 - 2 + bxn, j = y0 - 2 + byn, k = z0 - 2 + bzn;
    if (nb < NB && i >= 0 && i < F.nxn && j >= 0 && j < F.nyn && k >= 0 && k < F.nzn)
      m = F.mask[i + F.nxn * (j + F.nyn * k)];
  }
#pragma unroll
  for (int p = 0; p < RA; ++p) {
    const int n = tid + p * kTileBlock;
    if (n < NA) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        f[c * NA + n] = fv[p][c];
        u1[c * NA + n] = wv[p] * fv[p][c];  // f is zero at fixed DOFs
      }
      const int i = n % AX - 1, j = (n / AX) % AY - 1, k = n / (AX * AY) - 1;
      if (i >= 0 && i < BX && j >= 0 && j < BY && k >= 0 && k < BZ) wd[i + BX * (j + BY * k)] = wv[p];
    }
  }
#pragma unroll
  for (int p = 0; p < RE; ++p)
    if (tid + p * kTileBlock < NE) Em[tid + p * kTileBlock] = ev[p];
  if (tid < NB) mk[tid] = (unsigned char)m;
  __syncthreads();
  if (nb < NB) {
    const int c = (bxn + 1) + AX * ((byn + 1) + AY * (bzn + 1)), e = bxn + EX * (byn + EY * bzn);
    T Ku[3];
    if (tid < 256)  // uniform per wave
      tile_product<T, 0, 1, 0, 2>(k0, u1, NA, c, AX, AX * AY, Em, e, EX, EX * EY, Ku);
    else
      tile_product<T, 1, 2, 0, 2>(k0, u1, NA, c, AX, AX * AY, Em, e, EX, EX * EY, Ku);
#pragma unroll
    for (int q = 0; q < 3; ++q) half[tid >> 8][q * NB + nb] = Ku[q];
  }
  __syncthreads();
  if (tid < NB) {  // second sweep
    const int c = (bxn + 1) + AX * ((byn + 1) + AY * (bzn + 1));
    const T w = wd[tid];
    T v[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const T uq = u1[q * NA + c];
      v[q] = ((m >> q) & 1) ? T(0) : uq + w * (f[q * NA + c] - (half[0][q * NB + tid] + half[1][q * NB + tid]));
      u2[q * NB + tid] = v[q];
    }
    const int i = bxn - 2, j = byn - 2, k = bzn - 2;
    if (i >= 0 && i < kTx && j >= 0 && j < kTy && k >= 0 && k < kTz && x0 + i < F.nxn && y0 + j < F.nyn &&
        z0 + k < F.nzn) {
      const long long g = off + 3ll * ((x0 + i) + F.nxn * ((y0 + j) + F.nyn * (z0 + k)));
#pragma unroll
      for (int q = 0; q < 3; ++q) t.u[g + q] = v[q];
    }
  }
  __syncthreads();
  if ((tid & 127) < NC) {  // residual, a quarter of the elements per thread (the first one's with f)
    const int part = tid >> 7, n = tid & 127;
    const int i = n % CX, j = (n / CX) % CY, k = n / (CX * CY);
    const int c = (i + 1) + BX * ((j + 1) + BY * (k + 1)), e = (i + 1) + EX * ((j + 1) + EY * (k + 1));
    T Ku[3];
    if (part == 0)  // uniform per wave
      tile_product<T, 0, 1, 0, 1>(k0, u2, NB, c, BX, BX * BY, Em, e, EX, EX * EY, Ku);
    else if (part == 1)
      tile_product<T, 0, 1, 1, 2>(k0, u2, NB, c, BX, BX * BY, Em, e, EX, EX * EY, Ku);
    else if (part == 2)
      tile_product<T, 1, 2, 0, 1>(k0, u2, NB, c, BX, BX * BY, Em, e, EX, EX * EY, Ku);
    else
      tile_product<T, 1, 2, 1, 2>(k0, u2, NB, c, BX, BX * BY, Em, e, EX, EX * EY, Ku);
    const int fa = (i + 2) + AX * ((j + 2) + AY * (k + 2)), mm = mk[c];
#pragma unroll
    for (int q = 0; q < 3; ++q)
      r[part][q * NC + n] = ((mm >> q) & 1) ? T(0) : (part ? T(0) : f[q * NA + fa]) - Ku[q];
  }
  __syncthreads();
  // restriction: one thread per coarse DOF of the tile
  constexpr int DX = kTx / 2, DY = kTy / 2, DZ = kTz / 2;
  if (tid < 3 * DX * DY * DZ) {
    const int q = tid % 3, n = tid / 3;
    const int i = n % DX, j = (n / DX) % DY, k = n / (DX * DY);
    const int I = bx * DX + i, J = by * DY + j, K = bz * DZ + k;
    const int nxn = F.nx / 2 + 1, nyn = F.ny / 2 + 1, nzn = F.nz / 2 + 1;
    if (I < nxn && J < nyn && K < nzn) {
      T s = T(0);
#pragma unroll
      for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) {
            const T wgt = (dx == 1 ? T(1) : T(0.5)) * (dy == 1 ? T(1) : T(0.5)) * (dz == 1 ? T(1) : T(0.5));
            const int at = q * NC + (2 * i + dx) + CX * ((2 * j + dy) + CY * (2 * k + dz));
            s += wgt * ((r[0][at] + r[1][at]) + (r[2][at] + r[3][at]));
          }
      const int g = I + nxn * (J + nyn * K);
      const T fc = ((t.cmask[g] >> q) & 1) ? T(0) : s;
      const long long go = 3ll * nxn * nyn * nzn * rhs + 3ll * g + q;
      t.fc[go] = fc;
      if (t.wdc) t.tc[go] = t.wdc[g] * fc;
    }
  }
}

// Way up: u + P e_c and two sweeps of it to out (another vector than u: its
// neighbours still read u) at the tile's nodes; DOT: also one partial of f . out
// per tile and right-hand side.
template <typename T, bool DOT>
__device__ __forceinline__ void tile_up(const TileUpTask<T>& t, const K0Coef<T>& k0, int bx, int by, int bz, int rhs,
                                        int tile, int tiles) {
  const Level& F = t.F;
  if (t.act && !t.act[rhs]) return;
  constexpr int AX = kTx + 4, AY = kTy + 4, AZ = kTz + 4, NA = AX * AY * AZ;  // corrected u, from -2
  constexpr int BX = kTx + 2, BY = kTy + 2, BZ = kTz + 2, NB = BX * BY * BZ;  // first sweep, from -1
  constexpr int EX = kTx + 3, EY = kTy + 3, EZ = kTz + 3, NE = EX * EY * EZ;  // elements, from -2
  constexpr int NO = kTx * kTy * kTz;
  constexpr int HX = kTx / 2 + 3, HY = kTy / 2 + 3, HZ = kTz / 2 + 3, NH = HX * HY * HZ;  // coarse nodes, from -1
  static_assert(NB <= 256 && 8 * NO <= kTileBlock && NE <= kTileBlock && NH <= kTileBlock && kTileBlock == 512,
                "one round per stage");
  __shared__ T u3[3 * NA], u4[3 * NB], ec[3 * NH], Em[NE], half[3 * NB], part[8][3 * NO];
  const int tid = threadIdx.x;
  const int x0 = bx * kTx, y0 = by * kTy, z0 = bz * kTz;
  const long long off = 3ll * F.nn * rhs;
  const int nxn = F.nx / 2 + 1, nyn = F.ny / 2 + 1, nzn = F.nz / 2 + 1;
  constexpr int RA = (NA + kTileBlock - 1) / kTileBlock;
  T uv[RA][3], cv[3] = {T(0), T(0), T(0)}, ev = T(0), fb[3] = {T(0), T(0), T(0)}, wb = T(0);
  int mu[RA], mb = 0;
#pragma unroll
  for (int p = 0; p < RA; ++p) {
    const int n = tid + p * kTileBlock;
    const int i = x0 - 2 + n % AX, j = y0 - 2 + (n / AX) % AY, k = z0 - 2 + n / (AX * AY);
    const bool in = n < NA && i >= 0 && i < F.nxn && j >= 0 && j < F.nyn && k >= 0 && k < F.nzn;
    const int g = in ? i + F.nxn * (j + F.nyn * k) : 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) uv[p][c] = in ? t.u[off + 3ll * g + c] : T(0);
    mu[p] = in ? (int)F.mask[g] : 7;  // outside the grid: like a fixed node, zero
  }
  if (tid < NH) {
    const int I = x0 / 2 - 1 + tid % HX, J = y0 / 2 - 1 + (tid / HX) % HY, K = z0 / 2 - 1 + tid / (HX * HY);
    if (I >= 0 && I < nxn && J >= 0 && J < nyn && K >= 0 && K < nzn) {
      const long long g = 3ll * nxn * nyn * nzn * rhs + 3ll * (I + nxn * (J + nyn * K));
#pragma unroll
      for (int c = 0; c < 3; ++c) cv[c] = t.ec[g + c];
    }
  }
  if (tid < NE) {
    const int i = x0 - 2 + tid % EX, j = y0 - 2 + (tid / EX) % EY, k = z0 - 2 + tid / (EX * EY);
    if (i >= 0 && i < F.nx && j >= 0 && j < F.ny && k >= 0 && k < F.nz) ev = t.E[i + F.nx * (j + F.ny * k)];
  }
  // first-sweep node of this thread: two threads (halves of the block) per node
  const int nb = tid & 255, bi = nb % BX, bj = (nb / BX) % BY, bk = nb / (BX * BY);
  if (tid < NB) {
    const int i = x0 - 1 + bi, j = y0 - 1 + bj, k = z0 - 1 + bk;
    mb = 7;
    if (i >= 0 && i < F.nxn && j >= 0 && j < F.nyn && k >= 0 && k < F.nzn) {
      const int g = i + F.nxn * (j + F.nyn * k);
#pragma unroll
      for (int c = 0; c < 3; ++c) fb[c] = t.f[off + 3ll * g + c];
      wb = t.wd[g];
      mb = F.mask[g];
    }
  }
  if (tid < NH) {
#pragma unroll
    for (int c = 0; c < 3; ++c) ec[c * NH + tid] = cv[c];
  }
  if (tid < NE) Em[tid] = ev;
  __syncthreads();
#pragma unroll
  for (int p = 0; p < RA; ++p) {  // u + P e_c: the mean of the (one or two) coarse neighbours per axis
    const int n = tid + p * kTileBlock;
    if (n < NA) {
      const int i = n % AX, j = (n / AX) % AY, k = n / (AX * AY);  // node x0 - 2 + i, coarse from x0 / 2 - 1
      const int h = (i >> 1) + HX * ((j >> 1) + HY * (k >> 1));
      const int dx = i & 1, dy = (j & 1) * HX, dz = (k & 1) * HX * HY;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const T* e = ec + c * NH + h;
        const T s0 = T(0.5) * (T(0.5) * (e[0] + e[dx]) + T(0.5) * (e[dy] + e[dy + dx]));
        const T s1 = T(0.5) * (T(0.5) * (e[dz] + e[dz + dx]) + T(0.5) * (e[dz + dy] + e[dz + dy + dx]));
        u3[c * NA + n] = ((mu[p] >> c) & 1) ? uv[p][c] : uv[p][c] + T(0.5) * (s0 + s1);
      }
    }
  }
  __syncthreads();
  {
    const int c = (bi + 1) + AX * ((bj + 1) + AY * (bk + 1)), e = bi + EX * (bj + EY * bk);
    T Ku[3] = {T(0), T(0), T(0)};
    if (nb < NB) {
      if (tid < 256)  // uniform per wave
        tile_product<T, 0, 1, 0, 2>(k0, u3, NA, c, AX, AX * AY, Em, e, EX, EX * EY, Ku);
      else
        tile_product<T, 1, 2, 0, 2>(k0, u3, NA, c, AX, AX * AY, Em, e, EX, EX * EY, Ku);
    }
    if (tid >= 256 && nb < NB) {
#pragma unroll
      for (int q = 0; q < 3; ++q) half[q * NB + nb] = Ku[q];
    }
    __syncthreads();
    if (tid < NB) {  // first sweep
#pragma unroll
      for (int q = 0; q < 3; ++q)
        u4[q * NB + tid] =
            ((mb >> q) & 1) ? T(0) : u3[q * NA + c] + wb * (fb[q] - (Ku[q] + half[q * NB + tid]));
    }
  }
  __syncthreads();
  if (tid < 8 * NO) {  // second sweep: one element of a node per thread
    const int s = tid / NO, n = tid % NO;  // s: the element's side per axis
    const int i = n % kTx, j = (n / kTx) % kTy, k = n / (kTx * kTy);
    const int ex = s & 1, ey = (s >> 1) & 1, ez = s >> 2;
    const int c0 = (i + ex) + BX * ((j + ey) + BY * (k + ez));  // the element's first node
    const int sx = ex ? 1 : -1, syg = ey ? 1 : -1, szg = ez ? 1 : -1;
    // K0 is symmetric under reflection of an axis with the sign of that component
    // flipped: the rows of corner (1 - ex, ...) are those of corner 0 on the reflected element
    T v[8][3], sres[3] = {T(0), T(0), T(0)};
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      // reflected corner b: along a reflected axis the node on the other side
      const int ox = (b & 1) ^ (ex ? 0 : 1), oy = ((b >> 1) & 1) ^ (ey ? 0 : 1), oz = (b >> 2) ^ (ez ? 0 : 1);
      const int at = c0 + ox + BX * (oy + BY * oz);
      v[b][0] = T(sx) * u4[at];
      v[b][1] = T(syg) * u4[NB + at];
      v[b][2] = T(szg) * u4[2 * NB + at];
    }
#pragma unroll
    for (int b = 1; b < 8; ++b) {  // on the differences from the node (corner 0), as in tile_product
      const int bb[3] = {b & 1, (b >> 1) & 1, b >> 2};
#pragma unroll
      for (int d = 0; d < 3; ++d) v[b][d] -= v[0][d];
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          if (q == d) {
            sres[q] += k0.d[bb[q]][bb[(q + 1) % 3] + bb[(q + 2) % 3]] * v[b][d];
          } else {
            // node corner 0: derivative signs -1; those of b: +1 where it differs
            const int o = 3 - q - d;
            const bool pos = bb[d] == 0, same = pos == (bb[q] == 0);
            const T kk = same ? k0.p[bb[o]] : k0.m[bb[o]];
            if (pos)
              sres[q] += kk * v[b][d];
            else
              sres[q] -= kk * v[b][d];
          }
        }
    }
    const T E = Em[(i + 1 + ex) + EX * ((j + 1 + ey) + EY * (k + 1 + ez))];
    part[s][n] = E * T(sx) * sres[0];
    part[s][NO + n] = E * T(syg) * sres[1];
    part[s][2 * NO + n] = E * T(szg) * sres[2];
  }
  // the result's f and omega/D lie in the registers of its first-sweep thread
  __syncthreads();
  double dot = 0.0;
  {
    const int i = bi - 1, j = bj - 1, k = bk - 1;
    if (tid < NB && i >= 0 && i < kTx && j >= 0 && j < kTy && k >= 0 && k < kTz && x0 + i < F.nxn && y0 + j < F.nyn &&
        z0 + k < F.nzn) {
      const int n = i + kTx * (j + kTy * k);
      const long long g = off + 3ll * ((x0 + i) + F.nxn * ((y0 + j) + F.nyn * (z0 + k)));
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        T Ku = T(0);
#pragma unroll
        for (int s = 0; s < 8; ++s) Ku += part[s][q * NO + n];
        const T y = ((mb >> q) & 1) ? T(0) : u4[q * NB + tid] + wb * (fb[q] - Ku);
        t.out[g + q] = y;
        if (DOT) dot += (double)fb[q] * (double)y;
      }
    }
  }
  if (DOT) {  // one partial per tile, in a fixed order
    __shared__ double wsum[kTileBlock / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dot += __shfl_down(dot, o, 64);
    if ((tid & 63) == 0) wsum[tid >> 6] = dot;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kTileBlock / 64; ++w) s += wsum[w];
      t.dotp[(long long)tiles * rhs + tile] = s;
    }
  }
}

// Workgroup `local` of a grid's launch: tile, then right-hand side.
struct TileAt {
  int bx, by, bz, rhs, tile, tiles;
};
__device__ inline TileAt tile_at(const Level& F, int local) {
  const int gx = (F.nxn + kTx - 1) / kTx, gy = (F.nyn + kTy - 1) / kTy, gz = (F.nzn + kTz - 1) / kTz;
  TileAt t;
  t.tiles = gx * gy * gz;
  t.rhs = local / t.tiles;
  t.tile = local - t.rhs * t.tiles;
  t.bx = t.tile % gx;
  t.by = (t.tile / gx) % gy;
  t.bz = t.tile / (gx * gy);
  return t;
}
// One grid's launch is a batch of one (the task then lies at a fixed place of the arguments).
template <typename T>
__global__ __launch_bounds__(kTileBlock, sizeof(T) == 8 ? 3 : 4) void k_tile_down(Batch<TileDownTask<T>> b, K0Coef<T> k) {
  const int i = batch_task(b.begin, b.n, (int)blockIdx.x);
  const TileAt a = tile_at(b.a[i].F, (int)blockIdx.x - b.begin[i]);
  tile_down<T>(b.a[i], k, a.bx, a.by, a.bz, a.rhs);
}
template <typename T, bool DOT>
__global__ __launch_bounds__(kTileBlock, sizeof(T) == 8 ? 3 : 4) void k_tile_up(Batch<TileUpTask<T>> b, K0Coef<T> k) {
  const int i = batch_task(b.begin, b.n, (int)blockIdx.x);
  const TileAt a = tile_at(b.a[i].F, (int)blockIdx.x - b.begin[i]);
  tile_up<T, DOT>(b.a[i], k, a.bx, a.by, a.bz, a.rhs, a.tile, a.tiles);
}

}  // namespace

int tile_count(const Level& F) {
  return ((F.nxn + kTx - 1) / kTx) * ((F.nyn + kTy - 1) / kTy) * ((F.nzn + kTz - 1) / kTz);
}

template <typename T>
void launch_tile_down(const Batch<TileDownTask<T>>& b, const K0Coef<T>& k, hipStream_t s) {
  k_tile_down<T><<<b.begin[b.n], kTileBlock, 0, s>>>(b, k);
}
template <typename T>
void launch_tile_up(bool dot, const Batch<TileUpTask<T>>& b, const K0Coef<T>& k, hipStream_t s) {
  if (dot)
    k_tile_up<T, true><<<b.begin[b.n], kTileBlock, 0, s>>>(b, k);
  else
    k_tile_up<T, false><<<b.begin[b.n], kTileBlock, 0, s>>>(b, k);
}
template void launch_tile_down<float>(const Batch<TileDownTask<float>>&, const K0Coef<float>&, hipStream_t);
template void launch_tile_down<double>(const Batch<TileDownTask<double>>&, const K0Coef<double>&, hipStream_t);
template void launch_tile_up<float>(bool, const Batch<TileUpTask<float>>&, const K0Coef<float>&, hipStream_t);
template void launch_tile_up<double>(bool, const Batch<TileUpTask<double>>&, const K0Coef<double>&, hipStream_t);

bool k0_coefficients(const double* Ke, K0Coef<double>* k) {
  auto at = [&](int a, int c, int b, int d) { return Ke[(3 * a + c) * 24 + 3 * b + d]; };
  k->d[0][0] = at(0, 0, 0, 0);
  k->d[0][1] = at(0, 0, 2, 0);
  k->d[0][2] = at(0, 0, 6, 0);
  k->d[1][0] = at(0, 0, 1, 0);
  k->d[1][1] = at(0, 0, 3, 0);
  k->d[1][2] = at(0, 0, 7, 0);
  k->p[0] = at(0, 0, 0, 1);
  k->p[1] = at(0, 0, 4, 1);
  k->m[0] = at(0, 0, 1, 1);
  k->m[1] = at(0, 0, 5, 1);
  for (int a = 0; a < 8; ++a)
    for (int b = 0; b < 8; ++b)
      for (int c = 0; c < 3; ++c)
        for (int d = 0; d < 3; ++d) {
          auto bit = [](int n, int axis) { return (n >> axis) & 1; };
          double v;
          if (c == d) {
            v = k->d[bit(a, c) != bit(b, c)][(bit(a, (c + 1) % 3) != bit(b, (c + 1) % 3)) +
                                             (bit(a, (c + 2) % 3) != bit(b, (c + 2) % 3))];
          } else {
            const int o = 3 - c - d, third = bit(a, o) != bit(b, o);
            const bool pos = bit(a, c) == bit(b, d), same = pos == (bit(a, d) == bit(b, c));
            v = (pos ? 1.0 : -1.0) * (same ? k->p[third] : k->m[third]);
          }
          const double e = v - at(a, c, b, d);
          if (!(e < 1e-13 && e > -1e-13)) return false;
        }
  return true;
}

}  // namespace hexmg
