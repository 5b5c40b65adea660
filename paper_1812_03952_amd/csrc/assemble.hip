// assemble.hip -- the synthetic Jacobian on the device, and the chain rule
// back from dJ/dA to dJ/dlog k for the adjoint.
//
// Face transmissibility is tscale times the harmonic mean of the two cells'
// directional permeabilities (Section "Numerical Methods": harmonic
// averaging of the geometric part, one value shared by both cells of a
// face, zero on no-flow boundary faces).  Each row's diagonal block is the
// accumulation block over dt, plus T*M for every face of the row (the
// negated off-diagonal blocks), plus u*k*I in perforated cells (Peaceman
// form, well index proportional to k; Section "Well Modeling").
// FMA contraction is off so the blocks are the same products and sums as in
// a plain FP64 evaluation.
#pragma clang fp contract(off)
#include "rs_internal.h"
#include <math.h>

namespace {
#include "csr7.h"

__device__ __forceinline__ int64_t nbr_of(int64_t c, int s, int64_t nx, int64_t nxy) {
  switch (s) {
    case 0: return c - nxy;
    case 1: return c - nx;
    case 2: return c - 1;
    case 3: return c;
    case 4: return c + 1;
    case 5: return c + nx;
    default: return c + nxy;
  }
}
__device__ __forceinline__ int axis_of(int s) { return s == 0 || s == 6 ? 2 : (s == 1 || s == 5 ? 1 : 0); }

// index of cell c in the ascending well list, or -1
__device__ __forceinline__ int well_of(int nw, const int32_t *__restrict__ wc, int64_t c) {
  int lo = 0, hi = nw - 1;
  while (lo <= hi) {
    int mid = (lo + hi) >> 1;
    if (wc[mid] == c) return mid;
    if (wc[mid] < c) lo = mid + 1; else hi = mid - 1;
  }
  return -1;
}

// A cell's coordinates and its in-grid slots as a bit mask (grids hold fewer
// than 2^31 cells).
struct cell_at {
  int i, j, k;
  unsigned in;
};
__device__ __forceinline__ unsigned slots_in(int i, int j, int k, int nx, int ny, int nz) {
  return (k > 0 ? 1u : 0u) | (j > 0 ? 2u : 0u) | (i > 0 ? 4u : 0u) | 8u | (i < nx - 1 ? 16u : 0u) |
         (j < ny - 1 ? 32u : 0u) | (k < nz - 1 ? 64u : 0u);
}
__device__ __forceinline__ cell_at cell_of(int64_t c, int nx, int ny, int nz) {
  const uint32_t cu = (uint32_t)c, line = cu / (uint32_t)nx;
  cell_at a;
  a.i = (int)(cu - line * (uint32_t)nx);
  a.k = (int)(line / (uint32_t)ny);
  a.j = (int)(line - (uint32_t)a.k * (uint32_t)ny);
  a.in = slots_in(a.i, a.j, a.k, nx, ny, nz);
  return a;
}

// The kernels below move whole 4x4 blocks (HBM bound) and take 16 lanes a
// cell or face, one block entry each: every load and store of a block is one
// 128-byte run, with no more alignment than that of a double.  (One thread a
// cell touches 64 lines with each instruction.)

// Lane l < 7 of a cell forms the transmissibility of its slot l, so a cell
// takes one exp per lane; the entries see the operations of the definition in
// its order.  100x100x50: 153 us (5.9 TB/s of blocks read and written), 333 us
// with one thread a cell.
__global__ __launch_bounds__(256) void k_assemble(int nx, int ny, int nz, const double *__restrict__ logk, double kvkh,
                                                   double tscale, const double *__restrict__ Mf,
                                                   const double *__restrict__ Mb, const double *__restrict__ B,
                                                   double dt, int nw, const int32_t *__restrict__ wc,
                                                   const double *__restrict__ wu, const int32_t *__restrict__ rp,
                                                   double *__restrict__ vals) {
  const int64_t nxy = (int64_t)nx * ny, n = nxy * nz;
  const int64_t c = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
  if (c >= n) return;                                   // whole groups of 16
  const int e = threadIdx.x & 15, base = (threadIdx.x & 63) & ~15;
  const cell_at a = cell_of(c, nx, ny, nz);
  const int64_t p0 = rp[c];
  // every block's entry at once, from the accumulation block off the grid
  const double *Bc = B + 16 * c;
  double m[7];
#pragma unroll
  for (int s = 0; s < 7; ++s) {
    const double *M = Bc;
    if (s != 3 && ((a.in >> s) & 1u))
      M = s > 3 ? Mf + ((int64_t)axis_of(s) * n + c) * 16
                : Mb + ((int64_t)axis_of(s) * n + nbr_of(c, s, nx, nxy)) * 16;
    m[s] = M[e];
  }
  const bool in = e < 7 && ((a.in >> e) & 1u);
  const double kq = exp(logk[in ? nbr_of(c, e, nx, nxy) : c]);
  const double kc = __shfl(kq, base + 3, 64);
  double pa = e < 3 ? kq : kc, pb = e < 3 ? kc : kq;    // lower-numbered cell first
  if (e == 0 || e == 6) { pa = kvkh * pa; pb = kvkh * pb; }
  const double T = tscale * (((2.0 * pa) * pb) / (pa + pb));
  double acc = m[3] / dt;
  int64_t p = p0, diagpos = p0;
#pragma unroll
  for (int s = 0; s < 7; ++s) {
    const double Ts = __shfl(T, base + s, 64);
    if (!((a.in >> s) & 1u)) continue;
    if (s == 3) { diagpos = p++; continue; }
    const double t = Ts * m[s];
    vals[16 * p + e] = -t;
    acc = acc + t;
    ++p;
  }
  const int w = well_of(nw, wc, c);
  if (w >= 0) {
    const double ws = wu[w] * kc;
    if (ws != 0.0 && e % 5 == 0) acc = acc + ws;
  }
  vals[16 * diagpos + e] = acc;
}

// G = -lambda_i x_j^T for every stored block (i,j), caller layout: a row's
// blocks are one run, at the closed-form row start.  100x100x50: 108 us (4.5
// TB/s, written), 222 us slot by slot through an index array.
__global__ __launch_bounds__(256) void k_grad_vals(int nx, int ny, int nz, const double *__restrict__ lam,
                                                    const double *__restrict__ x, double *__restrict__ G) {
  const int64_t nxy = (int64_t)nx * ny, n = nxy * nz;
  const int64_t c = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
  if (c >= n) return;
  const int e = threadIdx.x & 15, r = e >> 2, col = e & 3;
  const csr7_row w = csr7_of((uint32_t)c, (uint32_t)nx, (uint32_t)ny, (uint32_t)nz);
  const double l = lam[4 * c + r];
  double xq[7];
#pragma unroll
  for (int s = 0; s < 7; ++s) xq[s] = x[4 * (((w.mask >> s) & 1u) ? nbr_of(c, s, nx, nxy) : c) + col];
  double *o = G + 16 * (int64_t)w.start + e;
#pragma unroll
  for (int s = 0; s < 7; ++s)
    if ((w.mask >> s) & 1u) {
      *o = -(l * xq[s]);
      o += 16;
    }
}

// sum over the 16 lanes of a DPP row, in every lane
template <int CTRL> __device__ __forceinline__ double row_add(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum(double v) {
  v = row_add<0x128>(v);                                // row_ror:8, 4, 2, 1
  v = row_add<0x124>(v);
  v = row_add<0x122>(v);
  return row_add<0x121>(v);
}

// dJ/dlog k_c = sum over the faces of c of dT/dlog k_c * (G : dA/dT)
//             + u_c k_c trace(G_cc) at wells
// G : dA/dT is the face's, the same from either side: a workgroup takes a tile
// of cells, forms it once for each face of the tile (16 lanes a face: four
// blocks of G, two of M), and sums the faces of its cells from LDS.  The
// tile's outer faces are formed by two tiles (1.29 times the faces in all).
// A workgroup's faces are a chain of loads, 16 of them side by side, so a tile
// has few cells: with 8 x 4 x 2 of them 15.7 us at 20x20x20 and 210 at
// 100x100x50, with 16 x 4 x 4 54 and 232, with one thread a cell that formed
// every face twice 40 and 1492.
// Along an axis with one cell in the tile the grid has one too: no faces there.
template <int TX_, int TY_, int TZ_> struct tile {
  static constexpr int TX = TX_, TY = TY_, TZ = TZ_;
  static constexpr int OX = TX > 1, OY = TY > 1, OZ = TZ > 1;           // cells around the tile
  static constexpr int FX = OX * (TX + 1) * TY * TZ, FY = OY * TX * (TY + 1) * TZ, FZ = OZ * TX * TY * (TZ + 1);
  static_assert(TX * TY * TZ == 64, "a wave's lanes at the end");
  static int64_t count(int nx, int ny, int nz) {
    return (int64_t)((nx + TX - 1) / TX) * ((ny + TY - 1) / TY) * ((nz + TZ - 1) / TZ);
  }
};

template <class TILE>
__global__ __launch_bounds__(256) void k_grad_logk(int nx, int ny, int nz, const double *__restrict__ logk, double kvkh,
                                                    double tscale, const double *__restrict__ Mf,
                                                    const double *__restrict__ Mb, int nw,
                                                    const int32_t *__restrict__ wc, const double *__restrict__ wu,
                                                    const int32_t *__restrict__ rp, const double *__restrict__ G,
                                                    double *__restrict__ g) {
  constexpr int TX = TILE::TX, TY = TILE::TY, TZ = TILE::TZ, OX = TILE::OX, OY = TILE::OY, OZ = TILE::OZ;
  constexpr int FX = TILE::FX, FY = TILE::FY, FZ = TILE::FZ, KX = TX + 2 * OX, KY = TY + 2 * OY, KZ = TZ + 2 * OZ;
  __shared__ double ef[FX + FY + FZ];
  __shared__ double kk[KZ][KY][KX];
  const int64_t nxy = (int64_t)nx * ny, n = nxy * nz;
  const int tx = (nx + TX - 1) / TX, ty = (ny + TY - 1) / TY;
  const int wg = (int)rs_wg(), bt = wg / tx, i0 = (wg - bt * tx) * TX;
  const int k0 = bt / ty * TZ, j0 = (bt - bt / ty * ty) * TY;
  if (k0 >= nz) return;                                 // past the last tile
  // permeabilities of the tile and its neighbours
  for (int t = threadIdx.x; t < KX * KY * KZ; t += 256) {
    const int a = t % KX, b = t / KX % KY, d = t / (KX * KY);
    const int i = i0 + a - OX, j = j0 + b - OY, k = k0 + d - OZ;
    if (i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz) kk[d][b][a] = exp(logk[i + nx * (j + (int64_t)ny * k)]);
  }
  // faces: below cell (a, b, d) of the tile along the axis
  const int e = threadIdx.x & 15;
#pragma unroll 2
  for (int f = threadIdx.x >> 4; f < FX + FY + FZ; f += 16) {
    const int axis = f < FX ? 0 : (f < FX + FY ? 1 : 2);
    const int t = axis == 0 ? f : (axis == 1 ? f - FX : f - FX - FY);
    const int ex = axis == 0 ? TX + 1 : TX, ey = axis == 1 ? TY + 1 : TY;
    const int q = t / ex, a = t - q * ex, d = q / ey, b = q - d * ey;
    const int i = i0 + a, j = j0 + b, k = k0 + d;       // the face's upper cell
    const int il = i - (axis == 0), jl = j - (axis == 1), kl = k - (axis == 2);
    if (il < 0 || jl < 0 || kl < 0 || i >= nx || j >= ny || k >= nz) continue;
    const int64_t hi = i + nx * (j + (int64_t)ny * k), lo = il + nx * (jl + (int64_t)ny * kl);
    const unsigned inl = slots_in(il, jl, kl, nx, ny, nz), inh = slots_in(i, j, k, nx, ny, nz);
    const double *Gl = G + 16 * (int64_t)rp[lo] + e, *Gh = G + 16 * (int64_t)rp[hi] + e;
    const int sd = 4 + axis, su = 2 - axis;             // lower cell's slot up, upper cell's slot down
    const double gll = Gl[16 * __popc(inl & 7u)], glh = Gl[16 * __popc(inl & ((1u << sd) - 1u))];
    const double ghh = Gh[16 * __popc(inh & 7u)], ghl = Gh[16 * __popc(inh & ((1u << su) - 1u))];
    const int64_t mo = ((int64_t)axis * n + lo) * 16 + e;
    const double v = row_sum((gll - glh) * Mf[mo] + (ghh - ghl) * Mb[mo]);
    if (e == 0) ef[f] = v;
  }
  __syncthreads();
  const int a = threadIdx.x % TX, b = threadIdx.x / TX % TY, d = threadIdx.x / (TX * TY);
  const int i = i0 + a, j = j0 + b, k = k0 + d;
  if (d >= TZ || i >= nx || j >= ny || k >= nz) return;   // the first wave takes the cells
  const int64_t c = i + nx * (j + (int64_t)ny * k);
  const unsigned in = slots_in(i, j, k, nx, ny, nz);
  const double kc = kk[d + OZ][b + OY][a + OX];
  double acc = 0.0;
#pragma unroll
  for (int s = 0; s < 7; ++s) {
    if (s == 3 || !((in >> s) & 1u)) continue;
    const int axis = axis_of(s), up = s > 3;
    const int fa = a + (axis == 0 && up), fb = b + (axis == 1 && up), fd = d + (axis == 2 && up);
    const int f = axis == 0 ? fa + (TX + 1) * (fb + TY * fd)
                            : (axis == 1 ? FX + fa + TX * (fb + (TY + 1) * fd) : FX + FY + fa + TX * (fb + TY * fd));
    const int sg = up ? 1 : -1;
    const double kq = kk[d + OZ + (axis == 2) * sg][b + OY + (axis == 1) * sg][a + OX + (axis == 0) * sg];
    const double sc = tscale * (axis == 2 ? kvkh : 1.0);
    const double den = (kc + kq) * (kc + kq);
    const double dT = sc * 2.0 * kc * kq * kq / den;
    acc = acc + dT * ef[f];
  }
  const int w = well_of(nw, wc, c);
  if (w >= 0) {
    const double *Gcc = G + 16 * ((int64_t)rp[c] + __popc(in & 7u));
    acc = acc + wu[w] * kc * (Gcc[0] + Gcc[5] + Gcc[10] + Gcc[15]);
  }
  g[c] = acc;
}

}  // namespace

extern "C" rs_status rs_assemble(int nx, int ny, int nz, const double *d_logk, double kvkh, double tscale,
                                 const double *d_Mf, const double *d_Mb, const double *d_B, double dt,
                                 int nw, const int32_t *d_wcell, const double *d_wu,
                                 const int32_t *d_row_ptr, double *d_vals, void *stream) {
  if (!rs_grid_dims_ok(nx, ny, nz) || nw < 0 || !d_logk || !d_Mf || !d_Mb || !d_B || !d_row_ptr || !d_vals ||
      (nw > 0 && (!d_wcell || !d_wu)) || !(dt > 0.0))
    return RS_E_ARG;
  int64_t n = (int64_t)nx * ny * nz;
  k_assemble<<<rs_grid(16 * n), RS_BLOCK, 0, rs_stream(stream)>>>(nx, ny, nz, d_logk, kvkh, tscale, d_Mf, d_Mb, d_B,
                                                             dt, nw, d_wcell, d_wu, d_row_ptr, d_vals);
  RS_HIP(hipGetLastError());
  return RS_OK;
}

extern "C" rs_status rs_grad_vals(rs_bsr A, const double *d_lambda, const double *d_x, double *d_G,
                                  void *stream) {
  if (!A || !d_lambda || !d_x || !d_G) return RS_E_ARG;
  const grid3 &g = A->g;
  k_grad_vals<<<rs_grid(16 * g.n), RS_BLOCK, 0, rs_stream(stream)>>>(g.nx, g.ny, g.nz, d_lambda, d_x, d_G);
  RS_HIP(hipGetLastError());
  return RS_OK;
}

extern "C" rs_status rs_grad_logk(int nx, int ny, int nz, const double *d_logk, double kvkh, double tscale,
                                  const double *d_Mf, const double *d_Mb, int nw, const int32_t *d_wcell,
                                  const double *d_wu, const int32_t *d_row_ptr, const double *d_G,
                                  double *d_g, void *stream) {
  if (!rs_grid_dims_ok(nx, ny, nz) || nw < 0 || !d_logk || !d_Mf || !d_Mb || !d_row_ptr || !d_G || !d_g ||
      (nw > 0 && (!d_wcell || !d_wu)))
    return RS_E_ARG;
  auto run = [&](auto t) {
    using TILE = decltype(t);
    k_grad_logk<TILE><<<rs_wgs(TILE::count(nx, ny, nz)), 256, 0, rs_stream(stream)>>>(
        nx, ny, nz, d_logk, kvkh, tscale, d_Mf, d_Mb, nw, d_wcell, d_wu, d_row_ptr, d_G, d_g);
  };
  // Grids one cell thick in y, in x, or in two directions take tiles in their
  // own shape.  With a thread per cell, tiles of 16 x 4 x 4 and now: 500x1x500
  // 482, 124 and 67 us; 1x400x700 566, 585 and 73; 300000x1x1 268, 395 and 37;
  // 1x300000x1 275, 1494 and 35; 1x1x300000 285, 1619 and 43.
  if (ny == 1 && nz == 1) run(tile<64, 1, 1>{});
  else if (nx == 1 && nz == 1) run(tile<1, 64, 1>{});
  else if (nx == 1 && ny == 1) run(tile<1, 1, 64>{});
  else if (nx == 1) run(tile<1, 8, 8>{});
  else if (ny == 1) run(tile<8, 1, 8>{});
  else run(tile<8, 4, 2>{});
  RS_HIP(hipGetLastError());
  return RS_OK;
}
