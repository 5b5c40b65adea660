// ras.hip -- second stage as zero-overlap restricted additive Schwarz (RAS)
// with the xy-layers of the grid as subdomains and block ILU(0) inside each
// layer (Section "Preconditioners": RAS with overlap 0 is block Jacobi over
// the subdomains; the subdomain problems are solved by ILU(k) or block
// ILU(k), here k = 0).  On the 7-point block pattern in natural order block
// ILU(0) only modifies the diagonal blocks, so it is DILU; restricted to a
// layer the stencil is the in-plane 5-point one.
//
// Layers are independent.  Inside a layer the recurrences run over the lines
// i + j = lambda (nx + ny - 1 levels): the thread group of line j handles
// cell (lambda - j, j) at level lambda, reads the previous level's values of
// its own line and of line j-1 (j+1 backward) from LDS, and one barrier
// separates the levels.  The factorisation gives each layer one workgroup,
// which never waits on another; the sweeps split a layer into strips of lines,
// one workgroup each, that hand the boundary line's values to the next strip
// level by level.
// The factorisation uses a quad of lanes per cell in FP64.
//
// The sweeps are written with D^{-1} folded in, which is the same operator
// in exact arithmetic:
//   forward   y = rh - Lh_y y_{c-nx} - Lh_x y_{c-1},   rh = D^{-1} r~2,
//   backward  z = y  - Uh_x z_{c+1}  - Uh_y z_{c+nx},
// with Lh = D^{-1} L and Uh = D^{-1} U formed once at set-up.  Their operands
// are stored level by level ("wavefront order": within a layer, by lambda,
// then by j), so the cells of one level are contiguous in memory; rh is
// formed (and permuted) by an elementwise pass over the whole grid.
//
// Layout: A~ blocks by stencil slot t7[7][n][16] (slots -z -y -x self +x +y
// +z, zeros off-grid), D^{-1} blocks dinv2[n][16]; scaled blocks
// blk[2][n][2][16] (Lh_y, Lh_x; Uh_x, Uh_y) in wavefront order; vectors [n][4];
// all in the preconditioner's precision.
#include "rs_internal.h"
#include <math.h>
#include <algorithm>
#include <type_traits>

namespace {
#pragma clang fp contract(off)
#include "block4.h"
#pragma clang fp contract(fast)
#include "quad4.h"
#include "quadinv.h"
#include "reduce.h"

// ---- wavefront order --------------------------------------------------------
// Number of cells (i, j) of an nx x ny layer with i + j < lambda.
__device__ __forceinline__ int64_t tri(int64_t x) { return x > 0 ? x * (x + 1) / 2 : 0; }
__device__ __forceinline__ int64_t wf_off(int lam, int nx, int ny) {
  return tri(lam) - tri(lam - nx) - tri(lam - ny) + tri(lam - nx - ny);
}
__device__ __forceinline__ int wf_jlo(int lam, int nx) { return max(0, lam - nx + 1); }
// position of cell (i, j) of its layer in wavefront order
__device__ __forceinline__ int64_t wf_pos(int i, int j, int nx, int ny) {
  return wf_off(i + j, nx, ny) + (j - wf_jlo(i + j, nx));
}

// ---- right-hand side of the forward sweep, per (cell, block row) ------------
// rh = D^{-1} (r~ - A~[:,0] x_p) in wavefront order, and x_p permuted alike.
// x_p carries nx*ny zero guard entries on each side, so every stencil
// neighbour is in bounds, and off-grid column-0 entries are zero.
// Per tile of RI x RJ cells of a layer (4 lanes per cell, one workgroup of
// 4*RI*RJ threads): the results are staged in LDS in the tile's own
// wavefront order, in which the cells of one anti-diagonal of the tile are
// consecutive in the layer's wavefront order too, and written back as runs
// of up to min(RI, RJ) cells instead of one scattered cell per quad.
// tickets: the ticket counters of the sweeps that follow on the stream, zeroed
// here.
constexpr int RAS_TICKETS = 5, RAS_CTL = 8;   // one per sweep of an apply; the error word after them
constexpr int RI = 16, RJ = 16;
template <class T>
__global__ __launch_bounds__(4 * RI * RJ) void k_ras_in_tile(int nx, int ny, int64_t n, const T *__restrict__ rt,
                                                             const T *__restrict__ col0, const T *__restrict__ xp,
                                                             const T *__restrict__ dinv2, T *__restrict__ rh,
                                                             T *__restrict__ xpw, int *__restrict__ tickets) {
  __shared__ T so[RI * RJ][4];
  if (blockIdx.x == 0 && threadIdx.x < RAS_TICKETS) tickets[threadIdx.x] = 0;
  __shared__ T sx[RI * RJ];
  __shared__ int sab[RI * RJ];
  const int tx = (nx + RI - 1) / RI, ty = (ny + RJ - 1) / RJ;
  const int layer = blockIdx.x / (tx * ty), tt = blockIdx.x - layer * (tx * ty);
  const int i0 = (tt % tx) * RI, j0 = (tt / tx) * RJ;
  const int ni = min(RI, nx - i0), nj = min(RJ, ny - j0);      // this tile's extent
  const int64_t nxy = (int64_t)nx * ny;
  const int tid = threadIdx.x, row = tid & 3, q = tid >> 2;
  const int a = q % RI, b = q / RI;
  if (a < ni && b < nj) {
    const int64_t c = layer * nxy + (int64_t)(j0 + b) * nx + (i0 + a);
    const int64_t off[7] = {-nxy, -(int64_t)nx, -1, 0, 1, (int64_t)nx, nxy};
    T col[8], dv[4];
    ld8v(col0 + c * 32 + 8 * row, col);
    ld4v(dinv2 + c * 16 + 4 * row, dv);
    T v = rt[4 * c + row];
#pragma unroll
    for (int sl = 0; sl < 7; ++sl) v = v - col[sl] * xp[c + off[sl]];
    const T o = quad_mv<T>(dv, v);
    const int w = (int)wf_pos(a, b, ni, nj);                   // tile-local wavefront index
    so[w][row] = o;
    if (row == 0) {
      sx[w] = xp[c];
      sab[w] = a | (b << 16);
    }
  }
  __syncthreads();
  if (q < ni * nj) {
    const int ab = sab[q], aa = ab & 0xffff, bb = ab >> 16;
    const int64_t p = layer * nxy + wf_pos(i0 + aa, j0 + bb, nx, ny);
    rh[4 * p + row] = so[q][row];
    if (row == 0) xpw[p] = sx[q];
  }
}

// ---- scaled blocks for the sweeps, per (cell, block row) ---------------------
// blk[b / 2][p][b % 2] = D_c^{-1} A~_{c, nb(b)} for b = 0..3: -y, -x, +x, +y
// (slots 1, 2, 4, 5), at the cell's wavefront position p: the two blocks that
// a sweep reads lie side by side; FP64 products rounded once.
template <class T>
__global__ __launch_bounds__(256) void k_ras_scale(int nx, int ny, int64_t n, const T *__restrict__ t7,
                                                   const T *__restrict__ dinv2, T *__restrict__ blk) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 4 * n) return;
  const int64_t nxy = (int64_t)nx * ny, c = t >> 2;
  const int row = (int)(t & 3);
  double dv[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) dv[m] = (double)dinv2[c * 16 + 4 * row + m];
  const int64_t k = c / nxy, rem = c - k * nxy;
  const int j = (int)(rem / nx), i = (int)(rem - (int64_t)j * nx);
  const int64_t p = k * nxy + wf_pos(i, j, nx, ny);
  const int slot[4] = {1, 2, 4, 5};
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const T *a = t7 + ((int64_t)slot[b] * n + c) * 16;
    T o[4];
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
      double v = 0.0;
#pragma unroll
      for (int m = 0; m < 4; ++m) v = fma(dv[m], (double)a[4 * m + cc], v);
      o[cc] = (T)v;
    }
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) blk[((b >> 1) * n + p) * 32 + 16 * (b & 1) + 4 * row + cc] = o[cc];
  }
}

template <class T> struct vec4t;
template <> struct vec4t<float> { typedef float4 type; };
template <> struct vec4t<double> { typedef double4 type; };

// The loads that refill a level's registers must come after the level's last
// use of them.  Loads from read-only restrict arguments are free to move, and
// once hoisted above that use the registers rotate through copies that wait
// for every load in flight; an empty asm statement that takes the level's
// result and "changes" the refill's line index pins the order (it emits no
// instruction).
template <class T> __device__ __forceinline__ void order_after(int &idx, T tok) {
  asm volatile("" : "+v"(idx) : "v"(tok));
}

// ---- factorisation, per layer: D_c = A~_cc - sum_{q in {c-nx, c-1}} A~_cq D_q^{-1} A~_qc
// A quad of lanes per cell, lane r holding block row r, computes in FP64
// (lines j = q + LW*u for quad q, U passes): the Schur terms and the inverse of
// quadinv.h, element by element the operations of the single-thread form.
// Bound by the chain of one cell: 1.6 us per level with one wave per SIMD, of
// which the four pivot steps are most.  Reading the pivot rows by DPP took the
// pass from 556 to 425 us at 100x100x50 and from 1388 to 1123 us at
// 200x200x100 (FP32); loads two levels ahead, one barrier per level, and the
// two Schur terms side by side gave nothing more.  D^{-1} blocks
// are rounded to the stored precision before the next cells use them; both
// neighbours' D^{-1} (cell before in x: same line, previous level; before in
// y: line j-1) come from an LDS slot per line, with a barrier after the
// reads of a level and one after its writes.  One writer wave copies the
// D^{-1} blocks of level lambda-1 from LDS to global memory while level
// lambda is computed.
// diag (optional, [n][16]) replaces the diagonal blocks A~_cc of t7: the
// overlapping RAS factors a layer whose diagonal already carries the Schur
// term of the layer below.
template <class T, int U>
__global__ __launch_bounds__(1024) void k_ras_setup(int nx, int ny, int64_t n, int LW, const T *__restrict__ t7,
                                                    const T *__restrict__ diag, T *__restrict__ dinv2,
                                                    int *__restrict__ flag) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) unsigned char smem[];
  T *ring = (T *)smem;                                  // [ny][16]
  const int tid = threadIdx.x;
  const bool compute = tid < 4 * LW;                    // wave-uniform (4 LW is a multiple of 64)
  const int64_t nxy = (int64_t)nx * ny, cl = nxy * blockIdx.x;
  const int Lv = nx + ny - 1;
  if (!compute) {
    const int w = tid - 4 * LW;
    auto write_level = [&](int m) {
      if (m < 0 || m >= Lv) return;
      const int jlo = max(0, m - nx + 1), jhi = min(ny - 1, m);
      for (int j = jlo + w; j <= jhi; j += 64) {
        const int64_t c = cl + (int64_t)j * nx + (m - j);
#pragma unroll
        for (int e = 0; e < 16; e += 4)
          *(typename vec4t<T>::type *)(dinv2 + c * 16 + e) = *(const typename vec4t<T>::type *)(ring + j * 16 + e);
      }
    };
    for (int lam = 0; lam < Lv; ++lam) {
      write_level(lam - 1);
      __syncthreads();
      __syncthreads();
    }
    write_level(Lv - 1);
    return;
  }
  const int q = tid >> 2, r = tid & 3, wq = (tid & 63) & ~3;
  const T *Ad = diag ? diag : t7 + 3 * n * 16, *Ay = t7 + 1 * n * 16, *Ax = t7 + 2 * n * 16;
  const T *Upx = t7 + 4 * n * 16, *Upy = t7 + 5 * n * 16;
  // this lane's row of A~_cc, A~_{c,c-nx}, A~_{c,c-1}, A~_{c-nx,c}, A~_{c-1,c}:
  // one level ahead with one pass, loaded at use with several
  T pre[5][4];
  auto load = [&](int lam, int u, T (&p)[5][4]) {
    const int j = min(q + LW * u, ny - 1);
    const int i = min(max(lam - j, 0), nx - 1);
    const int64_t c = cl + (int64_t)j * nx + i;
    const int64_t qy = j > 0 ? c - nx : c, qx = i > 0 ? c - 1 : c;
    ld4v(Ad + c * 16 + 4 * r, p[0]);
    ld4v(Ay + c * 16 + 4 * r, p[1]);
    ld4v(Ax + c * 16 + 4 * r, p[2]);
    ld4v(Upy + qy * 16 + 4 * r, p[3]);
    ld4v(Upx + qx * 16 + 4 * r, p[4]);
  };
  if constexpr (U == 1) load(0, 0, pre);
  int bad = 0;
  T orow[U][4];
  int ok[U];
  for (int lam = 0; lam < Lv; ++lam) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = q + LW * u, i = lam - j;
      T a[5][4];
      if constexpr (U == 1) {
#pragma unroll
        for (int b = 0; b < 5; ++b)
#pragma unroll
          for (int cc = 0; cc < 4; ++cc) a[b][cc] = pre[b][cc];
      } else {
        load(lam, u, a);
      }
      if (j < ny && i >= 0 && i < nx) {                 // the same for the four lanes of the cell
        double Lr[4], Rr[4];
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) Lr[cc] = (double)a[0][cc];
        T dq[4];                                        // -y, then -x (ascending column)
        if (j > 0) {
          ld4v(ring + (j - 1) * 16 + 4 * r, dq);
          quad_schur<T>(Lr, dq, a[3], a[1]);
        }
        if (i > 0) {
          ld4v(ring + j * 16 + 4 * r, dq);
          quad_schur<T>(Lr, dq, a[4], a[2]);
        }
        int mine;
        bad |= quad_inverse(Lr, Rr, r, wq, mine);
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) orow[u][cc] = (T)Rr[cc];
        ok[u] = mine;
      }
      if constexpr (U == 1) load(lam + 1, 0, pre);
    }
    __syncthreads();                                    // level lam-1 reads done
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = q + LW * u, i = lam - j;
      if (j < ny && i >= 0 && i < nx) {
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) ring[j * 16 + 4 * ok[u] + cc] = orow[u][cc];
      }
    }
    __syncthreads();                                    // level lam visible
  }
  if (bad) atomicOr(flag, bad);
}

// ---- sweeps -----------------------------------------------------------------
//   forward   y = rh - Lh_y y_{c-nx} - Lh_x y_{c-1}
//   backward  z = y - Uh_x z_{c+1} - Uh_y z_{c+nx}, output z + Pi_p x_p (x_p
//             added to unknown 0) in natural order
// A layer is split into S strips of H consecutive lines, one workgroup each.
// A quad of lanes owns a line; lane r owns block row r.  A strip needs, at
// every level, the value of the line just before it (after it, backward)
// computed one level earlier by the neighbouring strip:
//   - the writer wave publishes its boundary line, level by level, as 64-bit
//     words (launch tag << 32 | 32 bits of the value), with device-scope stores;
//   - the poller wave loads the neighbour's words 8 levels at a time, polls
//     those whose tag does not match yet, and puts each level's value into the
//     ghost slot of the LDS ring, ready for the level;
//   - workgroups take tickets in dependency order (every strip of a layer
//     after the one it reads), so a workgroup only waits on workgroups that
//     are already running; every wait is bounded, and a time-out latches an
//     error word that the host turns into RS_E_HIP.
// The waves each have one kind of memory traffic, because one counter tracks
// a wave's loads and stores and with both kinds in flight a wave can only wait
// for all of them: compute waves only load, with the next P levels in flight
// in registers; the writer only stores; the poller only loads words.
// Bound, on small and middling layers, by the chain of a level (LDS read, four
// dependent FMAs, LDS write, barrier) and by the instructions a wave issues
// between two barriers, one in 4 to 5 cycles: the level's place in wavefront
// order is a scalar that advances by a difference (ras_cursor), the two blocks
// of a cell lie side by side, and a line's own previous value comes by DPP.
// Both sweeps, against the kernels before these (per-lane addresses formed
// anew each level; strips of up to 224 lines, a layer per workgroup above):
// FP32 157 -> 97 us at 100x100x50, 398 -> 323 at 200x200x100 (1.3 GB, 4.0
// TB/s), 930 -> 800 at 256x256x160; FP64 342 -> 277 at 161x143x67.
// The level count is padded to a multiple of P and every load is issued
// unconditionally at a clamped (in-bounds) address, with the terms of inactive
// cells dropped by selects: then every path through a level issues the same
// loads, and the compiler waits only for the level's own data.
constexpr int RAS_SPIN_LIMIT = 1 << 20;     // polls with a short sleep: about a second
constexpr int RAS_H = 48;                   // most lines of a strip (at most 64: the writer's lanes)
constexpr int RAS_T = 4 * RAS_H + 128;      // most threads: compute, writer, poller

// A value in FP64 crosses strips as two words, high half first, each with the
// tag: words of value r of column i: [W r, W r + W), W = 1 or 2.
template <class T> struct ras_nw { static constexpr int W = sizeof(T) / 4; };
__device__ __forceinline__ void ras_put(uint64_t *p, uint32_t v, uint32_t tag) {
  __hip_atomic_store(p, ((uint64_t)tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ras_put_v(uint64_t *p, float v, uint32_t tag) { ras_put(p, __float_as_uint(v), tag); }
__device__ __forceinline__ void ras_put_v(uint64_t *p, double v, uint32_t tag) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  ras_put(p, (uint32_t)(b >> 32), tag);
  ras_put(p + 1, (uint32_t)b, tag);
}
// the low halves of words w, loaded from p earlier, once every tag is `tag`:
// re-read (bounded) until they match; false on time-out
template <int W>
__device__ __forceinline__ bool ras_get(uint64_t *p, const uint64_t (&w)[W], uint32_t tag, uint32_t (&v)[W],
                                        bool &failed) {
  for (int q = 0; q < W; ++q) {
    uint64_t x = w[q];
    int spins = 0;
    while ((uint32_t)(x >> 32) != tag) {
      if (failed || ++spins > RAS_SPIN_LIMIT) { failed = true; return false; }
      __builtin_amdgcn_s_sleep(1);
      x = __hip_atomic_load(p + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    v[q] = (uint32_t)x;
  }
  return true;
}
__device__ __forceinline__ float ras_value(const uint32_t (&v)[1]) { return __uint_as_float(v[0]); }
__device__ __forceinline__ double ras_value(const uint32_t (&v)[2]) {
  return __longlong_as_double((long long)(((uint64_t)v[0] << 32) | v[1]));
}

// word of the boundary value (row r) of strip s of layer k at column i
__device__ __forceinline__ int64_t ras_xword(int k, int s, int S, int nx, int i) {
  return (((int64_t)k * S + s) * nx + i) * 4;
}

// Place of a level in wavefront order, all scalar: line j's cell of level lam
// is at base + j, for the lines [jlo, jhi] of the level; levels past the
// layer's ends stay at its last (first) level.
struct ras_cursor {
  int lam, jlo, jhi;
  int64_t base;
  __device__ __forceinline__ void set(int64_t cl, int l, int nx, int ny) {
    lam = l;
    jlo = max(0, l - nx + 1);
    jhi = min(ny - 1, l);
    base = cl + wf_off(l, nx, ny) - jlo;
  }
  __device__ __forceinline__ void up(int nx, int ny) {
    if (lam >= nx + ny - 2) return;
    ++lam;
    const int lo = max(0, lam - nx + 1);
    base += jhi + 1 - lo;
    jlo = lo;
    jhi = min(ny - 1, lam);
  }
  __device__ __forceinline__ void down(int nx, int ny) {
    if (lam <= 0) return;
    --lam;
    const int hi = min(ny - 1, lam);
    base += jlo - hi - 1;
    jlo = max(0, lam - nx + 1);
    jhi = hi;
  }
};

// u = sum_m a[m] v_m, the 4-vector v spread over the quad, as dot4
template <class T> __device__ __forceinline__ T quad_dot(const T (&a)[4], T v) {
  T u = 0;
  u = fma(a[0], qb<0>(v), u);
  u = fma(a[1], qb<1>(v), u);
  u = fma(a[2], qb<2>(v), u);
  return fma(a[3], qb<3>(v), u);
}

// The poller wave: words of the neighbour's boundary line, 8 steps at a time
// (32 lanes: step offset, block row), loaded 5 steps before the first of them
// is needed and checked two steps before it.  A strip so runs 9 steps behind
// its neighbour's line; with 16 at a time, 17, and both sweeps took 12 % longer
// at 100x100x50 in FP64, 6 % at 200x200x100 in FP32 (loaded 7 steps before: the
// same).  Word i = i0 + di * step, if in
// [0, nx); xw: the neighbour's words, nullptr for none.  Value of step m to
// slot `slot` of the ring buffer that step m reads.
template <class T>
__device__ __forceinline__ void ras_poll(int w, int steps, int i0, int di, int nx, uint64_t *xw, uint32_t tag,
                                         T (*gh)[4], T *ring, int RS, int slot, int *err) {
  constexpr int W = ras_nw<T>::W;
  bool failed = false;
  const int r = w & 3;
  uint64_t pend[W] = {};
  auto issue8 = [&](int m8) {
    const int i = i0 + di * (m8 + (w >> 2));
    if (!xw || w >= 32 || i < 0 || i >= nx) return;
#pragma unroll
    for (int q = 0; q < W; ++q)
      pend[q] = __hip_atomic_load(xw + W * (4 * (int64_t)i + r) + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto finish8 = [&](int m8) {
    const int m = m8 + (w >> 2), i = i0 + di * m;
    if (!xw || w >= 32 || i < 0 || i >= nx) return;
    uint32_t v[W] = {};
    if (!ras_get<W>(xw + W * (4 * (int64_t)i + r), pend, tag, v, failed)) atomicOr(err, 1);
    gh[m & 31][r] = ras_value(v);
  };
  T val = 0;                                            // the next step's, read one step ahead
  auto hand = [&](int m) {                              // to the buffer that step m reads
    if (w < 4) ring[((m + 1) & 1) * RS * 4 + 4 * slot + w] = val;
    val = gh[(m + 1) & 31][r];
  };
  issue8(0);
  finish8(0);
  val = gh[0][r];
  hand(0);
  __syncthreads();
  for (int m = 0; m < steps; ++m) {
    if ((m & 7) == 3) issue8(m + 5);
    if ((m & 7) == 6) finish8(m + 2);
    hand(m + 1);
    __syncthreads();
  }
}

template <class T> struct ras_fpre { T r, a1[4], a2[4]; };

template <class T, int P>
__global__ __launch_bounds__(RAS_T) void k_ras_fwd(int nx, int ny, int nz, int S, int H, int64_t n, int NC,
                                                   const T *__restrict__ blk, const T *__restrict__ rh,
                                                   T *__restrict__ y, int *__restrict__ ticket, int *__restrict__ err,
                                                   uint64_t *__restrict__ xw, uint32_t tag) {
  extern __shared__ __align__(16) unsigned char smem[];
  T *ring = (T *)smem;                                  // [2][H+2][4]: slot of line j: j - j0 + 1, slot 0 the ghost
  __shared__ int s_t;
  __shared__ T gh[32][4];                               // ghost line j0-1, by step mod 32
  const int tid = threadIdx.x;
  constexpr int W = ras_nw<T>::W;
  if (tid == 0) s_t = atomicAdd(ticket, 1);
  __syncthreads();
  const int tk = __builtin_amdgcn_readfirstlane(s_t);
  const int s = tk / nz, k = tk - s * nz;
  const int j0 = s * H, j1 = min(ny, j0 + H), RS = H + 2;
  const int64_t nxy = (int64_t)nx * ny, cl = nxy * k;
  const int Lw = nx + (j1 - j0) - 1, Lpad = (Lw + P - 1) / P * P;    // levels j0 .. j0 + Lw - 1
  if (tid >= NC + 64) {
    ras_poll<T>(tid - NC - 64, Lpad, 0, 1, nx, s > 0 ? xw + W * ras_xword(k, s - 1, S, nx, 0) : nullptr, tag, gh, ring,
                RS, 0, err);
    return;
  }
  ras_cursor cur;
  cur.set(cl, j0, nx, ny);
  if (tid >= NC) {
    const int w = tid - NC, j = j0 + w, jl = j1 - 1, wl = min(w, jl - j0) + 1;
    uint64_t *xp = s < S - 1 ? xw + W * (ras_xword(k, s, S, nx, 0) + w) : nullptr;
    __syncthreads();
    for (int m = 1; m <= Lpad; ++m) {                   // the outputs of step m - 1
      __syncthreads();
      const T *src = ring + ((m + 1) & 1) * RS * 4;
      const int lam = j0 + m - 1;
      const typename vec4t<T>::type o = *(const typename vec4t<T>::type *)(src + 4 * wl);
      const T e = src[4 * (jl - j0 + 1) + (w & 3)];
      const int i = lam - jl;
      if (xp && w < 4 && i >= 0 && i < nx) ras_put_v(xp + W * 4 * (int64_t)i, e, tag);
      if (j < j1 && (unsigned)(lam - j) < (unsigned)nx) *(typename vec4t<T>::type *)(y + 4 * (cur.base + j)) = o;
      cur.up(nx, ny);
    }
    return;
  }
  const int row = tid & 3, q = tid >> 2, j = j0 + q;
  const int sl = min(q, j1 - 1 - j0) + 1;
  const int jn = j < j1 ? nx : 0;                       // no column is active on a line past the strip
  T *slot = ring + 4 * sl;
  ras_fpre<T> R[P];
  auto load = [&](ras_fpre<T> &p, T tok) {
    int jj = j;
    order_after(jj, tok);
    const uint32_t at = (uint32_t)min(max(jj, cur.jlo), cur.jhi);
    const T *b = blk + 32 * cur.base, *v = rh + 4 * cur.base;
    p.r = v[4u * at + row];
    ld4v(b + (32u * at + 4 * row), p.a1);
    ld4v(b + (32u * at + 16 + 4 * row), p.a2);
    cur.up(nx, ny);
  };
#pragma unroll
  for (int d = 0; d < P - 1; ++d) load(R[d], (T)0);
  __syncthreads();
  T v = 0;
  for (int m0 = 0; m0 < Lpad; m0 += P) {
#pragma unroll
    for (int d = 0; d < P; ++d) {
      const int i = j0 + m0 + d - j;
      T yy[4];
      ld4v(slot + ((d + 1) & 1) * RS * 4 - 4, yy);      // the line before, or the ghost
      load(R[(d + P - 1) % P], v);                      // into the previous level's, while the read is under way
      const T ty = dot4(R[d].a1, yy), tx = quad_dot(R[d].a2, v);
      v = R[d].r;
      v = j > 0 ? v - ty : v;
      v = i > 0 ? v - tx : v;
      if ((unsigned)i < (unsigned)jn) slot[(d & 1) * RS * 4 + row] = v;
      __syncthreads();
    }
  }
}

template <class T> struct ras_bpre { T yc, xpc, a4[4], a5[4]; };

template <class T, int P>
__global__ __launch_bounds__(RAS_T) void k_ras_bwd(int nx, int ny, int nz, int S, int H, int64_t n, int NC,
                                                   const T *__restrict__ blk, const T *__restrict__ y,
                                                   const T *__restrict__ xpw, T *__restrict__ out,
                                                   int *__restrict__ ticket, int *__restrict__ err,
                                                   uint64_t *__restrict__ xw, uint32_t tag) {
  extern __shared__ __align__(16) unsigned char smem[];
  T *ring = (T *)smem;                                  // [2][H+2][4]: z, slot j1 - j0 + 1 the ghost
  __shared__ int s_t;
  __shared__ T gh[32][4];                               // ghost line j1, by step mod 32
  const int tid = threadIdx.x;
  constexpr int W = ras_nw<T>::W;
  if (tid == 0) s_t = atomicAdd(ticket, 1);
  __syncthreads();
  const int tk = __builtin_amdgcn_readfirstlane(s_t);
  const int st = tk / nz, k = tk - st * nz, s = S - 1 - st;     // last strip first
  const int j0 = s * H, j1 = min(ny, j0 + H), RS = H + 2, nl = j1 - j0;
  T *ob = ring + 2 * RS * 4;                            // [H][16][4]: output of line j, by column mod 16
  const int64_t nxy = (int64_t)nx * ny, cl = nxy * k;
  const int Lw = nx + nl - 1, Lpad = (Lw + P - 1) / P * P;
  const int ltop = j1 - 1 + nx - 1;                     // step m handles level ltop - m
  if (tid >= NC + 64) {
    ras_poll<T>(tid - NC - 64, Lpad, nx - 1, -1, nx, s < S - 1 ? xw + W * ras_xword(k, s + 1, S, nx, 0) : nullptr, tag,
                gh, ring, RS, nl + 1, err);
    return;
  }
  if (tid >= NC) {
    // A line's output advances by one cell a level, so eight lanes write eight
    // cells of a line in a row (128 or 256 bytes) at the level that completes
    // them, for an eighth of the lines each: stored level by level, 16 bytes to
    // each line's row, the sweep took a third longer in FP64 at 161x143x67, a
    // quarter in FP32.
    const int w = tid - NC, sub = w & 7;
    uint64_t *xp = s > 0 ? xw + W * (ras_xword(k, s, S, nx, 0) + w) : nullptr;
    __syncthreads();
    for (int m = 1; m <= Lpad; ++m) {                   // the outputs of step m - 1
      __syncthreads();
      const int lam = ltop - m + 1;
      const int q = (((lam - j0) & 7) + (w & ~7)), jq = min(q, nl - 1);
      const int i0 = lam - j0 - q, io = i0 + sub;       // a multiple of 8, and this lane's column
      const typename vec4t<T>::type z4 = *(const typename vec4t<T>::type *)(ob + (jq * 16 + (io & 15)) * 4);
      const T e = ring[((m + 1) & 1) * RS * 4 + 4 + (w & 3)];
      const int i = lam - j0;
      if (xp && w < 4 && i >= 0 && i < nx) ras_put_v(xp + W * 4 * (int64_t)i, e, tag);
      if (q < nl && i0 >= 0 && io < nx)
        *(typename vec4t<T>::type *)(out + 4 * (cl + (int64_t)(j0 + q) * nx + io)) = z4;
    }
    return;
  }
  ras_cursor cur;
  cur.set(cl, ltop, nx, ny);
  const int row = tid & 3, q = tid >> 2, j = j0 + q;
  const int sl = min(q, nl - 1) + 1;
  const int jn = j < j1 ? nx : 0;
  const T *bb = blk + 32 * n;
  T *slot = ring + 4 * sl, *oq = ob + (sl - 1) * 64 + row;
  ras_bpre<T> R[P];
  auto load = [&](ras_bpre<T> &p, T tok) {
    int jj = j;
    order_after(jj, tok);
    const uint32_t at = (uint32_t)min(max(jj, cur.jlo), cur.jhi);
    const T *b = bb + 32 * cur.base, *v = y + 4 * cur.base, *x = xpw + cur.base;
    p.yc = v[4u * at + row];
    p.xpc = x[at];
    ld4v(b + (32u * at + 4 * row), p.a4);
    ld4v(b + (32u * at + 16 + 4 * row), p.a5);
    cur.down(nx, ny);
  };
#pragma unroll
  for (int d = 0; d < P - 1; ++d) load(R[d], (T)0);
  __syncthreads();
  T z = 0;
  for (int m0 = 0; m0 < Lpad; m0 += P) {
#pragma unroll
    for (int d = 0; d < P; ++d) {
      const int i = ltop - m0 - d - j;
      T zy[4];
      ld4v(slot + ((d + 1) & 1) * RS * 4 + 4, zy);      // the line after, or the ghost
      load(R[(d + P - 1) % P], z);
      const T tx = quad_dot(R[d].a4, z), ty = dot4(R[d].a5, zy);
      z = R[d].yc;
      z = i < nx - 1 ? z - tx : z;
      z = j < ny - 1 ? z - ty : z;
      if ((unsigned)i < (unsigned)jn) {
        slot[(d & 1) * RS * 4 + row] = z;
        oq[(i & 15) * 4] = row == 0 ? z + R[d].xpc : z;
      }
      __syncthreads();
    }
  }
}

// ---- RAS with overlap 1 over the layers -------------------------------------
// The extension of layer k is the layers k-1, k, k+1; its block ILU(0) in
// natural order factors them one after another: the first with the plain
// layer factors P0, the next two with their diagonals reduced by the Schur
// term of the layer below (P1 for layer k, P2 for layer k+1).  The sweeps of
// one extension are layer sweeps joined by the couplings across z:
//   y0 = fwd(P0, r2)                            on layer k-1
//   y1 = fwd(P1, r2 - A~_{-z} y0)               on layer k
//   y2 = fwd(P2, r2 - A~_{-z} y1)               on layer k+1
//   z2 = bwd(P2, y2)                            on layer k+1
//   z  = bwd(P1, y1 - P1^{-1} A~_{+z} z2)       on layer k (kept)
// so every layer is swept three times forward and twice backward, each sweep
// over all layers at once.

// E_c = A~_cc - A~_{c,c-nxy} P_{c-nxy} A~_{c-nxy,c} (A~_cc on the first
// layer), per (cell, block row), in FP64 with the DILU's operations in its
// order: T1 = P_{c-nxy} A~_{c-nxy,c}, then row r of A~_{c,c-nxy} T1, then the
// subtraction.
template <class T>
__global__ __launch_bounds__(256) void k_ras_zdiag(int64_t n, int64_t nxy, const T *__restrict__ t7,
                                                   const T *__restrict__ P, T *__restrict__ E) {
#pragma clang fp contract(off)
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 4 * n) return;
  const int64_t c = t >> 2;
  const int r = (int)(t & 3);
  const T *Acc = t7 + (3 * n + c) * 16;
  if (c < nxy) {
#pragma unroll
    for (int b = 0; b < 4; ++b) E[c * 16 + 4 * r + b] = Acc[4 * r + b];
    return;
  }
  const int64_t q = c - nxy;
  const T *Pq = P + q * 16, *Aqc = t7 + (6 * n + q) * 16, *Acq = t7 + c * 16;
  double T1[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      double v = 0.0;
#pragma unroll
      for (int m = 0; m < 4; ++m) v = v + (double)Pq[4 * a + m] * (double)Aqc[4 * m + b];
      T1[a][b] = v;
    }
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    double v = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) v = v + (double)Acq[4 * r + m] * T1[m][b];
    E[c * 16 + 4 * r + b] = (T)((double)Acc[4 * r + b] - v);
  }
}

// The three factorisations of overlap 1 in one launch: workgroup (stage, layer)
// factors a layer as k_ras_setup does, with the diagonal reduced by the Schur
// term of the layer below in the factors of the stage before (k_ras_zdiag's
// operations and rounding), a few levels behind the workgroup that forms them.
//   - the writer wave of a stage that another one reads stores its blocks at
//     device scope and publishes the number of finished levels;
//   - the poller wave waits (bounded) until the levels below are there;
//   - the compute waves load the block rows of the layer below at device scope.
// Tickets go stage by stage, so a workgroup only waits on one that is already
// running.  One after another the stages leave most CUs idle (nz workgroups
// each) and take their chains' sum.  All three, against three launches of
// k_ras_setup and two of k_ras_zdiag: FP32 538 us for 1337 at 120x90x40, 1067
// for 2261 at 161x143x67, 1938 for 3305 at 180x220x60; FP64 631 for 1445, 1489
// for 2636 and 3402 for 4057.  (With the writer's lanes on a cell each instead
// of on consecutive words FP64 took 964, 3110 and 5409.)
constexpr int RAS1_DONE = 32;                           // ints from one level count to the next: a cache line each
template <class T> __device__ __forceinline__ void ld_row_dev(const T *p, T (&o)[4]) {
  constexpr int N = 4 * sizeof(T) / 8;
  uint64_t w[N];
#pragma unroll
  for (int e = 0; e < N; ++e)
    w[e] = __hip_atomic_load(reinterpret_cast<uint64_t *>(const_cast<T *>(p)) + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_memcpy(o, w, sizeof(o));
}
// MT: most threads, so that shorter layers have more registers.
template <class T, int MT>
__global__ __launch_bounds__(MT) void k_ras1_setup(int nx, int ny, int nz, int64_t n, int LW,
                                                     const T *__restrict__ t7, T *P0, T *P1, T *P2,
                                                     int *__restrict__ flag, int *__restrict__ ticket, int *done,
                                                     int *__restrict__ err) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) unsigned char smem[];
  T *ring = (T *)smem;                                  // [ny][16]
  __shared__ int s_t;
  const int tid = threadIdx.x, NC = 4 * LW;
  if (tid == 0) s_t = atomicAdd(ticket, 1);
  __syncthreads();
  const int tk = __builtin_amdgcn_readfirstlane(s_t);
  const int stage = tk / nz, k = tk - stage * nz;
  T *dinv = stage == 0 ? P0 : (stage == 1 ? P1 : P2);
  const T *below = stage == 1 ? P0 : P1;
  const bool chained = stage > 0 && k > 0;              // the same for the workgroup
  int *mine = done + (int64_t)tk * RAS1_DONE;
  const int64_t nxy = (int64_t)nx * ny, cl = nxy * k;
  const int Lv = nx + ny - 1;
  if (tid >= NC + 64) {                                 // poller: two levels ahead of the compute waves' loads
    const int *at = done + (int64_t)(chained ? tk - nz - 1 : tk) * RAS1_DONE;
    int have = chained ? 0 : Lv;
    bool failed = false;
    auto need = [&](int m) {
      m = min(m, Lv);
      int spins = 0;
      while (have < m && !failed) {
        have = __hip_atomic_load(const_cast<int *>(at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (have >= m) break;
        if (++spins > RAS_SPIN_LIMIT) {
          failed = true;
          if (tid == NC + 64) atomicOr(err, 1);
        }
        __builtin_amdgcn_s_sleep(1);
      }
    };
    need(2);
    __syncthreads();
    for (int lam = 0; lam < Lv; ++lam) {
      need(lam + 3);
      __syncthreads();
      __syncthreads();
    }
    return;
  }
  if (tid >= NC) {                                      // writer
    const int w = tid - NC;
    auto write_level = [&](int m) {
      if (m < 0) return;
      const int jlo = max(0, m - nx + 1), jhi = min(ny - 1, m);
      if (stage < 2) {                                  // 8 bytes a lane, a cell's words side by side
        constexpr int N = 16 * sizeof(T) / 8;
        const uint64_t *v = (const uint64_t *)ring;
        for (int x = jlo * N + w; x < (jhi + 1) * N; x += 64) {
          const int j = x / N, e = x - j * N;
          __hip_atomic_store(reinterpret_cast<uint64_t *>(dinv + (cl + (int64_t)j * nx + (m - j)) * 16) + e, v[x],
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
      }
      for (int j = jlo + w; j <= jhi; j += 64) {
        T *o = dinv + (cl + (int64_t)j * nx + (m - j)) * 16;
#pragma unroll
        for (int e = 0; e < 16; e += 4)
          *(typename vec4t<T>::type *)(o + e) = *(const typename vec4t<T>::type *)(ring + j * 16 + e);
      }
    };
    auto publish = [&](int m) {                         // levels below m are stored
      if (stage == 2) return;
      stores_done();
      if (w == 0 && m > 0) __hip_atomic_store(mine, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    __syncthreads();
    for (int lam = 0; lam < Lv; ++lam) {
      publish(lam - 1);                                 // the stores of the level before last
      write_level(lam - 1);
      __syncthreads();
      __syncthreads();
    }
    publish(Lv - 1);
    write_level(Lv - 1);
    publish(Lv);
    return;
  }
  const int q = tid >> 2, r = tid & 3, wq = (tid & 63) & ~3;
  const int j = min(q, ny - 1);
  struct rows { T v[8][4]; };
  // this lane's row of A~_cc, A~_{c,c-nx}, A~_{c,c-1}, A~_{c-nx,c}, A~_{c-1,c}
  // and, chained, of A~_{c,c-nxy}, A~_{c-nxy,c} and D^{-1} below, one level ahead
  auto load = [&](int lam, rows &p) {
    const int i = min(max(lam - j, 0), nx - 1);
    const int64_t c = cl + (int64_t)j * nx + i;
    const int64_t qy = j > 0 ? c - nx : c, qx = i > 0 ? c - 1 : c;
    ld4v(t7 + (3 * n + c) * 16 + 4 * r, p.v[0]);
    ld4v(t7 + (n + c) * 16 + 4 * r, p.v[1]);
    ld4v(t7 + (2 * n + c) * 16 + 4 * r, p.v[2]);
    ld4v(t7 + (5 * n + qy) * 16 + 4 * r, p.v[3]);
    ld4v(t7 + (4 * n + qx) * 16 + 4 * r, p.v[4]);
    if (chained) {
      ld4v(t7 + c * 16 + 4 * r, p.v[5]);
      ld4v(t7 + (6 * n + c - nxy) * 16 + 4 * r, p.v[6]);
      ld_row_dev(below + (c - nxy) * 16 + 4 * r, p.v[7]);
    }
  };
  __syncthreads();
  rows p;
  load(0, p);
  int bad = 0;
  for (int lam = 0; lam < Lv; ++lam) {
    const int i = lam - q;
    const bool act = q < ny && i >= 0 && i < nx;        // the same for the four lanes of the cell
    T orow[4] = {0, 0, 0, 0};
    int ok = r;
    if (act) {
      double Lr[4], Rr[4];
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) Lr[cc] = (double)p.v[0][cc];
      if (chained) {
        quad_schur<T>(Lr, p.v[7], p.v[6], p.v[5]);
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) Lr[cc] = (double)(T)Lr[cc];   // stored as T between the stages
      }
      T dq[4];                                          // -y, then -x (ascending column)
      if (q > 0) {
        ld4v(ring + (q - 1) * 16 + 4 * r, dq);
        quad_schur<T>(Lr, dq, p.v[3], p.v[1]);
      }
      if (i > 0) {
        ld4v(ring + q * 16 + 4 * r, dq);
        quad_schur<T>(Lr, dq, p.v[4], p.v[2]);
      }
      bad |= quad_inverse(Lr, Rr, r, wq, ok);
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) orow[cc] = (T)Rr[cc];
    }
    if (lam + 1 < Lv) load(lam + 1, p);
    __syncthreads();                                    // level lam-1 reads done
    if (act) {
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) ring[q * 16 + 4 * ok + cc] = orow[cc];
    }
    __syncthreads();                                    // level lam visible
  }
  if (bad) atomicOr(flag, bad);
}

// rh = P^{-1} (r~ - A~[:,0] x_p - A~_{c,c-nxy} yb_{c-nxy}) in wavefront order,
// with yb the forward result of the layer below (wavefront order) and no
// z term on the first layer; x_p carries nx*ny zero guards on each side.
template <class T>
__global__ __launch_bounds__(256) void k_ras1_rhs(int nx, int ny, int64_t n, const T *__restrict__ rt,
                                                  const T *__restrict__ col0, const T *__restrict__ xp,
                                                  const T *__restrict__ t7, const T *__restrict__ yb,
                                                  const T *__restrict__ P, T *__restrict__ rh) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 4 * n) return;                               // whole quads
  const int64_t nxy = (int64_t)nx * ny, c = t >> 2;
  const int row = (int)(t & 3);
  const int64_t off[7] = {-nxy, -(int64_t)nx, -1, 0, 1, (int64_t)nx, nxy};
  T col[8], dv[4];
  ld8v(col0 + c * 32 + 8 * row, col);
  ld4v(P + c * 16 + 4 * row, dv);
  T v = rt[t];
#pragma unroll
  for (int s = 0; s < 7; ++s) v = v - col[s] * xp[c + off[s]];
  const int64_t k = c / nxy, rem = c - k * nxy;
  const int j = (int)(rem / nx), i = (int)(rem - (int64_t)j * nx);
  const int64_t p = k * nxy + wf_pos(i, j, nx, ny);
  if (k > 0) {
    T a[4], yv[4];
    ld4v(t7 + c * 16 + 4 * row, a);                     // slot 0: A~_{c,c-nxy}
    ld4v(yb + 4 * (p - nxy), yv);
    v = v - dot4(a, yv);
  }
  rh[4 * p + row] = quad_mv<T>(dv, v);
}

// y = y - P^{-1} A~_{c,c+nxy} za_{c+nxy} on every layer but the last; y in
// wavefront order, za (the backward result of the layer above) natural.
template <class T>
__global__ __launch_bounds__(256) void k_ras1_up(int nx, int ny, int nz, int64_t n, const T *__restrict__ t7,
                                                 const T *__restrict__ za, const T *__restrict__ P,
                                                 T *__restrict__ y) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 4 * n) return;                               // whole quads
  const int64_t nxy = (int64_t)nx * ny, c = t >> 2;
  const int row = (int)(t & 3);
  const int64_t k = c / nxy;
  if (k >= nz - 1) return;                              // the same for the quad
  const int64_t rem = c - k * nxy;
  const int j = (int)(rem / nx), i = (int)(rem - (int64_t)j * nx);
  const int64_t p = k * nxy + wf_pos(i, j, nx, ny);
  T a[4], zv[4], dv[4];
  ld4v(t7 + (6 * n + c) * 16 + 4 * row, a);             // slot 6: A~_{c,c+nxy}
  ld4v(za + 4 * (c + nxy), zv);
  ld4v(P + c * 16 + 4 * row, dv);
  const T u = dot4(a, zv);
  y[4 * p + row] = y[4 * p + row] - quad_mv<T>(dv, u);
}

template <class T>
__global__ void k_ras_zero(int64_t m, T *__restrict__ v) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < m) v[t] = (T)0;
}

// Strips per layer: at most RAS_H = 48 lines each.  Of 16 to 96 lines, 48 (three
// compute waves) measured fastest or within 4 % of it in FP32 everywhere and in
// FP64 on large grids: both sweeps at 200x200x100 take 323 us in FP32, against
// 366 with 32 lines and 347 with 64, and 800 against 789 and 777 at
// 256x256x160; in FP64 613 against 711 and 681 at 200x200x100.  In FP64 a
// strip's operands bind it at what one CU takes in, so strips of 32 lines are
// faster while each has a CU of its own and the layer is split anyway: 122 us
// against 138 at 100x100x50, but 342 against 277 at 161x143x67 (335 strips) and
// 54 against 50 at 60x40x30 (one strip).
struct ras_shape { int S, H; };
static ras_shape ras_strips(const grid3 &g, int prec) {
  int H = RAS_H;
  if (prec == 64 && g.ny > RAS_H && (int64_t)g.nz * ((g.ny + 31) / 32) <= 256) H = 32;
  const int S = (g.ny + H - 1) / H;
  H = (g.ny + S - 1) / S;
  return {(g.ny + H - 1) / H, H};                       // every strip non-empty
}

// Whether overlap 1 chains its three factorisations: layers of at most 224 lines
// (compute, writer and poller waves fit), and 3 nz workgroups that share CUs at
// most in pairs, or, above 160 lines, whose 13 waves and more leave a CU no room
// (and FP64 too few registers), not at all.  All three, chained against one
// after another: 100x100x190 (570 workgroups) 1577 us for 1519 in FP32,
// 161x143x160 (480) 2243 for 2611 and 3252 for 3560 in FP64, 200x200x100 (300)
// 3644 for 3597 and 6337 for 4546, 200x200x60 (180) 1844 for 3339 and 3117 for
// 3975.
static bool ras1_chained(const grid3 &g, int u, int lw) {
  return u == 1 && 4 * lw + 128 <= 1024 && 3 * (int64_t)g.nz <= (lw <= 160 ? 512 : 256);
}

}  // namespace

// ---------------------------------------------------------------------------
rs_status rs_ras_check_shape(const grid3 &g, int prec) {
  // the factorisation: at most 240 lines per pass and 2 passes (FP64) or 4
  // (FP32), and one D^{-1} block per line in LDS, within 64 KiB
  int max_ny = prec == 64 ? 480 : 960;
  if (g.ny < 1 || g.ny > max_ny || g.nx < 1 || g.nz < 1) return RS_E_ARG;
  return RS_OK;
}

rs_status rs_ras_setup_run(rs_cpr_s *M, int *flag, hipStream_t s) {
  const grid3 &g = M->A->g;
  RS_TRY(rs_ras_check_shape(g, M->prec));
  const bool ov1 = M->o.smoother == RS_SM_RAS1;
  // a quad of lanes per line, at most 240 lines per pass (U passes), and
  // one writer wave: at most 1024 threads
  int u = 1;
  while ((g.ny + u - 1) / u > 240) u *= 2;            // 1, 2 or 4
  const int lw = ((g.ny + u - 1) / u + 15) / 16 * 16;
  size_t es = M->prec == 64 ? sizeof(double) : sizeof(float);
  size_t lds = es * 16 * (size_t)g.ny;
  RS_TRY(M->rblk.alloc(es * 4 * 16 * (size_t)g.n));
  RS_TRY(M->rxp.alloc(es * (size_t)g.n));
  if (ov1) {
    RS_TRY(M->rdv0.alloc(es * 16 * (size_t)g.n));
    RS_TRY(M->rdv2.alloc(es * 16 * (size_t)g.n));
    RS_TRY(M->rblk1.alloc(es * 4 * 16 * (size_t)g.n));
    RS_TRY(M->rblk2.alloc(es * 4 * 16 * (size_t)g.n));
    RS_TRY(M->ry1.alloc(es * 4 * (size_t)g.n));
    RS_TRY(M->rz2.alloc(es * 4 * (size_t)g.n));
    RS_TRY(M->rzero.alloc(es * (size_t)g.n));
  }
  {
    const ras_shape h = ras_strips(g, M->prec);
    M->rs_strips = h.S; M->rs_h = h.H;
    const size_t words = (size_t)g.nz * h.S * g.nx * 4 * (M->prec == 64 ? 2 : 1);
    RS_TRY(M->rxw.alloc(sizeof(uint64_t) * words));
    RS_TRY(M->rctl.alloc(sizeof(int) * RAS_CTL));
    RS_TRY(rs_fill32(M->rxw.p, 0, 2 * (int64_t)words, s));
    RS_TRY(rs_fill32(M->rctl.p, 0, RAS_CTL, s));
    M->repoch = 0;
  }
  auto run = [&](auto tag) -> rs_status {
    using T = decltype(tag);
    const T *t7 = M->D->t7.as<T>();
    auto factor = [&](const T *diag, T *dinv) {
      if constexpr (sizeof(T) == 8) {
        if (u == 1) k_ras_setup<T, 1><<<g.nz, 4 * lw + 64, lds, s>>>(g.nx, g.ny, g.n, lw, t7, diag, dinv, flag);
        else k_ras_setup<T, 2><<<g.nz, 4 * lw + 64, lds, s>>>(g.nx, g.ny, g.n, lw, t7, diag, dinv, flag);
      } else {
        if (u == 1) k_ras_setup<T, 1><<<g.nz, 4 * lw + 64, lds, s>>>(g.nx, g.ny, g.n, lw, t7, diag, dinv, flag);
        else if (u == 2) k_ras_setup<T, 2><<<g.nz, 4 * lw + 64, lds, s>>>(g.nx, g.ny, g.n, lw, t7, diag, dinv, flag);
        else k_ras_setup<T, 4><<<g.nz, 4 * lw + 64, lds, s>>>(g.nx, g.ny, g.n, lw, t7, diag, dinv, flag);
      }
    };
    auto scale = [&](const T *dinv, T *blk) {
      k_ras_scale<T><<<rs_grid(4 * g.n), RS_BLOCK, 0, s>>>(g.nx, g.ny, g.n, t7, dinv, blk);
    };
    if (!ov1) {
      factor(nullptr, M->dinv2.as<T>());
      scale(M->dinv2.as<T>(), M->rblk.as<T>());
    } else if (ras1_chained(g, u, lw)) {
      // P0 (plain layers), P1 (middle of each extension, the owned cells':
      // dinv2), P2 (top of each extension), chained
      int *ctl = M->rctl.as<int>();
      RS_TRY(M->rdone.alloc(sizeof(int) * (3 * (size_t)g.nz * RAS1_DONE)));
      RS_TRY(rs_fill32(M->rdone.p, 0, 3 * (int64_t)g.nz * RAS1_DONE, s));
      auto chain = [&](auto kernel) {
        kernel<<<3 * g.nz, 4 * lw + 128, lds, s>>>(g.nx, g.ny, g.nz, g.n, lw, t7, M->rdv0.as<T>(), M->dinv2.as<T>(),
                                                   M->rdv2.as<T>(), flag, ctl, M->rdone.as<int>(), ctl + RAS_TICKETS);
      };
      if (4 * lw + 128 <= 512) chain(k_ras1_setup<T, 512>);
      else if (4 * lw + 128 <= 768) chain(k_ras1_setup<T, 768>);
      else chain(k_ras1_setup<T, 1024>);
      scale(M->rdv0.as<T>(), M->rblk.as<T>());
      scale(M->dinv2.as<T>(), M->rblk1.as<T>());
      scale(M->rdv2.as<T>(), M->rblk2.as<T>());
      k_ras_zero<T><<<rs_grid(g.n), RS_BLOCK, 0, s>>>(g.n, M->rzero.as<T>());
    } else {
      // P0 (plain layers), P1 (middle of each extension, the owned cells':
      // dinv2), P2 (top of each extension).  The reduced diagonals E live in
      // the P2 scaled blocks' buffer (16 n of its 64 n entries), written only
      // after the last factorisation has read E: no pool memory is released
      // while this stream (possibly a side stream) still uses it.
      T *E = M->rblk2.as<T>();
      factor(nullptr, M->rdv0.as<T>());
      k_ras_zdiag<T><<<rs_grid(4 * g.n), RS_BLOCK, 0, s>>>(g.n, g.nxy, t7, M->rdv0.as<T>(), E);
      factor(E, M->dinv2.as<T>());
      k_ras_zdiag<T><<<rs_grid(4 * g.n), RS_BLOCK, 0, s>>>(g.n, g.nxy, t7, M->dinv2.as<T>(), E);
      factor(E, M->rdv2.as<T>());
      scale(M->rdv0.as<T>(), M->rblk.as<T>());
      scale(M->dinv2.as<T>(), M->rblk1.as<T>());
      scale(M->rdv2.as<T>(), M->rblk2.as<T>());
      k_ras_zero<T><<<rs_grid(g.n), RS_BLOCK, 0, s>>>(g.n, M->rzero.as<T>());
    }
    RS_HIP(hipGetLastError());
    return RS_OK;
  };
  if (M->prec == 64) return run(double{});
  return run(float{});
}

template <class T>
rs_status rs_ras_apply_run(rs_cpr_s *M, const T *xp, T *out, hipStream_t s) {
  const grid3 &g = M->A->g;
  const rs_dcpl_s *D = M->D;
  const bool ov1 = M->o.smoother == RS_SM_RAS1;
  // rh goes to zt, the forward result (wavefront order) to yv
  T *rh = M->zt.as<T>(), *y = M->yv.as<T>(), *xpw = M->rxp.as<T>();
  // the layer factors of the first forward sweep: P0 (dinv2 for overlap 0)
  const T *P0 = ov1 ? M->rdv0.as<T>() : M->dinv2.as<T>();
  {
    const int64_t tiles = (int64_t)g.nz * ((g.nx + RI - 1) / RI) * ((g.ny + RJ - 1) / RJ);
    // the tickets of the sweeps below are zeroed here
    int *tk = M->rctl.as<int>();
    k_ras_in_tile<T><<<(unsigned)tiles, 4 * RI * RJ, 0, s>>>(g.nx, g.ny, g.n, M->rt.as<T>(), D->col0.as<T>(), xp,
                                                             P0, rh, xpw, tk);
  }
  RS_HIP(hipGetLastError());
  // Levels in flight, and with them the workgroups that share a CU: few of them
  // stream the operands of a large grid faster than many.  At 200x200x100, FP32,
  // the forward sweep with 12 levels and three workgroups takes 27 % longer than
  // with 16 levels and one; the backward one has 12 levels and two, by the LDS
  // asked for, and takes 4 % longer with three and 14 % with 10 levels.
  constexpr int PF = sizeof(T) == 4 ? 16 : 8, PB = sizeof(T) == 4 ? 12 : 6;
  constexpr size_t two_per_cu = 56000;
  const int S = M->rs_strips, H = M->rs_h;
  const unsigned nwg = (unsigned)(g.nz * S);
  const int NC = (H + 15) / 16 * 64, nt = NC + 128;    // compute lanes in whole waves, writer, poller
  const size_t ring = sizeof(T) * 8 * (size_t)(H + 2);
  int *ticket = M->rctl.as<int>(), *err = ticket + RAS_TICKETS;
  uint64_t *xw = M->rxw.as<uint64_t>();
  // one forward sweep over all layers: blocks blk, rhs r, result yo (wavefront order)
  auto fwd = [&](const T *blk, const T *r, T *yo) {
    k_ras_fwd<T, PF><<<nwg, nt, ring, s>>>(g.nx, g.ny, g.nz, S, H, g.n, NC, blk, r, yo, ticket++, err, xw, ++M->repoch);
  };
  // one backward sweep: result + x_p (x_p in wavefront order) in natural order
  auto bwd = [&](const T *blk, const T *yi, const T *x, T *o) {
    k_ras_bwd<T, PB><<<nwg, nt, std::max(ring + sizeof(T) * 64 * (size_t)H, two_per_cu), s>>>(g.nx, g.ny, g.nz, S, H, g.n, NC, blk, yi, x, o, ticket++, err, xw,
                                               ++M->repoch);
  };
  const T *blk = M->rblk.as<T>();
  if (!ov1) {
    fwd(blk, rh, y);
    RS_HIP(hipGetLastError());
    bwd(blk, y, xpw, out);
    RS_HIP(hipGetLastError());
    return RS_OK;
  }
  const T *t7 = D->t7.as<T>();
  T *y1 = M->ry1.as<T>(), *z2 = M->rz2.as<T>();
  const unsigned gq = rs_grid(4 * g.n);
  fwd(blk, rh, y);                                                       // y0
  k_ras1_rhs<T><<<gq, RS_BLOCK, 0, s>>>(g.nx, g.ny, g.n, M->rt.as<T>(), D->col0.as<T>(), xp, t7, y,
                                        M->dinv2.as<T>(), rh);
  fwd(M->rblk1.as<T>(), rh, y1);                                         // y1
  k_ras1_rhs<T><<<gq, RS_BLOCK, 0, s>>>(g.nx, g.ny, g.n, M->rt.as<T>(), D->col0.as<T>(), xp, t7, y1,
                                        M->rdv2.as<T>(), rh);
  fwd(M->rblk2.as<T>(), rh, y);                                          // y2
  bwd(M->rblk2.as<T>(), y, M->rzero.as<T>(), z2);                        // z2 (natural order)
  k_ras1_up<T><<<gq, RS_BLOCK, 0, s>>>(g.nx, g.ny, g.nz, g.n, t7, z2, M->dinv2.as<T>(), y1);
  bwd(M->rblk1.as<T>(), y1, xpw, out);                                   // z of the owned layer
  RS_HIP(hipGetLastError());
  return RS_OK;
}

template rs_status rs_ras_apply_run<double>(rs_cpr_s *, const double *, double *, hipStream_t);
template rs_status rs_ras_apply_run<float>(rs_cpr_s *, const float *, float *, hipStream_t);
