// dilu.hip -- block ILU(0) (DILU on the 7-point block pattern) in natural
// order: factorisation and forward/backward sweeps as persistent, pipelined
// kernels.
//
// The recurrences run over hyperplanes i+j+k = const.  One launch per
// hyperplane costs a few microseconds of launch and drain each (about 1000
// launches per application at 200x200x100), so instead the grid is cut into
// bricks of x-lines (j, k) running along the whole x extent, and one workgroup
// walks its brick hyperplane by hyperplane (local level h = i + jl + kl): a
// quad of lanes per cell (one block row each), the previous level of the brick
// in an LDS ring, one barrier per level.  A brick needs, at level h, the face
// values that the bricks before it in j and in k computed at their level
// h + edge - 1.
//
// Progress and visibility across workgroups (and across XCDs, whose L2 caches
// are not coherent with each other):
//   - the only values other bricks read are the brick's outgoing faces, stored
//     with device-scope stores by a wave that does nothing but store;
//   - the sweeps' values carry a tag; the factorisation's blocks are followed,
//     once they are complete, by a level count;
//   - a wave of its own in each brick reads them with device-scope loads, as
//     often as it takes, and puts them into the ring.
//   - bricks are handed out by a ticket counter in an order where every
//     brick comes after the bricks it waits on, so a waiting workgroup only
//     ever waits on workgroups that are already running: no deadlock,
//     whatever the residency.  Each wait is bounded; on time-out the kernel
//     records an error and finishes (the host reports RS_E_HIP).
// The arithmetic per cell is the same sequence of operations as the
// definition, so results are bitwise reproducible.
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

constexpr int FL = 32;                  // a brick's level count has a cache line of its own
constexpr int SPIN_LIMIT = 1 << 20;     // polls (each a device-scope load): about a second

template <class T>
__device__ __forceinline__ void st_dev(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class T>
__device__ __forceinline__ T ld_dev(const T *p) { return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// exchange words without a tag, no level done, no error
__global__ void k_pipe_clear(int64_t words, uint64_t *__restrict__ x, int nb, int *__restrict__ done,
                             int *__restrict__ ctl) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < 4) ctl[t] = 0;
  if (t < nb) done[FL * t] = 0;
  if (t < words) x[t] = 0;
}

// ---- tagged exchange of brick faces ------------------------------------------
// A face value travels as 64-bit words (tag << 32 | 32 data bits): one word
// per FP32 value, two (low, high halves) per FP64 value.  The tag is the
// launch's epoch, so a consumer that reads its word with a device-scope load
// knows the data is current when the tag matches; stale words from earlier
// launches carry older epochs and no reset is needed.
template <class T> struct xw;
template <> struct xw<float> {
  static constexpr int W = 1;
  __device__ static void put(uint64_t *p, float v, uint32_t tag) {
    st_dev(p, (uint64_t)(((uint64_t)tag << 32) | (uint64_t)__float_as_uint(v)));
  }
  __device__ static void get(const uint64_t *p, uint64_t (&w)[W]) { w[0] = ld_dev(p); }
  __device__ static bool ready(const uint64_t (&w)[W], uint32_t tag) { return (uint32_t)(w[0] >> 32) == tag; }
  __device__ static float value(const uint64_t (&w)[W]) { return __uint_as_float((uint32_t)w[0]); }
};
template <> struct xw<double> {
  static constexpr int W = 2;
  __device__ static void put(uint64_t *p, double v, uint32_t tag) {
    uint64_t b = (uint64_t)__double_as_longlong(v);
    st_dev(p, (uint64_t)(((uint64_t)tag << 32) | (b & 0xffffffffull)));
    st_dev(p + 1, (uint64_t)(((uint64_t)tag << 32) | (b >> 32)));
  }
  __device__ static void get(const uint64_t *p, uint64_t (&w)[W]) { w[0] = ld_dev(p); w[1] = ld_dev(p + 1); }
  __device__ static bool ready(const uint64_t (&w)[W], uint32_t tag) {
    return (uint32_t)(w[0] >> 32) == tag && (uint32_t)(w[1] >> 32) == tag;
  }
  __device__ static double value(const uint64_t (&w)[W]) {
    return __longlong_as_double((long long)(((w[1] & 0xffffffffull) << 32) | (w[0] & 0xffffffffull)));
  }
};

__device__ __forceinline__ void st4v(float *p, const float *v) { *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void st4v(double *p, const double *v) {
  ((double2 *)p)[0] = make_double2(v[0], v[1]);
  ((double2 *)p)[1] = make_double2(v[2], v[3]);
}

// A sweep's brick: BJ x BK x-lines in j and in k, BK = 4 or 8 (see
// rs_dilu_prepare).  One poller wave covers both incoming faces, and a face
// has BJ lines of exchange words.
constexpr int BJ = 8;
constexpr int RG = BJ + 2;               // ring row: the brick's lines, one outside, one to spread the LDS banks
template <int BK> constexpr int ring_lines = RG * (BK + 1);

// word of the value of block row r of face cell (face f, position pos, i) of brick b
template <class T>
__device__ __forceinline__ int64_t xslot(int b, int f, int pos, int i, int nx, int r) {
  return ((((int64_t)b * 2 + f) * BJ + pos) * nx + i) * (4 * xw<T>::W) + r * xw<T>::W;
}

// brick of ticket t in an order where every brick comes after the bricks
// before it in j and in k: by J + K, then by K
__device__ __forceinline__ int64_t diag_count(int64_t d, int64_t NJ, int64_t NK) {   // bricks with J + K < d
  auto tri = [](int64_t x) { return x > 0 ? x * (x + 1) / 2 : (int64_t)0; };
  return tri(d) - tri(d - NJ) - tri(d - NK) + tri(d - NJ - NK);
}
__device__ __forceinline__ void brick_of(int t, int NJ, int NK, int &J, int &K) {
  int lo = 0, hi = NJ + NK - 2;          // the largest d with diag_count(d) <= t
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (diag_count(mid, NJ, NK) <= t) lo = mid; else hi = mid - 1;
  }
  K = max(0, lo - (NJ - 1)) + (int)(t - diag_count(lo, NJ, NK));
  J = lo - K;
}

// ---- brick order -----------------------------------------------------------------
// What the sweeps read and hand on is stored brick by brick, each brick level
// by level (h = i + jl + kl), the lines of a level by jl + kl, then kl.  Lines
// start in that order and end in it, so the lines active at a level are a run
// of it and the storage has no gaps.  A level is then one contiguous run per
// plane: in the grid's own order its 64 cells lie whole x-lines apart, in
// FP32 half of every cache line fetched for them is the next level's, they
// crowd into a few L2 channels for many nx, and the sweeps ran at half the
// speed at 200x200x100.
template <int BK> struct brick_geo {
  static constexpr int BS = BJ + BK - 2;   // levels between the first and the last line of a full brick
  int nx, bj, bk, nl;      // lines in j, in k, in all
  int64_t base;            // cells stored before the brick
  __device__ static int tri(int x) { return x > 0 ? x * (x + 1) / 2 : 0; }
  __device__ static int tet(int x) { return x > 0 ? x * (x + 1) * (x + 2) / 6 : 0; }
  // lines with jl + kl <= x, and their sum over the levels before x
  __device__ int started(int x) const { return x >= bj + bk - 2 ? nl : tri(x + 1) - tri(x + 1 - bj) - tri(x + 1 - bk); }
  __device__ int64_t begun(int64_t x) const {
    const int e = bj + bk - 1;                          // from level e - 1 on every line has started
    if (x > e) return (int64_t)(tet(e) - tet(e - bj) - tet(e - bk)) + (x - e) * nl;
    return tet((int)x) - tet((int)x - bj) - tet((int)x - bk);
  }
  // index in brick order of rank 0's cell at level h, were it active there
  // (lines that have ended are left out of the level's run)
  __device__ int64_t rank0(int h) const { return base + begun(h) - begun(h - nx) - (h >= nx ? started(h - nx) : 0); }
  __device__ int rank(int jl, int kl) const {
    const int s = jl + kl;
    return (s > 0 ? started(s - 1) : 0) + kl - max(0, s - (bj - 1));
  }
  // line of rank q
  __device__ void line(int q, int &jl, int &kl) const {
    int s = 0;
    while (s < bj + bk - 2 && started(s) <= q) ++s;
    kl = max(0, s - (bj - 1)) + q - (s > 0 ? started(s - 1) : 0);
    jl = s - kl;
  }
};
template <int BK> __device__ __forceinline__ brick_geo<BK> geo_of(int J, int K, int nx, int ny, int nz) {
  brick_geo<BK> g;
  g.nx = nx;
  g.bj = min(BJ, ny - J * BJ);
  g.bk = min(BK, nz - K * BK);
  g.nl = g.bj * g.bk;
  g.base = ((int64_t)K * BK * ny + (int64_t)g.bk * J * BJ) * nx;
  return g;
}
// a wave-uniform value that the compiler cannot see to be one
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The two passes below take 16 cells of each line of a brick per workgroup, 16
// consecutive cells of a line per wave, and read in the grid's order in whole
// cache lines.  tab[h - i0]: rank0 of the levels that the 16 cells are on.
constexpr int CH = 16;
template <int BK> __device__ __forceinline__ void level_table(const brick_geo<BK> &g, int i0, int64_t *tab) {
  const int t = threadIdx.x;
  if (t < CH + brick_geo<BK>::BS) tab[t] = g.rank0(i0 + t);
  __syncthreads();
}

// The sweeps' operands in brick order, planes -z -y -x D^{-1} +x +y +z of each
// level one after another (so that the forward sweep reads the first four and
// the backward sweep the last four), after the factorisation.
template <class T, int BK>
__global__ __launch_bounds__(256) void k_dilu_order(int nx, int ny, int nz, int NJ, int NC, int64_t n,
                                                     const T *__restrict__ t7, const T *__restrict__ dinv2,
                                                     T *__restrict__ pb) {
  __shared__ int64_t tab[CH + BJ + BK];
  const int b = blockIdx.x / NC, i0 = (int)(blockIdx.x - (unsigned)b * NC) * CH;
  const int J = b % NJ, K = b / NJ;
  const brick_geo<BK> g = geo_of<BK>(J, K, nx, ny, nz);
  level_table(g, i0, tab);
  const int row = threadIdx.x & 3, i = i0 + ((threadIdx.x >> 2) & 15);
  if (i >= nx) return;
  for (int l = threadIdx.x >> 6; l < g.nl; l += 4) {
    const int kl = l / g.bj, jl = l - kl * g.bj;
    const int h = i + jl + kl, q = g.rank(jl, kl);
    const int64_t c = (((int64_t)(K * BK + kl) * ny + J * BJ + jl) * nx + i) * 16 + 4 * row;
    // the level's active lines, and the index of its first one
    const int ended = h >= nx ? g.started(h - nx) : 0, act = g.started(h) - ended;
    const int64_t r0 = tab[h - i0], f = r0 + ended;
    T *o = pb + (7 * f + r0 + q - f) * 16 + 4 * row;
    T v[7][4];
#pragma unroll
    for (int s = 0; s < 7; ++s) ld4v(s == 3 ? dinv2 + c : t7 + s * n * 16 + c, v[s]);
#pragma unroll
    for (int s = 0; s < 7; ++s) st4v(o + (int64_t)s * act * 16, v[s]);
  }
}

// Right-hand side of the forward sweep, v = r~ - A~[:,0] x_p, and x_p, in brick
// order: apart from the sweep, whose levels depend on each other and would
// have to stream 144 bytes a cell more (in FP32).  x_p carries nx*ny zero
// guard entries on each side and off-grid column-0 entries are zero.  The
// results go through LDS and out level by level, as runs of up to a level
// (133 us in FP32 at 200x200x100, 5.3 TB/s; 195 written cell by cell).  Also zeroes the two sweeps' tickets.
template <class T, int BK>
__global__ __launch_bounds__(256) void k_dilu_rhs(int nx, int ny, int nz, int NJ, int NC, const T *__restrict__ rt,
                                                   const T *__restrict__ col0, const T *__restrict__ xp,
                                                   T *__restrict__ rhs, T *__restrict__ xpb, int *__restrict__ ctl) {
  __shared__ int64_t tab[CH + BJ + BK];
  __shared__ T sv[BJ * BK][CH][4], sx[BJ * BK][CH];     // by rank of the line
  if (blockIdx.x == 0 && threadIdx.x < 2) ctl[2 * threadIdx.x] = 0;
  const int b = blockIdx.x / NC, i0 = (int)(blockIdx.x - (unsigned)b * NC) * CH;
  const int J = b % NJ, K = b / NJ;
  const brick_geo<BK> g = geo_of<BK>(J, K, nx, ny, nz);
  level_table(g, i0, tab);
  const int row = threadIdx.x & 3, ii = (threadIdx.x >> 2) & 15, i = min(i0 + ii, nx - 1);
  const int64_t nxy = (int64_t)nx * ny;
  const int64_t nb[7] = {-nxy, -(int64_t)nx, -1, 0, 1, (int64_t)nx, nxy};
#pragma unroll 2
  for (int l = threadIdx.x >> 6; l < g.nl; l += 4) {
    const int kl = l / g.bj, jl = l - kl * g.bj;
    const int64_t c = ((int64_t)(K * BK + kl) * ny + J * BJ + jl) * nx + i;
    T col[8], x[7];
    ld8v(col0 + c * 32 + 8 * row, col);
#pragma unroll
    for (int s = 0; s < 7; ++s) x[s] = xp[c + nb[s]];
    T v = rt[4 * c + row];
#pragma unroll
    for (int s = 0; s < 7; ++s) v = v - col[s] * x[s];
    const int q = g.rank(jl, kl);
    sv[q][ii][row] = v;
    if (row == 0) sx[q][ii] = x[3];
  }
  __syncthreads();
  constexpr int NL = BJ * BK, ST = 64 / NL;             // lines of a full brick, levels per step
  const int q = (threadIdx.x >> 2) % NL;
  if (q >= g.nl) return;
  int jl, kl;
  g.line(q, jl, kl);
  for (int d = (threadIdx.x >> 2) / NL; d < CH + brick_geo<BK>::BS; d += ST) {
    const int e = d - jl - kl;
    if (e < 0 || e >= CH || i0 + e >= nx) continue;
    const int64_t o = tab[d] + q;
    rhs[4 * o + row] = sv[q][e][row];
    if (row == 0) xpb[o] = sx[q][e];
  }
}

// ---- sweeps ------------------------------------------------------------------
//   forward   y_c = D_c^{-1} (v_c - sum_{lower k} A~_ck y_k)
//   backward  z_c = y_c - D_c^{-1} sum_{upper k} A~_ck z_k, output z + Pi_p x_p
// A brick of 8 x 4 or 8 x 8 x-lines per workgroup, one barrier per level: 2 or
// 4 compute waves with a quad of lanes per cell (lane r owns block row r), a
// writer wave and a poller wave.
//   - compute: the neighbours' 4-vectors come from the previous level in an
//     LDS ring with a slot for each line just outside the brick; the operands
//     of the next P levels (five loads a level) are in flight in registers;
//   - writer: copies the previous level from LDS to global memory, the values
//     of the outgoing faces as tagged words as well (a wave's loads and stores
//     complete in order, so that stores in a compute wave would make its loads
//     wait for the slow device-scope ones);
//   - poller: one lane per value of the incoming faces (16 lines x 4); loads
//     the words D levels ahead, checks a level's tags when it is due, re-reads
//     the ones that are not there yet (bounded), puts the values into the ring.
// What bounds the sweeps is the chain of nx + ny + nz levels, a level taking
// as long as its CU takes to bring the operands in (about 45 GB/s a CU from
// HBM: 0.39 us in FP32 and 0.75 in FP64 with 64 cells), and for every brick on
// the way from corner to corner the way of a face value through memory, 2 to
// 3 us.  Forward and backward, FP32 at 200x200x100: 459 and 458 us (1395 and
// 1206 with bricks of 4 x 4 lines whose waves took the levels in turn, polled
// their faces themselves and read the grid's order; 690 and 740 with these
// waves on the grid's order); FP64 at 100x100x50: 199 and 199 (567 and 577).
template <class T> __device__ __forceinline__ void poll_faces(
    int lane, int L, int nx, bool has, int shift, const uint64_t *__restrict__ src, bool rev, T *__restrict__ slot0,
    T *__restrict__ slot1, uint32_t tag, int *__restrict__ err) {
  // level m of this lane's line is cell m - shift along x (from the far end
  // with rev); src: words of cell 0, 4 W a cell; slot0/1: ring entries of the
  // line for odd and even m
  constexpr int W = xw<T>::W, D = 8;
  bool failed = false;
  uint64_t w[D][W];
  auto at = [&](int m, int &i) {
    i = rev ? nx - 1 - (m - shift) : m - shift;
    return has && i >= 0 && i < nx;
  };
  // issued by every lane, at a clamped cell: then the number of younger loads
  // is known where a word is tested, and only its own load is waited for
  auto issue = [&](int m, uint64_t (&x)[W]) {
    int i;
    at(m, i);
    xw<T>::get(src + (int64_t)min(max(i, 0), nx - 1) * 4 * W, x);
  };
  auto deliver = [&](int m, uint64_t (&x)[W]) {
    // the words loaded D levels ago are tested outside the loop that reads
    // them again: in one loop the test would wait for every load in flight
    int i;
    const bool in = at(m, i);
    T v = xw<T>::value(x);
    if (__ballot(in && !xw<T>::ready(x, tag)) != 0) {
      uint64_t z[W];
      int spins = 0;
      do {
        if (in) xw<T>::get(src + (int64_t)i * 4 * W, z);
        if (++spins > SPIN_LIMIT) { atomicOr(err, 1); failed = true; }
      } while (__ballot(in && !xw<T>::ready(z, tag)) != 0 && !failed);
      v = xw<T>::value(z);
    }
    if (in) *((m & 1) ? slot0 : slot1) = v;
  };
#pragma unroll
  for (int d = 0; d < D; ++d) issue(d, w[d]);
  for (int m0 = 0; m0 < L; m0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      deliver(m0 + d, w[d]);
      issue(m0 + d + D, w[d]);
      __syncthreads();
    }
  }
  __syncthreads();
}

// the writer wave: level m is in LDS after the barrier that starts level m + 1
template <class T, class F> __device__ __forceinline__ void write_levels(int L, F &&write) {
  __syncthreads();
  for (int m = 0; m < L; ++m) {
    __syncthreads();
    write(m);
  }
}

// refills of a level's registers stay behind the level's last use of them
// (see the layer sweeps)
template <class T> __device__ __forceinline__ void after(int &idx, T tok) { asm volatile("" : "+v"(idx) : "v"(tok)); }

// Walks a brick's levels up (from level 0) or down (from level `top`), with a
// wave-uniform pointer to the level's vectors and one to its blocks: in the
// middle of the brick, where every line is active, a step adds constants.
template <class T, int BK> struct walk {
  const T *v, *o;          // 4-vectors and blocks of level h
  int h, first, act;       // lines ended, lines active
  __device__ void at_level(const brick_geo<BK> &g) {
    first = 0;
    act = g.nl;
    if (h < g.BS || h >= g.nx) {
      first = h >= g.nx ? g.started(h - g.nx) : 0;
      act = max((h >= 0 ? g.started(h) : 0) - first, 0);
    }
  }
  __device__ void begin(const brick_geo<BK> &g, const T *v0, const T *pb) {
    v = v0 + 4 * g.base;
    o = pb + 112 * g.base;
    h = 0;
    at_level(g);
  }
  __device__ void up(const brick_geo<BK> &g) {
    v += 4 * act;
    o += 112 * act;
    ++h;
    at_level(g);
  }
  __device__ void begin_top(const brick_geo<BK> &g, const T *v0, const T *pb, int top) {
    h = top;
    at_level(g);
    const int64_t off = g.base + (int64_t)g.nl * g.nx - act;
    v = v0 + 4 * off;
    o = pb + 112 * off;
  }
  __device__ void down(const brick_geo<BK> &g) {
    --h;
    at_level(g);
    v -= 4 * act;
    o -= 112 * act;
  }
  // index within the level for the lane of rank q; lanes without an active
  // line take a cell that is in the brick (past the last level the one before)
  __device__ int lane(int q) const { return act > 0 ? min(max(q - first, 0), act - 1) : (h < 0 ? 0 : -1); }
};

// p + e at a wave-uniform p and a 32-bit lane offset
template <class T> __device__ __forceinline__ const T *at(const T *p, int e) {
  return (const T *)((const char *)p + (int64_t)e * (int)sizeof(T));
}

template <class T> struct sweep_pre { T v, a[3][4], dv[4]; };

// The blocks that a sweep reads: pb, in brick order, or, where there is no
// memory for that copy (NAT), the planes of t7 and dinv2 in the grid's order.
template <class T> struct sweep_blocks {
  const T *pb, *t7, *dinv2;
  int64_t n;
};

template <class T, int P, int BK, bool NAT>
__global__ __launch_bounds__(4 * BJ * BK + 128) void k_fwd_pipe(int nx, int ny, int nz, int NJ, int NK, int *__restrict__ ticket,
                                                  int *__restrict__ err, uint32_t tag, uint64_t *__restrict__ xch,
                                                  sweep_blocks<T> B, const T *__restrict__ rhs,
                                                  T *__restrict__ y) {
  constexpr int NC = 4 * BJ * BK, RN = ring_lines<BK>, BS = brick_geo<BK>::BS;
  __shared__ __align__(32) T ring[2][RN][4];       // line (jl, kl) at (kl + 1) RG + jl + 1
  __shared__ int s_t;
  const int tid = threadIdx.x;
  if (tid == 0) s_t = atomicAdd(ticket, 1);
  __syncthreads();
  int J, K;
  brick_of(uni(s_t), NJ, NK, J, K);
  const int b = J + NJ * K;
  const brick_geo<BK> g = geo_of<BK>(J, K, nx, ny, nz);
  const int L = (nx + BS + 7) / 8 * 8;                  // levels, a multiple of P and of the poller's lead
  if (tid >= NC + 64) {
    // the y face before the brick (lines kl), then the z face (lines jl)
    const int lane = tid - NC - 64, r = lane & 3;
    const bool yf = lane < 4 * BK;
    const int pos = yf ? lane >> 2 : (lane >> 2) - BK;   // (lanes beyond the faces: past bj)
    const bool has = yf ? J > 0 && pos < g.bk : K > 0 && pos < g.bj;
    const int gs = !has ? 0 : (yf ? (pos + 1) * RG : pos + 1);
    // lanes without a face to read load words of their own brick
    const uint64_t *src = xch + (has ? xslot<T>(yf ? b - 1 : b - NJ, yf ? 0 : 1, pos, 0, nx, r) : xslot<T>(b, 0, 0, 0, nx, r));
    poll_faces<T>(lane, L, nx, has, pos, src, false, &ring[0][gs][r], &ring[1][gs][r], tag, err);
    return;
  }
  if (tid >= NC) {
    const int lane = tid - NC;
    const bool yf = lane < 4 * BK;
    const int pos = yf ? lane >> 2 : min((lane >> 2) - BK, BJ - 1), fj = yf ? BJ - 1 : pos, fk = yf ? pos : BK - 1;
    const bool pub = lane < 4 * (BJ + BK) && (yf ? J + 1 < NJ && pos < g.bk : K + 1 < NK && pos < g.bj);
    int jl = 0, kl = 0;
    if (lane < g.nl) g.line(lane, jl, kl);
    const T *f0 = &ring[0][(fk + 1) * RG + fj + 1][lane & 3], *o0 = &ring[0][(kl + 1) * RG + jl + 1][0];
    uint64_t *dst = xch + xslot<T>(b, yf ? 0 : 1, pos, 0, nx, lane & 3);
    walk<T, BK> w;
    w.begin(g, y, y);
    write_levels<T>(L, [&](int m) {
      const int i = m - fj - fk, c = m - jl - kl;
      const T fv = f0[(m & 1) * RN * 4];
      T ov[4];
      ld4v(o0 + (m & 1) * RN * 4, ov);
      if (pub && i >= 0 && i < nx) xw<T>::put(dst + (int64_t)i * 4 * xw<T>::W, fv, tag);
      if (lane < g.nl && c >= 0 && c < nx) st4v(const_cast<T *>(at(w.v, 4 * (lane - w.first))), ov);
      w.up(g);
    });
    return;
  }
  const int row = tid & 3, q = tid >> 2;
  int jl = 0, kl = 0;
  if (q < g.nl) g.line(q, jl, kl);
  const bool hz = K * BK + kl > 0, hy = J * BJ + jl > 0;
  const int slot = (kl + 1) * RG + jl + 1;
  walk<T, BK> lw;                                           // the level that loads next
  lw.begin(g, rhs, B.pb);
  const int64_t cl = ((int64_t)(K * BK + kl) * ny + J * BJ + jl) * nx;
  auto load = [&](sweep_pre<T> &p, T tok) {
    int e = lw.lane(q);
    after(e, tok);
    p.v = *at(lw.v, 4 * e + row);
    if constexpr (NAT) {
      int i = min(max(lw.h - jl - kl, 0), nx - 1);
      after(i, tok);
      const int64_t c = (cl + i) * 16 + 4 * row;
#pragma unroll
      for (int b = 0; b < 3; ++b) ld4v(B.t7 + b * B.n * 16 + c, p.a[b]);
      ld4v(B.dinv2 + c, p.dv);
      lw.up(g);
      return;
    }
    e = 16 * e + 4 * row;
    ld4v(at(lw.o, e), p.a[0]);
    ld4v(at(lw.o + lw.act * 16, e), p.a[1]);
    ld4v(at(lw.o + lw.act * 32, e), p.a[2]);
    ld4v(at(lw.o + lw.act * 48, e), p.dv);
    lw.up(g);
  };
  sweep_pre<T> R[P];
#pragma unroll
  for (int d = 0; d < P; ++d) load(R[d], (T)0);
  for (int h0 = 0; h0 < L; h0 += P) {
#pragma unroll
    for (int d = 0; d < P; ++d) {
      const int h = h0 + d, i = h - jl - kl;
      const bool act = q < g.nl && i >= 0 && i < nx;
      __syncthreads();
      const T(*prev)[4] = ring[(h + 1) & 1];
      T yz[4], yy[4], yx[4];
      ld4v(&prev[slot - RG][0], yz);
      ld4v(&prev[slot - 1][0], yy);
      ld4v(&prev[slot][0], yx);
      const T tz = dot4(R[d].a[0], yz), ty = dot4(R[d].a[1], yy), tx = dot4(R[d].a[2], yx);
      T v = R[d].v;
      v = hz ? v - tz : v;
      v = hy ? v - ty : v;
      v = i > 0 ? v - tx : v;
      const T o = quad_mv<T>(R[d].dv, v);
      if (act) ring[h & 1][slot][row] = o;
      load(R[d], o);
    }
  }
  __syncthreads();
}

template <class T, int P, int BK, bool NAT>
__global__ __launch_bounds__(4 * BJ * BK + 128) void k_bwd_pipe(int nx, int ny, int nz, int NJ, int NK, int *__restrict__ ticket,
                                                  int *__restrict__ err, uint32_t tag, uint64_t *__restrict__ xch,
                                                  sweep_blocks<T> B, const T *__restrict__ y,
                                                  const T *__restrict__ xpb, T *__restrict__ out) {
  constexpr int NC = 4 * BJ * BK, RN = ring_lines<BK>, BS = brick_geo<BK>::BS;
  __shared__ __align__(32) T ring[2][RN][4];       // line (jl, kl) at kl RG + jl
  constexpr int OB = 16 * 4 + 4;                          // padded: the lines of a level start in different banks
  __shared__ __align__(32) T ob[BJ * BK][OB];             // output z + Pi_p x_p of line (jl, kl), by column mod 16
  __shared__ int s_t;
  const int tid = threadIdx.x;
  if (tid == 0) s_t = atomicAdd(ticket, 1);
  __syncthreads();
  int J, K;
  brick_of(NJ * NK - 1 - uni(s_t), NJ, NK, J, K);
  const int b = J + NJ * K;
  const brick_geo<BK> g = geo_of<BK>(J, K, nx, ny, nz);
  const int L = (nx + BS + 7) / 8 * 8;                  // levels, a multiple of P and of the poller's lead
  const int top = nx - 1 + BS;                 // step m handles level top - m
  if (tid >= NC + 64) {
    // the y face after the brick (lines kl), then the z face (lines jl)
    const int lane = tid - NC - 64, r = lane & 3;
    const bool yf = lane < 4 * BK;
    const int pos = yf ? lane >> 2 : (lane >> 2) - BK;   // (lanes beyond the faces: past bj)
    const bool has = yf ? J + 1 < NJ && pos < g.bk : K + 1 < NK && pos < g.bj;
    const int gs = !has ? 0 : (yf ? pos * RG + BJ : BK * RG + pos);
    // lanes without a face to read load words of their own brick
    const uint64_t *src = xch + (has ? xslot<T>(yf ? b + 1 : b + NJ, yf ? 0 : 1, pos, 0, nx, r) : xslot<T>(b, 0, 0, 0, nx, r));
    poll_faces<T>(lane, L, nx, has, (yf ? BK : BJ) - 1 - pos, src, true, &ring[0][gs][r], &ring[1][gs][r], tag, err);
    return;
  }
  if (tid >= NC) {
    const int lane = tid - NC;
    const bool yf = lane < 4 * BK;
    const int pos = yf ? lane >> 2 : min((lane >> 2) - BK, BJ - 1), fj = yf ? 0 : pos, fk = yf ? pos : 0;
    const bool pub = lane < 4 * (BJ + BK) && (yf ? J > 0 && pos < g.bk : K > 0 && pos < g.bj);
    const T *f0 = &ring[0][fk * RG + fj][lane & 3];
    uint64_t *dst = xch + xslot<T>(b, yf ? 0 : 1, pos, 0, nx, lane & 3);
    // a line's output advances by one cell a level: eight lanes write eight
    // cells of a row together at the level that completes them, which one line
    // of every kl does (16 bytes to each line's row at every level: 512 us
    // instead of 458 in FP32 at 200x200x100)
    const int kl = lane >> 3, sub = lane & 7;
    T *o = out + 4 * ((int64_t)(K * BK + kl) * ny + J * BJ) * nx;
    write_levels<T>(L, [&](int m) {
      const int i = top - m - fj - fk;
      const int jl = (top - m - kl) & 7, i0 = top - m - kl - jl, io = i0 + sub;
      const T fv = f0[(m & 1) * RN * 4];
      T ov[4];
      ld4v(&ob[(kl & (BK - 1)) * BJ + jl][(io & 15) * 4], ov);
      if (pub && i >= 0 && i < nx) xw<T>::put(dst + (int64_t)i * 4 * xw<T>::W, fv, tag);
      if (jl < g.bj && kl < g.bk && i0 >= 0 && io < nx) st4v(o + 4 * ((int64_t)jl * nx + io), ov);
    });
    return;
  }
  const int row = tid & 3, q = tid >> 2;
  int jl = 0, kl = 0;
  if (q < g.nl) g.line(q, jl, kl);
  const bool hz = K * BK + kl < nz - 1, hy = J * BJ + jl < ny - 1;
  const int slot = kl * RG + jl;
  T *oq = &ob[kl * BJ + jl][row];
  T xpc[P];
  walk<T, BK> lw;                                           // the level that loads next
  lw.begin_top(g, y, B.pb, top);
  const T *xl = xpb + (lw.v - y) / 4;
  const int64_t cl = ((int64_t)(K * BK + kl) * ny + J * BJ + jl) * nx;
  auto load = [&](sweep_pre<T> &p, T &x, T tok) {
    int e = lw.lane(q);
    after(e, tok);
    p.v = *at(lw.v, 4 * e + row);
    x = *at(xl, e);
    if constexpr (NAT) {
      int i = min(max(lw.h - jl - kl, 0), nx - 1);
      after(i, tok);
      const int64_t c = (cl + i) * 16 + 4 * row;
      ld4v(B.dinv2 + c, p.dv);
#pragma unroll
      for (int b = 0; b < 3; ++b) ld4v(B.t7 + (4 + b) * B.n * 16 + c, p.a[b]);
      lw.down(g);
      xl -= lw.act;
      return;
    }
    e = 16 * e + 4 * row;
    ld4v(at(lw.o + lw.act * 48, e), p.dv);
    ld4v(at(lw.o + lw.act * 64, e), p.a[0]);
    ld4v(at(lw.o + lw.act * 80, e), p.a[1]);
    ld4v(at(lw.o + lw.act * 96, e), p.a[2]);
    lw.down(g);
    xl -= lw.act;
  };
  sweep_pre<T> R[P];
#pragma unroll
  for (int d = 0; d < P; ++d) load(R[d], xpc[d], (T)0);
  for (int m0 = 0; m0 < L; m0 += P) {
#pragma unroll
    for (int d = 0; d < P; ++d) {
      const int m = m0 + d, i = top - m - jl - kl;
      const bool act = q < g.nl && i >= 0 && i < nx;
      __syncthreads();
      const T(*prev)[4] = ring[(m + 1) & 1];
      T zx[4], zy[4], zz[4];
      ld4v(&prev[slot][0], zx);
      ld4v(&prev[slot + 1][0], zy);
      ld4v(&prev[slot + RG][0], zz);
      const T tx = dot4(R[d].a[0], zx), ty = dot4(R[d].a[1], zy), tz = dot4(R[d].a[2], zz);
      T v = 0;
      v = i < nx - 1 ? v + tx : v;
      v = hy ? v + ty : v;
      v = hz ? v + tz : v;
      const T w = quad_mv<T>(R[d].dv, v);
      const T zc = R[d].v - w;
      if (act) {
        ring[m & 1][slot][row] = zc;
        oq[(i & 15) * 4] = row == 0 ? zc + xpc[d] : zc;
      }
      load(R[d], xpc[d], zc);
    }
  }
  __syncthreads();
}

// ---- factorisation: D_c = A~_cc - sum_{lower k} A~_ck D_k^{-1} A~_kc ----------
// Bricks of 8 x 8 x-lines, one workgroup each, walked by hyperplanes like the
// sweeps' bricks: 4 compute waves with a quad of lanes per cell (lane r holds
// block row r), a writer wave and a poller wave, one barrier per level.
//   - compute: the D^{-1} rows of the three lower neighbours come from the
//     previous level in an LDS ring (which has a slot for each line just
//     outside the brick), the seven block rows of the next two levels are in
//     flight in registers;
//   - writer: copies the previous level from the ring to dinv2, the brick's
//     outgoing faces with device-scope stores, waits for them and publishes
//     the level count;
//   - poller: waits for the two bricks before (bounded), loads their face
//     blocks two levels ahead and puts them into the ring.
// What bounds it is the chain nx + ny + nz of levels: a level is a cell's
// dependency chain (three Schur products, then four pivot steps with a
// division each), so the cells of a level are spread over as many SIMDs as
// the brick has waves, and the brick is as large as keeps one compute wave
// per SIMD: the step from a brick to the next costs the brick edge in levels
// plus the face's way through memory, and larger bricks have fewer of them.
// Measured: 1.45 ms in FP32 at 200x200x100 (5.83 ms with bricks of 4 x 4 lines
// and one thread per cell), 0.74 ms in FP64 at 100x100x50 (2.05); a level of a
// lone brick takes 1.85 us in FP32 (about 760 instructions in a compute
// wave), 2.1 in FP64.  Each level count has a cache line of its own: packed
// counts, polled by one brick and written by another, cost 15 % more.
constexpr int SB = 8;                    // brick edge
constexpr int SG = SB + 1;               // ring lines per side: one outside the brick

template <class T> __device__ __forceinline__ void st_dev16(T *p, const T (&v)[16]) {   // 16 values, 8 bytes a store
  constexpr int PER = 8 / sizeof(T);
#pragma unroll
  for (int e = 0; e < 16; e += PER) {
    uint64_t w;
    __builtin_memcpy(&w, &v[e], 8);
    st_dev((uint64_t *)(p + e), w);
  }
}

template <class T>
__global__ __launch_bounds__(6 * 64) void k_setup_pipe(int nx, int ny, int nz, int NJ, int NK, int *__restrict__ ticket,
                                                       int *done, int *__restrict__ err, const T *__restrict__ t7,
                                                       T *dinv2, int *__restrict__ flag) {
  constexpr int B = SB, NC = 4 * B * B;                 // compute lanes
  __shared__ __align__(16) T ring[2][SG * SG][16];      // line (jl, kl) at (kl + 1) SG + jl + 1
  __shared__ int s_t;
  const int tid = threadIdx.x;
  if (tid == 0) s_t = atomicAdd(ticket, 1);
  __syncthreads();
  int J, K;
  brick_of(s_t, NJ, NK, J, K);
  const int b = J + NJ * K;
  const int64_t nxy = (int64_t)nx * ny, n = nxy * nz;
  const int L = nx + 2 * (B - 1);
  if (tid >= NC + 64) {
    // poller: lane (line of a face, row): the y face before the brick (lines
    // kl), then the z face (lines jl)
    const int lane = tid - NC - 64, r = lane & 3, pos = (lane >> 2) & 7;
    const bool yf = lane < 32;
    const int j = yf ? J * B - 1 : J * B + pos, k = yf ? K * B + pos : K * B - 1;
    const bool has = yf ? J > 0 && k < nz : K > 0 && j < ny;
    const int gs = yf ? (pos + 1) * SG : pos + 1;
    const T *base = dinv2 + (has ? ((int64_t)k * nxy + (int64_t)j * nx) * 16 : 0) + 4 * r;
    constexpr int NW = 4 * sizeof(T) / 8;               // 8-byte words of a block row
    // the lanes of each face read their own predecessor's count, both in one
    // round trip
    const int *fl = done + FL * (yf ? b - 1 : b - NJ);
    const bool pred = yf ? J > 0 : K > 0;
    int seen = pred ? 0 : L;
    bool failed = false;
    auto issue = [&](int h, uint64_t (&w)[NW]) {
      if (h >= L) return;
      const int need = min(h + B, L);                   // the face cell of level h is at level h + B - 1 of its brick
      int spins = 0;
      while (__ballot(seen < need) != 0 && !failed) {
        if (pred) seen = ld_dev(fl);
        if (++spins > SPIN_LIMIT) { atomicOr(err, 1); failed = true; }
      }
      asm volatile("" ::: "memory");                    // the loads stay behind the polls
      const int i = h - pos;
      if (!has || i < 0 || i >= nx) return;
#pragma unroll
      for (int e = 0; e < NW; ++e) w[e] = ld_dev((const uint64_t *)(base + (int64_t)i * 16) + e);
    };
    auto put = [&](int h, const uint64_t (&w)[NW]) {
      const int i = h - pos;
      if (!has || h >= L || i < 0 || i >= nx) return;
#pragma unroll
      for (int e = 0; e < NW; ++e) *((uint64_t *)&ring[(h + 1) & 1][gs][4 * r] + e) = w[e];
    };
    uint64_t w[2][NW];
    issue(0, w[0]);
    put(0, w[0]);
    issue(1, w[1]);
    for (int h = 0; h < L; h += 2) {
      __syncthreads();
      put(h + 1, w[1]);
      issue(h + 2, w[0]);
      if (h + 1 >= L) break;
      __syncthreads();
      put(h + 2, w[0]);
      issue(h + 3, w[1]);
    }
    __syncthreads();
    return;
  }
  if (tid >= NC) {
    // writer: line `lane` of the brick
    const int lane = tid - NC, jl = lane & 7, kl = lane >> 3;
    const int j = J * B + jl, k = K * B + kl;
    const bool line = j < ny && k < nz, face = jl == B - 1 || kl == B - 1;
    T *base = dinv2 + (line ? ((int64_t)k * nxy + (int64_t)j * nx) * 16 : 0);
    auto write_level = [&](int h) {
      const int i = h - jl - kl;
      if (line && i >= 0 && i < nx) {
        T v[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          T t4[4];
          ld4v(&ring[h & 1][(kl + 1) * SG + jl + 1][4 * q], t4);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[4 * q + e] = t4[e];
        }
        if (face) {
          st_dev16(base + (int64_t)i * 16, v);
        } else {
#pragma unroll
          for (int e = 0; e < 16; e += 4) st4v(base + (int64_t)i * 16 + e, v + e);
        }
      }
    };
    // the stores of a level have a level's time to complete before its count
    // is published
    auto publish = [&](int cnt) {
      __builtin_amdgcn_s_waitcnt(0);
      asm volatile("" ::: "memory");
      if (lane == 0) st_dev(done + FL * b, cnt);
    };
    for (int h = 0; h < L; ++h) {
      __syncthreads();
      if (h > 1) publish(h - 1);
      if (h > 0) write_level(h - 1);
    }
    __syncthreads();
    write_level(L - 1);
    publish(L);
    return;
  }
  const int r = tid & 3, q = tid >> 2, jl = q & 7, kl = q >> 3, wq = (tid & 63) & ~3;
  const int j = J * B + jl, k = K * B + kl;
  const bool line = j < ny && k < nz, hz = k > 0, hy = j > 0;
  const int slot = (kl + 1) * SG + jl + 1;
  const int64_t c0 = line ? (int64_t)k * nxy + (int64_t)j * nx : 0;
  // this lane's rows of A~_cc, A~_cq and A~_qc for q before c in z, y, x
  struct rows { T d[4], lo[3][4], up[3][4]; };
  auto load = [&](int h, rows &p) {
    int i = min(max(h - jl - kl, 0), nx - 1);
    const int64_t c = c0 + i;
    const int64_t qz = line && hz ? c - nxy : c, qy = line && hy ? c - nx : c, qx = i > 0 ? c - 1 : c;
    ld4v(t7 + (3 * n + c) * 16 + 4 * r, p.d);
    ld4v(t7 + c * 16 + 4 * r, p.lo[0]);
    ld4v(t7 + (n + c) * 16 + 4 * r, p.lo[1]);
    ld4v(t7 + (2 * n + c) * 16 + 4 * r, p.lo[2]);
    ld4v(t7 + (6 * n + qz) * 16 + 4 * r, p.up[0]);
    ld4v(t7 + (5 * n + qy) * 16 + 4 * r, p.up[1]);
    ld4v(t7 + (4 * n + qx) * 16 + 4 * r, p.up[2]);
  };
  int bad = 0;
  auto level = [&](int h, rows &p) {
    __syncthreads();
    const int i = h - jl - kl;
    if (line && i >= 0 && i < nx) {                     // the same for the four lanes of the cell
      const T(*prev)[16] = ring[(h + 1) & 1];
      double Lr[4], Rr[4];
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) Lr[cc] = (double)p.d[cc];
      T dq[4];
      if (hz) { ld4v(&prev[slot - SG][4 * r], dq); quad_schur<T>(Lr, dq, p.up[0], p.lo[0]); }
      if (hy) { ld4v(&prev[slot - 1][4 * r], dq); quad_schur<T>(Lr, dq, p.up[1], p.lo[1]); }
      if (i > 0) { ld4v(&prev[slot][4 * r], dq); quad_schur<T>(Lr, dq, p.up[2], p.lo[2]); }
      int mine;
      bad |= quad_inverse(Lr, Rr, r, wq, mine);
      T *o = &ring[h & 1][slot][4 * mine];
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) o[cc] = (T)Rr[cc];
    }
    load(h + 2, p);
  };
  rows p0, p1;
  load(0, p0);
  load(1, p1);
  for (int h = 0; h < L; h += 2) {
    level(h, p0);
    if (h + 1 >= L) break;
    level(h + 1, p1);
  }
  __syncthreads();
  if (bad) atomicOr(flag, bad);
}

}  // namespace

// ---------------------------------------------------------------------------
// The grids that rs_cpr_setup documents for DILU.  (The bound comes from face
// words of bricks of 4 x 4 lines within 4 GiB; bricks are larger now and
// nothing of that size is allocated.)
rs_status rs_dilu_check_shape(const grid3 &g, int prec) {
  const int64_t c = (int64_t)((g.ny + 3) / 4) * ((g.nz + 3) / 4) * g.nx;
  return c < (prec == 64 ? 1 << 23 : 1 << 24) ? RS_OK : RS_E_ARG;
}

rs_status rs_dilu_prepare(rs_cpr_s *M, hipStream_t s) {
  const grid3 &g = M->A->g;
  // Bricks of 8 x 4 lines while they are few enough for one a CU, 8 x 8 beyond:
  // a CU takes in about 45 GB/s, whatever its brick's size, so that thinner
  // bricks walk their levels faster, but a grid has more of them between its
  // corners.  Forward sweep with 8 x 4 and with 8 x 8 lines, us, FP32 and FP64:
  // 100x100x50 (169 thin bricks) 168 and 177, 212 and 287; 128x128x64 (256)
  // 226 and 264, 323 and 402; 150x150x75 (361) 316 and 300, 554 and 491;
  // 200x200x100 (650) 580 and 480, 878 and 806.
  M->pnj = (g.ny + BJ - 1) / BJ;
  M->pbk = (int64_t)M->pnj * ((g.nz + 3) / 4) <= 256 ? 4 : 8;
  M->pnk = (g.nz + M->pbk - 1) / M->pbk;
  const size_t nb = (size_t)M->pnj * M->pnk, nbs = (size_t)((g.ny + SB - 1) / SB) * ((g.nz + SB - 1) / SB);
  RS_TRY(M->pdone.alloc(sizeof(int) * FL * nbs));
  const size_t es = M->prec == 64 ? sizeof(double) : sizeof(float);
  // The copy in brick order takes 448 (FP32) or 896 bytes a cell, an eighth of
  // what a solve holds.  Where memory ends it is left out (rs_cpr_setup) or given
  // back (rs_yield), and the sweeps read the grid's order: an application at
  // 200x200x100 takes 1.56 ms for 1.38 in FP32, 2.34 for 2.27 in FP64.
  if (M->pcopy) RS_TRY(M->pblk.alloc(es * 7 * 16 * (size_t)g.n));
  RS_TRY(M->pxp.alloc(es * (size_t)g.n));
  RS_TRY(M->pctl.alloc(sizeof(int) * 4));     // [0] ticket, [1] error, [2] second ticket
  // face exchange: 2 faces x 8 lines x nx cells x 4 values x (1 or 2) words
  const size_t words = nb * 2 * BJ * g.nx * 4 * (M->prec == 64 ? 2 : 1);
  RS_TRY(M->pxch.alloc(sizeof(uint64_t) * words));
  const size_t most = std::max(words, nbs);
  k_pipe_clear<<<rs_grid(most), RS_BLOCK, 0, s>>>((int64_t)words, M->pxch.as<uint64_t>(), (int)nbs, M->pdone.as<int>(),
                                                  M->pctl.as<int>());
  RS_HIP(hipGetLastError());
  M->pepoch = 0;
  return RS_OK;
}

template <class T>
static rs_status dilu_setup_t(rs_cpr_s *M, int *flag, hipStream_t s) {
  const grid3 &g = M->A->g;
  const int SJ = (g.ny + SB - 1) / SB, SK = (g.nz + SB - 1) / SB;
  int *ctl = M->pctl.as<int>();
  const T *t7 = M->D->t7.as<T>();
  T *dinv2 = M->dinv2.as<T>(), *pb = M->pblk.as<T>();
  k_setup_pipe<T><<<SJ * SK, 6 * 64, 0, s>>>(g.nx, g.ny, g.nz, SJ, SK, ctl, M->pdone.as<int>(), ctl + 1, t7, dinv2, flag);
  if (!pb) {
    RS_HIP(hipGetLastError());
    return RS_OK;
  }
  // the sweeps' operands in brick order
  const int NC = (g.nx + CH - 1) / CH;
  const unsigned ng = (unsigned)(M->pnj * M->pnk) * NC;
  if (M->pbk == 4) k_dilu_order<T, 4><<<ng, 256, 0, s>>>(g.nx, g.ny, g.nz, M->pnj, NC, g.n, t7, dinv2, pb);
  else k_dilu_order<T, 8><<<ng, 256, 0, s>>>(g.nx, g.ny, g.nz, M->pnj, NC, g.n, t7, dinv2, pb);
  RS_HIP(hipGetLastError());
  return RS_OK;
}

rs_status rs_dilu_setup_run(rs_cpr_s *M, int *flag, hipStream_t s) {
  return M->prec == 64 ? dilu_setup_t<double>(M, flag, s) : dilu_setup_t<float>(M, flag, s);
}

template <class T, int BK, bool NAT>
static rs_status dilu_apply_t(rs_cpr_s *M, const T *xp, T *out, hipStream_t s) {
  const grid3 &g = M->A->g;
  const int NJ = M->pnj, NK = M->pnk, NC = (g.nx + CH - 1) / CH, NT = 4 * BJ * BK + 128;
  int *ctl = M->pctl.as<int>();
  uint64_t *xch = M->pxch.as<uint64_t>();
  T *rhs = M->zt.as<T>(), *y = M->yv.as<T>(), *xpb = M->pxp.as<T>();
  const sweep_blocks<T> B{M->pblk.as<T>(), M->D->t7.as<T>(), M->dinv2.as<T>(), g.n};
  constexpr int P = sizeof(T) == 4 ? 8 : 4;   // levels in flight (6 to 12 and 3 to 6 measure the same)
  k_dilu_rhs<T, BK><<<(unsigned)(NJ * NK) * NC, 256, 0, s>>>(g.nx, g.ny, g.nz, NJ, NC, M->rt.as<T>(),
                                                            M->D->col0.as<T>(), xp, rhs, xpb, ctl);
  uint32_t tag = ++M->pepoch;
  k_fwd_pipe<T, P, BK, NAT><<<NJ * NK, NT, 0, s>>>(g.nx, g.ny, g.nz, NJ, NK, ctl, ctl + 1, tag, xch, B, rhs, y);
  tag = ++M->pepoch;
  k_bwd_pipe<T, P, BK, NAT><<<NJ * NK, NT, 0, s>>>(g.nx, g.ny, g.nz, NJ, NK, ctl + 2, ctl + 1, tag, xch, B, y, xpb, out);
  RS_HIP(hipGetLastError());
  return RS_OK;
}

template <class T>
rs_status rs_dilu_apply_run(rs_cpr_s *M, const T *xp, T *out, hipStream_t s) {
  if (!M->pblk.p) return M->pbk == 4 ? dilu_apply_t<T, 4, true>(M, xp, out, s) : dilu_apply_t<T, 8, true>(M, xp, out, s);
  return M->pbk == 4 ? dilu_apply_t<T, 4, false>(M, xp, out, s) : dilu_apply_t<T, 8, false>(M, xp, out, s);
}

template rs_status rs_dilu_apply_run<double>(rs_cpr_s *, const double *, double *, hipStream_t);
template rs_status rs_dilu_apply_run<float>(rs_cpr_s *, const float *, float *, hipStream_t);

// error words of the pipelined sweeps (DILU bricks, RAS strips): a bounded
// wait that timed out leaves a non-zero word
rs_status rs_dilu_check(rs_cpr_s *M, hipStream_t s) {
  const int *w[2];
  rs_sweep_errors(M, w);
  if (!w[0] && !w[1]) return RS_OK;
  int h = 0, e = 0;
  RS_TRY(rs_wait_read_err(&h, w[0] ? w[0] : w[1], sizeof(int), w, &e, s));
  return e ? RS_E_HIP : RS_OK;
}

void rs_sweep_errors(const rs_cpr_s *M, const int *(&w)[2]) {
  w[0] = M->pctl.p ? M->pctl.as<int>() + 1 : nullptr;
  w[1] = M->rctl.p ? M->rctl.as<int>() + 5 : nullptr;
}
