// thermal.hip -- the linear system of one Newton step of a water / oil /
// energy subset of the paper's thermal model, assembled on the device: the
// residual R(u) and the Jacobian dR/du as 4x4 blocks in the caller's CSR
// layout of the 7-point pattern, ready for rs_bsr_attach_decouple.
//
// Per cell, unknowns (p, N_w, N_o, T) and equations (water, oil, energy,
// saturation constraint in volume form), with Eqs. eq4.1-eq4.3 of Section
// "Mathematical Model" discretised as in Section "Numerical Methods"
// (backward Euler; face transmissibility = harmonic geometric part times the
// upstream fluid part); the model, its constants and their sources are
// listed with rs_thermal_assemble in rsolve.h.
//
// A workgroup takes a tile of 64 cells (8 x 4 x 2 but on thin grids): it
// evaluates the properties of the tile's cells and of the cells around it once,
// into LDS, and then forms the block rows and the residual with a quad of lanes
// per cell, lane r for equation r, so that a block is written as one 128-byte
// run.  No two lanes
// write the same place.  The face flow seen from either side is the same
// number (up to sign): the upstream cell is the one of higher pressure, on a
// tie the lower-numbered one, whichever cell computes it.
#include "rs_internal.h"
#include <math.h>

namespace {
#include "csr7.h"
#include "quad4.h"

// Fig. rela-swt of the paper: S_w, k_rw, k_row
__constant__ double kSwt[12][3] = {
    {0.45, 0.0, 0.4},       {0.47, 0.000056, 0.361},    {0.50, 0.000552, 0.30625},  {0.55, 0.00312, 0.225},
    {0.60, 0.00861, 0.15625}, {0.65, 0.01768, 0.1},     {0.70, 0.03088, 0.05625},   {0.75, 0.04871, 0.025},
    {0.77, 0.05724, 0.016}, {0.80, 0.07162, 0.00625},   {0.82, 0.08229, 0.00225},   {0.85, 0.1, 0.0}};
// Fig. rela-slt: S_l, k_rg, k_rog
__constant__ double kSlt[19][3] = {
    {0.45, 0.2, 0.0},         {0.55, 0.14202, 0.0},     {0.57, 0.13123, 0.00079}, {0.60, 0.11560, 0.00494},
    {0.62, 0.10555, 0.00968}, {0.65, 0.09106, 0.01975}, {0.67, 0.08181, 0.02844}, {0.70, 0.06856, 0.04444},
    {0.72, 0.06017, 0.05709}, {0.75, 0.04829, 0.07901}, {0.77, 0.04087, 0.09560}, {0.80, 0.03054, 0.12346},
    {0.83, 0.02127, 0.15486}, {0.85, 0.01574, 0.17778}, {0.87, 0.01080, 0.20227}, {0.90, 0.00467, 0.24198},
    {0.92, 0.00165, 0.27042}, {0.94, 0.0, 0.30044},     {1.0, 0.0, 0.4}};
// Fig. fig-wat-vis: deg C, cp
__constant__ double kWvis[28][2] = {
    {5.0, 1.5182},       {8.0, 1.386},       {10.0, 1.311},      {20.0, 1.005},      {30.0, 0.8004},
    {40.0, 0.6543},      {50.0, 0.5518},     {60.0, 0.4714},     {70.0, 0.4066},     {80.0, 0.3570},
    {90.0, 0.3182},      {100.0, 0.2828},    {125.0, 0.2227},    {150.0, 0.1848},    {175.0, 0.1586},
    {200.0, 0.1394},     {225.0, 0.1238},    {250.0, 0.1117},    {275.0, 0.1005},    {300.0, 9.9125e-2},
    {325.0, 8.4075e-2},  {350.0, 7.7437e-2}, {375.0, 7.2818e-2}, {400.0, 7.2818e-2}, {500.0, 7.2818e-2},
    {600.0, 7.2818e-2},  {700.0, 7.2818e-2}, {800.0, 7.2818e-2}};

// Tables in LDS: rows of COLS values, abscissa first, then the slopes of the
// following interval.  find: the interval at x, or -1 below the first and -2
// beyond the last abscissa, where the table is constant.
template <int ROWS, int COLS> struct lds_table {
  static constexpr int W = 2 * COLS - 1;
  double v[ROWS][W];
  __device__ __forceinline__ void fill(const double (&tab)[ROWS][COLS], int t) {
    if (t >= ROWS * W) return;
    const int r = t / W, c = t - r * W;
    if (c < COLS) v[r][c] = tab[r][c];
    else v[r][c] = r + 1 < ROWS ? (tab[r + 1][c - COLS + 1] - tab[r][c - COLS + 1]) / (tab[r + 1][0] - tab[r][0]) : 0.0;
  }
  __device__ __forceinline__ int find(double x) const {
    if (x <= v[0][0]) return -1;
    if (x >= v[ROWS - 1][0]) return -2;
    int lo = 0, hi = ROWS - 1;               // v[lo][0] <= x < v[hi][0]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (x < v[mid][0]) hi = mid; else lo = mid;
    }
    return lo;
  }
  // value and slope of column col
  __device__ __forceinline__ double at(int col, int lo, double x, double &slope) const {
    slope = lo < 0 ? 0.0 : v[lo][COLS + col - 1];
    if (lo < 0) return v[lo == -1 ? 0 : ROWS - 1][col];
    return v[lo][col] + slope * (x - v[lo][0]);
  }
};
typedef lds_table<12, 3> swt_t;
typedef lds_table<28, 2> wvis_t;
static_assert(12 * swt_t::W <= 128 && 28 * wvis_t::W <= 128, "filled by half a workgroup each");

// What the flows need of a cell: pressure, temperature, thermal conductivity,
// the mobilities of water, oil (k_r rho / mu) and energy (their sum times the
// enthalpies), and the u-gradients of the mobilities and the conductivity.
enum { C_P, C_T, C_KT, C_L, C_LU = C_L + 3, C_KTU = C_LU + 12, C_N = C_KTU + 4 };
// What the cell itself needs besides: gradients of the energy and of the
// volume constraint, their values, the phase terms of a producer.
enum { O_EU, O_VU = 4, O_E = 8, O_VOL, O_EOLD, O_N };

// The parameters with what follows from them alone (formed on the host: a
// division in FP64 is 15 instructions for every lane)
struct tpar : rs_thermal_params {
  double acc;                // V / dt
  double gc[3];              // area / length of a face along x, y, z
  double ch[5], href;        // coefficients of the water enthalpy's integral, its value at t_ref
  explicit tpar(const rs_thermal_params &q) : rs_thermal_params(q) {
    acc = dx * dy * dz / dt;
    gc[0] = dy * dz / dx;
    gc[1] = dx * dz / dy;
    gc[2] = dx * dy / dz;
    const double tr = (t_ref - 32.0) / 1.8;
    href = 0.0;
    double pr = tr;
    for (int k = 0; k < 5; ++k) {
      ch[k] = cpg[k] / (k + 1);
      href += ch[k] * pr;
      pr *= tr;
    }
  }
};

__device__ double water_h(const tpar &q, double t, double &dh) {
  const double tc = (t - 32.0) * (1.0 / 1.8);
  // integral of c0 + c1 s + ... + c4 s^4 from tr to tc, and the integrand at tc
  const double h = ((((q.ch[4] * tc + q.ch[3]) * tc + q.ch[2]) * tc + q.ch[1]) * tc + q.ch[0]) * tc - q.href;
  const double cp = (((q.cpg[4] * tc + q.cpg[3]) * tc + q.cpg[2]) * tc + q.cpg[1]) * tc + q.cpg[0];
  double hv = 0.0, dhv = 0.0;              // heat of vaporisation, zero above T_crit
  if (tc < q.tcrit_w) {
    const double g = pow(q.tcrit_w - tc, q.ev_w - 1.0);
    hv = q.hvr_w * g * (q.tcrit_w - tc);
    dhv = -q.hvr_w * q.ev_w * g;
  }
  dh = (cp - dhv) * q.jmol_btu * (1.0 / 1.8);
  return (h - hv) * q.jmol_btu;
}

__device__ void cell_eval(const tpar &q, const double *__restrict__ u4, const swt_t &swt,
                          const wvis_t &wvis, double *__restrict__ c, double *__restrict__ own) {
  const double p = u4[0], nw = u4[1], no = u4[2], t = u4[3];
  const double dp = p - q.p_ref, dT = t - q.t_ref;
  c[C_P] = p; c[C_T] = t;
  const double phi = q.por_ref * (1.0 + q.cpor * dp), phi_p = q.por_ref * q.cpor;
  const double rw = q.rhow_ref * exp(q.cpw * dp - q.ct1w * dT - 0.5 * q.ct2w * dT * dT + q.cptw * dp * dT);
  const double rw_p = rw * (q.cpw + q.cptw * dT), rw_t = rw * (q.cptw * dp - q.ct1w - q.ct2w * dT);
  const double ro = q.rhoo_ref * exp(q.cpo * dp - q.ct1o * dT - 0.5 * q.ct2o * dT * dT + q.cpto * dp * dT);
  const double ro_p = ro * (q.cpo + q.cpto * dT), ro_t = ro * (q.cpto * dp - q.ct1o - q.ct2o * dT);
  // S = N / (phi rho): gradients in (p, N_w, N_o, T)
  const double aw = phi * rw, ao = phi * ro;
  const double iaw = 1.0 / aw, iao = 1.0 / ao, irw = 1.0 / rw, iro = 1.0 / ro;   // a division is 15 instructions
  const double sw = nw * iaw, so = no * iao;
  const double sw_u[4] = {-sw * (phi_p * rw + phi * rw_p) * iaw, iaw, 0.0, -sw * phi * rw_t * iaw};
  const double so_u[4] = {-so * (phi_p * ro + phi * ro_p) * iao, 0.0, iao, -so * phi * ro_t * iao};
  // relative permeabilities: k_rw, and Stone II with no gas (S_l = 1, the
  // last entry of that table)
  double dkrw, dkrow;
  const int is = swt.find(sw);
  const double krw = swt.at(1, is, sw, dkrw), krow = swt.at(2, is, sw, dkrow);
  const double krg = kSlt[18][1], krog = kSlt[18][2], krocw = kSwt[0][2];
  const double ikr = 1.0 / krocw, kg = krog * ikr + krg;
  double kro = krocw * ((krow * ikr + krw) * kg - krw - krg);
  double dkro = krocw * ((dkrow * ikr + dkrw) * kg - dkrw);
  if (kro < 0.0) { kro = 0.0; dkro = 0.0; }
  // viscosities
  double dmw;
  const double tc = (t - 32.0) * (1.0 / 1.8), mw = wvis.at(1, wvis.find(tc), tc, dmw);
  dmw *= 1.0 / 1.8;
  const double ita = 1.0 / (t + 459.67);
  const double mo = q.avisc_o * exp(q.bvisc_o * ita), dmo = -mo * q.bvisc_o * ita * ita;
  const double imw = 1.0 / mw, imo = 1.0 / mo;
  const double lw = krw * rw * imw, lo = kro * ro * imo;
  // enthalpies
  double hw_t;
  const double hw = water_h(q, t, hw_t), ho = q.cpl_o * dT;
  c[C_L] = lw;
  c[C_L + 1] = lo;
  c[C_L + 2] = lw * hw + lo * ho;
  for (int m = 0; m < 4; ++m) {
    const double drw = m == 0 ? rw_p : (m == 3 ? rw_t : 0.0), dro = m == 0 ? ro_p : (m == 3 ? ro_t : 0.0);
    const double dmuw = m == 3 ? dmw : 0.0, dmuo = m == 3 ? dmo : 0.0;
    const double lwm = (dkrw * sw_u[m] * rw + krw * drw - lw * dmuw) * imw;
    const double lom = (dkro * sw_u[m] * ro + kro * dro - lo * dmuo) * imo;
    const double hwm = m == 3 ? hw_t : 0.0, hom = m == 3 ? q.cpl_o : 0.0;
    c[C_LU + m] = lwm;
    c[C_LU + 4 + m] = lom;
    c[C_LU + 8 + m] = lwm * hw + lw * hwm + lom * ho + lo * hom;
  }
  // conductivity (linear mixing)
  const double mix = sw * q.kw + so * q.ko;
  c[C_KT] = phi * mix + (1.0 - phi) * q.kr;
  for (int m = 0; m < 4; ++m) {
    const double dphi = m == 0 ? phi_p : 0.0;
    c[C_KTU + m] = dphi * (mix - q.kr) + phi * (sw_u[m] * q.kw + so_u[m] * q.ko);
  }
  if (!own) return;
  // internal energies U = H - p/rho, energy per bulk volume
  const double uw = hw - q.pv_btu * p * irw, uo = ho - q.pv_btu * p * iro;
  const double uw_p = -q.pv_btu * (irw - p * rw_p * irw * irw), uw_t = hw_t + q.pv_btu * p * rw_t * irw * irw;
  const double uo_p = -q.pv_btu * (iro - p * ro_p * iro * iro), uo_t = q.cpl_o + q.pv_btu * p * ro_t * iro * iro;
  own[O_E] = nw * uw + no * uo + (1.0 - q.por_ref) * q.cp_rock * dT;
  own[O_EU] = nw * uw_p + no * uo_p;
  own[O_EU + 1] = uw;
  own[O_EU + 2] = uo;
  own[O_EU + 3] = nw * uw_t + no * uo_t + (1.0 - q.por_ref) * q.cp_rock;
  // the saturation constraint
  own[O_VOL] = phi - nw * irw - no * iro;
  own[O_VU] = phi_p + nw * rw_p * irw * irw + no * ro_p * iro * iro;
  own[O_VU + 1] = -irw;
  own[O_VU + 2] = -iro;
  own[O_VU + 3] = nw * rw_t * irw * irw + no * ro_t * iro * iro;
}

// energy per bulk volume only (the previous time step's state)
__device__ double cell_energy(const tpar &q, const double *__restrict__ u4) {
  const double p = u4[0], nw = u4[1], no = u4[2], t = u4[3];
  const double dp = p - q.p_ref, dT = t - q.t_ref;
  const double rw = q.rhow_ref * exp(q.cpw * dp - q.ct1w * dT - 0.5 * q.ct2w * dT * dT + q.cptw * dp * dT);
  const double ro = q.rhoo_ref * exp(q.cpo * dp - q.ct1o * dT - 0.5 * q.ct2o * dT * dT + q.cpto * dp * dT);
  double dh;
  const double hw = water_h(q, t, dh), ho = q.cpl_o * dT;
  return nw * (hw - q.pv_btu * p / rw) + no * (ho - q.pv_btu * p / ro) + (1.0 - q.por_ref) * q.cp_rock * dT;
}

// Tile of a workgroup, and the LDS index of its cells and the ones around it:
// own cells, then the faces -x, +x, -y, +y, -z, +z.  Along an axis with one
// cell in the tile the grid has one too, and there are no faces.
template <int TX_, int TY_, int TZ_> struct tile {
  static constexpr int TX = TX_, TY = TY_, TZ = TZ_, TN = TX * TY * TZ;
  static constexpr int HX = TN, HY = HX + (TX > 1 ? 2 * TY * TZ : 0), HZ = HY + (TY > 1 ? 2 * TX * TZ : 0);
  static constexpr int HN = HZ + (TZ > 1 ? 2 * TX * TY : 0);
  static_assert(HN + TN + TY * TZ <= 256 && 4 * TN == 256, "one evaluation or search and one block row per thread");
  static int64_t count(int nx, int ny, int nz) {
    return (int64_t)((nx + TX - 1) / TX) * ((ny + TY - 1) / TY) * ((nz + TZ - 1) / TZ);
  }
  __device__ static __forceinline__ void cell(int t, int &a, int &b, int &d) {
    if (t < HX) {
      a = t % TX; b = t / TX % TY; d = t / (TX * TY);
    } else if (t < HY) {
      const int f = t - HX, e = f % (TY * TZ);
      a = f < TY * TZ ? -1 : TX; b = e % TY; d = e / TY;
    } else if (t < HZ) {
      const int f = t - HY, e = f % (TX * TZ);
      b = f < TX * TZ ? -1 : TY; a = e % TX; d = e / TX;
    } else {
      const int f = t - HZ, e = f % (TX * TY);
      d = f < TX * TY ? -1 : TZ; a = e % TX; b = e / TX;
    }
  }
};

// 2300 instructions per 16 cells and a chain of loads, evaluation, faces and
// stores; the blocks written (441 MB at 100x100x50) would take 90 us.  There:
// 169 us, 426 us with one thread per cell that evaluated its six neighbours
// as well and searched the tables in constant memory.
template <class TILE>
__global__ __launch_bounds__(256) void k_thermal(int nx, int ny, int nz, tpar q,
                                                 const double *__restrict__ kx, const double *__restrict__ ky,
                                                 const double *__restrict__ kz, const double *__restrict__ u,
                                                 const double *__restrict__ uold, int nw,
                                                 const int32_t *__restrict__ wcell, const int32_t *__restrict__ wkind,
                                                 const double *__restrict__ wval, double *__restrict__ vals,
                                                 double *__restrict__ res) {
  constexpr int TX = TILE::TX, TY = TILE::TY, TZ = TILE::TZ, TN = TILE::TN;
  constexpr int HX = TILE::HX, HY = TILE::HY, HZ = TILE::HZ, HN = TILE::HN;
  __shared__ double prop[HN][C_N + 1], own[TN][O_N];
  __shared__ int first_well[TY * TZ];
  __shared__ swt_t swt;
  __shared__ wvis_t wvis;
  const int64_t nxy = (int64_t)nx * ny;
  const int tid = threadIdx.x, tx = (nx + TX - 1) / TX, ty = (ny + TY - 1) / TY;
  const int wg = (int)rs_wg(), bt = wg / tx, i0 = (wg - bt * tx) * TX;
  const int k0 = bt / ty * TZ, j0 = (bt - bt / ty * ty) * TY;
  if (k0 >= nz) return;                                 // past the last tile
  // What the second half needs of global memory is asked for first: the
  // workgroup's time is latencies one after another.
  const int r = tid & 3, l = tid >> 2, a = l % TX, b = l / TX % TY, d = l / (TX * TY);
  const int i = i0 + a, j = j0 + b, k = k0 + d;
  const bool cell = i < nx && j < ny && k < nz;
  const int64_t c = cell ? i + nx * (j + (int64_t)ny * k) : 0;
  const csr7_row w = csr7_of((uint32_t)c, (uint32_t)nx, (uint32_t)ny, (uint32_t)nz);
  // lane r of a quad takes the permeabilities of faces r and r + 4 (in the
  // order -z -y -x +x +y +z)
  double k1[2], k2[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int f = min(r + 4 * h, 5);
    const int ax = h ? (f == 4 ? 1 : 2) : (f == 3 ? 0 : 2 - f);
    const bool in = (w.mask >> (f < 3 ? f : f + 1)) & 1u;
    const int64_t st = ax == 0 ? 1 : (ax == 1 ? (int64_t)nx : nxy);
    const double *kk = ax == 0 ? kx : (ax == 1 ? ky : kz);
    k1[h] = kk[c];
    k2[h] = kk[in ? (f < 3 ? c - st : c + st) : c];
  }
  const int mo = min(1 + r, 3);
  const double un = u[4 * c + mo], uo = uold[4 * c + mo];
  if (tid < 128) swt.fill(kSwt, tid);
  else wvis.fill(kWvis, tid - 128);
  double u4[4];
  bool eval = false;
  const bool old = tid >= HN;
  {
    int ta, tb, td;
    TILE::cell(old ? min(tid - HN, TN - 1) : tid, ta, tb, td);
    const int ti = i0 + ta, tj = j0 + tb, tk = k0 + td;
    if (ti >= 0 && ti < nx && tj >= 0 && tj < ny && tk >= 0 && tk < nz && tid < HN + TN) {
      eval = true;
      ld4v((old ? uold : u) + 4 * (ti + nx * (tj + (int64_t)ny * tk)), u4);
    }
  }
  __syncthreads();
  if (eval) {
    if (old) own[tid - HN][O_EOLD] = cell_energy(q, u4);
    else cell_eval(q, u4, swt, wvis, prop[tid], tid < TN ? own[tid] : nullptr);
  } else if (tid >= HN + TN && tid < HN + TN + TY * TZ) {
    // threads without an evaluation: where the wells of each of the tile's
    // lines start (cells ascending and unique)
    const int t = tid - HN - TN;
    const int64_t c0 = i0 + nx * (j0 + t % TY + (int64_t)ny * (k0 + t / TY));
    int lo = 0, hi = nw;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (wcell[mid] < c0) lo = mid + 1; else hi = mid;
    }
    first_well[t] = lo;
  }
  __syncthreads();
  if (!cell) return;
  const double *A = prop[l], *W = own[l];
  const double acc = q.acc;
  // this equation's residual and row of the diagonal block
  double R, D[4];
  if (r < 2) {
    R = acc * (un - uo);
    for (int m = 0; m < 4; ++m) D[m] = m == 1 + r ? acc : 0.0;
  } else {
    R = r == 2 ? acc * (W[O_E] - W[O_EOLD]) : acc * W[O_VOL];
    for (int m = 0; m < 4; ++m) D[m] = acc * W[(r == 2 ? O_EU : O_VU) + m];
  }
  const int rr = min(r, 2);                             // the constraint has no flows: its terms are dropped below
  // LDS index of the neighbour across each face (-z -y -x +x +y +z)
  int nb[6];
  nb[0] = d > 0 ? l - TX * TY : HZ + a + TX * b;
  nb[1] = b > 0 ? l - TX : HY + a + TX * d;
  nb[2] = a > 0 ? l - 1 : HX + b + TY * d;
  nb[3] = a < TX - 1 ? l + 1 : HX + TY * TZ + b + TY * d;
  nb[4] = b < TY - 1 ? l + TX : HY + TX * TZ + a + TX * d;
  nb[5] = d < TZ - 1 ? l + TX * TY : HZ + TX * TY + a + TX * b;
  // Face factors that are the same for the four equations, handed on within
  // the quad by DPP: the transmissibility and 1 / (sum of the conductivities)
  double Gf[2], If[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int f = min(r + 4 * h, 5);
    const bool in = (w.mask >> (f < 3 ? f : f + 1)) & 1u;
    const double ks = k1[h] + k2[h];
    Gf[h] = ks > 0.0 ? q.ctrans * q.gc[h ? (f == 4 ? 1 : 2) : (f == 3 ? 0 : 2 - f)] * 2.0 * k1[h] * k2[h] / ks : 0.0;
    const int nf = h ? (f == 4 ? nb[4] : nb[5]) : (f == 0 ? nb[0] : f == 1 ? nb[1] : f == 2 ? nb[2] : nb[3]);
    const double ksum = A[C_KT] + prop[in ? nf : l][C_KT];
    If[h] = ksum > 0.0 ? 1.0 / ksum : 0.0;
  }
#pragma unroll
  for (int f = 0; f < 6; ++f) {
    const int s = f < 3 ? f : f + 1, ax = f < 3 ? 2 - f : f - 3, fl = f & 3;
    const double gh = f < 4 ? Gf[0] : Gf[1], ih = f < 4 ? If[0] : If[1];
    const double G = fl == 0 ? qb<0>(gh) : fl == 1 ? qb<1>(gh) : fl == 2 ? qb<2>(gh) : qb<3>(gh);
    const double ik = fl == 0 ? qb<0>(ih) : fl == 1 ? qb<1>(ih) : fl == 2 ? qb<2>(ih) : qb<3>(ih);
    if (!((w.mask >> s) & 1u)) continue;                // the same for the quad
    const double *B = prop[nb[f]];
    // upstream: the higher pressure, on a tie the lower-numbered cell
    const double pa = A[C_P], pb = B[C_P];
    const bool up_b = f >= 3 ? (pb > pa) : !(pa > pb);
    const double *U = up_b ? B : A;
    const double dp = pb - pa, gdp = G * dp;            // flow into c is positive for dp > 0
    const double gl = G * U[C_L + rr];
    // -dF/du in u_c and in u_b: the mobility's part falls to the upstream cell
    double O[4], F = gl * dp;
    for (int m = 0; m < 4; ++m) {
      const double t = gdp * U[C_LU + 4 * rr + m], tb = up_b ? t : 0.0;
      if (r < 3) D[m] -= t - tb;
      O[m] = 0.0 - tb;
    }
    if (r < 3) D[0] += gl;
    O[0] -= gl;
    if (r == 2) {                                       // conduction, harmonic mean of the conductivities
      const double Gc = q.gc[ax];
      const double ka = A[C_KT] * ik, kb = B[C_KT] * ik, dt = B[C_T] - A[C_T];
      const double gk = Gc * 2.0 * ka * B[C_KT], gd = Gc * dt * 2.0, da = gd * kb * kb, db = gd * ka * ka;
      F = F + gk * dt;
      for (int m = 0; m < 4; ++m) {
        D[m] -= da * A[C_KTU + m];
        O[m] -= db * B[C_KTU + m];
      }
      D[3] += gk;
      O[3] -= gk;
    }
    if (r < 3) R -= F;
    else O[0] = O[1] = O[2] = O[3] = 0.0;
    if (vals) {
      double2 *ob = (double2 *)(vals + 16 * (int64_t)csr7_pos(w, s) + 4 * r);
      ob[0] = make_double2(O[0], O[1]);
      ob[1] = make_double2(O[2], O[3]);
    }
  }
  int lo = first_well[l / TX], wc = lo < nw ? wcell[lo] : -1;
  while (wc >= 0 && wc < c) wc = ++lo < nw ? wcell[lo] : -1;
  if (wc == c && r < 3) {
    if (wkind[lo] > 0) {                         // injector: water rate (bbl/day of cold water)
      double dh;
      const double qw = wval[lo] * q.bbl_ft3 * q.rhow_ref;
      if (r == 0) R -= qw;
      if (r == 2) R -= qw * water_h(q, q.t_inj, dh);
    } else if (A[C_P] > q.p_bh) {                // producer at bottom-hole pressure: Q = -WI lambda (p - p_bh)
      const double wi = q.ctrans * wval[lo], drive = A[C_P] - q.p_bh;
      R -= -wi * A[C_L + r] * drive;
      for (int m = 0; m < 4; ++m) {
        const double dd = m == 0 ? 1.0 : 0.0;
        D[m] -= -wi * (A[C_LU + 4 * r + m] * drive + A[C_L + r] * dd);
      }
    }
  }
  if (vals) {
    double2 *db = (double2 *)(vals + 16 * (int64_t)csr7_pos(w, 3) + 4 * r);
    db[0] = make_double2(D[0], D[1]);
    db[1] = make_double2(D[2], D[3]);
  }
  if (res) res[4 * c + r] = R;
}

// wells must be ascending and unique, inside the grid.  One workgroup writes
// the flag whatever it finds; several (of a thread per well) set a zeroed one.
__global__ __launch_bounds__(1024) void k_thermal_wells_check(int64_t n, int nw, const int32_t *__restrict__ wcell,
                                                               int *__restrict__ bad) {
  int b = 0;
  for (int t = blockIdx.x * 1024 + threadIdx.x; t < nw; t += gridDim.x * 1024)
    if (wcell[t] < 0 || wcell[t] >= n || (t > 0 && wcell[t - 1] >= wcell[t])) b = 1;
  b = __syncthreads_or(b);
  if (threadIdx.x == 0 && (b || gridDim.x == 1)) *bad = b;
}
// Most wells that one workgroup checks; beyond, its steps of 1024 wells take
// longer than a launch that zeroes the flag.  Residual of 100x100x32 cells, one
// workgroup and many: 116 and 118 us with 16 thousand wells, 133 and 120 with
// 65 thousand, 283 and 128 with 320 thousand.
constexpr int WELLS_ONE_WG = 16384;

// (p, N_w, N_o, T) from (p, S_w, S_o, T): N = phi rho S
__global__ void k_thermal_state(int64_t n, rs_thermal_params q, const double *__restrict__ p,
                                const double *__restrict__ sw, const double *__restrict__ so,
                                const double *__restrict__ t, double *__restrict__ u) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  const double dp = p[c] - q.p_ref, dT = t[c] - q.t_ref;
  const double phi = q.por_ref * (1.0 + q.cpor * dp);
  const double rw = q.rhow_ref * exp(q.cpw * dp - q.ct1w * dT - 0.5 * q.ct2w * dT * dT + q.cptw * dp * dT);
  const double ro = q.rhoo_ref * exp(q.cpo * dp - q.ct1o * dT - 0.5 * q.ct2o * dT * dT + q.cpto * dp * dT);
  double2 *o = (double2 *)(u + 4 * c);
  o[0] = make_double2(p[c], phi * rw * sw[c]);
  o[1] = make_double2(phi * ro * so[c], t[c]);
}

}  // namespace

extern "C" void rs_thermal_params_default(rs_thermal_params *q) {
  if (!q) return;
  *q = rs_thermal_params{};
  q->dx = 29.17; q->dy = 29.17; q->dz = 10.0;
  q->dt = 1.0;
  q->ctrans = 1.127e-3 * 5.614583;
  q->p_ref = 14.696; q->t_ref = 60.0;
  q->rhow_ref = 3.4605; q->cpw = 3.0e-6; q->ct1w = 1.0e-4; q->ct2w = 0.0; q->cptw = 0.0;
  q->rhoo_ref = 0.2092; q->cpo = 5.0e-6; q->ct1o = 3.8e-4; q->ct2o = 0.0; q->cpto = 0.0;
  q->avisc_o = 0.287352; q->bvisc_o = 3728.2;
  q->cpl_o = 125.0;
  q->cpg[0] = 34.49885; q->cpg[1] = -0.01426; q->cpg[2] = 4.7356e-5; q->cpg[3] = -3.56759e-8;
  q->cpg[4] = 9.35531e-12;
  q->hvr_w = 4820.0; q->ev_w = 0.38; q->tcrit_w = 374.15;
  q->por_ref = 0.3; q->cpor = 5.0e-4;
  q->cp_rock = 35.0;
  q->kw = 8.6; q->ko = 1.8; q->kr = 24.0;
  q->pv_btu = 144.0 / 778.169;
  q->jmol_btu = 453.59237 / 1055.05585;
  q->p_bh = 17.0; q->t_inj = 450.0;
  q->bbl_ft3 = 5.614583;
}

extern "C" rs_status rs_thermal_assemble(int nx, int ny, int nz, const rs_thermal_params *q, const double *d_kx,
                                         const double *d_ky, const double *d_kz, const double *d_u,
                                         const double *d_uold, int nw, const int32_t *d_wcell,
                                         const int32_t *d_wkind, const double *d_wval, double *d_vals,
                                         double *d_res, void *stream) {
  if (!rs_grid_dims_ok(nx, ny, nz) || !q || !d_kx || !d_ky || !d_kz || !d_u || !d_uold || nw < 0 ||
      (nw > 0 && (!d_wcell || !d_wkind || !d_wval)) || (!d_vals && !d_res))
    return RS_E_ARG;
  const int64_t n = (int64_t)nx * ny * nz;
  const int64_t nnzb = n + 2 * ((int64_t)(nx - 1) * ny * nz + (int64_t)nx * (ny - 1) * nz + (int64_t)nx * ny * (nz - 1));
  if (n > INT32_MAX / 2 || nnzb > INT32_MAX) return RS_E_ARG;
  if (((uintptr_t)d_u | (uintptr_t)d_uold | (uintptr_t)d_vals | (uintptr_t)d_res) & 15) return RS_E_ARG;
  if (!(q->dt > 0.0) || !(q->dx > 0.0) || !(q->dy > 0.0) || !(q->dz > 0.0)) return RS_E_ARG;
  hipStream_t s = rs_stream(stream);
  if (nw > 0) {
    dbuf flag;
    RS_TRY(flag.alloc(sizeof(int)));
    const bool one = nw <= WELLS_ONE_WG;
    if (!one) RS_TRY(rs_fill32(flag.p, 0, 1, s));
    k_thermal_wells_check<<<one ? 1 : rs_grid(nw, 1024), 1024, 0, s>>>(n, nw, d_wcell, flag.as<int>());
    int h = 0;
    RS_HIP(hipGetLastError());
    RS_TRY(rs_wait_read(&h, flag.p, sizeof(int), s));
    if (h) return RS_E_ARG;
  }
  // Tiles of 8 x 4 x 2 cells, and on a grid one cell thick in x, where they
  // would hold 8 cells, or in two directions, tiles in its own shape.  Where it
  // is thick in x they are fast enough: 500x1x500 198 us, 700x700x1 194 (200 and
  // 333 with a thread per cell).  Others, with tiles of 8 x 4 x 2, a thread per
  // cell and now: 1x400x700 419, 225 and 83 us; 300000x1x1 314, 167 and 83;
  // 1x300000x1 643, 159 and 78; 1x1x300000 1597, 168 and 82.
  auto run = [&](auto t) {
    using TILE = decltype(t);
    k_thermal<TILE><<<rs_wgs(TILE::count(nx, ny, nz)), 256, 0, s>>>(nx, ny, nz, tpar(*q), d_kx, d_ky, d_kz, d_u, d_uold,
                                                                      nw, d_wcell, d_wkind, d_wval, d_vals, d_res);
  };
  if (ny == 1 && nz == 1) run(tile<64, 1, 1>{});
  else if (nx == 1 && nz == 1) run(tile<1, 64, 1>{});
  else if (nx == 1 && ny == 1) run(tile<1, 1, 64>{});
  else if (nx == 1) run(tile<1, 8, 8>{});
  else run(tile<8, 4, 2>{});
  RS_HIP(hipGetLastError());
  return RS_OK;
}

extern "C" rs_status rs_thermal_state(int64_t n, const rs_thermal_params *q, const double *d_p, const double *d_sw,
                                      const double *d_so, const double *d_t, double *d_u, void *stream) {
  if (n < 1 || !q || !d_p || !d_sw || !d_so || !d_t || !d_u || ((uintptr_t)d_u & 15)) return RS_E_ARG;
  hipStream_t s = rs_stream(stream);
  k_thermal_state<<<rs_grid(n), RS_BLOCK, 0, s>>>(n, *q, d_p, d_sw, d_so, d_t, d_u);
  RS_HIP(hipGetLastError());
  return RS_OK;
}
