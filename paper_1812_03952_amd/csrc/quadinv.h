// quadinv.h -- steps of the block ILU(0) factorisations on a quad of lanes per
// cell (lane r of the quad holds row r of each 4x4 block): the Schur update of
// a diagonal block by one neighbour, and the inverse of the result.  FP64,
// every element with the operations of the single-thread form in the same
// order (one multiply and one add per term, no contraction).
// Include inside an anonymous namespace after block4.h and quad4.h.
#pragma once

// Lr -= row r of A_cq (D_q^{-1} A_qc): dq, aqc and acq are this lane's rows of
// D_q^{-1}, A_qc and A_cq; the other rows come from the quad by DPP.
template <class T>
__device__ __forceinline__ void quad_schur(double (&Lr)[4], const T (&dq)[4], const T (&aqc)[4], const T (&acq)[4]) {
#pragma clang fp contract(off)
  double Aqc[4][4], t[4], Tm[4][4];
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) {
    Aqc[0][cc] = (double)qb<0>(aqc[cc]); Aqc[1][cc] = (double)qb<1>(aqc[cc]);
    Aqc[2][cc] = (double)qb<2>(aqc[cc]); Aqc[3][cc] = (double)qb<3>(aqc[cc]);
  }
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) {
    double v = (double)dq[0] * Aqc[0][cc];
#pragma unroll
    for (int m = 1; m < 4; ++m) v = v + (double)dq[m] * Aqc[m][cc];
    t[cc] = v;
  }
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) {
    Tm[0][cc] = qb<0>(t[cc]); Tm[1][cc] = qb<1>(t[cc]);
    Tm[2][cc] = qb<2>(t[cc]); Tm[3][cc] = qb<3>(t[cc]);
  }
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) {
    double v = (double)acq[0] * Tm[0][cc];
#pragma unroll
    for (int m = 1; m < 4; ++m) v = v + (double)acq[m] * Tm[m][cc];
    Lr[cc] = Lr[cc] - v;
  }
}

// Gauss-Jordan with row pivoting on [L | I], row r of L in Lr; on return Rr is
// row `mine` of the inverse.  The quad tracks the row permutation instead of
// moving rows: every lane takes the same pivot decision from the broadcast
// column.  Call it with whole quads active; returns RSF_* flags (0 = fine).
// While no quad of the wave has to pivot, which is the rule after a decoupling
// that scales the diagonal blocks to I, the pivot row is a fixed lane: it is
// read by DPP instead of through the LDS permute network, and the identity
// columns of R that no step has reached yet are left out (their entries are
// zeros that stay zero).
__device__ __forceinline__ int quad_inverse(double (&Lr)[4], double (&Rr)[4], int r, int wq, int &mine) {
#pragma clang fp contract(off)
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) Rr[cc] = cc == r ? 1.0 : 0.0;
  double rmax = 0.0;
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) rmax = fmax(rmax, fabs(Lr[cc]));
  const double amax = fmax(fmax(fmax(fmax(0.0, qb<0>(rmax)), qb<1>(rmax)), qb<2>(rmax)), qb<3>(rmax));
  mine = r;
  if (!isfinite(amax)) return RSF_NONFINITE;
  int bad = 0;
  bool ident = true;                            // no quad of the wave has pivoted so far
  unsigned perm = 0xE4u;                        // 2 bits per logical row k: its lane
  auto lane_of = [&](int k) { return (int)((perm >> (2 * k)) & 3u); };
  auto step = [&](auto pc) {
    constexpr int p = decltype(pc)::value;
    const double c0 = qb<0>(Lr[p]), c1 = qb<1>(Lr[p]), c2 = qb<2>(Lr[p]), c3 = qb<3>(Lr[p]);
    auto col = [&](int l) { return l == 0 ? c0 : (l == 1 ? c1 : (l == 2 ? c2 : c3)); };
    if (ident) {
      const double best = fabs(col(p));
      bool sw = false;
#pragma unroll
      for (int k = p + 1; k < 4; ++k) sw = sw || fabs(col(k)) > best;
      ident = __ballot(sw) == 0;
    }
    double pL[4], pR[4];
    if (ident) {
      double pv = col(p);
      if (fabs(pv) <= 1e-300 || fabs(pv) <= 1e-14 * amax) { bad |= RSF_SINGULAR; pv = 1.0; }
      const double inv = 1.0 / pv;
#pragma unroll
      for (int cc = p + 1; cc < 4; ++cc) pL[cc] = qb<p>(Lr[cc]) * inv;
#pragma unroll
      for (int cc = 0; cc <= p; ++cc) pR[cc] = qb<p>(Rr[cc]) * inv;
      const double f = Lr[p];
      const bool me = r == p;
#pragma unroll
      for (int cc = p + 1; cc < 4; ++cc) {
        const double u = Lr[cc] - f * pL[cc];
        Lr[cc] = me ? pL[cc] : u;
      }
#pragma unroll
      for (int cc = 0; cc <= p; ++cc) {
        const double u = Rr[cc] - f * pR[cc];
        Rr[cc] = me ? pR[cc] : u;
      }
    } else {
      int piv = p;
      double best = fabs(col(lane_of(p)));
#pragma unroll
      for (int k = p + 1; k < 4; ++k)
        if (fabs(col(lane_of(k))) > best) { best = fabs(col(lane_of(k))); piv = k; }
      const unsigned lp = (unsigned)lane_of(p), lq = (unsigned)lane_of(piv);
      perm = (perm & ~(3u << (2 * p)) & ~(3u << (2 * piv))) | (lq << (2 * p)) | (lp << (2 * piv));
      mine = mine == p ? piv : (mine == piv ? p : mine);
      const int src = wq + (int)lq;
      double pv = col((int)lq);
      if (fabs(pv) <= 1e-300 || fabs(pv) <= 1e-14 * amax) { bad |= RSF_SINGULAR; pv = 1.0; }
      const double inv = 1.0 / pv;
#pragma unroll
      for (int cc = p + 1; cc < 4; ++cc) pL[cc] = __shfl(Lr[cc], src, 64) * inv;
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) pR[cc] = __shfl(Rr[cc], src, 64) * inv;
      if (mine == p) {
#pragma unroll
        for (int cc = p + 1; cc < 4; ++cc) Lr[cc] = pL[cc];
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) Rr[cc] = pR[cc];
      } else {
        const double f = Lr[p];
#pragma unroll
        for (int cc = p + 1; cc < 4; ++cc) Lr[cc] = Lr[cc] - f * pL[cc];
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) Rr[cc] = Rr[cc] - f * pR[cc];
      }
    }
  };
  step(std::integral_constant<int, 0>{});
  step(std::integral_constant<int, 1>{});
  step(std::integral_constant<int, 2>{});
  step(std::integral_constant<int, 3>{});
  return bad;
}
