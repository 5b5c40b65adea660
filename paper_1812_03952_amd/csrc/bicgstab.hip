// bicgstab.hip -- right-preconditioned BiCGSTAB with M = CPR, the Krylov
// method the paper's experiments use (Section "Linear Solver" names it beside
// GMRES).  Textbook recurrence (van der Vorst, 1992) with p^ = M^{-1} p and
// s^ = M^{-1} s, so the residual it updates is the original system's:
//   rho_i = (r^, r),  p = r + (rho_i / rho_{i-1})(alpha / omega)(p - omega v)
//   v = A p^,  alpha = rho_i / (r^, v),  s = r - alpha v
//   t = A s^,  omega = (t, s) / (t, t),  x += alpha p^ + omega s^,  r = s - omega t
// One iteration is seven launches besides the two CPR applications:
//   k_bcg_p      p = r + beta (p - omega v)    (beta from device scalars; not in a cycle's first)
//   SpMV         v = A p^  with the epilogue dot (r^, v), and its sum
//   k_bcg_s      s = r - alpha v in place of r, ||s||^2
//   SpMV         t = A s^  with the epilogue dots (t, s), (t, t), and their sums
//   k_bcg_xr     x += alpha p^ + omega s^, r = s - omega t, (r^, r), ||r||^2
// Every dot is reduced in two fixed-order stages, the second one by the last
// workgroup of the launch that forms the first, so a solve is bitwise
// reproducible.  alpha, beta and omega are formed on the device from the
// reduced dots; the device posts a few doubles to the host twice per iteration
// (after s and after r) to test convergence and breakdown.  p^ and s^ are stored in the
// preconditioner's precision and read as stored, so v = A p^ and t = A s^
// hold for the stored vectors.
#include "rs_internal.h"
#include <algorithm>
#include <math.h>
#include <string.h>

namespace {

#include "reduce.h"

// Device scalar block (doubles).
enum {
  B_RHO = 0,     // rho_i = (r^, r)
  B_RHOP,        // rho_{i-1}
  B_ALPHA,
  B_OMEGA,
  B_RV,          // (r^, v)
  B_SN,          // ||s||^2
  B_TS,          // (t, s)
  B_TT,          // (t, t)
  B_RN,          // ||r||^2
  B_CNT,         // the reductions' workgroup count (an unsigned)
  B_TOTAL
};

// out[k] = sum of part[k * nparts + b], b < nparts, in a fixed order, k < ND
// (the SpMV's lists of one partial per workgroup).  With a post: out[0] and
// whether a sweep's bounded wait has timed out go to the host.
template <int ND>
__global__ __launch_bounds__(RED_T) void k_bcg_sums(int64_t nparts, const double *__restrict__ part,
                                                    double *__restrict__ mid, unsigned *__restrict__ cnt,
                                                    double *__restrict__ out, const int *__restrict__ err0,
                                                    const int *__restrict__ err1, rs_post *__restrict__ post,
                                                    uint64_t seq) {
  double acc[ND], sum[1];
#pragma unroll
  for (int k = 0; k < ND; ++k) acc[k] = 0.0;
  for (int64_t b = (int64_t)blockIdx.x * RED_T + threadIdx.x; b < nparts; b += (int64_t)gridDim.x * RED_T)
#pragma unroll
    for (int k = 0; k < ND; ++k) acc[k] += part[k * nparts + b];
  if (!reduce_grid<ND>(acc, ND - 1, mid, cnt, sum)) return;
  if ((threadIdx.x & 63) == 0 && threadIdx.x < 64 * ND) out[threadIdx.x >> 6] = sum[0];
  if (post && threadIdx.x == 0) {
    const double v[2] = {sum[0], ((err0 && *err0) || (err1 && *err1)) ? 1.0 : 0.0};
    post_host(post, seq, v, 2);
  }
}

// The vector kernels take two consecutive entries per thread and step
// (16-byte loads; N = 4n is even), which streams markedly faster than one.
template <class TZ> struct pair_of;
template <> struct pair_of<double> {
  __device__ static double2 ld(const double *p, int64_t t) { return ((const double2 *)p)[t]; }
};
template <> struct pair_of<float> {
  __device__ static double2 ld(const float *p, int64_t t) {
    const float2 f = ((const float2 *)p)[t];
    return make_double2((double)f.x, (double)f.y);
  }
};

// partials of ||b||^2 as the SpMV's epilogue forms them (one workgroup per 256
// entries, the same tree): a norm and a dot of equal vectors are then equal,
// and so are a solve from a stored x = 0 and one with zero_guess.  Also zeroes
// the count of the later reductions.
__global__ __launch_bounds__(256) void k_bcg_norm2(int64_t N, const double *__restrict__ b, double *__restrict__ part,
                                                   unsigned *__restrict__ cnt) {
  __shared__ double sh[4];
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const double x = t < N ? b[t] : 0.0;
  double v = x * x;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
  if (blockIdx.x == 0 && threadIdx.x == 0) *cnt = 0u;
}

__global__ void k_bcg_zero(int64_t N, double *__restrict__ x) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < N) x[t] = 0.0;
}

// start of a cycle: r^ = p = r and rho = ||r||^2 (the shadow r^ is a copy of
// r, so (r^, r) = ||r||^2); with b given, x = 0 and r = b first
__global__ void k_bcg_start(int64_t N, const double *__restrict__ b, double *__restrict__ r, double *__restrict__ rh,
                            double *__restrict__ p, double *__restrict__ x, double *__restrict__ S) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < (N >> 1)) {
    const double2 v = b ? ((const double2 *)b)[t] : ((const double2 *)r)[t];
    if (b) {
      ((double2 *)r)[t] = v;
      ((double2 *)x)[t] = make_double2(0.0, 0.0);
    }
    ((double2 *)rh)[t] = v;
    ((double2 *)p)[t] = v;
  }
  if (t == 0) S[B_RHO] = S[B_RN];
}

// p = r + beta (p - omega v), beta = (rho / rho_prev) (alpha / omega)
__global__ __launch_bounds__(256) void k_bcg_p(int64_t N, const double *__restrict__ r, const double *__restrict__ v,
                                               double *__restrict__ p, const double *__restrict__ S) {
  const double beta = (S[B_RHO] / S[B_RHOP]) * (S[B_ALPHA] / S[B_OMEGA]), omega = S[B_OMEGA];
  double2 *p2 = (double2 *)p;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < (N >> 1); t += (int64_t)gridDim.x * blockDim.x) {
    const double2 rv = pair_of<double>::ld(r, t), vv = pair_of<double>::ld(v, t);
    double2 pv = p2[t];
    pv.x = rv.x + beta * (pv.x - omega * vv.x);
    pv.y = rv.y + beta * (pv.y - omega * vv.y);
    p2[t] = pv;
  }
}

// alpha = rho / (r^, v);  s = r - alpha v (in place);  ||s||^2
__global__ __launch_bounds__(RED_T) void k_bcg_s(int64_t N, double *__restrict__ r, const double *__restrict__ v,
                                                 double *__restrict__ S, double *__restrict__ part,
                                                 rs_post *__restrict__ post, uint64_t seq) {
  const double rv = S[B_RV], alpha = S[B_RHO] / rv;
  double acc[1] = {0.0}, sum[1];
  double2 *r2 = (double2 *)r;
  for (int64_t t = (int64_t)blockIdx.x * RED_T + threadIdx.x; t < (N >> 1); t += (int64_t)gridDim.x * RED_T) {
    const double2 vv = pair_of<double>::ld(v, t);
    double2 sv = r2[t];
    sv.x = sv.x - alpha * vv.x;
    sv.y = sv.y - alpha * vv.y;
    r2[t] = sv;
    acc[0] = fma(sv.x, sv.x, acc[0]);
    acc[0] = fma(sv.y, sv.y, acc[0]);
  }
  if (!reduce_grid<1>(acc, 0, part, (unsigned *)(S + B_CNT), sum) || threadIdx.x != 0) return;
  S[B_ALPHA] = alpha;
  S[B_SN] = sum[0];
  const double o[2] = {rv, sum[0]};
  post_host(post, seq, o, 2);
}

// x += alpha p^ (the iteration stopped at s)
template <class TZ>
__global__ void k_bcg_xa(int64_t N, const TZ *__restrict__ ph, const double *__restrict__ S, double *__restrict__ x) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < N) x[t] = x[t] + S[B_ALPHA] * (double)ph[t];
}

// omega = (t, s) / (t, t);  x += alpha p^ + omega s^;  r = s - omega t;
// (r^, r) and ||r||^2, and the scalars of the next iteration.  (t, t) == 0
// (breakdown) takes omega = 0: x += alpha p^ and r = s.
template <class TZ>
__global__ __launch_bounds__(RED_T) void k_bcg_xr(int64_t N, const TZ *__restrict__ ph, const TZ *__restrict__ sh,
                                                  const double *__restrict__ tv, const double *__restrict__ rh,
                                                  double *__restrict__ r, double *__restrict__ x,
                                                  double *__restrict__ S, double *__restrict__ part,
                                                  rs_post *__restrict__ post, uint64_t seq) {
  __shared__ double res[2];
  const double alpha = S[B_ALPHA], tt2 = S[B_TT], omega = tt2 != 0.0 ? S[B_TS] / tt2 : 0.0;
  double acc[2] = {0.0, 0.0}, sum[1];
  double2 *x2 = (double2 *)x, *r2 = (double2 *)r;
  for (int64_t t = (int64_t)blockIdx.x * RED_T + threadIdx.x; t < (N >> 1); t += (int64_t)gridDim.x * RED_T) {
    const double2 pp = pair_of<TZ>::ld(ph, t), ss = pair_of<TZ>::ld(sh, t);
    const double2 tt = pair_of<double>::ld(tv, t), hh = pair_of<double>::ld(rh, t);
    double2 xv = x2[t], rv = r2[t];
    xv.x = xv.x + alpha * pp.x + omega * ss.x;
    xv.y = xv.y + alpha * pp.y + omega * ss.y;
    rv.x = rv.x - omega * tt.x;
    rv.y = rv.y - omega * tt.y;
    x2[t] = xv;
    r2[t] = rv;
    acc[0] = fma(hh.x, rv.x, acc[0]);
    acc[0] = fma(hh.y, rv.y, acc[0]);
    acc[1] = fma(rv.x, rv.x, acc[1]);
    acc[1] = fma(rv.y, rv.y, acc[1]);
  }
  if (!reduce_grid<2>(acc, 1, part, (unsigned *)(S + B_CNT), sum)) return;
  if ((threadIdx.x & 63) == 0 && threadIdx.x < 128) res[threadIdx.x >> 6] = sum[0];
  __syncthreads();
  if (threadIdx.x != 0) return;
  S[B_OMEGA] = omega;
  S[B_RHOP] = S[B_RHO];
  S[B_RHO] = res[0];
  S[B_RN] = res[1];
  const double o[4] = {tt2, omega, res[0], res[1]};
  post_host(post, seq, o, 4);
}

}  // namespace

extern "C" void rs_bicgstab_opts_default(rs_bicgstab_opts *o) {
  if (!o) return;
  o->rtol = 1e-8;
  o->maxit = 300;
  o->zero_guess = 0;
}

template <class TZ>
static rs_status bicgstab_t(rs_bsr_s *A, rs_cpr_s *M, const double *b, double *x, const rs_bicgstab_opts &o,
                            rs_solve_info *info, hipStream_t s) {
  const int64_t N = 4 * A->g.n;
  const unsigned nsp = rs_spmv_blocks(A);
  const int zp = sizeof(TZ) == 8 ? 64 : 32;
  if (M->bprec != zp || !M->bvec.p) {
    RS_TRY(rs_yield(M, [&]() -> rs_status {
      RS_TRY(M->bvec.alloc(sizeof(double) * N * 5 + sizeof(TZ) * N * 2));
      RS_TRY(M->bpart.alloc(sizeof(double) * (2 * (size_t)nsp + 2 * RED_NB)));
      return M->bscal.alloc(sizeof(double) * B_TOTAL);
    }));
    M->bprec = zp;
  }
  double *r = M->bvec.as<double>(), *rh = r + N, *p = rh + N, *v = p + N, *tv = v + N;
  TZ *ph = (TZ *)(tv + N), *shv = ph + N;
  double *sp = M->bpart.as<double>(), *part = sp + 2 * (size_t)nsp, *S = M->bscal.as<double>();
  unsigned *cnt = (unsigned *)(S + B_CNT);
  rs_post *post = nullptr;
  RS_TRY(rs_post_slot(&post));
  const int *err[2];
  rs_sweep_errors(M, err);
  hipEvent_t e0, e1;
  RS_HIP(hipEventCreate(&e0));
  RS_HIP(hipEventCreate(&e1));
  RS_HIP(hipEventRecord(e0, s));
  rs_status st = RS_OK;
  int iters = 0, cycles = 0;
  double relres = 0.0, est = 0.0;
  const unsigned gN = rs_grid(N), gP = (unsigned)std::min<int64_t>(1024, rs_grid(N >> 1)), nv = red_grid(N >> 1), ns = red_grid(nsp);
  bool timed = false;                            // e1 is recorded after everything queued so far
  bool sweeps_failed = false;
  double rr = 0.0;                               // ||r||^2 of the last norm read
  uint64_t seq = 0;
  // the sum of the norm's partials into S[B_RN] and rr; e1 is recorded while
  // the host would only wait, for the case that the solve ends here
  auto read_norm = [&]() -> rs_status {
    seq = rs_post_next(post);
    k_bcg_sums<1><<<ns, RED_T, 0, s>>>(nsp, sp, part, cnt, S + B_RN, err[0], err[1], post, seq);
    RS_HIP(hipGetLastError());
    RS_HIP(hipEventRecord(e1, s));
    timed = true;
    RS_TRY(rs_wait_post(post, seq, s));
    rr = post->v[0];
    sweeps_failed = post->v[1] != 0.0;
    return RS_OK;
  };
  // r = b - A x and ||r||^2
  auto residual = [&]() -> rs_status {
    RS_TRY(rs_spmv_dots(A, x, 64, r, b, 1, nullptr, sp, s));
    return read_norm();
  };
  do {
    k_bcg_norm2<<<nsp, 256, 0, s>>>(N, b, sp, cnt);
    if ((st = read_norm()) != RS_OK) break;
    const double bnorm = sqrt(rr);
    if (!isfinite(bnorm)) { st = RS_E_NONFINITE; break; }
    if (bnorm == 0.0) {
      k_bcg_zero<<<gN, RS_BLOCK, 0, s>>>(N, x);
      timed = false;
      relres = 0.0;
      break;
    }
    bool zero_start = o.zero_guess != 0;
    for (;;) {
      // x0 = 0: r = b and ||r||^2 = ||b||^2 (already in S[B_RN])
      if (!zero_start && (st = residual()) != RS_OK) break;
      const double rn = sqrt(rr);
      relres = rn / bnorm;
      st = !isfinite(rn) ? RS_E_NONFINITE : (rn <= o.rtol * bnorm ? RS_OK : RS_NOT_CONVERGED);
      if (st != RS_NOT_CONVERGED || iters >= o.maxit) {
        if (zero_start) {
          k_bcg_zero<<<gN, RS_BLOCK, 0, s>>>(N, x);
          timed = false;
        }
        break;
      }
      st = RS_OK;
      ++cycles;
      timed = false;
      k_bcg_start<<<rs_grid(N >> 1), RS_BLOCK, 0, s>>>(N, zero_start ? b : nullptr, r, rh, p, x, S);
      zero_start = false;
      double rho = rr;                       // (r^, r) with r^ = r
      bool first = true, stop_early = false;
      while (iters < o.maxit) {
        if (rho == 0.0) { stop_early = first; break; }
        if (!first) k_bcg_p<<<gP, 256, 0, s>>>(N, r, v, p, S);
        if ((st = rs_cpr_apply_any(M, p, ph, zp, s)) != RS_OK) break;
        if ((st = rs_spmv_dots(A, ph, zp, v, nullptr, 1, rh, sp, s)) != RS_OK) break;
        k_bcg_sums<1><<<ns, RED_T, 0, s>>>(nsp, sp, part, cnt, S + B_RV, nullptr, nullptr, nullptr, 0);
        seq = rs_post_next(post);
        k_bcg_s<<<nv, RED_T, 0, s>>>(N, r, v, S, part, post, seq);
        if (hipGetLastError() != hipSuccess) { st = RS_E_HIP; break; }
        if ((st = rs_wait_post(post, seq, s)) != RS_OK) break;
        if (post->v[0] == 0.0) { stop_early = first; break; }   // r now holds garbage; x is untouched
        ++iters;
        const double sn = sqrt(post->v[1]);
        est = sn;
        if (!isfinite(sn)) { st = RS_E_NONFINITE; break; }
        if (sn <= o.rtol * bnorm) {
          k_bcg_xa<TZ><<<gN, RS_BLOCK, 0, s>>>(N, ph, S, x);
          break;
        }
        if ((st = rs_cpr_apply_any(M, r, shv, zp, s)) != RS_OK) break;
        if ((st = rs_spmv_dots(A, shv, zp, tv, nullptr, 2, r, sp, s)) != RS_OK) break;
        k_bcg_sums<2><<<ns, RED_T, 0, s>>>(nsp, sp, part, cnt, S + B_TS, nullptr, nullptr, nullptr, 0);
        seq = rs_post_next(post);
        k_bcg_xr<TZ><<<nv, RED_T, 0, s>>>(N, ph, shv, tv, rh, r, x, S, part, post, seq);
        if (hipGetLastError() != hipSuccess) { st = RS_E_HIP; break; }
        if ((st = rs_wait_post(post, seq, s)) != RS_OK) break;
        if (post->v[0] == 0.0) { stop_early = first; break; }   // x += alpha p^ was applied
        const double rnn = sqrt(post->v[3]), omega = post->v[1];
        est = rnn;
        rho = post->v[2];
        first = false;
        if (!isfinite(rnn)) break;
        if (rnn <= o.rtol * bnorm || omega == 0.0) break;
      }
      if (st != RS_OK) break;
      if (stop_early) {
        if ((st = residual()) != RS_OK) break;
        relres = sqrt(rr) / bnorm;
        st = relres <= o.rtol ? RS_OK : RS_NOT_CONVERGED;
        break;
      }
    }
    est = bnorm > 0.0 ? est / bnorm : 0.0;
  } while (0);
  // the last norm read came after every sweep of the solve
  if ((st == RS_OK || st == RS_NOT_CONVERGED) && sweeps_failed) st = RS_E_HIP;
  float ms = 0.f;
  if (!timed) (void)hipEventRecord(e1, s);
  (void)hipEventSynchronize(e1);
  (void)hipEventElapsedTime(&ms, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (info) {
    info->iters = iters;
    info->cycles = cycles;
    info->status = st;
    info->relres = relres;
    info->est_relres = est;
    info->ms = ms;
  }
  return st;
}

extern "C" rs_status rs_bicgstab_solve(rs_bsr A, rs_cpr M, const double *d_b, double *d_x,
                                       const rs_bicgstab_opts *o, rs_solve_info *info, void *stream) {
  if (info) memset(info, 0, sizeof(*info));
  if (!A || !M || !d_b || !d_x || d_b == d_x || M->A != A) return RS_E_ARG;
  if (((uintptr_t)d_b | (uintptr_t)d_x) & 15) return RS_E_ARG;     // read 16 bytes at a time
  rs_bicgstab_opts opts;
  if (o) opts = *o; else rs_bicgstab_opts_default(&opts);
  if (opts.maxit < 0 || !(opts.rtol >= 0.0)) return RS_E_ARG;
  hipStream_t s = rs_stream(stream);
  return M->prec == 64 ? bicgstab_t<double>(A, M, d_b, d_x, opts, info, s)
                       : bicgstab_t<float>(A, M, d_b, d_x, opts, info, s);
}
