// gmres.hip -- restarted, right-preconditioned flexible GMRES (the Krylov
// solver of Section "Linear Solver"), Arnoldi by classical Gram-Schmidt
// applied twice (CGS2), Givens rotations on the device.
//
// One Arnoldi step j after z_j = M^{-1} v_j and w = A z_j makes three passes
// over the basis, each reading every v_i (i <= j) once:
//   pass 1  h1 = V^T w,  ||w||^2
//   pass 2  h2 = V^T (w - V h1)            (w - V h1 in registers only)
//   pass 3  w = (w - V h1) - V h2;  ||w||^2
// which is classical Gram-Schmidt applied twice, with the same operations
// per entry as updating w in place after each pass.  Each pass reduces its
// dots itself (its last workgroup adds the partials in a fixed order), and the
// last workgroup of pass 3 also forms h = h1 + h2, applies the previous
// rotations, builds the new one and updates g: three launches where separate
// reductions and rotations took seven.  The normalisation v_{j+1} = w /
// h_{j+1,j} reads h_{j+1,j} from device memory.  The orders are functions of
// the length alone, so a solve is bitwise reproducible.  The host reads one
// posted status per step to decide whether to stop.
// Z (the preconditioned vectors of flexible GMRES) is stored in the
// preconditioner's precision; the SpMV and x += Z y read it as stored, so
// A Z = V H holds for the stored Z and x stays consistent in FP32 mode.
#include "rs_internal.h"
#include <math.h>
#include <string.h>

namespace {

#include "reduce.h"

// Device scalar block layout (doubles):
enum {
  S_H1 = 0,            // 64: pass-1 dots, [j+1] = ||w||^2 before orthogonalisation
  S_H2 = 64,           // 64: pass-2 dots
  S_HN = 129,          // h_{j+1,j}
  S_BETA = 130,        // norm of the residual at the cycle start
  S_STAT = 132,        // [0] |g_{j+1}|, [1] breakdown flag, [2] halt flag
  S_G = 136,           // 65: rotated rhs g
  S_CS = 208,          // 64
  S_SN = 272,          // 64
  S_Y = 336,           // 64
  S_H = 400,           // (m+1) x m Hessenberg, row-major with leading dim 64
  S_CNT = 400 + 65 * 64,   // the reductions' workgroup count (an unsigned)
  S_TOTAL
};

// the grid's sums of acc[0 .. K) and acc[MK] into out[0 .. K]
template <int MK>
__device__ __forceinline__ void store_dots(const double (&acc)[MK + 1], int K, double *__restrict__ part,
                                           unsigned *__restrict__ cnt, double *__restrict__ out) {
  double sum[(MK + 8) / 8];
  if (!reduce_grid<MK + 1>(acc, K, part, cnt, sum)) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int e = 0; e < (MK + 8) / 8; ++e)
    if (lane == 0 && wv + 8 * e <= K) out[wv + 8 * e] = sum[e];
}

// pass 1: out[k] = V_k . w (k < K), out[K] = w . w.  Two consecutive
// entries per thread and step (16-byte loads; N = 4n is even): this streams
// about 1.5x faster than one entry per step.
template <int MK>
__global__ __launch_bounds__(RED_T) void k_dots(int64_t N, int K, const double *__restrict__ V,
                                                const double *__restrict__ w, double *__restrict__ part,
                                                unsigned *__restrict__ cnt, double *__restrict__ out) {
  double acc[MK + 1];
#pragma unroll
  for (int k = 0; k <= MK; ++k) acc[k] = 0.0;
  const int64_t N2 = N >> 1;
  const double2 *w2 = (const double2 *)w;
  for (int64_t t = (int64_t)blockIdx.x * RED_T + threadIdx.x; t < N2; t += (int64_t)gridDim.x * RED_T) {
    const double2 wv = w2[t];
#pragma unroll
    for (int k = 0; k < MK; ++k)
      if (k < K) {
        const double2 v = ((const double2 *)(V + (int64_t)k * N))[t];
        acc[k] = fma(v.x, wv.x, acc[k]);
        acc[k] = fma(v.y, wv.y, acc[k]);
      }
    acc[MK] = fma(wv.x, wv.x, acc[MK]);
    acc[MK] = fma(wv.y, wv.y, acc[MK]);
  }
  store_dots<MK>(acc, K, part, cnt, out);
}

// pass 2: w' = w - sum_k h1[k] V_k formed in registers only,
//   out[k] = V_k . w', out[K] = w' . w'  (read-only: w is not written, which
//   saves a vector write per Arnoldi step, and a kernel that both streams
//   several vectors in and one out runs slower than a read-only one)
template <int MK>
__global__ __launch_bounds__(RED_T) void k_axpy_dots(int64_t N, int K, const double *__restrict__ V,
                                                     const double *__restrict__ h1, const double *__restrict__ w,
                                                     double *__restrict__ part, unsigned *__restrict__ cnt,
                                                     double *__restrict__ out) {
  double acc[MK + 1];
#pragma unroll
  for (int k = 0; k <= MK; ++k) acc[k] = 0.0;
  double g1[MK];
#pragma unroll
  for (int k = 0; k < MK; ++k) g1[k] = (k < K) ? h1[k] : 0.0;
  const int64_t N2 = N >> 1;
  const double2 *w2 = (const double2 *)w;
  for (int64_t t = (int64_t)blockIdx.x * RED_T + threadIdx.x; t < N2; t += (int64_t)gridDim.x * RED_T) {
    double2 vk[MK];
    double2 wv = w2[t];
#pragma unroll
    for (int k = 0; k < MK; ++k) {
      vk[k] = (k < K) ? ((const double2 *)(V + (int64_t)k * N))[t] : make_double2(0.0, 0.0);
      wv.x = fma(-g1[k], vk[k].x, wv.x);
      wv.y = fma(-g1[k], vk[k].y, wv.y);
    }
#pragma unroll
    for (int k = 0; k < MK; ++k)
      if (k < K) {
        acc[k] = fma(vk[k].x, wv.x, acc[k]);
        acc[k] = fma(vk[k].y, wv.y, acc[k]);
      }
    acc[MK] = fma(wv.x, wv.x, acc[MK]);
    acc[MK] = fma(wv.y, wv.y, acc[MK]);
  }
  store_dots<MK>(acc, K, part, cnt, out);
}

// The rotations of step j by one wave, nrm2 = ||w||^2 after pass 3.  Lane i
// holds entry i of the column and rotation i; the chain over them runs on
// values read from their lanes.  Posts |g_{j+1}| and the breakdown flag.
// S_STAT[2] = 1 when the solve stops after this step (converged within tol,
// broken down or not finite), else 0.
__device__ __forceinline__ void givens_step(int j, double nrm2, double *__restrict__ S, double tol,
                                            rs_post *__restrict__ post, uint64_t seq) {
  double *H = S + S_H, *g = S + S_G;
  const int lane = threadIdx.x;
  const int li = min(lane, j);
  double h = (0.0 + S[S_H1 + li]) + S[S_H2 + li];
  const double cl = S[S_CS + li], sl = S[S_SN + li], gj = g[j], wn0 = sqrt(S[S_H1 + j + 1]);
  const double hn = sqrt(nrm2);
  double a = lane_value(h, 0);
  for (int i = 0; i < j; ++i) {
    const double c = lane_value(h, i + 1), cs = lane_value(cl, i), sn = lane_value(sl, i);
    const double u = cs * a + sn * c;
    a = -sn * a + cs * c;
    if (lane == i) h = u;
  }
  const double d = hypot(a, hn), cj = a / d, sj = hn / d;
  if (lane == j) h = d;
  if (lane <= j) H[lane * 64 + j] = h;
  if (lane != 0) return;
  S[S_HN] = hn;
  H[(j + 1) * 64 + j] = 0.0;
  S[S_CS + j] = cj;
  S[S_SN + j] = sj;
  const double gn = -sj * gj;
  g[j + 1] = gn;
  g[j] = cj * gj;
  const double est = fabs(gn);
  const bool brk = hn <= 1e-14 * wn0;
  S[S_STAT + 0] = est;
  S[S_STAT + 1] = brk ? 1.0 : 0.0;
  S[S_STAT + 2] = (brk || !(est > tol) || isinf(est)) ? 1.0 : 0.0;
  const double v[2] = {est, brk ? 1.0 : 0.0};
  post_host(post, seq, v, 2);
}

// pass 3: w' formed again with the operations of pass 2, then
// w'' = w' - sum_k h2[k] V_k stored into w, ||w''||^2, and the rotations
template <int MK>
__global__ __launch_bounds__(RED_T) void k_axpy_norm(int64_t N, int K, const double *__restrict__ V,
                                                     double *__restrict__ w, double *__restrict__ part,
                                                     double *__restrict__ S, double tol,
                                                     rs_post *__restrict__ post, uint64_t seq) {
  double g1[MK], g2[MK];
#pragma unroll
  for (int k = 0; k < MK; ++k) {
    g1[k] = (k < K) ? S[S_H1 + k] : 0.0;
    g2[k] = (k < K) ? S[S_H2 + k] : 0.0;
  }
  double acc[1] = {0.0};
  const int64_t N2 = N >> 1;
  double2 *w2 = (double2 *)w;
  for (int64_t t = (int64_t)blockIdx.x * RED_T + threadIdx.x; t < N2; t += (int64_t)gridDim.x * RED_T) {
    double2 vk[MK];
    double2 wv = w2[t];
#pragma unroll
    for (int k = 0; k < MK; ++k) {
      vk[k] = (k < K) ? ((const double2 *)(V + (int64_t)k * N))[t] : make_double2(0.0, 0.0);
      wv.x = fma(-g1[k], vk[k].x, wv.x);
      wv.y = fma(-g1[k], vk[k].y, wv.y);
    }
#pragma unroll
    for (int k = 0; k < MK; ++k) {
      wv.x = fma(-g2[k], vk[k].x, wv.x);
      wv.y = fma(-g2[k], vk[k].y, wv.y);
    }
    w2[t] = wv;
    acc[0] = fma(wv.x, wv.x, acc[0]);
    acc[0] = fma(wv.y, wv.y, acc[0]);
  }
  double sum[1];
  if (reduce_grid<1>(acc, 0, part, (unsigned *)(S + S_CNT), sum) && threadIdx.x < 64)
    givens_step(K - 1, sum[0], S, tol, post, seq);
}

// partials of ||w||^2 for k_cycle
__global__ __launch_bounds__(RED_T) void k_norm(int64_t N, const double *__restrict__ w, double *__restrict__ part) {
  __shared__ double sh[RED_T / 64];
  double acc = 0.0;
  const int64_t N2 = N >> 1;
  const double2 *w2 = (const double2 *)w;
  for (int64_t t = (int64_t)blockIdx.x * RED_T + threadIdx.x; t < N2; t += (int64_t)gridDim.x * RED_T) {
    const double2 wv = w2[t];
    acc = fma(wv.x, wv.x, acc);
    acc = fma(wv.y, wv.y, acc);
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 63) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double v = sh[0];
#pragma unroll
    for (int q = 1; q < RED_T / 64; ++q) v += sh[q];
    part[blockIdx.x] = v;
  }
}

// Start of a cycle, one workgroup: beta = the norm whose nb partials k_norm
// left, g = beta e_1, and the words that the passes count on.  The halt flag
// is set where there is nothing to iterate on.  Posts ||.||^2 and whether a
// sweep's bounded wait has timed out (err0, err1, either may be null).
__global__ __launch_bounds__(RED_T) void k_cycle(int nb, const double *__restrict__ part, double *__restrict__ S,
                                                 double rtol, const int *__restrict__ err0,
                                                 const int *__restrict__ err1, rs_post *__restrict__ post,
                                                 uint64_t seq) {
  __shared__ double sh[RED_T / 64];
  const int t = threadIdx.x;
  double s = wave_sum(t < nb ? part[t] : 0.0);
  if ((t & 63) == 63) sh[t >> 6] = s;
  __syncthreads();
  double nrm2 = sh[0];
#pragma unroll
  for (int q = 1; q < RED_T / 64; ++q) nrm2 += sh[q];
  const double beta = sqrt(nrm2);
  if (t < 65) S[S_G + t] = t == 0 ? beta : 0.0;
  if (t != 0) return;
  S[S_BETA] = beta;
  S[S_STAT + 2] = (beta == 0.0 || !isfinite(beta) || beta <= rtol * beta) ? 1.0 : 0.0;
  *(unsigned *)(S + S_CNT) = 0u;
  const double v[2] = {nrm2, ((err0 && *err0) || (err1 && *err1)) ? 1.0 : 0.0};
  post_host(post, seq, v, 2);
}

__global__ void k_backsolve(int k, double *__restrict__ S) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double *H = S + S_H, *g = S + S_G, *y = S + S_Y;
  for (int i = k - 1; i >= 0; --i) {
    double s = g[i];
    for (int c = i + 1; c < k; ++c) s = s - H[i * 64 + c] * y[c];
    y[i] = s / H[i * 64 + i];
  }
}

// v = w / S[idx] (device scalar) or w / beta (host scalar when idx < 0)
__global__ void k_scale(int64_t N, const double *w, const double *__restrict__ S, int idx,
                        double beta, double *v) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= N) return;
  double d = idx >= 0 ? S[idx] : beta;
  v[t] = w[t] / d;
}

__global__ void k_zero(int64_t N, double *__restrict__ x) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < N) x[t] = 0.0;
}

template <class TZ>
__global__ void k_update_x(int64_t N, int k, const TZ *__restrict__ Z, const double *__restrict__ S,
                           double *__restrict__ x, int x_zero) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= N) return;
  const double *y = S + S_Y;
  double v = x_zero ? 0.0 : x[t];                // x_zero: x = 0, not yet written
  for (int i = 0; i < k; ++i) v = fma(y[i], (double)Z[(int64_t)i * N + t], v);
  x[t] = v;
}

}  // namespace

extern "C" void rs_gmres_opts_default(rs_gmres_opts *o) {
  if (!o) return;
  o->restart = 30;
  o->rtol = 1e-8;
  o->maxit = 300;
  o->zero_guess = 0;
}

extern "C" const char *rs_status_string(int st) {
  switch (st) {
    case RS_OK: return "ok";
    case RS_NOT_CONVERGED: return "not converged (maximum iterations reached)";
    case RS_E_ARG: return "invalid argument";
    case RS_E_HIP: return "HIP runtime error";
    case RS_E_NOMEM: return "device memory allocation failed";
    case RS_E_SINGULAR: return "singular block or coarsest matrix";
    case RS_E_NONFINITE: return "non-finite value";
    default: return "unknown status";
  }
}

// Gram-Schmidt of step K - 1: w against V_0 .. V_{K-1}, and its rotations
template <int MK>
static void run_cgs2(int64_t N, int K, const double *V, double *w, double *part, double *S, double tol,
                     rs_post *post, uint64_t seq, hipStream_t s) {
  const unsigned nb = red_grid(N >> 1);
  unsigned *cnt = (unsigned *)(S + S_CNT);
  k_dots<MK><<<nb, RED_T, 0, s>>>(N, K, V, w, part, cnt, S + S_H1);
  k_axpy_dots<MK><<<nb, RED_T, 0, s>>>(N, K, V, S + S_H1, w, part, cnt, S + S_H2);
  k_axpy_norm<MK><<<nb, RED_T, 0, s>>>(N, K, V, w, part, S, tol, post, seq);
}

template <class TZ>
static rs_status gmres_t(rs_bsr_s *A, rs_cpr_s *M, const double *b, double *x, const rs_gmres_opts &o,
                         rs_solve_info *info, hipStream_t s) {
  int64_t N = 4 * A->g.n;
  int m = o.restart;
  if (M->m != m) {
    M->m = 0;                                    // no workspace until every part of it is there
    RS_TRY(rs_yield(M, [&]() -> rs_status {
      RS_TRY(M->V.alloc(sizeof(double) * N * (m + 1)));
      RS_TRY(M->Z.alloc(sizeof(TZ) * N * m));
      RS_TRY(M->w.alloc(sizeof(double) * N));
      RS_TRY(M->part.alloc(sizeof(double) * RED_NB * 33));
      return M->scal.alloc(sizeof(double) * S_TOTAL);
    }));
    M->m = m;
  }
  double *V = M->V.as<double>(), *w = M->w.as<double>(), *part = M->part.as<double>(), *S = M->scal.as<double>();
  TZ *Z = M->Z.as<TZ>();
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
  unsigned gN = rs_grid(N);
  bool timed = false;                            // e1 is recorded after everything queued so far
  bool sweeps_failed = false;
  // ||v||^2 and the start of a cycle from v; e1 is recorded while the host
  // would only wait, for the case that the solve ends here
  auto start_cycle = [&](const double *v, uint64_t *seq) -> rs_status {
    *seq = rs_post_next(post);
    k_norm<<<red_grid(N >> 1), RED_T, 0, s>>>(N, v, part);
    k_cycle<<<1, RED_T, 0, s>>>((int)red_grid(N >> 1), part, S, o.rtol, err[0], err[1], post, *seq);
    RS_HIP(hipGetLastError());
    RS_HIP(hipEventRecord(e1, s));
    timed = true;
    return RS_OK;
  };
  auto read_norm = [&](uint64_t seq, double *nrm) -> rs_status {
    RS_TRY(rs_wait_post(post, seq, s));
    *nrm = sqrt(post->v[0]);
    sweeps_failed = post->v[1] != 0.0;
    return RS_OK;
  };
  do {
    // ||b||; from x0 = 0 the first step's first pass (V_0 = b / ||b||) is
    // queued behind it, and does nothing where the cycle has nothing to do
    uint64_t seq = 0;
    bool zero_start = o.zero_guess != 0;
    bool in_queued = false;                      // step j's first pass is already on the stream
    if ((st = start_cycle(b, &seq)) != RS_OK) break;
    if (zero_start && o.maxit > 0) {
      if ((st = rs_cpr_apply_in(M, b, S + S_BETA, V, S + S_STAT + 2, s)) != RS_OK) break;
      in_queued = true;
      timed = false;
    }
    double bnorm = 0.0;
    if ((st = read_norm(seq, &bnorm)) != RS_OK) break;
    if (!isfinite(bnorm)) { st = RS_E_NONFINITE; break; }
    if (bnorm == 0.0) {
      if (hipMemsetAsync(x, 0, sizeof(double) * N, s) != hipSuccess) st = RS_E_HIP;
      timed = false;
      relres = 0.0;
      break;
    }
    bool x_zero = false;                         // x = 0 is implied, not stored
    for (;;) {
      double beta;
      if (zero_start) {
        // x0 = 0: r0 = b, ||r0|| = ||b||, V_0 = b / ||b||
        x_zero = true;
        beta = bnorm;
      } else {
        // r = b - A x into V_0
        if ((st = rs_spmv_any(A, x, 64, V, b, s)) != RS_OK) break;
        if ((st = start_cycle(V, &seq)) != RS_OK) break;
        if ((st = read_norm(seq, &beta)) != RS_OK) break;
      }
      relres = beta / bnorm;
      if (!isfinite(beta)) { st = RS_E_NONFINITE; break; }
      if (beta <= o.rtol * bnorm) { st = RS_OK; break; }
      if (iters >= o.maxit) { st = RS_NOT_CONVERGED; break; }
      // V_0 = r0 / beta: from x0 = 0 (r0 = b) the preconditioner's first pass
      // forms it (with beta from S_BETA); a restart's residual is in V_0
      // itself and is scaled in place
      const bool v0_fused = zero_start;
      timed = false;
      if (!v0_fused) k_scale<<<gN, RS_BLOCK, 0, s>>>(N, V, S, -1, beta, V);
      zero_start = false;
      ++cycles;
      const double tol = o.rtol * bnorm;
      const int zp = sizeof(TZ) == 8 ? 64 : 32;
      int k = 0;
      for (int j = 0; j < m; ++j) {
        double *vj = V + (int64_t)j * N;
        TZ *zj = Z + (int64_t)j * N;
        // V_j = w / h_{j,j-1} is formed by the preconditioner's first pass
        if (j == 0 && !v0_fused) {
          st = rs_cpr_apply_any(M, vj, zj, zp, s);
        } else {
          if (!in_queued) st = rs_cpr_apply_in(M, j > 0 ? w : b, S + (j > 0 ? S_HN : S_BETA), vj, nullptr, s);
          if (st == RS_OK) st = rs_cpr_apply_rest(M, zj, zp, s);
        }
        in_queued = false;
        if (st != RS_OK) break;
        if ((st = rs_spmv_any(A, zj, zp, w, nullptr, s)) != RS_OK) break;
        seq = rs_post_next(post);
        if (j < 8) run_cgs2<8>(N, j + 1, V, w, part, S, tol, post, seq, s);
        else if (j < 16) run_cgs2<16>(N, j + 1, V, w, part, S, tol, post, seq, s);
        else run_cgs2<32>(N, j + 1, V, w, part, S, tol, post, seq, s);
        if (hipGetLastError() != hipSuccess) { st = RS_E_HIP; break; }
        ++iters;
        k = j + 1;
        // the device already runs the next step's first pass while the host
        // reads the status; it does nothing if the rotations set the halt
        // flag (the host stops on the same values)
        in_queued = j + 1 < m && iters < o.maxit;
        if (in_queued && (st = rs_cpr_apply_in(M, w, S + S_HN, vj + N, S + S_STAT + 2, s)) != RS_OK) break;
        if ((st = rs_wait_post(post, seq, s)) != RS_OK) break;
        est = post->v[0];
        if (!isfinite(est)) { st = RS_E_NONFINITE; break; }
        if (post->v[1] != 0.0) break;                            // happy breakdown
        if (est <= tol || iters >= o.maxit) break;
      }
      in_queued = false;
      if (st != RS_OK) break;
      k_backsolve<<<1, 64, 0, s>>>(k, S);
      k_update_x<TZ><<<gN, RS_BLOCK, 0, s>>>(N, k, Z, S, x, x_zero ? 1 : 0);
      x_zero = false;
      if (hipGetLastError() != hipSuccess) { st = RS_E_HIP; break; }
    }
    if (x_zero) {                                // stopped before any update
      k_zero<<<gN, RS_BLOCK, 0, s>>>(N, x);
      timed = false;
    }
    est = (bnorm > 0.0) ? est / bnorm : 0.0;
  } while (0);
  // the last cycle's start came after every sweep of the solve
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

extern "C" rs_status rs_gmres_solve(rs_bsr A, rs_cpr M, const double *d_b, double *d_x,
                                    const rs_gmres_opts *o, rs_solve_info *info, void *stream) {
  if (info) memset(info, 0, sizeof(*info));
  if (!A || !M || !d_b || !d_x || d_b == d_x || M->A != A) return RS_E_ARG;
  if (((uintptr_t)d_b | (uintptr_t)d_x) & 15) return RS_E_ARG;     // read 16 bytes at a time
  rs_gmres_opts opts;
  if (o) opts = *o; else rs_gmres_opts_default(&opts);
  if (opts.restart < 1 || opts.restart > 32 || opts.maxit < 0 || !(opts.rtol >= 0.0)) return RS_E_ARG;
  hipStream_t s = rs_stream(stream);
  return M->prec == 64 ? gmres_t<double>(A, M, d_b, d_x, opts, info, s)
                       : gmres_t<float>(A, M, d_b, d_x, opts, info, s);
}

extern "C" rs_status rs_adjoint_solve(rs_bsr A, int method, int prec, const rs_cpr_opts *co,
                                      const double *d_w, double *d_lambda, const rs_gmres_opts *o,
                                      rs_solve_info *info, void *stream) {
  if (info) memset(info, 0, sizeof(*info));
  if (!A || !d_w || !d_lambda || (((uintptr_t)d_w | (uintptr_t)d_lambda) & 15)) return RS_E_ARG;
  hipStream_t s = rs_stream(stream);
  rs_cpr_opts opts;
  if (co) opts = *co; else rs_cpr_opts_default(&opts);
  bool same = A->at_m && A->at_method == method && A->at_prec == prec &&
              memcmp(&A->at_opts, &opts, sizeof(opts)) == 0;
  if (!same) {
    if (A->at_m) { rs_cpr_destroy(A->at_m); A->at_m = nullptr; }
    if (A->at_d) { rs_dcpl_destroy(A->at_d); A->at_d = nullptr; }
    if (!A->at) {
      A->at = new rs_bsr_s();
      rs_status st = rs_transpose7(A, A->at, s);
      if (st != RS_OK) { delete A->at; A->at = nullptr; return st; }
    }
    RS_TRY(rs_decouple(A->at, method, prec, stream, &A->at_d));
    rs_status st = rs_cpr_setup(A->at, A->at_d, &opts, stream, &A->at_m);
    if (st != RS_OK) { rs_dcpl_destroy(A->at_d); A->at_d = nullptr; return st; }
    A->at_method = method; A->at_prec = prec; A->at_opts = opts;
  }
  return rs_gmres_solve(A->at, A->at_m, d_w, d_lambda, o, info, stream);
}
