// Krylov kernels of libhmps: the vector work of restarted, right-
// preconditioned GMRES on Z_l (Saad and Schultz 1986; the flexible form of
// Saad 1993, which keeps the preconditioned vectors), one independent
// Krylov space per right-hand side.  The paper names GMRES as the iterative
// solver its power series is compared with; here the series P_K of Sec. IV
// serves as the preconditioner, which gives a converged solve also where
// rho(D^{-1} R_l) >= 1 and the series alone diverges.
//
// Vectors are N x nrhs column-major blocks (leading dimension ld); basis
// vector i of a block list starts at base + i * vs.  Per right-hand side c:
//   dots     h[i] = sum_r conj(V_i[r, c]) w[r, c], i < nvec, in two passes
//            (per-workgroup partial sums, then a fixed-order sum), so the
//            result does not depend on timing
//   orth     w[r, c] -= sum_i V_i[r, c] h[c, i] and, from the new w on chip,
//            the partial sums of the next pass's dots or of ||w||^2
//   update   y[r, c] += alpha sum_i V_i[r, c] coef[c, i]
//   step     the new Hessenberg column: previous Givens rotations, a new
//            rotation, the residual estimate |g_{j+1}| / ||b||; one wave per
//            right-hand side
//   solve    the upper-triangular least-squares system R y = g
// The vectors stay in the caches: every kernel here is bound by its launch and
// its chain of dependent steps, so the passes of an Arnoldi step are few (seven
// launches) and their sums are spread over waves.  24,576 rows, 30 vectors, one
// right-hand side: 94 us of kernels a step (thirteen launches and two copies)
// before, 31 us in seven so.
#include <hip/hip_runtime.h>

#include "dev.h"
#include "krylov.h"

namespace hm {

namespace {

constexpr int kKT = 256;  // threads per workgroup (one row each)

__device__ __forceinline__ double2 kzero() { return make_double2(0.0, 0.0); }

// conj(a) b
__device__ __forceinline__ double2 conj_mul(double2 a, double2 b) {
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

unsigned blocks_of(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// What k_orth leaves in partial: the dots of the vectors with w, or ||w||^2.
enum { kDots = 0, kNorm = 1 };

// One workgroup = kKT rows of column c (grid (nblk, nrhs)).  UPD: w[r, c] -=
// sum_i V_i[r, c] coef[c ldc + i], a thread per row, then the sums over the
// workgroup's rows of the new w:
//   kDots  partial[(c nvec + i) nblk + blk] = sum conj(V_i[r, c]) w[r, c]:
//          wave v takes the vectors v, v + 4, .., so that each sum is one
//          wave's and no vector waits for another's
//   kNorm  partial[c nblk + blk] = sum |w[r, c]|^2
template <bool UPD, int SUM>
__global__ __launch_bounds__(kKT) void k_orth(const double2* __restrict__ V, int64_t vs,
                                              int64_t ld, const double2* __restrict__ coef,
                                              int ldc, int nvec, double2* __restrict__ w,
                                              int64_t n, double2* __restrict__ partial) {
  __shared__ double2 cf[kMaxKrylov + 1];
  __shared__ double2 wl[kKT];
  const int blk = blockIdx.x, c = blockIdx.y, nblk = gridDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blk * kKT;
  const int64_t r = r0 + threadIdx.x;
  const bool ok = r < n;
  double2 wv = ok ? w[r + (int64_t)c * ld] : kzero();
  if constexpr (UPD) {
    for (int i = threadIdx.x; i < nvec; i += kKT) cf[i] = coef[(int64_t)c * ldc + i];
    __syncthreads();
    if (ok) {
      const double2* v = V + r + (int64_t)c * ld;
      double2 s = kzero();
#pragma unroll 8
      for (int i = 0; i < nvec; ++i) {
        const double2 p = cmul(v[(int64_t)i * vs], cf[i]);
        s.x += p.x;
        s.y += p.y;
      }
      wv.x -= s.x;
      wv.y -= s.y;
      w[r + (int64_t)c * ld] = wv;
    }
  }
  if constexpr (SUM == kNorm) {
    double q = wv.x * wv.x + wv.y * wv.y;
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) q += __shfl_xor(q, sh);
    if (lane == 0) wl[wave].x = q;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = wl[0].x;
#pragma unroll
      for (int k = 1; k < kKT / 64; ++k) t += wl[k].x;
      partial[(int64_t)c * nblk + blk] = make_double2(t, 0.0);
    }
  } else {
    wl[threadIdx.x] = wv;  // zero past the last row
    __syncthreads();
    constexpr int R = kKT / 64;
    double2 wr[R];
    int64_t q[R];  // rows past the last one re-read it and meet a zero
#pragma unroll
    for (int k = 0; k < R; ++k) {
      wr[k] = wl[lane + 64 * k];
      q[k] = min(r0 + lane + 64 * k, n - 1) + (int64_t)c * ld;
    }
#pragma unroll 2
    for (int i = wave; i < nvec; i += kKT / 64) {
      const double2* v = V + (int64_t)i * vs;
      double2 p = kzero();
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const double2 t = conj_mul(v[q[k]], wr[k]);
        p.x += t.x;
        p.y += t.y;
      }
#pragma unroll
      for (int sh = 32; sh > 0; sh >>= 1) {
        p.x += __shfl_xor(p.x, sh);
        p.y += __shfl_xor(p.y, sh);
      }
      if (lane == 0) partial[((int64_t)c * nvec + i) * nblk + blk] = p;
    }
  }
}

// Sum of nblk partial sums by one wave, in a fixed order (every lane gets it).
__device__ __forceinline__ double2 wave_sum(const double2* __restrict__ p, int nblk, int lane) {
  double2 s = kzero();
  for (int b = lane; b < nblk; b += 64) {
    s.x += p[b].x;
    s.y += p[b].y;
  }
#pragma unroll
  for (int sh = 32; sh > 0; sh >>= 1) {
    s.x += __shfl_xor(s.x, sh);
    s.y += __shfl_xor(s.y, sh);
  }
  return s;
}

// out[c ldo + i] = sum_blk partial[(c nvec + i) nblk + blk], a wave per sum
__global__ __launch_bounds__(kKT) void k_kreduce(const double2* __restrict__ partial, int nblk,
                                                 int nvec, int nrhs, double2* __restrict__ out,
                                                 int ldo) {
  const int t = blockIdx.x * (kKT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= nvec * nrhs) return;
  const int c = t / nvec, i = t % nvec;
  const double2 s = wave_sum(partial + (int64_t)t * nblk, nblk, lane);
  if (lane == 0) out[(int64_t)c * ldo + i] = s;
}

// y[r, c] += alpha sum_{i < nvec} V_i[r, c] coef[c ldc + i]; grid (rows, nrhs)
__global__ __launch_bounds__(kKT) void k_kupdate(double alpha, const double2* __restrict__ V,
                                                 int64_t vs, int64_t ld,
                                                 const double2* __restrict__ coef, int ldc,
                                                 int nvec, double2* __restrict__ y, int64_t n) {
  const int c = blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * kKT + threadIdx.x;
  if (r >= n) return;
  const int64_t q = r + (int64_t)c * ld;
  const double2* cf = coef + (int64_t)c * ldc;
  double2 s = kzero();
  for (int i = 0; i < nvec; ++i) {
    const double2 p = cmul(V[(int64_t)i * vs + q], cf[i]);
    s.x += p.x;
    s.y += p.y;
  }
  y[q].x += alpha * s.x;
  y[q].y += alpha * s.y;
}

// v[r, c] = s[c] v[r, c] (in place), and in v2 and v3 (one column) where given
__global__ __launch_bounds__(kKT) void k_kscale(double2* v, int64_t ld, const double* __restrict__ s,
                                                int64_t n, double2* __restrict__ v2,
                                                double2* __restrict__ v3) {
  const int c = blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * kKT + threadIdx.x;
  if (r >= n) return;
  const int64_t q = r + (int64_t)c * ld;
  const double f = s[c];
  const double2 x = make_double2(f * v[q].x, f * v[q].y);
  v[q] = x;
  if (v2) v2[r] = x;
  if (v3) v3[r] = x;
}

// The column's residual estimate and flag, also where the host reads them.
__device__ __forceinline__ void publish(const KrylovState& S, int c, double rel, bool go) {
  S.resid[c] = rel;
  S.act[c] = go ? 1 : 0;
  S.host_resid[c] = rel;
  S.host_act[c] = go ? 1 : 0;
}

// Start of a cycle: r = b - Z x is in the first basis slot, rn2 = ||r||^2
// and bn2 = ||b||^2 per column (real parts of the dot results).
__global__ void k_kstart(KrylovState S, const double2* __restrict__ rn2,
                         const double2* __restrict__ bn2, double tol, int nrhs) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nrhs) return;
  // a NaN norm stays NaN (fmax would turn it into 0, i.e. b = 0)
  const double rq = rn2[c].x, bq = bn2[c].x;
  const double rn = rq > 0.0 ? sqrt(rq) : (rq <= 0.0 ? 0.0 : rq);
  const double bn = bq > 0.0 ? sqrt(bq) : (bq <= 0.0 ? 0.0 : bq);
  double2* g = S.g + (int64_t)c * (S.m + 1);
  g[0] = make_double2(rn, 0.0);
  for (int i = 1; i <= S.m; ++i) g[i] = kzero();
  // b = 0 has the solution x = 0: nothing to do; a non-finite b or r gives
  // a NaN or infinite estimate (inactive, reported as not converged)
  const double rel = bn > 0 ? rn / bn : (bn == 0.0 ? 0.0 : bn);
  const bool go = bn > 0 && rn > 0 && rel > tol && isfinite(rel);
  S.bnorm[c] = bn;
  S.kc[c] = 0;
  publish(S, c, rel, go);
  S.inv[c] = go ? 1.0 / rn : 0.0;
}

// Arnoldi step j of column c (one wave): h = h1 + h2 (the two Gram-Schmidt
// passes), h_{j+1,j} = ||w|| from its nblk partial sums; the column is rotated
// by the earlier rotations, the new rotation zeroes h_{j+1,j}, and g follows.
// A column stays active while its residual estimate is above tol and the new
// basis vector is nonzero.  The chain of rotations runs on the column and the
// rotations in LDS (every lane alike), not on memory.
__global__ __launch_bounds__(64) void k_kstep(KrylovState S, int j, const double2* __restrict__ h1,
                                              const double2* __restrict__ h2, int ldh,
                                              const double2* __restrict__ hn2, int nblk,
                                              double tol) {
  __shared__ double2 Rl[kMaxKrylov + 1], sl[kMaxKrylov];
  __shared__ double cl[kMaxKrylov];
  const int c = blockIdx.x, lane = threadIdx.x;
  const int m = S.m;
  if (!S.act[c]) {
    if (lane == 0) {
      S.inv[c] = 0.0;
      publish(S, c, S.resid[c], false);
    }
    return;
  }
  double2* R = S.R + ((int64_t)c * m + j) * (m + 1);
  double* cs = S.cs + (int64_t)c * m;
  double2* sn = S.sn + (int64_t)c * m;
  double2* g = S.g + (int64_t)c * (m + 1);
  const double2 gj = g[j];
  for (int i = lane; i <= j; i += 64) {
    const double2 a = h1[(int64_t)c * ldh + i], b = h2[(int64_t)c * ldh + i];
    Rl[i] = make_double2(a.x + b.x, a.y + b.y);
    if (i < j) {
      cl[i] = cs[i];
      sl[i] = sn[i];
    }
  }
  const double hb = sqrt(fmax(wave_sum(hn2 + (int64_t)c * nblk, nblk, lane).x, 0.0));
  __syncthreads();
  // earlier rotations: [a; b] <- [cs a + sn b; -conj(sn) a + cs b]
  double2 a = Rl[0];
  for (int i = 0; i < j; ++i) {
    const double2 b = Rl[i + 1];
    const double ci = cl[i];
    const double2 sb = cmul(sl[i], b);
    const double2 sa = conj_mul(sl[i], a);
    if (lane == 0) R[i] = make_double2(ci * a.x + sb.x, ci * a.y + sb.y);
    a = make_double2(ci * b.x - sa.x, ci * b.y - sa.y);
  }
  // new rotation for (a, hb), hb real and >= 0: cs = |a| / t,
  // sn = (a / |a|) hb / t with t = sqrt(|a|^2 + hb^2); it maps (a, hb) to
  // ((a / |a|) t, 0).  For a = 0 it swaps the two rows (cs = 0, sn = 1),
  // which keeps |g| (no progress) when hb is zero too.
  const double aa = hypot(a.x, a.y), t = hypot(aa, hb);
  double cj;
  double2 sj, rj;
  if (aa == 0.0) {
    cj = 0.0;
    sj = make_double2(1.0, 0.0);
    rj = make_double2(hb, 0.0);
  } else {
    cj = aa / t;
    sj = make_double2(a.x / aa * hb / t, a.y / aa * hb / t);
    rj = make_double2(a.x / aa * t, a.y / aa * t);
  }
  const double2 sg = conj_mul(sj, gj);
  const double bn = S.bnorm[c];
  const double rel = bn > 0 ? hypot(sg.x, sg.y) / bn : 0.0;
  const bool go = hb > 0.0 && rel > tol && isfinite(rel);
  if (lane == 0) {
    R[j] = rj;
    cs[j] = cj;
    sn[j] = sj;
    g[j] = make_double2(cj * gj.x, cj * gj.y);
    g[j + 1] = make_double2(-sg.x, -sg.y);
    S.kc[c] = j + 1;
    S.inv[c] = go ? 1.0 / hb : 0.0;
    publish(S, c, rel, go);
  }
}

// y = R^{-1} g over the column's kc steps (zeros past kc, up to m)
__global__ void k_ksolve(KrylovState S, double2* __restrict__ y, int nrhs) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nrhs) return;
  const int m = S.m, k = S.kc[c];
  const double2* g = S.g + (int64_t)c * (m + 1);
  double2* yc = y + (int64_t)c * m;
  for (int i = k; i < m; ++i) yc[i] = kzero();
  for (int i = k - 1; i >= 0; --i) {
    double2 s = g[i];
    for (int l = i + 1; l < k; ++l) {
      const double2 p = cmul(S.R[((int64_t)c * m + l) * (m + 1) + i], yc[l]);
      s.x -= p.x;
      s.y -= p.y;
    }
    const double2 d = S.R[((int64_t)c * m + i) * (m + 1) + i];
    const double dd = d.x * d.x + d.y * d.y;
    // s / d = s conj(d) / |d|^2; a zero pivot (a zero column) gives 0
    yc[i] = dd > 0 ? make_double2((s.x * d.x + s.y * d.y) / dd, (s.y * d.x - s.x * d.y) / dd)
                   : kzero();
  }
}

}  // namespace

static void kreduce(const double2* partial, unsigned nblk, int nvec, int nrhs, double2* out,
                    int ldo, hipStream_t st) {
  hipLaunchKernelGGL(k_kreduce, dim3(blocks_of((int64_t)nvec * nrhs, kKT / 64)), dim3(kKT), 0, st,
                     partial, (int)nblk, nvec, nrhs, out, ldo);
}

hipError_t launch_kdots(const double2* V, int64_t vs, int64_t ld, const double2* w, int64_t n,
                        int nvec, int nrhs, double2* partial, double2* out, int ldo,
                        hipStream_t st) {
  if (n <= 0 || nrhs <= 0 || nvec <= 0) return hipSuccess;
  if (nvec > kMaxKrylov + 1) return hipErrorInvalidValue;
  const unsigned nblk = blocks_of(n, kKT);
  hipLaunchKernelGGL((k_orth<false, kDots>), dim3(nblk, nrhs), dim3(kKT), 0, st, V, vs, ld, nullptr,
                     0, nvec, const_cast<double2*>(w), n, partial);
  kreduce(partial, nblk, nvec, nrhs, out, ldo, st);
  return hipGetLastError();
}

hipError_t launch_korth(const double2* V, int64_t vs, int64_t ld, const double2* h1, double2* h2,
                        int ldh, int nvec, double2* w, int64_t n, int nrhs, double2* partial,
                        hipStream_t st) {
  if (n <= 0 || nrhs <= 0 || nvec <= 0) return hipSuccess;
  if (nvec > kMaxKrylov + 1) return hipErrorInvalidValue;
  const unsigned nblk = blocks_of(n, kKT);
  const dim3 grid(nblk, nrhs);
  hipLaunchKernelGGL((k_orth<true, kDots>), grid, dim3(kKT), 0, st, V, vs, ld, h1, ldh, nvec, w, n,
                     partial);
  kreduce(partial, nblk, nvec, nrhs, h2, ldh, st);
  hipLaunchKernelGGL((k_orth<true, kNorm>), grid, dim3(kKT), 0, st, V, vs, ld, h2, ldh, nvec, w, n,
                     partial);
  return hipGetLastError();
}

int64_t kdots_partials(int64_t n, int nvec, int nrhs) {
  return (int64_t)blocks_of(n, kKT) * nvec * nrhs;
}

hipError_t launch_kupdate(double alpha, const double2* V, int64_t vs, int64_t ld,
                          const double2* coef, int ldc, int nvec, double2* y, int64_t n, int nrhs,
                          hipStream_t st) {
  if (n <= 0 || nrhs <= 0 || nvec <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_kupdate, dim3(blocks_of(n, kKT), nrhs), dim3(kKT), 0, st, alpha, V, vs, ld,
                     coef, ldc, nvec, y, n);
  return hipGetLastError();
}

hipError_t launch_kscale(double2* v, int64_t ld, const double* s, int64_t n, int nrhs,
                         double2* v2, double2* v3, hipStream_t st) {
  if (n <= 0 || nrhs <= 0) return hipSuccess;
  if ((v2 || v3) && nrhs != 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_kscale, dim3(blocks_of(n, kKT), nrhs), dim3(kKT), 0, st, v, ld, s, n, v2, v3);
  return hipGetLastError();
}

hipError_t launch_kstart(const KrylovState& S, const double2* rn2, const double2* bn2, double tol,
                         int nrhs, hipStream_t st) {
  if (nrhs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_kstart, dim3(blocks_of(nrhs, 64)), dim3(64), 0, st, S, rn2, bn2, tol, nrhs);
  return hipGetLastError();
}

hipError_t launch_kstep(const KrylovState& S, int j, const double2* h1, const double2* h2, int ldh,
                        const double2* partial, int64_t n, double tol, int nrhs, hipStream_t st) {
  if (nrhs <= 0) return hipSuccess;
  if (j < 0 || j >= S.m || j >= kMaxKrylov || j + 1 > ldh) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_kstep, dim3(nrhs), dim3(64), 0, st, S, j, h1, h2, ldh, partial,
                     (int)blocks_of(n, kKT), tol);
  return hipGetLastError();
}

hipError_t launch_ksolve(const KrylovState& S, double2* y, int nrhs, hipStream_t st) {
  if (nrhs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ksolve, dim3(blocks_of(nrhs, 64)), dim3(64), 0, st, S, y, nrhs);
  return hipGetLastError();
}

}  // namespace hm
