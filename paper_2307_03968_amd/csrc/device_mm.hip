// Many-right-hand-side kernels of libhmps for gfx950: the near/far panel
// products and the stage-A low-rank products become dense contractions
// (panel m x c times inputs c x nrhs), so they run on the matrix cores:
//   FP32 blocks: Gauss 3M complex product on v_mfma_f32_16x16x4f32,
//     T1 = Ar Xr, T2 = Ai Xi, T3 = (Ar + Ai)(Xr + Xi), Re = T1 - T2,
//     Im = T3 - T1 - T2 (three real products instead of four);
//   FP64 blocks: four real products on v_mfma_f64_16x16x4f64.
// MFMA 16x16x4 operand layout (lane l): A[i][k] with i = l % 16, k = l / 16;
// B[k][j] with k = l / 16, j = l % 16.  Result element v of lane l is
// D[4 (l / 16) + v][l % 16] for the FP32 instruction and D[l / 16 + 4 v][l % 16]
// for the FP64 one (both measured on gfx950).
//
// The inputs are kept in row layout (the right-hand sides of one source point
// contiguous), so the B operand of a k-step (4 panel columns x 16 right-hand
// sides) is four 128- or 256-byte rows read straight from L2 with one load
// per lane.  A workgroup takes a piece (panel columns [c0, c1) of a leaf) for
// one tile of right-hand sides; its four waves split the piece's rows or its
// columns (term_piece), and every wave streams its part with the loads of a
// few k-steps in flight.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dev.h"

namespace hm {

namespace {

// k-steps of four panel columns in flight per wave with R row tiles and T
// right-hand-side tiles (R + T loads per k-step, 16 bytes each in FP64, at
// most 16 in FP32): few enough registers that two workgroups fit a CU, whose
// waves cover each other's waits.  The 32^3 cube's 64-RHS term, one
// workgroup per CU and 12 (FP32) or 4 (FP64) deep: 850 and 1,840 us; two,
// 4 and 2 deep: 832 and 1,770 us.
template <int PM>
constexpr int mm_depth(int R, int T) {
  constexpr bool F32 = PM != 0;
  if (R == 1) return F32 ? (T == 4 ? 12 : 8) : 4;
  return F32 ? 4 : (R * T >= 8 ? 2 : (R + T <= 3 ? 6 : 4));
}

constexpr int kThreads = 256;
typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d4v __attribute__((ext_vector_type(4)));
typedef double dvec2 __attribute__((ext_vector_type(2)));
typedef float fvec2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// Device-coherent (agent-scope) loads and stores of the row-layout vectors
// and x in the multi-term launch, where one term's values are read by
// waves of any XCD in the next term.
__device__ __forceinline__ float2 load_co(const float2* p) {
  const uint64_t v =
      __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  float2 r;
  __builtin_memcpy(&r, &v, sizeof(r));
  return r;
}
__device__ __forceinline__ double2 load_co(const double2* p) {
  const double* d = reinterpret_cast<const double*>(p);
  return make_double2(__hip_atomic_load(d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                      __hip_atomic_load(d + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void store_co(float2* p, float2 v) {
  uint64_t u;
  __builtin_memcpy(&u, &v, sizeof(u));
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_co(double2* p, double2 v) {
  double* d = reinterpret_cast<double*>(p);
  __hip_atomic_store(d, v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(d + 1, v.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 16-byte device-coherent (agent-scope) load and store of entry idx of an
// array; the base is the same for the whole wave.
constexpr int kAgentScope = 16;  // buffer cache policy: sc1
typedef int ivec4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const double2* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const uint64_t u = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)a);
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), 0,
                                           __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}
__device__ __forceinline__ double2 load_rsrc(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off) {
  const dvec2 d = __builtin_bit_cast(
      dvec2, (ivec4)__builtin_amdgcn_raw_buffer_load_b128(rs, byte_off, 0, kAgentScope));
  return make_double2(d.x, d.y);
}
__device__ __forceinline__ void store_rsrc(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off, double2 v) {
  dvec2 d;
  d.x = v.x;
  d.y = v.y;
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(ivec4, d), rs, byte_off, 0, kAgentScope);
}

// Block precision and products of a kernel.
constexpr int kF64 = 0, kF32 = 1, kMix = 2;
template <int PM>
struct Prec;

template <>
struct Prec<kF32> {                      // FP32 blocks, 3M
  using A = float2;                      // panel element
  using X = float2;                      // input element (row layout)
  using Acc = f4v;
  static constexpr int NACC = 3;
  __device__ static __forceinline__ A load_a(const void* P, uint32_t byte_off) {
    const fvec2 v = __builtin_nontemporal_load(
        reinterpret_cast<const fvec2*>(reinterpret_cast<const char*>(P) + byte_off));
    return make_float2(v.x, v.y);
  }
  // the lane's elements of RTL row tiles of one column, from the byte offset
  // of row kLaneRows * (lane mod 16) of the column: row tiles in pairs of 32
  // rows by one 16-byte load (two consecutive rows per lane), an odd last
  // one by itself (lane_b: the bytes of lane mod 16 rows)
  static constexpr int kLaneRows = 2;
  template <int RTL>
  __device__ static __forceinline__ void load_col(const void* P, uint32_t off, uint32_t lane_b,
                                                  A (&a)[RTL]) {
#pragma unroll
    for (int r = 0; r + 1 < RTL; r += 2) {
      const f4v v = __builtin_nontemporal_load(
          reinterpret_cast<const f4v*>(reinterpret_cast<const char*>(P) + (off + 16 * r * 8)));
      a[r] = make_float2(v.x, v.y);
      a[r + 1] = make_float2(v.z, v.w);
    }
    if constexpr (RTL & 1) a[RTL - 1] = load_a(P, off - lane_b + 16 * (RTL - 1) * 8);
  }
  __device__ static __forceinline__ void mac(Acc (&acc)[3], float2 a, float as, X b, float bs) {
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc[1], 0, 0, 0);
    acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(as, bs, acc[2], 0, 0, 0);
  }
  __device__ static __forceinline__ float sum(float2 v) { return v.x + v.y; }
  __device__ static __forceinline__ double2 result(const Acc (&acc)[3], int v) {
    const double t1 = acc[0][v], t2 = acc[1][v], t3 = acc[2][v];
    return make_double2(t1 - t2, t3 - t1 - t2);
  }
  __device__ static __forceinline__ X from(double2 z) { return make_float2((float)z.x, (float)z.y); }
  // row of result element v within the 16 x 16 tile (kq = lane / 16)
  __device__ static __forceinline__ int row(int kq, int v) { return 4 * kq + v; }
};

template <>
struct Prec<kMix> : Prec<kF32> {         // FP32 blocks and inputs, FP64 products and sums
  using Acc = d4v;
  static constexpr int NACC = 2;
  __device__ static __forceinline__ void mac(Acc (&acc)[2], float2, double2 a, X, double2 b) {
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc[0], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, acc[1], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, acc[1], 0, 0, 0);
  }
  __device__ static __forceinline__ double2 sum(float2 v) { return make_double2(v.x, v.y); }
  __device__ static __forceinline__ double2 result(const Acc (&acc)[2], int v) {
    return make_double2(acc[0][v], acc[1][v]);
  }
  __device__ static __forceinline__ int row(int kq, int v) { return kq + 4 * v; }
};

template <>
struct Prec<kF64> {                      // FP64 blocks, four real products
  using A = double2;
  using X = double2;
  using Acc = d4v;
  static constexpr int NACC = 2;
  __device__ static __forceinline__ A load_a(const void* P, uint32_t byte_off) {
    const dvec2 v = __builtin_nontemporal_load(
        reinterpret_cast<const dvec2*>(reinterpret_cast<const char*>(P) + byte_off));
    return make_double2(v.x, v.y);
  }
  static constexpr int kLaneRows = 1;
  template <int RTL>
  __device__ static __forceinline__ void load_col(const void* P, uint32_t off, uint32_t, A (&a)[RTL]) {
#pragma unroll
    for (int r = 0; r < RTL; ++r) a[r] = load_a(P, off + 16 * r * 16);
  }
  __device__ static __forceinline__ void mac(Acc (&acc)[2], double2 a, double, X b, double) {
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc[0], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, acc[1], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, acc[1], 0, 0, 0);
  }
  __device__ static __forceinline__ double sum(double2) { return 0.0; }
  __device__ static __forceinline__ double2 result(const Acc (&acc)[2], int v) {
    return make_double2(acc[0][v], acc[1][v]);
  }
  __device__ static __forceinline__ X from(double2 z) { return z; }
  __device__ static __forceinline__ int row(int kq, int v) { return kq + 4 * v; }
};

template <int PM, int RT, int NT>
struct MMAcc {
  typename Prec<PM>::Acc a[RT][NT][Prec<PM>::NACC];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < Prec<PM>::NACC; ++q) a[r][t][q] = typename Prec<PM>::Acc{};
  }
};

// acc[r][t] += P[row0 + 16 r + (0..15), c0 : c1) X[src(c0 : c1), rhs0 + 16 t + (0..15)]
// for the RTL row tiles r < RTL of this wave.  P is column-major with
// leading dimension ld (its allocation extends at least 16 rows past the
// last column, so the row tiles need no clamp: rows past ld read the next
// column, and rows past m are never stored); srcf(c), c < c1, is the X row
// holding column c's input (columns past c1 take the row of zeros).  D k-steps
// of four columns are in flight: the panel loads of the first D start before
// `ready` is called, which makes srcf usable (it may hold a workgroup barrier).  Panel loads past c1 are issued
// at the clamped column c1 - 1; right-hand sides past the row length are
// read at the clamped column ldr - 1 (their products land in result columns
// that are never stored).  CO: the inputs are read with device-coherent
// loads (the multi-term launch).
template <int PM, int RT, int NT, int RTL, bool CO, typename SRCF, typename READY>
__device__ __forceinline__ void mm_wave(const void* __restrict__ P, uint32_t ld, int row0, int c0,
                                        int c1, const SRCF& srcf, const READY& ready,
                                        const typename Prec<PM>::X* __restrict__ xr, int64_t ldr,
                                        int zrow, int rhs0, MMAcc<PM, RT, NT>& acc, int lane) {
  using PR = Prec<PM>;
  using AV = typename PR::A;
  using XV = typename PR::X;
  constexpr int D = mm_depth<PM>(RT, NT);
  const int l16 = lane & 15, kq = lane >> 4;
  // byte offsets: the panel entries of a lane and the input rows stay
  // 32-bit (a panel set and a row-layout vector are below 2^32 bytes)
  constexpr uint32_t esz = sizeof(AV);
  const uint32_t a_first = (uint32_t)(row0 + PR::kLaneRows * l16 + (c0 + kq) * ld) * esz;
  const uint32_t a_last = (uint32_t)(row0 + PR::kLaneRows * l16 + (c1 - 1) * ld) * esz;
  const uint32_t a_step = 4u * ld * esz;
  uint32_t cx[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) cx[t] = (uint32_t)min<int64_t>(rhs0 + 16 * t + l16, ldr - 1);
  const uint32_t ldr32 = (uint32_t)ldr;
  const int nsteps = (c1 - c0 + 3) >> 2;
  AV ab[D][RTL];
  XV bb[D][NT];
  auto load_a = [&](int s, AV (&a)[RTL]) {
    PR::template load_col<RTL>(P, min(a_first + (uint32_t)s * a_step, a_last), (uint32_t)l16 * esz, a);
  };
  auto load_b = [&](int s, XV (&b)[NT]) {
    const int c = c0 + 4 * s + kq;
    const uint32_t rb = (uint32_t)(c < c1 ? srcf(c) : zrow) * ldr32;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if constexpr (CO) b[t] = load_co(xr + rb + cx[t]);
      else b[t] = xr[rb + cx[t]];
    }
  };
#pragma unroll
  for (int d = 0; d < D; ++d) load_a(d, ab[d]);
  ready();
#pragma unroll
  for (int d = 0; d < D; ++d) load_b(d, bb[d]);
  constexpr int U = (16 + D - 1) / D * D;
  for (int k = 0; k < nsteps; k += U) {
#pragma unroll
    for (int d = 0; d < U; ++d) {
      if (d > 0 && d % 2 == 0 && k + d >= nsteps) break;
      const int slot = d % D;
      decltype(PR::sum(XV{})) bs[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) bs[t] = PR::sum(bb[slot][t]);
#pragma unroll
      for (int r = 0; r < RTL; ++r) {
        const auto as = PR::sum(ab[slot][r]);
#pragma unroll
        for (int t = 0; t < NT; ++t) PR::mac(acc.a[r][t], ab[slot][r], as, bb[slot][t], bs[t]);
      }
      load_a(k + d + D, ab[slot]);
      load_b(k + d + D, bb[slot]);
      // keep this k-step's products and the refill of its ring slot where
      // they are: otherwise the scheduler gathers the products of many
      // k-steps first and issues the loads after them, leaving no time
      // between a load and its use
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// ---------------------------------------------------------------- term
// LDS of one workgroup, used in turn: the sources of the piece's columns
// while its products run, the exchange buffer of the column split (WK > 1),
// then the finished rows of sixteen right-hand sides z (right-hand side c,
// row i at c kZld + i; the odd leading dimension spreads the banks).
template <int RT, int NT, int WR>
struct MMShared {
  static constexpr int WK = 4 / WR;
  static constexpr int kZld = 16 * RT * WR + 1;
  union {
    int src[kMmMaxCols];
    double2 red[WK > 1 ? WR * WK * (WK - 1) * 256 : 1];
    double2 z[16 * kZld];
  };
  int s_last;
};

// Epilogue of a leaf's finished rows z (in LDS) for sixteen right-hand
// sides: y = alpha z + beta v and its stores.  The row-layout rows of y (the
// next term's input) go out with the right-hand sides of a row on
// consecutive threads; v, x, the column-layout y and the output have the
// rows of a right-hand side on consecutive threads (the other way round
// every lane of the x update touched its own cache line: 8 to 12 us a leaf
// of 47 rows and 16 right-hand sides).  MT: the multi-term launch, whose
// leaves' earlier terms may have run on another XCD (device-coherent
// accesses; the last term also writes the column-layout y and the output).
template <bool MT>
__device__ __forceinline__ void finish_tile(const TermArgs& A, const double2* z, int ldz, int64_t off,
                                            int m, int rhs0, int nrhs, const MMSeriesArgs* S, bool last) {
  constexpr int NRT = 16;
  const int nc = min(NRT, nrhs - rhs0);
  if (A.yrow || A.yrow32) {
    for (int idx = threadIdx.x; idx < m * NRT; idx += kThreads) {
      const int i = idx / NRT, c = idx % NRT;
      if (c >= nc) continue;
      const double2 q = z[c * ldz + i];
      const double2 y = make_double2(A.alpha * q.x, A.alpha * q.y);
      const int64_t at = (off + i) * A.ldr + rhs0 + c;
      if constexpr (MT) {
        if (A.yrow) store_co(A.yrow + at, y);
        if (A.yrow32) store_co(A.yrow32 + at, make_float2((float)y.x, (float)y.y));
      } else {
        if (A.yrow) A.yrow[at] = y;
        if (A.yrow32) A.yrow32[at] = make_float2((float)y.x, (float)y.y);
      }
    }
  }
  // rows padded to a power of two at least 16: thread -> (column, row)
  const int sh = m <= 16 ? 4 : (m <= 32 ? 5 : (m <= 64 ? 6 : (m <= 128 ? 7 : 8)));
  for (int idx = threadIdx.x; idx < (nc << sh); idx += kThreads) {
    const int i = idx & ((1 << sh) - 1), cl = idx >> sh, c = rhs0 + cl;
    if (i >= m) continue;
    const double2 q = z[cl * ldz + i];
    double2 y = make_double2(A.alpha * q.x, A.alpha * q.y);
    if constexpr (MT) {
      const int64_t at = off + i + (int64_t)c * A.ldxa;
      const double2 o = load_co(A.xacc + at);
      const double2 res = make_double2(y.x + o.x, y.y + o.y);
      store_co(A.xacc + at, res);
      if (last) {
        if (S->yout) S->yout[off + i + (int64_t)c * S->ldy] = y;
        if (S->out) S->out[S->out_perm[off + i] + (int64_t)c * S->ldo] = res;
      }
    } else {
      if (A.v) {
        const double2 v = A.v[off + i + (int64_t)c * A.ldv];
        y.x = fma(A.beta, v.x, y.x);
        y.y = fma(A.beta, v.y, y.y);
      }
      if (A.yout) A.yout[off + i + (int64_t)c * A.ldy] = y;
      double2 res = y;
      if (A.xacc) {
        const int64_t at = off + i + (int64_t)c * A.ldxa;
        if (A.accumulate) {
          const double2 o = A.xacc[at];
          res.x += o.x;
          res.y += o.y;
        }
        A.xacc[at] = res;
      }
      if (A.out) A.out[A.out_perm[off + i] + (int64_t)c * A.ldo] = res;
    }
  }
}

// Sum of the partial rows of all np pieces of a leaf for sixteen
// right-hand sides into z (LDS): every thread of the workgroup, the
// right-hand sides of a row on consecutive threads, the pieces in a fixed
// order.  A thread has the loads of four entries of four pieces in flight
// (the rows come from the device's coherence point, microseconds away).
__device__ __forceinline__ void sum_pieces(const TermArgs& A, int m, int np, int q0, int rhs0, int nrhs, int lane,
                           double2* z_out, int ldz) {
  constexpr int KE = 4, KP = 4, NRT = 16;
  const uint32_t rowb = (uint32_t)A.ldr * 16u;  // bytes of a row
  // every lane stays in the loop (entries past the end are clamped): the
  // piece rows are held across the lanes of the wave
  for (int b = 0; b < m * NRT; b += KE * kThreads) {
    const int e0 = b + (int)threadIdx.x;
    double2 z[KE];
    uint32_t bo[KE];
#pragma unroll
    for (int e = 0; e < KE; ++e) {
      const int idx = min(e0 + e * kThreads, m * NRT - 1);
      z[e] = make_double2(0.0, 0.0);
      // past the right-hand sides: the last one again, not used
      bo[e] = (uint32_t)(idx / NRT) * rowb + (uint32_t)min(rhs0 + idx % NRT, nrhs - 1) * 16u;
    }
    for (int p0 = 0; p0 < np; p0 += 64) {
      const int rows_l = A.lprow[q0 + min(p0 + lane, np - 1)];
      const int nc = min(64, np - p0);
      for (int p = 0; p < nc; p += KP) {
        double2 v[KP][KE];
#pragma unroll
        for (int u = 0; u < KP; ++u) {
          const int64_t row = __builtin_amdgcn_readlane(rows_l, min(p + u, nc - 1));
          const __amdgpu_buffer_rsrc_t rs = uniform_rsrc(A.partial + row * A.ldr, (uint32_t)m * rowb);
#pragma unroll
          for (int e = 0; e < KE; ++e) v[u][e] = load_rsrc(rs, bo[e]);
        }
#pragma unroll
        for (int u = 0; u < KP; ++u)
          if (p + u < nc) {
#pragma unroll
            for (int e = 0; e < KE; ++e) {
              z[e].x += v[u][e].x;
              z[e].y += v[u][e].y;
            }
          }
      }
    }
#pragma unroll
    for (int e = 0; e < KE; ++e) {
      const int idx = e0 + e * kThreads;
      if (idx < m * NRT) z_out[(idx % NRT) * ldz + idx / NRT] = z[e];
    }
  }
}

// The products of one wave over columns [c0, c1) for its rtl row tiles (at
// least one), the tile count a template argument from RT down.
template <int PM, int RT, int NT, int RTL, bool CO, typename SRCF, typename READY>
__device__ __forceinline__ void mm_wave_tiles(int rtl, const void* P, uint32_t ld, int row0, int c0,
                                              int c1, const SRCF& srcf, const READY& ready,
                                              const typename Prec<PM>::X* xr, int64_t ldr, int zrow,
                                              int rhs0, MMAcc<PM, RT, NT>& acc, int lane) {
  if constexpr (RTL > 1) {
    if (rtl < RTL) {
      mm_wave_tiles<PM, RT, NT, RTL - 1, CO>(rtl, P, ld, row0, c0, c1, srcf, ready, xr, ldr, zrow,
                                             rhs0, acc, lane);
      return;
    }
  }
  mm_wave<PM, RT, NT, RTL, CO>(P, ld, row0, c0, c1, srcf, ready, xr, ldr, zrow, rhs0, acc, lane);
}

// One piece on one workgroup.  Its four waves form WR row blocks (16 RT rows
// each) times WK = 4 / WR column ranges (the piece's columns in WK contiguous
// parts, multiples of four columns).  The waves of a row block add their
// tiles through LDS in FP64, in wave order: tile q goes to the wave q mod WK,
// which finishes it, so the sums are spread over the waves.  Then, for the
// leaf's only piece, the epilogue; else the partial sums are published with
// agent-scope stores and the workgroup that brings the (leaf, right-hand-side
// tile) counter to the piece count sums them and runs the epilogue.  Returns
// whether this workgroup ran it.  MT: the multi-term launch (coherent inputs
// and epilogue, S and last as in finish_tile).
template <int PM, int RT, int NT, int WR, bool MT = false>
__device__ __forceinline__ bool term_piece(const TermArgs& A, const MMPiece* __restrict__ pc, int tile,
                                           int ntiles, int nrhs, int w, int lane,
                                           MMShared<RT, NT, WR>& sh,
                                           const MMSeriesArgs* S = nullptr, bool last = false) {
  using PR = Prec<PM>;
  using XV = typename PR::X;
  constexpr int NRT = 16 * NT, WK = 4 / WR;
  // the piece is the same for the whole workgroup: keep it in scalar
  // registers (uniform branches, scalar base addresses)
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  auto uni64 = [&](int64_t v) {
    return (int64_t)(uint32_t)uni((int)(v & 0xffffffff)) | ((int64_t)uni((int)(v >> 32)) << 32);
  };
  const int a = uni(pc->leaf), m = uni(pc->m), pc0 = uni(pc->c0), pc1 = uni(pc->c1);
  const int np = uni(pc->np);
  const int64_t off = uni(pc->off);
  const int64_t prow = uni(pc->prow);
  const int64_t poff = uni64(pc->panel), coff = uni64(pc->col);
  const int rhs0 = tile * NRT;
  const int wr = w / WK, wk = w % WK;
  const uint32_t ld = (uint32_t)(m + (m & 1));
  const void* P = PM != kF64 ? (const void*)(reinterpret_cast<const float2*>(A.ps.data) + poff)
                      : (const void*)(reinterpret_cast<const double2*>(A.ps.data) + poff);
  const int32_t* __restrict__ src = A.ps.src + coff;
  const XV* xr = PM != kF64 ? reinterpret_cast<const XV*>(A.xr32) : reinterpret_cast<const XV*>(A.xr);
  MMAcc<PM, RT, NT> acc;
  acc.zero();
  const int row0 = wr * 16 * RT;
  const int rtl = min(RT, (m - row0 + 15) >> 4);
  // the wave's part of the columns
  const int part = ((pc1 - pc0 + 4 * WK - 1) / (4 * WK)) * 4;
  const int c0 = pc0 + wk * part, c1 = min(pc1, c0 + part);
  // every source of the piece in one pass, then the barrier
  auto ready = [&] {
    const int n = pc1 - pc0;
    for (int c = threadIdx.x; c < n; c += kThreads) sh.src[c] = src[pc0 + c];
    __syncthreads();
  };
  auto srcf = [&](int c) -> int { return sh.src[c - pc0]; };
  if (rtl > 0 && c1 > c0)
    mm_wave_tiles<PM, RT, NT, RT, MT>(rtl, P, ld, row0, c0, c1, srcf, ready, xr, A.ldr, A.zrow, rhs0,
                                      acc, lane);
  else
    ready();
  const int l16 = lane & 15, kq = lane >> 4;
  const __amdgpu_buffer_rsrc_t rs =
      uniform_rsrc(A.partial + prow * A.ldr, (uint32_t)m * (uint32_t)A.ldr * 16u);
  // row tiles the products ran with (the paired ones hold even and odd rows)
  const int tiles = max(rtl, 1);
  // element v of tile (r, t): the leaf's z (its only piece), or the piece's
  // partial row
  constexpr int kZld = MMShared<RT, NT, WR>::kZld;
  auto put = [&](int r, int t, int v, double2 z) {
    const int k = PR::row(kq, v);
    const int i = row0 + (PR::kLaneRows == 2 && (r | 1) < tiles ? 16 * (r & ~1) + 2 * k + (r & 1) : 16 * r + k);
    const int c = 16 * t + l16;
    if (i >= m || rhs0 + c >= nrhs) return;
    if (np == 1) sh.z[l16 * kZld + i] = z;
    else store_rsrc(rs, ((uint32_t)i * (uint32_t)A.ldr + (uint32_t)(rhs0 + c)) * 16u, z);
  };
  constexpr int kOwn = (RT * NT + WK - 1) / WK;
  double2 own[WK > 1 ? kOwn : 1][4];  // finished tiles of this wave
  __syncthreads();  // the sources are read: their LDS is free
  if constexpr (WK > 1) {
    // rounds of WK tiles: slot(o, u) holds writer u's values of owner o's tile
    auto slot = [&](int o, int u) -> double2* {
      return sh.red + ((wr * WK + o) * (WK - 1) + (u - (u > o))) * 256;
    };
#pragma unroll
    for (int q0 = 0; q0 < RT * NT; q0 += WK) {
      // row tiles past the leaf (the same for the whole workgroup when WR = 1)
      if (WR == 1 && q0 / NT >= tiles) break;
#pragma unroll
      for (int o = 0; o < WK; ++o) {
        const int q = q0 + o;
        if (q >= RT * NT || o == wk) continue;
        double2* d = slot(o, wk);
#pragma unroll
        for (int v = 0; v < 4; ++v) d[v * 64 + lane] = PR::result(acc.a[q / NT][q % NT], v);
      }
      __syncthreads();
#pragma unroll
      for (int o = 0; o < WK; ++o) {
        const int q = q0 + o;
        if (q >= RT * NT || o != wk) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double2 z = make_double2(0.0, 0.0);
#pragma unroll
          for (int u = 0; u < WK; ++u) {
            const double2 p = u == o ? PR::result(acc.a[q / NT][q % NT], v) : slot(o, u)[v * 64 + lane];
            z.x += p.x;
            z.y += p.y;
          }
          own[q0 / WK][v] = z;
        }
      }
      __syncthreads();
    }
  }
  // sixteen right-hand sides at a time
#pragma unroll
  for (int t = 0; t < NT; ++t) {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int q = r * NT + t;
      if (r >= tiles || (WK > 1 && q % WK != wk)) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if constexpr (WK > 1) put(r, t, v, own[q / WK][v]);
        else put(r, t, v, PR::result(acc.a[r][t], v));
      }
    }
    if (np == 1 && rhs0 + 16 * t < nrhs) {
      __syncthreads();
      finish_tile<MT>(A, sh.z, kZld, off, m, rhs0 + 16 * t, nrhs, S, last);
      __syncthreads();  // z is read: its LDS is free
    }
  }
  if (np == 1) return true;
  // the stores have completed at the device's coherence point before the
  // counter moves, so the workgroup that finishes the count reads them all
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  int32_t* cnt = A.counters + (int64_t)a * ntiles + tile;
  if (threadIdx.x == 0)
    sh.s_last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == np - 1;
  __syncthreads();
  const bool fin = sh.s_last != 0;
  if (fin) {
    for (int c = rhs0; c < min(nrhs, rhs0 + NRT); c += 16) {
      sum_pieces(A, m, np, uni(pc->lp0), c, nrhs, lane, sh.z, kZld);
      __syncthreads();
      finish_tile<MT>(A, sh.z, kZld, off, m, c, nrhs, S, last);
      __syncthreads();  // z is read: its LDS is free
    }
    if (threadIdx.x == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return fin;
}

// Term kernel: a workgroup runs the pieces of one unit for one tile of
// right-hand sides.  Bound by the matrix cores with 64 right-hand sides, by
// the panel reads with 16.  One wave per piece, and one wave to add up to 64
// partial rows a leaf, took 2,047 us a term on the sphere of 6,000 points (64
// RHS, FP32) where this split takes 62; with 16 RHS, FP64 on 16 instances 466
// us (now 300 to 340), FP32 on 64 instances 625 (now 547).
// Workgroups are dispatched to the eight XCDs in turn (workgroup b to XCD
// b mod 8), each XCD with its own L2.  XCD x runs a contiguous range of the
// units (their leaves read overlapping input rows), the tiles of one unit one
// after another, so that a panel is read from memory by one XCD at about one
// time; the plain order when the unit count is not a multiple of 8.
template <int PM, int RT, int NT, int WR>
__global__ __launch_bounds__(kThreads, 2) void k_term_mm(TermArgs A, int nrhs, int nunits, int ntiles) {
  __shared__ MMShared<RT, NT, WR> sh;
  const int lane = threadIdx.x & 63;
  const int w = wave_id();
  const int b = (int)blockIdx.x;
  const int j = (nunits & 7) ? b : b >> 3;
  const int unit = ((nunits & 7) ? 0 : (b & 7) * (nunits >> 3)) + j / ntiles;
  const int tile = j % ntiles;
  const int pe = A.wptr[unit + 1];
  for (int p = A.wptr[unit]; p < pe; ++p)
    term_piece<PM, RT, NT, WR>(A, A.mpieces + p, tile, ntiles, nrhs, w, lane, sh);
}

// ---------------------------------------------------------------- stage A
// t rows [row0, row0 + 16) of group g (one wave): W_g X[s_off .. s_off + n),
// written to the t rows of the same row-layout vector.  CO: device-coherent
// inputs and stores (the multi-term launch).
template <int PM, int NT, bool CO>
__device__ __forceinline__ void stageA_tile(const void* __restrict__ W, const Group& g, int row0,
                                            int rows, typename Prec<PM>::X* xr, int64_t ldr,
                                            int64_t N, int zrow, int rhs0, int nrhs, int lane) {
  using PR = Prec<PM>;
  if (row0 >= rows) return;
  const void* Wg = PM != kF64 ? (const void*)(reinterpret_cast<const float2*>(W) + g.w_off)
                       : (const void*)(reinterpret_cast<const double2*>(W) + g.w_off);
  MMAcc<PM, 1, NT> acc;
  acc.zero();
  const int s_off = g.s_off, n = g.n;
  auto srcf = [&](int c) -> int { return s_off + c; };
  mm_wave<PM, 1, NT, 1, CO>(Wg, (uint32_t)g.ld, row0, 0, n, srcf, [] {}, xr, ldr, zrow, rhs0, acc, lane);
  const int l16 = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int q = row0 + PR::row(kq, v);
      const int c = rhs0 + 16 * t + l16;
      if (q < rows && c < nrhs) {
        const auto z = PR::from(PR::result(acc.a[0][t], v));
        if constexpr (CO) store_co(xr + (N + g.t0 + q) * ldr + c, z);
        else xr[(N + g.t0 + q) * ldr + c] = z;
      }
    }
}

// One workgroup = a 64-row tile of a source group, wave w its rows
// [16 w, 16 w + 16).
template <int PM, int NT>
__global__ __launch_bounds__(kThreads) void k_stageA_mm(const void* __restrict__ W,
                                                        const Group* __restrict__ groups,
                                                        const GroupItem* __restrict__ items,
                                                        typename Prec<PM>::X* __restrict__ xr,
                                                        int64_t ldr, int64_t N, int zrow, int nrhs) {
  const GroupItem it = items[blockIdx.x];
  const int w = wave_id();
  stageA_tile<PM, NT, false>(W, groups[it.group], it.row0 + 16 * w, it.rows, xr, ldr, N, zrow,
                              blockIdx.y * 16 * NT, nrhs, threadIdx.x & 63);
}

// ---------------------------------------------------------------- multi-term
constexpr int kSeriesSpinLimit = 1 << 21;

// Waits (bounded) until *c reaches need; gives up setting *err.
__device__ __forceinline__ void wait_count(const int32_t* c, int need, int32_t* err) {
  if (need <= 0) return;
  for (int spins = 0; __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need; ++spins) {
    if (spins >= kSeriesSpinLimit ||
        __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
      __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    __builtin_amdgcn_s_sleep(2);
  }
}

// The K series terms of MMSeriesArgs in one launch; every workgroup takes
// items from the queue on its own.  The products and sums of an item are
// those of the per-term launches (term_piece, stageA_tile).
template <int PM, int NT>
__global__ __launch_bounds__(kThreads) void k_series_mm(TermArgs A, MMSeriesArgs S, int nrhs) {
  using PR = Prec<PM>;
  using XV = typename PR::X;
  __shared__ MMShared<4, NT, 1> sh;
  __shared__ int s_tk;
  const int lane = threadIdx.x & 63;
  const int w = wave_id();
  const int per = S.n_a + S.n_b;
  const int total = S.K * per;
  for (;;) {
    // one ticket per fetch: items differ widely in size, and a workgroup
    // holding several consecutive tickets leaves a long tail (measured)
    if (threadIdx.x == 0)
      s_tk = __hip_atomic_fetch_add(S.queue, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int tk = __builtin_amdgcn_readfirstlane(s_tk);
    if (tk >= total) break;
    const int k = tk / per + 1, j = tk - (k - 1) * per;
    const int kind = __builtin_amdgcn_readfirstlane(S.items[j].kind);
    const int inst = __builtin_amdgcn_readfirstlane(S.items[j].inst);
    const int ia = __builtin_amdgcn_readfirstlane(S.items[j].a);
    const int cur = (k - 1) & 1;
    int32_t* cnt_k = S.cnt + ((int64_t)inst * S.kmax + (k - 1)) * 2;  // [tiles, epilogues] of term k
    const int need_b = S.need_b[inst];
    if (threadIdx.x == 0) {
      // a term piece waits for its instance's t_k, both kinds for its y_{k-1}
      if (kind != 0) wait_count(cnt_k, S.need_a[inst], S.err);
      if (k > 1) wait_count(cnt_k - 2 + 1, need_b, S.err);
    }
    __syncthreads();  // also: s_tk has been read by every wave
    bool counted = true;
    if (kind == 0) {
      // stage-A tile: t_k rows [row0, row0 + kGroupTileMM) of group ia from y_{k-1}
      XV* xr = PM != kF64 ? reinterpret_cast<XV*>(S.r32[cur]) : reinterpret_cast<XV*>(S.r64[cur]);
      const int row0 = __builtin_amdgcn_readfirstlane(S.items[j].row0);
      const int rows = __builtin_amdgcn_readfirstlane(S.items[j].rows);
      stageA_tile<PM == kMix ? kF32 : PM, NT, true>(S.W, S.groups[ia], row0 + 16 * w, rows, xr, A.ldr, S.N, A.zrow, 0,
                                 nrhs, lane);
    } else {
      TermArgs T = A;
      T.xr = S.r64[cur];
      T.xr32 = S.r32[cur];
      T.yrow = PM != kF64 ? nullptr : S.r64[cur ^ 1];
      T.yrow32 = PM != kF64 ? S.r32[cur ^ 1] : nullptr;
      counted = term_piece<PM, 4, NT, 1, true>(T, A.mpieces + ia, 0, 1, nrhs, w, lane, sh, &S, k == S.K);
    }
    // the t rows, or y_k and x of a finished leaf, are complete before the count
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0 && counted)
      (void)__hip_atomic_fetch_add(cnt_k + (kind == 0 ? 0 : 1), 1, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
  }
  // the last workgroup out clears the queue and the counters for the next
  // launch.  Every count of a workgroup has landed before it counts itself
  // out: its later queue fetches return a value, and the wait for that value
  // covers all of that thread's earlier vector memory operations (gfx950
  // counts them with one in-order counter), so no increment arrives after
  // the clear.
  __syncthreads();
  if (threadIdx.x == 0)
    s_tk = __hip_atomic_fetch_add(S.queue + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (s_tk == (int)gridDim.x - 1) {
    for (int i = threadIdx.x; i < S.ninst * S.kmax * 2; i += kThreads)
      __hip_atomic_store(S.cnt + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x == 0) {
      __hip_atomic_store(S.queue, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(S.queue + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---------------------------------------------------------------- layout
// Column layout (n x nrhs, ld ldi, rows through perm when set) to row
// layout through a 64 x 16 LDS tile: reads coalesced along the rows, writes
// along the right-hand sides.
__global__ __launch_bounds__(kThreads) void k_rows(const double2* __restrict__ in, int64_t ldi,
                                                   const int64_t* __restrict__ perm, int64_t n,
                                                   int nrhs, double2* __restrict__ out,
                                                   float2* __restrict__ out32, int64_t ldr) {
  __shared__ double2 tile[16][65];
  const int64_t p0 = (int64_t)blockIdx.x * 64;
  const int c0 = blockIdx.y * 16;
  {
    const int pl = threadIdx.x & 63;
    const int64_t p = p0 + pl;
    const int64_t srow = (p < n) ? (perm ? perm[p] : p) : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int cl = (threadIdx.x >> 6) + 4 * j;
      const int c = c0 + cl;
      tile[cl][pl] = (p < n && c < nrhs) ? in[srow + (int64_t)c * ldi] : make_double2(0.0, 0.0);
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int cl = threadIdx.x & 15;
    const int pl = (threadIdx.x >> 4) + 16 * j;
    const int64_t p = p0 + pl;
    if (p >= n || c0 + cl >= ldr) continue;
    const double2 v = tile[cl][pl];
    if (out) out[p * ldr + c0 + cl] = v;
    if (out32) out32[p * ldr + c0 + cl] = make_float2((float)v.x, (float)v.y);
  }
}

// 16-column right-hand-side tiles per unit: the requested tile (16, 32 or
// 64), or by nrhs when 0; at most cap
inline int pick_nt(int nrhs, int tile, int cap) {
  int nt = (tile == 16 || tile == 32 || tile == 64) ? tile / 16 : (nrhs <= 16 ? 1 : (nrhs <= 32 ? 2 : 4));
  return nt < cap ? nt : cap;
}

// The same for the term kernel of a list of nunits units on cus compute
// units: the least padded work, a 16-RHS tile counted 1.2 times (it reads the
// panel per 16 right-hand sides: sphere 12,000, 64 RHS, FP64 1,495 us a solve
// against 1,226 with 32), a 64-RHS tile 1.03 times unless every CU has two
// units (128-row leaves: cube 20^3, 256 units, 1,547 against 1,538; cube 32^3,
// 512 units, the 64-RHS tile reads each panel once).  Narrower when that
// leaves fewer than two workgroups per CU (sphere 2,001, 64 RHS, FP32: 16-RHS
// tiles 167 us a solve, 32-RHS 213).
inline int pick_term_nt(int nrhs, int tile, int cap, int nunits, int cus) {
  if (tile != 0) return pick_nt(nrhs, tile, cap);
  const double weight[3] = {1.2, 1.0, nunits >= 2 * cus ? 0.97 : 1.03};
  int best = 1;
  double cost = 1e30;
  for (int q = 0, nt = 1; nt <= cap; ++q, nt *= 2) {
    const double c = (nrhs + 16 * nt - 1) / (16 * nt) * nt * weight[q];
    if (c < cost) {
      cost = c;
      best = nt;
    }
  }
  while (best > 1 && (int64_t)nunits * ((nrhs + 16 * best - 1) / (16 * best)) < 2 * cus) best /= 2;
  return best;
}

template <int PM, int RT, int NT, int WR>
hipError_t term_mm_launch(const TermArgs& a, int nunits, int nrhs, hipStream_t st) {
  const int ntiles = (nrhs + 16 * NT - 1) / (16 * NT);
  hipLaunchKernelGGL((k_term_mm<PM, RT, NT, WR>), dim3(nunits * ntiles), dim3(kThreads), 0, st, a,
                     nrhs, nunits, ntiles);
  return hipGetLastError();
}

// Row and column split of a workgroup by the largest leaf: at most 64 rows,
// every wave all rows of a quarter of the columns; at most 96, two row blocks
// of 48 and half the columns each (four blocks of 32 leave a wave idle on 86
// rows: cube 14^3, 64 RHS, FP64 593 us a solve against 482; sphere 24,576,
// leaves of 96, 2,665 against 2,273); else four row blocks.
template <int PM>
hipError_t term_mm_p(int max_m, const TermArgs& a, int nunits, int nrhs, int tile, int cus,
                     hipStream_t st) {
  const int nt = pick_term_nt(nrhs, tile, max_m <= 96 || max_m > 128 ? 2 : 4, nunits, cus);
  if (max_m <= kMmSmallLeaf)
    return nt == 1 ? term_mm_launch<PM, 4, 1, 1>(a, nunits, nrhs, st)
                   : term_mm_launch<PM, 4, 2, 1>(a, nunits, nrhs, st);
  if (max_m <= 96)
    return nt == 1 ? term_mm_launch<PM, 3, 1, 2>(a, nunits, nrhs, st)
                   : term_mm_launch<PM, 3, 2, 2>(a, nunits, nrhs, st);
  if (max_m <= 128)
    return nt == 1 ? term_mm_launch<PM, 2, 1, 4>(a, nunits, nrhs, st)
         : nt == 2 ? term_mm_launch<PM, 2, 2, 4>(a, nunits, nrhs, st)
                   : term_mm_launch<PM, 2, 4, 4>(a, nunits, nrhs, st);
  return nt == 1 ? term_mm_launch<PM, 4, 1, 4>(a, nunits, nrhs, st)
                 : term_mm_launch<PM, 4, 2, 4>(a, nunits, nrhs, st);
}

template <int PM>
hipError_t stageA_mm_p(const void* W, const Group* groups, const GroupItem* items, int nitems,
                       typename Prec<PM>::X* xr, int64_t ldr, int64_t N, int zrow, int nrhs,
                       int tile, hipStream_t st) {
  const int nt = pick_nt(nrhs, tile, 4);
  const dim3 grid(nitems, (nrhs + 16 * nt - 1) / (16 * nt));
  if (nt == 1)
    hipLaunchKernelGGL((k_stageA_mm<PM, 1>), grid, dim3(kThreads), 0, st, W, groups, items, xr, ldr,
                       N, zrow, nrhs);
  else if (nt == 2)
    hipLaunchKernelGGL((k_stageA_mm<PM, 2>), grid, dim3(kThreads), 0, st, W, groups, items, xr, ldr,
                       N, zrow, nrhs);
  else
    hipLaunchKernelGGL((k_stageA_mm<PM, 4>), grid, dim3(kThreads), 0, st, W, groups, items, xr, ldr,
                       N, zrow, nrhs);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_term_mm(bool f32, int max_m, const TermArgs& a, int nunits, int nrhs, int tile,
                          int cus, hipStream_t st) {
  if (nunits <= 0 || nrhs <= 0) return hipSuccess;
  if (max_m > 256 || a.ldr < row_ld(nrhs) || (f32 ? !a.xr32 : !a.xr)) return hipErrorInvalidValue;
  if (!f32) return term_mm_p<kF64>(max_m, a, nunits, nrhs, tile, cus, st);
  return a.fp64_sums ? term_mm_p<kMix>(max_m, a, nunits, nrhs, tile, cus, st)
                     : term_mm_p<kF32>(max_m, a, nunits, nrhs, tile, cus, st);
}

hipError_t launch_series_mm(bool f32, const TermArgs& a, const MMSeriesArgs& s, int nwg, int nrhs,
                            hipStream_t st) {
  if (nwg <= 0 || s.K <= 0) return hipSuccess;
  if (s.K > s.kmax || nrhs <= 0 || nrhs > 32 || a.ldr < row_ld(nrhs) || (f32 ? !a.xr32 : !a.xr) ||
      (int64_t)s.K * (s.n_a + s.n_b) >= ((int64_t)1 << 31))
    return hipErrorInvalidValue;
#define HM_SERIES_CASE(P, T)                                                                       \
  hipLaunchKernelGGL((k_series_mm<P, T>), dim3(nwg), dim3(kThreads), 0, st, a, s, nrhs)
  if (nrhs <= 16) {
    if (!f32) HM_SERIES_CASE(kF64, 1);
    else if (a.fp64_sums) HM_SERIES_CASE(kMix, 1);
    else HM_SERIES_CASE(kF32, 1);
  } else {
    if (!f32) HM_SERIES_CASE(kF64, 2);
    else if (a.fp64_sums) HM_SERIES_CASE(kMix, 2);
    else HM_SERIES_CASE(kF32, 2);
  }
#undef HM_SERIES_CASE
  return hipGetLastError();
}

int series_mm_occupancy(bool f32, int nrhs) {
  int n = 0;
  hipError_t e;
  if (nrhs <= 16)
    e = f32 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_series_mm<kF32, 1>, kThreads, 0)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_series_mm<kF64, 1>, kThreads, 0);
  else
    e = f32 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_series_mm<kF32, 2>, kThreads, 0)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_series_mm<kF64, 2>, kThreads, 0);
  return (e == hipSuccess && n > 0) ? n : 1;
}

hipError_t launch_stageA_mm(bool f32, const void* W, const Group* groups, const GroupItem* items,
                            int nitems, double2* xr, float2* xr32, int64_t ldr, int64_t N,
                            int zrow, int nrhs, int tile, hipStream_t st) {
  if (nitems <= 0 || nrhs <= 0) return hipSuccess;
  if (ldr < row_ld(nrhs) || (f32 ? !xr32 : !xr)) return hipErrorInvalidValue;
  return f32 ? stageA_mm_p<kF32>(W, groups, items, nitems, xr32, ldr, N, zrow, nrhs, tile, st)
             : stageA_mm_p<kF64>(W, groups, items, nitems, xr, ldr, N, zrow, nrhs, tile, st);
}

hipError_t launch_rows(const double2* in, int64_t ldi, const int64_t* perm, int64_t n, int nrhs,
                       double2* out, float2* out32, int64_t ldr, hipStream_t st) {
  if (n <= 0 || nrhs <= 0) return hipSuccess;
  if (ldr < row_ld(nrhs)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((n + 63) / 64), (unsigned)(ldr / 16));
  hipLaunchKernelGGL(k_rows, grid, dim3(kThreads), 0, st, in, ldi, perm, n, nrhs, out, out32, ldr);
  return hipGetLastError();
}

}  // namespace hm
