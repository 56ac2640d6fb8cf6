// Thin SVD of small matrices by one-sided (Hestenes) Jacobi rotations,
// the decomposition of the Spec's svd / trunc_svd for matrices whose
// smaller dimension is at most JACOBI_MAX_K.
//
// The Gram-matrix route of the large path squares the condition number, so
// singular values below about 1e-8 of the largest are not resolved there.
// One-sided Jacobi works on the columns of the matrix itself: every column
// pair (p, q) is rotated until |<a_p, a_q>| <= m 2^-53 ||a_p|| ||a_q||, and
// the singular values are the column norms.  They carry an absolute error of
// a few ulps of the largest one, which resolves the small values that the
// truncation of message products and of tiny bonds decides on.
//
// One workgroup per problem, 16 lanes per column pair (a DPP row, so that the
// inner product of a pair is summed without LDS round trips), or a wave per pair
// for a few long columns.  Pairs are scheduled by the round-robin (circle)
// ordering: n/2 disjoint pairs per step, n - 1 steps per sweep, a workgroup
// barrier between steps; a step has at most 32 pairs, and the workgroup processes
// all of them at once.  V and, when it fits, W live in LDS.  A step is a chain of
// latencies (LDS read, reduction, rotation scalars, LDS write, barrier), so the
// scalars come from reciprocal-square-root seeds refined by two Newton steps
// instead of the division and square-root sequences, the column norms are carried
// along within a sweep, and up to 64 rows a lane holds its elements in registers
// from the inner product to the rotation.  A call on one complex problem takes 383
// us at 32 x 32 (about 1 us per step) and 1131 us at 64 x 64 (a step moves up to
// 192 KiB of LDS); four waves that took the pairs in turn from global memory, a
// wave per pair, 1943 and 8174 us.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "jacobi.hpp"

namespace tci {

namespace {

__device__ inline double cj(double a) { return a; }
__device__ inline cd cj(cd a) { return cd{a.x, -a.y}; }
__device__ inline double sq(double a) { return a * a; }
__device__ inline double sq(cd a) { return a.x * a.x + a.y * a.y; }
__device__ inline double mulr(double a, double b) { return a * b; }
__device__ inline cd mulr(cd a, cd b) { return a * b; }
__device__ inline double scl(double s, double a) { return s * a; }
__device__ inline cd scl(double s, cd a) { return cd{s * a.x, s * a.y}; }
__device__ inline double addv(double a, double b) { return a + b; }
__device__ inline cd addv(cd a, cd b) { return a + b; }
__device__ inline double zero_of(double) { return 0.0; }
__device__ inline cd zero_of(cd) { return cd{0.0, 0.0}; }
__device__ inline double one_of(double) { return 1.0; }
__device__ inline cd one_of(cd) { return cd{1.0, 0.0}; }

__device__ inline double wsum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline cd wsum_c(cd v) { return cd{wsum(v.x), wsum(v.y)}; }
__device__ inline double wsum_c(double v) { return wsum(v); }

// Sum over the 16 lanes of a DPP row; every lane receives the same bits (the
// partners of each step add the same two values).
template <int CTRL>
__device__ inline double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
__device__ inline double row_sum(double v) {
  v = dpp_add<0xB1>(v);     // quad_perm [1,0,3,2]
  v = dpp_add<0x4E>(v);     // quad_perm [2,3,0,1]
  v = dpp_add<0x141>(v);    // row_half_mirror
  return dpp_add<0x140>(v); // row_mirror
}
__device__ inline cd row_sum(cd v) { return cd{row_sum(v.x), row_sum(v.y)}; }

__device__ inline double shfl_add(double v, int m) { return v + __shfl_xor(v, m, 64); }
__device__ inline cd shfl_add(cd v, int m) { return cd{shfl_add(v.x, m), shfl_add(v.y, m)}; }
// over the LP lanes of a column pair
template <int LP, typename T>
__device__ inline T pair_sum(T v) {
  v = row_sum(v);
  if constexpr (LP == 64) {
    v = shfl_add(v, 16);
    v = shfl_add(v, 32);
  }
  return v;
}

// 1 / sqrt(x) and 1 / x for positive finite x: hardware seed, two Newton steps
__device__ inline double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int k = 0; k < 2; ++k) y = __builtin_fma(y * 0.5, __builtin_fma(-x * y, y, 1.0), y);
  return y;
}
__device__ inline double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int k = 0; k < 2; ++k) y = __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
  return y;
}

// 1 / sqrt(1 + t^2).  As rsqrt_nr, but the last step's residual is taken from t,
// (1 - y^2) - (y t)^2: that of the rounded 1 + t^2 leaves c^2 + s^2 above one on
// average for small t, up to an ulp per rotation, and hundreds of rotations stretch
// the columns (by 35 u at 60 x 60).
__device__ inline double cos_of_tan(double t) {
  const double x = __builtin_fma(t, t, 1.0);
  double y = __builtin_amdgcn_rsq(x);
  y = __builtin_fma(y * 0.5, __builtin_fma(-x * y, y, 1.0), y);
  const double p = y * t;
  return __builtin_fma(y * 0.5, __builtin_fma(-p, p, __builtin_fma(-y, y, 1.0)), y);
}

// Modulus of z != 0, its reciprocal and the conjugate of its phase.  A real phase is exactly +-1: as z / |z| by a reciprocal it is below
// one by an ulp now and then, and hundreds of rotations shrink the columns.
// TINY: z may be 0 (then so are |z| and its reciprocal), and the square or the
// reciprocal of |z| outside the exponent range.
template <bool TINY>
__device__ inline void modulus(double z, double& r, double& ir, double& phc) {
  r = fabs(z);
  if constexpr (TINY) ir = r > 0.0 ? 1.0 / r : 0.0;
  else ir = rcp_nr(r);
  phc = copysign(1.0, z);
}
template <bool TINY>
__device__ inline void modulus(cd z, double& r, double& ir, cd& phc) {
  int ex = 0;
  if constexpr (TINY) {   // of z scaled to order one
    const double a = fmax(fabs(z.x), fabs(z.y));
    ex = a > 0.0 ? __builtin_amdgcn_frexp_exp(a) : 0;
    z = cd{__builtin_amdgcn_ldexp(z.x, -ex), __builtin_amdgcn_ldexp(z.y, -ex)};
  }
  const double r2 = z.x * z.x + z.y * z.y;
  ir = !TINY || r2 > 0.0 ? rsqrt_nr(r2) : 0.0;
  phc = cd{z.x * ir, -z.y * ir};
  r = r2 * ir;
  if constexpr (TINY) {
    r = __builtin_amdgcn_ldexp(r, ex);
    ir = __builtin_amdgcn_ldexp(ir, -ex);
  }
}

__device__ inline double amax_of(double v) { return fabs(v); }
__device__ inline double amax_of(cd v) { return fmax(fabs(v.x), fabs(v.y)); }
__device__ inline double ldexp_of(double v, int e) { return __builtin_amdgcn_ldexp(v, e); }
__device__ inline cd ldexp_of(cd v, int e) { return cd{__builtin_amdgcn_ldexp(v.x, e), __builtin_amdgcn_ldexp(v.y, e)}; }

// unit-modulus phase of z (1 for z = 0) and its modulus
__device__ inline void polar(double z, double& r, double& ph) {
  r = fabs(z);
  ph = z < 0.0 ? -1.0 : 1.0;
}
__device__ inline void polar(cd z, double& r, cd& ph) {
  r = sqrt(z.x * z.x + z.y * z.y);
  ph = r > 0.0 ? cd{z.x / r, z.y / r} : cd{1.0, 0.0};
}

// Orthonormal completion of vector r of the set vec(q)[i] = P[q*vs + i*is]
// (q < r already orthonormal, length len): the first unit vector e_t whose
// component orthogonal to them has norm > 1/2, or else the e_t with the largest
// one (a vector spread over all entries has no component above 1/2 anywhere),
// orthogonalised twice.  Run by one wave.
template <typename T>
__device__ void complete_vector(T* P, long long vs, long long is, int len, int r) {
  const int lane = threadIdx.x & 63;
  // v = e_t - sum_q conj(vec_q[t]) vec_q, twice; returns |v|^2
  auto attempt = [&](int t) -> double {
    for (int i = lane; i < len; i += 64) P[r * vs + i * is] = (i == t) ? one_of(T{}) : zero_of(T{});
    __threadfence_block();
    for (int pass = 0; pass < 2; ++pass) {
      for (int q = 0; q < r; ++q) {
        T c = zero_of(T{});
        for (int i = lane; i < len; i += 64) c = addv(c, mulr(cj(P[q * vs + i * is]), P[r * vs + i * is]));
        c = wsum_c(c);
        for (int i = lane; i < len; i += 64)
          P[r * vs + i * is] = addv(P[r * vs + i * is], scl(-1.0, mulr(c, P[q * vs + i * is])));
        __threadfence_block();
      }
    }
    double nn = 0.0;
    for (int i = lane; i < len; i += 64) nn += sq(P[r * vs + i * is]);
    return wsum(nn);
  };
  double nn = 0.0, best = 0.0;
  int tb = 0;
  for (int t = 0; t < len && nn <= 0.25; ++t) {
    nn = attempt(t);
    if (nn > best) {
      best = nn;
      tb = t;
    }
  }
  if (nn <= 0.25) nn = attempt(tb);
  const double inv = 1.0 / sqrt(nn);
  for (int i = lane; i < len; i += 64) P[r * vs + i * is] = scl(inv, P[r * vs + i * is]);
  __threadfence_block();
}

// A: problem b at A + b*sA, row-major with leading dimension lda.
// wide == 0: the matrix is A itself (m x n, m >= n).  wide == 1: the matrix
// is the conjugate transpose of A, A being n x m (so again m x n, m >= n).
// W: m x n column-major, V: n x n column-major.
// Outputs of the SVD of the ORIGINAL A (rows x cols, k = n):
//   wide == 0: u (m x k) = W_j / s_j,       vh (k x n) = V^H
//   wide == 1: u (n x k) = V,               vh (k x m) = (W_j / s_j)^H
// s (k) descending; the largest-modulus entry of each u column (first on
// ties) made real positive, the matching vh row scaled by the conjugate
// phase.  sweeps[b] receives the sweep count (-1 if not converged).
// LDS: bytes of shared memory; W_LDS: W fits there beside V (otherwise W is
// the global workspace Wk).  MI > 0: m <= 16 MI, and a lane keeps its elements
// of both columns in registers between the inner product and the rotation.  LP:
// lanes per column pair.
template <typename T, int NT, int LDS, bool W_LDS, int MI, int LP>
__global__ __launch_bounds__(NT) void jacobi_svd_kernel(const T* A, long long lda, long long sA, int m, int n,
                                                        int wide, T* Wk, long long sW, T* u, long long su, T* vh,
                                                        long long svh, double* s, long long ss, int* sweeps,
                                                        int max_sweeps) {
  __shared__ __align__(16) char smem[LDS];
  const int b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int sub = tid % LP, slot = tid / LP;   // lane of the pair, pair of the step
  static_assert(LP == 16 || (LP == 64 && MI == 0), "a DPP row or a wave per pair");
  const T* Ab = A + b * sA;
  T* V = reinterpret_cast<T*>(smem);
  T* W;
  if constexpr (W_LDS) W = reinterpret_cast<T*>(smem) + n * n;
  else W = Wk + b * sW;
  __shared__ int rotated, some_tiny;
  __shared__ double sig[JACOBI_MAX_K];   // squared column norms; at the end the singular values
  __shared__ int rank_of[JACOBI_MAX_K];
  using Idx = std::conditional_t<W_LDS, int, long long>;
  constexpr int UB = LP == 16 ? 2 : 4;   // elements of a column in flight per lane where they are not kept
  // load and V = I
  __shared__ double s_max[NT / 64];
  double am = 0.0;
  if (wide) {
    for (Idx e = tid; e < (Idx)m * n; e += NT) {
      const int j = (int)(e / m), i = (int)(e % m);
      const T v = cj(Ab[(long long)j * lda + i]);
      am = fmax(am, amax_of(v));
      W[e] = v;
    }
  } else {
    for (Idx e = tid; e < (Idx)m * n; e += NT) {   // consecutive threads along a row of A
      const int i = (int)(e / n), j = (int)(e % n);
      const T v = Ab[(long long)i * lda + j];
      am = fmax(am, amax_of(v));
      W[(Idx)j * m + i] = v;
    }
  }
  for (int e = tid; e < n * n; e += NT) V[e] = (e / n == e % n) ? one_of(T{}) : zero_of(T{});
  for (int off = 32; off > 0; off >>= 1) am = fmax(am, __shfl_xor(am, off, 64));
  if (lane == 0) s_max[wv] = am;
  if (tid == 0) some_tiny = 0;
  __syncthreads();
  // A matrix whose largest entry is beyond 2^+-100 is scaled by a power of two
  // (exact), so that squared inner products of its columns stay in range.
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) am = fmax(am, s_max[k]);
  const int ae = am > 0.0 && am < INFINITY ? __builtin_amdgcn_frexp_exp(am) : 0;
  const int ex = ae > 100 || ae < -100 ? ae : 0;
  if (ex != 0) {
    for (Idx e = tid; e < (Idx)m * n; e += NT) W[e] = ldexp_of(W[e], -ex);
    __syncthreads();
  }
  const int N = n + (n & 1);            // even player count (column n is a bye when n is odd)
  const double tol = (double)m * 0x1p-53;
  int sweep = 0;
  bool conv = (n < 2);
  // the steps of one sweep; TINY: with the scaled forms (a copy of the loop, as
  // the few instructions more would cost a step 3% of its time)
  auto steps = [&](auto tiny) __attribute__((always_inline)) {
    constexpr bool TINY = decltype(tiny)::value;
    // players of this slot: position 0 is fixed, the others advance by one per step
    int t1 = slot == 0 ? 0 : slot, t2 = N - 1 - slot;
    for (int r = 0; r < N - 1; ++r) {
      const int p = min(t1, t2), q = max(t1, t2);
      if (slot < N / 2 && q < n) {
        T* wp = W + (Idx)p * m;
        T* wq = W + (Idx)q * m;
        const double al = sig[p], be = sig[q];
        T ga = zero_of(T{});
        T x[MI > 0 ? MI : 1], y[MI > 0 ? MI : 1];
        if constexpr (MI > 0) {
#pragma unroll
          for (int k = 0; k < MI; ++k) {
            const int i = sub + 16 * k;
            x[k] = i < m ? wp[i] : zero_of(T{});
            y[k] = i < m ? wq[i] : zero_of(T{});
          }
#pragma unroll
          for (int k = 0; k < MI; ++k) ga = addv(ga, mulr(cj(x[k]), y[k]));
        } else {
          for (int i0 = sub; i0 < m; i0 += UB * LP) {
            T u0[UB], u1[UB];
#pragma unroll
            for (int k = 0; k < UB; ++k) {
              const int i = min(i0 + k * LP, m - 1);
              u0[k] = wp[i];
              u1[k] = wq[i];
            }
#pragma unroll
            for (int k = 0; k < UB; ++k)
              if (i0 + k * LP < m) ga = addv(ga, mulr(cj(u0[k]), u1[k]));
          }
        }
        ga = pair_sum<LP>(ga);
        // |g| > tol |w_p| |w_q|, squared where that cannot underflow (a column
        // that shrank below that within the sweep waits for the next one)
        bool rot = al > 0.0 && be > 0.0;
        double ag, ig;
        T phc;
        if constexpr (TINY) {
          modulus<true>(ga, ag, ig, phc);
          rot = rot && ag > tol * (al * rsqrt_nr(al)) * (be * rsqrt_nr(be));
        } else {
          rot = rot && sq(ga) > fmax((tol * al) * (tol * be), 0x1p-960);
        }
        if (rot) {
          if constexpr (!TINY) modulus<false>(ga, ag, ig, phc);
          // rotate [w_p, w_q e^{-i phi}] by the real Jacobi rotation of
          // [[al, |g|], [|g|, be]]
          double zeta = (be - al) * (0.5 * ig);
          if (TINY && ag < 0x1p-1000) zeta = (be - al) / (2.0 * ag);   // ig may be Inf
          const double az = fabs(zeta);
          double t;
          if (az < 0x1p500) {
            const double h2 = __builtin_fma(zeta, zeta, 1.0);
            t = rcp_nr(az + h2 * rsqrt_nr(h2));
          } else {
            t = 0.5 / az;
          }
          if (zeta < 0.0) t = -t;
          const double c = cos_of_tan(t), sn = c * t;
          if constexpr (MI > 0) {
#pragma unroll
            for (int k = 0; k < MI; ++k) {
              const int i = sub + 16 * k;
              const T z = mulr(y[k], phc);
              if (i < m) {
                wp[i] = addv(scl(c, x[k]), scl(-sn, z));
                wq[i] = addv(scl(sn, x[k]), scl(c, z));
              }
            }
          } else {
            for (int i0 = sub; i0 < m; i0 += UB * LP) {
              T u0[UB], u1[UB];
#pragma unroll
              for (int k = 0; k < UB; ++k) {
                const int i = min(i0 + k * LP, m - 1);
                u0[k] = wp[i];
                u1[k] = wq[i];
              }
#pragma unroll
              for (int k = 0; k < UB; ++k) {
                const int i = i0 + k * LP;
                const T z = mulr(u1[k], phc);
                if (i < m) {
                  wp[i] = addv(scl(c, u0[k]), scl(-sn, z));
                  wq[i] = addv(scl(sn, u0[k]), scl(c, z));
                }
              }
            }
          }
          T* vp = V + p * n;
          T* vq = V + q * n;
#pragma unroll 4
          for (int i = sub; i < n; i += LP) {
            const T u0 = vp[i], z = mulr(vq[i], phc);
            vp[i] = addv(scl(c, u0), scl(-sn, z));
            vq[i] = addv(scl(sn, u0), scl(c, z));
          }
          if (sub == 0) {
            rotated = 1;
            sig[p] = fmax(0.0, al - t * ag);
            sig[q] = fmax(0.0, be + t * ag);
          }
        }
      }
      if (t1 != 0) t1 = t1 == N - 1 ? 1 : t1 + 1;
      t2 = t2 == N - 1 ? 1 : t2 + 1;
      __syncthreads();
    }
  };
  for (; !conv && sweep < max_sweeps; ++sweep) {
    // squared norms afresh in every sweep; within it the rotations carry them
    // along (|w_p|^2 - t |g|, |w_q|^2 + t |g|).  Their rounding can only spoil an
    // angle or postpone a rotation: the sweep that ends the iteration rotated
    // nothing and used the fresh norms.
    if (tid == 0) rotated = 0;
    for (int j = slot; j < n; j += NT / LP) {
      double nn = 0.0;
#pragma unroll 4
      for (int i = sub; i < m; i += LP) nn += sq(W[(Idx)j * m + i]);
      nn = pair_sum<LP>(nn);
      if (sub == 0) {
        sig[j] = nn;
        if (nn > 0.0 && nn < 0x1p-400) some_tiny = 1;
      }
    }
    __syncthreads();
    // without such columns every |g|^2 to rotate is above 2^-960
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(some_tiny) == 0, 1)) steps(std::false_type{});
    else steps(std::true_type{});
    conv = (rotated == 0);
    __syncthreads();
  }
  if (tid == 0) sweeps[b] = conv ? sweep : -1;
  // singular values = column norms, ranks by descending value (stable)
  for (int j = wv; j < n; j += NT / 64) {
    double nn = 0.0;
    for (int i = lane; i < m; i += 64) nn += sq(W[(long long)j * m + i]);
    nn = wsum(nn);
    if (lane == 0) sig[j] = sqrt(nn);
  }
  __syncthreads();
  if (tid < n) {
    int rk = 0;
    const double sj = sig[tid];
    for (int i = 0; i < n; ++i) rk += (sig[i] > sj) || (sig[i] == sj && i < tid);
    rank_of[tid] = rk;
    s[b * ss + rk] = __builtin_amdgcn_ldexp(sj, ex);
  }
  __syncthreads();
  T* ub = u + b * su;
  T* vb = vh + b * svh;
  const int k = n;
  // the normalised columns W_j / s_j and the rotations V_j, at rank r
  if (!wide) {
    for (Idx e = tid; e < (Idx)m * n; e += NT) {
      const int j = (int)(e / m), i = (int)(e % m);
      const double sj = sig[j];
      ub[(long long)i * k + rank_of[j]] = sj > 0.0 ? scl(1.0 / sj, W[e]) : zero_of(T{});
    }
    for (int e = tid; e < n * n; e += NT) {
      const int j = e / n, i = e % n;
      vb[(long long)rank_of[j] * n + i] = cj(V[e]);
    }
  } else {
    for (int e = tid; e < n * n; e += NT) {
      const int j = e / n, i = e % n;
      ub[(long long)i * k + rank_of[j]] = V[e];
    }
    for (Idx e = tid; e < (Idx)m * n; e += NT) {
      const int j = (int)(e / m), i = (int)(e % m);
      const double sj = sig[j];
      vb[(long long)rank_of[j] * m + i] = sj > 0.0 ? cj(scl(1.0 / sj, W[e])) : zero_of(T{});
    }
  }
  __syncthreads();
  // orthonormal completion of the vectors of zero singular values (they
  // sort last); one wave, in rank order
  if (wv == 0) {
    for (int r = 0; r < k; ++r) {
      if (s[b * ss + r] > 0.0) continue;
      if (!wide) complete_vector(ub, 1, k, m, r);
      else complete_vector(vb, m, 1, m, r);
    }
  }
  __syncthreads();
  // gauge: largest-modulus entry of each u column real positive
  const int urows = wide ? n : m;
  const int vcols = wide ? m : n;
  for (int r = wv; r < k; r += NT / 64) {
    double best = -1.0;
    int bi = 0;
    for (int i = lane; i < urows; i += 64) {
      const double a = sq(ub[(long long)i * k + r]);
      if (a > best) { best = a; bi = i; }
    }
    for (int off = 32; off > 0; off >>= 1) {
      const double ob = __shfl_xor(best, off, 64);
      const int oi = __shfl_xor(bi, off, 64);
      if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    double mod;
    T ph;
    polar(ub[(long long)bi * k + r], mod, ph);
    const T phc = cj(ph);
    for (int i = lane; i < urows; i += 64) ub[(long long)i * k + r] = mulr(ub[(long long)i * k + r], phc);
    for (int i = lane; i < vcols; i += 64) vb[(long long)r * vcols + i] = mulr(vb[(long long)r * vcols + i], ph);
  }
}

}  // namespace

size_t jacobi_work_elems(int m, int n) { return (size_t)m * n; }

// LDS sizes: V and W of a 32 x 32 complex problem, several of which share a
// compute unit, and of a 64 x 64 one (the larger also takes V of any problem
// when W stays in global memory).
static constexpr int JACOBI_LDS_SMALL = 2 * 32 * 32 * 16, JACOBI_LDS = 9 * 64 * 64 * 4;

// Lanes per pair: 16, so that a step has all pairs of up to 64 columns in at most
// 512 threads; a wave for matrices of few columns and many rows, where 16 lanes
// would walk long columns with most of the workgroup idle: 2048 x 8 complex 0.51 ms
// (1.75 with 16 lanes), 20000 x 24 34 ms (131), 300 x 32 1.4 ms (1.7).  Up to about
// six rows per column 16 lanes are faster (128 x 32: 0.62 and 0.67 ms), and above 32
// columns they fill the workgroup.
template <typename T>
static void jacobi_launch(const T* A, long long lda, long long sA, int m, int n, int wide, T* W, T* u, long long su,
                          T* vh, long long svh, double* s, long long ss, int* sweeps, int batch, hipStream_t st) {
  const size_t need = sizeof(T) * ((size_t)m * n + (size_t)n * n);
  const bool w_lds = need <= (size_t)JACOBI_LDS;
  constexpr int V32 = 32 * 32 * (int)sizeof(T), V64 = 64 * 64 * (int)sizeof(T);
  const int max_sweeps = 80;
  const long long sW = (long long)m * n;
  auto go = [&](auto kernel, int nt) {
    hipLaunchKernelGGL(kernel, dim3(batch), dim3(nt), 0, st, A, lda, sA, m, n, wide, W, sW, u, su, vh, svh, s, ss,
                       sweeps, max_sweeps);
  };
  if (n <= 32 && m <= 32) {
    go(jacobi_svd_kernel<T, 256, JACOBI_LDS_SMALL, true, 2, 16>, 256);
  } else if (m <= 64) {
    if (n <= 32) go(jacobi_svd_kernel<T, 256, JACOBI_LDS, true, 4, 16>, 256);
    else go(jacobi_svd_kernel<T, 512, JACOBI_LDS, true, 4, 16>, 512);
  } else if (n <= 8) {
    if (w_lds) go(jacobi_svd_kernel<T, 256, JACOBI_LDS, true, 0, 64>, 256);
    else go(jacobi_svd_kernel<T, 256, V32, false, 0, 64>, 256);
  } else if (n <= 32 && m < 6 * n) {   // at most 192 x 32: W is in LDS
    go(jacobi_svd_kernel<T, 256, JACOBI_LDS, true, 0, 16>, 256);
  } else if (n <= 32) {
    if (w_lds) go(jacobi_svd_kernel<T, 1024, JACOBI_LDS, true, 0, 64>, 1024);
    else go(jacobi_svd_kernel<T, 1024, V32, false, 0, 64>, 1024);
  } else {
    if (w_lds) go(jacobi_svd_kernel<T, 512, JACOBI_LDS, true, 0, 16>, 512);
    else go(jacobi_svd_kernel<T, 512, V64, false, 0, 16>, 512);
  }
}

hipError_t jacobi_svd(int dtype, const void* A, long long lda, long long sA, int rows, int cols, void* work,
                      void* u, long long su, void* vh, long long svh, double* s, long long ss, int* sweeps,
                      int batch, hipStream_t st) {
  if (batch <= 0) return hipSuccess;
  const int wide = rows < cols;
  const int m = wide ? cols : rows, n = wide ? rows : cols;
  if (n > JACOBI_MAX_K || n < 1) return hipErrorInvalidValue;
  auto run = [&](auto tag) {
    using T = decltype(tag);
    jacobi_launch<T>((const T*)A, lda, sA, m, n, wide, (T*)work, (T*)u, su, (T*)vh, svh, s, ss, sweeps, batch, st);
  };
  if (dtype == C128) run(cd{});
  else if (dtype == F64) run(double{});
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace tci
