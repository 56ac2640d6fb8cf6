// Batched FP64 Hermitian eigensolver for the Gram matrix of the truncated SVD.
//
// The truncated SVD (paper, TCI-spec appendix, linear algebra: svd and
// trunc_svd) of theta (m x n) is taken from the Gram matrix G = theta theta^dagger:
// G = U diag(s^2) U^dagger.  Only the largest kmax eigenpairs are needed.
//
//   1. Householder reduction to real symmetric tridiagonal form,
//      G = Q T Q^dagger, blocked in panels of NB columns: per column one
//      Hermitian matrix-vector product with the trailing matrix (the only
//      O(n^2) step, memory bound) and one small fused kernel; per panel a
//      rank-2NB update of the trailing matrix on the matrix cores.
//      The last TRI_CHIP_N columns run in one workgroup per problem that
//      holds the trailing matrix on chip.
//   2. Multisection with Sturm counts for the top eigenvalues of T (1 to 64
//      lanes per eigenvalue).
//   3. Inverse iteration (tridiagonal LU with partial pivoting, two solves
//      from a fixed pseudo-random start) for their eigenvectors Z (one
//      thread per vector).
//   4. Back-transformation U = Q Z with the compact-WY form of each panel's
//      reflectors, on the matrix cores.
// Every kernel takes the whole batch of same-size problems at once.
#include "common.hpp"
#include "gemm.hpp"
#include "eig.hpp"
#include "vecops.hpp"
#include "prof.hpp"

namespace tci {

template <typename T> struct EigT;
template <> struct EigT<double> {
  static constexpr int dtype = F64;
  __host__ __device__ static double zero() { return 0.0; }
  __host__ __device__ static double one() { return 1.0; }
};
template <> struct EigT<cd> {
  static constexpr int dtype = C128;
  __host__ __device__ static cd zero() { return cd{0.0, 0.0}; }
  __host__ __device__ static cd one() { return cd{1.0, 0.0}; }
};

__device__ inline double cj(double a) { return a; }
__device__ inline cd cj(cd a) { return conjg(a); }
__device__ inline double re(double a) { return a; }
__device__ inline double re(cd a) { return a.x; }
__device__ inline double im(double) { return 0.0; }
__device__ inline double im(cd a) { return a.y; }
__device__ inline double nrm2(double a) { return a * a; }
__device__ inline double nrm2(cd a) { return a.x * a.x + a.y * a.y; }
__device__ inline double mulr(double a, double b) { return a * b; }
__device__ inline cd mulr(cd a, cd b) { return a * b; }
__device__ inline double scl(double s, double a) { return s * a; }
__device__ inline cd scl(double s, cd a) { return s * a; }
__device__ inline double add(double a, double b) { return a + b; }
__device__ inline cd add(cd a, cd b) { return a + b; }
__device__ inline double sub(double a, double b) { return a - b; }
__device__ inline cd sub(cd a, cd b) { return a - b; }
__device__ inline double shfl_xor_t(double v, int m) { return __shfl_xor(v, m); }
__device__ inline cd shfl_xor_t(cd v, int m) { return cd{__shfl_xor(v.x, m), __shfl_xor(v.y, m)}; }
__device__ inline double rl(double, double r) { return r; }   // a real number as the element type
__device__ inline cd rl(cd, double r) { return cd{r, 0.0}; }

// ---------------------------------------------------------------------------
// Per-column kernels of the blocked reduction (LAPACK latrd organisation,
// lower storage, panel of NB columns starting at j0; p = i - j0):
//
//  colA (row blocks of TT rows over [row0, n)):
//    finish w_ip (ip = i-1): with t1 = W^H v, t2 = V^H v and yv = v^H A22 v
//      (summed here from the chunk partials of the previous colC),  alpha = -|tau|^2/2 (yv - t1^H t2 - t2^H t1),
//      w(r) = tau (y(r) - V(r,:) t1 - W(r,:) t2) + alpha v(r),  y(r) = sum_t P[t][r];
//    update column i: a(r,i) -= V(r,:) conj(W(i,:)) + W(r,:) conj(V(i,:));
//    d_i = Re a(i,i); one partial of ||a(i+2:n,i)||^2 per workgroup.
//  colC (lower-triangle tiles TT x TT of the trailing matrix, CH tiles of a
//    block row per workgroup):
//    reflector of a(i+1:n,i): beta = -sign(Re a) ||.||, tau = (beta - a)/beta,
//    v = [1, x / (a - beta)];  the chunk of tiles (R, cA..cB) adds
//    sum_C A_RC v_C to P[cA][R rows], and each tile with C < R adds A_RC^H v_R
//    to P[R][C rows]; v^H A v, one partial per chunk, and with the diagonal tile
//    t1 = W^H v and t2 = V^H v over its rows, one partial per band.
// Every tile of the lower triangle is read once per column.  Partials are
// summed by the kernel that consumes them (colC sums colA's norm partials,
// colA the chunk partials of colC): the kernel boundary makes them visible,
// and no workgroup waits on a device-scope fence, which on this chip writes
// back the L2 of its XCD.
// ---------------------------------------------------------------------------
constexpr int TT = 64;
static_assert(TRIDIAG_BAND >= TT, "the reduction reads whole diagonal tiles");

template <typename T, int NB>
struct TriWs {
  // byte offsets inside one problem's workspace
  __host__ __device__ static size_t xv(int) { return 0; }
  __host__ __device__ static size_t P(int n) { return align(sizeof(T) * (size_t)n); }
  __host__ __device__ static size_t pa(int n) { return P(n) + align(sizeof(T) * (size_t)nbt(n) * n); }
  __host__ __device__ static size_t pc(int n) { return pa(n) + align(sizeof(double) * (size_t)nbt(n)); }
  __host__ __device__ static size_t pt(int n) { return pc(n) + align(sizeof(T) * (size_t)ntile(n)); }
  // [V_panel; W^T] and [W^T; V_panel], 2 NB rows of n each: operands of the
  // fused rank-2NB trailing update
  __host__ __device__ static size_t cat1(int n) { return pt(n) + align(sizeof(T) * (size_t)nbt(n) * 2 * NB); }
  __host__ __device__ static size_t cat2(int n) { return cat1(n) + align(sizeof(T) * (size_t)2 * NB * n); }
  __host__ __device__ static size_t bytes(int n) { return cat2(n) + align(sizeof(T) * (size_t)2 * NB * n); }
  __host__ __device__ static int nbt(int n) { return (n + TT - 1) / TT; }
  __host__ __device__ static int ntile(int n) { return nbt(n) * (nbt(n) + 1) / 2; }
  __host__ __device__ static size_t align(size_t x) { return (x + 255) & ~size_t(255); }
};

// Tiles per workgroup of the trailing matvec: band R (rows R*TT ...) is cut
// into chunks of up to ch consecutive tiles C, and one workgroup handles one
// chunk, so that the reflector set-up and the final reduction are paid once
// per chunk.  The row sums of a chunk starting at tile cA go to P[cA][rows];
// the column sums of an off-diagonal tile (R, C) go to P[R][columns of C].
__host__ __device__ inline int tri_chunks(int nact, int ch) {
  int k = 0;
  for (int t = 1; t <= nact; ++t) k += (t + ch - 1) / ch;
  return k;
}

// Chunk length of a launch over nact bands of each of batch problems: whole
// bands (32 tiles) when these already give the chip TRI_WG workgroups, else
// the longest power of two that does.  A workgroup streams a tile in about
// 1.9 us, so a launch takes as long as its longest chunk: four problems of
// order 2048 ran 61.7 us per column on average with whole bands (128
// workgroups) and 20.8 us so cut, sixteen 70.9 and 51.2 us (512 to 2048
// workgroups within 1% of each other, 4096 2% slower).
constexpr int TRI_CH_MAX = 32, TRI_WG = 1024;
static int tri_chunk_len(int nact, int batch) {
  int ch = TRI_CH_MAX;
  while (ch > 1 && (long long)tri_chunks(nact, ch) * batch < TRI_WG) ch >>= 1;
  return ch;
}

// Is P[t][r] written in the column step whose first active block is b0?
__device__ inline bool tri_slot_used(int t, int r, int b0, int ch) {
  const int Rr = r / TT;
  return t > Rr || ((t - b0) & (ch - 1)) == 0;
}

// Sum over the 16 lanes of a DPP row; every lane receives the total.
template <int CTRL>
__device__ inline double dpp_add(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
__device__ inline double row16_sum(double v) {
  v = dpp_add<0xB1>(v);     // quad_perm [1,0,3,2]
  v = dpp_add<0x4E>(v);     // quad_perm [2,3,0,1]
  v = dpp_add<0x141>(v);    // row_half_mirror
  return dpp_add<0x140>(v); // row_mirror
}
__device__ inline double row8_sum(double v) { return dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(v))); }   // over 8 lanes
__device__ inline cd row8_sum(cd v) { return cd{row8_sum(v.x), row8_sum(v.y)}; }
__device__ inline cd row16_sum(cd v) { return cd{row16_sum(v.x), row16_sum(v.y)}; }

// v + (v of the lane whose number differs in bit 4, or bit 5), by the lane
// swaps between rows: no LDS round trip as in __shfl_xor.
__device__ inline double xor16_add(double v) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ inline double xor32_add(double v) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// sum over the lanes of a wave that share lane % 16, and over the whole wave
__device__ inline double quarter_sum(double v) { return xor32_add(xor16_add(v)); }
__device__ inline cd quarter_sum(cd v) { return cd{quarter_sum(v.x), quarter_sum(v.y)}; }
// Sums of four values over the lanes that share lane % 16: lane l receives the
// sum of value l / 16.  A lane swap between two different values sums both at
// once, so the four need three swaps where separate sums need eight.
__device__ inline double swap16_sum(double a, double b) {   // rows 0, 2: a over two rows; 1, 3: b
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ inline double swap32_sum(double a, double b) {   // lanes 0..31: a over the two halves; 32..63: b
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ inline double quarter_sum4(const double (&v)[4]) {
  return swap32_sum(swap16_sum(v[0], v[1]), swap16_sum(v[2], v[3]));
}
__device__ inline cd quarter_sum4(const cd (&v)[4]) {
  return cd{swap32_sum(swap16_sum(v[0].x, v[1].x), swap16_sum(v[2].x, v[3].x)),
            swap32_sum(swap16_sum(v[0].y, v[1].y), swap16_sum(v[2].y, v[3].y))};
}
template <typename T> __device__ inline T wave64_sum(T v) { return quarter_sum(row16_sum(v)); }

// Reflector scalars from ||x(i+2:n)||^2 and alpha = x(i+1).
template <typename T>
__device__ inline void reflector(T alpha, double xn2, double& beta, T& tau, T& scal) {
  const double ar = re(alpha), ai = im(alpha);
  if (xn2 == 0.0 && ai == 0.0) {
    beta = ar;
    tau = EigT<T>::zero();
    scal = EigT<T>::zero();
    return;
  }
  const double nrm = sqrt(ar * ar + ai * ai + xn2);
  beta = ar >= 0.0 ? -nrm : nrm;
  if constexpr (sizeof(T) == sizeof(double)) {
    tau = (beta - ar) / beta;
    scal = 1.0 / (ar - beta);
  } else {
    tau = cd{(beta - ar) / beta, -ai / beta};
    const double xr = ar - beta, xi = ai, den = xr * xr + xi * xi;
    scal = cd{xr / den, -xi / den};
  }
}

// Reflector scalars as in reflector(), without the division and square-root
// sequences, which a column would wait for: refined hardware seeds.
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
template <typename T>
__device__ inline void reflector_nr(T alpha, double xn2, double& beta, T& tau, T& scal) {
  const double ar = re(alpha), ai = im(alpha), sum = ar * ar + ai * ai + xn2;
  if ((xn2 == 0.0 && ai == 0.0) || !(sum > 1e-280 && sum < 1e280)) {
    reflector(alpha, xn2, beta, tau, scal);
    return;
  }
  const double rs = rsqrt_nr(sum), sg = ar >= 0.0 ? -1.0 : 1.0, ib = sg * rs;
  beta = sum * ib;
  const double xr = ar - beta;
  if constexpr (sizeof(T) == sizeof(double)) {
    tau = -xr * ib;
    scal = rcp_nr(xr);
  } else {
    const double iden = rcp_nr(xr * xr + ai * ai);
    tau = cd{-xr * ib, -ai * ib};
    scal = cd{xr * iden, -ai * iden};
  }
}

// acc + a b, acc + conj(a) b, acc - a conj(b) with fused multiply-adds only
__device__ inline double mac(double c, double a, double b) { return __builtin_fma(a, b, c); }
__device__ inline double mac_cj(double c, double a, double b) { return __builtin_fma(a, b, c); }
__device__ inline double msub_cj(double c, double a, double b) { return __builtin_fma(-a, b, c); }
__device__ inline cd mac(cd c, cd a, cd b) {
  return cd{__builtin_fma(-a.y, b.y, __builtin_fma(a.x, b.x, c.x)), __builtin_fma(a.y, b.x, __builtin_fma(a.x, b.y, c.y))};
}
__device__ inline cd mac_cj(cd c, cd a, cd b) {
  return cd{__builtin_fma(a.y, b.y, __builtin_fma(a.x, b.x, c.x)), __builtin_fma(-a.y, b.x, __builtin_fma(a.x, b.y, c.y))};
}
__device__ inline cd msub_cj(cd c, cd a, cd b) {
  return cd{__builtin_fma(-a.y, b.y, __builtin_fma(-a.x, b.x, c.x)), __builtin_fma(-a.y, b.x, __builtin_fma(a.x, b.y, c.y))};
}

// Barrier for data exchanged through LDS only: __syncthreads would also wait
// for the column's stores to global memory, a memory round trip per barrier.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One workgroup per 64 rows: lane = row, the four waves share a row's sums (wave
// w takes every fourth slot of P and every fourth panel column).  A launch is
// one chain of latencies, so every global load is issued before the first
// wait, what all waves need of row icol and of the partials is reduced by each
// wave for itself, and two barriers remain before w and one in the column update.
template <typename T, int NB>
__global__ __launch_bounds__(256) void tri_colA_kernel(TriArgs a, int row0, int icol, int ifin, int j0, int ch) {
  constexpr int PU = NB / 4, SU = 8;   // panel columns and slots of P (the first 32) per wave
  static_assert(2 * NB == 64, "lane l: t1 (l < NB) or t2");
  __shared__ T s_part[4][64], s_col[4][64];
  __shared__ T s_t[4][64], s_row[4][64];
  __shared__ T s_q[4];
  const int b = blockIdx.y, n = a.n, tid = threadIdx.x, lane = tid & 63, part = tid >> 6;
  char* ws = reinterpret_cast<char*>(a.ws) + b * a.sws;
  T* xv = reinterpret_cast<T*>(ws + TriWs<T, NB>::xv(n));
  const T* P = reinterpret_cast<const T*>(ws + TriWs<T, NB>::P(n));
  double* pa = reinterpret_cast<double*>(ws + TriWs<T, NB>::pa(n));
  const T* pc = reinterpret_cast<const T*>(ws + TriWs<T, NB>::pc(n));
  const T* pt = reinterpret_cast<const T*>(ws + TriWs<T, NB>::pt(n));
  T* G = reinterpret_cast<T*>(a.G) + b * a.sG;
  const T* V = reinterpret_cast<const T*>(a.Vt) + b * a.sVt + (long)j0 * n;   // panel row q at V + q n
  T* W = reinterpret_cast<T*>(a.Wp) + b * a.sWp;                              // panel column q at W + q n
  const T zero = EigT<T>::zero();
  const int r = row0 + blockIdx.x * TT + lane, rc = min(r, n - 1);
  const bool rv = r < n;
  const int pp = ifin >= 0 ? ifin - j0 : 0;     // panel columns before the one finished here
  const int p = icol >= 0 ? icol - j0 : 0;      // panel columns of the column update

  // ---- loads, from clamped addresses: what lies outside the finished panel
  // columns or the used slots is replaced by zero where it is used
  T vq[PU], wq[PU];
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int q = min(part + 4 * u, max(pp - 1, 0));
    vq[u] = V[(long)q * n + rc];
    wq[u] = W[(long)q * n + rc];
  }
  const T gcol = G[(long)rc * a.ldg + max(icol, 0)];
  // row icol of V (lanes < NB) and of W (lanes >= NB): the finished columns
  const int lq = lane & (NB - 1);
  const T* vwsrc = lane < NB ? V : W;
  T vw = vwsrc[(long)min(lq, max(pp - 1, 0)) * n + max(icol, 0)];
  T wr = zero, wi = zero;                       // w of this row and of row icol
  T vfin = zero;
  if (ifin >= 0) {
    const int tb0 = (ifin + 1) / TT, nbt = TriWs<T, NB>::nbt(n), nband = nbt - tb0, nwg = tri_chunks(nband, ch);
    vfin = V[(long)pp * n + rc];
    const T tau = reinterpret_cast<const T*>(a.tau)[b * a.stau + ifin];
    T ps[SU], tv[SU], pi = zero, qv = zero;
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int t = tb0 + part + 4 * u, k = part + 4 * u;
      ps[u] = P[(long)min(t, nbt - 1) * n + rc];
      tv[u] = pt[(long)min(k, nband - 1) * (2 * NB) + lane];
    }
    if (icol >= 0)
      for (int t = tb0 + lane; t < nbt; t += 64)
        if (tri_slot_used(t, icol, tb0, ch)) pi = add(pi, P[(long)t * n + icol]);
    for (int w = tid; w < nwg; w += 256) qv = add(qv, pc[w]);
    // ---- t1, t2 from one partial per band, the quadratic form from one per chunk
    T tsum = zero, y = zero;
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int t = tb0 + part + 4 * u, k = part + 4 * u;
      if (k < nband) tsum = add(tsum, tv[u]);
      if (t < nbt && tri_slot_used(t, rc, tb0, ch)) y = add(y, ps[u]);
    }
    for (int k = part + 4 * SU; k < nband; k += 4) tsum = add(tsum, pt[(long)k * (2 * NB) + lane]);
    for (int t = tb0 + part + 4 * SU; t < nbt; t += 4)
      if (tri_slot_used(t, rc, tb0, ch)) y = add(y, P[(long)t * n + rc]);
    qv = wave64_sum(qv);
    s_part[part][lane] = tsum;
    if (lane == 0) s_q[part] = qv;
    lds_barrier();
    T t12 = add(add(s_part[0][lane], s_part[1][lane]), add(s_part[2][lane], s_part[3][lane]));
    if (lq >= pp) t12 = vw = zero;
    s_t[part][lane] = t12;                      // read back by this wave only
    const T yv = add(add(s_q[0], s_q[1]), add(s_q[2], s_q[3]));
    // yv - t1^H t2 - t2^H t1 (each product appears in both halves of the wave)
    const double cross = wave64_sum(re(mulr(cj(t12), shfl_xor_t(t12, NB))));
    const T alpha = scl(-0.5 * nrm2(tau), sub(yv, rl(T{}, cross)));
    // w of row icol: y(icol) - V(icol,:) t1 - W(icol,:) t2, v(icol) = 1
    if (icol >= 0) {
      const T yi = wave64_sum(sub(pi, mulr(vw, t12)));
      wi = add(mulr(tau, yi), alpha);
    }
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int q = part + 4 * u;
      if (q < pp) {
        y = sub(y, mulr(vq[u], s_t[part][q]));
        y = sub(y, mulr(wq[u], s_t[part][NB + q]));
      }
    }
    s_col[part][lane] = y;
    lds_barrier();
    y = add(add(s_col[0][lane], s_col[1][lane]), add(s_col[2][lane], s_col[3][lane]));
    wr = add(mulr(tau, y), mulr(alpha, vfin));
    if (part == 0 && rv) W[(long)pp * n + r] = wr;
  }
  if (icol < 0) return;

  // ---- column icol (= row0) minus its p panel terms
  s_row[part][lane] = vw;
  T acc = part == 0 ? gcol : zero;
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int q = part + 4 * u;
    if (q < pp) {
      acc = msub_cj(acc, vq[u], s_row[part][NB + q]);
      acc = msub_cj(acc, wq[u], s_row[part][q]);
    }
  }
  if (part == 0 && p > pp) {                    // the column finished above: V(icol) = 1
    acc = msub_cj(acc, vfin, wi);
    acc = sub(acc, wr);
  }
  s_part[part][lane] = acc;
  lds_barrier();
  if (part == 0) {
    acc = add(add(s_part[0][lane], s_part[1][lane]), add(s_part[2][lane], s_part[3][lane]));
    double xn2 = 0.0;
    if (rv) {
      G[(long)r * a.ldg + icol] = acc;
      if (r >= icol + 1) xv[r] = acc;
      if (r >= icol + 2) xn2 = nrm2(acc);
      if (r == icol) a.d[b * a.sde + icol] = re(acc);
    }
    // ||x||^2 partial of this block (summed by the next kernel)
    xn2 = wave64_sum(xn2);
    if (lane == 0) pa[blockIdx.x] = xn2;
  }
}

// Every wave forms the reflector scalars for itself, so that no barrier stands
// before the tiles.
template <typename T, int NB>
__global__ __launch_bounds__(256) void tri_colC_kernel(TriArgs a, int i, int j0, int ch) {
  __shared__ T s_vR[4][TT];
  __shared__ T s_q[4];
  __shared__ T s_colsum[2][4][TT];
  static_assert(2 * NB == TT, "t1/t2 mapping assumes 2 NB == TT");
  const int b = blockIdx.x, n = a.n, tid = threadIdx.x, lane = tid & 63, part = tid >> 6;
  const int wg = (int)gridDim.y - 1 - (int)blockIdx.y;   // chunk: largest bands first
  const int p = i - j0;
  char* ws = reinterpret_cast<char*>(a.ws) + b * a.sws;
  const T* xv = reinterpret_cast<const T*>(ws + TriWs<T, NB>::xv(n));
  T* P = reinterpret_cast<T*>(ws + TriWs<T, NB>::P(n));
  T* pc = reinterpret_cast<T*>(ws + TriWs<T, NB>::pc(n));
  T* pt = reinterpret_cast<T*>(ws + TriWs<T, NB>::pt(n));
  const double* pa = reinterpret_cast<const double*>(ws + TriWs<T, NB>::pa(n));
  const T* G = reinterpret_cast<const T*>(a.G) + b * a.sG;
  T* V = reinterpret_cast<T*>(a.Vt) + b * a.sVt;
  const T* W = reinterpret_cast<const T*>(a.Wp) + b * a.sWp;
  const T zero = EigT<T>::zero();
  // chunk -> (band R, first tile cA, last tile cB)
  const int b0 = (i + 1) / TT;
  int k = wg, R = b0;
  for (;;) {
    const int nch = (R - b0 + ch) / ch;
    if (k < nch) break;
    k -= nch;
    ++R;
  }
  const int cA = b0 + k * ch, cB = min(R, cA + ch - 1);
  const bool has_diag = (cB == R);
  T xc = xv[min(cA * TT + lane, n - 1)];
  const T xr = xv[min(R * TT + lane, n - 1)];
  const T x1 = xv[i + 1];
  double xn2 = 0.0;
  for (int q = lane; q < (n - i + TT - 1) / TT; q += 64) xn2 += pa[q];
  xn2 = wave64_sum(xn2);
  double beta;
  T tv, scal;
  reflector_nr(x1, xn2, beta, tv, scal);
  if (wg == 0 && tid == 0) {
    a.e[b * a.sde + i] = beta;
    reinterpret_cast<T*>(a.tau)[b * a.stau + i] = tv;
  }
  auto vval = [&](int c, T x) -> T {
    const T v = mulr(x, scal);
    return c <= i || c >= n ? zero : c == i + 1 ? EigT<T>::one() : v;
  };
  const T vR = vval(R * TT + lane, xr);
  s_vR[part][lane] = vR;                        // read back by this wave only
  // reflector i into Vt (the chunk holding the diagonal tile owns band R's
  // rows; chunk 0 zeroes the rows above the active blocks)
  if (has_diag && part == 0 && R * TT + lane < n) V[(long)i * n + R * TT + lane] = vR;
  if (wg == 0)
    for (int rr = tid; rr < b0 * TT; rr += 256) V[(long)i * n + rr] = zero;

  // row sums of the chunk: lane l of entry e = 2 h + m holds row
  // part + 4 (4 e + l / 16)
  T rs[4] = {zero, zero, zero, zero}, qd = zero, qo = zero;
#pragma unroll 1
  for (int C = cA; C <= cB; ++C) {
    const bool diag = (C == R);
    const int c = C * TT + lane;
    const bool cok = c > i && c < n;
    const T vc = vval(c, xc);
    if (C < cB) xc = xv[min(c + TT, n - 1)];
    T colacc = zero;
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
      T ps[8];
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const int rl = part + 4 * (kk + 8 * h), r = R * TT + rl;
        T g = zero;
        if (cok && r > i && r < n) g = G[(long)r * a.ldg + c];
        ps[kk] = mulr(g, vc);                              // row-sum term
        colacc = mac_cj(colacc, g, s_vR[part][rl]);        // column-sum term
      }
      T v[2];
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const T four[4] = {ps[4 * m], ps[4 * m + 1], ps[4 * m + 2], ps[4 * m + 3]};
        v[m] = row16_sum(quarter_sum4(four));
        const T w = s_vR[part][part + 4 * (8 * h + 4 * m + (lane >> 4))];
        if (diag) qd = mac_cj(qd, w, v[m]);
        else qo = mac_cj(qo, w, v[m]);
      }
      if (h == 0) { rs[0] = add(rs[0], v[0]); rs[1] = add(rs[1], v[1]); }
      else { rs[2] = add(rs[2], v[0]); rs[3] = add(rs[3], v[1]); }
    }
    if (!diag) {
      const int sb = (C - cA) & 1;
      s_colsum[sb][part][lane] = colacc;
      lds_barrier();
      if (part == 0 && c < n)
        P[(long)R * n + c] = add(add(s_colsum[sb][0][lane], s_colsum[sb][1][lane]),
                                 add(s_colsum[sb][2][lane], s_colsum[sb][3][lane]));
    } else {
      // t1 = W^H v and t2 = V^H v over the diagonal tile's rows: values
      // m = 16 part .. + 15, m < NB for W's column m, else V's row m - NB.
      // Rows <= i of W may never have been written, so they are selected away
      // and not left to v = 0
      const bool live = R * TT + lane > i && R * TT + lane < n;
#pragma unroll 1
      for (int m0 = 16 * part; m0 < 16 * part + 16; m0 += 8) {
        T tt[8];
        const int rr = min(R * TT + lane, n - 1);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const T* src = m0 < NB ? W : V + (long)j0 * n;
          tt[u] = src[(long)min((m0 + u) & (NB - 1), max(p - 1, 0)) * n + rr];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) tt[u] = ((m0 + u) & (NB - 1)) < p && live ? mulr(cj(tt[u]), vR) : zero;
#pragma unroll
        for (int u = 0; u < 8; u += 4) {
          const T four[4] = {tt[u], tt[u + 1], tt[u + 2], tt[u + 3]};
          const T v = row16_sum(quarter_sum4(four));
          if ((lane & 15) == 0) pt[(long)(R - b0) * (2 * NB) + m0 + u + (lane >> 4)] = v;
        }
      }
    }
  }
  // row sums of the chunk -> P[cA][rows]; quadratic-form pieces
  if ((lane & 15) == 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = R * TT + part + 4 * (4 * e + (lane >> 4));
      if (r < n) P[(long)cA * n + r] = rs[e];
    }
  }
  qd = quarter_sum(qd);   // the 16 lanes of a row hold the same sums
  qo = quarter_sum(qo);
  if (lane == 0) s_q[part] = add(add(qd, qo), cj(qo));
  lds_barrier();
  if (tid == 0) pc[wg] = add(add(s_q[0], s_q[1]), add(s_q[2], s_q[3]));
}

// Operands of the trailing update G -= V W^H + W V^H = [V W] [W V]^H over
// rows and columns >= t: cat1 = [V_panel; W^T], cat2 = [W^T; V_panel] (rows
// q < pe from V_panel = Vt rows j0 .., from W^T), columns >= t.
template <typename T, int NB>
__global__ __launch_bounds__(256) void tri_cat_kernel(TriArgs a, int j0, int pe, int t) {
  const int b = blockIdx.y, n = a.n;
  char* ws = reinterpret_cast<char*>(a.ws) + b * a.sws;
  T* c1 = reinterpret_cast<T*>(ws + TriWs<T, NB>::cat1(n));
  T* c2 = reinterpret_cast<T*>(ws + TriWs<T, NB>::cat2(n));
  const T* V = reinterpret_cast<const T*>(a.Vt) + b * a.sVt;
  const T* W = reinterpret_cast<const T*>(a.Wp) + b * a.sWp;
  const long long tot = (long long)pe * (n - t);
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < tot; e += (long long)gridDim.x * 256) {
    const int q = (int)(e / (n - t)), r = t + (int)(e % (n - t));
    const T v = V[(long)(j0 + q) * n + r];
    const T w = W[(long)q * n + r];
    c1[(long)q * n + r] = v;
    c1[(long)(pe + q) * n + r] = w;
    c2[(long)q * n + r] = w;
    c2[(long)(pe + q) * n + r] = v;
  }
}

// Largest order of a matrix that tri_chip_kernel (below) holds on chip.
template <typename T> constexpr int TRI_CHIP_N = sizeof(T) == 16 ? 192 : 320;
template <typename T> static void tri_chip(const TriArgs& a, int i0, int batch, hipStream_t s);

template <typename T, int NB>
static hipError_t tridiag_impl(const TriArgs& a, int batch, hipStream_t s) {
  const int n = a.n;
  const size_t es = sizeof(T);
  const int nbt = TriWs<T, NB>::nbt(n);
  for (int j0 = 0, pe; j0 < n; j0 += pe) {
    if (n - j0 <= TRI_CHIP_N<T>) {   // the rest fits on chip: one launch
      tri_chip<T>(a, j0, batch, s);
      break;
    }
    pe = min(NB, n - TRI_CHIP_N<T> - j0);   // the last panel leaves the largest order that fits
    for (int p = 0; p < pe; ++p) {
      const int i = j0 + p;
      const int rowsA = n - i;
      hipLaunchKernelGGL((tri_colA_kernel<T, NB>), dim3((rowsA + TT - 1) / TT, batch), dim3(256), 0, s, a, i, i,
                         p > 0 ? i - 1 : -1, j0, tri_chunk_len(nbt - i / TT, batch));
      const int nact = nbt - (i + 1) / TT, ch = tri_chunk_len(nact, batch);
      // algorithmic bytes: the lower triangle of the trailing matrix read once
      ProfScope ps(s, 0.5 * (double)(n - i - 1) * (n - i) * sizeof(T) * batch, "hemv");
      hipLaunchKernelGGL((tri_colC_kernel<T, NB>), dim3(batch, tri_chunks(nact, ch)), dim3(256), 0, s, a, i, j0, ch);
    }
    const int t = j0 + pe;
    // finish w of the panel's last column, then the trailing update
    hipLaunchKernelGGL((tri_colA_kernel<T, NB>), dim3((n - t + TT - 1) / TT, batch), dim3(256), 0, s, a, t, -1, t - 1,
                       j0, tri_chunk_len(nbt - t / TT, batch));
    const int m = n - t;
    const long long tot = (long long)pe * m;
    const unsigned gx = (unsigned)std::min<long long>(256, (tot + 255) / 256);
    hipLaunchKernelGGL((tri_cat_kernel<T, NB>), dim3(gx, batch), dim3(256), 0, s, a, j0, pe, t);
    // one rank-2pe update: G[t:, t:] -= cat1[:, t:]^T conj(cat2[:, t:])
    char* G = reinterpret_cast<char*>(a.G);
    char* ws = reinterpret_cast<char*>(a.ws);
    GemmArgs g = gemm_args(m, m, 2 * pe, OP_T, OP_R, ws + TriWs<T, NB>::cat1(n) + (size_t)t * es, n,
                           ws + TriWs<T, NB>::cat2(n) + (size_t)t * es, n, G + ((long)t * a.ldg + t) * es, a.ldg);
    g.sA = a.sws / (long long)es; g.sB = a.sws / (long long)es; g.sC = a.sG;
    g.alpha_re = -1.0; g.beta_re = 1.0; g.batch = batch;
    g.lower_band = TRIDIAG_BAND;
    hipError_t err = gemm(EigT<T>::dtype, PREC_FP64, g, s);
    if (err != hipSuccess) return err;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Unblocked reduction (LAPACK hetd2 order, lower storage) of a trailing matrix
// of order nt = n - i0 held on chip: rows and columns i0 .. n-1 of G, at most
// 32 NB of them, by one 512-thread workgroup per matrix, all columns in one
// launch; the blocked path pays two launches per column, which at these orders
// is latency.  Outputs as the blocked path: d, e, tau, reflector rows of Vt.  Thread (ty, tx) = (tid / 16, tid % 16)
// keeps the elements (32 I + ty, 16 J + tx) of the lower triangle, the slices
// J < JL (which are finished first) in LDS and the others in registers, so
// that a column touches no memory but its reflector row of Vt.  Per column:
//   the column goes to LDS; every wave forms the reflector from it;
//   y = A v: row sums over the 16 lanes of a row (DPP), column sums over the
//     4 rows of a wave, then over the 8 waves through LDS;
//   w = tau y - 1/2 tau (tau y)^H v v;  A -= v w^H + w v^H.
// Rows and columns <= i of the stored matrix are dead: v and w are zero there,
// and v is written to LDS once so that no use of it needs a select.
// Bound by LDS reads of the vectors and by the latency of a column (four
// barriers): 4.5 us per column at order 192 complex (0.87 ms per launch), 1.9 us
// at 100 real (0.19 ms).  The same reduction from global memory by one
// workgroup took 15 and 5.8 us per column (16 problems of order 200 complex
// 3.07 ms, one of order 100 real 0.58 ms).
// ---------------------------------------------------------------------------
template <typename T, int NB, int JL>
__global__ __launch_bounds__(512) void tri_chip_kernel(TriArgs a, int i0) {
  constexpr int NT = 512, NW = NT / 64, NC = 2 * NB, NN = 32 * NB, JC = 4;
  // row block I has the slices J < 2 I + 2, of which min(JL, 2 I + 2) are in LDS
  constexpr int SKIP0 = JL > 2 ? JL - 2 : 0, NREG = NB * (NB + 1) - JL * NB + SKIP0;
  static_assert(JL <= 4, "only row block 0 may have fewer than JL slices");
  __shared__ T s_l[JL > 0 ? JL * NB * NT : 1];
  __shared__ T s_x[NN], s_v[NN], s_w[NN], s_row[NN], s_part[NW][NN];
  __shared__ T s_dot[NW];
  const int b = blockIdx.x, n = a.n, nt = n - i0, tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4, lane = tid & 63, wid = tid >> 6;
  const long ldg = a.ldg;
  T* G = reinterpret_cast<T*>(a.G) + b * a.sG + (long)i0 * ldg + i0;
  T* V = reinterpret_cast<T*>(a.Vt) + b * a.sVt + (long)i0 * n;
  T* tau = reinterpret_cast<T*>(a.tau) + b * a.stau + i0;
  double* dd = a.d + b * a.sde + i0;
  double* ee = a.e + b * a.sde + i0;
  T areg[NREG];
  auto slot = [](int I, int J) constexpr { return I * (I + 1) - JL * I + SKIP0 + (J - JL); };
  auto get = [&](int I, int J) -> T { return J < JL ? s_l[(I * JL + J) * NT + tid] : areg[J < JL ? 0 : slot(I, J)]; };
  auto put = [&](int I, int J, T v) {
    if (J < JL) s_l[(I * JL + J) * NT + tid] = v;
    else areg[J < JL ? 0 : slot(I, J)] = v;
  };
#pragma unroll
  for (int J = 0; J < NC; ++J)
#pragma unroll
    for (int I = J / 2; I < NB; ++I) {
      const int r = 32 * I + ty, c = 16 * J + tx;
      put(I, J, (r < nt && c <= r) ? G[r * ldg + c] : EigT<T>::zero());
    }
#pragma unroll 1
  for (int i = 0; i + 1 < nt; ++i) {
#pragma unroll
    for (int J = 0; J < NC; ++J)
      if (J == i >> 4) {
        if (tx == (i & 15)) {
#pragma unroll
          for (int I = J / 2; I < NB; ++I) s_x[32 * I + ty] = get(I, J);
        }
      }
    lds_barrier();
    // ||x(i+2:)||^2 and the reflector, by every wave
    double xn2 = 0.0;
#pragma unroll
    for (int k = 0; k < NN / 64; ++k) {
      const int r = lane + 64 * k;
      const double t = nrm2(s_x[r]);
      xn2 += r >= i + 2 && r < nt ? t : 0.0;
    }
    xn2 = wave64_sum(xn2);
    double beta;
    T tv, scal;
    reflector_nr(s_x[i + 1], xn2, beta, tv, scal);
    if (tid == 0) {
      dd[i] = re(s_x[i]);
      ee[i] = beta;
      tau[i] = tv;
    }
    // v, zero outside i < c < nt, for plain reads of every use
    if (tid < NN) {
      T v = mulr(s_x[tid], scal);
      v = tid <= i || tid >= nt ? EigT<T>::zero() : tid == i + 1 ? EigT<T>::one() : v;
      s_v[tid] = v;
      if (tid < nt) V[(long)i * n + i0 + tid] = v;
    }
    for (int c = tid; c < i0; c += NT) V[(long)i * n + c] = EigT<T>::zero();
    lds_barrier();
    T vr[NB], acc[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) {
      vr[I] = s_v[32 * I + ty];
      acc[I] = EigT<T>::zero();
    }
    // slices in chunks of JC without a branch inside, so that the loads,
    // products and sums of a chunk overlap
#pragma unroll
    for (int J0 = 0; J0 < NC; J0 += JC) {
      if (16 * (J0 + JC) <= i + 1) continue;
      T vc[JC], col[JC];
#pragma unroll
      for (int k = 0; k < JC; ++k) {
        vc[k] = s_v[16 * (J0 + k) + tx];
        col[k] = EigT<T>::zero();
      }
#pragma unroll
      for (int I = J0 / 2; I < NB; ++I)
#pragma unroll
        for (int k = 0; k < JC; ++k) {
          const int J = J0 + k;
          if (J > 2 * I + 1) continue;
          const T g = get(I, J);
          acc[I] = mac(acc[I], g, vc[k]);
          // an element of the diagonal counts once
          const T gc = J >= 2 * I && 16 * J + tx == 32 * I + ty ? EigT<T>::zero() : g;
          col[k] = mac_cj(col[k], gc, vr[I]);
        }
      s_part[wid][16 * J0 + lane] = quarter_sum4(col);
    }
#pragma unroll
    for (int I = 0; I < NB; ++I) acc[I] = row16_sum(acc[I]);
#pragma unroll
    for (int I = 0; I < NB; ++I)
      if (tx == 0) s_row[32 * I + ty] = acc[I];
    lds_barrier();
    // w0 = tau y and w0^H v
    T pd = EigT<T>::zero();
    if (tid < NN) {
      T y = s_row[tid];
#pragma unroll
      for (int w = 0; w < NW; ++w) y = add(y, s_part[w][tid]);
      y = mulr(tv, y);
      y = tid > i && tid < nt ? y : EigT<T>::zero();
      s_w[tid] = y;
      pd = mulr(cj(y), s_v[tid]);
    }
    pd = wave64_sum(pd);
    if (lane == 0) s_dot[wid] = pd;
    lds_barrier();
    T al = s_dot[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) al = add(al, s_dot[w]);
    al = scl(-0.5, mulr(tv, al));
    T wr[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) wr[I] = mac(s_w[32 * I + ty], al, vr[I]);
#pragma unroll
    for (int J0 = 0; J0 < NC; J0 += JC) {
      if (16 * (J0 + JC) <= i + 1) continue;
      T vc[JC], wc[JC];
#pragma unroll
      for (int k = 0; k < JC; ++k) {
        vc[k] = s_v[16 * (J0 + k) + tx];
        wc[k] = mac(s_w[16 * (J0 + k) + tx], al, vc[k]);
      }
#pragma unroll
      for (int I = J0 / 2; I < NB; ++I)
#pragma unroll
        for (int k = 0; k < JC; ++k) {
          const int J = J0 + k;
          if (J > 2 * I + 1) continue;
          const T g = get(I, J);
          const T u = msub_cj(msub_cj(g, vr[I], wc[k]), wr[I], vc[k]);
          put(I, J, J >= 2 * I && 16 * J + tx > 32 * I + ty ? g : u);
        }
    }
  }
  // the last diagonal element, held by the thread of its place
  const int l = nt - 1;
#pragma unroll
  for (int J = 0; J < NC; ++J)
#pragma unroll
    for (int I = J / 2; I < NB; ++I)
      if (32 * I + ty == l && 16 * J + tx == l) {
        dd[l] = re(get(I, J));
        ee[l] = 0.0;
      }
}

// 6 row blocks of complex elements take 120 registers and 96 KiB of LDS per
// workgroup, 10 of real ones 162 and 120 KiB; one block more exceeds the
// register file beside the vectors.
template <typename T>
static void tri_chip(const TriArgs& a, int i0, int batch, hipStream_t s) {
  const int nt = a.n - i0;
  // work figure: the lower triangle of the trailing matrix, summed over the columns
  ProfScope ps(s, sizeof(T) * (double)nt * (nt - 1) * (nt + 1) / 6.0 * batch, "tri_chip");
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(batch), dim3(512), 0, s, a, i0); };
  if (nt <= 64) go(tri_chip_kernel<T, 2, 0>);
  else if (nt <= 128) go(tri_chip_kernel<T, 4, 0>);
  else if constexpr (sizeof(T) == 16) go(tri_chip_kernel<T, 6, 2>);
  else if (nt <= 192) go(tri_chip_kernel<T, 6, 0>);
  else if (nt <= 256) go(tri_chip_kernel<T, 8, 0>);
  else go(tri_chip_kernel<T, 10, 3>);
}

// One workgroup per diagonal tile.
template <typename T>
__global__ __launch_bounds__(256) void mirror_tiles_kernel(T* G, long long ldg, int n) {
  const int t0 = blockIdx.x * TT;
  for (int e = threadIdx.x; e < TT * TT; e += 256) {
    const int r = t0 + e / TT, c = t0 + e % TT;
    if (c > r && c < n) G[r * ldg + c] = cj(G[c * ldg + r]);
  }
}

hipError_t tridiag_mirror_tiles(int dtype, void* G, long long ldg, int n, hipStream_t s) {
  if (n <= (dtype == C128 ? TRI_CHIP_N<cd> : TRI_CHIP_N<double>)) return hipSuccess;   // read by its lower triangle
  const dim3 grid((n + TT - 1) / TT);
  if (dtype == C128) hipLaunchKernelGGL(mirror_tiles_kernel<cd>, grid, dim3(256), 0, s, (cd*)G, ldg, n);
  else if (dtype == F64) hipLaunchKernelGGL(mirror_tiles_kernel<double>, grid, dim3(256), 0, s, (double*)G, ldg, n);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

size_t tridiag_ws_bytes(int dtype, int n) {
  return dtype == C128 ? TriWs<cd, TRIDIAG_NB>::bytes(n) : TriWs<double, TRIDIAG_NB>::bytes(n);
}

hipError_t tridiagonalize(int dtype, const TriArgs& a, int batch, hipStream_t s) {
  if (dtype != C128 && dtype != F64) return hipErrorInvalidValue;
  if (a.n <= 0 || batch <= 0) return hipSuccess;
  if (a.n <= (dtype == C128 ? TRI_CHIP_N<cd> : TRI_CHIP_N<double>)) {
    if (dtype == C128) tri_chip<cd>(a, 0, batch, s);
    else tri_chip<double>(a, 0, batch, s);
    return hipGetLastError();
  }
  if (a.sws < (long long)tridiag_ws_bytes(dtype, a.n)) return hipErrorInvalidValue;
  // the partial sums start at zero; the trailing-update operands, and what is
  // used of the panel W, are written before they are read
  const size_t zb = dtype == C128 ? TriWs<cd, TRIDIAG_NB>::cat1(a.n) : TriWs<double, TRIDIAG_NB>::cat1(a.n);
  if (a.sws % 4 != 0) return hipErrorInvalidValue;
  hipError_t e = zero_fill_rows(a.ws, zb, (size_t)a.sws, batch, s);
  if (e != hipSuccess) return e;
  if (dtype == C128) return tridiag_impl<cd, TRIDIAG_NB>(a, batch, s);
  return tridiag_impl<double, TRIDIAG_NB>(a, batch, s);
}

// ---------------------------------------------------------------------------
// Bisection: lam[b][j] = j-th largest eigenvalue of the symmetric tridiagonal
// (d, e), j < kmax.  Sturm count: number of negative pivots q_i = d_i - x -
// e_{i-1}^2 / q_{i-1} of the LDL^T factorisation of T - x I = number of
// eigenvalues below x.
//
// With q_i = p_i / p_{i-1} the pivots' signs are the sign changes of
//   p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2},
// whose step is one fused multiply-add on the dependent chain instead of a
// division.  Its rounding errors are the division form's: each rounding of p_i
// enters the ratios q_i and q_{i+1} and amounts to relative changes of e^2 and
// of d - x by a few ulps.  T is scaled by a power of two to a norm in [1, 2),
// and p is rescaled after every block of STURM_BLK steps: a step grows |p| at
// most 8 times, and a pair (p_i, p_{i-1}) shrinks by about e^2 per two steps,
// so blocks whose e^2 are all above STURM_TINY cannot under- or overflow
// (an exact zero of one p_i counts its sign change one step later).  The other
// blocks (splits, padding) take the guarded division form; tridiag_scale_kernel
// marks them by the sign bit of their first e^2.
// ---------------------------------------------------------------------------
constexpr int STURM_BLK = 8;
constexpr double STURM_TINY = 1e-60;
constexpr double STURM_PIVMIN = 2.2250738585072014e-308 * 64.0;   // of the scaled matrix

__device__ inline int sign_of(double v) { return __double2hiint(v) >> 31; }   // 0 or -1

// Guarded division steps from q_{i-1} over m steps; returns q.
__device__ inline double sturm_steps_div(const double* __restrict__ d, const double* __restrict__ e2, int m, double sc,
                                         double x, double q, int& cnt) {
  for (int u = 0; u < m; ++u) {
    q = __builtin_fma(d[u], sc, -x) - fabs(e2[u]) / q;
    if (fabs(q) < STURM_PIVMIN) q = -STURM_PIVMIN;
    cnt += q < 0.0;
  }
  return q;
}

// e2: scaled squares with block marks; sc: the scale of d; x: a point of the scaled matrix.
__device__ inline int sturm_count(const double* __restrict__ d, const double* __restrict__ e2, int n, double sc,
                                  double x) {
  double p = __builtin_fma(d[0], sc, -x), pp = 1.0;
  if (fabs(p) < STURM_PIVMIN) p = -STURM_PIVMIN;
  int cnt = p < 0.0;
  auto ratio = [&]() -> double {   // q with the sign that was counted
    const double q = fmax(fabs(p / pp), STURM_PIVMIN);
    return sign_of(p) == sign_of(pp) ? q : -q;
  };
  int i = 1;
  double dd[STURM_BLK], ee[STURM_BLK];
  if (i + STURM_BLK <= n) {
#pragma unroll
    for (int u = 0; u < STURM_BLK; ++u) {
      dd[u] = d[i + u];
      ee[u] = e2[i - 1 + u];
    }
  }
  for (; i + STURM_BLK <= n; i += STURM_BLK) {
    // the next block's entries (the same for the whole wave) are loaded
    // while this one is evaluated
    double dn[STURM_BLK], en[STURM_BLK];
    const int nx = i + 2 * STURM_BLK <= n ? i + STURM_BLK : i;
#pragma unroll
    for (int u = 0; u < STURM_BLK; ++u) {
      dn[u] = d[nx + u];
      en[u] = e2[nx - 1 + u];
    }
    if (__builtin_amdgcn_readfirstlane(__double2hiint(ee[0])) < 0) {
      p = sturm_steps_div(d + i, e2 + i - 1, STURM_BLK, sc, x, ratio(), cnt);
      pp = 1.0;
    } else {
#pragma unroll
      for (int u = 0; u < STURM_BLK; ++u) {
        const double a = __builtin_fma(dd[u], sc, -x);
        const double pn = __builtin_fma(a, p, -(ee[u] * pp));
        pp = p;
        p = pn;
        cnt += (unsigned)(__double2hiint(p) ^ __double2hiint(pp)) >> 31;
      }
    }
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));
    p = __builtin_amdgcn_ldexp(p, ex);
    pp = __builtin_amdgcn_ldexp(pp, ex);
#pragma unroll
    for (int u = 0; u < STURM_BLK; ++u) {
      dd[u] = dn[u];
      ee[u] = en[u];
    }
  }
  if (i < n) sturm_steps_div(d + i, e2 + i - 1, n - i, sc, x, ratio(), cnt);
  return cnt;
}

// Per problem: Gershgorin bounds and the scale into bnd[3 b ..] (lo, hi of the
// scaled matrix, the scale), squares of the scaled e with block marks into e2.
__global__ __launch_bounds__(256) void tridiag_scale_kernel(const double* d, const double* e, double* e2,
                                                            long long sde, int n, double* bnd) {
  __shared__ double s_lo[4], s_hi[4];
  const int b = blockIdx.x, tid = threadIdx.x;
  const double* db = d + b * sde;
  const double* eb = e + b * sde;
  double lo = db[0], hi = db[0];
  for (int i = tid; i < n; i += 256) {
    const double r = (i > 0 ? fabs(eb[i - 1]) : 0.0) + (i < n - 1 ? fabs(eb[i]) : 0.0);
    lo = fmin(lo, db[i] - r);
    hi = fmax(hi, db[i] + r);
  }
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off));
    hi = fmax(hi, __shfl_xor(hi, off));
  }
  if ((tid & 63) == 0) { s_lo[tid >> 6] = lo; s_hi[tid >> 6] = hi; }
  __syncthreads();
  lo = fmin(fmin(s_lo[0], s_lo[1]), fmin(s_lo[2], s_lo[3]));
  hi = fmax(fmax(s_hi[0], s_hi[1]), fmax(s_hi[2], s_hi[3]));
  const double scale = fmax(fabs(lo), fabs(hi));
  // the scale stays a normal number at both ends of the exponent range
  const int ex = scale > 0.0 ? max(-1000, min(1000, 1 - __builtin_amdgcn_frexp_exp(scale))) : 0;
  const double sc = __builtin_amdgcn_ldexp(1.0, ex);
  if (tid == 0) {
    const double eps = 4.0 * 2.220446049250313e-16 * scale * sc + STURM_PIVMIN;
    bnd[3 * b] = lo * sc - eps;
    bnd[3 * b + 1] = hi * sc + eps;
    bnd[3 * b + 2] = sc;
  }
  for (int i0 = tid * STURM_BLK; i0 < n; i0 += 256 * STURM_BLK) {
    double v[STURM_BLK];
    bool tiny = false;
#pragma unroll
    for (int u = 0; u < STURM_BLK; ++u) {
      const double x = i0 + u < n - 1 ? eb[i0 + u] * sc : 0.0;
      v[u] = x * x;
      tiny = tiny || !(v[u] >= STURM_TINY);
    }
    if (tiny) v[0] = -v[0];
#pragma unroll
    for (int u = 0; u < STURM_BLK; ++u)
      if (i0 + u < n) e2[b * sde + i0 + u] = v[u];
  }
}

// Multisection, L lanes per wanted eigenvalue (64 / L per wave): the lanes of
// eigenvalue j evaluate the Sturm count at L interior points that cut its
// interval [lo, hi] (count(lo) <= t < count(hi), t the ascending index) into
// L + 1 parts, and all of them move to the part whose ends keep that invariant
// (the first point whose count exceeds t and the point before it), until the
// interval is at rounding level relative to the eigenvalue itself.  Small
// eigenvalues are resolved to that relative accuracy because inverse iteration
// with shifts only absolutely accurate leaves the vectors of closely spaced
// small eigenvalues far from orthogonal, which costs a second Cholesky-QR pass.
// The first counts, at +- BIS_ZERO of the scaled matrix, settle the sign and
// the exact zeros (padding); an interval whose ends differ more than 4 times is
// cut evenly in the exponent, so that a small eigenvalue takes about
// log2 log2(norm / |lambda|) rounds more than a large one, not log2.
constexpr double BIS_ZERO = 0x1p-900;

// piecewise linear logarithm to base 2 of a positive normal number, and its inverse
__device__ inline double plog2(double v) {
  return (double)(__builtin_amdgcn_frexp_exp(v) - 1) + (2.0 * __builtin_amdgcn_frexp_mant(v) - 1.0);
}
__device__ inline double pexp2(double g) {
  const double f = floor(g);
  return __builtin_amdgcn_ldexp(1.0 + (g - f), (int)f);
}

template <int L>
__global__ __launch_bounds__(64) void bisect_kernel(const double* __restrict__ d, const double* __restrict__ e2,
                                                    const double* __restrict__ bnd, long long sde, int n, int kmax,
                                                    double* __restrict__ lam, long long slam) {
  const int b = blockIdx.y;
  const int lane = threadIdx.x;
  const int sub = lane & (L - 1);
  const int j = blockIdx.x * (64 / L) + lane / L;
  const double* db = d + b * sde;
  const double* e2b = e2 + b * sde;
  double lo = bnd[3 * b], hi = bnd[3 * b + 1];
  const double sc = bnd[3 * b + 2];
  const int t = n - 1 - min(j, kmax - 1);  // ascending index of this lane group's eigenvalue
  const int q0 = lane & ~(L - 1);          // first lane of the group
  int cneg, cpos;
  if constexpr (L > 1) {
    const int c = sturm_count(db, e2b, n, sc, sub & 1 ? BIS_ZERO : -BIS_ZERO);
    cneg = __shfl(c, q0, 64);
    cpos = __shfl(c, q0 + 1, 64);
  } else {
    cneg = sturm_count(db, e2b, n, sc, -BIS_ZERO);
    cpos = sturm_count(db, e2b, n, sc, BIS_ZERO);
  }
  const bool neg = cneg > t;
  if (neg) hi = fmin(hi, -BIS_ZERO);
  else if (cpos <= t) lo = fmax(lo, BIS_ZERO);
  else lo = hi = 0.0;
  for (int it = 0; it < 128; ++it) {
    const bool done = hi - lo <= 2.220446049250313e-16 * fmax(fabs(lo), fabs(hi));
    if (__ballot(!done) == 0ull) break;
    const double near = neg ? -hi : lo, far = neg ? -lo : hi;   // the ends by magnitude
    const bool geo = !done && near > 0.0 && far > 4.0 * near;
    const double p0 = geo ? plog2(near) : 0.0, dp = geo ? plog2(far) - p0 : 0.0;
    auto point = [&](int k) -> double {
      if (!geo) return lo + (hi - lo) * (1.0 / (L + 1)) * k;
      const double v = pexp2(p0 + dp * (1.0 / (L + 1)) * (neg ? L + 1 - k : k));
      return neg ? -v : v;
    };
    const bool below = sturm_count(db, e2b, n, sc, point(sub + 1)) <= t;
    // the group's flags (bit s: count at point s <= t); c = leading points below
    unsigned long long above = ~(__ballot(below) >> q0);
    if constexpr (L < 64) above |= 1ull << L;
    const int c = above ? __builtin_ctzll(above) : 64;
    if (!done) {
      const double nlo = c > 0 ? point(c) : lo;
      const double nhi = c < L ? point(c + 1) : hi;
      if (nlo >= lo && nhi <= hi && nlo < nhi) {
        lo = nlo;
        hi = nhi;
      }
    }
  }
  if (sub == 0 && j < kmax) lam[b * slam + j] = 0.5 * (lo + hi) / sc;
}

size_t tridiag_e2_elems(int n, int batch) { return (size_t)(n + 3) * batch; }

hipError_t tridiag_eigvals_top(const double* d, const double* e, double* e2, long long sde, int n,
                               int kmax, double* lam, long long slam, int batch, hipStream_t s) {
  if (kmax <= 0 || batch <= 0 || n <= 0) return hipSuccess;
  double* bnd = e2 + (size_t)n * batch;
  if (sde != n) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tridiag_scale_kernel, dim3(batch), dim3(256), 0, s, d, e, e2, sde, n, bnd);
  auto go = [&](auto kernel, int L) {
    hipLaunchKernelGGL(kernel, dim3((kmax + 64 / L - 1) / (64 / L), batch), dim3(64), 0, s, d, (const double*)e2,
                       (const double*)bnd, sde, n, kmax, lam, slam);
  };
  // L lanes cut the rounds to 1 / log2(L + 1) of a bisection's at L times its
  // counts.  A wave alone on a SIMD takes about 100 cycles per step (it waits on
  // its scalar loads), four waves about 60 each: more lanes pay up to one or
  // two waves per SIMD (1024 SIMDs) and cost above (order 2048, 16 problems of
  // 1024 values: 2.06 ms with L = 4, 2.63 ms with L = 16; the division form with
  // L = 4 took 6.77 ms).
  const long long want = (long long)kmax * batch;
  if (want <= 1024) go(bisect_kernel<64>, 64);
  else if (want <= 8192) go(bisect_kernel<16>, 16);
  else if (want <= 32768) go(bisect_kernel<4>, 4);
  else go(bisect_kernel<1>, 1);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Inverse iteration.  Thread (b, j) with j < chi[b] factorises
// P (T - lam_j I) = L U (partial pivoting; U has two super-diagonals) and
// solves twice, starting from a fixed pseudo-random vector; the result is
// normalised to unit 2-norm.  Workspace arrays and Z share the layout
// [b][i][j] (row i of an n x ldz matrix) so that neighbouring threads touch
// neighbouring addresses.
// ---------------------------------------------------------------------------
__device__ inline double hash_uniform(unsigned b, unsigned j, unsigned i) {
  unsigned h = b * 0x9E3779B1u ^ (j * 0x85EBCA77u + 0x165667B1u) ^ (i * 0xC2B2AE3Du);
  h ^= h >> 15; h *= 0x2C1B3C6Du; h ^= h >> 12; h *= 0x297A2D39u; h ^= h >> 15;
  return ((double)h + 0.5) * (2.0 / 4294967296.0) - 1.0;
}

// The recurrences below are sequential in i, one lane per eigenvector; a launch
// has few waves (2 per problem at 100 vectors), so what bounds it is the chain
// of one step and the latency of its loads.  Each pass walks i in blocks of
// IV_BLK with the next block's loads issued before this block's arithmetic
// (the stores of a step could alias them, which keeps the compiler from moving
// them ahead by itself).  The first forward solve runs inside the elimination,
// the 2-norm is summed in the last backward one, a pivot's reciprocal comes
// from refined seeds and interchanges are selections.  16 complex problems of
// order 200, 100 vectors each: 202 us with divisions, branches, a pass of its
// own for each of these and loads at a block's start; 93 us now (300 of order
// 300: 308 and 140).
constexpr int IV_BLK = 16, IV_BK2 = 8;   // forward; backward, with twice the loads per step

// forward: b <- L^-1 P (pre * z[:, j]), in place
__device__ __forceinline__ void invit_forward(double* z, long ld, unsigned j, int n, const double* dl, double pre) {
  struct Blk { double z[IV_BLK], s[IV_BLK]; };
  double bi = z[j] * pre;
  auto load = [&](Blk& k, int i0) {
#pragma unroll
    for (int u = 0; u < IV_BLK; ++u) {
      const int i = min(i0 + u, n - 2);
      k.z[u] = (z + (long)(i + 1) * ld)[j];
      k.s[u] = (dl + (long)i * ld)[j];
    }
  };
  auto step = [&](const Blk& k, int u, int i) {
    const double bn = k.z[u] * pre, sv = k.s[u];
    const bool sw = fabs(sv) >= 4.0;
    const double m = sw ? sv - copysign(4.0, sv) : sv;
    (z + (long)i * ld)[j] = sw ? bn : bi;
    const double p = sw ? bn : bi, q = sw ? bi : bn;
    bi = q - m * p;
  };
  auto block = [&](const Blk& k, int i0) {
    if (i0 + IV_BLK <= n - 1) {
#pragma unroll
      for (int u = 0; u < IV_BLK; ++u) step(k, u, i0 + u);
    } else {
#pragma unroll
      for (int u = 0; u < IV_BLK; ++u)
        if (i0 + u < n - 1) step(k, u, i0 + u);
    }
  };
  if (n > 1) {
    Blk p, q;
    load(p, 0);
    for (int i0 = 0; i0 < n - 1; i0 += 2 * IV_BLK) {
      load(q, i0 + IV_BLK);
      block(p, i0);
      load(p, i0 + 2 * IV_BLK);
      block(q, i0 + IV_BLK);
    }
  }
  z[(long)(n - 1) * ld + j] = bi;
}

// backward: U x = b, in place; ru holds the reciprocals of U's diagonal.
// Returns max|x| and the sum of squares.
__device__ __forceinline__ double invit_backward(double* z, long ld, unsigned j, int n, const double* ru,
                                                 const double* du, const double* du2, double& sq) {
  struct Blk { double z[IV_BK2], c1[IV_BK2], c2[IV_BK2], r[IV_BK2]; };
  double x1 = 0.0, x2 = 0.0, amax = 0.0, nn = 0.0;
  auto load = [&](Blk& k, int i0) {
#pragma unroll
    for (int u = 0; u < IV_BK2; ++u) {
      const long o = (long)max(i0 - u, 0) * ld;
      k.z[u] = (z + o)[j];
      k.c1[u] = (du + o)[j];
      k.c2[u] = (du2 + o)[j];
      k.r[u] = (ru + o)[j];
    }
  };
  auto step = [&](const Blk& k, int u, int i) {
    const double x = ((k.z[u] - k.c2[u] * x2) - k.c1[u] * x1) * k.r[u];
    (z + (long)i * ld)[j] = x;
    x2 = x1;
    x1 = x;
    amax = fmax(amax, fabs(x));
    nn += x * x;
  };
  auto block = [&](const Blk& k, int i0) {
    if (i0 - IV_BK2 >= -1) {
#pragma unroll
      for (int u = 0; u < IV_BK2; ++u) step(k, u, i0 - u);
    } else {
#pragma unroll
      for (int u = 0; u < IV_BK2; ++u)
        if (i0 - u >= 0) step(k, u, i0 - u);
    }
  };
  Blk p, q;
  load(p, n - 1);
  for (int i0 = n - 1; i0 >= 0; i0 -= 2 * IV_BK2) {
    load(q, i0 - IV_BK2);
    block(p, i0);
    load(p, i0 - 2 * IV_BK2);
    block(q, i0 - IV_BK2);
  }
  sq = nn;
  return amax;
}

// A power of two near 1 / norm: in these units (the vectors do not depend on them)
// no reciprocal leaves the range.
__device__ inline double invit_unit(double tnorm) {
  int ex = 0;
  if (tnorm > 0.0 && tnorm < 1e308) (void)frexp(tnorm, &ex);
  return ldexp(1.0, -max(ex, -1000));
}
__device__ inline double invit_tiny(double tnorm, double un) { return fmax(tnorm * un, 0.5) * 2.220446049250313e-16; }

// P (un T - lamj I) = L U of column j, and its forward solve of the pseudo-random
// start vector in z[:, j].  un: a power of two near 1 / norm; tiny: the smallest pivot.
__device__ __forceinline__ void invit_factor(const double* __restrict__ db, const double* __restrict__ eb, int n,
                                             double lamj, double un, double tiny, int b, unsigned j, long ld, double* ru,
                                             double* du, double* du2, double* dl, double* z) {
  // Elimination keeps one "active" row (entries a_i, c_i in columns i, i+1)
  // and meets original row i+1 (e_i, d_{i+1} - lam, e_{i+1}).  U row i is
  // stored as (1 / pivot, du, du2); the multiplier goes to dl, offset by +-4
  // when the rows were interchanged (|multiplier| <= 1 in both cases).  bi is
  // the active row's right-hand side, from the pseudo-random start.
  double a_i = db[0] * un - lamj;  // current diagonal entry of the active row i
  double c_i = (n > 1) ? eb[0] * un : 0.0;  // super-diagonal of active row
  double bi = hash_uniform(b, j, 0);
  auto step = [&](int i, double sub, double dn, double c_n) {  // entries (i+1, i), (i+1, i+1), (i+1, i+2)
    const double a_n = dn - lamj;
    // interchange rows i and i+1, but for no pivot below the smallest: a block of
    // noise (what the reduction leaves of a null space) would otherwise be solved
    // to its own relative accuracy, each vector to the same direction
    const bool sw = (fabs(a_i) < fabs(sub)) & (fabs(sub) >= tiny);
    const double pa = fabs(a_i) < tiny ? (a_i >= 0 ? tiny : -tiny) : a_i;
    const double piv = sw ? sub : pa, num = sw ? a_i : sub;
    const double y0 = __builtin_amdgcn_rcp(piv);
    const double y1 = fma(y0, fma(-piv, y0, 1.0), y0);
    const double m0 = num * y1;
    const double m = fma(fma(-piv, m0, num), y1, m0);   // num / piv, the residual corrected once
    const long o = (long)i * ld;
    const double p = sw ? a_n : c_i, q = sw ? c_i : a_n;
    (ru + o)[j] = fma(y1, fma(-piv, y1, 1.0), y1);
    (du + o)[j] = p;
    (du2 + o)[j] = sw ? c_n : 0.0;
    (dl + o)[j] = sw ? m + copysign(4.0, m) : m;       // |stored| >= 4 marks an interchange
    a_i = q - m * p;
    c_i = sw ? -m * c_n : c_n;
    const double bn = hash_uniform(b, j, i + 1);
    const double bp = sw ? bn : bi, bq = sw ? bi : bn;
    (z + o)[j] = bp;
    bi = bq - m * bp;
  };
  int i0 = 0;
  for (; i0 + IV_BK2 < n - 1; i0 += IV_BK2) {
    double ev[IV_BK2 + 1], dv[IV_BK2];
#pragma unroll
    for (int u = 0; u <= IV_BK2; ++u) ev[u] = eb[i0 + u] * un;
#pragma unroll
    for (int u = 0; u < IV_BK2; ++u) dv[u] = db[i0 + 1 + u] * un;
#pragma unroll
    for (int u = 0; u < IV_BK2; ++u) step(i0 + u, ev[u], dv[u], ev[u + 1]);
  }
  for (; i0 < n - 1; ++i0) step(i0, eb[i0] * un, db[i0 + 1] * un, i0 + 1 < n - 1 ? eb[i0 + 1] * un : 0.0);
  {
    double piv = a_i;
    if (fabs(piv) < tiny) piv = (piv >= 0 ? tiny : -tiny);
    const long o = (long)(n - 1) * ld + j;
    ru[o] = 1.0 / piv;
    du[o] = 0.0;
    du2[o] = 0.0;
    z[o] = bi;
  }
}

// One solve with the stored factors of column j: z[:, j] <- (T - lam_j)^-1
// (pre * z[:, j]); returns the factor 1 / max|z| for the next right-hand side.
__device__ __forceinline__ double invit_solve(double* z, long ld, unsigned j, int n, const double* ru, const double* du,
                                     const double* du2, const double* dl, double pre) {
  double sq;
  invit_forward(z, ld, j, n, dl, pre);
  const double amax = invit_backward(z, ld, j, n, ru, du, du2, sq);
  return amax > 0.0 ? 1.0 / amax : 1.0;
}

__global__ __launch_bounds__(64) void invit_kernel(const double* __restrict__ d, const double* __restrict__ e,
                                                   long long sde, int n, const double* __restrict__ lam,
                                                   long long slam, const int* __restrict__ chi, int kmax, double* Z,
                                                   long long ldz, long long sZ, double* w_ru, double* w_du,
                                                   double* w_du2, double* w_dl, long long sw_, int batch) {
  const int b = blockIdx.y;
  const unsigned j = blockIdx.x * blockDim.x + threadIdx.x;
  const int cb = chi ? min(chi[b], kmax) : kmax;
  if ((int)(blockIdx.x * blockDim.x) >= cb) return;
  const double* db = d + b * sde;
  const double* eb = e + b * sde;
  double* ru = w_ru + b * sw_;
  double* du = w_du + b * sw_;
  double* du2 = w_du2 + b * sw_;
  double* dl = w_dl + b * sw_;
  double* z = Z + b * sZ;
  const long ld = ldz;
  double tnorm = 0.0;
  for (int i = threadIdx.x; i < n; i += 64)
    tnorm = fmax(tnorm, fabs(db[i]) + (i > 0 ? fabs(eb[i - 1]) : 0.0) + (i < n - 1 ? fabs(eb[i]) : 0.0));
  for (int off = 32; off > 0; off >>= 1) tnorm = fmax(tnorm, __shfl_xor(tnorm, off, 64));
  if ((int)j >= cb) return;
  const double un = invit_unit(tnorm);
  // An eigenvalue that equals the one before it to rounding gets a shift a few
  // ulps below: with both shifts the same, and exact, one direction of a
  // multiple eigenvalue can outgrow the others by 1 / u in a solve, and what the
  // orthonormalisation leaves of the next vector is noise (as in LAPACK's stein).
  double lamj = lam[b * slam + j];
  if (j > 0) lamj = fmin(lamj, lam[b * slam + j - 1] - 4.0 * 2.220446049250313e-16 * fabs(lamj));
  lamj *= un;
  const double tiny = invit_tiny(tnorm, un);

  invit_factor(db, eb, n, lamj, un, tiny, b, j, ld, ru, du, du2, dl, z);
  double nn;
  double amax = invit_backward(z, ld, j, n, ru, du, du2, nn);
  invit_forward(z, ld, j, n, dl, amax > 0.0 ? 1.0 / amax : 1.0);
  amax = invit_backward(z, ld, j, n, ru, du, du2, nn);
  // normalise to unit 2-norm; squares that could leave the range are summed
  // again after scaling by the largest entry
  double inv;
  if (amax > 1e-130 && amax < 1e130) {
    inv = 1.0 / sqrt(nn);
  } else {
    const double scale = amax > 0.0 ? 1.0 / amax : 1.0;
    nn = 0.0;
    for (int i = 0; i < n; ++i) {
      const double x = z[(long)i * ld + j] * scale;
      nn += x * x;
    }
    inv = scale / sqrt(nn);
  }
  for (int i0 = 0; i0 < n; i0 += 2 * IV_BLK) {
    double zb[2 * IV_BLK];
#pragma unroll
    for (int u = 0; u < 2 * IV_BLK; ++u) zb[u] = z[(long)min(i0 + u, n - 1) * ld + j];
#pragma unroll
    for (int u = 0; u < 2 * IV_BLK; ++u)
      if (i0 + u < n) z[(long)(i0 + u) * ld + j] = zb[u] * inv;
  }
}

// Tight clusters (consecutive eigenvalues closer than INVIT_CLUSTER_TOL of
// the matrix norm; exact multiplicities among them) make independent inverse
// iterations converge to nearly the same vector.  One wave per problem walks
// its clusters; the members of a cluster (64 at a time, one per lane) are
// iterated together with their own factors, and after every solve they are
// orthonormalised in order against the earlier members (modified
// Gram-Schmidt), as in LAPACK's stein.
// With shifts exact to the last bit of the eigenvalues themselves, one direction
// of a cluster can outgrow the others by 1 / u and more in a solve (u^2 beside 1 in
// a null space), and what the orthonormalisation leaves of a vector is noise.  Where
// it leaves less than 1e-2 of one in the last pass, the members are solved again
// with shifts 4 u ||T|| below: (T - shift)^-1 then stretches all directions of the
// cluster about alike, and any of them are eigenvectors to that accuracy.
// The threshold sits at about 90 u ||T||: for a larger gap g the vectors of
// independent solves overlap by at most about u ||T|| / g < 1/90, which the
// Cholesky-QR2 that follows on all vectors removes.  (Graded spectra, as the
// Gram matrices of power-law bonds, have consecutive gaps between 1e-14 and
// 1e-11 of the norm over hundreds of eigenvalues; treating those as one
// cluster made its serial orthonormalisation dominate the whole update.)
constexpr double INVIT_CLUSTER_TOL = 1e-14;

__device__ inline double wave_sum_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__global__ __launch_bounds__(64) void invit_cluster_kernel(const double* d, const double* e, long long sde, int n,
                                                           const double* lam, long long slam, const int* chi,
                                                           int kmax, double* Z, long long ldz, long long sZ,
                                                           double* w_ru, double* w_du, double* w_du2, double* w_dl,
                                                           long long sw) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const int cb = chi ? min(chi[b], kmax) : kmax;
  const double* db = d + b * sde;
  const double* eb = e + b * sde;
  const double* lb = lam + b * slam;
  double* z = Z + b * sZ;
  const long ld = ldz;
  double tn = 0.0;
  for (int i = lane; i < n; i += 64)
    tn = fmax(tn, fabs(db[i]) + (i > 0 ? fabs(eb[i - 1]) : 0.0) + (i < n - 1 ? fabs(eb[i]) : 0.0));
  for (int off = 32; off > 0; off >>= 1) tn = fmax(tn, __shfl_xor(tn, off, 64));
  const double tol = INVIT_CLUSTER_TOL * tn, un = invit_unit(tn);
  int j0 = 0;
  while (j0 < cb) {
    int j1 = j0;
    while (j1 + 1 < cb && lb[j1] - lb[j1 + 1] <= tol) ++j1;
    if (j1 > j0) {
      for (int c0 = j0; c0 <= j1; c0 += 64) {
        const int cn = min(64, j1 - c0 + 1);
        const int m = c0 + lane;
        for (int attempt = 0; attempt < 2; ++attempt) {
          double scale = 1.0, least = 1.0;
          if (attempt == 1 && lane < cn) {
            const double lamm = lb[m] - 4.0 * 2.220446049250313e-16 * tn;
            invit_factor(db, eb, n, lamm * un, un, invit_tiny(tn, un), b, m, ld, w_ru + b * sw, w_du + b * sw,
                         w_du2 + b * sw, w_dl + b * sw, z);
            double sq;
            const double amax = invit_backward(z, ld, m, n, w_ru + b * sw, w_du + b * sw, w_du2 + b * sw, sq);
            scale = amax > 0.0 ? 1.0 / amax : 1.0;
          }
          for (int it = 0; it < 3; ++it) {
            if (lane < cn)
              scale = invit_solve(z, ld, m, n, w_ru + b * sw, w_du + b * sw, w_du2 + b * sw, w_dl + b * sw, scale);
            __syncthreads();
            // members c0 .. c0+cn-1 in order: apply the pending scale, remove the
            // earlier members of the cluster, normalise
            least = 1.0;
            for (int q = c0; q < c0 + cn; ++q) {
              const double sq = __shfl(scale, q - c0, 64);
              for (int i = lane; i < n; i += 64) z[(long)i * ld + q] *= sq;
              double gone = 0.0;
              for (int r = j0; r < q; ++r) {
                double dot = 0.0;
                for (int i = lane; i < n; i += 64) dot += z[(long)i * ld + r] * z[(long)i * ld + q];
                dot = wave_sum_d(dot);
                gone += dot * dot;
                for (int i = lane; i < n; i += 64) z[(long)i * ld + q] -= dot * z[(long)i * ld + r];
              }
              double nn = 0.0;
              for (int i = lane; i < n; i += 64) nn += z[(long)i * ld + q] * z[(long)i * ld + q];
              nn = wave_sum_d(nn);
              least = fmin(least, nn / (nn + gone));
              const double inv = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
              for (int i = lane; i < n; i += 64) z[(long)i * ld + q] *= inv;
            }
            scale = 1.0;
            __syncthreads();
          }
          if (least > 1e-4) break;
        }
      }
    }
    j0 = j1 + 1;
  }
}

hipError_t tridiag_invit(const double* d, const double* e, long long sde, int n, const double* lam,
                         long long slam, const int* chi, int kmax, double* Z, long long ldz, long long sZ,
                         double* work, int batch, hipStream_t s) {
  if (kmax <= 0 || batch <= 0) return hipSuccess;
  const long long sw = (long long)n * ldz;  // each workspace array: n x ldz per problem
  double* ru = work;
  double* du = work + sw * batch;
  double* du2 = work + 2 * sw * batch;
  double* dl = work + 3 * sw * batch;
  hipLaunchKernelGGL(invit_kernel, dim3((kmax + 63) / 64, batch), dim3(64), 0, s, d, e, sde, n, lam,
                     slam, chi, kmax, Z, ldz, sZ, ru, du, du2, dl, sw, batch);
  hipLaunchKernelGGL(invit_cluster_kernel, dim3(batch), dim3(64), 0, s, d, e, sde, n, lam, slam, chi, kmax, Z, ldz,
                     sZ, ru, du, du2, dl, sw);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Back-transformation U <- Q U with Q = H_0 H_1 ... H_{n-2}, applied in groups
// of BT_GB consecutive reflectors (several reduction panels), so that the
// products with the reflector block have 128 rows / inner dimension.
// Compact-WY factor of a group (LAPACK larft, forward, columnwise):
// H_{j0} ... H_{j0+g-1} = I - V T V^H, T upper triangular g x g with
// T(i,i) = tau_i and T(0:i, i) = -tau_i T(0:i, 0:i) S(0:i, i),
// S = V^H V from a GEMM.  T is built column by column in LDS, packed by
// columns (column i holds rows 0..i at offset i(i+1)/2).
// ---------------------------------------------------------------------------
constexpr int BT_GB = 128;

// One workgroup per (problem, group): block (b, grp) reads S of the group at
// Sg + b * sF + grp * BT_GB^2 and writes T at Tg + b * sF + grp * BT_GB^2.
// Eight threads per row share the sum of a column's entry, and S arrives eight
// columns at a time, the next eight in flight: a chain of 128 short columns,
// bound by their latency and by reading T from LDS (5.6 MB complex).  With one
// thread per row that loaded its S entry per column a complex group took
// 651 us; now 107 us (real: 269 to 55 us at 99 reflectors).
template <typename T>
__global__ __launch_bounds__(8 * BT_GB) void larft_group_kernel(TriArgs a, const void* Sg, void* Tg, long long sF) {
  constexpr int SB = 8;
  __shared__ T Tp[BT_GB * (BT_GB + 1) / 2];
  __shared__ T scol[SB][BT_GB];
  __shared__ T s_tau[BT_GB];
  const int b = blockIdx.x, grp = blockIdx.y, tid = threadIdx.x, q = tid >> 3, part = tid & 7;
  const int j0 = grp * BT_GB, g = min(BT_GB, a.n - 1 - j0);
  const long long off = b * sF + (long long)grp * BT_GB * BT_GB;
  const T* S = reinterpret_cast<const T*>(Sg) + off;   // g x g, ld BT_GB
  const T* tau = reinterpret_cast<const T*>(a.tau) + b * a.stau;
  T* Tout = reinterpret_cast<T*>(Tg) + off;             // BT_GB x BT_GB, ld BT_GB
  if (tid < g) s_tau[tid] = tau[j0 + tid];
  auto load = [&](int i) -> T { return q < g && i + part < g ? S[q * BT_GB + i + part] : EigT<T>::zero(); };
  T next = load(0);
  for (int i0 = 0; i0 < g; i0 += SB) {
    lds_barrier();
    scol[part][q] = next;
    lds_barrier();
    next = load(i0 + SB);
    for (int i = i0; i < min(g, i0 + SB); ++i) {
      const T ti = s_tau[i];
      T* coli = Tp + i * (i + 1) / 2;
      if (q < i) {
        T acc = EigT<T>::zero();
        for (int r = q + part; r < i; r += 8) acc = mac(acc, Tp[r * (r + 1) / 2 + q], scol[i - i0][r]);
        acc = row8_sum(acc);
        if (part == 0) coli[q] = mulr(scl(-1.0, ti), acc);
      } else if (q == i && part == 0) {
        coli[i] = ti;
      }
      lds_barrier();
    }
  }
  for (int e = tid; e < BT_GB * BT_GB; e += 8 * BT_GB) {
    const int r = e / BT_GB, c = e % BT_GB;
    Tout[e] = (r < g && c < g && r <= c) ? Tp[c * (c + 1) / 2 + r] : EigT<T>::zero();
  }
}

static int bt_groups(int n) { return (n - 1 + BT_GB - 1) / BT_GB; }

template <typename T>
static hipError_t backtransform_impl(const TriArgs& a, void* Tf, long long sTf, void* U, long long ldu,
                                     long long sU, int kmax, void* work, int batch, hipStream_t s) {
  const int n = a.n;
  const int ng = bt_groups(n);
  if (ng <= 0 || kmax <= 0) return hipSuccess;
  const size_t es = sizeof(T);
  const int dt = EigT<T>::dtype;
  char* V = reinterpret_cast<char*>(a.Vt);
  char* Uc = reinterpret_cast<char*>(U);
  char* Tc = reinterpret_cast<char*>(Tf);
  char* Sc = Tc + (size_t)ng * BT_GB * BT_GB * es;   // per-problem S of every group after the T factors
  char* W1 = reinterpret_cast<char*>(work);
  char* W2 = W1 + (size_t)batch * BT_GB * kmax * es;
  char* kws = W2 + (size_t)batch * BT_GB * kmax * es;   // split-K scratch
  const long long sW = (long long)BT_GB * kmax;
  hipError_t err = hipSuccess;
  // S = V_g^H V_g of every group (over rows j0+1 .. n-1; V_g = columns of Vt
  // rows j0 ..), then the T factors of all groups in one launch
  for (int grp = 0; grp < ng; ++grp) {
    const int j0 = grp * BT_GB, g = min(BT_GB, n - 1 - j0), rows = n - j0 - 1;
    GemmArgs gs = gemm_args(g, g, rows, OP_R, OP_T, V + ((long)j0 * n + j0 + 1) * es, n,
                            V + ((long)j0 * n + j0 + 1) * es, n, Sc + (size_t)grp * BT_GB * BT_GB * es, BT_GB);
    gs.sA = a.sVt; gs.sB = a.sVt; gs.sC = sTf; gs.batch = batch;
    gs.kws = kws; gs.kws_bytes = GEMM_SPLITK_WS_BYTES;
    err = gemm(dt, PREC_FP64, gs, s);
    if (err != hipSuccess) return err;
  }
  hipLaunchKernelGGL(larft_group_kernel<T>, dim3(batch, ng), dim3(8 * BT_GB), 0, s, a, (const void*)Sc, (void*)Tc, sTf);
  // groups applied last to first: U <- U - V_g (T_g (V_g^H U))
  for (int grp = ng - 1; grp >= 0; --grp) {
    const int j0 = grp * BT_GB, g = min(BT_GB, n - 1 - j0), rows = n - j0 - 1;
    GemmArgs g1 = gemm_args(g, kmax, rows, OP_R, OP_N, V + ((long)j0 * n + j0 + 1) * es, n,
                            Uc + (long)(j0 + 1) * ldu * es, ldu, W1, kmax);
    g1.sA = a.sVt; g1.sB = sU; g1.sC = sW; g1.batch = batch;
    g1.kws = kws; g1.kws_bytes = GEMM_SPLITK_WS_BYTES;
    err = gemm(dt, PREC_FP64, g1, s);
    if (err != hipSuccess) return err;
    GemmArgs g2 = gemm_args(g, kmax, g, OP_N, OP_N, Tc + (size_t)grp * BT_GB * BT_GB * es, BT_GB, W1, kmax, W2,
                            kmax);
    g2.sA = sTf; g2.sB = sW; g2.sC = sW; g2.batch = batch;
    err = gemm(dt, PREC_FP64, g2, s);
    if (err != hipSuccess) return err;
    GemmArgs g3 = gemm_args(rows, kmax, g, OP_T, OP_N, V + ((long)j0 * n + j0 + 1) * es, n, W2, kmax,
                            Uc + (long)(j0 + 1) * ldu * es, ldu);
    g3.sA = a.sVt; g3.sB = sW; g3.sC = sU;
    g3.alpha_re = -1.0; g3.beta_re = 1.0; g3.batch = batch;
    err = gemm(dt, PREC_FP64, g3, s);
    if (err != hipSuccess) return err;
  }
  return hipGetLastError();
}

size_t tridiag_backtransform_tf_elems(int n) { return (size_t)2 * std::max(1, bt_groups(n)) * BT_GB * BT_GB; }
size_t tridiag_backtransform_work_bytes(int dtype, int kmax, int batch) {
  const size_t es = dtype == C128 ? sizeof(cd) : sizeof(double);
  return es * 2 * BT_GB * (size_t)kmax * batch + GEMM_SPLITK_WS_BYTES;
}

hipError_t tridiag_backtransform(int dtype, const TriArgs& a, void* Tf, long long sTf, void* U,
                                 long long ldu, long long sU, int kmax, void* work, int batch,
                                 hipStream_t s) {
  if (batch > 1 && sTf < (long long)tridiag_backtransform_tf_elems(a.n)) return hipErrorInvalidValue;
  if (dtype == C128) return backtransform_impl<cd>(a, Tf, sTf, U, ldu, sU, kmax, work, batch, s);
  if (dtype == F64) return backtransform_impl<double>(a, Tf, sTf, U, ldu, sU, kmax, work, batch, s);
  return hipErrorInvalidValue;
}

}  // namespace tci
