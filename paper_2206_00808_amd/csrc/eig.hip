// Eigenvectors of the largest eigenvalues of a Hermitian matrix, and all eigenvalues.
//
//   1. k_tri_step, one launch per column: Householder reduction to a tridiagonal
//      matrix.  The reflectors H_j = I - 2 v_j v_j^H (unit v_j) stay as rows of V.
//   2. The tridiagonal matrix, made real by a diagonal of phases, is divided at
//      leaves of at most 16 rows (k_dc_leaf, implicit QR) and conquered level by
//      level by rank-one updates (Cuppen 1981): deflation (k_dc_deflate), the secular
//      equation by rational interpolation (k_dc_secular; Bunch, Nielsen and Sorensen
//      1978), the vectors from the recomputed update vector, which makes them
//      orthogonal to working precision whatever the gaps (k_dc_zhat, k_dc_vec; Gu and
//      Eisenstat 1994), and one product on the FP64 matrix cores (k_dc_gemm).
//   3. The reflectors are applied to the wanted vectors in blocks of 32 (k_bt_*).
//
// A tenth of the eigenvectors of a 1000-row matrix take 6.9 ms, all of them 7.3; two-sided
// Jacobi rounds on 32 x 32 blocks took 50 ms (13 sweeps of 63 rounds of two kernels).
//
// Everything is in FP64.  The matrix is first scaled by a power of two to entries below
// one, so squares neither overflow nor lose what matters to underflow.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"

namespace gw {

typedef double v4f64 __attribute__((ext_vector_type(4)));

namespace {
constexpr double kU = 1.1102230246251565e-16;  // 2^-53
// The scaled matrix has a component of at least one half, so its norm is at least that:
// what vanishes against it is dropped, however small the leaf or node that it stands in.
constexpr double kNormMin = 0.5;
constexpr int kLeaf = 16;       // rows of a leaf, at most
constexpr int kTriFused = 2048; // rows whose step vectors a workgroup keeps in LDS
constexpr int kBt = 32;         // reflectors per back-transform block
}  // namespace

// sum over the wavefront, in every lane
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_val(double x, int lane) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wsum(double x) {
  x += dpp_mov<0x128>(x);  // row_ror:8, 4, 2, 1
  x += dpp_mov<0x124>(x);
  x += dpp_mov<0x122>(x);
  x += dpp_mov<0x121>(x);
  return (lane_val(x, 0) + lane_val(x, 16)) + (lane_val(x, 32) + lane_val(x, 48));
}
__device__ __forceinline__ double wprod(double x) {
  x *= dpp_mov<0x128>(x);
  x *= dpp_mov<0x124>(x);
  x *= dpp_mov<0x122>(x);
  x *= dpp_mov<0x121>(x);
  return (lane_val(x, 0) * lane_val(x, 16)) * (lane_val(x, 32) * lane_val(x, 48));
}
__device__ __forceinline__ int wsum_i(int x) {
  for (int h = 32; h > 0; h >>= 1) x += __shfl_xor(x, h);
  return x;
}

// p[i] where ok, else 0: the load is made in either case, at i or at 0, so that several in
// a row are in flight at once (a load under a branch waits for the one before)
__device__ __forceinline__ cpx<double> load_if(const cpx<double>* __restrict__ p, int i, bool ok) {
  const cpx<double> x = p[ok ? i : 0];
  return mk(ok ? x.x : 0.0, ok ? x.y : 0.0);
}

// ------------------------------------------------------------- norms, checks, scaling
// per block: the largest component, a non-finite flag, and, relative to the block's
// largest component, the sums of squares of the off-diagonal entries and of the
// off-diagonal anti-Hermitian part; the range of the diagonal's imaginary parts
__global__ void __launch_bounds__(256) k_eig_norms(const cpx<double>* __restrict__ A, int N,
                                                   double* __restrict__ part) {
  __shared__ double sh[256];
  const size_t nn = (size_t)N * N;
  const int t = threadIdx.x;
  auto reduce = [&](double x, auto op) {
    sh[t] = x;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (t < h) sh[t] = op(sh[t], sh[t + h]);
      __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
  };
  auto mx = [](double a, double b) { return fmax(a, b); };
  auto add = [](double a, double b) { return a + b; };
  double big = 0.0, bad = 0.0, dmin = INFINITY, dmax = -INFINITY;
  for (size_t e = (size_t)blockIdx.x * 256 + t; e < nn; e += (size_t)gridDim.x * 256) {
    const cpx<double> x = A[e];
    if (!(isfinite(x.x) && isfinite(x.y))) bad = 1.0;
    big = fmax(big, fmax(fabs(x.x), fabs(x.y)));
    if (e / N == e % N) {
      dmin = fmin(dmin, x.y);
      dmax = fmax(dmax, x.y);
    }
  }
  big = reduce(big, mx);
  const double inv = big > 0.0 ? 1.0 / big : 0.0;
  double all = 0.0, off = 0.0, anti = 0.0;
  if (isfinite(inv))
    for (size_t e = (size_t)blockIdx.x * 256 + t; e < nn; e += (size_t)gridDim.x * 256) {
      const int i = (int)(e / N), j = (int)(e % N);
      const cpx<double> x = scal(A[e], inv);
      const double s = x.x * x.x + x.y * x.y;
      all += s;
      if (i != j) {
        const cpx<double> y = scal(A[(size_t)j * N + i], inv);
        const double ax = 0.5 * (x.x - y.x), ay = 0.5 * (x.y + y.y);
        off += s;
        anti += ax * ax + ay * ay;
      }
    }
  bad = reduce(bad, mx);
  all = reduce(all, add);
  off = reduce(off, add);
  anti = reduce(anti, add);
  dmax = reduce(dmax, mx);
  dmin = -reduce(-dmin, mx);
  if (t == 0) {
    double* o = part + 7 * (size_t)blockIdx.x;
    o[0] = big;
    o[1] = bad;
    o[2] = all;
    o[3] = off;
    o[4] = anti;
    o[5] = dmin;
    o[6] = dmax;
  }
}

// A <- its Hermitian part times 2^-ex
__global__ void k_eig_scale(cpx<double>* __restrict__ A, int N, int ex) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)N * N) return;
  const int i = (int)(e / N), j = (int)(e % N);
  if (i > j) return;
  const cpx<double> x = A[e], y = A[(size_t)j * N + i];
  const double re = 0.5 * (ldexp(x.x, -ex) + ldexp(y.x, -ex));
  const double im = i == j ? 0.0 : 0.5 * (ldexp(x.y, -ex) - ldexp(y.y, -ex));
  A[e] = mk(re, im);
  A[(size_t)j * N + i] = mk(re, -im);
}

// ------------------------------------------------------------- tridiagonal reduction
// The reflector of a column c with |c|^2 = n2 below the diagonal and first entry c1:
// u = c - beta e_1 with beta = -(c1 / |c1|) |c|, v' = u / |u|.  A column of at most one
// entry below the diagonal, or of a norm that vanishes against the matrix (entries below
// one), is left as it is (v' = 0).  |c1| is not taken from a square that is subnormal or
// zero: u must have |u|^2 = 2 |c| (|c| + |c1|) to working precision for H to be unitary.
struct Reflector {
  cpx<double> u1, e;  // first entry of u; the off-diagonal entry that remains
  double inv;         // 1 / |u|, 0 where the column is left
};
__device__ __forceinline__ Reflector reflector(double n2, cpx<double> c1, int n) {
  Reflector r;
  r.u1 = c1;
  r.inv = 0.0;
  r.e = n == 2 ? c1 : mk(0.0, 0.0);
  if (n > 2 && n2 > 1e-290) {
    const double nrm = sqrt(n2), a2 = c1.x * c1.x + c1.y * c1.y;
    const double al = a2 > 1e-280 ? sqrt(a2) : hypot(c1.x, c1.y);
    const double ia = nrm / al;
    // below 1e-290 of a norm of at least 1e-145 c1 vanishes, and its phase is free
    const cpx<double> b = al > 1e-290 ? scal(c1, ia) : mk(nrm, 0.0);
    r.e = mk(-b.x, -b.y);
    r.u1 = c1 + b;
    r.inv = 1.0 / sqrt(2.0 * nrm * (nrm + al));
  }
  return r;
}

// The vectors of step j over rows j..N-1 (index 0 is row j): from the last reflector v
// and y = A v the update vector w = 2 (y - (v^H y) v), the column j of the updated
// matrix A - v w^H - w v^H, and its reflector.  A thread keeps its Q entries of each in
// registers, so that all loads are in flight at once; emit(i, v, w, v') receives them.
// red: LDS of 2 T / 64 + 2 doubles.  d[j], e[j] are written by `lead`.
template <int T, int Q, typename F>
__device__ __forceinline__ void tri_vectors(const cpx<double>* __restrict__ A, int N, int j,
                                            const cpx<double>* __restrict__ vprev,
                                            const cpx<double>* __restrict__ yprev, double* red,
                                            double* __restrict__ d, cpx<double>* __restrict__ e,
                                            bool lead, F emit) {
  const int t = threadIdx.x, n = N - j, lane = t & 63, wave = t >> 6;
  constexpr int W = T / 64;
  const cpx<double>* row = A + (size_t)j * N + j;
  const cpx<double> zero = mk(0.0, 0.0);
  cpx<double> v[Q], w[Q], c[Q], vj = zero, wj = zero;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = t + T * q;
    const bool in = i < n, pd = in && j > 0;
    v[q] = pd ? vprev[j + i] : zero;
    w[q] = pd ? yprev[j + i] : zero;
    c[q] = in ? row[i] : zero;
  }
  if (j > 0) {
    vj = vprev[j];
    wj = yprev[j];
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) s += v[q].x * w[q].x + v[q].y * w[q].y;
    s = wsum(s);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    s = 0.0;
#pragma unroll
    for (int q = 0; q < W; ++q) s += red[q];
    wj = scal(wj - scal(vj, s), 2.0);
#pragma unroll
    for (int q = 0; q < Q; ++q) w[q] = scal(w[q] - scal(v[q], s), 2.0);
  }
  double n2 = 0.0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    c[q] = mk(c[q].x, -c[q].y) - cmulc(wj, v[q]) - cmulc(vj, w[q]);
    if (q > 0 || t > 0) n2 += c[q].x * c[q].x + c[q].y * c[q].y;
  }
  n2 = wsum(n2);
  if (lane == 0) red[W + wave] = n2;
  if (t == 1) {
    red[2 * W] = c[0].x;
    red[2 * W + 1] = c[0].y;
  }
  __syncthreads();
  n2 = 0.0;
#pragma unroll
  for (int q = 0; q < W; ++q) n2 += red[W + q];
  const Reflector r = reflector(n2, mk(red[2 * W], red[2 * W + 1]), n);
  if (lead && t == 0) {
    d[j] = c[0].x;
    if (n > 1) e[j] = r.e;
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = t + T * q;
    const cpx<double> u = i == 0 ? zero : i == 1 ? r.u1 : c[q];
    if (i < n) emit(i, v[q], w[q], scal(u, r.inv));
  }
}

// Step j: the rows below j of the matrix take the pending rank-two update and their
// product with the new reflector, S wavefronts per row; a row, up to 1024 columns, is
// fetched before the vectors are formed.  Up to T Q rows every workgroup forms the vectors
// anew in its LDS, which costs less than a second launch; with Q = 0 they come from global
// memory (k_tri_vec).
//
// One kernel boundary per column orders the steps (each row of y needs the whole new
// reflector, and the next reflector all of y).  Bound: the latency of that chain, 5.9 us
// per column over the 1000 columns of a 1000-row matrix (7.2 above 512 rows, 4.1 below
// 256; 8.0 with the vectors' passes through LDS).  Of the 7.2, the launch and the vectors
// are about 4.  Above 256 rows two wavefronts share a row: 7.2 us above 512 rows, 7.4 with
// one, 7.7 with four (and 8.2 with one each for eight rows per workgroup).
// first group of `rows` rows (a workgroup's) of step j's grid: a multiple of the XCD count,
// so that a group, which is workgroup (group mod 8) of every step, stays with one XCD's L2
__host__ __device__ __forceinline__ int tri_group(int j, int rows) {
  return (j + 1) / rows / kXcd * kXcd;
}
template <int Q, int T, int S>
__global__ void __launch_bounds__(T) k_tri_step(cpx<double>* __restrict__ A, int N, int j,
                                                  const cpx<double>* __restrict__ vprev,
                                                  const cpx<double>* __restrict__ yprev,
                                                  const cpx<double>* __restrict__ wg,
                                                  cpx<double>* __restrict__ vout,
                                                  cpx<double>* __restrict__ yout,
                                                  double* __restrict__ d,
                                                  cpx<double>* __restrict__ e) {
  extern __shared__ char smem[];
  __shared__ double red[2 * (T / 64) + 2];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, n = N - j;
  constexpr int rows = T / 64 / S;
  __shared__ cpx<double> ysum[T / 64];
  const int first = 1 + lane + 64 * (wave % S);  // this wavefront's columns: first + 64 S q
  const int i = (tri_group(j, rows) + blockIdx.x) * rows + wave / S - j;  // row j + i
  const bool live = i > 0 && i < n;
  cpx<double>* row = A + (size_t)(j + (live ? i : 0)) * N + j;
  constexpr int kPre = Q == 0 ? 8 : Q * T / 64 / S < 16 / S ? Q * T / 64 / S : 16 / S;
  cpx<double> a[kPre];
#pragma unroll
  for (int q = 0; q < kPre; ++q) {
    const int k = first + 64 * S * q;
    a[q] = live && k < n ? row[k] : mk(0.0, 0.0);
  }
  const cpx<double>*w, *vo, *vn;
  if (Q > 0) {
    auto* ls = reinterpret_cast<cpx<double>*>(smem);
    const bool lead = blockIdx.x == 0;
    tri_vectors<T, Q ? Q : 1>(A, N, j, vprev, yprev, red, d, e, lead,
                                [&](int k, cpx<double> v, cpx<double> u, cpx<double> x) {
                                  ls[k] = u;
                                  ls[n + k] = v;
                                  ls[2 * n + k] = x;
                                  if (lead) vout[j + k] = x;
                                });
    __syncthreads();
    w = ls;
    vo = ls + n;
    vn = ls + 2 * n;
    if (lead)
      for (int k = t; k < j; k += T) vout[k] = mk(0.0, 0.0);
  } else {
    w = wg + j;
    vo = vprev + j;
    vn = vout + j;
  }
  const bool pend = j > 0;
  const cpx<double> vi = pend && live ? vo[i] : mk(0.0, 0.0),
                    wi = pend && live ? w[i] : mk(0.0, 0.0);
  cpx<double> acc = mk(0.0, 0.0);
  auto one = [&](int k, cpx<double> x) {
    if (pend) {
      const cpx<double> wk = w[k], vk = vo[k];
      x = x - cmulc(wk, vi) - cmulc(vk, wi);
      row[k] = x;
    }
    const cpx<double> vk = vn[k];
    acc = acc + cmul(x, vk);
  };
#pragma unroll
  for (int q = 0; q < kPre; ++q) {
    const int k = first + 64 * S * q;
    if (live && k < n) one(k, a[q]);
  }
  for (int k0 = first + 64 * S * kPre; live && k0 < n; k0 += 64 * S * kPre) {
#pragma unroll
    for (int q = 0; q < kPre; ++q) {
      const int k = k0 + 64 * S * q;
      if (k < n) a[q] = row[k];
    }
#pragma unroll
    for (int q = 0; q < kPre; ++q) {
      const int k = k0 + 64 * S * q;
      if (live && k < n) one(k, a[q]);
    }
  }
  const double yr = wsum(acc.x), yi = wsum(acc.y);
  if (S == 1) {
    if (live && lane == 0) yout[j + i] = mk(yr, yi);
    return;
  }
  if (lane == 0) ysum[wave] = mk(yr, yi);
  __syncthreads();
  if (live && lane == 0 && wave % S == 0) {
    cpx<double> y = ysum[wave];
#pragma unroll
    for (int q = 1; q < S; ++q) y = y + ysum[wave + q];
    yout[j + i] = y;
  }
}

// The vectors of a step above kTriFused rows, where every workgroup's own copy would not
// fit its LDS: one workgroup forms them in global memory.
__global__ void __launch_bounds__(1024) k_tri_vec(const cpx<double>* __restrict__ A, int N, int j,
                                                  const cpx<double>* __restrict__ vprev,
                                                  const cpx<double>* __restrict__ yprev,
                                                  cpx<double>* __restrict__ wg,
                                                  cpx<double>* __restrict__ vout,
                                                  double* __restrict__ d,
                                                  cpx<double>* __restrict__ e) {
  __shared__ double red[34];
  for (int k = threadIdx.x; k < j; k += 1024) vout[k] = mk(0.0, 0.0);
  tri_vectors<1024, 8>(A, N, j, vprev, yprev, red, d, e, true,
                       [&](int k, cpx<double>, cpx<double> u, cpx<double> x) {
                         wg[j + k] = u;
                         vout[j + k] = x;
                       });
}

// |e| and the phases D_0 = 1, D_{j+1} = D_j e_j / |e_j| that make the matrix real, by one
// workgroup: a scan over the threads' pieces
__global__ void __launch_bounds__(1024) k_tri_phase(const cpx<double>* __restrict__ e, int N,
                                                    double* __restrict__ er,
                                                    cpx<double>* __restrict__ D) {
  __shared__ cpx<double> sc[2][1024];
  const int t = threadIdx.x, per = (N + 1023) / 1024;
  auto unit = [&](int j, double* mag) {
    const cpx<double> x = e[j];
    const double m = hypot(x.x, x.y);
    *mag = m;
    // an entry so small vanishes against the norm, and a subnormal m gives no unit vector
    return m > 1e-290 ? mk(x.x / m, x.y / m) : mk(1.0, 0.0);
  };
  auto norm1 = [](cpx<double> z) { return scal(z, 1.0 / hypot(z.x, z.y)); };
  cpx<double> p = mk(1.0, 0.0);
  for (int q = 0; q < per; ++q) {
    const int j = t * per + q;
    if (j < N - 1) {
      double m;
      p = cmul(p, unit(j, &m));
      er[j] = m;
    }
  }
  sc[0][t] = p;
  __syncthreads();
  int cur = 0;
  for (int h = 1; h < 1024; h <<= 1) {
    cpx<double> x = sc[cur][t];
    if (t >= h) x = norm1(cmul(x, sc[cur][t - h]));
    sc[cur ^ 1][t] = x;
    cur ^= 1;
    __syncthreads();
  }
  p = t > 0 ? sc[cur][t - 1] : mk(1.0, 0.0);
  for (int q = 0; q < per; ++q) {
    const int j = t * per + q;
    if (j >= N) break;
    D[j] = p;
    double m;
    if (j < N - 1) p = norm1(cmul(p, unit(j, &m)));
  }
}

// ------------------------------------------------------------- divide and conquer
// Leaves are rows [b_q, b_{q+1}), b_q = q N / leaves; a level merges s leaves each side.
// Qt holds eigenvectors as rows: row c of a node's diagonal block is its c-th vector.
__host__ __device__ __forceinline__ int dc_bound(int q, int N, int leaves) {
  return (int)((long long)q * N / leaves);
}

// 1 / sqrt(x) for normal positive x: the hardware estimate and two Newton steps
__device__ __forceinline__ double rsq_newton(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// Implicit symmetric QR with Wilkinson's shift on one leaf per wavefront: every lane
// carries the scalar recurrence in registers (the entries ahead are loaded from LDS a
// step early), lane r the r-th components of the vectors.  Bound: the latency of its
// rotations in series, about 250 for 16 rows: 75 us.  Leaves of 32 rows took 264 us (494
// with the entries in LDS and library square roots and divisions), more than the level of
// merges that they save.
__global__ void __launch_bounds__(64) k_dc_leaf(const double* __restrict__ d,
                                                const double* __restrict__ e, int N, int leaves,
                                                double* __restrict__ lam, double* __restrict__ Qt,
                                                int* __restrict__ flag) {
  __shared__ double q[kLeaf][kLeaf + 1];
  __shared__ double sd[kLeaf + 2], se[kLeaf + 2];
  const int t = threadIdx.x, b = blockIdx.x;
  const int lo = dc_bound(b, N, leaves), hi = dc_bound(b + 1, N, leaves), n = hi - lo;
  const bool own = t < n;
  if (t < kLeaf + 2) sd[t] = se[t] = 0.0;
  __syncthreads();
  if (own) {
    double x = d[lo + t];
    if (t == 0 && lo > 0) x -= e[lo - 1];
    if (t == n - 1 && hi < N) x -= e[hi - 1];
    sd[t] = x;
    se[t] = t < n - 1 ? e[lo + t] : 0.0;
    for (int c = 0; c < n; ++c) q[c][t] = c == t ? 1.0 : 0.0;
  }
  __syncthreads();
  double nrm = 0.0;
  for (int k = 0; k < n; ++k) nrm = fmax(nrm, fmax(fabs(sd[k]), fabs(se[k])));
  const double tol = kU * fmax(nrm, kNormMin);
  int hiq = n - 1, budget = 40 * n;
  while (hiq > 0 && budget-- > 0) {
    // the last unreduced block [p, hiq]
    const unsigned long long big = __ballot(t < hiq && fabs(se[min(t, kLeaf)]) > tol);
    if (big == 0) {
      hiq = 0;
      break;
    }
    hiq = 64 - __builtin_clzll(big);
    const unsigned long long gap = ~big & ((1ull << hiq) - 1);
    const int p = gap ? 64 - __builtin_clzll(gap) : 0;
    const double a = sd[hiq - 1], bb = se[hiq - 1], c = sd[hiq];
    const double h = 0.5 * (a - c);
    const double mu = c - bb * bb / (h + copysign(sqrt(h * h + bb * bb), h));
    double dk = sd[p], ek = se[p], x = dk - mu, z = ek;
    double dl = sd[p + 1], en = se[p + 1];
    double u = own ? q[p][t] : 0.0, w = own ? q[p + 1][t] : 0.0;
    for (int k = p; k < hiq; ++k) {
      const double dn = sd[k + 2], ef = se[k + 2];
      const double wn = own && k + 2 <= hiq ? q[k + 2][t] : 0.0;
      const double r2 = x * x + z * z;
      // below 1e-290 both vanish against the leaf's norm
      const bool act = r2 > 1e-290;
      const double ri = act ? rsq_newton(r2) : 0.0;
      const double cs = act ? x * ri : 1.0, sn = z * ri;
      const double g = 2.0 * cs * sn * ek, c2 = cs * cs, s2 = sn * sn;
      const double nek = (c2 - s2) * ek - cs * sn * (dk - dl);
      if (t == 0) {
        if (k > p) se[k - 1] = r2 * ri;
        sd[k] = c2 * dk + g + s2 * dl;
      }
      if (own) q[k][t] = cs * u + sn * w;
      u = cs * w - sn * u;
      w = wn;
      dk = s2 * dk - g + c2 * dl;
      x = nek;
      ek = cs * en;
      z = sn * en;
      dl = dn;
      en = ef;
    }
    if (t == 0) {
      se[hiq - 1] = x;
      sd[hiq] = dk;
    }
    if (own) q[hiq][t] = u;
    __syncthreads();
  }
  if (t == 0 && hiq > 0) *flag = 1;
  if (own) {
    const double x = sd[t];
    int r = 0;
    for (int k = 0; k < n; ++k) r += sd[k] < x || (sd[k] == x && k < t);
    lam[lo + r] = x;
    for (int c = 0; c < n; ++c) Qt[(size_t)(lo + r) * N + lo + c] = q[t][c];
  }
}

struct DcWork {
  // per row of the matrix, a node's part at [lo, hi)
  double *ds, *zs;      // the node's eigenvalues and update vector in ascending order
  int* is;              // and their rows of Qt
  double *dl, *w;       // secular problem: poles and update vector (first k), deflated (rest)
  int* src;             // their rows of Qt
  double *tau, *zh;     // roots: distance from the pole org; recomputed update vector
  int *org, *dst;       // dst: the row of each vector in the merged order
  double *rc, *rs;      // rotations of the deflation and their rows
  int *ra, *rb;
  int *k, *nrot;        // per node
  double* rho;
};

// The rank-one update of a merge: z from the last row of the left vectors and the first
// of the right ones, in ascending order of the eigenvalues; an entry whose weight
// vanishes against the norm is deflated, and one of a pair of eigenvalues so close that
// rotating the weight to the other costs nothing.  One wavefront scans 64 entries at a
// time: the tests of neighbours are made at once, and only where one succeeds does it go
// through the entries one by one (a rotation changes the next test).
// 10 us at 1000 entries, 91 with one lane going through all of them.
__global__ void __launch_bounds__(256) k_dc_deflate(const double* __restrict__ lam,
                                                    const double* __restrict__ e,
                                                    const double* __restrict__ Qt, int N,
                                                    int leaves, int s, DcWork W) {
  __shared__ double red[256];
  const int t = threadIdx.x, b = blockIdx.x;
  const int lo = dc_bound(2 * s * b, N, leaves), mid = dc_bound(2 * s * b + s, N, leaves),
            hi = dc_bound(2 * s * b + 2 * s, N, leaves);
  const double rho = 2.0 * e[mid - 1];
  double big = rho;
  for (int i = lo + t; i < hi; i += 256) {
    const double x = lam[i];
    const bool left = i < mid;
    // entries of the other side below x (ties: left first)
    int a = left ? mid : lo, z = left ? hi : mid;
    while (a < z) {
      const int m = (a + z) >> 1;
      if (left ? lam[m] < x : lam[m] <= x) a = m + 1;
      else z = m;
    }
    const int pos = left ? i + (a - mid) : (i - mid) + a;
    W.ds[pos] = x;
    W.zs[pos] = 0.70710678118654752440 * Qt[(size_t)i * N + (left ? mid - 1 : mid)];
    W.is[pos] = i;
    big = fmax(big, fabs(x));
  }
  red[t] = big;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (t < h) red[t] = fmax(red[t], red[t + h]);
    __syncthreads();
  }
  if (t >= 64) return;
  const double tol = 8.0 * kU * fmax(red[0], kNormMin);
  int k = lo, nd = hi, nr = lo, sp = -1;  // sp: the row of the entry held back
  double dp = 0.0, zp = 0.0;
  auto close = [&](double d0, double z0, double d1, double z1) {
    return fabs((d1 - d0) * z1 * z0) <= tol * (z1 * z1 + z0 * z0);
  };
  for (int c0 = lo; c0 < hi; c0 += 64) {
    const bool in = c0 + t < hi;
    const double dj = in ? W.ds[c0 + t] : 0.0, zj = in ? W.zs[c0 + t] : 0.0;
    const int sj = in ? W.is[c0 + t] : 0;
    const bool heavy = in && rho * fabs(zj) > tol;
    const unsigned long long live = __ballot(heavy), below = live & ((1ull << t) - 1);
    const unsigned long long out = __ballot(in && !heavy);
    if (in && !heavy) {
      const int x = nd - 1 - __popcll(out & ((1ull << t) - 1));
      W.dl[x] = dj;
      W.src[x] = sj;
    }
    nd -= __popcll(out);
    if (live == 0) continue;
    // the heavy entry before this one: of this piece, or the one held back
    const int pl = below ? 63 - __builtin_clzll(below) : t;
    const double qd = __shfl(dj, pl), qz = __shfl(zj, pl);
    const int qs = __shfl(sj, pl);
    const double d0 = below ? qd : dp, z0 = below ? qz : zp;
    const int s0 = below ? qs : sp;
    if (__ballot(heavy && s0 >= 0 && close(d0, z0, dj, zj)) == 0) {
      // nothing rotates: every heavy entry passes on the one before it
      const int held = sp >= 0 ? 1 : 0;
      if (heavy && s0 >= 0) {
        const int x = k + __popcll(below) - (1 - held);
        W.dl[x] = d0;
        W.w[x] = z0;
        W.src[x] = s0;
      }
      k += __popcll(live) - (1 - held);
      const int l = 63 - __builtin_clzll(live);
      dp = lane_val(dj, l);
      zp = lane_val(zj, l);
      sp = __builtin_amdgcn_readlane(sj, l);
      continue;
    }
    for (unsigned long long m = live; m; m &= m - 1) {
      const int l = __builtin_ctzll(m);
      const double d1 = lane_val(dj, l), z1 = lane_val(zj, l);
      const int s1 = __builtin_amdgcn_readlane(sj, l);
      if (sp >= 0) {
        const double t2 = z1 * z1 + zp * zp;
        if (close(dp, zp, d1, z1)) {
          const double tau = sqrt(t2), c = z1 / tau, sn = zp / tau;
          --nd;
          if (t == 0) {
            W.ra[nr] = sp;
            W.rb[nr] = s1;
            W.rc[nr] = c;
            W.rs[nr] = sn;
            W.dl[nd] = dp * c * c + d1 * sn * sn;
            W.src[nd] = sp;
          }
          ++nr;
          dp = dp * sn * sn + d1 * c * c;
          zp = tau;
          sp = s1;
          continue;
        }
        if (t == 0) {
          W.dl[k] = dp;
          W.w[k] = zp;
          W.src[k] = sp;
        }
        ++k;
      }
      dp = d1;
      zp = z1;
      sp = s1;
    }
  }
  if (t == 0) {
    if (sp >= 0) {
      W.dl[k] = dp;
      W.w[k] = zp;
      W.src[k] = sp;
    }
    W.k[b] = k - lo + (sp >= 0 ? 1 : 0);
    W.nrot[b] = nr - lo;
    W.rho[b] = rho;
  }
}

__global__ void __launch_bounds__(256) k_dc_rotate(double* __restrict__ Qt, int N, int leaves,
                                                   int s, DcWork W) {
  const int b = blockIdx.y, nr = W.nrot[b];
  if (nr == 0) return;
  const int lo = dc_bound(2 * s * b, N, leaves), hi = dc_bound(2 * s * b + 2 * s, N, leaves);
  const int g = lo + blockIdx.x * 256 + threadIdx.x;
  if (g >= hi) return;
  int held = -1;  // the row in x: a chain of rotations goes on with the last one's second row
  double x = 0.0;
  for (int r = 0; r < nr; ++r) {
    const int ia = W.ra[lo + r], ib = W.rb[lo + r];
    const double c = W.rc[lo + r], sn = W.rs[lo + r];
    if (ia != held) {
      if (held >= 0) Qt[(size_t)held * N + g] = x;
      x = Qt[(size_t)ia * N + g];
    }
    const double y = Qt[(size_t)ib * N + g];
    Qt[(size_t)ia * N + g] = c * x - sn * y;
    x = sn * x + c * y;
    held = ib;
  }
  Qt[(size_t)held * N + g] = x;
}

// The root in (0, G) of c - p / x + q / (G - x), p, q > 0
__device__ __forceinline__ double two_pole(double c, double p, double q, double G) {
  const double B = c * G + p + q, C = p * G;
  const double sq = sqrt(fmax(B * B - 4.0 * c * C, 0.0));
  return B >= 0.0 ? 2.0 * C / (B + sq) : (B - sq) / (2.0 * c);
}

// Root i of 1 + sum_j p_j / (dl_j - x), p_j = rho w_j^2, between poles i and i + 1 (the
// last one above its pole), one wavefront per root.  The unknown is the distance sg from
// the nearer pole, mirrored where that is the right one, so that the function
// g(sg) = side + sum_j p_j / (side (dl_j - dl_org) - sg) rises from -inf at 0.  Each side's
// terms are replaced by a pole term of the same value and slope; iterates are kept
// inside a bracket.  Ends when g is below its own rounding error.
__global__ void __launch_bounds__(256) k_dc_secular(int N, int leaves, int s, DcWork W) {
  const int b = blockIdx.y, k = W.k[b];
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= k) return;
  const int lo = dc_bound(2 * s * b, N, leaves);
  const double* dl = W.dl + lo;
  const double* w = W.w + lo;
  const double rho = W.rho[b];
  const bool last = i == k - 1;
  const double di = dl[i], wi = w[i], pi = rho * wi * wi;
  double side = 1.0, G = 0.0, hi, sg;
  int org = i;
  if (!last) {
    G = dl[i + 1] - di;
    const double m = 0.5 * G, pn = rho * w[i + 1] * w[i + 1];
    double f = 0.0;
    for (int j = lane; j < k; j += 64)
      if (j != i && j != i + 1) f += rho * w[j] * w[j] / ((dl[j] - di) - m);
    const double c0 = 1.0 + wsum(f);
    hi = m;
    if (c0 + (pn - pi) / m >= 0.0) {
      sg = two_pole(c0, pi, pn, G);
    } else {
      side = -1.0;
      org = i + 1;
      sg = two_pole(-c0, pn, pi, G);
    }
  } else {
    double p = 0.0;
    for (int j = lane; j < k; j += 64) p += rho * w[j] * w[j];
    hi = wsum(p) * (1.0 + 8.0 * kU);
    double f = 0.0;
    for (int j = lane; j < k - 1; j += 64) f += rho * w[j] * w[j] / ((dl[j] - di) - hi);
    const double c = 1.0 + wsum(f);
    sg = c > 0.0 ? pi / c : 0.0;
  }
  const double d0 = dl[org];
  double a = 0.0;
  for (int it = 0; it < 100; ++it) {
    if (!(sg > a && sg < hi)) {
      if (it == 0 && last && sg >= hi) sg = hi;
      else sg = a > 0.0 ? sqrt(a) * sqrt(hi) : hi * 0.125;
    }
    double sn = 0.0, dn = 0.0, sf = 0.0, df = 0.0;
    for (int j = lane; j < k; j += 64) {
      const double den = side * (dl[j] - d0) - sg;
      const double r = 1.0 / den, tj = rho * w[j] * w[j] * r, sl = tj * r;
      if (den < 0.0) {
        sn += tj;
        dn += sl;
      } else {
        sf += tj;
        df += sl;
      }
    }
    sn = wsum(sn);
    dn = wsum(dn);
    sf = wsum(sf);
    df = wsum(df);
    const double g = side + sn + sf;
    if (fabs(g) <= 8.0 * kU * (1.0 + sf - sn)) break;
    if (g < 0.0) a = sg;
    else hi = sg;
    if (hi - a <= 2.0 * kU * hi) break;
    const double p = dn * sg * sg;
    double c = side + sn + dn * sg;
    if (last) {
      sg = c > 0.0 ? p / c : -1.0;
    } else {
      const double D = G - sg;
      c += sf - df * D;
      sg = two_pole(c, p, df * D * D, G);
    }
  }
  if (lane == 0) {
    W.tau[lo + i] = side * sg;
    W.org[lo + i] = org;
  }
}

// The update vector whose exact roots the computed ones are: |zh_j|^2 =
// |x_j - dl_j| prod_{i != j} |x_i - dl_j| / |dl_i - dl_j|, one wavefront per entry.
__global__ void __launch_bounds__(256) k_dc_zhat(int N, int leaves, int s, DcWork W) {
  const int b = blockIdx.y, k = W.k[b];
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (j >= k) return;
  const int lo = dc_bound(2 * s * b, N, leaves);
  const double* dl = W.dl + lo;
  const double dj = dl[j];
  double p = 1.0;
  for (int i = lane; i < k; i += 64) {
    const double x = (dl[W.org[lo + i]] - dj) + W.tau[lo + i];
    p *= fabs(i == j ? x : x / (dl[i] - dj));
  }
  p = wprod(p);
  if (lane == 0) W.zh[lo + j] = copysign(sqrt(p), W.w[lo + j]);
}

// Row i of Ut: the unit vector of root i in the basis of the k poles.  Every eigenvalue
// of the node, deflated ones included, also finds its place in ascending order.
// `first`: at the last level only places from it on are needed.
__global__ void __launch_bounds__(256) k_dc_vec(int N, int leaves, int s, int first, DcWork W,
                                                double* __restrict__ Ut,
                                                double* __restrict__ lam) {
  const int b = blockIdx.y, k = W.k[b];
  const int lo = dc_bound(2 * s * b, N, leaves), hi = dc_bound(2 * s * b + 2 * s, N, leaves);
  const int n = hi - lo;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n) return;
  const double* dl = W.dl + lo;
  auto value = [&](int q) { return q < k ? dl[W.org[lo + q]] + W.tau[lo + q] : dl[q]; };
  const double x = value(i);
  int r = 0;
  for (int q = lane; q < n; q += 64) {
    const double y = value(q);
    r += y < x || (y == x && q < i);
  }
  r = wsum_i(r);
  if (lane == 0) {
    lam[lo + r] = x;
    W.dst[lo + i] = lo + r;
  }
  if (i >= k || lo + r < first) return;
  const double d0 = dl[W.org[lo + i]], tau = W.tau[lo + i];
  double n2 = 0.0;
  for (int j = lane; j < k; j += 64) {
    const double u = W.zh[lo + j] / ((dl[j] - d0) - tau);
    n2 += u * u;
  }
  const double inv = 1.0 / sqrt(wsum(n2));
  for (int j = lane; j < k; j += 64)
    Ut[(size_t)(lo + i) * N + lo + j] = W.zh[lo + j] / ((dl[j] - d0) - tau) * inv;
}

// Qn[dst_i] = sum_j Ut[i][j] Qt[src_j] for the k secular vectors, a copy for the rest:
// 64 x 64 tiles, four wavefronts of 32 x 32, 16 poles per stage.
__global__ void __launch_bounds__(256) k_dc_gemm(const double* __restrict__ Ut,
                                                 const double* __restrict__ Qt,
                                                 double* __restrict__ Qn, int N, int leaves,
                                                 int s, int first, DcWork W) {
  constexpr int KB = 16;
  __shared__ double sa[KB][64 + 2], sb[KB][64 + 2];
  const int b = blockIdx.z, k = W.k[b];
  const int lo = dc_bound(2 * s * b, N, leaves), hi = dc_bound(2 * s * b + 2 * s, N, leaves);
  const int n = hi - lo, i0 = blockIdx.y * 64, g0 = blockIdx.x * 64, t = threadIdx.x;
  if (i0 >= n || g0 >= n) return;
  for (int i = max(i0, k) + (t >> 6); i < min(i0 + 64, n); i += 4) {
    const int g = g0 + (t & 63), dst = W.dst[lo + i];
    if (g < n && dst >= first) Qn[(size_t)dst * N + lo + g] = Qt[(size_t)W.src[lo + i] * N + lo + g];
  }
  const int last = min(i0 + 64, k) - 1;
  if (i0 >= k || W.dst[lo + last] < first) return;
  const int lane = t & 63, wave = t >> 6, l16 = lane & 15, lk = lane >> 4;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  v4f64 acc[2][2] = {};
  // a thread's share of a stage, fetched while the one before is multiplied
  double fa[4], fb[4];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = t / KB + 16 * q, j = k0 + t % KB;
      fa[q] = i0 + i < k && j < k ? Ut[(size_t)(lo + i0 + i) * N + lo + j] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = k0 + t / 64 + 4 * q, g = g0 + t % 64;
      fb[q] = j < k && g < n ? Qt[(size_t)W.src[lo + j] * N + lo + g] : 0.0;
    }
  };
  fetch(0);
  for (int k0 = 0; k0 < k; k0 += KB) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sa[t % KB][t / KB + 16 * q] = fa[q];
      sb[t / 64 + 4 * q][t % 64] = fb[q];
    }
    fetch(k0 + KB);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KB; j += 4) {
      const double a0 = sa[j + lk][wr + l16], a1 = sa[j + lk][wr + 16 + l16];
      const double b0 = sb[j + lk][wc + l16], b1 = sb[j + lk][wc + 16 + l16];
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + wr + 16 * x + lk + 4 * r, g = g0 + wc + 16 * y + l16;
        if (i < k && g < n) Qn[(size_t)W.dst[lo + i] * N + lo + g] = acc[x][y][r];
      }
}

// ------------------------------------------------------------- back transformation
// Row r of Z: D times the tridiagonal matrix's vector of the r-th largest eigenvalue
__global__ void k_bt_start(const double* __restrict__ Qt, const cpx<double>* __restrict__ D, int N,
                           int nb, cpx<double>* __restrict__ Z) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)nb * N) return;
  const int r = (int)(e / N), g = (int)(e % N);
  Z[e] = scal(D[g], Qt[(size_t)(N - 1 - r) * N + g]);
}

// V^H V of a block of reflectors over one of `splits` column ranges
constexpr int kTfSplit = 8;
__global__ void __launch_bounds__(1024) k_bt_tgram(const cpx<double>* __restrict__ V, int N, int R,
                                                   cpx<double>* __restrict__ part) {
  __shared__ cpx<double> sv[kBt][kBt + 1];
  const int t = threadIdx.x, m = t / kBt, c = t % kBt, j0 = blockIdx.x * kBt;
  cpx<double> g = mk(0.0, 0.0);
  auto fetch = [&](int i) {
    return j0 + m < R && i < N ? V[(size_t)(j0 + m) * N + i] : mk(0.0, 0.0);
  };
  const int i1 = j0 + blockIdx.y * kBt, step = kBt * gridDim.y;
  cpx<double> next = fetch(i1 + c);
  for (int i0 = i1; i0 < N; i0 += step) {
    sv[m][c] = next;
    __syncthreads();
    next = fetch(i0 + step + c);
#pragma unroll 8
    for (int x = 0; x < kBt; ++x) g = g + cmulc(sv[m][x], sv[c][x]);
    __syncthreads();
  }
  part[((size_t)blockIdx.x * gridDim.y + blockIdx.y) * kBt * kBt + t] = g;
}

// T of H_{j0} .. H_{j0+31} = I - V T V^H: the inverse of 1/2 I plus the strictly upper
// part of V^H V, one workgroup per block, rows from the last
__global__ void __launch_bounds__(1024) k_bt_tfac(const cpx<double>* __restrict__ part, int splits,
                                                  cpx<double>* __restrict__ T) {
  __shared__ cpx<double> sg[kBt][kBt + 1];
  __shared__ cpx<double> sx[2][kBt];
  const int t = threadIdx.x, m = t / kBt, c = t % kBt;
  cpx<double> g = mk(0.0, 0.0);
  for (int q = 0; q < splits; ++q)
    g = g + part[((size_t)blockIdx.x * splits + q) * kBt * kBt + t];
  sg[m][c] = g;
  cpx<double> acc = mk(m == c ? 1.0 : 0.0, 0.0), x = acc;
  for (int i = kBt - 1; i >= 0; --i) {
    if (m == i) {
      x = scal(acc, 2.0);
      sx[i & 1][c] = x;
    }
    __syncthreads();
    if (m < i) acc = acc - cmul(sg[m][i], sx[i & 1][c]);
  }
  T[(size_t)blockIdx.x * kBt * kBt + t] = x;
}

// Columns of Z per workgroup, 16 per wavefront: a block of reflectors is two dependent
// launches, and 100 vectors of 1000 rows give them 56 and 112 workgroups, 5.4 and 8.2 us
// (28 workgroups of 64 columns per wavefront: 13 and 18).
constexpr int kBtSpan = 64, kBtGram = 128;
// partial V^H Z over one span: part[span][b][m]
__global__ void __launch_bounds__(512) k_bt_gram(const cpx<double>* __restrict__ V,
                                                 const cpx<double>* __restrict__ Z, int N, int R,
                                                 int nb, int j0, cpx<double>* __restrict__ part) {
  __shared__ cpx<double> sg[8][16][kBt + 1];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, l16 = lane & 15, lk = lane >> 4;
  const int b0 = blockIdx.x * 16, i0 = j0 + blockIdx.y * kBtGram + wave * 16;
  const bool rz = b0 + l16 < nb, r0 = j0 + l16 < R, r1 = j0 + 16 + l16 < R;
  const cpx<double>* z = Z + (size_t)(rz ? b0 + l16 : 0) * N;
  const cpx<double>* va = V + (size_t)(r0 ? j0 + l16 : 0) * N;
  const cpx<double>* vb = V + (size_t)(r1 ? j0 + 16 + l16 : 0) * N;
  const cpx<double> o = mk(0.0, 0.0);
  v4f64 re[2] = {}, im[2] = {};
#pragma unroll
  for (int k = 0; k < 16; k += 4) {
    const int i = i0 + k + lk;
    const bool in = i < N;
    const cpx<double> zz = load_if(z, i, in && rz), x0 = load_if(va, i, in && r0),
                      x1 = load_if(vb, i, in && r1);
    // rows: vectors b, columns: reflectors
    re[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(zz.x, x0.x, re[0], 0, 0, 0);
    re[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(zz.x, x1.x, re[1], 0, 0, 0);
    im[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(zz.y, x0.x, im[0], 0, 0, 0);
    im[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(zz.y, x1.x, im[1], 0, 0, 0);
    re[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(zz.y, x0.y, re[0], 0, 0, 0);
    re[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(zz.y, x1.y, re[1], 0, 0, 0);
    im[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(-zz.x, x0.y, im[0], 0, 0, 0);
    im[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-zz.x, x1.y, im[1], 0, 0, 0);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) sg[wave][lk + 4 * r][16 * h + l16] = mk(re[h][r], im[h][r]);
  __syncthreads();
  {
    const int e = t, b = e / kBt, m = e % kBt;
    part[(((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 16 + b) * kBt + m] =
        ((sg[0][b][m] + sg[1][b][m]) + (sg[2][b][m] + sg[3][b][m])) +
        ((sg[4][b][m] + sg[5][b][m]) + (sg[6][b][m] + sg[7][b][m]));
  }
}

// Z -= V T (V^H Z) on one span of columns of 16 vectors
__global__ void __launch_bounds__(256) k_bt_apply(const cpx<double>* __restrict__ V,
                                                  const cpx<double>* __restrict__ T,
                                                  const cpx<double>* __restrict__ part, int nspan,
                                                  int N, int R, int nb, int j0,
                                                  cpx<double>* __restrict__ Z) {
  __shared__ cpx<double> sg[16][kBt + 1];
  __shared__ cpx<double> st[kBt][kBt + 1];
  __shared__ cpx<double> sm[16][kBt + 1];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, l16 = lane & 15, lk = lane >> 4;
  const int b0 = blockIdx.x * 16, i0 = j0 + blockIdx.y * kBtSpan + wave * 16;
  const cpx<double> o = mk(0.0, 0.0);
  const int i = i0 + l16;
  cpx<double> v[kBt / 4];
#pragma unroll
  for (int k = 0; k < kBt / 4; ++k)
    v[k] = load_if(V + (size_t)min(j0 + 4 * k + lk, R - 1) * N, i, i < N && j0 + 4 * k + lk < R);
  cpx<double> z[4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
    z[r] = load_if(Z + (size_t)min(b0 + lk + 4 * r, nb - 1) * N, i, i < N);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = t + 256 * q;
    st[e / kBt][e % kBt] = T[(size_t)j0 * kBt + e];
  }
  for (int e = t; e < 16 * kBt; e += 256) {
    const cpx<double>* p = part + (size_t)blockIdx.x * 16 * kBt + e;
    const size_t sp = (size_t)gridDim.x * 16 * kBt;
    cpx<double> x = o;
    for (int q0 = 0; q0 < nspan; q0 += 8) {
      cpx<double> y[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = load_if(p + min(q0 + q, nspan - 1) * sp, 0, q0 + q < nspan);
#pragma unroll
      for (int q = 0; q < 8; ++q) x = x + y[q];
    }
    sg[e / kBt][e % kBt] = x;
  }
  __syncthreads();
  for (int e = t; e < 16 * kBt; e += 256) {
    const int b = e / kBt, m = e % kBt;
    cpx<double> x = o, y = o;  // T is zero below its diagonal
#pragma unroll
    for (int q = 0; q < kBt; q += 2) {
      x = x + cmul(st[m][q], sg[b][q]);
      y = y + cmul(st[m][q + 1], sg[b][q + 1]);
    }
    sm[b][m] = x + y;
  }
  __syncthreads();
  v4f64 re = {}, im = {};
#pragma unroll
  for (int k = 0; k < kBt / 4; ++k) {
    const cpx<double> x = sm[l16][4 * k + lk];
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, v[k].x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, v[k].y, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.y, v[k].y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, v[k].x, im, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int b = b0 + lk + 4 * r;
    if (b < nb && i < N) Z[(size_t)b * N + i] = z[r] - mk(re[r], im[r]);
  }
}

// U[g][r] = Z[r][g] and, in place, Z <- conj(Z); lam: eigenvalues with the scale put back
__global__ void k_bt_finish(cpx<double>* __restrict__ Z, int N, int nb, cpx<double>* __restrict__ U,
                            const double* __restrict__ d, int ex, double* __restrict__ lam) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (lam && e < (size_t)N) lam[e] = ldexp(d[e], ex);
  if (e >= (size_t)nb * N) return;
  const int r = (int)(e / N), g = (int)(e % N);
  const cpx<double> z = Z[e];
  U[(size_t)g * nb + r] = z;
  Z[e] = mk(z.x, -z.y);
}

// U[g][r] and Uh[r][g] = conj(U[g][r]): the eigenvectors of the nb largest eigenvalues of
// the Hermitian A (destroyed) in descending order; lam (may be NULL): all N eigenvalues
// ascending.  Refuses non-finite entries and a matrix that is not Hermitian.
gw_status herm_eig_top(gw_ctx* c, int N, int nb, cpx<double>* A, cpx<double>* U, cpx<double>* Uh,
                       double* lam) {
  const size_t nn = (size_t)N * N;
  int levels = 0;
  while (((N + (1 << levels) - 1) >> levels) > kLeaf) ++levels;
  const int leaves = 1 << levels, R = std::max(0, N - 2), nblk = (R + kBt - 1) / kBt;
  const int nspan = (N + kBtGram - 1) / kBtGram, nbt = (nb + 15) / 16;
  const int nparts = (int)std::min<size_t>(1024, (nn + 255) / 256);
  const size_t row = align_up((size_t)N * 16);
  const size_t bytes = align_up(nn * 16) + align_up(nn * 8) + 24 * row +
                       4 * align_up((size_t)leaves * 8) +
                       align_up((size_t)std::max(nblk, 1) * kBt * kBt * 16) +
                       align_up((size_t)std::max(nblk, 1) * kTfSplit * kBt * kBt * 16) +
                       align_up((size_t)nspan * nbt * 16 * kBt * 16) +
                       align_up((size_t)nparts * 7 * 8) + 256;
  char* base = nullptr;
  if (hipMalloc(reinterpret_cast<void**>(&base), bytes) != hipSuccess)
    return fail(c, GW_ENOMEM, "eigenvector buffers of %zu bytes", bytes);
  struct Free {
    char* p;
    gw_ctx* c;
    ~Free() {
      (void)hipStreamSynchronize(c->stream);
      (void)hipFree(p);
    }
  } guard{base, c};
  size_t off = 0;
  auto take = [&](size_t b) {
    char* p = base + off;
    off += align_up(b);
    return p;
  };
  auto* V = reinterpret_cast<cpx<double>*>(take(nn * 16));
  auto* Ut = reinterpret_cast<double*>(take(nn * 8));
  auto vec = [&] { return reinterpret_cast<cpx<double>*>(take((size_t)N * 16)); };
  auto dvec = [&] { return reinterpret_cast<double*>(take((size_t)N * 8)); };
  auto ivec = [&] { return reinterpret_cast<int*>(take((size_t)N * 4)); };
  cpx<double>* y[2] = {vec(), vec()};
  cpx<double>*wv = vec(), *e = vec(), *D = vec();
  double *d = dvec(), *er = dvec(), *ev = dvec();
  DcWork W;
  W.ds = dvec();
  W.zs = dvec();
  W.is = ivec();
  W.dl = dvec();
  W.w = dvec();
  W.src = ivec();
  W.tau = dvec();
  W.zh = dvec();
  W.org = ivec();
  W.dst = ivec();
  W.rc = dvec();
  W.rs = dvec();
  W.ra = ivec();
  W.rb = ivec();
  W.k = reinterpret_cast<int*>(take((size_t)leaves * 4));
  W.nrot = reinterpret_cast<int*>(take((size_t)leaves * 4));
  W.rho = reinterpret_cast<double*>(take((size_t)leaves * 8));
  auto* T = reinterpret_cast<cpx<double>*>(take((size_t)std::max(nblk, 1) * kBt * kBt * 16));
  auto* tp = reinterpret_cast<cpx<double>*>(
      take((size_t)std::max(nblk, 1) * kTfSplit * kBt * kBt * 16));
  auto* part = reinterpret_cast<cpx<double>*>(take((size_t)nspan * nbt * 16 * kBt * 16));
  auto* np = reinterpret_cast<double*>(take((size_t)nparts * 7 * 8));
  auto* flag = reinterpret_cast<int*>(take(4));
  // the tridiagonal problem's two vector buffers take the matrix's place
  double* Q[2] = {reinterpret_cast<double*>(A), reinterpret_cast<double*>(A) + nn};
  int ex = 0;
  {
    std::vector<double> hp(7 * (size_t)nparts);
    {
      ProfScope ps(c, "lowrank_prep");
      hipLaunchKernelGGL(k_eig_norms, dim3(nparts), dim3(256), 0, c->stream, A, N, np);
      GW_CHECK_LAUNCH(c, "k_eig_norms");
    }
    GW_HIP(c, hipMemcpyAsync(hp.data(), np, hp.size() * 8, hipMemcpyDeviceToHost, c->stream));
    GW_HIP(c, hipStreamSynchronize(c->stream));
    double big = 0.0, all = 0.0, offn = 0.0, anti = 0.0, dmin = INFINITY, dmax = -INFINITY;
    for (int b = 0; b < nparts; ++b) {
      const double* p = hp.data() + 7 * (size_t)b;
      if (p[1] != 0.0) return fail(c, GW_EINVAL, "non-finite entries in epst(0)");
      big = std::max(big, p[0]);
    }
    for (int b = 0; b < nparts; ++b) {
      const double* p = hp.data() + 7 * (size_t)b;
      const double r = big > 0.0 ? p[0] / big : 0.0, r2 = r * r;
      all += p[2] * r2;
      offn += p[3] * r2;
      anti += p[4] * r2;
      dmin = std::min(dmin, p[5]);
      dmax = std::max(dmax, p[6]);
    }
    if (big > 0.0) {
      // a matrix further from Hermitian than rounding leaves it has no such basis; where
      // it is diagonal to rounding its real parts are the eigenvalues
      const double lim = 1e-11 * std::sqrt(all);
      const double spread = dmax / big - dmin / big;
      if (std::sqrt(anti) > lim || (std::sqrt(offn) > 1e-14 * std::sqrt(all) && spread > lim))
        return fail(c, GW_EINVAL, "epst(0) is not Hermitian: the eigen-decomposition does not exist (anti-Hermitian norm %.3g of the whole)", std::sqrt(anti / all));
      (void)std::frexp(big, &ex);
    }
  }
  const unsigned gnn = (unsigned)((nn + 255) / 256);
  {
    ProfScope ps(c, "lowrank_tridiag");
    if (N * 48 > 65536)
      GW_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tri_step<4, 512, 2>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kTriFused * 48));
    hipLaunchKernelGGL(k_eig_scale, dim3(gnn), dim3(256), 0, c->stream, A, N, ex);
    for (int j = 0; j < N; ++j) {
      const int n = N - j;
      const int T = n > 256 && n <= kTriFused ? 512 : 256, rows = 4;
      const dim3 grid(std::max(1, (N + rows - 1) / rows - tri_group(j, rows)));
      const cpx<double>* vp = V + (size_t)std::max(j - 1, 0) * N;
      cpx<double>* vo = V + (size_t)j * N;
      if (n > kTriFused)
        hipLaunchKernelGGL(k_tri_vec, dim3(1), dim3(1024), 0, c->stream, A, N, j, vp,
                           y[(j + 1) & 1], wv, vo, d, e);
      auto* step = n > kTriFused ? &k_tri_step<0, 256, 1>
                   : n > 1024    ? &k_tri_step<4, 512, 2>
                   : n > 512     ? &k_tri_step<2, 512, 2>
                   : n > 256     ? &k_tri_step<1, 512, 2>
                                 : &k_tri_step<1, 256, 1>;
      hipLaunchKernelGGL(step, grid, dim3(T), n > kTriFused ? 0 : (size_t)n * 48, c->stream, A,
                         N, j, vp, y[(j + 1) & 1], wv, vo, y[j & 1], d, e);
    }
    GW_CHECK_LAUNCH(c, "tridiagonal reduction");
  }
  {
    ProfScope ps(c, "lowrank_divide");
    hipLaunchKernelGGL(k_tri_phase, dim3(1), dim3(1024), 0, c->stream, e, N, er, D);
    GW_HIP(c, hipMemsetAsync(flag, 0, 4, c->stream));
    GW_HIP(c, hipMemsetAsync(Q[0], 0, nn * 16, c->stream));
    hipLaunchKernelGGL(k_dc_leaf, dim3(leaves), dim3(64), 0, c->stream, d, er, N, leaves, ev, Q[0],
                       flag);
    for (int l = 0, s = 1; l < levels; ++l, s <<= 1) {
      const int nodes = leaves / (2 * s);
      const int nmax = (int)(((long long)N * 2 * s + leaves - 1) / leaves) + 1;
      const int first = nodes == 1 ? N - nb : 0;
      const dim3 waves((nmax + 3) / 4, nodes);
      hipLaunchKernelGGL(k_dc_deflate, dim3(nodes), dim3(256), 0, c->stream, ev, er, Q[l & 1], N,
                         leaves, s, W);
      hipLaunchKernelGGL(k_dc_rotate, dim3((nmax + 255) / 256, nodes), dim3(256), 0, c->stream,
                         Q[l & 1], N, leaves, s, W);
      hipLaunchKernelGGL(k_dc_secular, waves, dim3(256), 0, c->stream, N, leaves, s, W);
      hipLaunchKernelGGL(k_dc_zhat, waves, dim3(256), 0, c->stream, N, leaves, s, W);
      hipLaunchKernelGGL(k_dc_vec, waves, dim3(256), 0, c->stream, N, leaves, s, first, W, Ut, ev);
      const int nt = (nmax + 63) / 64;
      hipLaunchKernelGGL(k_dc_gemm, dim3(nt, nt, nodes), dim3(256), 0, c->stream, Ut, Q[l & 1],
                         Q[(l + 1) & 1], N, leaves, s, first, W);
    }
    GW_CHECK_LAUNCH(c, "divide and conquer");
  }
  {
    ProfScope ps(c, "lowrank_basis");
    const unsigned gz = (unsigned)(((size_t)std::max(nb, 1) * N + 255) / 256);
    hipLaunchKernelGGL(k_bt_start, dim3(gz), dim3(256), 0, c->stream, Q[levels & 1], D, N, nb, Uh);
    if (nblk > 0)
      {
      hipLaunchKernelGGL(k_bt_tgram, dim3(nblk, kTfSplit), dim3(1024), 0, c->stream, V, N, R, tp);
      hipLaunchKernelGGL(k_bt_tfac, dim3(nblk), dim3(1024), 0, c->stream, tp, kTfSplit, T);
    }
    for (int b = nblk - 1; b >= 0; --b) {
      const int j0 = b * kBt, sp = (N - j0 + kBtSpan - 1) / kBtSpan,
                sg = (N - j0 + kBtGram - 1) / kBtGram;
      hipLaunchKernelGGL(k_bt_gram, dim3(nbt, sg), dim3(512), 0, c->stream, V, Uh, N, R, nb, j0,
                         part);
      hipLaunchKernelGGL(k_bt_apply, dim3(nbt, sp), dim3(256), 0, c->stream, V, T, part, sg, N, R,
                         nb, j0, Uh);
    }
    hipLaunchKernelGGL(k_bt_finish, dim3(gz), dim3(256), 0, c->stream, Uh, N, nb, U, ev, ex, lam);
    GW_CHECK_LAUNCH(c, "back transformation");
  }
  int hflag = 0;
  GW_HIP(c, hipMemcpyAsync(&hflag, flag, 4, hipMemcpyDeviceToHost, c->stream));
  GW_HIP(c, hipStreamSynchronize(c->stream));
  if (hflag) return fail(c, GW_EINVAL, "the eigen-decomposition of epst(0) did not converge");
  return GW_OK;
}

}  // namespace gw
