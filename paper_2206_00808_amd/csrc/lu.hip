// eps = I - diag(v) chi0 and its inverse in double (Sec. II, dielectric matrix;
// the Performance section names this inversion as a large part of Epsilon).
//
// Default path: on the static and imaginary-frequency axis chi0 is Hermitian
// negative semidefinite, so with S = diag(sqrt(v)) (v > 0)
//   eps = S (I - S chi0 S) S^-1 = S epst S^-1,  epst Hermitian positive definite
// (every eigenvalue >= 1).  epst is inverted in place by blocked Gauss-Jordan
// elimination without pivoting (stable for a positive-definite matrix), whose
// work is one rank-nb GEMM update of the whole matrix per block, and then
// eps^-1 = S epst^-1 S^-1.  Each diagonal pivot is checked to be real and
// positive (>= 1/2, since epst >= I); if any is not (or some v <= 0), the result
// is discarded and the general path below runs instead.
//
// General path: right-looking blocked LU with partial pivoting (PA = LU), every
// frequency in the same launches (grid.z / grid.y = frequency):
//   panel  : one workgroup per matrix factors the N x nb column panel
//            (pivot = largest |re|+|im|, lowest row on ties)
//   laswp  : the panel's row interchanges applied to the other columns
//   trsm   : U12 = L11^-1 A12
//   update : A22 -= L21 U12 on the FP64 matrix cores
// then eps^-1 = U^-1 L^-1 P by blocked forward/back substitution on P*I.
#include "common.h"
#include "gj.h"

#include <climits>

namespace gw {

constexpr int NB = 32;  // block width of the factorisation and the substitutions

__global__ void k_eps_build(const cpx<double>* __restrict__ chi, const double* __restrict__ v,
                            cpx<double>* __restrict__ A, int N) {
  const size_t nn = (size_t)N * N;
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nn) return;
  const size_t off = (size_t)blockIdx.y * nn + idx;
  const int i = (int)(idx / N), j = (int)(idx % N);
  const cpx<double> x = chi[off];
  A[off] = mk((i == j ? 1.0 : 0.0) - v[i] * x.x, -v[i] * x.y);
}

// 1 / p of a pivot whose square leaves the normal range (a subnormal square loses the
// pivot's digits and has no reciprocal): p is scaled by a power of two to order one first.
// The back substitution raises flag[1] at such a pivot, and the matrix is factored again
// with this inverse: any test in the panels' chain of columns cost 1.4% of them.
__device__ __forceinline__ cpx<double> scaled_inverse(cpx<double> p) {
  int e = 0;
  (void)frexp(fmax(fabs(p.x), fabs(p.y)), &e);
  const double x = ldexp(p.x, -e), y = ldexp(p.y, -e), den = x * x + y * y;
  return mk(ldexp(x / den, -e), ldexp(-y / den, -e));
}
__device__ __forceinline__ bool square_in_range(double abs1) {
  return abs1 > 1e-140 && abs1 < 1e140;
}

__global__ void __launch_bounds__(1024) k_lu_panel(cpx<double>* __restrict__ A, int N, int k,
                                                   int nbk, int* __restrict__ ipiv,
                                                   int* __restrict__ flag) {
  __shared__ double sv[1024];
  __shared__ int si[1024];
  __shared__ cpx<double> prow[NB];
  const int tid = threadIdx.x, nt = blockDim.x;
  A += (size_t)blockIdx.x * N * N;
  ipiv += (size_t)blockIdx.x * N;
  for (int jj = 0; jj < nbk; ++jj) {
    const int j = k + jj;
    double best = -1.0;
    int bi = N;
    for (int i = j + tid; i < N; i += nt) {
      const cpx<double> a = A[(size_t)i * N + j];
      const double m = fabs(a.x) + fabs(a.y);
      if (m > best) { best = m; bi = i; }
    }
    sv[tid] = best;
    si[tid] = bi;
    __syncthreads();
    for (int s = nt / 2; s > 0; s >>= 1) {
      if (tid < s) {
        const double o = sv[tid + s];
        const int oi = si[tid + s];
        if (o > sv[tid] || (o == sv[tid] && oi < si[tid])) { sv[tid] = o; si[tid] = oi; }
      }
      __syncthreads();
    }
    const double pm = sv[0];
    const int p = (si[0] < N) ? si[0] : j;  // no finite candidate: keep the diagonal
    if (tid == 0) {
      ipiv[j] = p;
      if (!(pm > 0.0)) flag[0] = 1;
    }
    if (p != j) {
      for (int c = tid; c < nbk; c += nt) {
        const cpx<double> t = A[(size_t)j * N + k + c];
        A[(size_t)j * N + k + c] = A[(size_t)p * N + k + c];
        A[(size_t)p * N + k + c] = t;
      }
    }
    __syncthreads();
    for (int c = tid; c < nbk; c += nt) prow[c] = A[(size_t)j * N + k + c];
    __syncthreads();
    if (pm > 0.0) {
      const cpx<double> piv = prow[jj];
      const double den = piv.x * piv.x + piv.y * piv.y;
      const cpx<double> inv =
          square_in_range(pm) ? mk(piv.x / den, -piv.y / den) : scaled_inverse(piv);
      for (int i = j + 1 + tid; i < N; i += nt) {
        cpx<double>* row = A + (size_t)i * N + k;
        const cpx<double> l = cmul(row[jj], inv);
        row[jj] = l;
        for (int c = jj + 1; c < nbk; ++c) row[c] = row[c] - cmul(l, prow[c]);
      }
    }
    __syncthreads();
  }
}

// The same factorisation with the panel in registers: a thread holds eight columns of
// up to R rows, and the panel is factored by sub-panels of eight.  Rows stay with
// their threads (only a row's position moves, so the choice and the order of the
// pivots are those of explicit interchanges); a column costs one barrier, because
// each wavefront publishes its candidate's position and its whole row before it and
// every thread picks the winner after it.  Sub-panels are left-looking: the eight
// columns take the earlier ones' L (kept in W by columns, so that a wavefront's rows
// are contiguous) times U (in LDS, solved by one wavefront) when they are loaded.  The
// finished panel is moved to the rows' final positions at the end.
//
// Bound: latency of the columns' chains; one workgroup per matrix.  A 32-column panel
// of up to 768 rows takes 101 us, of up to 512 rows 72 and of up to 256 rows 42 (mean
// over a 613-row factorisation; 265 us with the columns in global memory, two passes
// over them and 12 barriers per column).  eps^-1 of four 613-row matrices by LU alone:
// 7.73 ms before, 2.89 ms with these panels (5.36 -> 1.37 ms) and the four-lane
// triangular solves (1.50 -> 0.83 ms).
constexpr int SW = 8;           // sub-panel width
constexpr int kPanelT = 256;    // threads: one wavefront per SIMD, up to 12 rows each

// 1 / x for normal x: the hardware estimate and two Newton steps
__device__ __forceinline__ double rcp_newton(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// largest v of the wavefront, and the lowest position among the lanes that hold it
__device__ __forceinline__ int dpp16(int v, int step) {
  switch (step) {
    case 0: return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);   // lane ^ 1
    case 1: return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);   // lane ^ 2
    case 2: return __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true);  // mirror within 8
    default: return __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true); // mirror within 16
  }
}
__device__ __forceinline__ double dpp16(double v, int step) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp16((int)b, step), hi = dpp16((int)(b >> 32), step);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double readlane(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ void wave_best(double* v, int* pos) {
  double m = *v;
#pragma unroll
  for (int st = 0; st < 4; ++st) m = fmax(m, dpp16(m, st));
  m = fmax(fmax(readlane(m, 0), readlane(m, 16)), fmax(readlane(m, 32), readlane(m, 48)));
  int p = *v == m ? *pos : INT_MAX;
#pragma unroll
  for (int st = 0; st < 4; ++st) p = min(p, dpp16(p, st));
  p = min(min(__builtin_amdgcn_readlane(p, 0), __builtin_amdgcn_readlane(p, 16)),
          min(__builtin_amdgcn_readlane(p, 32), __builtin_amdgcn_readlane(p, 48)));
  *v = m;
  *pos = p;
}

template <int R>
__global__ void __launch_bounds__(kPanelT) k_lu_panel_reg(cpx<double>* __restrict__ A, int N, int k,
                                                          int nbk, int* __restrict__ ipiv,
                                                          int* __restrict__ flag,
                                                          cpx<double>* __restrict__ W) {
  constexpr int NW = kPanelT / 64;
  __shared__ cpx<double> slot[2][NW][SW];
  __shared__ double cv[2][NW];
  __shared__ int cp[2][NW];
  __shared__ cpx<double> P[NB][NB + 1];  // pivot rows: L left of the diagonal, U from it on
  __shared__ int prow[NB];               // their rows
  __shared__ int fin[kPanelT * R];       // final position of every row
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  A += (size_t)blockIdx.x * N * N;
  W += (size_t)blockIdx.x * N * NB;
  ipiv += (size_t)blockIdx.x * N;
  const int m = N - k;
  cpx<double> a[R][SW];
  int pos[R];
  bool act[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    pos[r] = k + tid + kPanelT * r;
    act[r] = tid + kPanelT * r < m;
  }
  for (int c0 = 0; c0 < nbk; c0 += SW) {
    const int w = min(SW, nbk - c0);
    bool had[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      had[r] = act[r];
      const cpx<double>* row = A + (size_t)(k + tid + kPanelT * r) * N + k + c0;
#pragma unroll
      for (int c = 0; c < SW; ++c) a[r][c] = act[r] && c < w ? row[c] : mk(0.0, 0.0);
    }
    if (c0) {
      // the pivot rows so far: their entries here, and the last sub-panel's L
      for (int e = tid; e < c0 * SW; e += kPanelT) {
        const int jj = e / SW, c = e % SW;
        P[jj][c0 + c] = c < w ? A[(size_t)(k + prow[jj]) * N + k + c0 + c] : mk(0.0, 0.0);
      }
      for (int e = tid; e < SW * (c0 - SW); e += kPanelT) {
        const int jj = c0 - SW + e / (c0 - SW), c = e % (c0 - SW);
        P[jj][c] = W[(size_t)c * N + prow[jj]];
      }
      __syncthreads();
      if (wave == 0) {  // U = L^-1 times them: lane = (row of the block, column)
        const int jr = lane / SW, c = c0 + lane % SW;
        for (int b = 0; b < c0; b += SW) {
          cpx<double> x = P[b + jr][c];
#pragma unroll 8
          for (int t = 0; t < b; ++t) x = x - cmul(P[b + jr][t], P[t][c]);
#pragma unroll
          for (int t = 0; t < SW - 1; ++t) {
            const cpx<double> y = mk(__shfl(x.x, t * SW + lane % SW), __shfl(x.y, t * SW + lane % SW));
            if (jr > t) x = x - cmul(P[b + jr][b + t], y);
          }
          P[b + jr][c] = x;
          __builtin_amdgcn_wave_barrier();
        }
      }
      __syncthreads();
      for (int e = tid; e < c0 * SW; e += kPanelT) {
        const int jj = e / SW, c = e % SW;
        W[(size_t)(c0 + c) * N + prow[jj]] = P[jj][c0 + c];
      }
      // rows no longer active take zeros: every row shares the reads of U
      constexpr int U = R <= 2 ? 8 : R <= 4 ? 4 : 2;  // columns of L in flight
      for (int j0 = 0; j0 < c0; j0 += U) {
        cpx<double> lv[U][R];
#pragma unroll
        for (int x = 0; x < U; ++x)
#pragma unroll
          for (int r = 0; r < R; ++r)
            lv[x][r] = act[r] ? W[(size_t)(j0 + x) * N + tid + kPanelT * r] : mk(0.0, 0.0);
#pragma unroll
        for (int x = 0; x < U; ++x) {
          cpx<double> u[SW];
#pragma unroll
          for (int c = 0; c < SW; ++c) u[c] = P[j0 + x][c0 + c];
#pragma unroll
          for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < SW; ++c) a[r][c] = a[r][c] - cmul(lv[x][r], u[c]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < SW; ++q) {
      if (q >= w) break;
      const int jj = c0 + q, j = k + jj, par = q & 1;
      double bv = -1.0;
      int bp = INT_MAX;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double v = fabs(a[r][q].x) + fabs(a[r][q].y);
        if (act[r] && (v > bv || (v == bv && pos[r] < bp))) { bv = v; bp = pos[r]; }
      }
      wave_best(&bv, &bp);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (act[r] && pos[r] == bp) {
#pragma unroll
          for (int c = 0; c < SW; ++c) slot[par][wave][c] = a[r][c];
        }
      if (lane == 0) {
        cv[par][wave] = bv;
        cp[par][wave] = bp;
      }
      __syncthreads();
      int bw = 0;
      bv = cv[par][0];
      bp = cp[par][0];
#pragma unroll
      for (int x = 1; x < NW; ++x) {
        const double v = cv[par][x];
        const int o = cp[par][x];
        if (v > bv || (v == bv && o < bp)) { bv = v; bp = o; bw = x; }
      }
      const bool none = !(bv >= 0.0);  // no comparable candidate: keep the diagonal
      const int p = none ? j : bp;
      if (tid == 0) {
        ipiv[j] = p;
        if (!(bv > 0.0)) flag[0] = 1;
      }
      cpx<double> u[SW];
#pragma unroll
      for (int c = 0; c < SW; ++c) u[c] = slot[par][bw][c];
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (act[r]) {
          if (pos[r] == p) {
            act[r] = false;
            pos[r] = j;
            prow[jj] = tid + kPanelT * r;
#pragma unroll
            for (int c = 0; c < SW; ++c) P[jj][c0 + c] = a[r][c];
          } else if (pos[r] == j) {
            pos[r] = p;
          }
        }
      if (bv > 0.0) {
        const double den = rcp_newton(u[q].x * u[q].x + u[q].y * u[q].y);
        const cpx<double> inv = mk(u[q].x * den, -u[q].y * den);
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (act[r]) {
            const cpx<double> l = cmul(a[r][q], inv);
            a[r][q] = l;
#pragma unroll
            for (int c = q + 1; c < SW; ++c) a[r][c] = a[r][c] - cmul(l, u[c]);
          }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (had[r]) {
        cpx<double>* l = W + (size_t)c0 * N + tid + kPanelT * r;
#pragma unroll
        for (int c = 0; c < SW; ++c) l[(size_t)c * N] = a[r][c];
      }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (tid + kPanelT * r < m) fin[tid + kPanelT * r] = pos[r];
  __syncthreads();
#pragma unroll 4
  for (int e = tid; e < m * NB; e += kPanelT) {
    const int i = e / NB, c = e % NB;
    if (c < nbk) A[(size_t)fin[i] * N + k + c] = W[(size_t)c * N + i];
  }
}

__global__ void k_lu_laswp(cpx<double>* __restrict__ A, int N, int k, int nbk,
                           const int* __restrict__ ipiv) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= N || (c >= k && c < k + nbk)) return;
  A += (size_t)blockIdx.y * N * N;
  ipiv += (size_t)blockIdx.y * N;
  for (int s = k; s < k + nbk; ++s) {
    const int p = ipiv[s];
    if (p != s) {
      const cpx<double> t = A[(size_t)s * N + c];
      A[(size_t)s * N + c] = A[(size_t)p * N + c];
      A[(size_t)p * N + c] = t;
    }
  }
}

// Solve T X = B in place on rows kb..kb+nbk of X for columns c0..c0+ncols, where
// T is the nbk x nbk diagonal block of the LU factors: unit lower (UPPER=false)
// or non-unit upper (UPPER=true).  Four neighbouring lanes share a right-hand side,
// lane l holding rows 4 r + l: each solved entry is passed inside the four and taken
// out of all later rows at once.  Bound: latency of 32 dependent entries; 613 columns of
// four matrices: 11 us lower, 13 upper (20-31 with one lane per column).
__device__ __forceinline__ double quad_get(double v, int from) {
  const long long b = __double_as_longlong(v);
  int lo = (int)b, hi = (int)(b >> 32);
  switch (from) {
    case 0: lo = __builtin_amdgcn_mov_dpp(lo, 0x00, 0xf, 0xf, true);
            hi = __builtin_amdgcn_mov_dpp(hi, 0x00, 0xf, 0xf, true); break;
    case 1: lo = __builtin_amdgcn_mov_dpp(lo, 0x55, 0xf, 0xf, true);
            hi = __builtin_amdgcn_mov_dpp(hi, 0x55, 0xf, 0xf, true); break;
    case 2: lo = __builtin_amdgcn_mov_dpp(lo, 0xAA, 0xf, 0xf, true);
            hi = __builtin_amdgcn_mov_dpp(hi, 0xAA, 0xf, 0xf, true); break;
    default: lo = __builtin_amdgcn_mov_dpp(lo, 0xFF, 0xf, 0xf, true);
             hi = __builtin_amdgcn_mov_dpp(hi, 0xFF, 0xf, 0xf, true);
  }
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <bool UPPER, bool SCALED>
__global__ void __launch_bounds__(64) k_trsm_block(const cpx<double>* __restrict__ LU, int N,
                                                   int kb, int nbk, cpx<double>* __restrict__ X,
                                                   int c0, int ncols, int* __restrict__ flag) {
  __shared__ cpx<double> T[NB][NB + 1];  // T[column][row]: the rows a column is taken out of
  __shared__ cpx<double> dinv[NB];
  LU += (size_t)blockIdx.y * N * N;
  X += (size_t)blockIdx.y * N * N;
  const int lane = threadIdx.x, l4 = lane & 3, cidx = blockIdx.x * 16 + (lane >> 2);
  const bool live = cidx < ncols;
  cpx<double>* xc = X + (size_t)kb * N + c0 + (live ? cidx : 0);
  cpx<double> x[NB / 4];
#pragma unroll
  for (int r = 0; r < NB / 4; ++r)
    x[r] = 4 * r + l4 < nbk ? xc[(size_t)(4 * r + l4) * N] : mk<double>(0, 0);
#pragma unroll 4
  for (int e = lane; e < NB * NB; e += 64) {
    const int r = e / NB, cc = e % NB;
    const bool in = r < nbk && cc < nbk;
    const cpx<double> t = in ? LU[(size_t)(kb + r) * N + kb + cc] : mk(0.0, 0.0);
    T[cc][r] = (UPPER ? r < cc : r > cc) ? t : mk(0.0, 0.0);
    if (UPPER && r == cc) {
      const double den = t.x * t.x + t.y * t.y;
      cpx<double> inv = mk(t.x / den, -t.y / den);
      const double abs1 = fabs(t.x) + fabs(t.y);
      if (in && !square_in_range(abs1)) {
        if (SCALED) inv = scaled_inverse(t);
        else if (abs1 != 0.0) flag[1] = 1;
      }
      dinv[r] = in ? inv : mk(0.0, 0.0);
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NB; ++s) {
    const int t = UPPER ? NB - 1 - s : s, rt = t / 4;
    cpx<double> y = mk(quad_get(x[rt].x, t & 3), quad_get(x[rt].y, t & 3));
    if (UPPER) {
      y = cmul(y, dinv[t]);
      if (l4 == (t & 3)) x[rt] = y;
    }
#pragma unroll
    for (int r = UPPER ? 0 : rt; r < (UPPER ? rt + 1 : NB / 4); ++r)
      x[r] = x[r] - cmul(T[t][4 * r + l4], y);
  }
#pragma unroll
  for (int r = 0; r < NB / 4; ++r)
    if (live && 4 * r + l4 < nbk) xc[(size_t)(4 * r + l4) * N] = x[r];
}

// Row s of P*I is e_perm[s], perm = identity after the interchanges s <-> ipiv[s].
__global__ void __launch_bounds__(256) k_perm_build(const int* __restrict__ ipiv, int N,
                                                    int* __restrict__ perm) {
  extern __shared__ int sp[];
  const int f = blockIdx.x;
  ipiv += (size_t)f * N;
  perm += (size_t)f * N;
  for (int i = threadIdx.x; i < N; i += blockDim.x) sp[i] = i;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int s = 0; s < N; ++s) {
      const int p = ipiv[s];
      const int t = sp[s];
      sp[s] = sp[p];
      sp[p] = t;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += blockDim.x) perm[i] = sp[i];
}

__global__ void k_perm_identity(const int* __restrict__ perm, int N, cpx<double>* __restrict__ Y) {
  const size_t nn = (size_t)N * N;
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nn) return;
  const int s = (int)(e / N), j = (int)(e % N);
  Y[(size_t)blockIdx.y * nn + e] = mk(j == perm[(size_t)blockIdx.y * N + s] ? 1.0 : 0.0, 0.0);
}


// ---------------------------------------------------------------- Gauss-Jordan path
__global__ void k_fill_int(int* p, int n, int v) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = v;
}


// epst = I - S chi0 S with S = diag(sqrt(v)), one 32x32 tile per workgroup
// (grid: tiles x tiles x nfreq). flag[1] = 1 if some v <= 0 or non-finite;
// flag[4] = 1 if some chi0 entry is not finite;
// flag[5] = 1 if chi0 is not exactly Hermitian;
// flag[3] = 1 if chi0 is not Hermitian: |chi_ij - conj(chi_ji)| above
// kHermRel (|chi_ij| + |chi_ji|) for some pair, checked against the mirror
// tile staged through LDS. The Gauss-Jordan pivot test alone cannot tell a
// Hermitian positive-definite epst from a non-Hermitian one whose pivots
// happen to look the same.
constexpr double kHermRel = 1e-12;
constexpr int ET = 32;
__global__ void __launch_bounds__(256) k_epst_build(const cpx<double>* __restrict__ chi,
                                                    const double* __restrict__ v,
                                                    cpx<double>* __restrict__ A, int N,
                                                    int* __restrict__ flag) {
  __shared__ cpx<double> mir[ET][ET + 1];
  const size_t nn = (size_t)N * N;
  const int ti = blockIdx.y, tj = blockIdx.x;
  chi += (size_t)blockIdx.z * nn;
  A += (size_t)blockIdx.z * nn;
  const int c = threadIdx.x % ET, r0 = threadIdx.x / ET;  // 8 rows per pass
  // mirror tile (tj, ti), read row-wise and stored transposed
  for (int r = r0; r < ET; r += 256 / ET) {
    const int i = tj * ET + r, j = ti * ET + c;
    if (i < N && j < N) mir[c][r] = chi[(size_t)i * N + j];
  }
  __syncthreads();
  bool bad = false, nonfinite = false, inexact = false;
  for (int r = r0; r < ET; r += 256 / ET) {
    const int i = ti * ET + r, j = tj * ET + c;
    if (i >= N || j >= N) continue;
    const double vi = v[i], vj = v[j];
    if (j == 0 && (!(vi > 0.0) || !(vi < INFINITY))) flag[1] = 1;
    const cpx<double> x = chi[(size_t)i * N + j];
    const cpx<double> y = mir[r][c];  // chi[j][i]
    const double dr = x.x - y.x, di = x.y + y.y;
    const double lim = kHermRel * (fabs(x.x) + fabs(x.y) + fabs(y.x) + fabs(y.y));
    inexact = inexact || !(dr == 0.0 && di == 0.0);
    nonfinite = nonfinite || !(fabs(x.x) < INFINITY && fabs(x.y) < INFINITY);
    bad = bad || !(fabs(dr) <= lim && fabs(di) <= lim);
    const double s = sqrt(vi) * sqrt(vj);
    A[(size_t)i * N + j] = mk((i == j ? 1.0 : 0.0) - s * x.x, -s * x.y);
  }
  if (bad) flag[3] = 1;
  if (nonfinite) flag[4] = 1;
  if (inexact) flag[5] = 1;
}

// ---------------------------------------------------------------- consumers of eps^-1
// W[f][G][G'] = eps^-1[f][G][G'] v(q+G')
__global__ void k_screened_w(const cpx<double>* __restrict__ einv, const double* __restrict__ v,
                             int N, cpx<double>* __restrict__ w) {
  const size_t nn = (size_t)N * N;
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nn) return;
  const size_t off = (size_t)blockIdx.y * nn + e;
  w[off] = scal(einv[off], v[e % N]);
}

// X[p][G] = conj(M[p][G]) in double (the left factor of the SX quadratic form)
template <typename Tin>
__global__ void k_conj_widen(const cpx<Tin>* __restrict__ m, size_t n, cpx<double>* __restrict__ x) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const cpx<Tin> a = m[e];
  x[e] = mk((double)a.x, -(double)a.y);
}

// sigma[n] += -pref sum_{n''} sum_G' U[(n'',n)][G'] v(G') M[(n'',n)][G'], U = conj(M) eps^-1;
// one workgroup per band n, the occupied bands and G' summed in a fixed order
template <typename Tin>
__global__ void __launch_bounds__(256) k_sx_reduce(const cpx<double>* __restrict__ U,
                                                   const cpx<Tin>* __restrict__ m,
                                                   const double* __restrict__ v, int nocc,
                                                   int nband, int N, double pref,
                                                   cpx<double>* __restrict__ sigma) {
  __shared__ double sr[256], si[256];
  const int n = blockIdx.x;
  double ar = 0.0, ai = 0.0;
  for (int o = 0; o < nocc; ++o) {
    const size_t row = ((size_t)o * nband + n) * N;
    for (int g = threadIdx.x; g < N; g += blockDim.x) {
      const cpx<double> u = U[row + g];
      const cpx<Tin> b = m[row + g];
      const double br = v[g] * (double)b.x, bi = v[g] * (double)b.y;
      ar += u.x * br - u.y * bi;
      ai += u.x * bi + u.y * br;
    }
  }
  sr[threadIdx.x] = ar;
  si[threadIdx.x] = ai;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sr[threadIdx.x] += sr[threadIdx.x + s];
      si[threadIdx.x] += si[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) sigma[n] = mk(sigma[n].x - pref * sr[0], sigma[n].y - pref * si[0]);
}

gw_status screened_w(gw_ctx* c, int N, int nfreq, const double* epsinv, const double* vcoul,
                     double* w) {
  const size_t nn = (size_t)N * N;
  ProfScope ps(c, "screened_w");
  hipLaunchKernelGGL(k_screened_w, dim3((unsigned)((nn + 255) / 256), nfreq), dim3(256), 0,
                     c->stream, reinterpret_cast<const cpx<double>*>(epsinv), vcoul, N,
                     reinterpret_cast<cpx<double>*>(w));
  GW_CHECK_LAUNCH(c, "k_screened_w");
  return GW_OK;
}

gw_status sigma_sx_static(gw_ctx* c, int nocc, int nband, int N, const void* mtxel, gw_dtype dt,
                          const double* epsinv, const double* vcoul, double prefactor,
                          double* sigma) {
  const int P = nocc * nband;
  const size_t np = (size_t)P * N;
  gw_status st = ws_begin(c, 2 * align_up(np * 16));
  if (st != GW_OK) return st;
  cpx<double>* X = static_cast<cpx<double>*>(ws_take(c, np * 16));
  double* U = static_cast<double*>(ws_take(c, np * 16));
  {
    ProfScope ps(c, "sx_conj");
    if (dt == GW_C128)
      hipLaunchKernelGGL(k_conj_widen<double>, dim3((unsigned)((np + 255) / 256)), dim3(256), 0,
                         c->stream, static_cast<const cpx<double>*>(mtxel), np, X);
    else
      hipLaunchKernelGGL(k_conj_widen<float>, dim3((unsigned)((np + 255) / 256)), dim3(256), 0,
                         c->stream, static_cast<const cpx<float>*>(mtxel), np, X);
    GW_CHECK_LAUNCH(c, "k_conj_widen");
  }
  // U = conj(M) eps^-1 on the matrix cores
  st = zgemm_nn(c, P, N, N, 1.0, reinterpret_cast<const double*>(X), 0, N, 0, epsinv, 0, N, 0, U,
                0, N, 0, 1, np, (size_t)N * N, np, 0.0);
  if (st != GW_OK) return st;
  ProfScope ps(c, "sx_reduce");
  if (dt == GW_C128)
    hipLaunchKernelGGL(k_sx_reduce<double>, dim3(nband), dim3(256), 0, c->stream,
                       reinterpret_cast<const cpx<double>*>(U),
                       static_cast<const cpx<double>*>(mtxel), vcoul, nocc, nband, N, prefactor,
                       reinterpret_cast<cpx<double>*>(sigma));
  else
    hipLaunchKernelGGL(k_sx_reduce<float>, dim3(nband), dim3(256), 0, c->stream,
                       reinterpret_cast<const cpx<double>*>(U),
                       static_cast<const cpx<float>*>(mtxel), vcoul, nocc, nband, N, prefactor,
                       reinterpret_cast<cpx<double>*>(sigma));
  GW_CHECK_LAUNCH(c, "k_sx_reduce");
  return GW_OK;
}

// one factorisation and its substitutions; *again: a pivot's square left the normal range
// and `scaled` was not set
static gw_status epsinv_pivoted(gw_ctx* c, int N, int nfreq, const double* chi0,
                                const double* vcoul, double* epsinv, bool scaled, bool* again) {
  const size_t nn = (size_t)N * N;
  const size_t bytes = align_up(nfreq * nn * 16) + 2 * align_up((size_t)nfreq * N * 4) +
                       align_up((size_t)nfreq * N * NB * 16);
  gw_status st = ws_begin(c, bytes);
  if (st != GW_OK) return st;
  cpx<double>* LU = static_cast<cpx<double>*>(ws_take(c, nfreq * nn * 16));
  int* ipiv = static_cast<int*>(ws_take(c, (size_t)nfreq * N * 4));
  int* perm = static_cast<int*>(ws_take(c, (size_t)nfreq * N * 4));
  cpx<double>* W = static_cast<cpx<double>*>(ws_take(c, (size_t)nfreq * N * NB * 16));
  cpx<double>* Y = reinterpret_cast<cpx<double>*>(epsinv);
  {
    ProfScope ps(c, "flags_clear");
    hipLaunchKernelGGL(k_fill_int, dim3(1), dim3(64), 0, c->stream, c->d_flag, 16, 0);
    GW_CHECK_LAUNCH(c, "k_fill_int");
  }
  {
    ProfScope ps(c, "eps_build");
    hipLaunchKernelGGL(k_eps_build, dim3((unsigned)((nn + 255) / 256), nfreq), dim3(256), 0,
                       c->stream, reinterpret_cast<const cpx<double>*>(chi0), vcoul, LU, N);
    GW_CHECK_LAUNCH(c, "k_eps_build");
  }
  const long long s2 = (long long)nn;  // batch stride in complex elements
  const size_t ext = (size_t)nfreq * nn;  // complex elements in LU and in epsinv
  double* LUd = reinterpret_cast<double*>(LU);
  for (int k = 0; k < N; k += NB) {
    const int nbk = std::min(NB, N - k);
    {
      ProfScope ps(c, "lu_panel");
      // rows per thread that fit the registers; more rows stay in global memory
      switch (scaled ? 0 : (N - k + kPanelT - 1) / kPanelT) {
#define GW_PANEL(R)                                                                          \
  case R:                                                                                    \
    hipLaunchKernelGGL(k_lu_panel_reg<R>, dim3(nfreq), dim3(kPanelT), 0, c->stream, LU, N, k, \
                       nbk, ipiv, c->d_flag, W);                                             \
    break;
        GW_PANEL(1) GW_PANEL(2) GW_PANEL(3) GW_PANEL(4) GW_PANEL(5) GW_PANEL(6) GW_PANEL(7)
        GW_PANEL(8) GW_PANEL(9) GW_PANEL(10) GW_PANEL(11) GW_PANEL(12)
#undef GW_PANEL
        default:
          hipLaunchKernelGGL(k_lu_panel, dim3(nfreq), dim3(1024), 0, c->stream, LU, N, k, nbk,
                             ipiv, c->d_flag);
      }
      GW_CHECK_LAUNCH(c, "k_lu_panel");
    }
    {
      ProfScope ps(c, "lu_laswp");
      hipLaunchKernelGGL(k_lu_laswp, dim3((N + 255) / 256, nfreq), dim3(256), 0, c->stream, LU,
                         N, k, nbk, ipiv);
      GW_CHECK_LAUNCH(c, "k_lu_laswp");
    }
    const int rest = N - k - nbk;
    if (rest > 0) {
      {
        ProfScope ps(c, "lu_trsm");
        hipLaunchKernelGGL((k_trsm_block<false, false>), dim3((rest + 15) / 16, nfreq), dim3(64), 0,
                           c->stream, LU, N, k, nbk, LU, k + nbk, rest, c->d_flag);
        GW_CHECK_LAUNCH(c, "k_trsm_block");
      }
      st = zgemm_nn(c, rest, rest, nbk, -1.0, LUd, (size_t)(k + nbk) * N + k, N, s2, LUd,
                    (size_t)k * N + k + nbk, N, s2, LUd, (size_t)(k + nbk) * N + k + nbk, N, s2,
                    nfreq, ext, ext, ext);
      if (st != GW_OK) return st;
    }
  }
  {
    ProfScope ps(c, "inv_perm");
    hipLaunchKernelGGL(k_perm_build, dim3(nfreq), dim3(256), (size_t)N * 4, c->stream, ipiv, N,
                       perm);
    GW_CHECK_LAUNCH(c, "k_perm_build");
    hipLaunchKernelGGL(k_perm_identity, dim3((unsigned)((nn + 255) / 256), nfreq), dim3(256), 0,
                       c->stream, perm, N, Y);
    GW_CHECK_LAUNCH(c, "k_perm_identity");
  }
  // forward: L Y = P I
  for (int kb = 0; kb < N; kb += NB) {
    const int nbk = std::min(NB, N - kb);
    {
      ProfScope ps(c, "inv_trsm_lower");
      hipLaunchKernelGGL((k_trsm_block<false, false>), dim3((N + 15) / 16, nfreq), dim3(64), 0,
                         c->stream, LU, N, kb, nbk, Y, 0, N, c->d_flag);
      GW_CHECK_LAUNCH(c, "k_trsm_block");
    }
    const int below = N - kb - nbk;
    if (below > 0) {
      st = zgemm_nn(c, below, N, nbk, -1.0, LUd, (size_t)(kb + nbk) * N + kb, N, s2, epsinv,
                    (size_t)kb * N, N, s2, epsinv, (size_t)(kb + nbk) * N, N, s2, nfreq, ext, ext,
                    ext);
      if (st != GW_OK) return st;
    }
  }
  // back: U X = Y
  const int nblk = (N + NB - 1) / NB;
  for (int b = nblk - 1; b >= 0; --b) {
    const int kb = b * NB;
    const int nbk = std::min(NB, N - kb);
    {
      ProfScope ps(c, "inv_trsm_upper");
      auto* solve = scaled ? &k_trsm_block<true, true> : &k_trsm_block<true, false>;
      hipLaunchKernelGGL(solve, dim3((N + 15) / 16, nfreq), dim3(64), 0, c->stream, LU, N, kb, nbk,
                         Y, 0, N, c->d_flag);
      GW_CHECK_LAUNCH(c, "k_trsm_block");
    }
    if (kb > 0) {
      st = zgemm_nn(c, kb, N, nbk, -1.0, LUd, (size_t)kb, N, s2, epsinv, (size_t)kb * N, N, s2,
                    epsinv, 0, N, s2, nfreq, ext, ext, ext);
      if (st != GW_OK) return st;
    }
  }
  int flag[2] = {0, 0};
  GW_HIP(c, hipMemcpyAsync(flag, c->d_flag, sizeof flag, hipMemcpyDeviceToHost, c->stream));
  GW_HIP(c, hipStreamSynchronize(c->stream));
  // what follows such a pivot is not finite, so it comes before the zero pivots
  *again = flag[1] && !scaled;
  if (flag[0] && !*again)
    return fail(c, GW_ESINGULAR, "eps has a zero pivot (singular dielectric matrix)");
  return GW_OK;
}

gw_status epsinv_pivoted_one(gw_ctx* c, int N, int nfreq, const double* chi0,
                             const double* vcoul, double* epsinv) {
  bool again = false;
  gw_status st = epsinv_pivoted(c, N, nfreq, chi0, vcoul, epsinv, false, &again);
  if (st == GW_OK && again) st = epsinv_pivoted(c, N, nfreq, chi0, vcoul, epsinv, true, &again);
  return st;
}

static gw_status epsinv_gauss_jordan(gw_ctx* c, int N, int nfreq, const double* chi0,
                                     const double* vcoul, double* epsinv) {
  const size_t nR = (size_t)nfreq * GB * N, nC = (size_t)nfreq * N * GB, nD = (size_t)nfreq * GB * GB;
  gw_status st = ws_begin(c, 2 * align_up(nR * 16) + align_up(nC * 16) + 3 * align_up(nD * 16));
  if (st != GW_OK) return st;
  GjStrided g;
  g.m.A = reinterpret_cast<cpx<double>*>(epsinv);
  g.m.chi = reinterpret_cast<const cpx<double>*>(chi0);
  g.m.v = vcoul;
  g.m.R0 = static_cast<cpx<double>*>(ws_take(c, nR * 16));
  g.m.R1 = static_cast<cpx<double>*>(ws_take(c, nR * 16));
  g.m.Cb = static_cast<cpx<double>*>(ws_take(c, nC * 16));
  g.m.D0 = static_cast<cpx<double>*>(ws_take(c, nD * 16));
  g.m.D1 = static_cast<cpx<double>*>(ws_take(c, nD * 16));
  g.m.Dn = static_cast<cpx<double>*>(ws_take(c, nD * 16));
  g.m.bad = c->d_flag + 2;
  g.m.full = c->d_flag + 5;
  g.m.N = N;
  g.m.pad = 0;
  {
    ProfScope ps(c, "flags_clear");
    hipLaunchKernelGGL(k_fill_int, dim3(1), dim3(64), 0, c->stream, c->d_flag, 16, 0);
    GW_CHECK_LAUNCH(c, "k_fill_int");
  }
  {
    ProfScope ps(c, "eps_build");
    const unsigned nt = (unsigned)((N + ET - 1) / ET);
    hipLaunchKernelGGL(k_epst_build, dim3(nt, nt, nfreq), dim3(256), 0, c->stream,
                       g.m.chi, vcoul, g.m.A, N, c->d_flag);
    GW_CHECK_LAUNCH(c, "k_epst_build");
  }
  return gj_steps(c, g, nfreq, N, "gj_diag", "gj_small", "gj_update", "eps_unscale");
}

// rmax[f] = max_ij |R_f[i][j] - delta_ij| (|re| + |im|), one workgroup per
// frequency; a non-finite entry makes the result non-finite
__global__ void __launch_bounds__(1024) k_resid_max(const cpx<double>* __restrict__ R, int N,
                                                    double* __restrict__ rmax) {
  __shared__ double sm[1024];
  const size_t nn = (size_t)N * N;
  R += (size_t)blockIdx.x * nn;
  double m = 0.0;
  for (size_t e = threadIdx.x; e < nn; e += blockDim.x) {
    const int i = (int)(e / N), j = (int)(e % N);
    const cpx<double> r = R[e];
    const double a = fabs(r.x - (i == j ? 1.0 : 0.0)) + fabs(r.y);
    m = (a > m || a != a) ? a : m;
  }
  sm[threadIdx.x] = m;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      const double o = sm[threadIdx.x + s];
      if (o > sm[threadIdx.x] || o != o) sm[threadIdx.x] = o;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) rmax[blockIdx.x] = sm[0];
}

// Whether X solves eps X = I for every frequency to max_ij |(eps X - I)_ij| <=
// kVerifyRel / N, with eps = I - diag(v) chi0 formed again. Since X - eps^-1 =
// eps^-1 (eps X - I), that bounds the relative error of X in the infinity norm
// by N max_ij |.| <= kVerifyRel.
constexpr double kVerifyRel = 1e-10;
static gw_status epsinv_verified(gw_ctx* c, int N, int nfreq, const double* chi0,
                                 const double* vcoul, const double* X, bool* ok) {
  const size_t nn = (size_t)N * N, ext = (size_t)nfreq * nn;
  gw_status st = ws_begin(c, 2 * align_up(ext * 16) + align_up((size_t)nfreq * 8));
  if (st != GW_OK) return st;
  cpx<double>* E = static_cast<cpx<double>*>(ws_take(c, ext * 16));
  double* R = static_cast<double*>(ws_take(c, ext * 16));
  double* d_rmax = static_cast<double*>(ws_take(c, (size_t)nfreq * 8));
  {
    ProfScope ps(c, "eps_build");
    hipLaunchKernelGGL(k_eps_build, dim3((unsigned)((nn + 255) / 256), nfreq), dim3(256), 0,
                       c->stream, reinterpret_cast<const cpx<double>*>(chi0), vcoul, E, N);
    GW_CHECK_LAUNCH(c, "k_eps_build");
  }
  st = zgemm_nn(c, N, N, N, 1.0, reinterpret_cast<const double*>(E), 0, N, (long long)nn, X, 0, N,
                (long long)nn, R, 0, N, (long long)nn, nfreq, ext, ext, ext, 0.0);
  if (st != GW_OK) return st;
  {
    ProfScope ps(c, "eps_verify");
    hipLaunchKernelGGL(k_resid_max, dim3(nfreq), dim3(1024), 0, c->stream,
                       reinterpret_cast<const cpx<double>*>(R), N, d_rmax);
    GW_CHECK_LAUNCH(c, "k_resid_max");
  }
  std::vector<double> rmax(nfreq);
  GW_HIP(c, hipMemcpyAsync(rmax.data(), d_rmax, (size_t)nfreq * 8, hipMemcpyDeviceToHost,
                           c->stream));
  GW_HIP(c, hipStreamSynchronize(c->stream));
  *ok = true;
  for (double r : rmax) *ok = *ok && r <= kVerifyRel / N;
  return GW_OK;
}

gw_status epsinv_run(gw_ctx* c, int N, int nfreq, const double* chi0, const double* vcoul,
                     double* epsinv) {
  gw_status st = epsinv_gauss_jordan(c, N, nfreq, chi0, vcoul, epsinv);
  if (st != GW_OK) return st;
  int flags[5] = {0, 0, 0, 0, 0};
  GW_HIP(c, hipMemcpyAsync(flags, c->d_flag, sizeof flags, hipMemcpyDeviceToHost, c->stream));
  GW_HIP(c, hipStreamSynchronize(c->stream));
  if (flags[4]) return fail(c, GW_EINVAL, "chi0 holds a non-finite entry");
  // some v <= 0: the symmetric form eps~ does not exist; general LU
  if (flags[1]) return epsinv_pivoted_one(c, N, nfreq, chi0, vcoul, epsinv);
  if (!flags[2] && !flags[3]) return GW_OK;
  // chi0 not Hermitian (as on the real frequency axis), or a pivot not of the
  // Hermitian positive-definite kind: Gauss-Jordan without pivoting carries no
  // stability guarantee there, so its result is kept only if it solves
  // eps X = I to within kVerifyRel / N per entry; otherwise general LU with
  // partial pivoting
  bool ok = false;
  if ((st = epsinv_verified(c, N, nfreq, chi0, vcoul, epsinv, &ok)) != GW_OK) return st;
  if (ok) return GW_OK;
  return epsinv_pivoted_one(c, N, nfreq, chi0, vcoul, epsinv);
}

}  // namespace gw
