// Blocked Gauss-Jordan inversion of eps~ = I - S chi0 S, several matrices in the same
// launches: one size and a stride (one call's frequencies) or a table of matrices of
// different sizes (a plan's).
//
// Step K of 64 rows is two launches:
//   - k_gj_panel, one workgroup per 64 columns: the column panel Cb = A[:, K] and the row
//     panel R = Dinv A[K, :]; R[:, K] = I + Dinv, so that A - Cb R leaves -Cb Dinv in the
//     column block, its Gauss-Jordan value.  The block row of the step before takes its
//     value here (R of that step, Dinv in its columns);
//   - k_gj_update: A -= Cb R, and on its first workgroups the next diagonal block and its
//     inverse.  The block row K is left out: the next step rewrites it.
//
// A matrix that is exactly Hermitian keeps only its lower blocks.  Blocks whose rows and
// columns are both finished, or both not, are Hermitian; A[finished, unfinished] is minus
// the conjugate transpose of A[unfinished, finished].  So the panels are read from the
// lower blocks, half the update's tiles are left out, and k_gj_final writes the upper half
// as the conjugate of the lower.  Nine matrices of 1000 rows: 1476 us (updates 65 us,
// panels 18), 2156 with every block updated (109 us) and the panels in two launches (20).
// A matrix that is not exactly Hermitian (m.full) takes every block, in the same launches.
#pragma once

#include "tiles.h"

namespace gw {

constexpr int GB = 64;  // Gauss-Jordan block width

struct GjM {
  cpx<double>* A;          // eps~ in place, then eps^-1 (the caller's epsinv slice)
  const cpx<double>* chi;  // chi0 slice
  const double* v;         // v(q+G)
  cpx<double>*R0, *R1;     // [GB][N], by step parity
  cpx<double>* Cb;         // [N][GB]
  cpx<double>*D0, *D1;     // [GB][GB], the inverse of a step's diagonal block, by parity
  cpx<double>* Dn;         // [GB][GB], the next diagonal block
  int* bad;                // set by v <= 0 or a pivot that is not real and >= 1/2
  int* full;               // set where chi0 is not exactly Hermitian
  int N, pad;
  __device__ __forceinline__ cpx<double>* r(int s) const { return s & 1 ? R1 : R0; }
  __device__ __forceinline__ cpx<double>* d(int s) const { return s & 1 ? D1 : D0; }
};

// matrix f of a table, or of equal matrices one after another
struct GjTable {
  const GjM* ms;
  __device__ __forceinline__ GjM operator()(int f) const { return ms[f]; }
};
struct GjStrided {
  GjM m;
  __device__ __forceinline__ GjM operator()(int f) const {
    GjM r = m;
    const size_t nn = (size_t)m.N * m.N, p = (size_t)m.N * GB, d = GB * GB;
    r.A += f * nn;
    r.chi += f * nn;
    r.R0 += f * p;
    r.R1 += f * p;
    r.Cb += f * p;
    r.D0 += f * d;
    r.D1 += f * d;
    r.Dn += f * d;
    return r;
  }
};

// ---- 64 x 64 inverse
__device__ __forceinline__ double gj_lane(double x, int lane) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// lane T of each row of 16 lanes, in all of them
template <int T>
__device__ __forceinline__ double gj_row(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x150 + T, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x150 + T, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// What the pivots were: bad() where one was not real and >= 1/2 (or not finite), which I
// minus a negative semidefinite matrix cannot give.
struct GjPivots {
  double least = INFINITY, skew = -INFINITY, finite = 0.0;
  __device__ __forceinline__ void add(cpx<double> p) {
    least = fmin(least, p.x);
    skew = fmax(skew, fma(-0.25, p.x, fabs(p.y)));
    finite = fma(p.x, 0.0, fma(p.y, 0.0, finite));
  }
  __device__ __forceinline__ bool bad() const {
    return !(least >= 0.5 && skew <= 0.0 && finite == 0.0);
  }
};

// Steps T.. of the 16 x 16 Gauss-Jordan inverse without pivoting in one wavefront: lane
// (l16, lk) holds columns 4 lk .. 4 lk + 3 of row l16.  1/p by the hardware reciprocal and
// two Newton steps.
template <int T>
__device__ __forceinline__ void gj_invert_16(cpx<double> (&d)[4], GjPivots& pv) {
  if constexpr (T < 16) {
    constexpr int ct = T & 3, lt = T >> 2;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
    const cpx<double> p = mk(gj_lane(d[ct].x, lt * 16 + T), gj_lane(d[ct].y, lt * 16 + T));
    const cpx<double> col = mk(__shfl(d[ct].x, lt * 16 + l16), __shfl(d[ct].y, lt * 16 + l16));
    pv.add(p);
    const double den = p.x * p.x + p.y * p.y;
    double r = __builtin_amdgcn_rcp(den);
    r = fma(r, fma(-den, r, 1.0), r);
    r = fma(r, fma(-den, r, 1.0), r);
    const cpx<double> pinv = den > 0.0 ? mk(p.x * r, -p.y * r) : mk(0.0, 0.0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const bool own = c == ct && lk == lt;  // column T
      const cpx<double> row = cmul(mk(gj_row<T>(d[c].x), gj_row<T>(d[c].y)), pinv);
      const cpx<double> rs = own ? pinv : row;
      const cpx<double> x = own ? mk(0.0, 0.0) : d[c];
      const double xr = fma(col.y, rs.y, fma(-col.x, rs.x, x.x));
      const double xi = fma(-col.y, rs.x, fma(-col.x, rs.y, x.y));
      d[c] = l16 == T ? rs : mk(xr, xi);
    }
    gj_invert_16<T + 1>(d, pv);
  }
}

struct GjInv {
  cpx<double> P[16][66];     // row panel
  cpx<double> C[64][17];     // column panel
  cpx<double> D[2][16][17];  // diagonal inverse, one copy per wavefront that needs it
};
// In-place inverse of a 64 x 64 matrix held by four wavefronts as 2 x 2 blocks of 32 x 32,
// each 2 x 2 tiles in the layout of v_mfma_f64_16x16x4_f64's result (entry r of a lane at
// row lk + 4r, column l16); rows and columns past the matrix hold the identity, which
// leaves its inverse unchanged.  Blocked Gauss-Jordan of width 16: the owners of the row
// and column panel publish them, every wavefront inverts the diagonal 16 x 16 for itself,
// and both products (Dinv P, and the update) run on the matrix cores, with k numbered so
// that each operand is in its lane's registers as it was produced.
// Bound: latency of 64 pivots in series, 36 us; a scalar elimination with one barrier per
// row took 43 us on 16 wavefronts and about 65 on the four of a look-ahead.
__device__ __forceinline__ bool gj_invert_64(d4 (&re)[2][2], d4 (&im)[2][2], GjInv& L) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wr = wave >> 1, wc = wave & 1;
  GjPivots pv;
  // one copy of the code for the four steps: unrolled, it is 70 KiB that the instruction
  // cache sees once (39 us)
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    const int h = q >> 1, x = q & 1;
#pragma unroll
    for (int a = 0; a < 2; ++a)
      if (wr == h && a == x) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            L.P[lk + 4 * r][wc * 32 + 16 * b + l16] = mk(re[a][b][r], im[a][b][r]);
      }
#pragma unroll
    for (int b = 0; b < 2; ++b)
      if (wc == h && b == x) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            L.C[wr * 32 + 16 * a + lk + 4 * r][l16] = mk(re[a][b][r], im[a][b][r]);
      }
    __syncthreads();
    cpx<double> d[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) d[c] = L.P[l16][16 * q + 4 * lk + c];
    gj_invert_16<0>(d, pv);
    __builtin_amdgcn_sched_barrier(0);
    // R = Dinv P, k = 4 lk + s; entry s of the result is then row k = lk + 4 s of the
    // update's second operand
    d4 rr[2], ri[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      d4 t1 = {}, t2 = {}, t3 = {};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const cpx<double> y = L.P[4 * lk + s][wc * 32 + 16 * b + l16];
        t1 = __builtin_amdgcn_mfma_f64_16x16x4f64(d[s].x, y.x, t1, 0, 0, 0);
        t2 = __builtin_amdgcn_mfma_f64_16x16x4f64(d[s].y, y.y, t2, 0, 0, 0);
        t3 = __builtin_amdgcn_mfma_f64_16x16x4f64(d[s].x + d[s].y, y.x + y.y, t3, 0, 0, 0);
      }
      rr[b] = t1 - t2;
      ri[b] = (t3 - t1) - t2;
      __builtin_amdgcn_sched_barrier(0);
    }
    if (wc == h) {  // the panel's own columns: Dinv, and no old value below
#pragma unroll
      for (int c = 0; c < 4; ++c) L.D[wr][l16][4 * lk + c] = d[c];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int b = 0; b < 2; ++b)
        if (b == x) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const cpx<double> y = L.D[wr][lk + 4 * r][l16];
            rr[b][r] = y.x;
            ri[b][r] = y.y;
          }
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            re[a][b] = (d4){0, 0, 0, 0};
            im[a][b] = (d4){0, 0, 0, 0};
          }
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      if (wr == h && a == x) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          re[a][b] = rr[b];
          im[a][b] = ri[b];
        }
        continue;
      }
      cpx<double> c[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) c[s] = L.C[wr * 32 + 16 * a + l16][lk + 4 * s];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        d4 t1 = {}, t2 = {}, t3 = {};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          t1 = __builtin_amdgcn_mfma_f64_16x16x4f64(c[s].x, rr[b][s], t1, 0, 0, 0);
          t2 = __builtin_amdgcn_mfma_f64_16x16x4f64(c[s].y, ri[b][s], t2, 0, 0, 0);
          t3 = __builtin_amdgcn_mfma_f64_16x16x4f64(c[s].x + c[s].y, rr[b][s] + ri[b][s], t3, 0, 0,
                                                    0);
        }
        re[a][b] -= t1 - t2;
        im[a][b] -= (t3 - t1) - t2;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
  }
  return pv.bad();
}

// The inverse of the nbk x nbk matrix at src (row stride ld) to dst (row stride GB)
__device__ __forceinline__ bool gj_block_inverse(const cpx<double>* src, int ld, int nbk,
                                                 cpx<double>* __restrict__ dst, GjInv& L) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4, wave = threadIdx.x >> 6;
  const int r0 = (wave >> 1) * 32 + lk, c0 = (wave & 1) * 32 + l16;
  d4 re[2][2], im[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 16 * a + 4 * r, j = c0 + 16 * b;
        const bool in = i < nbk && j < nbk;
        const cpx<double> x = src[(size_t)min(i, nbk - 1) * ld + min(j, nbk - 1)];
        re[a][b][r] = in ? x.x : i == j ? 1.0 : 0.0;
        im[a][b][r] = in ? x.y : 0.0;
      }
  const bool bad = gj_invert_64(re, im, L);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 16 * a + 4 * r, j = c0 + 16 * b;
        if (i < nbk && j < nbk) dst[i * GB + j] = mk(re[a][b][r], im[a][b][r]);
      }
  return bad;
}

// Inverse of the first diagonal block
template <typename M>
__global__ void __launch_bounds__(256) k_gj_diag(M ms) {
  __shared__ GjInv L;
  const GjM m = ms(blockIdx.x);
  if (gj_block_inverse(m.A, m.N, min(GB, m.N), m.D0, L)) *m.bad = 1;
}

// Step at k (s = k / GB), 64 columns of matrix blockIdx.y.  The 64 x 64 piece of the row
// panel passes through LDS (column j of row t at slot j ^ (t & 15), so that rows and
// columns of it are both written without bank conflicts) to the product with Dinv, each of
// eight wavefronts a 16 x 32 block, three real v_mfma_f64_16x16x4 products per complex
// one.  No entry is both read and written: the previous block's rows are taken from its R
// and Dinv.  Bound: latency of its loads, LDS and products in turn, 18 us (24 with the
// previous block's values loaded one after another).
template <typename M>
__global__ void __launch_bounds__(512) k_gj_panel(M ms, int k, int s) {
  __shared__ cpx<double> P[GB][GB];
  const GjM m = ms(blockIdx.y);
  const int N = m.N, j0 = blockIdx.x * GB;
  if (k >= N || j0 >= N) return;
  const int nbk = min(GB, N - k), w = min(GB, N - j0), kp = k - GB;
  const bool full = *m.full != 0;
  const int tid = threadIdx.x, fast = tid & 63, slow = tid >> 6;
  cpx<double>* R = m.r(s);
  const cpx<double>*Rp = m.r(s + 1), *D = m.d(s), *Dp = m.d(s + 1);
  auto slot = [](int t, int j) { return j ^ (t & 15); };
  // the finished value of row kp + t at column j0 + j
  auto fixed = [&](int t, int j) {
    return j0 == kp ? Dp[t * GB + j] : Rp[(size_t)t * N + j0 + j];
  };
  const int lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lk = lane >> 4;
  const int r0 = (wave >> 1) * 16, c0 = (wave & 1) * 32;
  cpx<double> a[GB / 4];
#pragma unroll
  for (int q = 0; q < GB / 4; ++q) {
    const int r = r0 + l16, t = 4 * q + lk;
    const cpx<double> x = D[min(r, nbk - 1) * GB + min(t, nbk - 1)];
    a[q] = r < nbk && t < nbk ? x : mk(0.0, 0.0);
  }
  if (full || j0 < k) {
    cpx<double> x[8], y[8];
    const int j = min(fast, w - 1);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      x[q] = m.A[(size_t)(k + min(slow + 8 * q, nbk - 1)) * N + j0 + j];
    if (k > 0) {
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = fixed(slow + 8 * q, j);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int t = slow + 8 * q;
      P[t][slot(t, fast)] = t < nbk && fast < w ? x[q] : mk(0.0, 0.0);
    }
    if (k > 0 && fast < w) {
#pragma unroll
      for (int q = 0; q < 8; ++q) m.A[(size_t)(kp + slow + 8 * q) * N + j0 + fast] = y[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int t = fast, j = slow + 8 * q;
      if (j < w && t < nbk) {
        const cpx<double> x = P[t][slot(t, j)];
        m.Cb[(size_t)(j0 + j) * GB + t] =
            !full                  ? mk(-x.x, x.y)
            : k > 0 && j0 == kp    ? Rp[(size_t)j * N + k + t]
                                   : m.A[(size_t)(j0 + j) * N + k + t];
      }
    }
  } else {
    cpx<double> x[8];
    const int t = fast;
#pragma unroll
    for (int q = 0; q < 8; ++q)
      x[q] = m.A[(size_t)(j0 + min(slow + 8 * q, w - 1)) * N + k + min(t, nbk - 1)];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = slow + 8 * q;
      const bool in = t < nbk && j < w;
      if (in) m.Cb[(size_t)(j0 + j) * GB + t] = x[q];
      P[t][slot(t, j)] = in ? mk(x[q].x, -x[q].y) : mk(0.0, 0.0);
    }
  }
  if (j0 == k) {
    for (int e = tid; e < nbk * nbk; e += 512) {
      const int t = e / nbk, j = e % nbk;
      const cpx<double> dv = D[t * GB + j];
      R[(size_t)t * N + k + j] = mk(dv.x + (t == j ? 1.0 : 0.0), dv.y);
    }
    return;
  }
  __syncthreads();
  d4 t1[2] = {}, t2[2] = {}, t3[2] = {};
#pragma unroll
  for (int q = 0; q < GB / 4; ++q) {
    const int t = 4 * q + lk;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const cpx<double> x = P[t][slot(t, c0 + 16 * b + l16)];
      t1[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q].x, x.x, t1[b], 0, 0, 0);
      t2[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q].y, x.y, t2[b], 0, 0, 0);
      t3[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q].x + a[q].y, x.x + x.y, t3[b], 0, 0, 0);
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = r0 + lk + 4 * r, j = c0 + 16 * b + l16;
      if (t < nbk && j < w)
        R[(size_t)t * N + j0 + j] = mk(t1[b][r] - t2[b][r], (t3[b][r] - t1[b][r]) - t2[b][r]);
    }
}

// The rank-nbk update A -= Cb R, the bulk of each Gauss-Jordan step, with the next step's
// diagonal inverse in the same launch.
//   - Update tiles: with K at most GB the product per output is short and the C
//     tile streams through once, so there is no LDS staging and no barrier.
//     Each wavefront computes a 32x32 block (2x2 v_mfma_f64_16x16x4_f64, three
//     real products per complex one) with its fragments loaded straight from
//     Cb (N x GB) and R (GB x N), which stay in L2; the next four K are loaded
//     while the current ones feed the matrix cores. C is read in the epilogue;
//     three workgroups per CU cover that latency with the other wavefronts'
//     products. From N = 2048 the operands pass through LDS instead
//     (gj_update_tile_lds), which loads each fragment once per workgroup.
//     Lower tiles of 64x64 are numbered matrix, row band, column band, then the upper
//     ones (needed by matrices with m.full only), each range renumbered per XCD, so one
//     XCD's L2 holds the panels of its tiles.
//   - Look-ahead (where another step follows): the first nmat workgroups each form the
//     next diagonal block Dn = A[K'][K'] - Cb[K'] R[:, K'] with the same tile code,
//     and its inverse (gj_block_inverse). The update skips tile (K', K'): that block
//     is only ever read into values that a later step overwrites (the next
//     panel's K' columns and row block K', which the step after rewrites from
//     R and Dinv), so no workgroup writes what another reads.
constexpr int UT = 64;  // workgroup tile (2x2 wavefronts of 32x32)

// A -= product on a wavefront's 32x32 block at (ia, ja): Re = t1 - t2, Im = t3 -
// t1 - t2 (f64 16x16x4 D layout: row lk + 4r, column l16). The 8 entries of
// each row block are loaded (at clamped, always valid addresses) before any is
// stored, so the loads are in flight together: with a load, a wait and a store
// per entry, each of the 16 entries cost a full memory round trip.
__device__ __forceinline__ void gj_epilogue(const d4 (&t1)[2][2], const d4 (&t2)[2][2],
                                            const d4 (&t3)[2][2], cpx<double>* A, int N, int ia,
                                            int ja) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    cpx<double> v[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = min(ia + a * 16 + lk + 4 * r, N - 1), j = min(ja + b * 16 + l16, N - 1);
        v[b][r] = A[(size_t)i * N + j];
      }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = ia + a * 16 + lk + 4 * r, j = ja + b * 16 + l16;
        if (i < N && j < N)
          A[(size_t)i * N + j] = mk(v[b][r].x - (t1[a][b][r] - t2[a][b][r]),
                                    v[b][r].y - ((t3[a][b][r] - t1[a][b][r]) - t2[a][b][r]));
      }
  }
}

// A -= Cb R on the 64x64 tile at (i0, j0) (rows and columns below N) with the
// operands staged in LDS: Cb[i0 .. i0 + 63][K] and R[K][j0 .. j0 + 63] pass in
// chunks of 8 K through two 16 KiB buffers, loaded by global_load_lds, so each
// fragment comes from L2 once per workgroup, where the 2x2 wavefronts loading
// their fragments directly fetch each twice.
//   - Cb chunk [64 rows][8 k of 16 B]: k stored at slot k ^ (row & 7). A
//     fragment read (16 rows, one k per group of 16 lanes) then takes as many
//     LDS cycles as a contiguous 1 KiB read, by the bank-conflict counter;
//     (row & 7) ^ ((row >> 3) & 1) took twice as many. R chunk [8 k][64
//     columns]: a fragment read is 256 contiguous bytes per k.
//   - K past kdim is read clamped and zeroed at the fragment (stale panel
//     entries may hold anything); rows and columns past N are clamped and
//     feed outputs that are not stored.
//   - Products as in gj_update_tile: 2x2 v_mfma_f64_16x16x4_f64 blocks per
//     wavefront, three real products per complex one, A read in the epilogue.
__device__ __forceinline__ void gj_update_tile_lds(const cpx<double>* __restrict__ Cb,
                                                   const cpx<double>* __restrict__ R,
                                                   cpx<double>* A, int N, int kdim, int i0,
                                                   int j0, cpx<double>* lds) {
  static_assert(sizeof(GjInv) >= 4 * UT * 8 * 16, "the chunks share the inverse's LDS");
  cpx<double>*Cs0 = lds, *Rs0 = Cs0 + UT * 8, *Cs1 = Rs0 + UT * 8, *Rs1 = Cs1 + UT * 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
  d4 t1[2][2], t2[2][2], t3[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      t1[a][b] = (d4){0, 0, 0, 0};
      t2[a][b] = (d4){0, 0, 0, 0};
      t3[a][b] = (d4){0, 0, 0, 0};
    }
  // chunk at K offset kc: 16 row blocks of 1 KiB (8 of Cb, 8 rows each; 8 of
  // R, one k each), 4 per wavefront
  auto issue = [&](cpx<double>* Cs, cpx<double>* Rs, int kc) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = wave * 4 + u;
      const int row = (idx & 7) * 8 + (lane >> 3);
      const int kb = (lane & 7) ^ (lane >> 3);  // row & 7 = lane >> 3
      const cpx<double>* sa = Cb + (size_t)min(i0 + row, N - 1) * GB + min(kc + kb, kdim - 1);
      const cpx<double>* sr = R + (size_t)min(kc + (idx & 7), kdim - 1) * N + min(j0 + lane, N - 1);
      if (idx < 8)
        __builtin_amdgcn_global_load_lds((const void*)sa, (lds_void*)(Cs + idx * 64), 16, 0, 0);
      else
        __builtin_amdgcn_global_load_lds((const void*)sr, (lds_void*)(Rs + (idx - 8) * 64), 16,
                                         0, 0);
    }
  };
  auto compute = [&](const cpx<double>* Cs, const cpx<double>* Rs, int kc) {
#pragma unroll
    for (int kk = 0; kk < 8; kk += 4) {
      const int k = kk + lk;
      const bool ok = kc + k < kdim;
      cpx<double> fa[2], fb[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int row = wi + a * 16 + l16;
        const cpx<double> v = Cs[row * 8 + (k ^ (l16 & 7))];
        fa[a] = ok ? v : mk(0.0, 0.0);
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const cpx<double> v = Rs[k * UT + wj + b * 16 + l16];
        fb[b] = ok ? v : mk(0.0, 0.0);
      }
      double sa[2], sb[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) sa[a] = fa[a].x + fa[a].y;
#pragma unroll
      for (int b = 0; b < 2; ++b) sb[b] = fb[b].x + fb[b].y;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          t1[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a].x, fb[b].x, t1[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          t2[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a].y, fb[b].y, t2[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          t3[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[a], sb[b], t3[a][b], 0, 0, 0);
    }
  };
  const int nch = (kdim + 7) / 8;
  issue(Cs0, Rs0, 0);
  __syncthreads();  // (its fence waits for the loads)
  for (int c = 0; c < nch; c += 2) {
    if (c + 1 < nch) issue(Cs1, Rs1, (c + 1) * 8);
    compute(Cs0, Rs0, c * 8);
    __syncthreads();
    if (c + 1 < nch) {
      if (c + 2 < nch) issue(Cs0, Rs0, (c + 2) * 8);
      compute(Cs1, Rs1, (c + 1) * 8);
      __syncthreads();
    }
  }
  gj_epilogue(t1, t2, t3, A, N, i0 + wi, j0 + wj);
}

__host__ __device__ __forceinline__ long long gj_lower(int nt) { return (long long)nt * (nt + 1) / 2; }
__host__ __device__ __forceinline__ long long gj_pad(long long x) {
  return (x + kXcd - 1) / kXcd * kXcd;
}
// workgroups of an update over nmat matrices of up to nmax rows
inline unsigned gj_update_grid(int nmat, int nmax) {
  const int nt = (nmax + UT - 1) / UT;
  return (unsigned)(nmat + gj_pad(gj_lower(nt) * nmat) + gj_pad(gj_lower(nt - 1) * nmat));
}

template <bool kLds, typename M>
__global__ void __launch_bounds__(256, 3) k_gj_update(M ms, int nmat, int nmax, int k, int s) {
  __shared__ __align__(16) char lds[sizeof(GjInv)];
  const int wave = threadIdx.x >> 6, k2 = k + GB;
  if ((int)blockIdx.x < nmat) {
    static_assert(GB == 64 && UT == GB, "the look-ahead block is one 64x64 tile");
    const GjM m = ms(blockIdx.x);
    const int N = m.N, nb2 = min(GB, N - k2);
    if (nb2 <= 0) return;
    gj_update_tile(m.Cb, GB, m.r(s), m.A, N, GB, k2 + (wave >> 1) * 32, k2 + (wave & 1) * 32,
                   k2 + nb2, m.Dn, GB, k2);
    __syncthreads();  // Dn complete and visible to the workgroup
    if (gj_block_inverse(m.Dn, GB, nb2, m.d(s + 1), *reinterpret_cast<GjInv*>(lds)))
      *m.bad = 1;
    return;
  }
  const int ntm = (nmax + UT - 1) / UT;
  const long long low = gj_lower(ntm), up = gj_lower(ntm - 1);
  long long b = (long long)blockIdx.x - nmat;
  const bool upper = b >= gj_pad(low * nmat);
  if (upper) b -= gj_pad(low * nmat);
  const long long per = upper ? up : low, lin = xcd_linear(b, per * nmat);
  if (lin < 0) return;
  const GjM m = ms((int)(lin / per));
  const int rem = (int)(lin % per), N = m.N;
  int ti = (int)((sqrtf(8.0f * rem + 1.0f) - 1.0f) * 0.5f);
  while (gj_lower(ti) > rem) --ti;
  while (gj_lower(ti + 1) <= rem) ++ti;
  int tj = rem - (int)gj_lower(ti);
  if (upper) {
    const int x = ti + 1;
    ti = tj;
    tj = x;
  }
  if (k >= N || ti * UT >= N || tj * UT >= N || ti == s) return;
  if (ti == s + 1 && tj == s + 1) return;
  if (upper && *m.full == 0) return;
  const int nbk = min(GB, N - k);
  if constexpr (kLds)
    gj_update_tile_lds(m.Cb, m.r(s), m.A, N, nbk, ti * UT, tj * UT,
                       reinterpret_cast<cpx<double>*>(lds));
  else
    gj_update_tile(m.Cb, GB, m.r(s), m.A, N, nbk, ti * UT + (wave >> 1) * 32,
                   tj * UT + (wave & 1) * 32, N, m.A, N, 0);
}

// eps^-1 = S epst^-1 S^-1, in place, 32 x 32 tiles; the last block row from its R and Dinv.
// Without m.full the tiles above the diagonal are written by those below.
constexpr int FT = 32;
template <typename M>
__global__ void __launch_bounds__(256) k_gj_final(M ms) {
  __shared__ cpx<double> x[FT][FT + 1];
  const GjM m = ms(blockIdx.z);
  const int N = m.N, i0 = blockIdx.y * FT, j0 = blockIdx.x * FT;
  const bool full = *m.full != 0;
  if (i0 >= N || j0 >= N || (j0 > i0 && !full)) return;
  const int s = (N - 1) / GB, kl = s * GB;
  const int c = threadIdx.x % FT, r0 = threadIdx.x / FT;
  __shared__ double root[2][FT];
  // rows of a tile are all before the last block or all in it (GB is a multiple of FT)
  const bool tail = i0 >= kl, corner = tail && j0 >= kl;
  const cpx<double>* p = corner ? m.d(s) + (i0 - kl) * GB + j0 - kl
                         : tail ? m.r(s) + (size_t)(i0 - kl) * N + j0
                                : m.A + (size_t)i0 * N + j0;
  const int ld = corner ? GB : N;
  if (threadIdx.x < 2 * FT) {
    const int g = (threadIdx.x < FT ? i0 : j0) + c;
    root[threadIdx.x / FT][c] = sqrt(m.v[min(g, N - 1)]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    x[r0 + 8 * q][c] = p[(size_t)min(r0 + 8 * q, N - 1 - i0) * ld + min(c, N - 1 - j0)];
  __syncthreads();
  const bool diag = i0 == j0 && !full;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = r0 + 8 * q, i = i0 + r, j = j0 + c;
    if (i < N && j < N) {
      const cpx<double> y = diag && c > r ? x[c][r] : x[r][c];
      const double f = root[0][r] / root[1][c];
      m.A[(size_t)i * N + j] = mk(f * y.x, diag && c > r ? -f * y.y : f * y.y);
    }
  }
  if (full || i0 == j0) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = r0 + 8 * q, i = j0 + r, j = i0 + c;  // the mirror tile
    if (i < N && j < N) {
      const cpx<double> y = x[c][r];
      const double f = root[1][r] / root[0][c];
      m.A[(size_t)i * N + j] = mk(f * y.x, -f * y.y);
    }
  }
}

// Every step of the inversion of nmat matrices of up to nmax rows whose eps~ is in place
template <typename M>
gw_status gj_steps(gw_ctx* c, M ms, int nmat, int nmax, const char* sdiag, const char* ssmall,
                   const char* supd, const char* sfin) {
  {
    ProfScope ps(c, sdiag);
    hipLaunchKernelGGL(k_gj_diag<M>, dim3(nmat), dim3(256), 0, c->stream, ms);
    GW_CHECK_LAUNCH(c, "k_gj_diag");
  }
  // (up to one block the inverse of it is the result)
  for (int k = 0, s = 0; nmax > GB && k < nmax; k += GB, ++s) {
    {
      ProfScope ps(c, ssmall);
      hipLaunchKernelGGL(k_gj_panel<M>, dim3((nmax + GB - 1) / GB, nmat), dim3(512), 0, c->stream,
                         ms, k, s);
      GW_CHECK_LAUNCH(c, "k_gj_panel");
    }
    ProfScope ps(c, supd);
    // Operands staged in LDS (each fetched once per workgroup) pay where the matrices pass
    // the last-level cache, or every block is updated, which the host does not know.  One
    // matrix, inversion with fragments straight from L2 / through LDS, half the blocks:
    // 2047 rows 2.50 / 2.65 ms, 3000 3.82 / 4.07, 4000 6.60 / 6.51, 5000 11.7 / 10.3, three
    // of 3000 8.67 / 6.94; every block: 2047 rows 2.70 / 2.82, 3000 5.23 / 4.94, 4000
    // 12.5 / 10.2.  At 2048 half the blocks lose at most 7%, every block at most 4%.
    auto* update = nmax >= 2048 ? &k_gj_update<true, M> : &k_gj_update<false, M>;
    hipLaunchKernelGGL(update, dim3(gj_update_grid(nmat, nmax)), dim3(256), 0, c->stream, ms, nmat,
                       nmax, k, s);
    GW_CHECK_LAUNCH(c, "k_gj_update");
  }
  ProfScope ps(c, sfin);
  const unsigned nt = (unsigned)((nmax + FT - 1) / FT);
  hipLaunchKernelGGL(k_gj_final<M>, dim3(nt, nt, nmat), dim3(256), 0, c->stream, ms);
  GW_CHECK_LAUNCH(c, "k_gj_final");
  return GW_OK;
}

}  // namespace gw
