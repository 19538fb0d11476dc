// Learned closure of the truncated conduction-band sum.
//
// A small network predicts chi0_full - chi0_trunc for one (q, omega = 0) matrix
// from per-(G <= G') features; chi0_trunc plus the Hermitised prediction is the
// corrected matrix, and the full band sum remains the fallback and the
// reference for its error.  The nearest idea in the paper is the static remainder used for
// the Coulomb-hole sum over empty states (Computational Details).
//
//   features  |q+G|, |q+G'|, (q+G).(q+G')/10, Re chi_t/s, Im chi_t/s, 10 gap, 2 emax
//             (zero-padded to 32), s = max_G |chi_t[G][G]|, rows = upper triangle
//   network   depth hidden layers of `width` with SiLU, then a linear output;
//             products on v_mfma_f32_16x16x32_bf16 (bf16 operands rounded to
//             nearest even from float, float accumulation), float master weights
//   training  MSE over the real outputs, backpropagation with the same products
//             on transposed operands, Adam with bias correction
//   fallback  a double-precision blocked Cholesky of -chi_out; if it meets a
//             pivot that is not positive, the full sum is returned instead
#include <cmath>
#include <cstring>

#include "tiles.h"

namespace gw {

constexpr int CL_KPAD = 32;  // input features padded to one MFMA K-step
constexpr int CL_OPAD = 32;  // outputs padded (the real ones first, the rest kept zero)
constexpr int CL_RT = 128;   // row tile
constexpr int CL_NFEAT = 7;
constexpr int CL_NOUT = 2;
constexpr uint32_t CL_MAGIC = 0x4C4D5747u;  // "GWML"

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }
__device__ __forceinline__ float dsilu_f(float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// row r of the upper triangle (row major) -> (i, j), i <= j < N
__device__ __forceinline__ void tri_rc(long long r, int N, int* oi, int* oj) {
  const double b = 2.0 * N + 1.0;
  long long i = (long long)floor((b - sqrt(b * b - 8.0 * (double)r)) * 0.5);
  auto off = [&](long long k) { return k * (2LL * N - k + 1) / 2; };
  if (i < 0) i = 0;
  while (i > 0 && off(i) > r) --i;
  while (off(i + 1) <= r) ++i;
  *oi = (int)i;
  *oj = (int)(i + (r - off(i)));
}

__global__ void k_cl_scale(const cpx<double>* __restrict__ chi, int N, double* __restrict__ s) {
  __shared__ double red[256];
  double m = 0.0;
  for (int i = threadIdx.x; i < N; i += blockDim.x) {
    const cpx<double> d = chi[(size_t)i * N + i];
    m = fmax(m, sqrt(d.x * d.x + d.y * d.y));
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int k = blockDim.x / 2; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + k]);
    __syncthreads();
  }
  if (threadIdx.x == 0) s[0] = red[0] > 0.0 ? red[0] : 1.0;
}

// X[r][0..31] and (when full != NULL) T[r][0..1]; rows >= n zero.
__global__ void k_cl_features(const double* __restrict__ qg, const cpx<double>* __restrict__ chi,
                              const cpx<double>* __restrict__ full, int N, long long n,
                              long long npad, double gap, double emax,
                              const double* __restrict__ sc, float* __restrict__ X,
                              float* __restrict__ T) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= npad) return;
  float* x = X + r * CL_KPAD;
  for (int k = 0; k < CL_KPAD; ++k) x[k] = 0.f;
  if (T) { T[r * 2] = 0.f; T[r * 2 + 1] = 0.f; }
  if (r >= n) return;
  int i, j;
  tri_rc(r, N, &i, &j);
  const double s = sc[0];
  const double* a = qg + 3 * (size_t)i;
  const double* b = qg + 3 * (size_t)j;
  const cpx<double> c = chi[(size_t)i * N + j];
  x[0] = (float)sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2]);
  x[1] = (float)sqrt(b[0] * b[0] + b[1] * b[1] + b[2] * b[2]);
  x[2] = (float)((a[0] * b[0] + a[1] * b[1] + a[2] * b[2]) / 10.0);
  x[3] = (float)(c.x / s);
  x[4] = (float)(c.y / s);
  x[5] = (float)(10.0 * gap);
  x[6] = (float)(2.0 * emax);
  if (T) {
    const cpx<double> f = full[(size_t)i * N + j];
    T[r * 2] = (float)((f.x - c.x) / s);
    T[r * 2 + 1] = (float)((f.y - c.y) / s);
  }
}

// ------------------------------------------------------------------ bf16 GEMMs
// Every product is v_mfma_f32_16x16x32_bf16 with bf16 (RNE) operands rounded from
// float as they are loaded and float accumulation.  Only the pre-activations Z_l
// and the gradients dZ_l cross HBM, in float: H = SiLU(Z) is formed again where
// it is an operand, and the last hidden layer's dZ (two outputs' worth of
// products) where it is one.
//
// These kernels are bound by HBM: 18 rows x width x 4 bytes per hidden unit and
// step for depth 3.  One epoch over 301 + 433 + 552 + 797 G vectors (width 256,
// depth 3, 609 k rows, 11 GB) took 36.1 ms with 64 x 64 tiles staged element by
// element, a separate column-sum pass and one launch per layer and split sum, and
// takes 4.35 ms with these kernels, half of it in k_cl_wgrad.

typedef float f8 __attribute__((ext_vector_type(8)));

// operand of a row: SiLU(Z), the value itself, or the last hidden layer's dZ
enum { A_ID = 0, A_SILU = 1, A_OUT = 2 };
// result: Z = v + bias; the real outputs Y = v + bias; dZ = v SiLU'(Zin)
enum { EPI_Z = 0, EPI_Y = 1, EPI_DZ = 2 };

__device__ __forceinline__ float bf16_round(float x) { return bf16_to_f(bf16_rn_bits(x)); }

constexpr int CG_KC = 64;         // K chunk of B staged in LDS
constexpr int CG_KP = CG_KC + 8;  // pitch: 16 rows x 16 bytes cover all 64 banks

// C[rows][N] = epi(op(A)[rows][K] B^T), B bf16 [N][K].  A workgroup takes 128 rows
// and 16 NB columns (the whole width up to 256, so that A is read once); each of
// its four wavefronts owns 32 rows and loads their operand fragments straight
// into registers, eight consecutive k per lane, one chunk ahead.
template <int NB, int AOP, int EPI>
__global__ void __launch_bounds__(256, 2) k_cl_gemm(
    int N, int K, const float* __restrict__ A, int lda, const unsigned short* __restrict__ B,
    const float* __restrict__ bias, const float* __restrict__ Zin, float* __restrict__ C, int ldc,
    const float2* __restrict__ dy, const float* __restrict__ wo) {
  __shared__ __align__(16) unsigned short Bs[16 * NB][CG_KP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  const size_t m0 = (size_t)blockIdx.x * CL_RT + wave * 32;
  const int n0 = blockIdx.y * 16 * NB;
  f4 acc[2][NB];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < NB; ++y) acc[x][y] = (f4){0, 0, 0, 0};
  float2 g[2];
  if (AOP == A_OUT) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      g[x] = dy[m0 + x * 16 + l16];
      g[x].x = bf16_round(g[x].x);
      g[x].y = bf16_round(g[x].y);
    }
  }
  f8 a[2][2];
  auto fetch = [&](int kc) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (kc + s * 32 < K) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
          a[s][x] = *reinterpret_cast<const f8*>(A + (m0 + x * 16 + l16) * lda + kc + s * 32 +
                                                 lk * 8);
      }
  };
  fetch(0);
  for (int kc = 0; kc < K; kc += CG_KC) {
    const int kl = min(CG_KC, K - kc), q8 = kl >> 3;  // 32 or 64: 4 or 8 chunks of 8 per row
    const int sh = q8 == 8 ? 3 : 2;
    if (kc) __syncthreads();
    for (int e = tid; e < 16 * NB * q8; e += 256) {
      const int n = e >> sh, k = (e & (q8 - 1)) * 8;
      *reinterpret_cast<uint4*>(&Bs[n][k]) =
          *reinterpret_cast<const uint4*>(B + (size_t)(n0 + n) * K + kc + k);
    }
    bf8 af[2][2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (s * 32 < kl) {
        f8 w0, w1;
        if (AOP == A_OUT) {
          w0 = *reinterpret_cast<const f8*>(wo + kc + s * 32 + lk * 8);
          w1 = *reinterpret_cast<const f8*>(wo + K + kc + s * 32 + lk * 8);
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          f8 v = a[s][x];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            if (AOP == A_SILU) v[i] = silu_f(v[i]);
            if (AOP == A_OUT) v[i] = (g[x].x * w0[i] + g[x].y * w1[i]) * dsilu_f(v[i]);
          }
          af[s][x] = __builtin_convertvector(v, bf8);
        }
      }
    __syncthreads();
    if (kc + CG_KC < K) fetch(kc + CG_KC);
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (s * 32 < kl) {
#pragma unroll
        for (int y = 0; y < NB; ++y) {
          const bf8 b = *reinterpret_cast<const bf8*>(&Bs[y * 16 + l16][s * 32 + lk * 8]);
#pragma unroll
          for (int x = 0; x < 2; ++x)
            acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[s][x], b, acc[x][y], 0, 0, 0);
        }
      }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < NB; ++y) {
      const int j = n0 + y * 16 + l16;
      if (EPI == EPI_Y && j >= CL_NOUT) continue;
      const size_t o = (m0 + x * 16 + lk * 4) * ldc + j;
      float z[4];
      if (EPI == EPI_DZ) {
#pragma unroll
        for (int r = 0; r < 4; ++r) z[r] = Zin[o + (size_t)r * ldc];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        C[o + (size_t)r * ldc] = EPI == EPI_DZ ? acc[x][y][r] * dsilu_f(z[r])
                                               : acc[x][y][r] + bias[j];
    }
}

// bf16 copies of the weights for the products: wb [out][in] as stored, wt its
// transpose [in][out]; wo the two real output rows, rounded, in float.
constexpr int CL_MAXL = 9;
struct ClShape {
  int layers;
  int din[CL_MAXL], dout[CL_MAXL];
  unsigned woff[CL_MAXL];
};
__global__ void k_cl_pack(const float* __restrict__ p, ClShape sh, unsigned short* __restrict__ wb,
                          unsigned short* __restrict__ wt, float* __restrict__ wo) {
  const int l = blockIdx.y, din = sh.din[l], dout = sh.dout[l];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= din * dout) return;
  const unsigned short h = bf16_rn_bits(p[sh.woff[l] + i]);
  const int o = i / din, k = i - o * din;
  wb[sh.woff[l] + i] = h;
  wt[sh.woff[l] + (unsigned)k * dout + o] = h;
  if (l == sh.layers - 1 && o < CL_NOUT) wo[o * din + k] = bf16_to_f(h);
}

// Weight and bias gradients of every layer in one launch: dW_l = dZ_l^T H_(l-1)
// over a split of the rows, 128 x 128 outputs per workgroup.  The contraction runs
// over rows, so 32 rows of the 256 operand columns pass through LDS transposed:
// one column per thread, its 32 loads coalesced across the wavefront and in
// flight while the previous slab is multiplied.  The thread of a dZ column also
// sums it for the bias.  The tiles of one split follow one another on one XCD,
// where the columns they share stay in L2.
constexpr int WG_T = 128, WG_P = 40;
struct ClWgLayer {
  const float *dz, *h;   // dmode A_ID: dZ, A_OUT: Z of the last hidden layer, A_SILU: dY (outputs)
  int dout, din, dmode, hmode, tn, tile0;
  unsigned woff, boff;
};
struct ClWg {
  int layers, tiles;
  ClWgLayer l[CL_MAXL];
};
__global__ void __launch_bounds__(256, 2) k_cl_wgrad(ClWg W, long long rows, int rchunk,
                                                     const float2* __restrict__ dy,
                                                     const float* __restrict__ wo, size_t count,
                                                     float* __restrict__ part) {
  __shared__ __align__(16) unsigned short S[2][2 * WG_T][WG_P];
  const int xcd = blockIdx.x % kXcd, idx = blockIdx.x / kXcd;
  const int tile = idx % W.tiles, split = (idx / W.tiles) * kXcd + xcd;
  int li = 0;
  while (li + 1 < W.layers && tile >= W.l[li + 1].tile0) ++li;
  const ClWgLayer L = W.l[li];
  const int tm = (tile - L.tile0) / L.tn, tn = (tile - L.tile0) % L.tn;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lk = lane >> 4, wr = wave >> 1, wc = wave & 1;
  const bool isd = tid < WG_T;
  const int col = isd ? tm * WG_T + tid : tn * WG_T + tid - WG_T;
  const int mode = isd ? L.dmode : L.hmode;
  const bool outs = isd && L.dmode == A_SILU;  // the output layer's dY columns
  const bool live = outs ? col < CL_NOUT : col < (isd ? L.dout : L.din);
  const int ld = outs ? CL_NOUT : isd ? L.dout : L.din;
  const float* src = (outs ? reinterpret_cast<const float*>(dy) : isd ? L.dz : L.h) +
                     (live ? col : 0);
  const long long r0 = (long long)split * rchunk, r1 = min(rows, r0 + rchunk);
  float w0 = 0.f, w1 = 0.f;
  if (isd && L.dmode == A_OUT && live) { w0 = wo[col]; w1 = wo[L.dout + col]; }
  f4 acc[4][4];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[x][y] = (f4){0, 0, 0, 0};
  float csum = 0.f;
  float v[32];
  auto fetch = [&](long long r) {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = src[(size_t)(r + i) * ld];
  };
  const bool work = tm * WG_T + wr * 64 < L.dout && tn * WG_T + wc * 64 < L.din;
  if (r0 < r1) fetch(r0);
  int buf = 0;
  for (long long r = r0; r < r1; r += 32, buf ^= 1) {
    if (mode == A_SILU && !outs) {
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = silu_f(v[i]);
    } else if (mode == A_OUT) {
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const float2 g = dy[r + i];
        v[i] = (bf16_round(g.x) * w0 + bf16_round(g.y) * w1) * dsilu_f(v[i]);
      }
    }
    if (!live) {
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = 0.f;
    }
    float slab = 0.f;  // 32 rows at a time: a chain over all rows would round each at its sum
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f8 t;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        t[k] = v[8 * i + k];
        slab += t[k];
      }
      *reinterpret_cast<bf8*>(&S[buf][tid][8 * i]) = __builtin_convertvector(t, bf8);
    }
    csum += slab;
    __syncthreads();
    if (r + 32 < r1) fetch(r + 32);
    if (work) {
      bf8 a[4], b[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        a[x] = *reinterpret_cast<const bf8*>(&S[buf][wr * 64 + x * 16 + l16][lk * 8]);
        b[x] = *reinterpret_cast<const bf8*>(&S[buf][WG_T + wc * 64 + x * 16 + l16][lk * 8]);
      }
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[x], b[y], acc[x][y], 0, 0, 0);
    }
  }
  float* out = part + (size_t)split * count;
  if (isd && tn == 0 && col < L.dout) out[L.boff + col] = csum;
  if (!work) return;
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = tm * WG_T + wr * 64 + x * 16 + lk * 4 + q;
        const int j = tn * WG_T + wc * 64 + y * 16 + l16;
        if (i < L.dout && j < L.din) out[L.woff + (size_t)i * L.din + j] = acc[x][y][q];
      }
}

// dY = 2 (Y - T) / (n nout); per-block partial sums of (Y-T)^2
__global__ void k_cl_dy(const float* __restrict__ Y, const float* __restrict__ T, long long n,
                        long long npad, float* __restrict__ dY, double* __restrict__ part) {
  __shared__ double red[256];
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  double s = 0.0;
  if (r < npad) {
    const double scale = 2.0 / ((double)n * CL_NOUT);
    for (int o = 0; o < CL_NOUT; ++o) {
      const float d = r < n ? Y[r * CL_NOUT + o] - T[r * CL_NOUT + o] : 0.f;
      dY[r * CL_NOUT + o] = (float)(scale * d);
      s += (double)d * d;
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = blockDim.x / 2; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void k_sum_f64(const double* __restrict__ part, int n, double* __restrict__ out) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = blockDim.x / 2; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0];
}

// Adam on the gradient summed over the row splits in their order
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ part, int splits,
                       float* __restrict__ m, float* __restrict__ v, size_t n, float lr, float b1,
                       float b2, float eps, float bc1, float bc2) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float gi = 0.f;
#pragma unroll 8
  for (int z = 0; z < splits; ++z) gi += part[(size_t)z * n + i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// out = chi_t + s * Hermitise(Y): (i<=j) gets y, (j,i) its conjugate, diagonal real
__global__ void k_cl_apply(const cpx<double>* __restrict__ chi, const float* __restrict__ Y, int N,
                           long long n, const double* __restrict__ sc,
                           cpx<double>* __restrict__ out) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  int i, j;
  tri_rc(r, N, &i, &j);
  const double s = sc[0];
  const double yr = s * (double)Y[r * CL_NOUT], yi = s * (double)Y[r * CL_NOUT + 1];
  const cpx<double> c = chi[(size_t)i * N + j];
  if (i == j) {
    out[(size_t)i * N + i] = mk(c.x + yr, c.y);
  } else {
    out[(size_t)i * N + j] = mk(c.x + yr, c.y + yi);
    const cpx<double> d = chi[(size_t)j * N + i];
    out[(size_t)j * N + i] = mk(d.x + yr, d.y - yi);
  }
}

// ------------------------------------------------------------------ Cholesky check
// A = -chi (lower Cholesky, right-looking, blocks of 32).  flag = 1 on a pivot
// that is not positive.
constexpr int CB = 32;

__global__ void k_set_i32(int* p, int v) { *p = v; }

__global__ void k_chol_neg(const cpx<double>* __restrict__ chi, cpx<double>* __restrict__ A,
                           size_t nn) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nn) A[i] = mk(-chi[i].x, -chi[i].y);
}

// factor the diagonal block in LDS; store L11 and W = L11^-H (upper) in Lw
__global__ void __launch_bounds__(1024) k_chol_diag(cpx<double>* __restrict__ A, int N, int k,
                                                    cpx<double>* __restrict__ Lw,
                                                    int* __restrict__ flag) {
  __shared__ cpx<double> L[CB][CB + 1];
  __shared__ cpx<double> Wi[CB][CB + 1];
  __shared__ double dpiv;
  const int nbk = min(CB, N - k);
  const int tid = threadIdx.x, i = tid / CB, j = tid % CB;
  if (i < nbk && j < nbk) L[i][j] = A[(size_t)(k + i) * N + k + j];
  __syncthreads();
  for (int t = 0; t < nbk; ++t) {
    if (tid == 0) {
      const double d = L[t][t].x;
      if (!(d > 0.0) || !(d < INFINITY)) { flag[0] = 1; dpiv = 1.0; } else dpiv = sqrt(d);
    }
    __syncthreads();
    const double p = dpiv;
    // column t below the pivot: l_it = a_it / p
    if (j == t && i > t && i < nbk) L[i][t] = scal(L[i][t], 1.0 / p);
    if (tid == 0) L[t][t] = mk(p, 0.0);
    __syncthreads();
    // trailing: a_ij -= l_it conj(l_jt), i >= j > t
    if (i > t && j > t && i < nbk && j <= i) L[i][j] = L[i][j] - cmulc(L[j][t], L[i][t]);
    __syncthreads();
  }
  // W = L^-1 (lower) by forward substitution on the identity, one column per thread
  if (tid < nbk) {
    const int c = tid;
    for (int r = 0; r < nbk; ++r) {
      cpx<double> s = mk(r == c ? 1.0 : 0.0, 0.0);
      for (int u = c; u < r; ++u) s = s - cmul(L[r][u], Wi[u][c]);
      Wi[r][c] = r >= c ? cmul(s, mk(1.0 / L[r][r].x, 0.0)) : mk(0.0, 0.0);
    }
  }
  __syncthreads();
  if (i < nbk && j < nbk) {
    A[(size_t)(k + i) * N + k + j] = j <= i ? L[i][j] : mk(0.0, 0.0);
    Lw[i * CB + j] = Wi[i][j];  // L11^-1, lower
  }
}

// rows below the block: L21 = A21 L11^-H, i.e. l_i = a_i (L11^-1)^H; also R = L21^H
__global__ void k_chol_panel(cpx<double>* __restrict__ A, int N, int k,
                             const cpx<double>* __restrict__ Lw, cpx<double>* __restrict__ R) {
  const int nbk = min(CB, N - k);
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  const int rows = N - k - nbk;
  if (e >= rows * nbk) return;
  const int i = k + nbk + e / nbk, t = e % nbk;
  // sum_u a_iu conj(W[t][u]), W = L11^-1 lower
  cpx<double> s = mk(0.0, 0.0);
  for (int u = 0; u <= t; ++u) s = s + cmul(A[(size_t)i * N + k + u], mk(Lw[t * CB + u].x, -Lw[t * CB + u].y));
  // written to R first: the row of A is still being read by the other t of this row
  R[(size_t)t * N + i] = mk(s.x, -s.y);
}

__global__ void k_chol_store(cpx<double>* __restrict__ A, int N, int k,
                             const cpx<double>* __restrict__ R) {
  const int nbk = min(CB, N - k);
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  const int rows = N - k - nbk;
  if (e >= rows * nbk) return;
  const int i = k + nbk + e / nbk, t = e % nbk;
  const cpx<double> r = R[(size_t)t * N + i];
  A[(size_t)i * N + k + t] = mk(r.x, -r.y);
}

__global__ void __launch_bounds__(256) k_chol_update(cpx<double>* __restrict__ A, int N, int k,
                                                     const cpx<double>* __restrict__ R) {
  const int nbk = min(CB, N - k);
  const int s = k + nbk, rest = N - s;
  const int i0 = blockIdx.y * ZTM, j0 = blockIdx.x * ZTM;
  if (i0 >= rest || j0 >= rest) return;
  // A22 -= L21 L21^H, L21 = A[s:, k:k+nbk] (ld N), L21^H = R[:, s:] (ld N)
  zgemm_tile(rest, rest, nbk, -1.0, 1.0, A + (size_t)s * N + k, N, R + s, N, A + (size_t)s * N + s, N,
             i0, j0);
}

}  // namespace gw

// ------------------------------------------------------------------ network object
struct gw_mlp {
  gw_ctx* ctx = nullptr;
  int nin = 0, width = 0, depth = 0, nout = 0;
  std::vector<int> din, dout;          // per linear layer (padded)
  std::vector<size_t> woff, boff;      // offsets (floats) into the flat parameter arrays
  size_t count = 0;
  float *p = nullptr, *m = nullptr, *v = nullptr;
  long long step = 0;
  bool ready = false;                  // trained or loaded
  double tol = 1e-4;                   // INFER with chi0_full: largest accepted rel_F
  char* act = nullptr;                 // activations and scratch
  size_t act_cap = 0;
};

namespace gw {

void mlp_free(gw_mlp* n) {
  if (n->p) (void)hipFree(n->p);
  if (n->act) (void)hipFree(n->act);
  delete n;
}

static uint64_t splitmix64(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// activation layout: X[npad][KPAD]; Z_l [npad][width] for l < depth (inference keeps
// two of them in turn); dZ_l [npad][width] for l < depth - 1 (training); Y, dY, T
// [npad][2]; gradient partials [splits][count]; bf16 weights; loss partials
struct ClBufs {
  float *X, *Y, *dY, *T, *part, *wo;
  unsigned short *wb, *wt;
  std::vector<float*> Z, dZ;
  double *lpart, *loss, *scale, *rpart, *rsum;
  cpx<double>* chol;
  cpx<double>* R;
  cpx<double>* Lw;
};

// Row splits of the weight gradients: a multiple of the XCDs.  64 splits of the 12
// tiles of a 256-wide, 3-deep network are 768 workgroups, and their partials
// (35 MB) stay below a tenth of the operands' bytes from 60 k rows on.  Larger
// networks have more tiles and take fewer splits, so that the partials stay within
// 256 MB, but not fewer than 32 of many rows: each split is a chain of sums in single
// precision, and rows / 32 / splits terms and the splits together are never more than
// with 32.
static int cl_splits(size_t count, long long npad) {
  const long long fit = std::min<long long>(64, (long long)((64u << 20) / count) / kXcd * kXcd);
  return (int)std::max(fit, std::min<long long>(32, (npad + 8191) / 8192 * kXcd));
}
static constexpr int kRelBlocks = 256;  // workgroups of the fixed-order rel_F reduction

static gw_status cl_buffers(gw_mlp* net, int N, long long npad, bool train, ClBufs* b) {
  gw_ctx* c = net->ctx;
  const size_t w = net->width;
  std::vector<std::pair<void**, size_t>> parts;
  auto add = [&](auto** p, size_t bytes) { parts.push_back({reinterpret_cast<void**>(p), bytes}); };
  const int nz = train ? net->depth : std::min(net->depth, 2), nd = train ? net->depth - 1 : 0;
  b->Z.assign(net->depth, nullptr);
  b->dZ.assign(net->depth, nullptr);
  add(&b->X, (size_t)npad * CL_KPAD * 4);
  for (int l = 0; l < nz; ++l) add(&b->Z[l], (size_t)npad * w * 4);
  for (int l = 0; l < nd; ++l) add(&b->dZ[l], (size_t)npad * w * 4);
  add(&b->Y, (size_t)npad * CL_NOUT * 4);
  add(&b->dY, (size_t)npad * CL_NOUT * 4);
  add(&b->T, (size_t)npad * CL_NOUT * 4);
  add(&b->part, train ? (size_t)cl_splits(net->count, npad) * net->count * 4 : 0);
  add(&b->wo, CL_NOUT * w * 4);
  add(&b->wb, net->count * 2);
  add(&b->wt, net->count * 2);
  add(&b->lpart, (size_t)((npad + 255) / 256) * 8);
  add(&b->loss, 8);
  add(&b->scale, 8);
  add(&b->rpart, 2 * kRelBlocks * 8);
  add(&b->rsum, 2 * 8);
  add(&b->chol, train ? 0 : (size_t)N * N * 16);
  add(&b->R, train ? 0 : (size_t)CB * N * 16);
  add(&b->Lw, (size_t)CB * CB * 16);
  size_t total = 0;
  for (auto& p : parts) total += align_up(p.second);
  if (total > net->act_cap) {
    if (net->act) {
      GW_HIP(c, hipStreamSynchronize(c->stream));
      (void)hipFree(net->act);
      net->act = nullptr;
      net->act_cap = 0;
    }
    void* q = nullptr;
    hipError_t e = hipMalloc(&q, total);
    if (e != hipSuccess) return fail(c, GW_ENOMEM, "closure workspace of %zu bytes", total);
    net->act = static_cast<char*>(q);
    net->act_cap = total;
  }
  size_t off = 0;
  for (auto& p : parts) {
    *p.first = net->act + off;
    off += align_up(p.second);
  }
  for (int l = nz; l < net->depth; ++l) b->Z[l] = b->Z[l % nz];
  return GW_OK;
}

// one product over all rows; the column tile is the largest of 256, 128, 64 that
// divides the width
template <int AOP, int EPI>
static gw_status cl_gemm(gw_ctx* c, long long npad, int N, int K, const float* A,
                         const unsigned short* B, const float* bias, const float* Zin, float* C,
                         const float* dy, const float* wo, const char* name) {
  const unsigned gx = (unsigned)(npad / CL_RT);
  const float2* g = reinterpret_cast<const float2*>(dy);
  ProfScope ps(c, name);
  if constexpr (EPI == EPI_Y) {
    hipLaunchKernelGGL((k_cl_gemm<1, AOP, EPI>), dim3(gx, 1), dim3(256), 0, c->stream, N, K, A, K,
                       B, bias, Zin, C, CL_NOUT, g, wo);
  } else if (N % 256 == 0) {
    hipLaunchKernelGGL((k_cl_gemm<16, AOP, EPI>), dim3(gx, N / 256), dim3(256), 0, c->stream, N, K,
                       A, K, B, bias, Zin, C, N, g, wo);
  } else if (N % 128 == 0) {
    hipLaunchKernelGGL((k_cl_gemm<8, AOP, EPI>), dim3(gx, N / 128), dim3(256), 0, c->stream, N, K,
                       A, K, B, bias, Zin, C, N, g, wo);
  } else {
    hipLaunchKernelGGL((k_cl_gemm<4, AOP, EPI>), dim3(gx, N / 64), dim3(256), 0, c->stream, N, K, A,
                       K, B, bias, Zin, C, N, g, wo);
  }
  GW_CHECK_LAUNCH(c, "k_cl_gemm");
  return GW_OK;
}

static gw_status cl_forward(gw_mlp* net, long long npad, ClBufs& b) {
  gw_ctx* c = net->ctx;
  const int L = net->depth;
  ClShape sh{};
  sh.layers = L + 1;
  int most = 0;
  for (int l = 0; l <= L; ++l) {
    sh.din[l] = net->din[l];
    sh.dout[l] = net->dout[l];
    sh.woff[l] = (unsigned)net->woff[l];
    most = std::max(most, net->din[l] * net->dout[l]);
  }
  {
    ProfScope ps(c, "closure_pack");
    hipLaunchKernelGGL(k_cl_pack, dim3((most + 255) / 256, L + 1), dim3(256), 0, c->stream, net->p,
                       sh, b.wb, b.wt, b.wo);
    GW_CHECK_LAUNCH(c, "k_cl_pack");
  }
  gw_status st = cl_gemm<A_ID, EPI_Z>(c, npad, net->dout[0], net->din[0], b.X, b.wb + net->woff[0],
                                      net->p + net->boff[0], nullptr, b.Z[0], nullptr, nullptr,
                                      "closure_fwd");
  for (int l = 1; l < L && st == GW_OK; ++l)
    st = cl_gemm<A_SILU, EPI_Z>(c, npad, net->dout[l], net->din[l], b.Z[l - 1],
                                b.wb + net->woff[l], net->p + net->boff[l], nullptr, b.Z[l],
                                nullptr, nullptr, "closure_fwd");
  if (st != GW_OK) return st;
  return cl_gemm<A_SILU, EPI_Y>(c, npad, net->dout[L], net->din[L], b.Z[L - 1],
                                b.wb + net->woff[L], net->p + net->boff[L], nullptr, b.Y, nullptr,
                                nullptr, "closure_fwd");
}

// gradients of the loss already expressed in dY, as row-split partials in b.part
static gw_status cl_backward(gw_mlp* net, long long npad, ClBufs& b) {
  gw_ctx* c = net->ctx;
  gw_status st = GW_OK;
  const int L = net->depth;
  // d(pre-activation of layer l-1) = (dZ_l W_l) SiLU'(Z_(l-1)); dZ of layer L-1 is
  // formed from dY where it is needed
  for (int l = L - 1; l >= 1; --l) {
    if (l == L - 1)
      st = cl_gemm<A_OUT, EPI_DZ>(c, npad, net->din[l], net->dout[l], b.Z[l], b.wt + net->woff[l],
                                  nullptr, b.Z[l - 1], b.dZ[l - 1], b.dY, b.wo, "closure_bwd");
    else
      st = cl_gemm<A_ID, EPI_DZ>(c, npad, net->din[l], net->dout[l], b.dZ[l], b.wt + net->woff[l],
                                 nullptr, b.Z[l - 1], b.dZ[l - 1], nullptr, nullptr,
                                 "closure_bwd");
    if (st != GW_OK) return st;
  }
  ClWg W{};
  W.layers = L + 1;
  for (int l = 0; l <= L; ++l) {
    ClWgLayer& y = W.l[l];
    y.dout = net->dout[l];
    y.din = net->din[l];
    y.dmode = l == L ? A_SILU : l == L - 1 ? A_OUT : A_ID;
    y.hmode = l == 0 ? A_ID : A_SILU;
    y.dz = l == L ? b.dY : l == L - 1 ? b.Z[l] : b.dZ[l];
    y.h = l == 0 ? b.X : b.Z[l - 1];
    y.woff = (unsigned)net->woff[l];
    y.boff = (unsigned)net->boff[l];
    y.tn = (y.din + WG_T - 1) / WG_T;
    y.tile0 = W.tiles;
    W.tiles += y.tn * ((y.dout + WG_T - 1) / WG_T);
  }
  const int splits = cl_splits(net->count, npad);
  const long long rchunk = ((npad + splits - 1) / splits + 31) / 32 * 32;
  ProfScope ps(c, "closure_wgrad");
  hipLaunchKernelGGL(k_cl_wgrad, dim3((unsigned)(W.tiles * splits)), dim3(256), 0, c->stream, W,
                     npad, (int)rchunk, reinterpret_cast<const float2*>(b.dY), b.wo, net->count,
                     b.part);
  GW_CHECK_LAUNCH(c, "k_cl_wgrad");
  return GW_OK;
}

// Per workgroup, in a fixed order: the sums of |a - b|^2 and of |b|^2 over
// the elements i = blockIdx.x * 256 + threadIdx.x + k * gridDim.x * 256, into
// part[blockIdx.x] and part[gridDim.x + blockIdx.x].
__global__ void __launch_bounds__(256) k_relf_part(const cpx<double>* __restrict__ a,
                                                   const cpx<double>* __restrict__ b, size_t n,
                                                   double* __restrict__ part) {
  __shared__ double sd[256], sr[256];
  double d = 0.0, r = 0.0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const cpx<double> x = a[i], y = b[i];
    const double ex = x.x - y.x, ey = x.y - y.y;
    d += ex * ex + ey * ey;
    r += y.x * y.x + y.y * y.y;
  }
  sd[threadIdx.x] = d;
  sr[threadIdx.x] = r;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) {
      sd[threadIdx.x] += sd[threadIdx.x + k];
      sr[threadIdx.x] += sr[threadIdx.x + k];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[blockIdx.x] = sd[0];
    part[gridDim.x + blockIdx.x] = sr[0];
  }
}

// rel_F(a, b) = ||a - b||_F / ||b||_F over N x N complex doubles, reduced on the
// device in a fixed order (the same inputs give the same bits); synchronises.
static gw_status cl_rel_f(gw_ctx* c, int N, const double* a, const double* b, ClBufs& bf,
                          double* rel) {
  const size_t nn = (size_t)N * N;
  {
    ProfScope ps(c, "closure_judge");
    hipLaunchKernelGGL(k_relf_part, dim3(kRelBlocks), dim3(256), 0, c->stream,
                       reinterpret_cast<const cpx<double>*>(a),
                       reinterpret_cast<const cpx<double>*>(b), nn, bf.rpart);
    GW_CHECK_LAUNCH(c, "k_relf_part");
    hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(256), 0, c->stream, bf.rpart, kRelBlocks, bf.rsum);
    GW_CHECK_LAUNCH(c, "k_sum_f64");
    hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(256), 0, c->stream, bf.rpart + kRelBlocks,
                       kRelBlocks, bf.rsum + 1);
    GW_CHECK_LAUNCH(c, "k_sum_f64");
  }
  double h[2] = {0.0, 0.0};
  GW_HIP(c, hipMemcpyAsync(h, bf.rsum, sizeof h, hipMemcpyDeviceToHost, c->stream));
  GW_HIP(c, hipStreamSynchronize(c->stream));
  *rel = h[1] > 0.0 ? std::sqrt(h[0] / h[1]) : (h[0] > 0.0 ? INFINITY : 0.0);
  return GW_OK;
}

static gw_status cl_cholesky_fails(gw_ctx* c, int N, const double* chi, ClBufs& b, bool* fails) {
  const size_t nn = (size_t)N * N;
  {
    ProfScope ps(c, "closure_chol");
    hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(1), 0, c->stream, c->d_flag + 2, 0);
    GW_CHECK_LAUNCH(c, "k_set_i32");
    hipLaunchKernelGGL(k_chol_neg, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, c->stream,
                       reinterpret_cast<const cpx<double>*>(chi), b.chol, nn);
    GW_CHECK_LAUNCH(c, "k_chol_neg");
    for (int k = 0; k < N; k += CB) {
      const int nbk = std::min(CB, N - k), rest = N - k - nbk;
      hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(1024), 0, c->stream, b.chol, N, k, b.Lw,
                         c->d_flag + 2);
      GW_CHECK_LAUNCH(c, "k_chol_diag");
      if (rest <= 0) break;
      hipLaunchKernelGGL(k_chol_panel, dim3((rest * nbk + 255) / 256), dim3(256), 0, c->stream,
                         b.chol, N, k, b.Lw, b.R);
      GW_CHECK_LAUNCH(c, "k_chol_panel");
      hipLaunchKernelGGL(k_chol_store, dim3((rest * nbk + 255) / 256), dim3(256), 0, c->stream,
                         b.chol, N, k, b.R);
      GW_CHECK_LAUNCH(c, "k_chol_store");
      const int t = (rest + ZTM - 1) / ZTM;
      hipLaunchKernelGGL(k_chol_update, dim3(t, t), dim3(256), 0, c->stream, b.chol, N, k, b.R);
      GW_CHECK_LAUNCH(c, "k_chol_update");
    }
  }
  int flag = 0;
  GW_HIP(c, hipMemcpyAsync(&flag, c->d_flag + 2, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  GW_HIP(c, hipStreamSynchronize(c->stream));
  *fails = flag != 0;
  return GW_OK;
}

}  // namespace gw

using namespace gw;

extern "C" {

gw_status gw_mlp_create(gw_ctx* c, gw_mlp** out, int nin, int width, int depth, int nout,
                        uint64_t seed) {
  if (!c || !out) return GW_EINVAL;
  *out = nullptr;
  c->err.clear();
  if (nin < 1 || nin > CL_KPAD || nout < 1 || nout > CL_OPAD || width < 64 || width % 64 ||
      width > 4096 || depth < 1 || depth > 8)
    return fail(c, GW_EINVAL, "network shape: 1<=nin<=32, 1<=nout<=32, width a multiple of 64 "
                              "(<=4096), 1<=depth<=8");
  gw_mlp* n = new gw_mlp();
  n->ctx = c;
  n->nin = nin;
  n->width = width;
  n->depth = depth;
  n->nout = nout;
  for (int l = 0; l <= depth; ++l) {
    n->din.push_back(l == 0 ? CL_KPAD : width);
    n->dout.push_back(l == depth ? CL_OPAD : width);
  }
  for (int l = 0; l <= depth; ++l) {
    n->woff.push_back(n->count);
    n->count += (size_t)n->din[l] * n->dout[l];
    n->boff.push_back(n->count);
    n->count += n->dout[l];
  }
  // Glorot-uniform weights on the real fan-in/fan-out (splitmix64 uniforms);
  // padded rows and columns and every bias start (and stay) at zero
  std::vector<float> h(n->count, 0.f);
  uint64_t s = seed;
  for (int l = 0; l <= depth; ++l) {
    const int ri = l == 0 ? nin : width, ro = l == depth ? nout : width;
    const double lim = std::sqrt(6.0 / (ri + ro));
    for (int o = 0; o < ro; ++o)
      for (int i = 0; i < ri; ++i) {
        const double u = (double)(splitmix64(s) >> 11) * (1.0 / 9007199254740992.0);
        h[n->woff[l] + (size_t)o * n->din[l] + i] = (float)((2.0 * u - 1.0) * lim);
      }
  }
  void* mem = nullptr;
  if (hipMalloc(&mem, 3 * n->count * sizeof(float)) != hipSuccess) {
    delete n;
    return fail(c, GW_ENOMEM, "network parameters");
  }
  n->p = static_cast<float*>(mem);
  n->m = n->p + n->count;
  n->v = n->m + n->count;
  hipError_t e = hipMemcpy(n->p, h.data(), n->count * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemset(n->m, 0, 2 * n->count * 4);
  if (e != hipSuccess) {
    (void)hipFree(mem);
    delete n;
    return hip_fail(c, e, "network init");
  }
  c->mlps.insert(n);
  *out = n;
  return GW_OK;
}

gw_status gw_mlp_set_tolerance(gw_mlp* n, double tol) {
  if (!n) return GW_EINVAL;
  if (!(tol >= 0.0) || !std::isfinite(tol))
    return fail(n->ctx, GW_EINVAL, "the closure tolerance must be finite and >= 0");
  n->tol = tol;
  return GW_OK;
}

gw_status gw_mlp_destroy(gw_mlp* n) {
  if (!n) return GW_EINVAL;
  (void)hipStreamSynchronize(n->ctx->stream);
  n->ctx->mlps.erase(n);
  gw::mlp_free(n);
  return GW_OK;
}

// layout: u32 magic, u32 version, i32 nin, width, depth, nout, kpad, opad,
//         i64 step, i64 count, then float params[count], m[count], v[count]
gw_status gw_mlp_save(const gw_mlp* n, void* buf, size_t* nbytes) {
  if (!n || !nbytes) return GW_EINVAL;
  const size_t need = 48 + 3 * n->count * 4;
  if (!buf) { *nbytes = need; return GW_OK; }
  if (*nbytes < need) return fail(n->ctx, GW_EINVAL, "buffer of %zu bytes, %zu needed", *nbytes, need);
  char* b = static_cast<char*>(buf);
  uint32_t hdr[2] = {CL_MAGIC, 1};
  int32_t dims[6] = {n->nin, n->width, n->depth, n->nout, CL_KPAD, CL_OPAD};
  int64_t tail[2] = {n->step, (int64_t)n->count};
  std::memcpy(b, hdr, 8);
  std::memcpy(b + 8, dims, 24);
  std::memcpy(b + 32, tail, 16);
  hipError_t e = hipStreamSynchronize(n->ctx->stream);
  if (e == hipSuccess) e = hipMemcpy(b + 48, n->p, n->count * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(b + 48 + n->count * 4, n->m, n->count * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(b + 48 + 2 * n->count * 4, n->v, n->count * 4, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(n->ctx, e, "gw_mlp_save");
  *nbytes = need;
  return GW_OK;
}

gw_status gw_mlp_load(gw_mlp* n, const void* buf, size_t nbytes) {
  if (!n || !buf) return GW_EINVAL;
  const char* b = static_cast<const char*>(buf);
  if (nbytes < 48) return fail(n->ctx, GW_EINVAL, "buffer too short");
  uint32_t hdr[2];
  int32_t dims[6];
  int64_t tail[2];
  std::memcpy(hdr, b, 8);
  std::memcpy(dims, b + 8, 24);
  std::memcpy(tail, b + 32, 16);
  if (hdr[0] != CL_MAGIC || hdr[1] != 1) return fail(n->ctx, GW_EINVAL, "not a saved network");
  if (dims[0] != n->nin || dims[1] != n->width || dims[2] != n->depth || dims[3] != n->nout ||
      dims[4] != CL_KPAD || dims[5] != CL_OPAD || tail[1] != (int64_t)n->count)
    return fail(n->ctx, GW_EINVAL, "saved network has another shape");
  if (nbytes < 48 + 3 * n->count * 4) return fail(n->ctx, GW_EINVAL, "buffer too short");
  hipError_t e = hipStreamSynchronize(n->ctx->stream);
  if (e == hipSuccess) e = hipMemcpy(n->p, b + 48, n->count * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(n->m, b + 48 + n->count * 4, n->count * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(n->v, b + 48 + 2 * n->count * 4, n->count * 4, hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(n->ctx, e, "gw_mlp_load");
  n->step = tail[0];
  n->ready = true;
  return GW_OK;
}

gw_status gw_chi0_closure(gw_ctx* c, gw_mlp* net, int mode, int N, const double* qG,
                          const double* chi0_trunc, double gap, double emax,
                          const double* chi0_full, float lr, float* loss, double* chi0_out) {
  if (!c) return GW_EINVAL;
  c->err.clear();
  if (mode != GW_CLOSURE_INFER && mode != GW_CLOSURE_TRAIN_STEP && mode != GW_CLOSURE_FULL_FALLBACK)
    return fail(c, GW_EINVAL, "unknown closure mode");
  if (N <= 0 || N > 16384) return fail(c, GW_EINVAL, "neps must be in 1..16384");
  (void)hipSetDevice(c->device);
  const size_t nn = (size_t)N * N;
  if (mode == GW_CLOSURE_FULL_FALLBACK) {
    if (!chi0_full || !chi0_out) return fail(c, GW_EINVAL, "FULL_FALLBACK needs chi0_full and chi0_out");
    GW_HIP(c, hipMemcpyAsync(chi0_out, chi0_full, nn * 16, hipMemcpyDeviceToDevice, c->stream));
    return GW_OK;
  }
  if (!net || net->ctx != c) return fail(c, GW_EINVAL, "network missing or from another context");
  if (net->nin != CL_NFEAT || net->nout != CL_NOUT)
    return fail(c, GW_EINVAL, "the closure network maps %d features to %d outputs", CL_NFEAT, CL_NOUT);
  if (!qG || !chi0_trunc) return fail(c, GW_EINVAL, "NULL qG or chi0_trunc");
  if (mode == GW_CLOSURE_TRAIN_STEP && !chi0_full) return fail(c, GW_EINVAL, "training needs chi0_full");
  if (mode == GW_CLOSURE_INFER && !chi0_out) return fail(c, GW_EINVAL, "INFER needs chi0_out");
  if (mode == GW_CLOSURE_INFER && !net->ready)
    return fail(c, GW_ENOTTRAINED, "the network has not been trained or loaded");
  if (!(lr >= 0.f) && mode == GW_CLOSURE_TRAIN_STEP) return fail(c, GW_EINVAL, "negative learning rate");
  const long long n = (long long)N * (N + 1) / 2;
  const long long npad = (n + CL_RT - 1) / CL_RT * CL_RT;
  ClBufs b;
  const bool train = mode == GW_CLOSURE_TRAIN_STEP;
  gw_status st = cl_buffers(net, N, npad, train, &b);
  if (st != GW_OK) return st;
  const cpx<double>* ct = reinterpret_cast<const cpx<double>*>(chi0_trunc);
  const cpx<double>* cf = reinterpret_cast<const cpx<double>*>(chi0_full);
  {
    ProfScope ps(c, "closure_features");
    hipLaunchKernelGGL(k_cl_scale, dim3(1), dim3(256), 0, c->stream, ct, N, b.scale);
    GW_CHECK_LAUNCH(c, "k_cl_scale");
    hipLaunchKernelGGL(k_cl_features, dim3((unsigned)((npad + 255) / 256)), dim3(256), 0,
                       c->stream, qG, ct, train ? cf : nullptr, N, n, npad,
                       gap, emax, b.scale, b.X, train ? b.T : nullptr);
    GW_CHECK_LAUNCH(c, "k_cl_features");
  }
  if ((st = cl_forward(net, npad, b)) != GW_OK) return st;
  if (train) {
    const int nblk = (int)((npad + 255) / 256);
    {
      ProfScope ps(c, "closure_loss");
      hipLaunchKernelGGL(k_cl_dy, dim3(nblk), dim3(256), 0, c->stream, b.Y, b.T, n, npad, b.dY,
                         b.lpart);
      GW_CHECK_LAUNCH(c, "k_cl_dy");
      hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(256), 0, c->stream, b.lpart, nblk, b.loss);
      GW_CHECK_LAUNCH(c, "k_sum_f64");
    }
    if ((st = cl_backward(net, npad, b)) != GW_OK) return st;
    net->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float bc1 = 1.f - std::pow(b1, (float)net->step), bc2 = 1.f - std::pow(b2, (float)net->step);
    {
      ProfScope ps(c, "closure_adam");
      hipLaunchKernelGGL(k_adam, dim3((unsigned)((net->count + 255) / 256)), dim3(256), 0,
                         c->stream, net->p, b.part, cl_splits(net->count, npad), net->m, net->v,
                         net->count, lr, b1, b2, 1e-8f, bc1, bc2);
      GW_CHECK_LAUNCH(c, "k_adam");
    }
    net->ready = true;
    if (loss) {
      double l = 0.0;
      GW_HIP(c, hipMemcpyAsync(&l, b.loss, 8, hipMemcpyDeviceToHost, c->stream));
      GW_HIP(c, hipStreamSynchronize(c->stream));
      *loss = (float)(l / ((double)n * CL_NOUT));
    }
    return GW_OK;
  }
  // INFER
  {
    ProfScope ps(c, "closure_apply");
    hipLaunchKernelGGL(k_cl_apply, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, ct,
                       b.Y, N, n, b.scale, reinterpret_cast<cpx<double>*>(chi0_out));
    GW_CHECK_LAUNCH(c, "k_cl_apply");
  }
  if (chi0_full) {
    // the full sum judges the prediction: it is kept only if it is within the
    // network's tolerance of the full sum and negative semidefinite
    double rel = 0.0;
    if ((st = cl_rel_f(c, N, chi0_out, chi0_full, b, &rel)) != GW_OK) return st;
    bool fails = !(rel <= net->tol);
    if (!fails && (st = cl_cholesky_fails(c, N, chi0_out, b, &fails)) != GW_OK) return st;
    if (fails) {
      GW_HIP(c, hipMemcpyAsync(chi0_out, chi0_full, nn * 16, hipMemcpyDeviceToDevice, c->stream));
      return GW_EFALLBACK;
    }
  }
  return GW_OK;
}

}  // extern "C"
