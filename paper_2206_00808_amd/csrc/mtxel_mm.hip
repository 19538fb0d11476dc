// Spinor matrix elements (Sec. II, Eq. (matrix_el)) as dense pruned transforms on the
// matrix cores:
//   rho_vc(r) = sum_s conj(u_v^s(r)) u_c^s(r),
//   M_vc(G)   = (1/N) sum_j rho_vc(r_j) exp(+2 pi i g.j/n),  G on the eps sphere.
//
// Grid.  M_vc(G) is a convolution of two finite spheres: any grid with
// n_a > max|gv_a| + max|gc_a| + max|geps_a| gives it without aliasing, whatever box
// the fields are quoted on, so the products are formed on n_a equal to that sum
// plus one (22 x 23 x 24 points for a 48^3 box of the Si-like system, 26 x 26 x 67
// for 60 x 60 x 160: an eighth and a thirteenth of the points).  No factorisation of
// n_a is needed.
//
// Transforms.  With 13-15 of about 24 frequencies kept per axis, a dense real product
// with cos and sin columns costs no more than a pruned FFT with its twiddles, and
// runs on v_mfma_f64_16x16x4_f64 / v_mfma_f32_16x16x4_f32 from registers:
//   - a tile of 16 rows y by 16 columns (cos, sin of eight |g2|) of one plane's
//     products, contracted over the row (K = the row's entries);
//   - its result has rows y in registers and lane groups, which is the B operand of
//     the product over y: Or, Oi = [cos; sin](|g1| y) X, no exchange in between.
// Each lane forms the products rho it feeds to the matrix cores itself, from its
// conduction entries (registers, for all valence bands) and the valence plane (LDS).
// The real and imaginary parts of rho are separate real products; the four
// combinations (cos|sin) x (cos|sin) of a (|g1|, |g2|) pair are kept as a quad of
// complex values and unfolded to (+-g1, +-g2) after the last transform, inside the
// four lanes that hold them.
//
// Fields are stored in the order the fragments are read: element (y, z) of a plane at
// [y / 16][z / 4][lane], lane = 16 (z % 4) + l, y % 16 = row_of(l), so that every
// wavefront load is 64 consecutive elements.
//
// One call, before (pruned FFTs on the box, on the vector ALU) and after: 48^3 box,
// 16 x 800 pairs in double 5.10 -> 0.93 ms; 60 x 60 x 160 box in float 13.5 -> 2.23 ms;
// a box of unequal axes outside the FFTs' list of lengths 3.07 -> 0.19 ms.
#include "mtxel_mm.h"

#include <cmath>
#include <vector>

namespace gw {

namespace {

template <typename T> struct MmType;
template <> struct MmType<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mfma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <> struct MmType<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mfma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// A 16-row tile's row in operand position m whose result sits in register r of lane
// group q has the logical index 4 r + q in both types: the FP64 result has row
// 4 r + q there, the FP32 one row 4 q + r.
template <typename T>
__host__ __device__ __forceinline__ int row_of(int m) {
  return sizeof(T) == 8 ? m : 4 * (m & 3) + (m >> 2);
}

// Sums over K steps run in chunks of two: eight products through the accumulator,
// the chunks added outside it.  The matrix cores add their products to the
// accumulator one after the other, so that one chain over all n steps would round
// 4 n times at the size of the running sum.
using D4 = MmType<double>::v4;
template <typename T>
__device__ __forceinline__ typename MmType<T>::v4 mfma2(T a0, T b0, T a1, T b1, bool two) {
  typename MmType<T>::v4 c = {0, 0, 0, 0};
  c = MmType<T>::mfma(a0, b0, c);
  return two ? MmType<T>::mfma(a1, b1, c) : c;
}

template <typename T>
__device__ __forceinline__ cpx<double> widen(cpx<T> v) {
  return mk((double)v.x, (double)v.y);
}
// a, b the values at +g and -g: a + b for the cosine, i (a - b) for the sine
__device__ __forceinline__ cpx<double> fold(cpx<double> a, cpx<double> b, bool sine) {
  return sine ? mk(b.y - a.y, a.x - b.x) : a + b;
}

typedef __attribute__((address_space(3))) void lds_ptr;

// folded index kappa of an axis with frequencies -G..G: cos of 0..G, then sin of 1..G
__host__ __device__ __forceinline__ int kappa_g(int k, int G, bool* sine) {
  *sine = k > G;
  return k > G ? k - G : k;
}

// One sphere's bands: coefficients, compact cube, tables, and where the results go.
// The band kernels take two sets (valence, then conduction) in one launch.
template <typename T>
struct BandSet {
  const cpx<T>* coef;
  const int* cube;
  long long s0, s1, s2;                // cube strides
  int ng, nbs, G0, G1, G2, kx, ky, ntz;
  const double *bx, *by, *bz;
  cpx<T>*t1, *u;
};

// ---------------------------------------------------------------- bands, axis 0
// t1[bs][x][col] = sum_g c(g, col) exp(+2 pi i g x / n0) over the sphere's columns
// (axes 1, 2 of its compact cube).  A wavefront takes 16 columns: the coefficients
// folded over +-g go to LDS once, then every tile of 16 x is
// [cos | sin](x, kappa) times them, two real products.  The band transforms run in
// double for both types: they are bound by memory and latency, and single precision
// keeps only the roundings of the stored fields.  816 bands of 1993 G: 71 us (211 for
// pruned FFTs of whole pencils).
template <typename T>
__global__ void __launch_bounds__(256) k_mm_band_x(BandSet<T> bv, BandSet<T> bc, int kmax, int n0) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const bool val = (int)blockIdx.x < bv.nbs;
  const BandSet<T>& B = val ? bv : bc;
  const size_t bs = val ? blockIdx.x : blockIdx.x - bv.nbs;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, q = lane >> 4;
  cpx<double>* D = reinterpret_cast<cpx<double>*>(smem_raw) + (size_t)wave * kmax * 64 + lane;
  const int e2 = 2 * B.G2 + 1, ncol = (2 * B.G1 + 1) * e2, G0 = B.G0, ksteps = B.kx;
  const int col = (blockIdx.y * (blockDim.x >> 6) + wave) * 16 + l16;
  if (col - l16 >= ncol) return;  // whole wavefront
  const cpx<T>* cf = B.coef + bs * B.ng;
  const int j1 = col / e2, j2 = col - j1 * e2;
  const int* cb = B.cube + j1 * B.s1 + j2 * B.s2;
#pragma unroll 4
  for (int s = 0; s < ksteps; ++s) {
    bool sine;
    const int k = 4 * s + q, g = kappa_g(k, G0, &sine);
    const bool in = k <= 2 * G0 && col < ncol;
    const int ia = in ? cb[(G0 + g) * B.s0] : -1, ib = in && g ? cb[(G0 - g) * B.s0] : -1;
    // unconditional loads (of element 0 where the sphere has none), so that they overlap
    const cpx<double> a = widen(cf[max(ia, 0)]), b = widen(cf[max(ib, 0)]), z = mk(0.0, 0.0);
    D[s * 64] = fold(ia >= 0 ? a : z, ib >= 0 ? b : z, sine);
  }
  __builtin_amdgcn_wave_barrier();  // a wavefront reads its own region only, in order
  for (int xt = 0; 16 * xt < n0; ++xt) {
    D4 re = {0, 0, 0, 0}, im = re;
    const double* w = B.bx + (size_t)xt * ksteps * 64 + lane;
#pragma unroll 2
    for (int s = 0; s < ksteps; s += 2) {
      const bool two = s + 1 < ksteps;
      const int s1 = two ? s + 1 : s;
      const cpx<double> d0 = D[s * 64], d1 = D[s1 * 64];
      const double a0 = w[s * 64], a1 = w[s1 * 64];
      re += mfma2(a0, d0.x, a1, d1.x, two);
      im += mfma2(a0, d0.y, a1, d1.y, two);
    }
    if (col < ncol) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = 16 * xt + 4 * r + q;
        if (x < n0) B.t1[(bs * n0 + x) * ncol + col] = mk((T)re[r], (T)im[r]);
      }
    }
  }
}

// ---------------------------------------------------------------- bands, axes 1 and 2
// RT wavefronts per plane of one band and spinor component, one for each tile of 16 rows.
// The plane's t1, folded over +-g1, goes to LDS by tiles of eight +-g2 pairs (rows g2, +g2
// and -g2 of a pair in one lane), each wavefront a part; then for every tile of g2,
// Y(g2, y) = sum_g1 t1 exp(+2 pi i g1 y / n1), folded over +-g2 in place into the B
// operand of u(z, y) += sum_g2 [cos | sin](z, g2) Y, whose result is in the fragment
// order of the fields.  Bound: latency of its loads and of the dependent products.
// One wavefront for a plane's tiles in turn took 183 us for 16 x 800 bands in a 48^3 box and
// 221 for 56 x 250 in single precision in 60 x 60 x 160; here 178 and 231.
template <typename T, int JT>
__global__ void __launch_bounds__(256, 3) k_mm_band_plane(BandSet<T> bv, BandSet<T> bc, int kmax,
                                                       int n0, int ns, int rt, int ks,
                                                       size_t plane) {
  using D = MmType<double>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = wave % rt;
  const int slot = wave / rt;                              // plane of the workgroup
  int p = blockIdx.x * ((blockDim.x >> 6) / rt) + slot;    // (band, spin, x)
  const bool val = p < bv.nbs * n0;
  const BandSet<T>& B = val ? bv : bc;
  if (!val) p -= bv.nbs * n0;
  const bool mine = p < B.nbs * n0;
  if (!mine) p = 0;
  cpx<double>* S = reinterpret_cast<cpx<double>*>(smem_raw) + (size_t)slot * kmax * 64 + lane;
  const int G1 = B.G1, G2 = B.G2, ky = B.ky, lr = l16 >> 2, e2 = 2 * G2 + 1;
  const int bs = p / n0, x = p - bs * n0, band = bs / ns, sp = bs - band * ns;
  const cpx<T>* src = B.t1 + (size_t)p * (2 * G1 + 1) * e2;
  if (mine)
    for (int tz = 0; tz < B.ntz; ++tz) {
      // this lane's operand row: g2 = +-ga
      const int ga = 8 * tz + (l16 & 3) + 4 * (lr >> 1), g2 = (lr & 1) ? -ga : ga;
      const bool live = ga <= G2 && !((lr & 1) && ga == 0);
      const cpx<T>* row = src + (live ? G2 + g2 : 0);
#pragma unroll 4
      for (int s = t; s < ky; s += rt) {
        bool sine;
        const int k = 4 * s + q, g = kappa_g(k, G1, &sine);
        const bool in = live && k <= 2 * G1;
        const int gi = in ? g : 0;
        const cpx<double> a = widen(row[(G1 + gi) * e2]), b = widen(row[(G1 - gi) * e2]),
                          z = mk(0.0, 0.0);
        S[(tz * ky + s) * 64] = fold(in ? a : z, in && g ? b : z, sine);
      }
    }
  __syncthreads();
  if (!mine) return;
  cpx<T>* dst = B.u + ((size_t)band * n0 + x) * plane + (size_t)sp * rt * ks * 64 + lane;
  D4 ur[JT], ui[JT];
#pragma unroll
  for (int j = 0; j < JT; ++j) ur[j] = ui[j] = (D4){0, 0, 0, 0};
  for (int tz = 0; tz < B.ntz; ++tz) {
    D4 yr = {0, 0, 0, 0}, yi = yr;
    const double* w = B.by + (size_t)t * ky * 64 + lane;
#pragma unroll 2
    for (int s = 0; s < ky; s += 2) {
      const bool two = s + 1 < ky;
      const int s1 = two ? s + 1 : s;
      const cpx<double> d0 = S[(tz * ky + s) * 64], d1 = S[(tz * ky + s1) * 64];
      const double w0 = w[s * 64], w1 = w[s1 * 64];
      yr += mfma2(d0.x, w0, d1.x, w1, two);
      yi += mfma2(d0.y, w0, d1.y, w1, two);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (8 * tz + 4 * h > G2) break;
      const double pr = yr[2 * h] + yr[2 * h + 1], pi = yi[2 * h] + yi[2 * h + 1];
      const double mr = yr[2 * h] - yr[2 * h + 1], mi = yi[2 * h] - yi[2 * h + 1];
      const D4 none = {0, 0, 0, 0};
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        const double* wz = B.bz + ((size_t)(j * B.ntz + tz) * 4 + 2 * h) * 64 + lane;
        const double wc = wz[0], wsn = wz[64];
        const D4 cr = D::mfma(wc, pr, none), ci = D::mfma(wc, pi, none);
        ur[j] += D::mfma(wsn, -mi, cr);
        ui[j] += D::mfma(wsn, mr, ci);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < JT; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * j + r < ks)
        dst[(size_t)(t * ks + 4 * j + r) * 64] = mk((T)ur[j][r], (T)ui[j][r]);
}

// ---------------------------------------------------------------- pair planes
// A workgroup owns plane x, four conduction bands (one per wavefront, their plane in
// registers) and one tile of eight |g2|, and walks a range of valence bands: the next
// valence plane is loaded straight into the other half of LDS while this one is
// multiplied.  One barrier per valence band.  Writes
// t2[pair][x][quad][cos|sin 1][cos|sin 2], pair = (c - c0) nvt + (v - v0).
//
// Bound: matrix cores (2 RT KS + up to 8 RT products of 16 x 16 x 4 per pair and
// plane per row tile of |g1|); the valence plane is read from L2 once per four pairs.
// 12,800 pairs of the Si-like case in double: 485 us, 25.5 TFLOP/s of products without
// padding (4.9 ms for both halves of the FFT planes on the vector ALU).
// Registers of a band's entries, the result and output tiles and the coefficients, in
// words: up to these counts the kernels take at most 256 registers, two wavefronts per
// SIMD, without scratch memory (one spinor component keeps more loads ahead).
__host__ __device__ constexpr bool mm_band_fits(bool dbl, int ns, int rt, int ks) {
  return rt <= 3 && ks <= 12 &&
         (2 * ns * rt * ks + 8 * rt + 16 + ks) * (dbl ? 2 : 1) <= (ns == 2 ? 172 : 160);
}

template <typename T, int NS, int RT, int KS>
__global__ void __launch_bounds__(256, 2) k_mm_pair(
    const cpx<T>* __restrict__ uv, const cpx<T>* __restrict__ uc, size_t plane, int nvt, int nct,
    int nvs, int n0, int n1, int ncz, int nry, const T* __restrict__ zc, const T* __restrict__ yc,
    const int* __restrict__ qpos, int G1, int G2, int nq4, cpx<T>* __restrict__ t2) {
  using V = typename MmType<T>::v4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int CH = (NS * RT * KS * (int)sizeof(cpx<T>) * 64 + 1023) / 1024;  // KiB per plane
  const int ncg = (nct + 3) / 4;
  const long long lin = xcd_linear(blockIdx.x, (long long)n0 * nvs * ncg * ncz);
  if (lin < 0) return;
  const int ct = (int)(lin % ncz), cg = (int)((lin / ncz) % ncg), vx = (int)(lin / ncz / ncg);
  const int x = vx / nvs, vb = (int)((long long)nvt * (vx % nvs) / nvs),
            ve = (int)((long long)nvt * (vx % nvs + 1) / nvs);
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  T* Y = reinterpret_cast<T*>(smem_raw + 2 * CH * 1024);
  int* Qp = reinterpret_cast<int*>(Y + (size_t)nry * RT * 4 * 64);
  auto stage = [&](int v, int buf) {
    const char* src = reinterpret_cast<const char*>(uv + ((size_t)v * n0 + x) * plane);
#pragma unroll
    for (int i = wave; i < CH; i += 4)
      __builtin_amdgcn_global_load_lds((const void*)(src + i * 1024 + lane * 16),
                                       (lds_ptr*)(smem_raw + (buf * CH + i) * 1024), 16, 0, 0);
  };
  stage(vb, 0);
  for (int i = tid; i < nry * RT * 4 * 64; i += 256) Y[i] = yc[i];
  for (int i = tid; i < nry * 64; i += 256) {
    const int g1 = i >> 3, g2 = ct * 8 + (i & 7);
    const int qd = g1 <= G1 && g2 <= G2 ? qpos[g1 * (G2 + 1) + g2] : -1;
    Qp[i] = qd < 0 ? -1 : 4 * qd;
  }
  const int cl = cg * 4 + wave;
  const bool mine = cl < nct;
  cpx<T> cr[NS][RT][KS];
  {
    const cpx<T>* src = uc + ((size_t)(mine ? cl : nct - 1) * n0 + x) * plane + lane;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int k = 0; k < KS; ++k) cr[s][t][k] = src[((s * RT + t) * KS + k) * 64];
  }
  T z[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) z[k] = zc[((size_t)ct * KS + k) * 64 + lane];
  __syncthreads();  // plane 0 and the tables in place
  int qd0[2];       // first tile of |g1|: this lane's places in a plane's quads
#pragma unroll
  for (int h = 0; h < 2; ++h) qd0[h] = mine ? Qp[(4 * h + q) * 8 + (l16 >> 1)] : -1;
  for (int vl = vb; vl < ve; ++vl) {
    const int buf = (vl - vb) & 1;
    if (vl + 1 < ve) stage(vl + 1, buf ^ 1);
    const cpx<T>* P = reinterpret_cast<const cpx<T>*>(smem_raw + buf * CH * 1024) + lane;
    V xr[RT], xi[RT];
    // chunks of CK K steps of one row tile, in order: once this chunk's rho are
    // formed, the next chunk's valence entries are read and the last chunk's result is
    // added while this one's products run.  The barriers keep the compiler from
    // forming every rho at once.
    constexpr int CK = 2, NC = (KS + CK - 1) / CK, NCH = NC * RT;
    V pr, pi;
    cpx<T> d[CK][NS];
    auto read = [&](int ch) {
      const int t = ch % RT, k2 = ch / RT * CK;
#pragma unroll
      for (int i = 0; i < CK; ++i)
        if (k2 + i < KS) {
#pragma unroll
          for (int s = 0; s < NS; ++s) d[i][s] = P[((s * RT + t) * KS + k2 + i) * 64];
        }
    };
    auto add = [&](int ch) {
      const int t = ch % RT;
      xr[t] = ch < RT ? pr : xr[t] + pr;
      xi[t] = ch < RT ? pi : xi[t] + pi;
      // Here and not at the end, where every chunk's result would be held until then: of 36
      // rows in single precision 240 -> 212 us, of 32 and 16 rows up to 2% slower.
      if constexpr (RT == 3) asm volatile("" : "+v"(xr[t]), "+v"(xi[t]));
    };
    read(0);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int t = ch % RT, k2 = ch / RT * CK;
      T re[CK], im[CK];
#pragma unroll
      for (int i = 0; i < CK; ++i)
        if (k2 + i < KS) {
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            const cpx<T> v = d[i][s], c = cr[s][t][k2 + i];
            re[i] = s ? fma(v.x, c.x, fma(v.y, c.y, re[i])) : fma(v.x, c.x, v.y * c.y);
            im[i] = s ? fma(v.x, c.y, fma(-v.y, c.x, im[i])) : fma(v.x, c.y, -(v.y * c.x));
          }
        }
      __builtin_amdgcn_sched_barrier(0);
      if (ch + 1 < NCH) read(ch + 1);
      __builtin_amdgcn_sched_barrier(0);
      V ar = {0, 0, 0, 0}, ai = {0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < CK; ++i)
        if (k2 + i < KS) {
          ar = MmType<T>::mfma(re[i], z[k2 + i], ar);
          ai = MmType<T>::mfma(im[i], z[k2 + i], ai);
        }
      if (ch) add(ch - 1);
      pr = ar;
      pi = ai;
      __builtin_amdgcn_sched_barrier(0);
    }
    add(NCH - 1);
    cpx<T>* out = t2 + (((size_t)cl * nvt + vl) * n0 + x) * (size_t)nq4 * 4 + (l16 & 1);
    for (int ty = 0; ty < nry; ++ty) {
      V orr, oi;
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int r2 = 0; r2 < 4; r2 += CK)
          if (t + r2 == 0 || 16 * t + 4 * r2 < n1) {  // rows past n1 have zero coefficients
            V br = {0, 0, 0, 0}, bi = {0, 0, 0, 0};
#pragma unroll
            for (int r = r2; r < r2 + CK; ++r) {
              const T a = Y[((ty * RT + t) * 4 + r) * 64 + lane];
              br = MmType<T>::mfma(a, xr[t][r], br);
              bi = MmType<T>::mfma(a, xi[t][r], bi);
            }
            orr = t + r2 ? orr + br : br;
            oi = t + r2 ? oi + bi : bi;
          }
      // the next plane's loads (and the last band's stores) have had the products'
      // time; waited for here, so that this band's stores are not
      if (ty == 0) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int qd = qd0[h];
        if (ty) qd = mine ? Qp[(ty * 8 + 4 * h + q) * 8 + (l16 >> 1)] : -1;
        if (qd >= 0) {
          out[(unsigned)qd] = mk(orr[2 * h], oi[2 * h]);
          out[(unsigned)qd + 2] = mk(orr[2 * h + 1], oi[2 * h + 1]);
        }
      }
    }
    // every wavefront's loads have landed and its reads of this plane are complete (the
    // products have used them): a bare barrier, since a fence would wait for the stores
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
}

// ---------------------------------------------------------------- pair planes by rows
// The same for planes whose conduction entries do not fit one wavefront's registers
// (mm_band_fits): rt wavefronts share a band, each with the entries of 16 rows.  A
// wavefront forms its rows' products once for all NZ column tiles and contracts them over
// the entries.  Then, with at least one output tile for each wavefront (EX), the results
// X are exchanged through LDS and the wavefronts take the tiles in turn, K over all rows;
// with fewer, every wavefront contracts its own rows for each tile, and the rt partial
// results go through LDS (two buffers, one barrier per tile) and are added while the next
// tile's products run.  The valence entries come straight from L2 in fragment order, D K
// steps ahead.
//
// Bound: issue of the matrix cores and of the products on the same ALUs (44-55% of the
// cycles are the matrix cores'), with three wavefronts of a 48-row plane on four SIMDs.
// 16 x 64 pairs in double, pair planes: 48 points per axis 2484 -> 781 us, 40 points 1374
// -> 566 us (with a whole band per wavefront, 130-930 spilled bytes), 52 x 52 x 34 points
// 1031 -> 326 us (general transforms).  31 points, 16 x 128 pairs: 579 -> 441 us.
template <typename T, int NS, int KS>
constexpr int mm_rows_depth() {
  // K steps in flight: a divisor of KS, so that slots keep their place from band to band
  return KS == 4 || KS == 6 ? KS : KS == 8 || KS == 12 || KS == 16 ? 4 : KS / 2;
}
constexpr int kPartPitch = 66;  // entries per register of a partial tile in LDS

template <typename T, int NS, int KS, int NZ, bool EX>
__global__ void __launch_bounds__(256, 2) k_mm_pair_rows(
    const cpx<T>* __restrict__ uv, const cpx<T>* __restrict__ uc, size_t plane, int nvt, int nct,
    int nvs, int n0, int n1, int rt, int ct0, int nry, const T* __restrict__ zc,
    const T* __restrict__ yc, const int* __restrict__ qpos, int G1, int G2, int nq4,
    cpx<T>* __restrict__ t2) {
  using V = typename MmType<T>::v4;
  constexpr int D = mm_rows_depth<T, NS, KS>(), NCH = KS / 2;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), t = wave % rt, b = wave / rt;
  const int nb = (blockDim.x >> 6) / rt, ncg = (nct + nb - 1) / nb;
  const long long lin = xcd_linear(blockIdx.x, (long long)n0 * nvs * ncg);
  if (lin < 0) return;
  const int cg = (int)(lin % ncg), vx = (int)(lin / ncg), x = vx / nvs;
  const int vb = (int)((long long)nvt * (vx % nvs) / nvs),
            ve = (int)((long long)nvt * (vx % nvs + 1) / nvs);
  T* Z = reinterpret_cast<T*>(smem_raw);
  T* Y = Z + NZ * KS * 64;
  int* Qp = reinterpret_cast<int*>(Y + (size_t)nry * rt * 256);
  // partial tiles [2][rt][4][kPartPitch], or the results X [rt][NZ][4][64]
  cpx<T>* Ps = reinterpret_cast<cpx<T>*>(Qp + nry * NZ * 64) +
               (size_t)b * rt * (EX ? NZ * 256 : 8 * kPartPitch);
  const int cl = cg * nb + b;
  const bool mine = cl < nct;
  // valence entries of this wavefront's rows, D K steps ahead of their use
  // (uniform base and one lane offset: the steps' addresses take no vector registers)
  const cpx<T>* src = uv + ((size_t)vb * n0 + x) * plane + (size_t)t * KS * 64;
  const size_t sps = (size_t)rt * KS * 64;  // from spinor component to component
  cpx<T> d[D][NS], cr[NS][KS];
#pragma unroll
  for (int k = 0; k < D; ++k)
#pragma unroll
    for (int s = 0; s < NS; ++s) d[k][s] = (src + s * sps + k * 64)[lane];
  {
    const cpx<T>* c = uc + ((size_t)(mine ? cl : nct - 1) * n0 + x) * plane + (size_t)t * KS * 64;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int k = 0; k < KS; ++k) cr[s][k] = (c + s * sps + k * 64)[lane];
  }
  for (int i = tid; i < NZ * KS * 64; i += blockDim.x) Z[i] = zc[(size_t)ct0 * KS * 64 + i];
  for (int i = tid; i < nry * rt * 256; i += blockDim.x) Y[i] = yc[i];
  for (int i = tid; i < nry * NZ * 64; i += blockDim.x) {
    const int g1 = i / (NZ * 8), g2 = ct0 * 8 + i % (NZ * 8);
    const int qd = g1 <= G1 && g2 <= G2 ? qpos[g1 * (G2 + 1) + g2] : -1;
    Qp[i] = qd < 0 ? -1 : 4 * qd;
  }
  __syncthreads();
  // the sum of a tile's partials, stored as whole quads
  int par = 0, last = -1;
  cpx<T>* lout = t2;
  auto flush = [&]() {
    if (last < 0) return;
    const cpx<T>* P = Ps + (size_t)(par ^ 1) * rt * 4 * kPartPitch;
    for (int e = t * 64 + lane; e < 256; e += 64 * rt) {
      const int slot = e & 3, g2i = (e >> 2) & 7, g1i = e >> 5;
      const int at = (2 * (g1i >> 2) + (slot >> 1)) * kPartPitch + (g1i & 3) * 16 + 2 * g2i + (slot & 1);
      const int qd = mine ? Qp[last + g1i * NZ * 8 + g2i] : -1;
      cpx<T> v = P[at];
      for (int w = 1; w < rt; ++w) v = v + P[(size_t)w * 4 * kPartPitch + at];
      if (qd >= 0) lout[(unsigned)(qd + slot)] = v;
    }
  };
  for (int vl = vb; vl < ve; ++vl) {
    const cpx<T>* nsrc = vl + 1 < ve ? src + (size_t)n0 * plane : src;
    V xr[NZ], xi[NZ], pr, pi;
    int zl = lane;
    asm volatile("" : "+v"(zl));  // the coefficients stay in LDS
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      T re[2], im[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int k = 2 * ch + i;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const cpx<T> v = d[k % D][s], c = cr[s][k];
          re[i] = s ? fma(v.x, c.x, fma(v.y, c.y, re[i])) : fma(v.x, c.x, v.y * c.y);
          im[i] = s ? fma(v.x, c.y, fma(-v.y, c.x, im[i])) : fma(v.x, c.y, -(v.y * c.x));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int k = 2 * ch + i;
#pragma unroll
        for (int s = 0; s < NS; ++s)
          d[k % D][s] = k + D < KS ? (src + s * sps + (k + D) * 64)[lane]
                                   : (nsrc + s * sps + (k + D - KS) * 64)[lane];
      }
      T z[NZ][2];
#pragma unroll
      for (int c = 0; c < NZ; ++c)
#pragma unroll
        for (int i = 0; i < 2; ++i) z[c][i] = Z[(c * KS + 2 * ch + i) * 64 + zl];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < NZ; ++c) {
        V ar = {0, 0, 0, 0}, ai = {0, 0, 0, 0};
        ar = MmType<T>::mfma(re[0], z[c][0], ar);
        ai = MmType<T>::mfma(im[0], z[c][0], ai);
        ar = MmType<T>::mfma(re[1], z[c][1], ar);
        ai = MmType<T>::mfma(im[1], z[c][1], ai);
        // the result before this one
        const int it = ch * NZ + c - 1, pc = (it + NZ) % NZ;
        if (it >= 0) {
          xr[pc] = it < NZ ? pr : xr[pc] + pr;
          xi[pc] = it < NZ ? pi : xi[pc] + pi;
          // here and not at the end, where every chunk's result would be held until then
          asm volatile("" : "+v"(xr[pc]), "+v"(xi[pc]));
        }
        pr = ar;
        pi = ai;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    xr[NZ - 1] = NCH == 1 ? pr : xr[NZ - 1] + pr;
    xi[NZ - 1] = NCH == 1 ? pi : xi[NZ - 1] + pi;
    cpx<T>* out = t2 + (((size_t)cl * nvt + vl) * n0 + x) * (size_t)nq4 * 4;
    // bare barriers: a fence would wait for the stores and loads in flight
    auto barrier = [] {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    if constexpr (EX) {
      barrier();  // the last band's X has been read
#pragma unroll
      for (int c = 0; c < NZ; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) Ps[((t * NZ + c) * 4 + r) * 64 + lane] = mk(xr[c][r], xi[c][r]);
      barrier();
      for (int i = t; i < nry * NZ; i += rt) {
        const int ty = i / NZ, c = i - ty * NZ;
        const cpx<T>* X = Ps + c * 256 + lane;
        const T* y = Y + (size_t)ty * rt * 256 + lane;
        cpx<T> xf[4];
        T yf[4];
        auto fetch = [&](int w) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            xf[r] = X[(size_t)w * NZ * 256 + r * 64];
            yf[r] = y[w * 256 + r * 64];
          }
        };
        fetch(0);
        V o_r = {0, 0, 0, 0}, o_i = {0, 0, 0, 0};
        for (int w = 0; w < rt; ++w) {
          cpx<T> xc[4];
          T yc4[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            xc[r] = xf[r];
            yc4[r] = yf[r];
          }
          if (w + 1 < rt) fetch(w + 1);
          V a_r = {0, 0, 0, 0}, a_i = {0, 0, 0, 0}, b_r = {0, 0, 0, 0}, b_i = {0, 0, 0, 0};
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            a_r = MmType<T>::mfma(yc4[r], xc[r].x, a_r);
            a_i = MmType<T>::mfma(yc4[r], xc[r].y, a_i);
          }
          if (16 * w + 8 < n1) {  // rows past n1 have zero coefficients
#pragma unroll
            for (int r = 2; r < 4; ++r) {
              b_r = MmType<T>::mfma(yc4[r], xc[r].x, b_r);
              b_i = MmType<T>::mfma(yc4[r], xc[r].y, b_i);
            }
          }
          o_r = (o_r + a_r) + b_r;
          o_i = (o_i + a_i) + b_i;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int qd = mine ? Qp[(ty * 8 + 4 * h + (lane >> 4)) * NZ * 8 + c * 8 + ((lane & 15) >> 1)] : -1;
          if (qd >= 0) {
            out[(unsigned)(qd + (lane & 1))] = mk(o_r[2 * h], o_i[2 * h]);
            out[(unsigned)(qd + 2 + (lane & 1))] = mk(o_r[2 * h + 1], o_i[2 * h + 1]);
          }
        }
      }
    } else {
#pragma unroll
      for (int c = 0; c < NZ; ++c)
        for (int ty = 0; ty < nry; ++ty) {
          const T* y = Y + (size_t)(ty * rt + t) * 256 + lane;
          V o_r = {0, 0, 0, 0}, o_i = {0, 0, 0, 0};
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const T a = y[r * 64];
            o_r = MmType<T>::mfma(a, xr[c][r], o_r);
            o_i = MmType<T>::mfma(a, xi[c][r], o_i);
          }
          if (16 * t + 8 < n1) {  // rows past n1 have zero coefficients
            V b_r = {0, 0, 0, 0}, b_i = {0, 0, 0, 0};
#pragma unroll
            for (int r = 2; r < 4; ++r) {
              const T a = y[r * 64];
              b_r = MmType<T>::mfma(a, xr[c][r], b_r);
              b_i = MmType<T>::mfma(a, xi[c][r], b_i);
            }
            o_r += b_r;
            o_i += b_i;
          }
          flush();
          cpx<T>* P = Ps + (size_t)(par * rt + t) * 4 * kPartPitch + lane;
#pragma unroll
          for (int r = 0; r < 4; ++r) P[r * kPartPitch] = mk(o_r[r], o_i[r]);
          last = ty * 8 * NZ * 8 + c * 8;
          lout = out;
          par ^= 1;
          barrier();  // this tile's partials are written, and the last tile's have been read
        }
    }
    src = nsrc;
  }
  if constexpr (!EX) flush();
}

// ---------------------------------------------------------------- axis 0 and scatter
__device__ __forceinline__ float quad_swap(float v, bool two) {
  const int i = __float_as_int(v);
  return __int_as_float(two ? __builtin_amdgcn_mov_dpp(i, 0x4E, 0xf, 0xf, true)
                            : __builtin_amdgcn_mov_dpp(i, 0xB1, 0xf, 0xf, true));
}
__device__ __forceinline__ double quad_swap(double v, bool two) {
  const long long b = __double_as_longlong(v);
  const int lo = (int)b, hi = (int)(b >> 32);
  const int l2 = two ? __builtin_amdgcn_mov_dpp(lo, 0x4E, 0xf, 0xf, true)
                     : __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xf, 0xf, true);
  const int h2 = two ? __builtin_amdgcn_mov_dpp(hi, 0x4E, 0xf, 0xf, true)
                     : __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xf, 0xf, true);
  return __longlong_as_double(((long long)h2 << 32) | (unsigned)l2);
}
// lane bit set: other - i own, clear: own + i other (own the sin, the other the cos
// value of the pair when the bit is set)
template <typename T>
__device__ __forceinline__ cpx<T> unfold_sign(cpx<T> v, bool bit, bool two) {
  const cpx<T> o = mk(quad_swap(v.x, two), quad_swap(v.y, two));
  return bit ? mk(o.x + v.y, o.y - v.x) : mk(v.x - o.y, v.y + o.x);
}

// One wavefront per pair and tile of four quads: C, S(|g0|) = [cos; sin] t2 over the
// planes (t2 read once, 16 lanes on consecutive values), then +-g0 from C +- i S,
// +-g2 and +-g1 by exchanges inside the quad, 1/N, and the scatter onto the eps
// sphere through tab[tile][|g0|][sign][16] (index or -1).  The tiles of a pair run
// on one XCD, where its scattered stores fill whole lines.  |g0| tiles i0 .. i0 + NX - 1
// of nx (a second launch reads t2 again when there are more).  Bound: memory; the 12,800
// pairs of the Si-like case take 205 us (417 with FFTs from the box's planes).
template <typename T, int NX>
__global__ void __launch_bounds__(256) k_mm_pair_x(const cpx<T>* __restrict__ t2, int n0, int nq4,
                                                   int kx, int i0, int nx,
                                                   const T* __restrict__ xc,
                                                   const int* __restrict__ tab, T invN, int nvt,
                                                   int c0, int nc_total, int neps,
                                                   long long ntasks, cpx<T>* __restrict__ M) {
  using V = typename MmType<T>::v4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* X = reinterpret_cast<T*>(smem_raw);
  const long long lin = xcd_linear(blockIdx.x, (ntasks + 3) / 4);
  if (lin < 0) return;
  for (int i = threadIdx.x; i < NX * kx * 64; i += 256) X[i] = xc[(size_t)i0 * kx * 64 + i];
  __syncthreads();
  const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
  const long long task = lin * 4 + (threadIdx.x >> 6);
  if (task >= ntasks) return;
  const int nt = nq4 / 4;
  const int pr = (int)(task / nt), tile = (int)(task - (long long)pr * nt);
  const int ld = nq4 * 4, last = n0 - 1;
  const cpx<T>* src = t2 + (size_t)pr * n0 * ld + tile * 16 + l16;
  // in float, two running sums per result, of every other chunk: the axis of the planes
  // is the long one (67 points in the layered cell)
  constexpr bool kTwo = sizeof(T) == 4;
  V ar[NX], ai[NX], br[NX], bi[NX];
#pragma unroll
  for (int i = 0; i < NX; ++i) ar[i] = ai[i] = br[i] = bi[i] = (V){0, 0, 0, 0};
  // four K steps at a time, the next four in flight
  constexpr int U = 4;
  cpx<T> b[U];
  auto fetch = [&](int s) {
#pragma unroll
    for (int i = 0; i < U; ++i) b[i] = src[(unsigned)(min(4 * (s + i) + q, last) * ld)];
  };
  fetch(0);
#pragma unroll 1
  for (int s = 0; s < kx; s += U) {
    cpx<T> d[U];
#pragma unroll
    for (int i = 0; i < U; ++i) d[i] = b[i];
    if (s + U < kx) fetch(s + U);
#pragma unroll
    for (int h = 0; h < U; h += 2)
      if (s + h < kx) {
        const bool two = s + h + 1 < kx;
        const int s1 = two ? s + h + 1 : s + h;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
          const T a0 = X[(i * kx + s + h) * 64 + lane], a1 = X[(i * kx + s1) * 64 + lane];
          V &sr = h && kTwo ? br[i] : ar[i], &si = h && kTwo ? bi[i] : ai[i];
          sr += mfma2<T>(a0, d[h].x, a1, d[h + 1].x, two);
          si += mfma2<T>(a0, d[h].y, a1, d[h + 1].y, two);
        }
      }
  }
  if constexpr (kTwo) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      ar[i] += br[i];
      ai[i] += bi[i];
    }
  }
  const int v = pr % nvt, c = c0 + pr / nvt;
  cpx<T>* dst = M + ((size_t)v * nc_total + c) * neps;
  const bool bz = l16 & 1, by = l16 & 2;
#pragma unroll
  for (int i = 0; i < NX; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const T cre = ar[i][2 * h], cim = ai[i][2 * h], sre = ar[i][2 * h + 1],
              sim = ai[i][2 * h + 1];
      const int* tb = tab + (((size_t)tile * nx + i0 + i) * 8 + 4 * h + q) * 32 + l16;
#pragma unroll
      for (int sg = 0; sg < 2; ++sg) {
        cpx<T> w = sg ? mk(cre + sim, cim - sre) : mk(cre - sim, cim + sre);
        w = unfold_sign<T>(unfold_sign<T>(w, bz, false), by, true);
        const int idx = tb[16 * sg];
        if (idx >= 0) dst[idx] = scal(w, invN);
      }
    }
}

// ---------------------------------------------------------------- tables
// cos and sin(2 pi m / n) with the argument folded to the first octant
void root(long long m, int n, double* c, double* s) {
  m %= n;
  if (m < 0) m += n;
  const long long q = (4 * m) / n, rem = 4 * m - q * n;
  double cc, ss;
  if (2 * rem <= n) {
    const double a = (M_PI / 2.0) * (double)rem / (double)n;
    cc = std::cos(a);
    ss = std::sin(a);
  } else {
    const double a = (M_PI / 2.0) * (double)(n - rem) / (double)n;
    cc = std::sin(a);
    ss = std::cos(a);
  }
  *c = q == 0 ? cc : q == 1 ? -ss : q == 2 ? -cc : ss;
  *s = q == 0 ? ss : q == 1 ? cc : q == 2 ? -ss : -cc;
}
double trig(bool sine, long long m, int n) {
  double c, s;
  root(m, n, &c, &s);
  return sine ? s : c;
}

struct Blob {
  std::vector<char> h;
  size_t begin() {
    h.resize(align_up(h.size()));
    return h.size();
  }
  void put(double v, bool as_double = true) {
    const float f = (float)v;
    const char* p = reinterpret_cast<const char*>(&v);
    if (!as_double) p = reinterpret_cast<const char*>(&f);
    h.insert(h.end(), p, p + (as_double ? 8 : 4));
  }
  void put_int(int v) {
    const char* p = reinterpret_cast<const char*>(&v);
    h.insert(h.end(), p, p + 4);
  }
};

int lrow(bool dbl, int m) { return dbl ? row_of<double>(m) : row_of<float>(m); }

// output rows: logical 4 r + q is |g| = 8 tile + q + 4 (r / 2), cos for even r
void put_out_rows(Blob& b, bool dbl, int tiles, int ksteps, int G, int n) {
  for (int t = 0; t < tiles; ++t)
    for (int s = 0; s < ksteps; ++s)
      for (int l = 0; l < 64; ++l) {
        const int i = lrow(dbl, l & 15), r = i >> 2, g = 8 * t + (i & 3) + 4 * (r >> 1);
        const int k = 4 * s + (l >> 4);
        b.put(g <= G && k < n ? trig(r & 1, (long long)g * k, n) : 0.0, dbl);
      }
}

int fold_steps(int g) { return (2 * g + 1 + 3) / 4; }

void put_band(Blob& b, const MmTables& t, const int* g, MmTables::Band* o) {
  o->kx = fold_steps(g[0]);
  o->ky = fold_steps(g[1]);
  o->ntz = g[2] / 8 + 1;
  o->ncol = (2 * g[1] + 1) * (2 * g[2] + 1);
  o->bx = b.begin();
  for (int xt = 0; 16 * xt < t.n[0]; ++xt)
    for (int s = 0; s < o->kx; ++s)
      for (int l = 0; l < 64; ++l) {
        bool sine;
        const int k = 4 * s + (l >> 4), f = kappa_g(k, g[0], &sine);
        const int x = 16 * xt + (l & 15);
        b.put(k <= 2 * g[0] && x < t.n[0] ? trig(sine, (long long)f * x, t.n[0]) : 0.0);
      }
  o->by = b.begin();
  for (int rt = 0; rt < t.rt; ++rt)
    for (int s = 0; s < o->ky; ++s)
      for (int l = 0; l < 64; ++l) {
        bool sine;
        const int k = 4 * s + (l >> 4), f = kappa_g(k, g[1], &sine);
        const int y = 16 * rt + lrow(t.dbl, l & 15);
        b.put(k <= 2 * g[1] && y < t.n[1] ? trig(sine, (long long)f * y, t.n[1]) : 0.0);
      }
  o->bz = b.begin();
  for (int j = 0; j < t.jt; ++j)
    for (int tz = 0; tz < o->ntz; ++tz)
      for (int hs = 0; hs < 4; ++hs)  // h, cos | sin
        for (int l = 0; l < 64; ++l) {
          const int z = 16 * j + (l & 15), f = 8 * tz + 4 * (hs >> 1) + (l >> 4);
          b.put(f <= g[2] && z < t.n[2] ? trig(hs & 1, (long long)f * z, t.n[2]) : 0.0);
        }
}

// K steps and row tiles the pair kernels are built for
constexpr int kKs[] = {2, 3, 4, 5, 6, 7, 8, 10, 12}, kKsRows[] = {4, 6, 8, 10, 12, 14, 16};
constexpr int kMaxRt = 4, kMaxNx = 4, kMaxNz = 3;
constexpr size_t kLds = 160 * 1024;

size_t pair_lds(bool dbl, int ns, int rt, int ks, int nry) {
  const size_t ch = ((size_t)ns * rt * ks * (dbl ? 1024 : 512) + 1023) / 1024;
  return 2 * ch * 1024 + (size_t)nry * rt * 4 * 64 * (dbl ? 8 : 4) + (size_t)nry * 64 * 4;
}
// bands of a workgroup of the rows kernel, whether it exchanges X, and its LDS
int rows_bands(int rt) { return rt == 1 ? 4 : rt == 2 ? 2 : 1; }
bool rows_exchange(int rt, int nz, int nry) { return nry * nz >= rt; }
size_t rows_lds(bool dbl, int rt, int ks, int nz, int nry) {
  const size_t w = dbl ? 8 : 4;
  return ((size_t)nz * ks * 64 + (size_t)nry * rt * 256) * w + (size_t)nry * nz * 256 +
         (size_t)rows_bands(rt) * rt * (rows_exchange(rt, nz, nry) ? nz * 256 : 8 * kPartPitch) *
             2 * w;
}
size_t pairx_lds(bool dbl, int nx, int kx) {
  return (size_t)std::min(nx, kMaxNx) * kx * 64 * (dbl ? 8 : 4);
}
// wavefronts (or planes) per workgroup of the band transforms, at most `most`, with `k` KiB
// of folded entries each: fewer where that puts half as many again on a CU (of 16)
int band_waves(int k, int most) {
  auto on_cu = [k](int w) { return std::min(16, 160 / (w * k) * w); };
  int best = most;
  for (int w = most - 1; w >= 1; --w)
    if (2 * on_cu(w) >= 3 * on_cu(best)) best = w;
  return best;
}

// Intermediate and band fields of a chunk of conduction bands.  Chunks that stay in the
// 256 MB last-level cache were slower: the Si-like case took 1.22 ms in chunks of 96 MB,
// 1.07 of 192 and 400 MB, 1.01 of 1,600 MB, the layered one 3.48, 3.01, 2.71 and
// 2.54 ms; short launches cost more than the reads from HBM.
constexpr size_t kChunkBytes = 1536ull << 20;
constexpr long long kPairGroups = 1500;

struct MmSizes {
  int ct;  // conduction bands per chunk
  size_t uv, uc, t1, t1v, t2;
};
MmSizes mm_sizes(const MmTables& t, int nv, int nc) {
  const size_t el = t.dbl ? 16 : 8;
  const size_t t2_band = (size_t)nv * t.n[0] * t.eps->nq4 * 4 * el;
  const size_t u_band = (size_t)t.n[0] * t.plane * el;
  const size_t t1_c = (size_t)t.nspinor * t.n[0] * t.bc.ncol * el;
  const size_t t1_v = (size_t)t.nspinor * t.n[0] * t.bv.ncol * el;
  MmSizes s;
  const size_t per = t2_band + u_band;
  long long ct = std::max<long long>(4, (long long)(kChunkBytes / per) / 4 * 4);
  s.ct = (int)std::min<long long>(ct, nc);
  s.uv = u_band * nv + 1024;  // planes are staged in whole KiB
  s.uc = u_band * s.ct;
  s.t1 = t1_c * s.ct;
  s.t1v = t1_v * (size_t)nv;
  s.t2 = t2_band * s.ct;
  return s;
}

template <typename K>
hipError_t allow(gw_ctx* c, K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <typename T>
BandSet<T> band_set(const MmTables& t, bool val, int nb, int ng, const cpx<T>* coef, cpx<T>* t1,
                    cpx<T>* u) {
  const int* g = val ? t.gv : t.gc;
  const long long* st = val ? t.sv : t.sc;
  const MmTables::Band& b = val ? t.bv : t.bc;
  auto tab = [&](size_t o) { return reinterpret_cast<const double*>(t.grid->p + o); };
  return BandSet<T>{coef, val ? t.cube_v : t.cube_c, st[0], st[1], st[2], ng, nb * t.nspinor, g[0],
                    g[1], g[2], b.kx, b.ky, b.ntz, tab(b.bx), tab(b.by), tab(b.bz), t1, u};
}

// coefficients -> fields in fragment order, valence and conduction in one launch each
template <typename T>
gw_status run_bands(gw_ctx* c, const MmTables& t, const BandSet<T>& v, const BandSet<T>& k) {
  const int kx = std::max(v.kx, k.kx), nw = band_waves(kx, 4);
  const int ky = std::max(v.ky * v.ntz, k.ky * k.ntz), nwp = band_waves(ky, 4 / t.rt);
  const int ncol = std::max(t.bv.ncol, t.bc.ncol), nbs = v.nbs + k.nbs;
  const size_t lx = (size_t)nw * kx * 1024, lp = (size_t)nwp * ky * 1024;
  {
    ProfScope ps(c, "band_xpass");
    if (!c->capturing) GW_HIP(c, allow(c, k_mm_band_x<T>, lx));
    hipLaunchKernelGGL(k_mm_band_x<T>, dim3(nbs, (ncol + 16 * nw - 1) / (16 * nw)), dim3(64 * nw),
                       lx, c->stream, v, k, kx, t.n[0]);
    GW_CHECK_LAUNCH(c, "k_mm_band_x");
  }
  ProfScope ps(c, "band_plane");
  const dim3 gr((unsigned)(((long long)nbs * t.n[0] + nwp - 1) / nwp)), bl(64 * nwp * t.rt);
#define GW_MM_BP(J)                                                                             \
  if (t.jt == J) {                                                                              \
    if (!c->capturing) GW_HIP(c, allow(c, k_mm_band_plane<T, J>, lp));                          \
    hipLaunchKernelGGL((k_mm_band_plane<T, J>), gr, bl, lp, c->stream, v, k, ky, t.n[0],         \
                       t.nspinor, t.rt, t.ks, t.plane);                                         \
  }
  GW_MM_BP(1) GW_MM_BP(2) GW_MM_BP(3) GW_MM_BP(4)
#undef GW_MM_BP
  GW_CHECK_LAUNCH(c, "k_mm_band_plane");
  return GW_OK;
}

template <typename T, int NS, int RT, int KS>
gw_status launch_pair(gw_ctx* c, const MmTables& t, const cpx<T>* uv, const cpx<T>* uc, int nv,
                      int nct, cpx<T>* t2) {
  auto k = k_mm_pair<T, NS, RT, KS>;
  const size_t lds = pair_lds(sizeof(T) == 8, NS, RT, KS, t.nry);
  if (!c->capturing) GW_HIP(c, allow(c, k, lds));
  // valence ranges: enough workgroups to even out over the CUs, of at least six bands
  const long long base = (long long)t.n[0] * ((nct + 3) / 4) * t.ncz;
  const int nvs = (int)std::max<long long>(1, std::min<long long>(nv / 6, (kPairGroups - 1) / base + 1));
  const long long tot = base * nvs;
  hipLaunchKernelGGL(k, dim3((unsigned)((tot + kXcd - 1) / kXcd * kXcd)), dim3(256), lds,
                     c->stream, uv, uc, t.plane, nv, nct, nvs, t.n[0], t.n[1], t.ncz, t.nry,
                     reinterpret_cast<const T*>(t.grid->p + t.o_zc),
                     reinterpret_cast<const T*>(t.grid->p + t.o_yc),
                     reinterpret_cast<const int*>(t.eps->dev.p + t.eps->o_qpos), t.ge[1], t.ge[2], t.eps->nq4, t2);
  GW_CHECK_LAUNCH(c, "k_mm_pair");
  return GW_OK;
}

template <typename T, int NS, int KS, int NZ>
gw_status launch_rows(gw_ctx* c, const MmTables& t, const cpx<T>* uv, const cpx<T>* uc, int nv,
                      int nct, int ct0, cpx<T>* t2) {
  auto* k = rows_exchange(t.rt, NZ, t.nry) ? &k_mm_pair_rows<T, NS, KS, NZ, true>
                                           : &k_mm_pair_rows<T, NS, KS, NZ, false>;
  const size_t lds = rows_lds(sizeof(T) == 8, t.rt, KS, NZ, t.nry);
  if (!c->capturing) GW_HIP(c, allow(c, k, lds));
  const int nb = rows_bands(t.rt);
  const long long base = (long long)t.n[0] * ((nct + nb - 1) / nb);
  const int nvs = (int)std::max<long long>(1, std::min<long long>(nv / 6, (kPairGroups - 1) / base + 1));
  const long long tot = base * nvs;
  hipLaunchKernelGGL(k, dim3((unsigned)((tot + kXcd - 1) / kXcd * kXcd)), dim3(64 * t.rt * nb), lds,
                     c->stream, uv, uc, t.plane, nv, nct, nvs, t.n[0], t.n[1], t.rt, ct0, t.nry,
                     reinterpret_cast<const T*>(t.grid->p + t.o_zc),
                     reinterpret_cast<const T*>(t.grid->p + t.o_yc),
                     reinterpret_cast<const int*>(t.eps->dev.p + t.eps->o_qpos), t.ge[1], t.ge[2],
                     t.eps->nq4, t2);
  GW_CHECK_LAUNCH(c, "k_mm_pair_rows");
  return GW_OK;
}

// column tiles in launches of up to kMaxNz, evenly
template <typename T, int NS, int KS>
gw_status run_rows(gw_ctx* c, const MmTables& t, const cpx<T>* uv, const cpx<T>* uc, int nv,
                   int nct, cpx<T>* t2) {
  const int parts = (t.ncz + kMaxNz - 1) / kMaxNz;
  for (int i = 0; i < parts; ++i) {
    const int c0 = t.ncz * i / parts, nz = t.ncz * (i + 1) / parts - c0;
    gw_status st = nz == 1   ? launch_rows<T, NS, KS, 1>(c, t, uv, uc, nv, nct, c0, t2)
                   : nz == 2 ? launch_rows<T, NS, KS, 2>(c, t, uv, uc, nv, nct, c0, t2)
                             : launch_rows<T, NS, KS, 3>(c, t, uv, uc, nv, nct, c0, t2);
    if (st != GW_OK) return st;
  }
  return GW_OK;
}

template <typename T, int NS, int RT, int KS>
gw_status band_or_rows(gw_ctx* c, const MmTables& t, const cpx<T>* uv, const cpx<T>* uc, int nv,
                       int nct, cpx<T>* t2) {
  if constexpr (mm_band_fits(sizeof(T) == 8, NS, RT, KS))
    return launch_pair<T, NS, RT, KS>(c, t, uv, uc, nv, nct, t2);
  return fail(c, GW_EUNSUPPORTED, "no pair kernel for %d row tiles, %d K steps", RT, KS);
}

template <typename T, int NS, int RT>
gw_status pick_ks(gw_ctx* c, const MmTables& t, const cpx<T>* uv, const cpx<T>* uc, int nv, int nct,
                  cpx<T>* t2) {
  switch (t.ks) {
    case 2: return band_or_rows<T, NS, RT, 2>(c, t, uv, uc, nv, nct, t2);
    case 3: return band_or_rows<T, NS, RT, 3>(c, t, uv, uc, nv, nct, t2);
    case 4: return band_or_rows<T, NS, RT, 4>(c, t, uv, uc, nv, nct, t2);
    case 5: return band_or_rows<T, NS, RT, 5>(c, t, uv, uc, nv, nct, t2);
    case 6: return band_or_rows<T, NS, RT, 6>(c, t, uv, uc, nv, nct, t2);
    case 7: return band_or_rows<T, NS, RT, 7>(c, t, uv, uc, nv, nct, t2);
    case 8: return band_or_rows<T, NS, RT, 8>(c, t, uv, uc, nv, nct, t2);
    case 10: return band_or_rows<T, NS, RT, 10>(c, t, uv, uc, nv, nct, t2);
    case 12: return band_or_rows<T, NS, RT, 12>(c, t, uv, uc, nv, nct, t2);
  }
  return fail(c, GW_EUNSUPPORTED, "no pair kernel for %d K steps", t.ks);
}

template <typename T, int NS>
gw_status run_pairs(gw_ctx* c, const MmTables& t, const cpx<T>* uv, const cpx<T>* uc, int nv,
                    int nct, cpx<T>* t2) {
  if (t.rows) {
    switch (t.ks) {
      case 4: return run_rows<T, NS, 4>(c, t, uv, uc, nv, nct, t2);
      case 6: return run_rows<T, NS, 6>(c, t, uv, uc, nv, nct, t2);
      case 8: return run_rows<T, NS, 8>(c, t, uv, uc, nv, nct, t2);
      case 10: return run_rows<T, NS, 10>(c, t, uv, uc, nv, nct, t2);
      case 12: return run_rows<T, NS, 12>(c, t, uv, uc, nv, nct, t2);
      case 14: return run_rows<T, NS, 14>(c, t, uv, uc, nv, nct, t2);
      case 16: return run_rows<T, NS, 16>(c, t, uv, uc, nv, nct, t2);
    }
    return fail(c, GW_EUNSUPPORTED, "no pair kernel for %d K steps", t.ks);
  }
  if (t.rt == 1) return pick_ks<T, NS, 1>(c, t, uv, uc, nv, nct, t2);
  if (t.rt == 2) return pick_ks<T, NS, 2>(c, t, uv, uc, nv, nct, t2);
  return pick_ks<T, NS, 3>(c, t, uv, uc, nv, nct, t2);
}

template <typename T>
gw_status run_mtxel(gw_ctx* c, const MmTables& t, int nv, int ngv, const cpx<T>* cv, int nc,
                    int ngc, const cpx<T>* cc, cpx<T>* M, char* ws) {
  const MmSizes s = mm_sizes(t, nv, nc);
  cpx<T>* uv = reinterpret_cast<cpx<T>*>(ws);
  ws += align_up(s.uv);
  cpx<T>* uc = reinterpret_cast<cpx<T>*>(ws);
  ws += align_up(s.uc);
  cpx<T>* t1 = reinterpret_cast<cpx<T>*>(ws);
  ws += align_up(s.t1) + align_up(s.t1v);
  cpx<T>* t2 = reinterpret_cast<cpx<T>*>(ws);
  cpx<T>* t1v = reinterpret_cast<cpx<T>*>(reinterpret_cast<char*>(t1) + align_up(s.t1));
  for (int c0 = 0; c0 < nc; c0 += s.ct) {
    const int nct = std::min(s.ct, nc - c0);
    gw_status st = run_bands<T>(
        c, t, band_set<T>(t, true, c0 ? 0 : nv, ngv, cv, t1v, uv),
        band_set<T>(t, false, nct, ngc, cc + (size_t)c0 * t.nspinor * ngc, t1, uc));
    if (st != GW_OK) return st;
    {
      ProfScope ps(c, "pair_plane");
      st = t.nspinor == 2 ? run_pairs<T, 2>(c, t, uv, uc, nv, nct, t2)
                          : run_pairs<T, 1>(c, t, uv, uc, nv, nct, t2);
      if (st != GW_OK) return st;
    }
    ProfScope ps(c, "pair_xpass");
    const long long tasks = (long long)nv * nct * (t.eps->nq4 / 4), blocks = (tasks + 3) / 4;
    const dim3 gr((unsigned)((blocks + kXcd - 1) / kXcd * kXcd)), bl(256);
    const T invN = (T)(1.0 / ((double)t.n[0] * t.n[1] * t.n[2]));
    for (int i0 = 0; i0 < t.nx; i0 += kMaxNx) {
      const int nx = std::min(kMaxNx, t.nx - i0);
      const size_t xl = pairx_lds(sizeof(T) == 8, nx, t.kx);
#define GW_MM_PX(N)                                                                              \
  if (nx == N) {                                                                                 \
    if (!c->capturing) GW_HIP(c, allow(c, k_mm_pair_x<T, N>, xl));                               \
    hipLaunchKernelGGL((k_mm_pair_x<T, N>), gr, bl, xl, c->stream, t2, t.n[0], t.eps->nq4, t.kx, i0,   \
                       t.nx, reinterpret_cast<const T*>(t.grid->p + t.o_xc),                         \
                       reinterpret_cast<const int*>(t.eps->dev.p + t.eps->o_tab), invN, nv, c0, nc, t.neps,  \
                       tasks, M);                                                                \
  }
      GW_MM_PX(1) GW_MM_PX(2) GW_MM_PX(3) GW_MM_PX(4)
#undef GW_MM_PX
      GW_CHECK_LAUNCH(c, "k_mm_pair_x");
    }
  }
  return GW_OK;
}

}  // namespace

DevBuf::~DevBuf() {
  if (p) (void)hipFree(p);
}

static bool being_captured(gw_ctx* c) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  return c->stream && hipStreamIsCapturing(c->stream, &cap) == hipSuccess &&
         cap != hipStreamCaptureStatusNone;
}

// Bounded caches: their entries are given back when they pass kCacheBytes together
// (freeing waits for the device), but not during a capture.  What a plan or a captured
// graph reads is held elsewhere too.
constexpr size_t kCacheBytes = 256u << 20;
template <typename M>
static void bound_cache(M* cache, size_t* bytes, size_t more, bool capture) {
  if (*bytes + more > kCacheBytes && !capture) {
    cache->clear();
    *bytes = 0;
  }
  *bytes += more;
}

// Axis order and coefficient tables for the spheres' largest |g|; null when no kernel is
// built for them.
static gw_status grid_tables(gw_ctx* c, const SphereMap* sv, const SphereMap* sc,
                             const SphereMap* se, int nspinor, bool dbl,
                             std::shared_ptr<MmTables>* out) {
  // the axis order with the least matrix-core time and intermediate traffic per pair
  // among those the kernels are built for
  auto t = std::make_shared<MmTables>();
  t->dbl = dbl;
  t->nspinor = nspinor;
  const double cyc = dbl ? 64.0 : 32.0, el = dbl ? 16.0 : 8.0;
  double best = INFINITY;
  static const int perms[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
  for (const auto& p : perms) {
    int n[3], g[3];
    for (int a = 0; a < 3; ++a) {
      g[a] = se->gmax[p[a]];
      n[a] = sv->gmax[p[a]] + sc->gmax[p[a]] + g[a] + 1;
    }
    const int rt = (n[1] + 15) / 16, need = (n[2] + 3) / 4;
    const int ncz = g[2] / 8 + 1, nry = g[1] / 8 + 1, nx = g[0] / 8 + 1, kx = (n[0] + 3) / 4;
    int ks = 0;
    for (int k : kKs)
      if (!ks && k >= need) ks = k;
    const bool rows = !ks || !mm_band_fits(dbl, nspinor, rt, ks) ||
                      pair_lds(dbl, nspinor, rt, ks, nry) > kLds;
    if (rows) {
      ks = 0;
      for (int k : kKsRows)
        if (!ks && k >= need) ks = k;
    }
    if (rt > kMaxRt || !ks || (rows && rows_lds(dbl, rt, ks, std::min(ncz, kMaxNz), nry) > kLds) ||
        pairx_lds(dbl, nx, kx) > kLds ||
        (size_t)fold_steps(std::max(sv->gmax[p[0]], sc->gmax[p[0]])) * 1024 > kLds ||
        (size_t)std::max(fold_steps(sv->gmax[p[1]]) * (sv->gmax[p[2]] / 8 + 1),
                         fold_steps(sc->gmax[p[1]]) * (sc->gmax[p[2]] / 8 + 1)) * 1024 > kLds)
      continue;
    // 16 x 16 x 4 products per pair over 1,024 SIMDs; the intermediate written and
    // read at about 1.6 bytes per SIMD and cycle
    // (the rows kernel keeps the matrix cores busy for two thirds of the time that the
    // other does: 64 x 21 x 22 points in single precision 136 us, 21 x 64 x 22 by rows 180)
    const double mm = n[0] * (double)ncz * (2.0 * rt * ks + 2.0 * nry * ((n[1] + 3) / 4)) * cyc *
                      (rows ? 1.4 : 1.0);
    const double tr = n[0] * (g[1] + 1.0) * (g[2] + 1.0) * 4.0 * 2.0 * el / 1.6;
    if (mm + tr < best) {
      best = mm + tr;
      t->rt = rt;
      t->ks = ks;
      t->rows = rows;
      t->jt = (ks + 3) / 4;
      t->ncz = ncz;
      t->nry = nry;
      t->nx = nx;
      t->kx = kx;
      for (int a = 0; a < 3; ++a) {
        t->perm[a] = p[a];
        t->n[a] = n[a];
        t->ge[a] = g[a];
        t->gv[a] = sv->gmax[p[a]];
        t->gc[a] = sc->gmax[p[a]];
        const long long stv[3] = {(long long)sv->ext[1] * sv->ext[2], sv->ext[2], 1};
        const long long stc[3] = {(long long)sc->ext[1] * sc->ext[2], sc->ext[2], 1};
        t->sv[a] = stv[p[a]];
        t->sc[a] = stc[p[a]];
      }
    }
  }
  if (best == INFINITY) return GW_OK;
  t->plane = (size_t)nspinor * t->rt * t->ks * 64;
  const int G0 = t->ge[0], G1 = t->ge[1], G2 = t->ge[2];
  Blob b;
  t->o_zc = b.begin();
  for (int ct = 0; ct < t->ncz; ++ct)
    for (int s = 0; s < t->ks; ++s)
      for (int l = 0; l < 64; ++l) {
        const int z = 4 * s + (l >> 4), g = ct * 8 + ((l & 15) >> 1);
        b.put(z < t->n[2] && g <= G2 ? trig(l & 1, (long long)g * z, t->n[2]) : 0.0, dbl);
      }
  t->o_yc = b.begin();
  put_out_rows(b, dbl, t->nry, t->rt * 4, G1, t->n[1]);
  t->o_xc = b.begin();
  put_out_rows(b, dbl, t->nx, t->kx, G0, t->n[0]);
  put_band(b, *t, t->gv, &t->bv);
  put_band(b, *t, t->gc, &t->bc);
  t->grid = std::make_shared<DevBuf>();
  gw_status st = upload(c, b.h.data(), b.h.size(), &t->grid->p);
  t->grid->bytes = b.h.size();
  if (st == GW_OK) *out = t;
  return st;
}

static gw_status eps_tables(gw_ctx* c, const MmTables& t, const SphereMap* se,
                            const int32_t* geps, std::shared_ptr<MmEps>* out) {
  const int G0 = t.ge[0], G1 = t.ge[1], G2 = t.ge[2];
  auto x = std::make_shared<MmEps>();
  Blob b;
  // quads (|g1|, |g2|) with a point of the eps sphere, and its compact index map
  const int e1 = 2 * G1 + 1, e2 = 2 * G2 + 1;
  std::vector<int> map((size_t)(2 * G0 + 1) * e1 * e2, -1), qpos((size_t)(G1 + 1) * (G2 + 1), -1);
  std::vector<std::pair<int, int>> quads;
  for (int i = 0; i < se->n; ++i) {
    const int g0 = geps[3 * i + t.perm[0]], g1 = geps[3 * i + t.perm[1]],
              g2 = geps[3 * i + t.perm[2]];
    map[((size_t)(g0 + G0) * e1 + g1 + G1) * e2 + g2 + G2] = i;
    qpos[(size_t)std::abs(g1) * (G2 + 1) + std::abs(g2)] = 0;
  }
  for (int g1 = 0; g1 <= G1; ++g1)
    for (int g2 = 0; g2 <= G2; ++g2) {
      int& q = qpos[(size_t)g1 * (G2 + 1) + g2];
      if (q < 0) continue;
      q = (int)quads.size();
      quads.push_back({g1, g2});
    }
  x->nq = (int)quads.size();
  x->nq4 = (x->nq + 3) / 4 * 4;
  x->o_qpos = b.begin();
  for (int q : qpos) b.put_int(q);
  x->o_tab = b.begin();
  for (int tile = 0; tile < x->nq4 / 4; ++tile)
    for (int g = 0; g < 8 * t.nx; ++g)
      for (int sg = 0; sg < 2; ++sg)
        for (int l = 0; l < 16; ++l) {
          const int q = tile * 4 + l / 4, s1 = (l >> 1) & 1, s2 = l & 1;
          int idx = -1;
          if (q < x->nq && g <= G0) {
            const int g1 = quads[q].first, g2 = quads[q].second;
            if (!(sg && !g) && !(s1 && !g1) && !(s2 && !g2))
              idx = map[((size_t)((sg ? -g : g) + G0) * e1 + (s1 ? -g1 : g1) + G1) * e2 +
                        (s2 ? -g2 : g2) + G2];
          }
          b.put_int(idx);
        }
  gw_status st = upload(c, b.h.data(), b.h.size(), &x->dev.p);
  x->dev.bytes = b.h.size();
  if (st == GW_OK) *out = x;
  return st;
}

gw_status mm_tables(gw_ctx* c, const SphereMap* sv, const SphereMap* sc, const SphereMap* se,
                    const int32_t* geps, int nspinor, bool dbl, std::shared_ptr<MmTables>* out) {
  out->reset();
  const bool capture = being_captured(c);
  MmGridKey key{};
  for (int a = 0; a < 3; ++a) {
    key[a] = sv->gmax[a];
    key[3 + a] = sc->gmax[a];
    key[6 + a] = se->gmax[a];
  }
  key[9] = 2 * nspinor + dbl;
  auto it = c->mm_grid.find(key);
  if (it == c->mm_grid.end()) {
    std::shared_ptr<MmTables> t;
    gw_status st = grid_tables(c, sv, sc, se, nspinor, dbl, &t);
    if (st != GW_OK) return st;
    bound_cache(&c->mm_grid, &c->mm_grid_bytes, t ? t->grid->bytes : 256, capture);
    it = c->mm_grid.emplace(key, t).first;
  }
  if (!it->second) return GW_OK;
  auto t = std::make_shared<MmTables>(*it->second);
  t->cube_v = sv->d_cube;
  t->cube_c = sc->d_cube;
  t->neps = se->n;
  // sphere maps are the context's, one per set of G vectors, for its lifetime
  const auto ek = std::make_pair(se, 9 * t->perm[0] + 3 * t->perm[1] + t->perm[2]);
  auto ie = c->mm_eps.find(ek);
  if (ie == c->mm_eps.end()) {
    std::shared_ptr<MmEps> e;
    gw_status st = eps_tables(c, *t, se, geps, &e);
    if (st != GW_OK) return st;
    bound_cache(&c->mm_eps, &c->mm_eps_bytes, e->dev.bytes, capture);
    ie = c->mm_eps.emplace(ek, e).first;
  }
  t->eps = ie->second;
  if (capture) {
    c->mm_held.insert(t->grid);
    c->mm_held.insert(t->eps);
  }
  *out = t;
  return GW_OK;
}

size_t mm_workspace(const MmTables& t, int nv, int nc) {
  const MmSizes s = mm_sizes(t, nv, nc);
  return align_up(s.uv) + align_up(s.uc) + align_up(s.t1) + align_up(s.t1v) + align_up(s.t2);
}

gw_status mm_mtxel(gw_ctx* c, const MmTables& t, int nv, int ngv, const void* cv, int nc, int ngc,
                   const void* cc, void* mtxel, void* ws) {
  char* w = static_cast<char*>(ws);
  return t.dbl ? run_mtxel<double>(c, t, nv, ngv, static_cast<const cpx<double>*>(cv), nc, ngc,
                                   static_cast<const cpx<double>*>(cc),
                                   static_cast<cpx<double>*>(mtxel), w)
               : run_mtxel<float>(c, t, nv, ngv, static_cast<const cpx<float>*>(cv), nc, ngc,
                                  static_cast<const cpx<float>*>(cc),
                                  static_cast<cpx<float>*>(mtxel), w);
}

}  // namespace gw
