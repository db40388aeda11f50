// Matrix-core transforms of short and odd-length axes (fm_mat.h): the x
// passes and the fused y-z pass of the spectral part of an iteration.
//
//  k_mat_xf     x forward: rows of the (Anderson-combined) residual ->
//               spectral planes T[kx][z][y], y fastest.
//  k_mat_plane  one block per (component, kx) plane: y forward, z forward,
//               Green operator, z inverse, y inverse.  The plane lives in
//               LDS between the axes, the z spectrum in registers, so global
//               memory sees one read and one write of the plane.
//  k_mat_xi     x inverse and the displacement update.
//
// Roles: the half matrices are the A operand of v_mfma_*_16x16x4 (lane l
// holds row l & 15, column group l >> 4), the data the B operand (lane l
// holds pencil l & 15).  The result has pencil l & 15 in every lane and rows
// mdim(l >> 4, r) in register r; the inverse z product takes the scaled
// result registers as its B operand directly, its matrix columns being
// stored in that order.
#include <hip/hip_runtime.h>

#include "fm_fft.h"
#include "fm_mat.h"

namespace fm {

namespace {

template <typename R> struct V4T;
template <> struct V4T<float> { typedef float t __attribute__((ext_vector_type(4))); };
template <> struct V4T<double> { typedef double t __attribute__((ext_vector_type(4))); };
template <typename R> using V4 = typename V4T<R>::t;
// the same at the alignment of one real (row starts are not aligned)
template <typename R> struct U4T;
template <> struct U4T<float> { typedef float t __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct U4T<double> { typedef double t __attribute__((ext_vector_type(4), aligned(8))); };
template <typename R> using U4 = typename U4T<R>::t;
template <typename R> struct U2T;
template <> struct U2T<float> { typedef float t __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct U2T<double> { typedef double t __attribute__((ext_vector_type(2), aligned(8))); };
template <typename R> using U2 = typename U2T<R>::t;

__device__ __forceinline__ V4<float> mfma(float a, float b, V4<float> c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ V4<double> mfma(double a, double b, V4<double> c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Row of register r of lane group g in a 16-row result tile.
template <typename R>
__host__ __device__ __forceinline__ constexpr int mdim(int g, int r) {
  return sizeof(R) == 4 ? 4 * g + r : 4 * r + g;
}

// Fragments of one 16-row tile of both half matrices.  They are fetched one
// row tile ahead of their use, so that their latency overlaps the products
// of the tile before.
template <typename R, int KT>
struct Frag {
  V4<R> a[KT], b[KT];
  __device__ __forceinline__ void load(const void* fU, const void* fV, int mt, int kt, int lane) {
    const FM_GLOBAL R* pU = gconst((const R*)fU) + mt * kt * 256 + lane * 4;
    const FM_GLOBAL R* pV = gconst((const R*)fV) + mt * kt * 256 + lane * 4;
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const int tc = t < kt ? t : 0;
      a[t] = *(const FM_GLOBAL V4<R>*)(pU + tc * 256);
      b[t] = *(const FM_GLOBAL V4<R>*)(pV + tc * 256);
    }
  }
};

// Both half products of one row tile for NS sets of pencils: u = P e,
// v = Q o.  Straight-line over the KT column tiles (operands of tiles past an
// axis' own are zero); the last one takes the rl steps that hold data, one
// or all four.  The steps accumulate in four chains (two where the registers
// of FP64 pairs do not hold four, eight from KT = 4 on), added at the end:
// the rounding error of a chain grows with the square root of its length
// (relative error of the FP32 Green operator at n = 100, 51 columns: 3.4e-7
// in one chain, 2.0e-7 in four, 2.0e-7 by the axis passes).  A chain takes even and odd nodes in
// turn, so that the alternating sums of the highest frequencies, which the
// HEX1 Green operator amplifies most, cancel as they are formed.
template <typename R, int KT, int NS>
__device__ __forceinline__ void mat_tile(const Frag<R, KT>& f, int rl, const V4<R> (&e)[NS][KT],
                                         const V4<R> (&o)[NS][KT], V4<R> (&u)[NS], V4<R> (&v)[NS]) {
  constexpr int CH = sizeof(R) == 8 ? (NS == 2 ? 2 : 4) : (NS == 1 && KT >= 4 ? 8 : 4);
  V4<R> uc[NS][CH], vc[NS][CH];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int r = 0; r < CH; ++r) uc[s][r] = vc[s][r] = (V4<R>)((R)0);
  auto step = [&](int t, int r) {
    const int c = (r >> 1) + 2 * (t & (CH / 2 - 1));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      uc[s][c] = mfma(f.a[t][r], e[s][t][r], uc[s][c]);
      vc[s][c] = mfma(f.b[t][r], o[s][t][r], vc[s][c]);
    }
  };
#pragma unroll
  for (int t = 0; t + 1 < KT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) step(t, r);
  step(KT - 1, 0);
  if (rl > 1) {
#pragma unroll
    for (int r = 1; r < 4; ++r) step(KT - 1, r);
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int w = CH / 2; w > 0; w >>= 1)
#pragma unroll
      for (int c = 0; c < w; ++c) {
        uc[s][c] += uc[s][c + w];
        vc[s][c] += vc[s][c + w];
      }
    u[s] = uc[s][0];
    v[s] = vc[s][0];
  }
}

// Forward operands of all tiles from a row contiguous in memory.  Lane group
// g takes nodes 16 t + 4 g .. + 3 and their mirror images (MC_SPLIT: nodes
// 2 (16 t + 4 g) .. + 7).  Every load is unconditional, at an index clamped
// into the row, so that all of them are in flight together; columns past the
// half matrix are zero there.
template <typename R, int KT>
struct RowRaw {
  V4<R> a[KT], b[KT];
  __device__ __forceinline__ void load(const FM_GLOBAL R* row, const MatAxis& x, int kt, int g) {
    const int n = x.n, h = n >> 1;
    if (x.cls != MC_SPLIT) {
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        // q <= h implies q + 3 <= n and n - q - 3 >= 0 for n >= 4
        const int q = min(16 * t + 4 * g, h & ~3);
        a[t] = (V4<R>)(*(const FM_GLOBAL U4<R>*)(row + q));
        b[t] = (V4<R>)(*(const FM_GLOBAL U4<R>*)(row + n - q - 3));
      }
    } else {
      // all tiles but the last lie in the row (n >= 32 (kt - 1))
#pragma unroll
      for (int t = 0; t + 1 < KT; ++t) {
        const int q = min(2 * (16 * t + 4 * g), max(n - 7, 0));
        a[t] = (V4<R>)(*(const FM_GLOBAL U4<R>*)(row + q));
        b[t] = (V4<R>)(*(const FM_GLOBAL U4<R>*)(row + min(q + 4, n - 3)));
      }
      V4<R> la, lb;
      const int j0 = 2 * (16 * (kt - 1) + 4 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        la[r] = row[min(j0 + r, n)];
        lb[r] = row[min(j0 + 4 + r, n)];
      }
#pragma unroll
      for (int t = 0; t < KT; ++t)
        if (t + 1 >= kt) { a[t] = la; b[t] = lb; }
    }
  }
  // Fold or split; nodes that carry no data (0 and n, by kind) enter as zero
  // whatever the memory holds.
  __device__ __forceinline__ void operands(const MatAxis& x, int kt, int g, V4<R> (&e)[KT], V4<R> (&o)[KT]) const {
    const int n = x.n, h = n >> 1;
    if (x.cls != MC_SPLIT) {
      const bool no0 = x.j0 > 0, non = x.j1 <= n;
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const bool first = min(16 * t + 4 * g, h & ~3) == 0;
        V4<R> m;
        m[0] = first && non ? (R)0 : b[t][3];
        m[1] = b[t][2]; m[2] = b[t][1]; m[3] = b[t][0];
        V4<R> v = a[t];
        v[0] = first && no0 ? (R)0 : v[0];
        e[t] = t < kt ? v + m : (V4<R>)((R)0);
        o[t] = t < kt ? v - m : (V4<R>)((R)0);
      }
    } else {
      const bool odd = x.kind == K_DST3;
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        V4<R> ev, ov;
        ev[0] = a[t][0]; ev[1] = a[t][2]; ev[2] = b[t][0]; ev[3] = b[t][2];
        ov[0] = a[t][1]; ov[1] = a[t][3]; ov[2] = b[t][1]; ov[3] = b[t][3];
        if (t == 0) ev[0] = (g == 0 && odd) ? (R)0 : ev[0];
        if (t + 1 >= kt) {      // DCT-III: node n
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = 2 * (16 * t + 4 * g + r);
            ev[r] = j < x.j1 ? ev[r] : (R)0;
            ov[r] = j + 1 < x.j1 ? ov[r] : (R)0;
          }
        }
        e[t] = odd ? ov : ev;
        o[t] = odd ? ev : ov;
      }
    }
  }
};

// The value as one the compiler knows nothing about: indexes formed from it
// inside a loop stay there, instead of taking a register each before it.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Sum and difference of two operand sets (the halves of a MC_SPLIT or
// MC_CPLX transform).
template <typename V>
__device__ __forceinline__ void butterfly(V& a, V& b) {
  const V s = a + b, t = a - b;
  a = s;
  b = t;
}

// Plane of slot a of half U / V after the x transform (complex: the real and
// imaginary planes of a frequency are neighbours).
__device__ __forceinline__ int plane_U(const MatAxis& x, int a) { return x.kind == K_DFT ? 2 * a : a; }
__device__ __forceinline__ int plane_V(const MatAxis& x, int a) { return x.kind == K_DFT ? 2 * a + 1 : x.cU + a; }

// ---------------------------------------------------------------------------
// x forward.  One wavefront per 16 rows, rows read as quads, spectral planes
// written with the 16 rows contiguous.
template <typename R, int KT>
__global__ void __launch_bounds__(64 * MAT_WAVES) k_mat_xf(const MatDesc* __restrict__ descs,
                                                           const int2* __restrict__ work) {
  const int2 wk = work[blockIdx.x];
  const MatDesc& d = descs[wk.x];
  const FM_GLOBAL Ctrl* C = gconst(d.ctrl);
  const MatAxis x = d.x[0];
  const int lane = threadIdx.x & 63, g = lane >> 4, p = lane & 15;
  const int64_t NR = (int64_t)(d.x[1].n + 1) * (d.x[2].n + 1);
  const int64_t r0 = ((int64_t)wk.y * MAT_WAVES + (threadIdx.x >> 6)) * 16;
  if (r0 >= NR || C->status != ST_RUNNING) return;
  Frag<R, KT> f;
  f.load(x.fU, x.fV, 0, KT, lane);
  V4<R> e[1][KT], o[1][KT];
  {
    const int64_t row = min(r0 + p, NR - 1) * (x.n + 1);
    const FM_GLOBAL R* ring = gconst((const R*)d.D);
    const int64_t stride = d.ring_stride;
    const int nd = C->n_d;
    RowRaw<R, KT> raw;
    raw.load(ring + C->slot_d[0] * stride + row, x, KT, g);
    {
      const R a0 = (R)C->alpha[0];
#pragma unroll
      for (int t = 0; t < KT; ++t) { raw.a[t] *= a0; raw.b[t] *= a0; }
    }
    for (int q = 1; q < nd; ++q) {      // Anderson combination
      RowRaw<R, KT> rq;
      rq.load(ring + C->slot_d[q] * stride + row, x, KT, g);
      const R aq = (R)C->alpha[q];
#pragma unroll
      for (int t = 0; t < KT; ++t) { raw.a[t] += aq * rq.a[t]; raw.b[t] += aq * rq.b[t]; }
    }
    raw.operands(x, KT, g, e[0], o[0]);
  }
  FM_GLOBAL R* T = gmut((R*)d.T) + r0 + p;
  const bool okr = r0 + p < NR;
  for (int mt = 0; mt < KT; ++mt) {
    V4<R> u[1], v[1];
    Frag<R, KT> fn;
    fn.load(x.fU, x.fV, mt + 1 < KT ? mt + 1 : 0, KT, lane);
    mat_tile<R, KT, 1>(f, x.rlf, e, o, u, v);
    f = fn;
    if (x.cls == MC_SPLIT) butterfly(u[0], v[0]);
    if (!okr) continue;
    if (16 * mt + 15 < x.cV) {      // (cV <= cU)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * mt + mdim<R>(g, r);
        T[plane_U(x, a) * NR] = u[0][r];
        T[plane_V(x, a) * NR] = v[0][r];
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * mt + mdim<R>(g, r);
        if (a < x.cU) T[plane_U(x, a) * NR] = u[0][r];
        if (a < x.cV) T[plane_V(x, a) * NR] = v[0][r];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// x inverse and displacement update u^f += w - sum_k beta_k delta_k; the new
// increment goes into the ring (FP64 accumulator).
template <typename R, int KT>
__global__ void __launch_bounds__(64 * MAT_WAVES) k_mat_xi(const MatDesc* __restrict__ descs,
                                                           const int2* __restrict__ work) {
  const int2 wk = work[blockIdx.x];
  const MatDesc& d = descs[wk.x];
  const FM_GLOBAL Ctrl* C = gconst(d.ctrl);
  const MatAxis x = d.x[0];
  const int lane = threadIdx.x & 63, g = lane >> 4, p = lane & 15;
  const int64_t NR = (int64_t)(d.x[1].n + 1) * (d.x[2].n + 1);
  const int64_t r0 = ((int64_t)wk.y * MAT_WAVES + (threadIdx.x >> 6)) * 16;
  if (r0 >= NR) return;
  Frag<R, KT> f;
  f.load(x.iU, x.iV, 0, KT, lane);
  V4<R> e[1][KT], o[1][KT];
  {
    const FM_GLOBAL R* T = gconst((const R*)d.T) + min(r0 + p, NR - 1);
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * t + mdim<R>(g, r);
        e[0][t][r] = T[plane_U(x, min(a, x.cU - 1)) * NR];
        o[0][t][r] = T[plane_V(x, max(min(a, x.cV - 1), 0)) * NR];
      }
    // (slots past the halves repeat the last one)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int a = 16 * (KT - 1) + mdim<R>(g, r);
      e[0][KT - 1][r] = a < x.cU ? e[0][KT - 1][r] : (R)0;
      o[0][KT - 1][r] = a < x.cV ? o[0][KT - 1][r] : (R)0;
      if (KT > 1) o[0][KT > 1 ? KT - 2 : 0][r] = a - 16 < x.cV ? o[0][KT > 1 ? KT - 2 : 0][r] : (R)0;
    }
    if (x.cls == MC_SPLIT)
#pragma unroll
      for (int t = 0; t < KT; ++t) butterfly(e[0][t], o[0][t]);
  }
  if (C->status != ST_RUNNING) return;
  const int nb = C->n_b;
  const FM_GLOBAL R* ring = gconst((const R*)d.delta);
  const int64_t stride = d.ring_stride;
  FM_GLOBAL R* dw = gmut((R*)d.delta) + (int64_t)C->slot_w * stride;
  FM_GLOBAL double* uf = gmut(d.uf);
  auto upd1 = [&](int64_t i, R w) {
    for (int q = 0; q < nb; ++q) w -= (R)C->beta[q] * ring[C->slot_b[q] * stride + i];
    dw[i] = w;
    uf[i] += (double)w;
  };
  // two quads of consecutive nodes
  auto upd4 = [&](int64_t i, V4<R> w, int64_t i2, V4<R> w2) {
    U4<double> a = *(const FM_GLOBAL U4<double>*)(uf + i), a2 = *(const FM_GLOBAL U4<double>*)(uf + i2);
    for (int q = 0; q < nb; ++q) {
      const FM_GLOBAL R* ds = ring + C->slot_b[q] * stride;
      const V4<R> b = (V4<R>)(*(const FM_GLOBAL U4<R>*)(ds + i)), b2 = (V4<R>)(*(const FM_GLOBAL U4<R>*)(ds + i2));
      const R be = (R)C->beta[q];
      w -= be * b;
      w2 -= be * b2;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      a[r] += (double)w[r];
      a2[r] += (double)w2[r];
    }
    *(FM_GLOBAL U4<R>*)(dw + i) = (U4<R>)w;
    *(FM_GLOBAL U4<R>*)(dw + i2) = (U4<R>)w2;
    *(FM_GLOBAL U4<double>*)(uf + i) = a;
    *(FM_GLOBAL U4<double>*)(uf + i2) = a2;
  };
  const int n = x.n, h = n >> 1;
  const bool okr = r0 + p < NR;
  const int64_t row = (r0 + p) * (x.n + 1);
  for (int mt = 0; mt < KT; ++mt) {
    V4<R> u[1], v[1];
    Frag<R, KT> fn;
    fn.load(x.iU, x.iV, mt + 1 < KT ? mt + 1 : 0, KT, lane);
    mat_tile<R, KT, 1>(f, x.rli, e, o, u, v);
    f = fn;
    if (!okr) continue;
    const int q = 16 * mt + 4 * g;
    if (x.cls != MC_SPLIT) {
      V4<R> A = u[0], B = v[0];
      butterfly(A, B);
      if (sizeof(R) == 4 && 2 * (q + 3) < n) {
        V4<R> Br;
        Br[0] = B[3]; Br[1] = B[2]; Br[2] = B[1]; Br[3] = B[0];
        upd4(row + q, A, row + n - q - 3, Br);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = 16 * mt + mdim<R>(g, r);
          if (j <= h) upd1(row + j, A[r]);
          if (2 * j < n) upd1(row + n - j, B[r]);
        }
      }
    } else {
      const bool odd = x.kind == K_DST3;     // U holds the odd nodes
      const V4<R> A = odd ? v[0] : u[0], B = odd ? u[0] : v[0];
      if (sizeof(R) == 4 && 2 * q + 7 <= n) {
        V4<R> lo, hi;
        lo[0] = A[0]; lo[1] = B[0]; lo[2] = A[1]; lo[3] = B[1];
        hi[0] = A[2]; hi[1] = B[2]; hi[2] = A[3]; hi[3] = B[3];
        upd4(row + 2 * q, lo, row + 2 * q + 4, hi);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = 2 * (16 * mt + mdim<R>(g, r));
          if (j <= n) upd1(row + j, A[r]);
          if (j + 1 <= n) upd1(row + j + 1, B[r]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// y and z transforms, Green operator and their inverses on one kx plane.
//
// Per-column Green data: den(kz) = A cos^2(xi_z/2) + B sin^2(xi_z/2).
template <typename R>
__device__ __forceinline__ void green_ab(const MatDesc& d, double s0, double c0, double s1, double c1, R& A, R& B) {
  double a[3], b[3];
  if (d.scheme == 0) {
    a[0] = s0 * c1; a[1] = c0 * s1; a[2] = 0;
    b[0] = 0; b[1] = 0; b[2] = c0 * c1;
  } else {
    a[0] = s0 * c1; a[1] = c0 * s1; a[2] = s0 * s1;
    b[0] = c0 * s1; b[1] = s0 * c1; b[2] = c0 * c1;
  }
  const double lam = d.green_lam ? d.lam0 : 0.0;
  const double f = 4.0 / (d.h * d.h);
  A = (R)(f * (2.0 * d.mu0 * (a[0] + a[1] + a[2]) + lam * a[d.q]));
  B = (R)(f * (2.0 * d.mu0 * (b[0] + b[1] + b[2]) + lam * b[d.q]));
}

template <typename R> __device__ __forceinline__ R rcp_of(R x) { return (R)1 / x; }
template <> __device__ __forceinline__ float rcp_of<float>(float x) { return __builtin_amdgcn_rcpf(x); }

// 1 / den, 0 on the null modes (exact zeros of den) and on slots without a
// frequency (their table entries are zero).  sc: (sin^2, cos^2) pair.
template <typename R>
__device__ __forceinline__ R green_f(R A, R B, const R* sc) {
  const R den = A * sc[1] + B * sc[0];
  return den == (R)0 ? (R)0 : rcp_of<R>(den);
}

// NS sets of pencils per wavefront.  NS = 1: real planes (a complex plane
// pair of real transforms is two blocks).  NS = 2: components with a DFT of
// complex data; the sets hold the real and imaginary parts, which are the
// two planes of a frequency (x periodic) or the two slots of a y frequency
// (y the first periodic axis).
//
// LDS: the plane as S[half][slot][z] with the slots of a half padded to whole
// 16-row tiles (padding rows hold zeros) and z padded to whole tiles, so
// that neither direction of access needs a bounds test; the Green
// coefficients of each row; the z slot frequencies.
template <typename R, int KT, int NS>
__global__ void __launch_bounds__(mat_plane_threads(sizeof(R), KT, NS), mat_plane_waves(sizeof(R), KT, NS)) k_mat_plane(
    const MatDesc* __restrict__ descs, const int2* __restrict__ work) {
  extern __shared__ __align__(16) char smem[];
  R* sm = (R*)smem;
  const int2 wk = work[blockIdx.x];
  const MatDesc& d = descs[wk.x];
  const FM_GLOBAL Ctrl* C = gconst(d.ctrl);
  const MatAxis X = d.x[0], Y = d.x[1], Z = d.x[2];
  const int lane = threadIdx.x & 63, g = lane >> 4, p = lane & 15;
  const int wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
  const int N1 = Y.n + 1, N2 = Z.n + 1, n1 = Y.n, n2 = Z.n;
  const int64_t NR = (int64_t)N1 * N2;
  const bool xc = X.kind == K_DFT;
  const bool pair = NS == 2 && d.pair;            // some transform of complex data
  const bool px = pair && xc;                     // sets are the real and imaginary planes
  const int npl = px ? 2 : 1;
  const int plane0 = px ? 2 * wk.y : wk.y;
  const int pitch = mat_pitch(N2, sizeof(R));
  const int HR = 16 * Y.kt, RW = 2 * HR;
  R* gab = sm + npl * RW * pitch;                 // [RW] pairs
  R* gz = gab + 2 * RW;                           // [2][16 Z.kt] pairs
  // matrix steps of tile KT - 1 (past the tiles of the shorter axis: zeros)
  const int yf = Y.kt == KT ? Y.rlf : 1, yi = Y.kt == KT ? Y.rli : 1;
  const int zf = Z.kt == KT ? Z.rlf : 1, zi = Z.kt == KT ? Z.rli : 1;
  FM_GLOBAL R* T = gmut((R*)d.T) + (int64_t)plane0 * NR;
  const int ntz = (N2 + 15) >> 4;
  const int nt1 = (NS == 1 || px) ? ntz : (ntz + 1) >> 1;
  // rows of this wavefront's first tile; z[s]: z position of set s of a tile
  // (a set past the plane repeats the last tile's work into its place)
  auto zpos = [&](int tile, int s) { return 16 * ((NS == 1 || px) ? tile : min(2 * tile + s, ntz - 1)) + p; };
  RowRaw<R, KT> raw[NS];
  auto load_rows = [&](int tile) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      raw[s].load(T + (px ? s * NR : 0) + (int64_t)min(zpos(tile, s), N2 - 1) * N1, Y, Y.kt, g);
  };
  load_rows(min(wave, nt1 - 1));
  Frag<R, KT> f;
  f.load(Y.fU, Y.fV, 0, Y.kt, lane);
  {
    // x frequency of the plane, Green coefficients of the y slots
    int hx = 0, ax = xc ? (px ? wk.y : wk.y >> 1) : wk.y;
    if (!xc && ax >= X.cU) { hx = 1; ax -= X.cU; }
    const FM_GLOBAL double* gx = gconst(X.gs) + 2 * (hx * 16 * X.kt + ax);
    const FM_GLOBAL double* gy = gconst(Y.gs);
    for (int i = threadIdx.x; i < RW; i += blockDim.x) {
      R A, B;
      green_ab<R>(d, gx[0], gx[1], gy[2 * i], gy[2 * i + 1], A, B);
      gab[2 * i] = A;
      gab[2 * i + 1] = B;
    }
    for (int i = threadIdx.x; i < 64 * Z.kt; i += blockDim.x) gz[i] = gconst((const R*)Z.gz)[i];
  }
  if (C->status != ST_RUNNING) return;

  // ---- y forward: rows of the plane -> S[slot][z] ----
  for (int tile = wave; tile < nt1; tile += nwave) {
    V4<R> e[NS][KT], o[NS][KT];
    int z[NS];
    const int gl = opaque(g);
    if (tile != wave) load_rows(tile);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      z[s] = zpos(tile, s);
      raw[s].operands(Y, Y.kt, g, e[s], o[s]);
    }
    for (int mt = 0; mt < Y.kt; ++mt) {
      V4<R> u[NS], v[NS];
      Frag<R, KT> fn;
      fn.load(Y.fU, Y.fV, mt + 1 < Y.kt ? mt + 1 : 0, Y.kt, lane);
      mat_tile<R, KT, NS>(f, yf, e, o, u, v);
      f = fn;
      if (Y.cls == MC_SPLIT) {
#pragma unroll
        for (int s = 0; s < NS; ++s) butterfly(u[s], v[s]);
      } else if (NS == 2 && Y.cls == MC_CPLX) {
        const V4<R> a0 = u[0] + v[NS - 1], a1 = u[NS - 1] - v[0], b0 = u[0] - v[NS - 1], b1 = u[NS - 1] + v[0];
        u[0] = a0; u[NS - 1] = a1; v[0] = b0; v[NS - 1] = b1;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * mt + mdim<R>(gl, r);
        // slots of the second half without a frequency of their own
        const bool none = (Y.cls == MC_CPLX && (a == 0 || 2 * a == n1)) || (Y.cls == MC_SPLIT && a >= Y.cV);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          R* b = sm + ((px ? s * RW : 0) + a) * pitch + z[s];
          b[0] = u[s][r];
          b[HR * pitch] = none ? (R)0 : v[s][r];
        }
      }
    }
  }
  f.load(Z.fU, Z.fV, 0, Z.kt, lane);
  __syncthreads();

  // ---- z forward, Green, z inverse: rows of S, in place ----
  {
    const bool zc = NS == 2 && Z.cls == MC_CPLX;
    // row tiles that hold frequencies: the halves' tiles, of every plane
    const int tU = (Y.cU + 15) >> 4, tV = (Y.cV + 15) >> 4, tP = tU + tV;
    const int all = zc ? (px ? tP : tU) : npl * tP;
    const int nt2 = zc ? all : (all + NS - 1) / NS;
    for (int tile = wave; tile < nt2; tile += nwave) {
      const int gl = opaque(g);
      V4<R> e[NS][KT], o[NS][KT], u[NS][KT], v[NS][KT];
      R* row[NS];
      R gA[NS], gB[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        // (the second set of the last tile may repeat a tile: same values, same place)
        int i = min(zc ? tile : NS * tile + s, all - 1);
        int pl = zc ? (px ? s : 0) : 0;
        if (!zc && i >= tP) { i -= tP; pl = 1; }
        int ri = i < tU ? 16 * i : HR + 16 * (i - tU);
        if (zc && !px) ri = s * HR + 16 * i;
        ri += p;
        gA[s] = gab[2 * ri];
        gB[s] = gab[2 * ri + 1];
        row[s] = sm + (pl * RW + ri) * pitch;
        // operands in the natural order 16 t + 4 r + g
        if (Z.cls != MC_SPLIT) {
          const int h = n2 >> 1;
#pragma unroll
          for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int j = min(16 * t + 4 * r + gl, h);
              e[s][t][r] = row[s][j];
              o[s][t][r] = row[s][n2 - j];
            }
          // nodes 0 and n carry no data for some kinds
          e[s][0][0] = g == 0 && Z.j0 > 0 ? (R)0 : e[s][0][0];
          o[s][0][0] = g == 0 && Z.j1 <= n2 ? (R)0 : o[s][0][0];
#pragma unroll
          for (int t = 0; t < KT; ++t) {
            butterfly(e[s][t], o[s][t]);
            e[s][t] = t < Z.kt ? e[s][t] : (V4<R>)((R)0);
            o[s][t] = t < Z.kt ? o[s][t] : (V4<R>)((R)0);
          }
        } else {
          const int od = Z.kind == K_DST3;      // U takes the odd nodes
#pragma unroll
          for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int j = 2 * (16 * t + 4 * r + gl);
              const int ju = j + od, jv = j + 1 - od;
              const R a = row[s][min(ju, n2)], b = row[s][min(jv, n2)];
              e[s][t][r] = ju < Z.j1 ? a : (R)0;
              o[s][t][r] = jv >= Z.j0 && jv < Z.j1 ? b : (R)0;
            }
        }
      }
#pragma unroll
      for (int mt = 0; mt < KT; ++mt) {
#pragma unroll
        for (int s = 0; s < NS; ++s) u[s][mt] = v[s][mt] = (V4<R>)((R)0);
        if (mt < Z.kt) {
          V4<R> tu[NS], tv[NS];
          Frag<R, KT> fn;
          if (mt + 1 < Z.kt) fn.load(Z.fU, Z.fV, mt + 1, Z.kt, lane);
          else fn.load(Z.iU, Z.iV, 0, Z.kt, lane);
          mat_tile<R, KT, NS>(f, zf, e, o, tu, tv);
          f = fn;
          // Green operator; MC_SPLIT and MC_CPLX fold the scaled frequencies
          // for the inverse product
          R s1[4][2], s2[4][2];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int a = 16 * mt + mdim<R>(gl, r);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              s1[r][k] = gz[2 * a + k];
              s2[r][k] = gz[2 * (16 * Z.kt + a) + k];
            }
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (zc) {
              const R f1 = green_f<R>(gA[0], gB[0], s1[r]), f2 = green_f<R>(gA[0], gB[0], s2[r]);
              const R u0 = tu[0][r], u1 = tu[NS - 1][r], v0 = tv[0][r], v1 = tv[NS - 1][r];
              const R pr = f1 * (u0 + v1), pi = f1 * (u1 - v0), qr = f2 * (u0 - v1), qi = f2 * (u1 + v0);
              u[0][mt][r] = pr + qr; u[NS - 1][mt][r] = pi + qi;
              v[0][mt][r] = pr - qr; v[NS - 1][mt][r] = pi - qi;
            } else {
#pragma unroll
              for (int s = 0; s < NS; ++s) {
                const R f1 = green_f<R>(gA[s], gB[s], s1[r]), f2 = green_f<R>(gA[s], gB[s], s2[r]);
                const R uu = tu[s][r], vv = tv[s][r];
                if (Z.cls == MC_SPLIT) {
                  const R w1 = f1 * (uu + vv), w2 = f2 * (uu - vv);
                  u[s][mt][r] = w1 + w2;
                  v[s][mt][r] = w1 - w2;
                } else {
                  u[s][mt][r] = f1 * uu;
                  v[s][mt][r] = f2 * vv;
                }
              }
            }
          }
        }
      }
      for (int mt = 0; mt < Z.kt; ++mt) {
        V4<R> tu[NS], tv[NS];
        Frag<R, KT> fn;
        if (mt + 1 < Z.kt) fn.load(Z.iU, Z.iV, mt + 1, Z.kt, lane);
        else fn.load(Z.fU, Z.fV, 0, Z.kt, lane);
        mat_tile<R, KT, NS>(f, zi, u, v, tu, tv);
        f = fn;
        if (zc) {       // the odd half times i
          const V4<R> a0 = -tv[NS - 1], a1 = tv[0];
          tv[0] = a0;
          tv[NS - 1] = a1;
        }
        const int h = n2 >> 1;
        // (values past the nodes go to the row's padding, at N2)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int a = 16 * mt + mdim<R>(gl, r);
            if (Z.cls != MC_SPLIT) {
              row[s][a <= h ? a : N2] = tu[s][r] + tv[s][r];
              row[s][2 * a < n2 ? n2 - a : N2] = tu[s][r] - tv[s][r];
            } else {
              const R A = Z.kind == K_DST3 ? tv[s][r] : tu[s][r], B = Z.kind == K_DST3 ? tu[s][r] : tv[s][r];
              row[s][min(2 * a, N2)] = A;
              row[s][min(2 * a + 1, N2)] = B;
            }
          }
      }
    }
  }
  f.load(Y.iU, Y.iV, 0, Y.kt, lane);
  __syncthreads();

  // ---- y inverse: S[slot][z] -> rows of the plane ----
  for (int tile = wave; tile < nt1; tile += nwave) {
    const int gl = opaque(g);
    V4<R> e[NS][KT], o[NS][KT];
    int z[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      z[s] = 16 * ((NS == 1 || px) ? tile : 2 * tile + s) + p;
      const R* b = sm + (px ? s * RW : 0) * pitch + min(z[s], N2 - 1);
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = min(16 * t, HR - 16) + mdim<R>(gl, r);
          e[s][t][r] = t < Y.kt ? b[a * pitch] : (R)0;
          o[s][t][r] = t < Y.kt ? b[(HR + a) * pitch] : (R)0;
        }
    }
    if (Y.cls != MC_FOLD)
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int t = 0; t < KT; ++t) butterfly(e[s][t], o[s][t]);
    for (int mt = 0; mt < Y.kt; ++mt) {
      V4<R> u[NS], v[NS];
      Frag<R, KT> fn;
      fn.load(Y.iU, Y.iV, mt + 1 < Y.kt ? mt + 1 : 0, Y.kt, lane);
      mat_tile<R, KT, NS>(f, yi, e, o, u, v);
      f = fn;
      if (NS == 2 && Y.cls == MC_CPLX) {
        const V4<R> a0 = -v[NS - 1], a1 = v[0];
        v[0] = a0;
        v[NS - 1] = a1;
      }
      const int h = n1 >> 1, q = 16 * mt + 4 * gl;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (z[s] >= N2) continue;
        FM_GLOBAL R* row = T + (px ? s * NR : 0) + (int64_t)z[s] * N1;
        if (Y.cls != MC_SPLIT) {
          const V4<R> A = u[s] + v[s], B = u[s] - v[s];
          if (sizeof(R) == 4 && 2 * (q + 3) < n1) {
            V4<R> Br;
#pragma unroll
            for (int r = 0; r < 4; ++r) Br[r] = B[3 - r];
            *(FM_GLOBAL U4<R>*)(row + q) = (U4<R>)A;
            *(FM_GLOBAL U4<R>*)(row + n1 - q - 3) = (U4<R>)Br;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int j = 16 * mt + mdim<R>(gl, r);
              if (j <= h) row[j] = A[r];
              if (2 * j < n1) row[n1 - j] = B[r];
            }
          }
        } else {
          const bool odd = Y.kind == K_DST3;
          const V4<R> A = odd ? v[s] : u[s], B = odd ? u[s] : v[s];
          if (sizeof(R) == 4 && 2 * q + 7 <= n1) {
            V4<R> lo, hi;
            lo[0] = A[0]; lo[1] = B[0]; lo[2] = A[1]; lo[3] = B[1];
            hi[0] = A[2]; hi[1] = B[2]; hi[2] = A[3]; hi[3] = B[3];
            *(FM_GLOBAL U4<R>*)(row + 2 * q) = (U4<R>)lo;
            *(FM_GLOBAL U4<R>*)(row + 2 * q + 4) = (U4<R>)hi;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int j = 2 * (16 * mt + mdim<R>(gl, r));
              if (j <= n1) row[j] = A[r];
              if (j + 1 <= n1) row[j + 1] = B[r];
            }
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Half matrices in fragment order: entry r of lane l of fragment (mt, t) is
// row 16 mt + (l & 15), column 16 t + kmap(l >> 4, r).  Forward columns run
// in quads (4 g + r) or, on the z axis, naturally (4 r + g); inverse columns
// run in the order of the product's result registers.
__device__ double mat_fwd(int kind, int cls, int n, int half, int a, int b, const double* cs) {
  auto c = [&](int64_t m) { return cs[m % (4 * n)]; };                    // cos(pi m / 2n)
  auto s = [&](int64_t m) { return cs[(m + 3 * n) % (4 * n)]; };          // sin(pi m / 2n)
  const int h = n / 2;
  if (cls == MC_SPLIT) {
    if (a >= (n + 1) / 2) return 0;
    const bool odd_first = kind == K_DST3;
    const int j = 2 * b + ((half == 0) == odd_first ? 1 : 0);
    if (kind == K_DCT3) {
      if (j > n - 1) return 0;
      return (j == 0 ? 1.0 : 2.0) * c((int64_t)(2 * a + 1) * j);
    }
    if (j < 1 || j > n) return 0;
    return (j == n ? 1.0 : 2.0) * s((int64_t)(2 * a + 1) * j);
  }
  if (b > h) return 0;
  const double mid = 2 * b == n ? 0.5 : 1.0;        // the fold counts the middle node twice
  if (cls == MC_CPLX || kind == K_DFT) {
    if (a > h) return 0;
    const double v = half == 0 ? c((int64_t)4 * a * b) : s((int64_t)4 * a * b);
    return mid * (half == 1 && cls == MC_FOLD ? -v : v);
  }
  if (kind == K_DCT1) {
    const int k = 2 * a + half;
    if (k > n) return 0;
    return (b == 0 ? 1.0 : 2.0) * mid * c((int64_t)2 * k * b);
  }
  const int k = 2 * a + 1 + half;                   // DST-I: sin(pi k j / n)
  if (k > n - 1) return 0;
  return 2.0 * mid * s((int64_t)2 * k * b);
}

__device__ double mat_inv(int kind, int cls, int n, int half, int a, int b, const double* cs) {
  auto c = [&](int64_t m) { return cs[m % (4 * n)]; };
  auto s = [&](int64_t m) { return cs[(m + 3 * n) % (4 * n)]; };
  const int h = n / 2;
  const double in = 1.0 / n;
  if (cls == MC_SPLIT) {                            // row a: node, column b: folded frequency
    if (b >= (n + 1) / 2) return 0;
    const bool odd_first = kind == K_DST3;
    const int j = 2 * a + ((half == 0) == odd_first ? 1 : 0);
    if (j > n || (kind == K_DCT3 && j == n)) return 0;
    return in * (kind == K_DCT3 ? c((int64_t)(2 * b + 1) * j) : s((int64_t)(2 * b + 1) * j));
  }
  if (a > h) return 0;
  if (cls == MC_CPLX) {
    if (b > h) return 0;
    return in * (half == 0 ? c((int64_t)4 * a * b) : s((int64_t)4 * a * b));
  }
  if (kind == K_DFT) {
    if (b > h) return 0;
    const double w = (b == 0 || 2 * b == n) ? 1.0 : 2.0;
    return in * w * (half == 0 ? c((int64_t)4 * a * b) : -s((int64_t)4 * a * b));
  }
  if (kind == K_DCT1) {
    const int k = 2 * b + half;
    if (k > n) return 0;
    return 0.5 * in * ((k == 0 || k == n) ? 1.0 : 2.0) * c((int64_t)2 * k * a);
  }
  const int k = 2 * b + 1 + half;
  if (k > n - 1) return 0;
  return in * s((int64_t)2 * k * a);
}

template <typename R>
__global__ void __launch_bounds__(256) k_mat_tables(MatTableArgs A) {
  const int f = blockIdx.x;                         // fragment mt * kt + t
  const int mt = f / A.kt, t = f - mt * A.kt;
  const int l = threadIdx.x >> 2, r = threadIdx.x & 3, g = l >> 4;
  const int row = 16 * mt + (l & 15);
  const int kf = 16 * t + (A.natural ? 4 * r + g : 4 * g + r), ki = 16 * t + mdim<R>(g, r);
  const int64_t o = (int64_t)f * 256 + threadIdx.x;
  ((R*)A.fU)[o] = (R)mat_fwd(A.kind, A.cls, A.n, 0, row, kf, A.base);
  ((R*)A.fV)[o] = (R)mat_fwd(A.kind, A.cls, A.n, 1, row, kf, A.base);
  ((R*)A.iU)[o] = (R)mat_inv(A.kind, A.cls, A.n, 0, row, ki, A.base);
  ((R*)A.iV)[o] = (R)mat_inv(A.kind, A.cls, A.n, 1, row, ki, A.base);
  if (t == 0 && threadIdx.x < 32) {
    // frequency of slot a of each half
    const int half = threadIdx.x >> 4, a = 16 * mt + (threadIdx.x & 15), n = A.n, h = n / 2;
    int k = -1;
    if (A.cls == MC_SPLIT) { if (half == 0 ? a < (n + 1) / 2 : a < n / 2) k = half == 0 ? a : n - 1 - a; }
    else if (A.cls == MC_CPLX) { if (a <= h && !(half == 1 && (a == 0 || 2 * a == n))) k = half == 0 ? a : n - a; }
    else if (A.kind == K_DFT) { if (a <= h) k = a; }
    else if (A.kind == K_DCT1) { if (2 * a + half <= n) k = 2 * a + half; }
    else { if (2 * a + 1 + half <= n - 1) k = 2 * a + half; }
    const double s2 = k >= 0 ? A.s2[k] : 0.0, c2 = k >= 0 ? A.c2[k] : 0.0;
    const int i = 2 * (half * 16 * A.kt + a);
    A.gs[i] = s2; A.gs[i + 1] = c2;
    ((R*)A.gz)[i] = (R)s2; ((R*)A.gz)[i + 1] = (R)c2;
  }
}

template <typename R, int INV>
bool launch_x_kt(int kt, unsigned grid, hipStream_t st, const MatDesc* M, const int2* wl) {
  const dim3 G(grid), T(64 * MAT_WAVES);
#define FM_MAT_X(K)                                                                                      \
  case K:                                                                                                \
    if constexpr (K <= mat_max_kt(sizeof(R), 1)) {                                                       \
      if (INV) hipLaunchKernelGGL((k_mat_xi<R, K>), G, T, 0, st, M, wl);                                 \
      else hipLaunchKernelGGL((k_mat_xf<R, K>), G, T, 0, st, M, wl);                                     \
      return true;                                                                                       \
    }                                                                                                    \
    return false;
  switch (kt) {
    FM_MAT_X(1) FM_MAT_X(2) FM_MAT_X(3) FM_MAT_X(4) FM_MAT_X(5) FM_MAT_X(6)
    default: return false;
  }
#undef FM_MAT_X
}

template <typename R, int NS>
bool launch_plane_kt(int kt, unsigned grid, size_t lds, hipStream_t st, const MatDesc* M, const int2* wl) {
  const dim3 G(grid), T(mat_plane_threads(sizeof(R), kt, NS));
#define FM_MAT_P(K)                                                                                      \
  case K:                                                                                                \
    if constexpr (K <= mat_max_kt(sizeof(R), NS)) {                                                      \
      hipLaunchKernelGGL((k_mat_plane<R, K, NS>), G, T, lds, st, M, wl);                                 \
      return true;                                                                                       \
    }                                                                                                    \
    return false;
  switch (kt) {
    FM_MAT_P(1) FM_MAT_P(2) FM_MAT_P(3) FM_MAT_P(4) FM_MAT_P(5) FM_MAT_P(6)
    default: return false;
  }
#undef FM_MAT_P
}

template <typename R, int NS, int K>
hipError_t plane_limit(int big) {
  if constexpr (K > mat_max_kt(sizeof(R), NS)) return hipSuccess;
  else {
    const hipError_t e =
        hipFuncSetAttribute((const void*)k_mat_plane<R, K, NS>, hipFuncAttributeMaxDynamicSharedMemorySize, big);
    return e != hipSuccess ? e : plane_limit<R, NS, K + 1>(big);
  }
}

}  // namespace

hipError_t mat_set_limits(int rbytes) {
  const int big = 160 * 1024;
  if (rbytes == 4) {
    const hipError_t e = plane_limit<float, 1, 1>(big);
    return e != hipSuccess ? e : plane_limit<float, 2, 1>(big);
  }
  const hipError_t e = plane_limit<double, 1, 1>(big);
  return e != hipSuccess ? e : plane_limit<double, 2, 1>(big);
}

void mat_build_tables(int rbytes, const MatTableArgs& a, hipStream_t st) {
  const dim3 G(a.kt * a.kt), T(256);
  if (rbytes == 4) hipLaunchKernelGGL(k_mat_tables<float>, G, T, 0, st, a);
  else hipLaunchKernelGGL(k_mat_tables<double>, G, T, 0, st, a);
}

bool mat_launch_x(int rbytes, int inverse, int kt, unsigned grid, hipStream_t st, const MatDesc* M, const int2* wl) {
  if (rbytes == 4) return inverse ? launch_x_kt<float, 1>(kt, grid, st, M, wl) : launch_x_kt<float, 0>(kt, grid, st, M, wl);
  return inverse ? launch_x_kt<double, 1>(kt, grid, st, M, wl) : launch_x_kt<double, 0>(kt, grid, st, M, wl);
}

bool mat_launch_plane(int rbytes, int kt, int ns, unsigned grid, size_t lds, hipStream_t st, const MatDesc* M,
                      const int2* wl) {
  if (rbytes == 4)
    return ns == 2 ? launch_plane_kt<float, 2>(kt, grid, lds, st, M, wl) : launch_plane_kt<float, 1>(kt, grid, lds, st, M, wl);
  return ns == 2 ? launch_plane_kt<double, 2>(kt, grid, lds, st, M, wl) : launch_plane_kt<double, 1>(kt, grid, lds, st, M, wl);
}

}  // namespace fm
