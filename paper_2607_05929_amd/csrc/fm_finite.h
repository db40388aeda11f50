// Lagrangian finite-strain formulation (Sec. 2.2, Eq. TF_initial and the
// discrete problem of Eq. GeneralBCtobesolved with P in place of sigma):
// F = 1 + grad u at the integration points, first Piola-Kirchhoff stress
// P = F Pi from a hyperelastic law, D = Div P at the nodes with the
// column-wise mirror rules of the small-strain divergence, which hold for a
// non-symmetric tensor as they stand.  The spectral part of an iteration is
// unchanged (B0 / 2mu0 act on the non-symmetric gradient).
//
//  k_fs_stress  one thread per voxel: gradient (FP64, from the FP64
//               displacement), law, S[l][q] = P[q][l] of every point into
//               the solve's stress buffer (9 x n_ppv x voxels, FP64 in both
//               precisions, so that the equilibrium error of an FP32-mixed
//               solve has no FP32 floor).
//  k_fs_div     one block per stress-divergence tile: D_q = sum over the 8
//               voxels J - 1 + b and the directions l of (2 b_l - 1) S_lq of
//               the point owning the corner (HEX1: the point; TETRA2: T1 on
//               odd b, T2 on even b), mirror corners dropped and the sum
//               doubled per reflecting face (reading R21), periodic images
//               along periodic axes of u_q; FP64 partials of sum w |P|^2,
//               <P> (11, 22, 33, 23, 13, 12) and sum |D|^2.
//  k_fs_out     outputs: Green-Lagrange strain and Cauchy stress (Voigt).
#pragma once
#include "fm_space.h"

namespace fm {

// Full displacement gradient g[l][q] = D_l u_q at point r of voxel (x, y, z),
// FP64 (HEX1 weights (2a_l - 1)/(4h); TETRA2 (2a_l - 1)/(2h) on the even (T1)
// and odd (T2) corners), plus the gradient of u*; u: the corner values.
template <int SCH>
__device__ __forceinline__ void point_grad64(const SolveDev& s, const FM_GLOBAL Ctrl* C, const double (&u)[3][8], int x,
                                             int y, int z, int r, double (&g)[3][3]) {
  double gA[3][3], gB[3][3], hc[3][3];
  ustar_grad_column<double>(s, C, x, y, gA, gB);
  tet_cross_terms<double>(s, C, hc);
  const double zc = (z + 0.5) * s.h;
  const double f = (SCH == 1 ? 0.5 : 0.25) / s.h;
#pragma unroll
  for (int l = 0; l < 3; ++l)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      double a = 0;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        if (SCH == 1 && ((c ^ (c >> 1) ^ (c >> 2)) & 1) != r) continue;
        a += ((c >> l) & 1) ? u[q][c] : -u[q][c];
      }
      double v = a * f + gA[l][q] + gB[l][q] * zc;
      if (SCH == 1) v += r == 0 ? -hc[l][q] : hc[l][q];
      g[l][q] = v;
    }
}

__device__ __forceinline__ double det3(const double F[3][3]) {
  return F[0][0] * (F[1][1] * F[2][2] - F[1][2] * F[2][1]) - F[0][1] * (F[1][0] * F[2][2] - F[1][2] * F[2][0]) +
         F[0][2] * (F[1][0] * F[2][1] - F[1][1] * F[2][0]);
}

// First Piola-Kirchhoff stress P[q][J] for F[q][J]: Saint Venant-Kirchhoff
// Pi = lambda tr(E) 1 + 2 mu E, P = F Pi (table entry: lambda, mu);
// compressible Neo-Hookean of Appendix B, P = mu J^-2/3 (F - tr(F F^T)/3
// F^-T) + K (J - 1) J F^-T (table entry: mu, K).
template <typename PT>
__device__ __forceinline__ void pk1_law(int law, PT M, const double F[3][3], double P[3][3]) {
  if (law == LAW_SVK) {
    const double lam = (double)M[0], mu = (double)M[1];
    double E[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        double a = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) a += F[k][i] * F[k][j];
        E[i][j] = 0.5 * (a - (i == j ? 1.0 : 0.0));
      }
    const double tr = E[0][0] + E[1][1] + E[2][2];
    double Pi[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) Pi[i][j] = 2.0 * mu * E[i][j] + (i == j ? lam * tr : 0.0);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        double a = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) a += F[i][k] * Pi[k][j];
        P[i][j] = a;
      }
  } else {
    const double mu = (double)M[0], K = (double)M[1];
    const double J = det3(F);
    // F^-T = cof(F) / J
    double cof[3][3];
    cof[0][0] = F[1][1] * F[2][2] - F[1][2] * F[2][1];
    cof[0][1] = F[1][2] * F[2][0] - F[1][0] * F[2][2];
    cof[0][2] = F[1][0] * F[2][1] - F[1][1] * F[2][0];
    cof[1][0] = F[0][2] * F[2][1] - F[0][1] * F[2][2];
    cof[1][1] = F[0][0] * F[2][2] - F[0][2] * F[2][0];
    cof[1][2] = F[0][1] * F[2][0] - F[0][0] * F[2][1];
    cof[2][0] = F[0][1] * F[1][2] - F[0][2] * F[1][1];
    cof[2][1] = F[0][2] * F[1][0] - F[0][0] * F[1][2];
    cof[2][2] = F[0][0] * F[1][1] - F[0][1] * F[1][0];
    double I1 = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) I1 += F[i][j] * F[i][j];
    const double a = mu * pow(J, -2.0 / 3.0), b = K * (J - 1.0) * J;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const double fit = cof[i][j] / J;
        P[i][j] = a * (F[i][j] - I1 / 3.0 * fit) + b * fit;
      }
  }
}

// First Piola-Kirchhoff stress of every point of voxel (x, y, z).  Scheme and
// tensor loops are fixed at compile time: the tensors stay in registers
// (with runtime loops they lived in scratch memory; 101 x 87 x 64 TETRA2
// Neo-Hooke: 47 us then, 35 us now, of which 30 us is the 148 MB it writes).
template <typename R, int SCH, typename F>
__device__ __forceinline__ void fs_points(const SolveDev& s, const FM_GLOBAL Ctrl* C, int x, int y, int z, int law,
                                          const FM_GLOBAL R* M, F&& use) {
  double u[3][8];
  voxel_corners<double>(s, x, y, z, u);
#pragma unroll
  for (int r = 0; r < (SCH == 1 ? 2 : 1); ++r) {
    double g[3][3], Fm[3][3], P[3][3];
    point_grad64<SCH>(s, C, u, x, y, z, r, g);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int J = 0; J < 3; ++J) Fm[q][J] = (q == J ? 1.0 : 0.0) + g[J][q];
    pk1_law(law, M, Fm, P);
    use(r, Fm, P);
  }
}
template <typename R, typename F>
__device__ __forceinline__ void fs_voxel(const SolveDev& s, const FM_GLOBAL Ctrl* C, int64_t v, F&& use) {
  const int n0 = s.n[0], n1 = s.n[1];
  const int x = (int)(v % n0);
  const int64_t t = v / n0;
  const int y = (int)(t % n1), z = (int)(t / n1);
  const int mt = gconst(s.mat)[v];
  const int law = gconst(s.mlaw)[mt];
  const FM_GLOBAL R* M = gconst((const R*)s.mtab) + (int64_t)mt * MT_STRIDE;
  if (s.scheme == 1) fs_points<R, 1>(s, C, x, y, z, law, M, use);
  else fs_points<R, 0>(s, C, x, y, z, law, M, use);
}

template <typename R>
__global__ void __launch_bounds__(256) k_fs_stress(const SolveDev* __restrict__ S, const int2* __restrict__ work) {
  const int2 w = work[blockIdx.x / (SPACE_TILE / 256)];
  const SolveDev& s = S[w.x];
  const FM_GLOBAL Ctrl* C = gconst(s.ctrl);
  if (C->status != ST_RUNNING) return;
  const int64_t v = (int64_t)w.y * SPACE_TILE + (blockIdx.x % (SPACE_TILE / 256)) * 256 + threadIdx.x;
  if (v >= s.Nv) return;
  fs_voxel<R>(s, C, v, [&](int r, const double (&)[3][3], const double (&P)[3][3]) {
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        gmut((double*)s.sig)[((int64_t)(l * 3 + q) * s.nppv + r) * s.Nv + v] = P[q][l];
  });
}

// Divergence of S at the nodes of one stress-divergence tile, two points per
// voxel (NP = 2) or one.  The 24 stresses of a component are loaded together,
// without a branch (mirror corners load a voxel of the grid and count as
// zero); with a branch per corner each load waited for the one before
// (101 x 87 x 64 TETRA2: 54 us then, 41 us now).
template <typename R, int NP>
__device__ __forceinline__ void fs_div_tile(const SolveDev& s, const FM_GLOBAL Ctrl* C, const SdBox& bx,
                                            double (&acc)[8]) {
  const int X0 = bx.X0, Y0 = bx.Y0, Z0 = bx.Z0;
  const int X1 = min(X0 + bx.W - 1, s.N[0]), Y1 = min(Y0 + bx.H - 1, s.N[1]), Z1 = min(Z0 + s.sd_zc, s.N[2]);
  const int nx = X1 - X0, ny = Y1 - Y0, nz = Z1 - Z0;
  const int n[3] = {s.n[0], s.n[1], s.n[2]};
  const FM_GLOBAL double* Sg = gconst((const double*)s.sig);
  FM_GLOBAL R* Dring = gmut((R*)s.Dring) + (int64_t)(C->m % s.depth) * 3 * s.Nn;
  const bool trac = C->has_trac;
  const double wip = 1.0 / NP;
  for (int idx = threadIdx.x; idx < nx * ny * nz; idx += blockDim.x) {
    const int J[3] = {X0 + idx % nx, Y0 + (idx / nx) % ny, Z0 + idx / (nx * ny)};
    const int64_t node = ((int64_t)J[2] * s.N[1] + J[1]) * s.N[0] + J[0];
    // voxel coordinates of the two sides, periodic images across the faces
    int vc[3][2];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      vc[i][0] = J[i] > 0 ? J[i] - 1 : n[i] - 1;
      vc[i][1] = J[i] < n[i] ? J[i] : 0;
    }
    const bool inner = J[0] < n[0] && J[1] < n[1] && J[2] < n[2];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      bool kept = true, drop[3][2];
      double fac = 0.25 / s.h;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const bool per = s.kinds[q][i] == K_DFT;
        kept = kept && node_kept(s.kinds[q][i], n[i], J[i]);
        if (!per && (J[i] == 0 || J[i] == n[i])) fac *= 2.0;
        drop[i][0] = !per && J[i] == 0;      // mirror corners
        drop[i][1] = !per && J[i] == n[i];
      }
      double v[8][3];
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int b0 = b & 1, b1 = (b >> 1) & 1, b2 = b >> 2;
        const int r = NP == 2 ? (((b0 + b1 + b2) & 1) ? 0 : 1) : 0;
        const int64_t vox = ((int64_t)vc[2][b2] * n[1] + vc[1][b1]) * n[0] + vc[0][b0];
#pragma unroll
        for (int l = 0; l < 3; ++l) v[b][l] = Sg[((int64_t)(l * 3 + q) * NP + r) * s.Nv + vox];
      }
      double D = 0;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int bb[3] = {b & 1, (b >> 1) & 1, b >> 2};
        const bool in = !(drop[0][bb[0]] || drop[1][bb[1]] || drop[2][bb[2]]);
#pragma unroll
        for (int l = 0; l < 3; ++l) {
          const double t = in ? v[b][l] : 0.0;
          D += bb[l] ? t : -t;
        }
      }
      D *= fac;
      if (trac) D += node_dstar<double>(s, C, J[0], J[1], J[2], q);
      D = kept ? D : 0.0;
      Dring[q * s.Nn + node] = (R)D;
      acc[7] += D * D;
      // the voxel whose lower corner is this node (corner 7) enters the
      // stress partials once: <P> entries P_11, P_22, P_33, P_23, P_13, P_12
      // (S[l][q] = P[q][l]); its point in v is r(7), the other one is loaded
      if (inner) {
        const int64_t vox = ((int64_t)J[2] * n[1] + J[1]) * n[0] + J[0];
#pragma unroll
        for (int r = 0; r < NP; ++r)
#pragma unroll
          for (int l = 0; l < 3; ++l) {
            const double t = NP == 2 && r == 1 ? Sg[((int64_t)(l * 3 + q) * NP + r) * s.Nv + vox] : v[7][l];
            acc[0] += wip * t * t;
            if (l == q) acc[1 + l] += wip * t;
            else if (l > q) acc[1 + vidx(l, q)] += wip * t;
          }
      }
    }
  }
}

template <typename R>
__global__ void __launch_bounds__(256) k_fs_div(const SolveDev* __restrict__ S, const int2* __restrict__ work) {
  const int2 w = work[blockIdx.x];
  const SolveDev& s = S[w.x];
  const FM_GLOBAL Ctrl* C = gconst(s.ctrl);
  if (C->status != ST_RUNNING) return;
  const SdBox bx = sd_box(s, w.y);
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (s.nppv == 2) fs_div_tile<R, 2>(s, C, bx, acc);
  else fs_div_tile<R, 1>(s, C, bx, acc);
  __shared__ double outp[8];
  block_sum<8>(acc, outp);
  __syncthreads();
  if (threadIdx.x < 8) gmut(s.part_s)[(int64_t)w.y * NPART_S + threadIdx.x] = outp[threadIdx.x];
}

// Outputs of a finite-strain solve: Green-Lagrange strain E and Cauchy
// stress J^-1 P F^T at every point (Voigt xx yy zz yz xz xy, FP64).
template <typename R>
__global__ void __launch_bounds__(256) k_fs_out(const SolveDev* __restrict__ S, const int2* __restrict__ work) {
  const int2 w = work[blockIdx.x];
  const SolveDev& s = S[w.x];
  const FM_GLOBAL Ctrl* C = gconst(s.ctrl);
  for (int sub = 0; sub < SPACE_TILE / 256; ++sub) {
    const int64_t v = (int64_t)w.y * SPACE_TILE + sub * 256 + threadIdx.x;
    if (v >= s.Nv) continue;
    fs_voxel<R>(s, C, v, [&](int r, const double (&F)[3][3], const double (&P)[3][3]) {
      constexpr int vi[6] = {0, 1, 2, 1, 0, 0}, vj[6] = {0, 1, 2, 2, 2, 1};
      const double J = det3(F);
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const int i = vi[k], j = vj[k];
        double e = 0, sg = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          e += F[a][i] * F[a][j];
          sg += P[i][a] * F[j][a];
        }
        if (s.out_eps) gmut(s.out_eps)[((int64_t)k * s.nppv + r) * s.Nv + v] = 0.5 * (e - (i == j ? 1.0 : 0.0));
        if (s.out_sig) gmut(s.out_sig)[((int64_t)k * s.nppv + r) * s.Nv + v] = sg / J;
      }
    });
  }
}

}  // namespace fm
