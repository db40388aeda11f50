// Matrix-core transforms: declarations shared by the engine and the kernels.
//
// Every Table 1 transform of an axis of n voxels splits into two real
// matrices of half its size (at most floor(n/2) + 1 rows and columns), by
// the reflection j <-> n - j of the nodes or k <-> n - 1 - k of the
// frequencies:
//   MC_FOLD   (DCT-I, DST-I, DFT of real data): e_j = x_j + x_{n-j},
//             o_j = x_j - x_{n-j}; even frequencies (or real parts) from e,
//             odd ones (imaginary parts) from o.  The inverse sums both
//             halves: x_j = E_j + O_j, x_{n-j} = E_j - O_j.
//   MC_SPLIT  (DCT-III, DST-III): nodes split by parity, frequencies k and
//             n - 1 - k are the sum and the difference of the halves; the
//             inverse folds the frequencies and splits the nodes.
//   MC_CPLX   (DFT of complex data): nodes and frequencies both fold, with
//             G_k = C_k - i S_k, G_{n-k} = C_k + i S_k.
// The products run on the matrix cores.  Data travel as the B operand (one
// pencil per lane of a 16-lane group), the half matrices as the A operand,
// stored in fragment order.  Spectral coefficients are kept by slot: slot a
// of the first half (U), slot a of the second half (V); their number per
// half and the physical frequency of each slot follow from the kind.
#pragma once
#include "fm_common.h"

namespace fm {

constexpr int MAT_WAVES = 4;          // wavefronts per block of the x kernels (each on its own pencils)
// Threads of a plane block: eight wavefronts while two fit a SIMD's registers.
__host__ __device__ constexpr int mat_plane_threads(int rbytes, int kt, int ns) {
  return kt * ns * (rbytes / 4) <= 3 ? 512 : 256;
}

// Wavefronts per SIMD a plane kernel's registers are held to.
__host__ __device__ constexpr int mat_plane_waves(int rbytes, int kt, int ns) {
  return kt * ns * (rbytes / 4) <= 4 ? 2 : 1;
}

// Largest half-matrix size in 16-row tiles the kernels are compiled for, by
// real size in bytes and by the sets of pencils a plane kernel carries.
__host__ __device__ constexpr int mat_max_kt(int rbytes, int ns) {
  return rbytes == 4 ? (ns == 2 ? 4 : 6) : (ns == 2 ? 3 : 4);
}

// Row pitch of the plane in LDS (reals) for N values padded to whole 16-wide
// tiles: conflict-free for the row-wise and the column-wise accesses of the
// 16 x 4 lane layout, and larger than N.
__host__ __device__ inline int mat_pitch(int N, int rbytes) { return (N + 15) / 16 * 16 + (rbytes == 4 ? 4 : 2); }
// Reals of LDS of a plane block: planes x 2 halves x 16 kty rows, Green
// coefficients per row, z slot frequencies.
__host__ __device__ inline size_t mat_plane_lds(int planes, int kty, int ktz, int N2, int rbytes) {
  return (size_t)planes * 32 * kty * mat_pitch(N2, rbytes) + 64 * kty + 64 * ktz;
}

struct MatTableArgs {
  int32_t kind, n, cls, kt, natural;   // natural: forward fragments in the natural k order (z axis)
  const double* base;                  // cos(pi m / (2 n)), m = 0 .. 4 n - 1
  const double* s2;                    // sin^2, cos^2 of the half frequency per coefficient index
  const double* c2;
  void *fU, *fV, *iU, *iV;             // fragments, kt * kt * 256 reals each
  double* gs;                          // [2][16 kt] pairs (sin^2, cos^2) per slot, (0, 0) where no frequency
  void* gz;                            // the same in the plan's precision
};

hipError_t mat_set_limits(int rbytes);
void mat_build_tables(int rbytes, const MatTableArgs& a, hipStream_t st);
// x passes (inverse = 0 / 1) and the fused y-z plane pass; kt: tiles of the
// longest axis involved, ns: pencil sets per wavefront of a plane block.
bool mat_launch_x(int rbytes, int inverse, int kt, unsigned grid, hipStream_t st, const MatDesc* M, const int2* wl);
bool mat_launch_plane(int rbytes, int kt, int ns, unsigned grid, size_t lds, hipStream_t st, const MatDesc* M,
                      const int2* wl);

}  // namespace fm
