// Full matrices around the triangles: the lower triangles of H and S from the upper ones, and the Hermitian
// parts of incoming gradients, both matrices in one launch each.  Bandwidth-bound: 16 bytes read and
// written per element of a triangle, or of the square, in 32 x 32 tiles turned through LDS.
#include "hs_internal.h"
#include "tiles.h"

namespace hsb {

namespace {

constexpr int kTile = 32, kTileRows = 8;  // rows of a tile per pass of the workgroup

// Tile pair blockIdx.x (bi <= bj) of the matrix blockIdx.z.
__global__ void __launch_bounds__(kTile* kTileRows) k_mirror(int n, double2* __restrict__ H, double2* __restrict__ S) {
  __shared__ double2 tile[kTile][kTile + 1];
  double2* M = blockIdx.z ? S : H;
  int bi, bj;
  tri_decode(blockIdx.x, (n + kTile - 1) / kTile, bi, bj);
  const int x = threadIdx.x % kTile, y0 = threadIdx.x / kTile;
  for (int y = y0; y < kTile; y += kTileRows) {
    const int r = bi * kTile + y, c = bj * kTile + x;
    if (r < n && c < n && c > r) tile[y][x] = M[(int64_t)r * n + c];
  }
  __syncthreads();
  for (int y = y0; y < kTile; y += kTileRows) {
    const int r = bj * kTile + y, c = bi * kTile + x;
    if (r < n && c < r) {
      const double2 v = tile[x][y];
      M[(int64_t)r * n + c] = make_double2(v.x, -v.y);
    }
  }
}

// out = (g + g^H) / 2, zero for g null.
__global__ void __launch_bounds__(kTile* kTileRows) k_hermitian_part(int n, const double2* __restrict__ gH,
                                                                     const double2* __restrict__ gS,
                                                                     double2* __restrict__ oH,
                                                                     double2* __restrict__ oS) {
  __shared__ double2 up[kTile][kTile + 1], lo[kTile][kTile + 1];  // tiles (bi, bj) and (bj, bi) of g
  const double2* g = blockIdx.z ? gS : gH;
  double2* out = blockIdx.z ? oS : oH;
  int bi, bj;
  tri_decode(blockIdx.x, (n + kTile - 1) / kTile, bi, bj);
  const int x = threadIdx.x % kTile, y0 = threadIdx.x / kTile;
  for (int y = y0; y < kTile; y += kTileRows) {
    const double2 z = make_double2(0.0, 0.0);
    const int r = bi * kTile + y, c = bj * kTile + x, r2 = bj * kTile + y, c2 = bi * kTile + x;
    up[y][x] = g && r < n && c < n ? g[(int64_t)r * n + c] : z;
    lo[y][x] = g && r2 < n && c2 < n ? g[(int64_t)r2 * n + c2] : z;
  }
  __syncthreads();
  for (int y = y0; y < kTile; y += kTileRows) {
    const int r = bi * kTile + y, c = bj * kTile + x, r2 = bj * kTile + y, c2 = bi * kTile + x;
    const double2 a = up[y][x], b = lo[x][y], a2 = lo[y][x], b2 = up[x][y];
    if (r < n && c < n) out[(int64_t)r * n + c] = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
    if (bi != bj && r2 < n && c2 < n)
      out[(int64_t)r2 * n + c2] = make_double2(0.5 * (a2.x + b2.x), 0.5 * (a2.y - b2.y));
  }
}

dim3 pairs(int n) {
  const int nb = (n + kTile - 1) / kTile;
  return dim3((unsigned)((int64_t)nb * (nb + 1) / 2), 1, 2);
}

}  // namespace

hipError_t launch_mirror(int n, double2* H, double2* S, hipStream_t s) {
  hipLaunchKernelGGL(k_mirror, pairs(n), dim3(kTile * kTileRows), 0, s, n, H, S);
  return hipGetLastError();
}

hipError_t launch_hermitian_part(int n, const double2* gH, const double2* gS, double2* oH, double2* oS,
                                 hipStream_t s) {
  hipLaunchKernelGGL(k_hermitian_part, pairs(n), dim3(kTile * kTileRows), 0, s, n, gH, gS, oH, oS);
  return hipGetLastError();
}

}  // namespace hsb
