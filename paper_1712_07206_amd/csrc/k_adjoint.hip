// Adjoint of the H/S build for a real loss L(H, S) with incoming gradients gH = dL/dRe H + i dL/dIm H
// and gS (likewise), in the type-factored form (k_fact.hip: R_t real, Y_t = T'_t R_t, phases E):
//
//   P_t   = E_t^H E_t,   M_t = R_t^T Y_t,   N_t = R_t^T Lam R_t                       (N_G x N_G)
//   Z_t   = gH .* conj(P_t),   Q_t = conj(gH) .* M_t + conj(gS) .* N_t
//   grad T'_t   = R_t Z_t R_t^T,  grad T_t = C grad T'_t C^H  (C: real to complex harmonics)
//   grad tau_a  = -2 sum_G K_G Im( E_a(G) sum_G' conj(E_a(G')) Q_t[G'][G] ),   a in t
//
// since T enters through M_t only and tau through the phases only (Eqs. 4-5).  Neither T nor gH, gS
// is taken to be Hermitian.  Per type and pair of columns: 6 N_L real products for M_t, N_t, as many
// for R Z, 6 N_t for the phases, where the atom by atom form takes 24 N_t N_L; nothing is kept
// from the forward.
//
//   k_adj_zq      P_t, M_t, N_t per tile (as k_fact_hs), Z_t and Q_t to memory
//   k_adj_uc      (R Z)^T = Z^T R^T, rows G; and the phase sums of grad tau, reduced over the rows
//                 of a tile to one partial per atom and segment of G'
//   k_adj_gt      R Z R^T in segments of G
//   k_adj_reduce  the segments' sums in order, turned back to complex harmonics; grad tau likewise
//
// All on v_mfma_f64_16x16x4f64; k_adj_uc and k_adj_gt read their operands straight into registers, one
// chunk ahead, and the transposed copies of R and E (k_fact_tables) keep every operand contiguous along
// the MFMA's row or column index.  Deterministic: fixed orders, no atomics.
#include "harmonics.h"
#include "hs_internal.h"
#include "wave_tile.h"

namespace hsb {

namespace {

// Z_t and Q_t (zeros outside n x n, up to n_pad): 64 x 64 tiles of the square (MI = 2) or their halves (MI = 1,
// interleaved in blockIdx.y), types over z.
template <int MI>
__global__ void __launch_bounds__(512, 2) k_adj_zq(FactCell c, FactK kk, int t0, const d2* __restrict__ gH,
                                                   const d2* __restrict__ gS, const char* __restrict__ ws,
                                                   d2* __restrict__ Z, d2* __restrict__ Q) {
  constexpr int PARTS = 2 / MI;
  __shared__ __align__(16) char lds[TypedTile<MI, false>::lds_bytes];
  const int n = kk.n;
  const int64_t n_pad = kk.n_pad;
  const int t = t0 + blockIdx.z;
  TypedTile<MI, false> tile(c, kk, ws, lds, blockIdx.y / PARTS, blockIdx.y % PARTS, blockIdx.x, t, t + 1);
  const bool active = tile.row0() < n && tile.col0() < n;
  const int col = tile.col();
  d2* z = Z + (int64_t)blockIdx.z * n_pad * n_pad + col;
  d2* qq = Q + (int64_t)blockIdx.z * n_pad * n_pad + col;
  d4 pR[MI], pI[MI], m1[MI], m2[MI], F[MI];
  tile.phase_sums(t, active, pR, pI);
  tile.row_sums(active, m1, m2, F);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = tile.row(i, q);
      d2 vz = d2{0.0, 0.0}, vq = d2{0.0, 0.0};  // (the sums of pad columns may hold anything)
      if (r < n && col < n) {
        const d2 h = gH[(int64_t)r * n + col], s = gS[(int64_t)r * n + col];
        const double a = m1[i][q], b = m2[i][q], d = F[i][q], pr = pR[i][q], pi = pI[i][q];
        vz = d2{h.x * pr + h.y * pi, h.y * pr - h.x * pi};
        vq = d2{h.x * a + h.y * b + s.x * d, h.x * b - h.y * a - s.y * d};
      }
      z[(int64_t)r * n_pad] = vz;
      qq[(int64_t)r * n_pad] = vq;
    }
}

// Complex A [k][row], real B [k][col]: re, im += sum over k in [4 k0, 4 k1) (4-row steps), both
// operands with their leading dimensions, in chunks of KC steps (k1 - k0 a multiple of KC).
template <int MI, int NJ, int KC>
__device__ __forceinline__ void product_cr(const d2* __restrict__ A, int64_t ldA, const double* __restrict__ B,
                                           int64_t ldB, int k0, int k1, d4 (&re)[MI][NJ], d4 (&im)[MI][NJ]) {
  typedef typename DVec<NJ>::T VB;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const d2* ap = A + (int64_t)lk * ldA + MI * lr;
  const double* bp = B + (int64_t)lk * ldB + NJ * lr;
  struct Chunk { d2 a[KC][MI]; VB b[KC]; };
  auto load = [&](int s, Chunk& x) {
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      const int64_t k = (int64_t)(s + q) * 4;
#pragma unroll
      for (int i = 0; i < MI; ++i) x.a[q][i] = ap[k * ldA + i];
      x.b[q] = *(const VB*)(bp + k * ldB);
    }
  };
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) re[i][j] = im[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  if (k0 >= k1) return;
  Chunk x;
  load(k0, x);
  for (int s = k0; s < k1; s += KC) {
    Chunk y;
    load(s + KC < k1 ? s + KC : s, y);
#pragma unroll
    for (int q = 0; q < KC; ++q)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const double b = DVec<NJ>::get(x.b[q], j);
          re[i][j] = MFMA(x.a[q][i].x, b, re[i][j]);
          im[i][j] = MFMA(x.a[q][i].y, b, im[i][j]);
        }
    x = y;
  }
}

// Workgroups blockIdx.x < nu: tiles of UT[G][k] = sum_G' Z[G'][G] RT[G'][k] (2 x 2 waves, rows G).
// Past them: the phase sums.  One wave per (16 MI columns G, 16 atoms, segment of G'):
// D[G][a] = sum_G' Q[G'][G] conj(ET[G'][a]) (three real products: P1 = q_r e_r, P2 = q_i e_i,
// P3 = (q_r + q_i)(e_r - e_i), Re = P1 + P2, Im = P3 - P1 + P2), then sum_G K_G Im(E_a(G) D[G][a])
// over the tile's columns into part[seg][column block][phase row][3].
template <int MI, int KC>
__global__ void __launch_bounds__(256, 2) k_adj_uc(FactCell c, FactK kk, FactAdj ad, int t0, int nu, int nab,
                                                   const char* __restrict__ ws, const d2* __restrict__ Z,
                                                   const d2* __restrict__ Q) {
  const int64_t n_pad = kk.n_pad;
  const int t = t0 + blockIdx.y;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int steps = kk.n_pad / 4;
  if ((int)blockIdx.x < nu) {
    const int nkb = (ad.Mt + 32 * MI - 1) / (32 * MI);
    const int row0 = blockIdx.x / nkb * 32 * MI + (wave >> 1) * 16 * MI;
    const int col0 = blockIdx.x % nkb * 32 * MI + (wave & 1) * 16 * MI;
    if (row0 >= kk.n_pad || col0 >= ad.Mt) return;
    d4 re[MI][MI], im[MI][MI];
    product_cr<MI, MI, KC>(Z + (int64_t)blockIdx.y * n_pad * n_pad + row0, n_pad,
                           (const double*)(ws + ad.RT) + (int64_t)t * n_pad * ad.Mt + col0, ad.Mt, 0, steps, re, im);
    d2* U = (d2*)(ws + ad.UT) + (int64_t)blockIdx.y * n_pad * ad.Mt;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < MI; ++j)
          U[(int64_t)(row0 + MI * (lk + 4 * q) + i) * ad.Mt + col0 + MI * lr + j] = d2{re[i][j][q], im[i][j][q]};
    return;
  }
  const int w = ((int)blockIdx.x - nu) * 4 + wave;  // (column block, atom block, segment), segment fastest
  const int seg = w % ad.nseg, ab = w / ad.nseg % nab, gb = w / ad.nseg / nab;
  const int row0 = gb * 16 * MI, a0 = ab * 16;
  if (row0 >= kk.n_pad || a0 >= c.nat[t]) return;
  const int nch = steps / KC;
  const int k0 = (int)((int64_t)nch * seg / ad.nseg) * KC, k1 = (int)((int64_t)nch * (seg + 1) / ad.nseg) * KC;
  const d2* ET = (const d2*)(ws + ad.ET) + c.eoff[t] + a0;
  const d2* qp = Q + (int64_t)blockIdx.y * n_pad * n_pad + (int64_t)lk * n_pad + row0 + MI * lr;
  const d2* ep = ET + (int64_t)lk * ad.et_ld + lr;
  struct Chunk { d2 a[KC][MI], b[KC]; };
  auto load = [&](int s, Chunk& x) {
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      const int64_t k = (int64_t)(s + q) * 4;
#pragma unroll
      for (int i = 0; i < MI; ++i) x.a[q][i] = qp[k * n_pad + i];
      x.b[q] = ep[k * ad.et_ld];
    }
  };
  d4 p1[MI], p2[MI], p3[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) p1[i] = p2[i] = p3[i] = d4{0.0, 0.0, 0.0, 0.0};
  if (k0 < k1) {
    Chunk x;
    load(k0, x);
    for (int s = k0; s < k1; s += KC) {
      Chunk y;
      load(s + KC < k1 ? s + KC : s, y);
#pragma unroll
      for (int q = 0; q < KC; ++q) {
        const double es = x.b[q].x - x.b[q].y;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          p1[i] = MFMA(x.a[q][i].x, x.b[q].x, p1[i]);
          p2[i] = MFMA(x.a[q][i].y, x.b[q].y, p2[i]);
          p3[i] = MFMA(x.a[q][i].x + x.a[q][i].y, es, p3[i]);
        }
      }
      x = y;
    }
  }
  // lane: atom a0 + lr, columns G = row0 + MI (lk + 4 q) + i; pads of E are zero
  const double* kv = (const double*)(ws + kk.kv);
  double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int G = row0 + MI * (lk + 4 * q) + i;
      const d2 e = ET[(int64_t)G * ad.et_ld + lr];
      const double re = p1[i][q] + p2[i][q], im = p3[i][q] - p1[i][q] + p2[i][q];
      const double s = e.x * im + e.y * re;
      v[0] += s * kv[4 * G + 0];
      v[1] += s * kv[4 * G + 1];
      v[2] += s * kv[4 * G + 2];
    }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    v[d] += __shfl_xor(v[d], 16, 64);
    v[d] += __shfl_xor(v[d], 32, 64);
  }
  if (lk == 0 && a0 + lr < c.nat[t]) {
    double* part = (double*)(ws + ad.partTau) + (((int64_t)seg * ad.ngb + gb) * ad.et_ld + c.eoff[t] + a0 + lr) * 3;
    part[0] = v[0];
    part[1] = v[1];
    part[2] = v[2];
  }
}

// part[t][seg][k][k'] = sum over the segment's G of UT[G][k] RT[G][k'].
template <int MI, int KC>
__global__ void __launch_bounds__(256, 2) k_adj_gt(FactCell c, FactK kk, FactAdj ad, int t0,
                                                   const char* __restrict__ ws) {
  const int64_t n_pad = kk.n_pad;
  const int t = t0 + blockIdx.y, seg = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int nkb = (ad.Mt + 32 * MI - 1) / (32 * MI);
  const int row0 = blockIdx.x / nkb * 32 * MI + (wave >> 1) * 16 * MI;
  const int col0 = blockIdx.x % nkb * 32 * MI + (wave & 1) * 16 * MI;
  if (row0 >= ad.Mt || col0 >= ad.Mt) return;
  const int nch = kk.n_pad / 4 / KC;
  const int k0 = (int)((int64_t)nch * seg / ad.ngt) * KC, k1 = (int)((int64_t)nch * (seg + 1) / ad.ngt) * KC;
  d4 re[MI][MI], im[MI][MI];
  product_cr<MI, MI, KC>((const d2*)(ws + ad.UT) + (int64_t)blockIdx.y * n_pad * ad.Mt + row0, ad.Mt,
                         (const double*)(ws + ad.RT) + (int64_t)t * n_pad * ad.Mt + col0, ad.Mt, k0, k1, re, im);
  d2* out = (d2*)(ws + ad.partT) + ((int64_t)t * ad.ngt + seg) * ad.Mt * ad.Mt;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < MI; ++j)
        out[(int64_t)(row0 + MI * (lk + 4 * q) + i) * ad.Mt + col0 + MI * lr + j] = d2{re[i][j][q], im[i][j][q]};
}

// grad T[(X,l,m)][(X',l',m')] = sum c(l,m,mu) (sum over segments of part)[mu][mu'] conj(c(l',m',mu')),
// zero for a type without atoms; and grad tau[a] = -2 sum of its partials (blocks past the T ones).
__global__ void __launch_bounds__(256) k_adj_reduce(FactCell c, FactAdj ad, int n_types, int ntb,
                                                    const char* __restrict__ ws, d2* __restrict__ gT,
                                                    double* __restrict__ gtau) {
  if ((int)blockIdx.x >= ntb) {
    const int i = ((int)blockIdx.x - ntb) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;  // wave: (atom, axis)
    int t = 0, a = i / 3;
    while (t < c.n_act && a >= c.nat[t]) a -= c.nat[t++];
    if (t >= c.n_act || blockIdx.y > 0) return;
    const double* part = (const double*)(ws + ad.partTau) + (int64_t)(c.eoff[t] + a) * 3 + i % 3;
    double s = 0.0;
    for (int b = lane; b < ad.nseg * ad.ngb; b += 64) s += part[(int64_t)b * ad.et_ld * 3];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) gtau[(c.atom0[t] + a) * 3 + i % 3] = -2.0 * s;
    return;
  }
  const int M = 2 * c.n_l;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)M * M) return;
  const int t = blockIdx.y, r = (int)(idx / M), k = (int)(idx % M);
  int at = 0;
  while (at < c.n_act && c.type[at] != t) ++at;
  d2 v = d2{0.0, 0.0};
  if (at < c.n_act) {
    const int xr = r >= c.n_l, xk = k >= c.n_l;
    int lr, mr, lk, mk;
    lm_of(r - xr * c.n_l, lr, mr);
    lm_of(k - xk * c.n_l, lk, mk);
    const int br = xr * c.n_l + lr * lr + lr, bk = xk * c.n_l + lk * lk + lk;
    const d2* part = (const d2*)(ws + ad.partT) + (int64_t)at * ad.ngt * ad.Mt * ad.Mt;
    for (int ir = 0; ir < (mr ? 2 : 1); ++ir)
      for (int ik = 0; ik < (mk ? 2 : 1); ++ik) {
        const int u1 = ir ? -mr : mr, u2 = ik ? -mk : mk;
        d2 s = d2{0.0, 0.0};
        for (int g = 0; g < ad.ngt; ++g) s += part[((int64_t)g * ad.Mt + br + u1) * ad.Mt + bk + u2];
        const double2 x = times_i(make_double2(s.x, s.y), harmonic_power(lr, mr, u1) - harmonic_power(lk, mk, u2));
        v += d2{x.x, x.y};
      }
    if (mr && mk) v *= 0.5;
    else if (mr || mk) v *= 0.70710678118654752440;
  }
  gT[(int64_t)t * M * M + idx] = v;
}

}  // namespace

hipError_t launch_adj_zq(const FactCell& c, const FactK& kk, int t0, int nt, int num_cus, const double2* gH,
                         const double2* gS, const char* ws, double2* Z, double2* Q, hipStream_t s) {
  const int nb = kk.n_pad / 64;
  const bool halves = 2 * nb * nb * nt <= num_cus;  // as in launch_fact_hs
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nb, halves ? 2 * nb : nb, nt), dim3(512), 0, s, c, kk, t0, (const d2*)gH,
                       (const d2*)gS, ws, (d2*)Z, (d2*)Q);
  };
  halves ? go(k_adj_zq<1>) : go(k_adj_zq<2>);
  return hipGetLastError();
}

hipError_t launch_adj_uc(const FactCell& c, const FactK& kk, const FactAdj& ad, int t0, int nt, int mi, char* ws,
                         const double2* Z, const double2* Q, hipStream_t s) {
  const int nkb = (ad.Mt + 32 * mi - 1) / (32 * mi);
  const int nu = kk.n_pad / (32 * mi) * nkb;
  int nab = 0;
  for (int t = t0; t < t0 + nt; ++t) nab = nab > (c.nat[t] + 15) / 16 ? nab : (c.nat[t] + 15) / 16;
  const int nc = (kk.n_pad / (16 * mi) * nab * ad.nseg + 3) / 4;
  const dim3 grid(nu + nc, nt);
  if (mi == 2)
    hipLaunchKernelGGL((k_adj_uc<2, 4>), grid, dim3(256), 0, s, c, kk, ad, t0, nu, nab, ws, (const d2*)Z, (const d2*)Q);
  else
    hipLaunchKernelGGL((k_adj_uc<1, 4>), grid, dim3(256), 0, s, c, kk, ad, t0, nu, nab, ws, (const d2*)Z, (const d2*)Q);
  return hipGetLastError();
}

hipError_t launch_adj_gt(const FactCell& c, const FactK& kk, const FactAdj& ad, int t0, int nt, char* ws,
                         hipStream_t s) {
  const int nkb = (ad.Mt + 63) / 64;
  hipLaunchKernelGGL((k_adj_gt<2, 4>), dim3(nkb * nkb, nt, ad.ngt), dim3(256), 0, s, c, kk, ad, t0, ws);
  return hipGetLastError();
}

hipError_t launch_adj_reduce(const FactCell& c, const FactAdj& ad, int n_types, int n_atoms, const char* ws,
                             double2* gT, double* gtau, hipStream_t s) {
  const int M = 2 * c.n_l, ntb = (M * M + 255) / 256;
  hipLaunchKernelGGL(k_adj_reduce, dim3(ntb + (3 * n_atoms + 3) / 4, n_types), dim3(256), 0, s, c, ad, n_types, ntb, ws,
                     (d2*)gT, gtau);
  return hipGetLastError();
}

}  // namespace hsb
