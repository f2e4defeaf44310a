// Type-factored H and S (the compression of A and B that Sec. 7 names as future work).
//
// Every coefficient of atom a (type t) is its type's coefficient at the origin times the atom's
// structure phase, W_a[k][G] = E_a(G) W0_t[k][G], E_a(G) = e^{i K_G . tau_a}, k = (A|B, l, m).
// T and the radial data are per type, so the atom sums of Eqs. 4-5 factor entry by entry:
//
//   H = sum_t P_t .* (W0_t^H T_t W0_t),  S = sum_t P_t .* (W0_t^H Lam_t W0_t),
//   P_t[G'][G] = sum_{a in t} conj(E_a(G')) E_a(G).
//
// W0_t is real up to a unitary map of m at fixed l: with the real harmonics s_{l,mu} of K_hat,
// i^l conj(Y_lm) = sum_mu c(l,m,mu) s_{l,mu}.  So with R_t[(X,l,mu)][G] = pre x_l(G) s_{l,mu}(G)
// (real; X = A|B, x_l = a_l|b_l) and T'_t = C^H T_t C,
//
//   W0^H T W0 = R^T (T' R),   W0^H Lam W0 = R^T (Lam R)   (Lam depends on l only),
//
// i.e. two real products per H entry and one per S entry and row, where the complex form takes
// three and three (3M) and stages complex operands.
//
//   k_fact_tables  K vectors, phases E, R, and T' per type (one launch, blocks by role)
//   k_fact_y       Y_t = T'_t R_t
//   k_fact_hs      the upper triangles of H and S
//
// k_fact_hs runs on v_mfma_f64_16x16x4f64 with its operands fed through LDS (TypedTile in wave_tile.h), two
// workgroups of 64 x 32 outputs to a compute unit; R, lam R, Y and E are block-major, so that what a tile reads of an
// array lies together.
// Bound by the FP64 matrix cores: at N_G = 12000, 128 atoms, l_max = 10 they are busy for 80 % of its 7.8 ms (at
// 2.3 GHz); the rest is waits at the ring's barriers and the copies.  One workgroup of 64 x 64 on eight waves took 8.3 ms;
// with its copies and their address arithmetic right behind the barrier 8.9; with a wave's row and column not
// known to be uniform, so that the ring ran on vector registers, 9.9; and 64 x 64 on 2 x 2 waves with operands read
// straight from global memory into registers, no barriers, 9.2.  The FP64 vector units share the matrix cores' pipe:
// the addition theorem's sum over l in place of the S product has fewer operations and was slower in every form
// tried.
#include "harmonics.h"
#include "hs_internal.h"
#include "special.h"
#include "tiles.h"
#include "wave_tile.h"

namespace hsb {

namespace {

__device__ inline int find_block(const FactK* ks, int nk, int b, int FactK::*first) {
  int lo = 0, hi = nk - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ks[mid].*first <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

constexpr int kTabG = 64;          // columns per workgroup of k_fact_tables
constexpr int kTabWaves = 16;
constexpr int kTabS = kTabG + 1;  // their stride in LDS: the transposed copies read along the rows

// Blocks x < ngb: type blockIdx.y's R rows and phases (and, for the first type, the K vectors) of 64
// columns; blocks past them: T'.  Latency-bound at small bases (a few hundred workgroups of short serial
// recurrences), bandwidth-bound on its writes at large ones, so the work is spread over the workgroup:
// wave 0 runs the backward Bessel recurrence of its 64 columns while the others run the power series (columns
// with x < 2; l dealt over the waves) and the Legendre recurrences (m dealt over the waves), whose
// coefficients are compile-time tables.  16 waves: 14.5 us at N_G = 1237 in 3 types, 44 us at 12000 in 4; with 4 waves
// 18.9 and 62.
__global__ void __launch_bounds__(64 * kTabWaves) k_fact_tables(FactCell c, RadialArgs ra, const TypeConsts* __restrict__ consts,
                                                     FactK one, const FactK* __restrict__ many, int nk, int ngb,
                                                     const int32_t* __restrict__ g, const double* __restrict__ tau,
                                                     const FactRep* __restrict__ rep, FactAdj ad,
                                                     const double2* __restrict__ T, char* __restrict__ ws) {
  extern __shared__ double sh[];
  const int t = blockIdx.y;
  const int tid = threadIdx.x;
  const int lmax = c.l_max, nl1 = lmax + 1;
  if ((int)blockIdx.x >= ngb) {  // T'[r][k], stored [k][r] zero-padded
    const int64_t e = (int64_t)(blockIdx.x - ngb) * (64 * kTabWaves) + tid;
    const int k = (int)(e / c.Mc), r = (int)(e % c.Mc);
    if (k >= c.Mr) return;
    const int M = 2 * c.n_l;
    double2 v = make_double2(0.0, 0.0);
    if (k < M && r < M) {
      const int xr = r >= c.n_l, xk = k >= c.n_l;
      int lr, mr, lk, mk;
      lm_of(r - xr * c.n_l, lr, mr);
      lm_of(k - xk * c.n_l, lk, mk);
      const double2* Tt = T + (int64_t)c.type[t] * M * M;
      const int br = xr * c.n_l + lr * lr + lr, bk = xk * c.n_l + lk * lk + lk;
      for (int ir = 0; ir < (mr ? 2 : 1); ++ir)
        for (int ik = 0; ik < (mk ? 2 : 1); ++ik) {
          const int m1 = ir ? -mr : mr, m2 = ik ? -mk : mk;
          const double2 x = times_i(Tt[(int64_t)(br + m1) * M + bk + m2],
                                    harmonic_power(lk, m2, mk) - harmonic_power(lr, m1, mr));
          v.x += x.x;
          v.y += x.y;
        }
      if (mr && mk) {
        v.x *= 0.5; v.y *= 0.5;
      } else if (mr || mk) {
        v.x *= 0.70710678118654752440; v.y *= 0.70710678118654752440;
      }
    }
    ((double2*)(ws + c.TT))[((int64_t)t * c.Mr + k) * c.Mc + r] = v;
    return;
  }
  const FactK& kk = many ? many[find_block(many, nk, blockIdx.x, &FactK::gblk0)] : one;
  const int64_t n_pad = kk.n_pad;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = (blockIdx.x - kk.gblk0) * kTabG + lane;
  const bool valid = G < kk.n;
  double* ang = sh;                            // [n_l][64] real harmonics times pre
  double* jl = ang + c.n_l * kTabS;            // [l_max + 2][64]
  double* ab = jl + (lmax + 2) * kTabS;        // [2][l_max + 1][64]
  double kx = 0.0, ky = 0.0, kz = 0.0;
  if (valid) {
    const int32_t* gi = g + 3 * (kk.g_row + G);
    const double n0 = gi[0] + kk.kfrac[0], n1 = gi[1] + kk.kfrac[1], n2 = gi[2] + kk.kfrac[2];
    kx = n0 * c.bvec[0] + n1 * c.bvec[3] + n2 * c.bvec[6];
    ky = n0 * c.bvec[1] + n1 * c.bvec[4] + n2 * c.bvec[7];
    kz = n0 * c.bvec[2] + n1 * c.bvec[5] + n2 * c.bvec[8];
  }
  const double kn = sqrt(kx * kx + ky * ky + kz * kz);
  const double x = kn * c.r_mt[t];
  if (wave == 0) {
    if (t == 0) {
      double* kv = (double*)(ws + kk.kv);
      kv[4 * G + 0] = kx; kv[4 * G + 1] = ky; kv[4 * G + 2] = kz; kv[4 * G + 3] = kn;
    }
    if (!(x < 2.0)) sph_bessel_back(lmax + 1, x, jl + lane, kTabS);
  } else {
    if (x < 2.0) {
      for (int l = wave - 1; l <= lmax + 1; l += kTabWaves - 1) jl[l * kTabS + lane] = sph_bessel_series(l, x);
    }
    double ct = 1.0, wr = 0.0, wi = 0.0;
    if (!(kn < 1e-12)) {
      const double r = 1.0 / kn;
      ct = kz * r; wr = kx * r; wi = ky * r;
    }
    double pr = c.pre, pi = 0.0;  // pre w^m
    int mp = 0;
    for (int m = wave - 1; m <= lmax; m += kTabWaves - 1) {
      for (; mp < m; ++mp) {
        const double q = pr * wr - pi * wi;
        pi = pr * wi + pi * wr;
        pr = q;
      }
      const double f = m ? 1.41421356237309504880 : 1.0;
      const double sr = f * pr, si = f * pi;
      double p0 = 0.0, p1 = kLegendre.diag[m];
      for (int l = m; l <= lmax; ++l) {
        if (l > m) {
          const double q = kLegendre.a[l][m] * (ct * p1 - kLegendre.b[l][m] * p0);
          p0 = p1;
          p1 = q;
        }
        ang[(l * l + l + m) * kTabS + lane] = p1 * sr;
        if (m) ang[(l * l + l - m) * kTabS + lane] = p1 * si;
      }
    }
  }
  __syncthreads();
  for (int l = wave; l <= lmax; l += kTabWaves) {
    double u, du, ud, dud;
    if (consts) {
      const double* q = consts->radial[c.type[t]][l];
      u = q[0]; du = q[1]; ud = q[2]; dud = q[3];
    } else {
      const double* q = ra.v[t * nl1 + l];
      u = q[0]; du = q[1]; ud = q[2]; dud = q[3];
    }
    const double det = u * dud - ud * du;
    const double val = jl[l * kTabS + lane];
    const double up = jl[(l + 1) * kTabS + lane];
    const double dj = l ? (l * jl[(l - 1) * kTabS + lane] - (l + 1) * up) / (2.0 * l + 1.0) : -up;
    const double slope = kn * dj;
    ab[l * kTabS + lane] = (val * dud - ud * slope) / det;
    ab[(nl1 + l) * kTabS + lane] = (u * slope - du * val) / det;
  }
  __syncthreads();
  const int blk = blockIdx.x - kk.gblk0;
  double* R = (double*)(ws + kk.R) + ((int64_t)blk * c.n_act + t) * c.Mr * 64 + lane;
  double* LR = (double*)(ws + kk.LR) + ((int64_t)blk * c.n_act + t) * c.Mr * 64 + lane;
  for (int L = wave; L < c.n_l; L += kTabWaves) {
    int l, m;
    lm_of(L, l, m);
    const double s = ang[L * kTabS + lane];
    const double xa = valid ? s * ab[l * kTabS + lane] : 0.0, xb = valid ? s * ab[(nl1 + l) * kTabS + lane] : 0.0;
    R[L * 64] = xa;
    LR[L * 64] = xa;
    R[(c.n_l + L) * 64] = xb;
    LR[(c.n_l + L) * 64] = (consts ? consts->udot2[c.type[t]][l] : ra.v[t * nl1 + l][4]) * xb;
  }
  for (int r = 2 * c.n_l + wave; r < c.Mr; r += kTabWaves) R[r * 64] = LR[r * 64] = 0.0;
  double2* E = (double2*)(ws + kk.E) + ((int64_t)blk * c.e_rows + c.eoff[t]) * 64 + lane;
  double2* EW = (double2*)(ws + kk.EW) + ((int64_t)blk * c.e_rows + c.eoff[t]) * 64 + lane;
  const int nt = c.nat[t], erows = (nt + kFactRows - 1) / kFactRows * kFactRows;
  for (int a = wave; a < erows; a += kTabWaves) {
    double2 v = make_double2(0.0, 0.0);
    double wt = 1.0;
    if (a < nt && valid) {
      const int at = rep ? rep[c.atom0[t] + a].atom : c.atom0[t] + a;
      if (rep) wt = rep[c.atom0[t] + a].weight;
      double s, q;
      sincos(kx * tau[3 * at + 0] + ky * tau[3 * at + 1] + kz * tau[3 * at + 2], &s, &q);
      v = make_double2(q, s);
    }
    E[a * 64] = v;
    if (rep) EW[a * 64] = make_double2(wt * v.x, wt * v.y);
  }
  if (!ad.Mt) return;
  double2* ET = (double2*)(ws + ad.ET) + ((int64_t)ad.etb[t] * n_pad + G) * 32;
  for (int a = wave; a < (nt + 31) / 32 * 32; a += kTabWaves)
    ET[(int64_t)(a / 32) * n_pad * 32 + a % 32] = a < nt ? E[a * 64] : make_double2(0.0, 0.0);
  // transposed copy of R: lanes along the rows
  const int G0 = (blockIdx.x - kk.gblk0) * kTabG;
  double* RT = (double*)(ws + ad.RT) + (int64_t)t * n_pad * ad.Mt + G0 * 64;
  for (int e = tid; e < kTabG * ad.Mt; e += 64 * kTabWaves) {
    const int q = e / ad.Mt, r = e - q * ad.Mt;
    double v = 0.0;
    if (r < 2 * c.n_l && G0 + q < kk.n) {
      const int x2 = r >= c.n_l, L = r - x2 * c.n_l;
      int l, m;
      lm_of(L, l, m);
      v = ang[L * kTabS + q] * ab[(x2 * nl1 + l) * kTabS + q];
    }
    RT[(int64_t)(r / 64) * n_pad * 64 + q * 64 + r % 64] = v;
  }
}


// Y_t = T'_t R_t (real parts only if REAL): workgroup of 2 x 2 waves, each 16 MI rows x 16 NJ columns.
template <int MI, int NJ, bool REAL>
__global__ void __launch_bounds__(256, 2) k_fact_y(FactCell c, FactK one, const FactK* __restrict__ many, int nk,
                                                   char* __restrict__ ws) {
  constexpr int KC = 4;
  const FactK& kk = many ? many[find_block(many, nk, blockIdx.x, &FactK::yblk0)] : one;
  const int t = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int row0 = blockIdx.y * 32 * MI + (wave >> 1) * 16 * MI;
  const int col0 = (blockIdx.x - kk.yblk0) * 32 * NJ + (wave & 1) * 16 * NJ;
  if (row0 >= c.Mr || col0 >= kk.n) return;
  const d2* tp = (const d2*)(ws + c.TT) + ((int64_t)t * c.Mr + lk) * c.Mc + row0 + MI * lr;
  const int64_t blk = col0 / 64;  // a workgroup's columns lie in one block
  const double* rp = (const double*)(ws + kk.R) + ((blk * c.n_act + t) * c.Mr + lk) * 64 + col0 % 64 + NJ * lr;
  typedef typename DVec<NJ>::T VB;
  d4 re[MI][NJ], im[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) re[i][j] = im[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  d2 a[KC][MI], an[KC][MI];
  VB b[KC], bn[KC];
  auto load = [&](int ch, d2 (&av)[KC][MI], VB (&bv)[KC]) {
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      const int64_t k = (int64_t)(ch * KC + q) * 4;
#pragma unroll
      for (int i = 0; i < MI; ++i) av[q][i] = tp[k * c.Mc + i];
      bv[q] = *(const VB*)(rp + k * 64);
    }
  };
  const int nch = c.Mr / (4 * KC);
  load(0, a, b);
  for (int ch = 0; ch < nch; ++ch) {
    load(ch + 1 < nch ? ch + 1 : ch, an, bn);
#pragma unroll
    for (int q = 0; q < KC; ++q)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const double bj = DVec<NJ>::get(b[q], j);
          re[i][j] = MFMA(a[q][i].x, bj, re[i][j]);
          if constexpr (!REAL) im[i][j] = MFMA(a[q][i].y, bj, im[i][j]);
        }
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      b[q] = bn[q];
#pragma unroll
      for (int i = 0; i < MI; ++i) a[q][i] = an[q][i];
    }
  }
  // D layout of the 16x16 f64 MFMA: lane l, element q -> row l/16 + 4q, column l%16
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = row0 + MI * (lk + 4 * q) + i;
      if (row >= c.Mr) continue;
      const int64_t o = ((blk * c.n_act + t) * c.Mr + row) * 64 + col0 % 64 + NJ * lr;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if constexpr (REAL) ((double*)(ws + kk.Y))[o + j] = re[i][j][q];
        else ((d2*)(ws + kk.Y))[o + j] = d2{re[i][j][q], im[i][j][q]};
      }
    }
}

// Upper triangles of H and S: per type P_t times the sums over its R rows (TypedTile), into the running H and S.
// 64 x 32 tiles, the halves of 64 x 64 ones (MI = 2), or quarters of those (MI = 1).
template <int MI, bool REAL>
__global__ void __launch_bounds__(256, 2) k_fact_hs(FactCell c, FactK one, const FactK* __restrict__ many, int nk,
                                                    int num_wg, int gr, const char* __restrict__ ws,
                                                    void* __restrict__ H, void* __restrict__ S) {
  constexpr int PARTS = 4 / MI;
  __shared__ __align__(16) char lds[TypedTile<MI, REAL>::lds_bytes];
  int start, len;
  xcd_range(blockIdx.x % kXcds, num_wg, start, len);
  const int w = start + blockIdx.x / kXcds;
  FactK kk = one;
  if (many) kk = many[find_block(many, nk, w / PARTS, &FactK::tile0)];
  const int n = kk.n, nb = (n + 63) / 64;
  int bi, bj;
  if (gr > 0) grouped_decode(w / PARTS - kk.tile0, nb, gr, bi, bj);
  else tri_decode(w / PARTS - kk.tile0, nb, bi, bj);
  const int part = w % PARTS;
  if (bi * 64 + part / 2 * 32 >= n || bj * 64 + part % 2 * 32 >= n) return;
  if (bi == bj && part == 2) return;  // below the diagonal
  TypedTile<MI, REAL> tile(c, kk, ws, lds, bi, part / 2, bj, part % 2, 0, c.n_act);
  const int r0 = tile.row0(), c0 = tile.col0();
  const bool active = r0 < n && c0 < n && c0 + 16 > r0;
  d4 hR[MI], hI[MI], sR[MI], sI[MI];
  clear(hR);
  clear(hI);
  clear(sR);
  clear(sI);
  for (int t = 0; t < c.n_act; ++t) {
    d4 pR[MI], pI[MI], m1[MI], m2[MI], F[MI];
    tile.phase_sums(t, active, pR, pI);
    tile.row_sums(active, m1, m2, F);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      sR[i] += pR[i] * F[i];
      if constexpr (REAL) {
        hR[i] += pR[i] * m1[i];
      } else {
        sI[i] += pI[i] * F[i];
        hR[i] += pR[i] * m1[i] - pI[i] * m2[i];
        hI[i] += pR[i] * m2[i] + pI[i] * m1[i];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = tile.row(i, q), col = tile.col();
      if (r < n && col < n && col >= r) {
        const int64_t o = kk.out_off + (int64_t)r * n + col;
        if constexpr (REAL) {
          ((double*)H)[o] = hR[i][q];
          ((double*)S)[o] = sR[i][q];
        } else {
          ((d2*)H)[o] = d2{hR[i][q], hI[i][q]};
          ((d2*)S)[o] = d2{sR[i][q], sI[i][q]};
        }
      }
    }
}

// XL[r][G] = lam[r] X[r][G]; one thread per G, rows over blockIdx.y.
__global__ void __launch_bounds__(256) k_scale_rows(const double2* __restrict__ X, const double* __restrict__ lam,
                                                    int rows, int n_pad, double2* __restrict__ XL) {
  const int G = blockIdx.x * blockDim.x + threadIdx.x;
  if (G >= n_pad) return;
  for (int r = blockIdx.y; r < rows; r += gridDim.y) {
    const double2 v = X[(int64_t)r * n_pad + G];
    XL[(int64_t)r * n_pad + G] = make_double2(lam[r] * v.x, lam[r] * v.y);
  }
}

}  // namespace

int fact_tiles(int n) {
  const int nb = (n + 63) / 64;
  return nb * (nb + 1) / 2;
}

hipError_t launch_fact_tables(const FactCell& c, const RadialArgs& ra, const TypeConsts* consts, const FactK& one,
                              const FactK* many, int nk, int ngb, const int32_t* g, const double* tau,
                              const FactRep* rep, const FactAdj& ad, const double2* T, char* ws, hipStream_t s) {
  const size_t lds = (size_t)(c.n_l + c.l_max + 2 + 2 * (c.l_max + 1)) * kTabS * sizeof(double);
  const int ntb = (int)(((int64_t)c.Mr * c.Mc + 64 * kTabWaves - 1) / (64 * kTabWaves));
  hipLaunchKernelGGL(k_fact_tables, dim3(ngb + ntb, c.n_act), dim3(64 * kTabWaves), lds, s, c, ra, consts, one, many, nk, ngb, g,
                     tau, rep, ad, T, ws);
  return hipGetLastError();
}

hipError_t launch_fact_y(const FactCell& c, const FactK& one, const FactK* many, int nk, int nblk, int mi, bool real,
                         char* ws, hipStream_t s) {
  const dim3 grid(nblk, (c.Mr + 32 * mi - 1) / (32 * mi), c.n_act);
  if (mi == 2 && real) hipLaunchKernelGGL((k_fact_y<2, 2, true>), grid, dim3(256), 0, s, c, one, many, nk, ws);
  else if (mi == 2) hipLaunchKernelGGL((k_fact_y<2, 2, false>), grid, dim3(256), 0, s, c, one, many, nk, ws);
  else if (real) hipLaunchKernelGGL((k_fact_y<1, 1, true>), grid, dim3(256), 0, s, c, one, many, nk, ws);
  else hipLaunchKernelGGL((k_fact_y<1, 1, false>), grid, dim3(256), 0, s, c, one, many, nk, ws);
  return hipGetLastError();
}

hipError_t launch_fact_hs(const FactCell& c, const FactK& one, const FactK* many, int nk, int tiles, bool real, int gr,
                          int num_cus, const char* ws, void* H, void* S, hipStream_t s) {
  // Quarters while there is one for every compute unit at most: half the products per workgroup, but each operand
  // read for half as many (3-type cell of l_max 7: 28 tiles 44 us as quarters, 51 as halves; 66 tiles 59 and 57; 1128 tiles
  // of a 2-type cell 253 and 224).
  const bool quarters = 4 * tiles <= num_cus;
  const int num_wg = (quarters ? 4 : 2) * tiles;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(num_wg), dim3(256), 0, s, c, one, many, nk, num_wg, gr, ws, H, S);
  };
  if (quarters) real ? go(k_fact_hs<1, true>) : go(k_fact_hs<1, false>);
  else real ? go(k_fact_hs<2, true>) : go(k_fact_hs<2, false>);
  return hipGetLastError();
}

hipError_t launch_scale_rows(const double2* X, const double* lam, int rows, int n_pad, double2* XL, hipStream_t s) {
  dim3 grid((n_pad + 255) / 256, rows < 256 ? rows : 256);
  hipLaunchKernelGGL(k_scale_rows, grid, dim3(256), 0, s, X, lam, rows, n_pad, XL);
  return hipGetLastError();
}

}  // namespace hsb
