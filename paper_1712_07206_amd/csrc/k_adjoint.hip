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
// All on v_mfma_f64_16x16x4f64, the first two through an LDS ring (wave_tile.h); Z, Q, R Z and the
// transposed copies of R and E (k_fact_tables) are block-major, so that chunks are contiguous runs.
// Deterministic: fixed orders, no atomics.
// At N_G = 6000, 64 atoms in two types, l_max = 10 (3.9 ms): k_adj_zq 2.3 ms, 71 % of it the matrix cores' time, the rest
// the 2.3 GB of Z and Q it writes, the reads of gH and gS and the ring's waits (2.6 ms with one type per workgroup and
// rows of n_pad); k_adj_uc 1.55 ms, of which its products take 1.15 at a large matrix product's rate (1.73 ms with one
// workgroup of 64 columns G on eight waves to a compute unit; at N_G = 801 in 3 types, where the tiles are fewer than
// the compute units, 37 and 61 us); k_adj_gt 0.07 ms.
#include <type_traits>

#include "harmonics.h"
#include "hs_internal.h"
#include "tiles.h"
#include "wave_tile.h"

namespace hsb {

namespace {

// Z_t and Q_t (zeros outside n x n, up to n_pad), block-major: [type][64 columns][n_pad rows][64]; 64 x 32 tiles of the
// square (MI = 2) or 32 x 32 ones (MI = 1), column halves interleaved in blockIdx.x and row halves in blockIdx.y, `per`
// types each.  Writes 32 bytes per type and element.
template <int MI>
__global__ void __launch_bounds__(256, 2) k_adj_zq(FactCell c, FactK kk, int t0, int per, const d2* __restrict__ gH,
                                                   const d2* __restrict__ gS, const char* __restrict__ ws,
                                                   d2* __restrict__ Z, d2* __restrict__ Q) {
  constexpr int PARTS = 2 / MI;
  const int bj = blockIdx.x / 2;
  __shared__ __align__(16) char lds[TypedTile<MI, false>::lds_bytes];
  const int n = kk.n;
  const int64_t n_pad = kk.n_pad;
  const int first = blockIdx.z * per;
  TypedTile<MI, false> tile(c, kk, ws, lds, blockIdx.y / PARTS, blockIdx.y % PARTS, bj, blockIdx.x % 2,
                            t0 + first, t0 + first + per);
  const bool active = tile.row0() < n && tile.col0() < n;
  const int col = tile.col();
  d2 h[MI][4], s[MI][4];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = tile.row(i, q);
      h[i][q] = s[i][q] = d2{0.0, 0.0};
      if (r < n && col < n) {
        h[i][q] = gH[(int64_t)r * n + col];
        s[i][q] = gS[(int64_t)r * n + col];
      }
    }
  for (int t = first; t < first + per; ++t) {
    const int64_t o = ((int64_t)t * (n_pad / 64) + bj) * n_pad * 64 + col % 64;
    d4 pR[MI], pI[MI], m1[MI], m2[MI], F[MI];
    tile.phase_sums(t0 + t, active, pR, pI);
    tile.row_sums(active, m1, m2, F);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = tile.row(i, q);
        d2 vz = d2{0.0, 0.0}, vq = d2{0.0, 0.0};  // (the sums of pad columns may hold anything)
        if (r < n && col < n) {
          const d2 gh = h[i][q], gs = s[i][q];
          const double a = m1[i][q], b = m2[i][q], d = F[i][q], pr = pR[i][q], pi = pI[i][q];
          vz = d2{gh.x * pr + gh.y * pi, gh.y * pr - gh.x * pi};
          vq = d2{gh.x * a + gh.y * b + gs.x * d, gh.x * b - gh.y * a - gs.y * d};
        }
        Z[o + (int64_t)r * 64] = vz;
        Q[o + (int64_t)r * 64] = vq;
      }
  }
}

// Complex A [k][64 rows], real B [k][64 columns]: re, im += sum over k in [4 k0, 4 k1) (4-row steps), in chunks of KC
// steps (k1 - k0 a multiple of KC).
template <int MI, int NJ, int KC>
__device__ __forceinline__ void product_cr(const d2* __restrict__ A, const double* __restrict__ B, int k0, int k1,
                                           d4 (&re)[MI][NJ], d4 (&im)[MI][NJ]) {
  typedef typename DVec<NJ>::T VB;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const d2* ap = A + lk * 64 + MI * lr;
  const double* bp = B + lk * 64 + NJ * lr;
  struct Chunk { d2 a[KC][MI]; VB b[KC]; };
  auto load = [&](int s, Chunk& x) {
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      const int64_t k = (int64_t)(s + q) * 4;
#pragma unroll
      for (int i = 0; i < MI; ++i) x.a[q][i] = ap[k * 64 + i];
      x.b[q] = *(const VB*)(bp + k * 64);
    }
  };
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

// Workgroups blockIdx.x < nu: 32 (G) x 64 tiles of UT[G][k] = sum_G' Z[G'][G] RT[G'][k], waves of 32 x 16; nu2 more: the
// last, partly empty ones in k.  With one or two blocks of 16 k the waves of one column of blocks take every fourth
// or second step, and their sums are added in the end, so that such a tile takes a quarter or half of the time.
// Past them: the phase sums of 32 columns G and 32 atoms over a segment of G', waves of 16 x 16:
// D[G][a] = sum_G' Q[G'][G] conj(ET[G'][a]) (three real products: P1 = q_r e_r, P2 = q_i e_i,
// P3 = (q_r + q_i)(e_r - e_i), Re = P1 + P2, Im = P3 - P1 + P2), then sum_G K_G Im(E_a(G) D[G][a])
// over the wave's columns into part[seg][16 columns][phase row][3].
// Types over the slowest index, so the largest tiles come first and the smaller fill up the end.
// Operands through an LDS ring in chunks of 16 G' (8 KB of Z or Q, half of each row of a block; 8 KB of RT or ET, one
// run); two workgroups to a compute unit, one's waits being the other's time.  32 columns G rather than 32 k, since Z has
// twice the bytes.  Three workgroups with three stages: the same.  The tiles of one 32 G on one XCD, which then reads
// that part of Z from memory once.
__global__ void __launch_bounds__(256, 2) k_adj_uc(FactCell c, FactK kk, FactAdj ad, int t0, int nu, int nu2, int nab,
                                                   const char* __restrict__ ws, const d2* __restrict__ Z,
                                                   const d2* __restrict__ Q) {
  typedef Ring<4, 16 * 1024, 4> R;
  __shared__ __align__(16) char lds[R::bytes];
  const int64_t np = kk.n_pad;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const bool is_u = (int)blockIdx.x < nu + nu2;
  const int first = (int)blockIdx.x < nu ? 0 : is_u ? nu : nu + nu2;
  const int num = (int)blockIdx.x < nu ? nu : is_u ? nu2 : (int)gridDim.x - nu - nu2;
  int start, len;
  xcd_range((blockIdx.x - first) % kXcds, num, start, len);
  const int w = start + (blockIdx.x - first) / kXcds;
  // type (slowest), 32 columns G, segment, block of k or of atoms
  const int full = c.n_l / 32;  // full 64-wide blocks of the 2 N_L k
  const int per = !is_u ? nab : (int)blockIdx.x < nu ? full : 1, segs = is_u ? 1 : ad.nseg;
  const int blk = (int)blockIdx.x >= nu && is_u ? full : w % per;
  const int seg = w / per % segs, gb = w / per / segs % (kk.n_pad / 32), y = w / per / segs / (kk.n_pad / 32);
  const int t = t0 + y;
  if (!is_u && blk * 32 >= c.nat[t]) return;
  const int nch = kk.n_pad / 16;
  const int c0 = is_u ? 0 : (int)((int64_t)nch * seg / ad.nseg);
  const int c1 = is_u ? nch : (int)((int64_t)nch * (seg + 1) / ad.nseg);
  const char* pa = uniform((const char*)((is_u ? Z : Q) + (((int64_t)y * (np / 64) + gb / 2) * np + c0 * 16) * 64 +
                                         gb % 2 * 32) + wave * 2048);
  const char* pb = uniform(ws + (is_u ? ad.RT + ((int64_t)t * (ad.Mt / 64) + blk) * np * 512
                                      : ad.ET + ((int64_t)(ad.etb[t] + blk) * np + c0 * 16) * 512) +
                           wave * 1024);
  R ring{lds, c1 - c0};
  const unsigned half = (lane >> 5) * 1024 + (lane & 31) * 16;  // of two rows of 512 bytes in rows of 1 KB
  int issued = c0;
  auto issue = [&]() {
    if (issued == c1) return;
    ++issued;
    char* st = ring.stage(wave);
    auto copy = [&](const char* p, unsigned off, int i) {
      __builtin_amdgcn_global_load_lds((const void*)(p + off), (lds_ptr)(st + i * 4096), 16, 0, 0);
    };
    copy(pa, half, 0);
    copy(pa + 8192, half, 1);
    copy(pb, lane * 16, 2);
    copy(pb + 4096, lane * 16, 3);
    pa += 16 * 1024;
    pb += 8 * 1024;
  };
  for (int i = 0; i < R::stages - 1; ++i) issue();
  if (is_u) {
    const int k16 = (2 * c.n_l + 15) / 16 - 4 * blk;       // blocks of 16 k left
    const int cols = k16 == 1 ? 1 : k16 == 2 ? 2 : 4;      // wave columns
    const int turns = 4 / cols, turn = wave / cols;  // this wave's steps: s = turn mod turns
    const int bcol = wave % cols * 16 + lr;
    d4 re[2], im[2];
    clear(re);
    clear(im);
    struct Ops { d2 a[2]; double b; };
    auto run = [&](auto per) {  // steps of a chunk per wave
      constexpr int PER = decltype(per)::value, TURNS = 4 / PER;
      section<PER, 2>(
          ring, PER * nch, true, issue,
          [&](const char* st, int s) {
            const int r = 4 * (s * TURNS + turn) + lk;
            const d2* A = (const d2*)(st + r * 512) + lr;
            return Ops{{A[0], A[16]}, ((const double*)(st + 8 * 1024 + r * 512))[bcol]};
          },
          [&](const Ops& o, int i) {
            re[i] = MFMA(o.a[i].x, o.b, re[i]);
            im[i] = MFMA(o.a[i].y, o.b, im[i]);
          });
    };
    if (turns == 1) run(std::integral_constant<int, 4>{});
    else if (turns == 2) run(std::integral_constant<int, 2>{});
    else run(std::integral_constant<int, 1>{});
    if (turns > 1) {  // all copies have landed: the ring's memory is free once everyone is here
      __syncthreads();
      double* mine = (double*)lds + wave * 1024 + lane;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          mine[(i * 4 + q) * 64] = re[i][q];
          mine[(8 + i * 4 + q) * 64] = im[i][q];
        }
      __syncthreads();
      if (turn > 0) return;
      for (int o = 1; o < turns; ++o) {
        const double* other = mine + o * cols * 1024;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            re[i][q] += other[(i * 4 + q) * 64];
            im[i][q] += other[(8 + i * 4 + q) * 64];
          }
      }
    }
    d2* U = (d2*)(ws + ad.UT) + (((int64_t)y * (ad.Mt / 64) + blk) * np + gb * 32) * 64 + bcol;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) U[(16 * i + lk + 4 * q) * 64] = d2{re[i][q], im[i][q]};
    return;
  }
  const int row = (wave >> 1) * 16, col = (wave & 1) * 16 + lr;
  d4 p1[1], p2[1], p3[1];
  clear(p1);
  clear(p2);
  clear(p3);
  struct Ops { d2 a, b; };
  section<4, 1>(
      ring, 4 * (c1 - c0), true, issue,
      [&](const char* st, int s) {
        return Ops{((const d2*)(st + (4 * s + lk) * 512))[row + lr],
                   ((const d2*)(st + 8 * 1024 + (4 * s + lk) * 512))[col]};
      },
      [&](const Ops& o, int) {
        p1[0] = MFMA(o.a.x, o.b.x, p1[0]);
        p2[0] = MFMA(o.a.y, o.b.y, p2[0]);
        p3[0] = MFMA(o.a.x + o.a.y, o.b.x - o.b.y, p3[0]);
      });
  // lane: atom 32 blk + col, columns G = 32 gb + row + lk + 4 q; pads of E are zero
  const double* kv = (const double*)(ws + kk.kv);
  const d2* ET = (const d2*)(ws + ad.ET) + (int64_t)(ad.etb[t] + blk) * np * 32 + col;
  double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t G = gb * 32 + row + lk + 4 * q;
    const d2 e = ET[G * 32];
    const double re = p1[0][q] + p2[0][q], im = p3[0][q] - p1[0][q] + p2[0][q];
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
  const int a = blk * 32 + col;
  if (lk == 0 && a < c.nat[t]) {
    double* part =
        (double*)(ws + ad.partTau) + (((int64_t)seg * ad.ngb + gb * 2 + (wave >> 1)) * c.e_rows + c.eoff[t] + a) * 3;
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
  const int nkb = ad.Mt / (32 * MI);
  const int row0 = blockIdx.x / nkb * 32 * MI + (wave >> 1) * 16 * MI;
  const int col0 = blockIdx.x % nkb * 32 * MI + (wave & 1) * 16 * MI;
  const int nch = kk.n_pad / 4 / KC;
  const int k0 = (int)((int64_t)nch * seg / ad.ngt) * KC, k1 = (int)((int64_t)nch * (seg + 1) / ad.ngt) * KC;
  d4 re[MI][MI], im[MI][MI];
  clear(re);
  clear(im);
  product_cr<MI, MI, KC>(
      (const d2*)(ws + ad.UT) + ((int64_t)blockIdx.y * nkb + row0 / 64) * n_pad * 64 + row0 % 64,
      (const double*)(ws + ad.RT) + ((int64_t)t * nkb + col0 / 64) * n_pad * 64 + col0 % 64, k0, k1, re, im);
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
// Latency-bound: the segments' loads are unrolled by 8 to be in flight together (28 -> 18 us for 16 segments at l_max = 10,
// 13 -> 9 us for 13 at l_max = 7).
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
#pragma unroll 4
    for (int b = lane; b < ad.nseg * ad.ngb; b += 64) s += part[(int64_t)b * c.e_rows * 3];
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
#pragma unroll 8
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
  const bool quarters = 4 * nb * nb * nt <= num_cus;  // as in launch_fact_hs
  // gH and gS are read once for all types where the tiles alone fill the compute units several times over
  const int per = nb * nb >= 4 * num_cus ? nt : 1;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(2 * nb, quarters ? 2 * nb : nb, nt / per), dim3(256), 0, s, c, kk, t0, per,
                       (const d2*)gH, (const d2*)gS, ws, (d2*)Z, (d2*)Q);
  };
  quarters ? go(k_adj_zq<1>) : go(k_adj_zq<2>);
  return hipGetLastError();
}

hipError_t launch_adj_uc(const FactCell& c, const FactK& kk, const FactAdj& ad, int t0, int nt, char* ws,
                         const double2* Z, const double2* Q, hipStream_t s) {
  const int nb = kk.n_pad / 32;
  int nab = 0;
  for (int t = t0; t < t0 + nt; ++t) nab = nab > (c.nat[t] + 31) / 32 ? nab : (c.nat[t] + 31) / 32;
  const int nu = nt * nb * (c.n_l / 32), nu2 = c.n_l % 32 ? nt * nb : 0;
  hipLaunchKernelGGL(k_adj_uc, dim3(nu + nu2 + nt * nb * ad.nseg * nab), dim3(256), 0, s, c, kk, ad, t0, nu, nu2, nab, ws,
                     (const d2*)Z, (const d2*)Q);
  return hipGetLastError();
}

hipError_t launch_adj_gt(const FactCell& c, const FactK& kk, const FactAdj& ad, int t0, int nt, char* ws,
                         hipStream_t s) {
  const int nkb = ad.Mt / 64;
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
