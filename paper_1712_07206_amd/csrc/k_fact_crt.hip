// Residue form of the type-factored build (k_fact.hip): per active type t
//
//   H += P_t o (R_t^T Y_t),  S += P_t o (R_t^T Lam R_t),  P_t = E_t^H E_t,
//
// with R^T Y by residues on the 8- or 16-bit matrix cores and P, the S product and the sums over the
// types in FP64.
//
// Every column of R_t and Y_t is scaled by a power of two and rounded to integers (complex for Y), with
// the 2-norms of the scaled columns bounded so that a product's integer sums stay below M / 2 in
// magnitude, M the product of the n moduli m_i.  The residues in [-(m-1)/2, (m-1)/2] of both, as signed bytes
// (or bfloat16 or half integers), give exact sums v_i over a type's at most 338 rows (338 * 120^2 <
// 2^23: int32, or integers in FP32), and the integer is M frac(sum_i v_i y_i / m_i), y_i = (M / m_i)^{-1}
// mod m_i.  With y_i / m_i = h_i + l_i (mod 1), |h_i| <= 1/2 on a 2^-27 grid, sum v_i h_i is exact
// (13 * 2^23 / 2 * 2^27 < 2^53), and so is its distance to the nearest integer; l_i <= 2^-28 adds its
// part to FP64 precision.  The v_i need no reduction modulo m_i for that.  The only approximation is
// the rounding of the scaled columns.  R is real, so a complex product takes two products per modulus.
//
// Measured at N_G = 12000, 128 atoms, l_max = 10, 11 moduli: k_fact_crt 7.15 ms (7.95 with chunks of half the
// size and the copies right behind the barrier), of which the FP64 and integer matrix cores take 3.2 and the FP64
// vector units, which share the FP64 ones' pipe, 0.7; its copies alone 4.9 (66 GB from L2).  k_fact_residues
// 0.18 ms.  The stacked residue contraction over the 30976 rows of all atoms took 110 ms, with H off by 2e-11 of its
// norm against 2e-12 here.
#include <cmath>

#include "hs_internal.h"
#include "residues.h"
#include "tiles.h"
#include "wave_tile.h"

namespace hsb {

namespace {

typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef int i4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// One 16 x 16 step over 4 units of rows: lane l holds the unit l / 16 of row (column) l % 16; output element q:
// row 4 (l / 16) + q, column l % 16.
template <int EK>
struct ResMma;
template <>
struct ResMma<0> {
  typedef i4v T;
  static __device__ __forceinline__ T mma(u4 a, u4 b, T c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i4v, a), __builtin_bit_cast(i4v, b), c, 0, 0, 0);
  }
};
template <>
struct ResMma<1> {
  typedef f4v T;
  static __device__ __forceinline__ T mma(u4 a, u4 b, T c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
  }
};
template <>
struct ResMma<2> {
  typedef f4v T;
  static __device__ __forceinline__ T mma(u4 a, u4 b, T c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
  }
};

// A tile reads chunks of 48 KB, per type
//   phases   24 rows (1 KB each): E of its 64 rows, EW of its 64 columns
//   R rows   48 rows (512 bytes each): R of its rows, lam R of its columns
//   residues SPC steps, [modulus][step]: of its rows R's 4 units of 64 columns, of its columns Y's
//            [4][NC][64 columns] (NC: real and imaginary part)
// The residues lie block-major, a stream of each 64 columns for R (A) and for Y (B), steps past the last
// modulus zero; A holds the columns of each 32 even ones first (k_fact_crt).  (The same pieces from arrays of whole
// rows, 1 KB out of every 192 at N_G = 12000, took 15.2 ms against 12.4.)
constexpr int kChunk = 48 * 1024, kRowsE = kChunk / 2048, kRowsF = kChunk / 1024;
typedef Ring<3, kChunk> CrtRing;
template <bool REAL>
struct Stream {
  static constexpr int NC = REAL ? 1 : 2;        // products per modulus
  static constexpr int SPC = kChunk / 1024 / (4 + 4 * NC);  // steps per chunk
  static constexpr int a_res = SPC * 4 * 1024;   // A's bytes of a residue chunk (of the others: half)
};

// Residues of R (blockIdx.z = 0, stream A) or Y (1, B) of type blockIdx.y and the 64 columns blockIdx.x, and the
// reciprocal scales.  The scale is the largest power of two 2^f with 2^f ||x|| + sqrt(2 M) / 2 <= bound (the second
// term bounds the norm of the rounding errors), 1 for a zero column.  Bandwidth-bound on what it writes (n_mod
// bytes or 16-bit values per value of 8 bytes read, twice, the second time from cache).
constexpr int kResWaves = 16;
template <int EK, bool REAL>
__global__ void __launch_bounds__(64 * kResWaves) k_fact_residues(FactCell c, FactK kk, FactCrt cr,
                                                               char* __restrict__ ws) {
  constexpr int RU = EK == 0 ? 16 : 8, EB = 16 / RU, PER = 4 / EB;
  typedef Stream<REAL> St;
  __shared__ double part[kResWaves][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = blockIdx.y, G = blockIdx.x * 64 + lane;
  const bool is_b = blockIdx.z;
  const int parts = is_b ? St::NC : 1;  // values per row
  const int64_t np = kk.n_pad;
  const int M = 2 * c.n_l;
  const int64_t len = (int64_t)cr.n_r * (is_b ? kChunk - St::a_res : St::a_res);  // a type's part
  char* out = ws + (is_b ? cr.B : cr.A) + ((int64_t)blockIdx.x * c.n_act + t) * len;
  const double* x = (const double*)(ws + (is_b ? kk.Y : kk.R)) +
                    (((int64_t)blockIdx.x * c.n_act + t) * c.Mr * 64 + lane) * parts;
  const int ld = 64 * parts;
  double sq = 0.0;
  for (int k = wave; k < M; k += kResWaves)
    for (int p = 0; p < parts; ++p) {
      const double v = x[k * ld + p];
      sq += v * v;
    }
  part[wave][lane] = sq;
  __syncthreads();
  sq = 0.0;
  for (int i = 0; i < kResWaves; ++i) sq += part[i][lane];
  double sc = 1.0, inv = 1.0;
  if (sq > 0.0) {
    const double q = (cr.bound - 0.5 * sqrt(2.0 * (double)M)) / sqrt(sq) * (1.0 - 0x1p-30);
    int e = 0;
    (void)frexp(q, &e);  // q = mant * 2^e, mant in [0.5, 1): 2^(e-1) <= q
    sc = ldexp(1.0, e - 1);
    inv = ldexp(1.0, 1 - e);
  }
  if (wave == 0) ((double*)(ws + cr.inv))[((int64_t)blockIdx.z * c.n_act + t) * np + G] = inv;
  u4* o = (u4*)out + (is_b ? lane : (lane & 32) | ((lane & 1) << 4) | ((lane & 31) >> 1));
  const int units = 4 * cr.ks;
  for (int u = wave; u < units * parts; u += kResWaves) {
    const int unit = u / parts, p = u - unit * parts;
    double v[RU];
#pragma unroll
    for (int r = 0; r < RU; ++r) {
      const int k = unit * RU + r;
      v[r] = k < M ? rint(x[k * ld + p] * sc) : 0.0;  // the scale is a power of two: the product is exact
    }
    for (int i = 0; i < cr.n_mod; ++i) {
      const double m = cr.m[i], im = cr.inv_m[i];
      u4 q = u4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int r = 0; r < RU; ++r) q[r / PER] |= residue_bits<EK>(smod_d(v[r], m, im)) << (8 * EB * (r % PER));
      o[((i * units + unit) * parts + p) * 64] = q;
    }
  }
  // steps past the last modulus
  for (int u = cr.n_mod * units * parts + wave; u < cr.n_r * St::SPC * 4 * parts;
       u += kResWaves) o[u * 64] = u4{0u, 0u, 0u, 0u};
}

// Upper triangles of H and S, 64 x 64 tiles on 2 x 4 waves of 32 x 16.
//
// A residue step is 64 cycles of a wave's matrix core and as many of its FP64 vector unit, and what misses L2
// takes thousands: operands read straight into registers two steps ahead took 14.0 ms.  P, H, S and the residue sums
// of 64 x 64 outputs fill the register file.
template <int EK, bool REAL>
__global__ void __launch_bounds__(512, 2) k_fact_crt(FactCell c, FactK kk, FactCrt cr, int num_wg, int gr,
                                                     const char* __restrict__ ws, void* __restrict__ H,
                                                     void* __restrict__ S) {
  typedef ResMma<EK> Mma;
  typedef Stream<REAL> St;
  constexpr int NC = St::NC, SPC = St::SPC;
  __shared__ __align__(16) char lds[CrtRing::bytes + 2 * HSB_MAX_TYPES * 64 * 8];
  double* const inv_row = (double*)(lds + CrtRing::bytes);  // [type][64]
  double* const inv_col = inv_row + HSB_MAX_TYPES * 64;
  int start, len;
  xcd_range(blockIdx.x % kXcds, num_wg, start, len);
  const int w = start + blockIdx.x / kXcds;
  const int n = kk.n, nb = (n + 63) / 64;
  int bi, bj;
  if (gr > 0) grouped_decode(w, nb, gr, bi, bj);
  else tri_decode(w, nb, bi, bj);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int row0 = bi * 64, col0 = bj * 64, wr = wave >> 2, wc = wave & 3;
  if (col0 >= n) return;
  const int r0 = row0 + wr * 32, c0 = col0 + wc * 16;
  const bool active = r0 < n && c0 < n && c0 + 16 > r0;
  const int64_t np = kk.n_pad;
  {
    const double* inv = (const double*)(ws + cr.inv);
    for (int i = threadIdx.x; i < c.n_act * 64; i += 512) {
      const int t = i >> 6, g = i & 63;
      inv_row[i] = inv[(int64_t)t * np + row0 + g];
      inv_col[i] = inv[(int64_t)(c.n_act + t) * np + col0 + g] * cr.M;
    }
  }

  const int M = 2 * c.n_l, steps = cr.n_mod * cr.ks;
  CrtRing ring{lds, 0};
  for (int t = 0; t < c.n_act; ++t) ring.left += (c.nat[t] + kRowsE - 1) / kRowsE + cr.n_f + cr.n_r;
  // The next chunk to issue: type, part (0 phases, 1 R rows, 2 residues), chunks left of the part, sources.
  int it = 0, part = 0, n_left = 0;
  const char *pa = nullptr, *pb = nullptr;
  auto enter = [&]() {
    const int64_t ta = (int64_t)bi * c.n_act + it, tb = (int64_t)bj * c.n_act + it;
    if (part == 0) {
      n_left = (c.nat[it] + kRowsE - 1) / kRowsE;
      pa = ws + kk.E + ((int64_t)bi * c.e_rows + c.eoff[it]) * 1024;
      pb = ws + kk.EW + ((int64_t)bj * c.e_rows + c.eoff[it]) * 1024;
    } else if (part == 1) {
      n_left = cr.n_f;
      pa = ws + kk.R + ta * c.Mr * 512;
      pb = ws + kk.LR + tb * c.Mr * 512;
    } else {
      n_left = cr.n_r;
      pa = ws + cr.A + ta * cr.n_r * St::a_res;
      pb = ws + cr.B + tb * cr.n_r * (kChunk - St::a_res);
    }
  };
  auto issue = [&]() {
    if (it >= c.n_act) return;
    char* st = ring.stage(wave);
    const int na = part == 2 ? St::a_res : kChunk / 2;
#pragma unroll
    for (int i = 0; i < CrtRing::copies; ++i) {
      const int o = (wave + 8 * i) * 1024;
      __builtin_amdgcn_global_load_lds((const void*)((o < na ? pa : pb - na) + o + lane * 16), (lds_ptr)(st + i * 8192),
                                       16, 0, 0);
    }
    pa += na;
    pb += kChunk - na;
    if (--n_left == 0) {
      if (++part == 3) {
        part = 0;
        ++it;
      }
      if (it < c.n_act) enter();
    }
  };
  enter();
  for (int i = 0; i < CrtRing::stages - 1; ++i) issue();

  const d4 z = d4{0.0, 0.0, 0.0, 0.0};
  d4 hR[2], hI[2], sR[2], sI[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) hR[i] = hI[i] = sR[i] = sI[i] = z;
  // Row of element q of block i: 2 (4 lk + q) + i of the wave's 32, for the residue operands (whose rows lie in
  // this order, even ones first) and, rows dealt to the lanes in this order, for the FP64 ones.
  const int arow = wr * 32 + 2 * ((lr >> 2) + 4 * (lr & 3)), bcol = wc * 16 + lr;
  for (int t = 0; t < c.n_act; ++t) {
    d4 pR[2], pI[2];
    {
      d4 p1[2], p2[2], p3[2];
      clear(p1);
      clear(p2);
      clear(p3);
      struct Phases { d2 a[2], b; };
      section<kRowsE / 4, 2>(
          ring, (c.nat[t] + 3) / 4, active, issue,
          [&](const char* st, int s) {
            const d2* A = (const d2*)(st + (4 * s + lk) * 1024) + arow;
            return Phases{{A[0], A[1]}, ((const d2*)(st + (kRowsE + 4 * s + lk) * 1024))[bcol]};
          },
          [&](const Phases& x, int i) {
            p1[i] = MFMA(x.a[i].x, x.b.x, p1[i]);
            if constexpr (REAL) {
              p1[i] = MFMA(x.a[i].y, x.b.y, p1[i]);
            } else {
              p2[i] = MFMA(x.a[i].y, x.b.y, p2[i]);
              p3[i] = MFMA(x.a[i].x - x.a[i].y, x.b.x + x.b.y, p3[i]);
            }
          });
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        pR[i] = REAL ? p1[i] : p1[i] + p2[i];
        pI[i] = p3[i] - p1[i] + p2[i];
      }
    }
    {
      d4 F[2];
      clear(F);
      struct Rows { d2 a; double b; };
      section<kRowsF / 4, 2>(
          ring, (M + 3) / 4, active, issue,
          [&](const char* st, int s) {
            return Rows{*(const d2*)((const double*)(st + (4 * s + lk) * 512) + arow),
                        ((const double*)(st + kChunk / 2 + (4 * s + lk) * 512))[bcol]};
          },
          [&](const Rows& x, int i) { F[i] = MFMA(x.a[i], x.b, F[i]); });
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        sR[i] += pR[i] * F[i];
        if constexpr (!REAL) sI[i] += pI[i] * F[i];
      }
    }
    d4 hs[NC][2], ls[NC][2];
    typename Mma::T acc[NC][2];
#pragma unroll
    for (int p = 0; p < NC; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        hs[p][i] = ls[p][i] = z;
        acc[p][i] = typename Mma::T{0, 0, 0, 0};
      }
    int mod = 0, k = 0;
    double h = cr.h[0], l = cr.l[0];  // of the modulus being summed
    struct Residues { u4 a[2], b[NC]; };
    section<SPC, 2>(
        ring, steps, active, issue,
        [&](const char* st, int s) {
          const u4* A = (const u4*)(st + (s * 4 + lk) * 1024) + wr * 32 + lr;
          const u4* B = (const u4*)(st + St::a_res + (s * 4 + lk) * NC * 1024) + bcol;
          Residues x;
#pragma unroll
          for (int i = 0; i < 2; ++i) x.a[i] = A[16 * i];
#pragma unroll
          for (int p = 0; p < NC; ++p) x.b[p] = B[64 * p];
          return x;
        },
        [&](const Residues& x, int i) {
#pragma unroll
          for (int p = 0; p < NC; ++p) acc[p][i] = Mma::mma(x.a[i], x.b[p], acc[p][i]);
          if (i == 1 && ++k == cr.ks) {  // uniform
            k = 0;
#pragma unroll
            for (int p = 0; p < NC; ++p)
#pragma unroll
              for (int e = 0; e < 2; ++e) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  const double v = (double)acc[p][e][q];
                  hs[p][e][q] = fma(v, h, hs[p][e][q]);
                  ls[p][e][q] = fma(v, l, ls[p][e][q]);
                }
                acc[p][e] = typename Mma::T{0, 0, 0, 0};
              }
            if (++mod < cr.n_mod) {
              h = cr.h[mod];
              l = cr.l[mod];
            }
          }
        });
    const double ic = inv_col[t * 64 + bcol];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double sc = ic * inv_row[t * 64 + wr * 32 + 2 * (4 * lk + q) + i];
        double x[NC];
#pragma unroll
        for (int p = 0; p < NC; ++p) {
          const double f = (hs[p][i][q] - rint(hs[p][i][q])) + ls[p][i][q];
          x[p] = (f - rint(f)) * sc;
        }
        if constexpr (REAL) {
          hR[i][q] += pR[i][q] * x[0];
        } else {
          hR[i][q] += pR[i][q] * x[0] - pI[i][q] * x[1];
          hI[i][q] += pR[i][q] * x[1] + pI[i][q] * x[0];
        }
      }
  }
  const int col = c0 + lr;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = r0 + 2 * (4 * lk + q) + i;
      if (r < n && col < n && col >= r) {
        const int64_t o = (int64_t)r * n + col;
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

}  // namespace

FactCrt fact_crt(const CrtConsts& cc, const FactCell& c, int ek, bool real) {
  FactCrt r{};
  const int rows = 4 * crt_unit_rows(ek), M = 2 * c.n_l;
  const int spc = real ? Stream<true>::SPC : Stream<false>::SPC;
  r.n_mod = cc.n_mod;
  r.ks = (M + rows - 1) / rows;
  r.n_f = (M + kRowsF - 1) / kRowsF;
  r.n_r = (r.n_mod * r.ks + spc - 1) / spc;
  r.a_bytes = (int64_t)c.n_act * r.n_r * (real ? Stream<true>::a_res : Stream<false>::a_res);
  r.b_bytes = (int64_t)c.n_act * r.n_r * kChunk - r.a_bytes;
  r.M = cc.M;
  r.bound = cc.bound;
  for (int i = 0; i < cc.n_mod; ++i) {
    const int m = cc.m[i];
    const int y = cc.y[i] > m / 2 ? cc.y[i] - m : cc.y[i];
    r.m[i] = m;
    r.inv_m[i] = 1.0 / m;
    r.h[i] = std::ldexp(std::rint(std::ldexp((double)y / m, 27)), -27);
    r.l[i] = ((double)y - r.h[i] * m) / m;  // the difference is exact: h has 27 fractional bits, m 8
  }
  return r;
}

hipError_t launch_fact_residues(const FactCell& c, const FactK& kk, const FactCrt& cr, int ek, bool real, char* ws,
                            hipStream_t s) {
  const dim3 grid(kk.n_pad / 64, c.n_act, 2), block(64 * kResWaves);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, c, kk, cr, ws); };
  if (ek == 0) real ? go(k_fact_residues<0, true>) : go(k_fact_residues<0, false>);
  else if (ek == 1) real ? go(k_fact_residues<1, true>) : go(k_fact_residues<1, false>);
  else real ? go(k_fact_residues<2, true>) : go(k_fact_residues<2, false>);
  return hipGetLastError();
}

hipError_t launch_fact_crt(const FactCell& c, const FactK& kk, const FactCrt& cr, int ek, bool real, int gr,
                           const char* ws, void* H, void* S, hipStream_t s) {
  const int num_wg = fact_tiles(kk.n);
  const dim3 grid(num_wg), block(512);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, c, kk, cr, num_wg, gr, ws, H, S); };
  if (ek == 0) real ? go(k_fact_crt<0, true>) : go(k_fact_crt<0, false>);
  else if (ek == 1) real ? go(k_fact_crt<1, true>) : go(k_fact_crt<1, false>);
  else real ? go(k_fact_crt<2, true>) : go(k_fact_crt<2, false>);
  return hipGetLastError();
}

}  // namespace hsb
