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
// Measured at N_G = 12000, 128 atoms, l_max = 10, 11 moduli: k_fact_crt 7.95 ms, of which the FP64
// and integer matrix cores are busy 3.2 and the FP64 vector units 0.7 (they share the FP64 ones' pipe);
// without its copies 5.9, its copies alone 4.9 (66 GB from L2).  k_fact_pack 0.26 ms.  The stacked residue
// contraction over the 30976 rows of all atoms took 110 ms, with H off by 2e-11 of its norm against 2e-12 here.
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

// Operand streams.  A tile reads the stream A of its 64 rows and the stream B of its 64 columns, one after the other
// in chunks of 24 KB (both streams' parts), per type:
//   phases   chunks of 12 rows (1 KB a row and stream): E; B's weighted with the atoms' multiplicities (real form)
//   R rows   chunks of 24 rows (512 bytes each): A R, B lam R
//   residues chunks of SPC steps, [modulus][step]: A R's 4 units of 64 columns, B Y's [4][NC][64 columns] (NC: real
//            and imaginary part)
// Rows and steps past the ends are zero.  A's residues hold the columns of each 32 even ones first (k_fact_crt).
// (The same pieces from arrays of whole rows, 1 KB out of every 192 at N_G = 12000: 15.2 ms against 12.4.)
constexpr int kRowsE = 12, kRowsF = 24, kChunk = 24 * 1024;
typedef Ring<6, kChunk> CrtRing;
template <bool REAL>
struct Stream {
  static constexpr int NC = REAL ? 1 : 2;        // products per modulus
  static constexpr int SPC = 24 / (4 + 4 * NC);  // steps per chunk
  static constexpr int a_res = SPC * 4 * 1024;   // A's bytes of a residue chunk (of the others: half)
};

// Stream A (blockIdx.z = 0) or B (1) of type blockIdx.y and the 64 columns blockIdx.x, and the reciprocal scales.
// The scale is the largest power of two 2^f with 2^f ||x|| + sqrt(2 M) / 2 <= bound (the second term bounds the
// norm of the rounding errors), 1 for a zero column.  Bandwidth-bound on what it writes (n_mod bytes or
// 16-bit values per value of 8 bytes read, twice, the second time from cache).
constexpr int kPackWaves = 16;
template <int EK, bool REAL>
__global__ void __launch_bounds__(64 * kPackWaves) k_fact_pack(FactCell c, FactK kk, FactCrt cr,
                                                               char* __restrict__ ws) {
  constexpr int RU = EK == 0 ? 16 : 8, EB = 16 / RU, PER = 4 / EB;
  typedef Stream<REAL> St;
  __shared__ double part[kPackWaves][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = blockIdx.y, G = blockIdx.x * 64 + lane;
  const bool is_b = blockIdx.z;
  const int parts = is_b ? St::NC : 1;  // values per row
  const int64_t np = kk.n_pad;
  const int M = 2 * c.n_l, nat = c.nat[t];
  const int n_e = (nat + kRowsE - 1) / kRowsE;
  char* out = ws + (is_b ? cr.B + blockIdx.x * cr.b_len + cr.boff[t] : cr.A + blockIdx.x * cr.a_len + cr.aoff[t]);
  {
    const d2* e = (const d2*)(ws + (is_b ? kk.EW : kk.E)) + ((int64_t)blockIdx.x * c.e_rows + c.eoff[t]) * 64 + lane;
    d2* o = (d2*)out + lane;
    for (int k = wave; k < n_e * kRowsE; k += kPackWaves) o[k * 64] = k < nat ? e[k * 64] : d2{0.0, 0.0};
    out += n_e * (kChunk / 2);
  }
  const int64_t r0 = ((int64_t)blockIdx.x * c.n_act + t) * c.Mr;
  const double* R = (const double*)(ws + kk.R) + r0 * 64 + lane;
  {
    const double* r = is_b ? (const double*)(ws + kk.LR) + r0 * 64 + lane : R;
    double* o = (double*)out + lane;
    for (int k = wave; k < cr.n_f * kRowsF; k += kPackWaves) o[k * 64] = k < M ? r[k * 64] : 0.0;
    out += cr.n_f * (kChunk / 2);
  }
  const double* x = is_b ? (const double*)(ws + kk.Y) + (r0 * 64 + lane) * parts : R;
  const int ld = 64 * parts;
  double sq = 0.0;
  for (int k = wave; k < M; k += kPackWaves)
    for (int p = 0; p < parts; ++p) {
      const double v = x[k * ld + p];
      sq += v * v;
    }
  part[wave][lane] = sq;
  __syncthreads();
  sq = 0.0;
  for (int i = 0; i < kPackWaves; ++i) sq += part[i][lane];
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
  for (int u = wave; u < units * parts; u += kPackWaves) {
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
       u += kPackWaves) o[u * 64] = u4{0u, 0u, 0u, 0u};
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
  // next chunk to issue: its parts of the streams, chunks until the type's residues and the next type
  const char* pa = ws + cr.A + bi * cr.a_len;
  const char* pb = ws + cr.B + bj * cr.b_len;
  int it = 0, to_res = (c.nat[0] + kRowsE - 1) / kRowsE + cr.n_f, to_type = cr.n_r;
  auto issue = [&]() {
    if (it >= c.n_act) return;
    char* st = ring.stage(wave);
    const int na = to_res > 0 ? kChunk / 2 : St::a_res;
#pragma unroll
    for (int i = 0; i < CrtRing::copies; ++i) {
      const int o = (wave + 8 * i) * 1024;
      __builtin_amdgcn_global_load_lds((const void*)((o < na ? pa : pb - na) + o + lane * 16), (lds_ptr)(st + i * 8192), 16, 0, 0);
    }
    pa += na;
    pb += kChunk - na;
    if (to_res > 0) {
      --to_res;
    } else if (--to_type == 0) {
      to_type = cr.n_r;
      if (++it < c.n_act) to_res = (c.nat[it] + kRowsE - 1) / kRowsE + cr.n_f;
    }
  };
  auto arrive = [&]() -> const char* {
    const char* st = ring.arrive();
    issue();
    return st;
  };
  for (int i = 0; i < CrtRing::stages - 1; ++i) issue();

  const d4 z = d4{0.0, 0.0, 0.0, 0.0};
  d4 hR[2], hI[2], sR[2], sI[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) hR[i] = hI[i] = sR[i] = sI[i] = z;
  // Row of element q of block i: 2 (4 lk + q) + i of the wave's 32, for the residue operands (whose rows lie in
  // this order, even ones first) and, rows dealt to the lanes in this order, for the FP64 ones.
  const int arow = wr * 32 + 2 * ((lr >> 2) + 4 * (lr & 3)), bcol = wc * 16 + lr;
  for (int t = 0; t < c.n_act; ++t) {
    const int nt = c.nat[t];
    d4 pR[2], pI[2];
    {
      d4 p1[2], p2[2], p3[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) p1[i] = p2[i] = p3[i] = z;
      for (int k0 = 0; k0 < nt; k0 += kRowsE) {
        const char* st = arrive();
#pragma unroll
        for (int s = 0; s < kRowsE / 4; ++s) {
          if (active && k0 + 4 * s < nt) {  // uniform
            const d2* A = (const d2*)(st + (4 * s + lk) * 1024) + arow;
            const d2 b = ((const d2*)(st + (kRowsE + 4 * s + lk) * 1024))[bcol];
            const double bs = b.x + b.y;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const d2 a = A[i];
              p1[i] = MFMA(a.x, b.x, p1[i]);
              if constexpr (REAL) {
                p1[i] = MFMA(a.y, b.y, p1[i]);
              } else {
                p2[i] = MFMA(a.y, b.y, p2[i]);
                p3[i] = MFMA(a.x - a.y, bs, p3[i]);
              }
            }
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        pR[i] = REAL ? p1[i] : p1[i] + p2[i];
        pI[i] = p3[i] - p1[i] + p2[i];
      }
    }
    {
      d4 F[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) F[i] = z;
      for (int k0 = 0; k0 < M; k0 += kRowsF) {
        const char* st = arrive();
        if (!active) continue;
        d2 a[kRowsF / 4];
        double b[kRowsF / 4];
#pragma unroll
        for (int s = 0; s < kRowsF / 4; ++s) {
          a[s] = *(const d2*)((const double*)(st + (4 * s + lk) * 512) + arow);
          b[s] = ((const double*)(st + 12 * 1024 + (4 * s + lk) * 512))[bcol];
        }
#pragma unroll
        for (int s = 0; s < kRowsF / 4; ++s) {
          if (k0 + 4 * s < M) {  // uniform
#pragma unroll
            for (int i = 0; i < 2; ++i) F[i] = MFMA(a[s][i], b[s], F[i]);
          }
        }
      }
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
    for (int s0 = 0; s0 < steps; s0 += SPC) {
      const char* st = arrive();
      if (!active) continue;
      u4 a[SPC][2], b[SPC][NC];
#pragma unroll
      for (int s = 0; s < SPC; ++s) {
        const u4* A = (const u4*)(st + (s * 4 + lk) * 1024) + wr * 32 + lr;
        const u4* B = (const u4*)(st + St::a_res + (s * 4 + lk) * NC * 1024) + bcol;
#pragma unroll
        for (int i = 0; i < 2; ++i) a[s][i] = A[16 * i];
#pragma unroll
        for (int p = 0; p < NC; ++p) b[s][p] = B[64 * p];
      }
#pragma unroll
      for (int s = 0; s < SPC; ++s) {
        if (s0 + s < steps) {  // uniform
#pragma unroll
          for (int p = 0; p < NC; ++p)
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[p][i] = Mma::mma(a[s][i], b[s][p], acc[p][i]);
          if (++k == cr.ks) {
            k = 0;
            const double h = cr.h[mod], l = cr.l[mod];
            ++mod;
#pragma unroll
            for (int p = 0; p < NC; ++p)
#pragma unroll
              for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  const double v = (double)acc[p][i][q];
                  hs[p][i][q] = fma(v, h, hs[p][i][q]);
                  ls[p][i][q] = fma(v, l, ls[p][i][q]);
                }
                acc[p][i] = typename Mma::T{0, 0, 0, 0};
              }
          }
        }
      }
    }
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
  for (int t = 0; t < c.n_act; ++t) {
    r.aoff[t] = r.a_len;
    r.boff[t] = r.b_len;
    const int64_t half = (int64_t)((c.nat[t] + kRowsE - 1) / kRowsE + r.n_f) * (kChunk / 2);
    const int64_t a = real ? Stream<true>::a_res : Stream<false>::a_res;
    r.a_len += half + r.n_r * a;
    r.b_len += half + r.n_r * (kChunk - a);
  }
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

hipError_t launch_fact_pack(const FactCell& c, const FactK& kk, const FactCrt& cr, int ek, bool real, char* ws,
                            hipStream_t s) {
  const dim3 grid(kk.n_pad / 64, c.n_act, 2), block(64 * kPackWaves);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, c, kk, cr, ws); };
  if (ek == 0) real ? go(k_fact_pack<0, true>) : go(k_fact_pack<0, false>);
  else if (ek == 1) real ? go(k_fact_pack<1, true>) : go(k_fact_pack<1, false>);
  else real ? go(k_fact_pack<2, true>) : go(k_fact_pack<2, false>);
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
