// Wave tiles of the type-factored kernels: 16 MI rows x 16 NJ columns per wave on
// v_mfma_f64_16x16x4f64, operands read straight from global memory into registers one chunk (KC
// steps of 4 rows) ahead.  A lane holds MI (NJ) neighbouring rows (columns), one for each block:
// block i covers the rows of index i modulo MI, so one load serves all blocks.
// Output of the 16x16 f64 MFMA: lane l, element q -> row l/16 + 4q, column l%16 of the block.
#pragma once

#include "hs_internal.h"

namespace hsb {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64((a), (b), (c), 0, 0, 0)

// A lane's values of N neighbouring columns, as one load.
template <int N>
struct DVec;
template <>
struct DVec<1> { typedef double T; static __device__ double get(T v, int) { return v; } };
template <>
struct DVec<2> { typedef d2 T; static __device__ double get(T v, int i) { return v[i]; } };

// The sums of one (G', G) wave tile for a type t with phases E, rows R and Y:
//   P = E^H E:  three real products per complex one (P1 = a_r b_r, P2 = a_i b_i,
//     P3 = (a_r - a_i)(b_r + b_i), Re = P1 + P2, Im = P3 - P1 + P2); the real form takes two, into
//     one sum, the columns' phases weighted with the atom's multiplicity;
//   m1 + i m2 = R^T Y (the real form: m1 only),  m3 = R^T lam R.
// P is summed in the registers of the m's, which come after it.
template <int MI, int NJ, int KC, bool REAL>
struct TypedTile {
  static_assert(kFactRows % (4 * KC) == 0, "rows are padded to whole chunks");
  typedef typename DVec<MI>::T VA;
  typedef typename DVec<NJ>::T VB;
  struct EChunk { d2 a[KC][MI], b[KC][NJ]; double w[KC]; };
  struct MChunk { VA a[KC]; VB b[KC]; VB yr[KC]; d2 y[KC][NJ]; double lam[KC]; };

  const FactCell& c;
  const FactK& kk;
  const FactRep* rep;
  const char* ws;
  int64_t n_pad;
  int lk, row, col;
  EChunk ec;
  MChunk mc;

  __device__ __forceinline__ TypedTile(const FactCell& cell, const FactK& k, int row0, int col0, const FactRep* reps,
                                       const char* base)
      : c(cell), kk(k), rep(reps), ws(base), n_pad(k.n_pad) {
    const int lane = threadIdx.x & 63;
    lk = lane >> 4;
    row = row0 + MI * (lane & 15);
    col = col0 + NJ * (lane & 15);
  }
  __device__ __forceinline__ void load_e(int t, int ch, EChunk& e) const {
    const d2* base = (const d2*)(ws + kk.E) + (int64_t)c.eoff[t] * n_pad;
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      const int k = (ch * KC + q) * 4 + lk;
      const d2* p = base + (int64_t)k * n_pad;
#pragma unroll
      for (int i = 0; i < MI; ++i) e.a[q][i] = p[row + i];
#pragma unroll
      for (int j = 0; j < NJ; ++j) e.b[q][j] = p[col + j];
      if constexpr (REAL) e.w[q] = k < c.nat[t] ? rep[c.atom0[t] + k].weight : 0.0;
    }
  }
  __device__ __forceinline__ void load_m(int t, int ch, MChunk& m) const {
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      const int64_t k = (int64_t)t * c.Mr + (ch * KC + q) * 4 + lk;
      const double* p = (const double*)(ws + kk.R) + k * n_pad;
      m.a[q] = *(const VA*)(p + row);
      m.b[q] = *(const VB*)(p + col);
      m.lam[q] = ((const double*)(ws + c.lam))[k];
      if constexpr (REAL) {
        m.yr[q] = *(const VB*)((const double*)(ws + kk.Y) + k * n_pad + col);
      } else {
        const d2* yp = (const d2*)(ws + kk.Y) + k * n_pad + col;
#pragma unroll
        for (int j = 0; j < NJ; ++j) m.y[q][j] = yp[j];
      }
    }
  }
  // ec holds type t's first phase chunk; with more, type t + 1's is loaded on the way.
  __device__ __forceinline__ void sums(int t, bool more, d4 (&m1)[MI][NJ], d4 (&m2)[MI][NJ], d4 (&m3)[MI][NJ],
                                       d4 (&pR)[MI][NJ], d4 (&pI)[MI][NJ]) {
    const d4 z = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) m1[i][j] = m2[i][j] = m3[i][j] = z;
    load_m(t, 0, mc);  // lands behind the phase sums
    const int kse = (c.nat[t] + 3) / 4, nce = (kse + KC - 1) / KC;
    for (int ch = 0; ch < nce; ++ch) {
      EChunk en;
      load_e(t, ch + 1 < nce ? ch + 1 : ch, en);
#pragma unroll
      for (int q = 0; q < KC; ++q) {
        if (ch * KC + q < kse) {  // uniform
          double ad[MI], bs[NJ];
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            if constexpr (REAL) ec.b[q][j] *= ec.w[q];
            bs[j] = ec.b[q][j].x + ec.b[q][j].y;
          }
#pragma unroll
          for (int i = 0; i < MI; ++i) ad[i] = ec.a[q][i].x - ec.a[q][i].y;
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
              m1[i][j] = MFMA(ec.a[q][i].x, ec.b[q][j].x, m1[i][j]);
              if constexpr (REAL) {
                m1[i][j] = MFMA(ec.a[q][i].y, ec.b[q][j].y, m1[i][j]);
              } else {
                m2[i][j] = MFMA(ec.a[q][i].y, ec.b[q][j].y, m2[i][j]);
                m3[i][j] = MFMA(ad[i], bs[j], m3[i][j]);
              }
            }
        }
      }
      ec = en;
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        pR[i][j] = REAL ? m1[i][j] : m1[i][j] + m2[i][j];
        pI[i][j] = m3[i][j] - m1[i][j] + m2[i][j];
        m1[i][j] = m2[i][j] = m3[i][j] = z;
      }
    if (more) load_e(t + 1, 0, ec);  // lands behind the R sums
    const int ksm = (2 * c.n_l + 3) / 4, ncm = (ksm + KC - 1) / KC;
    for (int ch = 0; ch < ncm; ++ch) {
      MChunk mn;
      load_m(t, ch + 1 < ncm ? ch + 1 : ch, mn);
#pragma unroll
      for (int q = 0; q < KC; ++q) {
        if (ch * KC + q < ksm) {  // uniform
          double ls[NJ];
#pragma unroll
          for (int j = 0; j < NJ; ++j) ls[j] = mc.lam[q] * DVec<NJ>::get(mc.b[q], j);
#pragma unroll
          for (int i = 0; i < MI; ++i) {
            const double ai = DVec<MI>::get(mc.a[q], i);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
              if constexpr (REAL) {
                m1[i][j] = MFMA(ai, DVec<NJ>::get(mc.yr[q], j), m1[i][j]);
              } else {
                m1[i][j] = MFMA(ai, mc.y[q][j].x, m1[i][j]);
                m2[i][j] = MFMA(ai, mc.y[q][j].y, m2[i][j]);
              }
              m3[i][j] = MFMA(ai, ls[j], m3[i][j]);
            }
          }
        }
      }
      mc = mn;
    }
  }
};

}  // namespace hsb
