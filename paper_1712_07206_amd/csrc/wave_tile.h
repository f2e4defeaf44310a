// Tiles of the type-factored kernels on v_mfma_f64_16x16x4f64 (A: lane l holds row l % 16 of step row l / 16; B
// likewise its column; output: lane l, element q -> row l / 16 + 4 q, column l % 16).
#pragma once

#include "hs_internal.h"

namespace hsb {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr;

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64((a), (b), (c), 0, 0, 0)

// A lane's values of N neighbouring columns, as one load.
template <int N>
struct DVec;
template <>
struct DVec<1> { typedef double T; static __device__ double get(T v, int) { return v; } };
template <>
struct DVec<2> { typedef d2 T; static __device__ double get(T v, int i) { return v[i]; } };

template <int MI, int NJ>
__device__ __forceinline__ void clear(d4 (&x)[MI][NJ]) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) x[i][j] = d4{0.0, 0.0, 0.0, 0.0};
}
template <int MI>
__device__ __forceinline__ void clear(d4 (&x)[MI]) {
#pragma unroll
  for (int i = 0; i < MI; ++i) x[i] = d4{0.0, 0.0, 0.0, 0.0};
}

// s_waitcnt immediate (gfx9 encoding): at most n vector-memory operations pending, LDS operations done.
constexpr int vm_pending(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

__device__ __forceinline__ const char* uniform(const char* p) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)p);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((uintptr_t)p >> 32));
  return (const char*)(((uintptr_t)hi << 32) | lo);
}

// LDS ring of a workgroup: chunks of BYTES, copied straight there (global_load_lds_dwordx4) as copies of 1 KB, copy
// WAVES i + w of a chunk by wave w; STAGES - 1 chunks ahead, one barrier per chunk.
// The ring has to be the kernel's only __shared__ array: with several the compiler waits for every pending
// copy before each read of one.
template <int STAGES, int BYTES, int WAVES = 8>
struct Ring {
  static constexpr int stages = STAGES, chunk = BYTES, copies = BYTES / 1024 / WAVES, bytes = STAGES * BYTES;
  char* lds;
  int left;  // chunks not yet waited for
  int istage = 0, cstage = 0;
  // This wave's part of the next stage.
  __device__ __forceinline__ char* stage(int wave) {
    char* st = lds + istage * BYTES + wave * 1024;
    istage = istage == STAGES - 1 ? 0 : istage + 1;
    return st;
  }
  // Waits for the next chunk, everyone's copies of it; the stage of the chunk before is free after it.
  __device__ __forceinline__ const char* arrive() {
    --left;
    if (left >= STAGES - 2) __builtin_amdgcn_s_waitcnt(vm_pending((STAGES - 2) * copies));
    else if (STAGES > 4 && left == 3) __builtin_amdgcn_s_waitcnt(vm_pending(3 * copies));
    else if (STAGES > 3 && left == 2) __builtin_amdgcn_s_waitcnt(vm_pending(2 * copies));
    else if (left == 1) __builtin_amdgcn_s_waitcnt(vm_pending(copies));
    else __builtin_amdgcn_s_waitcnt(vm_pending(0));
    // a plain s_barrier: __syncthreads would wait for the copies in flight as well
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const char* st = lds + cstage * BYTES;
    cstage = cstage == STAGES - 1 ? 0 : cstage + 1;
    return st;
  }
};

// A section (say, a type's rows) of `steps` steps of the matrix cores, PER of them a chunk: read(stage, s) gives a step's
// operands, mac(x, i) takes the products of block i of MI.  The next step's operands are read ahead, over
// the barrier too, behind the first block's products (the wait for a step's own operands is then not one for
// theirs too), and the copies of another chunk (issue) go out behind the first step's: right behind the
// barrier, where all waves are, they and their addresses leave the matrix cores idle.
template <int PER, int MI, class Ring, class Issue, class Read, class Mac>
__device__ __forceinline__ void section(Ring& ring, int steps, bool active, Issue issue, Read read, Mac mac) {
  const int chunks = (steps + PER - 1) / PER;
  if (!active) {  // uniform
    for (int i = 0; i < chunks; ++i) {
      ring.arrive();
      issue();
    }
    return;
  }
  auto step = [&](const auto& x, const char* st, int next) {
    if constexpr (MI == 2) {
      mac(x, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    auto y = read(st, next);
    __builtin_amdgcn_sched_barrier(0);
    mac(x, MI - 1);
    __builtin_amdgcn_sched_barrier(0);
    return y;
  };
  const char* st = ring.arrive();
  auto x = read(st, 0);
  for (int i = 1; i < chunks; ++i) {
#pragma unroll
    for (int s = 0; s < PER; ++s) {
      if (PER == 1) issue();  // arrive() counts on one issue before it
      if (s == PER - 1) st = ring.arrive();
      x = step(x, st, s == PER - 1 ? 0 : s + 1);
      if (PER > 1 && s == 0) issue();
    }
  }
  const int rest = steps - (chunks - 1) * PER;
  mac(x, 0);
  if constexpr (MI == 2) mac(x, 1);
  __builtin_amdgcn_sched_barrier(0);
  issue();
#pragma unroll
  for (int s = 1; s < PER; ++s)
    if (s < rest) {
      x = read(st, s);
      mac(x, 0);
      if constexpr (MI == 2) mac(x, 1);
    }
}

// One tile of 32 MI (G') x 32 (G) of the type-factored products on 2 x 2 waves of 16 MI x 16: one half of the columns
// and (MI = 1) one half of the rows of a 64 x 64 block of the arrays.  A lane holds MI neighbouring rows, one for
// each of its blocks: block i covers the rows of index i modulo MI.  Two workgroups to a compute unit, one wave
// of each per SIMD, so that one's waits at its barriers are the other's time.
//
// Chunks of 20 KB are 12 phase rows (E at G', EW at G), then 16 of the type's R rows (R at G'; lam R and Y at G; the
// real form 20) out of the block-major arrays; rows past a type's are copied but not used.
template <int MI, bool REAL>
struct TypedTile {
  static constexpr int RE = 12, RM = REAL ? 20 : 16;
  typedef Ring<4, 20 * 1024, 4> R;
  static constexpr int lds_bytes = R::bytes;
  // offsets in a stage: EW; lam R and Y, and the latter's row
  static constexpr int at_b = RE * 1024, at_l = RM * 512, at_y = RM * 768, y_row = REAL ? 256 : 512;
  typedef typename DVec<MI>::T VA;
  const FactCell& c;
  const FactK& kk;
  const char* ws;
  R ring;
  int bi, bj, part_i, part_j, t_end;
  int wave, lr, lk, arow, bcol;
  // The next chunk to issue: its type, chunks left of the type's phases or rows; this wave's next sources: of E and EW;
  // of R, lam R and Y (the real form's wave takes R or lam R in p1, lam R or Y in p2), and what takes them from the
  // last chunk of a type to the next type's first.
  int it, n_left;
  bool irows = false;
  const char *pa, *pb;
  const char *p0, *p1, *p2, *p3;
  unsigned off, off2, off4;  // a lane's offset in a copy: of whole rows of 1 KB, of halves of those, of halves of 512 bytes
  int adj, adj3;

  __device__ __forceinline__ TypedTile(const FactCell& cell, const FactK& k, const char* base, char* lds, int block_i,
                                       int half_i, int block_j, int half_j, int t0, int t1)
      : c(cell), kk(k), ws(base), bi(block_i), bj(block_j), part_i(half_i), part_j(half_j), t_end(t1), it(t0) {
    const int lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lr = lane & 15;
    lk = lane >> 4;
    arow = part_i * 32 + (wave >> 1) * 16 * MI + MI * lr;
    bcol = (wave & 1) * 16 + lr;
    off = lane * 16;
    off2 = (lane >> 5) * 1024 + (lane & 31) * 16;
    off4 = (lane >> 4) * 512 + (lane & 15) * 16;
    ring.lds = lds;
    ring.left = 0;
    for (int t = t0; t < t1; ++t) ring.left += (c.nat[t] + RE - 1) / RE + (2 * c.n_l + RM - 1) / RM;
    n_left = (c.nat[it] + RE - 1) / RE;
    const int n_f = (2 * c.n_l + RM - 1) / RM;
    const int64_t ra = ((int64_t)bi * c.n_act + it) * c.Mr, rb = ((int64_t)bj * c.n_act + it) * c.Mr;
    const char* r = ws + kk.R + ra * 512;
    const char* l = ws + kk.LR + rb * 512 + part_j * 256;
    const char* y = ws + kk.Y + rb * (REAL ? 512 : 1024) + part_j * y_row;
    p0 = uniform(r + wave * 1024);
    if constexpr (REAL) {  // copies 0-9 of R (2 rows each), 10-14 of lam R, 15-19 of Y (4 rows each)
      p1 = uniform(wave < 2 ? r + (8 + wave) * 1024 : l + (wave - 2) * 2048);
      p2 = uniform(wave < 3 ? l + (2 + wave) * 2048 : y);
      p3 = uniform(y + (1 + wave) * 2048);
    } else {  // copies 0-7 of R, 8-11 of lam R (4 rows), 12-19 of Y (2 rows)
      p2 = p1 = uniform(l + wave * 2048);
      p3 = uniform(y + wave * 2048);
    }
    adj = (c.Mr - n_f * RM) * 512;
    adj3 = adj * (REAL ? 1 : 2);
    phase_source();
    for (int i = 0; i < R::stages - 1; ++i) issue();
  }
  // First row and column of this wave's part (uniform).
  __device__ __forceinline__ int row0() const { return bi * 64 + part_i * 32 + (wave >> 1) * 16 * MI; }
  __device__ __forceinline__ int col0() const { return bj * 64 + part_j * 32 + (wave & 1) * 16; }
  // Row of element q of block i, and the column, of this lane's sums.
  __device__ __forceinline__ int row(int i, int q) const { return row0() + MI * (lk + 4 * q) + i; }
  __device__ __forceinline__ int col() const { return col0() + lr; }

  __device__ __forceinline__ void phase_source() {
    pa = uniform(ws + kk.E + ((int64_t)bi * c.e_rows + c.eoff[it]) * 1024 + wave * 1024);
    pb = uniform(ws + kk.EW + ((int64_t)bj * c.e_rows + c.eoff[it]) * 1024 + part_j * 512 + wave * 2048);
  }
  __device__ __forceinline__ void issue() {
    if (it >= t_end) return;
    char* st = ring.stage(wave);
    auto copy = [&](const char* p, unsigned o, int i) {
      __builtin_amdgcn_global_load_lds((const void*)(p + o), (lds_ptr)(st + i * 4096), 16, 0, 0);
    };
    if (!irows) {
#pragma unroll
      for (int i = 0; i < 3; ++i) copy(pa + i * 4096, off, i);
      copy(pb, off2, 3);
      copy(pb + 8192, off2, 4);  // waves 2 and 3: two rows past the chunk's, to memory not read
      pa += RE * 1024;
      pb += RE * 1024;
      if (--n_left == 0) {
        irows = true;
        n_left = (2 * c.n_l + RM - 1) / RM;
      }
    } else {
      copy(p0, off, 0);
      copy(p0 + 4096, off, 1);
      if constexpr (REAL) {
        copy(p1, wave < 2 ? off : off4, 2);
        copy(p2, off4, 3);
        copy(p3, off4, 4);
        p1 += RM * 512;
        p3 += RM * 512;
      } else {
        copy(p2, off4, 2);
        copy(p3, off2, 3);
        copy(p3 + 8192, off2, 4);
        p3 += RM * 1024;
      }
      p0 += RM * 512;
      p2 += RM * 512;
      if (--n_left == 0) {
        irows = false;
        if (++it < t_end) {
          p0 += adj;
          p1 += adj;
          p2 += adj;
          p3 += adj3;
          n_left = (c.nat[it] + RE - 1) / RE;
          phase_source();
        }
      }
    }
  }
  struct Phases { d2 a[MI], b; };
  __device__ __forceinline__ Phases read_phases(const char* st, int s) const {
    Phases x;
    const d2* A = (const d2*)(st + (4 * s + lk) * 1024) + arow;
#pragma unroll
    for (int i = 0; i < MI; ++i) x.a[i] = A[i];
    x.b = ((const d2*)(st + at_b + (4 * s + lk) * 512))[bcol];
    return x;
  }
  // P_t = E_t^H E_t: three real products per complex one (P1 = a_r b_r, P2 = a_i b_i,
  // P3 = (a_r - a_i)(b_r + b_i), Re = P1 + P2, Im = P3 - P1 + P2); the real form, its columns' phases weighted with the
  // atoms' multiplicities, takes two, into one sum (pI is not set).
  __device__ __forceinline__ void phase_sums(int t, bool active, d4 (&pR)[MI], d4 (&pI)[MI]) {
    d4 p1[MI], p2[MI], p3[MI];
    clear(p1);
    clear(p2);
    clear(p3);
    section<RE / 4, MI>(
        ring, (c.nat[t] + 3) / 4, active, [&] { issue(); }, [&](const char* st, int s) { return read_phases(st, s); },
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
    for (int i = 0; i < MI; ++i) {
      pR[i] = REAL ? p1[i] : p1[i] + p2[i];
      if constexpr (!REAL) pI[i] = p3[i] - p1[i] + p2[i];
    }
  }
  struct Rows { VA a; d2 y; double yr, l; };
  __device__ __forceinline__ Rows read_rows(const char* st, int s) const {
    Rows x;
    x.a = *(const VA*)((const double*)(st + (4 * s + lk) * 512) + arow);
    x.l = ((const double*)(st + at_l + (4 * s + lk) * 256))[bcol];
    if constexpr (REAL) x.yr = ((const double*)(st + at_y + (4 * s + lk) * y_row))[bcol];
    else x.y = ((const d2*)(st + at_y + (4 * s + lk) * y_row))[bcol];
    return x;
  }
  // m1 + i m2 = R_t^T Y_t (the real form: m1 only), F = R_t^T Lam_t R_t.
  __device__ __forceinline__ void row_sums(bool active, d4 (&m1)[MI], d4 (&m2)[MI], d4 (&F)[MI]) {
    clear(m1);
    if constexpr (!REAL) clear(m2);
    clear(F);
    section<RM / 4, MI>(
        ring, (2 * c.n_l + 3) / 4, active, [&] { issue(); }, [&](const char* st, int s) { return read_rows(st, s); },
        [&](const Rows& x, int i) {
          const double a = DVec<MI>::get(x.a, i);
          if constexpr (REAL) {
            m1[i] = MFMA(a, x.yr, m1[i]);
          } else {
            m1[i] = MFMA(a, x.y.x, m1[i]);
            m2[i] = MFMA(a, x.y.y, m2[i]);
          }
          F[i] = MFMA(a, x.l, F[i]);
        });
  }
};

}  // namespace hsb
