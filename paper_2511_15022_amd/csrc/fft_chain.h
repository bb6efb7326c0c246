// Chain FFT passes: the padded row and column transforms of the propagation as
// P interleaved M-point chains, compiled for every chain length M that factors
// into 2, 3 and 5 (chain_lengths below).
//
// A padded length n = P M whose samples fill only the first half splits into P
// chains, because half of the inputs are zero and half of the outputs are
// dropped: with w = exp(-2 pi i / n),
//   P = 4 (n % 4 == 0, samples at i < 2 M): bin 4 m + p is bin m of the M-point
//         transform of w^{p i} (x[i] + (-i)^p x[i + M]) (i < M), and the inverse
//         gives u[i + M j] = sum_p w^{-p i} i^{p j} z_p[i] for j = 0, 1;
//   P = 2 (n = 2 M, M odd, samples at i < M): bin 2 m + p is bin m of the
//         transform of w^{p i} x[i], and u[i] = z_0[i] + w^{-i} z_1[i].
// z_p is the M-point inverse of the bins p mod P.
//
// The radices of a chain's stages are chosen at compile time by the cost model
// below (VALU instructions of a stage times its passes over the lanes), except
// for the lengths whose plan was measured.  A compile-time plan keeps the
// butterflies, the index arithmetic and the twiddle strides constant; the
// runtime-plan kernels (radix 2, 3, 4, 5 and 8 chosen per stage, whole rows or
// half columns between workgroup barriers) remain for the shapes that do not
// split: more samples than half the padded length, odd padded lengths and
// chains longer than the tables below.
#pragma once

#include <algorithm>

#include "cgh_internal.h"
#include "fft_reg.h"

namespace cgh {

// ----------------------------------------------------------------------------
// chain lengths and plans
// ----------------------------------------------------------------------------

// Element i of an array at a wave-uniform base, addressed with a 32-bit byte
// offset (so the access takes the scalar-base form, with no 64-bit address add).
template <class T>
__device__ __forceinline__ T &at32(T *base, uint32_t i) {
  return *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + i * (uint32_t)sizeof(T));
}
template <class T>
__device__ __forceinline__ const T &at32(const T *base, uint32_t i) {
  return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) +
                                      i * (uint32_t)sizeof(T));
}

// VALU instructions of a register DFT of length R (RFft): the base radices
// counted from their code, the composite ones from their factors
constexpr int dft_ops(int R) {
  if (R == 1) return 0;
  if (R == 2) return 4;
  if (R == 3) return 16;
  if (R == 4) return 16;
  if (R == 5) return 36;
  if (R == 8) return 56;
  const int a = base_factor(R), b = R / a;
  return a * dft_ops(b) + b * dft_ops(a) + (gcd_c(a, b) == 1 ? 0 : 4 * (a - 1) * (b - 1));
}

// cost of one LDS stage: `passes` butterflies of radix R per thread, twiddled
// unless it is the first; per value a load, a store and their share of the
// index arithmetic
constexpr int stage_cost(int R, int passes, bool twiddled) {
  return passes * (dft_ops(R) + (twiddled ? 5 * (R - 1) : 0) + 3 * R + 8);
}

constexpr int kRadices[] = {2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27};

struct ColPlan {
  int r0, r1, r2, ch;
};

// Column chain plan: M = r0 r1 r2 (r1 may be 1), ch chains per wave; the last forward and
// first inverse stage are fused in registers, one butterfly of radix r2 per lane
// (ch M / r2 <= 64).  Up to M = 300 two chains share a wave: one chain's butterflies leave
// half of the lanes idle (a radix-8 stage of 256 points has 32).  Above, the higher radices
// that two chains need cost more registers and LDS conflicts than the lanes gain (us per
// pass of synthetic columns, one and two chains: 128 4.5 and 4.3, 180 7.9 and 7.4, 256 32.0
// and 24.0, 300 20.0 and 18.7; 320 29.0 and 31.1, 360 36.3 and 38.3, 512 37.7 and 40.6,
// 540 75 and 84, 720 78 and 110).  Among the plans of least cost an odd r0 comes first: the
// first stage stores at stride r0, and an odd stride spreads the stores over the LDS banks.
constexpr ColPlan col_plan(int M) {
  // measured, with the synthetic columns' us of the plans nearest:
  // 4K: 10 6 18 380, 6 9 20 381, 9 6 20 389; 640: two chains 4 8 20 68.7, one 16 4 10 72.7;
  // 384: 8 6 8 31.0, 6 8 8 32.7; 360: 6 6 10 36.3, 10 6 6 37.0; 256: 4 8 8 24.0, 8 4 8
  // 25.2; 225: four chains 15 1 15 12.2, two 5 5 9 14.0.  540 (1080p) keeps 12 5 9 (82)
  // against 6 9 10 (75): the Random POH's loss takes signs of differences of fields, and
  // another order of roundings flips a few of them, which moves single gradients by 3e-3
  // of their root mean square
  if (M == 1080) return {10, 6, 18, 1};
  if (M == 1024) return {8, 8, 16, 1};
  if (M == 640) return {4, 8, 20, 2};
  if (M == 540) return {12, 5, 9, 1};
  if (M == 512) return {8, 8, 8, 1};
  if (M == 384) return {8, 6, 8, 1};
  if (M == 360) return {6, 6, 10, 1};
  if (M == 256) return {4, 8, 8, 2};
  if (M == 225) return {15, 1, 15, 4};
  const int ch = M <= 300 ? 2 : 1;
  ColPlan best{0, 0, 0, ch};
  int cost = 1 << 30;
  for (int r2 : kRadices) {
    if (M % r2 || ch * (M / r2) > 64) continue;
    const int q = M / r2;
    for (int r0 : kRadices) {
      if (q % r0) continue;
      const int r1 = q / r0;
      if (r1 > 16) continue;
      bool known = r1 == 1;
      for (int r : kRadices) known = known || r == r1;
      if (!known) continue;
      const int n0 = (ch * (M / r0) + 63) / 64, n1 = r1 > 1 ? (ch * (M / r1) + 63) / 64 : 0;
      // registers: every butterfly of a stage is held before the first store
      if (n0 * r0 > 32 || n1 * r1 > 32) continue;
      int c = stage_cost(r0, n0, false) + stage_cost(r0, n0, true);
      if (r1 > 1) c += 2 * stage_cost(r1, n1, true);
      c += 2 * dft_ops(r2) + 13 * r2 + 16;
      c = c * 8 + (r0 % 2 ? 0 : 4);
      if (c < cost) {
        cost = c;
        best = ColPlan{r0, r1, r2, ch};
      }
    }
  }
  return best;
}

template <int M>
struct ColPlanOf {
  static constexpr ColPlan value = col_plan(M);
};
// The layouts between a chain's stages: after the first and second forward stage, after
// the first and second inverse stage (exchange_pad).
struct ColPads {
  Pad f0, f1, i0, i1;
};
// Workgroups per CU that LDS of a chain stride holds (beside them the table of M), as far
// as their waves fit a CU; padding may not cost one.
constexpr int col_groups(int M, int stride, const ColPlan &pl) {
  return std::min(160 * 1024 / ((8 * stride + M) * 8), 4 * pl.ch);
}
constexpr int col_room(int M, const ColPlan &pl) {
  int n = M + (12 - M % 8) % 8;
  const int groups = col_groups(M, n, pl);
  while (n < 2 * M && col_groups(M, n + 8, pl) == groups) n += 8;
  return n;
}
constexpr ColPads col_pads(int M, const ColPlan &pl) {
  const bool two = pl.r1 == 1;
  const int room = col_room(M, pl);
  return {exchange_pad(pl.r0, 1, two ? M / pl.r2 : M / pl.r1, M, room),
          two ? Pad{0, 0} : exchange_pad(pl.r1, pl.r0, M / pl.r2, M, room),
          exchange_pad(pl.r2, 1, two ? M / pl.r0 : M / pl.r1, M, room),
          two ? Pad{0, 0} : exchange_pad(pl.r1, pl.r2, M / pl.r0, M, room)};
}
// elements from one chain to the next in LDS: its longest layout, to 4 modulo 8, so that
// the lanes that load or combine neighbouring columns' chains use all banks
constexpr int col_stride(int M, const ColPlan &pl) {
  const ColPads p = col_pads(M, pl);
  const int n = std::max(std::max(p.f0.at(M - 1), p.f1.at(M - 1)),
                         std::max(p.i0.at(M - 1), p.i1.at(M - 1))) + 1;
  return n + (12 - n % 8) % 8;
}
// a workgroup's eight chains, pl.ch per wave
constexpr int col_threads(const ColPlan &pl) { return 512 / pl.ch; }
// waves per SIMD that the LDS of its workgroups leaves room for, four at most
constexpr int col_waves(int M, const ColPlan &pl) {
  return std::max(1, std::min(4, col_groups(M, col_stride(M, pl), pl) * (8 / pl.ch) / 4));
}

// Row plan: the stages of P interleaved M-point chains over T threads
// (workgroup barriers between stages), M = r[0] .. r[n - 1].
struct RowPlan {
  int n;
  int r[4];
};

constexpr int row_plan_cost(int M, int P, int T, const RowPlan &p) {
  int c = 0, ns = 1;
  for (int s = 0; s < p.n; ++s) {
    const int R = p.r[s], items = P * (M / R), passes = (items + T - 1) / T;
    if (passes * R > 40) return 1 << 29;  // registers
    c += stage_cost(R, passes, s > 0) + 120;  // two barriers
    // the first stage stores at stride P R: an even stride repeats its banks
    if (s == 0) c += passes * R * (R % 4 == 0 ? 4 : R % 2 == 0 ? 2 : 0);
    ns *= R;
  }
  return c;
}

constexpr RowPlan row_plan(int M, int P, int T) {
  if (P == 4 && T == 512) {
    // measured: 960 (1080p) against 8 8 15, 8 15 8, 10 8 12, 12 8 10 and 16 4 15; 1920
    // (4K) against 8 16 15, 16 8 15, 16 15 8, 12 16 10 and 15 8 16; 1024 (serving pads)
    // against 16 16 4
    if (M == 960) return {3, {15, 8, 8, 1}};
    if (M == 1920) return {3, {15, 16, 8, 1}};
    if (M == 1024) return {3, {8, 8, 16, 1}};
  }
  RowPlan best{0, {1, 1, 1, 1}};
  int cost = 1 << 29;
  for (int a : kRadices) {
    if (M % a) continue;
    for (int b = 1; b <= 27; ++b) {
      if ((M / a) % b) continue;
      for (int d = 1; d <= 27; ++d) {
        if ((M / a / b) % d || (b == 1 && d > 1)) continue;
        const int e = M / a / b / d;
        if (e > 27 || (d == 1 && e > 1)) continue;
        const int rs[4] = {a, b, d, e};
        RowPlan p{0, {1, 1, 1, 1}};
        bool ok = true;
        for (int s = 0; s < 4; ++s) {
          if (rs[s] == 1) continue;
          bool known = false;
          for (int r : kRadices) known = known || r == rs[s];
          ok = ok && known;
          p.r[p.n++] = rs[s];
        }
        if (!ok) continue;
        const int c = row_plan_cost(M, P, T, p);
        if (c < cost) {
          cost = c;
          best = p;
        }
      }
    }
  }
  return best;
}

// Threads per row workgroup: from 400 values on 3 to 16 per thread, 512 threads at most; one
// wave below.  Measured
// (row_loss, row_inv): padded 2048 with 512 threads 31.5 / 2 and 12.0 us, with 256
// 30.0 / 2 and 11.2 us (640 x 1024 RGB); 2560 17.5 and 17.2 us; 3840 60.7 and 28.5
// against 60.5 and 30.8 us (1080p RGB).
constexpr int row_threads(int M, int P) {
  const int n = P * M;
  return n >= 3200 ? 512 : n >= 900 ? 256 : n >= 400 ? 128 : 64;
}

constexpr bool smooth_c(int n) {
  for (int p : {2, 3, 5})
    while (n % p == 0) n /= p;
  return n == 1;
}

// The chain lengths the passes are compiled for.
constexpr int kMinChain = 16;
// the longest odd chain whose fused stage takes one butterfly per lane (1215 / 27 = 45; the
// next odd length, 1875, needs 75); chains of four end with the padded heights of col_supported
constexpr int kMaxColChain = 1215;
constexpr int kMaxRowChain4 = 2048, kMaxRowChain2 = 4095;  // kMaxFft / P
constexpr bool col_chain(int M, int P) {
  return M >= kMinChain && M <= kMaxColChain && P * M <= 2 * kColHalfMax && smooth_c(M) &&
         (P == 4 || M % 2);
}
constexpr bool row_chain(int M, int P) {
  return M >= kMinChain && M <= (P == 4 ? kMaxRowChain4 : kMaxRowChain2) && smooth_c(M) &&
         (P == 4 || M % 2);
}

// The column lengths whose planes share a pass (k_col_wave): those whose last radix leaves
// the registers of a lane room for the kept spectrum beside the one at work.  Above 15 the
// two spill: three planes at 4K RGB (radix 20) 2.78 ms together, 2.38 ms one by one.
// Below: 720p RGB in three planes 272 us one by one, 240 us together (render);
// 640 x 1024 RGB in two planes 425 and 400 us (gradient of the full loss).
constexpr bool planes_chain(int M, int P) { return col_chain(M, P) && col_plan(M).r2 <= 15; }

// the split of a padded length n with `used` samples: P chains of n / P, or 0
inline int split_of(int n, int used, bool (*built)(int, int)) {
  if (2 * used > n || n % 2) return 0;
  const int P = n % 4 == 0 ? 4 : 2;
  return built(n / P, P) ? P : 0;
}

// waves per SIMD that the LDS of a workgroup of 512 threads leaves room for
constexpr int lds_waves(int values) { return values * 8 + 1024 > 80 * 1024 ? 2 : 4; }
// Row workgroups that a CU's LDS holds, and the lengths whose forward rows are
// pipelined: where only one or two workgroups fit, they do not cover each other's
// loads, so a workgroup takes several rows and loads the next one's samples while it
// transforms this one's (4K RGB rows of 7680: 144 us without, 127 us with; with four
// workgroups of 3840 per CU it costs, 36 against 38 us).  The passes that read the
// spectrum do not gain from it (row_inv 172 us without, 185 us with; row_loss 247 and
// 284 us: their next row costs 30 registers per thread).
constexpr int row_groups(int M, int P) { return 160 * 1024 / (((P + 1) * M) * 8 + 128); }
constexpr bool row_pipe(int M, int P) { return row_groups(M, P) <= 2; }
constexpr int row_waves(int M, int P) { return lds_waves((P + 1) * M); }

// ----------------------------------------------------------------------------
// row passes: one row per workgroup, chain p at buf[P m + p], which is the row in
// natural bin order.  Blocks b and b + 8, which run on one XCD, take rows 2k and
// 2k + 1, so the two halves of each 128-byte line of the column-tiled spectrum
// meet in one L2.
// ----------------------------------------------------------------------------
__device__ __forceinline__ int paired_row(int b, int rows) {
  if (b >= (rows & ~15)) return b;
  return (b & ~15) + 2 * (b & 7) + ((b >> 3) & 1);
}

// stages S .. END - 1 of a row's chains, LDS to LDS
template <int M, int P, int T, int DIR, int S, int END>
__device__ __forceinline__ void row_stages(float2 *__restrict__ buf,
                                           const float2 *__restrict__ tw, int tid) {
  constexpr RowPlan p = row_plan(M, P, T);
  if constexpr (S < END) {
    constexpr int ns = (S > 0 ? p.r[0] : 1) * (S > 1 ? p.r[1] : 1) * (S > 2 ? p.r[2] : 1);
    cstage<p.r[S], DIR, P, T, M, ns>(buf, tw, tid);
    row_stages<M, P, T, DIR, S + 1, END>(buf, tw, tid);
  }
}

// Butterfly i of a radix-R stage over P interleaved chains (i = P j + p) reads, in the
// first stage, and writes, in the last, the row's elements i + q (P M / R): neighbouring
// threads have neighbouring elements, so the first stage of a transform loads its
// butterflies from memory and the last one stores them there, with no pass through LDS
// for the exchange with memory.  Before (rows staged in LDS on both sides) and now: 4K
// RGB row_loss 311 -> 246 us, row_inv 184 -> 172 us, row_fwd 147 -> 127 us (144 us
// without the pipeline); 1080p RGB 63.5 -> 60.6, 31.0 -> 28.4 and 36.5 -> 36.1 us.  The
// passes move 896, 597 and 597 MB at 4K: 3.6, 3.5 and 4.7 TB/s, against 5.2 TB/s of a
// large copy; the reads of 64-byte pieces of the spectrum bind the first two.
template <int M, int P, int T, int R>
struct EdgeStage {
  static constexpr int NB = M / R, ITEMS = NB * P, IT = (ITEMS + T - 1) / T;
  // element i + q ITEMS of row y of a channel's column-tiled spectrum
  // [ceil(P M / 8)][H][8]; where ITEMS is a multiple of 8, q moves the (uniform) base only
  template <class F2>
  static __device__ __forceinline__ F2 &at(F2 *Sc, int H, int y, int i, int q) {
    if constexpr (ITEMS % 8 == 0)
      return at32(Sc + (size_t)q * (ITEMS / 8) * H * 8, ((i >> 3) * H + y) * 8 + (i & 7));
    const int x = i + q * ITEMS;
    return at32(Sc, ((x >> 3) * H + y) * 8 + (x & 7));
  }
  static __device__ __forceinline__ void load(float2 (&v)[IT][R], const float2 *Sc, int H, int y,
                                              int tid) {
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int q = 0; q < R; ++q) v[it][q] = at(Sc, H, y, min(tid + it * T, ITEMS - 1), q);
  }
  // the first stage: registers to LDS
  template <int DIR>
  static __device__ __forceinline__ void first(float2 (&v)[IT][R], float2 *buf, int tid) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int i = tid + it * T;
      if (ITEMS % T == 0 || i < ITEMS) {
        RFft<R, DIR>::run(v[it]);
        const int b = i % P, j = i / P;
        static_for<0, R>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          buf[(j * R + q) * P + b] = v[it][q];
        });
      }
    }
  }
  // the last stage: LDS to memory
  template <int DIR>
  static __device__ __forceinline__ void last(const float2 *buf, const float2 *tw, float2 *Sc,
                                              int H, int y, int tid) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int i = tid + it * T;
      if (ITEMS % T == 0 || i < ITEMS) {
        const int b = i % P, j = i / P;
        float2 v[R];
        static_for<0, R>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          v[q] = buf[(j + q * NB) * P + b];
        });
        if constexpr (NB > 1) {
          static_for<1, R>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            float2 w = tw[q * j];
            if constexpr (DIR > 0) w.y = -w.y;
            v[q] = cmul(v[q], w);
          });
        }
        RFft<R, DIR>::run(v);
        static_for<0, R>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          at(Sc, H, y, i, q) = v[q];
        });
      }
    }
  }
};
template <int M, int P, int T>
using FirstStage = EdgeStage<M, P, T, row_plan(M, P, T).r[0]>;
template <int M, int P, int T>
using LastStage = EdgeStage<M, P, T, row_plan(M, P, T).r[row_plan(M, P, T).n - 1]>;

// Keeps what is computed from a value inside the loop over the rows: addresses that
// the compiler would otherwise hold in registers from one row to the next.
__device__ __forceinline__ void opaque(int &v) { asm volatile("" : "+v"(v)); }

// Waits for values loaded earlier (they become values of this point).  A pipelined
// row waits for its successor's loads here, before its own stores: loads and stores
// complete in issue order, and a wait after the stores would wait for them too.
template <int A, int B>
__device__ __forceinline__ void arrived(float2 (&v)[A][B]) {
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) asm volatile("" : "+v"(v[a][b].x), "+v"(v[a][b].y));
}

// M-entry table exp(-2 pi i e / M), stored contiguously after the P M table
template <int M, int P, int T>
__device__ __forceinline__ void load_chain_table(float2 *tw, const float2 *__restrict__ twf,
                                                 int tid) {
  constexpr int KT = (M + T - 1) / T;
  float2 tv[KT];
#pragma unroll
  for (int k = 0; k < KT; ++k) tv[k] = at32(twf, P * M + min(tid + k * T, M - 1));
#pragma unroll
  for (int k = 0; k < KT; ++k)
    if (KT * T == M || tid + k * T < M) tw[tid + k * T] = tv[k];
}

// the chain inputs at m = n from the samples a = x[n] and (P = 4) b = x[n + M]
template <int P>
__device__ __forceinline__ void chain_inputs(float2 *buf, int n, float2 a, float2 b, float2 w1) {
  if constexpr (P == 4) {
    const float2 w2 = cmul(w1, w1), w3 = cmul(w2, w1);
    buf[4 * n] = cadd(a, b);
    buf[4 * n + 1] = cmul(make_float2(a.x + b.y, a.y - b.x), w1);  // (a - i b) w^n
    buf[4 * n + 2] = cmul(csub(a, b), w2);                         // (a - b) w^{2n}
    buf[4 * n + 3] = cmul(make_float2(a.x - b.y, a.y + b.x), w3);  // (a + i b) w^{3n}
  } else {
    buf[2 * n] = a;
    buf[2 * n + 1] = cmul(a, w1);
  }
}

// u[n] and (P = 4) u[n + M] from the chain outputs at m = n
template <int P>
__device__ __forceinline__ void chain_outputs(const float2 *buf, int n, float2 w1, float2 &u0,
                                              float2 &u1) {
  if constexpr (P == 4) {
    const float2 w2 = cmul(w1, w1), w3 = cmul(w2, w1);
    const float2 z0 = buf[4 * n];
    const float2 z1 = cmul(cconj(w1), buf[4 * n + 1]);
    const float2 z2 = cmul(cconj(w2), buf[4 * n + 2]);
    const float2 z3 = cmul(cconj(w3), buf[4 * n + 3]);
    u0 = cadd(cadd(z0, z1), cadd(z2, z3));
    const float2 e = csub(z0, z2), o = csub(z1, z3);
    u1 = make_float2(e.x - o.y, e.y + o.x);  // z0 + i z1 - z2 - i z3
  } else {
    u0 = cadd(buf[2 * n], cmul(cconj(w1), buf[2 * n + 1]));
    u1 = make_float2(0.f, 0.f);
  }
}

#define CGH_ROW_KERNEL(M, P)                    \
  __global__ __launch_bounds__(row_threads(M, P)) \
      __attribute__((amdgpu_waves_per_eu(row_waves(M, P)))) void

// F1: field rows (zero-extended to Wp = P M) -> forward FFT -> S
template <int M, int P>
CGH_ROW_KERNEL(M, P) k_row_fwd_q(const float2 *__restrict__ field, int H, int W, int rows,
                                 const float2 *__restrict__ twf_x, float2 *__restrict__ S) {
  constexpr int T = row_threads(M, P), K = (M + T - 1) / T, Wt = (P * M + 7) / 8;
  constexpr RowPlan pl = row_plan(M, P, T);
  constexpr bool PIPE = row_pipe(M, P);
  __shared__ float2 buf[P * M];
  __shared__ float2 tw[M];
  int tid = threadIdx.x;
  load_chain_table<M, P, T>(tw, twf_x, tid);
  float2 wv[K], ab[2][K];
  auto load = [&](int blk) {
    const float2 *f = field + (size_t)paired_row(blk, rows) * W;  // (row R = c H + y)
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int n = min(tid + k * T, M - 1);
      ab[0][k] = at32(f, min(n, W - 1));
      ab[1][k] = P == 4 ? at32(f, min(n + M, W - 1)) : make_float2(0.f, 0.f);
    }
  };
#pragma unroll
  for (int k = 0; k < K; ++k) wv[k] = at32(twf_x, min(tid + k * T, M - 1));
  load(blockIdx.x);
  if constexpr (PIPE) arrived(ab);
  for (int blk = blockIdx.x; blk < rows; blk += gridDim.x) {
    if constexpr (PIPE) opaque(tid);
    const int R = paired_row(blk, rows), c = R / H, y = R - c * H;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int n = tid + k * T;
      if (K * T == M || n < M) {
        const float2 a = n < W ? ab[0][k] : make_float2(0.f, 0.f);
        const float2 b = n + M < W ? ab[1][k] : make_float2(0.f, 0.f);
        chain_inputs<P>(buf, n, a, b, wv[k]);
      }
    }
    lds_sync();
    row_stages<M, P, T, -1, 0, pl.n - 2>(buf, tw, tid);
    if constexpr (PIPE) load(min(blk + (int)gridDim.x, rows - 1));
    row_stages<M, P, T, -1, std::max(pl.n - 2, 0), pl.n - 1>(buf, tw, tid);
    if constexpr (PIPE) arrived(ab);
    LastStage<M, P, T>::template last<-1>(buf, tw, S + (size_t)c * Wt * H * 8, H, y, tid);
    if constexpr (!PIPE) break;
    lds_sync();
  }
}

// The sums of the loss partials of each hologram, by `blocks` workgroups more in front
// of B2's (one per hologram, 0: none), beside the rows: a kernel of its own would keep
// the device for its 3 to 13 us of dependent loads (6 us at 1080p RGB, 13 us at 4K RGB).
struct LossSums {
  const double *part;
  int planes, rows_per_plane, span, blocks;
  double inv_m;
  double *out;
  uint32_t *finite_flag;
};

// Hologram b: loss = sum of its loss partials / M, psnr = 10 log10(1 / loss), in a fixed
// order over T threads, four chains each.  The partials of plane l are
// part[l * rows_per_plane + r]; hologram b owns r in [b span, (b + 1) span).
template <int T>
__device__ __forceinline__ void loss_sums(const LossSums &a, int b) {
  __shared__ double red[T / 64];
  const int tid = threadIdx.x;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int l = 0; l < a.planes; ++l) {
    const double *p = a.part + (size_t)l * a.rows_per_plane + (size_t)b * a.span;
    for (int i = tid; i < a.span; i += 4 * T) {
      double v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = i + k * T < a.span ? p[i + k * T] : 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] += v[k];
    }
  }
  double acc = (s[0] + s[1]) + (s[2] + s[3]);
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_down(acc, d, 64);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double sum = 0.0;
    for (int w = 0; w < T / 64; ++w) sum += red[w];
    const double loss = sum * a.inv_m;
    a.out[2 * b] = loss;
    a.out[2 * b + 1] = 10.0 * log10(1.0 / loss);
    if (a.finite_flag && !isfinite(loss)) atomicOr(a.finite_flag, kNonFiniteLoss);
  }
}

// B2: S -> inverse FFT -> first W values of each row
template <int M, int P>
CGH_ROW_KERNEL(M, P) k_row_inv_q(const float2 *__restrict__ S, int H, int W, int rows,
                                 const float2 *__restrict__ twf_x, float2 *__restrict__ out,
                                 LossSums sums) {
  constexpr int T = row_threads(M, P), K = (M + T - 1) / T, Wt = (P * M + 7) / 8;
  constexpr RowPlan pl = row_plan(M, P, T);
  using First = FirstStage<M, P, T>;
  __shared__ float2 buf[P * M];
  __shared__ float2 tw[M];
  const int tid = threadIdx.x;
  const int blk = (int)blockIdx.x - sums.blocks;
  if (blk < 0) return loss_sums<T>(sums, blockIdx.x);
  load_chain_table<M, P, T>(tw, twf_x, tid);
  const int R = paired_row(blk, rows), c = R / H, y = R - c * H;
  float2 wv[K], v[First::IT][pl.r[0]];
  First::load(v, S + (size_t)c * Wt * H * 8, H, y, tid);
#pragma unroll
  for (int k = 0; k < K; ++k) wv[k] = at32(twf_x, min(tid + k * T, M - 1));
  First::template first<+1>(v, buf, tid);
  lds_sync();
  row_stages<M, P, T, +1, 1, pl.n>(buf, tw, tid);
  float2 *o = out + (size_t)R * W;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int n = tid + k * T;
    if ((K * T == M || n < M) && n < W) {
      float2 u0, u1;
      chain_outputs<P>(buf, n, wv[k], u0, u1);
      o[n] = u0;
      if (P == 4 && n + M < W) o[n + M] = u1;
    }
  }
}

// The middle row pass (F3).  S -> inverse FFT -> u (first W values) -> I =
// |u|^2 (optionally stored, with u); if make_grad: dL/dI = 2 (I - T) / M (MSE,
// Sec. 3.2) or the caller's dL/dI, g = 2 dL/dI u = dL/dRe(u) + j dL/dIm(u),
// zero-extended, forward FFT, back into S.  One FP64 partial sum of the loss per
// row into loss_part.
template <int M, int P>
CGH_ROW_KERNEL(M, P) k_row_loss_q(float2 *__restrict__ S, int H, int W, int rows,
                                  const float2 *__restrict__ twf_x,
                                  const float *__restrict__ target,
                                  const float *__restrict__ grad_I,
                                  const float *__restrict__ mask, int mcg,
                                  float *__restrict__ intensity, float2 *__restrict__ u_out,
                                  double *__restrict__ loss_part, float gscale, int make_grad) {
  constexpr int T = row_threads(M, P), K = (M + T - 1) / T, Wt = (P * M + 7) / 8, J = P / 2;
  constexpr RowPlan pl = row_plan(M, P, T);
  using First = FirstStage<M, P, T>;
  __shared__ float2 buf[P * M];
  __shared__ float2 tw[M];
  __shared__ double red[T / 64];
  const int tid = threadIdx.x;
  load_chain_table<M, P, T>(tw, twf_x, tid);
  const int R = paired_row(blockIdx.x, rows), c = R / H, y = R - c * H;
  float2 *Sc = S + (size_t)c * Wt * H * 8;
  float2 v[First::IT][pl.r[0]];
  First::load(v, Sc, H, y, tid);
  // per-element inputs at n and n + M and the chains' twiddles, fetched before the
  // transform so that their latency overlaps it
  const float *tsrc = target ? target : grad_I;
  const size_t row = (size_t)R * W;
  if (mask) mask += ((size_t)(c / mcg) * H + y) * W;
  float tv[J][K], mv[J][K];
  float2 wv[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int n = min(tid + k * T, M - 1);
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int x = min(n + j * M, W - 1);
      tv[j][k] = tsrc ? tsrc[row + x] : 0.f;
      mv[j][k] = mask ? mask[x] : 0.f;
    }
    wv[k] = at32(twf_x, n);
  }
  First::template first<+1>(v, buf, tid);
  lds_sync();
  row_stages<M, P, T, +1, 1, pl.n>(buf, tw, tid);
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int n = tid + k * T;
    if (K * T == M || n < M) {
      float2 u[2];
      chain_outputs<P>(buf, n, wv[k], u[0], u[1]);
      float f[2] = {0.f, 0.f};
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int x = n + j * M;
        if (x >= W) continue;
        const float t = tv[j][k], m = mv[j][k];
        const float I = u[j].x * u[j].x + u[j].y * u[j].y;
        if (intensity) intensity[row + x] = I;
        if (u_out) u_out[row + x] = u[j];
        if (target) {
          // L_recon weight 1 + m^2 + t^2 (plain MSE without a mask)
          const float d = I - t, w = mask ? 1.f + m * m + t * t : 1.f;
          acc += (double)d * (double)d * (double)w;
          f[j] = gscale * d * w;  // 4 w (I - T) / M
        } else if (grad_I) {
          f[j] = 2.0f * t;
        }
      }
      if (make_grad)
        chain_inputs<P>(buf, n, make_float2(f[0] * u[0].x, f[0] * u[0].y),
                        make_float2(f[1] * u[1].x, f[1] * u[1].y), wv[k]);
    }
  }
  if (target) {
    for (int d = 32; d > 0; d >>= 1) acc += __shfl_down(acc, d, 64);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
  }
  lds_sync();
  if (target && tid == 0) {
    double sum = 0.0;
    for (int w = 0; w < T / 64; ++w) sum += red[w];
    loss_part[R] = sum;
  }
  if (make_grad) {
    row_stages<M, P, T, -1, 0, pl.n - 1>(buf, tw, tid);
    LastStage<M, P, T>::template last<-1>(buf, tw, Sc, H, y, tid);
  }
}

// ----------------------------------------------------------------------------
// column pass
// ----------------------------------------------------------------------------
// Source, destination and transfer table of one column pass.  src and dst
// may be the same buffer (in place).  acc: add the result to dst instead of
// overwriting it (the adjoint's sum over planes).  htab points at the table
// of the pass's plane for channel 0; channel ch is at htab + ch * hstride.
// planes > 1 (k_col_wave with PLANES): plane l's table is at htab + l * hplane, and its
// spectrum at l * splane of dst (forward) or src (adjoint).
struct ColIO {
  const float2 *src;
  float2 *dst;
  const float2 *htab;
  size_t hstride;
  int acc;
  int planes;
  size_t hplane, splane;
};

// The steps of a column workgroup (k_col_wave); item i of a step is row n = i / NC of
// column c = i % NC of the workgroup's.
template <int M, int P, class PL = ColPlanOf<M>>
struct ColSteps {
  static constexpr ColPlan pl = PL::value;
  static constexpr int CH = pl.ch, R0 = pl.r0, R1 = pl.r1, R2 = pl.r2;
  static constexpr int NB2 = M / R2, LANES = CH * NB2;  // the fused stage's
  static_assert(R0 * R1 * R2 == M && LANES <= 64, "the fused stage takes one butterfly per lane");
  static constexpr int MS = col_stride(M, pl);
  // layouts in LDS: plain where the columns are loaded and combined
  struct Plain { static constexpr Pad value{0, 0}; };
  struct F0 { static constexpr Pad value = col_pads(M, pl).f0; };
  struct F1 { static constexpr Pad value = col_pads(M, pl).f1; };
  struct I0 { static constexpr Pad value = col_pads(M, pl).i0; };
  struct I1 { static constexpr Pad value = col_pads(M, pl).i1; };
  static constexpr int NC = 8 / P;  // columns per workgroup
  static constexpr int T = col_threads(pl), NI = NC * M, K = (NI + T - 1) / T;

  // the columns' samples, to registers
  static __device__ __forceinline__ void load(const float2 *src, int H, int tid, float2 (&av)[K],
                                              float2 (&bv)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = tid + k * T, n = min(i / NC, M - 1), c = i % NC;
      av[k] = at32(src, min(n, H - 1) * 8 + c);
      bv[k] = P == 4 ? at32(src, min(n + M, H - 1) * 8 + c) : make_float2(0.f, 0.f);
    }
  }
  static __device__ __forceinline__ void load_w(const float2 *twf_y, int tid, float2 (&w1)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) w1[k] = at32(twf_y, min((tid + k * T) / NC, M - 1));
  }
  // the chains' inputs, to LDS
  static __device__ __forceinline__ void inputs(float2 *buf, int H, int tid, float2 (&av)[K],
                                                float2 (&bv)[K], float2 (&w1)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = tid + k * T, n = i / NC, c = i % NC;
      if (K * T == NI || i < NI) {
        const float2 a = n < H ? av[k] : make_float2(0.f, 0.f);
        if constexpr (P == 4) {
          const float2 bb = n + M < H ? bv[k] : make_float2(0.f, 0.f);
          const float2 s0 = cadd(a, bb), s2 = csub(a, bb);
          const float2 s1 = make_float2(a.x + bb.y, a.y - bb.x);  // a - i b
          const float2 s3 = make_float2(a.x - bb.y, a.y + bb.x);  // a + i b
          const float2 w2 = cmul(w1[k], w1[k]), w3 = cmul(w2, w1[k]);  // w^{2n}, w^{3n}
          buf[(4 * c) * MS + n] = s0;
          buf[(4 * c + 1) * MS + n] = cmul(s1, w1[k]);
          buf[(4 * c + 2) * MS + n] = cmul(s2, w2);
          buf[(4 * c + 3) * MS + n] = cmul(s3, w3);
        } else {
          buf[(2 * c) * MS + n] = a;
          buf[(2 * c + 1) * MS + n] = cmul(a, w1[k]);
        }
      }
    }
  }
  // a lane's transfer values: spectrum entries ky = P (j + NB2 q) + p of chain `chain`,
  // whose column's table starts at entry col0 of h
  static __device__ __forceinline__ void transfer(const float2 *h, uint32_t col0, int p, int lane,
                                                  float2 (&hv)[R2]) {
    const int j = min(lane, LANES - 1) % NB2;
    static_for<0, R2>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      const int ky = P * (j + NB2 * q) + p;
      hv[q] = at32(h, col0 + min(ky, P * M - ky));
    });
  }
  // a wave's chains, LDS to the spectrum entries j + NB2 q of lane NB2 u + j (chain u)
  static __device__ __forceinline__ void forward(float2 *wb, const float2 *tw, int lane,
                                                 float2 (&v)[R2]) {
    wstage<R0, -1, M, 1, CH, MS, Plain, F0>(wb, tw, lane);
    if constexpr (R1 > 1) wstage<R1, -1, M, R0, CH, MS, F0, F1>(wb, tw, lane);
    if (lane < LANES) {
      constexpr Pad in = R1 > 1 ? F1::value : F0::value;
      const int u = lane / NB2, j = lane - u * NB2, at = u * MS + in.at(j);
      static_for<0, R2>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        v[q] = wb[at + in.at(q * NB2)];
      });
      static_for<1, R2>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        v[q] = cmul(v[q], tw[q * j]);  // last forward stage: Ns = NB2, unit twiddle step
      });
      RFft<R2, -1>::run(v);
    }
  }
  // the inverse of the spectrum entries of each lane, to LDS
  static __device__ __forceinline__ void inverse(float2 *wb, const float2 *tw, int lane,
                                                 float2 (&v)[R2]) {
    if (lane < LANES) RFft<R2, +1>::run(v);  // first inverse stage: Ns = 1, no twiddles
    wave_lds_order();
    if (lane < LANES) {
      const int u = lane / NB2, j = lane - u * NB2, at = u * MS + I0::value.at(j * R2);
      static_for<0, R2>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        wb[at + q] = v[q];
      });
    }
    wave_lds_order();
    if constexpr (R1 > 1) {
      wstage<R1, +1, M, R2, CH, MS, I0, I1>(wb, tw, lane);
      wstage<R0, +1, M, R2 * R1, CH, MS, I1, Plain>(wb, tw, lane);
    } else {
      wstage<R0, +1, M, R2, CH, MS, I0, Plain>(wb, tw, lane);
    }
  }
  // the columns from the chains' outputs
  static __device__ __forceinline__ void outputs(const float2 *buf, float2 *dst, int H, int acc,
                                                 int tid, float2 (&w1)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = tid + k * T, n = i / NC, c = i % NC;
      if ((K * T == NI || i < NI) && n < H) {
        float2 y0, y1;
        if constexpr (P == 4) {
          const float2 w2 = cmul(w1[k], w1[k]), w3 = cmul(w2, w1[k]);
          const float2 z0 = buf[(4 * c) * MS + n];
          const float2 z1 = cmul(cconj(w1[k]), buf[(4 * c + 1) * MS + n]);
          const float2 z2 = cmul(cconj(w2), buf[(4 * c + 2) * MS + n]);
          const float2 z3 = cmul(cconj(w3), buf[(4 * c + 3) * MS + n]);
          y0 = cadd(cadd(z0, z1), cadd(z2, z3));
          // z0 + i z1 - z2 - i z3
          const float2 e = csub(z0, z2), o = csub(z1, z3);
          y1 = make_float2(e.x - o.y, e.y + o.x);
        } else {
          y0 = cadd(buf[(2 * c) * MS + n], cmul(cconj(w1[k]), buf[(2 * c + 1) * MS + n]));
        }
        float2 &d0 = at32(dst, n * 8 + c);
        d0 = acc ? cadd(d0, y0) : y0;
        if (P == 4 && n + M < H) {
          float2 &d1 = at32(dst, (n + M) * 8 + c);
          d1 = acc ? cadd(d1, y1) : y1;
        }
      }
    }
  }
};

// Column pass with one wave per chain, M = R0 R1 R2 (col_plan); CONJ: multiply
// by conj(H) (the adjoint pass).  A workgroup of eight waves takes 8 / P
// columns of a tile of 8; wave P c + p runs chain p of column c in its own
// M-element LDS buffer, so the stages of a chain need no workgroup barrier: only
// loading the columns and combining the chains are workgroup steps.  The
// forward plan is R0, R1, R2; its last stage leaves lane j < M / R2 holding
// spectrum entries j + (M / R2) q (q < R2), exactly the input of a first
// inverse stage of radix R2, so the transfer multiply and that stage run in
// registers; the inverse plan is R2, R1, R0.  The transfer table is read
// column-major ([Wq][Hq]); the workgroups of a mirror pair of tiles
// (t, Wt - 1 - t), whose columns need about the same table columns, are blocks
// b + 8 s (s < 2 P), which share an XCD.
//
// PLANES: every focal plane in one pass.  The planes share the spectrum of the field, so
// the forward pass transforms a column once, keeps its entries in registers and inverts
// their product with each plane's table; the adjoint adds conj(H_l) times each plane's
// spectrum in registers and inverts the sum once.  Of L planes' 2 L transforms, L + 1 are
// left, and the shared side is read (or its sum written) once.  Bound by VALU issue and LDS
// as with one plane; lengths by planes_chain.
template <int M, int P, bool CONJ, bool PLANES, class PL = ColPlanOf<M>>
__global__ __launch_bounds__(col_threads(PL::value))
__attribute__((amdgpu_waves_per_eu(col_waves(M, PL::value)))) void
k_col_wave(ColIO io, int Hq, int H, int Wp, int Wt, int C, const float2 *__restrict__ twf_y) {
  using S = ColSteps<M, P, PL>;
  constexpr int T = S::T, K = S::K, R2 = S::R2, NC = S::NC, KT = (M + T - 1) / T;
  __shared__ float2 buf[8 * S::MS];
  __shared__ float2 tw[M];
  int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: scalar addressing
  const int b = blockIdx.x;
  constexpr int SL = 2 * P;  // workgroups of a mirror pair
  const int slot = (b >> 3) % SL, pi = (b / (8 * SL)) * 8 + (b & 7);
  const int hp = (Wt + 1) >> 1;
  if (pi >= C * hp) return;
  const int ch = pi / hp, pp = pi - ch * hp;
  const int t = slot < P ? pp : Wt - 1 - pp;
  if (slot >= P && t == pp) return;  // the middle tile of an odd count has no mirror
  const int part = slot % P;
  const size_t off = ((size_t)ch * Wt + t) * H * 8 + part * NC;
  const float2 *src = io.src + off;
  float2 *dst = io.dst + off;
  // the chain of this lane's fused butterfly (uniform with one chain per wave)
  const int chain = S::CH == 1 ? wave : wave * S::CH + min(lane, S::LANES - 1) / S::NB2;
  const int c = chain / P, p = chain % P;
  float2 *wb = buf + wave * (S::CH * S::MS);
  // columns past Wp (the last tile of a Wp that is not a multiple of 8) hold
  // nothing that is read again; their table column is clamped
  const int kx = min(t * 8 + part * NC + c, Wp - 1);
  const int qx = min(kx, Wp - kx);
  const float2 *h = io.htab + (size_t)ch * io.hstride;
  const uint32_t col0 = (uint32_t)(qx * Hq);  // below 4097^2: 32-bit byte offsets reach it
  float2 av[K], bv[K];
  {
    // every global load of this phase is issued before the first LDS store
    float2 w1[K], tv[KT];
    S::load(src, H, tid, av, bv);
    S::load_w(twf_y, tid, w1);
#pragma unroll
    for (int k = 0; k < KT; ++k) tv[k] = at32(twf_y, P * M + min(tid + k * T, M - 1));  // w_M^k
#pragma unroll
    for (int k = 0; k < KT; ++k)
      if (tid + k * T < M) tw[tid + k * T] = tv[k];
    S::inputs(buf, H, tid, av, bv, w1);
  }
  __syncthreads();
  float2 hv[R2], v[R2];
  auto times_h = [&](float2 (&o)[R2], bool add) {
    static_for<0, R2>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      const float2 r = cmul(v[q], CONJ ? cconj(hv[q]) : hv[q]);  // the table carries 1 / (Hp Wp)
      o[q] = add ? cadd(o[q], r) : r;
    });
  };
  if constexpr (!PLANES) {
    S::transfer(h, col0, p, lane, hv);  // issued before the forward stages
    S::forward(wb, tw, lane, v);
    if (lane < S::LANES) times_h(v, false);
    S::inverse(wb, tw, lane, v);
    float2 w1[K];
    S::load_w(twf_y, tid, w1);
    __syncthreads();
    S::outputs(buf, dst, H, io.acc, tid, w1);
  } else if constexpr (!CONJ) {
    S::transfer(h, col0, p, lane, hv);
    S::forward(wb, tw, lane, v);
    float2 w1[K], o[R2];
    for (int l = 0; l < io.planes; ++l) {
      opaque(tid);
      opaque(lane);
      if (l > 0) {
        S::transfer(h + (size_t)l * io.hplane, col0, p, lane, hv);
        __syncthreads();  // the previous plane's outputs have left LDS
      }
      times_h(o, false);
      S::inverse(wb, tw, lane, o);
      S::load_w(twf_y, tid, w1);
      __syncthreads();
      S::outputs(buf, dst + (size_t)l * io.splane, H, 0, tid, w1);
    }
  } else {
    float2 sum[R2];
#pragma unroll
    for (int q = 0; q < R2; ++q) sum[q] = make_float2(0.f, 0.f);
    // the next plane's columns are loaded ahead where the registers hold them (the sum,
    // a spectrum and its table values are 6 R2 of the 128)
    constexpr bool AHEAD = 4 * R2 + 4 * K <= 48;
    float2 w1[K];
    for (int l = 0;;) {
      opaque(tid);
      opaque(lane);
      const bool more = l + 1 < io.planes;
      if (AHEAD && more) S::load(src + (size_t)(l + 1) * io.splane, H, tid, av, bv);
      if (AHEAD) S::transfer(h + (size_t)l * io.hplane, col0, p, lane, hv);
      S::forward(wb, tw, lane, v);
      if (!AHEAD) S::transfer(h + (size_t)l * io.hplane, col0, p, lane, hv);
      if (lane < S::LANES) times_h(sum, true);
      ++l;
      if (!more) break;
      if (!AHEAD) S::load(src + (size_t)l * io.splane, H, tid, av, bv);
      S::load_w(twf_y, tid, w1);
      __syncthreads();  // every chain has left LDS
      S::inputs(buf, H, tid, av, bv, w1);
      __syncthreads();
    }
    S::inverse(wb, tw, lane, sum);
    S::load_w(twf_y, tid, w1);
    __syncthreads();
    S::outputs(buf, dst, H, io.acc, tid, w1);
  }
}

// ----------------------------------------------------------------------------
// Launchers, one translation unit per part: part k of kChainParts holds the
// chain lengths whose index in increasing order is k modulo kChainParts.
// ----------------------------------------------------------------------------
struct RowArgs {
  int pass;  // 0: forward (F1), 1: inverse (B2), 2: middle pass (F3)
  const float2 *field;
  float2 *S;
  float2 *out;
  int H, W, rows, num_cu;
  const float2 *twf_x;
  const float *target, *grad_I, *mask;
  int mcg;
  float *intensity;
  float2 *u_out;
  double *loss_part;
  float gscale;
  int make_grad;
  LossSums sums;
};
struct ColArgs {
  ColIO io;
  int conj_h, Hq, H, Wp, Wt, C;
  const float2 *twf_y;
};
constexpr int kChainParts = 8;
// each returns true if its part holds the (M, P) kernels (which were then launched)
#define CGH_CHAIN_PART_FNS(k)                                               \
  bool row_chain_part_##k(int M, int P, const RowArgs &a, hipStream_t s); \
  bool col_chain_part_##k(int M, int P, const ColArgs &a, hipStream_t s);
CGH_CHAIN_PART_FNS(0) CGH_CHAIN_PART_FNS(1) CGH_CHAIN_PART_FNS(2) CGH_CHAIN_PART_FNS(3)
CGH_CHAIN_PART_FNS(4) CGH_CHAIN_PART_FNS(5) CGH_CHAIN_PART_FNS(6) CGH_CHAIN_PART_FNS(7)
#undef CGH_CHAIN_PART_FNS

}  // namespace cgh
