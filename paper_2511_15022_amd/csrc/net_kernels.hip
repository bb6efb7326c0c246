// Kernels of the learned initialiser's U-Net (include/cgh_net.h): 3x3
// convolutions as implicit GEMMs on the matrix cores (BF16 inputs, FP32
// sums), their weight gradients, and the pooling, upsampling, ReLU and
// lattice glue around them.
//
// Matrix instruction (one wave, D = A B + D, D 32 x 32 FP32): in v_mfma_f32_32x32x16
// bf16 (A 32 x 16, B 16 x 32) lane l supplies A[l % 32][8 (l / 32) + i] and
// B[8 (l / 32) + i][l % 32] (i < 8) and holds D[8 (v / 4) + 4 (l / 32) + v % 4][l % 32] in
// accumulator v < 16.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "cgh_internal.h"
#include "cgh_net.h"
#include "fft_reg.h"

namespace cgh {
namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);  // nearest, ties to even
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

bool al16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

// ----------------------------------------------------------------------------
// Convolution.  A workgroup of four waves takes tiles of 32 columns x 4 R rows and
// 32 NB output channels; wave w takes R rows of a tile (all 32 columns), in R NB
// accumulators of 32 channels x 32 pixels.  For each block of 16 input channels (a
// stage) it holds in LDS the tile's input pixels with a border of one (4 R + 2 rows
// of 34) and its output channels' weights for the 9 taps.  A wave reads its 9 NB
// weight fragments once per stage, then walks its R + 2 staged rows: one fragment
// of a staged row serves the three output rows above, at and below it, so a stage
// costs 3 (R + 2) + 9 NB reads of 16 bytes per lane for 9 R NB matrix instructions
// (R = 4, NB = 2: 36 for 72; with one row per wave and a read of each operand per tap
// 27 for 18).  LDS feeds at most one such read per two matrix instructions of the
// CU's four SIMDs, so this ratio decides whether the matrix cores or LDS are the
// limit.  With at most 32 input channels (KC = 2) a stage is the whole tile and the
// weights stay in registers for the kernel: there HBM is the limit.
//
// The stages are loaded straight into LDS (buffer loads to LDS, 16 bytes per lane:
// no registers held while they are in flight), NBUF - 1 stages ahead of the
// products and across tiles: workgroups are persistent, so a tile's first stage
// loads during the last products and the stores of the tile before it.  One
// barrier per stage, which waits for LDS only.  A lane without a source (outside the
// image, past the last channel) has an offset past the buffer's end, which reads
// zero.  The loads fill LDS in lane order, so the arrangement against bank conflicts
// is made on the source side: slot 2 i + b of 16 bytes holds half
// b ^ ((column >> 3) & 1) of pixel i's 16 channels (of weight row i, its channel; with
// KC = 2, quarter b ^ ((column >> 2) & 3) in slot 4 i + b), which spreads the 16 lanes
// of an LDS phase over all banks and keeps a pixel's channels on neighbouring
// lanes of the load.
//
// The weights are the A operand and the pixels the B operand, so a lane ends up
// with groups of four consecutive channels of one pixel; exchanges between the
// wave's halves make them eight, and the outputs leave in 16-byte stores without
// passing through LDS.
//
// For every output the products are added in the order input block, tap
// (ky, kx), channel group of the instruction, whatever the tile: results do not
// depend on NB, R and FAR.
//
// A slot's offset from its tile's first pixel has 32 bits.  FAR: for images whose
// staged rows lie further apart than that (far_rows), each wave's slots, which lie in
// at most two staged rows, are loaded from a 64-bit base per row, and offsets count
// from the row's first staged pixel (64 -> 32 channels, 18 x 2^20 pixels: 1.95 ms, weight
// gradients 1.66 ms; as many pixels at 1024 x 18432, without it, 1.17 and 1.15 ms).
//
// Measured (1080 x 1920, C = 3, per layer, before and now): 24 -> 32 channels 96 and
// 53 us (4.4 TB/s), 32 -> 32 84 and 60 us, 96 -> 32 209 and 128 us; 128 -> 128 at
// 270 x 480 66 and 44 us, 384 -> 128 152 and 94 us (1214 TFLOP/s; a large library
// matrix product reaches 1227 on the same card).
// ----------------------------------------------------------------------------

// A buffer of `bytes` bytes from `base`; loads at or past the end return zero.
constexpr int kBufferBytes = 0x7fff0000;    // the end where offsets are valid by construction
constexpr uint32_t kOutside = 0x80000000u;  // an offset past the end of any buffer here
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const uint16_t *base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), 0, bytes, 0x00027000);
}

// 16 bytes per lane, at byte `off` + `sof` (wave-uniform) of `buf`, to LDS at `dst`
// (wave-uniform) + 16 lane
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t buf, uint32_t off, int sof,
                                            v8s *dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(
      buf, (__attribute__((address_space(3))) void *)dst, 16, off, sof, 0, 0);
}

// two BF16 (round to nearest, ties to even) in one word, by the hardware conversion
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  v2bf r;
  r[0] = (__bf16)a;
  r[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, r);
}

// the BF16 pair v where the pair m is > 0 (its bits 0x0001 .. 0x7f80: not NaN), else 0
__device__ __forceinline__ uint32_t gated(uint32_t v, uint32_t m) {
  const uint32_t lo = m & 0xffffu, hi = m >> 16;
  return (lo - 1u < 0x7f80u ? v & 0xffffu : 0u) | (hi - 1u < 0x7f80u ? v & 0xffff0000u : 0u);
}

// waits until at most N of this wave's vector memory operations are in flight (the
// builtin, so that the compiler knows)
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}

struct ConvArgs {
  const uint16_t *x1, *x2, *w;
  const float *bias;
  int c1, c2, up, H, W, cout, relu;
  float *out32;
  uint16_t *out16;
  uint16_t *pooled;      // 2 x 2 averages of out16, or null
  const uint16_t *gate;  // out16 is zero where gate <= 0 (gradient through ReLU), or null
  int tiles_x, nco, items;  // column tiles, channel tiles, tiles in all (channel tile fastest)
};

// Whether a tile's staged pixels (at most 18 rows and 34 columns) may lie past the end of
// a buffer from its first one, in an image of W columns and c channels.
bool far_rows(int W, int c) { return 2 * (int64_t)c * (18 * (int64_t)W + 64) > kBufferBytes; }

// 16 bytes per lane to LDS at `dst`, as load_to_lds, from byte `off` + `sof` of the staged
// row `row` of each lane, which is r0 or r0 + 1 (wave-uniform); from(r) is the (uniform)
// address of the first staged pixel of row r
template <class FROM>
__device__ __forceinline__ void load_two_rows(int row, int r0, FROM from, uint32_t off, int sof,
                                              v8s *dst) {
#pragma unroll
  for (int e = 0; e < 2; ++e)
    if (row == r0 + e) load_to_lds(buffer_of(from(r0 + e), kBufferBytes), off, sof, dst);
}

template <int R, int NB, int KC, int NBUF, bool TWO, bool GEN, bool FAR = false>
__global__ __launch_bounds__(256, 2) void k_conv3x3(ConvArgs a) {
  constexpr bool THIN = KC == 2;
  static_assert(!FAR || (!THIN && NBUF == 2), "far rows: one number of loads per wave is not kept");
  static_assert(!THIN || (!TWO && NB == 1 && NBUF == 2), "one input of at most 32 channels");
  constexpr int CO = 32 * NB, TY = 4 * R, SR = TY + 2, SC = 34, SP = 2 * KC;  // SP: slots per pixel
  constexpr int NA = SR * SC * SP, NW = THIN ? 0 : 9 * CO * 2;  // 16-byte slots
  constexpr int KA = (NA + 255) / 256, KW = (NW + 255) / 256;
  // With more than two buffers a wait counts the loads still in flight, so every
  // wave issues the same number: the slots are padded to whole rounds.
  constexpr bool PAD = NBUF > 2;
  constexpr int LA = PAD ? 256 * KA : NA, LW = PAD ? 256 * KW : NW, LB = LA + LW;
  __shared__ v8s smem[NBUF][LB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int px = lane & 31, half = lane >> 5;
  const int H = a.H, W = a.W, cin = TWO ? a.c1 + a.c2 : a.c1;
  const int W1 = TWO && a.up ? W >> 1 : W;  // (an upsampled input always has a skip here)
  const int nst = THIN ? 1 : (cin + 15) / 16;  // stages per tile (a last block of 8 is zero-filled)
  // Workgroup b runs on XCD b % 8.  Each XCD takes one contiguous run of the tiles and
  // its workgroups take them in turn, so neighbouring tiles, which share border
  // pixels or inputs, meet in one L2.
  const int xcd = blockIdx.x & 7, nx = (gridDim.x - xcd + 7) >> 3;
  const int share = a.items >> 3, extra = a.items & 7;
  const int run0 = xcd * share + min(xcd, extra), run1 = run0 + share + (xcd < extra ? 1 : 0);
  int item = run0 + (blockIdx.x >> 3);
  if (item >= run1) return;
  // The pixel slots this thread fills: the byte offsets of their channels in x1 and
  // x2 from the tile's first staged pixel.  Tiles start at multiples of 4 rows and
  // 32 columns, so with an upsampled x1 these are the same for every tile too.
  uint32_t o1[KA], o2[TWO ? KA : 1], ah = 0;  // ah bit k: the upper 8 channels
#pragma unroll
  for (int k = 0; k < KA; ++k) {
    const int s = tid + 256 * k, i = s / SP, row = i / SC, col = i - row * SC;
    const int g = (s % SP) ^ (THIN ? (col >> 2) & 3 : (col >> 3) & 1);
    if (g & 1) ah |= 1u << k;
    int q = FAR ? col : row * W + col;
    if constexpr (TWO) {
      o2[k] = s < NA ? 2u * (uint32_t)(q * a.c2 + 8 * g) : kOutside;
      if (a.up) q = FAR ? (col + 1) >> 1 : ((row + 1) >> 1) * W1 + ((col + 1) >> 1);
    }
    o1[k] = s < NA && (!THIN || 8 * g < cin) ? 2u * (uint32_t)(q * a.c1 + 8 * g) : kOutside;
  }
  uint32_t wo[KW > 0 ? KW : 1], wh = 0;
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const int s = tid + 256 * k, i = s >> 1, t = i / CO, c = i - t * CO;
    const int g = (s & 1) ^ ((c >> 3) & 1);
    if (g) wh |= 1u << k;
    wo[k] = s < NW ? 2u * (uint32_t)((c * 9 + t) * cin + 8 * g) : kOutside;
  }
  // the tile being loaded
  __amdgpu_buffer_rsrc_t b1, b2, bw;
  const uint16_t *f1 = nullptr, *f2 = nullptr;  // FAR: the bases of b1 and b2
  uint32_t out = 0;  // bit k: slot k's pixel lies outside the image
  auto aim = [&](int it) {
    const int tile = THIN ? it : it / a.nco, ty = tile / a.tiles_x;
    const int ax = (tile - ty * a.tiles_x) * 32 - 1, ay = ty * TY - 1;
    out = 0;
    if (ay < 0 || ax < 0 || ay + SR > H || ax + SC > W) {  // an edge tile
      int t0 = tid;
      asm volatile("" : "+v"(t0));  // worked out here, not kept
#pragma unroll
      for (int k = 0; k < KA; ++k) {
        const int i = (t0 + 256 * k) / SP, row = i / SC, col = i - row * SC;
        const bool in = ((uint32_t)(ay + row) < (uint32_t)H) & ((uint32_t)(ax + col) < (uint32_t)W);
        out |= in ? 0u : 1u << k;
      }
    }
    // the first staged pixel; before the first of the image where that lies outside
    const int64_t q2 = (int64_t)ay * W + ax;
    if constexpr (TWO) {
      const int64_t q1 = a.up ? (int64_t)(((ay + 1) >> 1) - 1) * W1 + ((ax + 1) >> 1) - 1 : q2;
      b1 = buffer_of(a.x1 + q1 * a.c1, kBufferBytes);
      b2 = buffer_of(a.x2 + q2 * a.c2, kBufferBytes);
      if constexpr (FAR) f1 = a.x1 + q1 * a.c1, f2 = a.x2 + q2 * a.c2;
    } else {
      b1 = buffer_of(a.x1 + q2 * a.c1, kBufferBytes);
    }
    if constexpr (!THIN) {
      const int co = (it - tile * a.nco) * CO;
      bw = buffer_of(a.w + (size_t)co * 9 * cin, (a.cout - co) * 9 * cin * 2);
    }
  };
  // slot k's 16 bytes at offset o + sof of src, which is b1 (or, with `second`, b2), to LDS
  auto load_pixel = [&](__amdgpu_buffer_rsrc_t src, bool second, uint32_t o, int sof, int k,
                        v8s *dst) {
    if constexpr (FAR) {
      static_assert(64 / SP <= SC, "a wave's slots lie in at most two rows");
      load_two_rows(
          (tid + 256 * k) / SP / SC, (64 * wave + 256 * k) / SP / SC,
          [&](int r) {
            return second ? f2 + (int64_t)r * W * a.c2
                          : f1 + (int64_t)(a.up ? (r + 1) >> 1 : r) * W1 * a.c1;
          },
          o, sof, dst);
    } else {
      load_to_lds(src, o, sof, dst);
    }
  };
  // offset o of slot k, past the buffer where its pixel is outside
  auto masked = [&](uint32_t o, int k) { return o | ((out << (31 - k)) & kOutside); };
  auto load_stage = [&](int st, int buf) {
    v8s *const sa = smem[buf] + 64 * wave, *const sw = sa + LA;
    const int c0 = 16 * st;  // the block's channels c0 .. c0 + 15
    if (!GEN || (c0 + 8 < cin && (c0 + 8 < a.c1 || c0 >= a.c1))) {
      // uniform: sixteen channels of one input
      const bool in1 = !TWO || c0 < a.c1;
      const __amdgpu_buffer_rsrc_t src = in1 ? b1 : b2;
      const int sof = 2 * (in1 ? c0 : c0 - a.c1);
#pragma unroll
      for (int k = 0; k < KA; ++k)
        if (PAD || 256 * (k + 1) <= NA || tid + 256 * k < NA)
          load_pixel(src, !in1, masked(in1 ? o1[k] : o2[TWO ? k : 0], k), sof, k, sa + 256 * k);
    } else {
      // the last eight channels, or x1's last eight and x2's first
      const bool both = TWO && c0 < a.c1 && c0 + 8 >= a.c1 && c0 + 8 < cin;
#pragma unroll
      for (int k = 0; k < KA; ++k) {
        if (!PAD && 256 * (k + 1) > NA && tid + 256 * k >= NA) continue;
        const bool up8 = (ah >> k) & 1;
        const uint32_t p1 = masked(o1[k], k), p2 = TWO ? masked(o2[k], k) : kOutside;
        if (TWO && (up8 || c0 >= a.c1))
          load_pixel(b2, true, up8 ? (both && p2 < kOutside ? p2 - 16u : kOutside)
                                   : p2 + 2u * (uint32_t)(c0 - a.c1),
                     0, k, sa + 256 * k);
        else
          load_pixel(b1, false, up8 ? kOutside : p1, 2 * c0, k, sa + 256 * k);
      }
    }
    if constexpr (!THIN) {
      const bool cut = GEN && c0 + 8 >= cin;  // the block's upper 8 channels are past the last
#pragma unroll
      for (int k = 0; k < KW; ++k)
        if (PAD || 256 * (k + 1) <= NW || tid + 256 * k < NW)
          load_to_lds(bw, cut && ((wh >> k) & 1) ? kOutside : wo[k], 2 * c0, sw + 256 * k);
    }
  };
  v16f acc[R][NB];
  v8bf wf[KC][9][NB];
  auto channel = [&](int it) { return THIN ? (int)blockIdx.y * CO : (it % a.nco) * CO; };
  // this lane's operands in a buffer: pixel (row wave R, column px + kx), group 2 u +
  // half, and weight row px
  int ia[3][KC];
#pragma unroll
  for (int kx = 0; kx < 3; ++kx)
#pragma unroll
    for (int u = 0; u < KC; ++u) {
      const int col = px + kx, g = 2 * u + half;
      ia[kx][u] = (wave * R * SC + col) * SP + (g ^ (THIN ? (col >> 2) & 3 : (col >> 3) & 1));
    }
  const int iw = LA + px * 2 + (half ^ ((px >> 3) & 1));
  auto products = [&](int buf) {
    const v8s *const sb = smem[buf];
    if constexpr (!THIN) {
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          wf[0][t][b] = __builtin_bit_cast(v8bf, sb[iw + (t * CO + 32 * b) * 2]);
    }
#pragma unroll
    for (int u = 0; u < KC; ++u) {
      // the three fragments of the next staged row are read before this row's products
      v8bf f[2][3];
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) f[0][kx] = __builtin_bit_cast(v8bf, sb[ia[kx][u]]);
#pragma unroll
      for (int sr = 0; sr < R + 2; ++sr) {
        if (sr + 1 < R + 2)
#pragma unroll
          for (int kx = 0; kx < 3; ++kx)
            f[(sr + 1) & 1][kx] =
                __builtin_bit_cast(v8bf, sb[ia[kx][u] + (sr + 1) * SC * SP]);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int ky = sr - r;
            if (ky < 0 || ky > 2) continue;
#pragma unroll
            for (int b = 0; b < NB; ++b)
              acc[r][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  wf[u][3 * ky + kx][b], f[sr & 1][kx], acc[r][b], 0, 0, 0);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // the stages are loaded in order, NBUF - 1 ahead of the products, across tiles
  int l_item = item, l_st = 0, l_buf = 0;
  auto load_next = [&]() -> bool {
    if (l_item >= run1) return false;
    load_stage(l_st, l_buf);
    l_buf = l_buf + 1 == NBUF ? 0 : l_buf + 1;
    if (++l_st == nst) {
      l_st = 0;
      l_item += nx;
      if (l_item < run1) aim(l_item);
    }
    return true;
  };
  // this wave's loads of the next stage have landed: with `ahead` stages loaded
  // after it still in flight
  auto landed = [&](bool ahead) {
    if (NBUF == 3 && ahead) wait_vm<KA + KW>();
    else wait_vm<0>();
  };
  static_assert(NBUF == 2 || (NBUF == 3 && KA + KW < 63), "buffers");
  aim(item);
  load_next();
  if constexpr (THIN) {
    // the weights of this workgroup's channels, for the whole kernel
    const int c = channel(0) + px;
#pragma unroll
    for (int u = 0; u < KC; ++u)
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int ci = 16 * u + 8 * half;
        v8s v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (c < a.cout && ci < cin)
          v = *reinterpret_cast<const v8s *>(a.w + ((size_t)c * 9 + t) * cin + ci);
        wf[u][t][0] = __builtin_bit_cast(v8bf, v);
      }
  }
  landed(NBUF == 3 && load_next());
  lds_sync();  // (a barrier that leaves the loads in flight)
  int buf = 0;
  while (true) {
    const int tile = THIN ? item : item / a.nco, ty = tile / a.tiles_x;
    const int x0 = (tile - ty * a.tiles_x) * 32, y0 = ty * TY, co0 = channel(item);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][b][v] = 0.f;
    for (int st = 0; st < nst; ++st) {
      // the stage in smem[buf] has landed for every wave, and no wave reads the buffer
      // of the stage before it any more, which the next load fills
      const bool ahead = load_next();
      products(buf);
      // (the stores of a tile's outputs are issued after this wait, so they complete
      // during the next stage's products)
      landed(ahead);
      buf = buf + 1 == NBUF ? 0 : buf + 1;
      if (st + 1 < nst) lds_sync();
    }
    // ---- outputs: lane l holds, of pixel l % 32, channels 8 g + 4 (l / 32) + e in
    // accumulator 4 g + e (g, e < 4)
    const int x = x0 + px;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
    const int cb = co0 + 32 * b;
    float bv[16];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool any = a.bias && cb + 8 * g < a.cout;  // uniform: scalar loads
        const float lo = any ? a.bias[cb + 8 * g + e] : 0.f;
        const float hi = any ? a.bias[cb + 8 * g + 4 + e] : 0.f;
        bv[4 * g + e] = half ? hi : lo;
      }
    uint32_t prev[8];  // the packed channels of the row above (pooling)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int y = y0 + wave * R + r;
      if (y >= H) break;  // uniform
      __builtin_amdgcn_sched_barrier(0);  // one row at a time: fewer registers
      const size_t row = ((size_t)y * W + x0) * a.cout + cb;  // of the tile's first pixel
      float f[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) f[v] = acc[r][b][v] + bv[v];
      if (a.out32 && x < W) {
        float *o = a.out32 + row;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = 8 * g + 4 * half;  // cout is a multiple of 8
          if (cb + c < a.cout)
            *reinterpret_cast<float4 *>(o + px * a.cout + c) =
                make_float4(f[4 * g], f[4 * g + 1], f[4 * g + 2], f[4 * g + 3]);
        }
      }
      if (!a.out16) continue;  // uniform
      uint32_t o[8];
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const float u0 = a.relu ? fmaxf(f[2 * v], 0.f) : f[2 * v];
        const float u1 = a.relu ? fmaxf(f[2 * v + 1], 0.f) : f[2 * v + 1];
        o[v] = pack_bf16(u0, u1);
      }
      // groups g and g + 1 of the two halves -> eight consecutive channels per lane:
      // lanes below 32 get 8 g .. 8 g + 7, the others 8 (g + 1) .. 8 (g + 1) + 7
      uint32_t s[8];
#pragma unroll
      for (int g = 0; g < 4; g += 2)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const auto sw2 = __builtin_amdgcn_permlane32_swap(o[2 * g + e], o[2 * g + 2 + e], false,
                                                            false);
          s[2 * g + e] = sw2[0];
          s[2 * g + 2 + e] = sw2[1];
        }
#pragma unroll
      for (int g = 0; g < 4; g += 2) {
        const int c = 8 * g + 8 * half;
        uint4 val = make_uint4(s[2 * g], s[2 * g + 1], s[2 * g + 2], s[2 * g + 3]);
        if (x < W && cb + c < a.cout) {
          if (a.gate) {
            const uint4 m = *reinterpret_cast<const uint4 *>(a.gate + row + px * a.cout + c);
            val = make_uint4(gated(val.x, m.x), gated(val.y, m.y), gated(val.z, m.z),
                             gated(val.w, m.w));
          }
          *reinterpret_cast<uint4 *>(a.out16 + row + px * a.cout + c) = val;
        }
      }
      static_assert(R % 2 == 0, "the pooling pairs rows of one wave");
      {
        if (a.pooled) {  // uniform; H and W are even, and so are y0 and x0
          if (r % 2 == 0) {
#pragma unroll
            for (int v = 0; v < 8; ++v) prev[v] = s[v];
          } else {
#pragma unroll
            for (int v = 0; v < 8; ++v) {
              // (left + right) of the row above plus (left + right) of this row
              auto pairs = [](uint32_t u, int hi) {
                const float me = from_bf16((uint16_t)(hi ? u >> 16 : u & 0xffffu));
                return me + __shfl_xor(me, 1, 64);
              };
              const float lo = pairs(prev[v], 0) + pairs(s[v], 0);
              const float hi = pairs(prev[v], 1) + pairs(s[v], 1);
              s[v] = pack_bf16(0.25f * lo, 0.25f * hi);
            }
            const size_t qp = (size_t)(y >> 1) * (W >> 1) + (x >> 1);
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
              const int c = cb + 8 * g + 8 * half;
              if (x < W && !(x & 1) && c < a.cout)
                *reinterpret_cast<uint4 *>(a.pooled + qp * a.cout + c) =
                    make_uint4(s[2 * g], s[2 * g + 1], s[2 * g + 2], s[2 * g + 3]);
            }
          }
        }
      }
    }
    }
    item += nx;
    if (item >= run1) break;
    lds_sync();  // the next tile's first stage has landed for every wave
  }
}

// The tile of a convolution (rows per wave, blocks of 32 output channels): the
// largest that still gives every CU about two workgroups (480 of 512), because a CU
// holds two and fewer leave the chip idle; else two rows per wave with a third buffer
// (66 x 98 with 384 input and 128 output channels: 26 us with four rows, 18 us with
// two, 21 us with one).
struct ConvTile {
  int r, nb;
};
ConvTile conv_tile(int H, int W, bool thin, int cout) {
  auto groups = [&](int r, int nb) {
    return (int64_t)((W + 31) / 32) * ((H + 4 * r - 1) / (4 * r)) * ((cout + 32 * nb - 1) / (32 * nb));
  };
  if (!thin && cout % 64 == 0 && groups(4, 2) >= 480) return {4, 2};
  return {groups(4, 1) >= 480 ? 4 : 2, 1};
}

hipError_t launch_conv(ConvArgs a, hipStream_t s) {
  // an upsampled input without a skip runs as one with an absent skip
  const bool far = far_rows(a.W, std::max(a.c1, a.c2));
  const bool two = a.c2 > 0 || a.up;
  const bool thin = !two && a.c1 <= 32 && !far;
  const bool gen = a.c1 % 16 != 0 || a.c2 % 16 != 0;
  ConvTile t = conv_tile(a.H, a.W, thin, a.cout);
  if (gen) t.nb = 1;
  if (far) t = {2, 1};
  a.tiles_x = (a.W + 31) / 32;
  a.nco = (a.cout + 32 * t.nb - 1) / (32 * t.nb);
  const int tiles = a.tiles_x * ((a.H + 4 * t.r - 1) / (4 * t.r));
  a.items = thin ? tiles : tiles * a.nco;
  // persistent workgroups, as many as the chip holds at once, in whole rounds over
  // the 8 XCDs
  const int most = 512 / (thin ? a.nco : 1);
  const dim3 grid(std::min(a.items, std::max(8, most & ~7)), thin ? a.nco : 1);
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, a); };
  auto rows = [&](auto twoc, auto genc) {
    constexpr bool TWO = decltype(twoc)::value, GEN = decltype(genc)::value;
    if constexpr (!GEN) {
      if (t.r == 4 && t.nb == 2) return go(k_conv3x3<4, 2, 1, 2, TWO, false>);
    }
    if (t.r == 4) go(k_conv3x3<4, 1, 1, 2, TWO, GEN>);
    else go(k_conv3x3<2, 1, 1, 3, TWO, GEN>);
  };
  using std::bool_constant;
  if (far) {
    go(k_conv3x3<2, 1, 1, 2, true, true, true>);
  } else if (thin) {
    if (t.r == 4) go(k_conv3x3<4, 1, 2, 2, false, false>);
    else go(k_conv3x3<2, 1, 2, 2, false, false>);
  } else if (two) {
    if (gen) rows(bool_constant<true>{}, bool_constant<true>{});
    else rows(bool_constant<true>{}, bool_constant<false>{});
  } else {
    if (gen) rows(bool_constant<false>{}, bool_constant<true>{});
    else rows(bool_constant<false>{}, bool_constant<false>{});
  }
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// Weight gradient: gw[co][t][ci] (tap t = 3 ky + kx) = sum_p gy[p][co]
// in[p + k(t) - 1][ci], a GEMM whose reduction runs over pixels (K = 16 pixels of a
// row per v_mfma_f32_32x32x16 bf16).  A workgroup of four waves takes 32 output x
// 32 input channels, all nine taps, over a share of the tiles of 16 rows x 32
// columns: the tile's dL/dout and its input with a border of one are loaded
// straight into LDS as [row][pixel][32 channels] and read transposed
// (ds_read_b64_tr_b16: a lane gets four consecutive pixels of one channel), so no
// channel-major copy of either exists in memory.  A tap's column shift is an address
// offset; one fragment of an input row serves the three taps ky with three rows of
// dL/dout held in registers.  Wave w takes rows 4 w .. 4 w + 3 of the tile; the four
// waves' sums are added in LDS, the shares' by k_wgrad_reduce, in fixed orders.  The
// bias gradient rides along in the workgroups of the first input channels.
//
// LDS reads bound the products (44 transposed reads for 36 matrix instructions); two
// workgroups per CU cover each other's loads.  Measured at 512 x 512 RGB, all 15
// layers: staging copies, products and reduction 1222 us before (one wave per range
// of pixels, operands from global memory), now 298 us of products and 59 us of
// reduction (k_wgrad_reduce).
// ----------------------------------------------------------------------------
struct WgradArgs {
  const uint16_t *x1, *x2, *gy;
  int c1, c2, up, H, W, cout;
  int tiles_x, tiles, splits;
  float *part, *part_b;
};

constexpr int kWgRows = 16, kWgCols = 32;  // pixels of a tile

// FAR: as the convolution's (a wave's slots lie in one row of dL/dout and in at most
// two of the input).
template <bool FAR>
__global__ __launch_bounds__(256, 2) void k_conv3x3_wgrad(WgradArgs a) {
  constexpr int SC = kWgCols + 2, NI = (kWgRows + 2) * SC * 4, NG = kWgRows * kWgCols * 4;
  constexpr int KI = (NI + 255) / 256, KG = NG / 256;
  static_assert(NG % 256 == 0, "whole rounds of dL/dout slots");
  __shared__ v8s smem[NI + NG];  // input slots, then dL/dout slots; at the end FP32 sums
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ci0 = blockIdx.x * 32, co0 = blockIdx.y * 32, share = blockIdx.z;
  const int H = a.H, W = a.W, cin = a.c1 + a.c2, W1 = a.up ? W >> 1 : W;
  // byte offsets of this thread's slots from the tile's first staged pixel (tiles
  // start at even rows and columns, so they hold for every tile with up too); bit k
  // of from2: slot k's channels are x2's
  uint32_t oi[KI], og[KG], from2 = 0;
#pragma unroll
  for (int k = 0; k < KI; ++k) {
    const int s = tid + 256 * k, i = s >> 2, row = i / SC, col = i - row * SC;
    const int c = ci0 + 8 * (s & 3);
    if (s >= NI || c >= cin) {
      oi[k] = kOutside;
    } else if (c < a.c1) {
      const int q = a.up ? (FAR ? 0 : ((row + 1) >> 1) * W1) + ((col + 1) >> 1)
                         : (FAR ? 0 : row * W) + col;
      oi[k] = 2u * (uint32_t)(q * a.c1 + c);
    } else {
      oi[k] = 2u * (uint32_t)(((FAR ? 0 : row * W) + col) * a.c2 + c - a.c1);
      from2 |= 1u << k;
    }
  }
#pragma unroll
  for (int k = 0; k < KG; ++k) {
    const int s = tid + 256 * k, i = s >> 2, row = i / kWgCols, col = i % kWgCols;
    const int c = co0 + 8 * (s & 3);
    og[k] = c < a.cout ? 2u * (uint32_t)(((FAR ? 0 : row * W) + col) * a.cout + c) : kOutside;
  }
  // this lane's part of a transposed read's address: pixel 8 (lane / 32) + (lane % 16) / 4,
  // channels 16 (lane / 16 % 2) + 4 (lane % 4)
  const int at = (8 * (lane >> 5) + ((lane & 15) >> 2)) * 32 + 16 * ((lane >> 4) & 1) +
                 4 * (lane & 3);
  uint16_t *const si = reinterpret_cast<uint16_t *>(smem) + at;
  uint16_t *const sg = reinterpret_cast<uint16_t *>(smem + NI) + at;
  // eight consecutive pixels of one channel per lane, from pixel index p of a staged array
  auto frag = [](uint16_t *s, int p) {
    typedef __attribute__((address_space(3))) v4s *lds4;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(s + 32 * p));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(s + 32 * (p + 4)));
    return __builtin_bit_cast(v8bf, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  v16f acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
  float bsum = 0.f;
  const int t0 = (int)((int64_t)a.tiles * share / a.splits);
  const int t1 = (int)((int64_t)a.tiles * (share + 1) / a.splits);
  for (int tile = t0; tile < t1; ++tile) {
    const int ty = tile / a.tiles_x, x0 = (tile - ty * a.tiles_x) * kWgCols, y0 = ty * kWgRows;
    const int64_t q2 = (int64_t)(y0 - 1) * W + x0 - 1;
    const int64_t q1 = a.up ? (int64_t)((y0 >> 1) - 1) * W1 + (x0 >> 1) - 1 : q2;
    const auto b1 = buffer_of(a.x1 + q1 * a.c1, kBufferBytes);
    const auto b2 = buffer_of(a.x2 + q2 * a.c2, kBufferBytes);
    const auto bg = buffer_of(a.gy + ((int64_t)y0 * W + x0) * a.cout, kBufferBytes);
    uint32_t out_i = 0, out_g = 0;  // slots whose pixel lies outside the image
    if (y0 == 0 || x0 == 0 || y0 + kWgRows + 1 > H || x0 + kWgCols + 1 > W) {
#pragma unroll
      for (int k = 0; k < KI; ++k) {
        const int i = (tid + 256 * k) >> 2, row = i / SC, col = i - row * SC;
        const bool in = ((uint32_t)(y0 - 1 + row) < (uint32_t)H) &
                        ((uint32_t)(x0 - 1 + col) < (uint32_t)W);
        out_i |= in ? 0u : 1u << k;
      }
#pragma unroll
      for (int k = 0; k < KG; ++k) {
        const int i = (tid + 256 * k) >> 2;
        out_g |= ((y0 + i / kWgCols < H) & (x0 + i % kWgCols < W)) ? 0u : 1u << k;
      }
    }
    lds_sync();  // every wave is done with the previous tile
    v8s *const li = smem + 64 * wave, *const lg = smem + NI + 64 * wave;
#pragma unroll
    for (int k = 0; k < KI; ++k) {
      if (256 * (k + 1) > NI && tid + 256 * k >= NI) continue;
      const uint32_t o = oi[k] | ((out_i << (31 - k)) & kOutside);
      if constexpr (FAR) {
        const int row = (tid + 256 * k) / 4 / SC, r0 = (64 * wave + 256 * k) / 4 / SC;
        if ((from2 >> k) & 1)
          load_two_rows(
              row, r0, [&](int r) { return a.x2 + (q2 + (int64_t)r * W) * a.c2; }, o, 0,
              li + 256 * k);
        else
          load_two_rows(
              row, r0,
              [&](int r) { return a.x1 + (q1 + (int64_t)(a.up ? (r + 1) >> 1 : r) * W1) * a.c1; },
              o, 0, li + 256 * k);
      } else {
        if ((from2 >> k) & 1) load_to_lds(b2, o, 0, li + 256 * k);
        else load_to_lds(b1, o, 0, li + 256 * k);
      }
    }
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      const uint32_t o = og[k] | ((out_g << (31 - k)) & kOutside);
      if constexpr (FAR) {
        const int r = (64 * wave + 256 * k) / 4 / kWgCols;
        load_to_lds(buffer_of(a.gy + ((int64_t)(y0 + r) * W + x0) * a.cout, kBufferBytes), o, 0,
                    lg + 256 * k);
      } else {
        load_to_lds(bg, o, 0, lg + 256 * k);
      }
    }
    wait_vm<0>();
    lds_sync();
#pragma unroll
    for (int xc = 0; xc < kWgCols; xc += 16) {
      v8bf g[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) g[r] = frag(sg, (4 * wave + r) * kWgCols + xc);
      if (blockIdx.x == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int i = 0; i < 8; ++i) bsum += (float)g[r][i];
      }
      v8bf f[2][3];
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) f[0][kx] = frag(si, 4 * wave * SC + xc + kx);
#pragma unroll
      for (int sr = 0; sr < 6; ++sr) {
        // the next row's fragments are read before this row's products
        if (sr + 1 < 6)
#pragma unroll
          for (int kx = 0; kx < 3; ++kx)
            f[(sr + 1) & 1][kx] = frag(si, (4 * wave + sr + 1) * SC + xc + kx);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
          for (int ky = 0; ky < 3; ++ky) {
            const int r = sr - ky;
            if (r < 0 || r > 3) continue;
            acc[3 * ky + kx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[r], f[sr & 1][kx],
                                                                       acc[3 * ky + kx], 0, 0, 0);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // the four waves' sums, three taps at a time: D[row = co][col = ci] of tap t has row
  // 8 (v / 4) + 4 (l / 32) + v % 4 and column l % 32 in register v of lane l
  const int N = 9 * cin;
  float *const red = reinterpret_cast<float *>(smem);
  float *dst = a.part + (size_t)share * a.cout * N;
#pragma unroll
  for (int tb = 0; tb < 9; tb += 3) {
    lds_sync();
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[(wave * 3 + t) * 1024 + 64 * v + lane] = acc[tb + t][v];
    lds_sync();
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = tid + 256 * j, v = i >> 6, l = i & 63;
        const int co = co0 + 8 * (v >> 2) + 4 * (l >> 5) + (v & 3), ci = ci0 + (l & 31);
        const float s = (red[t * 1024 + i] + red[(3 + t) * 1024 + i]) +
                        (red[(6 + t) * 1024 + i] + red[(9 + t) * 1024 + i]);
        if (co < a.cout && ci < cin) dst[(size_t)co * N + (tb + t) * cin + ci] = s;
      }
  }
  if (blockIdx.x == 0) {
    // lanes l and l + 32 hold the two halves of the pixels of channel co0 + l
    bsum += __shfl_down(bsum, 32, 64);
    lds_sync();
    if (lane < 32) red[32 * wave + lane] = bsum;
    lds_sync();
    if (tid < 32 && co0 + tid < a.cout)
      a.part_b[(size_t)share * a.cout + co0 + tid] =
          (red[tid] + red[32 + tid]) + (red[64 + tid] + red[96 + tid]);
  }
}

// Fixed-order sum over many shares (more than kFewShares): a workgroup takes 64 outputs,
// four consecutive ones per lane, with 16 lanes each; lane g of an output adds shares g,
// g + 16, ... in order (sixteen loads in flight), then one lane adds the 16 lane sums in
// order.  Outputs i < len are the weight gradients; the workgroups with i < cout also sum
// the bias partials the same way.  Bound by the reads of the shares.
constexpr int kFewShares = 16;

__device__ __forceinline__ float4 shares_sum(const float *__restrict__ part, int64_t stride,
                                             int splits, int g) {
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k = g; k < splits; k += 256) {
    float4 v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int kk = k + 16 * j;
      v[j] = kk < splits ? *reinterpret_cast<const float4 *>(part + (size_t)kk * stride)
                         : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j)
      s = make_float4(s.x + v[j].x, s.y + v[j].y, s.z + v[j].z, s.w + v[j].w);
  }
  return s;
}

// One layer's shares and where their sums go; its workgroups are blocks
// [first, next job's first).
struct SumJob {
  const float *part, *part_b;
  float *gw, *gb;
  int64_t len;
  int splits, cout;
  unsigned first;
};
constexpr int kSumJobs = 16;
struct SumJobs {
  SumJob job[kSumJobs];
  int count;
};

__device__ __forceinline__ void sum_many(const SumJob &a, unsigned block) {
  __shared__ float4 red[16][17];
  const int o = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int64_t i = (int64_t)block * 64 + 4 * o;  // len and cout are multiples of 4
  const auto total = [&](float *out) {
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int q = 0; q < 16; ++q) {
      const float4 v = red[q][o];
      t = make_float4(t.x + v.x, t.y + v.y, t.z + v.z, t.w + v.w);
    }
    out[0] = t.x; out[1] = t.y; out[2] = t.z; out[3] = t.w;  // (need not be 16-byte aligned)
  };
  if (i < a.len) red[g][o] = shares_sum(a.part + i, a.len, a.splits, g);
  __syncthreads();
  if (g == 0 && i < a.len) total(a.gw + i);
  if (a.gb == nullptr || (int64_t)block * 64 >= a.cout) return;  // uniform per workgroup
  __syncthreads();
  if (i < a.cout) red[g][o] = shares_sum(a.part_b + i, a.cout, a.splits, g);
  __syncthreads();
  if (g == 0 && i < a.cout) total(a.gb + i);
}

// The same for at most kFewShares shares: four consecutive outputs per thread, the
// shares in order; the threads after the weight gradients' take the biases, one each.
// len is a multiple of 4 (cout is one of 8).
__device__ __forceinline__ void sum_few(const SumJob &a, unsigned block) {
  const int64_t i = (int64_t)block * 256 + threadIdx.x, n4 = a.len / 4;
  if (i < n4) {
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int k = 0; k < a.splits; ++k) {
      const float4 v = *reinterpret_cast<const float4 *>(a.part + (size_t)k * a.len + 4 * i);
      s = make_float4(s.x + v.x, s.y + v.y, s.z + v.z, s.w + v.w);
    }
    float *d = a.gw + 4 * i;  // (gw need not be 16-byte aligned)
    d[0] = s.x; d[1] = s.y; d[2] = s.z; d[3] = s.w;
  } else if (a.gb && i < n4 + a.cout) {
    float s = 0.f;
    for (int k = 0; k < a.splits; ++k) s += a.part_b[(size_t)k * a.cout + (i - n4)];
    a.gb[i - n4] = s;
  }
}

// The sums of one or several layers.  A layer's shares are 5 to 19 MB, which a launch of
// its own added in 7.5 us, much of it start and drain: the 15 layers of 512 x 512 RGB
// took 109 us in 15 launches, 85 us in two (those with one float per lane and load), and
// take 59 us in two with four (247 MB: 4.2 TB/s; 5.2 TB/s is a large copy's rate).
__global__ __launch_bounds__(256) void k_wgrad_reduce(SumJobs js) {
  int k = 0;
  while (k + 1 < js.count && blockIdx.x >= js.job[k + 1].first) ++k;
  const SumJob &a = js.job[k];
  const unsigned block = blockIdx.x - a.first;
  if (a.splits <= kFewShares)
    sum_few(a, block);
  else
    sum_many(a, block);
}

__global__ void k_flip(const uint16_t *__restrict__ w, int cout, int cin,
                       uint16_t *__restrict__ wt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;  // over wt: [cin][9][cout]
  if (i >= cout * 9 * cin) return;
  const int co = i % cout, t = (i / cout) % 9, ci = i / (9 * cout);
  wt[i] = w[((size_t)co * 9 + (8 - t)) * cin + ci];  // (ky, kx) -> (2 - ky, 2 - kx)
}

__global__ void k_cast(const float *__restrict__ x, int64_t n, uint16_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = to_bf16(x[i]);
}

__global__ void k_relu_grad(const float *__restrict__ g, const uint16_t *__restrict__ a,
                            int64_t n, uint16_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = to_bf16((a == nullptr || from_bf16(a[i]) > 0.f) ? g[i] : 0.f);
}

// four BF16 values of v, zero where the gate's are not > 0 (no gate: all kept)
__device__ __forceinline__ uint2 gate4(float4 v, const uint16_t *__restrict__ gate, size_t at) {
  uint2 o = make_uint2(pack_bf16(v.x, v.y), pack_bf16(v.z, v.w));
  if (gate) {
    const uint2 m = *reinterpret_cast<const uint2 *>(gate + at);
    o = make_uint2(gated(o.x, m.x), gated(o.y, m.y));
  }
  return o;
}

// the same as k_relu_grad, four elements per thread (16-byte aligned g, 8-byte aligned
// a and out, n a multiple of 4): one load and one store per thread instead of four
// narrow ones (512 x 512 x 24: 12 -> 6 us)
__global__ void k_relu_grad4(const float *__restrict__ g, const uint16_t *__restrict__ a,
                             int64_t n4, uint16_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const float4 v = reinterpret_cast<const float4 *>(g)[i];
  *reinterpret_cast<uint2 *>(out + 4 * i) = gate4(v, a, 4 * (size_t)i);
}

// The upsampling's adjoint and the ReLU below it in one pass, four channels per thread
// (C, stride multiples of 4): the FP32 sum of k_up_adjoint is rounded once and never
// stored.
__global__ void k_up_adjoint_gated(const float *__restrict__ g, int H, int W, int stride, int C,
                                   const uint16_t *__restrict__ gate, uint16_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int Ho = H / 2, Wo = W / 2, C4 = C / 4;
  if (i >= (int64_t)Ho * Wo * C4) return;
  const int c = 4 * (int)(i % C4);
  const int64_t q = i / C4;
  const int y = (int)(q / Wo), x = (int)(q - (int64_t)y * Wo);
  const float *s = g + ((size_t)(2 * y) * W + 2 * x) * stride + c;
  const float4 p0 = *reinterpret_cast<const float4 *>(s);
  const float4 p1 = *reinterpret_cast<const float4 *>(s + stride);
  const float4 p2 = *reinterpret_cast<const float4 *>(s + (size_t)W * stride);
  const float4 p3 = *reinterpret_cast<const float4 *>(s + (size_t)W * stride + stride);
  const float4 v = make_float4((p0.x + p1.x) + (p2.x + p3.x), (p0.y + p1.y) + (p2.y + p3.y),
                               (p0.z + p1.z) + (p2.z + p3.z), (p0.w + p1.w) + (p2.w + p3.w));
  const size_t at = (size_t)q * C + c;
  *reinterpret_cast<uint2 *>(out + at) = gate4(v, gate, at);
}

// k_grad_combine and the ReLU below it in one pass, likewise
__global__ void k_grad_combine_gated(const float *__restrict__ gp, const float *__restrict__ gs,
                                     int stride, int off, int H, int W, int C,
                                     const uint16_t *__restrict__ gate,
                                     uint16_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int C4 = C / 4;
  if (i >= (int64_t)H * W * C4) return;
  const int c = 4 * (int)(i % C4);
  const int64_t q = i / C4;
  const int y = (int)(q / W), x = (int)(q - (int64_t)y * W);
  const float4 p = *reinterpret_cast<const float4 *>(
      gp + ((size_t)(y >> 1) * (W >> 1) + (x >> 1)) * C + c);
  const float4 k = *reinterpret_cast<const float4 *>(gs + (size_t)q * stride + off + c);
  // (the product is rounded before the sum, as in k_grad_combine)
  const float4 v = make_float4(__fadd_rn(__fmul_rn(0.25f, p.x), k.x),
                               __fadd_rn(__fmul_rn(0.25f, p.y), k.y),
                               __fadd_rn(__fmul_rn(0.25f, p.z), k.z),
                               __fadd_rn(__fmul_rn(0.25f, p.w), k.w));
  const size_t at = (size_t)q * C + c;
  *reinterpret_cast<uint2 *>(out + at) = gate4(v, gate, at);
}

__global__ void k_pool2(const uint16_t *__restrict__ x, int H, int W, int C,
                        uint16_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int Ho = H / 2, Wo = W / 2;
  if (i >= (int64_t)Ho * Wo * C) return;
  const int c = (int)(i % C);
  const int64_t q = i / C;
  const int y = (int)(q / Wo), xo = (int)(q - (int64_t)y * Wo);
  const uint16_t *s = x + ((size_t)(2 * y) * W + 2 * xo) * C + c;
  const float v = (from_bf16(s[0]) + from_bf16(s[C])) +
                  (from_bf16(s[(size_t)W * C]) + from_bf16(s[(size_t)W * C + C]));
  out[i] = to_bf16(0.25f * v);
}

__global__ void k_up_adjoint(const float *__restrict__ g, int H, int W, int stride, int C,
                             float *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int Ho = H / 2, Wo = W / 2;
  if (i >= (int64_t)Ho * Wo * C) return;
  const int c = (int)(i % C);
  const int64_t q = i / C;
  const int y = (int)(q / Wo), x = (int)(q - (int64_t)y * Wo);
  const float *s = g + ((size_t)(2 * y) * W + 2 * x) * stride + c;
  out[i] = (s[0] + s[stride]) + (s[(size_t)W * stride] + s[(size_t)W * stride + stride]);
}

__global__ void k_grad_combine(const float *__restrict__ gp, const float *__restrict__ gs,
                               int stride, int off, int H, int W, int C,
                               float *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)H * W * C) return;
  const int c = (int)(i % C);
  const int64_t q = i / C;
  const int y = (int)(q / W), x = (int)(q - (int64_t)y * W);
  float v = 0.f;
  if (gp) v = 0.25f * gp[((size_t)(y >> 1) * (W >> 1) + (x >> 1)) * C + c];
  if (gs) v += gs[(size_t)q * stride + off + c];
  out[i] = v;
}

// lattice point k = i gx + j: centre in FP64, its pixel
__device__ __forceinline__ void lattice_point(int k, int H, int W, int gy, int gx, double &cy,
                                              double &cx, int &iy, int &ix) {
  const int i = k / gx, j = k - i * gx;
  cy = (i + 0.5) * (double)H / gy;
  cx = (j + 0.5) * (double)W / gx;
  iy = (int)floor(cy);
  ix = (int)floor(cx);
}

constexpr double kLogScale0 = 0.69314718055994530942;  // ln 2
constexpr double kAmp0 = 0.5, kOpacity0 = -0.5;

__global__ void k_lattice_gather(const float *__restrict__ net, int H, int W, int gy, int gx,
                                 int C, float *__restrict__ params) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = gy * gx;
  if (k >= n) return;
  double cy, cx;
  int iy, ix;
  lattice_point(k, H, W, gy, gx, cy, cx, iy, ix);
  const float *o = net + ((size_t)iy * W + ix) * 8 * C;
  const double mx = fmin(fmax(cx + (double)o[0], 1e-3), W - 1e-3);
  const double my = fmin(fmax(cy + (double)o[1], 1e-3), H - 1e-3);
  // flat layout: mean_pre [n][2], log_scale [n][2], rotation [n], amplitude [n][C],
  // phase [n][C], opacity_pre [n]; colour c from output block c
  params[2 * k] = (float)atanh(2.0 * mx / W - 1.0);
  params[2 * k + 1] = (float)atanh(2.0 * my / H - 1.0);
  params[2 * (size_t)n + 2 * k] = (float)((double)o[2] + kLogScale0);
  params[2 * (size_t)n + 2 * k + 1] = (float)((double)o[3] + kLogScale0);
  params[4 * (size_t)n + k] = o[4];
  for (int c = 0; c < C; ++c) {
    params[5 * (size_t)n + (size_t)k * C + c] = (float)((double)o[8 * c + 5] + kAmp0);
    params[(size_t)(5 + C) * n + (size_t)k * C + c] = o[8 * c + 6];
  }
  params[(size_t)(5 + 2 * C) * n + k] = (float)((double)o[7] + kOpacity0);
}

__global__ void k_fill0(float *__restrict__ x, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = 0.f;
}

__global__ void k_lattice_scatter(const float *__restrict__ net, const float *__restrict__ g,
                                  int H, int W, int gy, int gx, int C,
                                  float *__restrict__ gnet) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = gy * gx;
  if (k >= n) return;
  double cy, cx;
  int iy, ix;
  lattice_point(k, H, W, gy, gx, cy, cx, iy, ix);
  const float *o = net + ((size_t)iy * W + ix) * 8 * C;
  float *d = gnet + ((size_t)iy * W + ix) * 8 * C;
  const double mx = cx + (double)o[0], my = cy + (double)o[1];
  const double ux = 2.0 * mx / W - 1.0, uy = 2.0 * my / H - 1.0;
  // d atanh(2m / S - 1) / dm = (2 / S) / (1 - u^2); zero where the clip is active
  d[0] = (mx > 1e-3 && mx < W - 1e-3) ? (float)((double)g[2 * k] * (2.0 / W) / (1.0 - ux * ux)) : 0.f;
  d[1] = (my > 1e-3 && my < H - 1e-3) ? (float)((double)g[2 * k + 1] * (2.0 / H) / (1.0 - uy * uy)) : 0.f;
  d[2] = g[2 * (size_t)n + 2 * k];
  d[3] = g[2 * (size_t)n + 2 * k + 1];
  d[4] = g[4 * (size_t)n + k];
  for (int c = 0; c < C; ++c) {
    d[8 * c + 5] = g[5 * (size_t)n + (size_t)k * C + c];
    d[8 * c + 6] = g[(size_t)(5 + C) * n + (size_t)k * C + c];
  }
  d[7] = g[(size_t)(5 + 2 * C) * n + k];
}

__global__ void k_sqrt_field(const float *__restrict__ t, int64_t n, float2 *__restrict__ f) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) f[i] = make_float2(sqrtf(fmaxf(t[i], 0.f)), 0.f);
}

// planar [C][n] inputs -> [n][8 C]: block c of pixel i from colour c
__global__ void k_features(const float *__restrict__ t, const float2 *__restrict__ b, int64_t n,
                           int C, uint16_t *__restrict__ out) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n * C) return;
  const int c = (int)(j / n);
  const int64_t i = j - (int64_t)c * n;
  const float v = t[j];
  const float2 u = b[j];
  uint16_t *o = out + (i * C + c) * 8;
  o[0] = to_bf16(v);
  o[1] = to_bf16(sqrtf(fmaxf(v, 0.f)));
  o[2] = to_bf16(u.x);
  o[3] = to_bf16(u.y);
  o[4] = to_bf16(sqrtf(u.x * u.x + u.y * u.y));
  o[5] = o[6] = o[7] = 0;
}

unsigned blocks_of(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }


// the split of the weight-gradient GEMM: about two workgroups per CU over the tiles
// of an image, and the byte offsets of its workspace parts
struct WgPlan {
  int tiles_x, tiles, splits;
  size_t part, part_b, bytes;
  size_t shares_b, shares;  // the shares alone: the bias's offset, bytes
};
size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }
WgPlan wgrad_plan(int H, int W, int cin, int cout) {
  WgPlan p;
  p.tiles_x = (W + kWgCols - 1) / kWgCols;
  p.tiles = p.tiles_x * ((H + kWgRows - 1) / kWgRows);
  const int pairs = ((cin + 31) / 32) * ((cout + 31) / 32);
  // The workspace's size is an interface callers allocate by: room for the partials
  // of up to 512 / pairs shares of whole 16-pixel row chunks and for channel-major
  // copies of both operands.  The copies are no longer made and the shares are of
  // tiles, never more of them than that room holds.
  const size_t Wr = (W + 15) & ~15;
  const int chunks = (int)(H * (Wr / 16));
  const int want = std::max(1, std::min(chunks, (512 + pairs - 1) / pairs));
  const int cps = (chunks + want - 1) / want, room = (chunks + cps - 1) / cps;
  p.splits = std::max(1, std::min(p.tiles, room));
  const size_t len = (size_t)cout * 9 * cin;
  p.part = 0;
  p.part_b = round256(room * len * sizeof(float));
  p.shares_b = round256((size_t)p.splits * len * sizeof(float));
  p.shares = p.shares_b + round256((size_t)p.splits * cout * sizeof(float));
  p.bytes = p.part_b + round256((size_t)room * cout * sizeof(float)) +
            round256((size_t)cout * H * Wr * sizeof(uint16_t)) +
            round256((size_t)3 * cin * (H + 2) * Wr * sizeof(uint16_t));
  return p;
}

}  // namespace
}  // namespace cgh

using namespace cgh;

#define NET_CHECK(cond, ...) \
  do {                       \
    if (!(cond)) return report(CGH_ERR_INVALID_ARG, __VA_ARGS__); \
  } while (0)
#define NET_LAUNCHED(where)                                                           \
  do {                                                                                \
    const hipError_t e_ = hipGetLastError();                                          \
    if (e_ != hipSuccess) return report(CGH_ERR_DEVICE, "%s: %s", where, hipGetErrorString(e_)); \
  } while (0)

static cgh_status check_conv_shape(const cgh_bf16 *x1, int32_t c1, int32_t up,
                                   const cgh_bf16 *x2, int32_t c2, int32_t H, int32_t W) {
  NET_CHECK(x1 && c1 > 0 && c1 % 8 == 0, "x1 NULL or c1 = %d not a positive multiple of 8", c1);
  NET_CHECK((x2 == nullptr) == (c2 == 0) && c2 >= 0 && c2 % 8 == 0,
            "x2 / c2 = %d: both absent, or c2 a positive multiple of 8", c2);
  NET_CHECK(H >= 1 && W >= 1 && (int64_t)H * W < (1LL << 31), "bad size %d x %d", H, W);
  NET_CHECK(!up || (H % 2 == 0 && W % 2 == 0), "upsampled input needs even H, W");
  NET_CHECK(al16(x1) && al16(x2), "inputs must be 16-byte aligned");
  return CGH_OK;
}

extern "C" {

cgh_status cgh_net_conv3x3(const cgh_bf16 *x1, int32_t c1, int32_t up, const cgh_bf16 *x2,
                           int32_t c2, int32_t H, int32_t W, const cgh_bf16 *w,
                           const float *bias, int32_t cout, int32_t relu, float *out32,
                           cgh_bf16 *out16, void *stream) {
  const cgh_status st = check_conv_shape(x1, c1, up, x2, c2, H, W);
  if (st != CGH_OK) return st;
  NET_CHECK(w && cout > 0 && cout % 8 == 0, "w NULL or cout = %d not a multiple of 8", cout);
  NET_CHECK(out32 || out16, "no output");
  NET_CHECK(al16(w) && al16(out32) && al16(out16), "w, out32 and out16 must be 16-byte aligned");
  ConvArgs a{x1, x2, w, bias, c1, c2, up, H, W, cout, relu, out32, out16, nullptr, nullptr, 0};
  const hipError_t e = launch_conv(a, (hipStream_t)stream);
  if (e != hipSuccess) return report(CGH_ERR_DEVICE, "conv3x3: %s", hipGetErrorString(e));
  return CGH_OK;
}

cgh_status cgh_net_conv3x3_pool2(const cgh_bf16 *x1, int32_t c1, int32_t up, const cgh_bf16 *x2,
                                 int32_t c2, int32_t H, int32_t W, const cgh_bf16 *w,
                                 const float *bias, int32_t cout, int32_t relu, cgh_bf16 *out16,
                                 cgh_bf16 *pooled, void *stream) {
  const cgh_status st = check_conv_shape(x1, c1, up, x2, c2, H, W);
  if (st != CGH_OK) return st;
  NET_CHECK(w && cout > 0 && cout % 8 == 0, "w NULL or cout = %d not a multiple of 8", cout);
  NET_CHECK(out16 && pooled, "no output");
  NET_CHECK(H % 2 == 0 && W % 2 == 0, "pooling needs even H, W");
  NET_CHECK(al16(w) && al16(out16) && al16(pooled), "w, out16 and pooled must be 16-byte aligned");
  ConvArgs a{x1, x2, w, bias, c1, c2, up, H, W, cout, relu, nullptr, out16, pooled, nullptr};
  const hipError_t e = launch_conv(a, (hipStream_t)stream);
  if (e != hipSuccess) return report(CGH_ERR_DEVICE, "conv3x3: %s", hipGetErrorString(e));
  return CGH_OK;
}

cgh_status cgh_net_conv3x3_gated(const cgh_bf16 *gy, int32_t cout, int32_t H, int32_t W,
                                 const cgh_bf16 *w_t, int32_t cin, const cgh_bf16 *gate,
                                 cgh_bf16 *out16, void *stream) {
  const cgh_status st = check_conv_shape(gy, cout, 0, nullptr, 0, H, W);
  if (st != CGH_OK) return st;
  NET_CHECK(w_t && cin > 0 && cin % 8 == 0, "w_t NULL or cin = %d not a multiple of 8", cin);
  NET_CHECK(gate && out16, "gate/out16 is NULL");
  NET_CHECK(al16(w_t) && al16(gate) && al16(out16), "w_t, gate and out16 must be 16-byte aligned");
  ConvArgs a{gy, nullptr, w_t, nullptr, cout, 0, 0, H, W, cin, 0, nullptr, out16, nullptr, gate};
  const hipError_t e = launch_conv(a, (hipStream_t)stream);
  if (e != hipSuccess) return report(CGH_ERR_DEVICE, "conv3x3: %s", hipGetErrorString(e));
  return CGH_OK;
}

cgh_status cgh_net_flip_weights(const cgh_bf16 *w, int32_t cout, int32_t cin, cgh_bf16 *w_t,
                                void *stream) {
  NET_CHECK(w && w_t && cout > 0 && cin > 0, "bad arguments");
  hipLaunchKernelGGL(k_flip, dim3(blocks_of((int64_t)cout * 9 * cin, 256)), dim3(256), 0,
                     (hipStream_t)stream, w, cout, cin, w_t);
  NET_LAUNCHED("flip_weights");
  return CGH_OK;
}

size_t cgh_net_wgrad_workspace(int32_t H, int32_t W, int32_t cin, int32_t cout) {
  if (H < 1 || W < 1 || cin < 1 || cout < 1) return 0;
  return wgrad_plan(H, W, cin, cout).bytes;
}

// the products of one layer's weight gradient: a share of the sums per workgroup plane
static cgh_status wgrad_shares(const cgh_bf16 *x1, int c1, int up, const cgh_bf16 *x2, int c2,
                               int H, int W, const cgh_bf16 *gy, int cout, const WgPlan &pl,
                               float *part, float *part_b, hipStream_t s) {
  const int cin = c1 + c2;
  const WgradArgs wa{x1, x2, gy,   c1,         c2,       up,        H,
                     W,  cout, pl.tiles_x, pl.tiles, pl.splits, part, part_b};
  const auto kern = far_rows(W, std::max(std::max(c1, c2), cout)) ? k_conv3x3_wgrad<true>
                                                                  : k_conv3x3_wgrad<false>;
  hipLaunchKernelGGL(kern, dim3((cin + 31) / 32, (cout + 31) / 32, pl.splits), dim3(256), 0, s,
                     wa);
  NET_LAUNCHED("conv3x3_wgrad");
  return CGH_OK;
}

// appends a layer's sums to js; returns the workgroups so far
static unsigned add_sums(SumJobs &js, unsigned blocks, const float *part, const float *part_b,
                         int splits, int cin, int cout, float *gw, float *gb) {
  const int64_t len = (int64_t)cout * 9 * cin;
  js.job[js.count++] = SumJob{part, part_b, gw, gb, len, splits, cout, blocks};
  return blocks + (splits <= kFewShares ? blocks_of(len / 4 + cout, 256)
                                        : blocks_of(std::max<int64_t>(len, cout), 64));
}

cgh_status cgh_net_conv3x3_wgrad(const cgh_bf16 *x1, int32_t c1, int32_t up, const cgh_bf16 *x2,
                                 int32_t c2, int32_t H, int32_t W, const cgh_bf16 *gy,
                                 int32_t cout, float *gw, float *gb, void *workspace,
                                 size_t workspace_bytes, void *stream) {
  cgh_status st = check_conv_shape(x1, c1, up, x2, c2, H, W);
  if (st != CGH_OK) return st;
  NET_CHECK(gy && gw && cout > 0 && cout % 8 == 0, "gy/gw NULL or cout = %d not a multiple of 8",
            cout);
  const int cin = c1 + c2;
  const WgPlan pl = wgrad_plan(H, W, cin, cout);
  if (!workspace || workspace_bytes < pl.bytes)
    return report(CGH_ERR_WORKSPACE, "wgrad workspace has %zu bytes, needs %zu", workspace_bytes,
                  pl.bytes);
  NET_CHECK(al16(workspace) && al16(gy), "workspace and gy must be 16-byte aligned");
  float *part = (float *)((char *)workspace + pl.part);
  float *part_b = (float *)((char *)workspace + pl.part_b);
  hipStream_t s = (hipStream_t)stream;
  st = wgrad_shares(x1, c1, up, x2, c2, H, W, gy, cout, pl, part, part_b, s);
  if (st != CGH_OK) return st;
  SumJobs js{};
  const unsigned blocks = add_sums(js, 0, part, part_b, pl.splits, cin, cout, gw, gb);
  hipLaunchKernelGGL(k_wgrad_reduce, dim3(blocks), dim3(256), 0, s, js);
  NET_LAUNCHED("wgrad_reduce");
  return CGH_OK;
}

size_t cgh_net_wgrad_shares_bytes(int32_t H, int32_t W, int32_t cin, int32_t cout) {
  if (H < 1 || W < 1 || cin < 1 || cout < 1) return 0;
  return wgrad_plan(H, W, cin, cout).shares;
}

cgh_status cgh_net_wgrad_shares(const cgh_bf16 *x1, int32_t c1, int32_t up, const cgh_bf16 *x2,
                                int32_t c2, int32_t H, int32_t W, const cgh_bf16 *gy,
                                int32_t cout, void *shares, size_t shares_bytes, void *stream) {
  const cgh_status st = check_conv_shape(x1, c1, up, x2, c2, H, W);
  if (st != CGH_OK) return st;
  NET_CHECK(gy && cout > 0 && cout % 8 == 0, "gy NULL or cout = %d not a multiple of 8", cout);
  const WgPlan pl = wgrad_plan(H, W, c1 + c2, cout);
  if (!shares || shares_bytes < pl.shares)
    return report(CGH_ERR_WORKSPACE, "the shares have %zu bytes, need %zu", shares_bytes,
                  pl.shares);
  NET_CHECK(al16(shares) && al16(gy), "shares and gy must be 16-byte aligned");
  return wgrad_shares(x1, c1, up, x2, c2, H, W, gy, cout, pl, (float *)shares,
                      (float *)((char *)shares + pl.shares_b), (hipStream_t)stream);
}

cgh_status cgh_net_wgrad_sums(const cgh_net_wgrad_job *jobs, int32_t count, void *stream) {
  NET_CHECK(count >= 0 && (count == 0 || jobs), "bad arguments");
  for (int k = 0; k < count; ++k) {
    const cgh_net_wgrad_job &j = jobs[k];
    NET_CHECK(j.H > 0 && j.W > 0 && j.cin > 0 && j.cin % 8 == 0 && j.cout > 0 && j.cout % 8 == 0,
              "job %d: bad shape", k);
    NET_CHECK(j.shares && j.gw && al16(j.shares), "job %d: shares/gw NULL or misaligned", k);
  }
  for (int k = 0; k < count;) {
    SumJobs js{};
    unsigned blocks = 0;
    for (; k < count && js.count < kSumJobs; ++k) {
      const cgh_net_wgrad_job &j = jobs[k];
      const WgPlan pl = wgrad_plan(j.H, j.W, j.cin, j.cout);
      blocks = add_sums(js, blocks, (const float *)j.shares,
                        (const float *)((const char *)j.shares + pl.shares_b), pl.splits, j.cin,
                        j.cout, j.gw, j.gb);
    }
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(blocks), dim3(256), 0, (hipStream_t)stream, js);
    NET_LAUNCHED("wgrad_reduce");
  }
  return CGH_OK;
}

cgh_status cgh_net_cast_bf16(const float *x, int64_t count, cgh_bf16 *out, void *stream) {
  NET_CHECK(count >= 0 && (count == 0 || (x && out)), "bad arguments");
  if (count == 0) return CGH_OK;
  hipLaunchKernelGGL(k_cast, dim3(blocks_of(count, 256)), dim3(256), 0, (hipStream_t)stream, x,
                     count, out);
  NET_LAUNCHED("cast_bf16");
  return CGH_OK;
}

cgh_status cgh_net_relu_grad(const float *g, const cgh_bf16 *a, int64_t count, cgh_bf16 *out,
                             void *stream) {
  NET_CHECK(count >= 0 && (count == 0 || (g && out)), "bad arguments");
  if (count == 0) return CGH_OK;
  if (al16(g) && al16(a) && al16(out) && count % 4 == 0) {
    hipLaunchKernelGGL(k_relu_grad4, dim3(blocks_of(count / 4, 256)), dim3(256), 0,
                       (hipStream_t)stream, g, a, count / 4, out);
    NET_LAUNCHED("relu_grad");
    return CGH_OK;
  }
  hipLaunchKernelGGL(k_relu_grad, dim3(blocks_of(count, 256)), dim3(256), 0,
                     (hipStream_t)stream, g, a, count, out);
  NET_LAUNCHED("relu_grad");
  return CGH_OK;
}

cgh_status cgh_net_pool2(const cgh_bf16 *x, int32_t H, int32_t W, int32_t C, cgh_bf16 *out,
                         void *stream) {
  NET_CHECK(x && out && H >= 2 && W >= 2 && H % 2 == 0 && W % 2 == 0 && C > 0, "bad arguments");
  hipLaunchKernelGGL(k_pool2, dim3(blocks_of((int64_t)(H / 2) * (W / 2) * C, 256)), dim3(256), 0,
                     (hipStream_t)stream, x, H, W, C, out);
  NET_LAUNCHED("pool2");
  return CGH_OK;
}

cgh_status cgh_net_up_adjoint(const float *g, int32_t H, int32_t W, int32_t stride, int32_t C,
                              float *out, void *stream) {
  NET_CHECK(g && out && H % 2 == 0 && W % 2 == 0 && H >= 2 && W >= 2 && C > 0 && stride >= C,
            "bad arguments");
  hipLaunchKernelGGL(k_up_adjoint, dim3(blocks_of((int64_t)(H / 2) * (W / 2) * C, 256)),
                     dim3(256), 0, (hipStream_t)stream, g, H, W, stride, C, out);
  NET_LAUNCHED("up_adjoint");
  return CGH_OK;
}

cgh_status cgh_net_grad_combine(const float *gp, const float *gs, int32_t stride, int32_t off,
                                int32_t H, int32_t W, int32_t C, float *out, void *stream) {
  NET_CHECK(out && H >= 1 && W >= 1 && C > 0, "bad arguments");
  NET_CHECK(!gp || (H % 2 == 0 && W % 2 == 0), "pooled gradient needs even H, W");
  NET_CHECK(!gs || (off >= 0 && off + C <= stride), "skip slice outside its rows");
  hipLaunchKernelGGL(k_grad_combine, dim3(blocks_of((int64_t)H * W * C, 256)), dim3(256), 0,
                     (hipStream_t)stream, gp, gs, stride, off, H, W, C, out);
  NET_LAUNCHED("grad_combine");
  return CGH_OK;
}

cgh_status cgh_net_up_adjoint_gated(const float *g, int32_t H, int32_t W, int32_t stride,
                                    int32_t C, const cgh_bf16 *gate, cgh_bf16 *out,
                                    void *stream) {
  NET_CHECK(g && gate && out && H % 2 == 0 && W % 2 == 0 && H >= 2 && W >= 2 && C > 0 &&
                stride >= C && C % 8 == 0 && stride % 8 == 0, "bad arguments");
  NET_CHECK(al16(g) && al16(gate) && al16(out), "buffers must be 16-byte aligned");
  hipLaunchKernelGGL(k_up_adjoint_gated,
                     dim3(blocks_of((int64_t)(H / 2) * (W / 2) * (C / 4), 256)), dim3(256), 0,
                     (hipStream_t)stream, g, H, W, stride, C, gate, out);
  NET_LAUNCHED("up_adjoint_gated");
  return CGH_OK;
}

cgh_status cgh_net_grad_combine_gated(const float *gp, const float *gs, int32_t stride,
                                      int32_t off, int32_t H, int32_t W, int32_t C,
                                      const cgh_bf16 *gate, cgh_bf16 *out, void *stream) {
  NET_CHECK(gp && gs && gate && out && H >= 2 && W >= 2 && H % 2 == 0 && W % 2 == 0 && C > 0 &&
                C % 8 == 0, "bad arguments");
  NET_CHECK(off >= 0 && off + C <= stride && off % 8 == 0 && stride % 8 == 0,
            "skip slice outside its rows");
  NET_CHECK(al16(gp) && al16(gs) && al16(gate) && al16(out), "buffers must be 16-byte aligned");
  hipLaunchKernelGGL(k_grad_combine_gated, dim3(blocks_of((int64_t)H * W * (C / 4), 256)),
                     dim3(256), 0, (hipStream_t)stream, gp, gs, stride, off, H, W, C, gate, out);
  NET_LAUNCHED("grad_combine_gated");
  return CGH_OK;
}

cgh_status cgh_net_lattice_gather(const float *net, int32_t H, int32_t W, int32_t gy,
                                  int32_t gx, int32_t C, float *params, void *stream) {
  NET_CHECK(net && params && gy >= 1 && gx >= 1 && gy <= H && gx <= W && C >= 1 &&
                C <= CGH_MAX_CHANNELS, "bad arguments");
  hipLaunchKernelGGL(k_lattice_gather, dim3(blocks_of((int64_t)gy * gx, 256)), dim3(256), 0,
                     (hipStream_t)stream, net, H, W, gy, gx, C, params);
  NET_LAUNCHED("lattice_gather");
  return CGH_OK;
}

cgh_status cgh_net_lattice_scatter(const float *net, const float *grads, int32_t H, int32_t W,
                                   int32_t gy, int32_t gx, int32_t C, float *g_net,
                                   void *stream) {
  NET_CHECK(net && grads && g_net && gy >= 1 && gx >= 1 && gy <= H && gx <= W && C >= 1 &&
                C <= CGH_MAX_CHANNELS, "bad arguments");
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_fill0, dim3(blocks_of((int64_t)H * W * 8 * C, 256)), dim3(256), 0, s,
                     g_net, (int64_t)H * W * 8 * C);
  hipLaunchKernelGGL(k_lattice_scatter, dim3(blocks_of((int64_t)gy * gx, 256)), dim3(256), 0, s,
                     net, grads, H, W, gy, gx, C, g_net);
  NET_LAUNCHED("lattice_scatter");
  return CGH_OK;
}

cgh_status cgh_net_sqrt_field(const float *target, int64_t count, cgh_c64 *field,
                              void *stream) {
  NET_CHECK(target && field && count > 0, "bad arguments");
  hipLaunchKernelGGL(k_sqrt_field, dim3(blocks_of(count, 256)), dim3(256), 0,
                     (hipStream_t)stream, target, count, reinterpret_cast<float2 *>(field));
  NET_LAUNCHED("sqrt_field");
  return CGH_OK;
}

cgh_status cgh_net_features(const float *target, const cgh_c64 *back, int64_t count, int32_t C,
                            cgh_bf16 *out, void *stream) {
  NET_CHECK(target && back && out && count > 0 && C >= 1 && C <= CGH_MAX_CHANNELS,
            "bad arguments");
  hipLaunchKernelGGL(k_features, dim3(blocks_of(count * C, 256)), dim3(256), 0,
                     (hipStream_t)stream, target, reinterpret_cast<const float2 *>(back), count, C,
                     out);
  NET_LAUNCHED("features");
  return CGH_OK;
}

}  // extern "C"
