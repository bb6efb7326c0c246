// Band-limited angular-spectrum propagation on gfx950: mixed-radix Stockham
// FFTs held in LDS, the transfer-function multiply fused into the column
// pass, and intensity / MSE / adjoint seed fused into the middle row pass.
//
// The propagation of one channel is u = crop(IFFT2(H . FFT2(pad(U0))))
// (Sec. 2; Alg. 1 ZeroPad + MultiPlanePropagate).  Because FFT2 -> H -> IFFT2
// is a circular convolution, padding the field at the start of each row and
// column (instead of centring it) and cropping the same leading window gives
// the same u; the kernels use that placement so the zero padding never exists
// in memory:
//   F1  row FFT:    U0 [C][H][W] -> S (rows zero-extended to Wp)
//   F2  column pass on S: FFT over Hp (zero-extended), x H/(Hp Wp), IFFT, keep H rows
//   F3  row pass:   IFFT, crop W -> u; I = |u|^2; loss; g = dL/du; zero-extend; FFT
//   B1  column pass with conj(H) (the adjoint, supplementary BLASM Backward Pass)
//   B2  row IFFT, crop W -> dL/dU0
// S is column-tiled: [C][ceil(Wp/8)][H][8] complex, so a column workgroup
// reads and writes pieces of one contiguous block.
//
// Lengths that split into chains run the kernels of fft_chain.h (four or two chains per
// row or column, plans compiled for each length).  The kernels below are for the other
// shapes: more samples than half the padded length, odd padded lengths, chains shorter or
// longer than those tables.  There a row workgroup takes two rows (or four), whose 64-byte
// pieces of a tile make whole 128-byte lines.
//
// Column pass there for even Hp = 2M: the input occupies rows [0, H) and only rows
// [0, H) of the output are kept, so the Hp-point transform splits into two
// M-point chains (radix-2 first and last stages done in registers):
//   even chain: FFT_M(x[n] + x[n+M])             -> x H(ky = 2m)   -> IFFT_M -> e
//   odd chain:  FFT_M((x[n] - x[n+M]) w^n)       -> x H(ky = 2m+1) -> IFFT_M -> o
//   y[n] = e[n] + w^-n o[n],  y[n+M] = e[n] - w^-n o[n],   w = exp(-2 pi i / Hp)
// which halves the LDS footprint of a column block.
#include <cmath>

#include "fft_chain.h"

namespace cgh {

// ----------------------------------------------------------------------------
// Twiddles w^e = exp(-2 pi i e / n) from a two-level table kept in LDS:
// hi[j] = w^{64 j} (j <= n/64), lo[j] = w^j (j < 64); w^e = hi[e >> 6] lo[e & 63].
// The global copy of a table is kTwEntries float2: hi at [0, 129), lo at [129, 193).
// ----------------------------------------------------------------------------
constexpr int kTwHi = 129;
constexpr int kTwEntries = kTwHi + 64;

struct TwLds {
  float2 hi[kTwHi];
  float2 lo[64];
};

__device__ __forceinline__ float2 tw_at(const TwLds &t, int e) {
  return cmul(t.hi[e >> 6], t.lo[e & 63]);
}

template <int T>
__device__ __forceinline__ void load_tw(TwLds &dst, const float2 *__restrict__ src, int tid) {
  for (int i = tid; i < kTwEntries; i += T) {
    if (i < kTwHi) dst.hi[i] = src[i];
    else dst.lo[i - kTwHi] = src[i];
  }
}

// ----------------------------------------------------------------------------
// One Stockham stage over B interleaved transforms held in LDS:
// element (index r, transform b) lives at buf[r * B + b].  Butterfly j of
// transform b reads r = j + q n/R (q < R), twiddles by exp(DIR 2 pi i q k /
// (Ns R)) with k = j mod Ns, and writes to (j / Ns) Ns R + k + q Ns.  All
// reads of a stage complete (barrier) before its writes, so one buffer
// suffices; each thread keeps its butterflies in registers across the barrier.
// ----------------------------------------------------------------------------
template <int R, int DIR, int B, int T, int MAXN>
__device__ __forceinline__ void fft_stage(float2 *__restrict__ buf, int n, int Ns,
                                          uint32_t magic, int tws, const TwLds &tw,
                                          int tid) {
  constexpr int MAXIT = (B * ((MAXN + R - 1) / R) + T - 1) / T;
  const int nb = n / R;
  const int items = nb * B;
  float2 v[MAXIT][R];
#pragma unroll
  for (int it = 0; it < MAXIT; ++it) {
    const int i = tid + it * T;
    if (i < items) {
      const int b = i % B, j = i / B;
#pragma unroll
      for (int q = 0; q < R; ++q) v[it][q] = buf[(j + q * nb) * B + b];
      if (Ns > 1) {
        const int grp = (int)__umulhi((uint32_t)j, magic);
        float2 w1 = tw_at(tw, (j - grp * Ns) * tws);
        if (DIR > 0) w1.y = -w1.y;
        float2 w = w1;
        v[it][1] = cmul(v[it][1], w);
#pragma unroll
        for (int q = 2; q < R; ++q) {
          w = cmul(w, w1);
          v[it][q] = cmul(v[it][q], w);
        }
      }
      Dft<R, DIR>::run(v[it]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < MAXIT; ++it) {
    const int i = tid + it * T;
    if (i < items) {
      const int b = i % B, j = i / B;
      const int grp = Ns > 1 ? (int)__umulhi((uint32_t)j, magic) : j;
      const int base = grp * Ns * R + (j - grp * Ns);
#pragma unroll
      for (int q = 0; q < R; ++q) buf[(base + q * Ns) * B + b] = v[it][q];
    }
  }
  __syncthreads();
}

template <int DIR, int B, int T, int MAXN>
__device__ void fft_lds(float2 *__restrict__ buf, const FftPlan &p, const TwLds &tw, int tid) {
  for (int s = 0; s < p.nstages; ++s) {
    const int r = p.radix[s];
    // An opaque per-stage copy of the thread index: without it the compiler
    // hoists every radix variant's per-butterfly index math out of this loop
    // and keeps it all live (about 2x the registers).
    int ts = tid;
    asm volatile("" : "+v"(ts));
    if (r == 8)
      fft_stage<8, DIR, B, T, MAXN>(buf, p.n, p.ns[s], p.magic[s], p.tws[s], tw, ts);
    else if (r == 4)
      fft_stage<4, DIR, B, T, MAXN>(buf, p.n, p.ns[s], p.magic[s], p.tws[s], tw, ts);
    else if (r == 3)
      fft_stage<3, DIR, B, T, MAXN>(buf, p.n, p.ns[s], p.magic[s], p.tws[s], tw, ts);
    else if (r == 5)
      fft_stage<5, DIR, B, T, MAXN>(buf, p.n, p.ns[s], p.magic[s], p.tws[s], tw, ts);
    else
      fft_stage<2, DIR, B, T, MAXN>(buf, p.n, p.ns[s], p.magic[s], p.tws[s], tw, ts);
  }
}

// ----------------------------------------------------------------------------
// Host-side planning
// ----------------------------------------------------------------------------
bool smooth235(int n) {
  if (n < 1) return false;
  for (int p : {2, 3, 5})
    while (n % p == 0) n /= p;
  return n == 1;
}

bool make_plan(int n, FftPlan *plan) {
  if (!smooth235(n) || n > kMaxFft) return false;
  int rad[kMaxStages];
  int ns = 0, m = n, twos = 0;
  while (m % 2 == 0) { m /= 2; ++twos; }
  // powers of two as radix 8 where possible, leftovers as 4 (or one 2)
  while (twos >= 3 && twos != 4) { rad[ns++] = 8; twos -= 3; }
  while (twos >= 2) { rad[ns++] = 4; twos -= 2; }
  if (twos == 1) rad[ns++] = 2;
  while (m % 3 == 0) { rad[ns++] = 3; m /= 3; }
  while (m % 5 == 0) { rad[ns++] = 5; m /= 5; }
  if (ns > kMaxStages) return false;
  plan->n = n;
  plan->nstages = ns;
  int prod = 1;
  for (int s = 0; s < ns; ++s) {
    plan->radix[s] = rad[s];
    plan->ns[s] = prod;
    plan->magic[s] = prod > 1 ? (uint32_t)((((uint64_t)1 << 32) + prod - 1) / prod) : 0u;
    plan->tws[s] = n / (prod * rad[s]);
    prod *= rad[s];
  }
  for (int s = ns; s < kMaxStages; ++s) {
    plan->radix[s] = 0; plan->ns[s] = 0; plan->magic[s] = 0; plan->tws[s] = 0;
  }
  return true;
}

bool col_supported(int Hp) {
  if (Hp % 2 == 0) return Hp / 2 <= kColHalfMax;
  return Hp <= kColFullMax;
}

// ----------------------------------------------------------------------------
// Tables (FP64 on the device, rounded to FP32 once)
// ----------------------------------------------------------------------------
__global__ void k_twiddles(float2 *tw, int n) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= kTwEntries) return;
  const long e = j < kTwHi ? (64L * j) % n : (long)(j - kTwHi) % n;
  double s, c;
  sincospi(2.0 * (double)e / (double)n, &s, &c);
  tw[j] = make_float2((float)c, (float)(-s));  // exp(-2 pi i e / n)
}

hipError_t launch_build_twiddles(float2 *tw, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_twiddles, dim3(1), dim3(256), 0, s, tw, n);
  return hipGetLastError();
}

// full table tw[e] = exp(-2 pi i e / n), e < n
__global__ void k_twiddles_full(float2 *tw, int n) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  double s, c;
  sincospi(2.0 * (double)e / (double)n, &s, &c);
  tw[e] = make_float2((float)c, (float)(-s));
}

hipError_t launch_build_twiddles_full(float2 *tw, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_twiddles_full, dim3((n + 255) / 256), dim3(256), 0, s, tw, n);
  return hipGetLastError();
}

// Band-limited angular-spectrum transfer function (Sec. 2; supplementary
// "Spatial Frequency Computation", "Bandlimit Computation", "Transfer Function
// Evaluation"), quarter table indexed by |fx| = qx / (Wp dx), |fy| = qy / (Hp dx).
// L_x, L_y are the extents of the padded grid.  Evanescent frequencies get 0.
// aperture > 0: the circular aperture of Alg. 3, centred on the zero frequency
// (bins with qx^2 + qy^2 >= aperture^2 are zeroed).
//
// One table entry per thread.  out: row-major [Hq][Wq] (x fastest over the
// threads); out_t: column-major [Wq][Hq] (y fastest), times t_scale (the
// 1 / (Hp Wp) of the inverse transform, applied in FP64).  The chain column pass
// reads only the column-major table, the other column kernels only the
// row-major one, so a context holds one of them.  optics: where lambda and z are
// kept on the device (2 doubles): written from the arguments, or, with `held`, read
// instead of them.
//
// held (cgh_get_transfer): the column-major table that the column pass reads.  Its
// entries carry t_scale, which cannot be divided out to the last bit, so an entry is
// worked out anew from the optics that are current in stream order and returned where
// `held` has its scaled value; elsewhere `held`'s own value, divided by t_scale, is.
__global__ void k_transfer(float2 *out, float2 *out_t, double t_scale, int Hq, int Wq, int Hp,
                           int Wp, double pitch, double lambda, double z, double aperture,
                           double *optics, const float2 *held) {
  const int fast = blockIdx.x * blockDim.x + threadIdx.x, slow = blockIdx.y;
  const int qx = out_t ? slow : fast, qy = out_t ? fast : slow;
  if (held) {
    lambda = optics[0];
    z = optics[1];
  } else if (optics && fast == 0 && slow == 0) {
    optics[0] = lambda;
    optics[1] = z;
  }
  if (qx >= Wq || qy >= Hq) return;
  const double Lx = Wp * pitch, Ly = Hp * pitch;
  const double fx = qx / Lx, fy = qy / Ly;
  const double ax = 2.0 * z / Lx, ay = 2.0 * z / Ly;
  const double fxmax = 1.0 / (lambda * sqrt(ax * ax + 1.0));
  const double fymax = 1.0 / (lambda * sqrt(ay * ay + 1.0));
  const double arg = 1.0 / (lambda * lambda) - fx * fx - fy * fy;
  double sn = 0.0, cs = 0.0;
  const bool open = aperture <= 0.0 || (double)qx * qx + (double)qy * qy < aperture * aperture;
  if (fx < fxmax && fy < fymax && arg >= 0.0 && open) {
    const double ph = 6.283185307179586476925 * z * sqrt(arg);  // 2 pi z sqrt(arg)
    sincos(ph, &sn, &cs);
  }
  if (held) {
    const float2 t = held[(size_t)qx * Hq + qy];
    if (t.x != (float)(cs * t_scale) || t.y != (float)(sn * t_scale)) {
      cs = t.x / t_scale;
      sn = t.y / t_scale;
    }
  }
  if (out) out[(size_t)qy * Wq + qx] = make_float2((float)cs, (float)sn);
  if (out_t)
    out_t[(size_t)qx * Hq + qy] = make_float2((float)(cs * t_scale), (float)(sn * t_scale));
}

hipError_t launch_build_transfer(const Ctx &c, int b0, int b1, hipStream_t s) {
  const bool t = c.htab_t != nullptr;
  const dim3 grid(((t ? c.Hq : c.Wq) + 255) / 256, t ? c.Wq : c.Hq);
  for (int b = b0; b < b1; ++b)
    for (int ch = 0; ch < c.C; ++ch)
      for (int l = 0; l < c.L; ++l) {
        // propagation channel b C + ch: colour ch of hologram b
        const size_t k = ((size_t)b * c.C + ch) * c.L + l, at = k * c.Hq * c.Wq;
        hipLaunchKernelGGL(k_transfer, grid, dim3(256), 0, s, t ? nullptr : c.htab + at,
                           t ? c.htab_t + at : nullptr, 1.0 / ((double)c.Hp * (double)c.Wp), c.Hq,
                           c.Wq, c.Hp, c.Wp, c.cfg.pitch_m, c.lam[b][ch], c.zd[b][l],
                           c.cfg.aperture, c.optics + 2 * k, nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
  return hipSuccess;
}

hipError_t launch_read_transfer(const Ctx &c, int channel, int plane, float2 *out,
                                hipStream_t s) {
  const size_t k = (size_t)channel * c.L + plane, elems = (size_t)c.Hq * c.Wq;
  if (c.htab)
    return hipMemcpyAsync(out, c.htab + k * elems, elems * sizeof(float2),
                          hipMemcpyDeviceToDevice, s);
  hipLaunchKernelGGL(k_transfer, dim3((c.Wq + 255) / 256, c.Hq), dim3(256), 0, s, out, nullptr,
                     1.0 / ((double)c.Hp * (double)c.Wp), c.Hq, c.Wq, c.Hp, c.Wp, c.cfg.pitch_m,
                     0.0, 0.0, c.cfg.aperture, c.optics + 2 * k, c.htab_t + k * elems);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// Row passes: two rows (y0, y0+1) of one channel per workgroup, interleaved in
// LDS as element (x, b) at sbuf[2 x + b].  Column-tiled global layout:
//   S[c][x / 8][y][x % 8]
// so sixteen consecutive threads move one 128-byte line (rows y0, y0+1 of a tile).
// ----------------------------------------------------------------------------
constexpr int kRowThreads = 512;

__device__ __forceinline__ size_t tiled(int c, int y, int x, int H, int Wt) {
  return (((size_t)c * Wt + (x >> 3)) * H + y) * 8 + (x & 7);
}

// Global -> LDS copy of n elements with G loads in flight per thread: every load
// of a group is issued (at a clamped, always valid index) before the first one
// is stored, so their latencies overlap instead of adding up.  ld(i) must be
// callable for every 0 <= i < n; st(i, v) stores element i.
template <int T, int G, class LD, class ST>
__device__ __forceinline__ void staged_copy(int n, int tid, LD ld, ST st) {
  for (int i0 = tid; i0 < n; i0 += T * G) {
    float2 v[G];
#pragma unroll
    for (int g = 0; g < G; ++g) v[g] = ld(min(i0 + g * T, n - 1));
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (i0 + g * T < n) st(i0 + g * T, v[g]);
  }
}

// row b (< ROWS) and column x of element i of ROWS consecutive rows of length w
template <int ROWS>
__device__ __forceinline__ int row_of(int i, int w) {
  int b = 0;
#pragma unroll
  for (int r = 1; r < ROWS; ++r) b += i >= r * w;
  return b;
}

// load the two rows of S into LDS (zero beyond Wp or H)
__device__ __forceinline__ void load_rows_tiled(float2 *sbuf, const float2 *__restrict__ S,
                                                int c, int y0, int H, int Wp, int Wt,
                                                int tid) {
  staged_copy<kRowThreads, 8>(
      Wt * 16, tid,
      [&](int i) {
        const int b = (i >> 3) & 1, x = (i >> 4) * 8 + (i & 7);
        const float2 v = S[tiled(c, min(y0 + b, H - 1), x, H, Wt)];
        return y0 + b < H ? v : make_float2(0.f, 0.f);
      },
      [&](int i, float2 v) {
        const int b = (i >> 3) & 1, x = (i >> 4) * 8 + (i & 7);
        if (x < Wp) sbuf[2 * x + b] = v;
      });
}

// rows y0, y0+1 of the field, zero-extended to n, into LDS (interleaved)
__device__ __forceinline__ void load_field_rows(float2 *sbuf, const float2 *__restrict__ field,
                                                int c, int y0, int H, int W, int n, int tid) {
  staged_copy<kRowThreads, 8>(
      2 * W, tid,
      [&](int i) {
        const int b = row_of<2>(i, W), x = i - b * W;
        const float2 v = field[((size_t)c * H + min(y0 + b, H - 1)) * W + x];
        return y0 + b < H ? v : make_float2(0.f, 0.f);
      },
      [&](int i, float2 v) {
        const int b = row_of<2>(i, W), x = i - b * W;
        sbuf[2 * x + b] = v;
      });
  for (int i = tid; i < 2 * (n - W); i += kRowThreads) sbuf[2 * W + i] = make_float2(0.f, 0.f);
}

__device__ __forceinline__ void store_rows_tiled(const float2 *sbuf, float2 *__restrict__ S,
                                                 int c, int y0, int H, int Wp, int Wt,
                                                 int tid) {
  for (int i = tid; i < Wt * 16; i += kRowThreads) {
    const int t = i >> 4, b = (i >> 3) & 1, x = t * 8 + (i & 7);
    if (x < Wp && y0 + b < H) S[tiled(c, y0 + b, x, H, Wt)] = sbuf[2 * x + b];
  }
}

// F1: field rows (zero-extended to Wp) -> forward FFT -> S
template <int MAXN>
__global__ __launch_bounds__(kRowThreads) void k_row_fwd(const float2 *__restrict__ field,
                                                         int H, int W, int Wt, FftPlan p,
                                                         const float2 *__restrict__ twx,
                                                         float2 *__restrict__ S) {
  extern __shared__ float2 sbuf[];
  __shared__ TwLds tw;
  const int tid = threadIdx.x, n = p.n;
  const int pairs = (H + 1) >> 1;
  const int c = blockIdx.x / pairs, y0 = 2 * (blockIdx.x % pairs);
  load_tw<kRowThreads>(tw, twx, tid);
  load_field_rows(sbuf, field, c, y0, H, W, n, tid);
  __syncthreads();
  fft_lds<-1, 2, kRowThreads, MAXN>(sbuf, p, tw, tid);
  store_rows_tiled(sbuf, S, c, y0, H, n, Wt, tid);
}

// B2: S -> inverse FFT -> first W values of each row -> grad field
template <int MAXN>
__global__ __launch_bounds__(kRowThreads) void k_row_inv(const float2 *__restrict__ S, int H,
                                                         int W, int Wt, FftPlan p,
                                                         const float2 *__restrict__ twx,
                                                         float2 *__restrict__ out) {
  extern __shared__ float2 sbuf[];
  __shared__ TwLds tw;
  const int tid = threadIdx.x, n = p.n;
  const int pairs = (H + 1) >> 1;
  const int c = blockIdx.x / pairs, y0 = 2 * (blockIdx.x % pairs);
  load_tw<kRowThreads>(tw, twx, tid);
  load_rows_tiled(sbuf, S, c, y0, H, n, Wt, tid);
  __syncthreads();
  fft_lds<+1, 2, kRowThreads, MAXN>(sbuf, p, tw, tid);
  for (int b = 0; b < 2; ++b) {
    if (y0 + b >= H) break;
    float2 *dst = out + ((size_t)c * H + y0 + b) * W;
    for (int x = tid; x < W; x += kRowThreads) dst[x] = sbuf[2 * x + b];
  }
}

// F3: S -> inverse FFT -> u (first W values) -> I = |u|^2 (optionally stored,
// with u); if make_grad: dL/dI = 2 (I - T) / M (MSE, Sec. 3.2) or the caller's
// dL/dI, g = 2 dL/dI u = dL/dRe(u) + j dL/dIm(u), zero-extended, forward FFT,
// back into S.  FP64 partial sums of (I - T)^2 per workgroup into loss_part.
template <int MAXN>
__global__ __launch_bounds__(kRowThreads) void k_row_loss(
    float2 *__restrict__ S, int H, int W, int Wt, FftPlan p, const float2 *__restrict__ twx,
    const float *__restrict__ target, const float *__restrict__ grad_I,
    const float *__restrict__ mask, int mcg, float *__restrict__ intensity, float2 *__restrict__ u_out,
    double *__restrict__ loss_part, float gscale, int make_grad) {
  extern __shared__ float2 sbuf[];
  __shared__ TwLds tw;
  __shared__ double red[kRowThreads / 64];
  const int tid = threadIdx.x, n = p.n;
  const int pairs = (H + 1) >> 1;
  const int c = blockIdx.x / pairs, y0 = 2 * (blockIdx.x % pairs);
  load_tw<kRowThreads>(tw, twx, tid);
  if (mask) mask += (size_t)(c / mcg) * H * W;
  load_rows_tiled(sbuf, S, c, y0, H, n, Wt, tid);
  __syncthreads();
  fft_lds<+1, 2, kRowThreads, MAXN>(sbuf, p, tw, tid);
  double acc = 0.0;
  for (int i = tid; i < 2 * n; i += kRowThreads) {
    const int b = i >= n, x = i - b * n;
    const int y = y0 + b;
    if (x < W && y < H) {
      const float2 u = sbuf[2 * x + b];
      const float I = u.x * u.x + u.y * u.y;
      const size_t o = ((size_t)c * H + y) * W + x;
      if (intensity) intensity[o] = I;
      if (u_out) u_out[o] = u;
      float f = 0.f;
      if (target) {
        const float t = target[o], d = I - t;
        // L_recon weight 1 + m^2 + t^2 (plain MSE without a mask)
        const float w = mask ? 1.f + mask[(size_t)y * W + x] * mask[(size_t)y * W + x] + t * t
                             : 1.f;
        acc += (double)d * (double)d * (double)w;
        f = gscale * d * w;  // 4 w (I - T) / M
      } else if (grad_I) {
        f = 2.0f * grad_I[o];
      }
      if (make_grad) sbuf[2 * x + b] = make_float2(f * u.x, f * u.y);
    } else if (make_grad) {
      sbuf[2 * x + b] = make_float2(0.f, 0.f);
    }
  }
  if (target) {
    // wave sums, then a fixed-order sum over the waves
    for (int d = 32; d > 0; d >>= 1) acc += __shfl_down(acc, d, 64);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int w = 0; w < kRowThreads / 64; ++w) s += red[w];
      loss_part[blockIdx.x] = s;
    }
  }
  if (make_grad) {
    __syncthreads();
    fft_lds<-1, 2, kRowThreads, MAXN>(sbuf, p, tw, tid);
    store_rows_tiled(sbuf, S, c, y0, H, n, Wt, tid);
  }
}

// ----------------------------------------------------------------------------
// Size-specialised row passes: compile-time plan (three large-radix stages for
// the workload lengths), ROWS rows per workgroup, full twiddle table in LDS.
// ----------------------------------------------------------------------------
template <int N, int ROWS, int T>
__device__ __forceinline__ void load_rows_c(float2 *sbuf, const float2 *__restrict__ S, int c,
                                            int y0, int H, int Wt, int tid) {
  constexpr int NT = (N + 7) / 8 * 8 * ROWS, G = (NT + T - 1) / T;
  staged_copy<T, G>(
      Wt * 8 * ROWS, tid,
      [&](int i) {
        const int t = i / (8 * ROWS), r = i % (8 * ROWS), b = r >> 3, x = t * 8 + (r & 7);
        const float2 v = S[tiled(c, min(y0 + b, H - 1), x, H, Wt)];
        return y0 + b < H ? v : make_float2(0.f, 0.f);
      },
      [&](int i, float2 v) {
        const int t = i / (8 * ROWS), r = i % (8 * ROWS), b = r >> 3, x = t * 8 + (r & 7);
        if (x < N) sbuf[ROWS * x + b] = v;
      });
}

template <int N, int ROWS, int T>
__device__ __forceinline__ void store_rows_c(const float2 *sbuf, float2 *__restrict__ S, int c,
                                             int y0, int H, int Wt, int tid) {
  for (int i = tid; i < Wt * 8 * ROWS; i += T) {
    const int t = i / (8 * ROWS), r = i % (8 * ROWS), b = r >> 3, x = t * 8 + (r & 7);
    if (x < N && y0 + b < H) S[tiled(c, y0 + b, x, H, Wt)] = sbuf[ROWS * x + b];
  }
}

template <int N, int T>
__device__ __forceinline__ void load_table(float2 *tw, const float2 *__restrict__ src, int tid) {
  for (int i = tid; i < N; i += T) tw[i] = src[i];
}

// Twiddles of a specialised row pass: the full length-N table when it fits in
// LDS beside the rows (FULL), otherwise the two-level table.
template <int N, bool FULL>
struct RowTw;
template <int N>
struct RowTw<N, true> {
  float2 t[N];
  template <int T>
  __device__ __forceinline__ void load(const float2 *full, const float2 *, int tid) { load_table<N, T>(t, full, tid); }
  template <int DIR, int B, int T>
  __device__ __forceinline__ void fft(float2 *buf, int tid) const { cfft<DIR, B, T, N>(buf, t, tid); }
};
template <int N>
struct RowTw<N, false> {
  TwLds t;
  template <int T>
  __device__ __forceinline__ void load(const float2 *, const float2 *two, int tid) { load_tw<T>(t, two, tid); }
  template <int DIR, int B, int T>
  __device__ __forceinline__ void fft(float2 *buf, int tid) const { cfft2<DIR, B, T, N>(buf, t, tid); }
};

template <int N, int ROWS, int T, bool FULL>
__global__ __launch_bounds__(T) void k_row_fwd_c(const float2 *__restrict__ field, int H, int W,
                                                 int Wt, const float2 *__restrict__ twf,
                                                 const float2 *__restrict__ tw2,
                                                 float2 *__restrict__ S) {
  __shared__ float2 sbuf[ROWS * N];
  __shared__ RowTw<N, FULL> tw;
  const int tid = threadIdx.x;
  const int groups = (H + ROWS - 1) / ROWS;
  const int c = blockIdx.x / groups, y0 = ROWS * (blockIdx.x % groups);
  tw.template load<T>(twf, tw2, tid);
  staged_copy<T, (ROWS * N + T - 1) / T>(
      ROWS * W, tid,
      [&](int i) {
        const int b = row_of<ROWS>(i, W), x = i - b * W;
        const float2 v = field[((size_t)c * H + min(y0 + b, H - 1)) * W + x];
        return y0 + b < H ? v : make_float2(0.f, 0.f);
      },
      [&](int i, float2 v) {
        const int b = row_of<ROWS>(i, W), x = i - b * W;
        sbuf[ROWS * x + b] = v;
      });
  for (int i = tid; i < ROWS * (N - W); i += T) sbuf[ROWS * W + i] = make_float2(0.f, 0.f);
  __syncthreads();
  tw.template fft<-1, ROWS, T>(sbuf, tid);
  store_rows_c<N, ROWS, T>(sbuf, S, c, y0, H, Wt, tid);
}

template <int N, int ROWS, int T, bool FULL>
__global__ __launch_bounds__(T) void k_row_inv_c(const float2 *__restrict__ S, int H, int W,
                                                 int Wt, const float2 *__restrict__ twf,
                                                 const float2 *__restrict__ tw2,
                                                 float2 *__restrict__ out) {
  __shared__ float2 sbuf[ROWS * N];
  __shared__ RowTw<N, FULL> tw;
  const int tid = threadIdx.x;
  const int groups = (H + ROWS - 1) / ROWS;
  const int c = blockIdx.x / groups, y0 = ROWS * (blockIdx.x % groups);
  tw.template load<T>(twf, tw2, tid);
  load_rows_c<N, ROWS, T>(sbuf, S, c, y0, H, Wt, tid);
  __syncthreads();
  tw.template fft<+1, ROWS, T>(sbuf, tid);
  for (int b = 0; b < ROWS; ++b) {
    if (y0 + b >= H) break;
    float2 *dst = out + ((size_t)c * H + y0 + b) * W;
    for (int x = tid; x < W; x += T) dst[x] = sbuf[ROWS * x + b];
  }
}

template <int N, int ROWS, int T, bool FULL>
__global__ __launch_bounds__(T) void k_row_loss_c(
    float2 *__restrict__ S, int H, int W, int Wt, const float2 *__restrict__ twf,
    const float2 *__restrict__ tw2, const float *__restrict__ target,
    const float *__restrict__ grad_I, const float *__restrict__ mask, int mcg,
    float *__restrict__ intensity, float2 *__restrict__ u_out, double *__restrict__ loss_part,
    float gscale, int make_grad) {
  __shared__ float2 sbuf[ROWS * N];
  __shared__ RowTw<N, FULL> tw;
  __shared__ double red[T / 64];
  constexpr int KT = (ROWS * N + T - 1) / T;  // cropped elements per thread (W <= N)
  const int tid = threadIdx.x;
  const int groups = (H + ROWS - 1) / ROWS;
  const int c = blockIdx.x / groups, y0 = ROWS * (blockIdx.x % groups);
  const int nw = ROWS * W;  // element i: row y0 + i / W, column i % W
  if (mask) mask += (size_t)(c / mcg) * H * W;
  tw.template load<T>(twf, tw2, tid);
  load_rows_c<N, ROWS, T>(sbuf, S, c, y0, H, Wt, tid);
  // the target (or the caller's dL/dI) of this thread's elements, fetched
  // before the transform (whose barriers do not wait for global loads) so
  // that the loads overlap it
  const float *tsrc = target ? target : grad_I;
  float tv[KT], mv[KT];
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const int i = min(tid + k * T, nw - 1);
    const int b = row_of<ROWS>(i, W), x = i - b * W, y = min(y0 + b, H - 1);
    tv[k] = tsrc ? tsrc[((size_t)c * H + y) * W + x] : 0.f;
    mv[k] = mask ? mask[(size_t)y * W + x] : 0.f;
  }
  lds_sync();
  tw.template fft<+1, ROWS, T>(sbuf, tid);
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const int i = tid + k * T;
    if (i < nw) {
      const int b = row_of<ROWS>(i, W), x = i - b * W, y = y0 + b;
      if (y < H) {
        const float2 u = sbuf[ROWS * x + b];
        const float I = u.x * u.x + u.y * u.y;
        const size_t o = ((size_t)c * H + y) * W + x;
        if (intensity) intensity[o] = I;
        if (u_out) u_out[o] = u;
        float f = 0.f;
        if (target) {
          // L_recon weight 1 + m^2 + t^2 (plain MSE without a mask)
          const float d = I - tv[k], w = mask ? 1.f + mv[k] * mv[k] + tv[k] * tv[k] : 1.f;
          acc += (double)d * (double)d * (double)w;
          f = gscale * d * w;  // 4 w (I - T) / M
        } else if (grad_I) {
          f = 2.0f * tv[k];
        }
        if (make_grad) sbuf[ROWS * x + b] = make_float2(f * u.x, f * u.y);
      } else if (make_grad) {
        sbuf[ROWS * x + b] = make_float2(0.f, 0.f);
      }
    }
  }
  if (make_grad)
    for (int i = tid; i < ROWS * (N - W); i += T) sbuf[ROWS * W + i] = make_float2(0.f, 0.f);
  if (target) {
    for (int d = 32; d > 0; d >>= 1) acc += __shfl_down(acc, d, 64);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
      double sum = 0.0;
      for (int w = 0; w < T / 64; ++w) sum += red[w];
      loss_part[blockIdx.x] = sum;
    }
  }
  if (make_grad) {
    __syncthreads();
    tw.template fft<-1, ROWS, T>(sbuf, tid);
    store_rows_c<N, ROWS, T>(sbuf, S, c, y0, H, Wt, tid);
  }
}

// rows per row-pass workgroup
int row_group_rows(const Ctx &c) {
  return c.row_p ? 1 : c.Wp == 512 ? 4 : 2;
}
static int row_blocks(const Ctx &c) {
  const int r = row_group_rows(c);
  return c.CF * ((c.H + r - 1) / r);
}
static size_t row_lds(const Ctx &c) { return (size_t)2 * c.Wp * sizeof(float2); }

static RowArgs row_args(const Ctx &c, int pass) {
  RowArgs a{};
  a.pass = pass;
  a.H = c.H;
  a.W = c.W;
  a.rows = row_blocks(c);
  a.num_cu = c.num_cu;
  a.twf_x = c.twf_x;
  return a;
}

// the chain kernels of c.row_p chains of Wp / c.row_p points (fft_chain.h)
static hipError_t launch_row_chain(const Ctx &c, const RowArgs &a, hipStream_t s) {
  const int P = c.row_p, M = c.Wp / P;
  const bool found =
      row_chain_part_0(M, P, a, s) || row_chain_part_1(M, P, a, s) ||
      row_chain_part_2(M, P, a, s) || row_chain_part_3(M, P, a, s) ||
      row_chain_part_4(M, P, a, s) || row_chain_part_5(M, P, a, s) ||
      row_chain_part_6(M, P, a, s) || row_chain_part_7(M, P, a, s);
  return found ? hipGetLastError() : hipErrorInvalidValue;
}

static LossSums loss_sums_of(const Ctx &c, double *loss) {
  const int rows = row_blocks(c);
  return LossSums{c.loss_part, c.L, rows, rows / c.B, c.B,
                  1.0 / ((double)c.L * c.C * c.H * c.W), loss, c.finite_flag};
}

int row_split(int Wp, int W) { return split_of(Wp, W, row_chain); }
int col_split(int Hp, int H) { return split_of(Hp, H, col_chain); }

hipError_t launch_row_fwd(const Ctx &c, const float2 *field, float2 *dst, hipStream_t s,
                          int planes) {
  if (c.row_p) {
    // planes follow one another as channels do
    RowArgs a = row_args(c, 0);
    a.rows *= planes;
    a.field = field;
    a.S = dst;
    return launch_row_chain(c, a, s);
  }
  if (planes > 1) {
    const hipError_t e = launch_row_fwd(c, field, dst, s, planes - 1);
    if (e != hipSuccess) return e;
    field += (size_t)(planes - 1) * c.CF * c.H * c.W;
    dst += (planes - 1) * spec_elems(c);
  }
  if (c.Wp == 3840)
    hipLaunchKernelGGL((k_row_fwd_c<3840, 2, 512, false>), dim3(row_blocks(c)), dim3(512), 0, s,
                       field, c.H, c.W, c.Wt, c.twf_x, c.tw_x, dst);
  else if (c.Wp == 512)
    hipLaunchKernelGGL((k_row_fwd_c<512, 4, 256, true>), dim3(row_blocks(c)), dim3(256), 0, s,
                       field, c.H, c.W, c.Wt, c.twf_x, c.tw_x, dst);
  else if (c.Wp <= 4096)
    hipLaunchKernelGGL(k_row_fwd<4096>, dim3(row_blocks(c)), dim3(kRowThreads), row_lds(c), s,
                       field, c.H, c.W, c.Wt, c.plan_x, c.tw_x, dst);
  else
    hipLaunchKernelGGL(k_row_fwd<8192>, dim3(row_blocks(c)), dim3(kRowThreads), row_lds(c), s,
                       field, c.H, c.W, c.Wt, c.plan_x, c.tw_x, dst);
  return hipGetLastError();
}

hipError_t launch_row_inv(const Ctx &c, const float2 *src, float2 *out, hipStream_t s,
                          double *loss) {
  if (c.row_p) {
    RowArgs a = row_args(c, 1);
    a.S = const_cast<float2 *>(src);  // only read by this pass
    a.out = out;
    if (loss) a.sums = loss_sums_of(c, loss);
    return launch_row_chain(c, a, s);
  }
  if (loss) {
    const hipError_t e = launch_loss_finalize(c, loss, s);
    if (e != hipSuccess) return e;
  }
  if (c.Wp == 3840)
    hipLaunchKernelGGL((k_row_inv_c<3840, 2, 512, false>), dim3(row_blocks(c)), dim3(512), 0, s,
                       src, c.H, c.W, c.Wt, c.twf_x, c.tw_x, out);
  else if (c.Wp == 512)
    hipLaunchKernelGGL((k_row_inv_c<512, 4, 256, true>), dim3(row_blocks(c)), dim3(256), 0, s,
                       src, c.H, c.W, c.Wt, c.twf_x, c.tw_x, out);
  else if (c.Wp <= 4096)
    hipLaunchKernelGGL(k_row_inv<4096>, dim3(row_blocks(c)), dim3(kRowThreads), row_lds(c), s,
                       src, c.H, c.W, c.Wt, c.plan_x, c.tw_x, out);
  else
    hipLaunchKernelGGL(k_row_inv<8192>, dim3(row_blocks(c)), dim3(kRowThreads), row_lds(c), s,
                       src, c.H, c.W, c.Wt, c.plan_x, c.tw_x, out);
  return hipGetLastError();
}

hipError_t launch_row_loss(const Ctx &c, int plane, int planes, float2 *buf, const float *target,
                           const float *grad_intensity, const float *mask, float *intensity,
                           float2 *u_out, int make_grad, hipStream_t s) {
  if (!c.row_p && planes > 1) {
    const hipError_t e = launch_row_loss(c, plane, planes - 1, buf, target, grad_intensity, mask,
                                         intensity, u_out, make_grad, s);
    if (e != hipSuccess) return e;
    plane += planes - 1;
    buf += (planes - 1) * spec_elems(c);
  }
  // the loss of each hologram is its own mean over L C H W
  const double M = (double)c.L * c.C * c.H * c.W;
  const float gscale = (float)(4.0 / M);
  // plane l of the [L][B C][H][W] arrays; its loss partials after those of planes < l
  const size_t po = (size_t)plane * c.CF * c.H * c.W;
  if (target) target += po;
  if (grad_intensity) grad_intensity += po;
  if (intensity) intensity += po;
  if (u_out) u_out += po;
  // [L][B][H][W]: propagation channel ch reads the mask of hologram ch / C
  if (mask) mask += (size_t)plane * c.B * c.H * c.W;
  const int mcg = c.C;
  double *lp = c.loss_part + (size_t)plane * row_blocks(c);
  if (c.row_p) {
    RowArgs a = row_args(c, 2);
    a.rows *= planes;
    a.S = buf;
    a.target = target;
    a.grad_I = grad_intensity;
    a.mask = mask;
    a.mcg = mcg;
    a.intensity = intensity;
    a.u_out = u_out;
    a.loss_part = lp;
    a.gscale = gscale;
    a.make_grad = make_grad;
    return launch_row_chain(c, a, s);
  }
  if (c.Wp == 3840)
    hipLaunchKernelGGL((k_row_loss_c<3840, 2, 512, false>), dim3(row_blocks(c)), dim3(512), 0, s,
                       buf, c.H, c.W, c.Wt, c.twf_x, c.tw_x, target, grad_intensity, mask, mcg, intensity,
                       u_out, lp, gscale, make_grad);
  else if (c.Wp == 512)
    hipLaunchKernelGGL((k_row_loss_c<512, 4, 256, true>), dim3(row_blocks(c)), dim3(256), 0, s,
                       buf, c.H, c.W, c.Wt, c.twf_x, c.tw_x, target, grad_intensity, mask, mcg, intensity,
                       u_out, lp, gscale, make_grad);
  else if (c.Wp <= 4096)
    hipLaunchKernelGGL(k_row_loss<4096>, dim3(row_blocks(c)), dim3(kRowThreads), row_lds(c), s,
                       buf, c.H, c.W, c.Wt, c.plan_x, c.tw_x, target, grad_intensity, mask, mcg,
                       intensity, u_out, lp, gscale, make_grad);
  else
    hipLaunchKernelGGL(k_row_loss<8192>, dim3(row_blocks(c)), dim3(kRowThreads), row_lds(c), s,
                       buf, c.H, c.W, c.Wt, c.plan_x, c.tw_x, target, grad_intensity, mask, mcg,
                       intensity, u_out, lp, gscale, make_grad);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// Column passes over one 8-column tile of one channel (a contiguous block of
// H x 8 complex in S), in place.
// ----------------------------------------------------------------------------
__device__ __forceinline__ void col_store(const ColIO &io, size_t i, float2 v) {
  io.dst[i] = io.acc ? cadd(io.dst[i], v) : v;
}

__device__ __forceinline__ float2 transfer_at(const float2 *__restrict__ hc, int ky, int kx,
                                              int Hp, int Wp, int Wq, int conj_h, float scale) {
  const int qx = min(kx, Wp - kx), qy = min(ky, Hp - ky);
  float2 h = hc[(size_t)qy * Wq + qx];
  if (conj_h) h.y = -h.y;
  return cscale(h, scale);
}

// X[i] *= H(2 (i >> 3) + parity, 8 t + (i & 7)) over one column block of M rows:
// all table loads of a thread are issued before the first is used, so their
// latencies overlap.
template <int M, int T>
__device__ __forceinline__ void apply_transfer(float2 *X, const float2 *__restrict__ hc,
                                               int parity, int t, int Wp, int Wq, int conj_h,
                                               float scale, int tid) {
  constexpr int total = 8 * M, K = (total + T - 1) / T, G = 3;
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += G) {
    float2 hv[G];
#pragma unroll
    for (int k = k0; k < k0 + G && k < K; ++k) {
      const int i = tid + k * T;
      hv[k - k0] = make_float2(0.f, 0.f);
      if (total % T == 0 || i < total) {
        const int kx = t * 8 + (i & 7), ky = 2 * (i >> 3) + parity;
        const int qx = min(kx, Wp - kx), qy = min(ky, 2 * M - ky);
        if (kx < Wp) hv[k - k0] = hc[(uint32_t)(qy * Wq + qx)];
      }
    }
#pragma unroll
    for (int k = k0; k < k0 + G && k < K; ++k) {
      const int i = tid + k * T;
      if (total % T == 0 || i < total) {
        float2 h = hv[k - k0];
        if (conj_h) h.y = -h.y;
        X[i] = cmul(X[i], cscale(h, scale));
      }
    }
  }
}

// even Hp = 2M: two M-point chains (see the file header)
template <int MAXM, int T>
__global__ __launch_bounds__(T, 2048 / T) void k_col_half(ColIO io, int H, int Wp, int Wt,
                                                FftPlan pm, const float2 *__restrict__ twm,
                                                const float2 *__restrict__ twh, int Wq,
                                                int conj_h, float scale) {
  __shared__ float2 sbuf[8 * MAXM];
  __shared__ TwLds tm, th;
  constexpr int K = (8 * MAXM + T - 1) / T;
  const int tid = threadIdx.x;
  const int M = pm.n, Hp = 2 * M;
  const int t = blockIdx.x, ch = blockIdx.y;
  const size_t off = ((size_t)ch * Wt + t) * H * 8;
  const float2 *base = io.src + off;
  const float2 *hc = io.htab + ch * io.hstride;
  const int total = 8 * M;
  load_tw<T>(tm, twm, tid);
  load_tw<T>(th, twh, tid);
  __syncthreads();
  float2 keep[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = tid + k * T;
    keep[k] = make_float2(0.f, 0.f);
    if (i < total) {
      const int n = i >> 3, kx = t * 8 + (i & 7);
      float2 x0 = make_float2(0.f, 0.f), x1 = x0;
      if (kx < Wp) {
        if (n < H) x0 = base[i];
        if (n + M < H) x1 = base[i + 8 * M];
      }
      sbuf[i] = cadd(x0, x1);
      keep[k] = cmul(csub(x0, x1), tw_at(th, n));
    }
  }
  __syncthreads();
  for (int parity = 0; parity < 2; ++parity) {
    fft_lds<-1, 8, T, MAXM>(sbuf, pm, tm, tid);
    for (int i = tid; i < total; i += T) {
      const int m = i >> 3, kx = t * 8 + (i & 7);
      sbuf[i] = kx < Wp ? cmul(sbuf[i], transfer_at(hc, 2 * m + parity, kx, Hp, Wp, Wq, conj_h,
                                                     scale))
                        : make_float2(0.f, 0.f);
    }
    __syncthreads();
    fft_lds<+1, 8, T, MAXM>(sbuf, pm, tm, tid);
    if (parity == 0) {
      // even result to registers, odd-chain input to LDS (each thread its own slots)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int i = tid + k * T;
        if (i < total) {
          const float2 e = sbuf[i];
          sbuf[i] = keep[k];
          keep[k] = e;
        }
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = tid + k * T;
    if (i < total) {
      const int n = i >> 3, kx = t * 8 + (i & 7);
      if (kx < Wp) {
        const float2 wo = cmul(cconj(tw_at(th, n)), sbuf[i]);
        if (n < H) col_store(io, off + i, cadd(keep[k], wo));
        if (n + M < H) col_store(io, off + i + 8 * M, csub(keep[k], wo));
      }
    }
  }
}

// odd Hp: one Hp-point transform per column
template <int MAXN, int T>
__global__ __launch_bounds__(T) void k_col_full(ColIO io, int H, int Wp, int Wt, FftPlan py,
                                                const float2 *__restrict__ twy, int Wq,
                                                int conj_h, float scale) {
  __shared__ float2 sbuf[8 * MAXN];
  __shared__ TwLds ty;
  const int tid = threadIdx.x;
  const int Hp = py.n;
  const int t = blockIdx.x, ch = blockIdx.y;
  const size_t off = ((size_t)ch * Wt + t) * H * 8;
  const float2 *base = io.src + off;
  const float2 *hc = io.htab + ch * io.hstride;
  const int total = 8 * Hp;
  load_tw<T>(ty, twy, tid);
  for (int i = tid; i < total; i += T) {
    const int r = i >> 3, kx = t * 8 + (i & 7);
    sbuf[i] = (r < H && kx < Wp) ? base[i] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  fft_lds<-1, 8, T, MAXN>(sbuf, py, ty, tid);
  for (int i = tid; i < total; i += T) {
    const int r = i >> 3, kx = t * 8 + (i & 7);
    sbuf[i] = kx < Wp ? cmul(sbuf[i], transfer_at(hc, r, kx, Hp, Wp, Wq, conj_h, scale))
                      : make_float2(0.f, 0.f);
  }
  __syncthreads();
  fft_lds<+1, 8, T, MAXN>(sbuf, py, ty, tid);
  for (int i = tid; i < 8 * H; i += T) {
    const int kx = t * 8 + (i & 7);
    if (kx < Wp) col_store(io, off + i, sbuf[i]);
  }
}

// size-specialised even/odd column pass: compile-time M-point plan, full
// M-entry twiddle table in LDS (the Hp-point pre/post twiddles use the small
// two-level table)
template <int M, int T>
__global__ __launch_bounds__(T) void k_col_half_c(ColIO io, int H, int Wp, int Wt,
                                                  const float2 *__restrict__ twf_m,
                                                  const float2 *__restrict__ twh, int Wq,
                                                  int conj_h, float scale) {
  __shared__ float2 sbuf[8 * M];
  __shared__ float2 tw[M];
  __shared__ TwLds th;
  constexpr int K = (8 * M + T - 1) / T;
  constexpr int total = 8 * M;
  constexpr int Hp = 2 * M;
  const int tid = threadIdx.x;
  const int t = blockIdx.x, ch = blockIdx.y;
  const size_t off = ((size_t)ch * Wt + t) * H * 8;
  const float2 *base = io.src + off;
  const float2 *hc = io.htab + ch * io.hstride;
  load_table<M, T>(tw, twf_m, tid);
  load_tw<T>(th, twh, tid);
  __syncthreads();
  float2 keep[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = tid + k * T;
    keep[k] = make_float2(0.f, 0.f);
    if (total % T == 0 || i < total) {
      const int n = i >> 3, kx = t * 8 + (i & 7);
      float2 x0 = make_float2(0.f, 0.f), x1 = x0;
      if (kx < Wp) {
        if (n < H) x0 = base[i];
        if (n + M < H) x1 = base[i + 8 * M];
      }
      sbuf[i] = cadd(x0, x1);
      keep[k] = cmul(csub(x0, x1), tw_at(th, n));
    }
  }
  __syncthreads();
  for (int parity = 0; parity < 2; ++parity) {
    cfft<-1, 8, T, M>(sbuf, tw, tid);
    apply_transfer<M, T>(sbuf, hc, parity, t, Wp, Wq, conj_h, scale, tid);
    __syncthreads();
    cfft<+1, 8, T, M>(sbuf, tw, tid);
    if (parity == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int i = tid + k * T;
        if (total % T == 0 || i < total) {
          const float2 e = sbuf[i];
          sbuf[i] = keep[k];
          keep[k] = e;
        }
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = tid + k * T;
    if (total % T == 0 || i < total) {
      const int n = i >> 3, kx = t * 8 + (i & 7);
      if (kx < Wp) {
        const float2 wo = cmul(cconj(tw_at(th, n)), sbuf[i]);
        if (n < H) col_store(io, off + i, cadd(keep[k], wo));
        if (n + M < H) col_store(io, off + i + 8 * M, csub(keep[k], wo));
      }
    }
  }
}

hipError_t launch_col_pass(const Ctx &c, int conj_h, int plane, int planes, const float2 *src,
                           float2 *dst, int acc, hipStream_t s) {
  if (planes > 1 && !(c.col_p && planes_chain(c.Hp / c.col_p, c.col_p))) {
    for (int l = 0; l < planes; ++l) {
      const size_t o = l * spec_elems(c);
      const hipError_t e = conj_h ? launch_col_pass(c, 1, plane + l, 1, src + o, dst, acc || l, s)
                                  : launch_col_pass(c, 0, plane + l, 1, src, dst + o, acc, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const float scale = (float)(1.0 / ((double)c.Hp * (double)c.Wp));
  const size_t tab = (size_t)c.Hq * c.Wq;
  const ColIO io{src, dst, c.htab + (size_t)plane * tab, (size_t)c.L * tab, acc,
                 planes, tab, spec_elems(c)};
  dim3 grid(c.Wt, c.CF);
  if (c.col_p) {
    const int P = c.col_p, M = c.Hp / P;
    ColArgs a{};
    a.io = io;
    a.io.htab = c.htab_t + (size_t)plane * tab;
    a.conj_h = conj_h;
    a.Hq = c.Hq;
    a.H = c.H;
    a.Wp = c.Wp;
    a.Wt = c.Wt;
    a.C = c.CF;
    a.twf_y = c.twf_y;
    const bool found =
        col_chain_part_0(M, P, a, s) || col_chain_part_1(M, P, a, s) ||
        col_chain_part_2(M, P, a, s) || col_chain_part_3(M, P, a, s) ||
        col_chain_part_4(M, P, a, s) || col_chain_part_5(M, P, a, s) ||
        col_chain_part_6(M, P, a, s) || col_chain_part_7(M, P, a, s);
    if (!found) return hipErrorInvalidValue;
  } else if (c.Hp == 2160) {
    hipLaunchKernelGGL((k_col_half_c<1080, 1024>), grid, dim3(1024), 0, s, io, c.H, c.Wp, c.Wt,
                       c.twf_m, c.tw_y, c.Wq, conj_h, scale);
  } else if (c.Hp == 512) {
    hipLaunchKernelGGL((k_col_half_c<256, 256>), grid, dim3(256), 0, s, io, c.H, c.Wp, c.Wt,
                       c.twf_m, c.tw_y, c.Wq, conj_h, scale);
  } else if (c.Hp % 2 == 0) {
    const int M = c.Hp / 2;
    if (M <= kColHalfSmall)
      hipLaunchKernelGGL((k_col_half<kColHalfSmall, 512>), grid, dim3(512), 0, s, io, c.H, c.Wp,
                         c.Wt, c.plan_m, c.tw_m, c.tw_y, c.Wq, conj_h, scale);
    else
      hipLaunchKernelGGL((k_col_half<kColHalfMax, 1024>), grid, dim3(1024), 0, s, io, c.H, c.Wp,
                         c.Wt, c.plan_m, c.tw_m, c.tw_y, c.Wq, conj_h, scale);
  } else {
    hipLaunchKernelGGL((k_col_full<kColFullMax, 1024>), grid, dim3(1024), 0, s, io, c.H, c.Wp,
                       c.Wt, c.plan_y, c.tw_y, c.Wq, conj_h, scale);
  }
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_loss_finalize(LossSums sums) {
  loss_sums<256>(sums, blockIdx.x);
}

hipError_t launch_loss_finalize(const Ctx &c, double *loss, hipStream_t s) {
  hipLaunchKernelGGL(k_loss_finalize, dim3(c.B), dim3(256), 0, s, loss_sums_of(c, loss));
  return hipGetLastError();
}

}  // namespace cgh
