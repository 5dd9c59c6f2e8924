// Bandwidth-bound kernels of the hot path: the W-maps (step 2 of the H_eff
// ordering of Sec. 5), deterministic FP64 reductions and vector updates of
// the Lanczos solver, layout helpers of the truncation, casts of the
// mixed-precision path and the reduction of the W-adjoint.
#include <algorithm>

#include <type_traits>

#include "d3s_internal.h"

namespace d3s {
namespace {

constexpr int kThreads = 256;
constexpr int kRedBlocks = 1024;   // fixed partial count: reductions are order-deterministic

__device__ __forceinline__ float bf16_to_f32(bf16_t h) {
  return __uint_as_float(((uint32_t)h) << 16);
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40);   // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);                                           // round to nearest even
  return (bf16_t)(u >> 16);
}

template <typename T> struct Cvt;
template <> struct Cvt<double> {
  __device__ static double ld(double x) { return x; }
  __device__ static double st(double x) { return x; }
};
template <> struct Cvt<float> {
  __device__ static float ld(float x) { return x; }
  __device__ static float st(float x) { return x; }
};
template <> struct Cvt<bf16_t> {
  __device__ static float ld(bf16_t x) { return bf16_to_f32(x); }
  __device__ static bf16_t st(float x) { return f32_to_bf16(x); }
};

// ---------------------------------------------------------------- W-maps
// One thread per (a, y): it holds the K = wl*d values T1[a, :, :, y] in
// registers and produces the d*wr outputs; W (pre-scaled by alpha and laid
// out as [(s,v)][(w,t)]) sits in LDS and is read by broadcast.
template <typename Tin, typename Tout, typename Tc, int MAXK>
__global__ __launch_bounds__(kThreads)
void wmap_l2r_kernel(const Tin* __restrict__ T1, const Tc* __restrict__ Wg, Tout* __restrict__ out,
                     long ld_out, int ml, int d, int mr, int wl, int wr, Tc alpha) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Tc* sW = reinterpret_cast<Tc*>(smem_raw);
  const int K = wl * d;
  const int nOut = d * wr;
  // rows of MAXK entries, zero beyond K: the inner loop has no bounds test and
  // reads W with vector LDS loads
  for (int i = threadIdx.x; i < MAXK * nOut; i += blockDim.x) {
    const int o = i / MAXK, k = i - o * MAXK;  // o = s*wr + v, k = w*d + t
    const int s = o / wr, v = o - s * wr;
    const int w = k / d, t = k - w * d;
    sW[i] = (k < K) ? alpha * Wg[((w * wr + v) * d + s) * d + t] : Tc(0);
  }
  __syncthreads();
  const int a = blockIdx.y;
  const int y = blockIdx.x * blockDim.x + threadIdx.x;
  if (y >= mr) return;
  Tc in[MAXK];
  const Tin* src = T1 + (long)a * K * mr + y;
#pragma unroll
  for (int k = 0; k < MAXK; ++k) in[k] = (k < K) ? (Tc)Cvt<Tin>::ld(src[(long)k * mr]) : Tc(0);
  for (int o = 0; o < nOut; ++o) {
    const Tc* wrow = sW + o * MAXK;
    Tc acc = 0;
#pragma unroll
    for (int k = 0; k < MAXK; ++k) acc += wrow[k] * in[k];
    const int s = o / wr, v = o - s * wr;
    out[(long)(a * d + s) * ld_out + (long)v * mr + y] = Cvt<Tout>::st(acc);
  }
}

// Four consecutive y per thread, moved by one vector load or store per channel,
// for elements of 4 bytes or less in rows of whole aligned vectors.  The sum
// runs over k in the order of wmap_l2r_kernel, so a product does not depend on
// which of the two ran.  With one point a thread every broadcast read of four W
// entries (8 cycles of the LDS that four SIMDs share) serves four multiply-adds
// of one wave; here 16.  T1 FP32 to T2 BF16, d = 4, w = 6, behind the GEMM that
// writes T1: m = 1920 111 us (152 us), 2048 143 to 160 us (159 to 164 us), 2500 185
// us (236 us), 4.2 to 4.8 TB/s, the rate of a copy.
template <typename T> struct alignas(4 * sizeof(T)) Vec4 { T v[4]; };

template <typename Tin, typename Tout, typename Tc, int MAXK>
__global__ __launch_bounds__(kThreads)
void wmap_l2r_vec4_kernel(const Tin* __restrict__ T1, const Tc* __restrict__ Wg, Tout* __restrict__ out,
                          long ld_out, int ml, int d, int mr, int wl, int wr, Tc alpha) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Tc* sW = reinterpret_cast<Tc*>(smem_raw);
  const int K = wl * d;
  const int nOut = d * wr;
  for (int i = threadIdx.x; i < MAXK * nOut; i += blockDim.x) {
    const int o = i / MAXK, k = i - o * MAXK;  // o = s*wr + v, k = w*d + t
    const int s = o / wr, v = o - s * wr;
    const int w = k / d, t = k - w * d;
    sW[i] = (k < K) ? alpha * Wg[((w * wr + v) * d + s) * d + t] : Tc(0);
  }
  __syncthreads();
  const int a = blockIdx.y;
  const int y = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
  if (y >= mr) return;
  Tc in[MAXK][4];
  const Tin* src = T1 + (long)a * K * mr + y;
#pragma unroll
  for (int k = 0; k < MAXK; ++k) {
    if (k < K) {
      const Vec4<Tin> q = *reinterpret_cast<const Vec4<Tin>*>(src + (long)k * mr);
#pragma unroll
      for (int j = 0; j < 4; ++j) in[k][j] = (Tc)Cvt<Tin>::ld(q.v[j]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) in[k][j] = Tc(0);
    }
  }
  int s = 0, v = 0;
  for (int o = 0; o < nOut; ++o) {
    const Tc* wrow = sW + o * MAXK;
    Tc acc[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < MAXK; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] += wrow[k] * in[k][j];
    Vec4<Tout> r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r.v[j] = Cvt<Tout>::st(acc[j]);
    *reinterpret_cast<Vec4<Tout>*>(out + (long)(a * d + s) * ld_out + (long)v * mr + y) = r;
    if (++v == wr) {
      v = 0;
      ++s;
    }
  }
}

// One thread per (x, b): inputs Y[x, t, b, :] for all t (K = d*wr values),
// outputs Z[w, x, s, b] for all (w, s).
template <typename Tin, typename Tout, typename Tc, int MAXK>
__global__ __launch_bounds__(kThreads)
void wmap_r2l_kernel(const Tin* __restrict__ Y, const Tc* __restrict__ Wg, Tout* __restrict__ Z,
                     int ml, int d, int mr, int wl, int wr, Tc alpha) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Tc* sW = reinterpret_cast<Tc*>(smem_raw);
  const int K = d * wr;
  const int nOut = wl * d;
  for (int i = threadIdx.x; i < MAXK * nOut; i += blockDim.x) {
    const int o = i / MAXK, k = i - o * MAXK;  // o = w*d + s, k = t*wr + v
    const int w = o / d, s = o - w * d;
    const int t = k / wr, v = k - t * wr;
    sW[i] = (k < K) ? alpha * Wg[((w * wr + v) * d + s) * d + t] : Tc(0);
  }
  __syncthreads();
  const int x = blockIdx.y;
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= mr) return;
  Tc in[MAXK];
#pragma unroll
  for (int k = 0; k < MAXK; ++k) {
    if (k < K) {
      const int t = k / wr, v = k - t * wr;
      in[k] = (Tc)Cvt<Tin>::ld(Y[((long)(x * d + t) * mr + b) * wr + v]);
    } else {
      in[k] = Tc(0);
    }
  }
  for (int o = 0; o < nOut; ++o) {
    const Tc* wrow = sW + o * MAXK;
    Tc acc = 0;
#pragma unroll
    for (int k = 0; k < MAXK; ++k) acc += wrow[k] * in[k];
    const int w = o / d, s = o - w * d;
    Z[((long)(w * ml + x) * d + s) * mr + b] = Cvt<Tout>::st(acc);
  }
}

// W-maps for MPO bonds too wide for the register/LDS kernels above (the
// channel-pair MPO of H^2): one thread per output element, W read from
// global memory (every lane of a wave reads the same W entry, a broadcast).
template <typename Tin, typename Tout, typename Tc>
__global__ __launch_bounds__(kThreads)
void wmap_l2r_wide_kernel(const Tin* __restrict__ T1, const Tc* __restrict__ Wg, Tout* __restrict__ out,
                          long ld_out, int ml, int d, int mr, int wl, int wr, Tc alpha) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long)ml * d * wr * mr) return;
  const int y = (int)(e % mr);
  long r = e / mr;
  const int v = (int)(r % wr);
  r /= wr;
  const int s = (int)(r % d);
  const int a = (int)(r / d);
  Tc acc = 0;
  for (int w = 0; w < wl; ++w)
    for (int t = 0; t < d; ++t)
      acc += Wg[((w * wr + v) * d + s) * d + t] * (Tc)Cvt<Tin>::ld(T1[(((long)a * wl + w) * d + t) * mr + y]);
  out[((long)a * d + s) * ld_out + (long)v * mr + y] = Cvt<Tout>::st(alpha * acc);
}

template <typename Tin, typename Tout, typename Tc>
__global__ __launch_bounds__(kThreads)
void wmap_r2l_wide_kernel(const Tin* __restrict__ Y, const Tc* __restrict__ Wg, Tout* __restrict__ Z, int ml,
                          int d, int mr, int wl, int wr, Tc alpha) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long)wl * ml * d * mr) return;
  const int b = (int)(e % mr);
  long r = e / mr;
  const int s = (int)(r % d);
  r /= d;
  const int x = (int)(r % ml);
  const int w = (int)(r / ml);
  Tc acc = 0;
  for (int t = 0; t < d; ++t)
    for (int v = 0; v < wr; ++v)
      acc += Wg[((w * wr + v) * d + s) * d + t] * (Tc)Cvt<Tin>::ld(Y[(((long)x * d + t) * mr + b) * wr + v]);
  Z[e] = Cvt<Tout>::st(alpha * acc);
}

template <typename Tin, typename Tout, typename Tc>
void wmap_l2r_t(Ctx* c, const void* T1, const void* W, void* out, long ld_out, int ml, int d,
                int mr, int wl, int wr, double alpha) {
  const int K = wl * d;
  dim3 grid((mr + kThreads - 1) / kThreads, ml);
  auto args = [&](auto kern, int maxk) {
    const size_t sh = sizeof(Tc) * (size_t)maxk * d * wr;
    hipLaunchKernelGGL(kern, grid, dim3(kThreads), sh, c->stream, (const Tin*)T1, (const Tc*)W,
                       (Tout*)out, ld_out, ml, d, mr, wl, wr, (Tc)alpha);
  };
  const bool fits = d * wr <= 80;
  if constexpr (sizeof(Tin) <= 4 && sizeof(Tout) <= 4) {
    // A quarter of the threads: they have to fill the chip.  Their waves, weighted
    // by the share of a row's last wave that is in use: 780 suffice for up to 16
    // inputs a point, 1030 beyond (BF16, d = 4, w = 8, 64 x 64 25 against 14 us, 512
    // x 512 29 against 25, 600 x 600 both 32; w = 6, 512 x 512 21 against 19, 500 x
    // 640 0.95 and 700 x 700 0.86 of the time; d = 2, w = 5, 384 x 384 1.09 and 512 x
    // 512 0.99).  Nor may a row's second workgroup be nearly empty (FP32, w = 6,
    // 1200 x 1200 1.15 of the time, 1400 1.00, 1600 0.99, 1800 0.88; BF16, w = 8,
    // 1200 1.19, 1536 0.95).  FP32 rows that large tensors stream from memory gain
    // nothing with many inputs a point (w = 6, 2048 159 against 149 us, 2500 234
    // against 230; d = 2, w = 8, 2500 145 against 152).
    const long rw = (mr + 255) / 256, waves = (long)ml * mr / 256 * mr / (256 * rw);
    const int two = K < 16 ? 0 : sizeof(Tout) == 4 ? (K <= 24 ? 1550 : 1700) : K <= 16 ? 0 : K <= 24 ? 1250 : 1500;
    const int last = sizeof(Tout) == 4 && K > 16 ? 2000 : 1 << 30;
    if (fits && K <= 32 && waves >= (K <= 16 ? 780 : 1030) && mr >= 192 && (mr <= 1024 || (mr >= two && mr < last)) &&
        mr % 4 == 0 && ld_out % 4 == 0 &&
        reinterpret_cast<uintptr_t>(T1) % (4 * sizeof(Tin)) == 0 &&
        reinterpret_cast<uintptr_t>(out) % (4 * sizeof(Tout)) == 0) {
      grid.x = (mr / 4 + kThreads - 1) / kThreads;
      if (K <= 8) args(wmap_l2r_vec4_kernel<Tin, Tout, Tc, 8>, 8);
      else if (K <= 16) args(wmap_l2r_vec4_kernel<Tin, Tout, Tc, 16>, 16);
      else if (K <= 24) args(wmap_l2r_vec4_kernel<Tin, Tout, Tc, 24>, 24);
      else args(wmap_l2r_vec4_kernel<Tin, Tout, Tc, 32>, 32);
      D3S_HIP(hipGetLastError());
      return;
    }
  }
  if (fits && K <= 8) args(wmap_l2r_kernel<Tin, Tout, Tc, 8>, 8);
  else if (fits && K <= 16) args(wmap_l2r_kernel<Tin, Tout, Tc, 16>, 16);
  else if (fits && K <= 24) args(wmap_l2r_kernel<Tin, Tout, Tc, 24>, 24);
  else if (fits && K <= 32) args(wmap_l2r_kernel<Tin, Tout, Tc, 32>, 32);
  else if (fits && K <= 48) args(wmap_l2r_kernel<Tin, Tout, Tc, 48>, 48);
  else if (fits && K <= 80) args(wmap_l2r_kernel<Tin, Tout, Tc, 80>, 80);
  else {
    const long n = (long)ml * d * wr * mr;
    hipLaunchKernelGGL((wmap_l2r_wide_kernel<Tin, Tout, Tc>), dim3((unsigned)((n + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, c->stream, (const Tin*)T1, (const Tc*)W, (Tout*)out, ld_out, ml, d, mr,
                       wl, wr, (Tc)alpha);
  }
  D3S_HIP(hipGetLastError());
}

template <typename Tin, typename Tout, typename Tc>
void wmap_r2l_t(Ctx* c, const void* Y, const void* W, void* Z, int ml, int d, int mr, int wl,
                int wr, double alpha) {
  const int K = d * wr;
  dim3 grid((mr + kThreads - 1) / kThreads, ml);
  auto args = [&](auto kern, int maxk) {
    const size_t sh = sizeof(Tc) * (size_t)maxk * d * wl;
    hipLaunchKernelGGL(kern, grid, dim3(kThreads), sh, c->stream, (const Tin*)Y, (const Tc*)W,
                       (Tout*)Z, ml, d, mr, wl, wr, (Tc)alpha);
  };
  const bool fits = d * wl <= 80;
  if (fits && K <= 8) args(wmap_r2l_kernel<Tin, Tout, Tc, 8>, 8);
  else if (fits && K <= 16) args(wmap_r2l_kernel<Tin, Tout, Tc, 16>, 16);
  else if (fits && K <= 24) args(wmap_r2l_kernel<Tin, Tout, Tc, 24>, 24);
  else if (fits && K <= 32) args(wmap_r2l_kernel<Tin, Tout, Tc, 32>, 32);
  else if (fits && K <= 48) args(wmap_r2l_kernel<Tin, Tout, Tc, 48>, 48);
  else if (fits && K <= 80) args(wmap_r2l_kernel<Tin, Tout, Tc, 80>, 80);
  else {
    const long n = (long)wl * ml * d * mr;
    hipLaunchKernelGGL((wmap_r2l_wide_kernel<Tin, Tout, Tc>), dim3((unsigned)((n + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, c->stream, (const Tin*)Y, (const Tc*)W, (Tout*)Z, ml, d, mr, wl, wr,
                       (Tc)alpha);
  }
  D3S_HIP(hipGetLastError());
}

// Block-sparse W-map over a table of tasks, one per (left sector i, right
// sector j) pair.  A task lists its allowed input channel pairs and output
// channel pairs as entries {offset within a row, partial W index}; for an
// element (a, y) of the D_i x D_j block
//   out[a*out_rs + e_out.off + y] = alpha * sum_k W[e_in[k].wp + e_out.wp] * in[a*in_rs + e_in[k].off + y]
// (the W index is the sum of the two partial indices).  Workgroups take
// chunks of kWmapChunk elements of a block (a per-chunk table names the
// task), four per thread, 256 apart so that loads and stores stay
// coalesced; the task's W sub-matrix sits in LDS.  Nothing outside the
// listed blocks is read or written.
template <typename Tin, typename Tout, typename Tc, int MAXK>
__global__ __launch_bounds__(kThreads)
void wmap_blocks_kernel(const Tin* __restrict__ in, const Tc* __restrict__ Wg, Tout* __restrict__ out,
                        const WmapTask* __restrict__ tasks, const int* __restrict__ ctask,
                        const WmapEnt* __restrict__ ents, long in_rs, long out_rs, Tc alpha) {
  constexpr int EPT = kWmapChunk / kThreads;
  __shared__ Tc sW[MAXK * MAXK];
  __shared__ long sInOff[MAXK], sOutOff[MAXK];
  __shared__ int sInW[MAXK], sOutW[MAXK];
  const WmapTask tk = tasks[ctask[blockIdx.x]];
  const int nin = tk.nin, nout = tk.nout;
  for (int i = threadIdx.x; i < nin; i += blockDim.x) {
    sInOff[i] = ents[tk.idx0 + i].off;
    sInW[i] = ents[tk.idx0 + i].wp;
  }
  for (int i = threadIdx.x; i < nout; i += blockDim.x) {
    sOutOff[i] = ents[tk.idx0 + nin + i].off;
    sOutW[i] = ents[tk.idx0 + nin + i].wp;
  }
  __syncthreads();
  // W rows zero-padded to MAXK; inputs past nin are zeros (the test is
  // uniform over the workgroup, so it costs no divergence and no loads)
  for (int i = threadIdx.x; i < nout * MAXK; i += blockDim.x) {
    const int o = i / MAXK, k = i - o * MAXK;
    sW[i] = (k < nin) ? alpha * Wg[sInW[k] + sOutW[o]] : Tc(0);
  }
  __syncthreads();
  const long n = (long)tk.di * tk.dj;
  const long e0 = (long)((int)blockIdx.x - tk.chunk0) * kWmapChunk + threadIdx.x;
  for (int r = 0; r < EPT; ++r) {
    const long e = e0 + (long)r * kThreads;
    if (e >= n) return;
    const long a = tk.i_off + e / tk.dj, y = tk.j_off + e % tk.dj;
    const Tin* src = in + a * in_rs + y;
    Tout* dst = out + a * out_rs + y;
    if (nin == 0) {
      for (int o = 0; o < nout; ++o) dst[sOutOff[o]] = Cvt<Tout>::st(Tc(0));
      continue;
    }
    Tc v[MAXK];
#pragma unroll
    for (int k = 0; k < MAXK; ++k) v[k] = (k < nin) ? (Tc)Cvt<Tin>::ld(src[sInOff[k]]) : Tc(0);
    for (int o = 0; o < nout; ++o) {
      Tc acc = 0;
#pragma unroll
      for (int k = 0; k < MAXK; ++k) acc += sW[o * MAXK + k] * v[k];
      dst[sOutOff[o]] = Cvt<Tout>::st(acc);
    }
  }
}

// Four consecutive elements of a block row per thread, moved with one
// vector load / store per channel pair: for tables whose offsets, row
// lengths and block widths are all multiples of 4 (so the four elements
// share a row and the vectors are aligned).  Same chunks and task table as
// wmap_blocks_kernel.

template <typename Tin, typename Tout, typename Tc, int MAXK>
__global__ __launch_bounds__(kThreads)
void wmap_blocks_vec4_kernel(const Tin* __restrict__ in, const Tc* __restrict__ Wg, Tout* __restrict__ out,
                             const WmapTask* __restrict__ tasks, const int* __restrict__ ctask,
                             const WmapEnt* __restrict__ ents, long in_rs, long out_rs, Tc alpha) {
  static_assert(kWmapChunk == 4 * kThreads, "one vector of four elements per thread");
  __shared__ Tc sW[MAXK * MAXK];
  __shared__ long sInOff[MAXK], sOutOff[MAXK];
  __shared__ int sInW[MAXK], sOutW[MAXK];
  const WmapTask tk = tasks[ctask[blockIdx.x]];
  const int nin = tk.nin, nout = tk.nout;
  for (int i = threadIdx.x; i < nin; i += blockDim.x) {
    sInOff[i] = ents[tk.idx0 + i].off;
    sInW[i] = ents[tk.idx0 + i].wp;
  }
  for (int i = threadIdx.x; i < nout; i += blockDim.x) {
    sOutOff[i] = ents[tk.idx0 + nin + i].off;
    sOutW[i] = ents[tk.idx0 + nin + i].wp;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nout * MAXK; i += blockDim.x) {
    const int o = i / MAXK, k = i - o * MAXK;
    sW[i] = (k < nin) ? alpha * Wg[sInW[k] + sOutW[o]] : Tc(0);
  }
  __syncthreads();
  const long e = (long)((int)blockIdx.x - tk.chunk0) * kWmapChunk + 4L * threadIdx.x;
  if (e >= (long)tk.di * tk.dj) return;
  const long a = tk.i_off + e / tk.dj, y = tk.j_off + e % tk.dj;
  const Tin* src = in + a * in_rs + y;
  Tout* dst = out + a * out_rs + y;
  if (nin == 0) {
    Vec4<Tout> z;
#pragma unroll
    for (int j = 0; j < 4; ++j) z.v[j] = Cvt<Tout>::st(Tc(0));
    for (int o = 0; o < nout; ++o) *reinterpret_cast<Vec4<Tout>*>(dst + sOutOff[o]) = z;
    return;
  }
  Tc v[MAXK][4];
#pragma unroll
  for (int k = 0; k < MAXK; ++k) {
    if (k < nin) {
      const Vec4<Tin> q = *reinterpret_cast<const Vec4<Tin>*>(src + sInOff[k]);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[k][j] = (Tc)Cvt<Tin>::ld(q.v[j]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[k][j] = Tc(0);
    }
  }
  for (int o = 0; o < nout; ++o) {
    Tc acc[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < MAXK; ++k) {
      const Tc wk = sW[o * MAXK + k];
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] += wk * v[k][j];
    }
    Vec4<Tout> r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r.v[j] = Cvt<Tout>::st(acc[j]);
    *reinterpret_cast<Vec4<Tout>*>(dst + sOutOff[o]) = r;
  }
}

template <typename Tin, typename Tout, typename Tc>
void wmap_blocks_t(Ctx* c, const void* in, const void* W, void* out, const WmapPlan& w, double alpha) {
  dim3 grid((unsigned)w.chunks), block(kThreads);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, 0, c->stream, (const Tin*)in, (const Tc*)W, (Tout*)out, w.d_tasks,
                       w.d_ctask, w.d_ents, w.in_rs, w.out_rs, (Tc)alpha);
  };
  // the vector form: 4-byte (or smaller) elements, vector-aligned buffers
  if constexpr (sizeof(Tin) <= 4 && sizeof(Tout) <= 4) {
    const bool v4 = w.vec4 && w.maxk <= 24 && (reinterpret_cast<uintptr_t>(in) % (4 * sizeof(Tin)) == 0) &&
                    (reinterpret_cast<uintptr_t>(out) % (4 * sizeof(Tout)) == 0);
    if (v4) {
      if (w.maxk <= 8) go(wmap_blocks_vec4_kernel<Tin, Tout, Tc, 8>);
      else if (w.maxk <= 16) go(wmap_blocks_vec4_kernel<Tin, Tout, Tc, 16>);
      else go(wmap_blocks_vec4_kernel<Tin, Tout, Tc, 24>);
      D3S_HIP(hipGetLastError());
      return;
    }
  }
  if (w.maxk <= 8) go(wmap_blocks_kernel<Tin, Tout, Tc, 8>);
  else if (w.maxk <= 16) go(wmap_blocks_kernel<Tin, Tout, Tc, 16>);
  else if (w.maxk <= 24) go(wmap_blocks_kernel<Tin, Tout, Tc, 24>);
  else if (w.maxk <= 32) go(wmap_blocks_kernel<Tin, Tout, Tc, 32>);
  else if (w.maxk <= 48) go(wmap_blocks_kernel<Tin, Tout, Tc, 48>);
  else if (w.maxk <= 80) go(wmap_blocks_kernel<Tin, Tout, Tc, 80>);
  else throw Error{D3S_EINVAL, "block W-map: more than 80 channel pairs"};
  D3S_HIP(hipGetLastError());
}

// ---------------------------------------------------------------- reductions
__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += sh[w];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(kThreads)
void dot_partial_kernel(const double* __restrict__ x, const double* __restrict__ y, long n,
                        double* __restrict__ part) {
  __shared__ double sh[kThreads / 64];
  double acc = 0.0;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    acc += x[i] * y[i];
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Sums over a wave of R running sums per lane at once: at every step a lane
// hands half of its rows to its partner and adds the partner's half of the
// others, so R rows take R - 1 exchanges (+ one per further step) instead of
// 6 R.  Returns the total of row `lane / (64 / P)`, P the power of two >= R;
// the order of the additions is fixed.
template <int R> constexpr int pow2_rows() { return R <= 8 ? 8 : R <= 16 ? 16 : R <= 32 ? 32 : 64; }
template <int R>
__device__ __forceinline__ double wave_row_sums(const double* acc) {
  constexpr int P = pow2_rows<R>();
  const int lane = threadIdx.x & 63;
  double v[P];
#pragma unroll
  for (int j = 0; j < P; ++j) v[j] = j < R ? acc[j] : 0.0;
#pragma unroll
  for (int h = P / 2, off = 32; off > 0; h /= 2, off /= 2) {
    if (h > 0) {
      const bool up = (lane & off) != 0;
#pragma unroll
      for (int j = 0; j < h; ++j) {
        double a = v[j], b = v[j + h];
        // else the choice becomes an index, and that a chain of P choices
        asm volatile("" : "+v"(a), "+v"(b));
        const double mine = up ? b : a, give = up ? a : b;
        v[j] = mine + __shfl_xor(give, off, 64);
      }
    } else {
      v[0] += __shfl_xor(v[0], off, 64);
    }
  }
  return v[0];
}

// sc[j] = -(the coefficient of row j), zero for rows <= j < 4 RW: read from
// coef, or (cpart given) summed here from the nbp partial sums of every row,
// by every workgroup in the same order, the first one storing them to coef.
// A wave takes the rows wave, wave + 4, ... and has all their partial sums in
// flight at once.  Ends with a barrier.
template <int RW>
__device__ __forceinline__ void load_coefs(double* sc, int rows, double* coef, const double* __restrict__ cpart,
                                           int nbp) {
  if (cpart && nbp <= 16) {
    // short rows: four lanes a row
    const int q = threadIdx.x & 3, j = threadIdx.x >> 2;
    if (j < 4 * RW) {
      const double* p = cpart + (long)min(j, rows - 1) * nbp;
      double u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) u[i] = (q + 4 * i < nbp) ? p[q + 4 * i] : 0.0;
      double t = (u[0] + u[1]) + (u[2] + u[3]);
      t += __shfl_xor(t, 1, 64);
      t += __shfl_xor(t, 2, 64);
      if (q == 0) {
        sc[j] = (j < rows) ? -t : 0.0;
        if (blockIdx.x == 0 && j < rows) coef[j] = t;
      }
    }
  } else if (cpart) {
    constexpr int W = 64 / pow2_rows<RW>();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double acc[RW];
#pragma unroll
    for (int j = 0; j < RW; ++j) {
      const double* p = cpart + (long)min(wave + 4 * j, rows - 1) * nbp;
      double t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = (lane + 64 * u < nbp) ? p[lane + 64 * u] : 0.0;
      acc[j] = (t[0] + t[1]) + (t[2] + t[3]);
    }
    const double t = wave_row_sums<RW>(acc);
    const int r = wave + 4 * (lane / W);
    if (lane % W == 0 && lane / W < RW) {
      sc[r] = (r < rows) ? -t : 0.0;
      if (blockIdx.x == 0 && r < rows) coef[r] = t;
    }
  } else {
    for (int j = threadIdx.x; j < 4 * RW; j += blockDim.x) sc[j] = (j < rows) ? -coef[j] : 0.0;
  }
  __syncthreads();
}

// One pass of Gram-Schmidt over at most 64 rows of V, kGsChunk elements of
// every row per workgroup and turn:
//   MODE 0: the partial sums of <V_j, w>
//   MODE 1: w <- w + sum_j sc_j V_j (sc = -coefficients) and the partial sums
//           of <V_j, w_new>
//   MODE 2: the same update and the partial sum of |w_new|^2
// The rows are dealt to the four waves; a wave holds its (at most 16) rows of
// the chunk in registers, four consecutive elements a lane, so V is read once
// in 16-byte loads that are all in flight together, and the update's four
// shares meet in LDS.  The row count may be read from device memory, so the
// kernel branches once, uniformly, to a body compiled for the rows a wave has
// (rows past the last one are clamped to it and weighted by zero).  Bound by
// the latency of one turn for short vectors and by L2 / HBM for long ones.
// Measured, MODE 0 / 1 / 2, about 20 rows: n = 61440 4.2 / 6.7 / 5.8 us (a
// thread per element with all rows in every wave, 64 workgroups: 15 / 12 / 8.5
// us and two launches of 4 us for the sums; since then 4.1 / 5.2 / 4.8 us),
// n = 2048 3.5 / 4.3 / 3.4 us (8.2 / 8.2 / 4.4 us and the two launches).
constexpr int kGsChunk = kThreads;
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

template <int MODE, int RW>
__device__ __forceinline__ void gs_pass_rows(const double* __restrict__ V, long ldv, int rows, const double* sc,
                                             double (*sx)[kGsChunk], double* __restrict__ w, long n,
                                             double* __restrict__ part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double acc[RW];
#pragma unroll
  for (int j = 0; j < RW; ++j) acc[j] = 0.0;
  const long chunks = (n + kGsChunk - 1) / kGsChunk;
  for (long ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
    const long i0 = ch * kGsChunk + lane * 4;
    const bool whole = (ch + 1) * kGsChunk <= n;
    auto load4 = [&](const double* p, double (&v)[4]) {
      if (whole) {
        const d2u a = *reinterpret_cast<const d2u*>(p + i0), b = *reinterpret_cast<const d2u*>(p + i0 + 2);
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (i0 + e < n) ? p[i0 + e] : 0.0;
      }
    };
    double x[4], v[RW][4];
    load4(w, x);
#pragma unroll
    for (int j = 0; j < RW; ++j) load4(V + (long)min(wave + 4 * j, rows - 1) * ldv, v[j]);
    if constexpr (MODE > 0) {
      double u[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int j = 0; j < RW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] += sc[wave + 4 * j] * v[j][e];
      __syncthreads();                   // the previous turn's shares have been read
#pragma unroll
      for (int e = 0; e < 4; ++e) sx[wave][lane * 4 + e] = u[e];
      __syncthreads();                   // ... and every wave has loaded w
#pragma unroll
      for (int e = 0; e < 4; ++e)
        x[e] += (sx[0][lane * 4 + e] + sx[1][lane * 4 + e]) + (sx[2][lane * 4 + e] + sx[3][lane * 4 + e]);
      if (wave == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i0 + e < n) w[i0 + e] = x[e];
      }
    }
    if constexpr (MODE < 2) {
#pragma unroll
      for (int j = 0; j < RW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j] += v[j][e] * x[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[0] += x[e] * x[e];
    }
  }
  if constexpr (MODE < 2) {
    constexpr int W = 64 / pow2_rows<RW>();
    const double t = wave_row_sums<RW>(acc);
    const int r = wave + 4 * (lane / W);
    if (lane % W == 0 && lane / W < RW && r < rows) part[(long)r * gridDim.x + blockIdx.x] = t;
  } else {
    double t = acc[0];
    for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
  }
}

template <int MODE>
__global__ __launch_bounds__(kThreads, 2)
void gs_pass_kernel(const double* __restrict__ V, long ldv, int k, const int* __restrict__ kdev,
                    double* __restrict__ coef, const double* __restrict__ cpart, int nbp, double* __restrict__ w,
                    long n, double* __restrict__ part, int* __restrict__ knext) {
  __shared__ double sc[64];
  __shared__ double sx[4][kGsChunk];
  const int rows = kdev ? (*kdev + 1) : k;
  // the next step's index: nothing in this step reads it
  if (knext && blockIdx.x == 0 && threadIdx.x == 0) *knext = rows;
  auto go = [&](auto rt) {
    constexpr int RW = decltype(rt)::value;
    if constexpr (MODE > 0) load_coefs<RW>(sc, rows, coef, cpart, nbp);
    gs_pass_rows<MODE, RW>(V, ldv, rows, sc, sx, w, n, part);
  };
  switch ((rows + 7) / 8) {
    case 1: go(std::integral_constant<int, 2>()); break;
    case 2: go(std::integral_constant<int, 4>()); break;
    case 3: go(std::integral_constant<int, 6>()); break;
    case 4: go(std::integral_constant<int, 8>()); break;
    case 5: go(std::integral_constant<int, 10>()); break;
    case 6: go(std::integral_constant<int, 12>()); break;
    case 7: go(std::integral_constant<int, 14>()); break;
    default: go(std::integral_constant<int, 16>()); break;
  }
}

// End of a Lanczos step k (k from the host, or *kdev): V_{k+1} = w / beta
// with beta = sqrt(|w|^2) (zero when beta is not positive; skipped when
// k+1 = kk), and ab[2k] = alpha_k (the projections of both Gram-Schmidt
// passes on V_k), ab[2k+1] = beta (ab may be pinned host memory).
__global__ __launch_bounds__(kThreads)
void lanczos_tail_kernel(const double* __restrict__ w, long n, const double* __restrict__ npart, int nnp,
                         const double* __restrict__ c1, const double* __restrict__ c2, int k,
                         const int* __restrict__ kdev, int kk, double* __restrict__ V, double* __restrict__ ab) {
  if (kdev) k = *kdev;
  // |w|^2 from the per-block partials, summed in a fixed order by every block
  __shared__ double sb;
  __shared__ double sh[kThreads / 64];
  double part = 0.0;
  for (int q = threadIdx.x; q < nnp; q += blockDim.x) part += npart[q];
  const double tot = block_sum(part, sh);
  if (threadIdx.x == 0) sb = tot;
  __syncthreads();
  const double b = sqrt(fmax(sb, 0.0));
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ab[2 * k] = c1[k] + c2[k];
    ab[2 * k + 1] = b;
  }
  if (k + 1 >= kk) return;
  double* vnext = V + (long)(k + 1) * n;
  const double f = (b > 0.0) ? 1.0 / b : 0.0;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    vnext[i] = w[i] * f;
}

// Gram-Schmidt twice and the end of a Lanczos step, as the passes and the tail
// above, for short vectors and few rows: one workgroup keeps V, E elements of
// up to KR rows a thread, in registers from the first sums to the last update.
// Bound by the load of V through one compute unit (64 bytes a clock) and the
// latency of the three sums; it saves three launches.  Up to 8 / 16 / 24 / 48
// rows it takes 3.8 / 5.3 / 7.2 / 12.3 us for n <= 1024 and 4.8 / 7.0 / 9.4 us
// for n <= 2048, where the four launches take 13 to 15 us and their gaps.
constexpr int kOrthoThreads = 512;

template <int E, int KR>
__global__ __launch_bounds__(kOrthoThreads)
void lanczos_ortho_kernel(double* __restrict__ V, long n, int k, int kk, const double* __restrict__ w,
                          double* __restrict__ ab) {
  constexpr int NW = kOrthoThreads / 64;
  static_assert(KR % 8 == 0, "rows are summed eight at a time");
  __shared__ double sp[NW][KR], sc[KR], sn[NW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rows = k + 1;
  auto at = [&](int q) { return 2L * (threadIdx.x + kOrthoThreads * q); };     // pair q of the thread
  // no branches: every load is a pair within the row.  An odd row's last
  // element is the second of a pair whose first belongs to another thread; x is
  // zero where the thread has no element, V whatever was loaded
  auto load = [&](const double* p, double (&v)[E]) {
#pragma unroll
    for (int q = 0; q < E / 2; ++q) {
      const d2u a = *reinterpret_cast<const d2u*>(p + min(at(q), n - 2));
      v[2 * q] = a.x;
      v[2 * q + 1] = a.y;
    }
  };
  double x[E], v[KR][E];
  auto cut = [&]() {
#pragma unroll
    for (int q = 0; q < E / 2; ++q) {
      x[2 * q] = at(q) < n - 1 ? x[2 * q] : 0.0;
      x[2 * q + 1] = at(q) < n ? x[2 * q + 1] : 0.0;
    }
  };
  load(w, x);
#pragma unroll
  for (int j = 0; j < KR; ++j) load(V + (long)min(j, rows - 1) * n, v[j]);
  cut();
  double alpha = 0.0;
  auto sums = [&](auto gt) {             // rows 8 g .. 8 g + 7
    constexpr int g = 8 * decltype(gt)::value;
    if constexpr (g < KR) {
      double acc[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        acc[j] = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[j] += v[g + j][e] * x[e];
      }
      const double t = wave_row_sums<8>(acc);
      if (lane % 8 == 0) sp[wave][g + lane / 8] = t;
    }
  };
  auto pass = [&]() {
    static_assert(KR <= 48, "six groups of rows");
    sums(std::integral_constant<int, 0>());
    sums(std::integral_constant<int, 1>());
    sums(std::integral_constant<int, 2>());
    sums(std::integral_constant<int, 3>());
    sums(std::integral_constant<int, 4>());
    sums(std::integral_constant<int, 5>());
    __syncthreads();
    if (threadIdx.x < KR) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < NW; ++q) s += sp[q][threadIdx.x];
      sc[threadIdx.x] = (int)threadIdx.x < rows ? s : 0.0;     // the rows past the last are copies of it
    }
    __syncthreads();
    alpha += sc[k];
#pragma unroll
    for (int j = 0; j < KR; ++j) {
      const double c = sc[j];
#pragma unroll
      for (int e = 0; e < E; ++e) x[e] -= c * v[j][e];
    }
    cut();
  };
  pass();
  pass();
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < E; ++e) s += x[e] * x[e];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) sn[wave] = s;
  __syncthreads();
  s = 0.0;
#pragma unroll
  for (int q = 0; q < NW; ++q) s += sn[q];
  const double b = sqrt(fmax(s, 0.0));
  if (threadIdx.x == 0) {
    ab[2 * k] = alpha;
    ab[2 * k + 1] = b;
  }
  if (rows >= kk) return;
  double* vnext = V + (long)rows * n;
  const double f = (b > 0.0) ? 1.0 / b : 0.0;
#pragma unroll
  for (int q = 0; q < E / 2; ++q) {
    const long i = at(q), ic = min(i, n - 2);
    if (i < n - 1) vnext[ic] = x[2 * q] * f;
    if (i < n) vnext[ic + 1] = x[2 * q + 1] * f;
  }
}

// dst = V_k and *kcur = k, k = *knext
__global__ __launch_bounds__(kThreads)
void copy_row_kernel(const double* __restrict__ V, long n, const int* __restrict__ knext, int* __restrict__ kcur,
                     double* __restrict__ dst) {
  const int k = *knext;
  if (blockIdx.x == 0 && threadIdx.x == 0) *kcur = k;
  const double* src = V + (long)k * n;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

__global__ void set_int_kernel(int* p, int v) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *p = v;
}

// out[j] = sum_b part[j * nb + b] in a fixed order; one block per j
__global__ __launch_bounds__(kThreads)
void reduce_rows_kernel(const double* __restrict__ part, int nb, double* __restrict__ out,
                        const int* __restrict__ kdev) {
  __shared__ double sh[kThreads / 64];
  const int j = blockIdx.x;
  if (kdev && j >= *kdev + 1) return;
  double acc = 0.0;
  for (int b = threadIdx.x; b < nb; b += blockDim.x) acc += part[(long)j * nb + b];
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) out[j] = s;
}

__global__ __launch_bounds__(kThreads)
void maxpy_kernel(const double* __restrict__ V, long ldv, int k, const int* __restrict__ kdev,
                  const double* __restrict__ coef, double sign, double* __restrict__ w, long n, int accumulate) {
  __shared__ double sc[128];
  if (kdev) k = *kdev + 1;
  for (int j = threadIdx.x; j < k; j += blockDim.x) sc[j] = sign * coef[j];
  __syncthreads();
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    double acc = accumulate ? w[i] : 0.0;
    for (int j = 0; j < k; ++j) acc += sc[j] * V[(long)j * ldv + i];
    w[i] = acc;
  }
}

__global__ void scale_kernel(double* __restrict__ x, long n, double s) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    x[i] *= s;
}

__global__ void scale_dev_kernel(double* __restrict__ x, long n, const double* __restrict__ s, int recip_sqrt) {
  const double f = recip_sqrt ? 1.0 / sqrt(*s) : *s;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    x[i] *= f;
}

// y = a x + b y; with b = 0 the old y is not read (it may hold anything,
// including NaN bit patterns of fresh workspace)
__global__ void axpby_kernel(double a, const double* __restrict__ x, double b, double* __restrict__ y, long n) {
  if (b == 0.0) {
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
      y[i] = a * x[i];
    return;
  }
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = a * x[i] + b * y[i];
}

__global__ void fill_kernel(double* __restrict__ x, long n, double v) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    x[i] = v;
}

__global__ void zero_kernel(uint4* __restrict__ x, long n16, unsigned char* __restrict__ tail, int ntail) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (long)gridDim.x * blockDim.x)
    x[i] = uint4{0, 0, 0, 0};
  if (blockIdx.x == 0 && (int)threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

// one workgroup per descriptor: a strided rows x cols block copy
__global__ void copy_desc_kernel(const double* __restrict__ src, double* __restrict__ dst,
                                 const CopyDesc* __restrict__ desc) {
  const CopyDesc dd = desc[blockIdx.x];
  const long total = (long)dd.rows * dd.cols;
  for (long i = threadIdx.x; i < total; i += blockDim.x) {
    const long r = i / dd.cols, c = i - r * dd.cols;
    dst[dd.dst_off + r * dd.dst_rs + c * dd.dst_cs] = src[dd.src_off + r * dd.src_rs + c * dd.src_cs];
  }
}

// M[a,s,b] = 0 unless key(q_a) + key(q_s) = key(q_b) (linear charge keys)
__global__ void mask_site_kernel(double* __restrict__ M, int ml, int d, int mr, const int* __restrict__ ka,
                                 const int* __restrict__ ks, const int* __restrict__ kb) {
  const long total = (long)ml * d * mr;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
    const long b = i % mr;
    const long as = i / mr;
    const int s = (int)(as % d), a = (int)(as / d);
    if (ka[a] + ks[s] != kb[b]) M[i] = 0.0;
  }
}

template <typename T>
__global__ void transpose_kernel(const T* __restrict__ in, long R, long C, T* __restrict__ out) {
  __shared__ T tile[32][33];
  const long r0 = (long)blockIdx.y * 32, c0 = (long)blockIdx.x * 32;
  for (int i = threadIdx.y; i < 32; i += blockDim.y) {
    const long r = r0 + i, cc = c0 + threadIdx.x;
    if (r < R && cc < C) tile[i][threadIdx.x] = in[r * C + cc];
  }
  __syncthreads();
  for (int i = threadIdx.y; i < 32; i += blockDim.y) {
    const long cc = c0 + i, r = r0 + threadIdx.x;
    if (r < R && cc < C) out[cc * R + r] = tile[threadIdx.x][i];
  }
}

// 2-byte elements in even rows and columns: 64 x 64 elements a workgroup, moved
// as pairs, so that a row of the tile is 128 bytes in both directions.  2048 x
// 8192: 20 us (35 us with 2-byte accesses and 64-byte rows).
__global__ __launch_bounds__(256)
void transpose_pairs_kernel(const unsigned short* __restrict__ in, long R, long C, unsigned short* __restrict__ out) {
  __shared__ unsigned tile[64][33];
  const long r0 = (long)blockIdx.y * 64, c0 = (long)blockIdx.x * 64;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
#pragma unroll
  for (int i = 0; i < 64; i += 8) {
    const long r = r0 + y + i, c = c0 + 2 * x;
    if (r < R && c < C) tile[y + i][x] = *reinterpret_cast<const unsigned*>(in + r * C + c);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 64; i += 8) {
    const int cl = y + i, sh = 16 * (cl & 1);
    const long c = c0 + cl, r = r0 + 2 * x;
    const unsigned lo = (tile[2 * x][cl >> 1] >> sh) & 0xffffu, hi = (tile[2 * x + 1][cl >> 1] >> sh) & 0xffffu;
    if (r < R && c < C) *reinterpret_cast<unsigned*>(out + c * R + r) = lo | (hi << 16);
  }
}

template <typename Tin, typename Tout>
__device__ __forceinline__ Tout rl_convert(Tin v) {
  if constexpr (std::is_same<Tin, Tout>::value) return v;
  else if constexpr (std::is_same<Tout, bf16_t>::value) return f32_to_bf16((float)v);
  else return (Tout)v;
}

// One destination tile of at most 32 x 32 per workgroup (32 x 8 threads, rows
// along x).  A thread's four rows are loaded, at clamped addresses, before any
// is stored: one after the other they wait for each load in turn.
// The input is the sum of `parts` FP32 products of n elements each, added up in
// the order of sum_partials_kernel (parts 1: a plain copy), so that partial
// products need no launch that reads them all and writes their sum to be read
// again here.  Site of 3000 x 2900 states, BF16: psi in 9.2 -> 8.3 us, two
// partial products out 17.5 us and a gap -> 13.4 us.
template <typename Tin, typename Tout>
__global__ __launch_bounds__(256)
void relayout_tiles_kernel(const Tin* __restrict__ in, int parts, long n, Tout* __restrict__ out,
                           const RlTile* __restrict__ tiles) {
  const RlTile t = tiles[blockIdx.x];
  const int x = threadIdx.x;
  if (x >= t.pcols) return;
  const bool any = t.rows > 0 && t.cols > 0;
  Tin v[4];
  if (any) {
    const Tin* p = in + t.src + min(x, t.cols - 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = p[(long)min((int)threadIdx.y + 8 * q, t.rows - 1) * t.src_ld];
    if constexpr (std::is_same<Tin, float>::value)
      for (int j = 1; j < parts; ++j) {
        p += n;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] += p[(long)min((int)threadIdx.y + 8 * q, t.rows - 1) * t.src_ld];
      }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = threadIdx.y + 8 * q;
    if (i < t.prows)
      out[t.dst + (long)i * t.dst_ld + x] =
          any && i < t.rows && x < t.cols ? rl_convert<Tin, Tout>(v[q]) : rl_convert<float, Tout>(0.0f);
  }
}

// One 32 x 32 tile per workgroup, staged through LDS so that both the
// reads and the writes run along rows.
template <typename T>
__global__ void transpose_tiles_kernel(const T* __restrict__ in, T* __restrict__ out,
                                       const TrTile* __restrict__ tiles) {
  __shared__ T tile[32][33];
  const TrTile t = tiles[blockIdx.x];
  if (t.rows > 0 && t.cols > 0) {
    // entries past the edge repeat the last one; none of them is stored
    const T* p = in + t.src + min((int)threadIdx.x, t.cols - 1);
    T v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = p[(long)min((int)threadIdx.y + 8 * q, t.rows - 1) * t.src_ld];
#pragma unroll
    for (int q = 0; q < 4; ++q) tile[threadIdx.y + 8 * q][threadIdx.x] = v[q];
  }
  __syncthreads();
  for (int i = threadIdx.y; i < t.cols; i += blockDim.y)
    if ((int)threadIdx.x < t.rows) out[t.dst + (long)i * t.dst_ld + threadIdx.x] = tile[threadIdx.x][i];
}

__global__ void copy2d_kernel(const double* __restrict__ src, long lds, double* __restrict__ dst, long ldd,
                              long rows, long cols) {
  const long total = rows * cols;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
    const long r = i / cols, cc = i - r * cols;
    dst[r * ldd + cc] = src[r * lds + cc];
  }
}

template <typename Tout>
__global__ void cast_kernel(const double* __restrict__ x, Tout* __restrict__ y, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    if constexpr (sizeof(Tout) == 2) y[i] = f32_to_bf16((float)x[i]);
    else y[i] = (Tout)x[i];
  }
}

__global__ void cast_f32_f64_kernel(const float* __restrict__ x, double* __restrict__ y, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = (double)x[i];
}

// Wbar[w, v, s, t] = sum_a part[a][(w,t)][(s,v)], fixed order over a: 32 threads
// share an entry, 16 neighbouring entries a workgroup (a thread per entry left
// the chip idle: 73 us for the 300 terms of 576 entries, now 5 us).
constexpr int kAdjCols = 16, kAdjParts = 32;
__global__ __launch_bounds__(kAdjCols * kAdjParts)
void adjoint_sum_kernel(const double* __restrict__ part, int ml, int d, int wl, int wr,
                                   double* __restrict__ Wbar) {
  __shared__ double red[kAdjParts][kAdjCols];
  const int n1 = wl * d, n2 = d * wr;
  const int col = threadIdx.x % kAdjCols, grp = threadIdx.x / kAdjCols;
  const int idx = blockIdx.x * kAdjCols + col, at = min(idx, n1 * n2 - 1);
  double acc = 0.0;
#pragma unroll 4
  for (int a = grp; a < ml; a += kAdjParts) acc += part[(long)a * n1 * n2 + at];
  red[grp][col] = acc;
  __syncthreads();
  if (grp != 0 || idx >= n1 * n2) return;
#pragma unroll
  for (int i = 1; i < kAdjParts; ++i) acc += red[i][col];
  const int r = idx / n2, cc = idx - r * n2;     // r = (w,t), cc = (s,v)
  const int w = r / d, t = r - w * d;
  const int s = cc / wr, v = cc - s * wr;
  Wbar[((w * wr + v) * d + s) * d + t] = acc;
}

inline int grid_for(long n) {
  long g = (n + kThreads - 1) / kThreads;
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

void wmap_l2r(Ctx* c, d3s_prec p, const void* T1, const void* W, void* out, long ld_out, int ml,
              int d, int mr, int wl, int wr, double alpha) {
  if (p == D3S_F64) wmap_l2r_t<double, double, double>(c, T1, W, out, ld_out, ml, d, mr, wl, wr, alpha);
  else if (p == D3S_F32) wmap_l2r_t<float, float, float>(c, T1, W, out, ld_out, ml, d, mr, wl, wr, alpha);
  else wmap_l2r_t<float, bf16_t, float>(c, T1, W, out, ld_out, ml, d, mr, wl, wr, alpha);
}

void wmap_r2l(Ctx* c, d3s_prec p, const void* Y, const void* W, void* Z, int ml, int d, int mr,
              int wl, int wr, double alpha) {
  if (p == D3S_F64) wmap_r2l_t<double, double, double>(c, Y, W, Z, ml, d, mr, wl, wr, alpha);
  else if (p == D3S_F32) wmap_r2l_t<float, float, float>(c, Y, W, Z, ml, d, mr, wl, wr, alpha);
  else wmap_r2l_t<float, bf16_t, float>(c, Y, W, Z, ml, d, mr, wl, wr, alpha);
}

void wmap_blocks(Ctx* c, d3s_prec p, const void* in, const void* W, void* out, const WmapPlan& w, double alpha) {
  if (w.tasks.empty() || w.chunks <= 0) return;
  if (p == D3S_F64) wmap_blocks_t<double, double, double>(c, in, W, out, w, alpha);
  else if (p == D3S_F32) wmap_blocks_t<float, float, float>(c, in, W, out, w, alpha);
  else wmap_blocks_t<float, bf16_t, float>(c, in, W, out, w, alpha);
}

void dot_f64(Ctx* c, const double* x, const double* y, long n, double* out_dev) {
  double* part = (double*)ws_get(c, WS_RED, sizeof(double) * kRedBlocks);
  hipLaunchKernelGGL(dot_partial_kernel, dim3(kRedBlocks), dim3(kThreads), 0, c->stream, x, y, n, part);
  hipLaunchKernelGGL(reduce_rows_kernel, dim3(1), dim3(kThreads), 0, c->stream, part, kRedBlocks, out_dev,
                     (const int*)nullptr);
  D3S_HIP(hipGetLastError());
}

void mdot_f64(Ctx* c, const double* V, long ldv, int k, const double* w, long n, double* coef_dev) {
  if (k <= 0) return;
  if (k > 128) throw Error{D3S_EINVAL, "mdot: more than 128 vectors"};
  // partial count fixed by n (deterministic), at most kGsMaxBlocks
  const int nb = gs_blocks(n);
  double* part = (double*)ws_get(c, WS_RED, sizeof(double) * (size_t)nb * 128);
  for (int j0 = 0; j0 < k; j0 += 64)
    hipLaunchKernelGGL(gs_pass_kernel<0>, dim3(nb), dim3(kThreads), 0, c->stream, V + (long)j0 * ldv, ldv,
                       std::min(64, k - j0), (const int*)nullptr, (double*)nullptr, (const double*)nullptr, 0,
                       const_cast<double*>(w), n, part + (size_t)j0 * nb, (int*)nullptr);
  hipLaunchKernelGGL(reduce_rows_kernel, dim3(k), dim3(kThreads), 0, c->stream, part, nb, coef_dev,
                     (const int*)nullptr);
  D3S_HIP(hipGetLastError());
}

int gs_blocks(long n) {
  return (int)std::max<long>(1, std::min<long>(kGsMaxBlocks, (n + kGsChunk - 1) / kGsChunk));
}

void gram_schmidt(Ctx* c, const double* V, long ldv, int k, const int* kdev, double* w, long n, double* coef1,
                  double* coef2, double* npart, int* knext) {
  if (k <= 0) return;
  if (k > 64) throw Error{D3S_EINVAL, "Gram-Schmidt: more than 64 vectors in the fused pass"};
  const int nb = gs_blocks(n);
  // Up to kGsFused partial sums a row every workgroup of the next pass adds
  // them up itself, which costs it a few loads per thread; beyond, a launch
  // between the passes does (about 4 us)
  const bool fused = nb <= kGsFused;
  double* p1 = (double*)ws_get(c, WS_RED, sizeof(double) * (size_t)nb * 128);
  double* p2 = p1 + (size_t)nb * 64;
  const dim3 grid(nb), block(kThreads);
  auto pass = [&](auto kern, double* coef, const double* cpart, double* part, int* kn) {
    hipLaunchKernelGGL(kern, grid, block, 0, c->stream, V, ldv, k, kdev, coef, fused ? cpart : (const double*)nullptr,
                       nb, w, n, part, kn);
  };
  auto sums = [&](const double* part, double* coef) {
    if (!fused) hipLaunchKernelGGL(reduce_rows_kernel, dim3(k), block, 0, c->stream, part, nb, coef, kdev);
  };
  pass(gs_pass_kernel<0>, nullptr, nullptr, p1, nullptr);
  sums(p1, coef1);
  pass(gs_pass_kernel<1>, coef1, p1, p2, nullptr);
  sums(p2, coef2);
  pass(gs_pass_kernel<2>, coef2, p2, npart, knext);
  D3S_HIP(hipGetLastError());
}

void lanczos_tail(Ctx* c, const double* w, long n, const double* npart, const double* c1, const double* c2, int k,
                  const int* kdev, int kk, double* V, double* ab) {
  hipLaunchKernelGGL(lanczos_tail_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, w, n, npart,
                     gs_blocks(n), c1, c2, k, kdev, kk, V, ab);
  D3S_HIP(hipGetLastError());
}

bool lanczos_ortho(Ctx* c, double* V, long n, int k, int kk, const double* w, double* ab) {
  auto go = [&](auto e, auto kr) {
    hipLaunchKernelGGL((lanczos_ortho_kernel<decltype(e)::value, decltype(kr)::value>), dim3(1), dim3(kOrthoThreads), 0,
                       c->stream, V, n, k, kk, w, ab);
    D3S_HIP(hipGetLastError());
    return true;
  };
  using E2 = std::integral_constant<int, 2>;
  using E4 = std::integral_constant<int, 4>;
  using E8 = std::integral_constant<int, 8>;
  using K8 = std::integral_constant<int, 8>;
  using K16 = std::integral_constant<int, 16>;
  using K24 = std::integral_constant<int, 24>;
  using K48 = std::integral_constant<int, 48>;
  const int rows = k + 1;
  if (n < 2) return false;
  if (n <= 2 * kOrthoThreads) {
    if (rows <= 8) return go(E2(), K8());
    if (rows <= 16) return go(E2(), K16());
    if (rows <= 24) return go(E2(), K24());
    if (rows <= 48) return go(E2(), K48());
  } else if (n <= 4 * kOrthoThreads) {
    if (rows <= 8) return go(E4(), K8());
    if (rows <= 16) return go(E4(), K16());
    if (rows <= 24) return go(E4(), K24());
  } else if (n <= 8 * kOrthoThreads) {
    if (rows <= 8) return go(E8(), K8());
  }
  return false;
}

void copy_row_f64(Ctx* c, const double* V, long n, const int* knext, int* kcur, double* dst) {
  hipLaunchKernelGGL(copy_row_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, V, n, knext, kcur, dst);
  D3S_HIP(hipGetLastError());
}

void set_int_dev(Ctx* c, int* p, int v) {
  hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(64), 0, c->stream, p, v);
  D3S_HIP(hipGetLastError());
}

void maxpy_f64(Ctx* c, const double* V, long ldv, int k, const double* coef_dev, double sign, double* w,
               long n, const int* kdev, bool accumulate) {
  if (k <= 0) return;
  if (k > 128) throw Error{D3S_EINVAL, "maxpy: more than 128 vectors"};
  hipLaunchKernelGGL(maxpy_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, V, ldv, k, kdev, coef_dev,
                     sign, w, n, accumulate ? 1 : 0);
  D3S_HIP(hipGetLastError());
}

void scale_f64(Ctx* c, double* x, long n, double s) {
  hipLaunchKernelGGL(scale_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, x, n, s);
  D3S_HIP(hipGetLastError());
}

void scale_by_dev_f64(Ctx* c, double* x, long n, const double* s_dev, bool reciprocal_sqrt) {
  hipLaunchKernelGGL(scale_dev_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, x, n, s_dev,
                     reciprocal_sqrt ? 1 : 0);
  D3S_HIP(hipGetLastError());
}

void axpby_f64(Ctx* c, double a, const double* x, double b, double* y, long n) {
  hipLaunchKernelGGL(axpby_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, a, x, b, y, n);
  D3S_HIP(hipGetLastError());
}

void copy_f64(Ctx* c, const double* x, double* y, long n) {
  if (n <= 0) return;
  D3S_HIP(hipMemcpyAsync(y, x, sizeof(double) * n, hipMemcpyDeviceToDevice, c->stream));
}

void fill_f64(Ctx* c, double* x, long n, double v) {
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, x, n, v);
  D3S_HIP(hipGetLastError());
}

// Channel-pair MPO of H^2 between bra and ket copies of the state:
// W2[(w,c), (v,u), p, q] = sum_r W[w,v,r,p] W[c,u,r,q].
__global__ __launch_bounds__(kThreads)
void mpo_square_kernel(const double* __restrict__ W, double* __restrict__ W2, int wl, int wr, int d) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n = (long)wl * wl * wr * wr * d * d;
  if (e >= n) return;
  const int q = (int)(e % d);
  long r = e / d;
  const int p = (int)(r % d);
  r /= d;
  const int vu = (int)(r % ((long)wr * wr));
  const int wc = (int)(r / ((long)wr * wr));
  const int v = vu / wr, u = vu % wr, w = wc / wl, cc = wc % wl;
  double acc = 0.0;
  for (int k = 0; k < d; ++k) acc += W[((w * wr + v) * d + k) * d + p] * W[((cc * wr + u) * d + k) * d + q];
  W2[e] = acc;
}

void mpo_square(Ctx* c, const double* W, double* W2, int wl, int wr, int d) {
  const long n = (long)wl * wl * wr * wr * d * d;
  hipLaunchKernelGGL(mpo_square_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     c->stream, W, W2, wl, wr, d);
  D3S_HIP(hipGetLastError());
}

// Metric of the residual's near-side vectors, ordered |S_y> (y < m), then
// H_v|S_y> at m + v*m + y:  G = [[1, E], [E^T, H2]] with E[y', (v,y)] =
// env[y', v, y] and H2[(v,y), (z,x)] = h2[y, v, z, x].
__global__ __launch_bounds__(kThreads)
void residual_metric_kernel(const double* __restrict__ env, const double* __restrict__ h2, int m, int w,
                            double* __restrict__ G) {
  const long n = (long)(1 + w) * m;
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * n) return;
  const long r = e / n, col = e % n;
  double val;
  if (r < m && col < m) {
    val = (r == col) ? 1.0 : 0.0;
  } else if (r < m) {
    val = env[r * w * m + (col - m)];
  } else if (col < m) {
    val = env[col * w * m + (r - m)];
  } else {
    const long rv = r - m, cz = col - m;
    const long v = rv / m, y = rv % m, z = cz / m, x = cz % m;
    val = h2[((y * w + v) * w + z) * m + x];
  }
  G[e] = val;
}

void residual_metric(Ctx* c, const double* env, const double* h2, int m, int w, double* G) {
  const long n = (long)(1 + w) * m;
  hipLaunchKernelGGL(residual_metric_kernel, dim3((unsigned)((n * n + kThreads - 1) / kThreads)), dim3(kThreads),
                     0, c->stream, env, h2, m, w, G);
  D3S_HIP(hipGetLastError());
}

__global__ __launch_bounds__(kThreads)
void scale2d_kernel(double* __restrict__ x, long ld, long rows, long cols, double f) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows * cols) return;
  const long r = e / cols, col = e % cols;
  x[r * ld + col] *= f;
}

void scale2d_f64(Ctx* c, double* x, long ld, long rows, long cols, double f) {
  const long n = rows * cols;
  if (n <= 0) return;
  hipLaunchKernelGGL(scale2d_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     c->stream, x, ld, rows, cols, f);
  D3S_HIP(hipGetLastError());
}

// Enlarged environment of the centre-matrix formalism:
// Lt[(a,s), v, (x,t)] = sum_w L[a,w,x] W[w,v,s,t]; one thread per (a, x) with
// L[a, :, x] in registers and W in LDS.
template <int MAXW>
__global__ __launch_bounds__(kThreads)
void cwf_env_kernel(const double* __restrict__ L, const double* __restrict__ Wg, double* __restrict__ Lt, int ml,
                    int d, int wl, int wr) {
  extern __shared__ double sW[];
  const int nw = wl * wr * d * d;
  for (int i = threadIdx.x; i < nw; i += blockDim.x) sW[i] = Wg[i];
  __syncthreads();
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long)ml * ml) return;
  const int a = (int)(e / ml), x = (int)(e % ml);
  double l[MAXW];
#pragma unroll
  for (int w = 0; w < MAXW; ++w) l[w] = (w < wl) ? L[((long)a * wl + w) * ml + x] : 0.0;
  const long mlp = (long)ml * d;
  for (int sg = 0; sg < d; ++sg)
    for (int v = 0; v < wr; ++v) {
      double* dst = Lt + (((long)a * d + sg) * wr + v) * mlp + (long)x * d;
      for (int t = 0; t < d; ++t) {
        double acc = 0.0;
#pragma unroll
        for (int w = 0; w < MAXW; ++w)
          if (w < wl) acc += l[w] * sW[((w * wr + v) * d + sg) * d + t];
        dst[t] = acc;
      }
    }
}

void cwf_environment(Ctx* c, int ml, int d, int wl, int wr, const double* L, const double* W, double* Lt) {
  const long n = (long)ml * ml;
  const size_t sh = sizeof(double) * (size_t)wl * wr * d * d;
  if (sh > 64 * 1024) throw Error{D3S_EINVAL, "centre-matrix environment: MPO tensor too large for LDS"};
  const dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
  if (wl <= 8)
    hipLaunchKernelGGL(cwf_env_kernel<8>, grid, dim3(kThreads), sh, c->stream, L, W, Lt, ml, d, wl, wr);
  else if (wl <= 32)
    hipLaunchKernelGGL(cwf_env_kernel<32>, grid, dim3(kThreads), sh, c->stream, L, W, Lt, ml, d, wl, wr);
  else
    throw Error{D3S_EINVAL, "centre-matrix environment: w_l > 32"};
  D3S_HIP(hipGetLastError());
}

template <typename T>
__global__ __launch_bounds__(kThreads)
void sum_partials_kernel(const T* __restrict__ part, int parts, long n, T* __restrict__ out) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    T acc = part[i];
    for (int j = 1; j < parts; ++j) acc += part[(long)j * n + i];
    out[i] = acc;
  }
}

void sum_partials(Ctx* c, bool f64, const void* part, int parts, long n, void* out) {
  if (n <= 0) return;
  if (f64)
    hipLaunchKernelGGL(sum_partials_kernel<double>, dim3(grid_for(n)), dim3(kThreads), 0, c->stream,
                       (const double*)part, parts, n, (double*)out);
  else
    hipLaunchKernelGGL(sum_partials_kernel<float>, dim3(grid_for(n)), dim3(kThreads), 0, c->stream,
                       (const float*)part, parts, n, (float*)out);
  D3S_HIP(hipGetLastError());
}

void zero_bytes(Ctx* c, void* x, size_t bytes) {
  if (bytes == 0) return;
  if ((reinterpret_cast<uintptr_t>(x) & 15) != 0) throw Error{D3S_EINVAL, "zero_bytes: buffer not 16-byte aligned"};
  const long n16 = (long)(bytes / 16);
  const int ntail = (int)(bytes - (size_t)n16 * 16);
  hipLaunchKernelGGL(zero_kernel, dim3(grid_for(std::max(n16, 1L))), dim3(kThreads), 0, c->stream, (uint4*)x, n16,
                     (unsigned char*)x + n16 * 16, ntail);
  D3S_HIP(hipGetLastError());
}

void copy_blocks(Ctx* c, const double* src, double* dst, const std::vector<CopyDesc>& desc_in) {
  if (desc_in.empty()) return;
  // one workgroup per descriptor: blocks of more than kPiece elements are
  // cut into row ranges (and long rows into column ranges) first
  constexpr long kPiece = 16384;
  std::vector<CopyDesc> desc;
  desc.reserve(desc_in.size());
  for (const CopyDesc& q : desc_in) {
    if ((long)q.rows * q.cols <= kPiece) {
      desc.push_back(q);
      continue;
    }
    const int cstep = (int)std::min<long>(q.cols, kPiece);
    const int rstep = (int)std::max<long>(1, kPiece / cstep);
    for (int r0 = 0; r0 < q.rows; r0 += rstep)
      for (int c0 = 0; c0 < q.cols; c0 += cstep) {
        CopyDesc p = q;
        p.src_off = q.src_off + (long)r0 * q.src_rs + (long)c0 * q.src_cs;
        p.dst_off = q.dst_off + (long)r0 * q.dst_rs + (long)c0 * q.dst_cs;
        p.rows = std::min(rstep, q.rows - r0);
        p.cols = std::min(cstep, q.cols - c0);
        desc.push_back(p);
      }
  }
  CopyDesc* d = (CopyDesc*)ws_get(c, WS_DESC, sizeof(CopyDesc) * desc.size());
  D3S_HIP(hipMemcpyAsync(d, desc.data(), sizeof(CopyDesc) * desc.size(), hipMemcpyHostToDevice, c->stream));
  hipLaunchKernelGGL(copy_desc_kernel, dim3((unsigned)desc.size()), dim3(kThreads), 0, c->stream, src, dst, d);
  D3S_HIP(hipGetLastError());
  // the descriptor upload reads pageable host memory: wait before it goes away
  D3S_HIP(hipStreamSynchronize(c->stream));
}

void mask_site(Ctx* c, double* M, int ml, int d, int mr, const std::vector<int>& ka, const std::vector<int>& ks,
               const std::vector<int>& kb) {
  std::vector<int> all(ka);
  all.insert(all.end(), ks.begin(), ks.end());
  all.insert(all.end(), kb.begin(), kb.end());
  int* dk = (int*)ws_get(c, WS_DESC, sizeof(int) * all.size());
  D3S_HIP(hipMemcpyAsync(dk, all.data(), sizeof(int) * all.size(), hipMemcpyHostToDevice, c->stream));
  const long n = (long)ml * d * mr;
  hipLaunchKernelGGL(mask_site_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, M, ml, d, mr, dk, dk + ml,
                     dk + ml + d);
  D3S_HIP(hipGetLastError());
  D3S_HIP(hipStreamSynchronize(c->stream));
}

void transpose_f64(Ctx* c, const double* in, long R, long C, double* out) {
  transpose_any(c, 8, in, R, C, out);
}

void transpose_any(Ctx* c, int esz, const void* in, long R, long C, void* out) {
  if (R <= 0 || C <= 0) return;
  if ((R + 31) / 32 > 65535) throw Error{D3S_EINVAL, "transpose: too many rows"};
  dim3 grid((unsigned)((C + 31) / 32), (unsigned)((R + 31) / 32));
  if (esz == 8)
    hipLaunchKernelGGL(transpose_kernel<double>, grid, dim3(32, 8), 0, c->stream, (const double*)in, R, C,
                       (double*)out);
  else if (esz == 4)
    hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(32, 8), 0, c->stream, (const float*)in, R, C,
                       (float*)out);
  else if (R % 2 == 0 && C % 2 == 0 && (reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) % 4 == 0)
    hipLaunchKernelGGL(transpose_pairs_kernel, dim3((unsigned)((C + 63) / 64), (unsigned)((R + 63) / 64)), dim3(256), 0,
                       c->stream, (const unsigned short*)in, R, C, (unsigned short*)out);
  else
    hipLaunchKernelGGL(transpose_kernel<unsigned short>, grid, dim3(32, 8), 0, c->stream,
                       (const unsigned short*)in, R, C, (unsigned short*)out);
  D3S_HIP(hipGetLastError());
}

void transpose_tiles(Ctx* c, int esz, const void* in, void* out, const TrTile* tiles, int ntiles) {
  if (ntiles <= 0) return;
  if (esz == 8)
    hipLaunchKernelGGL(transpose_tiles_kernel<double>, dim3(ntiles), dim3(32, 8), 0, c->stream,
                       (const double*)in, (double*)out, tiles);
  else if (esz == 4)
    hipLaunchKernelGGL(transpose_tiles_kernel<float>, dim3(ntiles), dim3(32, 8), 0, c->stream,
                       (const float*)in, (float*)out, tiles);
  else
    hipLaunchKernelGGL(transpose_tiles_kernel<unsigned short>, dim3(ntiles), dim3(32, 8), 0, c->stream,
                       (const unsigned short*)in, (unsigned short*)out, tiles);
  D3S_HIP(hipGetLastError());
}

void relayout_sum(Ctx* c, const float* part, int parts, long n, double* out, const RlTile* tiles, int ntiles) {
  if (ntiles <= 0) return;
  hipLaunchKernelGGL((relayout_tiles_kernel<float, double>), dim3(ntiles), dim3(32, 8), 0, c->stream, part, parts, n,
                     out, tiles);
  D3S_HIP(hipGetLastError());
}

void relayout_tiles(Ctx* c, int in_kind, int out_kind, const void* in, void* out, const RlTile* tiles,
                    int ntiles) {
  if (ntiles <= 0) return;
  const dim3 g(ntiles), b(32, 8);
  if (in_kind == RL_F64 && out_kind == RL_BF16)
    hipLaunchKernelGGL((relayout_tiles_kernel<double, bf16_t>), g, b, 0, c->stream, (const double*)in, 1, 0L, (bf16_t*)out,
                       tiles);
  else if (in_kind == RL_F64 && out_kind == RL_F32)
    hipLaunchKernelGGL((relayout_tiles_kernel<double, float>), g, b, 0, c->stream, (const double*)in, 1, 0L, (float*)out,
                       tiles);
  else if (in_kind == RL_F32 && out_kind == RL_F64)
    hipLaunchKernelGGL((relayout_tiles_kernel<float, double>), g, b, 0, c->stream, (const float*)in, 1, 0L, (double*)out,
                       tiles);
  else if (in_kind == RL_F32 && out_kind == RL_F32)
    hipLaunchKernelGGL((relayout_tiles_kernel<float, float>), g, b, 0, c->stream, (const float*)in, 1, 0L, (float*)out,
                       tiles);
  else if (in_kind == RL_BF16 && out_kind == RL_BF16)
    hipLaunchKernelGGL((relayout_tiles_kernel<bf16_t, bf16_t>), g, b, 0, c->stream, (const bf16_t*)in, 1, 0L, (bf16_t*)out, tiles);
  else
    throw Error{D3S_EINVAL, "relayout: unsupported element types"};
  D3S_HIP(hipGetLastError());
}

void copy2d_f64(Ctx* c, const double* src, long lds, double* dst, long ldd, long rows, long cols) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(copy2d_kernel, dim3(grid_for(rows * cols)), dim3(kThreads), 0, c->stream, src, lds,
                     dst, ldd, rows, cols);
  D3S_HIP(hipGetLastError());
}

void cast_f64_to_f32(Ctx* c, const double* x, float* y, long n) {
  hipLaunchKernelGGL(cast_kernel<float>, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, x, y, n);
  D3S_HIP(hipGetLastError());
}

void cast_f64_to_bf16(Ctx* c, const double* x, bf16_t* y, long n) {
  hipLaunchKernelGGL(cast_kernel<bf16_t>, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, x, y, n);
  D3S_HIP(hipGetLastError());
}

void cast_f32_to_f64(Ctx* c, const float* x, double* y, long n) {
  hipLaunchKernelGGL(cast_f32_f64_kernel, dim3(grid_for(n)), dim3(kThreads), 0, c->stream, x, y, n);
  D3S_HIP(hipGetLastError());
}

void adjoint_reduce_f64(Ctx* c, const double* T1, const double* U, double* Wbar, int ml, int d, int mr,
                        int wl, int wr) {
  const int n1 = wl * d, n2 = d * wr;
  double* part = (double*)ws_get(c, WS_MISC, sizeof(double) * (size_t)ml * n1 * n2);
  // part[a] = T1[a] (n1 x mr) * U[a]^T (mr x n2), batched over a
  GemmArgs g{n1, n2, mr, T1, mr, true, (long)n1 * mr, U, mr, true, (long)n2 * mr, part, n2,
             (long)n1 * n2, 1.0, 0.0, ml};
  gemm_f64(c, g);
  const int tot = n1 * n2;
  hipLaunchKernelGGL(adjoint_sum_kernel, dim3((tot + kAdjCols - 1) / kAdjCols), dim3(kAdjCols * kAdjParts), 0,
                     c->stream, part, ml, d, wl, wr, Wbar);
  D3S_HIP(hipGetLastError());
}

}  // namespace d3s
