// MFMA contractions of small and medium sizes in FP64 and FP32, and of any
// size whose tiles do not fill the device evenly: every wave owns a tile (or a
// share of its K) and runs its K loop without workgroup barriers.
//
// What bounds a short product is the latency of a load against the few K
// steps of a tile, and the idle compute units of a launch of few large
// workgroups.  An FP64 (FP32) MFMA of 16x16x4 keeps a SIMD busy for 64 (32)
// cycles and needs only 16 (8) bytes per lane, so wave tiles of 32x32, 64x32 and
// 32x64 are fed by L1 and L2 (16-32 bytes per cycle and compute unit), and those of
// 16x16, which read twice as much, serve where the chip would otherwise be idle;
// small tiles give many waves, the K steps of a tile can be shared by the waves of
// a workgroup (summed through LDS in a fixed order), and up to two K steps of each
// wave are in flight in registers.
//
// Fragments: a K step covers 128 bytes of K (16 doubles, 32 floats).  Lane
// group g = lane / 16 holds the two 16-byte pieces [16 g, 16 g + 16) and
// [64 + 16 g, ...) of its row.  Which k a slot of the MFMA holds is the same
// for both operands, which is all the sum needs.
//
// All loads go through a buffer resource based at the tile's first element;
// rows past the operand's edge get an offset outside the resource and read
// as zeros without touching memory.  16-byte buffer loads need 4-byte
// alignment only, so no size or leading dimension takes other instructions; rows
// that start off a 128-byte line cost long sums of large products L2 traffic (see
// gemm_auto's rule).
// The last K step, when it is not whole, is loaded element by element
// (predicated), first of all, so that its latency overlaps the pipeline's
// fill.
//
// Measured (MI355X, one product, against the workgroup-tiled kernel with
// split-K before): M x N x K = 148 x 29 x 174 FP64 5.3 us (12.3 us),
// 1024 x 250 x 1500 20.8 us (28.0 us), 600 x 3600 x 2068 186 us (242-290 us),
// FP32 1402 x 1013 x 8104 208 us (285-415 us).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "mfma_tile.h"

namespace d3s {
namespace {

using namespace tile;

constexpr unsigned kOut = 0x80000000u;   // beyond every resource: reads as zero
constexpr int kFrontRows = 48;           // A-side rows of front_kernel's largest tile

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_at(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, 0x7fffffff, 0x00020000);
}

typedef unsigned u2v __attribute__((ext_vector_type(2)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));

// LDS accesses of one wave run in program order; this keeps the compiler from
// moving a lane's accesses across another lane's
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The fragments of T blocks of 16 outer rows of one operand, for one wave.
// KC: X[o*ld + k], else X[k*ld + o].  A k-contiguous operand is read 128
// bytes of a row by eight lanes, passed through the wave's own LDS rows of
// 144 bytes (conflict-free for the fragment reads) and needs no barrier; the
// other layout's lanes read 16 consecutive outer elements each load, which is
// the fragment itself.
template <typename S, int T, bool KC>
struct Operand {
  static constexpr int SZ = (int)sizeof(S);
  static constexpr int BK = 128 / SZ;
  static constexpr int VE = 16 / SZ;          // elements of a 16-byte piece
  static constexpr int LDK = BK + VE;         // LDS row
  static constexpr int LDS = KC ? T * 16 * LDK : 0;   // LDS elements per wave
  static constexpr int NV = KC ? 2 * T : T;   // offsets per lane
  unsigned vo[NV];
  struct Stage {                              // one K step on its way
    uint4 q[2 * T];
  };

  // valid: rows left in the operand from the tile's first one; rstride: element
  // distance of the tile's rows (KC)
  __device__ __forceinline__ void init(int valid, int rstride, int ld) {
    const int lane = threadIdx.x & 63;
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int o = i * 8 + (lane >> 3);
        vo[i] = (o < valid) ? (unsigned)(o * rstride * SZ + (lane & 7) * 16) : kOut;
      }
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int o = i * 16 + (lane & 15);
        vo[i] = (o < valid) ? (unsigned)(o * SZ + (lane >> 4) * VE * ld * SZ) : kOut;
      }
    }
  }
  __device__ __forceinline__ static unsigned* words(Stage& s, int i) { return reinterpret_cast<unsigned*>(&s.q[i]); }
  // one whole K step; p = the tile's element (0, k0)
  __device__ __forceinline__ void load(Stage& s, const S* p, int ld) const {
    const __amdgpu_buffer_rsrc_t rs = rsrc_at(p);
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const u4v q = __builtin_amdgcn_raw_buffer_load_b128(rs, vo[i], 0, 0);
        s.q[i] = make_uint4(q.x, q.y, q.z, q.w);
      }
    } else {
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          unsigned w[4];
#pragma unroll
          for (int e = 0; e < VE; ++e) {
            const int so = (j * 4 * VE + e) * ld * SZ;
            if constexpr (SZ == 8) {
              const u2v q = __builtin_amdgcn_raw_buffer_load_b64(rs, vo[i], so, 0);
              w[2 * e] = q.x;
              w[2 * e + 1] = q.y;
            } else {
              w[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, vo[i], so, 0);
            }
          }
          s.q[2 * i + j] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
  }
  // the last K step: `rem` < BK elements of K are left
  __device__ __forceinline__ void load_tail(Stage& s, const S* p, int ld, int rem) const {
    const __amdgpu_buffer_rsrc_t rs = rsrc_at(p);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 2 * T; ++i) {
      unsigned w[4];
      const unsigned v = KC ? vo[KC ? i : 0] : vo[KC ? 0 : i / 2];
#pragma unroll
      for (int e = 0; e < VE; ++e) {
        const int k = KC ? (lane & 7) * VE + e : (i & 1) * 4 * VE + (lane >> 4) * VE + e;
        const unsigned off = v + (KC ? (unsigned)(e * SZ) : (unsigned)(((i & 1) * 4 * VE + e) * ld * SZ));
        const unsigned o = (k < rem && v != kOut) ? off : kOut;
        if constexpr (SZ == 8) {
          const u2v q = __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, 0);
          w[2 * e] = q.x;
          w[2 * e + 1] = q.y;
        } else {
          w[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0);
        }
      }
      s.q[i] = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
  // fragments of a loaded K step (a wave's LDS accesses run in order)
  __device__ __forceinline__ void frags(Frag (&f)[T], const Stage& s, S* lds) const {
    if constexpr (KC) {
      const int lane = threadIdx.x & 63;
#pragma unroll
      for (int i = 0; i < NV; ++i)
        *reinterpret_cast<uint4*>(lds + (i * 8 + (lane >> 3)) * LDK + (lane & 7) * VE) = s.q[i];
      wave_lds_order();
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          f[i].q[j] = *reinterpret_cast<const uint4*>(lds + (i * 16 + (lane & 15)) * LDK + (j * 4 + (lane >> 4)) * VE);
      wave_lds_order();
    } else {
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) f[i].q[j] = s.q[2 * i + j];
    }
  }
};

// row of accumulator element r within its 16 x 16 block
template <typename S>
__device__ __forceinline__ int acc_row(int r, int g) { return sizeof(S) == 8 ? r * 4 + g : g * 4 + r; }

// acc += A B over the K steps first, first + stride, ... of the `nfull` whole
// ones, and over the tail step when tail_rem > 0.  a / b: the tiles' element
// (0, 0).  NST K steps are on their way from memory; the fragments of the
// next step are taken through LDS while the MFMAs of the current one run.
template <typename S, int TM, int TN, bool AKC, bool BKC, int NST>
__device__ __forceinline__ void mma_loop(typename Acc<S>::V (&acc)[TM][TN], const Operand<S, TM, AKC>& oa,
                                         const Operand<S, TN, BKC>& ob, S* lds, const S* a, const S* b, int lda,
                                         int ldb, int nfull, int first, int stride, int tail_rem) {
  constexpr int BK = 128 / (int)sizeof(S);
  const long astep = AKC ? (long)BK : (long)BK * lda, bstep = BKC ? (long)BK : (long)BK * ldb;
  typename Operand<S, TM, AKC>::Stage sa[NST];
  typename Operand<S, TN, BKC>::Stage sb[NST];
  Frag fa[2][TM], fb[2][TN];
  S* la = lds;
  S* lb = lds + Operand<S, TM, AKC>::LDS;
  auto mma = [&](const Frag (&x)[TM], const Frag (&y)[TN]) {
#pragma unroll
    for (int s = 0; s < kSteps<S>(); ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) mma_step<S>(acc[i][j], x[i], y[j], s);
  };
  const int cnt = nfull > first ? (nfull - first + stride - 1) / stride : 0;
  // past the end the last step is loaded again (its data is not used), so
  // that the loads in flight are the same on every path
  auto fetch = [&](auto ub, int it) {
    constexpr int u = decltype(ub)::value;
    const long t = first + (long)min(it, cnt - 1) * stride;
    oa.load(sa[u], a + t * astep, lda);
    ob.load(sb[u], b + t * bstep, ldb);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, NST - 1>;
  static_assert(NST == 1 || NST == 2, "the loop is unrolled by two");
  if (tail_rem > 0) {
    typename Operand<S, TM, AKC>::Stage ta;
    typename Operand<S, TN, BKC>::Stage tb;
    oa.load_tail(ta, a + nfull * astep, lda, tail_rem);
    ob.load_tail(tb, b + nfull * bstep, ldb, tail_rem);
    if (cnt > 0) {
      fetch(I0(), 0);
      if constexpr (NST == 2) fetch(I1(), 1);
    }
    oa.frags(fa[1], ta, la);
    ob.frags(fb[1], tb, lb);
    mma(fa[1], fb[1]);
  } else if (cnt > 0) {
    fetch(I0(), 0);
    if constexpr (NST == 2) fetch(I1(), 1);
  }
  if (cnt <= 0) return;
  oa.frags(fa[0], sa[0], la);
  ob.frags(fb[0], sb[0], lb);
  fetch(I0(), NST);
  // step it: the fragments of step it + 1 (in stage (it + 1) % NST) are
  // taken, its stage refilled with step it + 1 + NST, step it multiplied
  for (int it = 0; it < cnt; it += 2) {
    oa.frags(fa[1], sa[NST - 1], la);
    ob.frags(fb[1], sb[NST - 1], lb);
    fetch(I1(), it + 1 + NST);
    mma(fa[0], fb[0]);
    if (it + 1 >= cnt) break;
    oa.frags(fa[0], sa[0], la);
    ob.frags(fb[0], sb[0], lb);
    fetch(I0(), it + 2 + NST);
    mma(fa[1], fb[1]);
  }
}

struct DParams {
  int M, N, K;
  const void* A; int lda; long sA;
  const void* B; int ldb; long sB;
  void* C; long ldc; long sC;
  double alpha, beta;
  int kchunk;        // K range of one grid split (a multiple of the K step)
  long sSplit;       // element stride between the partial products of two splits
};

// C = alpha A B + beta C on wave tiles of (16 TM) x (16 TN); a workgroup of
// WK waves owns one tile, the waves taking the K steps in turn, and their
// partial tiles are summed through LDS in a fixed order.
template <typename S, int TM, int TN, int WK, int NST, bool AKC, bool BKC>
__global__ __launch_bounds__(WK * 64)
void direct_gemm_kernel(DParams p) {
  typedef typename Acc<S>::T AT;
  typedef typename Acc<S>::V AV;
  constexpr int BM = TM * 16, BN = TN * 16, BK = 128 / (int)sizeof(S);
  constexpr int kLds = Operand<S, TM, AKC>::LDS + Operand<S, TN, BKC>::LDS;   // staging per wave
  constexpr int kRed = WK > 1 ? BM * BN : 0;
  __shared__ __align__(16) S smem[WK * (kLds > kRed ? kLds : kRed) + 1];
  const int nTm = (p.M + BM - 1) / BM, nTn = (p.N + BN - 1) / BN;
  int tm, tn;
  tile_coords(nTm, nTn, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const long bz = blockIdx.y;
  const int kbeg = blockIdx.z * p.kchunk, kend = min(p.K, kbeg + p.kchunk);
  const S* A = reinterpret_cast<const S*>(p.A) + bz * p.sA;
  const S* B = reinterpret_cast<const S*>(p.B) + bz * p.sB;
  AT* __restrict__ C = reinterpret_cast<AT*>(p.C) + bz * p.sC + (long)blockIdx.z * p.sSplit;
  A += AKC ? (long)m0 * p.lda + kbeg : (long)kbeg * p.lda + m0;
  B += BKC ? (long)n0 * p.ldb + kbeg : (long)kbeg * p.ldb + n0;
  const int lane = threadIdx.x & 63, lrow = lane & 15, g = lane >> 4;
  const int wk = WK > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  Operand<S, TM, AKC> oa;
  Operand<S, TN, BKC> ob;
  oa.init(p.M - m0, AKC ? p.lda : 1, p.lda);
  ob.init(p.N - n0, BKC ? p.ldb : 1, p.ldb);
  AV acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = AV{0, 0, 0, 0};
  const int nfull = (kend - kbeg) / BK, rem = (kend - kbeg) - nfull * BK;
  mma_loop<S, TM, TN, AKC, BKC, NST>(acc, oa, ob, smem + wk * kLds, A, B, p.lda, p.ldb, nfull, wk, WK,
                                     (nfull % WK == wk) ? rem : 0);
  const AT alpha = (AT)p.alpha, beta = (AT)p.beta;
  auto put = [&](int row, int col, AT v) {
    if (m0 + row < p.M && n0 + col < p.N) {
      AT* dst = C + (long)(m0 + row) * p.ldc + n0 + col;
      AT w = alpha * v;
      if (p.beta != 0.0) w += beta * *dst;
      *dst = w;
    }
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) put(i * 16 + acc_row<S>(r, g), j * 16 + lrow, acc[i][j][r]);
  } else {
    AT* red = smem;
    __syncthreads();                   // every wave is done with its staging rows
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          red[(wk * BM + i * 16 + acc_row<S>(r, g)) * BN + j * 16 + lrow] = acc[i][j][r];
    __syncthreads();
    for (int e = threadIdx.x; e < BM * BN; e += WK * 64) {
      AT v = red[e];
#pragma unroll
      for (int q = 1; q < WK; ++q) v += red[q * BM * BN + e];
      put(e / BN, e % BN, v);
    }
  }
}

template <typename S, int TM, int TN, int WK, int NST>
void direct_launch(Ctx* c, const GemmArgs& g, int kchunk, int splits, void* C, long ldc, long sSplit, double alpha,
                   double beta) {
  DParams p{g.M, g.N, g.K, g.A, (int)g.lda, g.sA, g.B, (int)g.ldb, g.sB, C, ldc, g.sC, alpha, beta, kchunk, sSplit};
  const int nTm = (g.M + 16 * TM - 1) / (16 * TM), nTn = (g.N + 16 * TN - 1) / (16 * TN);
  const dim3 grid((unsigned)(nTm * nTn), (unsigned)g.batch, (unsigned)splits), block(WK * 64);
  if (g.a_kc && g.b_kc)
    hipLaunchKernelGGL((direct_gemm_kernel<S, TM, TN, WK, NST, true, true>), grid, block, 0, c->stream, p);
  else if (g.a_kc)
    hipLaunchKernelGGL((direct_gemm_kernel<S, TM, TN, WK, NST, true, false>), grid, block, 0, c->stream, p);
  else if (g.b_kc)
    hipLaunchKernelGGL((direct_gemm_kernel<S, TM, TN, WK, NST, false, true>), grid, block, 0, c->stream, p);
  else
    hipLaunchKernelGGL((direct_gemm_kernel<S, TM, TN, WK, NST, false, false>), grid, block, 0, c->stream, p);
  D3S_HIP(hipGetLastError());
}

// ---------------------------------------------------------------- GEMM + W-map
// The first two contractions of H_eff (and of the expansion term and the
// environment updates) in one launch: T1 never leaves the compute unit.
// T1 = A B on a tile of MT*16 rows (i, u) (i < AM points, u the MPO index,
// row i*WX + u of A) and 64 columns (q, t) (four waves of 16), kept in LDS,
// then the W-map as a second MFMA contraction over k = (u, t):
//   L2R: out[(a,s), v, y] = alpha sum_{w,t} W[w,v,s,t] T1[(a,w),(t,y)],  A = L, B = psi
//   R2L: out[w, x, s, b]  = alpha sum_{v,t} W[w,v,s,t] T1[(b,v),(x,t)],  A = R, B = psi
struct FParams {
  int na, wx, nq, ld2, wo, K;    // points and MPO channels of the A side, points of the B side, log2 d, output channels, K
  const void* A; int lda;
  const void* B; int ldb;
  const void* W;
  void* out; long ld_out;
  double alpha;
  int am;                        // A-side points per tile
};

template <typename S, int MT, int TN, bool R2L>
__global__ __launch_bounds__(256, 2)
void front_kernel(FParams p) {
  typedef typename Acc<S>::V AV;
  constexpr int NC = 64 * TN;                        // columns of the tile
  constexpr int LDT = NC + 16 / (int)sizeof(S);
  constexpr int BK = 128 / (int)sizeof(S);
  constexpr int kLds = Operand<S, MT, true>::LDS + Operand<S, TN, R2L>::LDS;   // staging per wave
  constexpr int kTile = MT * 16 * LDT;
  __shared__ __align__(16) S sT[4 * kLds > kTile ? 4 * kLds : kTile];
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int ld2 = p.ld2, d = 1 << ld2, wx = p.wx, am = p.am, wo = p.wo;
  const int lnp = (TN == 1 ? 6 : 7) - ld2, np = 1 << lnp;     // B-side points per tile
  const int nTm = (p.na + am - 1) / am, nTn = (p.nq + np - 1) / np;
  int tm, tn;
  tile_coords(nTm, nTn, tm, tn);
  const int i0 = tm * am, q0 = tn * np;
  const int lane = threadIdx.x & 63, lrow = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kin = wx << ld2, nout = wo << ld2, ks = (kin + 3) / 4, mb = (nout + 15) / 16;
  long* sOff = reinterpret_cast<long*>(smem_raw);    // element offset of every output
  S* sW = reinterpret_cast<S*>(smem_raw + sizeof(long) * 16 * mb);   // W in fragment order: [(mb, ks)][lane]
  // T1 tile
  const S* A = reinterpret_cast<const S*>(p.A) + (long)i0 * wx * p.lda;
  const S* B = reinterpret_cast<const S*>(p.B);
  Operand<S, MT, true> oa;
  Operand<S, TN, R2L> ob;
  oa.init(min(am, p.na - i0) * wx, p.lda, p.lda);
  if constexpr (R2L) {                               // column (x, t) of the tile: row x0*d + c of psi
    B += (((long)q0 << ld2) + wave * (16 * TN)) * p.ldb;
    ob.init(((p.nq - q0) << ld2) - wave * (16 * TN), p.ldb, p.ldb);
  } else {                                           // column t*np + y: psi[x][(t, y)]
    const int c = wave * (16 * TN), t = c / np, y = c - t * np;
    B += (long)t * p.nq + q0 + y;
    ob.init(p.nq - q0 - y, 1, p.ldb);
  }
  AV acc[MT][TN];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = AV{0, 0, 0, 0};
  // W[o][k], o = s*wo + v (L2R) or w*d + s (R2L), k = u*d + t, in fragments
  // dealt to the waves; a wave's first kPre are on their way during the K loop
  const S* Wg = reinterpret_cast<const S*>(p.W);
  const int wr = R2L ? wx : wo, frags = mb * ks;
  const float rks = 1.0f / ks, rwo = 1.0f / wo;      // quotients of small numbers
  auto w_entry = [&](int f) {
    const int m = (int)((f + 0.5f) * rks), o = min(m * 16 + lrow, nout - 1), k = min((f - m * ks) * 4 + g, kin - 1);
    const int u = k >> ld2, t = k & (d - 1), os = (int)((o + 0.5f) * rwo);
    const int w = R2L ? o >> ld2 : u, s = R2L ? o & (d - 1) : os, vv = R2L ? u : o - os * wo;
    return Wg + ((((((w * wr + vv) << ld2) + s) << ld2)) + t);
  };
  auto put_w = [&](int f, S v) {
    const int m = (int)((f + 0.5f) * rks);
    sW[f * 64 + lane] = (m * 16 + lrow < nout && (f - m * ks) * 4 + g < kin) ? (S)p.alpha * v : S(0);
  };
  constexpr int kPre = 4;
  S wpre[kPre];
#pragma unroll
  for (int q = 0; q < kPre; ++q) wpre[q] = *w_entry(min(wave + 4 * q, frags - 1));
  const int nfull = p.K / BK;
  mma_loop<S, MT, TN, true, R2L, 2>(acc, oa, ob, sT + wave * kLds, A, B, p.lda, p.ldb, nfull, 0, 1,
                                    p.K - nfull * BK);
#pragma unroll
  for (int q = 0; q < kPre; ++q)
    if (wave + 4 * q < frags) put_w(wave + 4 * q, wpre[q]);
  for (int f = wave + 4 * kPre; f < frags; f += 4) put_w(f, *w_entry(f));
  for (int o = threadIdx.x; o < nout; o += 256) {
    if constexpr (R2L) {
      const int w = o >> ld2, s = o & (d - 1);
      sOff[o] = (((long)w * p.nq << ld2) + s) * p.na;
    } else {
      const int s = (int)((o + 0.5f) * rwo), v = o - s * wo;
      sOff[o] = s * p.ld_out + (long)v * p.nq;
    }
  }
  __syncthreads();                                   // the staging rows are free
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        sT[(i * 16 + acc_row<S>(r, g)) * LDT + wave * (16 * TN) + j * 16 + lrow] = acc[i][j][r];
  __syncthreads();
  // W-map: blocks of 16 points by 16 outputs dealt to the waves; lane group
  // g's k of step s is (u, t) with u = (4 s + g) / d, t = g mod d
  const int npts = am * np, npb = (npts + 15) / 16;
  const int ustep = 4 >> ld2, u0 = g >> ld2, toff = (g & (d - 1)) * (R2L ? 1 : np);
  S* out = reinterpret_cast<S*>(p.out);
  auto mma = [](S wv, S x, AV& o) {
    if constexpr (sizeof(S) == 8) o = __builtin_amdgcn_mfma_f64_16x16x4f64(wv, x, o, 0, 0, 0);
    else o = __builtin_amdgcn_mfma_f32_16x16x4f32(wv, x, o, 0, 0, 0);
  };
  const float ram = 1.0f / am;
  struct Point {
    const S* tb;                                     // its T1 values
    S* dst;
    bool live;
  };
  auto point = [&](int pb) {
    const int pt = pb * 16 + lrow, pc = min(pt, npts - 1);
    int ia, iq;                                      // A-side and B-side index within the tile
    if constexpr (R2L) { iq = (int)((pc + 0.5f) * ram); ia = pc - iq * am; }
    else { ia = pc >> lnp; iq = pc & (np - 1); }
    return Point{sT + ia * wx * LDT + (R2L ? iq << ld2 : iq) + toff,
                 out + (R2L ? ((long)(q0 + iq) << ld2) * p.na + i0 + ia : ((long)(i0 + ia) << ld2) * p.ld_out + q0 + iq),
                 pt < npts && i0 + ia < p.na && q0 + iq < p.nq};
  };
  auto store = [&](const Point& pt, const AV& o, const long (&off)[4], int m) {
    if (pt.live) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (m * 16 + acc_row<S>(r, g) < nout) pt.dst[off[r]] = o[r];
    }
  };
  // Steps past the last k are skipped, and the lane groups past it in a step (d =
  // 2 and odd w) have zeros of T1 beside those of W: an infinite T1 value makes
  // its outputs infinite, not NaN.
  const bool part = (kin & 3) != 0;
  auto past = [&](int s) { return 4 * s + g >= kin; };
  // Up to KS steps the W fragments and output offsets of 16 outputs stay in
  // registers and a wave has two blocks of points in flight: the map of a
  // small call's tile takes 4500 cycles that way, 6900 with one block after the
  // other and everything read per block (128 x 120, d = 4, w = 6).
  auto map = [&](auto kst) {
    constexpr int KS = decltype(kst)::value;
    for (int m = 0; m < mb; ++m) {
      const S* wf = sW + (long)m * ks * 64 + lane;
      S wv[KS];
      long off[4];
#pragma unroll
      for (int s = 0; s < KS; ++s) wv[s] = wf[min(s, ks - 1) * 64];
#pragma unroll
      for (int r = 0; r < 4; ++r) off[r] = sOff[min(m * 16 + acc_row<S>(r, g), nout - 1)];
#pragma unroll
      for (int s = 0; s < KS; ++s) wv[s] = s < ks ? wv[s] : S(0);
      for (int pb = 2 * wave; pb < npb; pb += 8) {
        const Point pa = point(pb), pz = point(pb + 1);
        S x[KS], z[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const int r = min(min(s, ks - 1) * ustep + u0, wx - 1) * LDT;
          x[s] = pa.tb[r];
          z[s] = pz.tb[r];
        }
        if (part) {
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            x[s] = past(s) ? S(0) : x[s];
            z[s] = past(s) ? S(0) : z[s];
          }
        }
        AV o = AV{0, 0, 0, 0}, q = AV{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s)
          if (s < ks) {
            mma(wv[s], x[s], o);
            mma(wv[s], z[s], q);
          }
        store(pa, o, off, m);
        store(pz, q, off, m);
      }
    }
  };
  if (ks <= 3) {
    map(std::integral_constant<int, 3>());
  } else if (ks <= 6) {
    map(std::integral_constant<int, 6>());
  } else {
    constexpr int KC = 6;                            // k steps held at a time
    for (int pb = wave; pb < npb; pb += 4) {
      const Point pa = point(pb);
      for (int m = 0; m < mb; ++m) {
        AV o = AV{0, 0, 0, 0};
        const S* wf = sW + (long)m * ks * 64 + lane;
        for (int s0 = 0; s0 < ks; s0 += KC) {
          S x[KC], wv[KC];
#pragma unroll
          for (int s = 0; s < KC; ++s) {
            const int ss = min(s0 + s, ks - 1);
            x[s] = pa.tb[min(ss * ustep + u0, wx - 1) * LDT];
            wv[s] = (s0 + s < ks) ? wf[ss * 64] : S(0);
          }
          if (part) {
#pragma unroll
            for (int s = 0; s < KC; ++s) x[s] = past(s0 + s) ? S(0) : x[s];
          }
#pragma unroll
          for (int s = 0; s < KC; ++s)
            if (s0 + s < ks) mma(wv[s], x[s], o);
        }
        long off[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) off[r] = sOff[min(m * 16 + acc_row<S>(r, g), nout - 1)];
        store(pa, o, off, m);
      }
    }
  }
}

template <typename S, int MT, int TN, bool R2L>
void front_launch(Ctx* c, FParams p, size_t sh) {
  p.am = MT * 16 / p.wx;
  const int np = (64 * TN) >> p.ld2;
  const dim3 grid((unsigned)(((p.na + p.am - 1) / p.am) * ((p.nq + np - 1) / np)));
  hipLaunchKernelGGL((front_kernel<S, MT, TN, R2L>), grid, dim3(256), sh, c->stream, p);
  D3S_HIP(hipGetLastError());
}

// the largest leading dimension whose 32-bit byte offsets within a tile (at
// most 128 rows, or a K step) stay inside the buffer resource
constexpr long kMaxLd = (1L << 30) / (128 * 8);

template <typename S>
bool direct_dispatch(Ctx* c, const GemmArgs& g) {
  typedef typename Acc<S>::T AT;
  constexpr int BK = 128 / (int)sizeof(S);
  if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.batch <= 0 || g.batch > 65535) return false;
  if (g.lda > kMaxLd || g.ldb > kMaxLd) return false;
  auto ceil_div = [](long a, long b) { return (a + b - 1) / b; };
  const long t32 = ceil_div(g.M, 32) * ceil_div(g.N, 32) * g.batch;
  if (t32 > (1L << 30)) return false;
  const int steps = g.K / BK;
  // Who shares a tile's K (measured on MI355X, FP64 and FP32):
  //  - too few 32x32 tiles for half of the chip: 16x16 tiles, a K loop a
  //    quarter as long, by four or (long sums) eight waves (FP64 384 x 96 x 576
  //    5.3 us, 32x32 tiles 9.6; 512 x 120 x 720 5.4 against 10.7; 640 x 160 x
  //    960 8.7 against 12.3; 768 x 192 x 1152 12.4 against 14.4; 1024 x 250 x
  //    1500 26.2 against 20.2, where operands come twice as often from L2);
  //  - fewer 32x32 tiles than compute units: eight waves a tile while each
  //    gets two K steps or more, else four; very long sums are split over the
  //    grid too, which costs a summing launch (about 5 us);
  //  - long sums: 64x32 tiles of four waves once there are nearly two for each
  //    compute unit, 900 tiles of 32x32 (2048 x 512 x 3072, 1024 tiles: 106 us,
  //    32x32 tiles of four waves 111 us), before that 32x32 ones (1200 x 280 x 1680,
  //    342 tiles: 33 against 43 us, 1600 x 400 x 2400, 650: 66 against 76 us; FP32
  //    36 against 44 us);
  //  - short sums: four waves a 32x32 tile while there are fewer tiles than
  //    SIMDs (768 x 512 x 128: 7.2 us, one wave 8.3 us), one wave then
  //    (1536 x 1000 x 256: 21.5 us, four waves 24.4 us), and 32x64 tiles once
  //    these give every SIMD two (2400 x 3102 x 517: 150 us, 32x32 173 us).
  int splits = 1;
  if (t32 <= 128 && g.batch == 1 && steps >= 512 && !c->splitk_off) {
    splits = (int)std::min<long>(512 / t32, steps / 64);
    if (g.part) splits = (int)std::min<size_t>((size_t)splits, g.part_cap / (sizeof(AT) * (size_t)g.M * g.N));
  }
  int chunk = g.K;
  void* C = g.C;
  long ldc = g.ldc, ss = 0;
  double alpha = g.alpha, beta = g.beta;
  AT* part = nullptr;
  if (splits > 1) {
    chunk = (int)(ceil_div(ceil_div(g.K, splits), BK) * BK);
    splits = (int)ceil_div(g.K, chunk);
    part = g.part ? (AT*)g.part : (AT*)ws_get(c, WS_SPLITK, sizeof(AT) * (size_t)splits * g.M * g.N);
    C = part;
    ldc = g.N;
    ss = (long)g.M * g.N;
    alpha = 1.0;
    beta = 0.0;
  } else {
    splits = 1;
  }
  auto go = [&](auto tm, auto tn, auto wk, auto nst) {
    direct_launch<S, decltype(tm)::value, decltype(tn)::value, decltype(wk)::value, decltype(nst)::value>(
        c, g, chunk, splits, C, ldc, ss, alpha, beta);
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I4 = std::integral_constant<int, 4>;
  using I8 = std::integral_constant<int, 8>;
  if (t32 <= 160 && splits == 1) {
    if (steps >= 40) go(I1(), I1(), I8(), I2());
    else go(I1(), I1(), I4(), I2());
  } else if (t32 <= 320) {
    if (steps >= 16) go(I2(), I2(), I8(), I2());
    else go(I2(), I2(), I4(), I2());
  } else if (t32 >= 900 && t32 < 4096 && steps >= 64) {
    go(I4(), I2(), I4(), I1());
  } else if (t32 < 1024) {
    go(I2(), I2(), I4(), I2());
  } else if (t32 < 4096) {
    go(I2(), I2(), I1(), I2());
  } else {
    go(I2(), I4(), I1(), I1());
  }
  if (splits > 1) splitk_reduce(c, sizeof(AT) == 8, part, splits, g.M, g.N, g.C, g.ldc, g.alpha, g.beta);
  return true;
}

template <typename S>
bool front_dispatch(Ctx* c, bool r2l, bool copied, FParams p) {
  constexpr bool f64 = sizeof(S) == 8;
  const int d = 1 << p.ld2;
  p.am = kFrontRows / p.wx;
  const int kin = p.wx * d, nout = p.wo * d, mb = (nout + 15) / 16;
  const size_t sh = sizeof(long) * 16 * (size_t)mb + sizeof(S) * 64 * (size_t)((kin + 3) / 4) * mb;
  if (sh > 12 * 1024) return false;
  auto ceil_div = [](long a, long b) { return (a + b - 1) / b; };
  const long ta = ceil_div(p.na, p.am), tiles2 = ta * ceil_div(p.nq, 128 / d), tiles1 = ta * ceil_div(p.nq, 64 / d);
  if (tiles1 > (1L << 30)) return false;
  // Against the launches it replaces (for H_eff a transposed copy of psi, the
  // GEMM, the W-map): over m = 300 ... 2400 the kernel reaches 50 to 63 (FP64)
  // and 85 to 118 (FP32) TFLOP/s of its whole tiles, 60 and 102 in the middle of
  // the sizes where the two are close, below the workgroup-tiled GEMM's best;
  // but T1 costs the others a write and a read of memory, at 5 TB/s, and the
  // launches and their gaps 20 us.  Expansion and environments have no copy of
  // psi, a GEMM on its own layout and a W-map into other rows: 7 % more for the
  // GEMM, 3.3 TB/s, 10 us (m = 1024 right to left 801 / 831 us, 1200 left to
  // right 1423 / 1483, 1800 4825 / 4625).  H_eff, d = 4, w = 6, this kernel against
  // the launches, FP64: m = 300 51 / 68 us, 512 125 / 141, 800 433 / 444, 900 646 /
  // 642, 1024 835 / 795, 1200 1452 / 1403, 1400 2466 / 2113, 1600 3211 / 3040; FP32:
  // 300 35 / 49, 600 122 / 142, 800 236 / 230, 1024 458 / 427, 1400 1235 / 1117.
  const double t_front = 2.0 * tiles2 * kFrontRows * 128.0 * p.K / (f64 ? 60e12 : 102e12);
  const double rows = (double)p.na * p.wx, cols = (double)p.nq * d;
  const double t_gemm = gemm_estimate(f64 ? D3S_F64 : D3S_F32, (int)rows, (int)cols, p.K).seconds;
  const double bytes = (double)sizeof(S) * (rows * cols + (double)p.na * p.nq * nout);
  if (t_front > (copied ? t_gemm + bytes / 5e12 + 20e-6 : 1.067 * t_gemm + bytes / 3.3e12 + 10e-6)) return false;
  // 64 columns a tile (one block a wave) until 128 give every compute unit
  // its second workgroup (FP64 m = 128 11.6 against 17.6 us; 512 162 against
  // 138 us)
  // ... and then as many 16-row blocks a tile (3, 2, 1) as give the fewest
  // block rounds over 256 compute units: a small call spreads over more of
  // them (FP64, 3 / 2 / 1 blocks, whole product: m = 37 13.3 / 12.6 / 11.7 us,
  // 128 x 120 22.2 / 20.5 / 21.3, 160 25.5 / 27.2 / 29.3, 192 35.3 / 31.8 /
  // 36.4, 256 43.8 / 50.0 / 54.7)
  int mt = 3;
  long rounds = 1L << 60;
  for (int m = 3; m >= 1 && m * 16 >= p.wx; --m) {
    const long r = m * ceil_div(ceil_div(p.na, m * 16 / p.wx) * ceil_div(p.nq, 64 / d), 256);
    if (r < rounds) {
      rounds = r;
      mt = m;
    }
  }
  auto go = [&](auto m, auto n) {
    if constexpr (f64) {                 // right to left: expansion and environments, in FP64 only
      if (r2l) return front_launch<S, decltype(m)::value, decltype(n)::value, true>(c, p, sh);
    }
    front_launch<S, decltype(m)::value, decltype(n)::value, false>(c, p, sh);
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  if (tiles2 >= 400) go(I3(), I2());
  else if (mt == 1) go(I1(), I1());
  else if (mt == 2) go(I2(), I1());
  else go(I3(), I1());
  return true;
}

}  // namespace

// Which kernel, tile and split of K a large FP64 or FP32 product should take:
// the least modelled time.  A compute unit works off ceil(tiles / 256) tiles
// at the share of its matrix peak that the kernel reaches on whole tiles
// (measured, FP64 / FP32: 256x128 workgroup tiles 94 / 92 %, 128x128 91 %,
// the 32x64 wave tiles here 84 %); a split adds its partial products' write,
// read and summing launch.  For example FP64 6004 x 1403 x 8418 (rounds of
// 256x128 tiles half empty): 36 TFLOP/s on 256x128 tiles, 48 on 128x128 ones.
GemmChoice gemm_estimate(d3s_prec p, int M, int N, int K) {
  const bool f64 = p == D3S_F64;
  const double cu = (f64 ? 78.6e12 : 157.3e12) / 256;     // matrix flops of a compute unit
  const int sz = f64 ? 8 : 4, bk = 128 / sz;
  auto ceil_div = [](double a, double b) { return std::ceil(a / b - 1e-9); };
  const double flop_k = 2.0 * K;
  // 32x64 wave tiles, four at a time on a compute unit
  GemmChoice best{-1, 1, 4 * ceil_div(ceil_div(M, 32) * ceil_div(N, 64), 1024) * 32 * 64 * flop_k / (0.84 * cu)};
  for (int cfg = 2; cfg <= 3; ++cfg) {
    const int bm = cfg == 2 ? 256 : 128;
    const double tiles = ceil_div(M, bm) * ceil_div(N, 128), eff = cfg == 2 ? (f64 ? 0.94 : 0.92) : 0.91;
    for (int s = 1; s <= 8 && (s == 1 || K / s >= 16 * bk); ++s) {
      const double extra = s > 1 ? (s + 1.0) * M * N * sz / 4e12 + 5e-6 : 0.0;
      const double t = ceil_div(tiles * s, 256) * bm * 128 * flop_k / s / (eff * cu) + extra;
      if (t < best.seconds) best = GemmChoice{cfg, s, t};
    }
  }
  return best;
}

bool gemm_direct(Ctx* c, d3s_prec p, const GemmArgs& g) {
  if (p == D3S_F64) return direct_dispatch<double>(c, g);
  if (p == D3S_F32) return direct_dispatch<float>(c, g);
  return false;
}

bool front_wmap(Ctx* c, d3s_prec p, d3s_dir dir, int ml, int d, int mr, int wl, int wr, const void* env,
                const void* W, const void* psi, void* out, long ld_out, double alpha, bool copied) {
  // a chosen tile configuration means the separate kernels
  if (p == D3S_BF16 || (d != 2 && d != 4) || c->tile_config >= 0) return false;
  const bool r2l = dir == D3S_R2L;
  if (r2l && p != D3S_F64) return false;
  FParams f{};
  f.na = r2l ? mr : ml;
  f.wx = r2l ? wr : wl;
  f.nq = r2l ? ml : mr;
  f.ld2 = d == 4 ? 2 : 1;
  f.wo = r2l ? wl : wr;
  f.K = r2l ? mr : ml;
  f.A = env;
  f.lda = f.K;
  f.B = psi;
  f.W = W;
  f.out = out;
  f.ld_out = ld_out;
  f.alpha = alpha;
  const long ldb = r2l ? mr : (long)d * mr;
  if (f.wx > kFrontRows || f.lda > kMaxLd || ldb > kMaxLd) return false;
  f.ldb = (int)ldb;
  return p == D3S_F64 ? front_dispatch<double>(c, r2l, copied, f) : front_dispatch<float>(c, r2l, copied, f);
}

}  // namespace d3s
