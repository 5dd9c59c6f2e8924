// FP64 symmetric eigensolver for one matrix of kEigSmallMax < n <= kEigMidMax:
// the steps of eigsmall.hip spread over the device.
//
// What bounds it is the chain of matrix columns: a column of the reduction
// needs the product of the whole remaining matrix with the column before it.
//  - Reduction: one launch per column.  Every wave works out the pending update
//    and the new Householder vector for itself (two wave reductions over
//    vectors of length n, no barrier), then updates its rows and multiplies
//    them, so the matrix is passed over once per column.  Rows and columns are
//    counted from the end of the matrix: the grid shrinks with the remaining
//    matrix and a row stays on its workgroup, hence on its XCD's L2.  The last
//    kTail columns are reduced in registers by one workgroup, two barriers a
//    column.
//  - Tridiagonal eigenproblem: leaves of at most 64 by one workgroup each, then
//    merges level by level: order and deflation (a workgroup per merge), roots
//    of the secular equation (a wave per root), coupling vector, eigenvectors of
//    the rank-one update, and one product per half with the vectors so far.
//  - Back-transformation: a wave holds an eigenvector in registers and applies
//    the reflections in turn (two to a wave: 209 instead of 128 us at n = 512).
// A matrix of n = 512 takes 2.3 ms, of which the columns 1.7 ms at 4 us, the
// tail 0.13, the tridiagonal problem 0.3 and the way back 0.13; syevd takes
// 11.2 ms.
#include "d3s_internal.h"
#include "eigdc.h"

namespace d3s {
namespace {

constexpr int kTail = 96;        // columns left to the tail
constexpr int kLeafMax = 64;
constexpr int kWg = 256;

struct Head {
  unsigned long long top;        // bits of the largest absolute entry
  int info, pad;                 // 0 done, 1 not converged, 2 not finite
};

__device__ int scale_of(const Head* h) {      // exponent the matrix is divided by
  const double mx = __longlong_as_double((long long)h->top);
  return mx > 0.0 && isfinite(mx) ? ilogb(mx) : 0;
}

__global__ __launch_bounds__(kWg) void top_entry_kernel(const double* __restrict__ A, long count, Head* h) {
  unsigned long long top = 0;
  for (long i = (long)blockIdx.x * kWg + threadIdx.x; i < count; i += (long)gridDim.x * kWg)
    top = max(top, (unsigned long long)__double_as_longlong(fabs(A[i])));
  for (int o = 32; o > 0; o >>= 1) top = max(top, (unsigned long long)__shfl_xor((long long)top, o, 64));
  if ((threadIdx.x & 63) == 0) atomicMax(&h->top, top);
}

// Column k: A holds the matrix after columns < k - 1, to which the update
// v w^T + w v^T of column k - 1 is still to be applied, with v = row k - 1 of V
// and w from p = tau A v; row k is left as it is (nothing reads it again).  One
// wave, one row: a wave's own chain is what the launch takes, and four rows to
// a wave took 6.4 instead of 4.4 us a column at n = 512.  Loads are issued at
// clamped addresses and masked afterwards, so that none waits for another.
template <int NE>
__global__ __launch_bounds__(64)
void reduce_column_kernel(double* __restrict__ A, int n, int k, double* __restrict__ V, const double* __restrict__ pin,
                          double* __restrict__ pout, double* __restrict__ tauv, double* __restrict__ d,
                          double* __restrict__ e, const Head* __restrict__ head) {
  const int lane = threadIdx.x, r = n - 1 - blockIdx.x;      // r > k
  const bool first = k == 0, writer = blockIdx.x == 0;
  const double* vin = V + (long)max(k - 1, 0) * (64 * NE);
  double x[NE], v[NE], w[NE], a[NE];
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const int c = max(n - 1 - lane - 64 * j, 0);
    v[j] = vin[c];
    w[j] = pin[c];
    x[j] = A[(long)k * n + c];
    a[j] = A[(long)r * n + c];
  }
  const double tp = first ? 0.0 : tauv[k - 1];
  const double vk = first ? 0.0 : vin[k], pk = first ? 0.0 : pin[k];
  const double vr = first ? 0.0 : vin[r], pr = first ? 0.0 : pin[r];
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    loaded(v[j]);
    loaded(w[j]);
  }
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const bool in = !first && n - 1 - lane - 64 * j >= k;
    v[j] = in ? v[j] : 0.0;
    w[j] = in ? w[j] : 0.0;
    s = fma(v[j], w[j], s);
  }
  const double kk = 0.5 * tp * sum64(s), wk = pk - kk * vk, wr = pr - kk * vr;
  const int scale = first ? -scale_of(head) : 0;
  double s2 = 0.0, x0 = 0.0;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const int c = n - 1 - lane - 64 * j;
    w[j] = fma(-kk, v[j], w[j]);
    x[j] = first ? ldexp(x[j], scale) : x[j] - fma(vk, w[j], wk * v[j]);
    a[j] = first ? ldexp(a[j], scale) : a[j] - fma(vr, w[j], wr * v[j]);
    const double t = c > k + 1 ? x[j] : 0.0;
    s2 = fma(t, t, s2);
    x0 += c == k + 1 ? x[j] : 0.0;
  }
  s2 = sum64(s2);
  x0 = sum64(x0);
  double tau = 0.0, v0 = 0.0, ek = x0;
  if (s2 > 0.0) {
    ek = -copysign(sqrt(fma(x0, x0, s2)), x0);
    v0 = x0 - ek;
    tau = 2.0 / fma(v0, v0, s2);
  }
  double y = 0.0;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const int c = n - 1 - lane - 64 * j;
    const double t = c > k + 1 ? x[j] : (c == k + 1 ? v0 : 0.0);
    if (writer && c == k) d[k] = x[j];
    if (writer && c > k) V[(long)k * (64 * NE) + c] = t;
    if (c > k) A[(long)r * n + c] = a[j];
    y = fma(c > k ? a[j] : 0.0, t, y);
  }
  y = tau * sum64(y);
  if (lane == 0) {
    pout[r] = y;
    if (writer) {
      e[k] = ek;
      tauv[k] = tau;
    }
  }
}

// The last kTail columns, from column K = n - kTail on, with the update of
// column K - 1 pending
__global__ __launch_bounds__(kLanes * kTail)
void reduce_tail_kernel(const double* __restrict__ A, int n, double* __restrict__ V, int ldv, const double* __restrict__ pin,
                        double* __restrict__ tauv, double* __restrict__ d, double* __restrict__ e) {
  constexpr int E = kTail / kLanes, LD = kTail + 1;
  __shared__ double sV[kTail * LD], sP[kTail], sTau[kTail], sX[kTail + 1], sd[kTail + 1], se[kTail + 1];
  const int tid = threadIdx.x, lane = tid & 63, row = tid / kLanes, part = tid % kLanes, K = n - kTail;
  const double* v = V + (long)(K - 1) * ldv + K;
  const double* p = pin + K;
  double a[E], vc[E], pc[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int c = part + kLanes * j;
    a[j] = A[(long)(K + row) * n + K + c];
    vc[j] = v[c];
    pc[j] = p[c];
  }
  double s = v[lane] * p[lane];
  s += lane < kTail - 64 ? v[lane + 64] * p[lane + 64] : 0.0;
  const double kk = 0.5 * tauv[K - 1] * sum64(s), vr = v[row], wr = p[row] - kk * vr;
#pragma unroll
  for (int j = 0; j < E; ++j) a[j] -= fma(vr, pc[j] - kk * vc[j], wr * vc[j]);
  reduce_tridiagonal<kTail>(a, kTail, sV, sX, sTau, sP, sd, se);
  __syncthreads();
  for (int i = tid; i < kTail * kTail; i += kLanes * kTail) {
    const int k = i / kTail, c = i % kTail;
    if (k < kTail - 2 && c > k) V[(long)(K + k) * ldv + K + c] = sV[k * LD + c];
  }
  if (tid < kTail) {
    d[K + tid] = sd[tid];
    if (tid < kTail - 1) e[K + tid] = se[tid];
    if (tid < kTail - 2) tauv[K + tid] = sTau[tid];
  }
}

__device__ __forceinline__ int part_at(int n, int i, int count) { return (int)((long)n * i / count); }

// Leaf b of `count`: eigenvalues to ev, vectors to the diagonal block of Z (a
// row per vector)
__global__ __launch_bounds__(kLanes * kLeafMax)
void leaf_kernel(const double* __restrict__ d, const double* __restrict__ e, int n, int count, double* __restrict__ ev,
                 double* __restrict__ Z, Head* head) {
  __shared__ TridiagDc<kLeafMax> S;
  const int tid = threadIdx.x, lo = part_at(n, blockIdx.x, count), m = part_at(n, blockIdx.x + 1, count) - lo;
  if (tid < m) {
    double x = d[lo + tid];
    if (tid == 0 && lo > 0) x -= fabs(e[lo - 1]);
    if (tid == m - 1 && lo + m < n) x -= fabs(e[lo + m - 1]);
    S.d[tid] = x;
    S.e[tid] = tid < m - 1 ? e[lo + tid] : 0.0;
  }
  __syncthreads();
  const int bad = tridiag_dc<kLeafMax>(S, m);
  if (bad && tid == 0) atomicMax(&head->info, bad);
  if (bad == 2) {                      // the merges need numbers
    for (int i = tid; i < m; i += kLanes * kLeafMax) S.d[i] = 0.0;
    for (int i = tid; i < kLeafMax * TridiagDc<kLeafMax>::LD; i += kLanes * kLeafMax) S.w[i] = 0.0;
    __syncthreads();
  }
  if (tid < m) ev[lo + tid] = S.d[tid];
  for (int i = tid; i < m * m; i += kLanes * kLeafMax) {
    const int j = i / m, c = i % m;
    Z[(long)(lo + j) * n + lo + c] = S.w[c * TridiagDc<kLeafMax>::LD + j];
  }
}

// Per level, by position lo + i of a merge's block [lo, hi): the secular
// equation's poles, squared and signed couplings, roots; which old vector a pole
// is and which pole (or -1, deflated) an old vector; the rotations
struct Merge {
  double *ds, *zs, *zg, *zh, *tau, *rc, *rs;
  int *list, *pole, *org, *rp, *rq;
  int *count, *nrot;               // per merge
};

// Couplings, ascending order and deflation of merge blockIdx.x
__global__ __launch_bounds__(1024)
void merge_prepare_kernel(int n, int merges, double* __restrict__ ev, const double* __restrict__ e,
                          const double* __restrict__ Z, Merge M) {
  __shared__ double sd[1024], sz[1024], dl[1024], zl[1024], wtop[16];
  __shared__ int order[1024], list[1024], wcount[16], close, total;
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int lo = part_at(n, b, merges), m = part_at(n, b + 1, merges) - lo, mid = part_at(n, 2 * b + 1, 2 * merges);
  const double beta = e[mid - 1], rho = 2.0 * fabs(beta);
  const bool in = t < m;
  double dv = 0.0, zv = 0.0;
  if (in) {
    dv = ev[lo + t];
    const double* z = Z + (long)(lo + t) * n;
    zv = 0.70710678118654752440 * (lo + t < mid ? z[mid - 1] : copysign(1.0, beta) * z[mid]);
  }
  sd[t] = dv;
  sz[t] = zv;
  list[t] = 0;
  order[t] = t;
  if (t == 0) close = 0;
  double top = fmax(fabs(dv), fabs(beta));
  for (int o = 32; o > 0; o >>= 1) top = fmax(top, __shfl_xor(top, o, 64));
  if (lane == 0) wtop[wave] = top;
  __syncthreads();
  for (int i = 0; i < 16; ++i) top = fmax(top, wtop[i]);
  const double tol = 8.0 * kUlp * top;
  if (in) {
    int rank = 0;
#pragma unroll 8
    for (int i = 0; i < m; ++i) rank += (sd[i] < dv || (sd[i] == dv && i < t)) ? 1 : 0;
    order[rank] = t;
  }
  __syncthreads();
  const int me = order[t];
  const bool live = in && rho * fabs(sz[me]) > tol;
  const unsigned long long mask = __ballot(live);
  if (lane == 0) wcount[wave] = __popcll(mask);
  __syncthreads();
  int at = __popcll(mask & ((1ull << lane) - 1)), k = 0;
  for (int i = 0; i < 16; ++i) {
    at += i < wave ? wcount[i] : 0;
    k += wcount[i];
  }
  if (live) {
    list[at] = me;
    dl[at] = sd[me];
    zl[at] = sz[me];
  }
  __syncthreads();
  if (t + 1 < k) {
    const double p = zl[t], q = zl[t + 1];
    if (fabs((dl[t + 1] - dl[t]) * p * q) <= tol * (p * p + q * q)) close = 1;
  }
  if (t == 0) M.nrot[b] = 0;
  __syncthreads();
  if (close) {                       // one lane walks the list, in place
    if (t == 0) {
      int out = 0, nr = 0, p = list[0];
      double dp = dl[0], zp = zl[0];
      int nq = list[1];
      double nd = dl[1], nz = zl[1];
      for (int i = 1; i < k; ++i) {
        const int q = nq, in = min(i + 1, k - 1);
        double dq = nd, zq = nz;
        nq = list[in];                 // read ahead of the writes below
        nd = dl[in];
        nz = zl[in];
        const double h = zp * zp + zq * zq;
        if (fabs((dq - dp) * zp * zq) <= tol * h) {
          const double r = rsqrt_f64(h), c = zq * r, s = -zp * r, x = dp;
          dp = x * c * c + dq * s * s;
          dq = x * s * s + dq * c * c;
          zq = h * r;
          ev[lo + p] = dp;
          M.rp[lo + nr] = p;
          M.rq[lo + nr] = q;
          M.rc[lo + nr] = c;
          M.rs[lo + nr] = s;
          ++nr;
        } else {
          list[out] = p;
          dl[out] = dp;
          zl[out] = zp;
          ++out;
        }
        p = q;
        dp = dq;
        zp = zq;
      }
      list[out] = p;
      dl[out] = dp;
      zl[out] = zp;
      total = out + 1;
      M.nrot[b] = nr;
    }
    __syncthreads();
    k = total;
  }
  if (in) M.pole[lo + t] = -1;
  __syncthreads();
  if (t < k) {
    M.list[lo + t] = list[t];
    M.ds[lo + t] = dl[t];
    M.zg[lo + t] = zl[t];
    M.zs[lo + t] = zl[t] * zl[t];
    M.pole[lo + list[t]] = t;
  }
  if (t == 0) M.count[b] = k;
}

// Roots: a wave each; blockIdx.y: the merge
__global__ __launch_bounds__(kWg)
void merge_roots_kernel(int n, int merges, double* __restrict__ ev, const double* __restrict__ e, Merge M, Head* head) {
  const int b = blockIdx.y, k = M.count[b], j = blockIdx.x * (kWg / 64) + (threadIdx.x >> 6);
  if (j >= k) return;
  const int lo = part_at(n, b, merges), mid = part_at(n, 2 * b + 1, 2 * merges);
  int org;
  double tau;
  secular_root<64>(M.ds + lo, M.zs + lo, k, j, 2.0 * fabs(e[mid - 1]), org, tau);
  if ((threadIdx.x & 63) == 0) {
    const double x = M.ds[lo + org] + tau;
    M.org[lo + j] = org;
    M.tau[lo + j] = tau;
    ev[lo + M.list[lo + j]] = isfinite(x) ? x : 0.0;
    if (!isfinite(x)) atomicMax(&head->info, 1);
  }
}

// The coupling vector that has exactly these roots (a wave per entry)
__global__ __launch_bounds__(kWg) void merge_couplings_kernel(int n, int merges, Merge M) {
  const int b = blockIdx.y, k = M.count[b], i = blockIdx.x * (kWg / 64) + (threadIdx.x >> 6);
  if (i >= k) return;
  const int lo = part_at(n, b, merges), lane = threadIdx.x & 63;
  const double di = M.ds[lo + i];
  double pr = 1.0;
  for (int j = lane; j < k; j += 64) {
    const double gap = (M.ds[lo + M.org[lo + j]] - di) + M.tau[lo + j];
    pr *= (j == i) ? gap : gap / (M.ds[lo + j] - di);
  }
  for (int o = 32; o > 0; o >>= 1) pr *= __shfl_xor(pr, o, 64);
  if (lane == 0) M.zh[lo + i] = copysign(sqrt(fabs(pr)), M.zg[lo + i]);
}

// Column j of S (new vector j in terms of the old ones, the rotations
// included), 16 columns a workgroup and 16 lanes a column
__global__ __launch_bounds__(kWg)
void merge_vectors_kernel(int n, int merges, Merge M, double* __restrict__ S) {
  __shared__ double part[16][17];
  const int b = blockIdx.y, lo = part_at(n, b, merges), m = part_at(n, b + 1, merges) - lo;
  const int col = threadIdx.x & 15, grp = threadIdx.x >> 4, j = blockIdx.x * 16 + col;
  if (blockIdx.x * 16 >= m) return;
  const bool in = j < m;
  const int k = M.count[b], root = in ? M.pole[lo + j] : -1;
  double dj = 0.0, tj = 0.0, nn = 0.0;
  if (root >= 0) {
    dj = M.ds[lo + M.org[lo + root]];
    tj = M.tau[lo + root];
    for (int i = grp; i < k; i += 16) {
      const double t = M.zh[lo + i] / ((M.ds[lo + i] - dj) - tj);
      nn = fma(t, t, nn);
    }
  }
  part[grp][col] = nn;
  __syncthreads();
  nn = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) nn += part[i][col];
  const double f = root >= 0 ? 1.0 / sqrt(nn) : 0.0;
  double* s = S + (long)lo * n + lo + j;
  if (in)
    for (int i = grp; i < m; i += 16) {
      const int q = M.pole[lo + i];
      double t = i == j ? 1.0 : 0.0;
      if (root >= 0) t = q >= 0 ? f * (M.zh[lo + q] / ((M.ds[lo + q] - dj) - tj)) : 0.0;
      s[(long)i * n] = t;
    }
  __syncthreads();
  // the rotations came before the update: from the last to the first
  const int nr = M.nrot[b];
  if (in && grp == 0) {
    constexpr int kAhead = 8;          // loads in flight
    int held = -1;
    double yq = 0.0;
    for (int i0 = nr - 1; i0 >= 0; i0 -= kAhead) {
      double yp[kAhead], c[kAhead], sn[kAhead];
      int p[kAhead], q[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int i = lo + max(i0 - u, 0);
        p[u] = M.rp[i];
        q[u] = M.rq[i];
        c[u] = M.rc[i];
        sn[u] = M.rs[i];
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) yp[u] = s[(long)p[u] * n];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (i0 - u < 0) break;
        if (held != q[u]) {
          if (held >= 0) s[(long)held * n] = yq;
          yq = s[(long)q[u] * n];
        }
        s[(long)q[u] * n] = fma(sn[u], yp[u], c[u] * yq);
        yq = fma(c[u], yp[u], -(sn[u] * yq));
        held = p[u];
      }
    }
    if (held >= 0) s[(long)held * n] = yq;
  }
}

// Eigenvectors of the matrix from those of the tridiagonal one, to the row of
// their ascending place
template <int NE>
__global__ __launch_bounds__(kWg)
void back_kernel(const double* __restrict__ Z, const double* __restrict__ V, const double* __restrict__ tauv,
                 const double* __restrict__ ev, int n, double* __restrict__ out, double* __restrict__ evals,
                 const Head* __restrict__ head, int* __restrict__ info) {
  const int lane = threadIdx.x & 63, j = blockIdx.x * (kWg / 64) + (threadIdx.x >> 6);
  if (j >= n) return;
  double z[NE], cnt = 0.0;
  const double val = ev[j];
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int c = lane + 64 * i;
    z[i] = c < n ? Z[(long)j * n + c] : 0.0;
    const double x = c < n ? ev[c] : INFINITY;
    cnt += (x < val || (x == val && c < j)) ? 1.0 : 0.0;
  }
  const int rank = (int)sum64(cnt);
  // groups of G reflections, the next group's on their way meanwhile
  constexpr int G = NE <= 8 ? 4 : 2;
  double va[G][NE], vb[G][NE], ta[G], tb[G];
  auto load = [&](double (&x)[G][NE], double (&t)[G], int k0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int k = max(k0 - g, 0);
#pragma unroll
      for (int i = 0; i < NE; ++i) x[g][i] = V[(long)k * (64 * NE) + lane + 64 * i];
      t[g] = k0 - g >= 0 ? tauv[k] : 0.0;              // past the last: no reflection
    }
  };
  auto apply = [&](const double (&x)[G][NE], const double (&t)[G]) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      double y = 0.0;
#pragma unroll
      for (int i = 0; i < NE; ++i) y = fma(z[i], x[g][i], y);
      y = t[g] * sum64(y);
#pragma unroll
      for (int i = 0; i < NE; ++i) z[i] = fma(-y, x[g][i], z[i]);
    }
  };
  load(va, ta, n - 3);
  for (int k = n - 3; k >= 0; k -= 2 * G) {
    load(vb, tb, k - G);
    apply(va, ta);
    load(va, ta, k - 2 * G);
    apply(vb, tb);
  }
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int c = lane + 64 * i;
    if (c < n) out[(long)rank * n + c] = z[i];
  }
  if (lane == 0) evals[rank] = ldexp(val, scale_of(head));
  if (j == 0 && lane == 0) *info = head->info;
}

template <int NE>
bool solve(Ctx* c, int n, double* A, double* evals, int* info) {
  hipStream_t st = c->stream;
  const size_t nn = (size_t)n * n;
  // head, V, Z twice, S, then vectors: p twice, tau, d, e, eigenvalues, 7
  // of doubles and 5 of ints per level, counts
  const size_t bytes = 256 + sizeof(double) * (3 * nn + 64 * NE * (size_t)n + 13 * (size_t)n) + sizeof(int) * (5 * (size_t)n + 2 * 64);
  char* ws = nullptr;
  try {
    ws = (char*)ws_get(c, WS_EIG_MID, bytes);
  } catch (const Error& err) {
    if (err.code != D3S_ENOMEM) throw;
    return false;
  }
  Head* head = (Head*)ws;
  double* x = (double*)(ws + 256);
  auto take = [&](size_t k) {
    double* p = x;
    x += k;
    return p;
  };
  double *V = take(64 * NE * (size_t)n), *Z = take(nn), *Z2 = take(nn), *S = take(nn), *p0 = take(n), *p1 = take(n), *tau = take(n),
         *d = take(n), *e = take(n), *ev = take(n);
  Merge M;
  M.ds = take(n), M.zs = take(n), M.zg = take(n), M.zh = take(n), M.tau = take(n), M.rc = take(n), M.rs = take(n);
  int* ix = (int*)x;
  M.list = ix, M.pole = ix + n, M.org = ix + 2 * n, M.rp = ix + 3 * n, M.rq = ix + 4 * n;
  M.count = ix + 5 * n, M.nrot = M.count + 64;
  zero_bytes(c, head, 256 + sizeof(double) * 64 * NE * (size_t)n);     // rows of V: zero outside their vector
  hipLaunchKernelGGL(top_entry_kernel, dim3(64), dim3(kWg), 0, st, A, (long)nn, head);
  const int K = n - kTail;
  for (int k = 0; k < K; ++k)
    hipLaunchKernelGGL(reduce_column_kernel<NE>, dim3(n - 1 - k), dim3(64), 0, st, A, n, k, V, (k & 1) ? p0 : p1,
                       (k & 1) ? p1 : p0, tau, d, e, head);
  hipLaunchKernelGGL(reduce_tail_kernel, dim3(1), dim3(kLanes * kTail), 0, st, A, n, V, 64 * NE, (K & 1) ? p0 : p1, tau, d, e);
  int leaves = 1;
  while ((n + leaves - 1) / leaves > kLeafMax) leaves *= 2;
  hipLaunchKernelGGL(leaf_kernel, dim3(leaves), dim3(kLanes * kLeafMax), 0, st, d, e, n, leaves, ev, Z, head);
  for (int merges = leaves / 2; merges >= 1; merges /= 2) {
    const int m = (n + merges - 1) / merges;
    hipLaunchKernelGGL(merge_prepare_kernel, dim3(merges), dim3(1024), 0, st, n, merges, ev, e, Z, M);
    hipLaunchKernelGGL(merge_roots_kernel, dim3((m + 3) / 4, merges), dim3(kWg), 0, st, n, merges, ev, e, M, head);
    hipLaunchKernelGGL(merge_couplings_kernel, dim3((m + 3) / 4, merges), dim3(kWg), 0, st, n, merges, M);
    hipLaunchKernelGGL(merge_vectors_kernel, dim3((m + 15) / 16, merges), dim3(kWg), 0, st, n, merges, M, S);
    for (int b = 0; b < merges; ++b) {
      const int lo = (int)((long)n * b / merges), hi = (int)((long)n * (b + 1) / merges);
      const int mid = (int)((long)n * (2 * b + 1) / (2 * merges)), h0 = mid - lo, h1 = hi - mid;
      auto half = [&](int at, int h, int batch) {
        GemmArgs g{};
        g.M = hi - lo, g.N = h, g.K = h;
        g.A = S + (long)at * n + lo, g.lda = n, g.a_kc = false, g.sA = (long)h * n;
        g.B = Z + (long)at * n + at, g.ldb = n, g.b_kc = false, g.sB = (long)h * (n + 1);
        g.C = Z2 + (long)lo * n + at, g.ldc = n, g.sC = h;
        g.alpha = 1.0, g.beta = 0.0, g.batch = batch;
        if (!gemm_direct(c, D3S_F64, g)) gemm_f64(c, g);
      };
      if (h0 == h1) {
        half(lo, h0, 2);
      } else {
        half(lo, h0, 1);
        half(mid, h1, 1);
      }
    }
    std::swap(Z, Z2);
  }
  const int pv = kWg / 64;                 // a wave per vector
  hipLaunchKernelGGL(back_kernel<NE>, dim3((n + pv - 1) / pv), dim3(kWg), 0, st, Z, V, tau, ev, n, A, evals, head, info);
  D3S_HIP(hipGetLastError());
  return true;
}

}  // namespace

bool eig_mid_used(const Ctx* c, int n, int batch) {
  if (batch != 1 || n <= kEigSmallMax || n > kEigMidMax) return false;
  return c->eig_kind == 3 || (c->eig_kind == 0 && n > c->eig_jacobi_max);
}

bool eig_mid_launch(Ctx* c, int n, double* A, double* evals, int* info) {
  if (n <= 256) return solve<4>(c, n, A, evals, info);
  if (n <= 512) return solve<8>(c, n, A, evals, info);
  if (n <= 768) return solve<12>(c, n, A, evals, info);
  return solve<16>(c, n, A, evals, info);
}

}  // namespace d3s
