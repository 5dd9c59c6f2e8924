// Batched FP64 symmetric eigensolver for n <= kEigSmallMax in one launch, one
// workgroup per matrix: Householder reduction to tridiagonal form, divide and
// conquer on the tridiagonal matrix, and the transformation back.
//
// A library call spends a launch or more per matrix column (1.7 ms for a single
// n = 64 matrix on MI355X); inside one workgroup a column costs two barriers.
//  - Reduction: the matrix is kept in registers, eight lanes a row and every
//    eighth column each, so that a matrix-vector product is a few multiplies
//    and three DPP additions; vectors shared by the rows go through LDS, and
//    sums over a whole vector are formed by every wave for itself.
//  - Tridiagonal eigenproblem: split into leaves of at most 4, each solved by
//    one wave with the implicit QL iteration (its scalar recurrence, about 350
//    cycles for each of about n^2 rotations, is why the whole matrix is not:
//    0.64 ms at n = 64), then merged in pairs by rank-one updates
//    (Cuppen's method with deflation, the secular equation solved between the
//    poles, and the coupling vector recomputed from the roots so that the
//    vectors come out orthogonal, as Gu and Eisenstat showed).  Eight lanes
//    share a root's sums.
//  - Back-transformation: eight lanes hold an eigenvector and apply the
//    Householder reflections in turn, without barriers.
// Bound by the latency of these chains (n = 64, in thousands of cycles:
// reduction 140, leaves 45, secular equations 47, vectors 27, back 23).  What
// they are made of counts: values that are loaded or chosen under a condition
// became branches that wait for every load in turn, and leaves of 16 took 144
// thousand cycles.  One matrix, or up to 256: n = 32 0.09 ms, 64 0.18 ms, 96
// 0.34 ms; the library solver takes 0.95, 2.1 and 1.5 ms for one.
#include "d3s_internal.h"
#include "eigdc.h"

namespace d3s {
namespace {

// info: 0 done, 1 not converged, 2 non-finite input
template <int NMAX>
__global__ __launch_bounds__(kLanes * NMAX)
void eig_small_kernel(double* __restrict__ A, double* __restrict__ evals, int n,
                      int* __restrict__ info) {
  constexpr int E = NMAX / kLanes;      // elements of a row per lane
  constexpr int LD = NMAX + 1;
  constexpr int NT = kLanes * NMAX;
  __shared__ double sV[NMAX * LD];      // Householder vectors, row k
  __shared__ double sP[NMAX], sTau[NMAX], sX[NMAX + 1];
  __shared__ TridiagDc<NMAX> D;
  double *d = D.d, *e = D.e, *sW = D.w;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = tid / kLanes, part = tid % kLanes;
  double* Ab = A + (long)blockIdx.x * n * n;
  double* wb = evals + (long)blockIdx.x * n;
  int* ib = info + blockIdx.x;
  // symmetric: the column-major input read row by row is the same matrix
  double a[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int col = part + kLanes * j;
    a[j] = (row < n && col < n) ? Ab[(long)row * n + col] : 0.0;
  }
  // scaled by a power of two to entries below 2: nothing under- or overflows
  double mx = 0.0;
#pragma unroll
  for (int j = 0; j < E; ++j) mx = fmax(mx, isfinite(a[j]) ? fabs(a[j]) : INFINITY);
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  if (lane == 0) sP[wave] = mx;
  __syncthreads();
  for (int i = 0; i < NT / 64; ++i) mx = fmax(mx, sP[i]);
  if (!isfinite(mx)) {                  // the same for every thread
    if (tid == 0) *ib = 2;
    return;
  }
  const int scale = mx > 0.0 ? ilogb(mx) : 0;
#pragma unroll
  for (int j = 0; j < E; ++j) a[j] = ldexp(a[j], -scale);
  __syncthreads();                      // sP is written again
  reduce_tridiagonal<NMAX>(a, n, sV, sX, sTau, sP, d, e);
  __syncthreads();
  const int bad = tridiag_dc<NMAX>(D, n);
  if (bad == 2) {                       // the same for every thread
    if (tid == 0) *ib = 2;
    return;
  }
  // ---- ascending order and back-transformation: the eight lanes of column
  // `row` apply H_0 H_1 ... to it
  if (row < n) {
    const double v = d[row];
    double rank = 0.0;
    for (int i = part; i < n; i += kLanes) rank += d[i] < v || (d[i] == v && i < row);
    const int r = (int)sum8(rank);
    if (part == 0) wb[r] = ldexp(v, scale);
#pragma unroll
    for (int j = 0; j < E; ++j) a[j] = sW[(part + kLanes * j) * LD + row];
    for (int k = n - 3; k >= 0; --k) {
      const double* x = sV + k * LD;
      double vc[E], y = 0.0;
#pragma unroll
      for (int j = 0; j < E; ++j) vc[j] = x[part + kLanes * j];
#pragma unroll
      for (int j = 0; j < E; ++j) y = fma(a[j], vc[j], y);
      y = sTau[k] * sum8(y);
#pragma unroll
      for (int j = 0; j < E; ++j) a[j] = fma(-y, vc[j], a[j]);
    }
#pragma unroll
    for (int j = 0; j < E; ++j)
      if (part + kLanes * j < n) Ab[(long)r * n + part + kLanes * j] = a[j];
  }
  if (tid == 0) *ib = bad;
}

}  // namespace

bool eig_small_used(const Ctx* c, int n) {
  if (n < 1 || n > kEigSmallMax) return false;
  return c->eig_kind == 3 || (c->eig_kind == 0 && n > c->eig_jacobi_max);
}

void eig_small_launch(Ctx* c, int n, int batch, double* A, double* evals, int* info) {
  const dim3 g((unsigned)batch);
  auto go = [&](auto kern, int nmax) {
    hipLaunchKernelGGL(kern, g, dim3(kLanes * nmax), 0, c->stream, A, evals, n, info);
  };
  if (n <= 32) go(eig_small_kernel<32>, 32);
  else if (n <= 64) go(eig_small_kernel<64>, 64);
  else go(eig_small_kernel<kEigSmallMax>, kEigSmallMax);
  D3S_HIP(hipGetLastError());
}

void eig_small_check(const int* info, int batch) {
  for (int b = 0; b < batch; ++b) {
    if (info[b] == 2) throw Error{D3S_ENUMERIC, "eigensolver: the matrix is not finite"};
    if (info[b] != 0) throw Error{D3S_EDEVICE, "small eigensolver: no convergence"};
  }
}

void eig_batched_f64(Ctx* c, int n, int batch, double* A, double* evals) {
  if (batch <= 0) return;
  int* info = (int*)ws_get(c, WS_INFO, sizeof(int) * (size_t)batch);
  if (eig_small_used(c, n)) {
    eig_small_launch(c, n, batch, A, evals, info);
  } else if (!eig_mid_used(c, n, batch) || !eig_mid_launch(c, n, A, evals, info)) {
    syevd_batched_f64(c, n, batch, A, evals);
    return;
  }
  std::vector<int> h(batch);
  D3S_HIP(hipMemcpyAsync(h.data(), info, sizeof(int) * batch, hipMemcpyDeviceToHost, c->stream));
  D3S_HIP(hipStreamSynchronize(c->stream));
  eig_small_check(h.data(), batch);
}

}  // namespace d3s
