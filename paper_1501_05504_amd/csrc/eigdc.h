// Device parts shared by the symmetric eigensolvers (eigsmall.hip, eigmid.hip):
// sums over groups of lanes, the QL iteration of a leaf, the secular equation,
// and divide and conquer on a tridiagonal matrix within one workgroup.
#pragma once
#include <hip/hip_runtime.h>

namespace d3s {
namespace {

constexpr int kLanes = 8;   // lanes per row (column) of the matrix

template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// total of the eight lanes l & ~7 .. l | 7, on each of them
__device__ __forceinline__ double sum8(double v) {
  v = dpp_add<0xB1>(v);     // quad_perm 1 0 3 2
  v = dpp_add<0x4E>(v);     // quad_perm 2 3 0 1
  return dpp_add<0x141>(v); // row_half_mirror
}
template <int CTRL>
__device__ __forceinline__ double dpp_mul(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return v * __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double product8(double v) { return dpp_mul<0x141>(dpp_mul<0x4E>(dpp_mul<0xB1>(v))); }
__device__ __forceinline__ double lane_of(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// keeps a load where it is written: moved under the condition that its value
// is used in, each one would wait for itself
__device__ __forceinline__ void loaded(double& x) { asm volatile("" : "+v"(x)); }
// total of a wave
__device__ __forceinline__ double sum64(double v) {
  v = dpp_add<0x140>(sum8(v));   // row_mirror: the sixteen lanes of a row
  return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}

// 1 / sqrt(x) for normal x > 0: the hardware estimate and one third-order step
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// 1 / x for normal x: the hardware estimate and two Newton steps, within an ulp
__device__ __forceinline__ double rcp_f64(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

constexpr double kUlp = 2.220446049250313e-16;
constexpr int kLeaf = 4;

// Implicit QL with shifts (the tql2 iteration of Wilkinson and Reinsch's Handbook)
// on the tridiagonal block of size m <= kLeaf at d, e by one wave; the block's
// eigenvectors (its rows and columns of w, identity on entry) are rotated along,
// lane r holding row r.  Every lane runs the same recurrence and control flow is
// uniform.  False: no convergence.
__device__ bool ql_leaf(double* d, const double* e, int m, double* w, int ld, double* dummy) {
  const int lane = threadIdx.x & 63;
  double dr = lane < m ? d[lane] : 0.0, er = lane < m - 1 ? e[lane] : 0.0;
  double* z = lane < m ? w + lane * ld : dummy;
  auto put = [&](double& x, int k, double v) { x = lane == k ? v : x; };
  int iter = 0;
  for (int l = 0; l < m;) {
    const double up = __shfl_down(dr, 1, 64), dd = fabs(dr) + fabs(up);
    const unsigned long long small = __ballot(lane >= m - 1 || fabs(er) + dd == dd);
    const int q = __builtin_amdgcn_readfirstlane(__ffsll(small >> l) - 1 + l);   // end of the unreduced block
    if (q == l) {
      ++l;
      iter = 0;
      continue;
    }
    if (++iter > 60) return false;
    const double el = lane_of(er, l), dl = lane_of(dr, l);
    double g = (lane_of(dr, l + 1) - dl) / (2.0 * el);
    const double r1 = sqrt(fma(g, g, 1.0));
    double dn = lane_of(dr, q), ei = lane_of(er, q - 1), di = lane_of(dr, q - 1);
    g = dn - dl + el / (g + copysign(r1, g));
    double sn = 1.0, cn = 1.0, p = 0.0, hi = z[q], zi = z[q - 1];
    for (int i = q - 1; i >= l; --i) {
      const int ip = max(i - 1, 0);
      const double en = lane_of(er, ip), dp = lane_of(dr, ip), zp = z[ip];        // the next plane's
      const double f = sn * ei, b = cn * ei, h = fma(f, f, g * g);
      const bool none = !(h > 1e-280);    // nothing to rotate (norm about 1: far below rounding)
      const double ri = rsqrt_f64(h), r = none ? g : h * ri;
      sn = none ? 0.0 : f * ri;
      cn = none ? 1.0 : g * ri;
      g = dn - p;
      const double t = fma(di - g, sn, 2.0 * cn * b);
      p = sn * t;
      put(er, i + 1, r);
      put(dr, i + 1, g + p);
      g = fma(cn, t, -b);
      z[i + 1] = fma(sn, zi, cn * hi);
      hi = fma(cn, zi, -(sn * hi));
      dn = di;
      di = dp;
      ei = en;
      zi = zp;
    }
    z[l] = hi;
    put(dr, l, dn - p);
    put(er, l, g);
    put(er, q, 0.0);
  }
  if (lane < m) d[lane] = isfinite(dr) ? dr : 0.0;
  return !__any(!isfinite(dr));
}

// total over the L = 8 or 64 lanes that share an item
template <int L>
__device__ __forceinline__ double sum_lanes(double v) {
  if constexpr (L == 8) return sum8(v);
  else return sum64(v);
}

// Root j of 1 + rho sum_i z2_i / (d_i - x) = 0 between d_j and d_{j+1} (beyond
// d_{k-1} for the last), d ascending, by the L lanes of a group: returned as the
// pole `org` next to it and the distance tau from that pole, NaN if neither the
// residual nor the bracket became small enough.  Each side of the root is
// interpolated by one pole and a constant with value and slope matched (the
// "middle way" of R.-C. Li, LAPACK Working Note 89), safeguarded by bisection.
// In one and a half million roots (random, graded and clustered poles, weights
// down to the deflation limit, k up to 1024) 99.6 % took fewer than 8 steps and
// none more than 49; from the 40th on every other step bisects, so that the
// bracket closes to rounding (150 halvings at that limit) well before the last.
template <int L>
__device__ void secular_root(const double* d, const double* z2, int k, int j, double rho, int& org, double& tau) {
  const int part = threadIdx.x & (L - 1);
  const bool last = j == k - 1;
  double total = 0.0;
  if (last)
    for (int i = part; i < k; i += L) total += z2[i];
  const double gap = last ? rho * sum_lanes<L>(total) : d[j + 1] - d[j];
  double lo = 0.0, hi = gap;
  org = j;
  if (!last) {
    double f = 0.0;
    for (int i = part; i < k; i += L) f += z2[i] / ((d[i] - d[j]) - 0.5 * gap);
    if (1.0 + rho * sum_lanes<L>(f) >= 0.0) {
      hi = 0.5 * gap;
    } else {
      org = j + 1;
      lo = -0.5 * gap;
      hi = 0.0;
    }
  }
  const double d0 = d[org], p1 = d[j] - d0, p2 = last ? 0.0 : d[j + 1] - d0;
  tau = 0.5 * (lo + hi);
  int it = 0;
  for (; it < 400; ++it) {
    double a1 = 0.0, b1 = 0.0, a2 = 0.0, b2 = 0.0;
    for (int i = part; i < k; i += L) {
      const double r = rcp_f64((d[i] - d0) - tau), t = z2[i] * r;
      if (i <= j) {
        a1 += t;
        b1 = fma(t, r, b1);
      } else {
        a2 += t;
        b2 = fma(t, r, b2);
      }
    }
    a1 = rho * sum_lanes<L>(a1);
    b1 = rho * sum_lanes<L>(b1);
    a2 = rho * sum_lanes<L>(a2);
    b2 = rho * sum_lanes<L>(b2);
    const double f = 1.0 + a1 + a2;
    if (f < 0.0) lo = tau;
    else hi = tau;
    if (fabs(f) <= 4.0 * kUlp * (1.0 + fabs(a1) + a2) || hi - lo <= 2.0 * kUlp * fmax(fabs(lo), fabs(hi))) break;
    const double e1 = p1 - tau, e2 = p2 - tau;
    double eta;
    if (last) {
      const double r = 1.0 + a1 - b1 * e1;
      eta = e1 + b1 * e1 * e1 / r;
    } else {
      const double c = f - e1 * b1 - e2 * b2, a = (e1 + e2) * f - e1 * e2 * (b1 + b2), b = e1 * e2 * f;
      const double s = sqrt(fmax(fma(a, a, -4.0 * b * c), 0.0));
      eta = a <= 0.0 ? (a - s) / (2.0 * c) : 2.0 * b / (a + s);
    }
    if (!(f * eta < 0.0)) eta = -f / (b1 + b2);
    const double next = tau + eta;
    tau = (next > lo && next < hi && (it < 40 || !(it & 1))) ? next : 0.5 * (lo + hi);
  }
  if (it == 400) tau = NAN;
}

// Householder reduction of a symmetric matrix of size n <= NMAX to tridiagonal
// form by a workgroup of kLanes NMAX threads; thread (row, part) holds elements
// (row, part + kLanes j) in a.  Step k annihilates column k below the
// subdiagonal with H = 1 - tau v v^T: v is row k of sV, zero up to column k.
// sX: NMAX + 1 entries for the subdiagonal entry of the column at hand.
template <int NMAX>
__device__ void reduce_tridiagonal(double (&a)[NMAX / kLanes], int n, double* sV, double* sX, double* sTau, double* sP,
                                   double* d, double* e) {
  constexpr int E = NMAX / kLanes;
  constexpr int LD = NMAX + 1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int row = tid / kLanes, part = tid % kLanes;
  // column k: its diagonal entry to d, the next to sX, the others to row k of
  // sV, which is zero elsewhere
  auto put_column = [&](int k) {
    double t = a[0];
#pragma unroll
    for (int j = 1; j < E; ++j) {
      t = j == k / kLanes ? a[j] : t;
      loaded(t);                        // else the array goes to memory for an indexed read
    }
    if (part == k % kLanes) {
      sV[k * LD + row] = (row > k + 1 && row < n) ? t : 0.0;
      if (row == k) d[k] = t;
      if (row == k + 1) sX[k] = t;
    }
  };
  // rows whose wave is done are no longer stored: zero from here on
  for (int i = tid; i < NMAX * LD; i += kLanes * NMAX) sV[i] = 0.0;
  if (part == 0) sP[row] = 0.0;
  __syncthreads();
  put_column(0);
  __syncthreads();
  for (int k = 0; k < n - 2; ++k) {
    double* x = sV + k * LD;
    const bool busy = (tid | 63) / kLanes >= k;        // below, the wave's rows and sP are done
    double tau = 0.0, p = 0.0, vc[E];
    if (busy) {
      const double x0 = sX[k];
      double s2 = 0.0;
#pragma unroll
      for (int i = 0; i < (NMAX + 63) / 64; ++i) {
        const int r = lane + 64 * i;
        double t = x[min(r, NMAX - 1)];
        loaded(t);
        t = (r == k + 1 || r >= NMAX) ? 0.0 : t;       // another wave may have stored v's entry
        s2 = fma(t, t, s2);
      }
      s2 = sum64(s2);
      double v0 = 0.0, ek = x0;
      if (s2 > 0.0) {
        ek = -copysign(sqrt(fma(x0, x0, s2)), x0);
        v0 = x0 - ek;
        tau = 2.0 / fma(v0, v0, s2);
      }
      x[k + 1] = v0;                                   // every wave, the same value: no barrier
      if (tid == kLanes * NMAX - 1) {
        e[k] = ek;
        sTau[k] = tau;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
      for (int j = 0; j < E; ++j) vc[j] = x[part + kLanes * j];
#pragma unroll
      for (int j = 0; j < E; ++j) p = fma(a[j], vc[j], p);
      p = tau * sum8(p);
      p = (row > k && row < n) ? p : 0.0;
      if (part == 0) sP[row] = p;
    }
    __syncthreads();
    if (busy) {
      double wc[E], pv = 0.0;
      const double vr = x[row];
#pragma unroll
      for (int j = 0; j < E; ++j) wc[j] = sP[part + kLanes * j];
#pragma unroll
      for (int i = 0; i < (NMAX + 63) / 64; ++i) {
        const int r = lane + 64 * i, rc = min(r, NMAX - 1);
        double pr = sP[rc], xr = x[rc];
        loaded(pr);
        loaded(xr);
        pv = fma(r < NMAX ? pr : 0.0, xr, pv);
      }
      const double kk = 0.5 * tau * sum64(pv);
      const double wr = p - kk * vr;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        wc[j] = fma(-kk, vc[j], wc[j]);
        a[j] -= fma(vr, wc[j], wr * vc[j]);
      }
      put_column(k + 1);
    }
    __syncthreads();
  }
  // the last diagonal entry, and for n = 2 .. the last off-diagonal one
  if (n >= 2) {
    put_column(n - 1);
    __syncthreads();
    if (tid == 0) e[n - 2] = sX[n - 2];
  }
}

// Workgroup state of tridiag_dc.
template <int NMAX>
struct TridiagDc {
  static constexpr int LD = NMAX + 1;
  static constexpr int kMerges = NMAX <= 32 ? 4 : (NMAX <= 64 ? 8 : 16);    // of the first level
  double w[NMAX * LD];                  // eigenvectors, column j belongs to d[j]
  double d[NMAX + 1], e[NMAX + 1];      // diagonal (eigenvalues on return) and off-diagonal
  double zv[NMAX], ds[NMAX], zs[NMAX], zh[NMAX], tau[NMAX], dummy[kLanes * NMAX / 64][kLeaf + 1];
  int order[NMAX], list[NMAX], org[NMAX], rotp[NMAX], rotn[NMAX], nlist[kMerges], nrot[kMerges], bad, close;
};

// Eigenpairs of the tridiagonal matrix S.d, S.e of size n <= NMAX by a
// workgroup of kLanes NMAX threads: eigenvalues (in no order) into S.d, vectors
// into the columns of S.w.  0 done, 1 not converged, 2 not finite; the same for
// every thread, and after a barrier.
template <int NMAX>
__device__ int tridiag_dc(TridiagDc<NMAX>& S, int n) {
  constexpr int E = NMAX / kLanes;
  constexpr int LD = NMAX + 1;
  constexpr int NT = kLanes * NMAX;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = tid / kLanes, part = tid % kLanes;
  double *sW = S.w, *d = S.d, *zv = S.zv, *ds = S.ds, *zs = S.zs, *zh = S.zh, *tau = S.tau;
  const double* e = S.e;
  int *order = S.order, *list = S.list, *org = S.org, *rotp = S.rotp, *rotn = S.rotn, *nlist = S.nlist,
      *nrot = S.nrot;
  int &bad = S.bad, &close = S.close;
  for (int i = tid; i < NMAX * LD; i += NT) sW[i] = (i / LD == i % LD) ? 1.0 : 0.0;
  if (tid == 0) bad = 0;
  __syncthreads();
  // ---- leaves: boundaries n i / nleaf; every boundary's coupling is taken out
  // of the two diagonal entries beside it
  int levels = 0;
  while ((n >> levels) >= kLeaf + (((n >> levels) << levels) == n ? 1 : 0)) ++levels;
  const int nleaf = 1 << levels;
  auto bound = [&](int i, int lg) { return (n * i) >> lg; };      // part i of 2^lg
  if (tid > 0 && tid < nleaf) {
    const int b = bound(tid, levels);
    const double c = fabs(e[b - 1]);
    d[b - 1] -= c;                       // leaves have two entries or more: no overlap
    d[b] -= c;
  }
  __syncthreads();
  double tnorm = 0.0, total = 0.0;
  for (int i = 0; i < n; ++i) {
    const double x = fabs(d[i]), y = i < n - 1 ? fabs(e[i]) : 0.0;
    tnorm = fmax(tnorm, fmax(x, y));
    total += x + y;
  }
  __syncthreads();                       // d is written from here on
  if (!isfinite(total)) return 2;        // the same for every thread
  const double tol = 8.0 * kUlp * tnorm;
  for (int leaf = wave; leaf < nleaf; leaf += NT / 64) {
    const int b = bound(leaf, levels), m = bound(leaf + 1, levels) - b;
    if (!ql_leaf(d + b, e + b, m, sW + b * LD + b, LD, S.dummy[wave]) && lane == 0) bad = 1;
  }
  __syncthreads();
  // ---- merges, all pairs of a level side by side.  Groups of eight lanes: of
  // column `row`, of the sorted list's entry, and of a root in turn
  for (int lg = levels - 1; lg >= 0; --lg) {
    int b = 0;                           // the block of this group's column
    while (b + 1 < (1 << lg) && row >= bound(b + 1, lg)) ++b;
    const int lo = bound(b, lg), hi = row < n ? bound(b + 1, lg) : lo, mid = bound(2 * b + 1, lg + 1);
    const double beta = e[mid - 1], rho = 2.0 * fabs(beta);
    const bool in = row < n;
    // coupling vector (unit norm) and ascending order within the block
    if (in) {
      const double z = 0.70710678118654752440 * (row < mid ? sW[(mid - 1) * LD + row]
                                                           : copysign(1.0, beta) * sW[mid * LD + row]);
      const double v = d[row];
      double rank = 0.0;
      for (int i = lo + part; i < hi; i += kLanes) rank += d[i] < v || (d[i] == v && i < row);
      const int r = lo + (int)sum8(rank);
      if (part == 0) {
        zv[row] = z;
        order[r] = row;
      }
    }
    if (tid < TridiagDc<NMAX>::kMerges) nrot[tid] = 0;
    if (tid == 0) close = 0;
    __syncthreads();
    // entries that couple too weakly keep their eigenpair; the others form the
    // list, still ascending
    if (in) {
      const int me = order[row];
      const bool live = rho * fabs(zv[me]) > tol;
      double before = 0.0, all = 0.0;
      for (int i = lo + part; i < hi; i += kLanes) {
        const double f = rho * fabs(zv[order[i]]) > tol;
        all += f;
        before += (i < row) ? f : 0.0;
      }
      const int at = lo + (int)sum8(before), tot = (int)sum8(all);
      if (part == 0 && live) list[at] = me;
      if (part == 0 && row == lo) nlist[b] = tot;
    }
    __syncthreads();
    // neighbours that are too close: one of the two is decoupled by a rotation
    if (in && part == 0 && row - lo + 1 < nlist[b]) {
      const int p = list[row], q = list[row + 1];
      const double h = zv[p] * zv[p] + zv[q] * zv[q];
      if (fabs((d[q] - d[p]) * zv[p] * zv[q]) <= tol * h) close = 1;
    }
    __syncthreads();
    if (close) {                         // one lane per block walks its list
      if (in && part == 0 && row == lo && nlist[b] > 0) {
        const int cnt = nlist[b];
        int k = 0, nr = 0, p = list[lo], nq = list[lo + min(1, cnt - 1)];
        double dp = d[p], zp = zv[p], nd = d[nq], nz = zv[nq];
        for (int i = 1; i < cnt; ++i) {
          const int q = nq;
          double dq = nd, zq = nz;
          nq = list[lo + min(i + 1, cnt - 1)];       // read ahead
          nd = d[nq];
          nz = zv[nq];
          const double h = zp * zp + zq * zq;
          if (fabs((dq - dp) * zp * zq) <= tol * h) {
            const double r = rsqrt_f64(h), c = zq * r, s = -zp * r, x = dp;
            dp = x * c * c + dq * s * s;
            dq = x * s * s + dq * c * c;
            zq = h * r;
            zv[q] = zq;
            d[p] = dp;
            d[q] = dq;
            rotp[lo + nr] = p;
            rotn[lo + nr] = q;
            ds[lo + nr] = c;
            zs[lo + nr] = s;
            ++nr;
          } else {
            list[lo + k++] = p;
          }
          p = q;
          dp = dq;
          zp = zq;
        }
        list[lo + k++] = p;
        nlist[b] = k;
        nrot[b] = nr;
      }
      __syncthreads();
      if (in && part == 0) {             // row `row` of the block
        double* w = sW + row * LD;
        int held = -1;                   // column of the value y, not stored yet
        double y = 0.0;
        for (int i = 0; i < nrot[b]; ++i) {
          const int p = rotp[lo + i], q = rotn[lo + i];
          const double c = ds[lo + i], s = zs[lo + i], v = w[q];
          if (held != p) {
            if (held >= 0) w[held] = y;
            y = w[p];
          }
          w[p] = fma(c, y, s * v);
          y = fma(c, v, -(s * y));
          held = q;
        }
        if (held >= 0) w[held] = y;
      }
      __syncthreads();
    }
    const int k = nlist[b], j = row - lo;
    const bool active = in && j < k;
    if (active && part == 0) {
      ds[row] = d[list[row]];
      zs[row] = zv[list[row]] * zv[list[row]];
    }
    __syncthreads();
    int o = 0;
    double tj = 0.0;
    if (active) {
      secular_root<kLanes>(ds + lo, zs + lo, k, j, rho, o, tj);
      if (part == 0) {
        org[row] = o;
        tau[row] = tj;
      }
    }
    __syncthreads();
    // coupling vector that has exactly these roots
    if (active) {
      const double di = ds[row];
      double pr = 1.0;
      for (int i = part; i < k; i += kLanes) {
        const double gap = (ds[lo + org[lo + i]] - di) + tau[lo + i];
        pr *= (i == j) ? gap : gap / (ds[lo + i] - di);
      }
      pr = product8(pr);
      if (part == 0) zh[row] = copysign(sqrt(fabs(pr)), zv[list[row]]);
    }
    __syncthreads();
    // eigenvectors: column list[j] of the block; lane `part` has every eighth row
    double out[E];
    if (active) {
      const double dj = ds[lo + o];
      double nn = 0.0, tv[E];            // entry part + 8 m of the rank-one update's vector
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int i = part + kLanes * m;
        tv[m] = 0.0;
        if (i < k) tv[m] = zh[lo + i] / ((ds[lo + i] - dj) - tj);
        nn = fma(tv[m], tv[m], nn);
      }
      const double f = 1.0 / sqrt(sum8(nn));
#pragma unroll
      for (int q = 0; q < E; ++q) out[q] = 0.0;
      const double* w0 = sW + (lo + part) * LD;
#pragma unroll
      for (int m = 0; m < E; ++m) {
        if (kLanes * m >= k) break;
        tv[m] *= f;
#pragma unroll 2
        for (int s = 0; s < kLanes; ++s) {
          const int i = min(kLanes * m + s, k - 1);
          const double t = __shfl(tv[m], (lane & ~(kLanes - 1)) + s, 64);     // zero past k
          const double* w = w0 + list[lo + i];
#pragma unroll
          for (int q = 0; q < E; ++q) out[q] = fma(t, w[min(q * kLanes, NMAX - 1 - lo - part) * LD], out[q]);
        }
      }
    }
    __syncthreads();
    if (active) {
      const int col = list[row];
#pragma unroll
      for (int q = 0; q < E; ++q)
        if (lo + part + q * kLanes < hi) sW[(lo + part + q * kLanes) * LD + col] = out[q];
      if (part == 0) {
        const double v = ds[lo + o] + tj;
        d[col] = isfinite(v) ? v : 0.0;  // the ordering needs numbers
        if (!isfinite(v)) bad = 1;
      }
    }
    __syncthreads();
  }
  return bad;
}

}  // namespace
}  // namespace d3s
