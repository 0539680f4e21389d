// Function-approximation weights on the device (eqn:fT): for every column's
// tridiagonal T (the recurrence coefficients in device memory), the common
// shift E0 = min over the columns of the smallest eigenvalue of T,
//   y_b = exp(-b (T - E0) / 2) e_1   for H_t's columns (the Gram's weights),
//   e_1^T exp(-b (T - E0b)) e_1 = |exp(-b (T - E0b) / 2) e_1|^2 for H_b's.
//
// One wave per column.  The smallest eigenvalue comes from Sturm counts
// (Givens' bisection) at 64 points at a time, the exponentials from their
// Chebyshev series on the column's own interval, from its smallest eigenvalue
// e to its Gershgorin bound,
//   exp(-z (t + 1)) = sum_n' 2 (-1)^n e^-z I_n(z) T_n(t),  |t| <= 1,
// times exp(-b (e - E0) / 2): the sum's rounding is 1e-16 of its own largest
// value, so the weights of a column that lies above E0 (a sector of a conserved
// quantity) keep their relative accuracy however far above.  Its terms are
// the modified Bessel functions by Miller's backward recurrence (normalised by
// e^z = I_0 + 2 sum I_n), each times a product with the tridiagonal T, one row
// per lane, so no eigenvectors are formed.
//
// What bounds it: the latency of these two chains (k x 9 dependent divisions,
// 21 us at k = 30, 35-41 at 60; 30 + 10 sqrt(z) products, 9-32 us), whatever
// the number of columns up to the chip's waves.  On 16 host threads (implicit QR per column,
// coefficients copied to the host and weights back) 3 x 500 columns with
// 8 temperatures took 25 ms of a solve, now 0.25 ms; 80 columns with
// 4 temperatures 1.6 ms, now 0.06 ms; 12 columns with k = 30 0.3 ms, now 0.04;
// the product-state estimate's 2 x 64 columns (2 + 18 sites) 0.4 ms of 9.3.
#include "internal.h"

namespace rdm {

namespace {

constexpr int kTriMax = kTriRows * 64;

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wave_add(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// column x of the launch: H_t's columns first (with the padding when PAD),
// then H_b's
struct TriCol {
  bool bath;
  int c;
};

}  // namespace

// Smallest eigenvalue and Gershgorin upper bound of one column's T; NaN when a
// coefficient is not finite or the column has no step.
__global__ __launch_bounds__(64) void k_tri_bounds(TriArgs a) {
  __shared__ double al[kTriMax], b2[kTriMax];
  const int lane = threadIdx.x;
  const TriCol col{(int)blockIdx.x >= a.t.C, (int)blockIdx.x >= a.t.C ? (int)blockIdx.x - a.t.C : (int)blockIdx.x};
  const TriSeg& s = col.bath ? a.b : a.t;
  const int c = col.c, cp = s.cpad, kk = s.kc[c];
  bool bad = kk < 1;
  double lo = INFINITY, amin = INFINITY, hi = -INFINITY;
  for (int i = lane; i < s.k; i += 64) {
    // (k - 1 off-diagonals: nothing writes row k - 1 of hb)
    const double x = s.ha[(uint64_t)i * cp + c], y = i + 1 < s.k ? s.hb[(uint64_t)i * cp + c] : 0.0;
    bad |= !(fabs(x) < INFINITY) || !(fabs(y) < INFINITY);
    if (i < kk) {
      const double bp = i > 0 ? fabs(s.hb[(uint64_t)(i - 1) * cp + c]) : 0.0;
      const double bn = i + 1 < kk ? fabs(y) : 0.0;
      al[i] = x;
      b2[i] = bp * bp;
      lo = fmin(lo, x - bp - bn);
      hi = fmax(hi, x + bp + bn);
      amin = fmin(amin, x);
    }
  }
  bad = __any(bad);
  lo = wave_min(lo);
  amin = wave_min(amin);
  hi = wave_max(hi);
  __syncthreads();
  double* tmin = a.scratch + (col.bath ? 2 * a.t.C : 0);
  if (bad) {
    if (lane == 0) tmin[c] = tmin[s.C + c] = NAN;
    return;
  }
  // lambda_min lies in [lo, amin] (amin: the smallest Rayleigh quotient of a
  // unit vector e_i); 64 interior points a pass
  const double top = hi, tiny = 1e-300;
  hi = amin;
  for (int pass = 0; pass < 12; ++pass) {
    const double w = hi - lo;
    if (!(w > 4.5e-16 * fmax(fabs(lo), fabs(hi)))) break;
    const double x = lo + w * ((lane + 1) * (1.0 / 65.0));
    bool neg = false;
    double q = 1.0;
    for (int i = 0; i < kk; ++i) {
      q = al[i] - x - b2[i] / q;
      if (fabs(q) < tiny) q = -tiny;
      neg |= q < 0.0;
    }
    const uint64_t m = __ballot(neg);      // lanes whose point lies above lambda_min
    const int f = m ? __builtin_ctzll(m) : 64;
    const double xl = __shfl(x, f > 0 ? f - 1 : 0, 64), xh = __shfl(x, f < 64 ? f : 63, 64);
    if (f > 0) lo = xl;
    if (f < 64) hi = xh;
  }
  if (lane == 0) {
    tmin[c] = 0.5 * (lo + hi);
    tmin[s.C + c] = top;
  }
}

// The weights (H_t's columns, in the recombination's layout and scaling; the
// quadratures when there is no place for them) and the quadratures (H_b's) of
// inverse temperature blockIdx.y.
template <typename T, int R>
__global__ __launch_bounds__(64) void k_tri_weights(TriArgs a) {
  extern __shared__ double cf[];           // e^-z I_n(z), n <= N
  const int lane = threadIdx.x;
  const TriCol col{(int)blockIdx.x >= a.t.cpad, (int)blockIdx.x >= a.t.cpad ? (int)blockIdx.x - a.t.cpad : (int)blockIdx.x};
  const TriSeg& s = col.bath ? a.b : a.t;
  const int c = col.c, cp = s.cpad, ib = a.beta0 + (int)blockIdx.y;
  const bool weights = !col.bath && a.yt;  // else the quadrature
  T* yt = (T*)a.yt + (uint64_t)ib * a.t.k * a.t.cpad + c;
  double* out = a.scratch + 2 * (a.t.C + a.b.C) + (uint64_t)a.n_beta * a.b.C;
  double* quad = col.bath ? out - (uint64_t)(a.n_beta - ib) * a.b.C : out + kTriOut + (uint64_t)ib * a.t.C;
  if (!col.bath && c >= s.C) {
    if (weights)
      for (int i = lane; i < s.k; i += 64) yt[(uint64_t)i * cp] = T(0);
    return;
  }
  const double* tmin = a.scratch + (col.bath ? 2 * a.t.C : 0);
  double e0 = INFINITY;
  bool bad = false;
  for (int i = lane; i < s.C; i += 64) {
    bad |= !(tmin[i] < INFINITY);
    e0 = fmin(e0, tmin[i]);
  }
  e0 = wave_min(e0);
  bad = __any(bad);
  if (c == 0 && blockIdx.y == 0) {
    int brk = 0;
    for (int i = lane; i < s.C; i += 64) brk += s.kc[i] < s.k ? 1 : 0;
    const double nb = wave_add((double)brk);
    if (lane == 0) {
      out[col.bath ? 1 : 0] = bad ? NAN : e0;
      out[col.bath ? 3 : 2] = nb;
    }
  }
  if (bad) return;                         // the host sees the NaN and drops the instance
  // T = mid + half t with |t| <= 1 on the column's spectrum (a little room
  // below its smallest eigenvalue for the rounding of that)
  const double ec = tmin[c], top = tmin[s.C + c];
  const double bot = ec - 1e-14 * fmax(fabs(ec), fabs(top));
  const double half = 0.5 * (top - bot), mid = 0.5 * (top + bot);
  const double hb = 0.5 * a.beta[blockIdx.y], z = hb * half;
  const double low = exp(hb * (e0 - bot));  // exp(-hb (T - E0)) = low exp(-z (t + 1))
  const int kk = s.kc[c];
  double y[R], t0[R], t1[R], ad[R], au[R], dn[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = lane * R + r;
    const double inv = half > 0.0 ? 1.0 / half : 0.0;
    ad[r] = i < kk ? (s.ha[(uint64_t)i * cp + c] - mid) * inv : 0.0;
    au[r] = i > 0 && i < kk ? s.hb[(uint64_t)(i - 1) * cp + c] * inv : 0.0;
    dn[r] = i + 1 < kk ? s.hb[(uint64_t)i * cp + c] * inv : 0.0;
    t0[r] = i == 0 ? 1.0 : 0.0;
  }
  // w = A t for the tridiagonal A = (T - mid) / half
  auto product = [&](const double (&t)[R], double (&w)[R]) {
    const double up = __shfl_up(t[R - 1], 1, 64), down = __shfl_down(t[0], 1, 64);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double tu = r > 0 ? t[r - 1] : up, td = r + 1 < R ? t[r + 1] : down;
      w[r] = fma(ad[r], t[r], fma(au[r], tu, dn[r] * td));
    }
  };
  if (half > 0.0 && z > 1e-17) {
    // Miller's recurrence I_(n-1) = I_(n+1) + (2 n / z) I_n downwards from N
    // terms: e^-z I_N(z) < 1e-21 there, and the start value does not overflow
    const int n_terms = z < 1e-4 ? 6 : z < 1.0 ? 20 : min(a.n_terms(z), a.max_terms);
    double pn1 = 0.0, pn = 1e-300, sum = 0.0;
    const double tz = 2.0 / z;
    for (int n = n_terms; n > 0; --n) {
      if (lane == 0) cf[n] = pn;
      sum += pn;
      const double p = fma(n * tz, pn, pn1);
      pn1 = pn;
      pn = p;
    }
    if (lane == 0) cf[0] = pn;
    __syncthreads();
    const double nrm = 1.0 / (pn + 2.0 * sum);
    product(t0, t1);
#pragma unroll
    for (int r = 0; r < R; ++r) y[r] = cf[0] * t0[r];
    double sg = -2.0;
    for (int n = 1; n <= n_terms; ++n) {
      const double f = sg * cf[n];
      double w[R];
      product(t1, w);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        y[r] = fma(f, t1[r], y[r]);
        w[r] = fma(2.0, w[r], -t0[r]);
        t0[r] = t1[r];
        t1[r] = w[r];
      }
      sg = -sg;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) y[r] *= nrm;
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) y[r] = t0[r];   // a single eigenvalue, or exp(-z (t + 1)) = 1 to rounding
  }
  const double s1 = s.hs[c];
  if (!weights) {
    double q = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) q = fma(y[r], y[r], q);
    q = wave_add(q);
    if (lane == 0) quad[c] = q * exp(2.0 * hb * (e0 - bot)) / (s1 * s1);  // (low^2 would vanish first)
    return;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = lane * R + r;
    if (i < s.k) yt[(uint64_t)i * cp] = i < kk ? (T)(a.bscale * (low * y[r]) * s.hs[(uint64_t)i * cp + c] / s1) : T(0);
  }
}

template <typename T>
hipError_t launch_tri(const TriArgs& args, const double* betas, int n_beta, double zmax, hipStream_t st) {
  hipLaunchKernelGGL(k_tri_bounds, dim3(args.t.C + args.b.C), dim3(64), 0, st, args);
  TriArgs a = args;
  a.max_terms = a.n_terms(zmax);
  const int k = args.t.k > args.b.k ? args.t.k : args.b.k;
  const size_t shm = sizeof(double) * ((size_t)a.max_terms + 1);
  for (a.beta0 = 0; a.beta0 < n_beta; a.beta0 += kTriBetas) {
    const int nb = n_beta - a.beta0 < kTriBetas ? n_beta - a.beta0 : kTriBetas;
    for (int b = 0; b < nb; ++b) a.beta[b] = betas[a.beta0 + b];
    const dim3 grid(args.t.cpad + args.b.C, nb);
    if (k <= 64) hipLaunchKernelGGL((k_tri_weights<T, 1>), grid, dim3(64), shm, st, a);
    else if (k <= 128) hipLaunchKernelGGL((k_tri_weights<T, 2>), grid, dim3(64), shm, st, a);
    else hipLaunchKernelGGL((k_tri_weights<T, kTriRows>), grid, dim3(64), shm, st, a);
  }
  return hipGetLastError();
}
template hipError_t launch_tri<float>(const TriArgs&, const double*, int, double, hipStream_t);
template hipError_t launch_tri<double>(const TriArgs&, const double*, int, double, hipStream_t);

}  // namespace rdm
