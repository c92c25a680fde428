// Internal declarations shared by the HIP translation units of libpic.
// Nothing here is part of the public ABI (include/pic.h).
#pragma once
#include <complex>

#include <hip/hip_runtime.h>
#include <cstdint>
#include <string>

namespace pic {

template <typename T>
struct alignas(2 * sizeof(T)) cplx {
  T x, y;
};

template <typename T>
__host__ __device__ inline cplx<T> cmake(T x, T y) { cplx<T> c; c.x = x; c.y = y; return c; }
template <typename T>
__host__ __device__ inline cplx<T> cadd(cplx<T> a, cplx<T> b) { return cmake(a.x + b.x, a.y + b.y); }
template <typename T>
__host__ __device__ inline cplx<T> csub(cplx<T> a, cplx<T> b) { return cmake(a.x - b.x, a.y - b.y); }
template <typename T>
__host__ __device__ inline cplx<T> cmul(cplx<T> a, cplx<T> b) {
  return cmake(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <typename T>
__host__ __device__ inline cplx<T> cscale(cplx<T> a, T s) { return cmake(a.x * s, a.y * s); }
template <typename T>
__host__ __device__ inline cplx<T> cconj(cplx<T> a) { return cmake(a.x, -a.y); }
// multiply by -i (sign < 0) or +i (sign > 0)
template <typename T, int SIGN>
__host__ __device__ inline cplx<T> cmul_i(cplx<T> a) {
  return SIGN > 0 ? cmake(-a.y, a.x) : cmake(a.y, -a.x);
}

constexpr int kMaxStages = 12;
constexpr int kMaxBatch = 12;

// One axis of the mixed-radix Stockham FFT.  Stage s has radix radix[s]; ns[s] is
// the product of the radices of the stages before it; the twiddles of stage s,
// exp(-2 pi i k r / (ns R)) for k < ns and 1 <= r < R, start at twoff[s] of the
// table (entry k*(R-1) + r-1).
struct FftPlan {
  int n;
  int nstages;
  int radix[kMaxStages];
  int ns[kMaxStages];
  int twoff[kMaxStages];
  int twcount;
};

// Stages of an axis of n = 2^a 3^b points: the fewest radices out of 2, 3, 4, 6, 8, 9, 12 with
// product n (every stage is a pass over LDS and a barrier), of those the smallest sum (registers,
// twiddles).
constexpr int kRadices[] = {2, 3, 4, 6, 8, 9, 12};
constexpr int plan_cost(int n) {  // 1000 per stage plus the sum of the radices; < 0: none
  if (n == 1) return 0;
  int best = -1;
  for (int r : kRadices)
    if (n % r == 0) {
      const int c = plan_cost(n / r);
      if (c >= 0 && (best < 0 || c + 1000 + r < best)) best = c + 1000 + r;
    }
  return best;
}

// The plan of an axis (nstages = -1 for other n).  Along z a line is contiguous in LDS and the first
// stage writes at a stride of its radix, which conflicts on the banks unless the radix is odd: there a
// length with a factor 3 starts with a stage of radix 9 or 3, also at the cost of one stage more
// (c2r of 768 points, FP32, 384 x 384 lines: 12 8 8 1.40 ms, 3 8 8 4 1.35; 384 points, FP64: 6 8 8
// 300 us, 3 8 4 4 293).  On the strided axes lanes run over lines, which never conflict, and the radices go
// odd first, then from large to small.  A constant expression, so that the kernels specialised for
// an axis length take the same stages and twiddle offsets as the table the host builds from it.
constexpr FftPlan plan_of(int n, bool z) {
  FftPlan p{};
  p.n = n;
  int cost = n > 0 ? plan_cost(n) : -1;
  if (cost < 0 || cost / 1000 > kMaxStages - 1) {
    p.nstages = -1;
    return p;
  }
  int left = n, k = 0, count[16] = {};
  if (z && n % 3 == 0) {
    const int f = n % 9 == 0 ? 9 : 3;
    p.radix[k++] = f;
    left /= f;
  }
  while (left > 1)
    for (int r : kRadices)
      if (left % r == 0 && plan_cost(left / r) >= 0 && plan_cost(left / r) + 1000 + r == plan_cost(left)) {
        ++count[r];
        left /= r;
        break;
      }
  const int order[] = {9, 3, 12, 8, 6, 4, 2};
  for (int r : order)
    for (int c = 0; c < count[r]; ++c) p.radix[k++] = r;
  p.nstages = k;
  int ns = 1, off = 0;
  for (int s = 0; s < k; ++s) {
    p.ns[s] = ns;
    p.twoff[s] = off;
    off += ns * (p.radix[s] - 1);
    ns *= p.radix[s];
  }
  p.twcount = off;
  return p;
}
inline FftPlan make_fft_plan(int n, bool z = false) { return plan_of(n, z); }
// FP64 twiddles of a plan, 2*twcount doubles (re, im) of exp(-2 pi i k r/(ns R)).
void fft_twiddles(const FftPlan& p, double* out);

// Pointer batches passed to kernels by value.
template <typename P>
struct Batch {
  P p[kMaxBatch];
};

// Host FP64 tables (tables.cpp).
void alpha_staggered(int m, double* out);                  // out[n-1], n = 1..m
void k_staggered_axis(int n, double d, int order, double* out);  // [k]_s on fftfreq order
// Standard Galilean PSATD coefficients of one mode (Sec. 4.3), w = c |[k]_s|, W = v_gal . [k]_c:
// out = theta^2 C, theta^2 S/w, X1, X2, theta^2 X3, X4 (complex, FP64).
void galilean_coefficients(double w, double W, double dt, std::complex<double>* out);
// Averaged Galilean PSATD coefficients of one mode (Sec. 4.4): Psi1, Psi2, Y1, Y2, Y3, Y4.
void averaged_coefficients(double w, double W, double dt, std::complex<double>* out);
void alpha_centered(int m, double* out);                   // out[n-1], n = 1..m
void k_centered_axis(int n, double d, int order, double* out);   // [k]_c on fftfreq order
void psatd_coefficients(double w, double dt, double* C, double* S_over_w, double* X1, double* X2, double* X3);

}  // namespace pic
