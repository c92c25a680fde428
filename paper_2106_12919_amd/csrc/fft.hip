// LDS-staged mixed-radix Stockham FFT for gfx950 (radices 2, 3, 4, 6, 8, 9, 12).
//
// The paper's field solve transforms every grid quantity to Fourier space and
// back (Sec. 2, "solve Maxwell's equations on the Yee grid in Fourier space";
// discrete transform of App. A).  The staggered half-cell phase factors are not
// applied here: they are folded into the per-mode update (psatd.hip), so these
// kernels compute the plain index-space DFT.
//
// A real 3D transform runs three passes, each one read and one write of the
// array in HBM:
//   z pass  (r2c/c2r): two real z-lines packed as one complex line, one
//           workgroup per group of line pairs, lines contiguous in LDS;
//   y, x    (c2c):     a tile of TL lines that are adjacent in memory (the kz
//           index, or the flattened (ky,kz) index for x), so every global
//           access is a TL-wide contiguous row; in LDS the tile is stored
//           element-major with the line index fastest, which keeps the
//           butterfly reads and writes free of bank conflicts.
// Each Stockham stage reads its radix-R butterfly inputs from LDS and writes the outputs in autosorted
// order, to a second buffer (z) or in place after a barrier (x, y).
//
// Every length has kernels of its own, with its stages, strides and divisions as compile-time constants.
// With the plan as a runtime argument (the earlier kernels of the lengths other than 64, 128, 256, 384 and
// 768) the passes were bound by address arithmetic: 216 x 216 x 288 FP64, 11 arrays forward, one axis
// 757 us against 532 (4.7 TB/s), z 715 against 486 (4.9 TB/s); 96 x 96 x 192 FP32, one axis 23.7
// against 15.3 us.  It also lets every grid centre inside its transforms.
#include <utility>

#include "fft_kernels.h"

namespace pic {

namespace {

// The launchers of an axis length, or null for a length that is not in kFftLengths.
template <typename T, int... U>
const FftOps<T>* length_ops(int n, std::integer_sequence<int, U...>) {
  const FftOps<T>* found = nullptr;
  (void)((found = fft_ops<T, U>(n)) || ...);
  return found;
}

// A twiddle (c, s) = (cos, sin) of an exact angle in the run precision.  Rounding c and s
// separately leaves |w|^2 - 1 up to ~1e-7 in FP32, the same factor on every pass through that
// twiddle, which the field energy carried by those modes then gains or loses step after step.  In
// FP32 the pair is chosen among the roundings of c and s and their neighbours (each within one
// unit in the last place) as the one whose squared modulus is closest to 1; FP64 rounds directly.
template <typename T>
cplx<T> unit_twiddle(double c, double s) {
  if (sizeof(T) == 8) return cmake((T)c, (T)s);
  cplx<T> best = cmake((T)c, (T)s);
  double err = std::fabs((double)best.x * best.x + (double)best.y * best.y - 1.0);
  const float c0 = (float)c, s0 = (float)s;
  const float cs[3] = {std::nextafter(c0, -2.0f), c0, std::nextafter(c0, 2.0f)};
  const float ss[3] = {std::nextafter(s0, -2.0f), s0, std::nextafter(s0, 2.0f)};
  for (float cc : cs)
    for (float sc : ss) {
      const double e = std::fabs((double)cc * cc + (double)sc * sc - 1.0);
      if (e < err) {
        err = e;
        best = cmake((T)cc, (T)sc);
      }
    }
  return best;
}

}  // namespace

template <typename T>
hipError_t Fft3D<T>::init(int nx_, int ny_, int nz_) {
  nx = nx_; ny = ny_; nz = nz_;
  nzh = nz / 2 + 1;
  const int align = (int)(128 / sizeof(cplx<T>));
  pz = (nzh + align - 1) / align * align;
  const int n[3] = {nx, ny, nz};
  for (int d = 0; d < 3; ++d) {
    plan[d] = make_fft_plan(n[d], d == 2);
    ops[d] = length_ops<T>(n[d], std::make_integer_sequence<int, kFftUnits>{});
    if (plan[d].nstages < 0 || !ops[d]) return hipErrorInvalidValue;
    const int cnt = plan[d].twcount > 0 ? plan[d].twcount : 1;
    double* h = new double[2 * (size_t)cnt]();
    fft_twiddles(plan[d], h);
    cplx<T>* hc = new cplx<T>[cnt];
    for (int i = 0; i < cnt; ++i) hc[i] = unit_twiddle<T>(h[2 * i], h[2 * i + 1]);
    hipError_t e = hipMalloc(&tw[d], cnt * sizeof(cplx<T>));
    if (e == hipSuccess) e = hipMemcpy(tw[d], hc, cnt * sizeof(cplx<T>), hipMemcpyHostToDevice);
    delete[] h;
    delete[] hc;
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
void Fft3D<T>::release() {
  for (int d = 0; d < 3; ++d) {
    if (tw[d]) (void)hipFree(tw[d]);
    tw[d] = nullptr;
  }
}

template <typename T>
void Fft3D<T>::forward(const Batch<const T*>& in, const Batch<cplx<T>*>& out, int count, hipStream_t s,
                       const LineCenter<T>* lcp, bool x_pass) const {
  const LineCenter<T> lc = lcp ? *lcp : LineCenter<T>();
  ops[2]->r2c(in, out, count, tw[2], nx * ny, pz, lc, s);
  Batch<const cplx<T>*> cin;
  for (int i = 0; i < count; ++i) cin.p[i] = out.p[i];
  ops[1]->strided[0](cin, out, count, tw[1], nx, nzh, (long long)ny * pz, pz, lc, 1, s);
  if (x_pass) ops[0]->strided[0](cin, out, count, tw[0], 1, ny * pz, 0, (long long)ny * pz, lc, 0, s);
}

// (the rule and its measurements: solve_from_kib)
template <typename T>
bool Fft3D<T>::solves_along_x() const {
  return ops[0]->solve_x != nullptr && (size_t)nx * ny * nz * sizeof(T) >= ops[0]->solve_from;
}

template <typename T>
void Fft3D<T>::solve_x(const SolveX<T>& a, hipStream_t s) const {
  ops[0]->solve_x(a, tw[0], s);
}

template <typename T>
void Fft3D<T>::inverse(const Batch<const cplx<T>*>& in, const Batch<cplx<T>*>& scratch, const Batch<T*>& out,
                       int count, double scale, hipStream_t s, const LineCenter<T>* lcp, bool x_pass) const {
  const LineCenter<T> lc = lcp ? *lcp : LineCenter<T>();
  const T sc_hi = (T)scale, sc_lo = (T)(scale - (double)sc_hi);
  if (x_pass) ops[0]->strided[1](in, scratch, count, tw[0], 1, ny * pz, 0, (long long)ny * pz, lc, 0, s);
  Batch<const cplx<T>*> cs;
  for (int i = 0; i < count; ++i) cs.p[i] = scratch.p[i];
  ops[1]->strided[1](cs, scratch, count, tw[1], nx, nzh, (long long)ny * pz, pz, lc, 1, s);
  ops[2]->c2r(cs, out, count, tw[2], nx * ny, pz, sc_hi, sc_lo, lc, s);
}

template struct Fft3D<float>;
template struct Fft3D<double>;

}  // namespace pic
