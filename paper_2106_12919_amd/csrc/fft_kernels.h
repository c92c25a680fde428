// LDS-staged mixed-radix Stockham FFT for gfx950: the kernels, templates on the axis length, and the
// table of launchers per length that fft.hip calls.  fft_len.hip instantiates the lengths.
#pragma once

#include <type_traits>

#include "kernels.h"

namespace pic {

// Launchers of one axis length.
template <typename T>
struct FftOps {
  void (*r2c)(const Batch<const T*>& in, const Batch<cplx<T>*>& out, int count, const cplx<T>* tw, int nlines, int pz,
              const LineCenter<T>& lc, hipStream_t s);
  void (*c2r)(const Batch<const cplx<T>*>& in, const Batch<T*>& out, int count, const cplx<T>* tw, int nlines, int pz,
              T scale, T scale_lo, const LineCenter<T>& lc, hipStream_t s);
  void (*strided[2])(const Batch<const cplx<T>*>& in, const Batch<cplx<T>*>& out, int count, const cplx<T>* tw,
                     int outer_count, int inner_count, long long outer_stride, long long elem_stride,
                     const LineCenter<T>& lc, int axis, hipStream_t s);  // forward, inverse
  // x pass, standard update and inverse x pass in one kernel (null where it is not built), and the bytes
  // per array from which it is the faster form
  void (*solve_x)(const SolveX<T>& a, const cplx<T>* tw, hipStream_t s);
  size_t solve_from;
};
// The axis lengths pic_init accepts: every even 2^a 3^b in [8, 1024].  fft_len.hip is compiled once per
// unit u = 0 .. kFftUnits - 1 (in parallel) with the lengths at u, u + kFftUnits, ...
constexpr int kFftLengths[] = {8,   12,  16,  18,  24,  32,  36,  48,  54,  64,  72,  96,  108, 128, 144, 162,
                               192, 216, 256, 288, 324, 384, 432, 486, 512, 576, 648, 768, 864, 972, 1024};
constexpr int kFftLengthCount = sizeof(kFftLengths) / sizeof(kFftLengths[0]);
constexpr int kFftUnits = 16;

// The launchers of length n if it is one of unit U's, else null (fft_len.hip).
template <typename T, int U>
const FftOps<T>* fft_ops(int n);

namespace {

constexpr int kBlock = 256;

template <typename T, int SIGN>
__device__ inline void dft2(cplx<T>* v) {
  cplx<T> a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

// x times an irrational constant c = hi + lo (hi the nearest T, lo the remainder), rounded once:
// the product carries c to twice the precision of T.  A constant rounded to T alone scales the
// modes it touches by |fl(c)/c| != 1 on every pass, and in FP32 that is a systematic loss or gain
// of field energy of ~1e-8 per butterfly stage, the same for every mode that goes through it.
template <typename T>
__device__ inline T mul_const(T x, T hi, T lo) {
  return fma(hi, x, lo * x);
}

template <typename T, int SIGN>
__device__ inline void dft3(cplx<T>* v) {
  // X1 = v0 - (v1+v2)/2 + SIGN i (sqrt3/2)(v1 - v2), X2 = conjugate combination.
  constexpr double hd = 0.86602540378443864676372317075294;
  const T hh = (T)hd, hl = (T)(hd - (double)(T)hd);
  cplx<T> t = cadd(v[1], v[2]);
  cplx<T> d = csub(v[1], v[2]);
  cplx<T> m = cmake(v[0].x - (T)0.5 * t.x, v[0].y - (T)0.5 * t.y);
  const cplx<T> id = cmul_i<T, SIGN>(d);
  cplx<T> r = cmake(mul_const(id.x, hh, hl), mul_const(id.y, hh, hl));
  v[0] = cadd(v[0], t);
  v[1] = cadd(m, r);
  v[2] = csub(m, r);
}

template <typename T, int SIGN>
__device__ inline void dft4(cplx<T>* v) {
  cplx<T> t0 = cadd(v[0], v[2]);
  cplx<T> t1 = csub(v[0], v[2]);
  cplx<T> t2 = cadd(v[1], v[3]);
  cplx<T> t3 = cmul_i<T, SIGN>(csub(v[1], v[3]));
  v[0] = cadd(t0, t2);
  v[2] = csub(t0, t2);
  v[1] = cadd(t1, t3);
  v[3] = csub(t1, t3);
}

template <typename T, int SIGN>
__device__ inline void dft8(cplx<T>* v) {
  constexpr double sd = 0.70710678118654752440084436210485;
  const T sh = (T)sd, sl = (T)(sd - (double)(T)sd);
  cplx<T> e[4] = {v[0], v[2], v[4], v[6]};
  cplx<T> o[4] = {v[1], v[3], v[5], v[7]};
  dft4<T, SIGN>(e);
  dft4<T, SIGN>(o);
  // twiddles w^k = exp(SIGN i 2 pi k / 8), k = 0..3
  cplx<T> o1 = cmake(mul_const(o[1].x - (T)SIGN * o[1].y, sh, sl), mul_const(o[1].y + (T)SIGN * o[1].x, sh, sl));
  cplx<T> o2 = cmul_i<T, SIGN>(o[2]);
  cplx<T> o3 = cmake(mul_const(-o[3].x - (T)SIGN * o[3].y, sh, sl), mul_const(-o[3].y + (T)SIGN * o[3].x, sh, sl));
  v[0] = cadd(e[0], o[0]);
  v[4] = csub(e[0], o[0]);
  v[1] = cadd(e[1], o1);
  v[5] = csub(e[1], o1);
  v[2] = cadd(e[2], o2);
  v[6] = csub(e[2], o2);
  v[3] = cadd(e[3], o3);
  v[7] = csub(e[3], o3);
}

// 6 = 2 x 3 and 12 = 4 x 3 as prime-factor transforms (index maps instead of twiddles):
// x[(N2 n1 + N1 n2) mod N] -> X[(N2 (N2^-1 mod N1) k1 + N1 (N1^-1 mod N2) k2) mod N].
template <typename T, int SIGN>
__device__ inline void dft6(cplx<T>* v) {
  cplx<T> a[3] = {v[0], v[2], v[4]}, b[3] = {v[3], v[5], v[1]};
  dft3<T, SIGN>(a);
  dft3<T, SIGN>(b);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    v[(4 * k) % 6] = cadd(a[k], b[k]);
    v[(3 + 4 * k) % 6] = csub(a[k], b[k]);
  }
}

template <typename T, int SIGN>
__device__ inline void dft12(cplx<T>* v) {
  cplx<T> a[3][4];
#pragma unroll
  for (int n1 = 0; n1 < 3; ++n1) {
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) a[n1][n2] = v[(4 * n1 + 3 * n2) % 12];
    dft4<T, SIGN>(a[n1]);
  }
#pragma unroll
  for (int k2 = 0; k2 < 4; ++k2) {
    cplx<T> c[3] = {a[0][k2], a[1][k2], a[2][k2]};
    dft3<T, SIGN>(c);
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) v[(4 * k1 + 9 * k2) % 12] = c[k1];
  }
}

// z times the unit (c + SIGN i s) with c, s given in FP64 and carried to twice the precision of T.
template <typename T, int SIGN>
__device__ inline cplx<T> mul_unit(cplx<T> z, double c, double s) {
  const T ch = (T)c, cl = (T)(c - (double)(T)c), sh = (T)(SIGN * s), sl = (T)(SIGN * s - (double)(T)(SIGN * s));
  return cmake(fma(ch, z.x, fma(-sh, z.y, fma(cl, z.x, -sl * z.y))), fma(ch, z.y, fma(sh, z.x, fma(cl, z.y, sl * z.x))));
}

// 9 = 3 x 3: three dft3 over n1 of x[3 n1 + n2], times exp(SIGN 2 pi i n2 k1 / 9), three over n2.
template <typename T, int SIGN>
__device__ inline void dft9(cplx<T>* v) {
  constexpr double c1 = 0.76604444311897803520239265055542, s1 = 0.64278760968653932632264340990726;   // 2 pi / 9
  constexpr double c2 = 0.17364817766693034885171662676931, s2 = 0.98480775301220805936674302458952;   // 4 pi / 9
  constexpr double c4 = -0.93969262078590838405410927732473, s4 = 0.34202014332566873304409961468226;  // 8 pi / 9
  cplx<T> a[3][3];
#pragma unroll
  for (int n2 = 0; n2 < 3; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < 3; ++n1) a[n2][n1] = v[3 * n1 + n2];
    dft3<T, SIGN>(a[n2]);
  }
  a[1][1] = mul_unit<T, SIGN>(a[1][1], c1, s1);
  a[1][2] = mul_unit<T, SIGN>(a[1][2], c2, s2);
  a[2][1] = mul_unit<T, SIGN>(a[2][1], c2, s2);
  a[2][2] = mul_unit<T, SIGN>(a[2][2], c4, s4);
#pragma unroll
  for (int k1 = 0; k1 < 3; ++k1) {
    cplx<T> c[3] = {a[0][k1], a[1][k1], a[2][k1]};
    dft3<T, SIGN>(c);
#pragma unroll
    for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = c[k2];
  }
}

template <typename T, int SIGN, int R>
__device__ inline void dft(cplx<T>* v) {
  if constexpr (R == 2) dft2<T, SIGN>(v);
  else if constexpr (R == 3) dft3<T, SIGN>(v);
  else if constexpr (R == 4) dft4<T, SIGN>(v);
  else if constexpr (R == 6) dft6<T, SIGN>(v);
  else if constexpr (R == 8) dft8<T, SIGN>(v);
  else if constexpr (R == 9) dft9<T, SIGN>(v);
  else dft12<T, SIGN>(v);
}

// One butterfly of a Stockham stage: reads src[(b + r*nb)] and writes dst[j0 + r*ns].
template <typename T, int SIGN, int R>
__device__ inline void butterfly(const cplx<T>* __restrict__ src, cplx<T>* __restrict__ dst, int lbase, int js,
                                 int b, int nb, int ns, const cplx<T>* __restrict__ tw) {
  cplx<T> v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = src[lbase + (b + r * nb) * js];
  const int k = b % ns;
  if (ns > 1) {
#pragma unroll
    for (int r = 1; r < R; ++r) {
      cplx<T> w = tw[k * (R - 1) + r - 1];
      if (SIGN > 0) w.y = -w.y;
      v[r] = cmul(v[r], w);
    }
  }
  dft<T, SIGN, R>(v);
  const int j0 = (b / ns) * ns * R + k;
#pragma unroll
  for (int r = 0; r < R; ++r) dst[lbase + (j0 + r * ns) * js] = v[r];
}

// The transform of lines whose length N and count NL per block are compile-time constants:
// every stage's radix, stride and twiddle offset is a constant of plan_of(N), so butterfly
// indices need no runtime division and LDS offsets become instruction immediates.  Returns the
// buffer holding the result.
template <typename T, int SIGN, int N, int NL, bool LINE_FASTEST, int S = 0>
__device__ inline cplx<T>* fft_lds_static(cplx<T>* a, cplx<T>* b, const cplx<T>* __restrict__ tw) {
  constexpr FftPlan P = plan_of(N, !LINE_FASTEST);
  if constexpr (S == P.nstages) {
    return a;
  } else {
    constexpr int R = P.radix[S], NS = P.ns[S], NB = N / R, TOTAL = NL * NB;
    constexpr int LS = LINE_FASTEST ? 1 : N, JS = LINE_FASTEST ? NL : 1;
    const cplx<T>* tws = tw + P.twoff[S];
#pragma unroll
    for (int w0 = 0; w0 < TOTAL; w0 += kBlock) {
      const int w = w0 + (int)threadIdx.x;
      if (TOTAL % kBlock == 0 || w < TOTAL) {
        const int l = LINE_FASTEST ? w % NL : w / NB;
        const int bi = LINE_FASTEST ? w / NL : w % NB;
        butterfly<T, SIGN, R>(a, b, l * LS, JS, bi, NB, NS, tws);
      }
    }
    __syncthreads();
    return fft_lds_static<T, SIGN, N, NL, LINE_FASTEST, S + 1>(b, a, tw);
  }
}

// The same stages in one LDS buffer: every thread first takes the inputs of all its butterflies
// of a stage into registers, and writes the outputs after the block's barrier.  Half the LDS of
// the two-buffer form for the same tile, at one more barrier per stage.
template <typename T, int SIGN, int N, int NL, bool LINE_FASTEST, int BLOCK = kBlock, int S = 0>
__device__ inline void fft_lds_static_inplace(cplx<T>* a, const cplx<T>* __restrict__ tw, int tid) {
  constexpr FftPlan P = plan_of(N, !LINE_FASTEST);
  if constexpr (S < P.nstages) {
    constexpr int R = P.radix[S], NS = P.ns[S], NB = N / R, TOTAL = NL * NB;
    constexpr int LS = LINE_FASTEST ? 1 : N, JS = LINE_FASTEST ? NL : 1;
    constexpr int IT = (TOTAL + BLOCK - 1) / BLOCK;
    const cplx<T>* tws = tw + P.twoff[S];
    cplx<T> v[IT][R];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int w = it * BLOCK + tid;
      if (TOTAL % BLOCK == 0 || w < TOTAL) {
        const int l = LINE_FASTEST ? w % NL : w / NB;
        const int bi = LINE_FASTEST ? w / NL : w % NB;
#pragma unroll
        for (int r = 0; r < R; ++r) v[it][r] = a[l * LS + (bi + r * NB) * JS];
        if (NS > 1) {
          const int k = bi % NS;
#pragma unroll
          for (int r = 1; r < R; ++r) {
            cplx<T> t = tws[k * (R - 1) + r - 1];
            if (SIGN > 0) t.y = -t.y;
            v[it][r] = cmul(v[it][r], t);
          }
        }
        dft<T, SIGN, R>(v[it]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int w = it * BLOCK + tid;
      if (TOTAL % BLOCK == 0 || w < TOTAL) {
        const int l = LINE_FASTEST ? w % NL : w / NB;
        const int bi = LINE_FASTEST ? w / NL : w % NB;
        const int j0 = (bi / NS) * NS * R + bi % NS;
#pragma unroll
        for (int r = 0; r < R; ++r) a[l * LS + (j0 + r * NS) * JS] = v[it][r];
      }
    }
    __syncthreads();
    fft_lds_static_inplace<T, SIGN, N, NL, LINE_FASTEST, BLOCK, S + 1>(a, tw, tid);
  }
}

// The centering stencil of LineCenter along the lines of an LDS tile (element (l, j) of NL lines
// of N points at l * LS + j * JS), in place: every thread forms the outputs of its elements from
// LDS into registers, then writes them after the block's barrier.  SHIFT is the stencil's (0
// before a forward transform, -1 after an inverse one).
template <typename T, int N, int NL, bool LINE_FASTEST, int SHIFT>
__device__ inline void center_tile(cplx<T>* a, const LineCenter<T>& lc) {
  constexpr int LS = LINE_FASTEST ? 1 : N, JS = LINE_FASTEST ? NL : 1;
  constexpr int TOTAL = N * NL, IT = (TOTAL + kBlock - 1) / kBlock;
  cplx<T> o[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int w = it * kBlock + (int)threadIdx.x;
    T sx = 0, sy = 0;
    if (TOTAL % kBlock == 0 || w < TOTAL) {
      const int l = LINE_FASTEST ? w % NL : w / N;
      const int j = LINE_FASTEST ? w / NL : w % N;
      const cplx<T>* line = a + l * LS;
      for (int n = 1; n <= lc.m; ++n) {
        int jp = j + n + SHIFT, jm = j - n + 1 + SHIFT;
        jp -= jp >= N ? N : 0;
        jm += jm < 0 ? N : 0;
        const cplx<T> u = line[jp * JS], v = line[jm * JS];
        sx = fma(lc.c[n - 1], u.x + v.x, sx);
        sy = fma(lc.c[n - 1], u.y + v.y, sy);
      }
    }
    o[it] = cmake(sx, sy);
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int w = it * kBlock + (int)threadIdx.x;
    if (TOTAL % kBlock == 0 || w < TOTAL) {
      const int l = LINE_FASTEST ? w % NL : w / N;
      const int j = LINE_FASTEST ? w / NL : w % N;
      a[l * LS + j * JS] = o[it];
    }
  }
  __syncthreads();
}

// LDS of one block's tile buffers and twiddles, elements per z-pass block (line pairs times the line
// length) and the largest strided tile.
#ifndef PIC_FFT_LDS_BUDGET
#define PIC_FFT_LDS_BUDGET 65536
#endif
constexpr size_t kLdsBudget = PIC_FFT_LDS_BUDGET;
#ifndef PIC_FFT_ZPASS_ELEMS
#define PIC_FFT_ZPASS_ELEMS 2048
#endif
#ifndef PIC_FFT_MAX_TL_SHIFT
#define PIC_FFT_MAX_TL_SHIFT 4
#endif

// The plan's twiddles, copied to LDS behind the two tile buffers.
template <typename T>
__device__ inline cplx<T>* stage_twiddles(cplx<T>* lds, const cplx<T>* __restrict__ tw, int count) {
  for (int e = threadIdx.x; e < count; e += blockDim.x) lds[e] = tw[e];
  return lds;
}

// Largest P (z pass) and TL (strided pass) that fit the LDS budget with the twiddles.
template <typename T>
constexpr int static_pairs(int n) {
  int P = PIC_FFT_ZPASS_ELEMS / n;
  if (P < 1) P = 1;
  while (P > 1 && (2 * (size_t)P * n + n) * sizeof(cplx<T>) > kLdsBudget) P /= 2;
  return P;
}
template <typename T>
constexpr int static_lines(int n) {  // one tile buffer: the strided stages run in place
  int sh = PIC_FFT_MAX_TL_SHIFT;
  while (sh > 0 && (((size_t)1 << sh) * n + n) * sizeof(cplx<T>) > kLdsBudget) --sh;
  return 1 << sh;
}

template <typename T, int N>
__global__ void __launch_bounds__(kBlock) k_r2c_z_n(Batch<const T*> in, Batch<cplx<T>*> out,
                                                    const cplx<T>* __restrict__ tw, int nlines, int pz,
                                                    LineCenter<T> lc, unsigned cmask) {
  constexpr int P = static_pairs<T>(N);
  constexpr int TW = N - 1;  // twiddles of a plan: sum of ns (R - 1) over the stages
  constexpr int PER = (P * N + kBlock - 1) / kBlock;
  constexpr int NH = N / 2 + 1;
  extern __shared__ __align__(16) unsigned char smem[];
  cplx<T>* a = reinterpret_cast<cplx<T>*>(smem);
  cplx<T>* b = a + (size_t)P * N;
  const int pair0 = blockIdx.x * P;
  const int np = min(P, nlines / 2 - pair0);
  const unsigned total = (unsigned)(np * N);
  const T* __restrict__ src = in.p[blockIdx.y] + (size_t)2 * pair0 * N;  // line 2 pair0 of this block
  cplx<T>* __restrict__ dst = out.p[blockIdx.y] + (size_t)2 * pair0 * pz;
  T v0[PER], v1[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const unsigned e = threadIdx.x + u * kBlock;
    if (e < total) {
      const unsigned q = e / N, j = e - q * N;
      v0[u] = src[2 * q * N + j];
      v1[u] = src[(2 * q + 1) * N + j];
    }
  }
  const cplx<T>* twl = stage_twiddles(b + (size_t)P * N, tw, TW);
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const unsigned e = threadIdx.x + u * kBlock;
    if (e < total) a[e] = cmake(v0[u], v1[u]);
  }
  __syncthreads();
  if ((cmask >> blockIdx.y) & 1u) center_tile<T, N, P, false, 0>(a, lc);
  cplx<T>* res = fft_lds_static<T, -1, N, P, false>(a, b, twl);
  constexpr int OUTER = (P * NH + kBlock - 1) / kBlock;
#pragma unroll
  for (int u = 0; u < OUTER; ++u) {
    const unsigned e = threadIdx.x + u * kBlock;
    if (e < (unsigned)(np * NH)) {
      const unsigned q = e / NH, k = e - q * NH;
      const cplx<T> zk = res[q * N + k];
      const cplx<T> zn = res[q * N + (k == 0 ? 0 : N - k)];
      const cplx<T> F = cmake((T)0.5 * (zk.x + zn.x), (T)0.5 * (zk.y - zn.y));
      const cplx<T> G = cmake((T)0.5 * (zk.y + zn.y), (T)0.5 * (zn.x - zk.x));
      dst[2 * q * pz + k] = F;
      dst[(2 * q + 1) * pz + k] = G;
    }
  }
}

template <typename T, int N>
__global__ void __launch_bounds__(kBlock) k_c2r_z_n(Batch<const cplx<T>*> in, Batch<T*> out,
                                                    const cplx<T>* __restrict__ tw, int nlines, int pz, T scale,
                                                    T scale_lo, LineCenter<T> lc, unsigned cmask) {
  constexpr int P = static_pairs<T>(N);
  constexpr int TW = N - 1;  // twiddles of a plan: sum of ns (R - 1) over the stages
  constexpr int PER = (P * N + kBlock - 1) / kBlock;
  constexpr int HALF = N / 2;
  extern __shared__ __align__(16) unsigned char smem[];
  cplx<T>* a = reinterpret_cast<cplx<T>*>(smem);
  cplx<T>* b = a + (size_t)P * N;
  const int pair0 = blockIdx.x * P;
  const int np = min(P, nlines / 2 - pair0);
  const unsigned total = (unsigned)(np * N);
  const cplx<T>* __restrict__ src = in.p[blockIdx.y] + (size_t)2 * pair0 * pz;
  T* __restrict__ dst = out.p[blockIdx.y] + (size_t)2 * pair0 * N;
  cplx<T> f[PER], g[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const unsigned e = threadIdx.x + u * kBlock;
    if (e < total) {
      const unsigned q = e / N, k = e - q * N;
      const unsigned kk = k <= HALF ? k : N - k;
      f[u] = src[2 * q * pz + kk];
      g[u] = src[(2 * q + 1) * pz + kk];
    }
  }
  const cplx<T>* twl = stage_twiddles(b + (size_t)P * N, tw, TW);
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const unsigned e = threadIdx.x + u * kBlock;
    if (e < total) {
      const unsigned k = e % N;
      cplx<T> F = f[u], G = g[u];
      if (k > HALF) {
        F = cconj(F);
        G = cconj(G);
      } else if (k == 0 || k == HALF) {
        F.y = 0;
        G.y = 0;
      }
      a[e] = cmake(F.x - G.y, F.y + G.x);
    }
  }
  __syncthreads();
  cplx<T>* res = fft_lds_static<T, +1, N, P, false>(a, b, twl);
  if ((cmask >> blockIdx.y) & 1u) center_tile<T, N, P, false, -1>(res, lc);
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const unsigned e = threadIdx.x + u * kBlock;
    if (e < total) {
      const unsigned q = e / N, j = e - q * N;
      const cplx<T> v = res[e];
      dst[2 * q * N + j] = mul_const(v.x, scale, scale_lo);
      dst[(2 * q + 1) * N + j] = mul_const(v.y, scale, scale_lo);
    }
  }
}

// Strided pass with N and TL constant.  Thread t holds line i = t mod TL of the tile (kBlock
// is a multiple of TL) at elements j = t / TL + u kBlock / TL, so its global address advances
// by a constant number of rows per u.
template <typename T, int SIGN, int N>
__global__ void __launch_bounds__(kBlock) k_fft_strided_n(Batch<const cplx<T>*> in, Batch<cplx<T>*> out,
                                                          const cplx<T>* __restrict__ tw, int inner_count,
                                                          int tiles_per_outer, long long outer_stride,
                                                          long long elem_stride, LineCenter<T> lc, unsigned cmask) {
  constexpr int TL = static_lines<T>(N);
  static_assert(kBlock % TL == 0, "a block covers whole rows of the tile");
  constexpr int TW = N - 1;  // twiddles of a plan: sum of ns (R - 1) over the stages
  constexpr int TOTAL = N * TL;
  constexpr int PER = (TOTAL + kBlock - 1) / kBlock;
  constexpr int ROWS = kBlock / TL;  // rows advanced per u
  extern __shared__ __align__(16) unsigned char smem[];
  cplx<T>* a = reinterpret_cast<cplx<T>*>(smem);
  // tiles next to each other read and write the two halves of the same memory lines: one XCD
  const int tile = xcd_major(blockIdx.x, gridDim.x);
  const int outer = tile / tiles_per_outer;
  const int inner0 = (tile - outer * tiles_per_outer) * TL;
  const int nl = min(TL, inner_count - inner0);
  const int i = (int)threadIdx.x % TL, j0 = (int)threadIdx.x / TL;
  const long long row0 = (long long)outer * outer_stride + inner0 + min(i, nl - 1) + (long long)j0 * elem_stride;
  const long long step = (long long)ROWS * elem_stride;
  const cplx<T>* __restrict__ src = in.p[blockIdx.y] + row0;
  cplx<T> v[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (TOTAL % kBlock == 0 || (int)threadIdx.x + u * kBlock < TOTAL) v[u] = src[u * step];
  const cplx<T>* twl = stage_twiddles(a + (size_t)TL * N, tw, TW);
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int e = (int)threadIdx.x + u * kBlock;
    if (TOTAL % kBlock == 0 || e < TOTAL) a[e] = i < nl ? v[u] : cmake((T)0, (T)0);
  }
  __syncthreads();
  const bool cen = (cmask >> blockIdx.y) & 1u;
  if (SIGN < 0 && cen) center_tile<T, N, TL, true, 0>(a, lc);  // forward: centre, then transform
  fft_lds_static_inplace<T, SIGN, N, TL, true>(a, twl, threadIdx.x);
  if (SIGN > 0 && cen) center_tile<T, N, TL, true, -1>(a, lc);  // inverse: transform, then centre
  if (i < nl) {
    cplx<T>* __restrict__ dst = out.p[blockIdx.y] + row0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = (int)threadIdx.x + u * kBlock;
      if (TOTAL % kBlock == 0 || e < TOTAL) dst[u * step] = a[e];
    }
  }
}

// ------------------------------------------------- x pass, update and inverse x pass in one kernel

// Lines and workgroup of the fused pass at length N (lines = 0: not built).  A thread holds six complex
// values (the updated E, B) for each of its elements, so a workgroup grows with the line: at most 6
// elements per thread in FP32, 3 in FP64 (2 in workgroups of 1024, which have 128 registers per thread).
// Tiles of 16 or 8 lines are 128- or 64-byte rows (FP64: 128 and 64 bytes at 8 and 4 lines).
template <typename T>
struct SolveShape {
  int lines, block;
};

// KiB per array from which the fused pass is the faster one along x lines of n points (0: on no grid, so it
// is not built).  psatd_push_fields timed with it and with the separate kernels at 3 to 100 MiB per array,
// all lengths (fused / separate): mostly 0.85 to 0.95 from 3 MiB on, 0.75 to 0.8 from 50.  Below, its chain
// of 17 transforms in one workgroup takes longer than three launches (FP32 32^3 31.6 against 27.8 us, FP64
// 33.5 against 31.7); lengths with few workgroups per array need some more (FP32, 3 MiB: 108 points 1.02 to
// 1.04, 192 1.10, 512 1.04, 768 1.11).  With more registers than the workgroup has (FP32 162 1.05 at 5 MiB
// and 0.95 at 6; 486 1.06 at 17 and 0.93 at 34; 648 1.06 at 16 and 0.99 at 100; FP64 144 1.10 at 23 and 0.95
// at 30; 486 1.01 at 173) or one workgroup per CU (FP64 108 1.14 at 10 MiB, 1.02 at 29, 0.94 at 51; 162 and
// 324 1.05 at 16, 0.93 at 29) only large grids gain, or none.  FP64 lines of 8 and 12 points occupy 64 and
// 96 of a workgroup's 256 threads: 1.14 and 1.08 at 16 MiB.
template <typename T>
constexpr int solve_from_kib(int n) {
  switch (sizeof(T) == 4 ? n : -n) {
    case 108: case 144: case -72: case -512: return 3584;
    case 192: case 512: case 768: return 4096;
    case 162: return 6 << 10;
    case -162: case -324: return 24 << 10;
    case -144: return 28 << 10;
    case 486: return 32 << 10;
    case -108: return 48 << 10;
    case 648: case -8: case -12: case -486: return 0;
    default: return 3 << 10;
  }
}
template <typename T>
constexpr SolveShape<T> solve_shape(int n) {
  const int per = sizeof(T) == 4 ? 6 : 3, wide = sizeof(T) == 4 ? 16 : 8;
  if (solve_from_kib<T>(n) == 0) return {0, 0};
  if (n * wide <= 256 * per) return {wide, 256};
  if (n * wide <= 512 * per) return {wide, 512};
  if (n * wide / 2 <= 512 * per) return {wide / 2, 512};
  if (n * wide / 2 <= 1024 * (sizeof(T) == 4 ? 6 : 2)) return {wide / 2, 1024};
  return {0, 0};
}

// The standard update of psatd.hip between the transforms along x, for psatd_push_fields.  A workgroup
// takes TL adjacent (ky, kz) columns for every x, transforms the eleven inputs along x one after the other
// in the same LDS tile, adds each one's part of the update to the six updated fields, which stay in
// registers, and transforms those back.  As three kernels (x pass, update, inverse x pass) they move 54
// spectra between HBM and the chip, here 18 (the tables are even in kx, so lines read them for
// kx <= N / 2 only).  The whole solve at 256^3: FP32 1890 -> 1485 us, FP64 3563 -> 2650.  Every sum is
// formed in the order of k_psatd_update, so the results are as accurate: terms that wait for a later
// source are kept in LDS (in registers they spilled, 96 x 96 x 192 FP64 267 -> 319 us).  Bound by its chain
// of 17 transforms (2 barriers per stage) at two workgroups per CU.  The same fusion of pic_step's resident
// state (40 arrays against 25) was no faster than the separate kernels (384 x 384 x 768 FP32 4.1 ms either
// way, 128 x 128 x 256 142 against 128 us).
template <typename T, int N>
__global__ void __launch_bounds__(solve_shape<T>(N).block, sizeof(T) == 4 ? 4 : 3) k_solve_x(SolveX<T> a, const cplx<T>* __restrict__ tw) {
  constexpr int TL = solve_shape<T>(N).lines, BLOCK = solve_shape<T>(N).block;
  constexpr int TOTAL = N * TL, PER = (TOTAL + BLOCK - 1) / BLOCK, ROWS = BLOCK / TL;
  extern __shared__ __align__(16) unsigned char smem[];
  cplx<T>* tile = reinterpret_cast<cplx<T>*>(smem);
  cplx<T>* kept = tile + TOTAL;  // two values per element, read by the thread that wrote them
  cplx<T>* twl = kept + 2 * TOTAL;
  for (int e = threadIdx.x; e < N - 1; e += BLOCK) twl[e] = tw[e];
  const int col0 = xcd_major(blockIdx.x, gridDim.x) * TL;
  const int i = (int)threadIdx.x % TL, j0 = (int)threadIdx.x / TL;
  const int col = col0 + i, ky = col / a.pz, kz = col - ky * a.pz;
  const bool mode = kz < a.nzh;  // not a padding column
  // element u of this thread: a uniform row offset plus a 32-bit byte offset of the thread's own
  const size_t step = (size_t)ROWS * a.ny * a.pz;
  const unsigned off = (unsigned)(j0 * a.ny * a.pz + col) * (unsigned)sizeof(cplx<T>);
  auto at = [&](auto* p, int u) -> decltype(*p) {
    using C = std::conditional_t<std::is_const_v<std::remove_pointer_t<decltype(p)>>, const char, char>;
    return *reinterpret_cast<decltype(p)>(reinterpret_cast<C*>(p + u * step) + off);
  };
  auto has = [&](int u) { return TOTAL % BLOCK == 0 || (int)threadIdx.x + u * BLOCK < TOTAL; };
  auto load = [&](const cplx<T>* src, cplx<T>* v) {
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u] = has(u) ? at(src, u) : cmake((T)0, (T)0);
  };
  // a fresh copy of the thread index: indices derived from it are recomputed by each transform instead of
  // being kept in registers from the first to the last
  auto tid = [&]() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
  };
  auto put = [&](const cplx<T>* v) {
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (has(u)) tile[threadIdx.x + u * BLOCK] = v[u];
    __syncthreads();
  };
  auto own = [&](int u) { return has(u) ? tile[threadIdx.x + u * BLOCK] : cmake((T)0, (T)0); };
  // per element: its row of the tables (kx and N - kx share it) and the operators along x
  auto table = [&](const T* t, int u) {
    const int j = tid() / TL + u * ROWS, jm = 2 * j > N ? N - j : j;
    const unsigned o = (unsigned)((jm * a.ny + ky) * a.nzh + kz) * (unsigned)sizeof(T);
    return mode && has(u) ? *reinterpret_cast<const T*>(reinterpret_cast<const char*>(t) + o) : (T)0;
  };
  auto dx = [&](const cplx<T>* d, int u) { return d[min(tid() / TL + u * ROWS, N - 1)]; };
  const int kzc = mode ? kz : 0;
  const cplx<T> py = a.Dp[1][ky], my = a.Dm[1][ky], pz = a.Dp[2][kzc], mz = a.Dm[2][kzc];

  cplx<T> F[6][PER];  // E, B, then their update
  // forms the six values of element u here: left alone, the compiler moves the additions towards their
  // last use and keeps every source's terms in registers until then (190 instead of 110 at 128 points)
  auto settle = [&](int u) {
#pragma unroll
    for (int c = 0; c < 6; ++c) asm volatile("" : "+v"(F[c][u].x), "+v"(F[c][u].y)::"memory");
  };
  cplx<T> v[PER];
  load(a.src[0], v);
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    put(v);
    load(a.src[c + 1], v);
    fft_lds_static_inplace<T, -1, N, TL, true, BLOCK>(tile, twl, tid());
#pragma unroll
    for (int u = 0; u < PER; ++u) F[c][u] = own(u);
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {  // the fields' own part: C E + Sw D- x B, C B - Sw D+ x E
    const T C = table(a.C, u), Sw = table(a.Sw, u);
    const cplx<T> px = dx(a.Dp[0], u), mx = dx(a.Dm[0], u);
    const cplx<T> ex = F[0][u], ey = F[1][u], ez = F[2][u], bx = F[3][u], by = F[4][u], bz = F[5][u];
    F[0][u] = cadd(cscale(ex, C), cscale(csub(cmul(my, bz), cmul(mz, by)), Sw));
    F[1][u] = cadd(cscale(ey, C), cscale(csub(cmul(mz, bx), cmul(mx, bz)), Sw));
    F[2][u] = cadd(cscale(ez, C), cscale(csub(cmul(mx, by), cmul(my, bx)), Sw));
    F[3][u] = csub(cscale(bx, C), cscale(csub(cmul(py, ez), cmul(pz, ey)), Sw));
    F[4][u] = csub(cscale(by, C), cscale(csub(cmul(pz, ex), cmul(px, ez)), Sw));
    F[5][u] = csub(cscale(bz, C), cscale(csub(cmul(px, ey), cmul(py, ex)), Sw));
    settle(u);
  }
  // J^d: -Sw J to E^d and X1 (D+ x J) to B, each component of the curl formed before it is added, as
  // k_psatd_update does: the earlier of its two terms waits in the thread's own places of LDS
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    put(v);
    load(a.src[7 + d], v);
    fft_lds_static_inplace<T, -1, N, TL, true, BLOCK>(tile, twl, tid());
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (!has(u)) continue;
      cplx<T>* const k0 = kept + tid() + u * BLOCK;
      cplx<T>* const k1 = k0 + TOTAL;
      const T X1 = table(a.X1, u);
      const cplx<T> j = own(u), px = dx(a.Dp[0], u);
      F[d][u] = csub(F[d][u], cscale(j, table(a.Sw, u)));
      if (d == 0) {
        *k0 = cmul(pz, j);
        *k1 = cmul(py, j);
      } else if (d == 1) {
        F[5][u] = cadd(F[5][u], cscale(csub(cmul(px, j), *k1), X1));
        *k1 = cmul(pz, j);
      } else {
        F[3][u] = cadd(F[3][u], cscale(csub(cmul(py, j), *k1), X1));
        F[4][u] = cadd(F[4][u], cscale(csub(*k0, cmul(px, j)), X1));
      }
      settle(u);
    }
  }
  // (X3 rho^n - X2 rho^{n+1}) D+ to E, the difference first
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    put(v);
    if (r == 0) load(a.src[10], v);  // rho^n
    fft_lds_static_inplace<T, -1, N, TL, true, BLOCK>(tile, twl, tid());
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (!has(u)) continue;
      cplx<T>* const k0 = kept + tid() + u * BLOCK;
      if (r == 0) {
        *k0 = cscale(own(u), table(a.X2, u));
      } else {
        const cplx<T> rr = csub(cscale(own(u), table(a.X3, u)), *k0);
        F[0][u] = cadd(F[0][u], cmul(rr, dx(a.Dp[0], u)));
        F[1][u] = cadd(F[1][u], cmul(rr, py));
        F[2][u] = cadd(F[2][u], cmul(rr, pz));
        settle(u);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    put(F[c]);
    fft_lds_static_inplace<T, +1, N, TL, true, BLOCK>(tile, twl, tid());
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (has(u)) at(a.out[c], u) = own(u);
  }
}

// ---------------------------------------------------------------- launchers of one length

template <typename T>
constexpr size_t fft_lds_bytes(size_t elems, int n) {  // tile buffers and twiddles
  return (elems + (size_t)(n - 1)) * sizeof(cplx<T>);
}

template <typename T, int N>
struct FftLength {
  static void r2c(const Batch<const T*>& in, const Batch<cplx<T>*>& out, int count, const cplx<T>* tw, int nlines,
                  int pz, const LineCenter<T>& lc, hipStream_t s) {
    constexpr int P = static_pairs<T>(N);
    constexpr size_t lds = fft_lds_bytes<T>(2 * (size_t)P * N, N);
    allow_lds((const void*)k_r2c_z_n<T, N>, lds);
    hipLaunchKernelGGL((k_r2c_z_n<T, N>), dim3((nlines / 2 + P - 1) / P, count), dim3(kBlock), lds, s, in, out, tw,
                       nlines, pz, lc, lc.m > 0 ? lc.mask[2] : 0u);
  }
  static void c2r(const Batch<const cplx<T>*>& in, const Batch<T*>& out, int count, const cplx<T>* tw, int nlines,
                  int pz, T scale, T scale_lo, const LineCenter<T>& lc, hipStream_t s) {
    constexpr int P = static_pairs<T>(N);
    constexpr size_t lds = fft_lds_bytes<T>(2 * (size_t)P * N, N);
    allow_lds((const void*)k_c2r_z_n<T, N>, lds);
    hipLaunchKernelGGL((k_c2r_z_n<T, N>), dim3((nlines / 2 + P - 1) / P, count), dim3(kBlock), lds, s, in, out, tw,
                       nlines, pz, scale, scale_lo, lc, lc.m > 0 ? lc.mask[2] : 0u);
  }
  template <int SIGN>
  static void strided(const Batch<const cplx<T>*>& in, const Batch<cplx<T>*>& out, int count, const cplx<T>* tw,
                      int outer_count, int inner_count, long long outer_stride, long long elem_stride,
                      const LineCenter<T>& lc, int axis, hipStream_t s) {
    constexpr int TL = static_lines<T>(N);
    constexpr size_t lds = fft_lds_bytes<T>((size_t)TL * N, N);
    const int tpo = (inner_count + TL - 1) / TL;
    allow_lds((const void*)k_fft_strided_n<T, SIGN, N>, lds);
    hipLaunchKernelGGL((k_fft_strided_n<T, SIGN, N>), dim3(outer_count * tpo, count), dim3(kBlock), lds, s, in, out,
                       tw, inner_count, tpo, outer_stride, elem_stride, lc, lc.m > 0 ? lc.mask[axis] : 0u);
  }
  static void solve_x(const SolveX<T>& a, const cplx<T>* tw, hipStream_t s) {
    constexpr SolveShape<T> S = solve_shape<T>(N);
    if constexpr (S.lines > 0) {
      constexpr size_t lds = fft_lds_bytes<T>(3 * (size_t)S.lines * N, N);
      static_assert(lds <= 160 * 1024, "fits the LDS");
      allow_lds((const void*)k_solve_x<T, N>, lds);
      hipLaunchKernelGGL((k_solve_x<T, N>), dim3((unsigned)(a.ny * a.pz / S.lines)), dim3(S.block), lds, s, a, tw);
    }
  }
  static constexpr FftOps<T> ops = {&r2c, &c2r, {&strided<-1>, &strided<+1>},
                                    solve_shape<T>(N).lines > 0 ? &solve_x : nullptr,
                                    (size_t)solve_from_kib<T>(N) << 10};
};

}  // namespace

}  // namespace pic
