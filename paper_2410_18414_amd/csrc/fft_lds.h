// Complex helpers, the LDS Stockham FFT and the spectral derivative symbols,
// shared by the field solve (field.hip) and its adjoint (adjoint.hip).
#pragma once

#include "pic_internal.h"

namespace pic {
namespace {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double2 mul_i(double2 a) { return make_double2(-a.y, a.x); }      // i a
__device__ __forceinline__ double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }     // -i a
__device__ __forceinline__ double2 cdivr(double2 a, double r) { return make_double2(a.x / r, a.y / r); }

// The R-point DFT of v in registers (INV: the conjugate one).
template <int R, bool INV>
__device__ __forceinline__ void dft(double2 (&v)[R]) {
  auto rot = [](double2 z) { return INV ? mul_i(z) : mul_mi(z); };  // times e^{-+ i pi/2}
  if constexpr (R == 2) {
    const double2 t = v[0];
    v[0] = cadd(t, v[1]);
    v[1] = csub(t, v[1]);
  } else if constexpr (R == 4) {
    const double2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
    const double2 s13 = cadd(v[1], v[3]), d13 = rot(csub(v[1], v[3]));
    v[0] = cadd(s02, s13);
    v[1] = cadd(d02, d13);
    v[2] = csub(s02, s13);
    v[3] = csub(d02, d13);
  } else {
    // odd R: outputs q and R - q from the sums and differences of the inputs
    // m and R - m, with cos and sin of 2 pi m / R
    constexpr int H = (R - 1) / 2;
    constexpr double c3[] = {-0.5}, s3[] = {0.86602540378443864676};
    constexpr double c5[] = {0.30901699437494742410, -0.80901699437494742410},
                     s5[] = {0.95105651629515357212, 0.58778525229247312917};
    double2 s[H], d[H], v0 = v[0];
#pragma unroll
    for (int m = 0; m < H; ++m) {
      s[m] = cadd(v[m + 1], v[R - 1 - m]);
      d[m] = rot(csub(v[m + 1], v[R - 1 - m]));
      v[0] = cadd(v[0], s[m]);
    }
#pragma unroll
    for (int q = 1; q <= H; ++q) {
      double2 a = v0, b = make_double2(0.0, 0.0);
#pragma unroll
      for (int m = 1; m <= H; ++m) {
        const int e = (q * m) % R, f = e <= H ? e : R - e;
        const double c = R == 3 ? c3[f - 1] : c5[f - 1];
        const double w = (R == 3 ? s3[f - 1] : s5[f - 1]) * (e <= H ? 1.0 : -1.0);
        a = cadd(a, cscale(s[m - 1], c));
        b = cadd(b, cscale(d[m - 1], w));
      }
      v[q] = cadd(a, b);
      v[R - q] = csub(a, b);
    }
  }
}

// Radix-4 passes, then a radix-2 one for an odd lN, over B transforms of length
// 2^lN with at most one butterfly per thread.  lN is a constant where this is
// called: a pass is then some thirty instructions besides its butterfly's
// arithmetic and its two LDS round trips.  N = 128, two transforms: 1.04 us;
// 1.24 us with run-time strides, 1.84 us with run-time divisions.  Radix 8 takes
// fewer passes but gives the few busy waves three times the instructions: 1.7 us.
// Transforms are pitch apart (0: 2^lN).
template <bool INV>
__device__ __forceinline__ double2* fft_pow2(double2* a, double2* b, const int lN, int B,
                                             const double2* __restrict__ tw, int pitch) {
  const int lq = lN - 2, q = 1 << lq, t = threadIdx.x;
  const bool act = t < B << lq;
  const int j = t & (q - 1), fo = pitch ? (t >> lq) * pitch : (t >> lq) << lN;
#pragma unroll
  for (int ls = 0; ls + 2 <= lN; ls += 2) {
    if (act) {
      const double2* x = a + fo + j;
      double2 v[4] = {x[0], x[q], x[2 * q], x[3 * q]};
      const int k = j & ((1 << ls) - 1);
      if (ls) {
        const int e = k << (lq - ls);
        const double2 w1 = tw[e], w2 = tw[2 * e], w3 = tw[3 * e];
        v[1] = cmul(v[1], INV ? cconj(w1) : w1);
        v[2] = cmul(v[2], INV ? cconj(w2) : w2);
        v[3] = cmul(v[3], INV ? cconj(w3) : w3);
      }
      dft<4, INV>(v);
      double2* y = b + fo + ((j - k) << 2) + k;
#pragma unroll
      for (int m = 0; m < 4; ++m) y[m << ls] = v[m];
    }
    __syncthreads();
    double2* s = a;
    a = b;
    b = s;
  }
  if (lN & 1) {  // two butterflies per thread
    const int h = 2 * q;
    if (act) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const double2 w = tw[j + u * q];
        const double2 v0 = a[fo + j + u * q], v1 = cmul(a[fo + j + u * q + h], INV ? cconj(w) : w);
        b[fo + j + u * q] = cadd(v0, v1);
        b[fo + j + u * q + h] = csub(v0, v1);
      }
    }
    __syncthreads();
    double2* s = a;
    a = b;
    b = s;
  }
  return a;
}

// One Stockham pass over B transforms of any length N: radix r after ns points
// have been combined.  Every value is wave-uniform.
struct FftPass {
  int N, r, ns, q, stride;  // q = N / r butterflies, twiddle stride N / (r ns)
  int pitch;                // from one transform to the next
  float inv_q, inv_ns;      // 1 / q, 1 / ns
};

template <int R, bool INV>
__device__ __forceinline__ void fft_pass(const double2* a, double2* b, const FftPass& s, int B,
                                         const double2* __restrict__ tw) {
  const int P = s.pitch, q = s.q, Ns = s.ns;
  for (int t = threadIdx.x; t < B * q; t += blockDim.x) {
    const int f = fdiv(t, s.inv_q), j = t - f * q;
    const int g = fdiv(j, s.inv_ns), k = j - g * Ns;
    const double2* x = a + f * P + j;
    double2 v[R], w[R];
#pragma unroll
    for (int m = 0; m < R; ++m) v[m] = x[m * q];
    if (Ns > 1) {
      const int e = k * s.stride;
#pragma unroll
      for (int m = 1; m < R; ++m) w[m] = tw[m * e];
#pragma unroll
      for (int m = 1; m < R; ++m) v[m] = cmul(v[m], INV ? cconj(w[m]) : w[m]);
    }
    dft<R, INV>(v);
    double2* y = b + f * P + g * Ns * R + k;
#pragma unroll
    for (int m = 0; m < R; ++m) y[m * Ns] = v[m];
  }
}

// A pass of any odd radix r: first, in place, the twiddled inputs m and r - m of
// each butterfly become their sum and difference; then the outputs o and r - o
// share the products of those with cos and sin, a quarter of the
// multiplications and a third of the LDS reads of r-term complex sums.
template <bool INV>
__device__ __forceinline__ void fft_pass_odd(double2* a, double2* b, const FftPass& s, int B,
                                             const double2* __restrict__ tw) {
  const int P = s.pitch, q = s.q, Ns = s.ns, r = s.r, h = (r - 1) >> 1;
  const float inv_h = __builtin_amdgcn_rcpf((float)h);
  for (int t = threadIdx.x; t < B * q * h; t += blockDim.x) {
    const int u = fdiv(t, inv_h);  // f * q + j
    const int m = t - u * h + 1;
    const int f = fdiv(u, s.inv_q), j = u - f * q;
    const int k = j - fdiv(j, s.inv_ns) * Ns;
    double2* x = a + f * P + j;
    double2 v0 = x[m * q], v1 = x[(r - m) * q];
    if (Ns > 1) {
      const double2 w0 = tw[m * k * s.stride], w1 = tw[(r - m) * k * s.stride];
      v0 = cmul(v0, INV ? cconj(w0) : w0);
      v1 = cmul(v1, INV ? cconj(w1) : w1);
    }
    x[m * q] = cadd(v0, v1);
    const double2 d = csub(v0, v1);
    x[(r - m) * q] = INV ? mul_i(d) : mul_mi(d);
  }
  __syncthreads();
  // two output pairs o, r - o per thread: they share the reads of the sums and
  // differences (the pass is bound by LDS reads)
  const int ho = (h + 2) >> 1;  // threads per butterfly, outputs o and o + ho
  const float inv_ho = __builtin_amdgcn_rcpf((float)ho);
  for (int t = threadIdx.x; t < B * q * ho; t += blockDim.x) {
    const int u = fdiv(t, inv_ho);
    const int o = t - u * ho;
    const int f = fdiv(u, s.inv_q), j = u - f * q;
    const int g = fdiv(j, s.inv_ns), k = j - g * Ns;
    const double2* x = a + f * P + j;
    double2 ye[2], yo[2];
    ye[0] = ye[1] = x[0];
    yo[0] = yo[1] = make_double2(0.0, 0.0);
    const int er = r * q;  // tw[e q] = exp(-2 pi i e / r)
    const int eo[2] = {o * q, (o + ho) * q};
    int e[2] = {0, 0}, im = 0, ir = er;
#pragma unroll 2
    for (int m = 1; m <= h; ++m) {
      im += q;
      ir -= q;
      const double2 sm = x[im], df = x[ir];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        e[c] += eo[c];
        e[c] = e[c] >= er ? e[c] - er : e[c];
        const double2 w = tw[e[c]];  // cos, -sin
        ye[c].x = __builtin_fma(sm.x, w.x, ye[c].x);
        ye[c].y = __builtin_fma(sm.y, w.x, ye[c].y);
        yo[c].x = __builtin_fma(df.x, -w.y, yo[c].x);
        yo[c].y = __builtin_fma(df.y, -w.y, yo[c].y);
      }
    }
    double2* y = b + f * P + g * Ns * r + k;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int oc = o + c * ho;
      if (oc > h) break;
      y[oc * Ns] = cadd(ye[c], yo[c]);
      if (oc) y[(r - oc) * Ns] = csub(ye[c], yo[c]);
    }
  }
}

// B independent FFTs of the plan's length held in LDS at a[f*N + j] (f*pitch + j
// if a pitch is given; Stockham autosort: fft_pow2 for a power of two with one
// butterfly per thread, else the passes of the plan's radices).  Ping-pongs
// between a and b and returns the buffer holding the result.
// tw[t] = exp(-2 pi i t / N), t < N.  INV: exp(+...) (unnormalised inverse).
// MAXLN: log2 of the longest power of two that the caller transforms.  All
// threads of the block must call it; the caller synchronises before.
template <bool INV, int MAXLN = 10>
__device__ __forceinline__ double2* fft_lds(double2* a, double2* b, const FftPlan& p, int B,
                                            const double2* __restrict__ tw, int pitch = 0) {
  const int N = p.n;
  if (B * N <= 4 * (int)blockDim.x) {
    switch (N) {
      case 8: return fft_pow2<INV>(a, b, 3, B, tw, pitch);
      case 16: return fft_pow2<INV>(a, b, 4, B, tw, pitch);
      case 32: return fft_pow2<INV>(a, b, 5, B, tw, pitch);
      case 64: return fft_pow2<INV>(a, b, 6, B, tw, pitch);
      case 128: return fft_pow2<INV>(a, b, 7, B, tw, pitch);
    }
    if constexpr (MAXLN > 7) {
      switch (N) {
        case 256: return fft_pow2<INV>(a, b, 8, B, tw, pitch);
        case 512: return fft_pow2<INV>(a, b, 9, B, tw, pitch);
        case 1024: return fft_pow2<INV>(a, b, 10, B, tw, pitch);
      }
    }
  }
  FftPass s;
  s.N = N;
  s.pitch = pitch ? pitch : N;
  s.ns = 1;
  uint64_t radices = p.radices[0], more = p.radices[1];
  while (s.ns < N) {
    s.r = (int)(radices & 0xffff);
    // exact quotients of wave-uniform numbers: N / r, and what remains after it
    s.q = udiv_exact(N, s.r);
    s.stride = udiv_exact(s.q, s.ns);
    s.inv_q = __builtin_amdgcn_rcpf((float)s.q);
    s.inv_ns = __builtin_amdgcn_rcpf((float)s.ns);
    switch (s.r) {
      case 4: fft_pass<4, INV>(a, b, s, B, tw); break;
      case 2: fft_pass<2, INV>(a, b, s, B, tw); break;
      case 3: fft_pass<3, INV>(a, b, s, B, tw); break;
      case 5: fft_pass<5, INV>(a, b, s, B, tw); break;
      default: fft_pass_odd<INV>(a, b, s, B, tw); break;
    }
    __syncthreads();
    double2* t = a;
    a = b;
    b = t;
    s.ns *= s.r;
    radices = radices >> 16 | more << 48;
    more >>= 16;
  }
  return a;
}

__device__ __forceinline__ double kx_sym(int kx, const GridP& g) {
  return (2 * kx == g.nx) ? 0.0 : 2.0 * M_PI * kx / g.lx;
}
__device__ __forceinline__ double ky_sym(int ky, const GridP& g) {
  if (2 * ky == g.ny) return 0.0;
  const int m = (2 * ky < g.ny) ? ky : ky - g.ny;
  return 2.0 * M_PI * m / g.ly;
}

}  // namespace
}  // namespace pic
