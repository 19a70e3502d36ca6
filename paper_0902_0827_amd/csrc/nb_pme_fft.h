// Complex FFTs in LDS for the reciprocal part: many lines of one length at once, in place,
// FP64.
//
// A length n = r_1 r_2 ... r_p (radices 8, 4, 2, 3, 5, 7) is transformed by p passes.  The
// forward pass of radix r over sub-length s (first s = n) replaces, in every block of s
// entries, the r entries m = s / r apart by their discrete Fourier transform times the
// twiddles exp(-2 pi i j p / s), and continues with sub-length m: decimation in frequency.
// Every butterfly writes the entries it read, so a pass needs no second buffer and one
// barrier, and the frequencies come out in digit-reversed order.  The inverse runs the
// mirrored passes from that order (conjugate twiddles before the butterfly), so nothing is
// ever reordered: between the two only the frequency of each position is needed
// (FftShape::freq).
#pragma once

#include <hip/hip_runtime.h>

namespace nb {

namespace {

constexpr int kFftMaxPasses = 10;

// Length and radices of one dimension (made on the host, passed by value).
struct FftShape {
  int n = 0, passes = 0;
  int radix[kFftMaxPasses] = {};

  // Frequency at position p after the forward transform.
  __device__ int freq(int p) const {
    int f = 0, w = 1, s = n;
    for (int k = 0; k < passes; ++k) {
      s /= radix[k];
      const int q = p / s;
      f += q * w;
      p -= q * s;
      w *= radix[k];
    }
    return f;
  }
};

// Radices of length n, false when it has a prime factor above 7.
inline bool fft_shape(int n, FftShape *out) {
  FftShape s;
  s.n = n;
  int rest = n, twos = 0;
  while (rest % 2 == 0) rest /= 2, ++twos;
  // eights, with one or two fours (or a lone two) for the remaining factors of two
  if (twos % 3 == 1 && twos >= 4) {
    s.radix[s.passes++] = 4;
    s.radix[s.passes++] = 4;
    twos -= 4;
  } else if (twos % 3 == 1) {
    s.radix[s.passes++] = 2;
    twos -= 1;
  } else if (twos % 3 == 2) {
    s.radix[s.passes++] = 4;
    twos -= 2;
  }
  for (; twos > 0; twos -= 3) s.radix[s.passes++] = 8;
  for (int r : {3, 5, 7})
    while (rest % r == 0) {
      if (s.passes == kFftMaxPasses) return false;
      s.radix[s.passes++] = r;
      rest /= r;
    }
  if (rest != 1) return false;
  *out = s;
  return true;
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a times conj(b)
__device__ __forceinline__ double2 cmulc(double2 a, double2 b) {
  return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
// a times -i (forward) or i (inverse)
template <bool INV>
__device__ __forceinline__ double2 crot(double2 a) {
  return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// x_p <- sum_q x_q exp(-+ 2 pi i p q / R), unnormalised.
template <int R, bool INV>
__device__ __forceinline__ void dft(double2 (&x)[R]) {
  if constexpr (R == 2) {
    const double2 a = x[0], b = x[1];
    x[0] = cadd(a, b);
    x[1] = csub(a, b);
  } else if constexpr (R == 4) {
    const double2 a = cadd(x[0], x[2]), b = csub(x[0], x[2]), c = cadd(x[1], x[3]), d = crot<INV>(csub(x[1], x[3]));
    x[0] = cadd(a, c);
    x[1] = cadd(b, d);
    x[2] = csub(a, c);
    x[3] = csub(b, d);
  } else if constexpr (R == 8) {
    double2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
    dft<4, INV>(e);
    dft<4, INV>(o);
    constexpr double h = 0.70710678118654752440;  // cos(pi/4)
    const double2 r1 = crot<INV>(o[1]), r3 = crot<INV>(o[3]);
    o[1] = make_double2(h * (o[1].x + r1.x), h * (o[1].y + r1.y));   // times exp(-+ i pi/4)
    o[2] = crot<INV>(o[2]);
    o[3] = make_double2(h * (r3.x - o[3].x), h * (r3.y - o[3].y));   // times exp(-+ 3 i pi/4)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = cadd(e[k], o[k]);
      x[k + 4] = csub(e[k], o[k]);
    }
  } else {
    // odd R: with a_k = x_k + x_{R-k} and b_k = x_k - x_{R-k},
    // x_p = x_0 + sum_k cos(2 pi k p / R) a_k -+ i sum_k sin(2 pi k p / R) b_k
    static_assert(R == 3 || R == 5 || R == 7, "radices 2, 3, 4, 5, 7 and 8");
    constexpr int M = (R - 1) / 2;
    constexpr double c3[1] = {-0.5}, s3[1] = {0.86602540378443864676};
    constexpr double c5[2] = {0.30901699437494742410, -0.80901699437494742410};
    constexpr double s5[2] = {0.95105651629515357212, 0.58778525229247312917};
    constexpr double c7[3] = {0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624};
    constexpr double s7[3] = {0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048};
    auto cs = [&](int k) { return R == 3 ? c3[k - 1] : R == 5 ? c5[k - 1] : c7[k - 1]; };
    auto sn = [&](int k) { return R == 3 ? s3[k - 1] : R == 5 ? s5[k - 1] : s7[k - 1]; };
    double2 a[M], b[M], y[R];
    y[0] = x[0];
#pragma unroll
    for (int k = 1; k <= M; ++k) {
      a[k - 1] = cadd(x[k], x[R - k]);
      b[k - 1] = csub(x[k], x[R - k]);
      y[0] = cadd(y[0], a[k - 1]);
    }
#pragma unroll
    for (int p = 1; p <= M; ++p) {
      double2 u = x[0], v = make_double2(0.0, 0.0);
#pragma unroll
      for (int k = 1; k <= M; ++k) {
        const int kp = (k * p) % R, at = kp <= M ? kp : R - kp;
        const double c = cs(at), s = kp <= M ? sn(at) : -sn(at);
        u.x += c * a[k - 1].x;
        u.y += c * a[k - 1].y;
        v.x += s * b[k - 1].x;
        v.y += s * b[k - 1].y;
      }
      const double2 w = crot<INV>(v);
      y[p] = cadd(u, w);
      y[R - p] = csub(u, w);
    }
#pragma unroll
    for (int p = 0; p < R; ++p) x[p] = y[p];
  }
}

// u / d for 0 <= u < 2^20, rd = 1/d rounded (its error moves the quotient by less than the
// half that is added).
__device__ __forceinline__ int small_div(int u, float rd) {
  return static_cast<int>((static_cast<float>(u) + 0.5f) * rd);
}

// One pass of radix R over sub-length s of `lines` lines of length n, in place; at(l) gives
// line l, whose entry e is the LDS slot at(l)(e).  Consecutive threads take consecutive lines.
template <int R, bool INV, typename At>
__device__ __forceinline__ void fft_pass(const At &at, int lines, int n, int s, const double2 *tw) {
  const int m = s / R, total = lines * (n / R), step = n / s;
  const float rl = __builtin_amdgcn_rcpf(static_cast<float>(lines)), rm = __builtin_amdgcn_rcpf(static_cast<float>(m));
  for (int t = static_cast<int>(threadIdx.x); t < total; t += static_cast<int>(blockDim.x)) {
    const int u = small_div(t, rl), l = t - u * lines;
    const int blk = small_div(u, rm), j = u - blk * m;
    const int e0 = blk * s + j;
    const auto line = at(l);
    double2 x[R];
#pragma unroll
    for (int q = 0; q < R; ++q) x[q] = *line(e0 + q * m);
    if (INV && m > 1) {  // (m = 1: every twiddle is 1)
#pragma unroll
      for (int q = 1; q < R; ++q) x[q] = cmulc(x[q], tw[j * q * step]);
    }
    dft<R, INV>(x);
    if (!INV && m > 1) {
#pragma unroll
      for (int q = 1; q < R; ++q) x[q] = cmul(x[q], tw[j * q * step]);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) *line(e0 + q * m) = x[q];
  }
  __syncthreads();
}

// Forward (natural order in, digit-reversed out) or inverse (the reverse; unnormalised)
// transform of every line, by the whole workgroup.  tw[k] = exp(-2 pi i k / n), k < n.  The
// caller's writes are visible (a barrier) before the call, and the results after it.
template <bool INV, typename At>
__device__ __forceinline__ void fft_lines(const At &at, int lines, const FftShape &f, const double2 *tw) {
  int s = INV ? 1 : f.n;
  for (int k = 0; k < f.passes; ++k) {
    const int r = f.radix[INV ? f.passes - 1 - k : k];
    if (INV) s *= r;
    switch (r) {
      case 8: fft_pass<8, INV>(at, lines, f.n, s, tw); break;
      case 4: fft_pass<4, INV>(at, lines, f.n, s, tw); break;
      case 2: fft_pass<2, INV>(at, lines, f.n, s, tw); break;
      case 3: fft_pass<3, INV>(at, lines, f.n, s, tw); break;
      case 5: fft_pass<5, INV>(at, lines, f.n, s, tw); break;
      default: fft_pass<7, INV>(at, lines, f.n, s, tw); break;
    }
    if (!INV) s /= r;
  }
}

}  // namespace

}  // namespace nb
