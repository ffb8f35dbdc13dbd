// 32-point complex FFTs held in registers, the building block of the frequency-domain
// 3-D convolution: shared by two neighbouring lanes in the kernels (fft32_lanes_dit,
// fft32_lanes_dif), and in one thread (fft32), which the host test compares them with.
//
// Convention: forward X[k] = sum_n x[n] e^{-2 pi i n k / 32}; inverse (INV = true)
// x[n] = sum_k X[k] e^{+2 pi i n k / 32}, unnormalised.  Radix-2 decimation in
// time over bit-reversed inputs; every index is a compile-time constant once the
// loops unroll, so the arrays stay in VGPRs and the twiddles become immediates.
#pragma once

namespace cf {

// cos and sin of 2 pi t / 32 for t = 0 .. 15
constexpr float kFftCos32[16] = {1.000000000e+00f,  9.807852804e-01f,  9.238795325e-01f,  8.314696123e-01f,
                                 7.071067812e-01f,  5.555702330e-01f,  3.826834324e-01f,  1.950903220e-01f,
                                 0.0f,              -1.950903220e-01f, -3.826834324e-01f, -5.555702330e-01f,
                                 -7.071067812e-01f, -8.314696123e-01f, -9.238795325e-01f, -9.807852804e-01f};
constexpr float kFftSin32[16] = {0.0f,             1.950903220e-01f, 3.826834324e-01f, 5.555702330e-01f,
                                 7.071067812e-01f, 8.314696123e-01f, 9.238795325e-01f, 9.807852804e-01f,
                                 1.000000000e+00f, 9.807852804e-01f, 9.238795325e-01f, 8.314696123e-01f,
                                 7.071067812e-01f, 5.555702330e-01f, 3.826834324e-01f, 1.950903220e-01f};

__host__ __device__ constexpr int fft_brev5(int i) {
  return ((i & 1) << 4) | ((i & 2) << 2) | (i & 4) | ((i & 8) >> 2) | ((i & 16) >> 4);
}

template <bool INV>
__host__ __device__ inline void fft32(float (&re)[32], float (&im)[32]) {
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const int j = fft_brev5(i);
    if (j > i) {
      const float tr = re[i], ti = im[i];
      re[i] = re[j];
      im[i] = im[j];
      re[j] = tr;
      im[j] = ti;
    }
  }
#pragma unroll
  for (int half = 1; half < 32; half <<= 1) {
#pragma unroll
    for (int i = 0; i < 32; i += 2 * half) {
#pragma unroll
      for (int j = 0; j < half; ++j) {
        const int t = j * (16 / half);  // twiddle e^{-+2 pi i t / 32}
        const int a = i + j, b = i + j + half;
        float br, bi;
        if (t == 0) {
          br = re[b];
          bi = im[b];
        } else if (t == 8) {  // times -i (forward) or +i (inverse)
          br = INV ? -im[b] : im[b];
          bi = INV ? re[b] : -re[b];
        } else {
          const float c = kFftCos32[t], s = INV ? kFftSin32[t] : -kFftSin32[t];
          br = re[b] * c - im[b] * s;
          bi = re[b] * s + im[b] * c;
        }
        re[b] = re[a] - br;
        im[b] = im[a] - bi;
        re[a] = re[a] + br;
        im[a] = im[a] + bi;
      }
    }
  }
}

// (r, i) times e^{-+2 pi i t / 32}, t = 0 .. 15 (NEG: times minus that), in place.  Which
// product of each part is rounded by itself is written out: left to the compiler, it
// depends on the code around the transform.
template <bool INV, bool NEG = false>
__host__ __device__ inline void twiddle32(float &r, float &i, int t) {
  const float c = NEG ? -kFftCos32[t] : kFftCos32[t], s = NEG ? -kFftSin32[t] : kFftSin32[t];
  if (t == 0) {
    r *= c;
    i *= c;
  } else if (t == 8) {
    const float is = INV ? i * -s : i * s;
    i = INV ? r * s : r * -s;
    r = is;
  } else if (INV) {
    const float is = i * -s, ic = i * c;
    i = __builtin_fmaf(r, s, ic);
    r = __builtin_fmaf(r, c, is);
  } else if (NEG && t < 8 && t != 4) {
    const float is = i * s, rs = r * -s;
    i = __builtin_fmaf(i, c, rs);
    r = __builtin_fmaf(r, c, is);
  } else {
    const float rs = r * -s, rc = r * c;
    r = __builtin_fmaf(i, s, rc);
    i = __builtin_fmaf(i, c, rs);
  }
}

// 16-point complex FFT in registers (same conventions; twiddles e^{-+2 pi i 2t / 32})
template <bool INV>
__host__ __device__ inline void fft16(float (&re)[16], float (&im)[16]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int j = ((i & 1) << 3) | ((i & 2) << 1) | ((i & 4) >> 1) | ((i & 8) >> 3);
    if (j > i) {
      const float tr = re[i], ti = im[i];
      re[i] = re[j];
      im[i] = im[j];
      re[j] = tr;
      im[j] = ti;
    }
  }
#pragma unroll
  for (int half = 1; half < 16; half <<= 1) {
#pragma unroll
    for (int a = 0; a < 16; ++a) {
      if (a & half) continue;
      const int b = a + half;
      float br = re[b], bi = im[b];
      twiddle32<INV>(br, bi, (a & (half - 1)) * (16 / half));
      re[b] = re[a] - br;
      im[b] = im[a] - bi;
      re[a] = re[a] + br;
      im[a] = im[a] + bi;
    }
  }
}

// A 32-point transform shared by two neighbouring lanes (h = 0, 1), each holding 16 points.
// add(re, im, s) adds s times the other lane's re and im to this lane's.  The half h = 1 is
// held negated across the exchange (by its twiddles, which is exact), so both lanes combine
// as mine + s * theirs with a sign s = +-1 per lane, in place of an add, a subtract, a
// select and a move for each value.
//
// Decimation in time: lane h holds x[2n + h] and ends with X[16 h + k], k = 0..15
// (each half-transform is a 16-point FFT; the odd half is twisted by e^{-+2 pi i k/32}
// and the two are combined as X[k] = E[k] + W^k O[k], X[k + 16] = E[k] - W^k O[k]).
template <bool INV, typename Add>
__host__ __device__ inline void fft32_lanes_dit(float (&re)[16], float (&im)[16], int h, Add add) {
  fft16<INV>(re, im);
  if (h) {
#pragma unroll
    for (int k = 0; k < 16; ++k) twiddle32<INV, true>(re[k], im[k], k);
  }
  add(re, im, h ? 1.0f : -1.0f);
}

// Decimation in frequency: lane h holds x[16 h + n] and ends with X[2k + h]
// (X[2k] is the 16-point FFT of x[n] + x[n + 16], X[2k + 1] that of
// (x[n] - x[n + 16]) e^{-+2 pi i n / 32}).
template <bool INV, typename Add>
__host__ __device__ inline void fft32_lanes_dif(float (&re)[16], float (&im)[16], int h, Add add) {
  add(re, im, h ? -1.0f : 1.0f);
  if (h) {
#pragma unroll
    for (int n = 0; n < 16; ++n) twiddle32<INV, true>(re[n], im[n], n);
  }
  fft16<INV>(re, im);
}

// The same transforms for two threads that exchange plain values: partner(v) returns the
// other thread's value of v, not negated.
template <bool INV, typename Partner>
__host__ __device__ inline void fft32_pair_dit(float (&re)[16], float (&im)[16], int h, Partner partner) {
  fft32_lanes_dit<INV>(re, im, h, [&](float (&r)[16], float (&i)[16], float s) {
    for (int k = 0; k < 16; ++k) {
      r[k] += (h ? s : -s) * partner(r[k]);
      i[k] += (h ? s : -s) * partner(i[k]);
    }
  });
}
template <bool INV, typename Partner>
__host__ __device__ inline void fft32_pair_dif(float (&re)[16], float (&im)[16], int h, Partner partner) {
  fft32_lanes_dif<INV>(re, im, h, [&](float (&r)[16], float (&i)[16], float s) {
    for (int n = 0; n < 16; ++n) {
      r[n] += s * partner(r[n]);
      i[n] += s * partner(i[n]);
    }
  });
}

}  // namespace cf
