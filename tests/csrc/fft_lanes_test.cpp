// Host check of the lane-pair transforms that the plane kernels run (cf_fft32.h): the two
// lanes are run with an exchange of the values they hold at that point, as the kernels'
// multiply-add across lanes does it, and compared with a direct DFT in double.
#define __host__
#define __device__
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "cf_fft32.h"

struct Held {
  float re[16], im[16];
};

// runs both lanes of `fft`; a first run of each lane records what it holds at the exchange
template <typename Fft>
static void both_lanes(float (&re)[2][16], float (&im)[2][16], Fft fft) {
  Held held[2];
  for (int h = 0; h < 2; ++h) {
    float r[16], i[16];
    for (int k = 0; k < 16; ++k) r[k] = re[h][k], i[k] = im[h][k];
    fft(r, i, h, [&](float (&a)[16], float (&b)[16], float) {
      for (int k = 0; k < 16; ++k) held[h].re[k] = a[k], held[h].im[k] = b[k];
    });
  }
  for (int h = 0; h < 2; ++h)
    fft(re[h], im[h], h, [&](float (&a)[16], float (&b)[16], float s) {
      for (int k = 0; k < 16; ++k) {
        a[k] = std::fma(held[1 - h].re[k], s, a[k]);
        b[k] = std::fma(held[1 - h].im[k], s, b[k]);
      }
    });
}

template <bool INV>
static double check(const float *xr, const float *xi) {
  float tr[2][16], ti[2][16], fr[2][16], fi[2][16];
  for (int h = 0; h < 2; ++h)
    for (int n = 0; n < 16; ++n) {
      tr[h][n] = xr[2 * n + h], ti[h][n] = xi[2 * n + h];    // decimation in time
      fr[h][n] = xr[16 * h + n], fi[h][n] = xi[16 * h + n];  // in frequency
    }
  both_lanes(tr, ti, [](float (&r)[16], float (&i)[16], int h, auto add) { cf::fft32_lanes_dit<INV>(r, i, h, add); });
  both_lanes(fr, fi, [](float (&r)[16], float (&i)[16], int h, auto add) { cf::fft32_lanes_dif<INV>(r, i, h, add); });
  double e = 0.0;
  for (int k = 0; k < 32; ++k) {
    double sr = 0.0, si = 0.0;
    for (int n = 0; n < 32; ++n) {
      const double a = (INV ? 2.0 : -2.0) * M_PI * n * k / 32.0;
      sr += xr[n] * std::cos(a) - xi[n] * std::sin(a);
      si += xr[n] * std::sin(a) + xi[n] * std::cos(a);
    }
    e = std::fmax(e, std::fmax(std::fabs(sr - tr[k >> 4][k & 15]), std::fabs(si - ti[k >> 4][k & 15])));
    e = std::fmax(e, std::fmax(std::fabs(sr - fr[k & 1][k >> 1]), std::fabs(si - fi[k & 1][k >> 1])));
  }
  return e;
}

int main() {
  float xr[32], xi[32];
  // every unit impulse, real and imaginary: each twiddle and sign by itself
  for (int n = 0; n < 64; ++n) {
    for (int k = 0; k < 32; ++k) xr[k] = n == k, xi[k] = n == k + 32;
    const double e = std::fmax(check<false>(xr, xi), check<true>(xr, xi));
    if (!(e < 4e-7)) {
      std::printf("FAIL impulse %d: %g\n", n, e);
      return 1;
    }
  }
  std::srand(1);
  for (int rep = 0; rep < 200; ++rep) {
    for (int n = 0; n < 32; ++n) {
      xr[n] = (float)std::rand() / RAND_MAX - 0.5f;
      xi[n] = (float)std::rand() / RAND_MAX - 0.5f;
    }
    const double e = std::fmax(check<false>(xr, xi), check<true>(xr, xi));
    // five butterfly levels on sums of at most 32 values of 0.5: 5 * 16 * 2^-24 at the most
    if (!(e < 5e-6)) {
      std::printf("FAIL random %d: %g\n", rep, e);
      return 1;
    }
  }
  std::printf("OK\n");
  return 0;
}
