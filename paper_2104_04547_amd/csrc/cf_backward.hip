// Backward pass of the Coherent Fusion score, for fine-tuning.
//
// Coherent Fusion trains the fusion layers and both branches together: the loss
// gradient reaches the 3D-CNN and the SG-CNN through the concatenated latents
// (Sec. 2.2; training hyper-parameters in Table V).  These kernels compute, for
// one upstream gradient per pose g_p = dL/ds_p, the vector-Jacobian product
// sum_p g_p ds_p/dtheta for every parameter theta, in float32.
//
// Design: every reduction in a fixed order (row chunks, then partial sums in order),
// so gradients are reproducible bit for bit and independent of the launch shape.
//   * per-atom matrix products of the SG-CNN and their weight gradients
//     sum_i U[i][a] V[i][b]: 32 x 32 blocks on the float32 matrix instruction
//     (32x32x2) straight from memory -- a few thousand atoms at widths up to 192 are
//     cache-resident, so a product is a few microseconds of latency (one thread per
//     output entry, each walking its row, took 97 us for 5500 atoms x 64 -> 192, the
//     weight gradients 38 + 32 us); weight gradients into partial sums per 128 rows, then
//     one pass adding the partials in order;
//   * conv weight and data gradients: products on the float32 matrix instruction
//     (32x32x2), see k_conv_wgrad and k_conv_dgrad.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "cf_internal.h"

namespace cf {

namespace {

constexpr int kT = 256;

inline dim3 grid1(int64_t n) { return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((n + kT - 1) / kT, 1 << 20))); }

__global__ __launch_bounds__(kT) void k_fill(float *p, int64_t n, float v) {
  for (int64_t i = blockIdx.x * (int64_t)kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) p[i] = v;
}

__global__ __launch_bounds__(kT) void k_add(float *dst, const float *src, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) dst[i] += src[i];
}

typedef float f32x16b __attribute__((ext_vector_type(16)));

// Four consecutive floats from p, of which `left` exist (zero past them)
__device__ inline float4 take4(const float *p, int left, bool aligned) {
  if (left >= 4 && aligned) return *reinterpret_cast<const float4 *>(p);
  return make_float4(left > 0 ? p[0] : 0.0f, left > 1 ? p[1] : 0.0f, left > 2 ? p[2] : 0.0f, left > 3 ? p[3] : 0.0f);
}

// TRANS = false: Y[i][j] (+)= b[j] + sum_k W[j][k] X[i][k], i < n, j < J, k < K
// TRANS = true:  Y[i][j] (+)= sum_k W[k][j] X[i][k]  (the transposed product dX = dY W)
// A wave takes 32 rows x 32 columns, a workgroup 64 x 64.  The matrix instruction adds its
// two products one after the other like two fused multiply-adds, so with k in ascending
// order an entry is bit for bit the plain sum (the SG-CNN's states are large sums that
// amplify rounding: taking k out of order doubled the gradient's distance from 64 bits).
template <bool TRANS>
__global__ __launch_bounds__(kT) void k_rowmat(const float *__restrict__ X, int ldx, int n, int K,
                                               const float *__restrict__ W, int ldw, const float *__restrict__ b,
                                               int J, float *__restrict__ Y, int ldy, int accumulate) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, khalf = lane >> 5, lrow = lane & 31;
  const int i0 = blockIdx.x * 64 + (wave & 1) * 32, j0 = blockIdx.y * 64 + (wave >> 1) * 32;
  if (i0 >= n || j0 >= J) return;
  const int i = min(i0 + lrow, n - 1), j = min(j0 + lrow, J - 1);  // rows past the end: read, not stored
  const float *x = X + (int64_t)i * ldx, *w = TRANS ? W + j : W + (int64_t)j * ldw;
  const bool xa = ldx % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
  const bool wa = !TRANS && ldw % 4 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0;
  const float bj = b ? b[j] : 0.0f;
  f32x16b acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = bj;
  // eight of K at k; WHOLE: they exist and lie aligned, so the loads of several such steps
  // are in flight together (a test per load waits for each)
  auto step = [&](int k, auto whole) {
    constexpr bool WHOLE = decltype(whole)::value;
    auto take = [&](const float *p, int left, bool al) {
      if constexpr (WHOLE) return *reinterpret_cast<const float4 *>(p);
      return take4(p, left, al);
    };
    float a[4], v[4];  // k + 2 s + khalf
    const float4 a0 = take(x + k, K - k, xa), a1 = take(x + k + 4, K - k - 4, xa);
    a[0] = khalf ? a0.y : a0.x;
    a[1] = khalf ? a0.w : a0.z;
    a[2] = khalf ? a1.y : a1.x;
    a[3] = khalf ? a1.w : a1.z;
    if (TRANS) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int kk = k + 2 * q + khalf;
        v[q] = WHOLE || kk < K ? w[(int64_t)kk * ldw] : 0.0f;
      }
    } else {
      const float4 w0 = take(w + k, K - k, wa), w1 = take(w + k + 4, K - k - 4, wa);
      v[0] = khalf ? w0.y : w0.x;
      v[1] = khalf ? w0.w : w0.z;
      v[2] = khalf ? w1.y : w1.x;
      v[3] = khalf ? w1.w : w1.z;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], v[q], acc, 0, 0, 0);
  };
  int k = 0;
  if (xa && (TRANS || wa)) {
#pragma unroll 8
    for (; k + 8 <= K; k += 8) step(k, std::true_type{});
  }
  for (; k < K; k += 8) step(k, std::false_type{});
  if (j0 + lrow >= J) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = i0 + 8 * (r >> 2) + 4 * khalf + (r & 3);
    if (row >= n) continue;
    float *y = Y + (int64_t)row * ldy + j;
    *y = accumulate ? *y + acc[r] : acc[r];
  }
}

// A[i][f] (+)= sum over the CSR row of atom i of S[col][f]; atom ids are local to
// the chunk (0 .. n-1).  A column outside the chunk is reported and skipped.
__global__ __launch_bounds__(kT) void k_agg(const int32_t *__restrict__ rowp, const int32_t *__restrict__ col,
                                            int64_t cap, const float *__restrict__ S, int n, int F,
                                            float *__restrict__ A, int accumulate, int64_t *status) {
  for (int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x; e < (int64_t)n * F; e += (int64_t)gridDim.x * kT) {
    const int i = (int)(e / F), f = (int)(e % F);
    int64_t e0 = rowp[i], e1 = rowp[i + 1];
    if (e1 > cap) e1 = cap;
    float acc = 0.0f;
    for (int64_t q = e0; q < e1; ++q) {
      const int j = col[q];
      if (j < 0 || j >= n) {
        if (f == 0) dev_fail(status, kDevBadGraph);
        continue;
      }
      acc += S[(int64_t)j * F + f];
    }
    A[e] = accumulate ? A[e] + acc : acc;
  }
}

__device__ inline float sigm(float x) { return 1.0f / (1.0f + expf(-x)); }

// GRU update from the stacked gate inputs GI = W_ih m + b_ih, GH = W_hh h + b_hh
// (gate rows r, z, n): h' = (1 - z) n + z h
__global__ __launch_bounds__(kT) void k_gru_fwd(const float *__restrict__ GI, const float *__restrict__ GH,
                                                const float *__restrict__ Hin, int n, int H, float *__restrict__ Hout) {
  for (int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x; e < (int64_t)n * H; e += (int64_t)gridDim.x * kT) {
    const int64_t i = e / H;
    const int j = (int)(e % H);
    const float *gi = GI + i * 3 * H, *gh = GH + i * 3 * H;
    const float r = sigm(gi[j] + gh[j]), z = sigm(gi[H + j] + gh[H + j]);
    const float nn = tanhf(gi[2 * H + j] + r * gh[2 * H + j]);
    Hout[e] = (1.0f - z) * nn + z * Hin[e];
  }
}

// GRU backward, elementwise: from dh' the gradients of the gate inputs dGI
// (dr_pre, dz_pre, dn_pre), dGH (dr_pre, dz_pre, r dn_pre) and the direct part
// z dh' of dh
__global__ __launch_bounds__(kT) void k_gru_bwd(const float *__restrict__ GI, const float *__restrict__ GH,
                                                const float *__restrict__ Hin, const float *__restrict__ dHout, int n,
                                                int H, float *__restrict__ dGI, float *__restrict__ dGH,
                                                float *__restrict__ dHd) {
  for (int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x; e < (int64_t)n * H; e += (int64_t)gridDim.x * kT) {
    const int64_t i = e / H;
    const int j = (int)(e % H);
    const float *gi = GI + i * 3 * H, *gh = GH + i * 3 * H;
    const float r = sigm(gi[j] + gh[j]), z = sigm(gi[H + j] + gh[H + j]);
    const float hn = gh[2 * H + j];
    const float nn = tanhf(gi[2 * H + j] + r * hn);
    const float d = dHout[e], h = Hin[e];
    const float dn = d * (1.0f - z), dz = d * (h - nn);
    const float dpn = dn * (1.0f - nn * nn);
    const float dpr = dpn * hn * r * (1.0f - r), dpz = dz * z * (1.0f - z);
    float *a = dGI + i * 3 * H, *b = dGH + i * 3 * H;
    a[j] = dpr;
    a[H + j] = dpz;
    a[2 * H + j] = dpn;
    b[j] = dpr;
    b[H + j] = dpz;
    b[2 * H + j] = dpn * r;
    dHd[e] = d * z;
  }
}

// readout s[p][j] = sum over the ligand atoms i of pose p (in order) of
// sigma(Gpre[i][j]) * V[i][j]
__global__ __launch_bounds__(kT) void k_readout(const float *__restrict__ Gpre, const float *__restrict__ V,
                                                const uint8_t *__restrict__ is_lig, const int32_t *__restrict__ atom_off,
                                                int p0, int np, int H, float *__restrict__ S) {
  const int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x;
  if (e >= (int64_t)np * H) return;
  const int p = (int)(e / H), j = (int)(e % H);
  const int base = atom_off[p0];
  const int a0 = atom_off[p0 + p], a1 = atom_off[p0 + p + 1];
  float acc = 0.0f;
  // eight atoms' loads in flight, added in order
  for (int a = a0; a < a1; a += 8) {
    uint8_t lig[8];
    float g[8], v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int au = min(a + u, a1 - 1);
      const int64_t i = (int64_t)(au - base) * H + j;
      lig[u] = is_lig[au];
      g[u] = Gpre[i];
      v[u] = V[i];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (a + u < a1 && lig[u]) acc = fmaf(sigm(g[u]), v[u], acc);
  }
  S[e] = acc;
}

__global__ __launch_bounds__(kT) void k_readout_bwd(const float *__restrict__ Gpre, const float *__restrict__ V,
                                                    const uint8_t *__restrict__ is_lig,
                                                    const int32_t *__restrict__ atom_off, int p0, int np, int H,
                                                    const float *__restrict__ dS, float *__restrict__ dGpre,
                                                    float *__restrict__ dV) {
  const int base = atom_off[p0], n = atom_off[p0 + np] - base;
  for (int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x; e < (int64_t)n * H; e += (int64_t)gridDim.x * kT) {
    const int i = (int)(e / H), j = (int)(e % H);
    // pose of atom i: binary search over the chunk's offsets
    int lo = 0, hi = np;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (atom_off[p0 + mid] - base <= i) lo = mid; else hi = mid;
    }
    float dg = 0.0f, dv = 0.0f;
    if (is_lig[base + i]) {
      const float g = sigm(Gpre[e]), ds = dS[(int64_t)lo * H + j];
      dg = ds * V[e] * g * (1.0f - g);
      dv = ds * g;
    }
    dGpre[e] = dg;
    dV[e] = dv;
  }
}

// C[a][b] (+)= sum_{i < n} U[i][a] V[i][b] (V = null: the column sums of U, B = 1).
// Pass 1: chunk s of kRowsPerChunk rows -> partial[s][a][b] (column sums here, products
// below); pass 2 adds the partials in chunk order.
constexpr int kRowsPerChunk = 128;

__global__ __launch_bounds__(kT) void k_outer_partial(const float *__restrict__ U, int ldu, int n, int A,
                                                      float *__restrict__ part) {
  const int64_t a = blockIdx.x * (int64_t)kT + threadIdx.x;
  const int s = blockIdx.y;
  if (a >= A) return;
  const int i0 = s * kRowsPerChunk, i1 = min(n, i0 + kRowsPerChunk);
  float acc = 0.0f;
#pragma unroll 16
  for (int i = i0; i < i1; ++i) acc += U[(int64_t)i * ldu + a];
  part[(int64_t)s * A + a] = acc;
}

// The same partials by matrix instruction (V given): a wave takes 32 x 32 entries (a, b) of
// one chunk, two rows a step.
__global__ __launch_bounds__(kT) void k_outer_mfma(const float *__restrict__ U, int ldu, const float *__restrict__ V,
                                                   int ldv, int n, int A, int B, float *__restrict__ part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, khalf = lane >> 5, lrow = lane & 31;
  const int nbb = (B + 31) / 32;
  const int blk = blockIdx.x * 4 + wave, a0 = blk / nbb * 32, b0 = blk % nbb * 32, s = blockIdx.y;
  if (a0 >= A) return;
  const int a = min(a0 + lrow, A - 1), b = min(b0 + lrow, B - 1);
  const int i0 = s * kRowsPerChunk, i1 = min(n, i0 + kRowsPerChunk);
  f32x16b acc = {};
  if (i1 - i0 == kRowsPerChunk) {
    // a whole chunk: no tests, so that many rows' loads are in flight
    const float *u = U + (int64_t)(i0 + khalf) * ldu + a, *v = V + (int64_t)(i0 + khalf) * ldv + b;
#pragma unroll 32
    for (int i = 0; i < kRowsPerChunk; i += 2)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u[(int64_t)i * ldu], v[(int64_t)i * ldv], acc, 0, 0, 0);
  } else {
#pragma unroll 8
    for (int i = i0; i < i1; i += 2) {
      const int r = i + khalf;
      const float u = r < i1 ? U[(int64_t)r * ldu + a] : 0.0f, v = r < i1 ? V[(int64_t)r * ldv + b] : 0.0f;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u, v, acc, 0, 0, 0);
    }
  }
  if (b0 + lrow >= B) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = a0 + 8 * (r >> 2) + 4 * khalf + (r & 3);
    if (row < A) part[(int64_t)s * A * B + (int64_t)row * B + b] = acc[r];
  }
}

__global__ __launch_bounds__(kT) void k_outer_sum(const float *__restrict__ part, int nchunk, int A, int B,
                                                  float *__restrict__ C, int ldc, int accumulate) {
  const int64_t ab = (int64_t)A * B;
  const int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x;
  if (e >= ab) return;
  float acc = 0.0f;
#pragma unroll 16
  for (int s = 0; s < nchunk; ++s) acc += part[(int64_t)s * ab + e];
  float *c = C + (e / B) * ldc + (e % B);
  *c = accumulate ? *c + acc : acc;
}

// ... for few entries and many chunks (a layer's bias gradient: 64 entries, hundreds of
// chunks): a wave per entry, lane q the chunks q, q + 64, ..., then the lanes in a fixed tree
__global__ __launch_bounds__(kT) void k_outer_sum_wave(const float *__restrict__ part, int nchunk, int A, int B,
                                                       float *__restrict__ C, int ldc, int accumulate) {
  const int64_t ab = (int64_t)A * B;
  const int64_t e = blockIdx.x * (int64_t)(kT / 64) + (threadIdx.x >> 6);
  if (e >= ab) return;
  const int lane = threadIdx.x & 63;
  float acc = 0.0f;
#pragma unroll 4
  for (int s = lane; s < nchunk; s += 64) acc += part[(int64_t)s * ab + e];
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  float *c = C + (e / B) * ldc + (e % B);
  if (lane == 0) *c = accumulate ? *c + acc : acc;
}

// ---- 3D-CNN ----

// pool[p][c] = mean over the voxels of act[p][v][c]: a workgroup takes 32 channels of a
// pose, its 32 groups of threads every 32nd voxel in order, and the groups are added in order
constexpr int kPoolT = 1024;
__global__ __launch_bounds__(kPoolT) void k_pool_mean(const float *__restrict__ act, int64_t vox, int cstride, int C,
                                                     float *__restrict__ pool) {
  __shared__ float sum[kPoolT];
  const int p = blockIdx.y, c = blockIdx.x * 32 + (threadIdx.x & 31), g = threadIdx.x >> 5;
  float acc = 0.0f;
  if (c < C) {
    const float *a = act + (int64_t)p * vox * cstride + c;
#pragma unroll 8
    for (int64_t v = g; v < vox; v += kPoolT / 32) acc += a[v * cstride];
  }
  sum[threadIdx.x] = acc;
  __syncthreads();
  if (g == 0 && c < C) {
    float m = 0.0f;
    for (int q = 0; q < kPoolT / 32; ++q) m += sum[q * 32 + threadIdx.x];
    pool[(int64_t)p * C + c] = m / (float)vox;
  }
}

// dact[p][v][c] = dpool[p][c] / vox (channels past C zero)
__global__ __launch_bounds__(kT) void k_pool_seed(const float *__restrict__ dpool, int np, int64_t vox, int cstride,
                                                  int C, float *__restrict__ dact) {
  const int64_t n = (int64_t)np * vox * cstride;
  for (int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT) {
    const int c = (int)(e % cstride);
    const int64_t p = e / (vox * cstride);
    dact[e] = c < C ? dpool[p * C + c] / (float)vox : 0.0f;
  }
}

// d *= (y > 0): the ReLU's gradient from its output (y = max(u, 0))
__global__ __launch_bounds__(kT) void k_relu_mask(float *__restrict__ d, const float *__restrict__ y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT)
    d[i] = y[i] > 0.0f ? d[i] : 0.0f;
}

// d *= (y > 0) for rows of width J laid out with stride ld
__global__ __launch_bounds__(kT) void k_relu_rows(float *__restrict__ y, int n, int J, int ld) {
  for (int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x; e < (int64_t)n * J; e += (int64_t)gridDim.x * kT) {
    float *p = y + (e / J) * ld + (e % J);
    *p = *p > 0.0f ? *p : 0.0f;
  }
}

__global__ __launch_bounds__(kT) void k_relu_grad_rows(float *__restrict__ d, const float *__restrict__ pre, int n,
                                                       int J) {
  for (int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x; e < (int64_t)n * J; e += (int64_t)gridDim.x * kT)
    d[e] = pre[e] > 0.0f ? d[e] : 0.0f;
}

// Folded weights for the data gradient, as MFMA B fragments: W[co][ci][t] * a[co],
// a = gamma / sqrt(var + eps) with BatchNorm, else 1, at
// WT[((t * nch + co / 8) * cpad + ci) * 8 + (co & 1) * 4 + (co % 8) / 2], nch chunks of 8
// output channels and cpad input channels (zero past the layer's): the four K values of
// a lane (one parity of eight channels) are one 16-byte load.
__global__ __launch_bounds__(kT) void k_fold_wt(const float *__restrict__ W, const float *__restrict__ gamma,
                                                const float *__restrict__ var, int cout, int cin, int taps, int nch,
                                                int cpad, float *__restrict__ WT) {
  const int64_t n = (int64_t)taps * nch * cpad * 8;
  for (int64_t e = blockIdx.x * (int64_t)kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT) {
    const int q = (int)(e % 8), ci = (int)((e / 8) % cpad);
    const int64_t tc = e / (8 * (int64_t)cpad);
    const int co = (int)(tc % nch) * 8 + 2 * (q & 3) + (q >> 2), t = (int)(tc / nch);
    float v = 0.0f;
    if (co < cout && ci < cin) {
      const float a = gamma ? (float)((double)gamma[co] / sqrt((double)var[co] + 1e-5)) : 1.0f;
      v = W[((int64_t)co * cin + ci) * taps + t] * a;
    }
    WT[e] = v;
  }
}

// Weight gradient of one conv layer w.r.t. its folded weights, per pose (and, with
// few poses, per row subset):
//   part[p][co][t * cin + ci] = sum_o dY[p][o][co] * X[p][s o + t - P][ci]
// A workgroup takes 32 MB output channels and 32 NB columns (tx, ci) of one (tz, ty);
// its four waves take the output rows (oz, oy) in turn, each with all MB x NB blocks of
// accumulators, and add up in order at the end.  Per row a wave stages its dY row and
// the X row that (tz, ty) pairs with it in LDS of its own, in runs of
// output voxels (so no barrier inside): with the X row packed at cin floats per voxel,
// column q = tx cin + ci at output voxel ox is float S ox cin + q, the same for every
// tap of the row.
// What bounds it: the float32 matrix instruction (64 cycles; MB NB of them per
// MB + NB LDS reads).  A run's loads wait in registers while the run before it is
// multiplied: with the loads between the runs, two waves per SIMD left the matrix cores
// idle for more than half of the time.  The two stride-2 layers of the full model, 8 poses
// at 48^3: 2.1 + 2.0 ms -> 1.28 + 0.87 ms (72 and 89 TFLOP/s; 17 % of the first one's
// columns are padding).
// voxels of a run at most, and pieces of X per lane that wait in registers (16 bytes each,
// or 4): what the registers hold beside 2 x 5 blocks
constexpr int wgrad_run(bool vec) { return vec ? 16 : 24; }
constexpr int wgrad_xregs(bool vec) { return vec ? 8 : 16; }
// floats of LDS per wave at a run of `run` voxels: dY run, X run, and zeros for the
// columns past the row's last (at most 4 blocks of 32 and 31 more)
inline int wgrad_wave_floats(int run, int KS, int S, int cin) {
  const int f = run * 64 + (S * (run - 1) + KS) * cin + 160;
  return (f < 1024 ? 1024 : f + 3) / 4 * 4;
}

// VEC: cin, xstride and the X pointer allow 16-byte loads of X.  A run's values are
// loaded into registers while the run before it is multiplied: six 16-byte pieces of dY
// (three with MB = 1) and the first kXV of X per lane; whatever X has beyond those
// (bw_conv_wgrad picks runs that have none where it can) is loaded when it is stored.
template <int MB, int NB, bool VEC>
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_wgrad(
    const float *__restrict__ X, int D, int xstride, int cin, const float *__restrict__ dY, int Do, int ystride,
    int cout, int KS, int S, int ncg, int nsplit, int run, int wave_floats, float *__restrict__ part) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  typedef typename std::conditional<VEC, float4, float>::type xv_t;
  constexpr int kXV = wgrad_xregs(VEC), kE = VEC ? 4 : 1;
  constexpr int kYQ = 8 * MB, kYV = 64 / kYQ, kYU = wgrad_run(VEC) / kYV;  // dY: pieces a voxel, voxels a pass, passes
  const int P = (KS - 1) / 2;
  const int cg = blockIdx.x % ncg, tzy = blockIdx.x / ncg, tz = tzy / KS, ty = tzy % KS;
  const int c0 = blockIdx.y * 32 * MB, q0 = cg * 32 * NB;
  const int p = blockIdx.z / nsplit, split = blockIdx.z % nsplit;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int khalf = lane >> 5, lrow = lane & 31;
  float *sA = lds + wave * wave_floats, *sB = sA + run * 64;
  const int xw = S * (run - 1) + KS;           // X positions of a run
  const int cw = cin / kE, xtot = xw * cw;     // their pieces
  const float *xp = X + (int64_t)p * D * D * D * xstride;
  const float *yp = dY + (int64_t)p * Do * Do * Do * ystride + c0;
  const int ca = (lane % kYQ) * 4, va = lane / kYQ, nca = c0 + ca < ystride ? cout - c0 - ca : 0;
  const int xi0 = lane / cw, xc0 = lane % cw, xdi = 64 / cw, xdc = 64 % cw;
  f32x16b acc[MB][NB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[m][n] = f32x16b{};
  for (int e = lane; e < 160; e += 64) sB[xw * cin + e] = 0.0f;  // columns past the row's last
  // this wave's output rows, those whose X row lies in the grid
  auto row_ok = [&](int r) {
    const int z = S * (r / Do) + tz - P, y = S * (r % Do) + ty - P;
    return z >= 0 && z < D && y >= 0 && y < D;
  };
  auto next_row = [&](int r) {
    while (r < Do * Do && !row_ok(r)) r += 4 * nsplit;
    return r;
  };
  float4 ya[kYU];
  xv_t xa[kXV];
  auto load = [&](int r, int o0) {
    const int no = min(run, Do - o0), x0 = S * o0 - P, xe = min(D, x0 + S * (no - 1) + KS);
    const float *yr = yp + ((int64_t)r * Do + o0) * ystride;
    int v0 = va;
    asm volatile("" : "+v"(v0));
#pragma unroll
    for (int u = 0; u < kYU; ++u) {
      const int v = u * kYV + v0;
      ya[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (v < no && nca > 0) ya[u] = *reinterpret_cast<const float4 *>(yr + (uint32_t)(v * ystride + ca));
    }
    const float *xr = xp + ((int64_t)(S * (r / Do) + tz - P) * D + S * (r % Do) + ty - P) * D * xstride;
    int i = xi0, c = xc0;
    asm volatile("" : "+v"(i), "+v"(c));  // positions are stepped anew for each run, not held
#pragma unroll
    for (int u = 0; u < kXV; ++u) {
      const int x = x0 + i;
      xa[u] = xv_t{};
      if (u * 64 + lane < xtot && x >= 0 && x < xe)
        xa[u] = *reinterpret_cast<const xv_t *>(xr + (uint32_t)(x * xstride + kE * c));
      i += xdi;
      c += xdc;
      if (c >= cw) c -= cw, ++i;
    }
  };
  auto store = [&](int r, int o0) {
    // dY run: [voxel][64], odd voxels with their two 32-channel halves swapped, so that
    // the two K halves of a fragment read fall on different banks
#pragma unroll
    for (int u = 0; u < kYU; ++u) {
      const int v = u * kYV + va;
      float4 t = ya[u];
      if (nca < 4) {
        if (nca < 1) t.x = 0.0f;
        if (nca < 2) t.y = 0.0f;
        if (nca < 3) t.z = 0.0f;
        t.w = 0.0f;
      }
      if (v < run) *reinterpret_cast<float4 *>(sA + v * 64 + (ca ^ ((v & 1) << 5))) = t;
    }
    // X run: positions S o0 - P + i, cin floats each; zero outside the grid and past the
    // last one an output voxel of the run reaches
    xv_t *xb = reinterpret_cast<xv_t *>(sB);
#pragma unroll
    for (int u = 0; u < kXV; ++u)
      if (u * 64 + lane < xtot) xb[u * 64 + lane] = xa[u];
    if (xtot > kXV * 64) {
      const int no = min(run, Do - o0), x0 = S * o0 - P, xe = min(D, x0 + S * (no - 1) + KS);
      const float *xr = xp + ((int64_t)(S * (r / Do) + tz - P) * D + S * (r % Do) + ty - P) * D * xstride;
      for (int e = kXV * 64 + lane; e < xtot; e += 64) {
        const int i = e / cw, c = e - i * cw, x = x0 + i;
        xv_t t = {};
        if (x >= 0 && x < xe) t = *reinterpret_cast<const xv_t *>(xr + (int64_t)x * xstride + kE * c);
        xb[e] = t;
      }
    }
  };
  int r = next_row(split * 4 + wave), o0 = 0;
  if (r < Do * Do) load(r, o0);
  while (r < Do * Do) {
    // the wave's own LDS: its operations stay in order, only the compiler is held
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    store(r, o0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    o0 += run;
    if (o0 >= Do) {
      o0 = 0;
      r = next_row(r + 4 * nsplit);
    }
    if (r < Do * Do) load(r, o0);
    const float *bp = sB + khalf * S * cin + q0 + lrow;
    for (int k = 0; k < run; k += 2) {
      const int v = k + khalf;
      float a[MB], b[NB];
#pragma unroll
      for (int m = 0; m < MB; ++m) a[m] = sA[v * 64 + ((32 * m + lrow) ^ (khalf << 5))];
#pragma unroll
      for (int n = 0; n < NB; ++n) b[n] = bp[k * S * cin + 32 * n];
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[m], b[n], acc[m][n], 0, 0, 0);
    }
  }
  // the waves' sums in order, a block at a time
  const int64_t Q = (int64_t)KS * KS * KS * cin;
  const int qn = KS * cin;
  float *out = part + (int64_t)blockIdx.z * cout * Q + (int64_t)tzy * qn;
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 16; ++j) lds[wave * 1024 + (8 * (j >> 2) + 4 * khalf + (j & 3)) * 32 + lrow] = acc[m][n][j];
      __syncthreads();
      for (int e = threadIdx.x; e < 1024; e += kT) {
        const int co = c0 + 32 * m + e / 32, q = q0 + 32 * n + e % 32;
        if (co < cout && q < qn) out[co * Q + q] = lds[e] + lds[1024 + e] + lds[2048 + e] + lds[3072 + e];
      }
    }
}

// Data gradient of one conv layer (the transposed conv as a gather):
//   dX[p][v][ci] += sum_{t, co} dY[p][o][co] * W'[co][ci][t],  s o = v + P - t
// Input voxels of one parity per axis (v = s u + r) see the same taps t = t0 + s m, and
// reach the output voxels o = u + c - m: per parity class this is a dense stride-1
// correlation over dY.  A workgroup takes a 4 x 4 x 4 tile of u of one class and 64 input
// channels, a wave 32 x 32 of them; K runs over 8-channel chunks of co (the tile's dY
// halo in LDS, even and odd channels apart) and the class's taps (weight fragments from
// L2, two taps ahead).
// What bounds it: the float32 matrix instruction, four per row and weight load.
// Five layers of the full model, 8 poses at 48^3: 13.0 ms, 101 TFLOP/s (LDS-tiled FMAs that
// tested every tap for parity: 65.7 ms).
constexpr int kDT = 4;                     // tile edge (class voxels)
constexpr int kDHalo = kDT + 6;            // halo edge at most (k = 7, stride 1)

__global__ __launch_bounds__(kT) void k_conv_dgrad(const float *__restrict__ dY, int Do, int ystride, int nch,
                                                   const float *__restrict__ WT, int cin, int cpad, int KS, int S,
                                                   int D, int xstride, float *__restrict__ dX) {
  __shared__ __attribute__((aligned(16))) float halo[kDHalo * kDHalo * kDHalo * 8];
  const int ncl = S * S * S, P = (KS - 1) / 2;
  const int p = blockIdx.z / ncl, cl = blockIdx.z % ncl;
  const int rr[3] = {cl / (S * S), (cl / S) % S, cl % S};
  int t0[3], nt[3], nu[3], base[3];  // first tap, taps, class voxels, first halo voxel - u0
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    t0[d] = (rr[d] + P) % S;
    nt[d] = (KS - t0[d] + S - 1) / S;
    nu[d] = (D - rr[d] + S - 1) / S;
    base[d] = (rr[d] + P - t0[d]) / S - (nt[d] - 1);
  }
  const int Dc = (D + S - 1) / S, ntl = (Dc + kDT - 1) / kDT;
  const int uz0 = (int)(blockIdx.x / (ntl * ntl)) * kDT, uy0 = (int)(blockIdx.x / ntl) % ntl * kDT,
            ux0 = (int)(blockIdx.x % ntl) * kDT;
  if (uz0 >= nu[0] || uy0 >= nu[1] || ux0 >= nu[2]) return;
  const int hz = kDT + nt[0] - 1, hy = kDT + nt[1] - 1, hx = kDT + nt[2] - 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, khalf = lane >> 5, lrow = lane & 31;
  const int m = (wave & 1) * 32 + lrow;                       // this lane's A row: tile voxel
  const int ci = blockIdx.y * 64 + (wave >> 1) * 32 + lrow;   // ... and B column
  const bool cols = blockIdx.y * 64 + (wave >> 1) * 32 < cin; // a wave past the channels only stages
  const int lz = m / 16, ly = (m / 4) % 4, lx = m % 4;
  const float *yp = dY + (int64_t)p * Do * Do * Do * ystride;
  f32x16b acc = {};
  for (int c = 0; c < nch; ++c) {
    __syncthreads();
    for (int e = threadIdx.x; e < hz * hy * hx; e += kT) {
      const int x = e % hx, y = (e / hx) % hy, z = e / (hx * hy);
      const int oz = uz0 + base[0] + z, oy = uy0 + base[1] + y, ox = ux0 + base[2] + x;
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
      if (oz >= 0 && oz < Do && oy >= 0 && oy < Do && ox >= 0 && ox < Do) {
        const float *src = yp + (((int64_t)oz * Do + oy) * Do + ox) * ystride + c * 8;
        a = *reinterpret_cast<const float4 *>(src);
        b = *reinterpret_cast<const float4 *>(src + 4);
      }
      float4 *dst = reinterpret_cast<float4 *>(halo + e * 8);
      dst[0] = make_float4(a.x, a.z, b.x, b.z);
      dst[1] = make_float4(a.y, a.w, b.y, b.w);
    }
    __syncthreads();
    if (!cols) continue;
    // weight fragments of the class's taps in turn (mx fastest; the last one again past
    // the end)
    const float *wb = WT + ((int64_t)c * cpad + ci) * 8 + khalf * 4;
    int fx = 0, fy = 0, fz = 0;
    auto next_frag = [&]() {
      const int t = ((t0[0] + S * fz) * KS + t0[1] + S * fy) * KS + t0[2] + S * fx;
      if (++fx == nt[2]) {
        fx = 0;
        if (++fy == nt[1]) {
          fy = 0;
          if (++fz == nt[0]) fx = nt[2] - 1, fy = nt[1] - 1, fz = nt[0] - 1;
        }
      }
      return *reinterpret_cast<const float4 *>(wb + (int64_t)t * nch * cpad * 8);
    };
    float4 w0 = next_frag(), w1 = next_frag();
    for (int mz = 0; mz < nt[0]; ++mz)
      for (int my = 0; my < nt[1]; ++my) {
        const float *row = halo + (((lz + nt[0] - 1 - mz) * hy + ly + nt[1] - 1 - my) * hx + lx) * 8 + khalf * 4;
        for (int mx = 0; mx < nt[2]; ++mx) {
          const float4 w = w0;
          w0 = w1;
          w1 = next_frag();
          const float4 a = *reinterpret_cast<const float4 *>(row + (nt[2] - 1 - mx) * 8);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, w.x, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, w.y, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, w.z, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, w.w, acc, 0, 0, 0);
        }
      }
  }
  if (!cols || ci >= cin) return;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int mm = (wave & 1) * 32 + 8 * (j >> 2) + 4 * khalf + (j & 3);
    const int uz = uz0 + mm / 16, uy = uy0 + (mm / 4) % 4, ux = ux0 + mm % 4;
    if (uz >= nu[0] || uy >= nu[1] || ux >= nu[2]) continue;
    const int64_t v = ((int64_t)(S * uz + rr[0]) * D + S * uy + rr[1]) * D + S * ux + rr[2];
    dX[((int64_t)p * D * D * D + v) * xstride + ci] += acc[j];
  }
}

// Folded-weight gradients -> gradients of the blob's parameters, one workgroup
// per output channel co.  Folding: W' = a W, b' = a (b - mu) + beta with
// a = gamma / sqrt(var + eps) (without BatchNorm: a = 1, b' = b).  So
//   dW = a dW', db = a db', dbeta = db', dmean = -a db',
//   dgamma = g_a / sqrt(var + eps), dvar = -g_a a / (2 (var + eps)),
// with g_a = sum dW' W + db' (b - mu).  dWf: [co][t][ci]; blob W: [co][ci][t].
constexpr int kFoldT = 1024;  // a workgroup per output channel: loads in flight count (256 threads: 48 us)
__global__ __launch_bounds__(kFoldT) void k_fold_grad(const float *__restrict__ dWf, const float *__restrict__ dbf,
                                                  const float *__restrict__ W, const float *__restrict__ b,
                                                  const float *__restrict__ gamma, const float *__restrict__ mean,
                                                  const float *__restrict__ var, int cin, int taps,
                                                  float *__restrict__ gW, float *__restrict__ gb,
                                                  float *__restrict__ ggamma, float *__restrict__ gbeta,
                                                  float *__restrict__ gmean, float *__restrict__ gvar) {
  __shared__ double red[kFoldT];
  const int co = blockIdx.x, tid = threadIdx.x;
  const double a = gamma ? (double)gamma[co] / sqrt((double)var[co] + 1e-5) : 1.0;
  const int64_t n = (int64_t)cin * taps;
  double ga = 0.0;
#pragma unroll 4
  for (int64_t e = tid; e < n; e += kFoldT) {
    const int ci = (int)(e / taps), t = (int)(e % taps);
    const float d = dWf[((int64_t)co * taps + t) * cin + ci];
    const int64_t wi = (int64_t)co * n + e;
    ga += (double)d * (double)W[wi];
    gW[wi] += (float)(a * (double)d);
  }
  red[tid] = ga;
  __syncthreads();
  for (int s = kFoldT / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  if (tid == 0) {
    const double db = dbf[co];
    gb[co] += (float)(a * db);
    if (gamma) {
      const double ve = (double)var[co] + 1e-5;
      const double g_a = red[0] + db * ((double)b[co] - (double)mean[co]);
      ggamma[co] += (float)(g_a / sqrt(ve));
      gbeta[co] += (float)db;
      gmean[co] += (float)(-a * db);
      gvar[co] += (float)(-g_a * a / (2.0 * ve));
    }
  }
}

// ---- Coherent Fusion head ----

__device__ inline float selu_f(float x) {
  constexpr float kL = 1.0507009873554805f, kA = 1.6732632423543772f;
  return x > 0.0f ? kL * x : kL * kA * expm1f(x);
}
__device__ inline float selu_d(float x) {
  constexpr float kL = 1.0507009873554805f, kA = 1.6732632423543772f;
  return x > 0.0f ? kL : kL * kA * expf(x);
}

// One workgroup per pose: the fusion block's forward (z_0 = [cnn; sg], hidden SELU
// layers, optionally residual after the first, linear output) and its backward
// from dscore.  Per-pose parameter gradients go to part[p][...] in the blob order
// of the head; dcnn / dsg are the latents' gradients.  prm: the head's blob
// parameters.
constexpr int kHeadMaxW = 512;

__global__ __launch_bounds__(kT) void k_head_bwd(const float *__restrict__ cnn, int lc, const float *__restrict__ sg,
                                                 int sgw, const float *__restrict__ prm, int nhid, int fh,
                                                 int residual, const float *__restrict__ dscore,
                                                 float *__restrict__ scores, float *__restrict__ dcnn,
                                                 float *__restrict__ dsg, float *__restrict__ part, int64_t nprm) {
  __shared__ float z[9][kHeadMaxW];    // z_0 .. z_nhid
  __shared__ float pre[8][kHeadMaxW];  // hidden pre-activations
  __shared__ float dz[2][kHeadMaxW];
  __shared__ float red[kT];
  const int p = blockIdx.x, tid = threadIdx.x;
  const int fin = lc + sgw;
  for (int k = tid; k < fin; k += kT) z[0][k] = k < lc ? cnn[(int64_t)p * lc + k] : sg[(int64_t)p * sgw + k - lc];
  __syncthreads();
  // forward
  int64_t off = 0;
  int w = fin;
  for (int l = 0; l < nhid; ++l) {
    const float *W = prm + off, *b = prm + off + (int64_t)fh * w;
    for (int j = tid; j < fh; j += kT) {
      float acc = b[j];
      for (int k = 0; k < w; ++k) acc = fmaf(W[(int64_t)j * w + k], z[l][k], acc);
      pre[l][j] = acc;
      const float y = selu_f(acc);
      z[l + 1][j] = (residual && l > 0) ? y + z[l][j] : y;
    }
    __syncthreads();
    off += (int64_t)fh * w + fh;
    w = fh;
  }
  const float *Wo = prm + off;
  float acc = 0.0f;
  for (int k = tid; k < w; k += kT) acc = fmaf(Wo[k], z[nhid][k], acc);
  red[tid] = acc;
  __syncthreads();
  for (int s = kT / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  const float g = dscore[p];
  float *pp = part + (int64_t)p * nprm;
  if (tid == 0) {
    if (scores) scores[p] = red[0] + Wo[w];
    pp[off + w] = g;  // d b_out
  }
  for (int k = tid; k < w; k += kT) {
    pp[off + k] = g * z[nhid][k];  // d W_out
    dz[nhid & 1][k] = g * Wo[k];
  }
  __syncthreads();
  // backward through the hidden layers
  for (int l = nhid - 1; l >= 0; --l) {
    const int wi = l == 0 ? fin : fh;
    off -= (int64_t)fh * wi + fh;
    const float *W = prm + off;
    const int cur = (l + 1) & 1, nxt = l & 1;
    for (int j = tid; j < fh; j += kT) {
      const float dp = dz[cur][j] * selu_d(pre[l][j]);
      pp[off + (int64_t)fh * wi + j] = dp;  // d b
      pre[l][j] = dp;                       // reuse: dpre
    }
    __syncthreads();
    for (int e = tid; e < fh * wi; e += kT) pp[off + e] = pre[l][e / wi] * z[l][e % wi];  // d W
    for (int k = tid; k < wi; k += kT) {
      float s = 0.0f;
      for (int j = 0; j < fh; ++j) s = fmaf(W[(int64_t)j * wi + k], pre[l][j], s);
      dz[nxt][k] = (residual && l > 0) ? s + dz[cur][k] : s;
    }
    __syncthreads();
  }
  for (int k = tid; k < fin; k += kT) {
    const float d = dz[0][k];
    if (k < lc) dcnn[(int64_t)p * lc + k] = d; else dsg[(int64_t)p * sgw + k - lc] = d;
  }
}

}  // namespace

// ---------------------------------------------------------------- launchers

hipError_t bw_fill(float *p, int64_t n, float v, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_fill, grid1(n), dim3(kT), 0, s, p, n, v);
  return hipGetLastError();
}
hipError_t bw_add(float *dst, const float *src, int64_t n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_add, grid1(n), dim3(kT), 0, s, dst, src, n);
  return hipGetLastError();
}
hipError_t bw_rowmat(const float *X, int ldx, int n, int K, const float *W, int ldw, const float *b, int J, float *Y,
                     int ldy, int accumulate, hipStream_t s) {
  if (n > 0 && J > 0)
    hipLaunchKernelGGL(k_rowmat<false>, dim3((n + 63) / 64, (J + 63) / 64), dim3(kT), 0, s, X, ldx, n, K, W, ldw, b, J, Y,
                       ldy, accumulate);
  return hipGetLastError();
}
hipError_t bw_rowmat_t(const float *X, int ldx, int n, int J, const float *W, int ldw, int K, float *Y, int ldy,
                       int accumulate, hipStream_t s) {
  if (n > 0 && K > 0)
    hipLaunchKernelGGL(k_rowmat<true>, dim3((n + 63) / 64, (K + 63) / 64), dim3(kT), 0, s, X, ldx, n, J, W, ldw, nullptr,
                       K, Y, ldy, accumulate);
  return hipGetLastError();
}
hipError_t bw_agg(const int32_t *rowp, const int32_t *col, int64_t cap, const float *S, int n, int F, float *A,
                  int accumulate, int64_t *status, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_agg, grid1((int64_t)n * F), dim3(kT), 0, s, rowp, col, cap, S, n, F, A, accumulate, status);
  return hipGetLastError();
}
hipError_t bw_gru_fwd(const float *GI, const float *GH, const float *Hin, int n, int H, float *Hout, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_gru_fwd, grid1((int64_t)n * H), dim3(kT), 0, s, GI, GH, Hin, n, H, Hout);
  return hipGetLastError();
}
hipError_t bw_gru_bwd(const float *GI, const float *GH, const float *Hin, const float *dHout, int n, int H, float *dGI,
                      float *dGH, float *dHd, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_gru_bwd, grid1((int64_t)n * H), dim3(kT), 0, s, GI, GH, Hin, dHout, n, H, dGI, dGH, dHd);
  return hipGetLastError();
}
hipError_t bw_readout(const float *Gpre, const float *V, const uint8_t *is_lig, const int32_t *atom_off, int p0,
                      int np, int H, float *S, hipStream_t s) {
  hipLaunchKernelGGL(k_readout, grid1((int64_t)np * H), dim3(kT), 0, s, Gpre, V, is_lig, atom_off, p0, np, H, S);
  return hipGetLastError();
}
hipError_t bw_readout_bwd(const float *Gpre, const float *V, const uint8_t *is_lig, const int32_t *atom_off, int p0,
                          int np, int H, int n_atoms, const float *dS, float *dGpre, float *dV, hipStream_t s) {
  if (n_atoms > 0)
    hipLaunchKernelGGL(k_readout_bwd, grid1((int64_t)n_atoms * H), dim3(kT), 0, s, Gpre, V, is_lig, atom_off, p0, np, H,
                       dS, dGpre, dV);
  return hipGetLastError();
}
int64_t bw_outer_scratch(int n, int A, int B) {
  return (int64_t)std::max(1, (n + kRowsPerChunk - 1) / kRowsPerChunk) * A * B;
}
hipError_t bw_outer(const float *U, int ldu, const float *V, int ldv, int n, int A, int B, float *C, int ldc,
                    int accumulate, float *part, hipStream_t s) {
  const int nchunk = std::max(1, (n + kRowsPerChunk - 1) / kRowsPerChunk);
  const int64_t ab = (int64_t)A * B;
  if (n > 0 && V)
    hipLaunchKernelGGL(k_outer_mfma, dim3((unsigned)((((A + 31) / 32) * ((B + 31) / 32) + 3) / 4), nchunk), dim3(kT), 0, s,
                       U, ldu, V, ldv, n, A, B, part);
  else if (n > 0)
    hipLaunchKernelGGL(k_outer_partial, dim3((unsigned)((ab + kT - 1) / kT), nchunk), dim3(kT), 0, s, U, ldu, n, A,
                       part);
  else
    hipLaunchKernelGGL(k_fill, grid1(ab), dim3(kT), 0, s, part, ab, 0.0f);
  if (nchunk >= 64 && ab <= 4096)
    hipLaunchKernelGGL(k_outer_sum_wave, dim3((unsigned)((ab + kT / 64 - 1) / (kT / 64))), dim3(kT), 0, s, part, nchunk, A,
                       B, C, ldc, accumulate);
  else
    hipLaunchKernelGGL(k_outer_sum, dim3((unsigned)((ab + kT - 1) / kT)), dim3(kT), 0, s, part, n > 0 ? nchunk : 1, A, B,
                       C, ldc, accumulate);
  return hipGetLastError();
}
hipError_t bw_pool_mean(const float *act, int np, int64_t vox, int cstride, int C, float *pool, hipStream_t s) {
  hipLaunchKernelGGL(k_pool_mean, dim3((C + 31) / 32, np), dim3(kPoolT), 0, s, act, vox, cstride, C, pool);
  return hipGetLastError();
}
hipError_t bw_pool_seed(const float *dpool, int np, int64_t vox, int cstride, int C, float *dact, hipStream_t s) {
  hipLaunchKernelGGL(k_pool_seed, grid1((int64_t)np * vox * cstride), dim3(kT), 0, s, dpool, np, vox, cstride, C, dact);
  return hipGetLastError();
}
hipError_t bw_relu_mask(float *d, const float *y, int64_t n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_relu_mask, grid1(n), dim3(kT), 0, s, d, y, n);
  return hipGetLastError();
}
hipError_t bw_relu_rows(float *y, int n, int J, int ld, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_relu_rows, grid1((int64_t)n * J), dim3(kT), 0, s, y, n, J, ld);
  return hipGetLastError();
}
hipError_t bw_relu_grad_rows(float *d, const float *pre, int n, int J, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_relu_grad_rows, grid1((int64_t)n * J), dim3(kT), 0, s, d, pre, n, J);
  return hipGetLastError();
}
int64_t bw_fold_wt_floats(int cout, int cin, int taps) {
  return (int64_t)taps * ((cout + 7) / 8) * ((cin + 31) / 32 * 32) * 8;
}
hipError_t bw_fold_wt(const float *W, const float *gamma, const float *var, int cout, int cin, int taps, float *WT,
                      hipStream_t s) {
  hipLaunchKernelGGL(k_fold_wt, grid1(bw_fold_wt_floats(cout, cin, taps)), dim3(kT), 0, s, W, gamma, var, cout, cin,
                     taps, (cout + 7) / 8, (cin + 31) / 32 * 32, WT);
  return hipGetLastError();
}
// row subsets per pose of the weight gradient: as many as nparts partials allow, while
// the launch has fewer workgroups than two per CU
int bw_conv_wgrad_split(int cin, int cout, int KS, int Do, int np, int nparts) {
  const int nb = (KS * cin + 31) / 32, ncg = (nb + 4) / 5, mb = cout <= 32 ? 1 : 2;
  const int64_t wg = (int64_t)KS * KS * ncg * ((cout + 32 * mb - 1) / (32 * mb)) * np;
  int split = 1;
  while (split < 8 && wg * split < 512 && (split * 2) * np <= nparts && split * 8 <= Do * Do) split *= 2;
  return split;
}
hipError_t bw_conv_wgrad(const float *X, int D, int xstride, int cin, const float *dY, int Do, int ystride, int cout,
                         int KS, int S, int np, int nsplit, float *part, hipStream_t s) {
  const int nb = (KS * cin + 31) / 32, ncg = (nb + 4) / 5, nbw = (nb + ncg - 1) / ncg;
  // voxels per run: even, two workgroups per CU (one needs a run of at most two voxels and
  // 256 channels to fit), X in its registers, and a row's runs alike
  const bool vec = (cin & 3) == 0 && (xstride & 3) == 0 && ((uintptr_t)X & 15) == 0;
  int run = std::min(wgrad_run(vec), (Do + 1) / 2 * 2);
  while (run > 2 && (wgrad_wave_floats(run, KS, S, cin) * 16 > 81920 ||
                     (S * (run - 1) + KS) * (vec ? cin / 4 : cin) > 64 * wgrad_xregs(vec)))
    run -= 2;
  const int nrun = (Do + run - 1) / run;
  run = ((Do + nrun - 1) / nrun + 1) / 2 * 2;
  const int wf = wgrad_wave_floats(run, KS, S, cin);
  const size_t lds = sizeof(float) * 4 * wf;
  if (lds > 163840) return hipErrorInvalidValue;
  const int mb = cout <= 32 ? 1 : 2;
  const dim3 grid(KS * KS * ncg, (cout + 32 * mb - 1) / (32 * mb), np * nsplit);
#define CF_WG(MB, NB) \
  do {                \
    if (vec) CF_WGV(MB, NB, true); else CF_WGV(MB, NB, false); \
  } while (0)
#define CF_WGV(MB, NB, V)                                                                                          \
  do {                                                                                                             \
    if (lds > 65536) {                                                                                             \
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_conv_wgrad<MB, NB, V>),              \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 163840);                \
      if (e != hipSuccess) return e;                                                                               \
    }                                                                                                              \
    hipLaunchKernelGGL((k_conv_wgrad<MB, NB, V>), grid, dim3(kT), lds, s, X, D, xstride, cin, dY, Do, ystride, cout,  \
                       KS, S, ncg, nsplit, run, wf, part);                                                              \
  } while (0)
  if (mb == 1) {
    if (nbw <= 3) CF_WG(1, 3); else CF_WG(1, 5);
  } else {
    if (nbw <= 3) CF_WG(2, 3); else CF_WG(2, 5);
  }
#undef CF_WG
#undef CF_WGV
  return hipGetLastError();
}
hipError_t bw_conv_dgrad(const float *dY, int Do, int ystride, int cout, const float *WT, int cin, int KS, int S, int D,
                         int xstride, int np, float *dX, hipStream_t s) {
  if (KS - 1 + kDT > kDHalo || ystride % 8) return hipErrorInvalidValue;
  const int ntl = ((D + S - 1) / S + kDT - 1) / kDT;
  hipLaunchKernelGGL(k_conv_dgrad, dim3(ntl * ntl * ntl, (cin + 63) / 64, np * S * S * S), dim3(kT), 0, s, dY, Do,
                     ystride, (cout + 7) / 8, WT, cin, (cin + 31) / 32 * 32, KS, S, D, xstride, dX);
  return hipGetLastError();
}
hipError_t bw_fold_grad(const float *dWf, const float *dbf, const float *W, const float *b, const float *gamma,
                        const float *mean, const float *var, int cout, int cin, int taps, float *gW, float *gb,
                        float *ggamma, float *gbeta, float *gmean, float *gvar, hipStream_t s) {
  hipLaunchKernelGGL(k_fold_grad, dim3(cout), dim3(kFoldT), 0, s, dWf, dbf, W, b, gamma, mean, var, cin, taps, gW, gb,
                     ggamma, gbeta, gmean, gvar);
  return hipGetLastError();
}
bool bw_head_ok(int fin, int fh, int nhid) { return fin <= kHeadMaxW && fh <= kHeadMaxW && nhid <= 8; }
hipError_t bw_head(const float *cnn, int lc, const float *sg, int sgw, const float *prm, int nhid, int fh, int residual,
                   const float *dscore, int np, float *scores, float *dcnn, float *dsg, float *part, int64_t nprm,
                   hipStream_t s) {
  hipLaunchKernelGGL(k_head_bwd, dim3(np), dim3(kT), 0, s, cnn, lc, sg, sgw, prm, nhid, fh, residual, dscore, scores,
                     dcnn, dsg, part, nprm);
  return hipGetLastError();
}

}  // namespace cf
