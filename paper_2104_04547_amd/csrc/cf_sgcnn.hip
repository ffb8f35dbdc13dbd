// SG-CNN forward: embedding, gated graph propagation and gated ligand readout.
//
// The paper's SG-CNN is PotentialNet built on gated graph sequence networks
// (Sec. 3.3.1, Table II): node states are propagated first over covalent edges
// (K_c rounds) and then over non-covalent edges (K_n rounds); each round sums
// the neighbours' states, applies a per-round message matrix and updates every
// state with a gated recurrent unit shared by the rounds of a stage; a gated sum
// over the ligand atoms ("gather") gives the latent that enters the fusion head.
//
// Design: a round is one launch over blocks of a pose's atoms (64 at width 64), so
// that a lone pose spreads over the chip and a batch's large poses do not outlast
// the rest; the states of all poses ping-pong between two buffers from launch to
// launch, and the workgroups of a pose are neighbours on one XCD, under one L2.  (One
// workgroup per pose walking its blocks round by round took 1.32 ms for one
// 690-atom pose, 2.9 ms for 200 poses of 200-1500 atoms and 4.8 ms for 33 poses of the
// staged plain form: its chain of dependent phases was the whole time.  Now 0.16, 0.56
// and 0.52 ms.)  The neighbour sums are segmented CSR reductions
// (consecutive lanes = consecutive features, so a neighbour row is one coalesced
// read) staged in LDS, then the message and GRU products run on the block.
//   * precision form (H = 32 or 64): the products run on the matrix cores as
//     v_mfma_f32_32x32x16_bf16 with every float32 operand split into a bfloat16
//     pair (hi + lo) and three products per term (hi*hi + hi*lo + lo*hi), float32
//     accumulation.  Single bfloat16 operands move the scores of this model by
//     ~0.1 pK; the split keeps ~16 mantissa bits.  Each wave owns a 32-atom x
//     32-feature tile of all six GRU gate products, so the gates, the state
//     update and the store happen straight from the accumulators.
//   * plain form: the same on the float32 matrix instruction (32x32x2); width 16,
//     which has no matrix-core tile, keeps one workgroup per pose with float32 FMAs
//     and the weights in LDS.
#include <algorithm>
#include <utility>

#include "cf_internal.h"

namespace cf {

namespace {

constexpr int kThreads = 256;

// 1 / d for d >= 1: the hardware's reciprocal and one Newton step, which is the correctly
// rounded quotient for every float in [1, 2^126) (all of them compared), in four
// instructions instead of a division's eleven.  Beyond, where the quotient is subnormal,
// it is 0.
__device__ inline float recip_ge1(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r), d, 1.0f);
}
__device__ inline float sigm(float x) { return recip_ge1(1.0f + expf(-x)); }

// ---- shared pieces ------------------------------------------------------------

// h = W_e x + b_e for the pose's atoms (float32)
template <int H>
__device__ inline void sg_embed(const SgWeights &W, const float *__restrict__ feat, int a0, int n, int64_t lb,
                                float *h0) {
  for (int e = threadIdx.x; e < n * H; e += kThreads) {
    const int i = e / H, oo = e % H;
    const float *x = feat + (int64_t)(a0 + i) * CF_NCH;
    float v = W.embed_b[oo];
    for (int c = 0; c < CF_NCH; ++c) v += W.embed_wT[c * H + oo] * x[c];
    h0[(lb + i) * H + oo] = v;
  }
}

// Neighbour sums of atoms [blk, blk+nblk) into A (row stride ld) and their current
// states into Hc; rows past the pose are zero.  Each thread owns four consecutive
// features of a row (one 16-byte load per neighbour row segment) and H / 4 threads
// share a row.  The block's CSR rows are consecutive, so their columns form one
// contiguous range: it is staged in LDS (idx, up to icap entries, as row numbers in the
// pose; a thread with rows beyond that reads columns from memory) with coalesced loads, and every thread then walks NU
// of the block's rows at once (OVER: idx lies where Hc goes; nblk <= NU * kThreads / (H / 4)), kSlots neighbours
// per row per step, so that up to 4 NU row loads are in flight with no index load
// in front of them.  Every feature's sum runs over the row's neighbours in CSR order.
template <int H, int NU, bool OVER = false>
__device__ inline void sg_aggregate(const float *__restrict__ cur, const int32_t *__restrict__ rowp,
                                    const int32_t *__restrict__ colp, int64_t cap, int csr_global, int a0, int base,
                                    int64_t lb, int n, int blk, int nblk, int ld, float *A, float *Hc, int32_t *idx,
                                    int icap, int64_t *status) {
  constexpr int TPR = H / 4;              // threads per row
  constexpr int RPI = kThreads / TPR;     // rows per pass
  constexpr int kSlots = 4;               // neighbours per row per step
  static_assert(H % 4 == 0 && kThreads % TPR == 0, "row split");
  const int tr = threadIdx.x / TPR, c4 = (threadIdx.x % TPR) * 4;
  const int nrow = min(nblk, n - blk);  // rows of the pose in this block (>= 1)
  const int64_t rb = csr_global ? (int64_t)a0 + blk : lb + blk;
  // this thread's rows and their edge ranges (empty for rows past the block)
  int64_t e0[NU], e1[NU];
  int64_t E0 = rowp[rb], E1 = rowp[rb + nrow];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int a = tr + RPI * u;
    e0[u] = e1[u] = 0;
    if (a < nrow) {
      e0[u] = rowp[rb + a];
      e1[u] = rowp[rb + a + 1];
    }
  }
  E1 = E1 < cap ? E1 : cap;
  const int64_t nst = E0 < 0 || E1 <= E0 ? 0 : (E1 - E0 < icap ? E1 - E0 : icap);
  // staged in batches of kStage loads per thread, all in flight together
  constexpr int kStage = 4;
  for (int64_t e0 = 0; e0 < nst; e0 += kStage * kThreads) {
    int32_t cv[kStage];
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
      const int64_t e = e0 + u * kThreads + threadIdx.x;
      cv[u] = e < nst ? colp[E0 + e] : 0;
    }
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
      const int64_t e = e0 + u * kThreads + threadIdx.x;
      if (e < nst) {
        // the neighbour's row in the pose, -1 for one outside of it
        const int64_t j = (csr_global ? (int64_t)cv[u] - base : (int64_t)cv[u]) - lb;
        idx[e] = j >= 0 && j < n ? (int32_t)j : -1;
      }
    }
  }
  bool anybad = false;
  int64_t len = 0;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    if (e1[u] > cap) e1[u] = cap;
    if (e0[u] < 0) {
      anybad = true;
      e0[u] = e1[u];
    }
    len = e1[u] - e0[u] > len ? e1[u] - e0[u] : len;
  }
  __syncthreads();
  float4 s[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) s[u] = make_float4(0.f, 0.f, 0.f, 0.f);
  // Whole steps with a branch-free body: slots past a row's end and neighbours outside
  // the pose read the row's own state (the pose's first row for rows past the block) and
  // add nothing; a bad neighbour is reported once after the loop.  Where the rows lie
  // within the staged range, indices and offsets are 32 bits wide: a step's index work in
  // 64 bits was two fifths of the round's vector instructions (200 ragged poses at width
  // 64: 112 us a round, now 91).
  bool staged = true;
#pragma unroll
  for (int u = 0; u < NU; ++u) staged &= e0[u] >= e1[u] || (e0[u] >= E0 && e1[u] <= E0 + nst);
  if (staged) {
    const float *rows = cur + lb * H;
    int q0[NU], cnt[NU], self[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int a = tr + RPI * u;
      cnt[u] = e1[u] > e0[u] ? (int)(e1[u] - e0[u]) : 0;
      q0[u] = cnt[u] ? (int)(e0[u] - E0) : 0;
      self[u] = a < nrow ? blk + a : 0;
    }
    const int last = nst > 0 ? (int)nst - 1 : 0;
    for (int k = 0; k < (int)len; k += kSlots) {
      float4 v[NU][kSlots];
      bool use[NU][kSlots];
      int j[NU][kSlots];
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int w = 0; w < kSlots; ++w) j[u][w] = idx[min(q0[u] + k + w, last)];
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int w = 0; w < kSlots; ++w) {
          const bool live = k + w < cnt[u];
          use[u][w] = live && j[u][w] >= 0;
          anybad |= live && j[u][w] < 0;
          v[u][w] = *reinterpret_cast<const float4 *>(rows + (uint32_t)((use[u][w] ? j[u][w] : self[u]) * H + c4));
        }
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int w = 0; w < kSlots; ++w) {
          s[u].x += use[u][w] ? v[u][w].x : 0.0f;
          s[u].y += use[u][w] ? v[u][w].y : 0.0f;
          s[u].z += use[u][w] ? v[u][w].z : 0.0f;
          s[u].w += use[u][w] ? v[u][w].w : 0.0f;
        }
    }
  } else {
    for (int64_t k = 0; k < len; k += kSlots) {
      float4 v[NU][kSlots];
      bool use[NU][kSlots];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int a = tr + RPI * u;
        const int64_t self = lb + (a < nrow ? blk + a : 0);
#pragma unroll
        for (int w = 0; w < kSlots; ++w) {
          const int64_t q = e0[u] + k + w;
          const bool live = q < e1[u];
          int64_t c = 0;
          if (live) c = colp[q];
          const int64_t j = csr_global ? c - base : c;
          const bool bad = j < lb || j >= lb + n;
          anybad |= live && bad;
          use[u][w] = live && !bad;
          v[u][w] = *reinterpret_cast<const float4 *>(cur + (use[u][w] ? j : self) * H + c4);
        }
      }
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int w = 0; w < kSlots; ++w) {
          s[u].x += use[u][w] ? v[u][w].x : 0.0f;
          s[u].y += use[u][w] ? v[u][w].y : 0.0f;
          s[u].z += use[u][w] ? v[u][w].z : 0.0f;
          s[u].w += use[u][w] ? v[u][w].w : 0.0f;
        }
    }
  }
  if (anybad) dev_fail(status, kDevBadGraph);
  if constexpr (OVER) __syncthreads();  // the staged rows are read, Hc lies over them
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int a = tr + RPI * u;
    if (a < nblk) {
      const float4 hc = a < nrow ? *reinterpret_cast<const float4 *>(cur + (lb + blk + a) * H + c4)
                                 : make_float4(0.f, 0.f, 0.f, 0.f);
      *reinterpret_cast<float4 *>(A + a * ld + c4) = s[u];
      *reinterpret_cast<float4 *>(Hc + a * ld + c4) = hc;
    }
  }
}

// s = sum over ligand atoms of sigmoid(W_g [h; x] + b_g) * (W_v h + b_v), float32.
// Wg, Wv: LDS copies of the transposed readout weights; red: >= kThreads floats.
template <int H>
__device__ inline void sg_readout(const SgWeights &W, const float *__restrict__ cur, const float *__restrict__ feat,
                                  const uint8_t *__restrict__ is_lig, int a0, int n, int64_t lb, const float *Wg,
                                  const float *Wv, float *red, float *out) {
  constexpr int G = kThreads / H;
  const int o = threadIdx.x % H, g = threadIdx.x / H;
  float acc = 0.0f;
  for (int i = g; i < n; i += G) {
    if (!is_lig[a0 + i]) continue;
    const float *hi = cur + (lb + i) * H;
    const float *xi = feat + (int64_t)(a0 + i) * CF_NCH;
    float gt = W.gate_b[o], vl = W.val_b[o];
    for (int k = 0; k < H; ++k) {
      const float hk = hi[k];
      gt += Wg[k * H + o] * hk;
      vl += Wv[k * H + o] * hk;
    }
    for (int c = 0; c < CF_NCH; ++c) gt += Wg[(H + c) * H + o] * xi[c];
    acc += sigm(gt) * vl;
  }
  red[g * H + o] = acc;
  __syncthreads();
  if ((int)threadIdx.x < H) {
    float s = 0.0f;
    for (int q = 0; q < G; ++q) s += red[q * H + threadIdx.x];
    out[threadIdx.x] = s;
  }
}

// ---- plain form: float32 on the vector ALUs ----------------------------------

constexpr int kBlk = 32;  // atoms per block (plain form)

template <int H>
struct SgShared {
  float Wt[H * H];
  float Wih[H * 3 * H];
  float Whh[H * 3 * H];
  float A[kBlk * H];
  float M[kBlk * H];
  float Hc[kBlk * H];
  // staged neighbours: 64 a row, an area of its own (in M, 16 a row at width 16, half of a
  // block's rows read their columns from memory: four 4096-atom poses took 1.70 ms, now 1.16)
  int32_t idx[kBlk * 64];
};

template <int H>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(H >= 32 ? 3 : 2))) void k_sgcnn_f32(SgWeights W, const int32_t *__restrict__ atom_off,
                                                        int n_atoms, const float *__restrict__ feat,
                                                        const uint8_t *__restrict__ is_lig, int p0,
                                                        const int32_t *__restrict__ cov_row,
                                                        const int32_t *__restrict__ cov_col, int64_t cov_cap,
                                                        const int32_t *__restrict__ nc_row,
                                                        const int32_t *__restrict__ nc_col, int64_t nc_cap,
                                                        int csr_global, float *__restrict__ hbuf, int64_t hcap,
                                                        float *__restrict__ sg_latent, int64_t *__restrict__ status) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  SgShared<H> &S = *reinterpret_cast<SgShared<H> *>(smem_raw);
  constexpr int G = kThreads / H;  // thread groups (one output feature per thread)
  constexpr int APT = kBlk / G;    // atoms per thread in a block
  const int t = threadIdx.x;
  const int o = t % H, g = t / H;
  const int pl = blockIdx.x;
  const int base = atom_off[p0];
  int a0, a1;
  const bool ok = pose_range(atom_off, p0 + pl, n_atoms, a0, a1);
  const int n = a1 - a0;
  const int64_t lb = (int64_t)a0 - base;
  if (!ok || n <= 0 || lb < 0 || lb + n > hcap) {
    if (t == 0 && (!ok || lb < 0 || lb + n > hcap)) dev_fail(status, kDevBadOffsets);
    if (t < H) sg_latent[(int64_t)pl * H + t] = 0.0f;
    return;
  }
  float *h0 = hbuf, *h1 = hbuf + hcap * H;
  sg_embed<H>(W, feat, a0, n, lb, h0);
  __threadfence();
  __syncthreads();

  float *cur = h0, *nxt = h1;
  const int rounds = W.K_c + W.K_n;
  for (int r = 0; r < rounds; ++r) {
    const int stage = r < W.K_c ? 0 : 1;
    const int32_t *rowp = stage ? nc_row : cov_row;
    const int32_t *colp = stage ? nc_col : cov_col;
    const int64_t cap = stage ? nc_cap : cov_cap;
    for (int e = t; e < H * H; e += kThreads) S.Wt[e] = W.msgT[r][e];
    if (r == 0 || r == W.K_c) {
      for (int e = t; e < 3 * H * H; e += kThreads) {
        S.Wih[e] = W.w_ihT[stage][e];
        S.Whh[e] = W.w_hhT[stage][e];
      }
    }
    const float *bih = W.b_ih[stage], *bhh = W.b_hh[stage];
    __syncthreads();
    for (int blk = 0; blk < n; blk += kBlk) {
      sg_aggregate<H, (kBlk + 4 * kThreads / H - 1) / (4 * kThreads / H)>(cur, rowp, colp, cap, csr_global, a0, base, lb, n, blk, kBlk, H, S.A, S.Hc,
                      S.idx, kBlk * 64, status);
      __syncthreads();
      // messages m = W_t a
      {
        float acc[APT];
#pragma unroll
        for (int u = 0; u < APT; ++u) acc[u] = 0.0f;
        for (int k = 0; k < H; ++k) {
          const float w = S.Wt[k * H + o];
#pragma unroll
          for (int u = 0; u < APT; ++u) acc[u] += w * S.A[(g * APT + u) * H + k];
        }
#pragma unroll
        for (int u = 0; u < APT; ++u) S.M[(g * APT + u) * H + o] = acc[u];
      }
      __syncthreads();
      // GRU update
      {
        float ir[APT], iz[APT], in_[APT], hr[APT], hz[APT], hn[APT];
#pragma unroll
        for (int u = 0; u < APT; ++u) {
          ir[u] = bih[o];
          iz[u] = bih[H + o];
          in_[u] = bih[2 * H + o];
          hr[u] = bhh[o];
          hz[u] = bhh[H + o];
          hn[u] = bhh[2 * H + o];
        }
        for (int k = 0; k < H; ++k) {
          const float wir = S.Wih[k * 3 * H + o], wiz = S.Wih[k * 3 * H + H + o], win = S.Wih[k * 3 * H + 2 * H + o];
          const float whr = S.Whh[k * 3 * H + o], whz = S.Whh[k * 3 * H + H + o], whn = S.Whh[k * 3 * H + 2 * H + o];
#pragma unroll
          for (int u = 0; u < APT; ++u) {
            const float m = S.M[(g * APT + u) * H + k];
            const float hk = S.Hc[(g * APT + u) * H + k];
            ir[u] += wir * m;
            iz[u] += wiz * m;
            in_[u] += win * m;
            hr[u] += whr * hk;
            hz[u] += whz * hk;
            hn[u] += whn * hk;
          }
        }
#pragma unroll
        for (int u = 0; u < APT; ++u) {
          const int a = g * APT + u;
          const int i = blk + a;
          if (i < n) {
            const float rr = sigm(ir[u] + hr[u]);
            const float zz = sigm(iz[u] + hz[u]);
            const float nn = tanhf(in_[u] + rr * hn[u]);
            nxt[(lb + i) * H + o] = (1.0f - zz) * nn + zz * S.Hc[a * H + o];
          }
        }
      }
      __syncthreads();
    }
    __threadfence();
    __syncthreads();
    float *tmp = cur;
    cur = nxt;
    nxt = tmp;
  }
  // readout (weights staged in the GRU areas)
  for (int e = t; e < (H + CF_NCH) * H; e += kThreads) S.Wih[e] = W.gate_wT[e];
  for (int e = t; e < H * H; e += kThreads) S.Whh[e] = W.val_wT[e];
  __syncthreads();
  sg_readout<H>(W, cur, feat, is_lig, a0, n, lb, S.Wih, S.Whh, S.A, sg_latent + (int64_t)pl * H);
}

// ---- precision form: split-bfloat16 MFMA --------------------------------------

typedef float f32x16v __attribute__((ext_vector_type(16)));

// hi/lo bfloat16 split of 8 consecutive floats
__device__ inline void split8(const float *p, bf16x8 &hi, bf16x8 &lo) {
  const float4 a = *reinterpret_cast<const float4 *>(p);
  const float4 b = *reinterpret_cast<const float4 *>(p + 4);
  const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const bf16_t h = (bf16_t)v[q];
    hi[q] = h;
    lo[q] = (bf16_t)(v[q] - (float)h);
  }
}

__device__ inline f32x16v mfma3(const bf16x8 &ah, const bf16x8 &al, const bf16x8 &bh, const bf16x8 &bl, f32x16v c) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, c, 0, 0, 0);
  return c;
}

// Tile of one stage at width H: each of the four waves owns a 32-atom x 32-feature
// tile of the block (FB feature blocks x MBK atom blocks); rows padded to LD.
template <int H>
struct SgTile {
  static constexpr int LD = H + 4;      // padded row stride (floats)
  static constexpr int FB = H / 32;     // 32-feature blocks
  static constexpr int MBK = 4 / FB;    // 32-atom blocks per workgroup block
  static constexpr int BLK = 32 * MBK;  // atoms per block
  static_assert(H % 32 == 0 && H <= 128, "matrix-core widths are 32, 64 or 128");
};

// LDS of a round: A | M (first the staged rows) | Hc, or in two regions (A, then M | the
// staged rows, then Hc) for two more barriers.  Two pay at width 32 in the split form,
// where they let three workgroups run on a CU in place of two (96 poses of the paper's
// model, covalent stage: 66 -> 58 us a round); at width 64 three run either way and the
// barriers cost 9 %.
template <int H, bool F32>
constexpr bool sg_two_regions() {
  return H == 32 && !F32;
}
template <int H, bool F32>
constexpr int sg_lds_floats() {
  return (sg_two_regions<H, F32>() ? 2 : 3) * SgTile<H>::BLK * SgTile<H>::LD;
}

// acc += A[row][0..K) W^T for this lane's output column `col` of N, W given as
// split-bfloat16 MFMA B operands ([K/16][N][16], hi and lo) -- three products per
// term -- or, for the plain form, as float32 W^T [K][N] on the 32x32x2 float32
// matrix instruction.
template <int K, bool F32>
__device__ inline f32x16v mm_row(const float *arow, const bf16_t *bhi, const bf16_t *blo, const float *bT, int N,
                                 int col, int khalf, f32x16v acc) {
  if constexpr (F32) {
#pragma unroll 8
    for (int k = 0; k < K; k += 2)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(arow[k + khalf], bT[(int64_t)(k + khalf) * N + col], acc, 0, 0, 0);
  } else {
#pragma unroll
    for (int ks = 0; ks < K / 16; ++ks) {
      bf16x8 ah, al;
      split8(arow + ks * 16 + khalf * 8, ah, al);
      const int64_t wo = ((int64_t)ks * N + col) * 16 + khalf * 8;
      acc = mfma3(ah, al, *reinterpret_cast<const bf16x8 *>(bhi + wo), *reinterpret_cast<const bf16x8 *>(blo + wo),
                  acc);
    }
  }
  return acc;
}

// One round of one stage at width H for the atoms [blk, blk + BLK) of a pose:
// neighbour sums of the current states (cur), the round's message product, the
// stage's GRU, the new states of those atoms written to nxt (row stride H).
// SEP (plain form without staging): the gates' input and hidden parts in accumulators of
// their own that start at the biases -- with k in ascending order and the matrix
// instruction adding its two products in turn, bit for bit the sums of plain fused
// multiply-adds, which sit closer to the 64-bit states than the merged accumulators.
template <int H, bool F32, bool SEP>
__device__ void sg_block(const SgWeights &W, int stage, int r, const int32_t *__restrict__ rowp,
                         const int32_t *__restrict__ colp, int64_t cap, int csr_global, int a0, int base, int64_t lb,
                         int n, int blk, const float *cur, float *nxt, float *lds, int64_t *status) {
  using T = SgTile<H>;
  constexpr int LD = T::LD, BLK = T::BLK;
  static_assert(BLK % (4 * kThreads / H) == 0, "whole rows per thread in the neighbour sums");
  constexpr bool TWO = sg_two_regions<H, F32>();
  float *A = lds, *M = TWO ? lds : lds + BLK * LD, *Hc = lds + (TWO ? 1 : 2) * BLK * LD;
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int mb = wave / T::FB, fb = wave % T::FB;  // this wave's 32-atom x 32-feature tile
  const int lrow = lane & 31, khalf = lane >> 5;
  const int ocol = fb * 32 + lrow;  // output feature of this lane's accumulator column
  const float *bih = W.b_ih[stage], *bhh = W.b_hh[stage];
  const float bir = bih[ocol], biz = bih[H + ocol], bin = bih[2 * H + ocol];
  const float bhr = bhh[ocol], bhz = bhh[H + ocol], bhn = bhh[2 * H + ocol];
    sg_aggregate<H, BLK / (4 * kThreads / H), TWO>(cur, rowp, colp, cap, csr_global, a0, base, lb, n, blk, BLK, LD, A, Hc,
                  reinterpret_cast<int32_t *>(TWO ? Hc : M), BLK * LD, status);
    __syncthreads();
    // messages: M[atoms, ocol] = sum_k A[atoms, k] W_t[ocol, k]
    {
      f32x16v acc = {};
      acc = mm_row<H, F32>(&A[(mb * 32 + lrow) * LD], W.msg_hi[r], W.msg_lo[r], W.msgT[r], H, ocol, khalf, acc);
      if constexpr (TWO) __syncthreads();  // A is read, M takes its place
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int row = mb * 32 + 8 * (j >> 2) + 4 * khalf + (j & 3);
        M[row * LD + ocol] = acc[j];
      }
    }
    __syncthreads();
    // GRU gates for this wave's tile: the reset and update gates accumulate their
    // input and hidden products in one accumulator each; the candidate keeps them
    // apart (the reset gate scales only the hidden part)
    {
      f32x16v gr = {}, gz = {}, gin = {}, ghn = {}, hr = {}, hz = {};
      const float *mrow = &M[(mb * 32 + lrow) * LD], *hrow = &Hc[(mb * 32 + lrow) * LD];
      if constexpr (F32) {
        const float *wi = W.w_ihT[stage], *wh = W.w_hhT[stage];
        if constexpr (SEP) {
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            gr[j] = bir;
            gz[j] = biz;
            gin[j] = bin;
            hr[j] = bhr;
            hz[j] = bhz;
            ghn[j] = bhn;
          }
          hr = mm_row<H, true>(hrow, nullptr, nullptr, wh, 3 * H, ocol, khalf, hr);
          hz = mm_row<H, true>(hrow, nullptr, nullptr, wh, 3 * H, H + ocol, khalf, hz);
        }
        gr = mm_row<H, true>(mrow, nullptr, nullptr, wi, 3 * H, ocol, khalf, gr);
        if constexpr (!SEP) gr = mm_row<H, true>(hrow, nullptr, nullptr, wh, 3 * H, ocol, khalf, gr);
        gz = mm_row<H, true>(mrow, nullptr, nullptr, wi, 3 * H, H + ocol, khalf, gz);
        if constexpr (!SEP) gz = mm_row<H, true>(hrow, nullptr, nullptr, wh, 3 * H, H + ocol, khalf, gz);
        gin = mm_row<H, true>(mrow, nullptr, nullptr, wi, 3 * H, 2 * H + ocol, khalf, gin);
        ghn = mm_row<H, true>(hrow, nullptr, nullptr, wh, 3 * H, 2 * H + ocol, khalf, ghn);
      } else {
        const bf16_t *ih = W.ih_hi[stage], *il = W.ih_lo[stage], *hh = W.hh_hi[stage], *hl = W.hh_lo[stage];
        constexpr int kUnroll = H <= 64 ? H / 16 : 2;  // wider: bounded unroll keeps it in registers
#pragma unroll kUnroll
        for (int ks = 0; ks < H / 16; ++ks) {
          bf16x8 mhi, mlo, hhi, hlo;
          split8(mrow + ks * 16 + khalf * 8, mhi, mlo);
          split8(hrow + ks * 16 + khalf * 8, hhi, hlo);
          const int64_t w0 = ((int64_t)ks * 3 * H + ocol) * 16 + khalf * 8;
          const int64_t gs = (int64_t)H * 16;  // next gate's rows
          gr = mfma3(mhi, mlo, *reinterpret_cast<const bf16x8 *>(ih + w0), *reinterpret_cast<const bf16x8 *>(il + w0), gr);
          gr = mfma3(hhi, hlo, *reinterpret_cast<const bf16x8 *>(hh + w0), *reinterpret_cast<const bf16x8 *>(hl + w0), gr);
          gz = mfma3(mhi, mlo, *reinterpret_cast<const bf16x8 *>(ih + w0 + gs), *reinterpret_cast<const bf16x8 *>(il + w0 + gs), gz);
          gz = mfma3(hhi, hlo, *reinterpret_cast<const bf16x8 *>(hh + w0 + gs), *reinterpret_cast<const bf16x8 *>(hl + w0 + gs), gz);
          gin = mfma3(mhi, mlo, *reinterpret_cast<const bf16x8 *>(ih + w0 + 2 * gs), *reinterpret_cast<const bf16x8 *>(il + w0 + 2 * gs), gin);
          ghn = mfma3(hhi, hlo, *reinterpret_cast<const bf16x8 *>(hh + w0 + 2 * gs), *reinterpret_cast<const bf16x8 *>(hl + w0 + 2 * gs), ghn);
        }
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int row = mb * 32 + 8 * (j >> 2) + 4 * khalf + (j & 3);
        const int i = blk + row;
        if (i < n) {
          const float rr = SEP ? sigm(gr[j] + hr[j]) : sigm(gr[j] + (bir + bhr));
          const float zz = SEP ? sigm(gz[j] + hz[j]) : sigm(gz[j] + (biz + bhz));
          const float nn = SEP ? tanhf(gin[j] + rr * ghn[j]) : tanhf(gin[j] + bin + rr * (ghn[j] + bhn));
          nxt[(lb + i) * H + ocol] = (1.0f - zz) * nn + zz * Hc[row * LD + ocol];
        }
      }
    }
    __syncthreads();
}

// The pose of work item `it` of n_poses * nbx (pose-major, renumbered so that the
// items of a pose run on one XCD): its first block of atoms, its atom range and its
// first row lb in the state buffers.  False (nothing to do) for an empty or malformed
// pose, which is reported when `report` is set.
__device__ inline bool sg_item(const int32_t *__restrict__ atom_off, int n_atoms, int p0, int nbx, int64_t hcap,
                               bool report, int &pl, int &b0, int &a0, int &n, int &base, int64_t &lb,
                               int64_t *status) {
  int x, y, z;
  xcd_order(x, y, z);
  pl = x / nbx;
  b0 = x % nbx;
  base = atom_off[p0];
  int a1;
  const bool ok = pose_range(atom_off, p0 + pl, n_atoms, a0, a1);
  n = a1 - a0;
  lb = (int64_t)a0 - base;
  const bool bad = !ok || lb < 0 || lb + n > hcap;
  if (bad && report && b0 == 0 && threadIdx.x == 0) dev_fail(status, kDevBadOffsets);
  return !bad && n > 0;
}

constexpr int kEmbedRows = 32;  // atoms per workgroup of the embedding and the covalent gather

template <int H>
__global__ __launch_bounds__(kThreads) void k_sg_embed(SgWeights W, const int32_t *__restrict__ atom_off, int n_atoms,
                                                       const float *__restrict__ feat, int p0, int nbx,
                                                       float *__restrict__ h0, int64_t hcap,
                                                       int64_t *__restrict__ status) {
  int pl, b0, a0, n, base;
  int64_t lb;
  if (!sg_item(atom_off, n_atoms, p0, nbx, hcap, true, pl, b0, a0, n, base, lb, status)) return;
  // h = W_e x + b_e as sg_embed, a thread's feature column in registers and the atoms' rows
  // in LDS: with both read per product, 38 loads per value filled the L1's address
  // pipeline (200 ragged poses at width 64: 33 us, now 18)
  constexpr int XP = (CF_NCH + 3) / 4 * 4;
  __shared__ __attribute__((aligned(16))) float xs[kEmbedRows * XP];
  const int o = threadIdx.x % H, g = threadIdx.x / H;
  float w[CF_NCH];
#pragma unroll
  for (int c = 0; c < CF_NCH; ++c) w[c] = W.embed_wT[c * H + o];
  const float b = W.embed_b[o];
  for (int blk = b0 * kEmbedRows; blk < n; blk += nbx * kEmbedRows) {
    const int nr = min(kEmbedRows, n - blk);
    __syncthreads();
    for (int e = threadIdx.x; e < nr * CF_NCH; e += kThreads)
      xs[e / CF_NCH * XP + e % CF_NCH] = feat[(int64_t)(a0 + blk) * CF_NCH + e];
    __syncthreads();
    for (int i = g; i < nr; i += kThreads / H) {
      const float *x = xs + i * XP;
      float v = b;
#pragma unroll
      for (int c = 0; c < CF_NCH; ++c) v += w[c] * x[c];
      h0[(lb + blk + i) * H + o] = v;
    }
  }
}

// One round: the states of cur advanced into nxt.
template <int H, bool F32, bool SEP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(H == 128 || F32 ? 2 : 3))) void k_sg_round(
    SgWeights W, int stage, int r, const int32_t *__restrict__ atom_off, int n_atoms, int p0, int nbx,
    const int32_t *__restrict__ rowp, const int32_t *__restrict__ colp, int64_t cap, int csr_global,
    const float *__restrict__ cur, float *__restrict__ nxt, int64_t hcap, int64_t *__restrict__ status) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  int pl, b0, a0, n, base;
  int64_t lb;
  if (!sg_item(atom_off, n_atoms, p0, nbx, hcap, false, pl, b0, a0, n, base, lb, status)) return;
  for (int blk = b0 * SgTile<H>::BLK; blk < n; blk += nbx * SgTile<H>::BLK)
    sg_block<H, F32, SEP>(W, stage, r, rowp, colp, cap, csr_global, a0, base, lb, n, blk, cur, nxt, lds, status);
}

// ---- PotentialNet staging: the covalent stage at width HC closes with a per-atom
// gather, g_i = sigmoid(W_g1 [h_i; x_i] + b) * (W_v1 h_i + b_v1), and a linear
// embedding to width HN, h_i = W_e2 g_i + b; the readout's gate reads [h; g].  Small
// per-atom work: float32 FMAs with the weights read through the caches. ----
template <int HC, int HN>
__global__ __launch_bounds__(kThreads) void k_sg_mid(SgWeights W, const int32_t *__restrict__ atom_off, int n_atoms,
                                                     const float *__restrict__ feat, int p0, int nbx,
                                                     const float *__restrict__ cur, float *__restrict__ gb,
                                                     float *__restrict__ h2, int64_t hcap,
                                                     int64_t *__restrict__ status) {
  __shared__ float g[kEmbedRows * HC];
  int pl, b0, a0, n, base;
  int64_t lb;
  if (!sg_item(atom_off, n_atoms, p0, nbx, hcap, false, pl, b0, a0, n, base, lb, status)) return;
  for (int blk = b0 * kEmbedRows; blk < n; blk += nbx * kEmbedRows) {
    const int nr = min(kEmbedRows, n - blk);
    for (int e = threadIdx.x; e < nr * HC; e += kThreads) {
      const int i = e / HC, o = e % HC;
      const float *hi = cur + (lb + blk + i) * HC;
      const float *xi = feat + (int64_t)(a0 + blk + i) * CF_NCH;
      float gt = W.mid_gate_b[o], vl = W.mid_val_b[o];
#pragma unroll 8
      for (int k = 0; k < HC; ++k) {
        const float hk = hi[k];
        gt += W.mid_gate_wT[k * HC + o] * hk;
        vl += W.mid_val_wT[k * HC + o] * hk;
      }
      for (int c = 0; c < CF_NCH; ++c) gt += W.mid_gate_wT[(HC + c) * HC + o] * xi[c];
      const float gv = sigm(gt) * vl;
      gb[(lb + blk + i) * HC + o] = gv;
      g[e] = gv;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < nr * HN; e += kThreads) {
      const int i = e / HN, o = e % HN;
      float v = W.embed2_b[o];
#pragma unroll 8
      for (int k = 0; k < HC; ++k) v += W.embed2_wT[k * HN + o] * g[i * HC + k];
      h2[(lb + blk + i) * HN + o] = v;
    }
    __syncthreads();
  }
}

// Gated readout, one workgroup per pose: s = sum over ligand atoms of
// sigmoid(W_g [h; u] + b_g) * (W_v h + b_v), u the atom's U raw features (row stride
// U) or its covalent gather.  The threads form G groups of H; group g sums the
// ligand atoms i = g mod G in ascending order, then the groups are added in order.  The
// ligand atoms are listed per group first (a pose has a few dozen in hundreds), and a
// thread takes four of its group's atoms together, so that a weight is read once for
// four of them.
template <int H, int U>
__global__ __launch_bounds__(kThreads) void k_sg_readout(SgWeights W, const int32_t *__restrict__ atom_off,
                                                         int n_atoms, const float *__restrict__ cur,
                                                         const float *__restrict__ u, int u_local,
                                                         const uint8_t *__restrict__ is_lig, int p0, int64_t hcap,
                                                         float *__restrict__ sg_latent) {
  constexpr int G = kThreads / H, NA = 4, WAVES = kThreads / 64;
  static_assert(64 % G == 0, "a wave holds whole turns of the groups");
  __shared__ uint16_t list[G][CF_MAX_POSE_ATOMS / G];
  __shared__ int cnt[WAVES][G];
  __shared__ float red[kThreads];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int pl = blockIdx.x;
  const int base = atom_off[p0];
  float *out = sg_latent + (int64_t)pl * H;
  int a0, a1;
  const bool ok = pose_range(atom_off, p0 + pl, n_atoms, a0, a1);
  const int n = a1 - a0;
  const int64_t lb = (int64_t)a0 - base;
  if (!ok || n <= 0 || lb < 0 || lb + n > hcap) {
    if (t < H) out[t] = 0.0f;
    return;
  }
  unsigned long long turn = 0;
#pragma unroll
  for (int q = 0; q < 64; q += G) turn |= 1ull << q;
  const int lg = lane % G;
  int run = 0;  // atoms listed so far for group lg
  for (int c0 = 0; c0 < n; c0 += kThreads) {
    const int i = c0 + t;
    const bool lig = i < n && is_lig[a0 + i];
    const unsigned long long m = __ballot(lig) & (turn << lg);
    if (lane < G) cnt[wave][lane] = __popcll(m);
    __syncthreads();
    int at = run;
    for (int w = 0; w < WAVES; ++w) {
      const int k = cnt[w][lg];
      if (w < wave) at += k;
      run += k;
    }
    if (lig) list[lg][at + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)i;
    __syncthreads();
  }
  if (t < G) cnt[0][t] = run;  // thread t < G holds the total of group t
  __syncthreads();
  const int o = t % H, g = t / H;
  const int total = cnt[0][g];
  float acc = 0.0f;
  for (int q0 = 0; q0 < total; q0 += NA) {
    const float *hi[NA], *ui[NA];
    float gt[NA], vl[NA];
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int i = list[g][min(q0 + q, total - 1)];
      hi[q] = cur + (lb + i) * H;
      ui[q] = u + (u_local ? lb + i : (int64_t)(a0 + i)) * U;
      gt[q] = W.gate_b[o];
      vl[q] = W.val_b[o];
    }
#pragma unroll 8
    for (int k = 0; k < H; ++k) {
      const float wg = W.gate_wT[k * H + o], wv = W.val_wT[k * H + o];
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        const float hk = hi[q][k];
        gt[q] += wg * hk;
        vl[q] += wv * hk;
      }
    }
#pragma unroll 8
    for (int c = 0; c < U; ++c) {
      const float wg = W.gate_wT[(H + c) * H + o];
#pragma unroll
      for (int q = 0; q < NA; ++q) gt[q] += wg * ui[q][c];
    }
#pragma unroll
    for (int q = 0; q < NA; ++q)
      if (q0 + q < total) acc += sigm(gt[q]) * vl[q];
  }
  red[t] = acc;
  __syncthreads();
  if (t < H) {
    float s = 0.0f;
    for (int q = 0; q < G; ++q) s += red[q * H + t];
    out[t] = s;
  }
}

// arguments of one SG-CNN call
struct SgCall {
  const int32_t *atom_off;
  int n_atoms;
  const float *feat;
  const uint8_t *is_lig;
  int p0, n_poses, mean_atoms;
  const int32_t *row[2], *col[2];  // covalent, non-covalent
  int64_t cap[2];
  int csr_global;
  float *hbuf;
  int64_t hcap;
  float *latent;
  int64_t *status;
};

// rounds r0 .. r0 + K - 1 of a stage; cur and nxt are swapped after each
template <int H, bool F32, bool SEP>
hipError_t launch_rounds(const SgWeights &W, const SgCall &c, int stage, int r0, int K, float *&cur, float *&nxt,
                         hipStream_t s) {
  constexpr size_t lds = sizeof(float) * sg_lds_floats<H, F32>();
  static_assert(lds <= 65536, "a launch needs no attribute for this much");
  const int nbx = pose_blocks(c.n_atoms, c.mean_atoms, SgTile<H>::BLK);
  for (int r = r0; r < r0 + K; ++r) {
    hipLaunchKernelGGL((k_sg_round<H, F32, SEP>), dim3((unsigned)c.n_poses * nbx), dim3(kThreads), lds, s, W, stage, r,
                       c.atom_off, c.n_atoms, c.p0, nbx, c.row[stage], c.col[stage], c.cap[stage], c.csr_global, cur,
                       nxt, c.hcap, c.status);
    std::swap(cur, nxt);
  }
  return hipGetLastError();
}

template <int H>
hipError_t launch_embed(const SgWeights &W, const SgCall &c, float *h0, hipStream_t s) {
  const int nbx = pose_blocks(c.n_atoms, c.mean_atoms, kEmbedRows);
  hipLaunchKernelGGL(k_sg_embed<H>, dim3((unsigned)c.n_poses * nbx), dim3(kThreads), 0, s, W, c.atom_off, c.n_atoms,
                     c.feat, c.p0, nbx, h0, c.hcap, c.status);
  return hipGetLastError();
}

template <int H, bool F32>
hipError_t launch_flat(const SgWeights &W, const SgCall &c, hipStream_t s) {
  float *cur = c.hbuf, *nxt = c.hbuf + c.hcap * H;
  hipError_t e = launch_embed<H>(W, c, cur, s);
  if (e == hipSuccess) e = launch_rounds<H, F32, F32>(W, c, 0, 0, W.K_c, cur, nxt, s);
  if (e == hipSuccess) e = launch_rounds<H, F32, F32>(W, c, 1, W.K_c, W.K_n, cur, nxt, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_sg_readout<H, CF_NCH>), dim3(c.n_poses), dim3(kThreads), 0, s, W, c.atom_off, c.n_atoms, cur,
                     c.feat, 0, c.is_lig, c.p0, c.hcap, c.latent);
  return hipGetLastError();
}

// Each stage has its own pair of state buffers at its own row stride.  Layout
// (floats): covalent states 2 x [hcap][HC], covalent gather [hcap][HC],
// non-covalent states 2 x [hcap][HN].
template <int HC, int HN, bool F32>
hipError_t launch_staged(const SgWeights &W, const SgCall &c, hipStream_t s) {
  float *cur = c.hbuf, *nxt = c.hbuf + c.hcap * HC, *gb = c.hbuf + 2 * c.hcap * HC;
  float *cur2 = gb + c.hcap * HC, *nxt2 = cur2 + c.hcap * HN;
  hipError_t e = launch_embed<HC>(W, c, cur, s);
  if (e == hipSuccess) e = launch_rounds<HC, F32, false>(W, c, 0, 0, W.K_c, cur, nxt, s);
  if (e != hipSuccess) return e;
  const int nbx = pose_blocks(c.n_atoms, c.mean_atoms, kEmbedRows);
  hipLaunchKernelGGL((k_sg_mid<HC, HN>), dim3((unsigned)c.n_poses * nbx), dim3(kThreads), 0, s, W, c.atom_off,
                     c.n_atoms, c.feat, c.p0, nbx, cur, gb, cur2, c.hcap, c.status);
  e = launch_rounds<HN, F32, false>(W, c, 1, W.K_c, W.K_n, cur2, nxt2, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_sg_readout<HN, HC>), dim3(c.n_poses), dim3(kThreads), 0, s, W, c.atom_off, c.n_atoms, cur2, gb,
                     1, c.is_lig, c.p0, c.hcap, c.latent);
  return hipGetLastError();
}

// width 16: one workgroup per pose
hipError_t launch_h16(const SgWeights &W, const SgCall &c, hipStream_t s) {
  constexpr int H = 16;
  static_assert((H + CF_NCH) * H <= 3 * H * H, "readout weights must fit the staging area");
  const size_t lds = sizeof(SgShared<H>);
  hipLaunchKernelGGL((k_sgcnn_f32<H>), dim3(c.n_poses), dim3(kThreads), lds, s, W, c.atom_off, c.n_atoms, c.feat,
                     c.is_lig, c.p0, c.row[0], c.col[0], c.cap[0], c.row[1], c.col[1], c.cap[1], c.csr_global, c.hbuf,
                     c.hcap, c.latent, c.status);
  return hipGetLastError();
}

}  // namespace

// widths the staged kernel is built for (covalent, non-covalent)
bool sgcnn_staged_supported(int hc, int hn) {
  return (hc == 32 && (hn == 64 || hn == 128)) || (hc == 64 && hn == 128);
}

hipError_t launch_sgcnn(const SgWeights &W, int bf16, const int32_t *atom_off, int n_atoms, const float *feat,
                        const uint8_t *is_lig, int p0, int n_poses, int mean_atoms, const int32_t *cov_row,
                        const int32_t *cov_col, int64_t cov_cap, const int32_t *nc_row,
                        const int32_t *nc_col, int64_t nc_cap, int csr_global, float *hbuf,
                        int64_t hcap_atoms, float *sg_latent, int64_t *status, hipStream_t s) {
  if (n_poses <= 0) return hipSuccess;
  const SgCall c{atom_off, n_atoms, feat,       is_lig,     p0,   n_poses,    mean_atoms, {cov_row, nc_row}, {cov_col, nc_col},
                 {cov_cap, nc_cap}, csr_global, hbuf, hcap_atoms, sg_latent,  status};
  // the split-bfloat16 products need the split weight copies (precision form, H >= 32)
  const bool split = bf16 && W.msg_hi[0] != nullptr;
  if (W.staged) {
    if (bf16 && !split) return hipErrorInvalidValue;
#define CF_ST(HC, HN)                                                                            \
  if (W.H == HC && W.H2 == HN)                                                                   \
    return split ? launch_staged<HC, HN, false>(W, c, s) : launch_staged<HC, HN, true>(W, c, s);
    CF_ST(32, 64)
    CF_ST(32, 128)
    CF_ST(64, 128)
#undef CF_ST
    return hipErrorInvalidValue;
  }
  if (W.H == 16) return launch_h16(W, c, s);
  if (W.H == 32) return split ? launch_flat<32, false>(W, c, s) : launch_flat<32, true>(W, c, s);
  if (W.H == 64) return split ? launch_flat<64, false>(W, c, s) : launch_flat<64, true>(W, c, s);
  return hipErrorInvalidValue;
}

}  // namespace cf
