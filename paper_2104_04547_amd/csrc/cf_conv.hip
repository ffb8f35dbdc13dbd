// conv3d as an implicit GEMM on the CDNA4 matrix cores (MFMA).
//
// The 3D-CNN head (Sec. 3.3.1, Table III) is a stack of 3-D convolutions with
// BatchNorm (folded into weights and bias at context creation), ReLU and
// residual adds; it holds >99 % of the scoring FLOPs, so it is the one place the
// path is a dense contraction: M = output voxels, N = output channels,
// K = input channels x k^3 taps.
//
// Design (per workgroup = one spatial output tile of one pose, all of N or an
// N-tile of 64/128 columns):
//   * activations are channels-last; K is walked as (channel chunk, tap).  For
//     each 16-channel chunk (bf16) or 8-channel chunk (fp32) the tile's input
//     halo is staged once in LDS (32 bytes per voxel), then all k^3 taps are read
//     from LDS as shifted windows: no im2col buffer, and each input byte is
//     fetched from L2 once per tile and chunk.
//   * LDS rows are padded by 16 bytes (so the 16 lanes of one ds_read_b128 phase
//     hit disjoint banks) and stride-2 layers store the halo parity-split per
//     axis, so consecutive output voxels stay 32 bytes apart for every tap.
//   * the weight (B) fragments are pre-packed so that one 16-byte load per lane
//     gives one MFMA operand; they stream from L2/L1 straight into VGPRs.
//   * bf16: v_mfma_f32_32x32x16_bf16, one per (32-row block, 32-column block)
//     per chunk-tap; fp32: four v_mfma_f32_32x32x2_f32 (channels stored
//     even/odd-interleaved within a chunk so a lane's four K values are
//     contiguous).  Accumulation is fp32 in both.
//   * epilogue: + folded bias, + residual tensor, ReLU, convert, store.
#include <algorithm>
#include <type_traits>

#include "cf_internal.h"

namespace cf {

namespace {

template <typename T>
struct Frag;
template <>
struct Frag<bf16_t> {
  static constexpr int CC = 16;  // channels per chunk
};
template <>
struct Frag<float> {
  static constexpr int CC = 8;
};

__device__ inline int stored_index(int h, int n, int S) { return S == 1 ? h : (h & 1) * ((n + 1) >> 1) + (h >> 1); }

template <typename T, int KS, int S, int TZ, int TY, int TX, int NW, int NT>
struct ConvCfg {
  static constexpr int CC = Frag<T>::CC;
  static constexpr int PAD = (KS - 1) / 2;
  static constexpr int HZ = TZ * S + KS - S, HY = TY * S + KS - S, HX = TX * S + KS - S;
  static constexpr int ROW = HX * 32 + 16;  // bytes
  static constexpr int SLAB = HY * ROW;
  static constexpr int LDS = HZ * SLAB;
  static constexpr int MT = TZ * TY * TX;
  static constexpr int WM = MT / NW;
  static constexpr int MB = WM / 32, NB = NT / 32;
  static_assert(WM % 32 == 0, "rows per wave must be a multiple of 32");
  static_assert(LDS <= 163840, "halo exceeds LDS");
};

template <typename T, int KS, int S, int TZ, int TY, int TX, int NW, int NT>
__global__ __launch_bounds__(NW * 64) void k_conv(const T *__restrict__ in, const T *__restrict__ wpk,
                                                   const float *__restrict__ bias,
                                                   const T *__restrict__ res, T *__restrict__ out, int D,
                                                   int Do, int cin_pad, int cout_pad32, int cout,
                                                   int cout_store, int nty, int ntx, int wbytes) {
  using C = ConvCfg<T, KS, S, TZ, TY, TX, NW, NT>;
  constexpr int CC = C::CC;
  __shared__ __attribute__((aligned(16))) char lds[C::LDS];

  int tile, pose, nblk;
  xcd_order(tile, pose, nblk);
  const int n0 = nblk * NT;
  const int tz0 = (tile / (nty * ntx)) * TZ, ty0 = ((tile / ntx) % nty) * TY, tx0 = (tile % ntx) * TX;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int khalf = lane >> 5, lrow = lane & 31;
  const int nchunks = cin_pad / CC;

  // per M-block LDS byte offset of this lane's output row (tap (0,0,0))
  int rowoff[C::MB];
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb) {
    const int m = wave * C::WM + mb * 32 + lrow;
    const int z = m / (TY * TX), y = (m / TX) % TY, x = m % TX;
    rowoff[mb] = z * C::SLAB + y * C::ROW + x * 32 + khalf * 16;
  }

  typedef float accv __attribute__((ext_vector_type(16)));
  accv acc[C::MB][C::NB];
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.0f;

  const int oz = tz0 * S - C::PAD, oy = ty0 * S - C::PAD, ox = tx0 * S - C::PAD;
  const int64_t pose_in = (int64_t)pose * D * D * D;
  constexpr int HZ2 = S == 1 ? 0 : (C::HZ + 1) / 2;
  constexpr int HY2 = S == 1 ? 0 : (C::HY + 1) / 2;
  constexpr int HX2 = S == 1 ? 0 : (C::HX + 1) / 2;

  // ---- halo staging: 32 bytes per voxel; iteration `it` of a thread covers voxel
  // it * threads + tid.  All of a thread's loads are issued before the first LDS
  // store, so a chunk's staging costs about one memory latency, which the other
  // workgroup on the CU covers with its MFMAs. ----
  constexpr int NV = C::HZ * C::HY * C::HX;
  constexpr int NTH = NW * 64;
  constexpr int HITER = (NV + NTH - 1) / NTH;
  auto halo_load = [&](int it, int ch, uint4 &lo, uint4 &hi) {
    const int v = it * NTH + (int)threadIdx.x;
    lo = make_uint4(0, 0, 0, 0);
    hi = lo;
    if (v < NV) {
      const int hx = v % C::HX, hy = (v / C::HX) % C::HY, hz = v / (C::HX * C::HY);
      const int gz = oz + hz, gy = oy + hy, gx = ox + hx;
      if ((unsigned)gz < (unsigned)D && (unsigned)gy < (unsigned)D && (unsigned)gx < (unsigned)D) {
        const T *src = in + ((pose_in + ((int64_t)gz * D + gy) * D + gx) * cin_pad + ch * CC);
        lo = reinterpret_cast<const uint4 *>(src)[0];
        hi = reinterpret_cast<const uint4 *>(src)[1];
      }
    }
  };
  auto halo_store = [&](int it, uint4 lo, uint4 hi) {
    const int v = it * NTH + (int)threadIdx.x;
    if (v < NV) {
      const int hx = v % C::HX, hy = (v / C::HX) % C::HY, hz = v / (C::HX * C::HY);
      if (sizeof(T) == 4) {  // fp32: channels (0..7) -> (0,2,4,6 | 1,3,5,7)
        const uint4 a = lo, b = hi;
        lo = make_uint4(a.x, a.z, b.x, b.z);
        hi = make_uint4(a.y, a.w, b.y, b.w);
      }
      const int off = stored_index(hz, C::HZ, S) * C::SLAB + stored_index(hy, C::HY, S) * C::ROW +
                      stored_index(hx, C::HX, S) * 32;
      *reinterpret_cast<uint4 *>(lds + off) = lo;
      *reinterpret_cast<uint4 *>(lds + off + 16) = hi;
    }
  };
  const int tap_bytes = nchunks * cout_pad32 * CC * (int)sizeof(T);
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(wpk), (short)0, wbytes, 0x00020000);
  for (int chunk = 0; chunk < nchunks; ++chunk) {
    if (chunk) __syncthreads();  // every wave is done reading the previous chunk's halo
    {
      uint4 hl[HITER], hh[HITER];
#pragma unroll
      for (int it = 0; it < HITER; ++it) halo_load(it, chunk, hl[it], hh[it]);
#pragma unroll
      for (int it = 0; it < HITER; ++it) halo_store(it, hl[it], hh[it]);
    }
    __syncthreads();
    // Taps are consecutive in the packed weights, so the B fragments of tap t+1 and
    // t+2 are in flight while tap t's MFMAs issue.  They are buffer loads with the
    // tap offset in a scalar register (no per-tap address arithmetic); past the last
    // tap they read the zero taps of the padding.
    static_assert(2 <= kConvPadTaps, "prefetch past the weight padding");
    int vb[C::NB];
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb)
      vb[nb] = (((chunk * cout_pad32 + n0 + nb * 32 + lrow) * CC) + khalf * (CC / 2)) * (int)sizeof(T);
    uint4 b1[C::NB], b2[C::NB];
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb) {
      b1[nb] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb[nb], 0, 0));
      b2[nb] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb[nb], tap_bytes, 0));
    }
    int soff = 2 * tap_bytes;
    for (int dz = 0; dz < KS; ++dz) {
      const int offz = (S == 1 ? dz : (dz & 1) * HZ2 + (dz >> 1)) * C::SLAB;
      for (int dy = 0; dy < KS; ++dy) {
        const int offzy = offz + (S == 1 ? dy : (dy & 1) * HY2 + (dy >> 1)) * C::ROW;
#pragma unroll
        for (int dx = 0; dx < KS; ++dx) {
          const int toff = offzy + (S == 1 ? dx : (dx & 1) * HX2 + (dx >> 1)) * 32;
          uint4 bfr[C::NB];
#pragma unroll
          for (int nb = 0; nb < C::NB; ++nb) {
            bfr[nb] = b1[nb];
            b1[nb] = b2[nb];
            b2[nb] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb[nb], soff, 0));
          }
          soff += tap_bytes;
          uint4 afr[C::MB];
#pragma unroll
          for (int mb = 0; mb < C::MB; ++mb) afr[mb] = *reinterpret_cast<const uint4 *>(lds + rowoff[mb] + toff);
#pragma unroll
          for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < C::NB; ++nb) {
              if constexpr (sizeof(T) == 2) {
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, afr[mb]), __builtin_bit_cast(bf16x8, bfr[nb]), acc[mb][nb], 0, 0, 0);
              } else {
                const float4 a = __builtin_bit_cast(float4, afr[mb]);
                const float4 b = __builtin_bit_cast(float4, bfr[nb]);
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc[mb][nb], 0, 0, 0);
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc[mb][nb], 0, 0, 0);
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc[mb][nb], 0, 0, 0);
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc[mb][nb], 0, 0, 0);
              }
            }
        }
      }
    }
  }

  // ---- epilogue: bias, residual, ReLU, store ----
  const int64_t pose_out = (int64_t)pose * Do * Do * Do;
  auto row_base = [&](int m, bool &valid) -> int64_t {
    const int z = tz0 + m / (TY * TX), y = ty0 + (m / TX) % TY, x = tx0 + m % TX;
    valid = z < Do && y < Do && x < Do;
    return (pose_out + ((int64_t)z * Do + y) * Do + x) * cout_store;
  };
  if constexpr (sizeof(T) == 2 && C::MT * NT * 2 <= C::LDS) {
    // bf16: the output tile goes through LDS so that residual reads and output
    // writes are 16-byte row segments instead of 2-byte scatters.
    bf16_t *ot = reinterpret_cast<bf16_t *>(lds);  // [MT][NT]
    constexpr int SEG = NT / 8;                       // 16-byte segments per row
    __syncthreads();                                  // halo no longer needed
    if (res) {
      for (int e = threadIdx.x; e < C::MT * SEG; e += NTH) {
        const int m = e / SEG, q = e % SEG;
        bool valid;
        const int64_t ob = row_base(m, valid);
        if (valid && n0 + q * 8 + 8 <= cout_store)
          *reinterpret_cast<uint4 *>(ot + m * NT + q * 8) = *reinterpret_cast<const uint4 *>(res + ob + n0 + q * 8);
      }
      __syncthreads();
    }
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = wave * C::WM + mb * 32 + 8 * (r >> 2) + 4 * khalf + (r & 3);
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) {
          const int col = nb * 32 + lrow;
          float v = acc[mb][nb][r] + bias[n0 + col];
          if (res) v += (float)ot[m * NT + col];
          ot[m * NT + col] = (bf16_t)(v > 0.0f ? v : 0.0f);
        }
      }
    __syncthreads();
    for (int e = threadIdx.x; e < C::MT * SEG; e += NTH) {
      const int m = e / SEG, q = e % SEG;
      bool valid;
      const int64_t ob = row_base(m, valid);
      if (valid && n0 + q * 8 + 8 <= cout_store)
        *reinterpret_cast<uint4 *>(out + ob + n0 + q * 8) = *reinterpret_cast<const uint4 *>(ot + m * NT + q * 8);
    }
  } else {
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = wave * C::WM + mb * 32 + 8 * (r >> 2) + 4 * khalf + (r & 3);
        bool valid;
        const int64_t ob = row_base(m, valid);
        if (!valid) continue;
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) {
          const int n = n0 + nb * 32 + lrow;
          if (n >= cout) continue;
          float v = acc[mb][nb][r] + bias[n];
          if (res) v += (float)res[ob + n];
          v = v > 0.0f ? v : 0.0f;
          out[ob + n] = (T)v;
        }
      }
    }
  }
}

// ---- bf16 with 8-channel chunks and tap pairs ---------------------------------
//
// Same implicit GEMM, but the K walk pairs two consecutive taps of one 8-channel
// chunk into each 16-deep MFMA step: lanes of the first K half read their row at
// tap 2p, lanes of the second half at tap 2p+1.  The halo then needs 16 bytes per
// voxel, so an 8x8x8 output tile (128 rows per wave, 8 MFMAs per step) fits twice
// per CU, halving the weight traffic per FLOP of the 64-row tiles; and a 19-channel
// input costs 3 chunks instead of the 2 x 16 = 32 padded channels.
//
// Two further knobs serve the 64 -> 128 stride-2 layer, whose 12^3 output tiles
// poorly and whose weights do not stay in L2: WN waves split the columns (each
// wave 64 x 64, half the weight loads per MFMA of a 32 x 128 wave), and PP poses
// share one workgroup (the same tile of consecutive poses, one halo each), so one
// pass over the weights serves PP times the rows.
template <int KS, int S, int TZ, int TY, int TX, int NW, int NT, int WN, int PP>
struct Conv8Cfg {
  static_assert(KS >= 3 && KS % 2 == 1, "odd kernel of at least 3 taps per axis");
  static constexpr int PAD = (KS - 1) / 2;
  static constexpr int HZ = TZ * S + KS - S, HY = TY * S + KS - S, HX = TX * S + KS - S;
  // Row pitch.  A 16-lane group of a 16-byte LDS read covers two 8-voxel output
  // rows; a pitch of 128 mod 256 bytes puts those rows on disjoint banks.  Taken
  // unless only a tighter pitch keeps two workgroups per CU (or fits at all):
  // then the tight pitch + 16 bytes, or without the 16 bytes as a last resort.
  static constexpr int ROW_CF = ((HX * 16 + 127) / 256) * 256 + 128, ROW_T = HX * 16 + 16;
  static constexpr int PLANES = PP * HZ * HY;
  static constexpr int ROW = (PLANES * ROW_CF <= 81920)   ? ROW_CF
                             : (PLANES * ROW_T <= 81920)  ? ROW_T
                             : (PLANES * ROW_CF <= 163840) ? ROW_CF
                             : (PLANES * ROW_T <= 163840)  ? ROW_T
                                                           : HX * 16;  // bytes
  static constexpr int SLAB = HY * ROW;
  // Rows of a 16-lane group: two runs of 8 voxels (TX = 8) YD rows apart, with YD
  // the smallest of 1, 2, 4 that puts them 128 mod 256 bytes apart (disjoint banks)
  // when the pitch itself cannot be (the tight pitch of one-workgroup halos).
  static constexpr int YD = (TX != 8 || ROW % 256 == 128)            ? 1
                            : ((2 * ROW) % 256 == 128 && TY % 4 == 0) ? 2
                            : ((4 * ROW) % 256 == 128 && TY % 8 == 0) ? 4
                                                                      : 1;
  // PP poses per workgroup (the same tile of consecutive poses): the halo of
  // pose pp sits at pp * HALO1, its rows are tile rows pp * MT1 .. + MT1.  Each
  // weight fragment then serves PP times the rows.
  static constexpr int HALO1 = HZ * SLAB, HALO = PP * HALO1;
  static constexpr int MT1 = TZ * TY * TX, MT = PP * MT1;
  // the NW waves form NWM row groups x WN column groups: wave w takes rows
  // (w / WN) * WM .. + WM and columns (w % WN) * NT / WN .. + NT / WN
  static constexpr int NWM = NW / WN;
  static constexpr int WM = MT / NWM;
  static constexpr int MB = WM / 32, NB = NT / WN / 32;
  static constexpr int TAPS = KS * KS * KS, PAIRS = (TAPS + 1) / 2;
  // epilogue: output rows go through LDS in groups of MBG 32-row blocks per row group
  static constexpr int MBG = (NWM * 32 * NT * 2 * MB <= HALO) ? MB : ((NWM * 32 * NT * 2 * 2 <= HALO && MB % 2 == 0) ? 2 : 1);
  static constexpr int EPI = NWM * 32 * MBG * NT * 2;
  // Fine tiles (one or two 32 x 32 blocks per wave): a pair has 32 or 64 MFMA cycles, less
  // than the scalar arithmetic of its tap offsets (~60 instructions, 230 cycles a pair
  // measured), so those come from a table in LDS: 16-bit counts of 16 bytes, [K half][entry],
  // entry p + 5 for pair p, read eight entries at a time a group ahead.
  static constexpr int BLOCKS = MB * NB;
  static constexpr bool FINE = BLOCKS <= 2 && PP == 1;
  static constexpr int ENT = (PAIRS + 5 + 32 + 7) / 8 * 8;
  static constexpr int TAB = FINE ? 2 * ENT * 2 : 0;
  static constexpr int LDS = TAB + (HALO > EPI ? HALO : EPI);
  // Waves per SIMD the tile allows: a halo above half the LDS leaves one
  // workgroup per CU, so a four-wave workgroup owns its SIMDs' whole register file
  // (512 per lane); six-wave workgroups run two per CU (three waves per SIMD).
  static constexpr int WPE = (NW == 6 || NW == 12) ? 3 : ((LDS > 81920 && NW <= 4) ? 1 : 2);
  // Halo voxels each thread loads per chunk, and how many of those loads are in
  // flight at once (one batch per L2 round trip): all of them where the
  // registers allow, else batches of 6 beside 128 accumulator registers.
  static constexpr int NV1 = HZ * HY * HX, HITER = (PP * NV1 + NW * 64 - 1) / (NW * 64);
  static constexpr int HB_MAX = WPE == 1 ? 40 : (MB * NB <= 4 ? 16 : 6);
  static constexpr int HB = HITER < HB_MAX ? HITER : HB_MAX;
  // Software pipeline of the pair walk: weight fragments PF pairs ahead, row fragments
  // AD - 1 pairs ahead (PF a multiple of AD).  Several poses per workgroup mean one
  // workgroup per CU and weights beyond L2 (the 64 -> 128 stride-2 layer): six pairs
  // ahead there (5 % faster than four; eight spill at 256 registers).  A wave of one or
  // two 32 x 32 blocks has 32 or 64 MFMA cycles per pair to cover an LDS and an L2
  // round trip: deeper rings, in the registers that the small accumulator leaves.
  static constexpr int AD = FINE ? 4 : 2;
  // fine tiles keep each thread's halo addresses in registers for all chunks and, where
  // the voxels themselves fit too, load the next chunk's during the walk of this one
  static constexpr bool AHEAD = FINE && HITER <= 9;
  static constexpr int PF = PP > 1 ? 6 : BLOCKS == 1 ? 16 : BLOCKS == 2 ? 8 : ((NB <= 2 && KS > 3) ? 4 : 2);
  static_assert(PF % AD == 0 && (!FINE || PF % 8 == 0), "the unrolled walk indexes the rings at compile time");
  static_assert(PF <= kConvPadSteps, "prefetch past the weight padding");
  static_assert(!FINE || HALO / 16 < 65536, "16-bit table entries");
  static constexpr int WGCU = (163840 / LDS < WPE * 4 / NW ? 163840 / LDS : WPE * 4 / NW) < 1 ? 1 : (163840 / LDS < WPE * 4 / NW ? 163840 / LDS : WPE * 4 / NW);
  static_assert(NW % WN == 0 && NT % (32 * WN) == 0, "waves split the columns in 32-column blocks");
  static_assert(WM % 32 == 0, "rows per wave must be a multiple of 32");
  static_assert(LDS <= 163840, "halo exceeds LDS");
};

// Output voxel (z, y, x) of tile row ml (one pose's tile): x fastest in runs of TX;
// with YD > 1 the y order pairs y with y + YD in consecutive runs.
template <int TY, int TX, int YD>
__device__ inline void tile_coord(int ml, int &z, int &y, int &x) {
  z = ml / (TY * TX);
  const int r = ml % (TY * TX), g = r / TX;
  x = r % TX;
  if (YD == 4)
    y = (g & ~7) + (g >> 1 & 3) + 4 * (g & 1);
  else if (YD == 2)
    y = (g & ~3) + (g >> 1 & 1) + 2 * (g & 1);
  else
    y = g;
}

template <int KS, int S, int TZ, int TY, int TX, int NW, int NT, int WN, int PP>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(Conv8Cfg<KS, S, TZ, TY, TX, NW, NT, WN, PP>::WPE))) void k_conv8(const bf16_t *__restrict__ in, const bf16_t *__restrict__ wpk,
                                                    const float *__restrict__ bias, const bf16_t *__restrict__ res,
                                                    bf16_t *__restrict__ out, int n_poses, int D, int Do, int cin_pad,
                                                    int nchunks, int cout_pad32, int cout, int cout_store, int nty,
                                                    int ntx, int wbytes) {
  using C = Conv8Cfg<KS, S, TZ, TY, TX, NW, NT, WN, PP>;
  __shared__ __attribute__((aligned(16))) char lds_all[C::LDS];
  char *lds = lds_all + C::TAB;  // halo; epilogue rows
  int tile, pblk, nblk;
  if constexpr (C::FINE)
    xcd_order_by_z(tile, pblk, nblk);
  else
    xcd_order(tile, pblk, nblk);
  const int pose0 = pblk * PP;
  const int n0 = nblk * NT;
  const int tz0 = (tile / (nty * ntx)) * TZ, ty0 = ((tile / ntx) % nty) * TY, tx0 = (tile % ntx) * TX;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wave_m = wave / WN, ncol0 = (wave % WN) * (NT / WN);
  const int khalf = lane >> 5, lrow = lane & 31;
  constexpr int NTH = NW * 64;

  int rowoff[C::MB];
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb) {
    const int m = wave_m * C::WM + mb * 32 + lrow;
    const int pp = m / C::MT1, ml = m % C::MT1;
    int z, y, x;
    tile_coord<TY, TX, C::YD>(ml, z, y, x);
    rowoff[mb] = pp * C::HALO1 + z * C::SLAB + y * C::ROW + x * 16;
  }
  typedef float accv __attribute__((ext_vector_type(16)));
  accv acc[C::MB][C::NB];
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.0f;

  const int oz = tz0 * S - C::PAD, oy = ty0 * S - C::PAD, ox = tx0 * S - C::PAD;
  const int64_t pose_in = (int64_t)pose0 * D * D * D;
  constexpr int HZ2 = S == 1 ? 0 : (C::HZ + 1) / 2;
  constexpr int HY2 = S == 1 ? 0 : (C::HY + 1) / 2;
  constexpr int HX2 = S == 1 ? 0 : (C::HX + 1) / 2;
  constexpr int NV = PP * C::NV1;
  constexpr int HITER = C::HITER, HB = C::HB;
  auto tapoff = [&](int dz, int dy, int dx) {
    return (S == 1 ? dz : (dz & 1) * HZ2 + (dz >> 1)) * C::SLAB +
           (S == 1 ? dy : (dy & 1) * HY2 + (dy >> 1)) * C::ROW + (S == 1 ? dx : (dx & 1) * HX2 + (dx >> 1)) * 16;
  };

  // LDS offset of this lane's tap in pair p whose first tap is (z, y, x): lanes of
  // the first K half read tap 2p, the second half tap 2p + 1 (the first tap again
  // past the last tap, whose weights are zero)
  auto pair_toff = [&](int p, int z, int y, int x) {
    int ez = z, ey = y, ex = x + 1;
    if (ex == KS) {
      ex = 0;
      if (++ey == KS) {
        ey = 0;
        ++ez;
      }
    }
    const int t0 = tapoff(z, y, x);
    const int t1 = (2 * p + 1 < C::TAPS) ? tapoff(ez, ey, ex) : t0;
    return khalf ? t1 : t0;
  };
  // the rings read past the last pair: zero weights of the padding, which reach no MFMA
  constexpr int kPF = C::PF, AD = C::AD;
  uint16_t *tab = reinterpret_cast<uint16_t *>(lds_all);
  if constexpr (C::FINE) {
    for (int e = threadIdx.x; e < 2 * C::ENT; e += NTH) {
      const int p = e % C::ENT - 5, t = 2 * p + e / C::ENT;
      // past the last tap (zero weights): the pair's first tap; past the last pair: offset 0
      const int u = p < 0 || p >= C::PAIRS ? 0 : t < C::TAPS ? t : t - 1;
      tab[e] = (uint16_t)(tapoff(u / (KS * KS), (u / KS) % KS, u % KS) >> 4);
    }
  }
  const int pair_bytes = nchunks * cout_pad32 * 16 * 2;
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(wpk), (short)0, wbytes, 0x00020000);
  // Fine tiles run when few workgroups do, all in step and all missing L2 on the same
  // weights, a ring's depth per trip to memory.  So the first workgroups of an XCD each
  // touch a share of the next chunk's weights (one word per 128-byte line) a chunk ahead.
  // Measured alone: one pose's score 390 us without, 378 with; 96 poses of the paper-sized
  // model 1923 and 1914; 19 poses of 64^3 and 77 of 32^3 0.2 % apart.
  constexpr int kLinesPair = NT * 32 / 128, kLines = kLinesPair * C::PAIRS;
  constexpr int kWarm = 4;  // lines per thread at most
  const int wg = (int)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) / 8;
  const int nwg = max(1, (int)(gridDim.x * gridDim.y * gridDim.z) / 8);
  const int share = min(nwg, 32);
  uint32_t touched[kWarm];
  auto warm = [&](int chunk) {
#pragma unroll
    for (int i = 0; i < kWarm; ++i) {
      const int l = wg + share * ((int)threadIdx.x + i * NTH);
      const int off = (l / kLinesPair) * pair_bytes + (chunk * cout_pad32 + n0) * 32 + (l % kLinesPair) * 128;
      touched[i] = 0;
      if (wg < share && l < kLines && chunk < nchunks) touched[i] = __builtin_amdgcn_raw_buffer_load_b32(wrs, off, 0, 0);
    }
  };
  auto warm_done = [&]() {
#pragma unroll
    for (int i = 0; i < kWarm; ++i) asm volatile("" ::"v"(touched[i]));  // keeps the loads
  };
  constexpr int kHv = C::FINE ? C::HITER : 1;
  int hsrc[kHv], hdst[kHv];  // element and LDS offsets of this thread's halo voxels, -1: none
  uint4 hnext[kHv];
  auto halo_fetch = [&](int chunk) {
    const bf16_t *cin0 = in + pose_in * cin_pad + chunk * 8;
#pragma unroll
    for (int it = 0; it < kHv; ++it)
      hnext[it] = hsrc[it] >= 0 ? *reinterpret_cast<const uint4 *>(cin0 + hsrc[it]) : make_uint4(0, 0, 0, 0);
  };
  if constexpr (C::FINE) {
#pragma unroll
    for (int it = 0; it < kHv; ++it) {
      const int v = it * NTH + (int)threadIdx.x;
      const int hx = v % C::HX, hy = (v / C::HX) % C::HY, hz = v / (C::HX * C::HY);
      const int gz = oz + hz, gy = oy + hy, gx = ox + hx;
      const bool inside = (unsigned)gz < (unsigned)D && (unsigned)gy < (unsigned)D && (unsigned)gx < (unsigned)D;
      hsrc[it] = v < NV && inside ? ((gz * D + gy) * D + gx) * cin_pad : -1;
      hdst[it] = v < NV ? stored_index(hz, C::HZ, S) * C::SLAB + stored_index(hy, C::HY, S) * C::ROW +
                              stored_index(hx, C::HX, S) * 16
                        : -1;
    }
    halo_fetch(0);
    warm(0);
    warm_done();
  }
  for (int chunk = 0; chunk < nchunks; ++chunk) {
    if (chunk) __syncthreads();
    if constexpr (C::FINE) {
      if (!C::AHEAD && chunk) halo_fetch(chunk);
#pragma unroll
      for (int it = 0; it < kHv; ++it)
        if (hdst[it] >= 0) *reinterpret_cast<uint4 *>(lds + hdst[it]) = hnext[it];
    } else {
      // the chunk's first channel of the workgroup's first pose (uniform); voxel
      // offsets from it fit 32 bits (PP * D^3 * cin_pad elements), which keeps the
      // per-voxel address arithmetic out of 64-bit multiplies
      const bf16_t *cin0 = in + pose_in * cin_pad + chunk * 8;
#pragma unroll
      for (int it0 = 0; it0 < HITER; it0 += HB) {
        uint4 hv[HB];
#pragma unroll
        for (int it = it0; it < it0 + HB && it < HITER; ++it) {
          const int v = it * NTH + (int)threadIdx.x;
          hv[it - it0] = make_uint4(0, 0, 0, 0);
          if (v < NV) {
            const int pp = PP == 1 ? 0 : v / C::NV1, vl = PP == 1 ? v : v % C::NV1;
            const int hx = vl % C::HX, hy = (vl / C::HX) % C::HY, hz = vl / (C::HX * C::HY);
            const int gz = oz + hz, gy = oy + hy, gx = ox + hx;
            if ((unsigned)gz < (unsigned)D && (unsigned)gy < (unsigned)D && (unsigned)gx < (unsigned)D &&
                (PP == 1 || pose0 + pp < n_poses))
              hv[it - it0] = *reinterpret_cast<const uint4 *>(cin0 + (((pp * D + gz) * D + gy) * D + gx) * cin_pad);
          }
        }
#pragma unroll
        for (int it = it0; it < it0 + HB && it < HITER; ++it) {
          const int v = it * NTH + (int)threadIdx.x;
          if (v < NV) {
            const int pp = PP == 1 ? 0 : v / C::NV1, vl = PP == 1 ? v : v % C::NV1;
            const int hx = vl % C::HX, hy = (vl / C::HX) % C::HY, hz = vl / (C::HX * C::HY);
            const int off = pp * C::HALO1 + stored_index(hz, C::HZ, S) * C::SLAB + stored_index(hy, C::HY, S) * C::ROW +
                            stored_index(hx, C::HX, S) * 16;
            *reinterpret_cast<uint4 *>(lds + off) = hv[it - it0];
          }
        }
      }
    }
    __syncthreads();
    int vb[C::NB];
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb) vb[nb] = ((chunk * cout_pad32 + n0 + ncol0 + nb * 32 + lrow) * 16 + khalf * 8) * 2;
    // software pipeline: the weight fragments of pair p + kPF and the LDS row
    // fragments of pair p + AD - 1 are in flight while the MFMAs of pair p issue.  The
    // pair loop is unrolled by kPF so that both rings are indexed at compile time
    // (no register moves, so no wait on the newest loads).
    uint4 bq[kPF][C::NB];
#pragma unroll
    for (int q = 0; q < kPF; ++q)
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb)
        bq[q][nb] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb[nb], q * pair_bytes, 0));
    int soff = kPF * pair_bytes;
    if constexpr (C::FINE) {
      if (C::AHEAD && chunk + 1 < nchunks) halo_fetch(chunk + 1);
      warm(chunk + 1);
    }
    uint4 ar[AD][C::MB];
    int dz = 0, dy = 0, dx = 0;  // first tap of the pair whose rows are read next
    auto next_pair = [&]() {
      dx += 2;
      if (dx >= KS) {
        dx -= KS;
        if (++dy == KS) {
          dy = 0;
          ++dz;
        }
      }
    };
    // fine tiles: packed offsets of the next kPF pairs to read (tw) and of those after (tx)
    constexpr int kTw = C::FINE ? kPF / 8 : 1;
    uint4 tw[kTw], tx[kTw];
    const uint4 *tab8 = reinterpret_cast<const uint4 *>(tab + khalf * C::ENT) + 1;  // entry 8 = pair 3
    if constexpr (C::FINE) {
#pragma unroll
      for (int i = 0; i < kTw; ++i) tw[i] = tab8[i];
    }
#pragma unroll
    for (int d = 0; d < AD - 1; ++d) {
      const int t0 = C::FINE ? tab[khalf * C::ENT + d + 5] * 16 : pair_toff(d, dz, dy, dx);
#pragma unroll
      for (int mb = 0; mb < C::MB; ++mb) ar[d][mb] = *reinterpret_cast<const uint4 *>(lds + rowoff[mb] + t0);
      if constexpr (!C::FINE) next_pair();
    }
    auto pair = [&](const int p, const int ph) {
      // past the last pair: offset 0 of its rows (inside the halo) instead
      int tn;
      if constexpr (C::FINE) {
        const uint4 g = tw[ph >> 3];
        const uint32_t t = (ph & 6) == 0 ? g.x : (ph & 6) == 2 ? g.y : (ph & 6) == 4 ? g.z : g.w;
        tn = (int)((ph & 1) ? t >> 16 : t & 0xffffu) * 16;
      } else {
        tn = (p + AD - 1 < C::PAIRS) ? pair_toff(p + AD - 1, dz, dy, dx) : 0;
      }
#pragma unroll
      for (int mb = 0; mb < C::MB; ++mb)
        ar[(ph + AD - 1) % AD][mb] = *reinterpret_cast<const uint4 *>(lds + rowoff[mb] + tn);
      __builtin_amdgcn_sched_barrier(0);  // keep those reads ahead of this pair's MFMAs
      if constexpr (!C::FINE) next_pair();
#pragma unroll
      for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ar[ph % AD][mb]),
                                                                 __builtin_bit_cast(bf16x8, bq[ph][nb]), acc[mb][nb],
                                                                 0, 0, 0);
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb)
        bq[ph][nb] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb[nb], soff, 0));
      soff += pair_bytes;
    };
    // whole groups of kPF pairs with no test inside (so that the compiler's wait
    // analysis keeps every weight load of the ring in flight), then the rest
    constexpr int kFull = C::PAIRS / kPF * kPF;
    for (int p0 = 0; p0 < kFull; p0 += kPF) {
      if constexpr (C::FINE) {
#pragma unroll
        for (int i = 0; i < kTw; ++i) tx[i] = tab8[(p0 + kPF) / 8 + i];
      }
#pragma unroll
      for (int ph = 0; ph < kPF; ++ph) pair(p0 + ph, ph);
      if constexpr (C::FINE) {
#pragma unroll
        for (int i = 0; i < kTw; ++i) tw[i] = tx[i];
      }
    }
#pragma unroll
    for (int ph = 0; ph < kPF; ++ph)
      if (kFull + ph < C::PAIRS) pair(kFull + ph, ph);
    if constexpr (C::FINE) warm_done();
  }

  // ---- epilogue through LDS, MBG row blocks per wave at a time ----
  const int64_t pose_out = (int64_t)pose0 * Do * Do * Do;
  auto row_base = [&](int m, bool &valid) -> int64_t {
    const int pp = m / C::MT1, ml = m % C::MT1;
    int z, y, x;
    tile_coord<TY, TX, C::YD>(ml, z, y, x);
    z += tz0;
    y += ty0;
    x += tx0;
    valid = z < Do && y < Do && x < Do && (PP == 1 || pose0 + pp < n_poses);
    return (pose_out + (((int64_t)pp * Do + z) * Do + y) * Do + x) * cout_store;
  };
  bf16_t *ot = reinterpret_cast<bf16_t *>(lds);  // [NWM][MBG*32][NT]
  constexpr int SEG = NT / 8;
  constexpr int GR = C::MBG * 32;  // rows per row group per epilogue group
  // local row lr of group g -> tile row (lr / GR) * WM + (g + (lr % GR) / 32) * 32 + lr % 32
#pragma unroll
  for (int g = 0; g < C::MB; g += C::MBG) {
    __syncthreads();
    if (res) {
      for (int e = threadIdx.x; e < C::NWM * GR * SEG; e += NTH) {
        const int lr = e / SEG, q = e % SEG;
        const int m = (lr / GR) * C::WM + g * 32 + lr % GR;
        bool valid;
        const int64_t ob = row_base(m, valid);
        if (valid && n0 + q * 8 + 8 <= cout_store)
          *reinterpret_cast<uint4 *>(ot + lr * NT + q * 8) = *reinterpret_cast<const uint4 *>(res + ob + n0 + q * 8);
      }
      __syncthreads();
    }
#pragma unroll
    for (int mb = g; mb < g + C::MBG; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int lr = wave_m * GR + (mb - g) * 32 + 8 * (r >> 2) + 4 * khalf + (r & 3);
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) {
          const int col = ncol0 + nb * 32 + lrow;
          float v = acc[mb][nb][r] + bias[n0 + col];
          if (res) v += (float)ot[lr * NT + col];
          ot[lr * NT + col] = (bf16_t)(v > 0.0f ? v : 0.0f);
        }
      }
    __syncthreads();
    for (int e = threadIdx.x; e < C::NWM * GR * SEG; e += NTH) {
      const int lr = e / SEG, q = e % SEG;
      const int m = (lr / GR) * C::WM + g * 32 + lr % GR;
      bool valid;
      const int64_t ob = row_base(m, valid);
      if (valid && n0 + q * 8 + 8 <= cout_store)
        *reinterpret_cast<uint4 *>(out + ob + n0 + q * 8) = *reinterpret_cast<const uint4 *>(ot + lr * NT + q * 8);
    }
  }
}

// ---- bf16 with 4-channel chunks and tap quads -----------------------------------
//
// For inputs whose channel count leaves much of an 8-channel chunk empty (the
// 19-channel grid: 24 padded channels, 21 % zeros) the K walk takes 4 channels x 4
// taps per 16-deep MFMA step: lanes of the first K half read taps 4q and 4q + 1,
// the second half 4q + 2 and 4q + 3, 8 bytes (4 channels) each.  19 channels cost
// 20, and the halo needs 8 bytes per voxel, so the 21^3 halo of an 8^3 stride-2
// tile fits twice per CU.  Tap offsets come from a table in LDS.
template <int KS, int S, int TZ, int TY, int TX, int NW, int NT>
struct Conv4Cfg {
  static_assert(KS >= 3 && KS % 2 == 1, "odd kernel of at least 3 taps per axis");
  static constexpr int PAD = (KS - 1) / 2;
  static constexpr int HZ = TZ * S + KS - S, HY = TY * S + KS - S, HX = TX * S + KS - S;
  static constexpr int ROW = HX * 8 + 8, SLAB = HY * ROW, HALO = HZ * SLAB;  // bytes
  static constexpr int TAPS = KS * KS * KS, QUADS = (TAPS + 3) / 4;
  static constexpr int MT = TZ * TY * TX, WM = MT / NW, MB = WM / 32, NB = NT / 32;
  // Software pipeline of the quad walk, as in k_conv8: weight fragments PF quads ahead,
  // row fragments AD - 1 quads ahead.
  static constexpr int BLOCKS = MB * NB, AD = BLOCKS <= 2 ? 4 : 2;
  static constexpr int PF = BLOCKS <= 2 ? 8 : 4;  // big tiles: weights stay in L2, six quads ahead measured 6 % slower
  // LDS table of tap offsets into the halo.  AD = 2: one word per tap, read a quad
  // ahead.  AD = 4: LDS reads return in order, so a table read per quad would wait for
  // the row reads before it; the offsets of a quad are packed instead (two 16-bit
  // counts of 8 bytes per K half) and read eight quads at a time, a group ahead:
  // [half][entry], entry q + 1 for quad q (eight entries from a multiple of 4)
  static constexpr int ENT = (QUADS + 2 * PF + 8) / 4 * 4;
  static constexpr int TAB = AD == 2 ? QUADS * 4 * 4 : 2 * ENT * 4;
  static constexpr int MBG = (NW * 32 * NT * 2 * MB <= HALO) ? MB : ((NW * 32 * NT * 2 * 2 <= HALO && MB % 2 == 0) ? 2 : 1);
  static constexpr int EPI = NW * 32 * MBG * NT * 2;
  static constexpr int LDS = TAB + (HALO > EPI ? HALO : EPI);
  static constexpr int WPE = LDS > 81920 ? 1 : 2;
  static constexpr int HITER = (HZ * HY * HX + NW * 64 - 1) / (NW * 64);
  // halo loads in flight per batch (one round trip each): all of them up to 20
  // voxels per thread, else two batches (the 21^3 halo of the first layer: 37
  // voxels per thread in 19 + 18 instead of batches of 8, 4-5 % faster)
  static constexpr int HB = HITER <= 20 ? HITER : (HITER + 1) / 2;
  static constexpr int WGCU = 163840 / LDS < WPE * 4 / NW ? 163840 / LDS : WPE * 4 / NW;
  static_assert(WM % 32 == 0, "rows per wave must be a multiple of 32");
  static_assert(LDS <= 163840, "halo exceeds LDS");
  static_assert(AD == 2 || (PF == 8 && AD == 4 && HALO / 8 < 65536), "packed table of the deep walk");
  static_assert(PF <= kConvPadSteps, "prefetch past the weight padding");
};

template <int KS, int S, int TZ, int TY, int TX, int NW, int NT>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(Conv4Cfg<KS, S, TZ, TY, TX, NW, NT>::WPE))) void k_conv4(
    const bf16_t *__restrict__ in, const bf16_t *__restrict__ wpk, const float *__restrict__ bias,
    const bf16_t *__restrict__ res, bf16_t *__restrict__ out, int D, int Do, int cin_pad, int nchunks, int cout_pad32,
    int cout_store, int nty, int ntx, int wbytes, int chunk_major) {
  using C = Conv4Cfg<KS, S, TZ, TY, TX, NW, NT>;
  __shared__ __attribute__((aligned(16))) char lds[C::LDS];
  constexpr int AD = C::AD;
  int *tab = reinterpret_cast<int *>(lds);  // tap offsets into the halo (Conv4Cfg)
  char *halo = lds + C::TAB;
  int tile, pose, nblk;
  xcd_order(tile, pose, nblk);
  const int n0 = nblk * NT;
  const int tz0 = (tile / (nty * ntx)) * TZ, ty0 = ((tile / ntx) % nty) * TY, tx0 = (tile % ntx) * TX;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int khalf = lane >> 5, lrow = lane & 31;
  constexpr int NTH = NW * 64;
  constexpr int HZ2 = (C::HZ + 1) / 2, HY2 = (C::HY + 1) / 2, HX2 = (C::HX + 1) / 2;
  auto tap_off = [&](int t) {
    if (t >= C::TAPS) return 0;  // taps past the last read offset 0 (their weights are zero)
    const int dz = t / (KS * KS), dy = (t / KS) % KS, dx = t % KS;
    return (S == 1 ? dz : (dz & 1) * HZ2 + (dz >> 1)) * C::SLAB + (S == 1 ? dy : (dy & 1) * HY2 + (dy >> 1)) * C::ROW +
           (S == 1 ? dx : (dx & 1) * HX2 + (dx >> 1)) * 8;
  };
  if constexpr (AD == 2) {
    for (int t = threadIdx.x; t < C::QUADS * 4; t += NTH) tab[t] = tap_off(t);
  } else {
    for (int e = threadIdx.x; e < 2 * C::ENT; e += NTH) {
      const int h = e / C::ENT, q = e % C::ENT - 1, t = 4 * q + 2 * h;
      tab[e] = q < 0 ? 0 : (tap_off(t) >> 3) | (tap_off(t + 1) >> 3) << 16;
    }
  }
  int rowoff[C::MB];
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb) {
    const int m = wave * C::WM + mb * 32 + lrow;
    const int z = m / (TY * TX), y = (m / TX) % TY, x = m % TX;
    rowoff[mb] = z * C::SLAB + y * C::ROW + x * 8;
  }
  typedef float accv __attribute__((ext_vector_type(16)));
  accv acc[C::MB][C::NB];
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.0f;
  const int oz = tz0 * S - C::PAD, oy = ty0 * S - C::PAD, ox = tx0 * S - C::PAD;
  const int64_t pose_in = (int64_t)pose * D * D * D;
  constexpr int NV = C::HZ * C::HY * C::HX;
  constexpr int kPF = C::PF;  // past the last quad: zero weights of the padding
  const int quad_bytes = nchunks * cout_pad32 * 16 * 2;
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(wpk), (short)0, wbytes, 0x00020000);
  for (int chunk = 0; chunk < nchunks; ++chunk) {
    __syncthreads();  // the table is written / the previous chunk's halo is read
    // the chunk's channels of this pose (uniform) and the elements per voxel: voxel
    // offsets from there fit 32 bits, which keeps the per-voxel address arithmetic
    // out of 64-bit multiplies
    const bf16_t *cin0 = chunk_major ? in + ((int64_t)pose * nchunks + chunk) * D * D * D * 4
                                     : in + pose_in * cin_pad + chunk * 4;
    const int vstride = chunk_major ? 4 : cin_pad;
    // batches of HB loads in flight; the batch loop is not unrolled, so the halo
    // addressing is recomputed per chunk rather than hoisted and held in registers
#pragma unroll 1
    for (int it0 = 0; it0 < C::HITER; it0 += C::HB) {
      uint2 hv[C::HB];  // static indices only, so the batch stays in registers
#pragma unroll
      for (int i = 0; i < C::HB; ++i) {
        const int v = (it0 + i) * NTH + (int)threadIdx.x;
        hv[i] = make_uint2(0, 0);
        if (it0 + i < C::HITER && v < NV) {
          const int hx = v % C::HX, hy = (v / C::HX) % C::HY, hz = v / (C::HX * C::HY);
          const int gz = oz + hz, gy = oy + hy, gx = ox + hx;
          if ((unsigned)gz < (unsigned)D && (unsigned)gy < (unsigned)D && (unsigned)gx < (unsigned)D)
            hv[i] = *reinterpret_cast<const uint2 *>(cin0 + ((gz * D + gy) * D + gx) * vstride);
        }
      }
#pragma unroll
      for (int i = 0; i < C::HB; ++i) {
        const int v = (it0 + i) * NTH + (int)threadIdx.x;
        if (it0 + i < C::HITER && v < NV) {
          const int hx = v % C::HX, hy = (v / C::HX) % C::HY, hz = v / (C::HX * C::HY);
          const int off = stored_index(hz, C::HZ, S) * C::SLAB + stored_index(hy, C::HY, S) * C::ROW +
                          stored_index(hx, C::HX, S) * 8;
          *reinterpret_cast<uint2 *>(halo + off) = hv[i];
        }
      }
    }
    __syncthreads();
    int vb[C::NB];
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb) vb[nb] = ((chunk * cout_pad32 + n0 + nb * 32 + lrow) * 16 + khalf * 8) * 2;
    uint4 bq[kPF][C::NB];
#pragma unroll
    for (int q = 0; q < kPF; ++q)
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb)
        bq[q][nb] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb[nb], q * quad_bytes, 0));
    int soff = kPF * quad_bytes;
    // row fragments AD - 1 quads ahead: two 8-byte reads per row block (taps t, t + 1)
    uint4 ar[AD][C::MB];
    auto rows = [&](uint4 (&dst)[C::MB], int t0, int t1) {
#pragma unroll
      for (int mb = 0; mb < C::MB; ++mb) {
        const uint2 lo = *reinterpret_cast<const uint2 *>(halo + rowoff[mb] + t0);
        const uint2 hi = *reinterpret_cast<const uint2 *>(halo + rowoff[mb] + t1);
        dst[mb] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
    };
    // deep walk: packed offsets of the next eight quads to read (tw) and of the eight
    // after them (tx)
    uint4 tw[2], tx[2];
    const uint4 *tab8 = reinterpret_cast<const uint4 *>(tab + khalf * C::ENT) + 1;  // entry 4 = quad 3
    if constexpr (AD == 2) {
      rows(ar[0], tab[2 * khalf], tab[2 * khalf + 1]);
    } else {
#pragma unroll
      for (int d = 0; d < AD - 1; ++d) {
        const uint32_t t = (uint32_t)tab[khalf * C::ENT + d + 1];
        rows(ar[d], (int)(t & 0xffffu) * 8, (int)(t >> 16) * 8);
      }
      tw[0] = tab8[0];
      tw[1] = tab8[1];
    }
    auto quad = [&](const int q, const int ph) {
      if constexpr (AD == 2) {
        const int qn = q + 1 < C::QUADS ? q + 1 : q;
        rows(ar[(ph + 1) & 1], tab[4 * qn + 2 * khalf], tab[4 * qn + 2 * khalf + 1]);
      } else {
        const uint4 g = tw[ph >> 2];
        const uint32_t t = (ph & 3) == 0 ? g.x : (ph & 3) == 1 ? g.y : (ph & 3) == 2 ? g.z : g.w;
        rows(ar[(ph + AD - 1) % AD], (int)(t & 0xffffu) * 8, (int)(t >> 16) * 8);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ar[ph % AD][mb]),
                                                                 __builtin_bit_cast(bf16x8, bq[ph][nb]), acc[mb][nb],
                                                                 0, 0, 0);
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb)
        bq[ph][nb] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb[nb], soff, 0));
      soff += quad_bytes;
    };
    // whole groups of kPF quads with no test inside (so that the compiler's wait
    // analysis keeps every weight load of the ring in flight), then the rest
    constexpr int kFull = C::QUADS / kPF * kPF;
    for (int q0 = 0; q0 < kFull; q0 += kPF) {
      if constexpr (AD > 2) {
        tx[0] = tab8[q0 / 4 + 2];
        tx[1] = tab8[q0 / 4 + 3];
      }
#pragma unroll
      for (int ph = 0; ph < kPF; ++ph) quad(q0 + ph, ph);
      if constexpr (AD > 2) {
        tw[0] = tx[0];
        tw[1] = tx[1];
      }
    }
#pragma unroll
    for (int ph = 0; ph < kPF; ++ph)
      if (kFull + ph < C::QUADS) quad(kFull + ph, ph);
  }

  // ---- epilogue through LDS (as k_conv8) ----
  const int64_t pose_out = (int64_t)pose * Do * Do * Do;
  auto row_base = [&](int m, bool &valid) -> int64_t {
    const int z = tz0 + m / (TY * TX), y = ty0 + (m / TX) % TY, x = tx0 + m % TX;
    valid = z < Do && y < Do && x < Do;
    return (pose_out + ((int64_t)z * Do + y) * Do + x) * cout_store;
  };
  bf16_t *ot = reinterpret_cast<bf16_t *>(halo);  // [NW][MBG*32][NT]
  constexpr int SEG = NT / 8;
  constexpr int GR = C::MBG * 32;
#pragma unroll
  for (int g = 0; g < C::MB; g += C::MBG) {
    __syncthreads();
    if (res) {
      for (int e = threadIdx.x; e < NW * GR * SEG; e += NTH) {
        const int lr = e / SEG, qq = e % SEG;
        const int m = (lr / GR) * C::WM + g * 32 + lr % GR;
        bool valid;
        const int64_t ob = row_base(m, valid);
        if (valid && n0 + qq * 8 + 8 <= cout_store)
          *reinterpret_cast<uint4 *>(ot + lr * NT + qq * 8) = *reinterpret_cast<const uint4 *>(res + ob + n0 + qq * 8);
      }
      __syncthreads();
    }
#pragma unroll
    for (int mb = g; mb < g + C::MBG; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int lr = wave * GR + (mb - g) * 32 + 8 * (r >> 2) + 4 * khalf + (r & 3);
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) {
          const int col = nb * 32 + lrow;
          float v = acc[mb][nb][r] + bias[n0 + col];
          if (res) v += (float)ot[lr * NT + col];
          ot[lr * NT + col] = (bf16_t)(v > 0.0f ? v : 0.0f);
        }
      }
    __syncthreads();
    for (int e = threadIdx.x; e < NW * GR * SEG; e += NTH) {
      const int lr = e / SEG, qq = e % SEG;
      const int m = (lr / GR) * C::WM + g * 32 + lr % GR;
      bool valid;
      const int64_t ob = row_base(m, valid);
      if (valid && n0 + qq * 8 + 8 <= cout_store)
        *reinterpret_cast<uint4 *>(out + ob + n0 + qq * 8) = *reinterpret_cast<const uint4 *>(ot + lr * NT + qq * 8);
    }
  }
}

// ---- fp32, small tiles ------------------------------------------------------------
//
// The fp32 form of k_conv (8-channel chunks, four 32x32x2 MFMAs per block and tap, the same
// sums in the same order) with tiles small enough for two workgroups per CU: a stride-2
// 7^3 halo at 32 bytes per voxel leaves one 4 x 4 x 8 tile per CU, one wave per SIMD, whose
// LDS row read, weight loads and staging were exposed (53 % of what a float32 matrix product
// reaches here).  A wave takes one 32 x 32 block; the four waves are RW row groups x 4 / RW
// column groups.  Row fragments are read a tap ahead, weight fragments four taps ahead, and
// the next chunk's halo is loaded during the walk.  Measured at 48^3: first layer of the full
// model 501 -> 142 us for one pose, 4002 -> 2266 for 24, 37.6 -> 22.9 ms for 256; its last layer
// 1866 -> 357, 3502 -> 1968, 29.2 -> 17.7 ms; 5^3 stride-1 layers of 32 channels 247 -> 72 us for
// one pose, 6295 -> 6205 for 256.  The MFMA steps of a last chunk's absent
// channels (5 of the 19-channel grid's 24) are left out: their products are zeros.
template <int KS, int S, int TZ, int TY, int TX, int RW>
struct ConvFCfg {
  static constexpr int PAD = (KS - 1) / 2;
  static constexpr int HZ = TZ * S + KS - S, HY = TY * S + KS - S, HX = TX * S + KS - S;
  static constexpr int ROW = HX * 32 + 16, SLAB = HY * ROW, LDS = HZ * SLAB;
  static constexpr int NV = HZ * HY * HX, HITER = (NV + 255) / 256, NT = 4 / RW * 32;
  static_assert(TZ * TY * TX == 32 * RW, "a wave per 32 rows");
  static_assert(LDS <= 81920, "two workgroups per CU");
};

template <int KS, int S, int TZ, int TY, int TX, int RW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_f32(
    const float *__restrict__ in, const float *__restrict__ wpk, const float *__restrict__ bias,
    const float *__restrict__ res, float *__restrict__ out, int D, int Do, int cin, int cin_pad, int cout_pad32, int cout,
    int cout_store, int nty, int ntx, int wbytes) {
  using C = ConvFCfg<KS, S, TZ, TY, TX, RW>;
  __shared__ __attribute__((aligned(16))) char lds[C::LDS];
  int tile, pose, nblk;
  xcd_order(tile, pose, nblk);
  const int tz0 = (tile / (nty * ntx)) * TZ, ty0 = ((tile / ntx) % nty) * TY, tx0 = (tile % ntx) * TX;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, khalf = lane >> 5, lrow = lane & 31;
  const int rg = wave % RW, n0 = nblk * C::NT + wave / RW * 32;
  const int nchunks = cin_pad / 8;
  constexpr int HZ2 = S == 1 ? 0 : (C::HZ + 1) / 2, HY2 = S == 1 ? 0 : (C::HY + 1) / 2, HX2 = S == 1 ? 0 : (C::HX + 1) / 2;
  int rowoff;
  {
    const int m = rg * 32 + lrow, z = m / (TY * TX), y = (m / TX) % TY, x = m % TX;
    rowoff = z * C::SLAB + y * C::ROW + x * 32 + khalf * 16;
  }
  // this thread's halo voxels: element offset in a pose's chunk (-1: outside) and LDS offset
  int hsrc[C::HITER], hdst[C::HITER];
#pragma unroll
  for (int it = 0; it < C::HITER; ++it) {
    const int v = it * 256 + (int)threadIdx.x;
    const int hx = v % C::HX, hy = (v / C::HX) % C::HY, hz = v / (C::HX * C::HY);
    const int gz = tz0 * S - C::PAD + hz, gy = ty0 * S - C::PAD + hy, gx = tx0 * S - C::PAD + hx;
    const bool inside = (unsigned)gz < (unsigned)D && (unsigned)gy < (unsigned)D && (unsigned)gx < (unsigned)D;
    hsrc[it] = v < C::NV && inside ? ((gz * D + gy) * D + gx) * cin_pad : -1;
    hdst[it] = v < C::NV ? stored_index(hz, C::HZ, S) * C::SLAB + stored_index(hy, C::HY, S) * C::ROW +
                               stored_index(hx, C::HX, S) * 32
                         : -1;
  }
  const float *src = in + (int64_t)pose * D * D * D * cin_pad;
  float4 hl[C::HITER], hh[C::HITER];
  auto fetch = [&](int chunk) {
#pragma unroll
    for (int it = 0; it < C::HITER; ++it) {
      hl[it] = hh[it] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (hsrc[it] >= 0) {
        const float4 *q = reinterpret_cast<const float4 *>(src + hsrc[it] + chunk * 8);
        hl[it] = q[0];
        hh[it] = q[1];
      }
    }
  };
  typedef float accv __attribute__((ext_vector_type(16)));
  accv acc = {};
  const int tap_bytes = nchunks * cout_pad32 * 32;
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(wpk), (short)0, wbytes, 0x00020000);
  // one chunk's taps, STEPS channel pairs of eight channels
  auto walk = [&](auto steps_c, int chunk) {
    constexpr int STEPS = decltype(steps_c)::value;
    const int vb = ((chunk * cout_pad32 + n0 + lrow) * 8 + khalf * 4) * 4;
    constexpr int PF = 4;
    static_assert(PF <= kConvPadTaps, "prefetch past the weight padding");
    float4 b[PF];
#pragma unroll
    for (int q = 0; q < PF; ++q)
      b[q] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb, q * tap_bytes, 0));
    int soff = PF * tap_bytes;
    float4 a = *reinterpret_cast<const float4 *>(lds + rowoff);
    for (int dz = 0; dz < KS; ++dz)
      for (int dy = 0; dy < KS; ++dy) {
        const int row = (S == 1 ? dz : (dz & 1) * HZ2 + (dz >> 1)) * C::SLAB + (S == 1 ? dy : (dy & 1) * HY2 + (dy >> 1)) * C::ROW;
        // first tap of the next (dz, dy); the last one reads its own row again
        const int ny = dy + 1 < KS ? dy + 1 : 0, nz = dy + 1 < KS ? dz : (dz + 1 < KS ? dz + 1 : dz);
        const int nrow = (S == 1 ? nz : (nz & 1) * HZ2 + (nz >> 1)) * C::SLAB + (S == 1 ? ny : (ny & 1) * HY2 + (ny >> 1)) * C::ROW;
#pragma unroll
        for (int dx = 0; dx < KS; ++dx) {
          const float4 an = *reinterpret_cast<const float4 *>(
              lds + rowoff + (dx + 1 < KS ? row + (S == 1 ? dx + 1 : ((dx + 1) & 1) * HX2 + ((dx + 1) >> 1)) * 32 : nrow));
          __builtin_amdgcn_sched_barrier(0);
          const float4 w = b[0];
#pragma unroll
          for (int q = 0; q + 1 < PF; ++q) b[q] = b[q + 1];
          b[PF - 1] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(wrs, vb, soff, 0));
          soff += tap_bytes;
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, w.x, acc, 0, 0, 0);
          if constexpr (STEPS > 1) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, w.y, acc, 0, 0, 0);
          if constexpr (STEPS > 2) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, w.z, acc, 0, 0, 0);
          if constexpr (STEPS > 2) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, w.w, acc, 0, 0, 0);
          a = an;
        }
      }
  };
  fetch(0);
  for (int chunk = 0; chunk < nchunks; ++chunk) {
    if (chunk) __syncthreads();
#pragma unroll
    for (int it = 0; it < C::HITER; ++it)
      if (hdst[it] >= 0) {  // channels (0 .. 7) -> (0, 2, 4, 6 | 1, 3, 5, 7)
        float4 *dst = reinterpret_cast<float4 *>(lds + hdst[it]);
        dst[0] = make_float4(hl[it].x, hl[it].z, hh[it].x, hh[it].z);
        dst[1] = make_float4(hl[it].y, hl[it].w, hh[it].y, hh[it].w);
      }
    __syncthreads();
    if (chunk + 1 < nchunks) fetch(chunk + 1);
    if (cin - chunk * 8 > 4)
      walk(std::integral_constant<int, 4>{}, chunk);
    else
      walk(std::integral_constant<int, 2>{}, chunk);
  }
  const int n = n0 + lrow;
  if (n >= cout) return;
  const float bn = bias[n];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = rg * 32 + 8 * (r >> 2) + 4 * khalf + (r & 3);
    const int z = tz0 + m / (TY * TX), y = ty0 + (m / TX) % TY, x = tx0 + m % TX;
    if (z >= Do || y >= Do || x >= Do) continue;
    const int64_t o = (((int64_t)pose * Do + z) * Do * Do + (int64_t)y * Do + x) * cout_store + n;
    float v = acc[r] + bn;
    if (res) v += res[o];
    out[o] = v > 0.0f ? v : 0.0f;
  }
}

template <int KS, int S, int TZ, int TY, int TX, int NW, int NT>
hipError_t launch_q(const ConvLayer &L, const void *in, const void *res, void *out, int n_poses, int D,
                    hipStream_t s) {
  const int Do = (D + 2 * ((KS - 1) / 2) - KS) / S + 1;
  const int ntz = (Do + TZ - 1) / TZ, nty = (Do + TY - 1) / TY, ntx = (Do + TX - 1) / TX;
  const dim3 grid(ntz * nty * ntx, n_poses, L.cout_pad32 / NT);
  hipLaunchKernelGGL((k_conv4<KS, S, TZ, TY, TX, NW, NT>), grid, dim3(NW * 64), 0, s,
                     reinterpret_cast<const bf16_t *>(in), reinterpret_cast<const bf16_t *>(L.wpk4), L.bias,
                     reinterpret_cast<const bf16_t *>(res), reinterpret_cast<bf16_t *>(out), D, Do, L.cin_pad,
                     (L.cin + 3) / 4, L.cout_pad32, L.cout_store, nty, ntx, (int)L.wbytes4, L.in_cm4);
  return hipGetLastError();
}

template <int KS, int S, int TZ, int TY, int TX, int RW>
hipError_t launch_f(const ConvLayer &L, const void *in, const void *res, void *out, int n_poses, int D, hipStream_t s) {
  const int Do = (D + 2 * ((KS - 1) / 2) - KS) / S + 1;
  const int ntz = (Do + TZ - 1) / TZ, nty = (Do + TY - 1) / TY, ntx = (Do + TX - 1) / TX;
  const dim3 grid(ntz * nty * ntx, n_poses, L.cout_pad32 / ConvFCfg<KS, S, TZ, TY, TX, RW>::NT);
  hipLaunchKernelGGL((k_conv_f32<KS, S, TZ, TY, TX, RW>), grid, dim3(256), 0, s, reinterpret_cast<const float *>(in),
                     reinterpret_cast<const float *>(L.wpk), L.bias, reinterpret_cast<const float *>(res),
                     reinterpret_cast<float *>(out), D, Do, L.cin, L.cin_pad, L.cout_pad32, L.cout, L.cout_store, nty,
                     ntx, (int)L.wbytes);
  return hipGetLastError();
}

struct Variant {
  const char *name;
  int ks, s, tz, ty, tx, nw, nt;
  // 0: k_conv; 1: bf16 8-channel tap-pair kernel (k_conv8, weights in wpk8); 2: 4-channel tap quads (k_conv4,
  // wpk4); 3: the plain form's small tiles (k_conv_f32)
  int pairs;
  hipError_t (*launch_bf16)(const ConvLayer &, const void *, const void *, void *, int, int, hipStream_t);
  hipError_t (*launch_f32)(const ConvLayer &, const void *, const void *, void *, int, int, hipStream_t);
  int pp, blocks, wgcu;  // poses per workgroup, 32 x 32 blocks per wave, workgroups per CU (tap kernels)
};

template <int KS, int S, int TZ, int TY, int TX, int NW, int NT, int WN, int PP>
hipError_t launch_p(const ConvLayer &L, const void *in, const void *res, void *out, int n_poses, int D,
                    hipStream_t s) {
  const int Do = (D + 2 * ((KS - 1) / 2) - KS) / S + 1;
  const int ntz = (Do + TZ - 1) / TZ, nty = (Do + TY - 1) / TY, ntx = (Do + TX - 1) / TX;
  const dim3 grid(ntz * nty * ntx, (n_poses + PP - 1) / PP, L.cout_pad32 / NT);
  hipLaunchKernelGGL((k_conv8<KS, S, TZ, TY, TX, NW, NT, WN, PP>), grid, dim3(NW * 64), 0, s,
                     reinterpret_cast<const bf16_t *>(in), reinterpret_cast<const bf16_t *>(L.wpk8), L.bias,
                     reinterpret_cast<const bf16_t *>(res), reinterpret_cast<bf16_t *>(out), n_poses, D, Do, L.cin_pad,
                     (L.cin + 7) / 8, L.cout_pad32, L.cout, L.cout_store, nty, ntx, (int)L.wbytes8);
  return hipGetLastError();
}

template <typename T, int KS, int S, int TZ, int TY, int TX, int NW, int NT>
hipError_t launch_t(const ConvLayer &L, const void *in, const void *res, void *out, int n_poses, int D,
                    hipStream_t s) {
  const int Do = (D + 2 * ((KS - 1) / 2) - KS) / S + 1;
  const int ntz = (Do + TZ - 1) / TZ, nty = (Do + TY - 1) / TY, ntx = (Do + TX - 1) / TX;
  const dim3 grid(ntz * nty * ntx, n_poses, L.cout_pad32 / NT);
  hipLaunchKernelGGL((k_conv<T, KS, S, TZ, TY, TX, NW, NT>), grid, dim3(NW * 64), 0, s,
                     reinterpret_cast<const T *>(in), reinterpret_cast<const T *>(L.wpk), L.bias,
                     reinterpret_cast<const T *>(res), reinterpret_cast<T *>(out), D, Do, L.cin_pad,
                     L.cout_pad32, L.cout, L.cout_store, nty, ntx, (int)L.wbytes);
  return hipGetLastError();
}

#define CF_VARIANT(KS, S, TZ, TY, TX, NW, NT)                                                 \
  Variant {                                                                                   \
    "k" #KS "s" #S "_t" #TZ "x" #TY "x" #TX "_w" #NW "_n" #NT, KS, S, TZ, TY, TX, NW, NT, 0,   \
        &launch_t<bf16_t, KS, S, TZ, TY, TX, NW, NT>, &launch_t<float, KS, S, TZ, TY, TX, NW, NT>, 1, 0, 1 \
  }
#define CF_VARIANT8(KS, S, TZ, TY, TX, NW, NT)                                                   \
  Variant {                                                                                      \
    "p8k" #KS "s" #S "_t" #TZ "x" #TY "x" #TX "_w" #NW "_n" #NT, KS, S, TZ, TY, TX, NW, NT, 1,   \
        &launch_p<KS, S, TZ, TY, TX, NW, NT, 1, 1>, nullptr, 1,                                  \
        Conv8Cfg<KS, S, TZ, TY, TX, NW, NT, 1, 1>::BLOCKS, Conv8Cfg<KS, S, TZ, TY, TX, NW, NT, 1, 1>::WGCU \
  }
// WN waves across the columns (each wave: NT / WN columns of its row group)
#define CF_VARIANT8N(KS, S, TZ, TY, TX, NW, NT, WN)                                                      \
  Variant {                                                                                              \
    "p8k" #KS "s" #S "_t" #TZ "x" #TY "x" #TX "_w" #NW "c" #WN "_n" #NT, KS, S, TZ, TY, TX, NW, NT, 1,   \
        &launch_p<KS, S, TZ, TY, TX, NW, NT, WN, 1>, nullptr, 1,                                         \
        Conv8Cfg<KS, S, TZ, TY, TX, NW, NT, WN, 1>::BLOCKS, Conv8Cfg<KS, S, TZ, TY, TX, NW, NT, WN, 1>::WGCU \
  }
#define CF_VARIANT4(KS, S, TZ, TY, TX, NW, NT)                                                   \
  Variant {                                                                                      \
    "q4k" #KS "s" #S "_t" #TZ "x" #TY "x" #TX "_w" #NW "_n" #NT, KS, S, TZ, TY, TX, NW, NT, 2,   \
        &launch_q<KS, S, TZ, TY, TX, NW, NT>, nullptr, 1,                                        \
        Conv4Cfg<KS, S, TZ, TY, TX, NW, NT>::BLOCKS, Conv4Cfg<KS, S, TZ, TY, TX, NW, NT>::WGCU   \
  }
#define CF_VARIANTF(KS, S, TZ, TY, TX, RW)                                                       \
  Variant {                                                                                      \
    "f32k" #KS "s" #S "_t" #TZ "x" #TY "x" #TX "_w4", KS, S, TZ, TY, TX, 4, ConvFCfg<KS, S, TZ, TY, TX, RW>::NT, 3, \
        nullptr, &launch_f<KS, S, TZ, TY, TX, RW>, 1, 1, 2                                       \
  }
// ... and PP poses per workgroup
#define CF_VARIANT8P(KS, S, TZ, TY, TX, NW, NT, WN, PP)                                                           \
  Variant {                                                                                                       \
    "p8k" #KS "s" #S "_t" #TZ "x" #TY "x" #TX "_w" #NW "c" #WN "_n" #NT "_p" #PP, KS, S, TZ, TY, TX, NW, NT, 1,   \
        &launch_p<KS, S, TZ, TY, TX, NW, NT, WN, PP>, nullptr, PP,                                                \
        Conv8Cfg<KS, S, TZ, TY, TX, NW, NT, WN, PP>::BLOCKS, Conv8Cfg<KS, S, TZ, TY, TX, NW, NT, WN, PP>::WGCU    \
  }

const Variant kVariants[] = {
    CF_VARIANT(7, 1, 8, 8, 8, 4, 64),   // 0: full-model residual layers
    CF_VARIANT(7, 1, 4, 8, 8, 4, 64),   // 1
    CF_VARIANT(7, 1, 8, 8, 8, 8, 64),   // 2
    CF_VARIANT(7, 2, 4, 4, 8, 4, 64),   // 3: stride-2 layers
    CF_VARIANT(7, 2, 4, 4, 8, 4, 128),  // 4
    CF_VARIANT(7, 2, 2, 8, 8, 4, 64),   // 5
    CF_VARIANT(5, 1, 8, 8, 8, 4, 32),   // 6: tiny model
    CF_VARIANT(5, 1, 4, 8, 8, 4, 32),   // 7
    CF_VARIANT(7, 1, 4, 8, 8, 2, 64),   // 8: 128 rows per wave, two workgroups per CU
    CF_VARIANT(7, 2, 4, 4, 8, 2, 64),   // 9
    CF_VARIANT(7, 2, 4, 4, 8, 2, 128),  // 10
    CF_VARIANT(7, 2, 2, 8, 8, 2, 64),   // 11
    CF_VARIANT8(7, 1, 8, 8, 8, 4, 64),  // 12: tap pairs, 128 rows per wave
    CF_VARIANT8(7, 1, 4, 8, 8, 4, 64),  // 13
    CF_VARIANT8(7, 1, 4, 8, 8, 2, 64),  // 14
    CF_VARIANT8(7, 2, 4, 4, 8, 4, 64),  // 15
    CF_VARIANT8(7, 2, 4, 8, 8, 4, 64),  // 16
    CF_VARIANT8(7, 2, 4, 4, 8, 4, 128), // 17
    CF_VARIANT8(7, 2, 4, 8, 8, 4, 128), // 18
    CF_VARIANT8(5, 1, 8, 8, 8, 4, 32),  // 19
    CF_VARIANT8(7, 2, 8, 8, 8, 4, 64),  // 20: stride-2 first layer, 512-row tile
    CF_VARIANT8(7, 1, 8, 8, 8, 8, 64),  // 21
    CF_VARIANT8(7, 2, 4, 4, 12, 6, 128), // 22: 12^3 outputs of a 24^3 input in 9 whole tiles
    // 5^3 and 3^3 kernels (the paper-shaped model: 32 filters of 5^3, 64 of 3^3)
    CF_VARIANT8(5, 2, 8, 8, 8, 4, 32),   // 23
    CF_VARIANT8(5, 2, 4, 8, 8, 4, 32),   // 24
    CF_VARIANT8(5, 1, 4, 8, 8, 2, 32),   // 25
    CF_VARIANT8(3, 1, 8, 8, 8, 4, 64),   // 26
    CF_VARIANT8(3, 1, 4, 8, 8, 4, 64),   // 27
    CF_VARIANT8(3, 2, 8, 8, 8, 4, 64),   // 28
    CF_VARIANT8(3, 2, 4, 8, 8, 4, 64),   // 29
    CF_VARIANT(5, 2, 4, 8, 8, 4, 32),    // 30
    CF_VARIANT(3, 1, 8, 8, 8, 4, 64),    // 31
    CF_VARIANT(3, 1, 4, 8, 8, 4, 64),    // 32
    CF_VARIANT(3, 2, 4, 8, 8, 4, 64),    // 33
    CF_VARIANT(3, 2, 4, 4, 8, 4, 64),    // 34
    // stride-2 tiles whose halo allows one workgroup per CU: eight waves hide more latency
    CF_VARIANT8(7, 2, 8, 8, 8, 8, 64),   // 35
    CF_VARIANT8(7, 2, 4, 8, 8, 8, 128),  // 36
    CF_VARIANT8(5, 2, 8, 8, 8, 8, 32),   // 37
    // 128-column stride-2 layers with the columns split over two waves (64 rows x
    // 64 columns per wave: half the weight-fragment loads per MFMA of 17/22)
    CF_VARIANT8N(7, 2, 4, 4, 12, 6, 128, 2),  // 38: 12^3 outputs in 9 whole tiles
    CF_VARIANT8N(7, 2, 4, 4, 8, 4, 128, 2),   // 39
    // two poses per workgroup: 384 rows share each weight fragment (the 5.6 MB of
    // weights of the 64 -> 128 layer exceed an XCD's L2, so weight traffic per row
    // sets its speed); 12^3 outputs in 9 whole tiles
    CF_VARIANT8P(7, 2, 4, 4, 12, 8, 128, 2, 2),   // 40
    // 4-channel tap quads for the 19-channel grid
    CF_VARIANT4(7, 2, 8, 8, 8, 4, 64),   // 41: 21^3 halo at 8 bytes per voxel, two workgroups per CU
    CF_VARIANT4(5, 2, 8, 8, 8, 4, 32),   // 42
    CF_VARIANT4(5, 1, 8, 8, 8, 4, 32),   // 43
    CF_VARIANT4(7, 1, 8, 8, 8, 4, 32),   // 44  (the bf16 grid is read by tap-quad kernels only: one per
    CF_VARIANT4(3, 1, 8, 8, 8, 4, 32),   // 45   first-layer shape)
    CF_VARIANT4(3, 2, 8, 8, 8, 4, 32)    // 46
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

// Finer tiles for batches that leave the chip idle at the variants above, then the plain
// form's small tiles (64 columns before 32).  Their ids follow the frequency-domain path's,
// so that the ids callers may have stored stay what they were.
const Variant kFineTiles[] = {
    CF_VARIANT8N(7, 2, 4, 4, 4, 4, 64, 2),   // 12^3 outputs exactly, one 32 x 32 block per wave
    CF_VARIANT8N(3, 1, 4, 4, 4, 4, 64, 2),
    CF_VARIANT8N(3, 2, 4, 4, 4, 4, 64, 2),
    CF_VARIANT8(5, 1, 4, 4, 8, 4, 32),
    CF_VARIANT4(7, 2, 4, 4, 8, 4, 64),
    CF_VARIANT4(5, 2, 4, 4, 8, 4, 32),
    CF_VARIANT4(5, 1, 4, 4, 8, 4, 32),
    CF_VARIANTF(7, 2, 4, 4, 4, 2),
    CF_VARIANTF(5, 2, 4, 4, 4, 2),
    CF_VARIANTF(3, 2, 4, 4, 4, 2),
    CF_VARIANTF(7, 1, 4, 4, 4, 2),
    CF_VARIANTF(5, 1, 4, 4, 4, 2),
    CF_VARIANTF(3, 1, 4, 4, 4, 2),
    CF_VARIANTF(5, 2, 4, 4, 8, 4),
    CF_VARIANTF(3, 2, 4, 4, 8, 4),
    CF_VARIANTF(7, 1, 4, 4, 8, 4),
    CF_VARIANTF(5, 1, 4, 4, 8, 4),
    CF_VARIANTF(3, 1, 4, 4, 8, 4)
};
constexpr int kNumFine = sizeof(kFineTiles) / sizeof(kFineTiles[0]);
// one id past the direct kernels: the frequency-domain path
constexpr int kFftVariant = kNumVariants;

// the direct kernel of an id (null: the frequency-domain path, or no such id)
const Variant *variant_of(int v) {
  if (v >= 0 && v < kNumVariants) return &kVariants[v];
  return v > kFftVariant && v <= kFftVariant + kNumFine ? &kFineTiles[v - kFftVariant - 1] : nullptr;
}

bool tap_kernel_ok(const Variant &V, const ConvLayer &L) {
  if (V.ks != L.k || V.s != L.stride || L.cout_pad32 % V.nt != 0) return false;
  return V.pairs == 2 ? L.wpk4 && L.cin_pad % 4 == 0 : V.pairs == 1 && L.wpk8 && L.cin_pad % 8 == 0;
}

// Estimated time of a tap kernel, in cycles per K step: rounds of resident workgroups,
// each as long as the matrix cores of its fullest CU need, but no less than one step
// takes a lone workgroup.  Measured: the matrix cores reach 60 % with eight 32 x 32
// blocks per wave, 50 % with four to six, 42 % with two and 33 % with one (each block
// then reads its own row and weight fragment); a lone workgroup's step is ~550 cycles
// with big tiles, 120 with fine ones and 250 with fine tap quads (their halo loads).
double tile_cost(const Variant &V, const ConvLayer &L, int Do, int n_poses) {
  constexpr int kCUs = 256;
  const int64_t tiles = (int64_t)((Do + V.tz - 1) / V.tz) * ((Do + V.ty - 1) / V.ty) * ((Do + V.tx - 1) / V.tx);
  const int64_t wg = tiles * ((n_poses + V.pp - 1) / V.pp) * (L.cout_pad32 / V.nt);
  const double busy = V.blocks >= 8 ? 0.6 : V.blocks >= 4 ? 0.5 : V.blocks >= 2 ? 0.42 : 0.33;
  const double step = V.blocks * 32.0 * (V.nw > 4 ? V.nw / 4.0 : 1.0) / busy;
  const double lat = V.blocks > 2 ? 550.0 : V.pairs == 2 ? 250.0 : 120.0;
  auto round = [&](int64_t per_cu) { return std::max(lat, per_cu * step); };
  const int64_t full = wg / (kCUs * V.wgcu), rest = wg % (kCUs * V.wgcu);
  return full * round(V.wgcu) + (rest ? round((rest + kCUs - 1) / kCUs) : 0.0);
}

// The tile for a batch of n_poses: the variant itself, unless another tile of the same
// kernel is estimated a tenth faster.  Tiles of one kernel add the same products in
// the same order, so the choice changes no result (a pose scores the same in any batch).
// Measured, 64 -> 128 7^3 stride-2 layer, 384-row tiles of two poses against 64 x 64
// tiles: 411 / 73 us for one 24^3 pose (9 workgroups of the big tile on 256 CUs), 492 /
// 381 for 24, 537 / 539 for 40, 996 / 873 for 64 (a second round), 1065 / 671 for 19 poses
// of 32^3; first layer, 512- against 128-row tiles: 110 / 51 us for one pose, 120 / 75 for four.
int fit_tile(int v, const ConvLayer &L, int D_in, int n_poses) {
  const Variant &V = *variant_of(v);
  const int Do = (D_in + 2 * ((L.k - 1) / 2) - L.k) / L.stride + 1;
  int best = v;
  double cost = 0.9 * tile_cost(V, L, Do, n_poses);
  auto consider = [&](int id) {
    const Variant &C = *variant_of(id);
    if (C.pairs != V.pairs || !tap_kernel_ok(C, L)) return;
    const double t = tile_cost(C, L, Do, n_poses);
    if (t < cost) {
      cost = t;
      best = id;
    }
  };
  for (int i = 0; i < kNumFine; ++i) consider(kFftVariant + 1 + i);
  for (int i = 0; i < kNumVariants; ++i) consider(i);
  return best;
}

}  // namespace

int conv_num_variants() { return kNumVariants + 1 + kNumFine; }
const char *conv_variant_name(int v) {
  const Variant *V = variant_of(v);
  return V ? V->name : (v == kFftVariant ? "fft32" : "?");
}

bool conv_variant_ok(int v, const ConvLayer &L, int bf16, int D_in) {
  if (v == kFftVariant) return (bf16 ? !L.spec_f32 : L.spec_f32) && fft_conv_ok(L, D_in);
  const Variant *p = variant_of(v);
  if (!p) return false;
  const Variant &V = *p;
  if (V.pairs == 1 || V.pairs == 2) return bf16 && tap_kernel_ok(V, L);
  if (V.pairs == 3 && bf16) return false;
  const int cc = bf16 ? 16 : 8;
  return V.ks == L.k && V.s == L.stride && L.cout_pad32 % V.nt == 0 && L.cin_pad % cc == 0;
}

int conv_default_variant(const ConvLayer &L, int D_in, int bf16) {
  // measured on MI355X at 48^3: 7^3 stride-1 layers in the frequency domain (bf16:
  // 3x the tap-pair kernel), tap quads for the 19-channel first layer, tap pairs
  // for the 128-column stride-2 layer (two poses per workgroup); fp32 has no tap
  // kernels
  if (L.k == 7 && conv_variant_ok(kFftVariant, L, bf16, D_in)) return kFftVariant;
  const int pref[] = {12, 40, 41, 17, 20, 19, 23, 26, 28, 4, 3, 6, 1, 0, 2, 5, 7, 8, 9, 10, 11, 13, 14, 15, 16, 18,
                      21, 22, 24, 25, 27, 29, 30, 31, 32, 33, 34, 35, 36, 37, 38, 39, 42, 43, 44, 45, 46};
  for (int v : pref)
    if (conv_variant_ok(v, L, bf16, D_in)) return v;
  return -1;
}

bool conv_variant_is_fft(int v) { return v == kFftVariant; }

int64_t conv_work_bytes(int v, const ConvLayer &L, int D_in, int n_poses) {
  return v == kFftVariant ? fft_conv_work_bytes(L, D_in, n_poses) : 0;
}

namespace {
// Seeded values uniform in [0, 0.5) (SplitMix64 finaliser of seed + index): the
// autotuner times kernels on data that toggles like real activations, since
// the chip sustains a higher clock on constant operands.
__global__ __launch_bounds__(256) void k_fill_random(void *p, int64_t n, int bf16, uint64_t seed) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    uint64_t z = seed + (uint64_t)i * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    const float v = (float)(z >> 40) * (0.5f / 16777216.0f);
    if (bf16)
      reinterpret_cast<bf16_t *>(p)[i] = (bf16_t)v;
    else
      reinterpret_cast<float *>(p)[i] = v;
  }
}
}  // namespace

hipError_t launch_fill_random(void *p, int64_t bytes, int bf16, uint64_t seed, hipStream_t s) {
  const int64_t n = bytes / (bf16 ? 2 : 4);
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 16384);
  hipLaunchKernelGGL(k_fill_random, dim3((unsigned)blocks), dim3(256), 0, s, p, n, bf16, seed);
  return hipGetLastError();
}

int conv_fit_variant(int v, const ConvLayer &L, int bf16, int D_in, int n_poses) {
  const Variant *V = variant_of(v);
  if (!V || !conv_variant_ok(v, L, bf16, D_in)) return v;
  if (bf16) return V->pairs ? fit_tile(v, L, D_in, n_poses) : v;
  // the plain form's small tiles are the faster ones at every batch size measured (1 .. 256
  // poses, see k_conv_f32)
  for (int i = 0; i < kNumFine; ++i)
    if (kFineTiles[i].pairs == 3 && conv_variant_ok(kFftVariant + 1 + i, L, bf16, D_in)) return kFftVariant + 1 + i;
  return v;
}

hipError_t launch_conv(int variant, const ConvLayer &L, int bf16, const void *in, const void *res,
                       void *out, int n_poses, int D_in, void *work, hipStream_t s) {
  if (!conv_variant_ok(variant, L, bf16, D_in)) return hipErrorInvalidValue;
  if (variant == kFftVariant) return launch_fft_conv(L, in, res, out, n_poses, D_in, work, s);
  const Variant &V = *variant_of(variant);
  return bf16 ? V.launch_bf16(L, in, res, out, n_poses, D_in, s) : V.launch_f32(L, in, res, out, n_poses, D_in, s);
}

}  // namespace cf
