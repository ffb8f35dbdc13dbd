// Covalent and non-covalent neighbour lists by exact integer distance tests.
//
// The SG-CNN reads a spatial graph with two edge types chosen by distance
// threshold (Sec. 1; thresholds are hyper-parameters, Table I / Table II).  An
// edge (i, j) exists for i != j in the same pose when |x_i - x_j|^2 <= r^2 with
// coordinates and r in 2^-10 A integers, so the lists are exact.
//
// Design: a workgroup takes 64 atoms i of one pose (one per lane of each of its
// four waves) and sweeps all atoms j of the pose through a 1024-atom LDS tile that
// every lane reads at one address (a broadcast).  The waves share the sweep by
// 32-atom words of j and each lane gathers its hits of a word in a bit mask, with
// no branch and no store inside the sweep; the columns of a row are then the set
// bits in ascending order, so nothing is sorted.  Pass 1 counts the bits (degrees),
// per-pose totals are scanned into edge offsets, and pass 2 sweeps again and writes
// the rows from the masks.
//
// What bounds it: the n^2 tests on the vector ALUs.  One workgroup per pose (each
// thread an atom i, branching to a store per hit) left a single pose on one CU and a
// ragged batch waiting for its largest pose: 512 poses of 200-1500 atoms took 547 us
// to count and 1110 us to fill (134 and 170 here, 1.8e12 tests/s), one 690-atom pose
// 112 + 290 us (14 + 17).
//
// Exactness.  16-bit form (10 instructions a test): coordinates relative to the middle
// of the block's 64 atoms, saturated to 16 bits; saturating packed differences and two
// 2-way dot products give the sum of squares, < 3 * 2^30.  With every atom i of the
// block within 32766 - r of the middle on each axis, an atom j that saturates is more
// than r away from each of them, in truth and as computed, and the rest is exact.  A
// block that spans more (27 A to either side at the usual cutoffs), and every block at a
// cutoff above 32766 u, which a saturated difference does not exceed, takes the 32-bit form
// (15 instructions; the whole batch in it: 174 + 204 us): |x_i - x_j| of two int32 is an exact unsigned 32-bit number
// (v_sad_u32 on offset-binary values); clamped to C = r + 1 per axis, the sum of
// squares is exact where it decides (all axes <= r) and above r^2 where an axis was
// clamped.  For 3 C^2 < 2^32 (r <= 37836 u, 36.9 A) it takes 24-bit multiplies and
// 32-bit sums, above that 64-bit ones.
#include "cf_internal.h"
#include "cf_launch.h"

namespace cf {

namespace {

constexpr int kThreads = 256;
constexpr int kRows = 64;            // atoms i of a workgroup
constexpr int kTile = 1024;          // atoms of the j tile in LDS (16 KB)
constexpr int kWords = kTile / 32;   // mask words of a tile
constexpr int kParts = kThreads / kRows;
constexpr int kR32 = 37836;          // largest cutoff of the 32-bit form: 3 (r + 1)^2 < 2^32

typedef short short2v __attribute__((ext_vector_type(2)));

struct GraphShared {
  union {
    uint4 tile[kTile];     // offset-binary coordinates
    uint2 tile16[kTile];   // 16-bit coordinates from the block's middle: (x, y), (z, 0)
  };
  uint32_t mask[2][kWords][kRows];  // [covalent, non-covalent][word of j][atom i]
  int cnt[2][kParts][kRows];
  long long red[2][kThreads / 64];
};

// The pose of work item `it` (a pose and a first block of kRows atoms): atoms a0 ..
// a0 + n - 1, n = 0 for a malformed pose (reported once, by the pose's first item).
__device__ inline int item_pose(const int32_t *__restrict__ atom_off, int n_atoms, int p0, int pl, int base,
                                bool report, int &a0, int64_t *status) {
  int a1;
  const bool ok = pose_range(atom_off, p0 + pl, n_atoms, a0, a1) && a0 >= base;
  if (!ok && report) dev_fail(status, kDevBadOffsets);
  if (a0 < base) a0 = a1 = base;
  const int n = a1 - a0;
  if (n < 0 || n > CF_MAX_POSE_ATOMS) {
    if (report) dev_fail(status, n < 0 ? kDevBadOffsets : kDevPoseTooLarge);
    return 0;
  }
  return n;
}

// offset-binary coordinates (unsigned order = signed order)
__device__ inline uint4 atom_pos(const int32_t *__restrict__ xyz, int64_t a) {
  const int32_t *q = xyz + 3 * a;
  return make_uint4((uint32_t)q[0] ^ 0x80000000u, (uint32_t)q[1] ^ 0x80000000u, (uint32_t)q[2] ^ 0x80000000u, 0);
}

// |a - b|, exact for any two values (one instruction; the compiler makes three of it)
__device__ inline uint32_t abs_diff(uint32_t a, uint32_t b) {
  uint32_t d;
  asm("v_sad_u32 %0, %1, %2, 0" : "=v"(d) : "v"(a), "v"(b));
  return d;
}

// The frame of a block for the 16-bit form: the middle of its atoms' bounding box,
// and whether all of them lie within reach of it (every wave holds the same 64 atoms
// and gets the same answer).
struct Frame {
  uint32_t mx, my, mz;
  bool ok;
};
__device__ inline Frame block_frame(uint4 me, uint32_t r_nc) {
  uint32_t lo[3] = {me.x, me.y, me.z}, hi[3] = {me.x, me.y, me.z};
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      lo[d] = min(lo[d], (uint32_t)__shfl_xor((int)lo[d], o, 64));
      hi[d] = max(hi[d], (uint32_t)__shfl_xor((int)hi[d], o, 64));
    }
  Frame f;
  f.mx = lo[0] + (hi[0] - lo[0]) / 2;
  f.my = lo[1] + (hi[1] - lo[1]) / 2;
  f.mz = lo[2] + (hi[2] - lo[2]) / 2;
  // a cutoff above 32766 lets no block through, not even one whose atoms share a place
  const uint32_t reach = 32766u - r_nc;
  f.ok = r_nc <= 32766u && hi[0] - f.mx <= reach && hi[1] - f.my <= reach && hi[2] - f.mz <= reach;
  return f;
}
__device__ inline int sat16(uint32_t q, uint32_t m) {
  const int64_t d = (int64_t)q - m;
  return d < -32768 ? -32768 : d > 32767 ? 32767 : (int)d;
}
__device__ inline uint2 to_frame(const Frame &f, uint4 q) {
  return make_uint2((uint32_t)(uint16_t)sat16(q.x, f.mx) | (uint32_t)sat16(q.y, f.my) << 16,
                    (uint32_t)(uint16_t)sat16(q.z, f.mz));
}

// Masks of the tile's atoms j0 .. j0 + jn - 1 within r_nc / r_cov of this lane's atom
// i (index in the pose), its own bit cleared: S.mask[.][word][lane].  Called by all
// threads between barriers; wave w takes words w, w + 4, ...
// FORM: 16 (me16, tile16), 32 or 64.
template <int FORM>
__device__ inline void sweep_form(GraphShared &S, uint4 me, uint2 me16, int i, int j0, int jn, uint32_t r_cov,
                                  uint32_t r_nc) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t C = r_nc + 1;
  const int words = (jn + 31) / 32;
  const short2v mxy = __builtin_bit_cast(short2v, me16.x), mz = __builtin_bit_cast(short2v, me16.y);
  for (int k = wave; k < words; k += kThreads / 64) {
    uint32_t mc = 0, mn = 0;
    // eight atoms at a time, their bits as small constants
#pragma unroll 1
    for (int g = 0; g < 32; g += 8) {
      uint32_t gc = 0, gn = 0;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        bool hc, hn;
        if constexpr (FORM == 16) {
          const uint2 q = S.tile16[k * 32 + g + b];
          const short2v dxy = __builtin_elementwise_sub_sat(__builtin_bit_cast(short2v, q.x), mxy);
          const short2v dz = __builtin_elementwise_sub_sat(__builtin_bit_cast(short2v, q.y), mz);
          const uint32_t D = (uint32_t)__builtin_amdgcn_sdot2(dxy, dxy, __builtin_amdgcn_sdot2(dz, dz, 0, false), false);
          hc = D <= r_cov * r_cov;
          hn = D <= r_nc * r_nc;
        } else {
          const uint4 q = S.tile[k * 32 + g + b];
          const uint32_t ax = min(abs_diff(q.x, me.x), C), ay = min(abs_diff(q.y, me.y), C), az = min(abs_diff(q.z, me.z), C);
          if constexpr (FORM == 32) {
            const uint32_t D = __umul24(ax, ax) + __umul24(ay, ay) + __umul24(az, az);
            hc = D <= r_cov * r_cov;
            hn = D <= r_nc * r_nc;
          } else {
            const unsigned long long D =
                (unsigned long long)ax * ax + (unsigned long long)ay * ay + (unsigned long long)az * az;
            hc = D <= (unsigned long long)r_cov * r_cov;
            hn = D <= (unsigned long long)r_nc * r_nc;
          }
        }
        gc |= hc ? 1u << b : 0u;
        gn |= hn ? 1u << b : 0u;
      }
      mc |= gc << g;
      mn |= gn << g;
    }
    const int left = jn - k * 32;
    const uint32_t live = left >= 32 ? 0xffffffffu : (1u << left) - 1u;
    const int self = i - j0 - k * 32;
    const uint32_t keep = live & ~(self >= 0 && self < 32 ? 1u << self : 0u);
    S.mask[0][k][lane] = mc & keep;
    S.mask[1][k][lane] = mn & keep;
  }
}

// Stages atoms j0 .. j0 + jn - 1 and sweeps them, in the 16-bit form where the block's
// frame allows it (the answer is the same for every wave).
template <bool R32>
__device__ inline void sweep(GraphShared &S, const int32_t *__restrict__ xyz, int a0, uint4 me, const Frame &f, int i,
                             int j0, int jn, uint32_t r_cov, uint32_t r_nc) {
  __syncthreads();  // the tile and the masks are free
  for (int t = threadIdx.x; t < (jn + 31) / 32 * 32; t += kThreads) {
    const uint4 q = t < jn ? atom_pos(xyz, (int64_t)a0 + j0 + t) : make_uint4(0, 0, 0, 0);
    if (f.ok)
      S.tile16[t] = to_frame(f, q);
    else
      S.tile[t] = q;
  }
  __syncthreads();
  if (f.ok)
    sweep_form<16>(S, me, to_frame(f, me), i, j0, jn, r_cov, r_nc);
  else
    sweep_form<R32 ? 32 : 64>(S, me, make_uint2(0, 0), i, j0, jn, r_cov, r_nc);
}

// Pass 1: degrees.  Work items (pose, block) in a grid-stride loop; a pose of more
// than nbx blocks gives each of its items several.  WHOLE (nbx = 1): an item is a whole pose
// and writes its edge totals too.
template <bool R32, bool WHOLE>
__global__ __launch_bounds__(kThreads) void k_graph_count(const int32_t *__restrict__ atom_off, int n_atoms,
                                                          const int32_t *__restrict__ xyz, int p0, int n_poses,
                                                          int nbx, int r_cov, int r_nc,
                                                          int32_t *__restrict__ deg,  // [2][n_chunk_cap]
                                                          int64_t n_chunk_cap, int64_t *__restrict__ pose_tot,
                                                          int64_t *status) {
  __shared__ GraphShared S;
  const int base = atom_off[p0];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t it = blockIdx.x; it < (int64_t)n_poses * nbx; it += gridDim.x) {
    const int pl = (int)(it / nbx), b0 = (int)(it % nbx);
    int a0;
    const int n = item_pose(atom_off, n_atoms, p0, pl, base, b0 == 0 && threadIdx.x == 0, a0, status);
    long long tot = 0;  // edges of this lane's atoms, by waves 0 and 1
    for (int i0 = b0 * kRows; i0 < n; i0 += nbx * kRows) {
      const int i = i0 + lane;
      const uint4 me = atom_pos(xyz, (int64_t)a0 + (i < n ? i : i0));
      const Frame f = block_frame(me, (uint32_t)r_nc);
      int cc = 0, cn = 0;
      for (int j0 = 0; j0 < n; j0 += kTile) {
        const int jn = min(n - j0, kTile);
        sweep<R32>(S, xyz, a0, me, f, i, j0, jn, r_cov, r_nc);
        // a lane's own words, as its wave wrote them
        for (int k = wave; k < (jn + 31) / 32; k += kThreads / 64) {
          cc += __popc(S.mask[0][k][lane]);
          cn += __popc(S.mask[1][k][lane]);
        }
      }
      S.cnt[0][wave][lane] = cc;
      S.cnt[1][wave][lane] = cn;
      __syncthreads();
      const int64_t li = (int64_t)(a0 - base) + i;
      if (wave < 2 && i < n && li < n_chunk_cap) {
        int d = 0;
        for (int w = 0; w < kParts; ++w) d += S.cnt[wave][w][lane];
        deg[wave * n_chunk_cap + li] = d;
        if constexpr (WHOLE) tot += d;
      }
    }
    if (WHOLE && wave < 2) {
      for (int o = 32; o >= 1; o >>= 1) tot += __shfl_xor(tot, o, 64);
      if (lane == 0) pose_tot[(int64_t)wave * n_poses + pl] = tot;
    }
  }
}

// Edge totals of a pose from its degrees, by one wave
__device__ inline void pose_totals(const int32_t *__restrict__ deg, int64_t n_chunk_cap, int64_t lb, int n, int lane,
                                   long long &tc, long long &tn) {
  tc = tn = 0;
  const int64_t end = lb + n < n_chunk_cap ? lb + n : n_chunk_cap;
#pragma unroll 4
  for (int64_t q = lb + lane; q < end; q += 64) {
    tc += deg[q];
    tn += deg[n_chunk_cap + q];
  }
  for (int o = 32; o >= 1; o >>= 1) {
    tc += __shfl_xor(tc, o, 64);
    tn += __shfl_xor(tn, o, 64);
  }
}

__global__ __launch_bounds__(kThreads) void k_graph_tot(const int32_t *__restrict__ atom_off, int n_atoms, int p0,
                                                        int n_poses, const int32_t *__restrict__ deg,
                                                        int64_t n_chunk_cap, int64_t *__restrict__ pose_tot) {
  const int base = atom_off[p0];
  const int lane = threadIdx.x & 63;
  const int pl = (int)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (pl >= n_poses) return;
  int a0;
  const int n = item_pose(atom_off, n_atoms, p0, pl, base, false, a0, nullptr);
  long long tc, tn;
  pose_totals(deg, n_chunk_cap, (int64_t)(a0 - base), n, lane, tc, tn);
  if (lane == 0) {
    pose_tot[pl] = tc;
    pose_tot[n_poses + pl] = tn;
  }
}

// Exclusive scan of per-pose edge totals (one workgroup); writes the closing
// row_ptr entries and checks capacities.  With TOT the totals are summed here, a
// wave per pose (few poses: one launch less).
template <bool TOT>
__global__ __launch_bounds__(1024) void k_graph_scan(const int32_t *__restrict__ atom_off, int n_atoms, int p0,
                                                     int n_poses, const int32_t *__restrict__ deg, int64_t n_chunk_cap,
                                                     int64_t *__restrict__ pose_tot,
                                                     int32_t *cov_row, int64_t cov_cap, int32_t *nc_row,
                                                     int64_t nc_cap, int64_t *status) {
  __shared__ long long tmp[2][1024];
  if (TOT) {
    const int base = atom_off[p0];
    for (int pl = threadIdx.x >> 6; pl < n_poses; pl += 16) {
      int a0;
      const int n = item_pose(atom_off, n_atoms, p0, pl, base, false, a0, nullptr);
      long long tc, tn;
      pose_totals(deg, n_chunk_cap, (int64_t)(a0 - base), n, threadIdx.x & 63, tc, tn);
      if ((threadIdx.x & 63) == 0) {
        pose_tot[pl] = tc;
        pose_tot[n_poses + pl] = tn;
      }
    }
    __threadfence_block();
    __syncthreads();
  }
  long long carry[2] = {0, 0};
  for (int b0 = 0; b0 < n_poses; b0 += 1024) {
    const int p = b0 + threadIdx.x;
    for (int t = 0; t < 2; ++t) tmp[t][threadIdx.x] = p < n_poses ? pose_tot[t * n_poses + p] : 0;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      long long v[2];
      for (int t = 0; t < 2; ++t) v[t] = threadIdx.x >= o ? tmp[t][threadIdx.x - o] : 0;
      __syncthreads();
      for (int t = 0; t < 2; ++t) tmp[t][threadIdx.x] += v[t];
      __syncthreads();
    }
    for (int t = 0; t < 2; ++t) {
      const long long incl = tmp[t][threadIdx.x];
      const long long own = p < n_poses ? pose_tot[t * n_poses + p] : 0;
      if (p < n_poses) pose_tot[(2 + t) * n_poses + p] = carry[t] + incl - own;  // exclusive offset
    }
    __syncthreads();
    for (int t = 0; t < 2; ++t) carry[t] += tmp[t][1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const int64_t nchunk = (int64_t)atom_off[p0 + n_poses] - atom_off[p0];
    const bool over = carry[0] > cov_cap || carry[1] > nc_cap || carry[0] > INT32_MAX || carry[1] > INT32_MAX;
    if (over) {
      dev_fail(status, kDevCapacity);
      atomicMax(reinterpret_cast<unsigned long long *>(status + 1), (unsigned long long)carry[0]);
      atomicMax(reinterpret_cast<unsigned long long *>(status + 2), (unsigned long long)carry[1]);
    }
    if (nchunk >= 0 && nchunk <= n_chunk_cap) {
      cov_row[nchunk] = (int32_t)(carry[0] > INT32_MAX ? INT32_MAX : carry[0]);
      nc_row[nchunk] = (int32_t)(carry[1] > INT32_MAX ? INT32_MAX : carry[1]);
    } else {
      dev_fail(status, kDevBadOffsets);
    }
  }
}

// Pass 2: rows.  Workgroups as in pass 1; the part w of a lane's atom i (wave w)
// writes the columns of a quarter of the tile's words.  A row is written only if it
// fits its capacity whole.
template <bool R32>
__global__ __launch_bounds__(kThreads) void k_graph_fill(const int32_t *__restrict__ atom_off, int n_atoms,
                                                         const int32_t *__restrict__ xyz, int p0, int n_poses, int nbx,
                                                         int r_cov, int r_nc, const int32_t *__restrict__ deg,
                                                         int64_t n_chunk_cap, const int64_t *__restrict__ pose_tot,
                                                         int32_t *__restrict__ cov_row, int32_t *__restrict__ cov_col,
                                                         int64_t cov_cap, int32_t *__restrict__ nc_row,
                                                         int32_t *__restrict__ nc_col, int64_t nc_cap,
                                                         int64_t *status) {
  __shared__ GraphShared S;
  const int base = atom_off[p0];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t it = blockIdx.x; it < (int64_t)n_poses * nbx; it += gridDim.x) {
    const int pl = (int)(it / nbx), b0 = (int)(it % nbx);
    int a0;
    const int n = item_pose(atom_off, n_atoms, p0, pl, base, false, a0, nullptr);  // reported by pass 1
    const int lb = a0 - base;
    for (int i0 = b0 * kRows; i0 < n; i0 += nbx * kRows) {
      // first slots of the block: the pose's offset and the degrees of its earlier atoms
      long long pc = 0, pn = 0;
      for (int q = threadIdx.x; q < i0; q += kThreads)
        if ((int64_t)lb + q < n_chunk_cap) {
          pc += deg[lb + q];
          pn += deg[n_chunk_cap + lb + q];
        }
      for (int o = 32; o >= 1; o >>= 1) {
        pc += __shfl_xor(pc, o, 64);
        pn += __shfl_xor(pn, o, 64);
      }
      __syncthreads();  // the previous block's reads of S are done
      if (lane == 0) {
        S.red[0][wave] = pc;
        S.red[1][wave] = pn;
      }
      __syncthreads();
      int64_t run[2] = {pose_tot[2 * n_poses + pl], pose_tot[3 * n_poses + pl]};
      for (int w = 0; w < kThreads / 64; ++w) {
        run[0] += S.red[0][w];
        run[1] += S.red[1][w];
      }
      const int i = i0 + lane;
      const bool act = i < n && (int64_t)lb + i < n_chunk_cap;
      int d[2] = {act ? deg[lb + i] : 0, act ? deg[n_chunk_cap + lb + i] : 0};
      int ex[2] = {d[0], d[1]};
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(ex[0], o, 64), v = __shfl_up(ex[1], o, 64);
        if (lane >= o) {
          ex[0] += u;
          ex[1] += v;
        }
      }
      const int64_t s0[2] = {run[0] + ex[0] - d[0], run[1] + ex[1] - d[1]};
      if (wave == 0 && act) {
        cov_row[lb + i] = (int32_t)(s0[0] > INT32_MAX ? INT32_MAX : s0[0]);
        nc_row[lb + i] = (int32_t)(s0[1] > INT32_MAX ? INT32_MAX : s0[1]);
      }
      const bool fits[2] = {act && s0[0] + d[0] <= cov_cap, act && s0[1] + d[1] <= nc_cap};
      const uint4 me = atom_pos(xyz, (int64_t)a0 + (i < n ? i : i0));
      const Frame f = block_frame(me, (uint32_t)r_nc);
      int done[2] = {0, 0};  // columns of the earlier tiles
      for (int j0 = 0; j0 < n; j0 += kTile) {
        const int jn = min(n - j0, kTile), words = (jn + 31) / 32;
        sweep<R32>(S, xyz, a0, me, f, i, j0, jn, r_cov, r_nc);
        __syncthreads();
        const int wper = (words + kParts - 1) / kParts, k0 = wave * wper, k1 = min(words, k0 + wper);
        int c[2] = {0, 0};
        for (int k = k0; k < k1; ++k) {
          c[0] += __popc(S.mask[0][k][lane]);
          c[1] += __popc(S.mask[1][k][lane]);
        }
        S.cnt[0][wave][lane] = c[0];
        S.cnt[1][wave][lane] = c[1];
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          int at = done[t];
          for (int w = 0; w < kParts; ++w) {
            const int m = S.cnt[t][w][lane];
            if (w < wave) at += m;
            done[t] += m;
          }
          if (!fits[t]) continue;
          int32_t *col = (t ? nc_col : cov_col) + s0[t];
          for (int k = k0; k < k1; ++k)
            for (uint32_t m = S.mask[t][k][lane]; m; m &= m - 1) {
              if (at < d[t]) col[at] = lb + j0 + k * 32 + __ffs((int)m) - 1;
              ++at;
            }
        }
      }
    }
  }
}

}  // namespace

hipError_t launch_graph(const int32_t *atom_off, int n_atoms, const int32_t *xyz, int p0, int n_poses, int mean_atoms,
                        int r_cov, int r_nc, int32_t *cov_row, int32_t *cov_col, int64_t cov_cap, int32_t *nc_row,
                        int32_t *nc_col, int64_t nc_cap, int32_t *deg_scratch, int64_t n_chunk_cap,
                        int64_t *pose_scratch, int64_t *status, hipStream_t s) {
  // deg_scratch: 2 * n_chunk_cap ints; pose_scratch: 4 * n_poses int64
  if (n_poses <= 0) return hipSuccess;
  // items per pose: blocks for poses up to twice the mean (larger ones loop), never
  // more than the largest pose has
  const int nbx = pose_blocks(n_atoms, mean_atoms, kRows);
  const dim3 grid(item_groups((int64_t)n_poses * nbx));
  const bool small = r_nc <= kR32;
  const bool whole = nbx == 1;  // poses of one block each: totals with the degrees
#define CF_COUNT(R32, WHOLE)                                                                                        \
  hipLaunchKernelGGL((k_graph_count<R32, WHOLE>), grid, dim3(kThreads), 0, s, atom_off, n_atoms, xyz, p0, n_poses, nbx, \
                     r_cov, r_nc, deg_scratch, n_chunk_cap, pose_scratch, status)
  if (small) {
    if (whole) CF_COUNT(true, true); else CF_COUNT(true, false);
  } else {
    if (whole) CF_COUNT(false, true); else CF_COUNT(false, false);
  }
#undef CF_COUNT
  // Totals of larger poses: inside the scan's 16 waves while that is at most two poses a wave,
  // else a launch of their own.  Inside and apart, for ragged poses of 200-1500 atoms: one pose
  // 22.4 and 23.4 us for the whole build, 16 poses 35.5 and 36.6, 19 poses 64.3 and 64.8, 32
  // poses 70.3 and 69.1.  (300 poses of 12 atoms: 21.9 us apart, 18.7 with the degrees.)
  if (n_poses <= 32 && !whole) {
    hipLaunchKernelGGL(k_graph_scan<true>, dim3(1), dim3(1024), 0, s, atom_off, n_atoms, p0, n_poses, deg_scratch,
                       n_chunk_cap, pose_scratch, cov_row, cov_cap, nc_row, nc_cap, status);
  } else {
    if (!whole)
      hipLaunchKernelGGL(k_graph_tot, dim3((n_poses + 3) / 4), dim3(kThreads), 0, s, atom_off, n_atoms, p0, n_poses,
                         deg_scratch, n_chunk_cap, pose_scratch);
    hipLaunchKernelGGL(k_graph_scan<false>, dim3(1), dim3(1024), 0, s, atom_off, n_atoms, p0, n_poses, deg_scratch,
                       n_chunk_cap, pose_scratch, cov_row, cov_cap, nc_row, nc_cap, status);
  }
  if (small)
    hipLaunchKernelGGL(k_graph_fill<true>, grid, dim3(kThreads), 0, s, atom_off, n_atoms, xyz, p0, n_poses, nbx, r_cov,
                       r_nc, deg_scratch, n_chunk_cap, pose_scratch, cov_row, cov_col, cov_cap, nc_row, nc_col, nc_cap,
                       status);
  else
    hipLaunchKernelGGL(k_graph_fill<false>, grid, dim3(kThreads), 0, s, atom_off, n_atoms, xyz, p0, n_poses, nbx, r_cov,
                       r_nc, deg_scratch, n_chunk_cap, pose_scratch, cov_row, cov_col, cov_cap, nc_row, nc_col, nc_cap,
                       status);
  return hipGetLastError();
}

}  // namespace cf
