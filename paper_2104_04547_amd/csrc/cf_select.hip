// Selection after scoring: best pose per compound and top-k compounds.
//
// In the paper's screen each compound has up to 10 docked poses per binding site
// (40 over four sites) and is represented by its strongest prediction -- the
// maximum Coherent Fusion pK over its poses (Sec. 5.2); compounds are then ranked
// and the best few purchased for assays (the 100-of-1,000,000 example, Sec. 3.4).
//
// cf_compound_max: a group of 8 lanes per segment (64 for long segments), NaN scores are
// ignored, ties go to the lowest pose index.
// cf_top_k: exact selection on 64-bit keys (order-preserving 32-bit image of
// the value, then the complemented index, so every key is distinct and the
// ranking is "value descending, index ascending").
//   * up to 65,536 values: one workgroup, up to 16,384 of them in registers.  The k-th largest
//     of its 1024 threads' maxima bounds the k-th largest value from below; the few values
//     at or above it are ranked.  Where too many are (ties, or values in an order that
//     defeats the bound), histograms narrow the k-th value's range and ties are counted in
//     the order of their indices.
//   * more: radix select, 8 passes of an 8-bit digit histogram and the digit's choice (passes
//     after the key is certain return at once), one pass collects the keys at or above the
//     k-th, and a single workgroup sorts those k keys.
// What bounds it: launches, and latency on one CU.  For 50,000 values 19 launches took 75 us
// (102 us with the maxima of 50,000 segments of 10^6 scores before them), one takes 23
// (27), of which reading the values twice on one CU is about ten.  Results are
// deterministic.
#include <algorithm>
#include <cfloat>
#include <climits>
#include <mutex>

#include "cf_internal.h"
#include "cf_launch.h"
#include "cf_topk_pick.h"

namespace cf {

namespace {

constexpr int kSelThreads = 256;

__device__ inline uint64_t topk_key(float v, int i) {
  uint32_t u = v == 0.0f ? 0u : __float_as_uint(v);  // -0 and +0 are the same value
  uint32_t k;
  if (v != v)
    k = 0u;  // NaN ranks last
  else
    k = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((uint64_t)k << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)i);
}

// LPS lanes per segment; lane q takes the scores q, q + LPS, ... and the lanes' maxima are
// merged (the lowest index wins a tie)
template <int LPS>
__global__ __launch_bounds__(kSelThreads) void k_segmax(const float *__restrict__ scores, int n_scores,
                                                        const int32_t *__restrict__ off, int n_seg,
                                                        float *__restrict__ best, int32_t *__restrict__ best_idx,
                                                        int64_t *status) {
  const int q = threadIdx.x % LPS;
  const int64_t t = (blockIdx.x * (int64_t)kSelThreads + threadIdx.x) / LPS, step = (int64_t)gridDim.x * kSelThreads / LPS;
  for (int64_t seg_id = t; seg_id < n_seg; seg_id += step) {  // whole groups
    const int c = (int)seg_id;
    int a = off[c], b = off[c + 1];
    if (a < 0 || b < a || b > n_scores) {
      if (q == 0) dev_fail(status, kDevBadOffsets);
      a = b = 0;
    }
    float m = -FLT_MAX;
    int idx = -1;
    // counted from the segment's start, unsigned: past the end of one that ends near 2^31 too
    const uint32_t len = (uint32_t)(b - a);
    const float *seg = scores + a;
    for (uint32_t d = 0; d < len; d += 4 * LPS) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t p = d + u * LPS + q;
        v[u] = p < len ? seg[p] : __builtin_nanf("");
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (v[u] == v[u] && (idx < 0 || v[u] > m)) {
          m = v[u];
          idx = (int)(d + u * LPS + q);
        }
    }
#pragma unroll
    for (int o = LPS / 2; o >= 1; o >>= 1) {
      const float mo = __shfl_xor(m, o, LPS);
      const int io = __shfl_xor(idx, o, LPS);
      if (io >= 0 && (idx < 0 || mo > m || (mo == m && io < idx))) {
        m = mo;
        idx = io;
      }
    }
    if (q == 0) {
      best[c] = idx < 0 ? -INFINITY : m;
      best_idx[c] = idx < 0 ? -1 : a + idx;
    }
  }
}

// bitonic sort of m (a power of two) keys in LDS by nth threads, descending
__device__ inline void sort_keys(uint64_t *s, int m, int nth) {
  for (int size = 2; size <= m; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < m; i += nth) {
        const int j = i ^ stride;
        if (j > i) {
          const bool desc = (i & size) == 0;
          const uint64_t a = s[i], b = s[j];
          if (desc ? (a < b) : (a > b)) {
            s[i] = b;
            s[j] = a;
          }
        }
      }
      __syncthreads();
    }
}

// ---- up to kSmallN values: one workgroup ----

// Candidates beyond kSmallCap are narrowed first: a pass over 50,000 values takes about 7 us,
// a sort of 2048 keys 20 and one of 8192 115.  Every call measured (n 1,024 .. 65,536, k 1 ..
// 1024, random, sorted, rounded and equal values) is below the separate launches' 57 - 123 us:
// the 1024 best of 50,000 random values 60 us, of equal ones 53.
constexpr int kSmallT = 1024, kSmallN = 64 * kSmallT, kSmallCap = 2048;
// keys that are ranked by counting instead of sorted: a wave reads all of them, so the
// count grows with the square; a sort of 256 is 36 steps with a barrier each
constexpr int kSmallRank = 256;

// 1 <= k <= min(n, 1024).  HOLD: n <= E * 1024 and a thread keeps its E values; else it
// reads them again for each pass, E at a time (64 values do not fit beside their range
// tests: spilled and unrolled they took 26 us for 50,000 values).
template <int E, bool HOLD>
__global__ __launch_bounds__(kSmallT) void k_topk_small(const float *__restrict__ v, int n, int k,
                                                       int32_t *__restrict__ idx_out, float *__restrict__ val_out) {
  __shared__ uint64_t cand[kSmallCap];
  __shared__ uint32_t thr, top;
  __shared__ int cnt, pick[3], wsum[kSmallT / 64];
  __shared__ int bin[kSmallN / 64];  // counts of a digit's 256 values, or of the 64-index groups
  const int tid = threadIdx.x, lane = tid & 63;
  uint32_t key[E];  // images of the values e * 1024 + tid; 0 past the end (as a NaN's, but never counted)
  // buffer loads: past the end of the values they return zero, which takes the whole offset
  // in the vector operand (the scalar one is not part of the range check)
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(v), (short)0, n * 4, 0x00020000);
  auto load = [&](int base) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      key[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, (base + e * kSmallT + tid) * 4, 0, 0);
#pragma unroll
    for (int e = 0; e < E; ++e)
      key[e] = base + e * kSmallT + tid < n ? (uint32_t)(topk_key(__uint_as_float(key[e]), 0) >> 32) : 0u;
  };
  if constexpr (HOLD) load(0);
  // f(image, index) of this thread's values
  auto each = [&](auto f) {
    const int batches = HOLD ? 1 : (n + E * kSmallT - 1) / (E * kSmallT);
    for (int q = 0; q < batches; ++q) {
      if constexpr (!HOLD) load(q * E * kSmallT);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = (q * E + e) * kSmallT + tid;
        if (i < n) f(key[e], i);
      }
    }
  };
  uint32_t mx = 0;
  each([&](uint32_t y, int) { mx = y > mx ? y : mx; });
  uint32_t *maxima = reinterpret_cast<uint32_t *>(cand);
  maxima[tid] = mx;
  if (tid == 0) cnt = 0;
  __syncthreads();
  if (tid < 64) {  // the k-th largest of the maxima: the largest t that at least k of them reach
    uint32_t q[kSmallT / 64];
#pragma unroll
    for (int u = 0; u < kSmallT / 64; ++u) q[u] = maxima[u * 64 + lane];
    uint32_t t = 0;
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t c = t | 1u << bit;
      int have = 0;
#pragma unroll
      for (int u = 0; u < kSmallT / 64; ++u) have += __popcll(__ballot(q[u] >= c));
      if (have >= k) t = c;
      if (have == k) {  // exactly these: the smallest of them
        uint32_t least = 0xFFFFFFFFu;
#pragma unroll
        for (int u = 0; u < kSmallT / 64; ++u) least = q[u] >= c && q[u] < least ? q[u] : least;
        for (int o = 32; o >= 1; o >>= 1) least = min(least, (uint32_t)__shfl_xor((int)least, o, 64));
        t = least;
        break;
      }
    }
    uint32_t most = 0;
#pragma unroll
    for (int u = 0; u < kSmallT / 64; ++u) most = q[u] > most ? q[u] : most;
    for (int o = 32; o >= 1; o >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, o, 64));
    if (lane == 0) {
      thr = t;
      top = most;
    }
  }
  __syncthreads();
  const uint32_t lo = thr;
  // keys at or above the bound (each key's slot is arbitrary: they are sorted)
  auto take = [&](uint32_t y, int i) {
    const int slot = atomicAdd(&cnt, 1);
    if (slot < kSmallCap) cand[slot] = ((uint64_t)y << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)i);
  };
  each([&](uint32_t y, int i) {
    if (y >= lo) take(y, i);
  });
  __syncthreads();
  int m = cnt;
  if (m > kSmallCap) {
    // Too many: the range [lo2, hi2] of the k-th largest image is split 256-fold, by a
    // histogram of the images in it, until few enough keys reach its lower end or it is a
    // single image, of which the keys with the lowest indices are taken.  The keys of a wave
    // that share the first one's digit are added together: where many are too many, they
    // are mostly equal.
    uint32_t lo2 = lo, hi2 = top;
    int krem = k, reach = m;  // the krem-th largest of the range is sought; keys at or above lo2
    while (reach > kSmallCap && lo2 != hi2) {
      const int shift = max(0, 24 - __clz((int)(hi2 - lo2)));
      if (tid < 256) bin[tid] = 0;
      __syncthreads();
      each([&](uint32_t y, int) {
        if (y < lo2 || y > hi2) return;
        const int d = (int)((y - lo2) >> shift);
        const uint64_t same = __ballot(d == __builtin_amdgcn_readfirstlane(d));
        if (!(same >> lane & 1))
          atomicAdd(&bin[d], 1);
        else if (lane == __ffsll((unsigned long long)same) - 1)
          atomicAdd(&bin[d], __popcll(same));
      });
      __syncthreads();
      if (tid < 64) {
        int own[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) sum += own[u] = bin[4 * lane + u];
        int at = sum;  // keys of this lane's digits and of larger ones
        for (int o = 1; o < 64; o <<= 1) {
          const int w = __shfl_down(at, o, 64);
          if (lane + o < 64) at += w;
        }
        int above = at - sum;
#pragma unroll
        for (int u = 3; u >= 0; --u) {
          if (above < krem && above + own[u] >= krem) {  // exactly one digit
            pick[0] = 4 * lane + u;
            pick[1] = above;
            pick[2] = own[u];
          }
          above += own[u];
        }
      }
      __syncthreads();
      lo2 += (uint32_t)pick[0] << shift;
      hi2 = lo2 + min(hi2 - lo2, (1u << shift) - 1u);
      krem -= pick[1];
      reach = k - krem + pick[2];
    }
    const bool ties = reach > kSmallCap;  // of image lo2, of which the first krem indices are taken
    if (ties) {
      // the ties before each group of 64 indices (one wave's share of one load)
      each([&](uint32_t y, int i) {
        const uint64_t b = __ballot(y == lo2);
        if (lane == 0) bin[i >> 6] = __popcll(b);
      });
      __syncthreads();
      const int own = tid * 64 < n ? bin[tid] : 0;
      int in = own;
      for (int o = 1; o < 64; o <<= 1) {
        const int w = __shfl_up(in, o, 64);
        if (lane >= o) in += w;
      }
      if (lane == 63) wsum[tid >> 6] = in;
      __syncthreads();
      int before = in - own;
      for (int w = 0; w < tid >> 6; ++w) before += wsum[w];
      bin[tid] = before;
    }
    if (tid == 0) cnt = 0;
    __syncthreads();
    each([&](uint32_t y, int i) {
      bool mine = y >= lo2;
      if (ties) {
        const uint64_t b = __ballot(y == lo2);
        if (y == lo2) mine = bin[i >> 6] + __popcll(b & ((1ull << lane) - 1ull)) < krem;
      }
      if (mine) take(y, i);
    });
    __syncthreads();
    m = cnt;
  }
  if (m <= kSmallRank) {
    // few: a key's rank is the number of keys above it (all keys differ), with no barrier
    if (tid < m) {
      const uint64_t mine = cand[tid];
      int r = 0;
#pragma unroll 8
      for (int i = 0; i < m; ++i) r += cand[i] > mine ? 1 : 0;
      if (r < k) {
        const int j = (int)(0xFFFFFFFFu - (uint32_t)(mine & 0xFFFFFFFFu));
        idx_out[r] = j;
        if (val_out) val_out[r] = v[j];
      }
    }
    return;
  }
  int p2 = 1;
  while (p2 < m) p2 <<= 1;
  for (int i = m + tid; i < p2; i += kSmallT) cand[i] = 0ull;
  __syncthreads();
  sort_keys(cand, p2, kSmallT);
  for (int i = tid; i < k; i += kSmallT) {
    const int j = (int)(0xFFFFFFFFu - (uint32_t)(cand[i] & 0xFFFFFFFFu));
    idx_out[i] = j;
    if (val_out) val_out[i] = v[j];
  }
}

// ---- more values: radix select ----

// state: see topk_pick
__global__ void k_topk_init(uint32_t *hist, uint64_t *state, int k) {
  for (int i = threadIdx.x; i < 256; i += blockDim.x) hist[i] = 0;
  if (threadIdx.x < 6) state[threadIdx.x] = threadIdx.x == 2 ? (uint64_t)k : 0;
}

// Histogram of one digit of the keys under the prefix
__global__ __launch_bounds__(kSelThreads) void k_topk_hist(const float *__restrict__ v, int n, int shift,
                                                           uint32_t *hist, const uint64_t *state) {
  __shared__ uint32_t h[256];
  if (state[5]) return;
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t prefix = state[0], mask = state[1];
  for (int64_t i = blockIdx.x * (int64_t)kSelThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kSelThreads) {
    const uint64_t key = topk_key(v[i], (int)i);
    if ((key & mask) == prefix) atomicAdd(&h[(key >> shift) & 0xFF], 1u);
  }
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

// The digit whose bucket holds the k-th largest key, a thread per digit (one workgroup); the
// histogram is cleared for the next pass.  A launch of its own: picked by the last workgroup
// of the histogram's launch, each of that launch's workgroups made its counts visible to all
// eight XCDs first, and the 100 best of 1,000,000 values took 211 us in place of 116.
__global__ __launch_bounds__(256) void k_topk_digit(uint32_t *hist, uint64_t *state, int shift) {
  __shared__ uint32_t h[256];
  const uint64_t prefix = state[0], mask = state[1], krem = state[2], certain = state[5];
  const uint32_t own = hist[threadIdx.x];
  h[threadIdx.x] = own;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {  // suffix sums over the digits
    const uint32_t add = threadIdx.x + o < 256 ? h[threadIdx.x + o] : 0u;
    __syncthreads();
    h[threadIdx.x] += add;
    __syncthreads();
  }
  if (certain) return;
  topk_pick(prefix, mask, krem, threadIdx.x, shift, own, h[threadIdx.x], state);
  hist[threadIdx.x] = 0;
}

__global__ __launch_bounds__(kSelThreads) void k_topk_collect(const float *__restrict__ v, int n, uint64_t *state,
                                                              uint64_t *cand, int k) {
  const uint64_t thr = state[0];  // exactly k keys are at or above it (all keys are distinct)
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint64_t key = topk_key(v[i], i);
    if (key >= thr) {
      const unsigned long long slot = atomicAdd(reinterpret_cast<unsigned long long *>(&state[3]), 1ull);
      if (slot < (unsigned long long)k) cand[slot] = key;
    }
  }
}

// bitonic sort of k <= 1024 keys (padded to a power of two with zeros), descending
__global__ __launch_bounds__(1024) void k_topk_sort(const uint64_t *cand, int k, const float *__restrict__ v,
                                                    int32_t *idx_out, float *val_out) {
  __shared__ uint64_t s[1024];
  int m = 1;
  while (m < k) m <<= 1;
  for (int i = threadIdx.x; i < m; i += blockDim.x) s[i] = i < k ? cand[i] : 0ull;
  __syncthreads();
  sort_keys(s, m, 1024);
  for (int i = threadIdx.x; i < k; i += blockDim.x) {
    const int idx = (int)(0xFFFFFFFFu - (uint32_t)(s[i] & 0xFFFFFFFFu));
    idx_out[i] = idx;
    if (val_out) val_out[i] = v[idx];
  }
}

}  // namespace

hipError_t launch_segmax(const float *scores, int n_scores, const int32_t *off, int n_seg, float *best,
                         int32_t *best_idx, int64_t *status, hipStream_t s) {
  if (n_seg <= 0) return hipSuccess;
  // 8 lanes per segment (a compound has up to 40 poses), a wave where segments are long; a
  // launch has fewer than 2^32 threads, so the workgroups of more segments take several
  const int lps = (int64_t)n_scores > 128 * (int64_t)n_seg ? 64 : 8;
  const unsigned blocks = item_groups(((int64_t)n_seg * lps + kSelThreads - 1) / kSelThreads);
  if (lps == 64)
    hipLaunchKernelGGL(k_segmax<64>, dim3(blocks), dim3(kSelThreads), 0, s, scores, n_scores, off, n_seg, best, best_idx,
                       status);
  else
    hipLaunchKernelGGL(k_segmax<8>, dim3(blocks), dim3(kSelThreads), 0, s, scores, n_scores, off, n_seg, best, best_idx,
                       status);
  return hipGetLastError();
}

// Scratch of the allocation-free top-k: the 256-bin histogram (1 KB), the select
// state (64 B) and the k <= 1024 collected keys (8 KB).  One copy per GPU, held
// until the process ends; every allocation-free call on a GPU shares it.
static __device__ __align__(256) unsigned char scratch[kTopkScratchBytes];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of the current device's copy of `scratch`, looked up once per
// device (the array's name in host code is a host-side stand-in, not a device
// address).  Later calls read the cached pointer.
hipError_t topk_static_scratch(void **out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_topk(const float *v, int n, int k, int32_t *idx_out, float *val_out, void *scratch,
                       hipStream_t s) {
  if (n <= kSmallN && k <= kTopkMaxK) {
    if (n <= 4 * kSmallT)
      hipLaunchKernelGGL((k_topk_small<4, true>), dim3(1), dim3(kSmallT), 0, s, v, n, k, idx_out, val_out);
    else if (n <= 16 * kSmallT)
      hipLaunchKernelGGL((k_topk_small<16, true>), dim3(1), dim3(kSmallT), 0, s, v, n, k, idx_out, val_out);
    else
      hipLaunchKernelGGL((k_topk_small<32, false>), dim3(1), dim3(kSmallT), 0, s, v, n, k, idx_out, val_out);
    return hipGetLastError();
  }
  uint32_t *hist = reinterpret_cast<uint32_t *>(scratch);
  uint64_t *state = reinterpret_cast<uint64_t *>(reinterpret_cast<char *>(scratch) + 1024);
  uint64_t *cand = reinterpret_cast<uint64_t *>(reinterpret_cast<char *>(scratch) + 1024 + 64);
  const int blocks = (int)std::min<int64_t>(1024, ((int64_t)n + kSelThreads - 1) / kSelThreads);
  hipLaunchKernelGGL(k_topk_init, dim3(1), dim3(256), 0, s, hist, state, k);
  for (int shift = 56; shift >= 0; shift -= 8) {
    hipLaunchKernelGGL(k_topk_hist, dim3(blocks), dim3(kSelThreads), 0, s, v, n, shift, hist, state);
    hipLaunchKernelGGL(k_topk_digit, dim3(1), dim3(256), 0, s, hist, state, shift);
  }
  hipLaunchKernelGGL(k_topk_collect, dim3(blocks), dim3(kSelThreads), 0, s, v, n, state, cand, k);
  hipLaunchKernelGGL(k_topk_sort, dim3(1), dim3(1024), 0, s, cand, k, v, idx_out, val_out);
  return hipGetLastError();
}

}  // namespace cf
