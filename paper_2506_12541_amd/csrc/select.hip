// Group selection (Section 2.2, Eq. 10-12 with the importance scores of Eq. 6 and the
// top-k of Eq. 7): every contiguous group of g queries pools its real queries into
// q_p = (1/g) * sum q_t, scores every compressed key by the unscaled product <q_p, k_c>,
// scores each selection block of r = l'/l compressed blocks by the mean of their scores,
// excludes blocks of the group's own ball and blocks without a real token, and keeps the
// k* best blocks (higher score first, lower block index on equal scores), stored in
// ascending block order with -1 in unused slots.
//
// Scores are the f32 sums of six bf16 matrix products of the operands' three parts (x = hi +
// mid + lo up to 2^-27 |x|; the products whose weight reaches 2^-16), key by key, and a block's
// score is the mean of its keys': f32 accuracy, whatever the layer's storage type, so equal
// scores (and those closer than f32 rounding) rank by block index alike in every path below.
//
// The score matrix (N/g x N/l' per head) is never stored, and only the few blocks that can be
// among the k* best are scored. A workgroup owns 64 groups of one head, 16 per wave; the block
// keys (the sum of a block's compressed keys, less a vector common to the head's blocks, which
// shifts every score of a group alike) are streamed twice in tiles shared by its waves:
//   1. Scores from unit vectors in f16 (one MFMA per 32 dimensions), times the key's norm,
//      less a bound on their error: a lower bound of each block's score. Every lane keeps
//      the largest of each of a few disjoint sets of blocks; the k*-th largest of a
//      group's set maxima bounds its k*-th best score from below.
//   2. The same scores plus the bound: blocks that reach the group's threshold (about
//      1.15 k* of them; every block of the k* best is one) go to the wave's list.
//   3. The listed blocks are scored by f32 dots of the pooled query and the summed keys and
//      ranked within their group. Groups where a block of the k* best lies above one of the rest
//      by no more than the errors of their scores (about one in thirty) are ranked again by the
//      six products, 16 keys at a time as the rows of a product whose columns are the wave's
//      groups; elsewhere the six products give the same k* best. The selected blocks are ordered
//      by block index.
// Groups whose list overflows (e.g. all scores equal) and zero queries are left over: their
// workgroup then streams the compressed keys once, in three bf16 parts through LDS, scores
// every block for them and keeps a running top-k per lane, merged at the end. Heads whose keys
// are nearly equal, so that every list would overflow, skip the two streams.
// The common vector is a trimmed mean of blocks sampled over the head: without it, a component
// that all keys share (a bias, slowly varying features) widens the bound below, though it cannot
// change a ranking, until the lists overflow (65536 queries in groups of 16, keys N(0, 1) plus a
// common vector 20 times as long: 0.39 ms, with it 0.12). Any vector would do, so a few blocks serve.
// Error of a unit-vector score against the score it stands for, in units of |q| times the
// block's norm bound w = max(|its vector|, sum of its keys' norms / 16) (an upper bound of
// the vector's length serves as its scale): f16 rounds each of the two operands by at most 2^-11
// of its magnitude, so by Cauchy-Schwarz the product errs by at most 2^-10 (+ 2^-22); the
// vectors are scaled by 2^7, which keeps what f16 cannot hold (below 2^-24, or below 2^-14
// if subnormal numbers were flushed) under 2^-17; f32 sums and norms add under 2^-17. The score
// from six products errs by at most 2^-15 |q| (sum of the keys' norms) (224 sums of at most
// |q||k| in two 32-dimension steps, each off by an ulp at most), so by 2^-11 |q| w. kUnitErr
// is 1.6 * 2^-10.
// A dot errs by at most 12 * 2^-24 |q| |sum of the keys| (11 roundings, one in the summed key);
// kDotErr adds the six products' 2^-15.
// What bounds it: at 65536 queries in groups of 16 (two waves per SIMD) the latency of each tile
// and of the ranking, issue taking 26% of the time; with more waves VALU issue (75 instructions per
// 64 blocks and 16 groups in both streams, about 3000 per 16 groups for the ranking).
// Measured with its preparation, k* = 16, d = 64, r = 2, N(0, 1) tensors (in brackets: one
// stream of all compressed keys with the six products and a 16-deep list in every lane): 65536
// queries x 8 heads in groups of 16 0.10 ms (0.27), one by one 0.91 (2.73); 2^20 queries x 16
// heads in groups of 32 4.8 ms (15.7). Two sets of 16 groups per wave, which halve the LDS reads
// per group, left fewer waves (the kernel alone at 65536 queries 0.109 instead of 0.074 ms, one
// by one 0.86 instead of 0.82). With every group left over (keys N(0, 1) plus a common
// vector 1000 times as long) the three take 0.27, 3.0 and 18 ms.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "attn_common.hpp"

namespace bsa {
namespace {

constexpr int kWaves = 4;
constexpr int kFlat = 512;                // listed blocks of a wave (about 18 per group for k* = 16)
constexpr int kRing = 4, kAhead = 3;     // key tiles in LDS; of these, loads in flight
constexpr int kPerGroup = 64;             // listed blocks of a group
constexpr int kNoBlock = 0x7FFFFFFF;
constexpr float kUnit = 128.0f;           // scale of the f16 unit vectors
constexpr float kUnitErr = 1.6f / 1024 * kUnit * kUnit;
constexpr float kSpread = 1.0f / 16;      // least norm bound of a block, over the sum of its keys' norms
// Heads whose blocks' vectors are shorter than this share of their keys' norms skip the filter: its
// error bound, held up by kSpread, is then 7 times that of spread keys and lists overflow (a common
// vector 100 times as long as the keys at 65536 queries: 0.28 ms, 0.40 with the filter first).
constexpr float kEqual = 1.0f / 112;
constexpr float kDotErr = 1.0f / 32768 + 12.0f / (1 << 24);

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint32_t ordered_bits(float x) {
  x = x + 0.0f;
  uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The score of a key.
__device__ __forceinline__ float key_score(uint64_t key) {
  const uint32_t b = (uint32_t)(key >> 32);
  return __uint_as_float((b & 0x80000000u) ? (b & 0x7FFFFFFFu) : ~b);
}

// Keys order by score, then lower block first (blocks have 20 bits: N <= 2^24, l' >= 16); the low
// nine bits name the block's entry in its wave's list.
__device__ __forceinline__ uint64_t make_key(float score, int blk, int entry = 0) {
  return ((uint64_t)ordered_bits(score) << 32) | (uint64_t)(((0xFFFFFu - (uint32_t)blk) << 9) + (uint32_t)entry);
}
__device__ __forceinline__ int key_block(uint64_t key) { return (int)(0xFFFFFu - ((uint32_t)key >> 9)); }

// Insert x into the descending list (keys are unique, x > lst[K - 1]): every entry compares
// with x independently, then each slot keeps its entry, takes x, or takes its upper
// neighbour (slots are rewritten from the bottom, so the neighbour is still the old one).
template <int K>
__device__ __forceinline__ void topk_insert(uint64_t (&lst)[K], uint64_t x) {
  bool gt[K];
#pragma unroll
  for (int t = 0; t < K; ++t) gt[t] = lst[t] > x;
#pragma unroll
  for (int t = K - 1; t >= 1; --t) lst[t] = gt[t] ? lst[t] : (gt[t - 1] ? x : lst[t - 1]);
  lst[0] = gt[0] ? lst[0] : x;
}

// Over the group's four lanes L, L ^ 16, L ^ 32, L ^ 48.
__device__ __forceinline__ uint64_t group_min(uint64_t x) {
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    const uint64_t y = __shfl_xor(x, o, 64);
    x = x < y ? x : y;
  }
  return x;
}
__device__ __forceinline__ uint64_t group_max(uint64_t x) {
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    const uint64_t y = __shfl_xor(x, o, 64);
    x = x > y ? x : y;
  }
  return x;
}

// Rows of HD values, one 8-value chunk per lane of HD / 8 lanes, to f16 unit vectors times
// 2^7, and the row's norm (0 for a zero row, whose vector is zero; a row that is not
// finite gives NaN products). Scaling by a power of two first keeps the sum of squares in
// range for any magnitude.
template <typename MaxF, typename SumF>
__device__ __forceinline__ float unit_scale(const float* x, int n, int& e, MaxF rmax, SumF rsum) {
  float mx = 0.f;
  for (int i = 0; i < n; ++i) mx = fmaxf(mx, fabsf(x[i]));
  mx = rmax(mx);
  e = mx > 0.f ? __builtin_amdgcn_frexp_expf(mx) : 0;
  float ss = 0.f;
  for (int i = 0; i < n; ++i) {
    const float y = ldexpf(x[i], -e);
    ss += y * y;
  }
  ss = rsum(ss);
  return ss;
}

// Preparation of the selection in one launch. Workgroups below `pool_blocks`: pooled
// queries (Eq. 11), q_p = (1/g) * sum of the group's real queries in slot order, eight
// channels per thread (HBM: one read of Q in 16-byte loads; a thread per channel took 33
// instead of 14 us at 65536 queries x 8 heads of 64). The others: the sum of every selection
// block's compressed keys in f32 (ksum, not written for r = 1: kcmp holds them), less the head's
// common vector and over its norm bound (see above) in f16, the negated norm bound and the sum of
// its keys' norms (kabs), HD / 8 threads per block; blocks without a real token get the norms NaN,
// which no comparison passes. A head's norm bounds are padded with NaN to a whole tile of the
// selection kernel. Every workgroup forms its head's common vector from the same 16 blocks (a
// launch of its own for it would cost more than the loads): per channel the mean without the
// smallest and the largest. Heads whose blocks all fit the candidate lists do without. The
// head's first workgroup notes whether most sampled blocks are as good as equal (flags).
template <typename T, int HD>
__global__ void __launch_bounds__(256) select_prep_kernel(const T* __restrict__ q, const uint8_t* __restrict__ valid,
                                                          int H, int lgn, int lgg, long long pool_n8, int pool_blocks,
                                                          float* __restrict__ qpool, const float* __restrict__ kcmp,
                                                          const uint8_t* __restrict__ cvalid, int lgb, int lgr,
                                                          long long blocks, uint16_t* __restrict__ kunit,
                                                          float* __restrict__ knorm, float* __restrict__ kabs,
                                                          float* __restrict__ ksum, int* __restrict__ flags) {
  constexpr int CPR = HD / 8, NS = 16;   // sampled blocks
  static_assert(2 * kFlat / 16 >= 256 / CPR, "heads with a common vector hold whole workgroups");
  __shared__ float sample[NS][HD], common[HD];
  if ((int)blockIdx.x < pool_blocks) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= pool_n8) return;
    const int c = (int)(i % CPR) * 8, g = 1 << lgg;
    const long long tok = (i / CPR) << lgg;   // (b*H + h) * N + the group's first slot
    const T* qr = q + tok * HD + c;
    const uint8_t* vb =
        valid ? valid + ((long long)((uint32_t)(tok >> lgn) / (uint32_t)H) << lgn) + (tok & ((1LL << lgn) - 1))
              : nullptr;
    float s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = 0.f;
#pragma unroll 8
    for (int t = 0; t < g; ++t) {
      const typename Chunk<T>::type v = load_chunk(qr + (size_t)t * HD);
      const bool ok = vb == nullptr || vb[t];
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] = ok ? s[e] + (float)v[e] : s[e];
    }
    f32x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = s[e] / (float)g;
    *reinterpret_cast<f32x8*>(qpool + 8 * i) = o;
    return;
  }
  const long long i = (long long)(blockIdx.x - pool_blocks) * 256 + threadIdx.x;
  if (i >= blocks * CPR) return;   // whole rows: 256 is a multiple of CPR
  const long long blk = i / CPR;   // (b*H + h) * nblk + block, nblk = 2^lgb
  const int r = 1 << lgr, c = 8 * (int)(i % CPR);
  const int nblk = 1 << lgb;
  const bool centred = nblk > kFlat / 16;   // (then the workgroup's blocks are of one head)
  const int row = (int)threadIdx.x / CPR, srow = row % NS;
  // eight channels of the thread's block and of the block it samples: the keys' sum (rounded once
  // when used: within 2^-24 of the true sum, whatever cancels), an upper bound of the sum of their
  // norms, and whether the block holds a real token
  const long long bk[2] = {blk, centred ? (blk >> lgb << lgb) + ((2 * srow + 1) * nblk) / (2 * NS) : blk};
  double sum[2][8], sq[2] = {0.0, 0.0};
  uint32_t any[2] = {0, 0};
  float norms[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[t][e] = 0.0;
  const uint8_t* cv = cvalid + ((long long)((uint32_t)(blk >> lgb) / (uint32_t)H) << (lgb + lgr));
  for (int k = 0; k < r; ++k) {
    f32x8 v[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      v[t] = load_chunk(kcmp + ((bk[t] << lgr) + k) * HD + c);
      any[t] |= cv[((bk[t] & (nblk - 1)) << lgr) + k];
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sum[t][e] += (double)v[t][e];
        sq[t] = fma((double)v[t][e], (double)v[t][e], sq[t]);
      }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int o = 1; o < CPR; o <<= 1) sq[t] += __shfl_xor(sq[t], o, 64);
    norms[t] = (float)sqrt((double)r * sq[t]);   // sum of r norms <= sqrt(r sum of squares)
  }
  const float least = kSpread * norms[0];
  float mean[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) mean[e] = 0.f;
  bool equal = false;
  if (centred) {
    if (row < NS) {
#pragma unroll
      for (int e = 0; e < 8; ++e) sample[row][c + e] = any[1] ? (float)sum[1][e] : __builtin_nanf("");
    }
    __syncthreads();
    if (threadIdx.x < HD) {
      float s = 0.f, lo = __builtin_huge_valf(), hi = kNegInf;
      int n = 0;
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const float x = sample[t][threadIdx.x];
        const bool ok = fabsf(x) < 1e30f;   // not NaN, and the sum stays in range
        s += ok ? x : 0.f;
        lo = ok ? fminf(lo, x) : lo;
        hi = ok ? fmaxf(hi, x) : hi;
        n += ok;
      }
      common[threadIdx.x] = n > 2 ? (s - lo - hi) / (float)(n - 2) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) mean[e] = common[c + e];
    if (((blk - row) & (nblk - 1)) == 0) {   // the head's first workgroup
      float d2 = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float d = (float)(sum[1][e] - (double)mean[e]);
        d2 = fmaf(d, d, d2);
      }
#pragma unroll
      for (int o = 1; o < CPR; o <<= 1) d2 += __shfl_xor(d2, o, 64);
      const float lim = kEqual * norms[1];
      equal = 2 * __syncthreads_count(any[1] && d2 < lim * lim) > __syncthreads_count(any[1]);
    }
  }
  if (c == 0 && (blk & (nblk - 1)) == 0) flags[blk >> lgb] = equal;
  float a[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = (float)(sum[0][e] - (double)mean[e]);
  int ex;
  const float ss = unit_scale(
      a, 8, ex,
      [](float x) {
#pragma unroll
        for (int o = 1; o < CPR; o <<= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
        return x;
      },
      [](float x) {
#pragma unroll
        for (int o = 1; o < CPR; o <<= 1) x += __shfl_xor(x, o, 64);
        return x;
      });
  const float nrm = sqrtf(ss);
  const float rn = ss == 0.f ? 0.f : kUnit / fmaxf(nrm, ldexpf(least, -ex));
  f16x8 u;
  f32x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    u[e] = (_Float16)(ldexpf(a[e], -ex) * rn);
    o[e] = (float)sum[0][e];
  }
  *reinterpret_cast<f16x8*>(kunit + 8 * i) = u;
  if (r > 1) *reinterpret_cast<f32x8*>(ksum + 8 * i) = o;
  if (c == 0) {
    kabs[blk] = any[0] ? norms[0] : __builtin_nanf("");
    float* kn = knorm + (blk >> lgb) * (long long)max(1 << lgb, 4096 / HD);
    const int t = (int)(blk & ((1LL << lgb) - 1));
    kn[t] = any[0] ? -fmaxf(ldexpf(nrm, ex), least) : __builtin_nanf("");
    for (int p = t + (1 << lgb); p < 4096 / HD; p += 1 << lgb) kn[p] = __builtin_nanf("");
  }
}

// Sum over aligned runs of eight lanes, in every lane of the run.
__device__ __forceinline__ float sum8(float x) {
  auto dpp = [](float v, auto ctrl) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  x += dpp(x, std::integral_constant<int, 0xB1>{});    // lane ^ 1
  x += dpp(x, std::integral_constant<int, 0x4E>{});    // lane ^ 2
  x += dpp(x, std::integral_constant<int, 0x141>{});   // mirrored within eight lanes
  return x;
}

// Score of a selection block in f32 (r times it: <q, sum of its compressed keys>), by eight
// lanes (sub = lane % 8, four dimensions of each 32 per lane, so a row is read as whole
// 128-byte lines).
template <int NCH>
__device__ __forceinline__ float dot8(const f32x4 (&x)[NCH], const f32x4 (&y)[NCH]) {
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fmaf(x[c][e], y[c][e], s);
  return sum8(s);
}

// hi = bf16(x), mid = bf16(x - hi), lo = bf16(x - hi - mid) (the differences are exact in f32).
__device__ __forceinline__ void split3(const f32x8& v, bf16x8& hi, bf16x8& mid, bf16x8& lo) {
  float h[8], md[8], lw[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float ah = bf2f(f2bf(v[e]));
    const float r1 = v[e] - ah;
    const float am = bf2f(f2bf(r1));
    h[e] = ah;
    md[e] = am;
    lw[e] = r1 - am;
  }
  hi = make_chunk<bf16_t>(h);
  mid = make_chunk<bf16_t>(md);
  lo = make_chunk<bf16_t>(lw);
}

// a[0 .. n) sorted descending from a bitonic sequence (n a power of two).
template <int N>
__device__ __forceinline__ void bitonic_merge(float (&a)[N]) {
#pragma unroll
  for (int h = N / 2; h >= 1; h >>= 1)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if ((i & h) == 0) {
        const float x = a[i], y = a[i + h];
        a[i] = fmaxf(x, y);
        a[i + h] = fminf(x, y);
      }
}
template <int N>
__device__ __forceinline__ void sort_desc(float (&a)[N]) {
#pragma unroll
  for (int w = 2; w <= N; w <<= 1)
#pragma unroll
    for (int h = w / 2; h >= 1; h >>= 1)
#pragma unroll
      for (int i = 0; i < N; ++i)
        if ((i & h) == 0) {
          const bool desc = w == N || (i & w) == 0;
          const float x = a[i], y = a[i + h];
          a[i] = desc ? fmaxf(x, y) : fminf(x, y);
          a[i + h] = desc ? fminf(x, y) : fmaxf(x, y);
        }
}

// The K-th largest of the group's 4 K values, K per lane.
template <int K>
__device__ __forceinline__ float group_kth(float (&a)[K]) {
  sort_desc(a);
  float t[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {   // the best K of the lane pair's lists, bitonic
    float lo, hi, lo2, hi2;
    lo = xor16_pair(a[i], hi);
    lo2 = xor16_pair(a[K - 1 - i], hi2);
    (void)hi;
    (void)lo2;
    t[i] = fmaxf(lo, hi2);
  }
  bitonic_merge(t);
  float best = __builtin_huge_valf();
#pragma unroll
  for (int i = 0; i < K; ++i) {
    float lo, hi, lo2, hi2;
    lo = xor32_pair(t[i], hi);
    lo2 = xor32_pair(t[K - 1 - i], hi2);
    (void)hi;
    (void)lo2;
    best = fminf(best, fmaxf(lo, hi2));
  }
  return best;
}

// Eight row fragments of a key tile: at a0 plus 16 rows each (128-byte rows: four at a0, the
// same four rows' second half at a1). One statement that also waits: the compiler would
// otherwise wait for the tile loads in flight, whose stages it cannot tell apart.
template <int HD>
__device__ __forceinline__ void lds_frags8(uint32_t a0, uint32_t a1, f16x8 (&f)[8]) {
  if (HD == 64)
    asm volatile(
        "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:2048\n\tds_read_b128 %2, %8 offset:4096\n\t"
        "ds_read_b128 %3, %8 offset:6144\n\tds_read_b128 %4, %9\n\tds_read_b128 %5, %9 offset:2048\n\t"
        "ds_read_b128 %6, %9 offset:4096\n\tds_read_b128 %7, %9 offset:6144\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7])
        : "v"(a0), "v"(a1)
        : "memory");
  else
    asm volatile(
        "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:1024\n\tds_read_b128 %2, %8 offset:2048\n\t"
        "ds_read_b128 %3, %8 offset:3072\n\tds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %5, %8 offset:5120\n\t"
        "ds_read_b128 %6, %8 offset:6144\n\tds_read_b128 %7, %8 offset:7168\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7])
        : "v"(a0)
        : "memory");
}
// Norms of a tile: lane j's four blocks of every sub-tile (64 bytes apart).
template <int NST>
__device__ __forceinline__ void lds_norms(uint32_t a, f32x4 (&n)[NST]) {
  static_assert(NST == 4 || NST == 8, "sub-tiles");
  if constexpr (NST == 4)
    asm volatile(
        "ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:64\n\tds_read_b128 %2, %4 offset:128\n\t"
        "ds_read_b128 %3, %4 offset:192\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(n[0]), "=&v"(n[1]), "=&v"(n[2]), "=&v"(n[3])
        : "v"(a)
        : "memory");
  else
    asm volatile(
        "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:64\n\tds_read_b128 %2, %8 offset:128\n\t"
        "ds_read_b128 %3, %8 offset:192\n\tds_read_b128 %4, %8 offset:256\n\tds_read_b128 %5, %8 offset:320\n\t"
        "ds_read_b128 %6, %8 offset:384\n\tds_read_b128 %7, %8 offset:448\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(n[0]), "=&v"(n[1]), "=&v"(n[2]), "=&v"(n[3]), "=&v"(n[4]), "=&v"(n[5]), "=&v"(n[6]), "=&v"(n[7])
        : "v"(a)
        : "memory");
}

// s_waitcnt with vmcnt = V (expcnt and lgkmcnt left at their maxima)
template <int V>
__device__ __forceinline__ void vm_wait() {
  static_assert(V >= 0 && V < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((V & 15) | ((V >> 4) << 14) | (7 << 4) | (15 << 8));
}

// lgr: log2 of the compressed keys per selection block; lgls, lgm, lgg: log2 of l', m and g.
template <int HD, int K>
__global__ void __launch_bounds__(kWaves * 64)
    select_kernel(const float* __restrict__ qpool, const float* __restrict__ ksum, const float* __restrict__ kcmp,
                  const uint16_t* __restrict__ kunit, const float* __restrict__ knorm, const float* __restrict__ kabs,
                  const int* __restrict__ flags, int N, int lgr, int lgls, int lgm, int lgg, int mask_own, int kk,
                  int* __restrict__ sel) {
  constexpr int NCH = HD / 32;
  constexpr int KT = 4096 / HD;     // blocks per staged tile (8 KB)
  constexpr int GW = 16 * kWaves;   // groups per workgroup
  constexpr int NST = KT / 16;      // 16-block sub-tiles of a tile
  constexpr int NC = 4 * NST;       // blocks per lane and tile
  static_assert(NC % K == 0, "sets");   // K sets per lane: a block's set is its place in the tile
  // a ring of key tiles (8 KB each) and their norms, kAhead of them in flight
  __shared__ __attribute__((aligned(1024))) bf16_t ring[kRing][KT * HD];
  __shared__ __attribute__((aligned(256))) float nring[kRing][KT];
  __shared__ uint32_t flat_s[kWaves][kFlat];   // block | group << 20
  __shared__ int cnt_s[kWaves][16];            // a group's keys
  __shared__ __attribute__((aligned(16))) int best_s[kWaves][16 * 16];
  static_assert(sizeof(ring) >= kWaves * 16 * kPerGroup * 8, "reused tiles");
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, j = lane >> 4;
  const int ngroups = N >> lgg;
  const int bh = blockIdx.y;
  const int p0 = blockIdx.x * GW + 16 * wid;   // the wave's first group
  const int nblk = N >> lgls;
  const bf16_t* ku = kunit + (size_t)bh * nblk * HD;
  const float* kn = knorm + (size_t)bh * max(nblk, KT);   // negated; padded with NaN to a tile
  const float* ka = kabs + (size_t)bh * nblk;
  const float* ks = ksum + (size_t)bh * nblk * HD;
  const float* kc = kcmp + ((size_t)bh * nblk << lgr) * HD;
  const float* qb = qpool + (size_t)bh * ngroups * HD;

  // tiles u = 0 .. 2 nt - 1: the keys once per pass. Every wave loads its share of a tile
  // and all of the tile's norms, so that its loads in flight count alike.
  const int nt = (nblk + KT - 1) / KT;
  constexpr int PER = 8 / kWaves + KT / 64;
  auto issue = [&](int u) {
    if (u >= 2 * nt) return;
    const int t0 = (u >= nt ? u - nt : u) * KT;
    dma_tile<HD, KT, kWaves>(ring[u % kRing], ku, t0, nblk, wid, lane);
#pragma unroll
    for (int i = 0; i < KT / 64; ++i)
      __builtin_amdgcn_global_load_lds(kn + t0 + 64 * i + lane, &nring[u % kRing][64 * i], 4, 0, 0);
  };
  // tile u is in LDS for every wave, and the stage of tile u - 1 is free for tile u + kAhead
  auto advance = [&](int u) {
    if (u + kAhead <= 2 * nt)
      vm_wait<(kAhead - 1) * PER>();
    else
      vm_drain();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(u + kAhead);
  };

#pragma unroll
  for (int u = 0; u < kAhead; ++u) issue(u);
  const int ntu = flags[bh] ? 0 : nt;   // tiles used

  // this lane's group: unit query (B operand)
  const int pg = p0 + r;
  const bool live = pg < ngroups;
  f16x8 qf[NCH];
  bool zero, over;   // over: the group's scores are all formed instead (a zero query: all blocks tie)
  float qnorm;
  {
    const float* qr = qb + (size_t)(live ? pg : 0) * HD;
    float a[8 * NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const f32x8 v = load_chunk(qr + 32 * c + 8 * j);
#pragma unroll
      for (int e = 0; e < 8; ++e) a[8 * c + e] = v[e];
    }
    int ex;
    const float ss = unit_scale(a, 8 * NCH, ex, [](float x) { return col_max(x); }, [](float x) { return col_sum(x); });
    qnorm = ldexpf(sqrtf(ss), ex);
    zero = ss == 0.f;
    over = live && zero;
    const float rn = ss == 0.f ? 0.f : kUnit / sqrtf(ss);
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[c][e] = (_Float16)(ldexpf(a[8 * c + e], -ex) * rn);
  }

  // blocks of the group's own ball (excluded when mask_own); a wave compares only in tiles
  // that touch a ball of one of its groups
  const int lgb = lgm - lgls;   // blocks per ball
  const int own_lo = (pg >> (lgm - lgg)) << lgb;
  const int wave_lo = mask_own ? (p0 >> (lgm - lgg)) << lgb : 0;
  const int wave_hi = mask_own ? (((p0 + 15) >> (lgm - lgg)) + 1) << lgb : 0;
  auto own = [&](int blk) { return (uint32_t)(blk - own_lo) < (1u << lgb); };

  // the unit scores of tile u (plus `start`) and the blocks' negated norms: fn(index of the
  // block, norm, score); their product is minus the block's score over the query's norm.
  // Row fragments of sub-tile st lie 16 rows apart (one swizzle), so two addresses serve all.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)&ring[0][0];
  const uint32_t ldsn = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)&nring[0][0] + 16 * j;
  auto scores = [&](int u, float start, auto&& fn) {
    const f32x4 st4 = {start, start, start, start};
    const uint32_t base = lds0 + (u % kRing) * (KT * HD * 2) + r * HD * 2;
    f16x8 kf[8];
    lds_frags8<HD>(base + 16 * (j ^ swz<HD>(r)), base + 16 * ((4 + j) ^ swz<HD>(r)), kf);
    f32x4 acc[NST], nn[NST];
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int st = 0; st < NST; ++st)
        acc[st] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[c * NST + st], qf[c], c ? acc[st] : st4, 0, 0, 0);
    lds_norms<NST>(ldsn + (u % kRing) * (KT * 4), nn);
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int t = 0; t < 4; ++t) fn(4 * st + t, nn[st][t], acc[st][t]);
  };
  // the block of index t in a tile that starts at block t0
  auto block_of = [&](int t0, int t) { return t0 + 16 * (t / 4) + 4 * j + t % 4; };

  float top[K];   // minus each set's largest lower bound
#pragma unroll
  for (int t = 0; t < K; ++t) top[t] = __builtin_huge_valf();
#pragma unroll 1
  for (int u = 0; u < ntu; ++u) {
    advance(u);
    const int t0 = u * KT;
    if (t0 < wave_hi && t0 + KT > wave_lo)
      scores(u, -kUnitErr, [&](int t, float n, float sc) {
        float& x = top[t % K];
        x = fminf(x, own(block_of(t0, t)) ? __builtin_huge_valf() : n * sc);
      });
    else
      scores(u, -kUnitErr, [&](int t, float n, float sc) {
        float& x = top[t % K];
        x = fminf(x, n * sc);
      });
  }
  // just below the k*-th largest lower bound (-inf: fewer than K sets hold a block), so that
  // blocks that reach it lie above; NaN passes no block
#pragma unroll
  for (int t = 0; t < K; ++t) top[t] = -top[t];
  float thr = group_kth<K>(top);
  thr = thr == 0.f ? __int_as_float((int)0x80000001)
                   : thr > kNegInf ? __int_as_float(__float_as_int(thr) + (thr > 0.f ? -1 : 1)) : thr;
  thr = live && !over ? thr : __builtin_nanf("");

  // Hits (threshold minus upper bound below zero) are collected as sign bits, a tile's NC
  // candidates at a time, and moved to the wave's list every 32 candidates: a few rounds, each
  // taking one hit of every lane that has one. (A branch per candidate took 57 instead of 45 us
  // at 65536 queries in groups of 16.)
  uint32_t* flat = flat_s[wid];
  int total = 0;   // wave-uniform; entries past kFlat are counted, not kept
  const uint32_t tag = ((uint32_t)r << 20) + (uint32_t)(4 * j);
  uint32_t bits = 0;
  constexpr int TF = 32 / NC;   // tiles per move
  auto move = [&](int tile, int pushed) {   // `pushed` candidates since tile `tile`
    for (;;) {
      const uint64_t has = __builtin_amdgcn_ballot_w64(bits != 0);
      if (!has) break;
      const int at = total + __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0));
      const int top1 = 31 - __builtin_clz(bits | 1);
      const int ord = pushed - 1 - top1, t = ord % NC;
      if (bits != 0 && at < kFlat) flat[at] = tag + (uint32_t)((tile + ord / NC) * KT + 16 * (t / 4) + t % 4);
      bits &= ~(1u << top1);
      total += __popcll(has);
    }
  };
#pragma unroll 1
  for (int u = nt; u < nt + ntu; ++u) {
    advance(u);
    const int t0 = (u - nt) * KT;
    if (t0 < wave_hi && t0 + KT > wave_lo)
      scores(u, kUnitErr, [&](int t, float n, float sc) {
        const float x = own(block_of(t0, t)) ? 0.f : fmaf(n, sc, thr);
        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(x), 31);
      });
    else
      scores(u, kUnitErr, [&](int, float n, float sc) {
        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(fmaf(n, sc, thr)), 31);
      });
    const int done = (u - nt) % TF + 1;
    if (done == TF || u == 2 * nt - 1) move(u - nt - done + 1, done * NC);
  }
  if (ntu == 0) vm_drain();   // the first tiles have landed
  __syncthreads();   // the tiles are free: they hold the groups' lists from here

  // the listed blocks' dots, each to its group's list as a key (in no particular order)
  uint64_t* keys = reinterpret_cast<uint64_t*>(ring) + wid * 16 * kPerGroup;   // [group][kPerGroup]
  int* cnt = cnt_s[wid];
  int* best16 = best_s[wid];   // [group][16] the k* best blocks
  if (lane < 16) cnt[lane] = 0;
  *reinterpret_cast<int4*>(best16 + 4 * lane) = make_int4(kNoBlock, kNoBlock, kNoBlock, kNoBlock);
  wave_sync();
  if (total > kFlat || ntu == 0) {
    over = live;
    total = 0;
  }
  const int sub = lane & 7;
  // four rounds of eight entries at a time, all their rows in flight together
  constexpr int PF = 4;
#pragma unroll 1
  for (int e0 = 0; e0 < total; e0 += 8 * PF) {
    uint32_t x[PF];
    f32x4 qv[PF][NCH], kv[PF][NCH];
    float a[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) x[i] = flat[min(e0 + 8 * i + (lane >> 3), total - 1)];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int grp = (int)((x[i] >> 20) & 15), blk = min((int)(x[i] & 0xFFFFF), nblk - 1);
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        qv[i][c] = *reinterpret_cast<const f32x4*>(qb + (size_t)(p0 + grp) * HD + 32 * c + 4 * sub);
        kv[i][c] = *reinterpret_cast<const f32x4*>(ks + (size_t)blk * HD + 32 * c + 4 * sub);
      }
      a[i] = ka[blk];
    }
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const float s = dot8<NCH>(qv[i], kv[i]);
      const int grp = (int)((x[i] >> 20) & 15), blk = (int)(x[i] & 0xFFFFF);
      if (sub == 0 && e0 + 8 * i + (lane >> 3) < total && a[i] >= 0.f && blk < nblk) {
        // a score beyond f32's range may tie with blocks that the list need not hold
        const bool finite = fabsf(s) < __builtin_huge_valf();
        const int at = atomicAdd(&cnt[grp], finite ? 1 : kPerGroup + 1);
        const int e = e0 + 8 * i + (lane >> 3);
        flat[e] = __float_as_uint(a[i]);   // the entry has been read
        if (at < kPerGroup) keys[grp * kPerGroup + at] = make_key(s, blk, e);
      }
    }
  }
  wave_sync();
  const int n = cnt[r];
  over = over || (live && n > kPerGroup);
  const uint64_t* list = keys + r * kPerGroup;
  // each key's rank within its group (nr keys): lane j takes the group's keys j, j + 4, ..., eight
  // at a time, and compares them with all of the group's keys
  auto rank_keys = [&](int nr, auto&& each) {
    for (int b0 = 0; __builtin_amdgcn_ballot_w64(b0 < nr); b0 += 32) {
      uint64_t own8[8];
      int rank[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int y = b0 + 4 * i + j;
        own8[i] = y < nr ? list[y] : 0;
        rank[i] = 0;
      }
#pragma unroll 4
      for (int y = 0; y < nr; ++y) {
        const uint64_t k2 = list[y];
#pragma unroll
        for (int i = 0; i < 8; ++i) rank[i] += k2 > own8[i];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (own8[i] == 0) continue;
        if (rank[i] < kk) best16[16 * r + rank[i]] = key_block(own8[i]);
        each(own8[i], rank[i]);
      }
    }
  };
  float lo = __builtin_huge_valf(), hi = kNegInf;   // least score of the k* best, largest of the rest
  rank_keys(over ? 0 : n, [&](uint64_t key, int rank) {
    const float sc = key_score(key), err = kDotErr * qnorm * __uint_as_float(flat[(uint32_t)key & 511u]);
    if (rank < kk)
      lo = fminf(lo, sc - err);
    else
      hi = fmaxf(hi, sc + err);
  });
  lo = -col_max(-lo);
  hi = col_max(hi);

  // the group's pooled query and a row of 8 j .. of a compressed key in three bf16 parts
  bf16x8 qh[NCH], qm[NCH], ql[NCH];
  auto load_query = [&]() {
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      split3(load_chunk(qb + (size_t)(live ? pg : 0) * HD + 32 * c + 8 * j), qh[c], qm[c], ql[c]);
  };
  auto load_key = [&](int key, f32x8 (&v)[NCH]) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) v[c] = load_chunk(kc + (size_t)key * HD + 32 * c + 8 * j);
  };
  // scores of 16 keys (rows) for the wave's groups (columns), smaller products first
  auto six = [&](int c, const bf16x8& ah, const bf16x8& am, const bf16x8& al, f32x4 acc) {
    acc = mma(al, qh[c], acc);
    acc = mma(ah, ql[c], acc);
    acc = mma(am, qm[c], acc);
    acc = mma(am, qh[c], acc);
    acc = mma(ah, qm[c], acc);
    return mma(ah, qh[c], acc);
  };
  const int rr = 1 << lgr;
  const float rcp_r = 1.0f / (float)rr;

  // groups whose cut the dots do not decide: the blocks of their lists, gathered in `flat` as
  // (group, place in its list), are scored by the six products
  wave_sync();
  const bool near = live && !over && !(lo > hi);
  if (__builtin_amdgcn_ballot_w64(near)) {
    const int nn = near ? n : 0;
    int end = nn;   // of the group's entries
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int y = __shfl_up(end, o, 16);
      end += r >= o ? y : 0;
    }
    for (int i = j; i < nn; i += 4) flat[end - nn + i] = (uint32_t)(r * kPerGroup + i);
    const int tot = __builtin_amdgcn_readlane(end, 15);   // at most the kFlat entries there were
    load_query();
    wave_sync();
    bool bad = false;
    const int per = 16 >> lgr;   // blocks per product; four products' keys in flight together
#pragma unroll 1
    for (int b0 = 0; b0 < tot; b0 += 4 * per) {
      f32x8 kv[4][NCH];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int blk = key_block(keys[flat[min(b0 + b * per + (r >> lgr), tot - 1)]]);
        load_key((blk << lgr) + (r & (rr - 1)), kv[b]);
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int e0 = b0 + b * per;
        if (e0 >= tot) break;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          bf16x8 ah, am, al;
          split3(kv[b][c], ah, am, al);
          acc = six(c, ah, am, al, acc);
        }
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s += acc[i];
          if (((i + 1) & (rr - 1)) != 0) continue;
          const int e = e0 + ((4 * j + i) >> lgr);
          const int at = (int)flat[min(e, tot - 1)];
          s *= rcp_r;
          if (e < tot && at / kPerGroup == r) {   // the entry's own group's column
            bad = bad || !(fabsf(s) < __builtin_huge_valf());
            keys[at] = make_key(s, key_block(keys[at]));
          }
          s = 0.f;
        }
      }
    }
    wave_sync();
    over = over || col_max(bad ? 1.f : 0.f) > 0.f;
    rank_keys(near && !over ? n : 0, [](uint64_t, int) {});
  }
  wave_sync();
  // stored ascending with -1 in unused slots: lane j places the blocks of ranks 4j .. 4j + 3
  int* out = sel + ((size_t)bh * ngroups + p0) * kk;
  auto store = [&](bool mine_too) {
    int4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = reinterpret_cast<const int4*>(best16 + 16 * r)[i];
    const int all[16] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w,
                         v[2].x, v[2].y, v[2].z, v[2].w, v[3].x, v[3].y, v[3].z, v[3].w};
    const int4 m4 = reinterpret_cast<const int4*>(best16 + 16 * r)[j];
    const int mine[4] = {m4.x, m4.y, m4.z, m4.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int pos = 0;
#pragma unroll
      for (int t = 0; t < 16; ++t) pos += all[t] < mine[i];
      const bool used = mine[i] != kNoBlock;
      if (!used) pos = 4 * j + i;   // ranks are filled from 0: the slots past them stay unused
      if (mine_too && pos < kk) out[r * kk + pos] = used ? mine[i] : -1;
    }
  };
  store(live && !over);

  // Groups left over: the workgroup streams the compressed keys, 64 at a time, wave w splits
  // rows 16 w .. of a tile into the fragments of its three parts, and every wave with such a
  // group scores the tile for it. A lane keeps the K best of its rows' blocks; each lane's K / 4
  // best are all at least the smallest of the four lanes' (K / 4)-th, so the group already holds
  // K >= k* at or above that value and nothing below it can enter.
  if (!__syncthreads_or(over)) return;
  const bool some_zero = __syncthreads_or(over && zero);
  constexpr int TS = 4;   // 16-key sub-tiles of a tile, one per wave
  static_assert(kWaves == TS && sizeof(ring) >= TS * 3 * NCH * 64 * 16, "parts of a tile");
  bf16x8* const frag = reinterpret_cast<bf16x8*>(ring);   // [sub-tile][part][chunk][lane]
  const int ntok = nblk << lgr;
  const bool wave_over = __builtin_amdgcn_ballot_w64(over) != 0;
  uint64_t lst[K];
#pragma unroll
  for (int t = 0; t < K; ++t) lst[t] = 0;
  if (wave_over) load_query();
  // a tile's blocks into the lane's list: rows t0 + 16 st + 4 j + i, R keys per block
  auto take_tile = [&](auto rc, int t0, const f32x4 (&acc)[TS], uint64_t least) {
    constexpr int R = decltype(rc)::value, NPS = 4 / R;
    float cand[NPS * TS];   // in ascending block order; -inf: none
    const int blk0 = (t0 + 4 * j) / R;
#pragma unroll
    for (int st = 0; st < TS; ++st)
#pragma unroll
      for (int u = 0; u < NPS; ++u) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < R; ++i) s += acc[st][u * R + i];
        const int blk = blk0 + st * (16 / R) + u;
        cand[st * NPS + u] = over && !(mask_own && own(blk)) ? s * (1.0f / R) : kNegInf;
      }
    // best first; the wave repeats as often as its busiest lane needs
    for (;;) {
      float bs = kNegInf;
      int bi = 0;
#pragma unroll
      for (int t = 0; t < NPS * TS; ++t) {   // first maximum: the lowest block among equal scores
        const bool better = cand[t] > bs;
        bs = better ? cand[t] : bs;
        bi = better ? t : bi;
      }
      const uint64_t key = bs > kNegInf ? make_key(bs, blk0 + bi / NPS * (16 / R) + bi % NPS) : 0;
      const bool take = key > (least > lst[K - 1] ? least : lst[K - 1]);
      if (!__builtin_amdgcn_ballot_w64(take)) break;
      if (take) topk_insert<K>(lst, key);
#pragma unroll
      for (int t = 0; t < NPS * TS; ++t) cand[t] = take && t != bi ? cand[t] : kNegInf;
    }
  };
  f32x8 kv[NCH];
  float norm;   // NaN where the row's block holds no real token: no score passes
  auto fetch = [&](int t0) {
    const int row = t0 + 16 * wid + r, rc = min(row, ntok - 1);
    norm = row < ntok ? ka[rc >> lgr] : __builtin_nanf("");
    load_key(rc, kv);
  };
  fetch(0);
#pragma unroll 1
  for (int t0 = 0; t0 < ntok; t0 += 16 * TS) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      bf16x8 ah, am, al;
      split3(norm >= 0.f ? kv[c] : kv[c] + __builtin_nanf(""), ah, am, al);
      frag[((3 * wid + 0) * NCH + c) * 64 + lane] = ah;
      frag[((3 * wid + 1) * NCH + c) * 64 + lane] = am;
      frag[((3 * wid + 2) * NCH + c) * 64 + lane] = al;
    }
    const uint64_t least = group_min(lst[K / 4 - 1]);
    // a zero query scores every block 0: the first k* eligible blocks are the result
    if (!some_zero)
      __syncthreads();
    else if (__syncthreads_and(!over || (zero && least != 0)))
      break;
    if (t0 + 16 * TS < ntok) fetch(t0 + 16 * TS);
    if (wave_over) {
      f32x4 acc[TS];
#pragma unroll
      for (int st = 0; st < TS; ++st) {
        acc[st] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          const bf16x8* f = frag + (3 * st * NCH + c) * 64 + lane;
          acc[st] = six(c, f[0], f[NCH * 64], f[2 * NCH * 64], acc[st]);
        }
      }
      if (lgr == 0)
        take_tile(std::integral_constant<int, 1>{}, t0, acc, least);
      else if (lgr == 1)
        take_tile(std::integral_constant<int, 2>{}, t0, acc, least);
      else
        take_tile(std::integral_constant<int, 4>{}, t0, acc, least);
    }
    __syncthreads();
  }
  if (over) *reinterpret_cast<int4*>(best16 + 16 * r + 4 * j) = make_int4(kNoBlock, kNoBlock, kNoBlock, kNoBlock);
  wave_sync();
  // k* rounds of a 4-way merge of a group's sorted lists: the best head is chosen and its owner
  // drops it (keys are unique)
#pragma unroll 1
  for (int t = 0; t < kk; ++t) {
    const uint64_t w = group_max(lst[0]);
    const bool pop = w != 0 && lst[0] == w;
#pragma unroll
    for (int i = 0; i < K - 1; ++i) lst[i] = pop ? lst[i + 1] : lst[i];
    lst[K - 1] = pop ? 0 : lst[K - 1];
    if (over && j == 0 && w != 0) best16[16 * r + t] = key_block(w);
  }
  wave_sync();
  store(over);
}

// Workspace: unit vectors, norm bounds (a head's padded to a whole tile), sums of norms, a flag per
// head and, for several keys per block, their sums, each 256-byte aligned.
struct SelectWs {
  size_t norm, abs, flags, sum, total;
};
SelectWs select_ws(const Dims& D) {
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t heads = (size_t)D.B * D.H, nblk = D.N / D.ls, tile = 4096 / D.d;
  SelectWs W;
  W.norm = up(2 * heads * nblk * D.d);
  W.abs = W.norm + up(4 * heads * (nblk > tile ? nblk : tile));
  W.flags = W.abs + up(4 * heads * nblk);
  W.sum = W.flags + up(4 * heads);
  W.total = W.sum + (D.ls > D.l ? up(4 * heads * nblk * D.d) : 0);
  return W;
}

template <typename T, int HD, int K>
hipError_t select_k(const Dims& D, const void* q, const uint8_t* valid, const float* kcmp, const uint8_t* cvalid,
                    int* sel, float* qpool, bool given, uint16_t* kunit, hipStream_t st) {
  auto lg = [](int x) { return __builtin_ctz((unsigned)x); };
  const int ngroups = D.N / D.g, nblk = D.N / D.ls, R = D.ls / D.l;
  const long long blocks = (long long)D.B * D.H * nblk;
  const long long pool_n8 = given ? 0 : (long long)D.B * D.H * ngroups * (HD / 8);
  const long long pool_blocks = (pool_n8 + 255) / 256, key_blocks = (blocks * (HD / 8) + 255) / 256;
  const SelectWs W = select_ws(D);
  char* const w = reinterpret_cast<char*>(kunit);
  float *knorm = (float*)(w + W.norm), *kabs = (float*)(w + W.abs), *ksum = (float*)(w + W.sum);
  int* flags = (int*)(w + W.flags);
  hipLaunchKernelGGL((select_prep_kernel<T, HD>), dim3((unsigned)(pool_blocks + key_blocks)), dim3(256), 0, st,
                     (const T*)q, valid, D.H, lg(D.N), lg(D.g), pool_n8, (int)pool_blocks, qpool, kcmp, cvalid,
                     lg(nblk), lg(R), blocks, kunit, knorm, kabs, ksum, flags);
  const dim3 grid((ngroups + 16 * kWaves - 1) / (16 * kWaves), D.B * D.H);
  hipLaunchKernelGGL((select_kernel<HD, K>), grid, dim3(kWaves * 64), 0, st, (const float*)qpool,
                     R > 1 ? (const float*)ksum : kcmp, kcmp, (const uint16_t*)kunit, (const float*)knorm,
                     (const float*)kabs, (const int*)flags, D.N, lg(R), lg(D.ls), lg(D.m), lg(D.g), D.mask_own,
                     D.k, sel);
  return hipGetLastError();
}

template <typename T, int HD>
hipError_t select_hd(const Dims& D, const void* q, const uint8_t* valid, const float* kcmp, const uint8_t* cvalid,
                     int* sel, float* qpool, bool given, uint16_t* kunit, hipStream_t st) {
  if (D.k <= 4) return select_k<T, HD, 4>(D, q, valid, kcmp, cvalid, sel, qpool, given, kunit, st);
  if (D.k <= 8) return select_k<T, HD, 8>(D, q, valid, kcmp, cvalid, sel, qpool, given, kunit, st);
  return select_k<T, HD, 16>(D, q, valid, kcmp, cvalid, sel, qpool, given, kunit, st);
}

}  // namespace

hipError_t launch_select_topk(const Dims& D, const void* q, const uint8_t* valid, const float* kcmp,
                              const uint8_t* cvalid, int* sel, float* qpool, bool given, uint16_t* kunit,
                              hipStream_t st) {
  if (D.bf16)
    return D.d == 64 ? select_hd<bf16_t, 64>(D, q, valid, kcmp, cvalid, sel, qpool, given, kunit, st)
                     : select_hd<bf16_t, 32>(D, q, valid, kcmp, cvalid, sel, qpool, given, kunit, st);
  return select_hd<float, 32>(D, q, valid, kcmp, cvalid, sel, qpool, given, kunit, st);   // float32: head_dim 32
}

size_t select_ws_bytes(const Dims& D) { return select_ws(D).total; }

}  // namespace bsa
