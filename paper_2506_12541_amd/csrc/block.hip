// The dense parts of the transformer block around the layer (Section 3.1: each block holds
// an RMSNorm, the BSA layer and a SwiGLU): the channel matrix products on the bf16 matrix
// cores with f32 accumulation, RMSNorm forward/backward, SwiGLU forward/backward, and the
// casts, layout changes and deterministic reductions between them.
#include "common.hpp"
#include "kernels.hpp"

namespace bsa {
namespace {

constexpr float kNormEps = 1e-6f;

// ---- matrix products C[M, N] = sum_k A(m, k) B(n, k) ----
//
// Workgroup tiles of 256 x 256 (eight waves of 64 x 128, contraction tiles of 32 in four LDS
// stages), 128 x 128 (four waves of 64 x 64, contraction tiles of 64 in two) or 64 x 64 (four
// waves of 32 x 32, contraction tiles of 64 in four) in 16 x 16 accumulator tiles. Stages are
// filled by direct global->LDS loads while another feeds the matrix cores (launch_gemm picks
// the tile from the shape).
//   plain form (trans = false): A [M, K] and B [N, K], contraction index fastest; tiles are
//     staged as rows x contraction (row fragments read with ds_read_b128);
//   transposed form (trans = true): A [K, M] and B [K, N], the contraction runs over their
//     rows (the weight gradients dW = dY^T X over tokens); tiles are staged as contraction
//     x columns and read with transposing LDS reads (ds_read_b64_tr_b16).
// Accumulator lane L holds C[m0 + L % 16][n0 + 4 (L / 16) + e], e = 0..3 (the B fragment
// is the first MFMA operand).

// 16-byte chunk swizzle of a staged tile row: 4 or 8 chunks per row (row-fragment reads
// of 16 consecutive rows on distinct banks) or 16 and more chunks per row (transposing
// reads of 8 consecutive rows, chunk pairs on distinct banks).
template <int COLS>
__device__ __forceinline__ int tile_swz(int x) {
  return COLS == 32 ? ((x >> 1) & 3) : COLS == 64 ? (x & 7) : 2 * (x & 7);
}

// Staging of ROWS x COLS tiles of a logical row-major operand into LDS by the NW waves of
// the workgroup. Each wave instruction fills 1 KB of consecutive LDS; lane L's 16 bytes
// land at bytes [16 L, 16 L + 16) and the lane fetches the chunk the swizzle puts there.
// The element offset of that chunk splits into a per-lane part fixed for the kernel and a
// wave-uniform part per contraction tile (kt_offset; shapes are whole tiles, as the
// launcher checks).
template <int ROWS, int COLS, int NW>
struct TileLoader {
  static constexpr int CPR = COLS / 8;
  static constexpr int NU = ROWS * CPR / (64 * NW);   // wave instructions per wave
  static_assert(NU * 64 * NW == ROWS * CPR, "tile / wave split");
  const bf16_t* p;
  long long lane_off[NU];

  // (r0, c0): the tile origin of the operand block this workgroup owns, as (row, column)
  // of the logical matrix at kt = 0.
  __device__ __forceinline__ void init(const GemmMat& m, long long r0, int c0, int wid, int lane) {
    p = reinterpret_cast<const bf16_t*>(m.p);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int idx = (wid * NU + u) * 64 + lane;
      const int row = idx / CPR;
      const int col = 8 * ((idx % CPR) ^ tile_swz<COLS>(row));
      const long long r = r0 + row;
      const int c = c0 + col;
      if (m.heads == 0) {
        lane_off[u] = r * m.ld + c;
      } else {
        const long long b = r >> m.lgn, t = r & ((1LL << m.lgn) - 1);
        lane_off[u] = ((((b * m.heads + (c >> m.lgd)) << m.lgn) + t) << m.lgd) + (c & ((1 << m.lgd) - 1));
      }
    }
  }
  __device__ __forceinline__ void issue(bf16_t* lds, long long kt_off, int wid) const {
#pragma unroll
    for (int u = 0; u < NU; ++u)
      __builtin_amdgcn_global_load_lds(p + kt_off + lane_off[u], lds + (wid * NU + u) * 512, 16, 0, 0);
  }
};

// Wave-uniform element offset of contraction tile kt (BK wide) of an operand.
// Plain form: columns BK kt; in the heads layout a tile stays inside one head (BK <= d) or
// covers whole heads (d divides BK), n d elements per head. Transposed form: rows BK kt;
// in the heads layout BK divides n, so a tile stays inside one cloud.
template <bool TR, int BK>
__device__ __forceinline__ long long kt_offset(const GemmMat& m, int kt) {
  const long long k0 = (long long)kt * BK;
  if (!TR) {
    if (m.heads == 0) return k0;
    return ((k0 >> m.lgd) << (m.lgn + m.lgd)) + (k0 & ((1LL << m.lgd) - 1));
  }
  if (m.heads == 0) return k0 * m.ld;
  const long long b = k0 >> m.lgn, t = k0 & ((1LL << m.lgn) - 1);
  return ((b * m.heads << m.lgn) + t) << m.lgd;
}

template <int BK>
__device__ __forceinline__ bf16x8 frag_row(const bf16_t* t, int row, int lc) {
  return *reinterpret_cast<const bf16x8*>(t + row * BK + 8 * (lc ^ tile_swz<BK>(row)));
}

// Workgroup barrier without a memory fence: the waves' direct-to-LDS loads are already
// waited for by each wave (vmcnt), and later tiles stay in flight across it (the fence of
// __syncthreads would wait for every outstanding load). The empty statements keep the
// compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// s_waitcnt with vmcnt = V (expcnt and lgkmcnt left at their maxima)
template <int V>
__device__ __forceinline__ void vm_wait() {
  static_assert(V >= 0 && V < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((V & 15) | ((V >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Wait for this wave's LDS reads; no LDS access moves across it.
__device__ __forceinline__ void lgkm_drain() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// LDS byte addresses of the two transposing reads that give lane (p = L % 16, j = L / 16)
// the operand X[k0 + 4j + i][m0 + p] (i = 0..3) and X[k0 + 16 + 4j + i][m0 + p] of a
// [BK][COLS] tile X (BK = 32 or 64): within each 16-lane group, ds_read_b64_tr_b16 hands lane l element
// l % 4 of the 4-element runs addressed by lanes l / 4, 4 + l / 4, 8 + l / 4, 12 + l / 4, so
// lane p addresses row k0 + 4j + p / 4 (then + 16) at columns m0 + 4 (p % 4) + [0, 4).
template <int COLS>
__device__ __forceinline__ void tr_addr(const bf16_t* t, int k0, int m0, int lane, uint32_t& o0, uint32_t& o1) {
  const int p = lane & 15, j = lane >> 4;
  const int col = m0 + 4 * (p & 3);
  const int lc = col >> 3, sub = col & 7;
  const int x0 = k0 + 4 * j + (p >> 2), x1 = x0 + 16;
  const bf16_t* a0 = t + x0 * COLS + 8 * (lc ^ tile_swz<COLS>(x0)) + sub;
  const bf16_t* a1 = t + x1 * COLS + 8 * (lc ^ tile_swz<COLS>(x1)) + sub;
  o0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)a0;
  o1 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)a1;
}

// Four operand fragments (columns m0 + 16 i, i = 0..3) of one 32-deep contraction step of
// the transposed form, issued as one statement that also waits for them: every use of the
// results follows the wait.
template <int COLS>
__device__ __forceinline__ void tr_frags4(const bf16_t* t, int k0, int m0, int lane, bf16x8 (&f)[4]) {
  uint32_t a[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) tr_addr<COLS>(t, k0, m0 + 16 * i, lane, a[2 * i], a[2 * i + 1]);
  uint2 r[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %9\n\t"
      "ds_read_b64_tr_b16 %2, %10\n\tds_read_b64_tr_b16 %3, %11\n\t"
      "ds_read_b64_tr_b16 %4, %12\n\tds_read_b64_tr_b16 %5, %13\n\t"
      "ds_read_b64_tr_b16 %6, %14\n\tds_read_b64_tr_b16 %7, %15\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7])
      : "memory");
#pragma unroll
  for (int i = 0; i < 4; ++i)
    f[i] = __builtin_bit_cast(bf16x8, make_uint4(r[2 * i].x, r[2 * i].y, r[2 * i + 1].x, r[2 * i + 1].y));
}

// 1 / (1 + exp(-x)): the hardware reciprocal and one Newton step (within an ulp of the divided
// value, at a third of the division's instructions). Where exp(-x) leaves the range in which the
// reciprocal is a normal number (x below -87) the reciprocal stands: the step would give NaN.
__device__ __forceinline__ float sigmoid(float x) {
  const float y = 1.0f + __expf(-x);
  const float r = __builtin_amdgcn_rcpf(y);
  return y < 0x1p126f ? fmaf(fmaf(-y, r, 1.0f), r, r) : r;
}

struct GemmArgs {
  GemmMat a, b;
  int ntn;        // column tiles
  int kt_per;     // contraction tiles per split
  GemmOut o;
  long long split_stride;   // elements between the partial products of two splits
  bool stream_out;          // SwiGLU forward: stores that bypass the caches
};

// Rows of a wave's tile that pass through LDS at a time in the epilogue: as many as fit the
// four arrays of the first two stages.
constexpr int epi_rows(int array_bytes, int tmw, int tnw, int nw) {
  int rp = tmw;
  while (rp > 16 && 4 * (array_bytes / (rp * tnw * 4)) < nw) rp /= 2;
  return rp;
}

// Workgroup tile BM x BN of WM x WN waves (wave tile BM / WM x BN / WN in 16 x 16
// accumulator tiles); contraction tiles of BK in a ring of NS LDS stages, NS - 1 of them in
// flight while one feeds the matrix cores.
template <bool TR, int BM, int BN, int WM, int WN, int BK, int NS>
__global__ void __launch_bounds__(64 * WM * WN) gemm_kernel(GemmArgs g) {
  constexpr int NW = WM * WN;
  constexpr int TMW = BM / WM, TNW = BN / WN;
  constexpr int FI = TMW / 16, FJ = TNW / 16;
  static_assert(!TR || (FI % 4 == 0 && FJ % 4 == 0), "wave tile");
  static_assert(NS >= 2 && NS <= 4 && (BK == 32 || BK == 64), "pipeline");
  constexpr int AE = BM * BK, BE = BN * BK;
  __shared__ __attribute__((aligned(1024))) bf16_t as0[AE], bs0[BE], as1[AE], bs1[BE];
  __shared__ __attribute__((aligned(1024))) bf16_t as2[NS > 2 ? AE : 8], bs2[NS > 2 ? BE : 8];
  __shared__ __attribute__((aligned(1024))) bf16_t as3[NS > 3 ? AE : 8], bs3[NS > 3 ? BE : 8];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int wm = wid / WN, wn = wid % WN;
  // workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous run of
  // tiles (row panels walked column tile by column tile) so it re-reads A from its own L2
  const int nt = gridDim.x;
  int id = blockIdx.x;
  if ((nt & 7) == 0) id = (id & 7) * (nt >> 3) + (id >> 3);
  const int tm = id / g.ntn, tn = id - tm * g.ntn;
  const long long m0 = (long long)tm * BM, n0 = (long long)tn * BN;
  const int kt0 = blockIdx.y * g.kt_per, kt1 = kt0 + g.kt_per;

  TileLoader<TR ? BK : BM, TR ? BM : BK, NW> la;
  TileLoader<TR ? BK : BN, TR ? BN : BK, NW> lb;
  if (!TR) {
    la.init(g.a, m0, 0, wid, lane);
    lb.init(g.b, n0, 0, wid, lane);
  } else {
    la.init(g.a, 0, (int)m0, wid, lane);
    lb.init(g.b, 0, (int)n0, wid, lane);
  }
  constexpr int PER = decltype(la)::NU + decltype(lb)::NU;   // wave load instructions per tile
  bf16_t* const AS[4] = {as0, as1, as2, as3};
  bf16_t* const BS[4] = {bs0, bs1, bs2, bs3};
  auto issue = [&](int kt, int st) {
    la.issue(AS[st], kt_offset<TR, BK>(g.a, kt), wid);
    lb.issue(BS[st], kt_offset<TR, BK>(g.b, kt), wid);
  };
  f32x4 acc[FI][FJ];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < FJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  bf16x8 af[FI], bfr[FJ];
  auto read = [&](const bf16_t* as, const bf16_t* bs, int ks) {
    if (!TR) {
#pragma unroll
      for (int i = 0; i < FI; ++i) af[i] = frag_row<BK>(as, wm * TMW + 16 * i + (lane & 15), 4 * ks + (lane >> 4));
#pragma unroll
      for (int j = 0; j < FJ; ++j) bfr[j] = frag_row<BK>(bs, wn * TNW + 16 * j + (lane & 15), 4 * ks + (lane >> 4));
    } else {
#pragma unroll
      for (int i = 0; i < FI; i += 4)
        tr_frags4<BM>(as, 32 * ks, wm * TMW + 16 * i, lane, *reinterpret_cast<bf16x8(*)[4]>(&af[i]));
#pragma unroll
      for (int j = 0; j < FJ; j += 4)
        tr_frags4<BN>(bs, 32 * ks, wn * TNW + 16 * j, lane, *reinterpret_cast<bf16x8(*)[4]>(&bfr[j]));
    }
  };
  auto multiply = [&]() {
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int j = 0; j < FJ; ++j) acc[i][j] = mma(bfr[j], af[i], acc[i][j]);
  };

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (kt0 + s < kt1) issue(kt0 + s, s);
  if constexpr (NW == 8) {
    // Two waves share a SIMD; the second four waves run one phase behind the first four, so
    // that one wave of each SIMD multiplies while the other reads its fragments from LDS
    // (reads of both, then products of both, left each pipe idle half of the time). Phases
    // end with a barrier; wave group 0 reads tile t in phase 2t and multiplies in 2t + 1,
    // group 1 one phase later. Stage (t - 1) % NS is last read in phase 2t - 1, so tile
    // t + NS - 1 may be loaded into it from phase 2t on (both groups: as they read tile t);
    // tile t + 1 is first read in phase 2t + 2, so every wave waits for its part of it before
    // the barrier that ends phase 2t + 1.
    static_assert(BK == 32 && NS == 4, "one fragment depth per phase");
    const int n = kt1 - kt0, grp = wid >> 2;
    auto landed = [&](int t) {   // tile t + 1, with at most tiles t + 2 and t + 3 in flight
      if (t + 3 < n)
        vm_wait<2 * PER>();
      else if (t + 2 < n)
        vm_wait<PER>();
      else
        vm_drain();
    };
    landed(-1);
    lds_barrier();
    if (grp == 1) lds_barrier();
    for (int t0 = 0; t0 < n; t0 += NS) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int t = t0 + s;
        if (t < n) {
          if (t + NS - 1 < n) issue(kt0 + t + NS - 1, (s + NS - 1) % NS);
          read(AS[s], BS[s], 0);
          lgkm_drain();
          if (grp == 1) landed(t);
          lds_barrier();
          __builtin_amdgcn_s_setprio(1);
          multiply();
          __builtin_amdgcn_s_setprio(0);
          if (grp == 0) landed(t);
          lds_barrier();
        }
      }
    }
    if (grp == 0) lds_barrier();
  } else {
    for (int kt = kt0; kt < kt1; kt += NS) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int t = kt + s;
        if (t < kt1) {
          // tile t has landed once at most the NS - 2 tiles issued after it are in flight
          if (t + NS - 2 < kt1)
            vm_wait<(NS - 2) * PER>();
          else
            vm_drain();
          lds_barrier();     // every wave's loads of tile t are visible; stage s - 1 is free
          if (t + NS - 1 < kt1) issue(t + NS - 1, (s + NS - 1) % NS);
#pragma unroll
          for (int ks = 0; ks < BK / 32; ++ks) {
            read(AS[s], BS[s], ks);
            multiply();
          }
        }
      }
    }
  }

  // Epilogue. The accumulators go through LDS (the stages are free by then), RP rows of the
  // wave's tile at a time in f32, so that every global access is a run of whole 128-byte
  // lines: a lane stores 8 consecutive columns (4 of f32 outputs). Storing 4 columns of 16
  // rows straight from the accumulators left 32-byte pieces: at 65536 rows, C = 512, F = 2048
  // the SwiGLU forward took 477 instead of 402 us, its backward 497 instead of 340, the Q/K/V
  // product 174 instead of 140. (Without any epilogue the same products take 209, 122 and 90 us:
  // the writes are HBM-bound and the workgroups of a round write together.) 16-byte chunk c of
  // row x sits at c ^ (x mod 16) (mod 8 for 32-column tiles): rows written and rows read spread
  // over the banks.
  constexpr int AB = 2 * (AE < BE ? AE : BE);                          // bytes used of a stage array
  constexpr int RP = epi_rows(AB, TMW, TNW, NW);
  constexpr int WPA = AB / (RP * TNW * 4);                             // waves per stage array
  static_assert(WPA >= 1 && 4 * WPA >= NW && RP % 16 == 0, "epilogue regions");
  const GemmOut& o = g.o;
  const int r = lane & 15, jq = lane >> 4;
  constexpr int SM = TNW >= 64 ? 15 : 7;
  lds_barrier();   // every wave has read the last tile
  bf16_t* const arr = wid / WPA == 0 ? as0 : wid / WPA == 1 ? bs0 : wid / WPA == 2 ? as1 : bs1;
  float* const reg = reinterpret_cast<float*>(arr) + (wid % WPA) * RP * TNW;
  auto at = [&](int row, int chunk) { return reinterpret_cast<f32x4*>(reg + row * TNW + 4 * (chunk ^ (row & SM))); };
  auto row8 = [&](int row, int col, float (&v)[8]) {   // 8 consecutive columns of a row
    const f32x4 x = *at(row, col / 4), y = *at(row, col / 4 + 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = x[e];
      v[4 + e] = y[e];
    }
  };
#pragma unroll
  for (int i0 = 0; i0 < FI; i0 += RP / 16) {
#pragma unroll
    for (int i = 0; i < RP / 16; ++i)
#pragma unroll
      for (int j = 0; j < FJ; ++j) *at(16 * i + r, 4 * j + jq) = acc[i0 + i][j];
    wave_sync();
    const long long mw = m0 + wm * TMW + 16 * i0;
    if (o.epi == kEpiF32 || o.epi == kEpiPart) {
      constexpr int LPR = TNW / 4, RPI = 64 / LPR;
      const int c = lane % LPR;
      float* const dst = reinterpret_cast<float*>(o.out) + (o.epi == kEpiPart ? blockIdx.y * g.split_stride : 0) + n0 +
                         wn * TNW + 4 * c;
      const float* const res = o.epi == kEpiF32 && o.res ? o.res + n0 + wn * TNW + 4 * c : nullptr;
#pragma unroll 8
      for (int x0 = 0; x0 < RP; x0 += RPI) {
        const int x = x0 + lane / LPR;
        f32x4 v = *at(x, c);
        if (res) v += *reinterpret_cast<const f32x4*>(res + (mw + x) * o.ldr);
        *reinterpret_cast<f32x4*>(dst + (mw + x) * o.ldc) = v;
      }
    } else if (o.epi == kEpiSwigluFwd) {
      // B rows interleaved in groups of TNW (TNW / 2 rows of W_1, then the same rows of
      // W_3; launch_cast_weights with gemm_wave_cols): columns c and c + TNW / 2 hold u and w of
      // the same hidden unit
      constexpr int LPR = TNW / 16, RPI = 64 / LPR;
      const int c = 8 * (lane % LPR), F = o.ffn;
      const long long f = (n0 + wn * TNW) / 2 + c;
#pragma unroll 2
      for (int x0 = 0; x0 < RP; x0 += RPI) {
        const int x = x0 + lane / LPR;
        float u[8], w[8], av[8];
        row8(x, c, u);
        row8(x, TNW / 2 + c, w);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          u[e] = bf2f(f2bf(u[e]));
          w[e] = bf2f(f2bf(w[e]));
          av[e] = u[e] * sigmoid(u[e]) * w[e];
        }
        bf16x8* const up = reinterpret_cast<bf16x8*>(reinterpret_cast<bf16_t*>(o.out) + (mw + x) * 2 * F + f);
        bf16x8* const wp = reinterpret_cast<bf16x8*>(reinterpret_cast<bf16_t*>(o.out) + (mw + x) * 2 * F + F + f);
        bf16x8* const ap = reinterpret_cast<bf16x8*>(reinterpret_cast<bf16_t*>(o.out2) + (mw + x) * F + f);
        if (g.stream_out) {
          asm volatile("" ::: "memory");   // keeps the two branches' stores from being merged
          __builtin_nontemporal_store(make_chunk<bf16_t>(u), up);
          __builtin_nontemporal_store(make_chunk<bf16_t>(w), wp);
          __builtin_nontemporal_store(make_chunk<bf16_t>(av), ap);
          asm volatile("" ::: "memory");
        } else {
          *up = make_chunk<bf16_t>(u);
          *wp = make_chunk<bf16_t>(w);
          *ap = make_chunk<bf16_t>(av);
        }
      }
    } else {
      constexpr int LPR = TNW / 8, RPI = 64 / LPR;
      const int c = 8 * (lane % LPR), n = (int)n0 + wn * TNW + c;
      if (o.epi == kEpiSwigluBwd) {
        // v = da for hidden units n .. n + 7; u, w from the forward pass (bf16 [M, 2F])
        const int F = o.ffn;
#pragma unroll 2
        for (int x0 = 0; x0 < RP; x0 += RPI) {
          const int x = x0 + lane / LPR;
          const bf16_t* const uwp = reinterpret_cast<const bf16_t*>(o.aux) + (mw + x) * 2 * F + n;
          const bf16x8 ub = load_chunk(uwp), wb = load_chunk(uwp + F);
          float v[8], du[8], dw[8];
          row8(x, c, v);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float uf = (float)ub[e], wf = (float)wb[e], sg = sigmoid(uf);
            du[e] = v[e] * wf * sg * (1.0f + uf * (1.0f - sg));
            dw[e] = v[e] * uf * sg;
          }
          bf16_t* const dst = reinterpret_cast<bf16_t*>(o.out) + (mw + x) * 2 * F + n;
          *reinterpret_cast<bf16x8*>(dst) = make_chunk<bf16_t>(du);
          *reinterpret_cast<bf16x8*>(dst + F) = make_chunk<bf16_t>(dw);
        }
      } else {
        // token rows, or [part][b][head][token][d]: eight columns lie in one head's row
        int hp = 0;
        long long coff = n;
        if (o.epi == kEpiHeads) {
          hp = n / o.part_cols;
          const int cc = n - hp * o.part_cols;
          coff = ((long long)(cc >> o.lgd) << (o.lgn + o.lgd)) + (cc & ((1 << o.lgd) - 1));
        }
#pragma unroll 4
        for (int x0 = 0; x0 < RP; x0 += RPI) {
          const int x = x0 + lane / LPR;
          const long long m = mw + x;
          float v[8];
          row8(x, c, v);
          bf16_t* dst;
          if (o.epi == kEpiBf16) {
            dst = reinterpret_cast<bf16_t*>(o.out) + m * o.ldc + coff;
          } else {
            const long long b = m >> o.lgn, t = m & ((1LL << o.lgn) - 1);
            dst = reinterpret_cast<bf16_t*>(o.parts[hp]) + ((b * o.heads) << (o.lgn + o.lgd)) + coff + (t << o.lgd);
          }
          *reinterpret_cast<bf16x8*>(dst) = make_chunk<bf16_t>(v);
        }
      }
    }
    wave_sync();
  }
}

// ---- RMSNorm: one wave per row; lane L holds columns 2L + 128 t, t < C / 128 ----

template <int CT>
__global__ void __launch_bounds__(256) rmsnorm_fwd_kernel(const float* __restrict__ x, const float* __restrict__ gain,
                                                          const float* __restrict__ wg, long long rows,
                                                          bf16_t* __restrict__ xn, float* __restrict__ rstd,
                                                          float* __restrict__ gate) {
  constexpr int C = 128 * CT;
  const int lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const float* xr = x + row * C;
  float2 v[CT];
  float ss = 0.f;
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    v[t] = *reinterpret_cast<const float2*>(xr + 128 * t + 2 * lane);
    ss += v[t].x * v[t].x + v[t].y * v[t].y;
  }
  ss = wave_sum(ss);
  const float rs = 1.0f / sqrtf(ss / (float)C + kNormEps);
  float gd[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int c = 128 * t + 2 * lane;
    const float2 gg = *reinterpret_cast<const float2*>(gain + c);
    const float a0 = v[t].x * rs * gg.x, a1 = v[t].y * rs * gg.y;
    *reinterpret_cast<uint32_t*>(xn + row * C + c) = (uint32_t)f2bf(a0) | ((uint32_t)f2bf(a1) << 16);
    if (wg) {
#pragma unroll
      for (int jj = 0; jj < 3; ++jj) {
        const float2 w = *reinterpret_cast<const float2*>(wg + jj * C + c);
        gd[jj] += a0 * w.x + a1 * w.y;
      }
    }
  }
  if (wg) {
#pragma unroll
    for (int jj = 0; jj < 3; ++jj) gd[jj] = wave_sum(gd[jj]);
    if (lane == 0) {
#pragma unroll
      for (int jj = 0; jj < 3; ++jj) gate[row * 3 + jj] = gd[jj];
    }
  }
  if (lane == 0) rstd[row] = rs;
}

// dx = dres + r (dxh - xh mean(dxh xh)) with xh = x r, dxh = (dxn + dgate W_g) g, per row.
// Workgroup b owns a contiguous run of rows (wave w takes every fourth row from w); the
// sums over its rows of dg = (dxn + dgate W_g) xh and dW_g = dgate (xh g) go to
// part[b][4C] (dg, then dW_g row by row; zero without dgate), the four waves' sums added in
// wave order.
template <int CT>
__global__ void __launch_bounds__(256) rmsnorm_bwd_kernel(const float* __restrict__ dxn, const float* __restrict__ x,
                                                          const float* __restrict__ rstd, const float* __restrict__ gain,
                                                          const float* __restrict__ dres, const float* __restrict__ dgate,
                                                          const float* __restrict__ wg, long long rows, int rpg,
                                                          float* __restrict__ dx, bf16_t* __restrict__ dx16,
                                                          float* __restrict__ part) {
  constexpr int C = 128 * CT;
  __shared__ float red[3][4 * C];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long long g0 = (long long)blockIdx.x * rpg, g1 = g0 + rpg < rows ? g0 + rpg : rows;
  float2 gg[CT], ag[CT], w[3][CT], aw[3][CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int c = 128 * t + 2 * lane;
    gg[t] = *reinterpret_cast<const float2*>(gain + c);
    ag[t] = make_float2(0.f, 0.f);
#pragma unroll
    for (int jj = 0; jj < 3; ++jj) {
      w[jj][t] = dgate ? *reinterpret_cast<const float2*>(wg + jj * C + c) : make_float2(0.f, 0.f);
      aw[jj][t] = make_float2(0.f, 0.f);
    }
  }
  for (long long row = g0 + wid; row < g1; row += 4) {
    const float rs = rstd[row];
    float dga[3] = {0.f, 0.f, 0.f};
    if (dgate) {
#pragma unroll
      for (int jj = 0; jj < 3; ++jj) dga[jj] = dgate[row * 3 + jj];
    }
    float2 dn[CT], xh[CT], dr[CT];
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int c = 128 * t + 2 * lane;
      dn[t] = *reinterpret_cast<const float2*>(dxn + row * C + c);
      dr[t] = *reinterpret_cast<const float2*>(dres + row * C + c);
      const float2 xv = *reinterpret_cast<const float2*>(x + row * C + c);
#pragma unroll
      for (int jj = 0; jj < 3; ++jj) {
        dn[t].x += dga[jj] * w[jj][t].x;
        dn[t].y += dga[jj] * w[jj][t].y;
      }
      xh[t] = make_float2(xv.x * rs, xv.y * rs);
      s += dn[t].x * gg[t].x * xh[t].x + dn[t].y * gg[t].y * xh[t].y;
      ag[t].x += dn[t].x * xh[t].x;
      ag[t].y += dn[t].y * xh[t].y;
#pragma unroll
      for (int jj = 0; jj < 3; ++jj) {
        aw[jj][t].x += dga[jj] * xh[t].x * gg[t].x;
        aw[jj][t].y += dga[jj] * xh[t].y * gg[t].y;
      }
    }
    s = wave_sum(s) / (float)C;
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int c = 128 * t + 2 * lane;
      const float d0 = rs * (dn[t].x * gg[t].x - xh[t].x * s) + dr[t].x;
      const float d1 = rs * (dn[t].y * gg[t].y - xh[t].y * s) + dr[t].y;
      *reinterpret_cast<float2*>(dx + row * C + c) = make_float2(d0, d1);
      if (dx16) *reinterpret_cast<uint32_t*>(dx16 + row * C + c) = (uint32_t)f2bf(d0) | ((uint32_t)f2bf(d1) << 16);
    }
  }
  if (wid > 0) {
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int c = 128 * t + 2 * lane;
      *reinterpret_cast<float2*>(&red[wid - 1][c]) = ag[t];
#pragma unroll
      for (int jj = 0; jj < 3; ++jj) *reinterpret_cast<float2*>(&red[wid - 1][(1 + jj) * C + c]) = aw[jj][t];
    }
  }
  __syncthreads();
  if (wid == 0) {
    float* pw = part + (long long)blockIdx.x * 4 * C;
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int c = 128 * t + 2 * lane;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float2 v = q == 0 ? ag[t] : aw[q - 1][t];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const float2 o = *reinterpret_cast<const float2*>(&red[k][q * C + c]);
          v.x += o.x;
          v.y += o.y;
        }
        *reinterpret_cast<float2*>(pw + q * C + c) = v;
      }
    }
  }
}

// out[by * ncols + c] = sum over rows p in [32 by, 32 by + 32) (below P) of
// part[p * ld + col0 + c], c < ncols; wave w sums rows 32 by + 8 w .. + 8 and the four
// waves' sums are added in wave order.
__global__ void __launch_bounds__(256) colsum_kernel(const float* __restrict__ part, int P, long long ld, int col0,
                                                     int ncols, float* __restrict__ out) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + lane;
  const int p0 = blockIdx.y * 32 + w * 8;
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = c < ncols && p0 + i < P ? part[(long long)(p0 + i) * ld + col0 + c] : 0.f;
  float s = v[0];
#pragma unroll
  for (int i = 1; i < 8; ++i) s += v[i];
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && c < ncols) out[(long long)blockIdx.y * ncols + c] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// out[i] = sum over s of part[s * stride + i], four elements per thread, splits in order.
__global__ void __launch_bounds__(256) splitk_sum_kernel(const float* __restrict__ part, int S, long long stride,
                                                         long long count4, float* __restrict__ out) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= count4) return;
  float4 s = reinterpret_cast<const float4*>(part)[i];
  for (int k = 1; k < S; ++k) {
    const float4 v = reinterpret_cast<const float4*>(part + k * stride)[i];
    s.x += v.x;
    s.y += v.y;
    s.z += v.z;
    s.w += v.w;
  }
  reinterpret_cast<float4*>(out)[i] = s;
}

// [M, 3C] bf16 token-major rows from dq, dk, dv [B, H, N, d] f32, eight elements per thread.
__global__ void __launch_bounds__(256) pack_qkv_kernel(const float* __restrict__ dq, const float* __restrict__ dk,
                                                       const float* __restrict__ dv, long long rows, int C, int H,
                                                       int lgn, int lgd, bf16_t* __restrict__ out) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  const int c8 = 3 * C / 8;
  if (idx >= rows * c8) return;
  const long long m = idx / c8;
  const int col = (int)(idx - m * c8) * 8;
  const int p = col / C, c = col - p * C;
  const float* src = p == 0 ? dq : (p == 1 ? dk : dv);
  const long long b = m >> lgn, t = m & ((1LL << lgn) - 1);
  const long long h = c >> lgd, dd = c & ((1 << lgd) - 1);
  const f32x8 v = load_chunk(src + ((((b * H + h) << lgn) + t) << lgd) + dd);
  float o[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = v[e];
  *reinterpret_cast<bf16x8*>(out + m * 3 * C + col) = make_chunk<bf16_t>(o);
}

__global__ void __launch_bounds__(256) cast_bf16_kernel(const float* __restrict__ src, long long n8,
                                                        bf16_t* __restrict__ dst) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  const f32x8 v = load_chunk(src + 8 * i);
  float o[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = v[e];
  *reinterpret_cast<bf16x8*>(dst + 8 * i) = make_chunk<bf16_t>(o);
}

// The block's weights in bf16 as the forward's products read them, one launch for all (four
// launches of a few microseconds each before): eight values per thread, the segments one after
// the other (wqkv, wo, w2 as they are, then w13). Rows of the interleaved [W_1; W_3] operand
// come in groups of G: row r takes row (G / 2)(r / G) + r % G of W_1 when r % G < G / 2, else
// row (G / 2)(r / G) + r % G - G / 2 of W_3 (C a multiple of 8).
struct CastWeights {
  const float* src[5];   // wqkv, wo, w2, w1, w3
  bf16_t* dst[4];        // wqkv, wo, w2, w13
  long long n8[4];       // eight-value pieces of each
  int C, G;
};
__global__ void __launch_bounds__(256) cast_weights_kernel(CastWeights a) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  const float* src = a.src[0];
  bf16_t* dst = a.dst[0];
  int seg = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (seg == k && i >= a.n8[k]) {
      i -= a.n8[k];
      seg = k + 1;
      src = a.src[k + 1];
      dst = a.dst[k + 1];
    }
  if (seg == 3) {
    if (i >= a.n8[3]) return;
    const int c8 = a.C / 8, r = (int)(i / c8), c = (int)(i - (long long)r * c8) * 8;
    const int g = r / a.G, wi = r % a.G, h = a.G / 2;
    src = (wi < h ? a.src[3] + (long long)(h * g + wi) * a.C : a.src[4] + (long long)(h * g + wi - h) * a.C) + c;
  } else {
    src += 8 * i;
  }
  const f32x8 v = load_chunk(src);
  float o[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = v[e];
  *reinterpret_cast<bf16x8*>(dst + 8 * i) = make_chunk<bf16_t>(o);
}

// Five transposed casts in one launch: dst[c * ldd + r] = bf16(src[r * cols + c]) for [rows,
// cols] f32 matrices (32 x 32 tiles through LDS; rows and cols multiples of 32), the matrices'
// tiles one after the other.
struct CastWeightsT {
  const float* src[5];
  bf16_t* dst[5];
  int rows[5], cols[5], ldd[5];
};
__global__ void __launch_bounds__(256) cast_weights_t_kernel(CastWeightsT a) {
  __shared__ float tile[32][33];
  int id = blockIdx.x, k = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int nt = (a.rows[q] / 32) * (a.cols[q] / 32);
    if (k == q && id >= nt) {
      id -= nt;
      k = q + 1;
    }
  }
  const int cols = a.cols[k], tpr = cols / 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int r0 = id / tpr * 32, c0 = id % tpr * 32;
  const float* src = a.src[k];
  bf16_t* dst = a.dst[k];
#pragma unroll
  for (int q = 0; q < 4; ++q) tile[ty + 8 * q][tx] = src[(long long)(r0 + ty + 8 * q) * cols + c0 + tx];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) dst[(long long)(c0 + ty + 8 * q) * a.ldd[k] + r0 + tx] = f2bf(tile[tx][ty + 8 * q]);
}

unsigned blocks_for(long long n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

// Workgroup tile of a product: 256 x 256 (8 waves of 64 x 128, tiles of 32 along the
// contraction in four stages) where the shape allows and gives at least 256 tiles; else 128 x
// 128 (4 waves of 64 x 64, two workgroups per CU) if that gives at least 256 tiles; else 64 x
// 64 (4 waves of 32 x 32, four stages: few workgroups, each bound by the latency of its
// tiles). At 65536 rows 256 x 128 and 128 x 256 tiles of 4 waves, two workgroups per CU, took
// 2.32-2.34 ms for the block's products instead of 2.18; at 1024 rows, C = 512, F = 2048 the
// forward's four products take 40 us with 64 x 64 tiles instead of 66 with 128 x 128.
int gemm_tile(int M, int N) {
  if (M % 256 == 0 && N % 256 == 0 && (long long)(M / 256) * (N / 256) >= 256) return 256;
  return (long long)(M / 128) * (N / 128) >= 256 ? 128 : 64;
}

// Tile of a weight gradient with `splits` splits of the contraction: 128 x 128 where 256 x 256
// tiles and the base number of splits leave a quarter of the CUs or more without a workgroup.
int wgrad_tile(int M, int N, long long K) {
  return M % 256 == 0 && N % 256 == 0 && (long long)(M / 256) * (N / 256) * gemm_splits(M, N, K) >= 192 ? 256 : 128;
}

hipError_t launch_gemm(bool trans, const GemmMat& a, const GemmMat& b, int M, int N, long long K, int splits,
                       const GemmOut& o, hipStream_t st) {
  if (M <= 0 || N <= 0 || K <= 0 || M % 128 || N % 128 || K % 64 || splits < 1 || (K / 64) % splits)
    return hipErrorInvalidValue;
  if (o.epi != kEpiPart && splits != 1) return hipErrorInvalidValue;
  const int T = trans ? wgrad_tile(M, N, K) : gemm_tile(M, N);
  GemmArgs g{a, b, N / T, (int)((K / 64) / splits), o, (long long)M * o.ldc, false};
  if (T == 256) g.kt_per *= 2;   // tiles of 32
  // u, w and silu(u) w together larger than the last-level cache: storing them past the caches
  // leaves those to the operands (65536 rows, F = 2048: 413 -> 348 us); smaller ones are
  // better found there by the next product
  g.stream_out = o.epi == kEpiSwigluFwd && 6LL * M * o.ffn >= (256LL << 20);
  const dim3 grid((unsigned)((M / T) * (N / T)), (unsigned)splits);
  if (T == 256) {
    if (trans)
      gemm_kernel<true, 256, 256, 4, 2, 32, 4><<<grid, 512, 0, st>>>(g);
    else
      gemm_kernel<false, 256, 256, 4, 2, 32, 4><<<grid, 512, 0, st>>>(g);
  } else if (trans) {
    gemm_kernel<true, 128, 128, 2, 2, 64, 2><<<grid, 256, 0, st>>>(g);
  } else if (T == 128) {
    gemm_kernel<false, 128, 128, 2, 2, 64, 2><<<grid, 256, 0, st>>>(g);
  } else {
    gemm_kernel<false, 64, 64, 2, 2, 64, 4><<<grid, 256, 0, st>>>(g);
  }
  return hipGetLastError();
}

int gemm_wave_cols(int M, int N) { return gemm_tile(M, N) / 2; }

int gemm_splits(int M, int N, long long K) {
  const int T = M % 256 == 0 && N % 256 == 0 ? 256 : 128;
  const long long tiles = (long long)(M / T) * (N / T);
  const long long nkt = K / 64;
  int s = 1;
  // about one workgroup per CU (each split adds a partial product the sum reads back), at
  // least 16 contraction tiles per split
  while (tiles * s < 256 && nkt % (2 * s) == 0 && nkt / (2 * s) >= 16) s *= 2;
  return s;
}

int wgrad_splits(int M, int N, long long K, size_t part_bytes) {
  int s = gemm_splits(M, N, K);
  if (wgrad_tile(M, N, K) == 256) return s;
  // 128 x 128 tiles: up to two workgroups per CU, at least 8 contraction tiles per split, and
  // partial products that fit the workspace
  const long long tiles = (long long)(M / 128) * (N / 128), nkt = K / 64;
  while (tiles * s < 512 && nkt % (2 * s) == 0 && nkt / (2 * s) >= 8 &&
         sizeof(float) * (size_t)(2 * s) * M * N <= part_bytes)
    s *= 2;
  return s;
}

hipError_t launch_rmsnorm_fwd(const float* x, const float* gain, const float* wg, long long rows, int C, uint16_t* xn,
                              float* rstd, float* gate, hipStream_t st) {
  const unsigned nb = blocks_for(rows, 4);
  bf16_t* o = reinterpret_cast<bf16_t*>(xn);
  switch (C) {
    case 128: rmsnorm_fwd_kernel<1><<<nb, 256, 0, st>>>(x, gain, wg, rows, o, rstd, gate); break;
    case 256: rmsnorm_fwd_kernel<2><<<nb, 256, 0, st>>>(x, gain, wg, rows, o, rstd, gate); break;
    case 512: rmsnorm_fwd_kernel<4><<<nb, 256, 0, st>>>(x, gain, wg, rows, o, rstd, gate); break;
    case 1024: rmsnorm_fwd_kernel<8><<<nb, 256, 0, st>>>(x, gain, wg, rows, o, rstd, gate); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// row groups of the RMSNorm backward: up to 1024 workgroups, at least 16 rows each
int rmsnorm_bwd_groups(long long rows) {
  const long long g = (rows + 15) / 16;
  return (int)(g < 1024 ? g : 1024);
}

// deterministic column sums of part [P][ld] (columns col0 .. col0 + ncols - 1) into out, in
// two levels (32-row partial sums in tmp [ceil(P / 32)][ncols], then their sum)
hipError_t colsum(const float* part, int P, long long ld, int col0, int ncols, float* tmp, float* out, hipStream_t st) {
  const int rs = (P + 31) / 32;
  if (rs == 1) {
    colsum_kernel<<<dim3(blocks_for(ncols, 64), 1), 256, 0, st>>>(part, P, ld, col0, ncols, out);
    return hipGetLastError();
  }
  colsum_kernel<<<dim3(blocks_for(ncols, 64), rs), 256, 0, st>>>(part, P, ld, col0, ncols, tmp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return colsum(tmp, rs, ncols, 0, ncols, tmp + (long long)rs * ncols, out, st);
}

hipError_t launch_rmsnorm_bwd(const float* dxn, const float* x, const float* rstd, const float* gain, const float* dres,
                              const float* dgate, const float* wg, long long rows, int C, float* dx, uint16_t* dx16,
                              float* part, float* dgain, float* dwg, hipStream_t st) {
  const int ng = rmsnorm_bwd_groups(rows);
  const int rpg = (int)((rows + ng - 1) / ng);
  bf16_t* o16 = reinterpret_cast<bf16_t*>(dx16);
  switch (C) {
    case 128: rmsnorm_bwd_kernel<1><<<ng, 256, 0, st>>>(dxn, x, rstd, gain, dres, dgate, wg, rows, rpg, dx, o16, part); break;
    case 256: rmsnorm_bwd_kernel<2><<<ng, 256, 0, st>>>(dxn, x, rstd, gain, dres, dgate, wg, rows, rpg, dx, o16, part); break;
    case 512: rmsnorm_bwd_kernel<4><<<ng, 256, 0, st>>>(dxn, x, rstd, gain, dres, dgate, wg, rows, rpg, dx, o16, part); break;
    case 1024: rmsnorm_bwd_kernel<8><<<ng, 256, 0, st>>>(dxn, x, rstd, gain, dres, dgate, wg, rows, rpg, dx, o16, part); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  float* tmp = part + (long long)ng * 4 * C;
  e = colsum(part, ng, 4LL * C, 0, C, tmp, dgain, st);
  if (e != hipSuccess || !dgate) return e;
  return colsum(part, ng, 4LL * C, C, 3 * C, tmp, dwg, st);
}

size_t rmsnorm_bwd_part_bytes(long long rows, int C) {
  // partial rows, then the first level of the column sums (at most 32 rows) and the second
  const long long ng = rmsnorm_bwd_groups(rows);
  return sizeof(float) * (size_t)(ng + 32 + 1) * 4 * C;
}

hipError_t launch_splitk_sum(const float* part, int S, long long stride, long long count, float* out, hipStream_t st) {
  if (count % 4 || stride % 4) return hipErrorInvalidValue;
  splitk_sum_kernel<<<blocks_for(count / 4, 256), 256, 0, st>>>(part, S, stride, count / 4, out);
  return hipGetLastError();
}

hipError_t launch_pack_qkv(const float* dq, const float* dk, const float* dv, long long rows, int C, int H, int lgn,
                           int lgd, uint16_t* out, hipStream_t st) {
  if (C % 8) return hipErrorInvalidValue;
  pack_qkv_kernel<<<blocks_for(rows * (3 * C / 8), 256), 256, 0, st>>>(dq, dk, dv, rows, C, H, lgn, lgd,
                                                                        reinterpret_cast<bf16_t*>(out));
  return hipGetLastError();
}

hipError_t launch_cast_bf16(const float* src, long long n, uint16_t* dst, hipStream_t st) {
  if (n % 8) return hipErrorInvalidValue;
  cast_bf16_kernel<<<blocks_for(n / 8, 256), 256, 0, st>>>(src, n / 8, reinterpret_cast<bf16_t*>(dst));
  return hipGetLastError();
}

hipError_t launch_cast_weights(const float* wqkv, const float* wo, const float* w1, const float* w3, const float* w2,
                               int C, int F, int G, uint16_t* oqkv, uint16_t* oo, uint16_t* o13, uint16_t* o2,
                               hipStream_t st) {
  if (G <= 0 || G % 2 || (2 * F) % G || C % 8) return hipErrorInvalidValue;
  const long long cc = (long long)C * C / 8, cf = (long long)C * F / 8;
  const CastWeights a{{wqkv, wo, w2, w1, w3}, {oqkv, oo, o2, o13}, {3 * cc, cc, cf, 2 * cf}, C, G};
  cast_weights_kernel<<<blocks_for(4 * cc + 3 * cf, 256), 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_cast_weights_t(const float* wqkv, const float* wo, const float* w1, const float* w3, const float* w2,
                                 int C, int F, uint16_t* oqkv, uint16_t* oo, uint16_t* o13, uint16_t* o2,
                                 hipStream_t st) {
  if (C % 32 || F % 32) return hipErrorInvalidValue;
  const CastWeightsT a{{wqkv, wo, w1, w3, w2},
                       {oqkv, oo, o13, o13 + F, o2},
                       {3 * C, C, F, F, C},
                       {C, C, C, C, F},
                       {3 * C, C, 2 * F, 2 * F, C}};
  cast_weights_t_kernel<<<(unsigned)((C / 32) * (4 * (C / 32) + 3 * (F / 32))), 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace bsa
