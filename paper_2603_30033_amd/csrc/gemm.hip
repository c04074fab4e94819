// Dense products of the Tucker-attention forward that are plain GEMMs, on bf16/fp32 MFMA:
//   projection   [Qlat | K | V](tok) = [U2 | U3 | U~3]^T x(tok)      (Qlat = X U2, K = X U3,
//                V = X U~3 of Section "KV Caching"), with latent RoPE on K in the epilogue
//                (Definition "Latent RoPE": the key rotation is computed once for all heads)
//   latent merge Z(tok) = sum_i G~_i O_i(tok)                          (head merge through the
//                post-softmax core, from the contraction of H1 and H2 over heads)
//   output       Y(tok) = U~2 Z(tok)                                   (output-mode basis; prefill-sized
//                calls with a short contraction use the dedicated kernel of out_proj.hip)
// With a shared key-value latent the projection has no V rows: the K block's accumulators are
// stored unrotated as V (and as the cache row) before they are rotated.
// All three compute acc[m][tok] = sum_k A[m][k] B[tok][k] with the weight side as MFMA rows
// and tokens as MFMA columns, so that an accumulator lane owns one token and four
// consecutive output channels per register quad.
//
// Tiling: workgroup = 4 or 8 waves on a TM x TN tile (weights x tokens).  A stage is RB bytes of every tile row,
// moved from global memory straight into LDS (range-checked buffer loads, no register stage; chunks of a
// row XOR-swizzled against bank conflicts), ST stages in a ring, one barrier per stage.  The waves are dealt
// over the tile AND over the contraction: WGK groups of waves each multiply their own part of every stage, so
// that a wave's piece of the tile stays large (few LDS bytes per matrix instruction) even where the tile is
// small, and the groups' accumulators are added through LDS at the end, in a fixed order.  Split-K over
// workgroups (ksplit > 1, decode) leaves partial tiles for the caller's next kernel to sum.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "params.h"
#include "epilogue.h"

namespace ta {

template <typename T, int TM, int TN, int WGM, int WGN, int WGK, int RB, int ST> struct GemmCfg {
  static constexpr int kWaves = WGM * WGN * WGK;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int CE = 16 / (int)sizeof(T);                // elements per 16-byte chunk
  static constexpr int CPR = RB / 16;                           // chunks per row of a stage
  static constexpr int KS = RB / (int)sizeof(T);                // contraction elements of a stage
  static constexpr int RPP = 1024 / RB;                         // tile rows per 1 KB piece
  // pieces of the two operands of a stage, rounded up so that every wave moves the same number
  static constexpr int PA = (TM / RPP + kWaves - 1) / kWaves, PB = (TN / RPP + kWaves - 1) / kWaves;   // per wave
  static constexpr int kOps = PA + PB;
  static constexpr int kAElems = PA * kWaves * 1024 / (int)sizeof(T);
  static constexpr int kStageElems = kOps * kWaves * 1024 / (int)sizeof(T);
  static constexpr int MB = TM / WGM / 32, NB = TN / WGN / 32;
  static constexpr int CS = CPR / WGK / 2;                      // chunks of a stage per wave and half
  static_assert(CS >= 1 && CS * WGK * 2 == CPR, "every group of waves gets whole chunks");
  static_assert((ST - 2) * kOps < 64, "six-bit counter");
  // reduction over the WGK groups: blocks per round
  static constexpr int kMost = ST < 3 ? 1 : (sizeof(T) == 2 ? 4 : 2);   // what fits beside the rows' patches
  static constexpr int kLess = MB * NB < WGK ? MB * NB : WGK;
  static constexpr int RS = WGK == 1 ? 1 : (kLess < kMost ? kLess : kMost);
  static constexpr size_t kReduceBytes = WGK > 1 ? (size_t)kWaves * RS * 4096 : 0;
  static constexpr int kPatchElems = WGK > 1 ? 32 * (32 + CE) : NB * 32 * (MB * 32 + CE);   // one wave's output rows
  static constexpr size_t kPatchBytes = (size_t)kWaves * kPatchElems * sizeof(T);
  static constexpr size_t kRing = (size_t)ST * kStageElems * sizeof(T);
  static constexpr size_t kTail = kReduceBytes + (WGK > 1 ? kPatchBytes : 0) > kPatchBytes
                                      ? kReduceBytes + (WGK > 1 ? kPatchBytes : 0) : kPatchBytes;
  static constexpr size_t kBytes = kRing > kTail ? kRing : kTail;
  static_assert(kBytes <= 160 * 1024, "fits the LDS of a compute unit");
};

// acc += (16-byte chunk of a row of A) x (chunk of a row of B), both halves of the wave holding different chunks
__device__ __forceinline__ void mma_chunk(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma_chunk(f32x16& acc, const f32x4& a, const f32x4& b) {
#pragma unroll
  for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
}

// Output tile of one wave written as whole rows: accumulators go to a wave-private LDS patch as
// [token][channel], then 16-byte chunks of consecutive channels are stored, eight rows per
// instruction (the accumulator layout itself would store 8-byte pieces 8 KB apart).
template <typename T, int MB, int NB>
__device__ __forceinline__ void store_rows_y(const GemmArgs& g, const f32x16 (&acc)[MB][NB], T* patch,
                                             int m_base, int t_base) {
  constexpr int CW = MB * 32;                                   // channels per patch row
  constexpr int PRE = CW + 16 / sizeof(T);                      // padded row, elements
  constexpr int CE = 16 / sizeof(T);
  constexpr int CPR = CW / CE;                                  // chunks per row
  const int lane = threadIdx.x % kWave, h = lane / 32, lr = lane % 32;
  const int TP = g.Bsz * g.Npad;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        store4(patch + (j * 32 + lr) * PRE + i * 32 + 8 * q + 4 * h, acc[i][j][4 * q], acc[i][j][4 * q + 1],
               acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
  T* Y = static_cast<T*>(g.Out);
#pragma unroll
  for (int it = 0; it < NB * 32 * CPR / kWave; ++it) {
    const int ci = it * kWave + lane;
    const int row = ci / CPR, cc = ci % CPR;
    const int tp = t_base + row, m = m_base + cc * CE;
    if (tp >= TP || m >= g.M) continue;
    const int b = tp / g.Npad, n = tp % g.Npad;
    if (n >= g.N) continue;
    u32x4 v = *reinterpret_cast<const u32x4*>(patch + row * PRE + cc * CE);
    *reinterpret_cast<u32x4*>(Y + ((long)b * g.N + n) * g.ldo + m) = v;
  }
}

// DIRECT: both operands start on 16 bytes, and stages go straight into LDS.
template <typename T, int TM, int TN, int WGM, int WGN, int WGK, int RB, int ST, bool DIRECT>
__global__ __launch_bounds__(64 * WGM * WGN * WGK) void gemm_kernel(GemmArgs g) {
  using Cfg = GemmCfg<T, TM, TN, WGM, WGN, WGK, RB, ST>;
  constexpr int MB = Cfg::MB, NB = Cfg::NB, CE = Cfg::CE, CPR = Cfg::CPR, NW = Cfg::kWaves;
  using Vec = std::conditional_t<sizeof(T) == 2, bf16x8, f32x4>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  T* smem = reinterpret_cast<T*>(smem_raw);

  // Workgroups go to the eight XCDs round-robin in dispatch order (x fastest).  Remap the index
  // so that each XCD works through one contiguous range of (token tile, weight tile) pairs: the
  // weight tiles of one token tile then run on the same XCD back to back, and the token rows
  // they share are fetched into that XCD's L2 once.
  int bx = blockIdx.x, by = blockIdx.y;
  {
    const int gx = gridDim.x, per = gridDim.x * gridDim.y / 8;
    const int lin = bx + gx * by;
    if (lin < per * 8) {
      const int logical = (lin % 8) * per + lin / 8;
      bx = logical % gx;
      by = logical / gx;
    }
  }
  const int m_tile = bx * TM, t_tile = by * TN;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int wm = wave % WGM, wn = (wave / WGM) % WGN, kg = wave / (WGM * WGN);
  const int h = lane / 32, lr = lane % 32;
  const int TP = g.Bsz * g.Npad;

  // Operands as buffers that start at the tile's first row; a row that does not exist (past the weights, a
  // padding token of the caller's unpadded X) and elements past the contraction get an offset beyond the
  // descriptor's size, and the range check of the load supplies zeros for them.
  constexpr uint32_t kNone = 0x80000000u;
  auto buffer = [](const T* base, long bytes) {
    const long lim = 0x7fffffffl;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), 0, (int)(bytes < 0 ? 0 : (bytes > lim ? lim : bytes)),
                                             0x00020000);
  };
  const long TR = g.src_padded ? (long)TP : (long)g.Bsz * g.N;  // rows the token source holds
  auto src_row = [&](int tp) -> long {                          // source row of padded token tp, -1 if none
    if (tp >= TP) return -1l;
    if (g.src_padded) return tp;
    const int b = tp / g.Npad, n = tp % g.Npad;
    return n < g.N ? (long)b * g.N + n : -1l;
  };
  long row0 = TR;                                               // first source row the tile touches
  {
    const int tp = t_tile < TP ? t_tile : TP;
    if (g.src_padded) row0 = tp;
    else if (tp < TP) row0 = (long)(tp / g.Npad) * g.N + min(tp % g.Npad, g.N);
  }
  const __amdgpu_buffer_rsrc_t ra = buffer(static_cast<const T*>(g.A) + (long)m_tile * g.lda,
                                           (long)(g.M - m_tile) * g.lda * (long)sizeof(T));
  const __amdgpu_buffer_rsrc_t rb = buffer(static_cast<const T*>(g.Bsrc) + row0 * g.ldb, (TR - row0) * g.ldb * (long)sizeof(T));
  // piece i of this wave holds tile rows (wave + NW i) RPP ..; the chunk a lane moves is the same in all pieces
  const int prow = lane / CPR;
  const int koff = ((lane % CPR) ^ swz_x<CPR>(wave * Cfg::RPP + prow)) * CE;
  static_assert((NW * Cfg::RPP) % 16 == 0, "the swizzle repeats from piece to piece");
  uint32_t aoff[Cfg::PA], boff[Cfg::PB];
#pragma unroll
  for (int i = 0; i < Cfg::PA; ++i) {
    const int r = (wave + NW * i) * Cfg::RPP + prow;
    aoff[i] = r < TM && m_tile + r < g.M ? (uint32_t)(((long)r * g.lda + koff) * (long)sizeof(T)) : kNone;
  }
#pragma unroll
  for (int i = 0; i < Cfg::PB; ++i) {
    const int r = (wave + NW * i) * Cfg::RPP + prow;
    const long sr = r < TN ? src_row(t_tile + r) : -1l;
    boff[i] = sr < 0 ? kNone : (uint32_t)(((sr - row0) * g.ldb + koff) * (long)sizeof(T));
  }

  // stages of this workgroup's part of the contraction
  const int nk_all = (g.K + Cfg::KS - 1) / Cfg::KS;
  const int per = (nk_all + g.ksplit - 1) / g.ksplit;
  const int s0 = blockIdx.z * per;
  const int cnt = max(min(nk_all, s0 + per) - s0, 0);
  auto issue = [&](int i) {                                     // fetch stage i (past the end: zeros, no memory traffic)
    constexpr int kPiece = 1024 / (int)sizeof(T);
    T* st = smem + (long)(i % ST) * Cfg::kStageElems;
    const int k0 = (s0 + i) * Cfg::KS;
    const bool ok = i < cnt && k0 + koff < g.K;
    const uint32_t kb = (uint32_t)k0 * (uint32_t)sizeof(T);
    auto move = [&](__amdgpu_buffer_rsrc_t r, T* to, uint32_t off) {
      off = ok && off != kNone ? off + kb : kNone;
      if constexpr (DIRECT) buffer_to_lds(r, to, off);
      else buffer_to_lds_by_register(r, to, off, lane);          // (wait_lds in front of the barrier covers the store)
    };
#pragma unroll
    for (int p = 0; p < Cfg::PA; ++p) move(ra, st + (wave + NW * p) * kPiece, aoff[p]);
#pragma unroll
    for (int p = 0; p < Cfg::PB; ++p) move(rb, st + Cfg::kAElems + (wave + NW * p) * kPiece, boff[p]);
  };

  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

#pragma unroll
  for (int i = 0; i < ST - 1; ++i) issue(i);
  const int x = swz_x<CPR>(lr);                                 // swizzle of this lane's fragment rows
  for (int i = 0; i < cnt; ++i) {
    // this wave's share of stage i has landed, and its reads of stage i - 1 have returned; behind the barrier
    // both hold for every wave: stage i is whole, and the slot of stage i - 1 may be filled again
    wait_vm<(ST - 2) * Cfg::kOps>();
    wait_lds();
    __builtin_amdgcn_s_barrier();
    // the next loads are issued behind the products (they hold the wave while the LDS reads could start), except in
    // a two-stage ring, where they are needed at once: 8192 x 384 x 4096 36.0 against 38.4 us, but 65536 x 192 x 768
    // with two stages 32.3 issued first, 35.6 behind
    if (ST == 2) issue(i + ST - 1);
    const T* st = smem + (long)(i % ST) * Cfg::kStageElems;
    const T* la = st + (wm * MB * 32 + lr) * Cfg::KS;
    const T* lb = st + Cfg::kAElems + (wn * NB * 32 + lr) * Cfg::KS;
#pragma unroll
    for (int c = 0; c < Cfg::CS; ++c) {
      const int ch = (((kg * Cfg::CS + c) * 2 + h) ^ x) * CE;
      Vec fa[MB], fb[NB];
#pragma unroll
      for (int m = 0; m < MB; ++m) fa[m] = *reinterpret_cast<const Vec*>(la + m * 32 * Cfg::KS + ch);
#pragma unroll
      for (int n = 0; n < NB; ++n) fb[n] = *reinterpret_cast<const Vec*>(lb + n * 32 * Cfg::KS + ch);
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) mma_chunk(acc[m][n], fa[m], fb[n]);
    }
    if (ST > 2) issue(i + ST - 1);
  }
  wait_vm<0>();                                                 // nothing may land in LDS from here on
  __syncthreads();

  const int Mp = g.epi == 0 ? g.R2 + (g.shared_kv ? 1 : 2) * g.D : pad32(g.M);
  auto finish = [&](const f32x16& v, int m0, int t0, T* patch) {  // one 32x32 block of finished sums
    const int tp = t0 + lr;
    if (m0 >= Mp) return;
    if (g.ksplit > 1) {
      if (tp < TP) {
        float* dst = g.part + ((long)blockIdx.z * TP + tp) * Mp + m0 + 4 * h;
#pragma unroll
        for (int q = 0; q < 4; ++q) store4(dst + 8 * q, v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
      }
    } else if (g.epi == 2) {
      const f32x16 one[1][1] = {{v}};
      store_rows_y<T, 1, 1>(g, one, patch, m0, t0);
    } else {
      epilogue_block<T>(g, v, m0, tp, 0);                       // (not a decode step: see launch_gemm)
    }
  };
  constexpr int NBLK = MB * NB;
  // (the block loops are not unrolled: one copy of the epilogue's code)
  if constexpr (WGK == 1) {
    T* patch = smem + (long)wave * Cfg::kPatchElems;
    if (g.epi == 2 && g.ksplit <= 1) {                          // Y: whole rows through LDS
      store_rows_y<T, MB, NB>(g, acc, patch, m_tile + wm * MB * 32, t_tile + wn * NB * 32);
      return;
    }
#pragma clang loop unroll(disable)
    for (int k = 0; k < NBLK; ++k) {
      f32x16 v;
#pragma unroll
      for (int u = 0; u < NBLK; ++u)
        if (u == k) v = acc[u / NB][u % NB];
      finish(v, m_tile + (wm * MB + k / NB) * 32, t_tile + (wn * NB + k % NB) * 32, patch);
    }
  } else {
    // RS blocks of every wave per round: all groups leave them in LDS, then one wave per block adds the WGK
    // parts in group order and finishes it
    constexpr int RS = Cfg::RS, WMN = WGM * WGN;
    f32x4* red = reinterpret_cast<f32x4*>(smem_raw);
    T* patch = reinterpret_cast<T*>(smem_raw + Cfg::kReduceBytes) + (long)wave * Cfg::kPatchElems;
    static_assert(RS * WMN <= NW, "one wave per block of a round");
#pragma clang loop unroll(disable)
    for (int r0 = 0; r0 < NBLK; r0 += RS) {
      if (r0 > 0) __syncthreads();
#pragma unroll
      for (int u = 0; u < NBLK; ++u) {
        if (u < r0 || u >= r0 + RS) continue;
        f32x4* slot = red + (((long)kg * WMN + wn * WGM + wm) * RS + (u - r0)) * 256 + lane;
        const f32x16 v = acc[u / NB][u % NB];
#pragma unroll
        for (int q = 0; q < 4; ++q) slot[q * 64] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
      }
      __syncthreads();
      const int xs = wave % RS, wmn = wave / RS, u = r0 + xs;
      if (wmn < WMN && u < NBLK) {
        f32x16 v;
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = 0.f;
#pragma unroll
        for (int o = 0; o < WGK; ++o) {
          const f32x4* slot = red + (((long)o * WMN + wmn) * RS + xs) * 256 + lane;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 y = slot[q * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * q + e] += y[e];
          }
        }
        finish(v, m_tile + ((wmn % WGM) * MB + u / NB) * 32, t_tile + ((wmn / WGM) * NB + u % NB) * 32, patch);
      }
    }
  }
}

template <typename T, int TM, int TN, int WGM, int WGN, int WGK, int RB, int ST, bool DIRECT = true>
static hipError_t launch_one(const GemmArgs& a, int m_rows, hipStream_t s) {
  using Cfg = GemmCfg<T, TM, TN, WGM, WGN, WGK, RB, ST>;
  const int TP = a.Bsz * a.Npad;
  dim3 grid((m_rows + TM - 1) / TM, (TP + TN - 1) / TN, a.ksplit > 1 ? a.ksplit : 1);
  auto kern = gemm_kernel<T, TM, TN, WGM, WGN, WGK, RB, ST, DIRECT>;
  static LdsOnce lds_once;                                       // one per kernel instantiation
  if (hipError_t ae = allow_dynamic_lds(lds_once, kern, Cfg::kBytes); ae != hipSuccess) return ae;
  hipLaunchKernelGGL(kern, grid, dim3(Cfg::kThreads), Cfg::kBytes, s, a);
  return hipGetLastError();
}

// Which tile a product runs with.  Times in us of one launch, operands partly cached (M x K x tokens, bf16):
//                                    32x32/8  64x64/4  96x128/8  128x128/8  96x128/4     (tile / waves)
//   384 x 4096 x  8192 (projection)     81       41       35         41        42
//   256 x 4096 x 16384                 105       54       63         43        49
//   192 x  768 x 65536                 101       46       46         51        33
//   192 x  768 x  8192                15.7      8.9     12.1       13.8      12.5
//   128 x 4096 x  8192 (head merge)     30       18       33         36        39
//   128 x 4096 x 16384                  58       29       35         38        41
//    64 x  768 x  8192                 6.4      7.0     10.5       11.8      11.4
//   384 x 4096 x   384                 9.1       17       29         35        36
//  4096 x  384 x  8192                 211       74       82         71        53
// (before, four waves that split the tile only: 48, 63, 39, 14, 25, 36, 7.7, 22.6, 59).  Few tiles: as many
// workgroups as possible, the eight waves of each dealt over the contraction.  A long contraction with enough
// tiles for every compute unit is bound by the bytes that the caches deliver, hence the largest tile that still
// gives each one a workgroup; a short one by the start and the end of a workgroup, hence 56 to 80 KB of LDS,
// so that two workgroups share a compute unit, and by the number of rounds that 512 workgroups at a time make:
//                                    96x128/4  128x128/8  192x128/8
//   192 x  768 x 24576                   15.8      17.8       17.8      1, 1, 1 rounds
//   192 x  768 x 65536 (50432 exist)     30.2      32.6       26.4      2, 2, 1
//   128 x  768 x 34816                   25.4      18.4       23.2      2, 1, 1
//   128 x  768 x 65536                   31.6      23.0       27.1      2, 1, 1
//   256 x  768 x 36864                   29.0      29.3       34.8      2, 2, 2
//   256 x  768 x 65536                   51.8      45.1       52.9      3, 2, 2
//   320 x  768 x 36864                   46.8      37.1       41.7      3, 2, 2
//   320 x  768 x 65536                   75.2      60.2       59.8      4, 3, 2
// A round takes about as long as 30 rows more than a tile has (96x128 alone before; a forward pass over 256 x 197 tokens of 768
// channels 126.9 us then, 120.3 now).  That is for the projection; outputs as whole rows gain nothing (training of 64 x 1024 tokens
// 1183 us with the one tile, 1227 with all three).  fp32 is bound by its matrix instructions (64 cycles each): only
// the number of workgroups matters (192 x 768 x 1018 tokens 8.9 us with 32x32 and four waves, 8.0 with eight, 19
// with 64x64, 21 before; 768 x 192 x 1018 tokens 7.5, 10.0, 8.2, 8.9 before).
template <typename T> static hipError_t launch_tiles(const GemmArgs& a, hipStream_t s) {
  const int m_rows = (a.epi == 0) ? a.R2 + (a.shared_kv ? 1 : 2) * a.D : a.M;
  const long tokens = (long)a.Bsz * a.Npad;
  auto tiles = [&](int tm, int tn) { return (long)((m_rows + tm - 1) / tm) * ((tokens + tn - 1) / tn); };
  const bool few = tiles(64, 64) < kComputeUnits * 3 / 4 || a.ksplit > 1;
  // An operand of the caller's that does not start on 16 bytes (a piece of a larger buffer) is staged through registers,
  // with one tile for all sizes: rows are whole chunks from there on, so only the start decides.
  const bool direct = (reinterpret_cast<uintptr_t>(a.A) | reinterpret_cast<uintptr_t>(a.Bsrc)) % 16 == 0;
  if constexpr (sizeof(T) == 4) {
    if (!direct) return launch_one<T, 32, 32, 1, 1, 4, 128, 4, false>(a, m_rows, s);
    if (few) return launch_one<T, 32, 32, 1, 1, 4, 128, 4>(a, m_rows, s);
    return launch_one<T, 64, 64, 2, 2, 1, 128, 4>(a, m_rows, s);
  } else {
    if (!direct) return launch_one<T, 32, 32, 1, 1, 8, 256, 4, false>(a, m_rows, s);
    if (few) return launch_one<T, 32, 32, 1, 1, 8, 256, 4>(a, m_rows, s);
    if (a.K >= 1024) {
      if (m_rows % 96 == 0 && tiles(96, 128) >= kComputeUnits) return launch_one<T, 96, 128, 1, 2, 4, 128, 4>(a, m_rows, s);
      if (m_rows > 64 && tiles(128, 128) >= kComputeUnits) return launch_one<T, 128, 128, 1, 2, 4, 128, 4>(a, m_rows, s);
    } else if (tiles(96, 128) >= kComputeUnits) {
      auto cost = [&](int tm) { return ((tiles(tm, 128) + 2 * kComputeUnits - 1) / (2 * kComputeUnits)) * (tm + 30); };
      const long least = std::min(cost(96), std::min(cost(128), cost(192)));
      if (a.epi != 0 || cost(96) == least) return launch_one<T, 96, 128, 1, 4, 1, 128, 2>(a, m_rows, s);
      if (cost(128) == least) return launch_one<T, 128, 128, 2, 4, 1, 128, 2>(a, m_rows, s);
      return launch_one<T, 192, 128, 2, 4, 1, 128, 2>(a, m_rows, s);
    }
    return launch_one<T, 64, 64, 1, 1, 4, 128, 4>(a, m_rows, s);
  }
}
hipError_t launch_gemm(int dtype, const GemmArgs& a, hipStream_t s) {
  if (a.decode && a.ksplit < 2) return hipErrorInvalidValue;      // the positions are its caller's next kernel's
  return dtype == 0 ? launch_tiles<float>(a, s) : launch_tiles<bf16>(a, s);
}

}  // namespace ta
