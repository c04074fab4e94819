// Products that contract over tokens, out[m][n] = sum_t A[t][m] B[t][n], for the weight gradients
// of the backward pass (dU = X^T dLatent, dU~2 = dY^T Z, dG = Qlat^T dQ, dG~ = dZ^T O: the
// derivatives of the factor projections and of the head-mixed cores of Definition "Tucker
// Attention").  Both operands are token-major, as the forward and backward kernels leave them, so
// the contraction index is the slow index in memory.  A stage of 64 tokens of each operand goes straight
// into LDS as it lies in memory (range-checked loads, chunks of a row XOR-swizzled) and the MFMA operand
// fragments, which want the contraction index inside a lane, are read with transposing LDS loads: no
// token-minor copy of any operand is made.  Stages never straddle two sequences; rows of padding tokens
// read as zeros.
//
// All products of a backward call run in ONE launch (they are independent; each alone leaves part of the chip
// idle), every workgroup one TM x TN tile of one product over one part of the tokens.  The waves of a workgroup
// are dealt over the tile and over the tokens of a stage, and their sums are added through LDS, as in gemm.hip.
// With the tokens split over workgroups a second launch adds the partial tiles, which are kept in the order in
// which the lanes hold them (whole kilobytes per access).
#include <type_traits>

#include "common.h"
#include "params.h"

namespace ta {

constexpr int kTS = 64;   // tokens per stage

template <typename T, int TM, int TN, int WGM, int WGN, int WGK, int ST> struct TnCfg {
  static constexpr int kWaves = WGM * WGN * WGK, kThreads = 64 * kWaves;
  static constexpr int CE = 16 / (int)sizeof(T);
  static constexpr int CPA = TM / CE, CPB = TN / CE;             // chunks per token row
  static constexpr int PA = kTS * CPA / 64 / kWaves, PB = kTS * CPB / 64 / kWaves;   // 1 KB pieces per wave
  static_assert(PA * kWaves * 64 == kTS * CPA && PB * kWaves * 64 == kTS * CPB, "whole pieces per wave");
  static constexpr int kOps = PA + PB;
  static_assert((ST - 2) * kOps < 64, "six-bit counter");
  static constexpr int kAElems = kTS * TM, kStageElems = kTS * (TM + TN);
  static constexpr int MB = TM / WGM / 32, NB = TN / WGN / 32;
  static constexpr int kTokens = kTS / WGK;                      // tokens of a stage per group of waves
  static_assert(kTokens % (sizeof(T) == 2 ? 16 : 8) == 0, "whole matrix instructions");
  static constexpr int NBLK = MB * NB;
  static constexpr int RS = WGK == 1 ? 1 : (NBLK < WGK ? NBLK : (WGK < 4 ? WGK : 4));   // blocks per reduction round
  static constexpr size_t kRing = (size_t)ST * kStageElems * sizeof(T);
  static constexpr size_t kReduce = (size_t)kWaves * RS * 4096;
  static constexpr size_t kBytes = kRing > kReduce ? kRing : kReduce;
  static_assert(kBytes <= 160 * 1024, "fits the LDS of a compute unit");
};

// operand pieces of one 32-column block for the tokens row0 .. of a swizzled [token][column] tile: bf16 16 tokens
// (two transposing reads, which hand a lane tokens 4h + r and 8 + 4h + r of its column), fp32 8 tokens
struct TnFrag16 { u32x2 q[2]; };
struct TnFrag32 { float v[4]; };
// the pieces of one step: MB blocks of A from column ca on, NB blocks of B from column cb on
template <int CPA, int CPB, int MB, int NB>
__device__ __forceinline__ void tn_read(TnFrag16 (&fa)[MB], TnFrag16 (&fb)[NB], const bf16* la, const bf16* lb, int row0, int ca,
                                        int cb, int lane) {
  uint32_t at[2 * (MB + NB)];
  u32x2 v[2 * (MB + NB)];
#pragma unroll
  for (int k = 0; k < 2 * MB; ++k) at[k] = tr16_address<CPA>(la, row0, ca + 32 * (k / 2), k % 2, lane);
#pragma unroll
  for (int k = 0; k < 2 * NB; ++k) at[2 * MB + k] = tr16_address<CPB>(lb, row0, cb + 32 * (k / 2), k % 2, lane);
  lds_read_tr16(v, at);
#pragma unroll
  for (int k = 0; k < 2 * MB; ++k) fa[k / 2].q[k % 2] = v[k];
#pragma unroll
  for (int k = 0; k < 2 * NB; ++k) fb[k / 2].q[k % 2] = v[2 * MB + k];
}
template <int CPR> __device__ __forceinline__ void tn_read_one(TnFrag32& f, const float* tile, int row0, int col0, int lane) {
  const int h = lane / 32, col = col0 + lane % 32;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = row0 + 4 * h + r;
    f.v[r] = tile[row * (CPR * 4) + (((col / 4) ^ swz_x<CPR>(row)) * 4) + col % 4];
  }
}
template <int CPA, int CPB, int MB, int NB>
__device__ __forceinline__ void tn_read(TnFrag32 (&fa)[MB], TnFrag32 (&fb)[NB], const float* la, const float* lb, int row0, int ca,
                                        int cb, int lane) {
#pragma unroll
  for (int m = 0; m < MB; ++m) tn_read_one<CPA>(fa[m], la, row0, ca + 32 * m, lane);
#pragma unroll
  for (int n = 0; n < NB; ++n) tn_read_one<CPB>(fb[n], lb, row0, cb + 32 * n, lane);
}
__device__ __forceinline__ void tn_mma(f32x16& acc, const TnFrag16& a, const TnFrag16& b) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
      __builtin_bit_cast(bf16x8, u32x4{a.q[0][0], a.q[0][1], a.q[1][0], a.q[1][1]}),
      __builtin_bit_cast(bf16x8, u32x4{b.q[0][0], b.q[0][1], b.q[1][0], b.q[1][1]}), acc, 0, 0, 0);
}
__device__ __forceinline__ void tn_mma(f32x16& acc, const TnFrag32& a, const TnFrag32& b) {
#pragma unroll
  for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[r], b.v[r], acc, 0, 0, 0);
}

// one finished 32x32 block: column ranges routed to their destinations as fp32, a row or column that sits at an
// acc-order position of its 32-block stored at its natural index
__device__ __forceinline__ void tn_store(const TnProduct& p, const f32x16& v, int m0, int n0, int lane) {
  const int h = lane / 32, np = n0 + lane % 32;
  const int nn = p.perm_n ? (np & ~31) + acc_index(np & 31) : np;
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const TnProduct::Out& o = p.out[u];
    if (o.ptr == nullptr || nn < o.n0 || nn >= o.n1) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int mp = 8 * q + 4 * h + e;
        const int m = m0 + (p.perm_m ? acc_index(mp) : mp);
        if (m < p.M) o.ptr[(long)m * o.ld + (nn - o.n0)] = v[4 * q + e];
      }
  }
}

// DIRECT: every operand starts on 16 bytes, and stages go straight into LDS.
template <typename T, int TM, int TN, int WGM, int WGN, int WGK, int ST, bool DIRECT>
__global__ __launch_bounds__(64 * WGM * WGN * WGK) void gemm_tn_kernel(TnArgs a) {
  using Cfg = TnCfg<T, TM, TN, WGM, WGN, WGK, ST>;
  using F = std::conditional_t<sizeof(T) == 2, TnFrag16, TnFrag32>;
  constexpr int MB = Cfg::MB, NB = Cfg::NB, CE = Cfg::CE, NW = Cfg::kWaves;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  T* smem = reinterpret_cast<T*>(smem_raw);

  // Work items in the order (token split, product, row tile, column tile), dealt to the eight XCDs in contiguous
  // ranges: items that run together on an XCD read the same tokens, and neighbours the same columns of A.
  int lin = blockIdx.x;
  if (const int per = gridDim.x / 8; lin < per * 8) lin = (lin % 8) * per + lin / 8;
  // (readfirstlane: what the buffer descriptors are made of must be known to be uniform)
  const int z = __builtin_amdgcn_readfirstlane(lin / a.tiles);
  int t = lin - z * a.tiles, pi = 0;
  while (pi + 1 < a.n && t >= a.p[pi + 1].first_tile) ++pi;
  const TnProduct& p = a.p[__builtin_amdgcn_readfirstlane(pi)];
  t -= p.first_tile;
  const int n_ntiles = (p.cols + TN - 1) / TN;
  const int mt = __builtin_amdgcn_readfirstlane(t / n_ntiles);
  const int m_tile = mt * TM, n_tile = (t - mt * n_ntiles) * TN;

  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int wm = wave % WGM, wn = (wave / WGM) % WGN, kg = wave / (WGM * WGN);

  constexpr uint32_t kNone = 0x80000000u;
  uint32_t aoff[Cfg::PA], boff[Cfg::PB];
#pragma unroll
  for (int i = 0; i < Cfg::PA; ++i) {
    const int ci = (wave + NW * i) * 64 + lane, row = ci / Cfg::CPA;
    const int col = ((ci % Cfg::CPA) ^ swz_x<Cfg::CPA>(row)) * CE;
    aoff[i] = m_tile + col < p.M_ld ? (uint32_t)(((long)row * p.lda + col) * (long)sizeof(T)) : kNone;
  }
#pragma unroll
  for (int i = 0; i < Cfg::PB; ++i) {
    const int ci = (wave + NW * i) * 64 + lane, row = ci / Cfg::CPB;
    const int col = ((ci % Cfg::CPB) ^ swz_x<Cfg::CPB>(row)) * CE;
    boff[i] = n_tile + col < p.cols ? (uint32_t)(((long)row * p.ldb + col) * (long)sizeof(T)) : kNone;
  }
  const int spp = a.Npad / kTS, n_slices = a.Bsz * spp;
  const int per = __builtin_amdgcn_readfirstlane((n_slices + a.ksplit - 1) / a.ksplit);
  const int s0 = __builtin_amdgcn_readfirstlane(min(z * per, n_slices));
  const int cnt = __builtin_amdgcn_readfirstlane(min(n_slices, s0 + per) - s0);   // this workgroup's stages
  // Stages are fetched in order: sequence sb, its tokens sn .. sn + 63 next.  The size of the descriptor makes rows
  // that do not exist (padding tokens of an unpadded operand, stages past the end of this workgroup's range) read
  // as zeros.
  int sb = __builtin_amdgcn_readfirstlane(s0 / spp), sn = (s0 - sb * spp) * kTS, left = cnt;
  auto buffer = [&](const void* mat, long ld, int padded, int tile0) {
    const long row0 = padded ? (long)sb * a.Npad + sn : (long)sb * a.N + sn;
    int rows = padded ? kTS : max(0, min(kTS, a.N - sn));
    if (left <= 0) rows = 0;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(static_cast<const T*>(mat) + (left > 0 ? row0 * ld : 0l) + tile0), 0,
                                             (int)(rows * ld * (long)sizeof(T)), 0x00020000);
  };
  auto issue = [&](int slot) {
    constexpr int kPiece = 1024 / (int)sizeof(T);
    T* st = smem + (long)slot * Cfg::kStageElems;
    const __amdgpu_buffer_rsrc_t ra = buffer(p.At, p.lda, p.a_padded, m_tile);
    const __amdgpu_buffer_rsrc_t rb = buffer(p.Bt, p.ldb, p.b_padded, n_tile);
    auto move = [&](__amdgpu_buffer_rsrc_t r, T* to, uint32_t off) {
      if constexpr (DIRECT) buffer_to_lds(r, to, off);
      else buffer_to_lds_by_register(r, to, off, lane);          // (wait_lds in front of the barrier covers the store)
    };
#pragma unroll
    for (int k = 0; k < Cfg::PA; ++k) move(ra, st + (wave + NW * k) * kPiece, aoff[k]);
#pragma unroll
    for (int k = 0; k < Cfg::PB; ++k) move(rb, st + Cfg::kAElems + (wave + NW * k) * kPiece, boff[k]);
    --left;
    sn += kTS;
    if (sn == a.Npad) { sn = 0; ++sb; }
  };

  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  if (cnt > 0) {                                                // (the same for the whole workgroup)
#pragma unroll
    for (int i = 0; i < ST - 1; ++i) issue(i);
    for (int i = 0; i < cnt; ++i) {
      wait_vm<(ST - 2) * Cfg::kOps>();                          // as in gemm.hip: stage i whole, the slot of i - 1 free
      wait_lds();
      __builtin_amdgcn_s_barrier();
      const T* la = smem + (long)(i % ST) * Cfg::kStageElems;
      const T* lb = la + Cfg::kAElems;
      constexpr int kStep = sizeof(T) == 2 ? 16 : 8;
#pragma unroll
      for (int c = 0; c < Cfg::kTokens; c += kStep) {
        F fa[MB], fb[NB];
        tn_read<Cfg::CPA, Cfg::CPB>(fa, fb, la, lb, kg * Cfg::kTokens + c, wm * MB * 32, wn * NB * 32, lane);
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < NB; ++n) tn_mma(acc[m][n], fa[m], fb[n]);
      }
      issue((i + ST - 1) % ST);                                 // behind the products: it would hold the wave before them
    }
    wait_vm<0>();                                               // nothing may land in LDS from here on
  }
  __syncthreads();

  auto finish = [&](const f32x16& v, int m0, int n0) {
    const int mb = pad32(p.M) / 32, nb = (p.cols + 31) / 32;
    if (m0 / 32 >= mb || n0 / 32 >= nb) return;
    if (a.ksplit > 1) {
      f32x4* dst = reinterpret_cast<f32x4*>(a.part) + (((long)z * a.blocks + p.first_block + (m0 / 32) * nb + n0 / 32) * 256) + lane;
#pragma unroll
      for (int q = 0; q < 4; ++q) dst[q * 64] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    } else {
      tn_store(p, v, m0, n0, lane);
    }
  };
  // RS blocks of every wave per round go through LDS; one wave per block adds the WGK parts in group order
  constexpr int NBLK = Cfg::NBLK, RS = Cfg::RS, WMN = WGM * WGN;
  static_assert(RS * WMN <= NW, "one wave per block of a round");
  f32x4* red = reinterpret_cast<f32x4*>(smem_raw);
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
      finish(v, m_tile + ((wmn % WGM) * MB + u / NB) * 32, n_tile + ((wmn / WGM) * NB + u % NB) * 32);
    }
  }
}

// sum of the partial tiles of all products, in split order; one wave per 32x32 block
__global__ __launch_bounds__(64) void tn_reduce_kernel(TnArgs a) {
  const int lane = threadIdx.x, blk = blockIdx.x;
  int pi = 0;
  while (pi + 1 < a.n && blk >= a.p[pi + 1].first_block) ++pi;
  const TnProduct& p = a.p[pi];
  const f32x4* src = reinterpret_cast<const f32x4*>(a.part) + (long)blk * 256 + lane;
  f32x16 v;
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = 0.f;
  constexpr int U = 4;                                          // splits whose loads are in flight together
  for (int z0 = 0; z0 < a.ksplit; z0 += U) {
    f32x4 y[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) y[u][q] = src[(long)min(z0 + u, a.ksplit - 1) * a.blocks * 256 + q * 64];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (z0 + u < a.ksplit)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[4 * q + e] += y[u][q][e];
  }
  const int nb = (p.cols + 31) / 32, lb = blk - p.first_block;
  tn_store(p, v, lb / nb * 32, lb % nb * 32, lane);
}

// Tile edge: 128 where the products have enough 128-wide tiles to occupy half the chip (bf16), else 64.
static int tn_edge(int dtype, const TnArgs& a) {
  if (dtype == 0) return 64;
  int tiles = 0;
  for (int i = 0; i < a.n; ++i) tiles += (a.p[i].M / 128) * (a.p[i].cols / 128);
  return tiles >= kComputeUnits / 2 ? 128 : 64;
}
static int tn_tiles(int edge, const TnArgs& a) {
  int tiles = 0;
  for (int i = 0; i < a.n; ++i) tiles += ((a.p[i].M + edge - 1) / edge) * ((a.p[i].cols + edge - 1) / edge);
  return tiles;
}
static int tn_blocks(const TnArgs& a) {
  int blocks = 0;
  for (int i = 0; i < a.n; ++i) blocks += (pad32(a.p[i].M) / 32) * ((a.p[i].cols + 31) / 32);
  return blocks;
}
// Most parts for these products and this many tokens: four rounds of workgroups over the chip (the choice below never
// took more: 192 tiles four parts from 184 stages on, 320 in fp32 four), one part per stage, 16.
static int tn_ksplit_most(const TnArgs& a, int tiles) {
  const int slices = a.Bsz * (a.Npad / kTS), fill = (4 * kComputeUnits + tiles - 1) / tiles, most = fill < 16 ? fill : 16;
  return most < slices ? most : slices;
}
// Parts the tokens are split into: the count with the least estimated time, from what was measured (us): a stage of
// 64 tokens 0.76 with 128-wide tiles, 0.34 with 64-wide ones, 1.2 in fp32; 9, 5.4 and 7 for a workgroup's start and
// reduction; 4.5 for the second launch and 0.001 per partial block.  A compute unit holds one workgroup, one and a
// half effective ones of the 64-wide bf16 tiles (64 KB of LDS).  Measured, launch + second launch: LLaMA-7B shape
// (192 tiles of 128, 128 stages) 102 unsplit, 107 + 9 in two, 116 + 11 in three, 106 + 16 in five parts; GPT-2 shape
// (72 tiles of 64, 128 stages) 44, 25 + 5, 19 + 6, 19 + 7; the same in fp32 with 16 stages 26, 16 + 5, 14 + 6, 21 + 7.
// (Before, one launch per product and one per reduction: 168 + 40, 55 + 25 and 42 + 24.)
static int tn_ksplit(int dtype, const TnArgs& a) {
  const int edge = tn_edge(dtype, a), tiles = tn_tiles(edge, a), blocks = tn_blocks(a), slices = a.Bsz * (a.Npad / kTS);
  const double stage = dtype == 0 ? 1.2 : edge == 128 ? 0.76 : 0.34, fixed = dtype == 0 ? 7. : edge == 128 ? 9. : 5.4;
  int best = 1;
  double cost = 1e30;
  for (int ks = 1; ks <= tn_ksplit_most(a, tiles); ++ks) {
    double rounds = dtype == 1 && edge == 64 ? tiles * ks / (1.5 * kComputeUnits) : (tiles * ks + kComputeUnits - 1) / kComputeUnits;
    if (rounds < 1.) rounds = 1.;
    const double c = rounds * ((slices + ks - 1) / ks * stage + fixed) + (ks > 1 ? 4.5 + 0.001 * ks * blocks : 0.);
    if (c < cost) { cost = c; best = ks; }
  }
  return best;
}
// Scratch for the most parts, not for the chosen count: that one moves up and down with the tokens, and a workspace made for
// more tokens is to serve fewer.
size_t tn_part_bytes(int dtype, const TnArgs& a) {
  const int ks = tn_ksplit_most(a, tn_tiles(tn_edge(dtype, a), a));
  return ks > 1 ? (size_t)ks * tn_blocks(a) * 4096 : 0;
}

template <typename T, int TM, int TN, int WGM, int WGN, int WGK, int ST, bool DIRECT = true>
static hipError_t tn_one(const TnArgs& a, hipStream_t s) {
  using Cfg = TnCfg<T, TM, TN, WGM, WGN, WGK, ST>;
  auto kern = gemm_tn_kernel<T, TM, TN, WGM, WGN, WGK, ST, DIRECT>;
  static LdsOnce lds_once;
  if (hipError_t ae = allow_dynamic_lds(lds_once, kern, Cfg::kBytes); ae != hipSuccess) return ae;
  hipLaunchKernelGGL(kern, dim3(a.tiles * a.ksplit), dim3(Cfg::kThreads), Cfg::kBytes, s, a);
  if (hipError_t e = hipGetLastError(); e != hipSuccess || a.ksplit <= 1) return e;
  hipLaunchKernelGGL(tn_reduce_kernel, dim3(a.blocks), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gemm_tn(int dtype, const TnArgs& args, hipStream_t s) {
  TnArgs a = args;
  // operands of the caller's that do not start on 16 bytes: through registers, with 64-wide tiles for all sizes
  uintptr_t starts = 0;
  for (int i = 0; i < a.n; ++i) starts |= reinterpret_cast<uintptr_t>(a.p[i].At) | reinterpret_cast<uintptr_t>(a.p[i].Bt);
  const bool direct = starts % 16 == 0;
  const int edge = direct ? tn_edge(dtype, a) : 64;
  a.ksplit = tn_ksplit(dtype, a);                               // (the split that tn_part_bytes has counted with)
  a.tiles = a.blocks = 0;
  for (int i = 0; i < a.n; ++i) {
    a.p[i].first_tile = a.tiles;
    a.p[i].first_block = a.blocks;
    a.tiles += ((a.p[i].M + edge - 1) / edge) * ((a.p[i].cols + edge - 1) / edge);
    a.blocks += (pad32(a.p[i].M) / 32) * ((a.p[i].cols + 31) / 32);
  }
  if (!direct) return dtype == 0 ? tn_one<float, 64, 64, 1, 1, 8, 4, false>(a, s) : tn_one<bf16, 64, 64, 1, 1, 4, 4, false>(a, s);
  if (dtype == 0) return tn_one<float, 64, 64, 1, 1, 8, 4>(a, s);
  if (edge == 128) return tn_one<bf16, 128, 128, 1, 2, 4, 4>(a, s);
  return tn_one<bf16, 64, 64, 1, 1, 4, 4>(a, s);
}

}  // namespace ta
