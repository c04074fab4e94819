// Backward pass of the fused prefill attention (the paper trains the layer, Section
// "Experiments", and its timing tables carry a backward column; the gradient itself is the
// derivative of Definition "Latent RoPE for Tucker Attention" followed by softmax attention over
// the shared latent keys and values).  Flash-style: no N x N matrix is kept; probabilities are
// recomputed from the saved log-sum-exp.
//
// With P_i = softmax(S_i), S_i = Q_i K^T (Q_i the rotated, scaled per-head query; K the rotated
// latent keys), O_i = P_i V, and upstream dO_i = dZ G~_i:
//     delta_i = rowsum(dO_i * O_i)          dP_i = dO_i V^T        dS_i = P_i * (dP_i - delta_i)
//     dQ_i = dS_i K                         dK = sum_i dS_i^T Q_i  dV = sum_i P_i^T dO_i
// Two kernels, neither with atomics:
//   bwd_dq   one wave = 32 queries of one head, walks the key tiles like the forward kernel:
//            builds Q_i and dO_i in a prologue from the latent query and dZ (and leaves copies of
//            both for the second kernel), accumulates dQ_i, removes the rotation and stores it.
//   bwd_dkv  a pair of waves = 32 keys kept in registers as operands, walks (head, query block)
//            pairs staged in LDS; one wave of the pair accumulates dV^T, the other dK^T; heads are
//            split into groups over workgroups, each writing a partial sum that kv_reduce adds up
//            (and un-rotates).
// Products are computed in the orientation that keeps the contraction index inside a lane (see
// the fragment model in common.h): bwd_dq keeps queries as MFMA columns, bwd_dkv keeps keys.
#include <type_traits>

#include "common.h"
#include "params.h"

namespace ta {

namespace {

constexpr float kLn2 = 0.6931471805599453f;

// acc[cb] = (32 rows c of core block cb) x (this wave's 32 tokens): sum_b G[c][b] xrow[token][b].
// G: one head's fragment-major blocks [cb][bb]; xrow: this lane's token row + 16*h.
template <typename T, int CB>
__device__ __forceinline__ void core_product(f32x16 (&acc)[CB], const T* G, const T* xrow, int nbb, int lane) {
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[cb][e] = 0.f;
  for (int bb = 0; bb < nbb; ++bb) {
    const Frag<T> x = load_frag<T>(xrow + bb * 32);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const Frag<T> g = load_frag_major<T>(G + (long)(cb * nbb + bb) * kFragBlockElems, lane);
      mma32(acc[cb], g, x);
    }
  }
}

// rotate (sign = +1) or un-rotate (sign = -1) the channel pairs of accumulator blocks whose column
// (lane) sits at table position pos
template <int CB>
__device__ __forceinline__ void rotate_blocks(f32x16 (&a)[CB], const float4* rope, int rope_ld, int pos, int h,
                                              float sign) {
  const f32x4* tab = reinterpret_cast<const f32x4*>(rope) + (long)h * rope_ld + pos;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    f32x4 cs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) cs[q] = tab[(long)(cb * 8 + 2 * q) * rope_ld];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        const float x0 = a[cb][4 * q + e], x1 = a[cb][4 * q + e + 1];
        const float c = cs[q][e], s = sign * cs[q][e + 1];
        a[cb][4 * q + e] = x0 * c - x1 * s;
        a[cb][4 * q + e + 1] = x0 * s + x1 * c;
      }
  }
}

// element e of a fragment (same index as the accumulator register it came from)
__device__ __forceinline__ float frag_elem(const Frag<float>& f, int e) { return f.v[e / 4][e % 4]; }
__device__ __forceinline__ float frag_elem(const Frag<bf16>& f, int e) { return (float)f.v[e / 8][e % 8]; }

}  // namespace

// ---- dQ ----------------------------------------------------------------------------------------------
template <typename T, int D, int BC> struct DqLds {
  static constexpr int kRow = D + 16 / sizeof(T);               // K / V tile rows
  static constexpr int kTRow = BC + 16 / sizeof(T);             // K^T tile rows
  static constexpr int kKElems = BC * kRow;
  static constexpr int kTElems = D * kTRow;
  static constexpr int kStage = 2 * kKElems + kTElems;
  static constexpr size_t kBytes = 2ul * kStage * sizeof(T);
};

// Workgroup = HW heads x QW blocks of 32 queries (two: waves w and w+4 share a SIMD; one for calls with few
// workgroups), whose keys KS waves share (those with few workgroups: each takes every KS-th tile, the sums meet in LDS); key
// tiles of BC keys, one for each part, are staged once per workgroup and walked in 32-key halves, so that only one half's
// scores live in registers at a time.
template <typename T, int D, int BC, int QW, int HW, int KS>
__global__ __launch_bounds__(64 * QW * HW * KS) void bwd_dq_kernel(BwdArgs p) {
  constexpr int CB = D / 32, NB = BC / 32, TQ = 32 * QW, NT = 64 * HW * QW * KS;
  constexpr int CE = 16 / sizeof(T);
  using L = DqLds<T, D, BC>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  T* smem = reinterpret_cast<T*>(smem_raw);

  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int ks = wave / (QW * HW), wq = wave % (QW * HW);       // part of the keys; wave within the part
  const int h = lane / 32, lr = lane % 32;
  const int n_qtiles = p.Npad / TQ;
  const int qt = n_qtiles - 1 - blockIdx.y;                     // heavy (late causal) tiles first
  const int n_hg = (p.nH + HW - 1) / HW;
  // consecutive workgroups go to the 8 XCDs in turn: re-index the (sequence, head group) items of a row so
  // that one XCD, with its own L2, gets neighbouring items and sees the K/V of as few sequences as possible
  int item = blockIdx.x;
  if (gridDim.x % 8 == 0) item = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int b = item / n_hg;
  const int head_raw = (item % n_hg) * HW + wq % HW;
  const bool head_ok = head_raw < p.nH;
  const int head = head_ok ? head_raw : p.nH - 1;
  const int t0 = qt * TQ;
  const int tw = t0 + (wq / HW) * 32;                           // first query of this wave
  const int m = tw + lr;                                        // this lane's query, < Npad
  const long tok_base = (long)b * p.Npad;
  const long TP = (long)p.Bsz * p.Npad;

  // staging of the key tiles t KS .. t KS + KS - 1: K rows, V rows, K^T columns
  const int kv_end = p.causal ? min(p.N, t0 + TQ) : p.N;
  const int last = (kv_end + BC - 1) / BC - 1;                  // last key tile
  constexpr int RCH = BC * D / CE;                              // chunks of a row tile (and of the transposed one)
  constexpr int PT = (KS * RCH + NT - 1) / NT;
  constexpr bool FULL = KS * RCH % NT == 0;
  constexpr int RCPR = D / CE, TCPR = BC / CE;
  const T* Kg = static_cast<const T*>(p.Kr) + tok_base * D;
  const T* Vg = static_cast<const T*>(p.Vr) + tok_base * D;
  const T* Tg = static_cast<const T*>(p.Krt) + (long)b * D * p.Npad;
  u32x4 kreg[PT], vreg[PT], treg[PT];
  auto g_load = [&](int t) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int at = threadIdx.x + i * NT, ci = at % RCH;
      if (!FULL && at >= KS * RCH) break;
      const int tile = min(t * KS + at / RCH, last);
      const int row = ci / RCPR, cc = ci % RCPR;
      kreg[i] = *reinterpret_cast<const u32x4*>(Kg + (long)(tile * BC + row) * D + cc * CE);
      vreg[i] = *reinterpret_cast<const u32x4*>(Vg + (long)(tile * BC + row) * D + cc * CE);
      const int trow = ci / TCPR, tc = ci % TCPR;
      treg[i] = *reinterpret_cast<const u32x4*>(Tg + (long)trow * p.Npad + tile * BC + tc * CE);
    }
  };
  auto s_store = [&](int stage) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int at = threadIdx.x + i * NT, ci = at % RCH;
      if (!FULL && at >= KS * RCH) break;
      T* rows = smem + (long)(stage * KS + at / RCH) * L::kStage;
      T* vs = rows + L::kKElems;
      T* ts = vs + L::kKElems;
      const int row = ci / RCPR, cc = ci % RCPR;
      *reinterpret_cast<u32x4*>(rows + row * L::kRow + cc * CE) = kreg[i];
      *reinterpret_cast<u32x4*>(vs + row * L::kRow + cc * CE) = vreg[i];
      const int trow = ci / TCPR, tc = ci % TCPR;
      *reinterpret_cast<u32x4*>(ts + trow * L::kTRow + tc * CE) = treg[i];
    }
  };

  g_load(0);

  // ---- prologue: Q_i^T and dO_i^T of this wave's 32 tokens, delta, copies for the dK/dV kernel ----
  Frag<T> qf[CB], dof[CB];
  f32x16 negl, negd;                                            // -log-sum-exp and -delta of this lane's query
  {
    f32x16 qa[CB], da[CB];
    const T* Gt = static_cast<const T*>(p.Gt) + (long)head * D * p.R2;
    const T* Ql = static_cast<const T*>(p.Qlat) + (tok_base + m) * p.R2 + 16 * h;
    core_product<T, CB>(qa, Gt, Ql, p.R2 / 32, lane);
    if (p.rope != nullptr) rotate_blocks<CB>(qa, p.rope, p.rope_ld, p.pos0 + min(m, p.N - 1), h, 1.f);
    const T* Gtt = static_cast<const T*>(p.Gtil_t) + (long)head * D * p.RT2;
    const T* dZ = static_cast<const T*>(p.dZ) + (tok_base + m) * p.RT2 + 16 * h;
    core_product<T, CB>(da, Gtt, dZ, p.RT2 / 32, lane);
    const T* Orow = static_cast<const T*>(p.O) + ((tok_base + m) * p.nH + head) * D + 16 * h;
    float dsum = 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      qf[cb] = to_frag<T>(qa[cb]);
      dof[cb] = to_frag<T>(da[cb]);
      const Frag<T> of = load_frag<T>(Orow + cb * 32);
#pragma unroll
      for (int e = 0; e < 16; ++e) dsum += frag_elem(dof[cb], e) * frag_elem(of, e);   // the rounded dO that forms dP
    }
    const float delta = halves_sum(dsum);
    const float nlse = p.lse[((long)b * p.nH + head) * p.Npad + m];   // -inf for padding tokens
#pragma unroll
    for (int e = 0; e < 16; ++e) { negl[e] = nlse; negd[e] = -delta; }
    if (head_ok && ks == 0) {
      if (h == 0) p.delta[((long)b * p.nH + head) * p.Npad + m] = -delta;
      T* Qr = static_cast<T*>(p.Qr) + ((tok_base + m) * p.nH + head) * D + 16 * h;
      T* dOr = static_cast<T*>(p.dO) + ((tok_base + m) * p.nH + head) * D + 16 * h;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        store_frag<T>(Qr + cb * 32, qf[cb]);
        store_frag<T>(dOr + cb * 32, dof[cb]);
      }
    }
  }

  // ---- key tiles ------------------------------------------------------------------------------------
  f32x16 dq[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[cb][e] = 0.f;
  const int n_int = last / KS + 1;                              // intervals: tiles of part 0
  const int lim = p.causal ? min(m, p.N - 1) : p.N - 1;         // last key visible to this lane's query
  s_store(0);
  __syncthreads();
  for (int t = 0; t < n_int; ++t) {
    g_load(min(t + 1, n_int - 1));
    const T* st = smem + (long)((t & 1) * KS + ks) * L::kStage;
    const T* kbase = st + lr * L::kRow + 16 * h;
    const T* vbase = kbase + L::kKElems;
    const T* tbase = st + 2 * L::kKElems + lr * L::kTRow + 16 * h;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int n0 = (t * KS + ks) * BC + nb * 32;
      if (p.causal && n0 > tw + 31) continue;                   // every key of the half follows every query
      if (KS > 1 && n0 >= p.N) continue;                        // a tile past the last one
      // scores start from -log-sum-exp and dP from -delta, so the products form S - lse and dP - delta
      f32x16 s, dp;
      mma32_from(s, negl, load_frag<T>(kbase + nb * 32 * L::kRow), qf[0]);
#pragma unroll
      for (int cb = 1; cb < CB; ++cb) mma32(s, load_frag<T>(kbase + nb * 32 * L::kRow + cb * 32), qf[cb]);
      mma32_from(dp, negd, load_frag<T>(vbase + nb * 32 * L::kRow), dof[0]);
#pragma unroll
      for (int cb = 1; cb < CB; ++cb) mma32(dp, load_frag<T>(vbase + nb * 32 * L::kRow + cb * 32), dof[cb]);
      if (n0 + 31 >= p.N || (p.causal && n0 + 31 > tw)) {       // a key past the sequence or after a query
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (n0 + 8 * (e / 4) + 4 * h + (e % 4) > lim) s[e] = -INFINITY;
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = fast_exp2(s[e]) * dp[e];
      const Frag<T> dsf = to_frag<T>(s);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) mma32(dq[cb], load_frag<T>(tbase + cb * 32 * L::kTRow + nb * 32), dsf);
    }
    s_store((t + 1) & 1);
    __syncthreads();
  }

  // ---- the other parts' sums, in their order ------------------------------------------------------------
  if constexpr (KS > 1) {
    float* sums = reinterpret_cast<float*>(smem_raw);           // [KS - 1][QW * HW][16 CB][64]
    auto at = [&](int part) { return sums + (long)((part - 1) * QW * HW + wq) * (16 * CB * 64) + lane; };
    if (ks > 0) {                                               // (behind the loop's last barrier: the tiles are done with)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int e = 0; e < 16; ++e) at(ks)[(16 * cb + e) * 64] = dq[cb][e];
    }
    __syncthreads();
    if (ks > 0) return;
#pragma unroll
    for (int part = 1; part < KS; ++part)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int e = 0; e < 16; ++e) dq[cb][e] += at(part)[(16 * cb + e) * 64];
  }

  // ---- epilogue: remove the rotation, store -----------------------------------------------------------
  if (p.rope != nullptr) rotate_blocks<CB>(dq, p.rope, p.rope_ld, p.pos0 + min(m, p.N - 1), h, -1.f);
  if (head_ok) {
    T* dQ = static_cast<T*>(p.dQ) + ((tok_base + m) * p.nH + head) * D + 16 * h;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) store_frag<T>(dQ + cb * 32, to_frag<T>(dq[cb]));
  }
}

// ---- dK, dV ------------------------------------------------------------------------------------------
template <typename T, int D, int TQ, int KB> struct DkvLds {
  static constexpr int kStages = 3;
  static constexpr int kRow = D;                                // Q / dO rows, unpadded, chunks swizzled
  static constexpr int kRElems = TQ * kRow;
  static constexpr int kStageElems = 2 * kRElems;
  // behind the rows: -log-sum-exp and -delta of the queries, 64 places each (a direct-to-LDS load fills 64)
  static constexpr size_t kStageBytes = kStageElems * sizeof(T) + 2ul * 64 * sizeof(float);
  static_assert(TQ <= 64, "one load per vector");
  // probabilities handed from the dV^T waves to the dK^T waves: [2][KB key blocks][TQ/32] fragment blocks
  static constexpr size_t kPBytes = 2ul * KB * (TQ / 32) * kFragBlockElems * sizeof(T);
  static constexpr size_t kBytes = kStages * kStageBytes + kPBytes;
};

// Workgroup = 2 KB waves over 32 KB keys (KB = 4, or 2 for calls with few workgroups): waves w and w+KB own the same
// 32 keys (KB = 4: on one SIMD).  Wave w holds
// the keys in registers as MFMA column operands, forms the probabilities P of a (head, query block)
// pair, leaves them in LDS and accumulates dV^T += dO^T P; wave w+KB holds the values, forms dP one
// interval later, takes P from LDS, and accumulates dK^T += Q^T (P (dP - delta)).  Two resident
// waves per SIMD let one wave's exponentials overlap the other's matrix products.  The Q and dO rows
// of a pair are staged once, row-major (straight from global memory into LDS, three stages, two pairs
// ahead); the transposed operands Q^T and dO^T are read from the same
// tiles with transposing LDS loads, so their rows (the channels) come out in the stored channel
// order of Q and dO (acc order within 32-blocks), which kv_reduce undoes.
template <typename T, int D, int TQ, int KB>
__global__ __launch_bounds__(128 * KB) void bwd_dkv_kernel(BwdArgs p) {
  constexpr int CB = D / 32, QBN = TQ / 32, KT = 32 * KB, NT = 128 * KB;
  constexpr int CE = 16 / sizeof(T);
  using L = DkvLds<T, D, TQ, KB>;
  constexpr int NS = L::kStages;
  static_assert(swz_x<D / CE>(32) == 0, "blocks of 32 rows are swizzled alike");
  static_assert(sizeof(T) == 2 || QBN == 1, "one block of 32 queries in fp32");
  static_assert(L::kStageBytes % 16 == 0, "stages stay 16-byte aligned");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  T* pbuf = reinterpret_cast<T*>(smem_raw + NS * L::kStageBytes);

  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int h = lane / 32, lr = lane % 32;
  const bool k_role = wave >= KB;                               // dK^T wave (else dV^T wave)
  const int kb = wave % KB;                                     // key block of this wave
  const int n_parts = p.n_hg * p.qsplit;                        // partial sums: head groups, their queries in qsplit parts
  const int b = blockIdx.x / n_parts, part = blockIdx.x % n_parts, hg = part / p.qsplit;
  const int key0 = blockIdx.y * KT + 32 * kb;                   // first key of this wave
  const int nk = key0 + lr;                                     // this lane's key
  const bool key_ok = nk < p.Npad;
  const long tok_base = (long)b * p.Npad;
  const long TP = (long)p.Bsz * p.Npad;

  // column operand of this wave's keys for the whole kernel: the rotated keys in a dV^T wave (it
  // forms the scores), the values in a dK^T wave (it forms dP)
  Frag<T> kop[CB];
  {
    const long row = tok_base + (key_ok ? nk : 0);
    const T* src = static_cast<const T*>(k_role ? p.Vr : p.Kr) + row * D + 16 * h;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) kop[cb] = key_ok ? load_frag<T>(src + cb * 32) : zero_frag<T>();
  }
  f32x16 acc[CB];                                               // dV^T or dK^T of this wave's keys
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[cb][e] = 0.f;

  // (head, query block) pairs of this workgroup
  const int head0 = hg * p.hpg;
  const int n_heads = min(p.hpg, p.nH - head0);
  const int qb_first = p.causal ? (blockIdx.y * KT) / TQ : 0;
  const int n_qb = p.Npad / TQ - qb_first;                      // >= 1: the grid covers Npad
  const int it0 = n_heads * n_qb * (part % p.qsplit) / p.qsplit;        // the pairs of this part
  const int n_it = n_heads * n_qb * (part % p.qsplit + 1) / p.qsplit;
  // Query blocks are walked from the last one down: the workgroups of one (sequence, head group),
  // which run on the same XCD at the same time, then all read the same block at the same moment
  // (with causal masking their ranges start at different blocks but all end at the last).
  auto q_of = [&](int it) { return (qb_first + n_qb - 1 - it % n_qb) * TQ; };

  // The Q and dO rows of a pair and its two per-query vectors go from global memory straight into LDS (see dma_piece in
  // common.h), into the stage that the lagging dK^T waves have just left, one interval before the dV^T waves need
  // them.  Nothing else of the loop is in flight in vector memory, and the interval waits for it only at its end: the
  // compiler's own wait in front of a transposing read (every direct-to-LDS load has landed) would come in the
  // middle, hence load_frags_tr_swz.  Two sequences of 4096 tokens, 32 heads, D = 128:
  // 763 -> 716 us, and with the query blocks of a pair in step (below) 650 us; eight of 1024 tokens, 12 heads, D = 64: 66.1 ->
  // 62.1 -> 58.5 us.
  constexpr int CPR = D / CE;                                    // chunks per row
  constexpr int PIECES = TQ * CPR / 64;                          // 1 KB pieces per tensor
  constexpr int NW = NT / 64;
  auto issue = [&](int it, int stage) {
    const int head = head0 + it / n_qb, q0 = q_of(it);
    const T* Qg = static_cast<const T*>(p.Qr) + ((tok_base + q0) * p.nH + head) * D;
    const T* Og = static_cast<const T*>(p.dO) + ((tok_base + q0) * p.nH + head) * D;
    T* qs = reinterpret_cast<T*>(smem_raw + (size_t)stage * L::kStageBytes);
    T* os = qs + L::kRElems;
    const long rs = (long)p.nH * D;
#pragma unroll
    for (int i = 0; i < (PIECES + NW - 1) / NW; ++i) {
      const int q = i * NW + wave;
      if (q < PIECES) {
        dma_piece<T, CPR>(qs, q, lane, [&](int row) { return Qg + row * rs; });
        dma_piece<T, CPR>(os, q, lane, [&](int row) { return Og + row * rs; });
      }
    }
    if (wave < 2) {                                             // (lanes past TQ fetch the first ones again)
      const float* src = (wave == 0 ? p.lse : p.delta) + ((long)b * p.nH + head) * p.Npad + q0 + lane % TQ;
      float* st = reinterpret_cast<float*>(os + L::kRElems) + 64 * wave;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)st, 4, 0, 0);
    }
  };
  auto meet = [&]() {                                           // loads landed, LDS reads and writes done, all waves here
    wait_vm<0>();
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  if (it0 < n_it) issue(it0, it0 % NS);
  meet();
  if (it0 + 1 < n_it) issue(it0 + 1, (it0 + 1) % NS);
  // one interval: the dV^T waves work on pair t (stage t % 3), the dK^T waves on pair t-1; behind the meeting pair t+2
  // is fetched into stage (t+2) % 3, which held pair t-1.
  for (int t = it0; t < n_it + 1; ++t) {
    const int it = k_role ? t - 1 : t;                          // pair this wave works on in this interval
    if (it >= it0 && it < n_it) {
      const unsigned char* sb = smem_raw + (size_t)(it % NS) * L::kStageBytes;
      const T* qs = reinterpret_cast<const T*>(sb);
      const T* os = qs + L::kRElems;
      const float* stat = reinterpret_cast<const float*>(os + L::kRElems);
      const int q0 = q_of(it);
      // all 32 keys of the wave lie after all queries of the pair: nothing to do
      if (!p.causal || key0 <= q0 + TQ - 1) {
        constexpr int FC = 16 / CE;                             // chunks per fragment half
        constexpr int TF = CB < 2 ? 1 : 2;
        // A first query block that lies before all 32 keys has probabilities of zero, but a value that is not finite in
        // its rows (an overflown dY) would not vanish when multiplied by them: the rows of the second block stand in.
        // (Costs 3 us of 578 at 2 x 4096 tokens; a second copy of this code for one block cost 50.)
        const int row0 = QBN > 1 && p.causal && key0 > q0 + 31 ? 32 : 0;
        auto block_row = [&](int qb) { return qb == 0 ? row0 : qb * 32; };
        // The query blocks of the pair go through every phase together: their products are independent chains, and the
        // first transposed operands are read while those of the scores are still in the matrix pipe.
        f32x16 a[QBN];
        Frag<T> rf[QBN][CB];
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
          // rows of a block start from -log-sum-exp (scores) or -delta (dP)
          const float* st4 = stat + (k_role ? 64 : 0) + block_row(qb) + 4 * h;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v4 = *reinterpret_cast<const f32x4*>(st4 + 8 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) a[qb][4 * q + e] = v4[e];
          }
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int qb = 0; qb < QBN; ++qb)
            rf[qb][cb] = load_frag_swz<T>((k_role ? os : qs) + (block_row(qb) + lr) * L::kRow, cb * 2 * FC + h * FC, swz_x<CPR>(lr));
        if constexpr (sizeof(T) == 2) __builtin_amdgcn_sched_barrier(0);   // all reads on their way before the first product
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int qb = 0; qb < QBN; ++qb) mma32(a[qb], rf[qb][cb], kop[cb]);
        if constexpr (sizeof(T) == 2) __builtin_amdgcn_sched_barrier(0);
        const T* tile = k_role ? qs : os;                       // dK^T += Q^T dS,  dV^T += dO^T P
        Frag<T> tf[QBN][TF];
        if constexpr (sizeof(T) == 2) {
#pragma unroll
          for (int qb = 0; qb < QBN; ++qb) load_frags_tr_swz<CPR>(tf[qb], tile + block_row(qb) * L::kRow, 0, 0, lane);
        }
        Frag<T> bf[QBN];                                        // P (dV^T wave) or dS (dK^T wave), k = queries
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
          const int qfirst = q0 + 32 * qb;
          T* pblk = pbuf + (long)(((it & 1) * KB + kb) * QBN + qb) * kFragBlockElems;
          if (!k_role) {
            if (key0 + 31 >= p.N || (p.causal && key0 + 31 > qfirst)) {   // a key past the sequence or after a query
              // register e holds query qfirst + 4 h + 8 (e / 4) + e % 4
              const int first = nk >= p.N ? 64 : (p.causal ? nk - qfirst - 4 * h : 0);
#pragma unroll
              for (int e = 0; e < 16; ++e) a[qb][e] = 8 * (e / 4) + (e % 4) < first ? -INFINITY : a[qb][e];
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) a[qb][e] = fast_exp2(a[qb][e]);
            bf[qb] = to_frag<T>(a[qb]);
            store_frag_major<T>(pblk, lane, bf[qb]);
          } else {
            const Frag<T> pf = load_frag_major<T>(pblk, lane);
#pragma unroll
            for (int e = 0; e < 16; ++e) a[qb][e] *= frag_elem(pf, e);
            bf[qb] = to_frag<T>(a[qb]);
          }
        }
        if constexpr (sizeof(T) == 4) load_frags_tr_swz<CPR>(tf[0], tile, 0, 0, lane);   // (no registers for it earlier)
#pragma unroll
        for (int cb = 0; cb < CB; cb += TF) {
#pragma unroll
          for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
            for (int n = 0; n < TF; ++n) mma32(acc[cb + n], tf[qb][n], bf[qb]);
          if (cb + TF < CB)
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb) load_frags_tr_swz<CPR>(tf[qb], tile + block_row(qb) * L::kRow, 0, (cb + TF) * 32, lane);
        }
      }
    }
    meet();
    if (t + 2 < n_it) issue(t + 2, (t + 2) % NS);               // nothing is left in flight at the end
  }

  // rows of the accumulators are stored channel positions: position 16h'+4q'+r of a 32-block
  if (key_ok) {
    float* dst = (k_role ? p.dKp : p.dVp) + ((long)part * TP + tok_base + nk) * D + 4 * h;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        store4(dst + cb * 32 + 8 * q, acc[cb][4 * q], acc[cb][4 * q + 1], acc[cb][4 * q + 2], acc[cb][4 * q + 3]);
  }
}

// ---- sum of the head-group partials, rotation removed from the key part -----------------------------
// The scores carry a factor log2(e) (the per-head query is pre-scaled so that the softmax runs on
// exp2), so the key gradient formed from those queries is multiplied by ln 2 here.
// SP threads share the partials of a channel quad (every SP-th each, four loads of either kind in flight): with few tokens one
// thread's chain of loads is what the launch takes (D = 64, 2 x 509 tokens, 48 partials 7.1 us, 17.3 with one thread, 8.9 with
// eight loads of it in flight; 32 partials of 150 tokens, D = 128: 12.1 -> 64 of them 6.9).  With many tokens the launch reads at 5.8
// TB/s as it is.
template <typename T, int SP>
__global__ __launch_bounds__(256) void kv_reduce_kernel(KvReduceArgs a) {
  constexpr int QT = 256 / SP;                                  // quads of a workgroup
  const long TP = (long)a.Bsz * a.Npad;
  const int quads = a.D / 4;
  const long idx = (long)blockIdx.x * QT + threadIdx.x % QT;
  const bool live = idx < TP * quads;
  if (SP == 1 && !live) return;
  const long tp = live ? idx / quads : 0;
  const int k = (int)(idx % quads);
  const int n = (int)(tp % a.Npad);
  f32x4 sk = {0.f, 0.f, 0.f, 0.f}, sv = {0.f, 0.f, 0.f, 0.f};
  // the partials hold channel quad k at its stored (acc-order) position inside its 32-block
  const int c32 = (4 * k) % 32;
  const int spos = (4 * k) / 32 * 32 + 16 * ((c32 / 4) % 2) + 4 * (c32 / 8);
  if constexpr (SP == 1) {
    for (int g = 0; g < a.n_hg; ++g) {
      const long off = ((long)g * TP + tp) * a.D + spos;
      const f32x4 x = *reinterpret_cast<const f32x4*>(a.dKp + off);
      const f32x4 y = *reinterpret_cast<const f32x4*>(a.dVp + off);
#pragma unroll
      for (int e = 0; e < 4; ++e) { sk[e] += x[e]; sv[e] += y[e]; }
    }
  } else {
    constexpr int RD = 4;
    const int part = threadIdx.x / QT;
    for (int g0 = part; g0 < a.n_hg; g0 += RD * SP) {
      f32x4 x[RD], y[RD];
#pragma unroll
      for (int r = 0; r < RD; ++r) {
        const long off = ((long)min(g0 + r * SP, a.n_hg - 1) * TP + tp) * a.D + spos;
        x[r] = *reinterpret_cast<const f32x4*>(a.dKp + off);
        y[r] = *reinterpret_cast<const f32x4*>(a.dVp + off);
      }
#pragma unroll
      for (int r = 0; r < RD; ++r)
        if (g0 + r * SP < a.n_hg)
#pragma unroll
          for (int e = 0; e < 4; ++e) { sk[e] += x[r][e]; sv[e] += y[r][e]; }
    }
    __shared__ f32x4 sums[SP - 1][2][QT];
    if (part > 0) {
      sums[part - 1][0][threadIdx.x % QT] = sk;
      sums[part - 1][1][threadIdx.x % QT] = sv;
    }
    __syncthreads();
    if (part > 0 || !live) return;
#pragma unroll
    for (int q = 0; q < SP - 1; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sk[e] += sums[q][0][threadIdx.x][e];
        sv[e] += sums[q][1][threadIdx.x][e];
      }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) sk[e] *= kLn2;
  if (a.rope != nullptr && n < a.N) {
    const f32x4 cs = reinterpret_cast<const f32x4*>(a.rope)[(long)k * a.rope_ld + a.pos0 + n];
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      const float x0 = sk[e], x1 = sk[e + 1];
      sk[e] = x0 * cs[e] + x1 * cs[e + 1];
      sk[e + 1] = -x0 * cs[e + 1] + x1 * cs[e];
    }
  }
  T* row = static_cast<T*>(a.dLat) + tp * a.ld;
  if (a.shared_kv) {
    store4(row + a.colK + 4 * k, sk[0] + sv[0], sk[1] + sv[1], sk[2] + sv[2], sk[3] + sv[3]);
  } else {
    store4(row + a.colK + 4 * k, sk[0], sk[1], sk[2], sk[3]);
    store4(row + a.colV + 4 * k, sv[0], sv[1], sv[2], sv[3]);
  }
}

// ---- launchers ---------------------------------------------------------------------------------------
template <typename T, int D, int BC, int QW, int HW, int KS>
static hipError_t dq_launch(const BwdArgs& a, hipStream_t s) {
  dim3 grid(((a.nH + HW - 1) / HW) * a.Bsz, a.Npad / (32 * QW));
  const size_t smem = KS * DqLds<T, D, BC>::kBytes;
  auto kern = bwd_dq_kernel<T, D, BC, QW, HW, KS>;
  static LdsOnce lds_once;
  if (hipError_t ae = allow_dynamic_lds(lds_once, kern, smem); ae != hipSuccess) return ae;
  hipLaunchKernelGGL(kern, grid, dim3(64 * QW * HW * KS), smem, s, a);
  return hipGetLastError();
}
// Fewer workgroups than compute units: one block of queries each, so that a wave has a SIMD to itself, and its keys dealt
// to two waves, or four.  One block of queries and one, two, four waves (us): fp32, D = 64, 12 heads, 2 x 509 tokens 70.1,
// 44.5; 5 x 100 28.0, 21.4; bf16, D = 64, 1024 tokens 29.6, 22.2; D = 128 (tiles of 32 keys when they are shared), 32 heads, 450
// tokens 31.1, 25.5, 900 tokens (464 workgroups) 46.6, 48.7; D = 32, 4 heads, 512 tokens 12.1, 9.1, 7.8.
template <typename T, int D, int BC> static constexpr int shared_tile() {   // keys of a tile that is shared
  return 2 * DqLds<T, D, BC>::kBytes <= 160 * 1024 ? BC : 32;
}
template <typename T, int D, int BC> static constexpr bool by_two() {
  return 2 * DqLds<T, D, shared_tile<T, D, BC>()>::kBytes <= 160 * 1024;
}
// waves that share a query block's keys; 0: two query blocks a workgroup
template <typename T, int D, int BC> static int dq_key_parts(const BwdArgs& a) {
  const long blocks = (long)a.Bsz * (a.Npad / 32), tiles = (a.N + BC - 1) / BC;
  if ((a.nH + 3) / 4 * (blocks / 2) >= kComputeUnits) return 0;
  if (D == 32 && tiles >= 4 && a.nH * blocks <= kComputeUnits * 3 / 2) return 4;
  return by_two<T, D, BC>() && tiles >= 2 && (a.nH + 1) / 2 * blocks <= kComputeUnits ? 2 : 1;
}
template <typename T, int D, int BC>
static hipError_t dq_one(const BwdArgs& a, hipStream_t s) {
  switch (dq_key_parts<T, D, BC>(a)) {
    case 0: return dq_launch<T, D, BC, 2, 4, 1>(a, s);
    case 4:
      if constexpr (D == 32) return dq_launch<T, D, BC, 1, 1, 4>(a, s);
      break;
    case 2:
      if constexpr (by_two<T, D, BC>()) return dq_launch<T, D, shared_tile<T, D, BC>(), 1, 2, 2>(a, s);
      break;
    case 1: return dq_launch<T, D, BC, 1, 4, 1>(a, s);
  }
  return hipErrorInvalidValue;
}

int bwd_dq_key_parts(int dtype, const BwdArgs& a) {
  if (dtype == 0) return a.D == 32 ? dq_key_parts<float, 32, 32>(a) : a.D == 64 ? dq_key_parts<float, 64, 32>(a) : dq_key_parts<float, 128, 32>(a);
  return a.D == 32 ? dq_key_parts<bf16, 32, 64>(a) : a.D == 64 ? dq_key_parts<bf16, 64, 64>(a) : dq_key_parts<bf16, 128, 64>(a);
}

hipError_t launch_bwd_dq(int dtype, const BwdArgs& a, hipStream_t s) {
  if (dtype == 0) {
    switch (a.D) {
      case 32: return dq_one<float, 32, 32>(a, s);
      case 64: return dq_one<float, 64, 32>(a, s);
      case 128: return dq_one<float, 128, 32>(a, s);
    }
  } else {
    switch (a.D) {
      case 32: return dq_one<bf16, 32, 64>(a, s);
      case 64: return dq_one<bf16, 64, 64>(a, s);
      case 128: return dq_one<bf16, 128, 64>(a, s);
    }
  }
  return hipErrorInvalidValue;
}

// Few workgroups: 64 keys each instead of 128 (fp32, D = 64, 12 heads, 2 x 509 tokens: 81 -> 54 us).
template <typename T, int D, int TQ, int KB>
static hipError_t dkv_launch(const BwdArgs& a, hipStream_t s) {
  using L = DkvLds<T, D, TQ, KB>;
  static_assert(L::kBytes <= 160 * 1024, "fits the LDS of a compute unit");
  dim3 grid(a.n_hg * a.qsplit * a.Bsz, (a.Npad + 32 * KB - 1) / (32 * KB));
  auto kern = bwd_dkv_kernel<T, D, TQ, KB>;
  static LdsOnce lds_once;
  if (hipError_t ae = allow_dynamic_lds(lds_once, kern, L::kBytes); ae != hipSuccess) return ae;
  hipLaunchKernelGGL(kern, grid, dim3(128 * KB), L::kBytes, s, a);
  return hipGetLastError();
}
template <typename T, int D, int TQ>
static hipError_t dkv_one(const BwdArgs& a, hipStream_t s) {
  const long wgs = (long)a.n_hg * a.qsplit * a.Bsz * ((a.Npad + 127) / 128);
  return wgs < kComputeUnits ? dkv_launch<T, D, TQ, 2>(a, s) : dkv_launch<T, D, TQ, 4>(a, s);
}

hipError_t launch_bwd_dkv(int dtype, const BwdArgs& a, hipStream_t s) {
  if (dtype == 0) {
    switch (a.D) {
      case 32: return dkv_one<float, 32, 32>(a, s);
      case 64: return dkv_one<float, 64, 32>(a, s);
      case 128: return dkv_one<float, 128, 32>(a, s);
    }
  } else {
    switch (a.D) {
      case 32: return dkv_one<bf16, 32, 64>(a, s);
      case 64: return dkv_one<bf16, 64, 64>(a, s);
      case 128: return dkv_one<bf16, 128, 64>(a, s);
    }
  }
  return hipErrorInvalidValue;
}

template <typename T> static void kv_reduce(const KvReduceArgs& a, hipStream_t s) {
  const long total = (long)a.Bsz * a.Npad * (a.D / 4);
  if (total <= 256l * kComputeUnits) hipLaunchKernelGGL((kv_reduce_kernel<T, 4>), dim3((total + 63) / 64), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((kv_reduce_kernel<T, 1>), dim3((total + 255) / 256), dim3(256), 0, s, a);
}
hipError_t launch_kv_reduce(int dtype, const KvReduceArgs& a, hipStream_t s) {
  if (dtype == 0) kv_reduce<float>(a, s);
  else kv_reduce<bf16>(a, s);
  return hipGetLastError();
}

}  // namespace ta
