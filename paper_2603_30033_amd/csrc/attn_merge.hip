// Prefill attention and head merge in one kernel, for many short sequences of narrow latents (bf16, D <= 64): the keys and values
// of a sequence fit the LDS of a compute unit, all heads share them, and one wave takes 32 queries through all the heads (or
// every hs-th pair of them) and keeps their merged latent Z = sum_i G~_i O_i in its accumulators.  The per-head outputs
// are never stored, K and V are staged once, and behind that no wave waits for another.
//   The products are those of the prefill kernel (transposed, a lane owns one query; see there and the fragment model in
// common.h), followed by Z^T[b][m] += sum_c G~_i[b][c] O_i^T[c][m] with the normalised O_i rounded to bf16 as if it were stored.
// A wave works on two heads at a time: they share every K and V fragment read from LDS, and give the matrix and the vector unit
// independent work.
//   256 sequences of 197 tokens, 12 heads, D = 64: 66 us against 113 + 21 for the prefill kernel and the product behind it.  Half of
// its time a SIMD issues vector instructions (exponentials first), 0.4 of it its matrix unit is busy; the rest is the
// latency of a pair's start and end with two waves on a SIMD.  Tried: four waves of one head on 128 registers with the outputs
// stored 66 + 21; two heads in turn, probabilities of one under the products of the other, outputs stored 71 + 21; the
// cores of a pair staged in LDS 74 (a barrier per pair); the online softmax for all scores 75.
//   With latents of 64 channels and merged ones of 64, 96 and 128, 7, 24 and 38 registers go through scratch memory, at the start and
// the end of a pair; the loops over the keys touch none.
//   Without a reference exponent the largest probability of a row is rounded to bf16 like the others, where with one it is exactly
// 1: the error of those 256 sequences against fp64 is 4.916e-3, 4.896e-3 in the prefill kernel, whose first 64 keys give the
// reference.  With that reference here the whole pass takes 5 % more, with the one of the first 32 keys (4.900e-3) 2 to 5 %.
#include <type_traits>

#include "common.h"
#include "params.h"

namespace ta {

// Scores of at most kPlainScore in magnitude need no reference exponent over values between 2^-40 and 2^32 (or zero):
// probabilities up to 2^64 of 1280 keys times values up to 2^32 stay below 2^107, and one of 2^-64 times 2^-40 is 2^22 times the
// smallest normal number, so that what a sum of 1280 such products loses below it is less than the rounding to bf16.
constexpr float kPlainScore = 64.f;
constexpr unsigned kPlainMost = (127 + 32) << 7, kPlainLeast = (127 - 40) << 7;   // magnitudes as bf16 bits
template <int CB, int ZB>
__global__ __launch_bounds__(512) void attn_merge_kernel(AttnMergeArgs p) {
  typedef bf16 T;
  constexpr int D = 32 * CB, HP = 2;                            // heads at a time
  constexpr int KCPR = D / 8, VCPR = 4;                         // 16-byte chunks per row of a K tile [32][D], a V^T tile [D][32]
  constexpr int kTile = 32 * D;                                 // elements of either
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  T* smem = reinterpret_cast<T*>(smem_raw);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, h = lane / 32, lr = lane % 32;
  const int n_chunks = (p.nqb + p.qpw - 1) / p.qpw;
  const int b = blockIdx.x / n_chunks, chunk = n_chunks - 1 - blockIdx.x % n_chunks;   // (causal) heavy chunks first
  const int hg = wave / p.qpw, w = wave % p.qpw;
  // the two waves of a SIMD (w and w + 4) take query blocks from either end: with a causal mask their work adds up alike
  const int wq = w < 4 ? w : p.qpw + 3 - w;
  const int qb = chunk * p.qpw + wq;
  const bool live = qb < p.nqb;
  const long tok_base = (long)b * p.Npad;

  // ---- all keys and values this workgroup needs, straight into LDS: tile j = K rows and V^T columns 32 j .. 32 j + 31 ----
  const int n_keys = p.causal ? min(p.N, 32 * min((chunk + 1) * p.qpw, p.nqb)) : p.N;
  const int nkb = (n_keys + 31) / 32;
  {
    const T* Kg = static_cast<const T*>(p.Kr) + tok_base * D;
    const T* Vg = static_cast<const T*>(p.Vt) + (long)b * D * p.Npad;
    const int n_waves = blockDim.x / kWave;
    constexpr int PT = kTile / 512;                             // 1 KB pieces of a tile
    for (int q = wave; q < 2 * PT * nkb; q += n_waves) {
      const int j = q / (2 * PT), piece = q % (2 * PT);
      T* tile = smem + (long)(2 * j) * kTile;
      if (piece < PT) dma_piece<T, KCPR>(tile, piece, lane, [&](int row) { return Kg + (long)(32 * j + row) * D; });
      else dma_piece<T, VCPR>(tile + kTile, piece - PT, lane, [&](int row) { return Vg + (long)row * p.Npad + 32 * j; });
    }
  }
  const int nbb = p.R2 / 32;
  const int n_pairs = (p.nH + HP - 1) / HP;
  const int m = 32 * qb + lr;                                   // this lane's query (< Npad where live)
  const T* Ql = static_cast<const T*>(p.Qlat) + (tok_base + (live ? m : lr)) * p.R2 + 16 * h;
  // the latent query, the same for all heads: its first two blocks are kept
  const Frag<T> x0 = load_frag<T>(Ql), x1 = load_frag<T>(Ql + 32 * min(1, nbb - 1));
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // largest |k|^2 (infinite where a value is too large or too small for plain probabilities); the last channel of the values, where it is
  // padding, becomes ones, so that the products with the probabilities sum them along the way
  __shared__ float most[8];
  float k2 = 0.f;
  {
    unsigned v_most = 0u, v_least = ~0u;                        // least: less one, so that zero does not count
    for (int r = threadIdx.x; r < 32 * nkb; r += blockDim.x) {
      const T* row = smem + (long)(2 * (r / 32)) * kTile + (r % 32) * D;
      float n2 = 0.f;
#pragma unroll
      for (int u = 0; u < KCPR; ++u) {
        const bf16x8 x8 = *reinterpret_cast<const bf16x8*>(row + 8 * u);
#pragma unroll
        for (int e = 0; e < 8; ++e) n2 += (float)x8[e] * (float)x8[e];
      }
      k2 = n2 > k2 || n2 != n2 ? n2 : k2;                       // a NaN stays
      const T* val = smem + (long)(2 * (r / 32) + 1) * kTile + (r % 32) * D;
#pragma unroll
      for (int u = 0; u < KCPR; ++u) {
        const u32x4 x8 = *reinterpret_cast<const u32x4*>(val + 8 * u);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const unsigned size = (e % 2 ? x8[e / 2] >> 16 : x8[e / 2]) & 0x7fffu;
          v_most = max(v_most, size);
          v_least = min(v_least, size - 1u);
        }
      }
    }
    if (v_most > kPlainMost || v_least < kPlainLeast - 1u) k2 = INFINITY;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      const float y = __shfl_xor(k2, d);
      k2 = y > k2 || y != y ? y : k2;
    }
    if (lane == 0) most[wave] = k2;
    __syncthreads();
    for (int i = 0; i < (int)blockDim.x / kWave; ++i) k2 = most[i] > k2 || most[i] != most[i] ? most[i] : k2;
    if (p.ones) {
      for (int r = threadIdx.x; r < 32 * nkb; r += blockDim.x)
        smem[(long)(2 * (r / 32) + 1) * kTile + (D - 1) * 32 + r % 32] = (T)1.0f;
      __syncthreads();
    }
  }

  f32x16 zacc[ZB];
#pragma unroll
  for (int z = 0; z < ZB; ++z)
#pragma unroll
    for (int e = 0; e < 16; ++e) zacc[z][e] = 0.f;
  const int last_visible = p.causal ? min(m, p.N - 1) : p.N - 1;
  const int my_kb = p.causal ? min(qb + 1, nkb) : nkb;
  const f32x4* tab = reinterpret_cast<const f32x4*>(p.rope) + (long)h * p.rope_ld + p.pos0 + min(m, p.N - 1);

  const T* Gt = static_cast<const T*>(p.Gt);
  const T* G2 = static_cast<const T*>(p.Gtil2) + (long)lr * p.nH * D + 16 * h;
  for (int pair = hg; live && pair < n_pairs; pair += p.hs) {
    const int head[HP] = {HP * pair, min(HP * pair + 1, p.nH - 1)};
    // ---- per-head queries: Qhat^T = Gt_i Qlat^T, rotated ----
    Frag<T> qf[HP][CB];
    f32x16 o[HP][CB];
    {
#pragma unroll
      for (int i = 0; i < HP; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
          for (int e = 0; e < 16; ++e) o[i][c][e] = 0.f;
      auto multiply = [&](int bb, const Frag<T>& xb) {
#pragma unroll
        for (int i = 0; i < HP; ++i)
#pragma unroll
          for (int c = 0; c < CB; ++c)
            mma32(o[i][c], load_frag_major<T>(Gt + (long)head[i] * D * p.R2 + (long)(c * nbb + bb) * kFragBlockElems, lane), xb);
      };
      multiply(0, x0);
      if (nbb > 1) multiply(1, x1);
      for (int bb = 2; bb < nbb; ++bb) multiply(bb, load_frag<T>(Ql + bb * 32));
      if (p.rope != nullptr) {
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 cs = tab[(long)(c * 8 + 2 * q) * p.rope_ld];
#pragma unroll
            for (int i = 0; i < HP; ++i)
#pragma unroll
              for (int e = 0; e < 4; e += 2) {
                const float u0 = o[i][c][4 * q + e], u1 = o[i][c][4 * q + e + 1];
                o[i][c][4 * q + e] = u0 * cs[e] - u1 * cs[e + 1];
                o[i][c][4 * q + e + 1] = u0 * cs[e + 1] + u1 * cs[e];
              }
          }
      }
#pragma unroll
      for (int i = 0; i < HP; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) {
          qf[i][c] = to_frag<T>(o[i][c]);
#pragma unroll
          for (int e = 0; e < 16; ++e) o[i][c][e] = 0.f;
        }
    }

    // ---- softmax over the key blocks ----
    // PLAIN: |s| <= |q| max |k| bounds every score of this wave, so that exp2(s) needs no reference (and the loop no
    // reductions across lanes).  Otherwise the online form, reference refreshed only when a block exceeds it by 2^kLazy.
    constexpr float kLazy = 8.f;
    float m_ref[HP], l_run[HP];
    bool plain = true;
#pragma unroll
    for (int i = 0; i < HP; ++i) {
      m_ref[i] = l_run[i] = 0.f;
      float q2 = 0.f;
#pragma unroll
      for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const bf16x2 two = {qf[i][c].v[u][e], qf[i][c].v[u][e + 1]};
            q2 = __builtin_amdgcn_fdot2_f32_bf16(two, two, q2, false);
          }
      plain = plain && halves_sum(q2) * k2 <= kPlainScore * kPlainScore;   // false for a NaN
    }
    auto key_loop = [&](auto plain_c) {
      constexpr bool PLAIN = decltype(plain_c)::value;
      for (int j = 0; j < my_kb; ++j) {
        const T* kt = smem + (long)(2 * j) * kTile;
        const T* vt = kt + kTile;
        f32x16 s[HP];
#pragma unroll
        for (int i = 0; i < HP; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) s[i][e] = 0.f;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
          const Frag<T> k = load_frag_swz<T>(kt + lr * D, 4 * c + 2 * h, swz_x<KCPR>(lr));
#pragma unroll
          for (int i = 0; i < HP; ++i) mma32(s[i], k, qf[i][c]);
        }
        Frag<T> v[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) v[c] = load_frag_swz<T>(vt + (32 * c + lr) * 32, 2 * h, swz_x<VCPR>(32 * c + lr));
        if (32 * j + 32 > p.N || (p.causal && j == qb)) {
#pragma unroll
          for (int i = 0; i < HP; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (32 * j + 8 * (e / 4) + 4 * h + (e % 4) > last_visible) s[i][e] = -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < HP; ++i) {
          if constexpr (!PLAIN) {
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[i][e]);
            mx = halves_max(mx) - m_ref[i];
            const bool upd = (j == 0 || mx > kLazy) && mx != -INFINITY;
            if (__builtin_amdgcn_ballot_w64(upd) != 0ull) {
              const float delta = upd ? mx : 0.f, alpha = j == 0 ? 1.f : fast_exp2(-delta);   // block 0: O and l are still zero
              m_ref[i] += delta;
              l_run[i] *= alpha;
#pragma unroll
              for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[i][c][e] *= alpha;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) s[i][e] = fast_exp2(s[i][e] - m_ref[i]);
          } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) s[i][e] = fast_exp2(s[i][e]);
          }
          const Frag<T> pf = to_frag<T>(s[i]);
          // the rounded probabilities, as they are multiplied: a row of one key then has the value itself as its result
          if (!p.ones) l_run[i] = frag_sum(pf, l_run[i]);
#pragma unroll
          for (int c = 0; c < CB; ++c) mma32(o[i][c], v[c], pf);
        }
      }
    };
    if (__builtin_amdgcn_ballot_w64(!plain) == 0ull) key_loop(std::true_type{});
    else key_loop(std::false_type{});

    // ---- normalise, round as a stored O would be, merge ----
#pragma unroll
    for (int i = 0; i < HP; ++i) {
      Frag<T> g[CB][ZB];
#pragma unroll
      for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int z = 0; z < ZB; ++z) g[c][z] = load_frag<T>(G2 + (long)(32 * z) * p.nH * D + (long)head[i] * D + 32 * c);
      // row D - 1 of O: half 1, last register
      const float l_tot = halves_sum(p.ones ? (h == 1 ? o[i][CB - 1][15] : 0.f) : l_run[i]);
      const bool counts = m < p.N && HP * pair + i < p.nH;      // padding queries, and the second head of an odd last pair
      const float inv = counts ? 1.f / l_tot : 0.f;
#pragma unroll
      for (int c = 0; c < CB; ++c) {
#pragma unroll
        for (int e = 0; e < 16; ++e) o[i][c][e] = counts ? o[i][c][e] * inv : 0.f;
        const Frag<T> of = to_frag<T>(o[i][c]);
#pragma unroll
        for (int z = 0; z < ZB; ++z) mma32(zacc[z], g[c][z], of);
      }
    }
  }

  // ---- the head groups' sums in their order, then Z[tok][RT2] in natural order ----
  if (p.hs > 1) {
    __syncthreads();                                            // K and V are done with
    float* sums = reinterpret_cast<float*>(smem_raw);           // [hs - 1][qpw][16 ZB][64]
    if (hg > 0) {
      float* to = sums + (long)((hg - 1) * p.qpw + w) * (16 * ZB * 64) + lane;
#pragma unroll
      for (int z = 0; z < ZB; ++z)
#pragma unroll
        for (int e = 0; e < 16; ++e) to[(16 * z + e) * 64] = zacc[z][e];
    }
    __syncthreads();
    if (hg == 0)
      for (int g = 1; g < p.hs; ++g) {
        const float* from = sums + (long)((g - 1) * p.qpw + w) * (16 * ZB * 64) + lane;
#pragma unroll
        for (int z = 0; z < ZB; ++z)
#pragma unroll
          for (int e = 0; e < 16; ++e) zacc[z][e] += from[(16 * z + e) * 64];
      }
  }
  if (live && hg == 0) {
    T* Z = static_cast<T*>(p.Z) + (tok_base + m) * p.RT2 + 4 * h;
#pragma unroll
    for (int z = 0; z < ZB; ++z)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        store4(Z + 32 * z + 8 * q, zacc[z][4 * q], zacc[z][4 * q + 1], zacc[z][4 * q + 2], zacc[z][4 * q + 3]);
    if (qb == p.nqb - 1 && 32 * p.nqb < p.Npad) {               // a block of padding tokens behind the last one: zeros
      Z += 32l * p.RT2;
#pragma unroll
      for (int z = 0; z < ZB; ++z)
#pragma unroll
        for (int q = 0; q < 4; ++q) store4(Z + 32 * z + 8 * q, 0.f, 0.f, 0.f, 0.f);
    }
  }
}

namespace {
constexpr size_t kLdsMost = 160 * 1024 - 256;                   // beside the few words of the norms

// Waves below which the chip is better filled by the prefill kernel, whose workgroups split the heads (the time here is then that
// of one wave).  D = 64: 12 heads, ranks up to 64, 1024 waves 54.8 -> 51.4 us (128 x 128 tokens) and 94.4 -> 92.9 (128 x
// 250), 896 waves 93.2 -> 83.7 (128 x 197), 560 waves 67.3 -> 70.1; 1600 waves 143 -> 99.  So the two meet between 560 and 896, and
// the line stands above, where every SIMD has a wave.  Ranks of 128 have twice the products outside the key loop: 1280 waves
// 169 -> 180, 2048 116 -> 103.  D = 32 has half of them: 512 waves 19.8 -> 19.1.
long fewest_waves(const AttnMergeArgs& a) {
  return (a.R2 > 64 || a.RT2 > 64 ? 2048 : 1024) / (a.D == 32 ? 2 : 1);
}

// Query blocks dealt evenly to workgroups of at most eight waves; where that leaves waves free, the heads are split.  False
// where the LDS has no room for the keys.
bool plan(AttnMergeArgs& a, size_t& smem) {
  const int chunks = (a.nqb + 7) / 8, pairs = (a.nH + 1) / 2;
  a.qpw = (a.nqb + chunks - 1) / chunks;
  a.hs = 8 / a.qpw < pairs ? 8 / a.qpw : pairs;
  const size_t sums = (size_t)(a.hs - 1) * a.qpw * 16 * (a.RT2 / 32) * 64 * sizeof(float);
  smem = (size_t)a.nqb * 2 * 32 * a.D * sizeof(bf16);
  if (sums > smem) smem = sums;
  return smem <= kLdsMost;
}

template <int CB, int ZB> hipError_t launch_one(const AttnMergeArgs& a, size_t smem, hipStream_t s, hipEvent_t k0, hipEvent_t k1) {
  const dim3 grid(a.Bsz * ((a.nqb + a.qpw - 1) / a.qpw)), block(64 * a.qpw * a.hs);
  auto kern = attn_merge_kernel<CB, ZB>;
  static LdsOnce lds_once;
  if (hipError_t e = allow_dynamic_lds(lds_once, kern, kLdsMost); e != hipSuccess) return e;
  if (k0 != nullptr && k1 != nullptr) hipExtLaunchKernelGGL(kern, grid, block, (uint32_t)smem, s, k0, k1, 0, a);
  else hipLaunchKernelGGL(kern, grid, block, smem, s, a);
  return hipGetLastError();
}
}  // namespace

bool attn_merge_supported(int dtype, const AttnMergeArgs& in) {
  if (dtype != 1 || (in.D != 32 && in.D != 64) || in.RT2 > 128) return false;
  AttnMergeArgs a = in;
  size_t smem;
  return plan(a, smem) && (long)a.Bsz * a.nqb * a.hs >= fewest_waves(a);
}

hipError_t launch_attn_merge(const AttnMergeArgs& in, hipStream_t s, hipEvent_t k0, hipEvent_t k1) {
  AttnMergeArgs a = in;
  size_t smem;
  if (!plan(a, smem)) return hipErrorInvalidValue;
  if (a.D == 32) switch (a.RT2) {
      case 32: return launch_one<1, 1>(a, smem, s, k0, k1);
      case 64: return launch_one<1, 2>(a, smem, s, k0, k1);
      case 96: return launch_one<1, 3>(a, smem, s, k0, k1);
      case 128: return launch_one<1, 4>(a, smem, s, k0, k1);
    }
  if (a.D == 64) switch (a.RT2) {
      case 32: return launch_one<2, 1>(a, smem, s, k0, k1);
      case 64: return launch_one<2, 2>(a, smem, s, k0, k1);
      case 96: return launch_one<2, 3>(a, smem, s, k0, k1);
      case 128: return launch_one<2, 4>(a, smem, s, k0, k1);
    }
  return hipErrorInvalidValue;
}

}  // namespace ta
