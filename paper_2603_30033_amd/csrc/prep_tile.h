// One tile of the weight preparation (see prep.hip), as a device function: the preparation kernel runs
// one tile per workgroup, and a decode step lets the tiles ride along in the launch of its factor projection.
#pragma once
#include <type_traits>

#include "common.h"
#include "params.h"

namespace ta {

constexpr int kPrepTile = 64;

// workgroups (output tiles) of one job: 64 x 64 tiles of a copy, 32 x 32 tiles of kMixHeads mixed heads
constexpr int kMixTile = 32, kMixHeads = 4;
inline __host__ __device__ int prep_tiles(const PrepJob& j) {
  if (j.coef != nullptr)
    return ((j.Z + kMixHeads - 1) / kMixHeads) * ((j.rows_pad + kMixTile - 1) / kMixTile) * ((j.cols_pad + kMixTile - 1) / kMixTile);
  return j.Z * ((j.rows_pad + kPrepTile - 1) / kPrepTile) * ((j.cols_pad + kPrepTile - 1) / kPrepTile);
}

// 16 bytes of stored elements -> out (CE of them)
template <typename T> __device__ __forceinline__ void store_chunk(T* out, const float* x);
template <> __device__ __forceinline__ void store_chunk<bf16>(bf16* out, const float* x) {
  u32x4 pk;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f32x2 two = {x[2 * e], x[2 * e + 1]};
    pk[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
  }
  *reinterpret_cast<u32x4*>(out) = pk;
}
template <> __device__ __forceinline__ void store_chunk<float>(float* out, const float* x) {
  *reinterpret_cast<f32x4*>(out) = f32x4{x[0], x[1], x[2], x[3]};
}

// A 32 x 32 tile of kMixHeads head-mixed cores, sum_a coef[z][a] src[a]: every element of the core is fetched once for four heads
// (one head a workgroup read the core through the L2 once per head, 64 MB for 32 heads x 32 slices of 128 x 128, in batches of
// eight slices).  Thread = four neighbouring elements; 16 slices in flight.  Under the profiler, projection launch of a decode step
// with these tiles, 32 heads x 32 slices of 128 x 128, 24 sequences: 11.0 -> 8.7 us; 8 slices, 16 sequences: 7.5 -> 6.9; preparation
// alone, 32 heads x 8 slices and three factors of 4096 rows: 9.2 -> 6.3; 12 heads x 4 of 64 x 64: 5.7 -> 4.9.
template <typename T>
__device__ __forceinline__ void mix_tile(const PrepJob& jb, int local, float* lds) {
  constexpr int TS = kMixTile, NH = kMixHeads, CE = 16 / (int)sizeof(T);
  const int tiles_r = (jb.rows_pad + TS - 1) / TS, tiles_c = (jb.cols_pad + TS - 1) / TS;
  const int z0 = local / (tiles_r * tiles_c) * NH, rem = local % (tiles_r * tiles_c);
  const int r0 = (rem / tiles_c) * TS, c0 = (rem % tiles_c) * TS;
  const T* src = static_cast<const T*>(jb.src);
  const T* coef = static_cast<const T*>(jb.coef);
  // a head's coefficients (at most 64), one per lane, broadcast from there; 0 past the last slice
  const int lane = threadIdx.x % kWave;
  float cl[NH];
#pragma unroll
  for (int k = 0; k < NH; ++k)
    cl[k] = lane < jb.A ? to_f32(coef[(long)min(z0 + k, jb.Z - 1) * jb.A + min(lane, jb.A - 1)]) : 0.f;

  const int tr = threadIdx.x / 8, tc = (threadIdx.x % 8) * 4;      // this thread's row and first column in the tile
  const int row = min(r0 + tr, jb.rows - 1);
  float acc[NH][4];
#pragma unroll
  for (int k = 0; k < NH; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[k][e] = 0.f;
  auto add = [&](int a, const float (&x)[4]) {
#pragma unroll
    for (int k = 0; k < NH; ++k) {
      const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cl[k]), min(a, kWave - 1)));
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[k][e] += w * x[e];
    }
  };
  if (jb.cols % 4 == 0 && reinterpret_cast<uintptr_t>(src) % (4 * sizeof(T)) == 0) {
    typedef typename std::conditional<sizeof(T) == 2, u32x2, u32x4>::type Quad;
    const T* at = src + (long)row * jb.cols + min(c0 + tc, jb.cols - 4);   // a quad past the end re-reads the last one
    const long slice = (long)jb.rows * jb.cols;
    auto batch = [&](auto n_c, int a0) {                           // n slices from a0 on, all their loads in front of the first use
      constexpr int N = decltype(n_c)::value;
      Quad v[N];
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = *reinterpret_cast<const Quad*>(at + min(a0 + u, jb.A - 1) * slice);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < N; ++u) {
        float x[4];
        if constexpr (sizeof(T) == 2) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            x[2 * e] = __uint_as_float(v[u][e] << 16);
            x[2 * e + 1] = __uint_as_float(v[u][e] & 0xffff0000u);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(v[u][e]);
        }
        add(a0 + u, x);
      }
    };
    int a0 = 0;
    for (; jb.A - a0 > 8; a0 += 16) batch(std::integral_constant<int, 16>{}, a0);
    if (jb.A - a0 > 4) batch(std::integral_constant<int, 8>{}, a0);
    else if (jb.A > a0) batch(std::integral_constant<int, 4>{}, a0);
  } else {
    for (int a = 0; a < jb.A; ++a) {
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = to_f32(src[((long)a * jb.rows + row) * jb.cols + min(c0 + tc + e, jb.cols - 1)]);
      add(a, x);
    }
  }
  // element (r, c) of head k stands at column (c + r) % 32 of its row: reads along either direction spread over the banks
  auto place = [&](int k, int r, int c) -> float& { return lds[(k * TS + r) * TS + ((c + r) & (TS - 1))]; };
#pragma unroll
  for (int k = 0; k < NH; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool inside = r0 + tr < jb.rows && c0 + tc + e < jb.cols;   // the padded part of the output is zero
      place(k, tr, tc + e) = inside ? acc[k][e] * jb.scale : 0.f;
    }
  __syncthreads();

  const int u_ext = jb.transposed ? jb.cols_pad : jb.rows_pad, v_ext = jb.transposed ? jb.rows_pad : jb.cols_pad;
  const int u0 = jb.transposed ? c0 : r0, v0 = jb.transposed ? r0 : c0;
  constexpr int CPU = TS / CE;                                    // chunks per output row of the tile
  for (int ci = threadIdx.x; ci < NH * TS * CPU; ci += 256) {
    const int k = ci / (TS * CPU), ul = ci / CPU % TS, vc = (ci % CPU) * CE;
    const int u = u0 + ul, v = v0 + vc;
    if (z0 + k >= jb.Z || u >= u_ext || v >= v_ext) continue;
    float x[CE];
#pragma unroll
    for (int e = 0; e < CE; ++e) {
      const int vn = jb.perm ? acc_index(vc + e) : vc + e;        // natural index inside the tile (v0 is a multiple of 32)
      x[e] = jb.transposed ? place(k, vn, ul) : place(k, ul, vn);
    }
    long off;
    if (jb.frag) off = ((long)(u / 32) * (v_ext / 32) + v / 32) * kFragBlockElems + frag_major_offset<T>(u % 32, v % 32);
    else off = (long)u * jb.out_stride_u + v;
    store_chunk<T>(static_cast<T*>(jb.out) + (long)(z0 + k) * jb.out_stride_z + off, x);
  }
}

// one tile (workgroup index blk over all jobs); `tile` is kPrepTile x (kPrepTile + 1) floats of LDS
template <typename T>
__device__ __forceinline__ void prep_tile(const PrepArgs& args, int blk, float (*tile)[kPrepTile + 1]) {
  constexpr int TS = kPrepTile, CE = 16 / (int)sizeof(T);
  int ji = 0;
#pragma unroll
  for (int j = 1; j < kMaxPrepJobs; ++j)
    if (j < args.n_jobs && blk >= args.job[j].first_block) ji = j;
  const PrepJob& jb = args.job[ji];
  const int local = blk - jb.first_block;
  static_assert(kMixHeads * kMixTile * kMixTile <= TS * (TS + 1), "the mixed heads fit the tile");
  if (jb.coef != nullptr) {
    mix_tile<T>(jb, local, &tile[0][0]);
    return;
  }
  const int tiles_r = (jb.rows_pad + TS - 1) / TS, tiles_c = (jb.cols_pad + TS - 1) / TS;
  const int z = local / (tiles_r * tiles_c);
  const int rem = local % (tiles_r * tiles_c);
  const int r0 = (rem / tiles_c) * TS, c0 = (rem % tiles_c) * TS;
  const T* src = static_cast<const T*>(jb.src);
  T* out = static_cast<T*>(jb.out) + (long)z * jb.out_stride_z;

  // ---- source tile (rows r0.., columns c0..) -> LDS ---------------------------------------------------
  // Rows whose length and base keep every 16-byte chunk aligned are read a chunk per load (thread = chunk tx of rows ty,
  // ty+32); other shapes an element per load (thread = column tx of rows ty, ty+4, ...).
  const bool chunked = jb.cols % CE == 0 && reinterpret_cast<uintptr_t>(src) % 16 == 0;
  if (chunked) {
    constexpr int CPR = TS / CE;                                  // chunks per tile row
    constexpr int RPT = TS * CPR / 256;                           // rows per thread
    const int tx = threadIdx.x % CPR, ty = threadIdx.x / CPR;
    const int col = c0 + tx * CE;
    const int colc = min(col, jb.cols - CE);                      // a chunk past the end re-reads the last one
    u32x4 v[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i)
      v[i] = *reinterpret_cast<const u32x4*>(src + (long)min(r0 + ty + (256 / CPR) * i, jb.rows - 1) * jb.cols + colc);
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = ty + (256 / CPR) * i;
      float x[CE];
      if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[2 * e] = __uint_as_float(v[i][e] << 16);
          x[2 * e + 1] = __uint_as_float(v[i][e] & 0xffff0000u);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(v[i][e]);
      }
#pragma unroll
      for (int e = 0; e < CE; ++e) {
        const bool inside = r0 + r < jb.rows && col + e < jb.cols; // the padded part of the output is zero
        tile[r][tx * CE + e] = inside ? x[e] * jb.scale : 0.f;
      }
    }
  } else {
    constexpr int RPT = TS / 4;                                   // rows per thread
    const int tx = threadIdx.x % TS, ty = threadIdx.x / TS;
    const int col = min(c0 + tx, jb.cols - 1);
    T v[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) v[i] = src[(long)min(r0 + ty + 4 * i, jb.rows - 1) * jb.cols + col];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = ty + 4 * i;
      const bool inside = r0 + r < jb.rows && c0 + tx < jb.cols;
      tile[r][tx] = inside ? to_f32(v[i]) * jb.scale : 0.f;
    }
  }
  __syncthreads();

  // ---- output chunks of CE consecutive stored positions -----------------------------------------------
  // (u, v) = (column, row) of the source when transposed, (row, column) otherwise; with perm the stored
  // position p of a 32-block holds natural index acc_index(p)
  const int u_ext = jb.transposed ? jb.cols_pad : jb.rows_pad, v_ext = jb.transposed ? jb.rows_pad : jb.cols_pad;
  const int u0 = jb.transposed ? c0 : r0, v0 = jb.transposed ? r0 : c0;
  constexpr int CPU = TS / CE;                                    // chunks per output row of the tile
  for (int ci = threadIdx.x; ci < TS * CPU; ci += 256) {
    // consecutive threads take consecutive chunks of one output row
    const int ul = ci / CPU, vc = (ci % CPU) * CE;
    const int u = u0 + ul, v = v0 + vc;
    if (u >= u_ext || v >= v_ext) continue;
    float x[CE];
#pragma unroll
    for (int e = 0; e < CE; ++e) {
      const int p = (v + e) % 32, vb = (v + e) - p;
      const int vn = vb + (jb.perm ? acc_index(p) : p) - v0;       // natural index inside the tile
      x[e] = jb.transposed ? tile[vn][ul] : tile[ul][vn];
    }
    long off;
    if (jb.frag) {
      const int nvb = v_ext / 32;
      off = ((long)(u / 32) * nvb + v / 32) * kFragBlockElems + frag_major_offset<T>(u % 32, v % 32);
    } else {
      off = (long)u * jb.out_stride_u + v;
    }
    store_chunk<T>(out + off, x);
  }
}

}  // namespace ta
