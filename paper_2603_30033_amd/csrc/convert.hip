// Weight front-ends: classic attention weights -> Tucker-attention weights, on the device.
//   * GQA / MQA / MHA and MLA: the exact representations of the appendix "Tucker Representations
//     of MQA, GQA, and MLA" (selector cores; down-projections as bases, products of the
//     up-projections as core slices).
//   * MHA -> Tucker by a truncated higher-order SVD (appendix "Converting pretrained MHA
//     parameters to approximate attention parameters"), in fp64: Gram matrices of the mode
//     unfoldings from the dH-wide factors, their leading eigenvectors (all the d x d problems side by side
//     through a reduction to tridiagonal form, eigen.hip; the head mode and what that path does not take by a
//     one-sided Jacobi iteration), core by contraction with the transposed factors.
#include "../../include/tucker_attn.h"
#include "../../include/tucker_convert.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

#include "common.h"
#include "eigen.h"

namespace ta {
namespace {

// ---------------------------------------------------------------------------------------------
// element-wise builders of the exact representations
// ---------------------------------------------------------------------------------------------

template <typename T> __device__ __forceinline__ T from_f64(double v);
template <> __device__ __forceinline__ float from_f64<float>(double v) { return (float)v; }
template <> __device__ __forceinline__ bf16 from_f64<bf16>(double v) { return (bf16)(float)v; }

// C[i][row][col] = 1 iff row = (i,l) and col = (g(i),l); one pass over the whole core
template <typename T>
__global__ __launch_bounds__(256) void selector_core_kernel(T* C, int nH, int dH, int nG) {
  const long rows = (long)nH * dH, cols = (long)nG * dH;
  const long total = (long)nH * rows * cols;
  const int per = nH / nG;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const long col = e % cols, row = (e / cols) % rows, i = e / (cols * rows);
    const bool one = row / dH == i && col / dH == i / per && row % dH == col % dH;
    C[e] = from_f64<T>(one ? 1.0 : 0.0);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void identity_kernel(T* U, int n) {
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < (long)n * n; e += (long)gridDim.x * 256)
    U[e] = from_f64<T>(e / n == e % n ? 1.0 : 0.0);
}

// out[c][r] = in[r][c] through a 32x32 LDS tile; in is [rows, cols]
template <typename T>
__global__ __launch_bounds__(256) void transpose_copy_kernel(const T* in, T* out, int rows, int cols) {
  __shared__ T tile[32][33];
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int j = ty; j < 32; j += 8)
    if (r0 + j < rows && c0 + tx < cols) tile[j][tx] = in[(long)(r0 + j) * cols + c0 + tx];
  __syncthreads();
  for (int j = ty; j < 32; j += 8)
    if (c0 + j < cols && r0 + tx < rows) out[(long)(c0 + j) * rows + r0 + tx] = tile[tx][j];
}

// MLA pre-softmax core slice C[i][a][c] = sum_l WUQ[a][(i,l)] WUK[c][(i,l)]
template <typename T>
__global__ __launch_bounds__(256) void mla_core_kernel(const T* WUQ, const T* WUK, T* C, int nH, int dH, int dcQ, int dcK) {
  const long n = (long)nH * dH;
  const long total = (long)nH * dcQ * dcK;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const long c = e % dcK, a = (e / dcK) % dcQ, i = e / ((long)dcK * dcQ);
    const T* q = WUQ + a * n + i * dH;
    const T* k = WUK + c * n + i * dH;
    float acc = 0.f;
    for (int l = 0; l < dH; ++l) acc += to_f32(q[l]) * to_f32(k[l]);
    C[e] = from_f64<T>((double)acc);
  }
}

// MLA post-softmax core slice C~[i][(j,l)][c] = (j == i) ? WUV[c][(i,l)] : 0
template <typename T>
__global__ __launch_bounds__(256) void mla_post_core_kernel(const T* WUV, T* Ct, int nH, int dH, int dcK) {
  const long n = (long)nH * dH;
  const long total = (long)nH * n * dcK;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const long c = e % dcK, row = (e / dcK) % n, i = e / (dcK * n);
    Ct[e] = row / dH == i ? WUV[c * n + row] : from_f64<T>(0.0);
  }
}

// ---------------------------------------------------------------------------------------------
// fp64 pieces of the higher-order SVD
// ---------------------------------------------------------------------------------------------

// out[r][c] = in[r*sr + c*sc] as fp64, out row-major [rows, cols]
template <typename T>
__global__ __launch_bounds__(256) void to_f64_kernel(const T* in, long sr, long sc, double* out, int rows, int cols) {
  const long total = (long)rows * cols;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256)
    out[e] = (double)to_f32(in[(e / cols) * sr + (e % cols) * sc]);
}

template <typename T>
__global__ __launch_bounds__(256) void from_f64_kernel(const double* in, T* out, long total) {
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) out[e] = from_f64<T>(in[e]);
}

// C[m][n] = sum_k A(m,k) B(k,n) with element strides for every index (any transposition is a
// choice of strides) and a batch stride.
struct DgemmArgs {
  const double* A; long a_m, a_k, a_b;
  const double* B; long b_k, b_n, b_b;
  double* C; long c_m, c_n, c_b;
  int M, N, K;
};

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Tile of 32 BT x 32 BT, four waves with BT x BT blocks of the 16 x 16 x 4 fp64 matrix instruction each (lane l
// supplies A[l%16][l/16] and B[l/16][l%16] and receives D[l/16 + 4i][l%16] in register i); the next slice is
// loaded into registers while the current one is multiplied.  Bound by the matrix instruction (64 cycles) once
// every SIMD has a wave.
template <int BT>
__global__ __launch_bounds__(256) void dgemm_kernel(DgemmArgs g) {
  constexpr int TM = 32 * BT, KS = 32 / BT, E = TM * KS / 256;
  __shared__ double As[2][KS][TM + 2], Bs[2][KS][TM + 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
  const int mw = (wave >> 1) * 16 * BT, nw = (wave & 1) * 16 * BT;
  const double* A = g.A + (long)blockIdx.z * g.a_b;
  const double* B = g.B + (long)blockIdx.z * g.b_b;
  double* C = g.C + (long)blockIdx.z * g.c_b;
  f64x4 acc[BT][BT];
#pragma unroll
  for (int i = 0; i < BT; ++i)
#pragma unroll
    for (int j = 0; j < BT; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  double va[E], vb[E];
  // lanes run along the contiguous index of each operand
  auto at_a = [&](int j, int& k, int& m) { const int e = tid + 256 * j; k = g.a_k == 1 ? e % KS : e / TM; m = g.a_k == 1 ? e / KS : e % TM; };
  auto at_b = [&](int j, int& k, int& n) { const int e = tid + 256 * j; k = g.b_n == 1 ? e / TM : e % KS; n = g.b_n == 1 ? e % TM : e / KS; };
  auto load = [&](int k0) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      int k, m;
      at_a(j, k, m);
      va[j] = (m0 + m < g.M && k0 + k < g.K) ? A[(long)(m0 + m) * g.a_m + (long)(k0 + k) * g.a_k] : 0.0;
      at_b(j, k, m);
      vb[j] = (n0 + m < g.N && k0 + k < g.K) ? B[(long)(k0 + k) * g.b_k + (long)(n0 + m) * g.b_n] : 0.0;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      int k, m;
      at_a(j, k, m);
      As[buf][k][m] = va[j];
      at_b(j, k, m);
      Bs[buf][k][m] = vb[j];
    }
  };
  const int ns = (g.K + KS - 1) / KS;
  load(0);
  store(0);
  __syncthreads();
  for (int s = 0; s < ns; ++s) {
    if (s + 1 < ns) load((s + 1) * KS);
    const int buf = s & 1;
#pragma unroll
    for (int kk = 0; kk < KS / 4; ++kk) {
      double a[BT], b[BT];
#pragma unroll
      for (int i = 0; i < BT; ++i) a[i] = As[buf][4 * kk + lq][mw + 16 * i + lr];
#pragma unroll
      for (int j = 0; j < BT; ++j) b[j] = Bs[buf][4 * kk + lq][nw + 16 * j + lr];
#pragma unroll
      for (int i = 0; i < BT; ++i)
#pragma unroll
        for (int j = 0; j < BT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (s + 1 < ns) store((s + 1) & 1);                 // last read before the previous barrier
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < BT; ++i)
#pragma unroll
    for (int j = 0; j < BT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + mw + 16 * i + lq + 4 * r, n = n0 + nw + 16 * j + lr;
        if (m < g.M && n < g.N) C[(long)m * g.c_m + (long)n * g.c_n] = acc[i][j][r];
      }
}

// M1[i][j] = <W_i, W_j> = sum_{l,m} (A_i^T A_j)[l][m] (B_i^T B_j)[l][m]; GA = A^T A, GB = B^T B [n, n]
__global__ __launch_bounds__(256) void head_gram_kernel(const double* GA, const double* GB, double* M1, int nH, int dH) {
  const int i = blockIdx.y, j = blockIdx.x;
  const long n = (long)nH * dH;
  double s = 0.0;
  for (int e = threadIdx.x; e < dH * dH; e += 256) {
    const long at = ((long)i * dH + e / dH) * n + (long)j * dH + e % dH;
    s += GA[at] * GB[at];
  }
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int sft = 128; sft > 0; sft >>= 1) {
    if ((int)threadIdx.x < sft) red[threadIdx.x] += red[threadIdx.x + sft];
    __syncthreads();
  }
  if (threadIdx.x == 0) M1[(long)i * nH + j] = red[0];
}

// sums of up to three doubles over the 256 threads of a block; every thread receives them
__device__ __forceinline__ void block_sum3(double& a, double& b, double& c, double (*red)[3]) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_down(a, o);
    b += __shfl_down(b, o);
    c += __shfl_down(c, o);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[w][0] = a; red[w][1] = b; red[w][2] = c; }
  __syncthreads();
  a = red[0][0] + red[1][0] + red[2][0] + red[3][0];
  b = red[0][1] + red[1][1] + red[2][1] + red[3][1];
  c = red[0][2] + red[1][2] + red[2][2] + red[3][2];
}

// One step of a blocked one-sided Jacobi sweep on the rows of G [m, len].  The rows are grouped in
// blocks of 8; workgroup k takes the k-th pair (P, Q) of round `step` of a round-robin tournament
// over the blocks (pairs of one round are disjoint, so workgroups touch disjoint rows) and
//   1. forms the 16 x 16 Gram matrix S = R R^T of its 16 rows with the fp64 matrix instruction
//      (D[16x16] += A[16x4] B[4x16]; lane l supplies A[l%16][l/16] and B[l/16][l%16], which for
//      B = A^T is the same register, and receives D[l/16 + 4i][l%16] in register i),
//   2. runs one cyclic sweep of two-sided Jacobi rotations on S in LDS (15 rounds of 8 disjoint
//      rotations, worked out once per round), accumulating them in V,
//   3. replaces the rows by V^T R, again with the matrix instruction.
// A rotation is applied only if the inner product exceeds tol times the product of the two norms (the
// relative test, which keeps the small rows accurate relative to their own size).  Rows whose squared
// norm is at most `tiny` are numerically zero and are left alone.  Rows >= m of the last block
// read as zero and are never written.  `rotations` counts the rotations applied.
// One workgroup holds all rows of a matrix of at most 16 (m <= 16, step 0): with LOOP it goes on until a sweep finds
// nothing to rotate, and `rotations` receives the number of sweeps, 0 if `max_sweeps` were not enough; tiny is then
// worked out from the rows themselves.
template <int NW, bool LOOP>   // NW waves per workgroup: they share the columns in steps 1 and 3; the first four run step 2
__global__ __launch_bounds__(64 * NW) void jacobi_block_kernel(double* G, int m, int len, int step, double tol, double tiny,
                                                               int* rotations, int max_sweeps) {
  __shared__ double part[NW][16][17];                   // per-wave partial Gram matrices
  __shared__ double S[2][16][17];                       // double-buffered Gram matrix
  __shared__ double V[2][16][17];                       // accumulated rotations
  __shared__ int n_rot;
  const int nb = (m + 7) / 8, nbp = nb + (nb & 1), n1 = nbp - 1;
  const int k = blockIdx.x;
  const int P = k == 0 ? n1 : (step + k) % n1;
  const int Q = k == 0 ? step : (step - k + n1) % n1;
  // with an odd number of blocks one workgroup per round holds the bye (block index nb): its rows lie
  // beyond m and read as zero, so the workgroup still rotates the rows of its real block among themselves
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  auto row_of = [&](int r) { return (r < 8 ? P * 8 : Q * 8 - 8) + r; };
  const int chunks = (len + 15) / 16;
  for (int sweep = 0;; ++sweep) {
  if (LOOP && sweep == max_sweeps) {
    if (tid == 0) *rotations = 0;
    return;
  }

  // 1. Gram matrix: lane (lr, lq) of a wave loads columns c0 + 4 lq .. + 3 of row lr of a 16-column chunk
  {
    const int grow = row_of(lr);
    const double* src = G + (long)grow * len;
    // four values of this lane's row at columns c .. c+3 (zero beyond the matrix)
    auto load4 = [&](int ch, double* x) __attribute__((always_inline)) {
      const int c = ch * 16 + 4 * lq;
      if (grow < m && c + 3 < len && (len & 1) == 0) {    // even rows start 16-byte aligned
        const f64x2 lo = *reinterpret_cast<const f64x2*>(src + c), hi = *reinterpret_cast<const f64x2*>(src + c + 2);
        x[0] = lo[0]; x[1] = lo[1]; x[2] = hi[0]; x[3] = hi[1];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = (grow < m && ch < chunks && c + j < len) ? src[c + j] : 0.0;
      }
    };
    f64x4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
    for (int ch = wave; ch < chunks; ch += 2 * NW) {      // two chunks in flight, two accumulation chains
      double x0[4], x1[4];
      load4(ch, x0);
      load4(ch + NW, x1);                                 // a chunk index beyond the row loads zeros
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0[j], x0[j], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x1[j], x1[j], acc1, 0, 0, 0);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) part[wave][lq + 4 * i][lr] = acc0[i] + acc1[i];
  }
  if (tid == 0) n_rot = 0;
  __syncthreads();
  const int ti = (tid >> 4) & 15, tj = tid & 15;        // this thread's element of S and V (threads 0..255)
  const bool solver = tid < 256;
  if (solver) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) sum += part[w][ti][tj];
    S[0][ti][tj] = sum;
    V[0][ti][tj] = ti == tj ? 1.0 : 0.0;
  }
  __syncthreads();
  if (LOOP && sweep == 0) {
    double fro2 = 0.0;
    for (int i = 0; i < 16; ++i) fro2 += S[0][i][i];
    tiny = 1e-28 * m * fro2;
  }

  // 2. one sweep over the 120 pairs of the 16 rows: 15 rounds of 8 disjoint rotations.  Eight threads work
  // out the rotations of a round (new_x = co[x] old_x + si[x] old_partner), then the 256 solver threads
  // update their elements of S and V; the other waves only keep the barriers company.
  __shared__ double co[16], si[16];
  int cur = 0;
  for (int s = 0; s < 15; ++s) {
    if (tid < 8) {
      const int x = tid == 0 ? 15 : (s + tid) % 15, y = tid == 0 ? s : (s - tid + 15) % 15;
      const int p = x < y ? x : y, q = x < y ? y : x;
      const double a = S[cur][p][p], b = S[cur][q][q], c = S[cur][p][q];
      double cs = 1.0, sn = 0.0;
      if (a > tiny && b > tiny && fabs(c) > tol * sqrt(a * b)) {
        const double zeta = (b - a) / (2.0 * c);
        const double t = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
        cs = 1.0 / sqrt(1.0 + t * t);
        sn = cs * t;
        atomicAdd(&n_rot, 1);
      }
      co[p] = cs; si[p] = -sn;                            // row p: cs p - sn q
      co[q] = cs; si[q] = sn;                             // row q: sn p + cs q
    }
    __syncthreads();
    if (solver) {
      const int pi = ti == 15 ? s : (ti == s ? 15 : (2 * s - ti + 30) % 15);
      const int pj = tj == 15 ? s : (tj == s ? 15 : (2 * s - tj + 30) % 15);
      const double ci = co[ti], zi = si[ti], cj = co[tj], zj = si[tj];
      const double snew = ci * (cj * S[cur][ti][tj] + zj * S[cur][ti][pj]) + zi * (cj * S[cur][pi][tj] + zj * S[cur][pi][pj]);
      const double vnew = cj * V[cur][ti][tj] + zj * V[cur][ti][pj];
      S[cur ^ 1][ti][tj] = snew;
      V[cur ^ 1][ti][tj] = vnew;
    }
    __syncthreads();
    cur ^= 1;
  }
  if (n_rot == 0) {                                     // uniform: read after the barrier
    if (LOOP && tid == 0) *rotations = sweep + 1;
    return;
  }
  if (!LOOP && tid == 0) atomicAdd(rotations, n_rot);

  // 3. rows <- V^T R, 16 columns at a time: A[r][k] = V[k][r], B[k][n] = R[k][c0 + n]
  double va[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) va[kk] = V[cur][4 * kk + lq][lr];
  for (int ch = wave; ch < chunks; ch += NW) {
    const int c = ch * 16 + lr;
    double xb[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int grow = row_of(4 * kk + lq);
      xb[kk] = (grow < m && c < len) ? G[(long)grow * len + c] : 0.0;
    }
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[kk], xb[kk], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int grow = row_of(lq + 4 * i);
      if (grow < m && c < len) G[(long)grow * len + c] = acc[i];
    }
  }
  if (!LOOP) return;
  __threadfence_block();
  __syncthreads();                                      // the rows are whole; n_rot has been read
  }
}

// norms2[row] = squared norm of row `row` of G [m, len]
__global__ __launch_bounds__(256) void row_norms_kernel(const double* G, int len, double* norms2) {
  __shared__ double red[4][3];
  const double* g = G + (long)blockIdx.x * len;
  double a = 0.0, b = 0.0, c = 0.0;
  for (int j = threadIdx.x; j < len; j += 256) a += g[j] * g[j];
  block_sum3(a, b, c, red);
  if (threadIdx.x == 0) norms2[blockIdx.x] = a;
}

// Factor column k = row idx[k] (row k without idx) of G, normalised, signed so that its entry of largest magnitude
// (the first one on ties) is positive: U64 [len, r] fp64 and U [len, r] in the storage type.
template <typename T>
__global__ __launch_bounds__(256) void extract_factor_kernel(const double* G, int len, const int* idx, const double* norms2,
                                                             int r, double* U64, T* U) {
  __shared__ double best_v[256];
  __shared__ int best_j[256];
  const int k = blockIdx.x;
  const int src = idx ? idx[k] : k;
  const double* g = G + (long)src * len;
  double bv = -1.0;
  int bj = 0x7fffffff;
  for (int j = threadIdx.x; j < len; j += 256) {
    const double v = fabs(g[j]);
    if (v > bv) { bv = v; bj = j; }                     // j ascending: the first maximum of this thread
  }
  best_v[threadIdx.x] = bv;
  best_j[threadIdx.x] = bj;
  __syncthreads();
  for (int sft = 128; sft > 0; sft >>= 1) {
    if ((int)threadIdx.x < sft) {
      const double ov = best_v[threadIdx.x + sft];
      const int oj = best_j[threadIdx.x + sft];
      if (ov > best_v[threadIdx.x] || (ov == best_v[threadIdx.x] && oj < best_j[threadIdx.x])) {
        best_v[threadIdx.x] = ov;
        best_j[threadIdx.x] = oj;
      }
    }
    __syncthreads();
  }
  const int at = best_j[0] < len ? best_j[0] : 0;       // (a row without a number has no largest entry; the caller refuses it)
  const double scale = (g[at] < 0.0 ? -1.0 : 1.0) / sqrt(norms2[src]);
  for (int j = threadIdx.x; j < len; j += 256) {
    const double v = scale * g[j];
    U64[(long)j * r + k] = v;
    U[(long)j * r + k] = from_f64<T>(v);
  }
}

inline int blocks_for(long total) { return (int)std::min<long>((total + 255) / 256, 1 << 16); }

hipError_t dgemm(hipStream_t s, int batch, int M, int N, int K, const double* A, long a_m, long a_k, long a_b,
                 const double* B, long b_k, long b_n, long b_b, double* C, long c_m, long c_n, long c_b) {
  DgemmArgs g{A, a_m, a_k, a_b, B, b_k, b_n, b_b, C, c_m, c_n, c_b, M, N, K};
  // small tiles until the large ones fill every compute unit twice
  const long large = (long)((N + 63) / 64) * ((M + 63) / 64) * batch;
  if (large >= 2 * kComputeUnits) hipLaunchKernelGGL(dgemm_kernel<2>, dim3((N + 63) / 64, (M + 63) / 64, batch), dim3(256), 0, s, g);
  else hipLaunchKernelGGL(dgemm_kernel<1>, dim3((N + 31) / 32, (M + 31) / 32, batch), dim3(256), 0, s, g);
  return hipGetLastError();
}

#define CK(expr)                                  \
  do {                                            \
    if ((expr) != hipSuccess) return TUCKER_ATTN_HIP_ERROR; \
  } while (0)

constexpr int kJacobiWaves = 16;

struct JacobiStats {
  int sweeps = 0;
  long launches = 0;
  double ms = 0.0;
  double bytes = 0.0;
};

// The second half of an iteration: rows of G ordered by norm, the r longest -> U64 / U; synchronises the stream.
// (Rotations keep the sum of the squared norms, so the threshold is the one of the iteration.)
template <typename T>
int order_and_extract(hipStream_t s, const double* G, int m, int r, double* norms2, int* idx, double* U64, T* U, double* sv) {
  std::vector<double> h(m);
  hipLaunchKernelGGL(row_norms_kernel, dim3(m), dim3(256), 0, s, G, m, norms2);
  CK(hipGetLastError());
  CK(hipMemcpyAsync(h.data(), norms2, sizeof(double) * m, hipMemcpyDeviceToHost, s));
  CK(hipStreamSynchronize(s));
  const double tiny = 1e-28 * m * std::accumulate(h.begin(), h.end(), 0.0);
  std::vector<int> order(m);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return h[x] > h[y]; });
  if (sv)
    for (int k = 0; k < m; ++k) sv[k] = std::sqrt(std::sqrt(h[order[k]]));   // row norm = eigenvalue = sigma^2
  if (!(h[order[r - 1]] > 1e8 * tiny) || !(h[order[r - 1]] > 0.0)) return TUCKER_ATTN_UNSUPPORTED_SHAPE;
  CK(hipMemcpyAsync(idx, order.data(), sizeof(int) * r, hipMemcpyHostToDevice, s));
  CK(hipStreamSynchronize(s));                          // `order` is pageable host memory
  hipLaunchKernelGGL((extract_factor_kernel<T>), dim3(r), dim3(256), 0, s, G, m, idx, norms2, r, U64, U);
  CK(hipGetLastError());
  return TUCKER_ATTN_OK;
}

// The head mode (m = heads) where one workgroup holds the matrix: enqueued without a wait, finished behind the d x d
// problems.  counter receives the sweeps, 0 without convergence.
constexpr int kSmallJacobi = 16;
hipError_t enqueue_small_jacobi(hipStream_t s, double* G, int m, int* counter) {
  const double tol = std::max(2e-15, std::sqrt((double)m) * 2.3e-16);
  hipLaunchKernelGGL((jacobi_block_kernel<4, true>), dim3(1), dim3(256), 0, s, G, m, m, 0, tol, 0.0, counter, 60);
  return hipGetLastError();
}
// idx: rows in the order of their norms, largest first (the first of equal ones first); any order where they are no numbers
__global__ __launch_bounds__(64) void small_order_kernel(const double* norms2, int m, int* idx) {
  const int i = threadIdx.x;
  if (i < m) idx[i] = i;
  __syncthreads();
  if (i >= m) return;
  int rank = 0;
  for (int j = 0; j < m; ++j) rank += norms2[j] > norms2[i] || (norms2[j] == norms2[i] && j < i);
  idx[rank] = i;
}
// Enqueues the second half: norms, order, factor.  The host looks at norms2 and counter later (check_small_jacobi).
template <typename T>
hipError_t finish_small_jacobi(hipStream_t s, const double* G, int m, int r, double* norms2, int* idx, double* U64, T* U) {
  hipLaunchKernelGGL(row_norms_kernel, dim3(m), dim3(256), 0, s, G, m, norms2);
  hipLaunchKernelGGL(small_order_kernel, dim3(1), dim3(64), 0, s, norms2, m, idx);
  hipLaunchKernelGGL((extract_factor_kernel<T>), dim3(r), dim3(256), 0, s, G, m, idx, norms2, r, U64, U);
  return hipGetLastError();
}
// what the iteration has to have given, by its norms on the host: as order_and_extract
int check_small_jacobi(const double* norms2, int m, int r, int sweeps, double* sv, JacobiStats* stats) {
  if (stats) stats->sweeps += m > 1 ? sweeps : 0;
  if (sweeps == 0) return TUCKER_ATTN_UNSUPPORTED_SHAPE;
  std::vector<double> h(norms2, norms2 + m);
  const double tiny = 1e-28 * m * std::accumulate(h.begin(), h.end(), 0.0);
  std::stable_sort(h.begin(), h.end(), [](double x, double y) { return x > y; });
  if (sv)
    for (int k = 0; k < m; ++k) sv[k] = std::sqrt(std::sqrt(h[k]));   // row norm = eigenvalue = sigma^2
  return !(h[r - 1] > 1e8 * tiny) || !(h[r - 1] > 0.0) ? TUCKER_ATTN_UNSUPPORTED_SHAPE : TUCKER_ATTN_OK;
}

// Eigenvectors of the symmetric positive semi-definite G [m, m] (destroyed) with the r largest
// eigenvalues -> U64 / U [m, r]; sv (host, nullable) receives the square roots of all
// eigenvalues in decreasing order.  Synchronises the stream.
template <typename T>
int leading_eigenvectors(hipStream_t s, double* G, int m, int r, double* norms2, int* idx, int* counter,
                         double* U64, T* U, double* sv, JacobiStats* stats) {
  std::vector<double> h(m);
  hipLaunchKernelGGL(row_norms_kernel, dim3(m), dim3(256), 0, s, G, m, norms2);
  CK(hipGetLastError());
  CK(hipMemcpyAsync(h.data(), norms2, sizeof(double) * m, hipMemcpyDeviceToHost, s));
  CK(hipStreamSynchronize(s));
  const double fro2 = std::accumulate(h.begin(), h.end(), 0.0);
  const double tiny = 1e-28 * m * fro2;                 // rows below the rounding noise of G's entries
  const double tol = std::max(2e-15, std::sqrt((double)m) * 2.3e-16);
  const int nb = (m + 7) / 8, nbp = nb + (nb & 1), n_steps = nbp - 1;   // rounds of the block tournament
  int rotated = 0;
  hipEvent_t ev[2] = {nullptr, nullptr};
  if (stats) {
    CK(hipEventCreate(&ev[0]));
    if (hipEventCreate(&ev[1]) != hipSuccess) {
      (void)hipEventDestroy(ev[0]);
      return TUCKER_ATTN_HIP_ERROR;
    }
    (void)hipEventRecord(ev[0], s);
  }
  struct EventGuard {
    hipEvent_t* e;
    ~EventGuard() {
      if (e[0]) (void)hipEventDestroy(e[0]);
      if (e[1]) (void)hipEventDestroy(e[1]);
    }
  } guard{ev};
  for (int sweep = 0; sweep < 60 && m > 1; ++sweep) {
    if (stats) {
      ++stats->sweeps;
      stats->launches += n_steps;
      stats->bytes += 16.0 * m * m * n_steps;           // every round reads and writes all rows once
    }
    CK(hipMemsetAsync(counter, 0, sizeof(int), s));
    for (int step = 0; step < n_steps; ++step)
      hipLaunchKernelGGL((jacobi_block_kernel<kJacobiWaves, false>), dim3(nbp / 2), dim3(64 * kJacobiWaves), 0, s, G, m, m, step,
                         tol, tiny, counter, 1);
    CK(hipGetLastError());
    CK(hipMemcpyAsync(&rotated, counter, sizeof(int), hipMemcpyDeviceToHost, s));
    CK(hipStreamSynchronize(s));
    if (rotated == 0) break;
  }
  if (stats) {
    float ms = 0.f;
    CK(hipEventRecord(ev[1], s));
    CK(hipEventSynchronize(ev[1]));
    CK(hipEventElapsedTime(&ms, ev[0], ev[1]));
    stats->ms += ms;
  }
  if (rotated != 0) return TUCKER_ATTN_UNSUPPORTED_SHAPE;   // no convergence within the sweep limit
  return order_and_extract<T>(s, G, m, r, norms2, idx, U64, U, sv);
}

// Polish of nearly orthonormal rows, S = Z Z^T: S <- 1.5 I - 0.5 S in place, err[blockIdx.x] = largest |S - I| of a row
// blockIdx.y: problems, their S r^2 and their err err_stride apart
__global__ __launch_bounds__(256) void newton_schulz_kernel(double* S, int r, double* err, long err_stride) {
  __shared__ double red[4];
  S += (long)blockIdx.y * r * r;
  err += blockIdx.y * err_stride;
  double* row = S + (long)blockIdx.x * r;
  double worst = 0.0;
  for (int j = threadIdx.x; j < r; j += 256) {
    const double one = j == (int)blockIdx.x ? 1.0 : 0.0, off = fabs(row[j] - one);
    worst = off > worst || off != off ? off : worst;    // a NaN stays
    row[j] = 1.5 * one - 0.5 * row[j];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double x = __shfl_xor(worst, o);
    worst = x > worst || x != x ? x : worst;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = worst;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) worst = red[w] > worst || red[w] != red[w] ? red[w] : worst;
    err[blockIdx.x] = worst;
  }
}

// the report of the eigen-problems: a summary of each, then value | resid | err | diagonal | subdiagonal of each
constexpr int kSummary = 8, kReportHead = 4 * kSummary;
constexpr int kFailed = 0, kFro2 = 1, kLeast = 2, kResid = 3, kMissing = 4;   // (kFailed: by the reduction)
// squared Frobenius norm, least of the r eigenvalues, largest residual and largest deviation from orthogonality (a NaN stays)
__global__ __launch_bounds__(256) void eigen_summary_kernel(EigenBatch b, double* report) {
  __shared__ double red[256][4];
  const int p = blockIdx.x, m = b.m, r = b.r[p];
  double fro2 = 0.0, least = INFINITY, resid = 0.0, missing = 0.0;
  auto more = [](double x, double y) { return y > x || y != y ? y : x; };
  auto less = [](double x, double y) { return y < x || y != y ? y : x; };
  for (int k = threadIdx.x; k < m; k += 256) {
    const double on = b.tri[p][k], off = k + 1 < m ? b.tri[p][m + k] : 0.0;
    fro2 += on * on + 2.0 * off * off;
    if (k < r) {
      least = less(least, b.value[p][k]);
      resid = more(resid, b.resid[p][k]);
      missing = more(missing, b.value[p][2l * m + k]);
    }
  }
  double* mine = red[threadIdx.x];
  mine[0] = fro2; mine[1] = least; mine[2] = resid; mine[3] = missing;
  for (int n = 128; n > 0; n >>= 1) {
    __syncthreads();
    if ((int)threadIdx.x < n) {
      const double* other = red[threadIdx.x + n];
      mine[0] += other[0];
      mine[1] = less(mine[1], other[1]);
      mine[2] = more(mine[2], other[2]);
      mine[3] = more(mine[3], other[3]);
    }
  }
  if (threadIdx.x == 0) {
    double* to = report + kSummary * p;
    to[kFro2] = mine[0]; to[kLeast] = mine[1]; to[kResid] = mine[2]; to[kMissing] = mine[3];
  }
}
struct HosvdWs {
  double *A, *B, *T, *GA, *GB, *SA, *SB, *M1[2], *U1[2], *U2[2], *U3[2], *P, *Q, *H, *C, *norms2;
  double *M[4];                                         // Gram matrices: modes 2 and 3 of W, then of W~ (one for all where
                                                        // the problems are solved one by one)
  double *Z[4], *Z2[4], *work[4];                       // eigenvector rows before and behind the polish; scratch
  double* report;                                       // see kReportHead
  double* S;
  int *idx, *counter;
  double* small_norms;                                  // the head mode of both tensors, where it is small
  int* small_idx;
  size_t bytes;
};

// The reduction to tridiagonal form takes the sizes whose vectors fit the LDS (whole conversions: d = 768 6.7 ms
// against 206 ms by the Jacobi iteration, d = 4096 0.36 s against 4.3 s).
bool by_tridiagonal_form(int d) { return d >= kEigenMinSize && d <= kEigenMaxSize; }

HosvdWs carve_hosvd(void* base, int d, int nH, int dH) {
  const size_t n = (size_t)nH * dH, D = d;
  const size_t rmax = std::min<size_t>(D, 512);         // the layer's own rank limit bounds P, Q, H, C
  size_t off = 0;
  auto take = [&](size_t elems, size_t size) {
    void* p = base ? static_cast<char*>(base) + off : nullptr;
    off += (elems * size + 255) / 256 * 256;
    return p;
  };
  HosvdWs w;
  w.A = (double*)take(D * n, 8);
  w.B = (double*)take(D * n, 8);
  w.T = (double*)take(D * n, 8);
  w.GA = (double*)take(n * n, 8);
  w.GB = (double*)take(n * n, 8);
  w.SA = (double*)take(n * dH, 8);
  w.SB = (double*)take(n * dH, 8);
  for (int t = 0; t < 2; ++t) {
    w.M1[t] = (double*)take((size_t)nH * nH, 8);
    w.U1[t] = (double*)take((size_t)nH * nH, 8);
    w.U2[t] = (double*)take(D * rmax, 8);
    w.U3[t] = (double*)take(D * rmax, 8);
  }
  const bool batched = by_tridiagonal_form(d);
  for (int e = 0; e < 4; ++e) {
    w.M[e] = batched || e == 0 ? (double*)take(D * D, 8) : w.M[0];
    w.Z[e] = w.Z2[e] = w.work[e] = nullptr;
    if (!batched) continue;
    w.Z[e] = (double*)take(D * rmax, 8);
    w.Z2[e] = (double*)take(D * rmax, 8);
    w.work[e] = (double*)take(eigen_work_elems(d), 8);
  }
  w.report = batched ? (double*)take(kReportHead + 4 * 5 * D, 8) : nullptr;
  w.S = batched ? (double*)take(4 * rmax * rmax, 8) : nullptr;
  w.P = (double*)take(rmax * n, 8);
  w.Q = (double*)take(rmax * n, 8);
  w.H = (double*)take((size_t)nH * rmax * rmax, 8);
  w.C = (double*)take((size_t)nH * rmax * rmax, 8);
  w.norms2 = (double*)take(D + nH, 8);
  w.idx = (int*)take(D + nH, 4);
  w.counter = (int*)take(64, 4);
  w.small_norms = (double*)take(2 * kSmallJacobi, 8);
  w.small_idx = (int*)take(2 * kSmallJacobi, 4);
  w.bytes = off;
  return w;
}

// Gram matrices of the mode unfoldings of one tensor (A_i B_i^T)_i, A and B [d, n] fp64 in the workspace.
// Per-head dH x dH Gram matrices SA_i = A_i^T A_i, SB_i = B_i^T B_i, which modes 2 and 3 start from:
hipError_t head_products(hipStream_t s, const HosvdWs& w, int d, int nH, int dH) {
  const long n = (long)nH * dH;
  if (hipError_t e = dgemm(s, nH, dH, dH, d, w.A, 1, n, dH, w.A, n, 1, dH, w.SA, dH, 1, (long)dH * dH)) return e;
  return dgemm(s, nH, dH, dH, d, w.B, 1, n, dH, w.B, n, 1, dH, w.SB, dH, 1, (long)dH * dH);
}
// mode 1: <W_i, W_j> from the full Gram matrices of the factors
hipError_t head_mode_gram(hipStream_t s, const HosvdWs& w, int d, int nH, int dH, double* M1) {
  const long n = (long)nH * dH;
  const long ab = w.B - w.A;                            // both factors in one launch
  if (hipError_t e = dgemm(s, 2, (int)n, (int)n, d, w.A, 1, n, ab, w.A, n, 1, ab, w.GA, n, 1, w.GB - w.GA)) return e;
  hipLaunchKernelGGL(head_gram_kernel, dim3(nH, nH), dim3(256), 0, s, w.GA, w.GB, M1, nH, dH);
  return hipGetLastError();
}
hipError_t mode_gram(hipStream_t s, const HosvdWs& w, int d, int nH, int dH, int mode, double* M) {
  const long n = (long)nH * dH;
  // mode 2: sum_i W_i W_i^T = sum_i (A_i SB_i) A_i^T;  mode 3: sum_i W_i^T W_i = sum_i (B_i SA_i) B_i^T
  const double *F = mode == 2 ? w.A : w.B, *S = mode == 2 ? w.SB : w.SA;
  if (hipError_t e = dgemm(s, nH, d, dH, dH, F, n, 1, dH, S, dH, 1, (long)dH * dH, w.T, n, 1, dH)) return e;
  return dgemm(s, 1, d, d, (int)n, w.T, n, 1, 0, F, 1, n, 0, M, d, 1, 0);
}

// one d x d eigen-problem of a conversion
template <typename T> struct EigenJob {
  int tensor, mode;                                     // 0: W, 1: W~; 2 or 3
  int r;
  double* U64;
  T* U;
  double* sv;                                           // host, nullable
  JacobiStats* stats;                                   // nullable
};

// The problems of `jobs` (Gram matrices in w.M[j]) through the reduction to tridiagonal form.  done[j] is left false
// where the vectors are no certified answer (eigenvalues too close for the twisted factorisation); w.M[j] is lost
// either way.  Synchronises the stream.
template <typename T>
int tridiagonal_jobs(hipStream_t s, const HosvdWs& w, int d, const EigenJob<T>* jobs, int n_jobs, const TridiagWay& way, bool* done) {
  EigenBatch b;
  b.n = n_jobs;
  b.m = d;
  const bool timed = jobs[0].stats != nullptr;
  for (int j = 0; j < n_jobs; ++j) {
    done[j] = false;
    b.r[j] = jobs[j].r;
    b.n_values[j] = jobs[j].sv ? d : jobs[j].r;
    b.G[j] = w.M[j];
    b.Z[j] = w.Z[j];
    b.work[j] = w.work[j];
    b.failed[j] = w.report + kSummary * j + kFailed;
    b.value[j] = w.report + kReportHead + 5 * (size_t)d * j;
    b.resid[j] = b.value[j] + d;
    b.tri[j] = b.value[j] + 3 * (size_t)d;
  }
  double *from[4], *to[4];                              // eigenvector rows, before and behind a polish
  for (int j = 0; j < n_jobs; ++j) { from[j] = w.Z[j]; to[j] = w.Z2[j]; }
  struct Events {
    hipEvent_t e[2] = {nullptr, nullptr};
    ~Events() {
      for (hipEvent_t x : e)
        if (x) (void)hipEventDestroy(x);
    }
  } ev;
  if (timed) {
    for (hipEvent_t& x : ev.e) CK(hipEventCreate(&x));
    CK(hipEventRecord(ev.e[0], s));
  }
  bool resident = false;
  CK(launch_tridiag(b, s, ev.e[1], &resident, way));
  CK(launch_tridiag_vectors(b, s));
  // rows of close eigenvalues are orthogonal only to rounding / gap: one Newton-Schulz step Z <- (1.5 I - 0.5 Z Z^T) Z,
  // which squares what is missing and moves no vector by more than its own uncertainty
  // (problems j .. j + n - 1 of one rank together, their rows lie `apart`: a product of 64 rows alone leaves most of the chip idle;
  // four of 64 x 768: 122 us one by one, 31 together)
  const long apart = w.Z[1] - w.Z[0];
  auto polish = [&](int j, int n) -> hipError_t {
    const int r = b.r[j];
    if (hipError_t e = dgemm(s, n, r, r, d, from[j], d, 1, apart, from[j], 1, d, apart, w.S, r, 1, (long)r * r)) return e;
    hipLaunchKernelGGL(newton_schulz_kernel, dim3(r, n), dim3(256), 0, s, w.S, r, b.value[j] + 2 * (size_t)d, 5l * d);
    for (int i = j; i < j + n; ++i) std::swap(from[i], to[i]);
    return dgemm(s, n, r, d, r, w.S, r, 1, (long)r * r, to[j], d, 1, apart, from[j], d, 1, apart);
  };
  for (int j = 0, n; j < n_jobs; j += n) {
    for (n = 1; j + n < n_jobs && b.r[j + n] == b.r[j]; ++n) {}
    CK(polish(j, n));
  }
  hipLaunchKernelGGL(eigen_summary_kernel, dim3(n_jobs), dim3(256), 0, s, b, w.report);
  CK(hipGetLastError());
  bool want_values = false;
  for (int j = 0; j < n_jobs; ++j) want_values = want_values || jobs[j].sv;
  std::vector<double> report(kReportHead + (want_values ? 5 * (size_t)d * n_jobs : 0));
  CK(hipMemcpyAsync(report.data(), w.report, sizeof(double) * report.size(), hipMemcpyDeviceToHost, s));
  CK(hipStreamSynchronize(s));
  if (timed) {
    float ms = 0.f;
    CK(hipEventElapsedTime(&ms, ev.e[0], ev.e[1]));
    const int steps = resident ? 1 : tridiag_steps_of(d);
    if (steps > 0) jobs[0].stats->ms += ms;             // one set of launches for all
    jobs[0].stats->launches += steps;
    // the resident launch reads every matrix and writes its reflectors; step k reads and writes the d - 1 - k rows and
    // columns that remain
    if (resident) jobs[0].stats->bytes += 12.0 * n_jobs * d * d;
    else
      for (int k = 0; k < steps; ++k) jobs[0].stats->bytes += 16.0 * n_jobs * (d - 1. - k) * (d - 1. - k);
  }
  for (int j = 0; j < n_jobs; ++j) {
    const int r = b.r[j];
    const double* sum = report.data() + kSummary * j;
    if (resident && sum[kFailed] != 0.0) continue;
    const double fro2 = sum[kFro2], least = sum[kLeast];
    const double top = std::sqrt(fro2);
    // the rank test of the Jacobi path, on the squared eigenvalue
    if (!(least > 0.0) || !(least * least > 1e8 * 1e-28 * d * fro2)) return TUCKER_ATTN_UNSUPPORTED_SHAPE;
    double missing = sum[kMissing];
    const double resid = sum[kResid];
    // residuals of 2.1e-16 of the norm at most were seen (d = 8 .. 5056, repeated and graded spectra among them), whatever
    // the size: a vector that is further off than the rounding of G explains is no answer
    if (!(resid <= 4e-15 * top) || !(missing <= 1e-3 / r)) continue;
    for (; missing > 1e-8 / r; missing = r * missing * missing) CK(polish(j, 1));   // rare: very close eigenvalues
    if (jobs[j].sv) {
      const double* rep = report.data() + kReportHead + 5 * (size_t)d * j;
      std::vector<double> value(rep, rep + d);
      std::sort(value.begin(), value.end(), [](double x, double y) { return x > y; });
      for (int k = 0; k < d; ++k) jobs[j].sv[k] = std::sqrt(std::max(value[k], 0.0));
    }
    hipLaunchKernelGGL(row_norms_kernel, dim3(r), dim3(256), 0, s, from[j], d, w.norms2);
    hipLaunchKernelGGL((extract_factor_kernel<T>), dim3(r), dim3(256), 0, s, from[j], d, nullptr, w.norms2, r, jobs[j].U64, jobs[j].U);
    CK(hipGetLastError());
    done[j] = true;
  }
  return TUCKER_ATTN_OK;
}

// core: C[a] = sum_i U1[i][a] (U2^T A_i)(U3^T B_i)^T
template <typename T>
int core_of(hipStream_t s, const HosvdWs& w, int d, int nH, int dH, int r1, int r2, int r3, const double* U1, const double* U2,
            const double* U3, T* C) {
  const long n = (long)nH * dH;
  if (r2 == r3) {                                       // both in one launch
    CK(dgemm(s, 2, r2, (int)n, d, U2, 1, r2, U3 - U2, w.A, n, 1, w.B - w.A, w.P, n, 1, w.Q - w.P));
  } else {
    CK(dgemm(s, 1, r2, (int)n, d, U2, 1, r2, 0, w.A, n, 1, 0, w.P, n, 1, 0));
    CK(dgemm(s, 1, r3, (int)n, d, U3, 1, r3, 0, w.B, n, 1, 0, w.Q, n, 1, 0));
  }
  CK(dgemm(s, nH, r2, r3, dH, w.P, n, 1, dH, w.Q, 1, n, dH, w.H, r3, 1, (long)r2 * r3));
  CK(dgemm(s, 1, r1, r2 * r3, nH, U1, 1, r1, 0, w.H, (long)r2 * r3, 1, 0, w.C, (long)r2 * r3, 1, 0));
  const long total = (long)r1 * r2 * r3;
  hipLaunchKernelGGL((from_f64_kernel<T>), dim3(blocks_for(total)), dim3(256), 0, s, w.C, C, total);
  CK(hipGetLastError());
  return TUCKER_ATTN_OK;
}

template <typename T>
int from_gqa(int d, int nH, int dH, int nG, const T* WQ, const T* WK, const T* WV, const T* WO,
             const tucker_convert_weights_out& o, hipStream_t s) {
  const long n = (long)nH * dH, g = (long)nG * dH;
  const long core = (long)nH * n * g;
  hipLaunchKernelGGL((selector_core_kernel<T>), dim3(blocks_for(core)), dim3(256), 0, s, (T*)o.C, nH, dH, nG);
  hipLaunchKernelGGL((selector_core_kernel<T>), dim3(blocks_for(core)), dim3(256), 0, s, (T*)o.Ct, nH, dH, nG);
  hipLaunchKernelGGL((identity_kernel<T>), dim3(blocks_for((long)nH * nH)), dim3(256), 0, s, (T*)o.U1, nH);
  hipLaunchKernelGGL((identity_kernel<T>), dim3(blocks_for((long)nH * nH)), dim3(256), 0, s, (T*)o.Ut1, nH);
  hipLaunchKernelGGL((transpose_copy_kernel<T>), dim3((d + 31) / 32, (int)((n + 31) / 32)), dim3(256), 0, s, WO, (T*)o.Ut2, (int)n, d);
  CK(hipGetLastError());
  CK(hipMemcpyAsync(o.U2, WQ, sizeof(T) * d * n, hipMemcpyDeviceToDevice, s));
  CK(hipMemcpyAsync(o.U3, WK, sizeof(T) * d * g, hipMemcpyDeviceToDevice, s));
  CK(hipMemcpyAsync(o.Ut3, WV, sizeof(T) * d * g, hipMemcpyDeviceToDevice, s));
  return TUCKER_ATTN_OK;
}

template <typename T>
int from_mla(int d, int nH, int dH, int dcQ, int dcK, const T* WDQ, const T* WUQ, const T* WDKV, const T* WUK,
             const T* WDV, const T* WUV, const T* WO, const tucker_convert_weights_out& o, hipStream_t s) {
  const long n = (long)nH * dH;
  hipLaunchKernelGGL((mla_core_kernel<T>), dim3(blocks_for((long)nH * dcQ * dcK)), dim3(256), 0, s, WUQ, WUK, (T*)o.C, nH, dH, dcQ, dcK);
  hipLaunchKernelGGL((mla_post_core_kernel<T>), dim3(blocks_for((long)nH * n * dcK)), dim3(256), 0, s, WUV, (T*)o.Ct, nH, dH, dcK);
  hipLaunchKernelGGL((identity_kernel<T>), dim3(blocks_for((long)nH * nH)), dim3(256), 0, s, (T*)o.U1, nH);
  hipLaunchKernelGGL((identity_kernel<T>), dim3(blocks_for((long)nH * nH)), dim3(256), 0, s, (T*)o.Ut1, nH);
  hipLaunchKernelGGL((transpose_copy_kernel<T>), dim3((d + 31) / 32, (int)((n + 31) / 32)), dim3(256), 0, s, WO, (T*)o.Ut2, (int)n, d);
  CK(hipGetLastError());
  CK(hipMemcpyAsync(o.U2, WDQ, sizeof(T) * d * dcQ, hipMemcpyDeviceToDevice, s));
  CK(hipMemcpyAsync(o.U3, WDKV, sizeof(T) * d * dcK, hipMemcpyDeviceToDevice, s));
  if (WDV) CK(hipMemcpyAsync(o.Ut3, WDV, sizeof(T) * d * dcK, hipMemcpyDeviceToDevice, s));
  return TUCKER_ATTN_OK;
}

template <typename T>
int from_mha_hosvd(int d, int nH, int dH, const T* WQ, const T* WK, const T* WV, const T* WO, int r1, int r2, int r3,
                   int rt1, int rt2, int rt3, bool shared, const tucker_convert_weights_out& o, double* sv,
                   tucker_convert_hosvd_info* info, void* workspace, hipStream_t s, const TridiagWay& way) {
  JacobiStats stats[6];
  struct Report {                                       // filled on every return path
    tucker_convert_hosvd_info* info;
    const JacobiStats* st;
    ~Report() {
      if (!info) return;
      info->jacobi_launches = 0;
      info->jacobi_bytes = 0.0;
      info->jacobi_ms = 0.0;
      for (int k = 0; k < 6; ++k) {
        info->sweeps[k] = st[k].sweeps;
        if (k % 3 != 0) {
          info->jacobi_launches += st[k].launches;
          info->jacobi_ms += st[k].ms;
          info->jacobi_bytes += st[k].bytes;
        }
      }
    }
  } report{info, stats};
  const HosvdWs w = carve_hosvd(workspace, d, nH, dH);
  const long n = (long)nH * dH;
  const int cb = blocks_for((long)d * n);
  // the two tensors: A = WQ, B = WK before the softmax; A = WO^T (output index first), B = WV behind it
  auto load = [&](int t) -> hipError_t {
    hipLaunchKernelGGL((to_f64_kernel<T>), dim3(cb), dim3(256), 0, s, t ? WO : WQ, t ? 1 : n, t ? (long)d : 1, w.A, d, (int)n);
    hipLaunchKernelGGL((to_f64_kernel<T>), dim3(cb), dim3(256), 0, s, t ? WV : WK, n, 1, w.B, d, (int)n);
    return hipGetLastError();
  };
  EigenJob<T> jobs[4];
  int n_jobs = 0;
  for (int t = 0; t < 2; ++t)
    for (int mode = 2; mode <= 3; ++mode) {
      const long at = t * (nH + 2l * d) + nH + (mode - 2) * (long)d;
      if (t && mode == 3 && shared) {
        if (sv) std::fill(sv + at, sv + at + d, 0.0);
        continue;
      }
      jobs[n_jobs++] = EigenJob<T>{t, mode, t ? (mode == 2 ? rt2 : rt3) : (mode == 2 ? r2 : r3), mode == 2 ? w.U2[t] : w.U3[t],
                                   (T*)(t ? (mode == 2 ? o.Ut2 : o.Ut3) : (mode == 2 ? o.U2 : o.U3)), sv ? sv + at : nullptr,
                                   info ? &stats[3 * t + mode - 1] : nullptr};
    }
  const bool tridiagonal = by_tridiagonal_form(d);
  for (int t = 0; t < 2; ++t) {
    CK(load(t));
    CK(head_products(s, w, d, nH, dH));
    CK(head_mode_gram(s, w, d, nH, dH, w.M1[t]));
    if (nH <= kSmallJacobi) {
      CK(enqueue_small_jacobi(s, w.M1[t], nH, w.counter + 1 + t));
    } else {
      const int st = leading_eigenvectors<T>(s, w.M1[t], nH, t ? rt1 : r1, w.norms2, w.idx, w.counter, w.U1[t],
                                             (T*)(t ? o.Ut1 : o.U1), sv ? sv + t * (nH + 2l * d) : nullptr,
                                             info ? &stats[3 * t] : nullptr);
      if (st != TUCKER_ATTN_OK) return st;
    }
    for (int j = 0; j < n_jobs; ++j)
      if (tridiagonal && jobs[j].tensor == t) CK(mode_gram(s, w, d, nH, dH, jobs[j].mode, w.M[j]));
  }
  // A problem that the reduction to tridiagonal form cannot certify and every other size go through the Jacobi iteration, one
  // Gram matrix at a time, formed in front of it.
  bool done[4] = {false, false, false, false};
  if (tridiagonal)
    if (const int st = tridiagonal_jobs<T>(s, w, d, jobs, n_jobs, way, done); st != TUCKER_ATTN_OK) return st;
  int loaded = 1;
  for (int j = n_jobs - 1; j >= 0; --j) {
    if (done[j]) continue;
    if (loaded != jobs[j].tensor) {
      CK(load(jobs[j].tensor));
      CK(head_products(s, w, d, nH, dH));
    }
    loaded = jobs[j].tensor;
    CK(mode_gram(s, w, d, nH, dH, jobs[j].mode, w.M[j]));
    const int st = leading_eigenvectors<T>(s, w.M[j], d, jobs[j].r, w.norms2, w.idx, w.counter, jobs[j].U64, jobs[j].U,
                                           jobs[j].sv, jobs[j].stats);
    if (st != TUCKER_ATTN_OK) return st;
  }
  for (int t = 0; t < 2 && nH <= kSmallJacobi; ++t)
    CK(finish_small_jacobi<T>(s, w.M1[t], nH, t ? rt1 : r1, w.small_norms + t * kSmallJacobi, w.small_idx + t * kSmallJacobi, w.U1[t],
                              (T*)(t ? o.Ut1 : o.U1)));
  for (int t = 1; t >= 0; --t) {
    if (loaded != t) CK(load(t));
    loaded = t;
    const int st = core_of<T>(s, w, d, nH, dH, t ? rt1 : r1, t ? rt2 : r2, t ? rt3 : r3, w.U1[t], w.U2[t],
                              t && !shared ? w.U3[1] : w.U3[0], (T*)(t ? o.Ct : o.C));
    if (st != TUCKER_ATTN_OK) return st;
  }
  if (nH > kSmallJacobi) {
    CK(hipStreamSynchronize(s));
    return TUCKER_ATTN_OK;
  }
  double small[2 * kSmallJacobi];                       // the head mode's norms, sweeps behind them
  int sweeps[2];
  CK(hipMemcpyAsync(small, w.small_norms, sizeof(small), hipMemcpyDeviceToHost, s));
  CK(hipMemcpyAsync(sweeps, w.counter + 1, sizeof(sweeps), hipMemcpyDeviceToHost, s));
  CK(hipStreamSynchronize(s));
  for (int t = 0; t < 2; ++t)
    if (const int st = check_small_jacobi(small + t * kSmallJacobi, nH, t ? rt1 : r1, sweeps[t], sv ? sv + t * (nH + 2l * d) : nullptr,
                                          info ? &stats[3 * t] : nullptr);
        st != TUCKER_ATTN_OK)
      return st;
  return TUCKER_ATTN_OK;
}

}  // namespace
}  // namespace ta

extern "C" {

int tucker_convert_from_gqa(int32_t dtype, int32_t d, int32_t nH, int32_t dH, int32_t nG, const void* WQ, const void* WK,
                            const void* WV, const void* WO, const tucker_convert_weights_out* out, void* hip_stream) {
  if (dtype != TUCKER_ATTN_F32 && dtype != TUCKER_ATTN_BF16) return TUCKER_ATTN_INVALID_ARG;
  if (d < 1 || nH < 1 || dH < 1 || nG < 1 || nH % nG != 0) return TUCKER_ATTN_INVALID_ARG;
  if (!WQ || !WK || !WV || !WO || !out) return TUCKER_ATTN_INVALID_ARG;
  if (!out->C || !out->U1 || !out->U2 || !out->U3 || !out->Ct || !out->Ut1 || !out->Ut2 || !out->Ut3)
    return TUCKER_ATTN_INVALID_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (dtype == TUCKER_ATTN_F32)
    return ta::from_gqa<float>(d, nH, dH, nG, (const float*)WQ, (const float*)WK, (const float*)WV, (const float*)WO, *out, s);
  return ta::from_gqa<ta::bf16>(d, nH, dH, nG, (const ta::bf16*)WQ, (const ta::bf16*)WK, (const ta::bf16*)WV,
                                (const ta::bf16*)WO, *out, s);
}

int tucker_convert_from_mla(int32_t dtype, int32_t d, int32_t nH, int32_t dH, int32_t dcQ, int32_t dcK, const void* WDQ,
                            const void* WUQ, const void* WDKV, const void* WUK, const void* WDV, const void* WUV,
                            const void* WO, const tucker_convert_weights_out* out, void* hip_stream) {
  if (dtype != TUCKER_ATTN_F32 && dtype != TUCKER_ATTN_BF16) return TUCKER_ATTN_INVALID_ARG;
  if (d < 1 || nH < 1 || dH < 1 || dcQ < 1 || dcK < 1) return TUCKER_ATTN_INVALID_ARG;
  if (!WDQ || !WUQ || !WDKV || !WUK || !WUV || !WO || !out) return TUCKER_ATTN_INVALID_ARG;
  if (!out->C || !out->U1 || !out->U2 || !out->U3 || !out->Ct || !out->Ut1 || !out->Ut2) return TUCKER_ATTN_INVALID_ARG;
  if (WDV && !out->Ut3) return TUCKER_ATTN_INVALID_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (dtype == TUCKER_ATTN_F32)
    return ta::from_mla<float>(d, nH, dH, dcQ, dcK, (const float*)WDQ, (const float*)WUQ, (const float*)WDKV,
                               (const float*)WUK, (const float*)WDV, (const float*)WUV, (const float*)WO, *out, s);
  return ta::from_mla<ta::bf16>(d, nH, dH, dcQ, dcK, (const ta::bf16*)WDQ, (const ta::bf16*)WUQ, (const ta::bf16*)WDKV,
                                (const ta::bf16*)WUK, (const ta::bf16*)WDV, (const ta::bf16*)WUV, (const ta::bf16*)WO, *out, s);
}

size_t tucker_convert_hosvd_workspace_bytes(int32_t d, int32_t nH, int32_t dH) {
  if (d < 1 || nH < 1 || dH < 1 || d > 8192 || nH > 256 || (long)nH * dH > 8192) return 0;
  return ta::carve_hosvd(nullptr, d, nH, dH).bytes;
}

// tucker_convert_from_mha_hosvd with the way of its reduction stated (TridiagWay), so that tests reach the ways out of it
int tucker_test_from_mha_hosvd(int32_t dtype, int32_t d, int32_t nH, int32_t dH, const void* WQ, const void* WK, const void* WV,
                               const void* WO, int32_t r1, int32_t r2, int32_t r3, int32_t rt1, int32_t rt2, int32_t rt3,
                               int32_t shared_kv, const tucker_convert_weights_out* out, double* singular_values,
                               tucker_convert_hosvd_info* info, void* workspace, size_t workspace_bytes, void* hip_stream,
                               int32_t one_launch, int32_t looks) {
  const ta::TridiagWay way{one_launch != 0, looks};
  if (dtype != TUCKER_ATTN_F32 && dtype != TUCKER_ATTN_BF16) return TUCKER_ATTN_INVALID_ARG;
  if (d < 1 || nH < 1 || dH < 1) return TUCKER_ATTN_INVALID_ARG;
  if (d > 8192 || nH > 256 || (long)nH * dH > 8192) return TUCKER_ATTN_UNSUPPORTED_SHAPE;
  if (r1 < 1 || r2 < 1 || r3 < 1 || rt1 < 1 || rt2 < 1 || rt3 < 1) return TUCKER_ATTN_INVALID_ARG;
  if (r1 > nH || rt1 > nH || r2 > d || r3 > d || rt2 > d || rt3 > d) return TUCKER_ATTN_INVALID_ARG;
  if (r2 > 512 || r3 > 512 || rt2 > 512 || rt3 > 512) return TUCKER_ATTN_UNSUPPORTED_SHAPE;
  if (shared_kv != 0 && shared_kv != 1) return TUCKER_ATTN_INVALID_ARG;
  if (shared_kv && rt3 != r3) return TUCKER_ATTN_INVALID_ARG;
  if (!WQ || !WK || !WV || !WO || !out || !workspace) return TUCKER_ATTN_INVALID_ARG;
  if (!out->C || !out->U1 || !out->U2 || !out->U3 || !out->Ct || !out->Ut1 || !out->Ut2) return TUCKER_ATTN_INVALID_ARG;
  if (!shared_kv && !out->Ut3) return TUCKER_ATTN_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0) return TUCKER_ATTN_INVALID_ARG;
  if (workspace_bytes < tucker_convert_hosvd_workspace_bytes(d, nH, dH)) return TUCKER_ATTN_WORKSPACE_TOO_SMALL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (dtype == TUCKER_ATTN_F32)
    return ta::from_mha_hosvd<float>(d, nH, dH, (const float*)WQ, (const float*)WK, (const float*)WV, (const float*)WO, r1,
                                     r2, r3, rt1, rt2, rt3, shared_kv != 0, *out, singular_values, info, workspace, s, way);
  return ta::from_mha_hosvd<ta::bf16>(d, nH, dH, (const ta::bf16*)WQ, (const ta::bf16*)WK, (const ta::bf16*)WV,
                                      (const ta::bf16*)WO, r1, r2, r3, rt1, rt2, rt3, shared_kv != 0, *out, singular_values,
                                      info, workspace, s, way);
}

int tucker_convert_from_mha_hosvd(int32_t dtype, int32_t d, int32_t nH, int32_t dH, const void* WQ, const void* WK,
                                  const void* WV, const void* WO, int32_t r1, int32_t r2, int32_t r3, int32_t rt1,
                                  int32_t rt2, int32_t rt3, int32_t shared_kv, const tucker_convert_weights_out* out,
                                  double* singular_values, tucker_convert_hosvd_info* info, void* workspace,
                                  size_t workspace_bytes, void* hip_stream) {
  const ta::TridiagWay way;
  return tucker_test_from_mha_hosvd(dtype, d, nH, dH, WQ, WK, WV, WO, r1, r2, r3, rt1, rt2, rt3, shared_kv, out, singular_values,
                                    info, workspace, workspace_bytes, hip_stream, way.one_launch, way.looks);
}

}  // extern "C"
