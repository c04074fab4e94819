// Leading eigenpairs of symmetric matrices in fp64: Householder reduction to tridiagonal form, eigenvalues by
// multisection on Sturm counts, eigenvectors of the tridiagonal matrix from its twisted factorisation, and the
// reflectors applied back.  Up to four matrices of one size go through every launch side by side.
//
// The reduction is a chain of m dependent steps (each needs a product of the whole remaining matrix with a vector
// that the previous step determines), so a step is ONE launch: the rank-two update of step k-1, the column of
// step k and the product with its reflector are fused, every workgroup working out the reflector for itself.
#include "eigen.h"

#include "common.h"
#include "params.h"

namespace ta {
namespace {

// layout of a problem's work array, in vectors of m doubles
constexpr int kTau = 0, kV = 1, kY = 3;                 // kV, kY: two vectors each, used in turn

// x of the lane that the DPP control CTRL names
template <int CTRL> __device__ __forceinline__ double dpp(double x) {
  const long b = __builtin_bit_cast(long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (long)(((unsigned long)hi << 32) | lo));
}
// sum over a wave, every lane receives it (register moves: with LDS permutes a step of four 768 x 768 matrices takes 7.1 us, not 6.4)
__device__ __forceinline__ double wave_sum(double x) {
  x += dpp<0xb1>(x);                                    // lane ^ 1, lane ^ 2
  x += dpp<0x4e>(x);
  x += dpp<0x141>(x);                                   // mirrored in 8, in 16
  x += dpp<0x140>(x);
  {
    const long b = __builtin_bit_cast(long, x);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    x = __builtin_bit_cast(double, (long)(((unsigned long)hi[0] << 32) | lo[0])) +
        __builtin_bit_cast(double, (long)(((unsigned long)hi[1] << 32) | lo[1]));
  }
  const long b = __builtin_bit_cast(long, x);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return __builtin_bit_cast(double, (long)(((unsigned long)hi[0] << 32) | lo[0])) +
         __builtin_bit_cast(double, (long)(((unsigned long)hi[1] << 32) | lo[1]));
}
// sum over a workgroup of NW waves; every thread receives it.  `red` [NW] is not shared with the next call.
template <int NW> __device__ __forceinline__ double block_sum(double x, double* red) {
  x = wave_sum(x);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) s += red[w];
  return s;
}

// Step k of the reduction.  With v = the reflector of step k-1 (v_k = 1, zero before k), y = A v and
// w = tau (y - tau/2 (v.y) v), the remaining matrix becomes A - v w^T - w v^T; its row k gives the diagonal and
// subdiagonal entry k and the next reflector u, and the launch leaves A u for step k+1.
// Workgroup = 16 waves, RW rows each.  The grid stays the same for all steps; workgroups above the
// remaining matrix return, the last one stores what all work out.  Row k is read by every workgroup and
// written by none; row k-1, read by none any more, receives v for the way back.
// NC > 0: a row fits NC chunks of 64 lanes and is loaded before the reflector is known.
// Small matrices are bound by the latency of a launch, its loads and its two workgroup sums (four of 768: 9.6 us for
// the first steps, 6.3 for the last before the tail), large ones by memory (four of 4096: 78 us a step, 4.6 TB/s).
template <int NC, int RW>
__global__ __launch_bounds__(1024) void tridiag_step_kernel(EigenBatch b, int k) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ double red[2][16];
  const int m = b.m, p = blockIdx.y;
  double* A = b.G[p];
  double* work = b.work[p];
  double* v = reinterpret_cast<double*>(smem_raw);
  double* w = v + m;
  double* u = w + m;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.x * 16 * RW + wave;                 // this wave's rows: row0 + 16 t
  const int c0 = k + 1;                                         // first column that is still needed
  const bool writer = blockIdx.x == gridDim.x - 1;
  if (!writer && (int)(blockIdx.x + 1) * 16 * RW <= c0) return;

  double x[NC > 0 ? NC : 1];
  if constexpr (NC > 0) {
    if (row0 >= c0 && row0 < m) {
#pragma unroll
      for (int t = 0; t < NC; ++t) {
        const int j = c0 + lane + 64 * t;
        x[t] = j < m ? A[(long)row0 * m + j] : 0.0;
      }
    }
  }
  const double* vp = work + (long)(kV + ((k + 1) & 1)) * m;
  const double* yp = work + (long)(kY + ((k + 1) & 1)) * m;
  const double tau = k > 0 ? work[(long)kTau * m + k - 1] : 0.0;
  const double yk = k > 0 ? yp[k] : 0.0;                        // v_k = 1
  double dot = 0.0;
  for (int i = k + tid; i < m; i += 1024) {
    const double vi = k > 0 ? vp[i] : 0.0, yi = k > 0 ? yp[i] : 0.0;
    v[i] = vi;
    w[i] = yi;
    u[i] = A[(long)k * m + i];
    dot += vi * yi;
  }
  const double half = 0.5 * tau * block_sum<16>(dot, red[0]);
  const double wk = tau * (yk - half);
  double tail = 0.0;
  for (int i = k + tid; i < m; i += 1024) {
    const double vi = v[i], wi = tau * (w[i] - half * vi);
    const double c = u[i] - vi * wk - wi;                       // row k of the updated matrix (v_k = 1)
    w[i] = wi;
    u[i] = c;
    if (i > c0) tail += c * c;
    if (i == k && writer) b.tri[p][k] = c;
  }
  tail = block_sum<16>(tail, red[1]);
  if (c0 >= m) return;                                          // the last diagonal entry (v is the unit vector by then)
  const double x0 = u[c0];
  double beta = x0, tau_k = 0.0, scale = 0.0;
  if (tail > 0.0) {
    beta = -copysign(sqrt(x0 * x0 + tail), x0);
    tau_k = (beta - x0) / beta;
    scale = 1.0 / (x0 - beta);
  }
  __syncthreads();                                              // x0 has been read
  for (int i = c0 + tid; i < m; i += 1024) u[i] = i == c0 ? 1.0 : u[i] * scale;
  __syncthreads();
  if (writer) {
    if (tid == 0) {
      b.tri[p][m + k] = beta;
      work[(long)kTau * m + k] = tau_k;
    }
    double* vn = work + (long)(kV + (k & 1)) * m;
    for (int i = c0 + tid; i < m; i += 1024) vn[i] = u[i];
    if (k > 0)
      for (int i = k + tid; i < m; i += 1024) A[(long)(k - 1) * m + i] = v[i];
  }
  double* yn = work + (long)(kY + (k & 1)) * m;
#pragma unroll 1
  for (int t = 0; t < RW; ++t) {
    const int row = row0 + 16 * t;
    if (row < c0 || row >= m) continue;
    const double vi = v[row], wi = w[row];
    double* Ar = A + (long)row * m;
    double sum = 0.0;
    if constexpr (NC > 0) {
      static_assert(NC == 0 || RW == 1, "one row in registers");
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int j = c0 + lane + 64 * c;
        if (j < m) {
          const double z = x[c] - vi * w[j] - wi * v[j];
          Ar[j] = z;
          sum += z * u[j];
        }
      }
    } else {
      // eight loads in flight per lane
      for (int j0 = c0 + lane; j0 < m; j0 += 512) {
        double q[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) q[c] = j0 + 64 * c < m ? Ar[j0 + 64 * c] : 0.0;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int j = j0 + 64 * c;
          if (j < m) {
            const double z = q[c] - vi * w[j] - wi * v[j];
            Ar[j] = z;
            sum += z * u[j];
          }
        }
      }
    }
    sum = wave_sum(sum);
    if (lane == 0) yn[row] = sum;
  }
}

// interval that holds every eigenvalue, from Gershgorin's circles of the tridiagonal matrix (all lanes alike)
__device__ __forceinline__ void spectrum_bounds(const double* d, const double* e, int m, int lane, double& lo, double& hi) {
  lo = INFINITY;
  hi = -INFINITY;
  for (int i = lane; i < m; i += 64) {
    const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < m ? fabs(e[i]) : 0.0);
    lo = fmin(lo, d[i] - r);
    hi = fmax(hi, d[i] + r);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o));
    hi = fmax(hi, __shfl_xor(hi, o));
  }
  const double slack = 4e-16 * m * fmax(fabs(lo), fabs(hi)) + 1e-300;
  lo -= slack;
  hi += slack;
}
constexpr double kPivot = 1e-290;                       // smallest pivot magnitude, relative to max(1, e^2)

// Eigenvalue number 4 blockIdx.x + wave of a problem, counted from the largest: the 64 lanes of a wave count the
// eigenvalues below 64 points of the current interval, which shrinks 65-fold per round (10 rounds: below the
// rounding of the largest eigenvalue).  The count is that of the sign changes in the sequence of leading minors
// p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}: a serial chain of one fused multiply-add a row, where the pivots p_i / p_{i-1} would take
// a reciprocal (four problems of 768, 128 values each: 312 us by pivots, 165 so).  With the matrix scaled to a norm of 1 to 2 and
// an off-diagonal of less than 1e-20 taken as 1e-20 (far below the rounding of the diagonal), eight rows change the larger of two
// neighbouring minors by less than 2^20 upwards and 1e-205 downwards: a common power of two is taken out of both every eight rows,
// and what underflows next to the other is a zero minor, whose sign does not matter.
__global__ __launch_bounds__(256) void tridiag_values_kernel(EigenBatch b) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int m = b.m, p = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double* d = b.tri[p];
  const double* e = b.tri[p] + m;
  double* pd = reinterpret_cast<double*>(smem_raw);     // (d_i, e_{i-1}^2) pairs, scaled
  double lo, hi;
  spectrum_bounds(d, e, m, lane, lo, hi);
  const int shift = -ilogb(fmax(fabs(lo), fabs(hi)));   // (the bounds are never zero)
  for (int i = threadIdx.x; i < m; i += 256) {
    const double o = i > 0 ? ldexp(e[i - 1], shift) : 0.0;
    pd[2 * i] = ldexp(d[i], shift);
    pd[2 * i + 1] = fmax(o * o, 1e-40);
  }
  __syncthreads();
  const int idx = blockIdx.x * 4 + wave;
  if (idx >= b.n_values[p]) return;
  lo = ldexp(lo, shift);
  hi = ldexp(hi, shift);
  const int below = m - idx;                            // count at and above the eigenvalue wanted
  for (int round = 0; round < 10; ++round) {
    const double x = lo + (hi - lo) * ((lane + 1) / 65.0);
    // p1, p0: minors i and i-1.  A zero minor has either sign: the next one is -e^2 times the one before, so that the two
    // steps count one change together.
    double p1 = 1.0, p0 = 0.0;
    int cnt = 0, i = 0;
    auto high = [](double v) { return (unsigned)(__builtin_bit_cast(unsigned long, v) >> 32); };
    auto row = [&](int at) {
      const double q = fma(pd[2 * at] - x, p1, -(pd[2 * at + 1] * p0));
      cnt += (int)((high(q) ^ high(p1)) >> 31);
      p0 = p1;
      p1 = q;
    };
    for (; i + 8 <= m; i += 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u) row(i + u);
      const int e2 = -ilogb(fmax(fabs(p0), fabs(p1)));  // (not both are zero)
      p0 = ldexp(p0, e2);
      p1 = ldexp(p1, e2);
    }
    for (; i < m; ++i) row(i);
    const unsigned long long up = __builtin_amdgcn_ballot_w64(cnt >= below);
    const int f = up == 0ull ? 64 : __builtin_ctzll(up);
    const double nhi = f < 64 ? __shfl(x, f & 63) : hi;
    const double nlo = f > 0 ? __shfl(x, (f - 1) & 63) : lo;
    lo = nlo;
    hi = nhi;
  }
  if (lane == 0) b.value[p][idx] = ldexp(0.5 * (lo + hi), -shift);
}

// Unit eigenvector of the tridiagonal matrix for its eigenvalue blockIdx.x: pivots of the factorisations from the top
// (D+) and from the bottom (D-) are worked out by two lanes side by side; the vector starts from 1 where
// |D+ + D- - (d - lambda)| is least and follows the factors both ways.  That least value over the norm is the
// residual.  Row blockIdx.x of Z [r, m] receives the vector.
__global__ __launch_bounds__(64) void tridiag_vector_kernel(EigenBatch b) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int m = b.m, p = blockIdx.y, idx = blockIdx.x, lane = threadIdx.x;
  if (idx >= b.r[p]) return;
  double* d = reinterpret_cast<double*>(smem_raw);
  double* e = d + m;                                    // e[m-1] unused
  double* up = e + m;                                   // D+, then the factor from i+1 to i
  double* dn = up + m;                                  // D-, then the factor from i-1 to i
  const double lam = b.value[p][idx];
  double e2max = 0.0;
  for (int i = lane; i < m; i += 64) {
    d[i] = b.tri[p][i] - lam;
    const double o = i + 1 < m ? b.tri[p][m + i] : 0.0;
    e[i] = o;
    e2max = fmax(e2max, o * o);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) e2max = fmax(e2max, __shfl_xor(e2max, o));
  const double pivot = kPivot * fmax(1.0, e2max);
  __syncthreads();
  if (lane < 2) {
    double* out = lane == 0 ? up : dn;
    double q = 1.0;
#pragma unroll 4
    for (int i = 0; i < m; ++i) {
      const int at = lane == 0 ? i : m - 1 - i, prev = lane == 0 ? i - 1 : m - 1 - i;
      const double o = i > 0 ? e[prev] : 0.0;
      q = d[at] - o * o / q;
      if (fabs(q) < pivot) q = -pivot;
      out[at] = q;
    }
  }
  __syncthreads();
  double best = INFINITY;
  int at = 0;
  for (int i = lane; i < m; i += 64) {
    const double g = fabs(up[i] + dn[i] - d[i]);
    if (g < best) { best = g; at = i; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o);
    const int oa = __shfl_xor(at, o);
    if (ob < best || (ob == best && oa < at)) { best = ob; at = oa; }
  }
  // factors: z_i = up[i] z_{i+1} above the twist, z_i = dn[i] z_{i-1} below it
  for (int i = lane; i < m; i += 64) {
    const double f = i < at ? -e[i] / up[i] : 0.0;
    const double g = i > at ? -e[i - 1] / dn[i] : 0.0;
    up[i] = f;
    dn[i] = g;
  }
  __syncthreads();
  if (lane < 2) {
    double z = 1.0;
    const int n = lane == 0 ? at : m - 1 - at;
    if (lane == 0) d[at] = 1.0;
#pragma unroll 4
    for (int i = 1; i <= n; ++i) {
      const int j = lane == 0 ? at - i : at + i;
      z *= lane == 0 ? up[j] : dn[j];
      d[j] = z;
    }
  }
  __syncthreads();
  double n2 = 0.0;
  for (int i = lane; i < m; i += 64) n2 += d[i] * d[i];
  n2 = wave_sum(n2);
  const double inv = 1.0 / sqrt(n2);
  double* z = b.Z[p] + (long)idx * m;
  for (int i = lane; i < m; i += 64) z[i] = d[i] * inv;
  if (lane == 0) b.resid[p][idx] = best * inv;
}

// Row blockIdx.x of Z times the reflectors, last to first: z -= tau_k v_k (v_k . z), v_k in row k of G from column
// k+1 on.  NW waves hold the row, NC elements per thread; PF reflectors are in flight.
template <int NW, int NC, int PF>
__global__ __launch_bounds__(64 * NW) void apply_reflectors_kernel(EigenBatch b) {
  __shared__ double red[2][NW];
  const int m = b.m, p = blockIdx.y, tid = threadIdx.x;
  if ((int)blockIdx.x >= b.r[p]) return;
  const double* G = b.G[p];
  const double* tau = b.work[p] + (long)kTau * m;
  double* zr = b.Z[p] + (long)blockIdx.x * m;
  double z[NC], v[PF][NC], t[PF];
  auto load = [&](double (&q)[NC], double& tk, int k) {
    tk = k >= 0 ? tau[k] : 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int i = tid + 64 * NW * c;
      q[c] = k >= 0 && i > k && i < m ? G[(long)k * m + i] : 0.0;
    }
  };
#pragma unroll
  for (int c = 0; c < NC; ++c) z[c] = tid + 64 * NW * c < m ? zr[tid + 64 * NW * c] : 0.0;
  const int last = m - 3;                               // the reflectors of the last two steps are the identity
#pragma unroll
  for (int f = 0; f < PF; ++f) load(v[f], t[f], last - f);
  for (int k = last; k >= 0; k -= PF) {
#pragma unroll
    for (int f = 0; f < PF; ++f) {                      // past the first reflector: zeros
      double dot = 0.0;
#pragma unroll
      for (int c = 0; c < NC; ++c) dot += v[f][c] * z[c];
      if constexpr (NW == 1) dot = wave_sum(dot);
      else dot = block_sum<NW>(dot, red[f & 1]);
      dot *= t[f];
#pragma unroll
      for (int c = 0; c < NC; ++c) z[c] -= dot * v[f][c];
      load(v[f], t[f], k - f - PF);
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (tid + 64 * NW * c < m) zr[tid + 64 * NW * c] = z[c];
}

// The last kTail steps (k0 = m - kTail, or all of them with k0 = 0 in a smaller matrix) in one launch, one workgroup per
// problem: wave w holds the rows k0 + w, k0 + w + 16, ... in registers, and A u is summed over rows (A is symmetric), so
// that no sum runs across lanes.  Otherwise a step is the one of tridiag_step_kernel.
// The last 192 steps of four problems: 0.58 ms; as launches of their own 4.8 us each plus the gaps, 1.0 ms.
constexpr int kTail = kEigenTail;                       // 72 of a thread's 128 registers
__global__ __launch_bounds__(1024) void tridiag_tail_kernel(EigenBatch b, int k0) {
  constexpr int R = kTail / 16, C = kTail / 64;                 // rows per wave, chunks of 64 columns per row
  __shared__ double red[2][16], v[kTail], w[kTail], u[kTail], part[16][kTail];
  const int m = b.m, p = blockIdx.x, n = m - k0;                // all indices below count from k0
  double* A = b.G[p] + (long)k0 * m + k0;
  double* work = b.work[p];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double x[R][C];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int i = wave + 16 * r, j = lane + 64 * c;
      x[r][c] = i < n && j < n ? A[(long)i * m + j] : 0.0;
    }
  double tau = 0.0;
  if (tid < kTail) {                                            // the step before this launch
    const bool live = k0 > 0 && tid < n;
    v[tid] = live ? work[(long)(kV + ((k0 + 1) & 1)) * m + k0 + tid] : 0.0;
    w[tid] = live ? work[(long)(kY + ((k0 + 1) & 1)) * m + k0 + tid] : 0.0;
    u[tid] = 0.0;
  }
  if (k0 > 0) tau = work[(long)kTau * m + k0 - 1];
  if (k0 > 0 && tid < n) A[(long)tid - m] = work[(long)(kV + ((k0 + 1) & 1)) * m + k0 + tid];   // row k0 - 1 keeps v
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    const int c0 = k + 1;
    // row k of the matrix before the update, from its owner
    if (wave == (k & 15)) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r == (k >> 4))
#pragma unroll
          for (int c = 0; c < C; ++c) part[0][lane + 64 * c] = x[r][c];
    }
    const bool mine = tid >= k && tid < n;                      // the vector element of this thread (tid < kTail)
    const double vi = mine ? v[tid] : 0.0, yi = mine ? w[tid] : 0.0, yk = w[k];
    const double half = 0.5 * tau * block_sum<16>(vi * yi, red[0]);
    const double wk = tau * (yk - half), wi = tau * (yi - half * vi);
    const double cur = mine ? part[0][tid] - vi * wk - wi : 0.0;   // v_k = 1
    const double tail = block_sum<16>(mine && tid > c0 ? cur * cur : 0.0, red[1]);
    if (mine) u[tid] = cur;
    if (tid < kTail) w[tid] = mine ? wi : 0.0;
    if (tid == k) b.tri[p][k0 + k] = cur;
    if (c0 >= n) break;
    __syncthreads();
    const double x0 = u[c0];
    double beta = x0, tau_k = 0.0, scale = 0.0;
    if (tail > 0.0) {
      beta = -copysign(sqrt(x0 * x0 + tail), x0);
      tau_k = (beta - x0) / beta;
      scale = 1.0 / (x0 - beta);
    }
    __syncthreads();                                            // x0 has been read
    const double un = mine && tid > k ? (tid == c0 ? 1.0 : cur * scale) : 0.0;
    if (tid < kTail) u[tid] = un;
    if (tid == 0) {
      b.tri[p][m + k0 + k] = beta;
      work[(long)kTau * m + k0 + k] = tau_k;
    }
    if (mine && tid > k) A[(long)k * m + tid] = un;             // row k keeps its reflector for the way back
    __syncthreads();
    // update and product
    double sum[C], vj[C], wj[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      sum[c] = 0.0;
      vj[c] = v[lane + 64 * c];
      wj[c] = w[lane + 64 * c];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = wave + 16 * r;
      if (i < c0 || i >= n) continue;                           // (the same for the whole wave)
      const double vr = v[i], wr = w[i], ur = u[i];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        x[r][c] = x[r][c] - vr * wj[c] - wr * vj[c];
        sum[c] += ur * x[r][c];
      }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) part[wave][lane + 64 * c] = sum[c];
    __syncthreads();
    if (tid < kTail) {
      double y = 0.0;
#pragma unroll
      for (int q = 0; q < 16; ++q) y += part[q][tid];
      v[tid] = un;
      w[tid] = y;
    }
    tau = tau_k;
    __syncthreads();
  }
}

// All m steps in one launch: the rows stay in registers (workgroup = NW waves of RW rows; lane l holds columns l + 64 c), and
// what a step needs from the others is exchanged through memory.  At the end of step k the owner of every remaining row i
// posts the pair (y_i, a_i): the product of step k and the entry of column k+1 that stands in front of its update.  That
// is all that the next step waits for, so a step costs one such exchange and three barriers.
//   The exchange goes past the L2 caches (agent scope: those of the XCDs do not see each other's plain stores), through four
// slots of m pairs, used in turn.  A word of a pair not yet posted holds kUnset, a signalling NaN that no arithmetic
// returns, and a reader polls until every word it needs differs.  A workgroup that has gathered step k knows that all have
// gathered step k-1 and sets its pairs of that slot back to kUnset; these stores have arrived when it has gathered step
// k+1 (the polls wait for every memory operation before them), so in front of its post of that step, without which nobody
// comes to look at the slot again.
//   The launch is cooperative (every workgroup is resident, so every wait ends); polls are bounded all the same, and a
// workgroup that gives up marks the problem as failed, which takes it to the caller's other path.  A workgroup whose
// rows are done leaves; the last one stores what all work out.
// Bound by the latency of the exchange: four of 768 x 768 take 3.4 us a step against 7.3 by a launch per column and 3.0
// in the tail launch (reduction 5.0 -> 2.6 ms); 512: 3.0, 1024: 3.9.  A bare exchange of 16 bytes a row and one barrier take 2.0 us,
// 32 bytes a row 4.1; eight waves of two rows 2.7 ms, sixteen of one 3.4 (each wave reads the three vectors from LDS).
constexpr unsigned long kUnset = 0x7ff4a5c3965a3c69ul;
constexpr int kSlots = kEigenSlots;
static_assert(kY + 2 <= kEigenExchange && kEigenExchange % 2 == 0, "16-byte words on 16 bytes, also where m is odd");
typedef unsigned long u64x2 __attribute__((ext_vector_type(2)));
// pairs p[at[0]] .. p[at[E-1]], past the L2 of this XCD
template <int E> __device__ __forceinline__ void peek(u64x2 (&v)[E], const u64x2* p, const int (&at)[E]) {
  static_assert(E >= 2 && E <= 4, "");
  if constexpr (E == 2)
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %3, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]) : "v"(p + at[0]), "v"(p + at[1]) : "memory");
  else if constexpr (E == 3)
    asm volatile("global_load_dwordx4 %0, %3, off sc1\n\tglobal_load_dwordx4 %1, %4, off sc1\n\t"
                 "global_load_dwordx4 %2, %5, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]) : "v"(p + at[0]), "v"(p + at[1]), "v"(p + at[2]) : "memory");
  else
    asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
                 "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[E - 1])
                 : "v"(p + at[0]), "v"(p + at[1]), "v"(p + at[2]), "v"(p + at[E - 1]) : "memory");
}
__device__ __forceinline__ void post(unsigned long* p, unsigned long x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// lane l of the wave, as a scalar
__device__ __forceinline__ double from_lane(double x, int l) {
  const long b = __builtin_bit_cast(long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, l), hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
  return __builtin_bit_cast(double, (long)(((unsigned long)hi << 32) | lo));
}

__global__ __launch_bounds__(256) void exchange_clear_kernel(EigenBatch b) {
  const int p = blockIdx.y, n = 2 * kSlots * b.m;
  unsigned long* x = reinterpret_cast<unsigned long*>(b.work[p] + (long)kEigenExchange * b.m);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) x[i] = kUnset;
  if (blockIdx.x == 0 && threadIdx.x == 0) *b.failed[p] = 0.0;
}

template <int NW, int RW, int NC>
__global__ __launch_bounds__(64 * NW) void tridiag_resident_kernel(EigenBatch b, int looks) {
  constexpr int NT = 64 * NW, ROWS = NW * RW, W = 64 * NC, E = W / NT;   // E vector elements per thread
  static_assert(W % NT == 0 && ROWS == kResidentRows, "");
  __shared__ double vl[2][W], wl[2][W], ul[2][W], red[2][2][NW], pick[2][2];
  __shared__ int gave_up;
  const int m = b.m, p = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double* A = b.G[p];
  double* work = b.work[p];
  unsigned long* slots = reinterpret_cast<unsigned long*>(work + (long)kEigenExchange * m);
  const bool writer = blockIdx.x == gridDim.x - 1;
  const int row0 = blockIdx.x * ROWS + wave * RW;
  double x[RW][NC];
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int i = row0 + r, j = lane + 64 * c;
      x[r][c] = i < m && j < m ? A[(long)i * m + j] : 0.0;
    }
  if (tid == 0) gave_up = 0;
  double v[E], tau = 0.0;
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = 0.0;
  __syncthreads();
  for (int k = 0; k < m; ++k) {
    const int c0 = k + 1, q = k & 1;
    if (!writer && (int)(blockIdx.x + 1) * ROWS <= c0) return;
    // gather: y and column k in front of its update
    double y[E], a[E];
    if (k == 0) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        y[e] = 0.0;
        a[e] = A[min(tid + NT * e, m - 1)];
      }
    } else {
      const u64x2* slot = reinterpret_cast<const u64x2*>(slots + (long)(k % kSlots) * 2 * m);
      u64x2 got[E];
      int at[E], spins = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) {                             // elements that are not needed look at the last row
        const int i = tid + NT * e;
        at[e] = i >= k && i < m ? i : m - 1;
      }
      bool all;
      do {
        peek(got, slot, at);
        all = true;
#pragma unroll
        for (int e = 0; e < E; ++e) all = all && got[e][0] != kUnset && got[e][1] != kUnset;
      } while (!all && ++spins < looks);
      if (spins >= looks) gave_up = 1;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const unsigned long w0 = got[e][0], w1 = got[e][1];     // (scalars: a cast of a vector's element takes the first)
        y[e] = __builtin_bit_cast(double, w0);
        a[e] = __builtin_bit_cast(double, w1);
      }
    }
    double dot = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + NT * e;
      if (i >= k && i < m) dot += v[e] * y[e];
      if (i == k) pick[q][0] = y[e];
    }
    dot = wave_sum(dot);
    if (lane == 0) red[q][0][wave] = dot;
    __syncthreads();
    if (gave_up) {
      if (tid == 0) *b.failed[p] = 1.0;
      return;
    }
    dot = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) dot += red[q][0][i];
    if (k > 0 && lane < 2 * RW && row0 + lane / 2 < m)          // all have gathered step k-1: its pairs are free
      post(slots + (long)((k - 1) % kSlots) * 2 * m + 2 * row0 + lane, kUnset);
    const double half = 0.5 * tau * dot, wk = tau * (pick[q][0] - half);
    double cur[E], tail = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + NT * e;
      const bool mine = i >= k && i < m;
      const double w = mine ? tau * (y[e] - half * v[e]) : 0.0;
      cur[e] = mine ? a[e] - v[e] * wk - w : 0.0;               // column k of the updated matrix (v_k = 1)
      vl[q][i] = mine ? v[e] : 0.0;
      wl[q][i] = w;
      if (i > c0) tail += cur[e] * cur[e];
      if (i == c0) pick[q][1] = cur[e];
      if (writer && mine) {
        if (k > 0) A[(long)(k - 1) * m + i] = v[e];             // row k-1 keeps its reflector for the way back
        if (i == k) b.tri[p][k] = cur[e];
      }
    }
    tail = wave_sum(tail);
    if (lane == 0) red[q][1][wave] = tail;
    __syncthreads();
    if (c0 >= m) return;                                        // the last diagonal entry
    tail = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) tail += red[q][1][i];
    const double x0 = pick[q][1];
    double beta = x0, tau_k = 0.0, scale = 0.0;
    if (tail > 0.0) {
      beta = -copysign(sqrt(x0 * x0 + tail), x0);
      tau_k = (beta - x0) / beta;
      scale = 1.0 / (x0 - beta);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + NT * e;
      v[e] = i < c0 ? 0.0 : (i == c0 ? 1.0 : cur[e] * scale);
      ul[q][i] = v[e];
    }
    tau = tau_k;
    if (writer && tid == 0) {
      b.tri[p][m + k] = beta;
      work[(long)kTau * m + k] = tau_k;
    }
    __syncthreads();
    if (row0 + RW - 1 < c0 || row0 >= m) continue;              // (the same for the whole wave)
    double vr[RW], wr[RW], sum[RW], next[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      vr[r] = vl[q][row0 + r];
      wr[r] = wl[q][row0 + r];
      sum[r] = next[r] = 0.0;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (64 * (c + 1) <= c0 || 64 * c >= m) continue;          // columns that are done, or none
      const int j = lane + 64 * c;
      const double vj = vl[q][j], wj = wl[q][j], uj = ul[q][j];
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        x[r][c] = x[r][c] - vr[r] * wj - wr[r] * vj;
        sum[r] += x[r][c] * uj;
        if (c == c0 >> 6) next[r] = x[r][c];
      }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) sum[r] = wave_sum(sum[r]);
    // lane 2r (+ 1) posts the first (second) word of row r's pair
    double mine = 0.0;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const double n = from_lane(next[r], c0 & 63);
      if (lane / 2 == r) mine = lane & 1 ? n : sum[r];
    }
    if (lane < 2 * RW && row0 + lane / 2 >= c0 && row0 + lane / 2 < m)
      post(slots + (long)(c0 % kSlots) * 2 * m + 2 * row0 + lane, __builtin_bit_cast(unsigned long, mine));
  }
}

template <int NC> hipError_t tridiag_resident(const EigenBatch& b, int looks, hipStream_t s) {
  const int wgs = (b.m + kResidentRows - 1) / kResidentRows;
  hipLaunchKernelGGL(exchange_clear_kernel, dim3(8, b.n), dim3(256), 0, s, b);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  EigenBatch args = b;
  void* list[] = {&args, &looks};
  constexpr int kWaves = 4;
  auto kern = tridiag_resident_kernel<kWaves, kResidentRows / kWaves, NC>;
  return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(kern), dim3(wgs, b.n), dim3(64 * kWaves), list, 0, s);
}

template <int NC, int RW> hipError_t tridiag_steps(const EigenBatch& b, int steps, hipStream_t s) {
  const size_t lds = 3ul * b.m * sizeof(double);
  auto kern = tridiag_step_kernel<NC, RW>;
  static LdsOnce lds_once;
  if (hipError_t e = allow_dynamic_lds(lds_once, kern, 3ul * kEigenMaxSize * sizeof(double)); e != hipSuccess) return e;
  constexpr int kRows = 16 * RW;
  const int wgs = (b.m + kRows - 1) / kRows;
  for (int k = 0; k < steps; ++k) hipLaunchKernelGGL(kern, dim3(wgs, b.n), dim3(1024), lds, s, b, k);
  return hipGetLastError();
}

template <int NW, int NC, int PF> void apply_reflectors(const EigenBatch& b, int r, hipStream_t s) {
  hipLaunchKernelGGL((apply_reflectors_kernel<NW, NC, PF>), dim3(r, b.n), dim3(64 * NW), 0, s, b);
}

}  // namespace

hipError_t launch_tridiag(const EigenBatch& b, hipStream_t s, hipEvent_t steps_done, bool* resident, const TridiagWay& way) {
  *resident = false;
  if (b.n < 1 || b.n > kEigenBatch || b.m < kEigenMinSize || b.m > kEigenMaxSize) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  if (way.one_launch && tridiag_is_resident(b.m)) {
    e = b.m <= 512 ? tridiag_resident<8>(b, way.looks, s)
                   : (b.m <= 768 ? tridiag_resident<12>(b, way.looks, s) : tridiag_resident<16>(b, way.looks, s));
    if (e == hipSuccess) {
      *resident = true;
      return steps_done != nullptr ? hipEventRecord(steps_done, s) : e;
    }
    // fewer compute units than it takes, or no cooperative launch at all: by steps, which say what else is wrong
    (void)hipGetLastError();
  }
  const int steps = tridiag_steps_of(b.m);
  e = hipSuccess;
  if (steps > 0) e = b.m <= 512 ? tridiag_steps<8, 1>(b, steps, s) : (b.m <= 1024 ? tridiag_steps<16, 1>(b, steps, s) : tridiag_steps<0, 4>(b, steps, s));
  if (e == hipSuccess && steps_done != nullptr) e = hipEventRecord(steps_done, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tridiag_tail_kernel, dim3(b.n), dim3(1024), 0, s, b, steps);
  return hipGetLastError();
}

hipError_t launch_tridiag_vectors(const EigenBatch& b, hipStream_t s) {
  if (b.n < 1 || b.n > kEigenBatch || b.m < kEigenMinSize || b.m > kEigenMaxSize) return hipErrorInvalidValue;
  int r = 0, nv = 0;
  for (int p = 0; p < b.n; ++p) {
    if (b.r[p] < 1 || b.n_values[p] < b.r[p] || b.n_values[p] > b.m) return hipErrorInvalidValue;
    r = b.r[p] > r ? b.r[p] : r;
    nv = b.n_values[p] > nv ? b.n_values[p] : nv;
  }
  const size_t lv = 2ul * b.m * sizeof(double), lt = 4ul * b.m * sizeof(double);
  static LdsOnce values_once, vector_once;
  if (hipError_t e = allow_dynamic_lds(values_once, tridiag_values_kernel, 2ul * kEigenMaxSize * sizeof(double)); e != hipSuccess) return e;
  if (hipError_t e = allow_dynamic_lds(vector_once, tridiag_vector_kernel, 4ul * kEigenMaxSize * sizeof(double)); e != hipSuccess) return e;
  hipLaunchKernelGGL(tridiag_values_kernel, dim3((nv + 3) / 4, b.n), dim3(256), lv, s, b);
  hipLaunchKernelGGL(tridiag_vector_kernel, dim3(r, b.n), dim3(64), lt, s, b);
  static_assert(kEigenMaxSize <= 64 * 8 * 10, "a row fits the workgroup");
  if (b.m <= 256) apply_reflectors<1, 4, 8>(b, r, s);
  else if (b.m <= 512) apply_reflectors<4, 2, 8>(b, r, s);
  else if (b.m <= 1024) apply_reflectors<4, 4, 4>(b, r, s);
  else if (b.m <= 2048) apply_reflectors<4, 8, 4>(b, r, s);
  else apply_reflectors<8, 10, 4>(b, r, s);                // 5120 elements
  return hipGetLastError();
}

}  // namespace ta
