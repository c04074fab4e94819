// Leading eigenpairs of a batch of symmetric positive semi-definite fp64 matrices of one size (eigen.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace ta {

constexpr int kEigenBatch = 4;                          // matrices solved side by side
// four vectors of the matrix size have to fit the LDS of a workgroup
constexpr int kEigenMinSize = 8, kEigenMaxSize = 5056;

struct EigenBatch {
  int n, m;                                             // matrices in the batch, size of each
  int r[kEigenBatch];                                   // eigenvectors wanted of each, 1 .. m
  double* G[kEigenBatch];                               // [m, m], full storage; destroyed (holds the reflectors)
  double* Z[kEigenBatch];                               // [r, m] eigenvectors, largest eigenvalue first
  double* work[kEigenBatch];                            // eigen_work_elems(m) doubles each
  double* tri[kEigenBatch];                             // [2, m] diagonal and subdiagonal of the tridiagonal matrix
  double* value[kEigenBatch];                           // [m] eigenvalues, largest first (the first n_values written)
  double* resid[kEigenBatch];                           // [m] residual of each vector in the tridiagonal matrix
  int n_values[kEigenBatch];                            // eigenvalues wanted of each, r .. m
  double* failed[kEigenBatch];                          // 1.0: the resident reduction gave up (see there), nothing else holds
};
// vectors of m doubles in a work array: those of the steps, one place left free, and behind them the exchange of the resident
// reduction, whose 16-byte words start on 16 bytes for every m because an even number of vectors stands in front of them
constexpr int kEigenExchange = 6, kEigenSlots = 4;
inline size_t eigen_work_elems(int m) { return (kEigenExchange + 2ul * kEigenSlots) * m; }

// Sizes whose whole reduction is one launch with the matrices in registers; its workgroups hold kResidentRows rows each, so that
// four matrices of 1024 take the 256 compute units once.  Up to 256 most columns are the tail launch's either way.
constexpr int kResidentRows = 16;
inline bool tridiag_is_resident(int m) { return m > 256 && m <= 1024; }
// Otherwise: columns that the reduction takes by one launch each; the rest goes in one launch
constexpr int kEigenTail = 192;
inline int tridiag_steps_of(int m) { return m > kEigenTail ? m - kEigenTail : 0; }

// The ways a reduction may take; other values than these are for tests of the ways out.
struct TridiagWay {
  bool one_launch = true;                               // where tridiag_is_resident
  int looks = 1 << 20;                                  // of a workgroup of that launch at words not yet posted, before it gives up:
                                                        // each at least one round trip to memory, 0.5 s and more.  0: at once
};
// Enqueues the reduction to tridiagonal form; G, work and tri are written.  steps_done (nullable) is recorded behind the
// launches of one column each, or the one launch of all columns; `resident` receives which of the two it was.
hipError_t launch_tridiag(const EigenBatch& b, hipStream_t s, hipEvent_t steps_done, bool* resident, const TridiagWay& way);
// Enqueues eigenvalues and eigenvectors of the tridiagonal matrices, vectors carried back to the basis of G.
// The vectors are unit rows; rows of close eigenvalues are orthogonal only up to (rounding / gap).
hipError_t launch_tridiag_vectors(const EigenBatch& b, hipStream_t s);

}  // namespace ta
