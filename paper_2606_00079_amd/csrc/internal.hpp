// Host-side helpers shared by the translation units of libbitsmoe.
#pragma once

#include <cstddef>
#include <cstdint>
#include <initializer_list>
#include <string>

#include "bitsmoe.h"

namespace bitsmoe {

// Records `msg` as the calling thread's last error and returns `st`.
bitsmoe_status fail(bitsmoe_status st, const std::string& msg);
// Clears the calling thread's last error; returns BITSMOE_OK.
bitsmoe_status ok();

// Named scratch regions.  Each is a grow-only device buffer per device.
enum ScratchSlot : int {
  kScratchA = 0,     // operand staging (transposes, bf16 splits)
  kScratchB = 1,     // second operand staging
  kScratchPart = 2,  // split-K / row partials
  kScratchD = 3,     // score: bf16 error rows
  kScratchMisc = 4,  // small tables
  kScratchCount = 5
};

// Returns a device buffer of at least `bytes` bytes for `slot` on the
// current device.  Growing synchronizes `stream` first (calls on a device
// are stream-ordered, so no queued work still reads the old buffer).
// Returns nullptr after recording ERR_NOMEM / ERR_DEVICE.
void* scratch(int slot, size_t bytes, void* stream, bitsmoe_status* st);

// HIP error -> status with a message naming `what`.
bitsmoe_status device_error(const char* what, int hip_err);

// Compute units of the current device (cached per device; 256 if the query
// fails).
int device_cus();

// Records HIP events around a kernel launch when timing is enabled
// (bitsmoe_timing); construct right before the launch, destroy right after.
// A null name records nothing.
class KernelTimer {
 public:
  KernelTimer(const char* name, void* stream);
  ~KernelTimer();
 private:
  const char* name_;
  void* stream_;
  void* start_ = nullptr;
};

// Tridiagonal reduction of the symmetric fp64 M [n][n] in one cooperative
// launch (tridiag.hip): the diagonals d [n] and e [n-1], tau [n-1] and the
// reflectors by rows into V [n][n].  `fits`: whether this device holds an
// n x n matrix that way; `work` has `bytes` bytes, *err is nonzero after a
// run in which a reader of the exchange gave up, after `poll_limit` polls (the
// outputs are then of no use; M is as it was).  False if the launch was refused
// (nothing was computed).
constexpr int kTridiagPolls = 1 << 22;  // (seconds)
bool tridiag_resident_fits(int64_t n);
size_t tridiag_resident_bytes(int64_t n);
bool tridiag_resident(const double* M, int64_t n, double* V, double* dvec, double* evec,
                      double* tau, void* work, int* err, int poll_limit, void* stream);

// The same by one workgroup, for n that `fits`.
bool tridiag_small_fits(int64_t n);
void tridiag_small(const double* M, int64_t n, double* V, double* dvec, double* evec, double* tau,
                   void* stream);

// The r largest eigenvalues w [r] (ascending) of the tridiagonal (d, e) and
// their eigenvectors, the rows of Zt [r][n] (trieig.hip).  info [7]: scaled
// bounds (2) and norm, then the norm of T, max e^2, exponent of the scale and
// 1 if an entry is not finite; bad [r]: 1 where no vector was found.  `buf`
// has `bytes` bytes.  Vectors of eigenvalues closer than about 1e-7 of the
// norm are not orthogonal to full precision.
size_t tri_eigenpairs_bytes(int64_t n, int64_t r);
bitsmoe_status tri_eigenpairs(const double* d, const double* e, int64_t n, int64_t r, double* w,
                              double* Zt, double* info, uint8_t* bad, void* buf, void* stream);

// Back-transformation of the eigenvectors Zt [r][n] of the tridiagonal by the
// reflectors V, tau of the reduction, with order, sign and fp32 rounding, into
// Ut [r][n] (eigback.hip), for n that `fits`.  `panels` forms the compact
// factors T (`bytes` bytes) first.
bool backtransform_fits(int64_t n);
size_t backtransform_bytes(int64_t n);
bitsmoe_status backtransform_panels(const double* V, const double* tau, int64_t n, double* T,
                                    void* stream);
bitsmoe_status backtransform(const double* V, const double* T, const double* Zt, int64_t n, int64_t r,
                             float* Ut, void* stream);

// bitsmoe_shared_basis_gpu with its own poll limit for the one-launch reduction;
// *gave_up_host (may be null) is 1 where a reader gave up and the panel form took
// over.  For the test of that route; not part of the interface.
extern "C" bitsmoe_status bitsmoe_shared_basis_gpu_polls(const double* M_dev, int64_t d_out, int64_t r,
                                                         float* Ut_dev, double* eigvals_host,
                                                         double* host_ms, int poll_limit,
                                                         int* gave_up_host, void* stream);

// True when every pointer is 16-byte aligned (the kernels use 16-byte
// vector accesses on device buffers).
inline bool aligned16(std::initializer_list<const void*> ptrs) {
  for (const void* p : ptrs)
    if (reinterpret_cast<uintptr_t>(p) % 16 != 0) return false;
  return true;
}

inline bool is_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }

}  // namespace bitsmoe
