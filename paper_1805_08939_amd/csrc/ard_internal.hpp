// Internal helpers shared by the library's translation units: error state,
// argument checks and HIP error propagation. Not part of the public ABI.
#pragma once

#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "../../include/ard.h"

namespace ard {

// Records a formatted message as the calling thread's last error and returns
// `status`, so that a check reads `return fail(ARD_ERR_INVALID_ARG, ...)`.
int fail(int status, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Validates a row plan against the neuron count it is applied to. A NULL plan
// is "everything kept". needs_list: the caller reads the device kept-index
// list, so a plan that drops neurons must carry one. Returns ARD_OK or an
// error with a message.
int check_row_plan(const ard_row_plan* plan, int32_t n, const char* what, bool needs_list);

// Part of an fp32 tile-layer product (ard_tile.hip), for the tile-pattern LSTM.
constexpr int kTilePartSplits = 8;  // largest split of the kept-tile lists
struct TilePart {
  const void* act;
  const void* W;
  void* out;
  int32_t own0, own_count;  // output tile rows (fwd) or columns
  int32_t lo, hi;           // other index of the kept tiles used
  int32_t cols, lda;        // columns of the product, row stride of act
  int32_t ldo, nb, nv;      // output addressing (see TileWaveArgs)
  int64_t bstride;
  float* partial;           // kTilePartSplits * own_count * tile * cols floats, or NULL
  bool chains;              // add an output's terms in sixteen chains
};
// The plan's and W's checks of the tile-layer calls.
int tile_part_check(const ard_tile_plan* p, int32_t cols, const void* W);
int tile_part_f32(bool fwd, const ard_tile_plan* p, const TilePart& t, void* stream, int* splits_left);

// Kept count of a row pattern (see ard_row_kept).
inline int32_t kept_count(int32_t n, int32_t period, int32_t offset) {
  if (offset >= n) return 0;
  return (n - offset + period - 1) / period;
}

}  // namespace ard

// Propagates a HIP error from a launch or runtime call as ARD_ERR_HIP.
#define ARD_HIP_CHECK(expr)                                                           \
  do {                                                                                \
    hipError_t _e = (expr);                                                           \
    if (_e != hipSuccess)                                                             \
      return ::ard::fail(ARD_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(_e)); \
  } while (0)

#define ARD_LAUNCH_CHECK()                                                            \
  do {                                                                                \
    hipError_t _e = hipGetLastError();                                                \
    if (_e != hipSuccess)                                                             \
      return ::ard::fail(ARD_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(_e)); \
  } while (0)
