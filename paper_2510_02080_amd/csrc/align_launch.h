// Host-side launch helpers shared by the API translation unit and the kernels.
#pragma once

#include "s3a_internal.h"
#include "tuning.h"

namespace s3a {

// BF16 planes (xyz or depth) load 8 elements per 16 bytes, FP32 ones 4.
inline int vec_of(int dtype) { return (dtype == S3A_BF16 || dtype == DT_DEPTH_BF16) ? 8 : 4; }
inline int64_t tile_elems(int dtype, const LaunchCfg& lc) { return (int64_t)lc.wg * lc.items * vec_of(dtype); }
// Threads of one launch (HIP holds them below 2^32).
constexpr int64_t GRID_THREADS = 1ll << 31;

// Upper bound of the tile count of any batch (see k_sched).
inline int64_t max_tiles(int64_t n_points, int n_pairs, int64_t tile) { return n_points / tile + 2 * (int64_t)n_pairs + 1; }

// The call's schedule (tile table, per-pair ranges, depth cameras in pass form; a
// depth pair of invalid geometry is marked bad); stores the descriptor c to *cd.
hipError_t launch_sched(const Shape& sh, const CallDesc& c, CallDesc* cd, const Work& w, hipStream_t st);
hipError_t launch_pass(int dtype, int mode, const LaunchCfg& lc, const Shape& sh, const CallDesc* cd, const Work& w,
                       int32_t tile_lo, int32_t tile_hi, int grid, hipStream_t st);
// A Gauss-Newton pass (>= 1) that solves the pass before it first, at the untuned
// shapes (256 threads; 4 items FP32, 2 BF16, 16 depth), and the solve after the last.
hipError_t launch_pass_solve(int dtype, const Shape& sh, const CallDesc* cd, const Work& w, int pass, int grid,
                             hipStream_t st);
hipError_t launch_solve_last(const Shape& sh, const CallDesc* cd, const Work& w, int pass, hipStream_t st);
hipError_t launch_finalize(const Shape& sh, const CallDesc* cd, const Work& w, int pass, int32_t pair_lo, int32_t n,
                           hipStream_t st);
hipError_t launch_prep(const Shape& sh, const CallDesc* cd, const Work& w, int adjoint, hipStream_t st);
hipError_t launch_finalize_cost(const Shape& sh, const CallDesc* cd, const Work& w, hipStream_t st);
hipError_t launch_adjoint(int dtype, const LaunchCfg& lc, const Shape& sh, const CallDesc* cd, const Work& w, int grid,
                          hipStream_t st);
hipError_t launch_finalize_adjoint(const Shape& sh, const CallDesc* cd, const Work& w, hipStream_t st);
hipError_t launch_persistent(int dtype, const LaunchCfg& lc, const Shape& sh, const CallDesc* cd, const Work& w,
                             int grid, hipStream_t st);
hipError_t launch_fill_zero(uint32_t* p, int64_t n, hipStream_t st);
hipError_t launch_init_outputs(const Shape& sh, const CallDesc* cd, hipStream_t st);

}  // namespace s3a
