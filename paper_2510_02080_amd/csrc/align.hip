// Dense Sim(3) alignment kernels: tile scheduling, point passes, and the FP64
// per-pair finalize (Sec. III-C.2, eq. (sim3); Huber IRLS refinement).
//
// A call runs 1 + K (+1) passes over every pair: the moments pass of the
// weighted Umeyama closed form, K Gauss-Newton passes, and optionally a cost
// pass at the final iterate. Between passes each pair's tile partials are
// summed in a fixed order and its 7x7 (or 3x3 / 4x4) system is solved in FP64.
#include <algorithm>

#include "align_kernels.h"
#include "align_launch.h"
#include "finalize.h"

namespace s3a {

// ------------------------------------------------------------------ schedule

// The caller's cameras of depth pair k in pass form (reciprocal focal lengths,
// offsets), geometry checked and sanitised. Returns false for a pair with invalid
// geometry, or with more elements (n) than its frames hold.
__device__ inline bool depth_prep(const s3a_depth_pair& src, int64_t n, DepthPair* out) {
  int W = src.width, HW = src.frame_pixels, nf = src.n_frames;
  const bool ok = W >= 1 && HW >= W && HW % W == 0 && nf >= 1 && nf <= DEPTH_MAX_FRAMES && src.reserved == 0 &&
                  n <= (int64_t)nf * HW;
  if (!ok) {
    W = 1;
    HW = 1;
    nf = 1;
  }
  DepthPair dp;
  dp.width = W;
  dp.rows = HW / W;
  dp.frame_pixels = HW;
  dp.n_frames = nf;
  dp.inv_width = 1.0f / (float)W;
  dp.pad[0] = dp.pad[1] = dp.pad[2] = 0;
  for (int f = 0; f < DEPTH_MAX_FRAMES; ++f) {
    const s3a_camera* in[2] = {src.p + f, src.q + f};
    DepthCam* cam[2] = {dp.p + f, dp.q + f};
    for (int side = 0; side < 2; ++side) {
      const s3a_camera& c = *in[side];
      DepthCam& o = *cam[side];
      o.ifx = 1.0f / c.fx;
      o.ify = 1.0f / c.fy;
      o.ox = -c.cx / c.fx;
      o.oy = -c.cy / c.fy;
      for (int i = 0; i < 9; ++i) o.R[i] = c.R[i];
      for (int i = 0; i < 3; ++i) o.t[i] = c.t[i];
    }
  }
  *out = dp;
  return ok;
}

// A camera without NaN or infinities (also a focal length of zero), whose rays and
// centre are such that a depth below EXTREME / PLAIN_RAY gives no extreme point, and one
// below 1e30 a finite one.
__device__ inline bool camera_plain(const s3a_camera& c, int width, int rows) {
  float G = 0.0f, t = 0.0f;
  for (int i = 0; i < 9; ++i) G += fabsf(c.R[i]);
  for (int i = 0; i < 3; ++i) t += fabsf(c.t[i]);
  const float ray = fabsf(1.0f / c.fx) * (float)width + fabsf(c.cx / c.fx) + fabsf(1.0f / c.fy) * (float)rows + fabsf(c.cy / c.fy);
  return G * (ray + 1.0f) < PLAIN_RAY && t < EXTREME;  // (false for a NaN)
}

// Tile j of a pair's range [a, b); depth: the pair's frames, or null. Frames narrower
// than a vector of vec pixels count as spanned (see DepthWalk), and so do frames whose
// camera is lost or out of all scale: the walk of a frame masks a pixel by
// its depths, which such a camera takes to NaN all the same, while the spanning walk
// masks the points themselves.
__device__ inline TileDesc make_tile(int64_t a, int64_t b, int pair, int tile0, int ntiles, int j, int64_t T,
                                     const s3a_depth_pair* depth, int vec) {
  const int64_t b0 = a & ~(TILE_ALIGN - 1);
  TileDesc t;
  t.pair = pair;
  t.tile0 = tile0;
  t.ntiles = ntiles;
  t.frame = -1;
  t.head = j == 0 ? (int16_t)(a - b0) : (int16_t)0;
  if (b > a) {
    t.begin = b0 + (int64_t)j * T;
    t.end = t.begin + T < b ? t.begin + T : b;
    t.lo = a;
    if (depth && depth->width >= vec && depth->frame_pixels >= depth->width) {
      const int64_t first = t.begin > a ? t.begin : a;
      const int f0 = (int)((first - a) / depth->frame_pixels), f1 = (int)((t.end - 1 - a) / depth->frame_pixels);
      const int rows = depth->frame_pixels / depth->width;
      if (f0 == f1 && f0 < depth->n_frames && f0 < DEPTH_MAX_FRAMES && t.end > first &&
          camera_plain(depth->p[f0], depth->width, rows) && camera_plain(depth->q[f0], depth->width, rows))
        t.frame = (int16_t)f0;
    }
  } else {
    t.begin = t.end = t.lo = a;
    t.head = 0;
  }
  return t;
}
__device__ inline int tiles_of(int64_t a, int64_t b, int64_t T) {
  return b > a ? (int)((b - (a & ~(TILE_ALIGN - 1)) + T - 1) / T) : 1;
}

// The whole schedule of a call of at most SCHED_PAIRS pairs in one launch: every
// workgroup checks the offsets and scans the pairs' tile counts for itself (the
// offsets are a few kilobytes, read once from L2), then writes its share of the
// tiles, a thread each, found by bisection of the scan in LDS, and of the pairs
// (with the depth cameras' pass form). The call's descriptor arrives as an argument
// and the first workgroup stores it for the kernels that follow. One launch of
// about 5 us takes the place of a copy, a one-workgroup scan and a fill with one
// thread per pair, 4 + 4 + 17 us for 256 pairs of 32 tiles. If any pair is
// malformed, every pair is marked bad (so that a malformed offsets array cannot
// make the tile table larger than the host-side bound).
constexpr int SCHED_PAIRS = 2048;
constexpr int SCHED_WG = 256;
__global__ __launch_bounds__(SCHED_WG) void k_sched_tiles(Shape sh, CallDesc c, CallDesc* cd, Work w) {
  __shared__ int32_t tile0[SCHED_PAIRS + 1];
  __shared__ int32_t wave[SCHED_WG / 64];
  const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6, n = sh.n_pairs;
  const int64_t T = sh.tile_elems;
  const int per = (n + SCHED_WG - 1) / SCHED_WG, k0 = min(tid * per, n), k1 = min(k0 + per, n);
  int bad = 0;
  for (int k = k0; k < k1; ++k) {
    const int64_t a = c.offsets[k], b = c.offsets[k + 1];
    bad |= !(a >= 0 && a <= b && b <= sh.n_points);
  }
  const int any_bad = __syncthreads_or(bad);
  int mine = 0;
  for (int k = k0; k < k1; ++k) mine += any_bad ? 1 : tiles_of(c.offsets[k], c.offsets[k + 1], T);
  int incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int x = __shfl_up(incl, o, 64);
    if (lane >= o) incl += x;
  }
  if (lane == 63) wave[wv] = incl;
  __syncthreads();
  int at = incl - mine;
  for (int q = 0; q < wv; ++q) at += wave[q];
  for (int k = k0; k < k1; ++k) {
    tile0[k] = at;
    at += any_bad ? 1 : tiles_of(c.offsets[k], c.offsets[k + 1], T);
  }
  if (tid == SCHED_WG - 1) tile0[n] = at;
  __syncthreads();
  const int total = tile0[n], gt = (int)blockIdx.x * SCHED_WG + tid, gs = (int)gridDim.x * SCHED_WG;
  if (gt == 0) {
    *cd = c;
    *w.total_tiles = total;
  }
  for (int k = gt; k < n; k += gs) {
    PairSched s;
    s.a = any_bad ? 0 : c.offsets[k];
    s.b = any_bad ? 0 : c.offsets[k + 1];
    s.tile0 = tile0[k];
    s.ntiles = tile0[k + 1] - tile0[k];
    s.bad = any_bad;
    s.extreme = 0;
    if (c.depth && !depth_prep(c.depth[k], s.b - s.a, w.dpairs + k)) s.bad = 1;
    w.sched[k] = s;
  }
  for (int t = gt; t < total; t += gs) {
    int lo = 0, hi = n - 1;  // the last pair whose first tile is at most t
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (tile0[mid] <= t) lo = mid;
      else hi = mid - 1;
    }
    const int64_t a = any_bad ? 0 : c.offsets[lo], b = any_bad ? 0 : c.offsets[lo + 1];
    w.tiles[t] = make_tile(a, b, lo, tile0[lo], tile0[lo + 1] - tile0[lo], t - tile0[lo], T,
                           c.depth ? c.depth + lo : nullptr, sh.vec);
  }
}

// Calls of more pairs. One workgroup checks every pair's range, then makes an
// exclusive scan of the tile counts; k_sched_fill writes the tiles, k_depth_prep the
// cameras.
__global__ __launch_bounds__(1024) void k_sched(Shape sh, CallDesc c, CallDesc* cd, Work w) {
  __shared__ int32_t buf[1024];
  __shared__ int32_t carry;
  const int n = sh.n_pairs;
  const int64_t T = sh.tile_elems;
  int bad_local = 0;
  for (int k = threadIdx.x; k < n; k += 1024) {
    const int64_t a = c.offsets[k], b = c.offsets[k + 1];
    bad_local |= !(a >= 0 && a <= b && b <= sh.n_points);
  }
  const int any_bad = __syncthreads_or(bad_local);
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < n; base += 1024) {
    const int k = base + threadIdx.x;
    int32_t nt = 0;
    PairSched s{};
    if (k < n) {
      int64_t a = c.offsets[k], b = c.offsets[k + 1];
      s.bad = any_bad;
      if (any_bad) { a = 0; b = 0; }
      s.a = a;
      s.b = b;
      nt = tiles_of(a, b, T);
      s.ntiles = nt;
    }
    buf[threadIdx.x] = nt;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const int32_t x = (int)threadIdx.x >= off ? buf[threadIdx.x - off] : 0;
      __syncthreads();
      buf[threadIdx.x] += x;
      __syncthreads();
    }
    if (k < n) {
      s.tile0 = carry + buf[threadIdx.x] - nt;
      w.sched[k] = s;
    }
    __syncthreads();
    if (threadIdx.x == 1023) carry += buf[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *cd = c;
    *w.total_tiles = carry;
  }
}

__global__ void k_sched_fill(Shape sh, const s3a_depth_pair* depth, Work w) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= sh.n_pairs) return;
  const PairSched s = w.sched[k];
  for (int j = 0; j < s.ntiles; ++j) w.tiles[s.tile0 + j] = make_tile(s.a, s.b, k, s.tile0, s.ntiles, j, sh.tile_elems,
                                                                    depth ? depth + k : nullptr, sh.vec);
}

__global__ void k_depth_prep(Shape sh, const CallDesc* __restrict__ cd, Work w) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= sh.n_pairs) return;
  const PairSched sc = w.sched[k];
  if (!depth_prep(cd->depth[k], sc.b - sc.a, w.dpairs + k)) w.sched[k].bad = 1;
}

// ------------------------------------------------------------------ point passes

// ONE: a workgroup per tile, no loop over tiles (what the loop keeps in registers
// costs a wavefront of occupancy on depth input).
template <int DT, int MODE, int WG, int ITEMS, bool ONE>
__global__ __launch_bounds__(WG) void k_pass(Shape sh, const CallDesc* __restrict__ cd, Work w,
                                              int32_t tile_lo, int32_t tile_hi) {
  __shared__ double red[WG / 64][NSTAT];
  const int total = tile_hi >= 0 ? tile_hi : *w.total_tiles;
  const void* pl[7];
#pragma unroll
  for (int j = 0; j < 7; ++j) pl[j] = cd->planes[j];
  for (int t = tile_lo + (int)blockIdx.x; t < total; t += (int)gridDim.x) {
    const TileDesc td = load_tile(w.tiles + t);
    typename TileRaw<DT>::type first;
    if constexpr (ONE) tile_begin<DT, WG>(sh, pl, td, first);
    const PointParams P = load_params(w.params + td.pair);
    const SrcCtx<DT> src = make_src<DT>(pl, w, td);
    tile_body<DT, MODE, WG, ITEMS, ONE>(sh, src, td, P, first, red, w.partials + (int64_t)t * NSTAT,
                                        &w.sched[td.pair].extreme);
    if constexpr (ONE) return;
  }
}

// ------------------------------------------------------------------ passes that solve

// By a whole workgroup of 256: pair k's sums of pass `done`, and the solve that
// follows that pass. The workgroup `first` of the pair also stores the state for the
// next pass and, where no pass follows, the outputs. Returns whether passes follow.
// States and partials take turns in two buffers, by the parity of their pass, since
// the pair's other workgroups still read the old ones.
template <SolveKind KIND>
__device__ inline bool solve_pass(const Shape& sh, const CallDesc* __restrict__ cd, const Work& w, int k, int tile0,
                                  int ntiles, int done, bool first, SolveLds& S) {
  const int wv = (int)threadIdx.x >> 6;
  double word = 0.0;
  if (KIND != SOLVE_MOMENTS && wv == 0) word = state_word(w.state + (size_t)((done + 1) & 1) * w.pairs_cap + k);
  const int bad = KIND != SOLVE_GN ? w.sched[k].bad : 0, extreme = KIND != SOLVE_GN ? w.sched[k].extreme : 0;
  gather_groups(w.partials + ((size_t)(done & 1) * w.tiles_cap + tile0) * NSTAT, ntiles, wv, 4, S.part);
  if (KIND != SOLVE_MOMENTS && wv == 0) set_state_word(&S.st, word);
  __syncthreads();
  if (wv == 0) {
    solve_wave<KIND>(sh, cd, k, done, bad != 0, extreme != 0, first, S);
    if (first) set_state_word(w.state + (size_t)(done & 1) * w.pairs_cap + k, state_word(&S.st));
  }
  __syncthreads();
  return S.more != 0;
}

// Gauss-Newton pass `pass` >= 1 with the solve that precedes it: every workgroup
// (one per tile) sums its pair's partials of the pass before and solves its 7x7
// system itself, while its own first loads are in flight, so the launch between two
// passes is gone. A call of few tiles is bound by that chain alone: pass 5.0 +
// finalize 5.0 us for one pair of 3,072 points. With more tiles than the chip holds
// at once the repeated solves cost more than the launch (see passes_solve).
// FIRST: the solve is the closed form's (pass 1), which takes registers that the
// later passes' kernels then need not hold: three of those share a SIMD.
template <int DT, int MODE, int WG, int ITEMS, bool FIRST>
__global__ __launch_bounds__(WG) void k_pass_solve(Shape sh, const CallDesc* __restrict__ cd, Work w, int pass) {
  static_assert(WG == 256, "solve_pass");
  __shared__ double red[WG / 64][NSTAT];
  __shared__ SolveLds S;
  const int t = (int)blockIdx.x;
  const TileDesc td = load_tile(w.tiles + t);  // the grid lies within the table; past the call's tiles it is not used
  if (t >= *w.total_tiles) return;
  const void* pl[7];
#pragma unroll
  for (int j = 0; j < 7; ++j) pl[j] = cd->planes[j];
  typename TileRaw<DT>::type first;
  tile_begin<DT, WG>(sh, pl, td, first);
  const SrcCtx<DT> src = make_src<DT>(pl, w, td);
  if (!solve_pass<FIRST ? SOLVE_MOMENTS : SOLVE_GN>(sh, cd, w, td.pair, td.tile0, td.ntiles, pass - 1, t == td.tile0, S)) return;
  PointParams P;
#pragma unroll
  for (int i = 0; i < 9; ++i) P.Mf[i] = uniform_f32((float)(S.st.S.s * S.st.S.R[i]));
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    P.tcf[i] = uniform_f32((float)(S.st.S.t[i] - S.st.cq[i]));
    P.cf[i] = uniform_f32((float)S.st.cq[i]);
  }
  P.active = 1;
  P.mask = uniform_i32(S.st.mask);
  tile_gn<DT, WG, ITEMS, MODE == MODE_GN, true>(sh, src, td, P, first, red,
                                                w.partials + ((size_t)(pass & 1) * w.tiles_cap + t) * NSTAT);
}

// The solve after the last pass.
__global__ __launch_bounds__(256) void k_solve_last(Shape sh, const CallDesc* __restrict__ cd, Work w, int pass) {
  __shared__ SolveLds S;
  const int k = (int)blockIdx.x;
  const PairSched sc = w.sched[k];
  solve_pass<SOLVE_ANY>(sh, cd, w, k, sc.tile0, sc.ntiles, pass, true, S);
}

// The solve after pass `pass` as a launch of its own, a workgroup per pair, with one
// buffer each of states and partials: publishes the iterate for the next pass.
__global__ __launch_bounds__(256) void k_finalize(Shape sh, const CallDesc* __restrict__ cd, Work w, int pass,
                                                  int32_t pair_lo) {
  __shared__ SolveLds S;
  const int k = pair_lo + (int)blockIdx.x, wv = (int)threadIdx.x >> 6;
  if (k >= sh.n_pairs) return;
  const PairSched sc = w.sched[k];
  double word = 0.0;
  if (wv == 0 && pass > 0) word = state_word(w.state + k);
  gather_groups(w.partials + (int64_t)sc.tile0 * NSTAT, sc.ntiles, wv, 4, S.part);
  if (wv == 0 && pass > 0) set_state_word(&S.st, word);
  __syncthreads();
  if (wv != 0) return;
  solve_wave<SOLVE_ANY>(sh, cd, k, pass, sc.bad != 0, sc.extreme != 0, true, S);
  set_state_word(w.state + k, state_word(&S.st));
  if (threadIdx.x == 0) publish(w.params + k, S.st.S, S.st.cq, S.more, S.st.mask);
}

// ------------------------------------------------------------------ cost / adjoint prep

// S' = Exp(xi) S per pair; the adjoint also needs 1/C, gL and L.
__global__ void k_prep(Shape sh, const CallDesc* __restrict__ cd, Work w, int adjoint) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= sh.n_pairs) return;
  Sim3d S = load_sim3(cd->S_in + k);
  if (cd->xi) S = sim3_compose(sim3_exp(cd->xi + 7 * k), S);
  const double c0[3] = {0.0, 0.0, 0.0};
  int active = 1;
  if (adjoint) active = cd->C_in[k] > 0.0;
  publish(w.params + k, S, c0, active);
  if (adjoint) {
    w.params[k].inv_C = active ? (float)(1.0 / cd->C_in[k]) : 0.0f;
    w.params[k].scale = (float)cd->gL[k];
    w.params[k].L = (float)cd->L_in[k];
  }
}

__global__ __launch_bounds__(64) void k_finalize_cost(Shape sh, const CallDesc* __restrict__ cd, Work w) {
  const int k = blockIdx.x;
  if (k >= sh.n_pairs) return;
  const PairSched sc = w.sched[k];
  double s[NSTAT];
  pair_sums(w, sc, 3, s);
  if (threadIdx.x != 0) return;
  const double C = s[0];
  cd->C_out[k] = C;
  cd->L_out[k] = C > 0.0 ? s[1] / C : __builtin_nan("");
}

}  // namespace s3a

// ------------------------------------------------------------------ launchers

namespace s3a {

template <int DT, int MODE>
static hipError_t launch_pass_t(const LaunchCfg& lc, const Shape& sh, const CallDesc* cd, const Work& w,
                                int32_t tile_lo, int32_t tile_hi, int grid, hipStream_t st) {
#define S3A_CASE(WGV, IT)                                                                                   \
  if (lc.wg == WGV && lc.items == IT) {                                                                     \
    hipLaunchKernelGGL((k_pass<DT, MODE, WGV, IT, false>), dim3(grid), dim3(WGV), 0, st, sh, cd, w, tile_lo, \
                       tile_hi);                                                                            \
    return hipGetLastError();                                                                               \
  }
  if constexpr (DT == DT_DEPTH_F32 || DT == DT_DEPTH_BF16) {
    if (lc.wg == 256 && lc.items == 16 && lc.occupancy == 0 && grid < GRID_THREADS / 256) {  // the untuned depth shape
      hipLaunchKernelGGL((k_pass<DT, MODE, 256, 16, true>), dim3(grid), dim3(256), 0, st, sh, cd, w, tile_lo, tile_hi);
      return hipGetLastError();
    }
  }
  S3A_CASE(256, 2) S3A_CASE(256, 4) S3A_CASE(256, 8) S3A_CASE(256, 16)
  S3A_CASE(512, 2) S3A_CASE(512, 4) S3A_CASE(512, 8)
#undef S3A_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_pass(int dtype, int mode, const LaunchCfg& lc, const Shape& sh, const CallDesc* cd,
                       const Work& w, int32_t tile_lo, int32_t tile_hi, int grid, hipStream_t st) {
  if (dtype == DT_DEPTH_F32) {
    if (mode == MODE_MOMENTS) return launch_pass_t<DT_DEPTH_F32, MODE_MOMENTS>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_GN) return launch_pass_t<DT_DEPTH_F32, MODE_GN>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_GN_NC) return launch_pass_t<DT_DEPTH_F32, MODE_GN_NC>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    return hipErrorInvalidValue;
  }
  if (dtype == DT_DEPTH_BF16) {
    if (mode == MODE_MOMENTS) return launch_pass_t<DT_DEPTH_BF16, MODE_MOMENTS>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_GN) return launch_pass_t<DT_DEPTH_BF16, MODE_GN>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_GN_NC) return launch_pass_t<DT_DEPTH_BF16, MODE_GN_NC>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    return hipErrorInvalidValue;
  }
  if (dtype == S3A_F32) {
    if (mode == MODE_MOMENTS) return launch_pass_t<S3A_F32, MODE_MOMENTS>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_GN) return launch_pass_t<S3A_F32, MODE_GN>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_GN_NC) return launch_pass_t<S3A_F32, MODE_GN_NC>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_COST) return launch_pass_t<S3A_F32, MODE_COST>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
  } else {
    if (mode == MODE_MOMENTS) return launch_pass_t<S3A_BF16, MODE_MOMENTS>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_GN) return launch_pass_t<S3A_BF16, MODE_GN>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_GN_NC) return launch_pass_t<S3A_BF16, MODE_GN_NC>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
    if (mode == MODE_COST) return launch_pass_t<S3A_BF16, MODE_COST>(lc, sh, cd, w, tile_lo, tile_hi, grid, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_sched(const Shape& sh, const CallDesc& c, CallDesc* cd, const Work& w, hipStream_t st) {
  if (sh.n_pairs <= SCHED_PAIRS) {
    const int64_t most = sh.n_points / sh.tile_elems + 2 * (int64_t)sh.n_pairs + 1;
    const int grid = (int)std::max<int64_t>((sh.n_pairs + SCHED_WG - 1) / SCHED_WG,
                                            std::min<int64_t>((most + SCHED_WG - 1) / SCHED_WG, 256));
    hipLaunchKernelGGL(k_sched_tiles, dim3(grid), dim3(SCHED_WG), 0, st, sh, c, cd, w);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_sched, dim3(1), dim3(1024), 0, st, sh, c, cd, w);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sched_fill, dim3((sh.n_pairs + 255) / 256), dim3(256), 0, st, sh, c.depth, w);
  if ((e = hipGetLastError()) != hipSuccess || !c.depth) return e;
  hipLaunchKernelGGL(k_depth_prep, dim3((sh.n_pairs + 63) / 64), dim3(64), 0, st, sh, cd, w);
  return hipGetLastError();
}

template <int DT, int ITEMS>
static hipError_t launch_pass_solve_t(int mode, const Shape& sh, const CallDesc* cd, const Work& w, int pass, int grid,
                                      hipStream_t st) {
#define S3A_SOLVE(MODE, FIRST) \
  hipLaunchKernelGGL((k_pass_solve<DT, MODE, 256, ITEMS, FIRST>), dim3(grid), dim3(256), 0, st, sh, cd, w, pass)
  if (mode == MODE_GN && pass == 1) S3A_SOLVE(MODE_GN, true);
  else if (mode == MODE_GN) S3A_SOLVE(MODE_GN, false);
  else if (pass == 1) S3A_SOLVE(MODE_GN_NC, true);
  else S3A_SOLVE(MODE_GN_NC, false);
#undef S3A_SOLVE
  return hipGetLastError();
}

hipError_t launch_pass_solve(int dtype, const Shape& sh, const CallDesc* cd, const Work& w, int pass, int grid,
                             hipStream_t st) {
  const int mode = pass_mode(pass, sh.K);
  if (dtype == S3A_F32) return launch_pass_solve_t<S3A_F32, 4>(mode, sh, cd, w, pass, grid, st);
  if (dtype == S3A_BF16) return launch_pass_solve_t<S3A_BF16, 2>(mode, sh, cd, w, pass, grid, st);
  if (dtype == DT_DEPTH_F32) return launch_pass_solve_t<DT_DEPTH_F32, 16>(mode, sh, cd, w, pass, grid, st);
  return launch_pass_solve_t<DT_DEPTH_BF16, 16>(mode, sh, cd, w, pass, grid, st);
}

hipError_t launch_solve_last(const Shape& sh, const CallDesc* cd, const Work& w, int pass, hipStream_t st) {
  hipLaunchKernelGGL(k_solve_last, dim3(sh.n_pairs), dim3(256), 0, st, sh, cd, w, pass);
  return hipGetLastError();
}

hipError_t launch_finalize(const Shape& sh, const CallDesc* cd, const Work& w, int pass, int32_t pair_lo, int32_t n,
                           hipStream_t st) {
  for (int32_t k = 0; k < n; k += (int32_t)(GRID_THREADS / 256)) {
    const int32_t m = std::min(n - k, (int32_t)(GRID_THREADS / 256));
    hipLaunchKernelGGL(k_finalize, dim3(m), dim3(256), 0, st, sh, cd, w, pass, pair_lo + k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_prep(const Shape& sh, const CallDesc* cd, const Work& w, int adjoint, hipStream_t st) {
  if (sh.n_pairs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_prep, dim3((sh.n_pairs + 127) / 128), dim3(128), 0, st, sh, cd, w, adjoint);
  return hipGetLastError();
}

hipError_t launch_finalize_cost(const Shape& sh, const CallDesc* cd, const Work& w, hipStream_t st) {
  if (sh.n_pairs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_finalize_cost, dim3(sh.n_pairs), dim3(64), 0, st, sh, cd, w);
  return hipGetLastError();
}

}  // namespace s3a
