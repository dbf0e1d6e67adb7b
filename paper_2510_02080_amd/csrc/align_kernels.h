// Point passes of the dense Sim(3) alignment, its cost and its adjoint.
//
// One pass streams the seven SoA planes of every pair once and reduces
// per-point terms to NSTAT values per tile (see s3a_internal.h for the
// layout). Reads are 16-byte vectors (4 FP32 or 8 BF16 elements per plane per
// load), consecutive lanes on consecutive vectors. A tile is WG * ITEMS
// vectors of one pair; its reduction goes lane -> wavefront (butterfly) ->
// workgroup (LDS, FP64) -> one FP64 partial per tile. Per-pair totals are
// summed later over the pair's tiles in a fixed order, so results are
// bitwise reproducible run to run.
#pragma once

#include <stddef.h>

#include <type_traits>

#include "s3a_internal.h"

namespace s3a {

// ---------------------------------------------------------------- loads

template <int DT>
struct Planes;

// The planes live in global memory: loads go through global (not flat)
// address-space pointers, and are marked non-temporal. Each stored point is
// read once per pass and a pass streams far more than the caches hold, so
// keeping the lines buys nothing; on gfx950 the streaming hint lifts a
// read-only SoA sweep from about 6.2 to about 7.0 TB/s.
#if defined(__HIP_DEVICE_COMPILE__)
#define S3A_GLOBAL __attribute__((address_space(1)))
#else
#define S3A_GLOBAL
#endif
typedef float s3a_f4 __attribute__((ext_vector_type(4)));
typedef unsigned int s3a_u4 __attribute__((ext_vector_type(4)));

// What a tile's loads need besides the element index: the stored xyz planes,
// or for depth input the three planes and the tile's pair (start element and
// cameras, in uniform registers when the whole tile lies in one frame).
template <int DT>
struct SrcCtx {
  const void* const* pl;
};

struct DepthCtx {
  const void* pl[3];
  const DepthPair* dp;
  int64_t a;            // first element of the pair
  int width, rows, frame_pixels, n_frames;
  float inv_width;
  int frame;            // the tile's frame when it lies in one, else -1
  DepthCam cp, cq;      // that frame's cameras (valid when frame >= 0)
};
template <>
struct SrcCtx<DT_DEPTH_F32> : DepthCtx {};
template <>
struct SrcCtx<DT_DEPTH_BF16> : DepthCtx {};

// Stored xyz planes are read in two steps: fetch() issues one 16-byte vector
// per plane into raw registers (so a tile body can have the next vectors in
// flight while it works on the current ones), unpack() turns them into floats.
// A vector that runs past the end of the planes is gathered element by element
// (zeros past the end) into the same raw form.
typedef s3a_u4 RawVec[7];

template <>
struct Planes<S3A_F32> {
  static constexpr int VEC = 4;
  __device__ static inline void fetch(const SrcCtx<S3A_F32>& src, int64_t g0, int64_t n, RawVec& r) {
    const void* const* pl = src.pl;
    if (g0 + 4 <= n) {
#pragma unroll
      for (int j = 0; j < 7; ++j)
        r[j] = __builtin_nontemporal_load((const S3A_GLOBAL s3a_u4*)(static_cast<const uint32_t*>(pl[j]) + g0));
    } else {
#pragma unroll
      for (int j = 0; j < 7; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          r[j][e] = (g0 + e < n) ? static_cast<const uint32_t*>(pl[j])[g0 + e] : 0u;
    }
  }
  __device__ static inline void unpack(const RawVec& r, float (&v)[7][4]) {
#pragma unroll
    for (int j = 0; j < 7; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[j][e] = __uint_as_float(r[j][e]);
  }
  __device__ static inline void load(const SrcCtx<S3A_F32>& src, int64_t g0, int64_t n, float (&v)[7][4]) {
    RawVec r;
    fetch(src, g0, n, r);
    unpack(r, v);
  }
  // element e of plane j of a raw vector; its finiteness; zeroing it
  __device__ static inline float elem(const RawVec& r, int j, int e) { return __uint_as_float(r[j][e]); }
  __device__ static inline bool elem_finite(const RawVec& r, int j, int e) {
    return (r[j][e] & 0x7f800000u) != 0x7f800000u;
  }
  __device__ static inline void keep_elem(RawVec& r, int e, bool keep) {
#pragma unroll
    for (int j = 0; j < 7; ++j) r[j][e] = keep ? r[j][e] : 0u;
  }
};

template <>
struct Planes<S3A_BF16> {
  static constexpr int VEC = 8;
  __device__ static inline float lo(uint32_t u) { return __uint_as_float(u << 16); }
  __device__ static inline float hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
  __device__ static inline void fetch(const SrcCtx<S3A_BF16>& src, int64_t g0, int64_t n, RawVec& r) {
    const void* const* pl = src.pl;
    if (g0 + 8 <= n) {
#pragma unroll
      for (int j = 0; j < 7; ++j)
        r[j] = __builtin_nontemporal_load((const S3A_GLOBAL s3a_u4*)(static_cast<const uint16_t*>(pl[j]) + g0));
    } else {
#pragma unroll
      for (int j = 0; j < 7; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint16_t* h = static_cast<const uint16_t*>(pl[j]);
          const uint32_t a = (g0 + 2 * i < n) ? h[g0 + 2 * i] : 0u;
          const uint32_t b = (g0 + 2 * i + 1 < n) ? h[g0 + 2 * i + 1] : 0u;
          r[j][i] = a | (b << 16);
        }
    }
  }
  __device__ static inline void unpack(const RawVec& r, float (&v)[7][8]) {
#pragma unroll
    for (int j = 0; j < 7; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[j][2 * i] = lo(r[j][i]);
        v[j][2 * i + 1] = hi(r[j][i]);
      }
  }
  __device__ static inline void load(const SrcCtx<S3A_BF16>& src, int64_t g0, int64_t n, float (&v)[7][8]) {
    RawVec r;
    fetch(src, g0, n, r);
    unpack(r, v);
  }
  // element e (half e % 2 of word e / 2) of plane j of a raw vector; its finiteness; zeroing it
  __device__ static inline float elem(const RawVec& r, int j, int e) {
    return (e & 1) ? hi(r[j][e >> 1]) : lo(r[j][e >> 1]);
  }
  __device__ static inline bool elem_finite(const RawVec& r, int j, int e) {
    const uint32_t m = (e & 1) ? 0x7f800000u : 0x00007f80u;
    return (r[j][e >> 1] & m) != m;
  }
  __device__ static inline void keep_elem(RawVec& r, int e, bool keep) {
    const uint32_t m = (e & 1) ? 0x0000ffffu : 0xffff0000u;  // the other half
#pragma unroll
    for (int j = 0; j < 7; ++j) r[j][e >> 1] = keep ? r[j][e >> 1] : (r[j][e >> 1] & m);
  }
};

// Walk the lane's vectors of a tile: item it = 0 .. ITEMS-1 starts at element
// rel0 = (it * WG + lane) * VEC after the tile's first. Two raw buffers
// alternate: the next item's loads are issued before the current item is
// worked on, so every wavefront keeps loads in flight while it computes.
// fetch(rel, raw) issues the loads of the vector at rel; body(raw, rel0)
// consumes one. ITEMS is even. A lane runs the items with rel0 < end_rel. BEGUN:
// the caller has issued the first item's loads into A (pipelined_begin) some time
// before, to cover other latency with them.
template <int WG, int VEC, typename Raw, typename Fetch>
__device__ inline void pipelined_begin(int end_rel, Fetch&& fetch, Raw& A) {
  const int first = (int)threadIdx.x * VEC;
  if (first < end_rel) fetch(first, A);
}
template <int WG, int ITEMS, int VEC, typename Raw, bool BEGUN, typename Fetch, typename Body>
__device__ inline void pipelined_walk(int end_rel, Fetch&& fetch, Body&& body, Raw& A) {
  static_assert(ITEMS % 2 == 0, "items per lane must be even");
  constexpr int STRIDE = WG * VEC;
  Raw B;
  const int first = (int)threadIdx.x * VEC;
  if (first >= end_rel) return;
  if constexpr (!BEGUN) fetch(first, A);
#pragma unroll 1
  for (int it = 0; it < ITEMS; it += 2) {
    const int r0 = first + it * STRIDE;
    const int r1 = r0 + STRIDE;
    const bool more1 = r1 < end_rel;
    if (more1) fetch(r1, B);
    body(A, r0);
    if (!more1) break;
    const int r2 = r1 + STRIDE;
    const bool more2 = it + 2 < ITEMS && r2 < end_rel;
    if (more2) fetch(r2, A);
    body(B, r1);
    if (!more2) break;
  }
}
template <int WG, int ITEMS, int VEC, typename Raw, typename Fetch, typename Body>
__device__ inline void pipelined_items(int end_rel, Fetch&& fetch, Body&& body) {
  Raw A;
  pipelined_walk<WG, ITEMS, VEC, Raw, false>(end_rel, fetch, body, A);
}

// The walk of a full tile (every lane runs every item, every vector in bounds): the
// next items' loads have no branch around them, so that the wait before an item
// covers its own loads only (where a path may skip a load the compiler waits for
// everything in flight, and a wavefront's next loads do not overlap its work). The
// last item's loads are issued once more in place of those past the end.
template <int WG, int ITEMS, int VEC, typename Raw, bool BEGUN, typename Fetch, typename Body>
__device__ inline void full_walk(Fetch&& fetch, Body&& body, Raw& A) {
  static_assert(ITEMS % 2 == 0, "two buffers in turn");
  constexpr int STRIDE = WG * VEC;
  const int first = (int)threadIdx.x * VEC;
  Raw B;
  if constexpr (!BEGUN) fetch(first, A);
#pragma unroll 1
  for (int it = 0; it < ITEMS; it += 2) {
    const int r = first + it * STRIDE;
    fetch(r + STRIDE, B);
    body(A, r);
    fetch(it + 2 < ITEMS ? r + 2 * STRIDE : r + STRIDE, A);
    body(B, r + STRIDE);
  }
}

// Gradients are written once and not read back by the library: streaming
// (non-temporal) global stores.
__device__ inline void store_grad_vec(float* base, int64_t g0, int64_t n, const float* v, int VEC, int64_t lo,
                                 int64_t hi) {
  if (!base) return;
  if (g0 >= lo && g0 + VEC <= hi && g0 + VEC <= n) {
    for (int e = 0; e < VEC; e += 4) {
      const s3a_f4 x = {v[e], v[e + 1], v[e + 2], v[e + 3]};
      __builtin_nontemporal_store(x, (S3A_GLOBAL s3a_f4*)(base + g0 + e));
    }
  } else {
    for (int e = 0; e < VEC; ++e) {
      const int64_t g = g0 + e;
      if (g >= lo && g < hi && g < n) base[g] = v[e];
    }
  }
}

// A gradient pass's last act where the caller asked for it (SHAPE_ZERO_REST): the
// entries outside every pair's range, which no tile writes, become zero. Ranges that
// passed the schedule's check are joined end to end, so these are [0, a) and [b, n),
// usually nothing; else every pair's range is empty and all entries are. (Clearing the
// planes beforehand wrote them twice: 50 us of 13 M points' seven planes.)
__device__ inline void zero_rest(const Shape& sh, const Work& w, float* const (&gout)[7]) {
  if (!(sh.flags & SHAPE_ZERO_REST)) return;
  const int64_t a = w.sched[0].a, b = w.sched[sh.n_pairs - 1].b, rest = sh.n_points - (b - a);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rest; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t g = i < a ? i : i + (b - a);
#pragma unroll
    for (int j = 0; j < 7; ++j)
      if (gout[j]) gout[j][g] = 0.0f;
  }
}

__device__ inline float max3_abs(float x, float y, float z) { return fmaxf(fmaxf(fabsf(x), fabsf(y)), fabsf(z)); }

// Whether a lane of a moments pass has met a point whose largest value `size` (NaN
// apart) lies in [from, infinity): the bits of such a size, less from's, are the
// small unsigned numbers, whose least is kept. (Counted by masks instead, the moments of
// 256 depth pairs took 225 us against 187.)
struct ExtremeSeen {
  float from;
  uint32_t least = ~0u;
  __device__ inline void look(bool in, float size) {
    const uint32_t u = __float_as_uint(size) - __float_as_uint(from);
    least = min(least, in ? u : ~0u);
  }
  // (In the persistent launch the pair's solve is in the same launch: the flag is out
  // before the workgroup's barrier and arrival.)
  __device__ inline void mark(int32_t* flag) const {
    if (least >= __float_as_uint(__builtin_inff()) - __float_as_uint(from)) return;
    __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence();
  }
};

__device__ inline bool finite7(const float* x) {
  bool f = true;
#pragma unroll
  for (int j = 0; j < 7; ++j) f = f && __builtin_isfinite(x[j]);
  return f;
}

// ---------------------------------------------------------------- uniform parameters

// The per-pair parameters are the same for every lane of a tile: read them
// once and keep them in scalar registers.
__device__ inline float uniform_f32(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
__device__ inline int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline double uniform_f64(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ inline PointParams load_params(const PointParams* p) {
  PointParams r;
#pragma unroll
  for (int i = 0; i < 9; ++i) { r.M[i] = uniform_f64(p->M[i]); r.Mf[i] = uniform_f32(p->Mf[i]); }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    r.t[i] = uniform_f64(p->t[i]);
    r.c[i] = uniform_f64(p->c[i]);
    r.tcf[i] = uniform_f32(p->tcf[i]);
    r.cf[i] = uniform_f32(p->cf[i]);
  }
  r.inv_C = uniform_f32(p->inv_C);
  r.scale = uniform_f32(p->scale);
  r.L = uniform_f32(p->L);
  r.active = uniform_i32(p->active);
  r.mask = uniform_i32(p->mask);
  return r;
}

__device__ inline TileDesc load_tile(const TileDesc* p) {
  TileDesc r;
  const long long b = p->begin, e = p->end, l = p->lo;
  r.begin = ((long long)(unsigned)uniform_i32((int)(b >> 32)) << 32) | (unsigned)uniform_i32((int)b);
  r.end = ((long long)(unsigned)uniform_i32((int)(e >> 32)) << 32) | (unsigned)uniform_i32((int)e);
  r.lo = ((long long)(unsigned)uniform_i32((int)(l >> 32)) << 32) | (unsigned)uniform_i32((int)l);
  r.pair = uniform_i32(p->pair);
  r.tile0 = uniform_i32(p->tile0);
  r.ntiles = uniform_i32(p->ntiles);
  static_assert(offsetof(TileDesc, head) == offsetof(TileDesc, frame) + 2, "read as one word");
  int at;
  __builtin_memcpy(&at, &p->frame, sizeof(at));
  at = uniform_i32(at);
  r.frame = (int16_t)at;
  r.head = (int16_t)(at >> 16);
  return r;
}

// Depth input: three planes (d_p, d_q, c), the pixel's frame, row and column
// from its index in the pair, and each side unprojected with its camera:
// x = R (d ((col, row) * inv_f + o, 1)) + t. Elements before the pair's start
// (the head of a boundary vector) count back from its first pixel; the tile bodies
// mask them.
__device__ inline DepthCam load_cam_uniform(const DepthCam* c) {
  DepthCam r;
  r.ifx = uniform_f32(c->ifx);
  r.ify = uniform_f32(c->ify);
  r.ox = uniform_f32(c->ox);
  r.oy = uniform_f32(c->oy);
#pragma unroll
  for (int i = 0; i < 9; ++i) r.R[i] = uniform_f32(c->R[i]);
#pragma unroll
  for (int i = 0; i < 3; ++i) r.t[i] = uniform_f32(c->t[i]);
  return r;
}

// q = floor(x / m) for 0 <= x < 2^31, m >= 1 and quotients below 2^22: a float estimate,
// corrected (unsigned: the next multiple may pass 2^31).
__device__ inline int div_floor(int x, int m, float inv_m) {
  const unsigned ux = (unsigned)x, um = (unsigned)m;
  unsigned q = (unsigned)((float)x * inv_m);
  q -= (q * um > ux) ? 1u : 0u;
  q += ((q + 1u) * um <= ux) ? 1u : 0u;
  q -= (q * um > ux) ? 1u : 0u;
  return (int)q;
}

// floor(x / m) for x of either sign (an element before the frame's first counts back)
__device__ inline int row_of(int x, int m, float inv_m) { return x < 0 ? ~div_floor(~x, m, inv_m) : div_floor(x, m, inv_m); }

template <int DT>
struct DepthPlanes {
  static constexpr bool BF = DT == DT_DEPTH_BF16;
  static constexpr int VEC = BF ? 8 : 4;
  // Loads in two steps, as the stored planes' (see RawVec): d[0], d[1], d[2] = d_p, d_q,
  // c of elements g0 .. g0 + VEC - 1 (0 past n)
  typedef s3a_u4 Raw[3];
  __device__ static inline void fetch(const SrcCtx<DT>& s, int64_t g0, int64_t n, Raw& r) {
    if (g0 + VEC <= n) {
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if constexpr (BF)
          r[j] = __builtin_nontemporal_load((const S3A_GLOBAL s3a_u4*)(static_cast<const uint16_t*>(s.pl[j]) + g0));
        else
          r[j] = __builtin_nontemporal_load((const S3A_GLOBAL s3a_u4*)(static_cast<const uint32_t*>(s.pl[j]) + g0));
      }
    } else {
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (BF) {
            const uint16_t* h = static_cast<const uint16_t*>(s.pl[j]);
            const uint32_t a = (g0 + 2 * i < n) ? h[g0 + 2 * i] : 0u;
            const uint32_t b = (g0 + 2 * i + 1 < n) ? h[g0 + 2 * i + 1] : 0u;
            r[j][i] = a | (b << 16);
          } else {
            r[j][i] = (g0 + i < n) ? static_cast<const uint32_t*>(s.pl[j])[g0 + i] : 0u;
          }
        }
    }
  }
  // element rel of a tile from begin, every element in bounds (uniform bases and a
  // 32-bit offset a lane)
  __device__ static inline void fetch_full(const SrcCtx<DT>& s, int64_t begin, int rel, Raw& r) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const S3A_GLOBAL char* p = (const S3A_GLOBAL char*)s.pl[j] + begin * (BF ? 2 : 4);
      r[j] = __builtin_nontemporal_load((const S3A_GLOBAL s3a_u4*)(p + (unsigned)rel * (BF ? 2u : 4u)));
    }
  }
  __device__ static inline void unpack(const Raw& r, float (&d)[3][VEC]) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (BF) {
          d[j][2 * i] = __uint_as_float(r[j][i] << 16);
          d[j][2 * i + 1] = __uint_as_float(r[j][i] & 0xffff0000u);
        } else {
          d[j][i] = __uint_as_float(r[j][i]);
        }
      }
  }
};

template <>
struct Planes<DT_DEPTH_F32> : DepthPlanes<DT_DEPTH_F32> {};
template <>
struct Planes<DT_DEPTH_BF16> : DepthPlanes<DT_DEPTH_BF16> {};

// The load context of a tile (see SrcCtx).
template <int DT>
__device__ inline SrcCtx<DT> make_src(const void* const* pl, const Work& w, const TileDesc& td) {
  if constexpr (DT == DT_DEPTH_F32 || DT == DT_DEPTH_BF16) {
    SrcCtx<DT> s;
    s.pl[0] = pl[0];
    s.pl[1] = pl[1];
    s.pl[2] = pl[2];
    s.dp = w.dpairs + td.pair;
    s.a = td.lo;
    s.width = uniform_i32(s.dp->width);
    s.rows = uniform_i32(s.dp->rows);
    s.frame_pixels = uniform_i32(s.dp->frame_pixels);
    s.n_frames = uniform_i32(s.dp->n_frames);
    s.inv_width = uniform_f32(s.dp->inv_width);
    s.frame = td.frame;
    if (s.frame >= 0) {
      s.cp = load_cam_uniform(s.dp->p + s.frame);
      s.cq = load_cam_uniform(s.dp->q + s.frame);
    }
    return s;
  } else {
    (void)w;
    (void)td;
    return SrcCtx<DT>{pl};
  }
}

// ---------------------------------------------------------------- per-point terms

// Residual r = s R p + t - q and centred model point y_c = s R p + t - c,
// formed in FP64 (so that r keeps full FP32 relative precision however far
// the points are from the origin), then rounded to FP32.
__device__ inline void residual(const PointParams& P, const float* x, float (&r)[3], float (&yc)[3]) {
  const double p0 = x[0], p1 = x[1], p2 = x[2];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double y = fma(P.M[3 * i], p0, fma(P.M[3 * i + 1], p1, fma(P.M[3 * i + 2], p2, P.t[i])));
    r[i] = (float)(y - (double)x[3 + i]);
    yc[i] = (float)(y - P.c[i]);
  }
}

// Cost at S: 0 sum w, 1 sum w rho, 2 V (FP64 per lane).
__device__ inline void point_cost(double (&a)[3], const PointParams& P, float* x, bool in, float tau,
                                  float delta) {
  const bool valid = in && finite7(x) && x[6] >= tau;
  if (!valid) {
#pragma unroll
    for (int j = 0; j < 7; ++j) x[j] = 0.0f;
  }
  float r[3], y[3];
  residual(P, x, r, y);
  const float e2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
  float rho;
  if (e2 <= delta * delta) rho = 0.5f * e2;
  else rho = delta * (e2 * rsqrtf(e2) - 0.5f * delta);
  a[0] += (double)x[6];
  a[1] = fma((double)x[6], (double)rho, a[1]);
  a[2] += valid ? 1.0 : 0.0;
}

// ---------------------------------------------------------------- reductions

template <typename T>
__device__ inline T wave_sum(T v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// FP32 sums over the 64 lanes of a wavefront with DPP row operations (a fixed
// pairwise tree: neighbours within quads, half rows, rows, then across rows;
// the total ends in lane 63). All NSTAT sums advance one step at a time, so
// consecutive DPP operations never read a register written just before.
template <int N>
__device__ inline void wave_totals_f32(float (&v)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j)  // quad_perm [1,0,3,2]
    v[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), 0xb1, 0xf, 0xf, false));
#pragma unroll
  for (int j = 0; j < N; ++j)  // quad_perm [2,3,0,1]
    v[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), 0x4e, 0xf, 0xf, false));
#pragma unroll
  for (int j = 0; j < N; ++j)  // row_half_mirror
    v[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), 0x141, 0xf, 0xf, false));
#pragma unroll
  for (int j = 0; j < N; ++j)  // row_mirror
    v[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), 0x140, 0xf, 0xf, false));
#pragma unroll
  for (int j = 0; j < N; ++j)  // row_bcast:15 into rows 1 and 3
    v[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), 0x142, 0xa, 0xf, false));
#pragma unroll
  for (int j = 0; j < N; ++j)  // row_bcast:31 into rows 2 and 3
    v[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), 0x143, 0xc, 0xf, false));
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[j]), 63));
}

// Reduce NSTAT per-lane FP32 values over the workgroup (DPP within a
// wavefront, then FP64 across wavefronts through LDS) and store one FP64
// partial.
template <int WG>
__device__ inline void block_store_f32(float (&acc)[NSTAT], double (*red)[NSTAT], double* out) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  wave_totals_f32(acc);
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < NSTAT; ++j) red[wv][j] = (double)acc[j];
  }
  __syncthreads();
  if ((int)threadIdx.x < NSTAT) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < WG / 64; ++q) s += red[q][threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

// One DPP step on a double: both 32-bit halves move with the same control.
template <int CTRL, int ROWS>
__device__ inline double dpp_f64(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// FP64 sums over the 64 lanes of a wavefront: the same fixed DPP tree as the
// FP32 reduction above, advanced step-major over the N sums; every lane ends
// with the totals (read from lane 63).
template <int N>
__device__ inline void wave_totals_f64(double (&v)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] += dpp_f64<0xb1, 0xf>(v[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] += dpp_f64<0x4e, 0xf>(v[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] += dpp_f64<0x141, 0xf>(v[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] += dpp_f64<0x140, 0xf>(v[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] += dpp_f64<0x142, 0xa>(v[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] += dpp_f64<0x143, 0xc>(v[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v[j]);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 63);
    v[j] = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
  }
}

// Reduce N <= NSTAT per-lane FP64 values over the workgroup (DPP within a
// wavefront, then across wavefronts through LDS) and store N FP64 sums.
template <int WG, int N>
__device__ inline void block_store_f64(double (&acc)[N], double (*red)[NSTAT], double* out) {
  static_assert(N <= NSTAT, "too many sums");
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  wave_totals_f64(acc);
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < N; ++j) red[wv][j] = acc[j];
  }
  __syncthreads();
  if ((int)threadIdx.x < N) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < WG / 64; ++q) s += red[q][threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

// ---------------------------------------------------------------- tile bodies

// One point of the Gauss-Newton statistics: centred model point y, residual
// r, weight w (0 for masked points); Huber weight branch-free. COST: also the
// cost and inlier count (statistics 17 and 18), which only the pass at the
// last linearisation point reports; the other passes leave them at zero.
template <bool COST = true>
__device__ inline void gn_point(float (&a)[NSTAT], float y0, float y1, float y2, float r0, float r1, float r2, float w,
                                float d2, float delta, float hd2) {
  const float e2 = fmaf(r0, r0, fmaf(r1, r1, r2 * r2));
  const float ie = __builtin_amdgcn_rsqf(e2);
  const bool inl = e2 <= d2;
  const float psi = inl ? 1.0f : delta * ie;
  const float om = w * psi;
  const float oy0 = om * y0, oy1 = om * y1, oy2 = om * y2;
  a[0] += om;
  a[1] += oy0; a[2] += oy1; a[3] += oy2;
  a[4] = fmaf(oy0, y0, a[4]); a[5] = fmaf(oy0, y1, a[5]); a[6] = fmaf(oy0, y2, a[6]);
  a[7] = fmaf(oy1, y1, a[7]); a[8] = fmaf(oy1, y2, a[8]); a[9] = fmaf(oy2, y2, a[9]);
  a[10] = fmaf(om, r0, a[10]); a[11] = fmaf(om, r1, a[11]); a[12] = fmaf(om, r2, a[12]);
  a[13] = fmaf(oy1, r2, fmaf(-oy2, r1, a[13]));
  a[14] = fmaf(oy2, r0, fmaf(-oy0, r2, a[14]));
  a[15] = fmaf(oy0, r1, fmaf(-oy1, r0, a[15]));
  a[16] = fmaf(oy0, r0, fmaf(oy1, r1, fmaf(oy2, r2, a[16])));
  if constexpr (COST) {
    const float rho = inl ? 0.5f * e2 : fmaf(delta * e2, ie, -hd2);
    a[17] = fmaf(w, rho, a[17]);
    a[18] += (inl && w > 0.0f) ? 1.0f : 0.0f;
  }
}

// Pixel positions of a lane's vectors in a depth tile that lies in one frame, and
// what a row shares. A pixel's ray is affine in its column, so for a camera form
// (G, f): G0 (col ifx + ox) + [G1 (row ify + oy) + G2], the bracket is one value a row
// and component. The walk keeps (row, col) of the vector's first pixel and steps it
// by the lane stride; a vector crosses at most one row end (frames at least a vector
// wide). Every product and sum is the one that a pixel on its own would form, so
// sharing a row changes no bit. Elements before the pair count back from its first
// row (their values are masked).
template <int DT>
struct DepthWalk {
  int row, col, drow, dcol, width;
  __device__ inline DepthWalk(const SrcCtx<DT>& s, const TileDesc& td, int first, int stride) {
    width = s.width;
    const int j = (int)(td.begin + first - td.lo - (int64_t)s.frame * s.frame_pixels);
    row = row_of(j, width, s.inv_width);
    col = j - row * width;
    drow = uniform_i32(div_floor(stride, width, s.inv_width));
    dcol = stride - drow * width;
  }
  __device__ inline void next() {
    row += drow;
    col += dcol;
    if (col >= width) {
      col -= width;
      ++row;
    }
  }
};

// A value kept in a vector register: an operation reads one scalar register, so of
// two uniform operands the compiler would copy one for every pixel.
__device__ inline float in_vgpr(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

// A camera form: G (rows of three) with its column's intrinsics, ray_i = G_i0 rx + h_i.
struct CamForm {
  float g0[3], g1[3], g2[3], ifx, ox, ify, oy;
  __device__ inline CamForm(const float* G, const DepthCam& c) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      g0[i] = uniform_f32(G[3 * i]);
      g1[i] = uniform_f32(G[3 * i + 1]);
      g2[i] = in_vgpr(G[3 * i + 2]);
    }
    ifx = c.ifx;
    ox = in_vgpr(c.ox);
    ify = c.ify;
    oy = in_vgpr(c.oy);
  }
  // the row's share of the ray
  __device__ inline void row(float r, float (&h)[3]) const {
    const float ry = fmaf(r, ify, oy);
#pragma unroll
    for (int i = 0; i < 3; ++i) h[i] = fmaf(g1[i], ry, g2[i]);
  }
};

// Calls pixel(e, hp, hq, col) for the VEC pixels from (row, col), hp and hq the
// row shares of the forms: one row's where no lane of the wavefront crosses a row
// end, else the first or the next row's, chosen per pixel. NARROW: frames narrower than a
// vector too, where each pixel forms its own row's share.
template <int VEC, bool NARROW = false, typename Pixel>
__device__ inline void walk_pixels(int row, int col, int width, const CamForm& P, const CamForm& Q, Pixel&& pixel) {
  float hp[3], hq[3];
  const float fr = (float)row, fc = (float)col;
  P.row(fr, hp);
  Q.row(fr, hq);
  const bool cross = col > width - VEC;
  if (__builtin_amdgcn_ballot_w64(cross) == 0ull) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) pixel(e, hp, hq, fc + (float)e);
  } else if (NARROW && width < VEC) {
    int r = row, c = col;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      P.row((float)r, hp);
      Q.row((float)r, hq);
      pixel(e, hp, hq, (float)c);
      if (++c == width) {
        c = 0;
        ++r;
      }
    }
  } else {
    float hp1[3], hq1[3];
    P.row(fr + 1.0f, hp1);
    Q.row(fr + 1.0f, hq1);
    const float fw = (float)width;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const bool over = col >= width - e;
      float sp[3], sq[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        sp[i] = over ? hp1[i] : hp[i];
        sq[i] = over ? hq1[i] : hq[i];
      }
      pixel(e, sp, sq, over ? fc + (float)e - fw : fc + (float)e);
    }
  }
}

// A depth tile that spans frames: point(x, in) takes (p, q, c) of each element in the
// pair's submap frames, frame after frame, each lane's elements in order (in: the
// element lies in the tile, the pair and the frame at hand; a vector that holds a
// frame's end comes once with each). Frames of a few thousand pixels put every tile
// here. Bound by issue: with cameras and rows taken per segment instead of per element,
// 150 pairs of one to three 160 x 120 BF16 frames 722 -> 413 us a call, 60 pairs of
// 300 x 200 779 -> 475, and 256 pairs of 518 x 392 FP32, whose last tiles these are,
// 1863 -> 1681. So are frames narrower than a vector (13 M pixels in rows of 1 to 3,
// FP32, 700 us a call; an element at a time 1118, 615 when the one-frame walk took them
// element-wise too; BF16 rows of 1 to 7 590, 1185 and 670).
template <int DT, int WG, int ITEMS, typename Point>
__device__ inline void span_walk(const Shape& sh, const SrcCtx<DT>& s, const TileDesc& td, Point&& point) {
  using L = DepthPlanes<DT>;
  constexpr int VEC = L::VEC, STRIDE = WG * VEC;
  const int lo_rel = td.head, end_rel = (int)(td.end - td.begin);
  const int64_t at = td.begin - s.a;
  int seg = lo_rel > 0 ? lo_rel : 0;
#pragma unroll 1
  while (seg < end_rel) {
    int f = 0;  // the frame of at + seg: a pair has few
    while (f + 1 < s.n_frames && (int64_t)(f + 1) * s.frame_pixels <= at + seg) ++f;
    const int from = (int)((int64_t)f * s.frame_pixels - at);  // where the frame starts, and ends
    const int64_t here = (int64_t)(f + 1) * s.frame_pixels - at;
    const int seg_end = f + 1 < s.n_frames && here < end_rel ? (int)here : end_rel;
    const DepthCam cp = load_cam_uniform(s.dp->p + f), cq = load_cam_uniform(s.dp->q + f);
    const CamForm fp(cp.R, cp), fq(cq.R, cq);
#pragma unroll 1
    for (int it = seg / STRIDE; it * STRIDE < seg_end; ++it) {
      const int rel0 = (it * WG + (int)threadIdx.x) * VEC;
      if (rel0 >= seg_end || rel0 + VEC <= seg) continue;
      typename L::Raw r;
      L::fetch(s, td.begin + rel0, sh.n_points, r);
      float d[3][VEC];
      L::unpack(r, d);
      const int j = rel0 - from;  // above -VEC: the vector may begin in the frame before
      const int row = row_of(j, s.width, s.inv_width);
      walk_pixels<VEC, true>(row, j - row * s.width, s.width, fp, fq,
                       [&](int e, const float (&hp)[3], const float (&hq)[3], float fc) {
        const float rxp = fmaf(fc, fp.ifx, fp.ox), rxq = fmaf(fc, fq.ifx, fq.ox);
        float x[7];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          x[i] = fmaf(d[0][e], fmaf(fp.g0[i], rxp, hp[i]), cp.t[i]);
          x[3 + i] = fmaf(d[1][e], fmaf(fq.g0[i], rxq, hq[i]), cq.t[i]);
        }
        x[6] = d[2][e];
        point(x, rel0 + e >= seg && rel0 + e < seg_end);
      });
    }
    seg = seg_end;
  }
}

// The raw buffers of a tile's walk, whatever the input kind.
template <int DT>
struct TileRaw {
  typedef RawVec type;
};
template <>
struct TileRaw<DT_DEPTH_F32> {
  typedef DepthPlanes<DT_DEPTH_F32>::Raw type;
};
template <>
struct TileRaw<DT_DEPTH_BF16> {
  typedef DepthPlanes<DT_DEPTH_BF16>::Raw type;
};

// Issue the loads of the lane's first vector of a tile (before its cameras are known).
template <int DT, int WG>
__device__ inline void tile_begin(const Shape& sh, const void* const* pl, const TileDesc& td,
                                  typename TileRaw<DT>::type& r) {
  using Raw = typename TileRaw<DT>::type;
  SrcCtx<DT> src;
  if constexpr (DT == DT_DEPTH_F32 || DT == DT_DEPTH_BF16) {
    if (td.frame < 0) return;  // a tile that spans frames does not walk raw vectors
    for (int j = 0; j < 3; ++j) src.pl[j] = pl[j];
  } else {
    src.pl = pl;
  }
  pipelined_begin<WG, Planes<DT>::VEC, Raw>(
      (int)(td.end - td.begin), [&](int rel, Raw& x) { Planes<DT>::fetch(src, td.begin + rel, sh.n_points, x); }, r);
}

// Gauss-Newton pass over a depth tile that lies in one frame: the pair's
// current similarity is folded into each side's camera once per tile, so a
// pixel costs one affine map per side on its ray:
//   y_c = d_p (A ray_p) + b,  A = sR R_p, b = sR t_p + t - c;   q_c = d_q (R_q ray_q) + t_q - c.
// Bound by instruction issue, not by the loads: 65 vector operations a pixel in the compiled
// loop, 71 where a row ends in the vector, four cycles each on a SIMD, are 1.6 to 1.7 us a
// million pixels for the chip at its clock, and the loads alone as long. Forming a row's share of the ray, the positions and the
// masks once a vector, and the fourth wavefront per SIMD that the saved registers give:
// 256 pairs of 518 x 392 frames (62 M pixels) 169 -> 159 us a pass (140
// since extreme pairs have a walk of their own, by the registers it leaves); a few pairs, bound
// by one wavefront's chain, 345 -> 200 us a call of 10 steps.
template <int DT, int WG, int ITEMS, bool COST, bool BEGUN>
__device__ inline void tile_gn_depth_frame(const Shape& sh, const SrcCtx<DT>& src, const TileDesc& td,
                                           const PointParams& P, typename DepthPlanes<DT>::Raw& first,
                                           float (&a)[NSTAT]) {
  using L = DepthPlanes<DT>;
  constexpr int VEC = L::VEC;
  const DepthCam& cp = src.cp;
  const DepthCam& cq = src.cq;
  float A[9], b[3], bq[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
      A[3 * i + j] = fmaf(P.Mf[3 * i], cp.R[j], fmaf(P.Mf[3 * i + 1], cp.R[3 + j], P.Mf[3 * i + 2] * cp.R[6 + j]));
    b[i] = uniform_f32(fmaf(P.Mf[3 * i], cp.t[0], fmaf(P.Mf[3 * i + 1], cp.t[1], fmaf(P.Mf[3 * i + 2], cp.t[2], P.tcf[i]))));
    bq[i] = uniform_f32(cq.t[i] - P.cf[i]);
  }
  const float tau = sh.tau, delta = sh.delta_f;
  const float d2 = delta * delta, hd2 = 0.5f * delta * delta;
  const int lo_rel = td.head, end_rel = (int)(td.end - td.begin);
  const bool check_finite = P.mask != MASK_NONE;
  auto fetch = [&](int rel, typename L::Raw& r) { L::fetch(src, td.begin + rel, sh.n_points, r); };
  DepthWalk<DT> pos(src, td, (int)threadIdx.x * VEC, WG * VEC);
  const CamForm fp(A, cp), fq(cq.R, cq);
  auto body = [&](const typename L::Raw& raw, int rel0) {
    float d[3][VEC];
    L::unpack(raw, d);
    // a pair's first and last vectors, and in pairs that hold any, pixels that are not
    // finite: zeroed, so of weight zero and finite. (A finite depth of 1e30 or more gives
    // a point that is not, or the pair is MASK_EXTREME and not walked here.)
    if (check_finite || rel0 < lo_rel || rel0 + VEC > end_rel) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const bool in = rel0 + e >= lo_rel && rel0 + e < end_rel && fabsf(d[0][e]) < 1e30f && fabsf(d[1][e]) < 1e30f &&
                        __builtin_isfinite(d[2][e]);
#pragma unroll
        for (int j = 0; j < 3; ++j) d[j][e] = in ? d[j][e] : 0.0f;
      }
    }
    walk_pixels<VEC>(pos.row, pos.col, pos.width, fp, fq, [&](int e, const float (&hp)[3], const float (&hq)[3], float fc) {
      const float rxp = fmaf(fc, fp.ifx, fp.ox), rxq = fmaf(fc, fq.ifx, fq.ox);
      float y[3], q[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        y[i] = fmaf(d[0][e], fmaf(fp.g0[i], rxp, hp[i]), b[i]);
        q[i] = fmaf(d[1][e], fmaf(fq.g0[i], rxq, hq[i]), bq[i]);
      }
      const float c = d[2][e];
      gn_point<COST>(a, y[0], y[1], y[2], y[0] - q[0], y[1] - q[1], y[2] - q[2], c >= tau ? c : 0.0f, d2, delta, hd2);
    });
    pos.next();
  };
  if (end_rel == WG * ITEMS * VEC && td.begin + end_rel <= sh.n_points) {
    full_walk<WG, ITEMS, VEC, typename L::Raw, BEGUN>(
        [&](int rel, typename L::Raw& r) { L::fetch_full(src, td.begin, rel, r); }, body, first);
    return;
  }
  pipelined_walk<WG, ITEMS, VEC, typename L::Raw, BEGUN>(end_rel, fetch, body, first);
}


// Gauss-Newton pass over one tile. Every quantity is formed in FP32 in
// coordinates centred on the pair's centre c (the weighted target centroid):
//   y_c = Mf p + (t - c),  q_c = q - c,  r = y_c - q_c,
// so no product or difference involves coordinates far from the data, and the
// 17 statistics (plus cost and inlier count when COST) accumulate per lane
// over the few points the lane handles in this tile (then pairwise across
// lanes, FP64 across wavefronts and tiles). Points outside the pair's range,
// below the confidence threshold, or (in pairs that hold any) with a NaN/Inf
// value get zero weight and zeroed coordinates; in pairs that hold extreme values
// (PairMask), so does every point of weight zero.
// Elements of a raw vector that lie outside the pair's range [lo_rel, end_rel),
// or (check_finite) hold a NaN/Inf in any plane, are zeroed in place: zero
// weight and zero coordinates. Both cases are rare (a pair's first and last
// vectors; pairs the moments pass found non-finite values in), so the common
// vector pays one uniform test each. check_extreme: so are
// elements of weight zero.
// APART: that test stands by itself, which takes the walks' registers from 146 to 114
// or less (BF16, 256 pairs of 32 M points: 80 -> 75 us a pass). A FP32 walk, bound by the
// loads, is a hundredth faster without the fourth wavefront (133.8 against 134.5 us), so
// there it lies inside the other; but not in the solving passes, for whose registers
// that is worse (one pair of 203,056 points: 120 us a call against 116).
template <int DT, bool APART>
__device__ inline void mask_raw(RawVec& r, int rel0, int lo_rel, int end_rel, bool check_finite, bool check_extreme,
                                float tau) {
  constexpr int VEC = Planes<DT>::VEC;
  if (rel0 < lo_rel || rel0 + VEC > end_rel) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) Planes<DT>::keep_elem(r, e, rel0 + e >= lo_rel && rel0 + e < end_rel);
  }
  if (check_finite) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      bool fin = true;
#pragma unroll
      for (int j = 0; j < 7; ++j) fin = fin && Planes<DT>::elem_finite(r, j, e);
      Planes<DT>::keep_elem(r, e, fin);
    }
    if (!APART && check_extreme) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float c = Planes<DT>::elem(r, 6, e);
        Planes<DT>::keep_elem(r, e, c >= tau && c > 0.0f);
      }
    }
  }
  if (APART && __builtin_expect(check_extreme, 0)) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float c = Planes<DT>::elem(r, 6, e);
      Planes<DT>::keep_elem(r, e, c >= tau && c > 0.0f);
    }
  }
}

template <int DT, bool COST, bool APART>
__device__ inline void gn_vector(const Shape& sh, const PointParams& P, RawVec& r, int rel0, int lo_rel,
                                 int end_rel, bool check_finite, bool check_extreme, float (&a)[NSTAT]) {
  constexpr int VEC = Planes<DT>::VEC;
  using L = Planes<DT>;
  const float tau = sh.tau, delta = sh.delta_f;
  const float d2 = delta * delta, hd2 = 0.5f * delta * delta;
  mask_raw<DT, APART>(r, rel0, lo_rel, end_rel, check_finite, check_extreme, tau);
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    const float px = L::elem(r, 0, e), py = L::elem(r, 1, e), pz = L::elem(r, 2, e);
    const float c = L::elem(r, 6, e);
    const float w = c >= tau ? c : 0.0f;
    const float y0 = fmaf(P.Mf[0], px, fmaf(P.Mf[1], py, fmaf(P.Mf[2], pz, P.tcf[0])));
    const float y1 = fmaf(P.Mf[3], px, fmaf(P.Mf[4], py, fmaf(P.Mf[5], pz, P.tcf[1])));
    const float y2 = fmaf(P.Mf[6], px, fmaf(P.Mf[7], py, fmaf(P.Mf[8], pz, P.tcf[2])));
    gn_point<COST>(a, y0, y1, y2, y0 - (L::elem(r, 3, e) - P.cf[0]), y1 - (L::elem(r, 4, e) - P.cf[1]),
                   y2 - (L::elem(r, 5, e) - P.cf[2]), w, d2, delta, hd2);
  }
}

template <int DT, int WG, int ITEMS, bool COST, bool BEGUN = false>
__device__ inline void tile_gn(const Shape& sh, const SrcCtx<DT>& pl, const TileDesc& td, const PointParams& P,
                               typename TileRaw<DT>::type& first, double (*red)[NSTAT], double* out) {
  constexpr int VEC = Planes<DT>::VEC;
  float a[NSTAT];
#pragma unroll
  for (int j = 0; j < NSTAT; ++j) a[j] = 0.0f;
  if constexpr (DT == DT_DEPTH_F32 || DT == DT_DEPTH_BF16) {
    if (P.active && pl.frame >= 0 && P.mask != MASK_EXTREME) {
      tile_gn_depth_frame<DT, WG, ITEMS, COST, BEGUN>(sh, pl, td, P, first, a);
      block_store_f32<WG>(a, red, out);
      return;
    }
  }
  if (P.active) {
    const int lo_rel = td.head, end_rel = (int)(td.end - td.begin);
    const bool check_finite = P.mask != MASK_NONE, check_extreme = P.mask == MASK_EXTREME;
    if constexpr (DT == S3A_F32 || DT == S3A_BF16) {
      auto fetch = [&](int rel, RawVec& r) { Planes<DT>::fetch(pl, td.begin + rel, sh.n_points, r); };
      auto body = [&](RawVec& r, int rel0) {
        gn_vector<DT, COST, BEGUN || DT != S3A_F32>(sh, P, r, rel0, lo_rel, end_rel, check_finite, check_extreme, a);
      };
      pipelined_walk<WG, ITEMS, VEC, RawVec, BEGUN>(end_rel, fetch, body, first);
    } else {
      // depth input whose tile spans frames, or whose pair holds extreme values: a point at a time
      const float tau = sh.tau, delta = sh.delta_f;
      const float d2 = delta * delta, hd2 = 0.5f * delta * delta;
      span_walk<DT, WG, ITEMS>(sh, pl, td, [&](float (&x)[7], bool in) {
        const bool keep = in && (!check_finite || finite7(x)) && (!check_extreme || (x[6] >= tau && x[6] > 0.0f));
#pragma unroll
        for (int j = 0; j < 7; ++j) x[j] = keep ? x[j] : 0.0f;
        const float w = x[6] >= tau ? x[6] : 0.0f;
        const float y0 = fmaf(P.Mf[0], x[0], fmaf(P.Mf[1], x[1], fmaf(P.Mf[2], x[2], P.tcf[0])));
        const float y1 = fmaf(P.Mf[3], x[0], fmaf(P.Mf[4], x[1], fmaf(P.Mf[5], x[2], P.tcf[1])));
        const float y2 = fmaf(P.Mf[6], x[0], fmaf(P.Mf[7], x[1], fmaf(P.Mf[8], x[2], P.tcf[2])));
        gn_point<COST>(a, y0, y1, y2, y0 - (x[3] - P.cf[0]), y1 - (x[4] - P.cf[1]), y2 - (x[5] - P.cf[2]), w,
                       d2, delta, hd2);
      });
    }
  }
  block_store_f32<WG>(a, red, out);
}

// Moments of a depth-input tile whose pixels all lie in one frame. Each side is
// formed in its camera's frame, x' = d (R ray) (coordinates of the size of the
// scene, so FP32 products keep their precision), the products of the VEC pixels of
// one vector are summed in FP32 and added to FP64 lane sums (the weight sum itself
// in FP64 per pixel), and the lane sums are moved to the submap frame
// (x = x' + t) once, in FP64, at the end. Bound by issue as the Gauss-Newton pass (189
// registers, two wavefronts per SIMD; a bound of three spills 130 and is no faster):
// 233 -> 194 us on the same 256 pairs, their spanning tiles walked by vectors too.
template <int DT, int WG, int ITEMS, bool BEGUN>
__device__ inline void tile_moments_depth_frame(const Shape& sh, const SrcCtx<DT>& src, const TileDesc& td,
                                                typename DepthPlanes<DT>::Raw& first,
                                                double (&a)[NSTAT], int& nvalid, int& nbad, ExtremeSeen& extreme) {
  using L = DepthPlanes<DT>;
  constexpr int VEC = L::VEC;
  const DepthCam& cp = src.cp;
  const DepthCam& cq = src.cq;
  const float tau = sh.tau;
  const int lo_rel = td.head, end_rel = (int)(td.end - td.begin);
  DepthWalk<DT> pos(src, td, (int)threadIdx.x * VEC, WG * VEC);
  const CamForm fp(cp.R, cp), fq(cq.R, cq);
  auto body = [&](const typename L::Raw& raw, int rel0) {
    float d[3][VEC];
    L::unpack(raw, d);
    float s[17];
#pragma unroll
    for (int j = 0; j < 17; ++j) s[j] = 0.0f;
    walk_pixels<VEC>(pos.row, pos.col, pos.width, fp, fq, [&](int e, const float (&hp)[3], const float (&hq)[3], float fc) {
      const bool in = rel0 + e >= lo_rel && rel0 + e < end_rel;
      const float rxp = fmaf(fc, fp.ifx, fp.ox), rxq = fmaf(fc, fq.ifx, fq.ox);
      float x[3], y[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        x[i] = d[0][e] * fmaf(fp.g0[i], rxp, hp[i]);
        y[i] = d[1][e] * fmaf(fq.g0[i], rxq, hq[i]);
      }
      const float c = d[2][e];
      const bool fin = __builtin_isfinite(x[0] + x[1] + x[2] + y[0] + y[1] + y[2]) && __builtin_isfinite(c);
      const bool valid = in && fin && c >= tau;
      nvalid += valid ? 1 : 0;
      nbad += (in && !fin) ? 1 : 0;
      extreme.look(in, fmaxf(fabsf(d[0][e]), fabsf(d[1][e])));
      const float w = valid ? c : 0.0f;
      if (!fin) {  // (a finite pixel of weight zero adds nothing whatever its coordinates)
#pragma unroll
        for (int i = 0; i < 3; ++i) x[i] = y[i] = 0.0f;
      }
      const float wx0 = w * x[0], wx1 = w * x[1], wx2 = w * x[2];
      const float wy0 = w * y[0], wy1 = w * y[1], wy2 = w * y[2];
      a[0] += (double)w;  // the weight sum stays exact
      s[1] += wx0; s[2] += wx1; s[3] += wx2;
      s[4] += wy0; s[5] += wy1; s[6] += wy2;
      s[7] = fmaf(wx0, x[0], fmaf(wx1, x[1], fmaf(wx2, x[2], s[7])));
      s[8] = fmaf(wy0, x[0], s[8]);  s[9] = fmaf(wy0, x[1], s[9]);  s[10] = fmaf(wy0, x[2], s[10]);
      s[11] = fmaf(wy1, x[0], s[11]); s[12] = fmaf(wy1, x[1], s[12]); s[13] = fmaf(wy1, x[2], s[13]);
      s[14] = fmaf(wy2, x[0], s[14]); s[15] = fmaf(wy2, x[1], s[15]); s[16] = fmaf(wy2, x[2], s[16]);
    });
    pos.next();
#pragma unroll
    for (int j = 1; j < 17; ++j) a[j] += (double)s[j];
  };
  if (end_rel == WG * ITEMS * VEC && td.begin + end_rel <= sh.n_points)
    full_walk<WG, ITEMS, VEC, typename L::Raw, BEGUN>(
        [&](int rel, typename L::Raw& r) { L::fetch_full(src, td.begin, rel, r); }, body, first);
  else
    pipelined_walk<WG, ITEMS, VEC, typename L::Raw, BEGUN>(
        end_rel, [&](int rel, typename L::Raw& r) { L::fetch(src, td.begin + rel, sh.n_points, r); }, body, first);
  // to the submap frame: x = x' + tp, y = y' + tq
  const double tp[3] = {cp.t[0], cp.t[1], cp.t[2]}, tq[3] = {cq.t[0], cq.t[1], cq.t[2]};
  const double W = a[0], Sx[3] = {a[1], a[2], a[3]}, Sy[3] = {a[4], a[5], a[6]};
  a[7] += 2.0 * (tp[0] * Sx[0] + tp[1] * Sx[1] + tp[2] * Sx[2]) + (tp[0] * tp[0] + tp[1] * tp[1] + tp[2] * tp[2]) * W;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) a[8 + 3 * i + j] += tq[i] * Sx[j] + Sy[i] * tp[j] + tq[i] * tp[j] * W;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    a[1 + i] += tp[i] * W;
    a[4 + i] += tq[i] * W;
  }
}

// Moments pass over one tile: FP64 products and per-lane FP64 sums (the
// coordinates are uncentred here, so the second moments must keep more than
// FP32 precision), integer counts, DPP wavefront reduction.
template <int DT, int WG, int ITEMS, bool BEGUN>
__device__ inline void tile_moments(const Shape& sh, const SrcCtx<DT>& pl, const TileDesc& td,
                                   typename TileRaw<DT>::type& first, double (*red)[NSTAT], double* out,
                                   int32_t* extreme_out) {
  constexpr int VEC = Planes<DT>::VEC;
  ExtremeSeen extreme{DT == DT_DEPTH_F32 || DT == DT_DEPTH_BF16 ? EXTREME / PLAIN_RAY : EXTREME};
  double a[NSTAT];
#pragma unroll
  for (int j = 0; j < NSTAT; ++j) a[j] = 0.0;
  int nvalid = 0, nbad = 0;
  const float tau = sh.tau;
  const int lo_rel = td.head, end_rel = (int)(td.end - td.begin);
  if constexpr (DT == DT_DEPTH_F32 || DT == DT_DEPTH_BF16) {
    if (pl.frame >= 0) {
      tile_moments_depth_frame<DT, WG, ITEMS, BEGUN>(sh, pl, td, first, a, nvalid, nbad, extreme);
      extreme.mark(extreme_out);
      a[17] = (double)nvalid;
      a[18] = (double)nbad;
      block_store_f64<WG, NSTAT>(a, red, out);
      return;
    }
  }
  // one point: validity (counted), then the weighted raw moments in FP64. The largest
  // coordinate tells infinities too, and a comparison a NaN in either of two, which pays for
  // looking at it (32 M BF16 points, the closed form alone: a class test per value 113 us
  // a call, with the largest beside it 120, this 110).
  auto point = [&](float (&x)[7], bool in) {
    const float size = fmaxf(max3_abs(x[0], x[1], x[2]), max3_abs(x[3], x[4], x[5]));  // NaN apart
    const bool nans =
        __builtin_isunordered(x[0], x[1]) | __builtin_isunordered(x[2], x[3]) | __builtin_isunordered(x[4], x[5]);
    const bool fin = !nans & (size < __builtin_inff()) & __builtin_isfinite(x[6]);
    const bool valid = in && fin && x[6] >= tau;
    nvalid += valid ? 1 : 0;
    nbad += (in && !fin) ? 1 : 0;
    // (a neighbour's element in a vector of stored points may be seen too: the masks it
    // brings change no sum)
    extreme.look(in || DT == S3A_F32 || DT == S3A_BF16, size);
#pragma unroll
    for (int j = 0; j < 7; ++j) x[j] = valid ? x[j] : 0.0f;
    const double w = x[6];
    const double p0 = x[0], p1 = x[1], p2 = x[2], q0 = x[3], q1 = x[4], q2 = x[5];
    const double wp0 = w * p0, wp1 = w * p1, wp2 = w * p2;
    const double wq0 = w * q0, wq1 = w * q1, wq2 = w * q2;
    a[0] += w;
    a[1] += wp0; a[2] += wp1; a[3] += wp2;
    a[4] += wq0; a[5] += wq1; a[6] += wq2;
    a[7] = fma(wp0, p0, fma(wp1, p1, fma(wp2, p2, a[7])));
    a[8] = fma(wq0, p0, a[8]);  a[9] = fma(wq0, p1, a[9]);  a[10] = fma(wq0, p2, a[10]);
    a[11] = fma(wq1, p0, a[11]); a[12] = fma(wq1, p1, a[12]); a[13] = fma(wq1, p2, a[13]);
    a[14] = fma(wq2, p0, a[14]); a[15] = fma(wq2, p1, a[15]); a[16] = fma(wq2, p2, a[16]);
  };
  if constexpr (DT == S3A_F32 || DT == S3A_BF16) {
    pipelined_items<WG, ITEMS, VEC, RawVec>(
        end_rel, [&](int rel, RawVec& r) { Planes<DT>::fetch(pl, td.begin + rel, sh.n_points, r); },
        [&](RawVec& r, int rel0) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            float x[7];
#pragma unroll
            for (int j = 0; j < 7; ++j) x[j] = Planes<DT>::elem(r, j, e);
            point(x, rel0 + e >= lo_rel && rel0 + e < end_rel);
          }
        });
  } else {
    span_walk<DT, WG, ITEMS>(sh, pl, td, point);
  }
  extreme.mark(extreme_out);
  a[17] = (double)nvalid;
  a[18] = (double)nbad;
  block_store_f64<WG, NSTAT>(a, red, out);
}

// Cost pass over one tile: sum w, sum w rho (FP64 residuals, FP64 sums), V.
template <int DT, int WG, int ITEMS>
__device__ inline void tile_cost(const Shape& sh, const SrcCtx<DT>& pl, const TileDesc& td, const PointParams& P,
                                 double (*red)[NSTAT], double* out) {
  constexpr int VEC = Planes<DT>::VEC;
  double acc[3] = {0.0, 0.0, 0.0};
  if (P.active) {
    const int lo_rel = td.head, end_rel = (int)(td.end - td.begin);
#pragma unroll 1
    for (int it = 0; it < ITEMS; ++it) {
      const int rel0 = (it * WG + (int)threadIdx.x) * VEC;
      if (rel0 >= end_rel) break;
      float v[7][VEC];
      Planes<DT>::load(pl, td.begin + rel0, sh.n_points, v);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const bool in = rel0 + e >= lo_rel && rel0 + e < end_rel;
        float x[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) x[j] = v[j][e];
        point_cost(acc, P, x, in, sh.tau, sh.delta_f);
      }
    }
  }
  block_store_f64<WG, 3>(acc, red, out);
}

// extreme: the pair's flag, which a moments pass sets. BEGUN: first holds the lane's first
// vector, its loads issued (tile_begin).
template <int DT, int MODE, int WG, int ITEMS, bool BEGUN = false>
__device__ inline void tile_body(const Shape& sh, const SrcCtx<DT>& pl, const TileDesc& td, const PointParams& P,
                                 typename TileRaw<DT>::type& first, double (*red)[NSTAT], double* out,
                                 int32_t* extreme = nullptr) {
  if constexpr (MODE == MODE_GN || MODE == MODE_GN_NC) {
    tile_gn<DT, WG, ITEMS, MODE == MODE_GN, BEGUN>(sh, pl, td, P, first, red, out);
  } else if constexpr (MODE == MODE_MOMENTS) {
    tile_moments<DT, WG, ITEMS, BEGUN>(sh, pl, td, first, red, out, extreme);
  } else {
    static_assert(MODE == MODE_COST, "unknown pass mode");
    tile_cost<DT, WG, ITEMS>(sh, pl, td, P, red, out);
  }
}

// Sum the pair's tile partials in a fixed order (lane-strided, then the fixed
// DPP tree): the same value on every run, in every lane.
__device__ inline void pair_sums(const Work& w, const PairSched& sc, int nstat, double (&s)[NSTAT]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < NSTAT; ++j) s[j] = 0.0;
  for (int t = sc.tile0 + lane; t < sc.tile0 + sc.ntiles; t += 64) {
    const double* p = w.partials + (int64_t)t * NSTAT;
#pragma unroll
    for (int j = 0; j < NSTAT; ++j)
      if (j < nstat) s[j] += p[j];
  }
  wave_totals_f64(s);
}

}  // namespace s3a
