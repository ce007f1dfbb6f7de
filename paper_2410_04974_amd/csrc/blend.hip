// Per-tile alpha compositing on gfx950 (the 3D Gaussian splatting rasteriser's
// blending, Sec. 4.4): forward front-to-back with the final transmittance and
// the last contributor saved per pixel, and the reverse walk that turns dL/dI
// into per-Gaussian screen-space gradients.
//
// One workgroup of 256 threads per screen tile (forward) or per chunk of a
// tile's list (backward), one pixel per thread; each 64-lane wavefront owns an
// 8x8 block of the tile.  Each Gaussian's alpha >= 1/255 ellipse is tested
// exactly against a block before that block's pixels see it, so the
// per-pixel loop -- the kernels' critical path -- never visits a Gaussian its
// block cannot reach.  The forward's wavefronts walk the list independently
// (a tile's blocks differ in depth complexity, and a shared batch would hold
// every wavefront to the slowest); the backward stages one LDS batch for the
// workgroup and builds the four per-block lists from it.
#include <type_traits>

#include "internal.h"

namespace sixdgs {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kLog2AlphaMin = -7.994353436858858f;  // log2(1/255)
constexpr int kWaves = kBlock / 64;

// Whether a Gaussian's alpha can reach its clamp of 0.99 at some pixel.  Alpha
// is at most alpha_cond up to the rounding of the exponent, whose terms are up
// to q_max / (1 - rho^2) large (rho: the conic's correlation): below
// 1 / (1 - rho^2) = 1000 they round by under 3e-3, or 0.2% of alpha.
__device__ __forceinline__ bool may_clamp(float alpha_cond, float qxx, float qxy, float qyy) {
  return alpha_cond > 0.985f || qxy * qxy > 0.999f * qxx * qyy;
}

// Staged record: the conic pre-scaled so that alpha exp(-q/2) = exp2(p2 + log2 alpha).
struct Staged {
  float4 a;  // u, v, cA = -log2e/2 Qxx, cB = -log2e Qxy
  float4 b;  // cC = -log2e/2 Qyy, log2(alpha_cond), 1/alpha_cond (negated: may_clamp), entry id (bits)
  float4 c;  // r, g, b, -
};

__device__ __forceinline__ Staged stage(const Rec& r, uint32_t e) {
  Staged s;
  s.a = make_float4(r.a.x, r.a.y, -0.5f * kLog2e * r.a.z, -kLog2e * r.a.w);
  const float ia = __builtin_amdgcn_rcpf(r.b.y);
  s.b = make_float4(-0.5f * kLog2e * r.b.x, __log2f(r.b.y), may_clamp(r.b.y, r.a.z, r.a.w, r.b.x) ? -ia : ia,
                    __uint_as_float(e));
  s.c = make_float4(r.c.x, r.c.y, r.c.z, 0.f);
  return s;
}

// log2 of the unclamped alpha of a Gaussian at a pixel: the one evaluation both
// directions use, written with explicit roundings so both compile to the same
// arithmetic.
__device__ __forceinline__ float log2_alpha(const float4& A, const float4& B, float dx, float dy) {
  const float t = __fmaf_rn(A.z, dx, __fmul_rn(A.w, dy));
  return __fmaf_rn(t, dx, __fmaf_rn(__fmul_rn(B.x, dy), dy, B.y));
}

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }

// Does the extent box (with a one-pixel margin) reach the 8x8 block of pixel
// centres [x0, x0 + 7] x [y0, y0 + 7]?
__device__ __forceinline__ bool box_hits(const Rec& r, float x0, float y0) {
  return (r.a.x + r.b.z >= x0 - 1.0f) && (r.a.x - r.b.z <= x0 + 8.0f) && (r.a.y + r.b.w >= y0 - 1.0f) &&
         (r.a.y - r.b.w <= y0 + 8.0f);
}

// Can any pixel centre of the 8x8 block reach alpha >= 1/255, i.e. does the
// ellipse q(x) = (x - m)^T Q (x - m) <= q_max = 2 ln(255 alpha_cond) meet the
// block's rectangle of centres?  The minimum of the convex q over the
// rectangle is 0 when the centre m lies inside; otherwise it lies on an edge
// whose line separates m from the rectangle, and along an edge q is a 1D
// quadratic minimised by clamping.  A relative margin keeps the test
// conservative under float32 rounding, so it only skips Gaussians that no
// pixel of the block would take.  The margins (0.1% and 1e-3) are far wider
// than the errors of the hardware log and reciprocal used here: q_max is off
// by about 1e-7, and an edge minimiser off by a relative 1e-7 moves q by its
// square (q is flat there).
__device__ __forceinline__ bool ellipse_hits(const Rec& r, float x0, float y0) {
  if (!box_hits(r, x0, y0)) return false;
  const float qa = r.a.z, qb = r.a.w, qc = r.b.x;
  const float lim = (2.0f * kLn2) * __builtin_amdgcn_logf(255.0f * r.b.y) * 1.001f + 1e-3f;
  const float xl = x0 - r.a.x, xh = xl + 7.0f;
  const float yl = y0 - r.a.y, yh = yl + 7.0f;
  const bool inx = xl <= 0.f && xh >= 0.f, iny = yl <= 0.f && yh >= 0.f;
  if (inx && iny) return true;
  float best = 3.0e38f;
  if (!inx) {
    const float dx = xl > 0.f ? xl : xh;
    const float dy = fminf(fmaxf(-qb * dx * __builtin_amdgcn_rcpf(qc), yl), yh);
    best = fminf(best, qa * dx * dx + 2.0f * qb * dx * dy + qc * dy * dy);
  }
  if (!iny) {
    const float dy = yl > 0.f ? yl : yh;
    const float dx = fminf(fmaxf(-qb * dy * __builtin_amdgcn_rcpf(qa), xl), xh);
    best = fminf(best, qa * dx * dx + 2.0f * qb * dx * dy + qc * dy * dy);
  }
  return best <= lim;
}

__device__ __forceinline__ int find_view(const ViewTable& vt, int tile) {
  int v = 0;
  for (int k = 1; k < vt.nview; k++)
    if (tile >= vt.v[k].tile_base) v = k;
  return v;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
  return v;
}

template <int TW>
struct TileMap {
  static constexpr int TH = 256 / TW;
  static constexpr int BX = TW / 8;  // 8x8 blocks per tile row
  __device__ static int bx(int w) { return (w % BX) * 8; }
  __device__ static int by(int w) { return (w / BX) * 8; }
};

// Shared staging state of one backward batch of at most MAXB list positions.
template <int MAXB>
struct BatchLDS {
  Staged rec[MAXB];
  uint8_t list[kWaves][MAXB];     // per wavefront: staged slots in list order
  uint32_t wcnt[kWaves][kWaves];  // [block][staging wave] hits
};

// Stages pairs [b0, b0 + nb) of the tile list and builds the four per-block
// lists; returns the list length of this thread's wavefront.  Up to 128 pairs
// the two halves of the workgroup take the same pairs and two blocks each (the
// ellipse tests are most of the work), beyond every thread takes one pair and
// all four blocks.
template <int TW, int MAXB>
__device__ __forceinline__ uint32_t stage_batch(BatchLDS<MAXB>& L, const Rec* __restrict__ rec,
                                                const uint32_t* __restrict__ pval, uint32_t b0, uint32_t nb,
                                                float ox, float oy) {
  constexpr int kShare = kBlock / MAXB;        // threads per pair
  constexpr int kTests = kWaves / kShare;      // blocks per thread
  constexpr int kStageWaves = kWaves / kShare; // wavefronts over the pairs
  const int t = threadIdx.x & (MAXB - 1), lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int w0 = (int)__builtin_amdgcn_readfirstlane(wv / kStageWaves) * kTests;  // first block
  const int sw = wv % kStageWaves;
  uint32_t mask = 0;
  if ((uint32_t)t < nb) {
    const uint32_t e = pval[b0 + t];
    const Rec r = rec[e];
    if (w0 == 0) L.rec[t] = stage(r, e);
#pragma unroll
    for (int w = 0; w < kTests; w++)
      if (ellipse_hits(r, ox + TileMap<TW>::bx(w0 + w), oy + TileMap<TW>::by(w0 + w))) mask |= 1u << w;
  }
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t rank[kTests];
#pragma unroll
  for (int w = 0; w < kTests; w++) {
    const uint64_t bal = __ballot((mask >> w) & 1u);
    rank[w] = __popcll(bal & lt);
    if (lane == 0) L.wcnt[w0 + w][sw] = __popcll(bal);
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kTests; w++) {
    if ((mask >> w) & 1u) {
      uint32_t off = rank[w];
      for (int s = 0; s < sw; s++) off += L.wcnt[w0 + w][s];
      L.list[w0 + w][off] = (uint8_t)t;
    }
  }
  uint32_t cnt = 0;
#pragma unroll
  for (int s = 0; s < kStageWaves; s++) cnt += L.wcnt[wv][s];
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(cnt);  // uniform over the wavefront
}

// Forward staging: every wavefront walks the tile's list on its own, 64 list
// entries per step, keeps the Gaussians whose alpha >= 1/255 ellipse meets
// its 8x8 block, compacted in its own LDS buffer, and composites them once 64
// have gathered (or at a chunk boundary, or at the list's end).  No wavefront
// waits for another, and the loads of the next step are in flight while the
// current one is tested and blended.
constexpr int kFwdStep = 64;
constexpr int kFwdBuf = 128;  // pending hits stay below 64 before a step adds at most 64
struct FwdWaveLDS {
  float4 a[kFwdBuf];  // u, v, cA, cB
  float2 b[kFwdBuf];  // cC, log2(alpha_cond)
  float4 c[kFwdBuf];  // r, g, b, 1-based list position (bits)
};

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A pixel's running state in the forward.
struct FwdPixel {
  float T = 1.0f, C[3] = {0.f, 0.f, 0.f};
  float K[3] = {0.f, 0.f, 0.f};  // colour of the current chunk alone
  uint32_t last = 0, cnt = 0;
};

// One Gaussian of exponent p, (clamped) alpha a, colour c and 1-based list
// position pos, for the pixels of `live` that take it (p >= log2(1/255)): the
// weight a T enters the colour and T becomes T (1 - a), or the pixel stops and
// leaves `live` where that would fall below 1e-4.  Written over the execution
// mask: the two compares narrow it, so nothing after them needs a select
// (a select costs as much as a compare here, 4.3 cycles per wavefront and
// SIMD against 2.5 for the moves, products and sums).
// CHUNK: also the chunk's own colour.
template <bool SAVE, bool COUNTS, bool CHUNK>
__device__ __forceinline__ void blend_one(FwdPixel& P, uint64_t& live, float p, float a, const float4& c) {
  float Tn, w;
  uint64_t take;
  // (all lanes are active around this)
#define SIXDGS_TAKE                              \
  "s_mov_b64 exec, %[live]\n\t"                  \
  "v_cmpx_le_f32_e64 %[take], %[pmin], %[p]\n\t" \
  "v_fma_f32 %[tn], -%[T], %[a], %[T]\n\t"       \
  "v_mul_f32_e32 %[w], %[a], %[T]\n\t"           \
  "v_cmpx_le_f32_e32 vcc, %[tmin], %[tn]\n\t"    \
  "v_fmac_f32_e32 %[c0], %[r], %[w]\n\t"         \
  "v_fmac_f32_e32 %[c1], %[g], %[w]\n\t"         \
  "v_fmac_f32_e32 %[c2], %[b], %[w]\n\t"         \
  "v_mov_b32_e32 %[T], %[tn]\n\t"                \
  "s_xor_b64 %[take], %[take], vcc\n\t"          \
  "s_xor_b64 %[live], %[live], %[take]\n\t"
#define SIXDGS_END "s_mov_b64 exec, -1"
#define SIXDGS_IO                                                                                              \
  [T] "+v"(P.T), [c0] "+v"(P.C[0]), [c1] "+v"(P.C[1]), [c2] "+v"(P.C[2]), [live] "+s"(live), [take] "=&s"(take), \
      [tn] "=&v"(Tn), [w] "=&v"(w)
#define SIXDGS_IN                                                                                          \
  [p] "v"(p), [a] "v"(a), [r] "v"(c.x), [g] "v"(c.y), [b] "v"(c.z), [pmin] "s"(kLog2AlphaMin), [tmin] "s"(kTMin)
  if constexpr (!SAVE) {
    asm volatile(SIXDGS_TAKE SIXDGS_END : SIXDGS_IO : SIXDGS_IN : "vcc", "scc");
  } else if constexpr (!CHUNK) {
    asm volatile(SIXDGS_TAKE "v_mov_b32_e32 %[last], %[pos]\n\t" SIXDGS_END
                 : SIXDGS_IO, [last] "+v"(P.last)
                 : SIXDGS_IN, [pos] "v"(c.w)
                 : "vcc", "scc");
  } else {
    asm volatile(SIXDGS_TAKE
                 "v_fmac_f32_e32 %[k0], %[r], %[w]\n\t"
                 "v_fmac_f32_e32 %[k1], %[g], %[w]\n\t"
                 "v_fmac_f32_e32 %[k2], %[b], %[w]\n\t"
                 "v_mov_b32_e32 %[last], %[pos]\n\t" SIXDGS_END
                 : SIXDGS_IO, [last] "+v"(P.last), [k0] "+v"(P.K[0]), [k1] "+v"(P.K[1]), [k2] "+v"(P.K[2])
                 : SIXDGS_IN, [pos] "v"(c.w)
                 : "vcc", "scc");
  }
#undef SIXDGS_TAKE
#undef SIXDGS_END
#undef SIXDGS_IO
#undef SIXDGS_IN
  // (positions count from 1; the filler past the list has 0)
  if constexpr (COUNTS) P.cnt += P.last != 0 && P.last == __float_as_uint(c.w) ? 1u : 0u;
}

// SAVE = false renders the image only (inference): no chunk boundaries, no
// final transmittance, last contributor or chunk counts for a backward.
// COUNTS additionally counts each pixel's contributors (a debug export).
// G: Gaussians whose records a step reads and whose exponents it forms at
// once; WAVES: the wavefronts per SIMD to fit.  Bound by the vector
// instructions where there are many tiles, which more wavefronts then keep
// issuing: pairs and six wavefronts (80 registers) take 1352 us on sixteen
// uneven views of 500k Gaussians, fours and four 1506; image only, 1408x1408 of
// 12.7k Gaussians, pairs and seven 103, fours and five 107.  With few tiles the
// longest walks bound it, and a step of four shortens them: one 800x800 view of
// 300k, fours and four 134 us, pairs and six 141; 403x301 of 20k 34 and 38.
// (By selects instead of the execution mask: 1622, 110, 152 and 38 us.)
template <int TW, bool SAVE, bool COUNTS, int G, int WAVES>
__global__ void __launch_bounds__(kBlock, WAVES) k_blend_fwd(ViewTable vt, DevSettings ds, const Rec* __restrict__ rec,
                                                          const uint2* __restrict__ ranges,
                                                          const uint32_t* __restrict__ pval, BlendState bs) {
  __shared__ FwdWaveLDS W[kWaves];
  __shared__ uint32_t s_maxlast, s_ibase;
  __shared__ float s_l1[kWaves];
  const int tile = (int)bs.order[blockIdx.x];
  const int vi = find_view(vt, tile);
  const ViewDesc& vd = vt.v[vi];
  const int local = tile - vd.tile_base;
  const int tx = local % vd.ntx, ty = local / vd.ntx;
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  const float bx0 = (float)(tx * TW + TileMap<TW>::bx(wv)) + 0.5f;
  const float by0 = (float)(ty * TileMap<TW>::TH + TileMap<TW>::by(wv)) + 0.5f;
  const int px = tx * TW + TileMap<TW>::bx(wv) + (l & 7);
  const int py = ty * TileMap<TW>::TH + TileMap<TW>::by(wv) + (l >> 3);
  const bool inside = px < vd.W && py < vd.H;
  const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
  FwdWaveLDS& B = W[wv];
  const uint64_t lt = (l == 0) ? 0ull : (~0ull >> (64 - l));

  if constexpr (SAVE) {
    if (threadIdx.x == 0) s_maxlast = 0;
    __syncthreads();
  }
  const uint2 rg = ranges[tile];
  const uint32_t n = rg.y - rg.x;
  const uint32_t* pv = pval + rg.x;
  const uint32_t chunk = bs.chunk;
  FwdPixel P;
  uint32_t nbd = 0;
  uint64_t live = __ballot(inside);  // the pixels still composited
  bool opaque = false;               // a pending Gaussian may reach alpha's clamp (uniform)

  // CHUNK: the chunk's colour is wanted (past the first chunk: what lies
  // behind a boundary never includes the first)
  auto walk = [&](uint32_t nh, auto chunk_colour, auto clamp) {
    for (uint32_t g = 0; G * g < nh && live; g++) {
      float4 A[G], Cc[G];
      float2 Bq[G];
#pragma unroll
      for (int u = 0; u < G; u++) {
        A[u] = B.a[G * g + u];
        Bq[u] = B.b[G * g + u];
        Cc[u] = B.c[G * g + u];
      }
      // what does not depend on the pixel's state for all of the group first,
      // so its records are read at once
      float p[G], a[G];
#pragma unroll
      for (int u = 0; u < G; u++) {
        p[u] = log2_alpha(A[u], make_float4(Bq[u].x, Bq[u].y, 0.f, 0.f), fx - A[u].x, fy - A[u].y);
        a[u] = exp2_fast(p[u]);
        if constexpr (decltype(clamp)::value) a[u] = fminf(kAlphaMax, a[u]);
      }
#pragma unroll
      for (int u = 0; u < G; u++)
        blend_one<SAVE, COUNTS, decltype(chunk_colour)::value>(P, live, p[u], a[u], Cc[u]);
    }
  };
  auto composite = [&](uint32_t nh) {
    // the group that ends past nh would read stale slots: fill them with a
    // Gaussian no pixel takes (exponent -1e30) and a zero colour, so that
    // every slot of a group is evaluated alike
    if ((uint32_t)l < (G - nh % G) % G) {
      B.a[nh + l] = make_float4(0.f, 0.f, 0.f, 0.f);
      B.b[nh + l] = make_float2(0.f, -1e30f);
      B.c[nh + l] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    wave_lds_sync();
    using Yes = std::true_type;
    using No = std::false_type;
    if (SAVE && nbd > 0) {
      if (opaque)
        walk(nh, Yes{}, Yes{});
      else
        walk(nh, Yes{}, No{});
    } else {
      if (opaque)
        walk(nh, No{}, Yes{});
      else
        walk(nh, No{}, No{});
    }
    opaque = false;
  };

  // software pipeline: entry ids two steps ahead, records one step ahead
  // (past the list the ids stay 0, an entry that exists whenever the list is
  // not empty: every lane loads a record and the ones past the list go
  // unused, which spares zeroing the twelve registers every step)
  uint32_t e_cur = 0, e_nxt = 0;
  if ((uint32_t)l < n) e_cur = pv[l];
  if ((uint32_t)(kFwdStep + l) < n) e_nxt = pv[kFwdStep + l];
  Rec r_cur;
  if (n > 0) r_cur = rec[e_cur];
  uint32_t nh = 0;  // pending hits in B (uniform)
  for (uint32_t s0 = 0; s0 < n; s0 += kFwdStep) {
    if (!live) break;
    const Rec r_nxt = rec[e_nxt];
    uint32_t e_nn = 0;
    if (s0 + 2 * kFwdStep + l < n) e_nn = pv[s0 + 2 * kFwdStep + l];
    if (SAVE && s0 != 0 && (s0 & (chunk - 1)) == 0) {
      // a backward work item starts here: finish the chunk, then keep this
      // pixel's transmittance and the colour of the chunk that ends here
      composite(nh);
      nh = 0;
      const int64_t slot = ((int64_t)rg.x + s0) >> bs.chunk_shift;
      if (slot < bs.nbound) bs.bound[slot * kBlock + threadIdx.x] = make_float4(P.T, P.K[0], P.K[1], P.K[2]);
      P.K[0] = P.K[1] = P.K[2] = 0.f;
      nbd++;
    }
    const bool hit = (s0 + l < n) && ellipse_hits(r_cur, bx0, by0);
    const uint64_t bal = __ballot(hit);
    opaque = opaque || __ballot(hit && may_clamp(r_cur.b.y, r_cur.a.z, r_cur.a.w, r_cur.b.x)) != 0;
    if (hit) {
      const uint32_t k = nh + (uint32_t)__popcll(bal & lt);
      B.a[k] = make_float4(r_cur.a.x, r_cur.a.y, -0.5f * kLog2e * r_cur.a.z, -kLog2e * r_cur.a.w);
      B.b[k] = make_float2(-0.5f * kLog2e * r_cur.b.x, __log2f(r_cur.b.y));
      B.c[k] = make_float4(r_cur.c.x, r_cur.c.y, r_cur.c.z, __uint_as_float(s0 + l + 1));
    }
    nh += (uint32_t)__popcll(bal);
    wave_lds_sync();
    if (nh >= kFwdStep) {
      composite(nh);
      nh = 0;
      wave_lds_sync();
    }
    r_cur = r_nxt;
    e_nxt = e_nn;
  }
  composite(nh);
  if constexpr (!SAVE) {
    if (inside) {
      const int64_t HW = (int64_t)vd.W * vd.H;
      const int64_t pix = (int64_t)py * vd.W + px;
#pragma unroll
      for (int c = 0; c < 3; c++) vd.img[c * HW + pix] = P.C[c] + P.T * ds.bg[c];
    }
    return;
  }

  // turn the per-chunk colours into the colour behind each boundary: sums of
  // positive terms from the back, so no cancellation against the total
  float S0 = P.K[0], S1 = P.K[1], S2 = P.K[2];
  for (uint32_t m = nbd; m >= 1; m--) {
    const int64_t slot = ((int64_t)rg.x + (int64_t)m * chunk) >> bs.chunk_shift;
    if (slot >= bs.nbound) continue;
    float4* q = bs.bound + slot * kBlock + threadIdx.x;
    const float4 v = *q;
    *q = make_float4(v.x, S0, S1, S2);
    S0 += v.y;
    S1 += v.z;
    S2 += v.w;
  }
  float l1 = 0.f;  // this pixel's |I - I*| summed over the channels
  if (inside) {
    const int64_t HW = (int64_t)vd.W * vd.H;
    const int64_t pix = (int64_t)py * vd.W + px;
    // the running sum, whose rounding does not depend on where chunks begin
    const float o[3] = {P.C[0] + P.T * ds.bg[0], P.C[1] + P.T * ds.bg[1], P.C[2] + P.T * ds.bg[2]};
#pragma unroll
    for (int c = 0; c < 3; c++) vd.img[c * HW + pix] = o[c];
    bs.T_final[vd.pix_base + pix] = P.T;
    bs.last[vd.pix_base + pix] = P.last;
    if constexpr (COUNTS) bs.counts[vd.pix_base + pix] = P.cnt;
    if (bs.l1_partial) {
      // the L1 loss of the step (Sec. 4.4, Sec. 5.1): dL/dI = sign(I - I*) / count
#pragma unroll
      for (int c = 0; c < 3; c++) {
        const float d = o[c] - vd.tgt[c * HW + pix];
        l1 += fabsf(d);
        vd.dl[c * HW + pix] = (d > 0.f) ? bs.l1_inv : ((d < 0.f) ? -bs.l1_inv : 0.f);
      }
    }
  }
  if (bs.l1_partial) {
    // the tile's sum in a fixed order: lanes, then wavefronts
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l1 += __shfl_xor(l1, off);
    if (l == 0) s_l1[wv] = l1;
  }
  const uint32_t wlast = wave_max(P.last);
  if (l == 0) atomicMax(&s_maxlast, wlast);
  __syncthreads();
  // the tile's backward work items (tile, 0 .. nch - 1), appended to the list
  // where the tiles finished so far end (*n_items is zero before the launch)
  const uint32_t nch = (s_maxlast + chunk - 1) >> bs.chunk_shift;
  if (threadIdx.x == 0) {
    bs.tile_nch[tile] = nch;
    s_ibase = nch ? atomicAdd(bs.n_items, nch) : 0u;
    if (bs.l1_partial) {
      float sum = 0.f;
      for (int w = 0; w < kWaves; w++) sum += s_l1[w];
      bs.l1_partial[tile] = sum;
    }
  }
  __syncthreads();
  for (uint32_t k = threadIdx.x; k < nch; k += kBlock) {
    const int64_t slot = (int64_t)s_ibase + k;
    if (slot < bs.items_cap) bs.items[slot] = make_uint2((uint32_t)tile, k);
  }
}

// ------------------------------------------------------------ backward walk
// One wavefront, one 8x8 block: the reverse walk takes the block's list in
// groups of 16 Gaussians, each of the wavefront's four rows of 16 lanes holding
// the group (lane j: Gaussian j), and steps through the block's pixels four at a
// time: step `it` takes pixel 16 row + it in every row.  So the Gaussians'
// gradient sums are per-lane registers added up over the steps (nothing is
// reduced across lanes per Gaussian), and the two quantities that do chain
// along the list -- the transmittance and the colour behind -- are scans over
// the 16 lanes of a row.  A pixel's state lives in lane 16 row + it; a step
// reads it with row_newbcast as the operand of the instruction that needs it.
//
// The chained parts are inline assembly: there a scan step is one instruction
// in place (a lane without a source keeps its value), which the compiler's
// lane-move builtins do not reach.  gfx950's DPP reads need two wait states
// after the VALU write of the register they read.  The compiler provides them
// for its own instructions, not across these statements: each begins and ends
// with the wait, and four steps are interleaved, so that a result is read four
// instructions after it is written.
typedef float F4v __attribute__((ext_vector_type(4)));

template <int IT>
__device__ __forceinline__ uint32_t row_bcast(uint32_t x) {  // lane IT of each row
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + IT, 0xF, 0xF, true);
}

// One instruction for each of four steps: operands a b c d of the four, and
// the lane operation.
#define SIXDGS_DPP4(op, a0, b0, a1, b1, a2, b2, a3, b3, lanes)       \
  op " " a0 ", " b0 " " lanes "\n\t" op " " a1 ", " b1 " " lanes     \
     "\n\t" op " " a2 ", " b2 " " lanes "\n\t" op " " a3 ", " b3 " " \
     lanes "\n\t"
#define SIXDGS_ALL " row_mask:0xf bank_mask:0xf"
#define SIXDGS_SCAN(op, n) \
  SIXDGS_DPP4(op, "%0", "%0, %0", "%1", "%1, %1", "%2", "%2, %2", "%3", "%3, %3", "row_shl:" n SIXDGS_ALL)

// Steps 4K .. 4K + 3: x[j] = 1 / (1 - alpha) becomes the transmittance in
// front of each lane's Gaussian, T(pixel 4K + j) times the product of x[j]
// over the lanes from this one on, and T(pixel) the row's first of these.
template <int K>
__device__ __forceinline__ void transmittances(float& T, float (&x)[4]) {
  constexpr uint64_t kOne = 0x0001000100010001ull << (4 * K);
  asm("s_nop 1\n\t" SIXDGS_SCAN("v_mul_f32_dpp", "1") SIXDGS_SCAN("v_mul_f32_dpp", "2")
          SIXDGS_SCAN("v_mul_f32_dpp", "4") SIXDGS_SCAN("v_mul_f32_dpp", "8")
      "v_mul_f32_dpp %0, %4, %0 row_newbcast:%c9" SIXDGS_ALL "\n\t"
      "v_mul_f32_dpp %1, %4, %1 row_newbcast:%c10" SIXDGS_ALL "\n\t"
      "v_mul_f32_dpp %2, %4, %2 row_newbcast:%c11" SIXDGS_ALL "\n\t"
      "v_mul_f32_dpp %3, %4, %3 row_newbcast:%c12" SIXDGS_ALL "\n\t"
      "s_mov_b64 vcc, %5\n\t"
      "v_cndmask_b32_dpp %4, %0, %4, vcc row_newbcast:0" SIXDGS_ALL "\n\t"
      "s_mov_b64 vcc, %6\n\t"
      "v_cndmask_b32_dpp %4, %1, %4, vcc row_newbcast:0" SIXDGS_ALL "\n\t"
      "s_mov_b64 vcc, %7\n\t"
      "v_cndmask_b32_dpp %4, %2, %4, vcc row_newbcast:0" SIXDGS_ALL "\n\t"
      "s_mov_b64 vcc, %8\n\t"
      "v_cndmask_b32_dpp %4, %3, %4, vcc row_newbcast:0" SIXDGS_ALL "\n\t"
      "s_nop 1"
      : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(T)
      : "s"(~kOne), "s"(~(kOne << 1)), "s"(~(kOne << 2)), "s"(~(kOne << 3)), "i"(4 * K), "i"(4 * K + 1),
        "i"(4 * K + 2), "i"(4 * K + 3)
      : "vcc");
}

// Steps 4K .. 4K + 3: q[j] = dL/dC . c times the weight becomes
// q[j] + f[j] (D(pixel 4K + j) + the sum of q[j] over the lanes past this one),
// and D(pixel) grows by the row's sum of q[j].  one[j] is 1 in the lanes
// 4 i + j and 0 in the others; the bank mask keeps to the four lanes 4K ...
template <int K>
__device__ __forceinline__ void behind_terms(float& D, float (&q)[4], const float (&f)[4], const float (&one)[4]) {
  float s0, s1, s2, s3;
  asm("s_nop 1\n\t"
      SIXDGS_DPP4("v_add_f32_dpp", "%0", "%4, %4", "%1", "%5, %5", "%2", "%6, %6", "%3", "%7, %7",
                  "row_shl:1" SIXDGS_ALL " bound_ctrl:1")
      SIXDGS_SCAN("v_add_f32_dpp", "2") SIXDGS_SCAN("v_add_f32_dpp", "4") SIXDGS_SCAN("v_add_f32_dpp", "8")
      SIXDGS_DPP4("v_fmac_f32_dpp", "%4", "%0, %9", "%5", "%1, %10", "%6", "%2, %11", "%7", "%3, %12",
                  "row_shl:1" SIXDGS_ALL " bound_ctrl:1")
      "v_fmac_f32_dpp %4, %8, %9 row_newbcast:%c17" SIXDGS_ALL "\n\t"
      "v_fmac_f32_dpp %5, %8, %10 row_newbcast:%c18" SIXDGS_ALL "\n\t"
      "v_fmac_f32_dpp %6, %8, %11 row_newbcast:%c19" SIXDGS_ALL "\n\t"
      "v_fmac_f32_dpp %7, %8, %12 row_newbcast:%c20" SIXDGS_ALL "\n\t"
      "v_fmac_f32_dpp %8, %0, %13 row_newbcast:0 row_mask:0xf bank_mask:%c21\n\t"
      "v_fmac_f32_dpp %8, %1, %14 row_newbcast:0 row_mask:0xf bank_mask:%c21\n\t"
      "v_fmac_f32_dpp %8, %2, %15 row_newbcast:0 row_mask:0xf bank_mask:%c21\n\t"
      "v_fmac_f32_dpp %8, %3, %16 row_newbcast:0 row_mask:0xf bank_mask:%c21\n\t"
      "s_nop 1"
      : "=&v"(s0), "=&v"(s1), "=&v"(s2), "=&v"(s3), "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]), "+v"(D)
      : "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "v"(one[0]), "v"(one[1]), "v"(one[2]), "v"(one[3]), "i"(4 * K),
        "i"(4 * K + 1), "i"(4 * K + 2), "i"(4 * K + 3), "i"(1 << K));
}

// Steps 4K .. 4K + 3: sum[c] += dL/dC_c(pixel 4K + j) w[j].
template <int K>
__device__ __forceinline__ void colour_terms(float (&sum)[3], const float (&dC)[3], const float (&w)[4]) {
#pragma unroll
  for (int c = 0; c < 3; c++)
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:%c6" SIXDGS_ALL "\n\t"
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:%c7" SIXDGS_ALL "\n\t"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:%c8" SIXDGS_ALL "\n\t"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:%c9" SIXDGS_ALL
        : "+v"(sum[c])
        : "v"(dC[c]), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "i"(4 * K), "i"(4 * K + 1), "i"(4 * K + 2),
          "i"(4 * K + 3));
}
#undef SIXDGS_SCAN
#undef SIXDGS_ALL
#undef SIXDGS_DPP4

// a + b after swapping the upper half of a with the lower half of b: lanes
// 0-31 get a[i] + a[i+32], lanes 32-63 get b[i-32] + b[i].
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
  return __int_as_float(r[0]) + __int_as_float(r[1]);
}

// a + b after swapping the odd rows of a with the even rows of b: rows 0, 1,
// 2, 3 get a0 + a1, b0 + b1, a2 + a3, b2 + b3 (rows of 16 lanes).
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
  return __int_as_float(r[0]) + __int_as_float(r[1]);
}

// The walk's state: pixel state by lane, and the constant operands of the
// matrix products.
struct BwdWave {
  float T, D;           // transmittance in front of / dL/dC . colour behind the last group taken (lane = pixel)
  uint32_t lastcmp;     // list positions from here on are not taken (lane = pixel)
  float dC[3];          // dL/dC (lane = pixel)
  float dcA[4];         // dL/dC as the pixel operand of dL/dC . c
  float one[4];         // 1 in the lanes 4 i + j
  uint32_t qlast[4];    // per quad of pixels: list positions from here on no pixel takes,
  uint32_t qmin;        // list positions before here no pixel compares
};

// The gradients are moments of w = dL/d(exponent).  Far along a long thin
// Gaussian dx and dy are large and, in the gradients of its mean and covariance,
// nearly cancel.  So the walk takes the moments of (x, dy) with x = dx + r dy,
// the pixel's distance along its line from the Gaussian's axis, and they become
// those of (dx, dy) once per staged Gaussian (needles of 40 to 300 pixels: mean
// off by 3e-8 of its terms' sum, covariance by 2e-6 to 5e-6 in the root mean;
// moments of (dx, dy) throughout: 1e-7, and 2e-6 to 9e-6).  r = 0 where cB/2 / cA
// is not a number that serves.
__device__ __forceinline__ float axis_slope(float cA, float cB) {
  const float r = 0.5f * cB * rcp_fast(cA);
  return fabsf(r) < 1e12f ? r : 0.f;
}

// A group's Gaussian in this lane, and its sums over the pixels of the row.
struct BwdGauss {
  float cA;
  float dx[8];                // pixel columns
  float r, dy[2];             // axis_slope; the row's two pixel lines (4 apart)
  float bdy[2], cdy[2];       // the exponent's terms of the lines
  uint32_t pos;               // list position
  float s0[2], s1[2], s2[2];  // per pixel line: sums of w, w x, w x^2 (w = dL/d(exponent))
  float col[3];               // colour gradient
};

// How a group is walked: all pixels take every Gaussian that reaches 1/255
// (kFree), pixels may stop inside the group (kStops, by lastcmp), or also
// alpha's clamp may act (kExact).
enum BwdForm { kFree, kStops, kExact };

// Steps 4K .. 4K + 3 of a group.  col: the Gaussian's colour channel `row` (the
// fourth is 0), the operand of dL/dC . c.
template <int K, BwdForm FORM>
__device__ __forceinline__ void bwd_steps(BwdWave& W, BwdGauss& G, float col) {
  constexpr int h = K >> 1;
  const F4v zero = {0.f, 0.f, 0.f, 0.f};
  const F4v dc = __builtin_amdgcn_mfma_f32_16x16x4f32(W.dcA[K], col, zero, 0, 0, 0);
  float a[4], f[4], x[4], e[4];
#pragma unroll
  for (int j = 0; j < 4; j++) {
    const float dx = G.dx[(4 * K + j) & 7];
    // the operations and roundings of log2_alpha
    const float p = __fmaf_rn(__fmaf_rn(G.cA, dx, G.bdy[h]), dx, G.cdy[h]);
    bool take = p >= kLog2AlphaMin;
    e[j] = exp2_fast(p);
    if constexpr (FORM != kFree) {
      const uint32_t lc = j == 0   ? row_bcast<4 * K>(W.lastcmp)
                          : j == 1 ? row_bcast<4 * K + 1>(W.lastcmp)
                          : j == 2 ? row_bcast<4 * K + 2>(W.lastcmp)
                                   : row_bcast<4 * K + 3>(W.lastcmp);
      take = take && G.pos < lc;
    }
    a[j] = take ? e[j] : 0.f;
    if constexpr (FORM == kExact) a[j] = fminf(kAlphaMax, a[j]);
    x[j] = rcp_fast(1.0f - a[j]);
    f[j] = -a[j] * x[j];
  }
  // (f is formed here: the products below take x's registers)
  asm("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
  transmittances<K>(W.T, x);
  float wgt[4], q[4];
#pragma unroll
  for (int j = 0; j < 4; j++) {
    wgt[j] = a[j] * x[j];
    q[j] = dc[j] * wgt[j];
  }
  colour_terms<K>(G.col, W.dC, wgt);
  // alpha dL/dalpha = T alpha dL/dC . c - alpha / (1 - alpha) dL/dC . (colour behind)
  behind_terms<K>(W.D, q, f, W.one);
  if constexpr (FORM == kExact) {
#pragma unroll
    for (int j = 0; j < 4; j++) q[j] = e[j] <= kAlphaMax ? q[j] : 0.f;  // zero derivative above the clamp
  }
  // the four pixels' moments about the second's column, then about the axis
  const float a02 = q[0] + q[2];
  const float m0 = a02 + (q[1] + q[3]);
  const float m1 = __fmaf_rn(2.f, q[3], q[2] - q[0]);
  const float m2 = __fmaf_rn(4.f, q[3], a02);
  const float x1 = __fmaf_rn(G.r, G.dy[h], G.dx[(4 * K + 1) & 7]);
  const float c1 = __fmaf_rn(x1, m0, m1);
  G.s0[h] += m0;
  G.s1[h] += c1;
  G.s2[h] += __fmaf_rn(x1, m1 + c1, m2);
}

// pos0: the group's first list position; a 4 x 4 quad of pixels that all ended
// before it is left out (16 uneven views of 500k Gaussians 3410 -> 3325 us, one
// 800x800 view of 300k 169 -> 166; a form chosen for each quad: 3450, 174).
template <BwdForm FORM>
__device__ __forceinline__ void bwd_group(BwdWave& W, BwdGauss& G, float col, uint32_t pos0) {
  // keeps the forms' exponents apart: formed ahead of the choice between
  // them, all sixteen would be held in registers
  asm volatile("" : "+v"(G.cA));
  if (FORM == kFree || pos0 < W.qlast[0]) bwd_steps<0, FORM>(W, G, col);
  if (FORM == kFree || pos0 < W.qlast[1]) bwd_steps<1, FORM>(W, G, col);
  if (FORM == kFree || pos0 < W.qlast[2]) bwd_steps<2, FORM>(W, G, col);
  if (FORM == kFree || pos0 < W.qlast[3]) bwd_steps<3, FORM>(W, G, col);
}

__device__ __forceinline__ bool finite(float x) { return fabsf(x) < __builtin_huge_valf(); }

// The pixels of the block (first at x0, y0) whose dL/dC is not finite, by the
// lane that holds them, against staged Gaussian s at list position pos: where
// such a pixel takes it, its channels that are not finite go to the Gaussian's
// colour sums, and its other sums become undefined.  Every lane calls; `in`:
// whether it has a Gaussian.
__device__ __forceinline__ void not_finite(const Staged& s, bool in, uint32_t pos, float* sums, uint64_t odd,
                                           uint32_t lastcmp, const ViewDesc& vd, int x0, int y0) {
  for (; odd; odd &= odd - 1) {
    const int q = __ffsll((unsigned long long)odd) - 1;
    const int x = x0 + (q & 7), y = y0 + 4 * ((q >> 3) & 1) + (q >> 4);
    const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)lastcmp, q);
    const float p = log2_alpha(s.a, s.b, ((float)x + 0.5f) - s.a.x, ((float)y + 0.5f) - s.a.y);
    if (!(in && p >= kLog2AlphaMin && pos < last)) continue;
    for (int c = 0; c < 3; c++) {
      const float d = vd.dimg[((int64_t)c * vd.H + y) * vd.W + x];
      if (!finite(d)) atomicAdd(sums + 6 + c, d);
    }
    if (exp2_fast(p) <= kAlphaMax)
      for (int k = 0; k < 6; k++) atomicAdd(sums + k, __builtin_nanf(""));
  }
}

// One work item = one chunk of `chunk` list positions of one tile, walked
// back to front from the state the forward saved where the next chunk begins
// (or from the pixel's final state for the tile's last chunk).
//
// Bound by the vector instructions it issues.  With a pixel per lane for the
// whole walk, a Gaussian cost 65 of them, 24 for the sums of its nine values
// over the wavefront; here a group of 16 takes 30 a step and Gaussian without
// a reduction (the product dL/dC . c is four f32 matrix products a group, which
// share the vector units' rate but replace 48 instructions by 32 issue slots;
// the colour sums are cheaper as vector instructions: 3465 against 3780 us
// with matrix products on sixteen uneven views of 500k Gaussians).  Vector
// instructions there 2.81 -> 1.6 G, time 4803 -> 3313 us; one 800x800 view of
// 300k Gaussians 224 -> 164 us; eight 1080p views of 1M 4950 -> 3371.
// Registers: 95 hold the walk without spills, five wavefronts per SIMD; six
// (80, a few spilled outside the steps) are 2% faster where the launch has
// many long lists (MAXB = 256) and 8% slower on one 403x301 view.
template <int TW, int MAXB>
__global__ void __launch_bounds__(kBlock, MAXB <= 128 ? 5 : 6)
    k_blend_bwd(ViewTable vt, DevSettings ds, const Rec* __restrict__ rec, const uint2* __restrict__ ranges,
                const uint32_t* __restrict__ pval, BlendState bs, float* __restrict__ g2d, int batch) {
  __shared__ BatchLDS<MAXB> L;
  __shared__ float s_g[kG2D * MAXB];  // per staged Gaussian, summed over the four wavefronts
  __shared__ uint32_t s_maxlast;
  // the list holds the items in the order the forward's tiles finished
  // (measured: 5 us faster on c2 than taking it from the back, the long
  // tiles' chunks first)
  const uint32_t ni = (uint32_t)min<int64_t>(*bs.n_items, bs.items_cap);
  if (blockIdx.x >= ni) return;  // uniform
  const uint2 item = bs.items[blockIdx.x];
  const int tile = (int)item.x;
  const uint32_t chunk = bs.chunk;
  const uint32_t cstart = item.y * chunk;  // list positions [cstart, cstart + chunk) of the tile
  const int vi = find_view(vt, tile);
  const ViewDesc& vd = vt.v[vi];
  const int local = tile - vd.tile_base;
  const int tx = local % vd.ntx, ty = local / vd.ntx;
  const int wv = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  // a pixel per lane for the walk's state: lane 16 row + s holds that of step s,
  // so that steps 4 K .. 4 K + 3 of the four rows are a 4 x 4 quad of the block
  const int gj = l & 15, row = l >> 4;
  const float ox = (float)(tx * TW) + 0.5f, oy = (float)(ty * TileMap<TW>::TH) + 0.5f;
  const int px = tx * TW + TileMap<TW>::bx(wv) + (l & 7);
  const int py = ty * TileMap<TW>::TH + TileMap<TW>::by(wv) + 4 * (gj >> 3) + row;
  const bool inside = px < vd.W && py < vd.H;
  // pixel centres of the wavefront's block: its columns, and the row's first line
  float fx[8];
#pragma unroll
  for (int k = 0; k < 8; k++)
    fx[k] = __uint_as_float(__builtin_amdgcn_readfirstlane(
        __float_as_uint((float)(tx * TW + TileMap<TW>::bx(wv) + k) + 0.5f)));
  const float by0 = (float)(ty * TileMap<TW>::TH + TileMap<TW>::by(wv) + row) + 0.5f;

  float Tf = 0.f, dC0 = 0.f, dC1 = 0.f, dC2 = 0.f;
  uint32_t last = 0;
  if (inside) {
    const int64_t HW = (int64_t)vd.W * vd.H;
    const int64_t pix = (int64_t)py * vd.W + px;
    Tf = bs.T_final[vd.pix_base + pix];
    last = bs.last[vd.pix_base + pix];
    dC0 = vd.dimg[pix];
    dC1 = vd.dimg[HW + pix];
    dC2 = vd.dimg[2 * HW + pix];
  }
  // An infinite or undefined dL/dC would outlive the products with 0 by which
  // the walk leaves out Gaussians and pixels: such a channel is walked as 0, and
  // the Gaussians that its pixel takes get it afterwards (not_finite).
  const uint64_t odd = __ballot(!(finite(dC0) && finite(dC1) && finite(dC2)));
  dC0 = finite(dC0) ? dC0 : 0.f;
  dC1 = finite(dC1) ? dC1 : 0.f;
  dC2 = finite(dC2) ? dC2 : 0.f;
  // dL/dC passes through the (not yet used) staging records into the operand
  // of dL/dC . c
  static_assert(sizeof(L.rec) >= sizeof(float4) * kBlock, "dL/dC fits the staged records");
  float4* s_dc = reinterpret_cast<float4*>(L.rec);
  s_dc[threadIdx.x] = make_float4(dC0, dC1, dC2, 0.f);
  if (threadIdx.x == 0) s_maxlast = 0;
  for (int k = threadIdx.x; k < kG2D * MAXB; k += kBlock) s_g[k] = 0.f;
  __syncthreads();
  const uint32_t wlast = __builtin_amdgcn_readfirstlane(wave_max(last));
  if (l == 0) atomicMax(&s_maxlast, wlast);
  BwdWave W;
  W.dC[0] = dC0;
  W.dC[1] = dC1;
  W.dC[2] = dC2;
  {
    const float* q = reinterpret_cast<const float*>(s_dc + wv * 64);
    // operand lane (i, k) = (l & 15, l >> 4): result row / column i, contraction index k
#pragma unroll
    for (int k = 0; k < 4; k++) W.dcA[k] = q[4 * ((gj >> 2) * 16 + 4 * k + (gj & 3)) + row];
#pragma unroll
    for (int j = 0; j < 4; j++) W.one[j] = (l & 3) == j ? 1.f : 0.f;
  }
  __syncthreads();
  const uint2 rg = ranges[tile];
  const uint32_t maxlast = s_maxlast;
  // state behind the chunk: transmittance T in front of it and the colour S
  // behind it (background included), carried as D = dL/dC . S.  A pixel
  // outside the image has T = 0 and dL/dC = 0: it adds exact zeros.
  float S0 = Tf * ds.bg[0], S1 = Tf * ds.bg[1], S2 = Tf * ds.bg[2];
  W.T = Tf;
  if (cstart + chunk < last) {
    // the pixel takes Gaussians past this chunk: resume from the state saved
    // where the next chunk begins (otherwise its final state is that state)
    const int64_t slot = ((int64_t)rg.x + cstart + chunk) >> bs.chunk_shift;
    const float4 st = slot < bs.nbound ? bs.bound[slot * kBlock + wv * 64 + (4 * (gj >> 3) + row) * 8 + (l & 7)] : make_float4(1.f, 0.f, 0.f, 0.f);
    W.T = st.x;
    S0 += st.y;
    S1 += st.z;
    S2 += st.w;
  }
  W.D = dC0 * S0 + dC1 * S1 + dC2 * S2;
  // The walk of a pixel stops before its transmittance would fall below 1e-4,
  // which takes alpha <= 0.99 from at most 1e-2: a pixel that ended above
  // that took every Gaussian that reaches 1/255 there, so only the others
  // compare list positions.
  W.lastcmp = (Tf > 0.0101f || !inside) ? 0xFFFFFFFFu : last;
  W.qmin = __builtin_amdgcn_readfirstlane(~wave_max(~W.lastcmp));
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const bool mine = gj >> 2 == k;
    W.qlast[k] = __builtin_amdgcn_readfirstlane(wave_max(mine ? last : 0u));
  }
  const uint32_t cend = min(cstart + chunk, maxlast);

  for (uint32_t bend = rg.x + cend; bend > rg.x + cstart;) {
    const uint32_t b0 = (bend - (rg.x + cstart) > (uint32_t)batch) ? bend - batch : rg.x + cstart;
    const uint32_t nb = bend - b0;
    const uint32_t wn = stage_batch<TW, MAXB>(L, rec, pval, b0, nb, ox, oy);
    const uint32_t posb = b0 - rg.x;
    for (int g = (int)((wn + 15) >> 4) - 1; g >= 0; g--) {
      // lane j takes list slot 16 g + j; past the list a Gaussian that no pixel takes
      const uint32_t i = 16 * (uint32_t)g + gj;
      const uint32_t slot = L.list[wv][min(i, wn - 1)];
      BwdGauss G;
      G.pos = posb + slot;
      if (__builtin_amdgcn_readfirstlane(G.pos) >= wlast) continue;  // behind every pixel's last
      const Staged& sr = L.rec[slot];
      const float4 A = sr.a;
      const float2 B = make_float2(sr.b.x, i < wn ? sr.b.y : -1e30f);
      const bool clamps = sr.b.z < 0.f;
      const float col = reinterpret_cast<const float*>(&sr.c)[row];  // channel `row` (the fourth is 0)
      G.cA = A.z;
#pragma unroll
      for (int k = 0; k < 8; k++) G.dx[k] = fx[k] - A.x;
      G.r = axis_slope(A.z, A.w);
#pragma unroll
      for (int h = 0; h < 2; h++) {
        const float dy = (by0 + 4.f * (float)h) - A.y;
        G.dy[h] = dy;
        G.bdy[h] = __fmul_rn(A.w, dy);
        G.cdy[h] = __fmaf_rn(__fmul_rn(B.x, dy), dy, B.y);
        G.s0[h] = G.s1[h] = G.s2[h] = 0.f;
      }
      G.col[0] = G.col[1] = G.col[2] = 0.f;
      const uint32_t pos0 = __builtin_amdgcn_readfirstlane(G.pos), pos1 = __builtin_amdgcn_readlane(G.pos, 15);
      if (__ballot(clamps))
        bwd_group<kExact>(W, G, col, pos0);
      else if (pos1 >= W.qmin)
        bwd_group<kStops>(W, G, col, pos0);
      else
        bwd_group<kFree>(W, G, col, pos0);
      // the moments of w in (x, dy) and the colour gradient, summed over the
      // four rows (halving exchanges) and added in LDS
      const float v[kG2D] = {G.s1[0] + G.s1[1],
                             G.dy[0] * G.s0[0] + G.dy[1] * G.s0[1],
                             G.s2[0] + G.s2[1],
                             G.dy[0] * G.s1[0] + G.dy[1] * G.s1[1],
                             G.dy[0] * G.dy[0] * G.s0[0] + G.dy[1] * G.dy[1] * G.s0[1],
                             G.s0[0] + G.s0[1],
                             G.col[0],
                             G.col[1],
                             G.col[2]};
      const float k0 = swap16_add(swap32_add(v[0], v[1]), swap32_add(v[2], v[3]));
      const float k1 = swap16_add(swap32_add(v[4], v[5]), swap32_add(v[6], v[7]));
      const float h8 = swap32_add(v[8], v[8]);
      const float k2 = swap16_add(h8, h8);
      if (i < wn) {
        // rows 0 .. 3 of k0 hold v0 v2 v1 v3, of k1 v4 v6 v5 v7, every row of k2 v8
        float* const to = s_g + slot * kG2D;
        const int f = row == 0 ? 0 : row == 1 ? 2 : row == 2 ? 1 : 3;
        atomicAdd(to + f, k0);
        atomicAdd(to + f + 4, k1);
        if (row == 0) atomicAdd(to + 8, k2);
      }
    }
    if (odd)
      for (uint32_t i0 = 0; i0 < wn; i0 += 64) {  // (uniform)
        const uint32_t i = i0 + l, slot = L.list[wv][min(i, wn - 1)];
        not_finite(L.rec[slot], i < wn, posb + slot, s_g + slot * kG2D, odd, W.lastcmp, vd,
                   tx * TW + TileMap<TW>::bx(wv), ty * TileMap<TW>::TH + TileMap<TW>::by(wv));
      }
    __syncthreads();
    // one set of global atomics per (chunk, Gaussian).  Each staged
    // Gaussian's thread turns its column of sums into the nine components in
    // place (the conic gradient goes from the pre-scaled coefficients back to
    // the conic's full-matrix gradient); the adds then go Gaussian-major, so
    // that consecutive lanes add to consecutive words of one Gaussian's row (a
    // memory request per row instead of one per component), zero components
    // skipped.
    const int t = threadIdx.x;
    static_assert(sizeof(L.list) >= sizeof(uint32_t) * MAXB, "entry ids fit the slot lists");
    uint32_t* s_ent = reinterpret_cast<uint32_t*>(L.list);  // the slot lists are no longer read
    if ((uint32_t)t < nb) {
      float v[kG2D];
#pragma unroll
      for (int k = 0; k < kG2D; k++) v[k] = s_g[t * kG2D + k];
      // exponent p2 = log2(alpha) = cA dx^2 + cB dx dy + cC dy^2 + log2(alpha_cond), with
      // dx = x - r dy: dp2/dmean = -2 (cA dx + hB dy, hB dx + cC dy) for hB = cB / 2, and
      // dp2/dcA = dx^2 etc., cA = kq Qxx, cB = 2 kq Qxy, cC = kq Qyy
      const Staged& sr = L.rec[t];
      const float cA = sr.a.z, hB = 0.5f * sr.a.w, r = axis_slope(sr.a.z, sr.a.w);
      const float e = __fmaf_rn(-cA, r, hB), g = __fmaf_rn(-hB, r, sr.b.x);
      constexpr float kMean = -2.f * kLn2, kConic = -0.5f * kLog2e * kLn2;  // (dL/dp2 = ln 2 w)
      s_g[t * kG2D + 0] = kMean * (cA * v[0] + e * v[1]);
      s_g[t * kG2D + 1] = kMean * (hB * v[0] + g * v[1]);
      const float xy = __fmaf_rn(-r, v[4], v[3]);  // the sum of w dx dy
      s_g[t * kG2D + 2] = kConic * __fmaf_rn(-r, v[3] + xy, v[2]);
      s_g[t * kG2D + 3] = kConic * xy;
      s_g[t * kG2D + 4] = kConic * v[4];
      s_g[t * kG2D + 5] = v[5] * fabsf(sr.b.z);  // d alpha / d alpha_cond = alpha / alpha_cond
      s_ent[t] = __float_as_uint(sr.b.w);
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t idx = t; idx < nb * kG2D; idx += kBlock) {
      const uint32_t jg = idx / kG2D, k = idx - jg * kG2D;
      const float val = s_g[idx];
      s_g[idx] = 0.f;
      if (val != 0.f) unsafeAtomicAdd(g2d + (int64_t)s_ent[jg] * kG2D + k, val);
    }
    __syncthreads();
    bend = b0;
  }
}

}  // namespace

namespace {
constexpr int kFoursTiles = 3072;  // from this many tiles on the forward goes by pairs

template <int TW>
void launch_fwd(const ViewTable& vt, const DevSettings& s, const Rec* rec, const uint2* ranges, const uint32_t* pval,
                const BlendState& bs, bool save, hipStream_t st) {
  auto k = !save                          ? k_blend_fwd<TW, false, false, 2, 7>
           : bs.counts                    ? k_blend_fwd<TW, true, true, 4, 4>
           : vt.total_tiles < kFoursTiles ? k_blend_fwd<TW, true, false, 4, 4>
                                          : k_blend_fwd<TW, true, false, 2, 6>;
  hipLaunchKernelGGL(k, dim3(vt.total_tiles), dim3(kBlock), 0, st, vt, s, rec, ranges, pval, bs);
}
}  // namespace

void launch_blend_fwd(const ViewTable& vt, const DevSettings& s, const Rec* rec, const uint2* ranges,
                      const uint32_t* pval, BlendState bs, bool save, hipStream_t st) {
  if (vt.total_tiles <= 0) return;
  switch (vt.tile_w) {
    case 8: launch_fwd<8>(vt, s, rec, ranges, pval, bs, save, st); break;
    case 32: launch_fwd<32>(vt, s, rec, ranges, pval, bs, save, st); break;
    default: launch_fwd<16>(vt, s, rec, ranges, pval, bs, save, st); break;
  }
}

namespace {
template <int TW>
void launch_bwd(const ViewTable& vt, const DevSettings& s, const Rec* rec, const uint2* ranges, const uint32_t* pval,
                const BlendState& bs, float* g2d, int batch, dim3 grid, hipStream_t st) {
  if (batch <= 128)
    hipLaunchKernelGGL((k_blend_bwd<TW, 128>), grid, dim3(kBlock), 0, st, vt, s, rec, ranges, pval, bs, g2d, batch);
  else
    hipLaunchKernelGGL((k_blend_bwd<TW, 256>), grid, dim3(kBlock), 0, st, vt, s, rec, ranges, pval, bs, g2d, batch);
}
}  // namespace

void launch_blend_bwd(const ViewTable& vt, const DevSettings& s, const Rec* rec, const uint2* ranges,
                      const uint32_t* pval, BlendState bs, float* g2d, int batch, int64_t items, hipStream_t st) {
  if (vt.total_tiles <= 0 || items <= 0) return;
  const dim3 grid((unsigned)items);
  switch (vt.tile_w) {
    case 8: launch_bwd<8>(vt, s, rec, ranges, pval, bs, g2d, batch, grid, st); break;
    case 32: launch_bwd<32>(vt, s, rec, ranges, pval, bs, g2d, batch, grid, st); break;
    default: launch_bwd<16>(vt, s, rec, ranges, pval, bs, g2d, batch, grid, st); break;
  }
}

}  // namespace sixdgs
