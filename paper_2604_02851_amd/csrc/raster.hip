// Front-to-back compositing per tile and its adjoint.
//
// One workgroup per tile.  Each thread owns PPT pixels of the tile; each
// wavefront owns an SW x WROWS sub-tile (a band of whole rows when SW = TW,
// squarer blocks otherwise, which a splat's box misses more often).  The
// tile's list is consumed in batches of BATCH splat records staged in LDS:
// every pixel of the tile reads every record, so a record leaves HBM once per
// tile.  Before evaluating a splat, a wavefront tests the splat's 3-sigma box
// against its own sub-tile and skips it as a whole when they do not meet; the box
// is widened so that it contains every pixel whose FP32 ellipse test can
// pass, so skipping never changes a result.
//
// Forward: stops a pixel once its transmittance would fall below 1e-4 and
// the workgroup once every pixel has stopped; saves T_final, the contributor
// count and the last composited list position.
// The forward stores each list entry's strip bits (which wavefront pixel
// slots its splat may reach), and the backward stages them with the records
// instead of testing the strips again: it only walks list positions before
// the tile's largest last position, all of which the forward has staged.
// Backward: walks the list back to front from each pixel's last position,
// rebuilding the transmittance by division (FP32 reciprocal); a splat's screen-space
// gradient is summed over the thread's pixels in registers, then over the
// wavefront with DPP row operations, then over the wavefronts of the tile in
// LDS, and finally added once per (tile, splat, field) to the global
// accumulator.
//
// Both kernels are bound by issue slots of the SIMDs, not by memory (under
// 1 TB/s).  Per wavefront instruction, measured with eight wavefronts per SIMD:
// multiply, add, FMA 2 cycles; compare, select, DPP add, minimum, readlane 4;
// exp2, reciprocal 8; a scalar instruction about 4 of a unit of its own.  So
// the loops spend FMAs where they can save a compare or a select: decisions
// stay in scalar lane masks (a pixel that stopped is a cleared bit, not a sign
// of T to test), the clamp runs only where an opacity can reach it, and a
// splat's own factors are applied once to its totals at the flush.  1M
// Gaussians, 16 mixed views, 32x32 tiles in batches of 64 at four pixels per lane
// and sub-tiles 16 wide: forward 1.27 -> 0.98 ms (0.99e9 -> 0.71e9 vector
// instructions), adjoint 2.14 -> 1.87 ms (1.53e9 -> 1.23e9); both at eight
// wavefronts per SIMD instead of seven.
#include "internal.h"

namespace gs {
namespace {

// A wavefront owns an SW x WROWS sub-tile of PPT pixel slots, SLW x SLH blocks
// of 64 pixels side by side (NX across, NY down); lane l covers pixel
// (l % SLW, l / SLW) of each.  Slots are as square as the sub-tile allows: a
// splat then misses more of them (8 x 8 instead of 16 x 4 pixels evaluates
// about 7% fewer pixels for a splat of 20 pixels radius), and the slots of a
// row share the splat's vertical offset, those of a column the horizontal one.
template <int TW, int TH, int PPT, int SW>
struct Geom {
  static constexpr int NT = TW * TH / PPT;       // threads per workgroup
  static constexpr int NWAVES = NT / 64;
  static constexpr int WROWS = 64 / SW * PPT;    // sub-tile height
  static constexpr int WPR = TW / SW;            // wavefronts per tile row
  static constexpr int NX = PPT % (SW / 8) == 0 ? SW / 8 : (SW >= 16 && PPT % (SW / 16) == 0 ? SW / 16 : 1);
  static constexpr int NY = PPT / NX;
  static constexpr int SLW = SW / NX, SLH = 64 / SLW;
  // splats a wavefront works on at once: with one pixel per lane a single
  // splat leaves the wavefront waiting on its LDS reads and its chain of
  // dependent instructions, and two hide half of each other's (5k Gaussians in
  // three small views: forward 306 -> 249 us, adjoint 370 -> 286); with more
  // pixels per lane the registers serve more wavefronts instead
  static constexpr int SPLATS = PPT == 1 ? 2 : 1;
  static_assert(NX * NY == PPT && SLH * NY == WROWS, "slot shape");
  static_assert(NT % 64 == 0 && 64 % SW == 0 && TW % SW == 0 && TH % WROWS == 0 &&
                    NWAVES == WPR * (TH / WROWS),
                "tile / pixels-per-thread / wave shape");
  static_assert(NWAVES * PPT <= 30, "one strip bit per wavefront and pixel slot, below the flag bits");
  // strip bits of the first half of the wavefronts (two threads share a
  // splat's strip tests when the tile has several wavefronts)
  static constexpr int HALF_BITS = (NWAVES >= 2 ? NWAVES / 2 : NWAVES) * PPT;
  static_assert(HALF_BITS <= 16, "each half of the strip bits fits 16 bits");
};

// Workgroup -> tile.  Schedule 0: row-major tile order.  Schedule 1: each
// XCD (workgroups are dealt to the 8 XCDs round-robin) receives a contiguous
// run of tiles, so neighbouring tiles share splat records in that XCD's L2.
__device__ __forceinline__ uint32_t tile_of_block(uint32_t b, uint32_t ntiles, int schedule) {
  if (schedule == 0) return b;
  const uint32_t xcd = b & 7u, k = b >> 3;
  return xcd * (ntiles >> 3) + min(xcd, ntiles & 7u) + k;
}

// Culling of a splat against rectangles of pixel centres [x0, x1] x [y0, y1]:
// a pixel can pass the 3-sigma test only where q = a (dx + r dy)^2 + s dy^2 <= 9
// (P = -q/2).  The part of that ellipse with y in [y0, y1] is convex, so it
// meets the rectangle exactly when its extent in x meets [x0, x1]: its
// right end is the largest -r dy + sqrt((q - s dy^2) / a), a concave function
// of dy with its maximum at -r t, t = sqrt(q a / (s (s + a r^2))), clamped to
// the dy there are; its left end likewise at +r t.  One such extent serves a
// whole row of rectangles.  The threshold is widened by 0.1% + 0.01 and the
// extent by 0.01 pixels and 1e-5 of its shear for FP32 rounding of all
// evaluations, so culling never changes a result; a NaN culls nothing.
// (Per rectangle, from the minimum of q over its edges, the strip tests were a
// tenth of the forward's vector cycles, about 1660 per splat and tile of
// 16 strips instead of 500: forward of 500k Gaussians in eight views 461 -> 422
// us, of the 2M world 661 -> 595.)
constexpr float kCullQ = 9.0f * 1.001f + 0.01f;
constexpr float kMinus2Ln2 = -1.38629436111989061f;   // undoes the staged conic's -log2(e)/2
// an opacity below this cannot reach the alpha clamp (alpha <= opacity, as P <= 0)
constexpr float kMayClamp = 0.98f;
// flags of the adjoint in the per-splat strip mask (at most 30 strip bits)
constexpr uint32_t kActiveBit = 0x80000000u;   // trainable
constexpr uint32_t kClampBit = 0x40000000u;    // opaque enough to reach the alpha clamp

// Minimum of q over a rectangle, for shapes with one rectangle per row (an
// extent would serve only one there: 253 instead of 243 us for 5k Gaussians in
// three small views at 16x16 tiles and one pixel per thread).  q is convex, so
// its minimum is 0 at the centre when the centre lies inside, else it lies on an
// edge: along a horizontal edge (dy fixed) at dx = -r dy, along a vertical edge
// (dx fixed) at dy = -a r dx / (a r^2 + s), each clamped to the edge.
__device__ __forceinline__ float rect_qmin(float a, float r, float s, float inv, float cu, float cw, float x0,
                                           float x1, float y0, float y1) {
  if (cu >= x0 && cu <= x1 && cw >= y0 && cw <= y1) return 0.f;
  float best = INFINITY;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float dy = (k ? y1 : y0) - cw;
    const float xs = fminf(fmaxf(cu - r * dy, x0), x1);
    const float e = (xs - cu) + r * dy;
    best = fminf(best, a * e * e + s * dy * dy);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float dx = (k ? x1 : x0) - cu;
    const float dys = fminf(fmaxf(-a * r * dx * inv, y0 - cw), y1 - cw);
    const float e = dx + r * dys;
    best = fminf(best, a * e * e + s * dys * dys);
  }
  return best;
}

// Bit (w * PPT + q) set when the splat may reach a pixel of pixel slot q of
// wavefront w (a strip of SLW x SLH pixels of the tile whose top-left pixel
// is (tx0, ty0)), for the wavefronts w in [w0, w1).
template <class G, int SW, int PPT>
__device__ __forceinline__ uint32_t splat_strip_mask(const float4& r0, const float4& r1, int tx0, int ty0, int w0,
                                                     int w1) {
  const float cu = r0.x + r0.z, cw = r0.y + r0.w;
  const float a = r1.x, r = r1.y, s = r1.z;
  uint32_t m = 0;
  if constexpr (G::WPR * G::NX == 1) {
    const float inv = 1.f / fmaf(a * r, r, s);
#pragma unroll 1
    for (int w = w0; w < w1; ++w) {
      const int wy = ty0 + w * G::WROWS;
#pragma unroll 1
      for (int q = 0; q < PPT; ++q) {
        const float x0 = (float)tx0 + 0.5f, x1 = x0 + (float)(G::SLW - 1);
        const float y0 = (float)(wy + q * G::SLH) + 0.5f, y1 = y0 + (float)(G::SLH - 1);
        if (!(rect_qmin(a, r, s, inv, cu, cw, x0, x1, y0, y1) > kCullQ)) m |= 1u << (w * PPT + q);
      }
    }
    return m;
  }
  const float ia = __builtin_amdgcn_rcpf(a), is = __builtin_amdgcn_rcpf(s);
  const float ymax = __builtin_amdgcn_sqrtf(kCullQ * is);
  const float rt = r * __builtin_amdgcn_sqrtf(kCullQ * a * is * __builtin_amdgcn_rcpf(fmaf(a * r, r, s)));
  // not unrolled: the compositing kernels' register budget is set by their
  // main loops, and unrolled strip tests would raise it
#pragma unroll 1
  for (int wr = w0 / G::WPR; wr * G::WPR < w1; ++wr) {   // rows of wavefronts
    const int wa = max(w0, wr * G::WPR), wb = min(w1, (wr + 1) * G::WPR);
#pragma unroll 1
    for (int k = 0; k < G::NY; ++k) {                    // their rows of slots
      const float d0 = (float)(ty0 + wr * G::WROWS + k * G::SLH) + 0.5f - cw, d1 = d0 + (float)(G::SLH - 1);
      if (d0 > ymax || d1 < -ymax) continue;
      const float lo = fmaxf(d0, -ymax), hi = fminf(d1, ymax);
      const float dr = fminf(fmaxf(-rt, lo), hi), dl = fminf(fmaxf(rt, lo), hi);
      const float sr = -r * dr, sl = -r * dl;
      const float xr = (cu + sr) + __builtin_amdgcn_sqrtf(fmaxf(fmaf(-s * dr, dr, kCullQ), 0.f) * ia) +
                       fmaf(fabsf(sr), 1e-5f, 0.01f);
      const float xl = (cu + sl) - __builtin_amdgcn_sqrtf(fmaxf(fmaf(-s * dl, dl, kCullQ), 0.f) * ia) -
                       fmaf(fabsf(sl), 1e-5f, 0.01f);
#pragma unroll 1
      for (int w = wa; w < wb; ++w) {
        const float x0 = (float)(tx0 + (w - wr * G::WPR) * SW) + 0.5f;
        const int bit = w * PPT + k * G::NX;
#pragma unroll
        for (int c = 0; c < G::NX; ++c) {
          const float xa = x0 + (float)(c * G::SLW);
          if (!(xl > xa + (float)(G::SLW - 1) || xr < xa)) m |= 1u << (bit + c);
        }
      }
    }
  }
  return m;
}

// Largest value over the wavefront's 64 lanes (every lane receives it).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
  return v;
}

// The strip bits of staged splat j (the halves' words combined).
template <uint32_t H>
__device__ __forceinline__ uint32_t strip_word(const uint32_t* m, uint32_t j) {
  return H == 2 ? (m[2 * j] | m[2 * j + 1]) : m[j];
}

// Ranges are clamped to the key capacity so that a workspace whose lists were
// never built cannot send a read past the key buffers.
__device__ __forceinline__ uint2 clamp_range(uint2 rg, uint32_t cap) {
  rg.y = min(rg.y, cap);
  rg.x = min(rg.x, rg.y);
  return rg;
}

// Sum over the 64 lanes: inclusive scan inside each row of 16 lanes, then the
// row totals are carried across rows; lane 63 ends with the total.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float v) {
  const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, false);
  return v + __builtin_bit_cast(float, o);
}

__device__ __forceinline__ float wave_total_lane63(float v) {
  v = dpp_add<0x111, 0xf>(v);   // row_shr:1
  v = dpp_add<0x112, 0xf>(v);   // row_shr:2
  v = dpp_add<0x114, 0xf>(v);   // row_shr:4
  v = dpp_add<0x118, 0xf>(v);   // row_shr:8
  v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

template <int CTRL>
__device__ __forceinline__ float dpp_get(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// a + b after exchanging the upper 32 lanes of a with the lower 32 lanes of b
// (resp. the odd 16-lane rows of a with the even rows of b): each result lane
// holds a partial sum of one of the two inputs.  Written as inline assembly
// because the compiler's builtin for these gfx950 swaps loses one of its two
// results here; the s_nop gives the two wait states a cross-lane read needs
// after a VALU write of its operands.
__device__ __forceinline__ float swap32_sum(float a, float b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  return a + b;
}
__device__ __forceinline__ float swap16_sum(float a, float b) {
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  return a + b;
}

// Transposed reduction of eight per-lane values over the wavefront: two
// levels of lane-group swaps halve the values per lane while folding lanes,
// then a row mirror merges the last pair and three DPP steps finish the
// 8-lane groups.  Afterwards every lane of 8-lane group k holds the wave
// total of one field; which field is fixed by the lane position and found
// once per kernel by reducing one-hot tags (reduce8_field).
__device__ __forceinline__ float reduce8(const float* g, bool lo8) {
  const float w0 = swap32_sum(g[0], g[1]);
  const float w1 = swap32_sum(g[2], g[3]);
  const float w2 = swap32_sum(g[4], g[5]);
  const float w3 = swap32_sum(g[6], g[7]);
  const float x0 = swap16_sum(w0, w1);
  const float x1 = swap16_sum(w2, w3);
  const float s = lo8 ? x0 : x1, z = lo8 ? x1 : x0;
  float y = s + dpp_get<0x140>(z);   // row_mirror: lane i of a row reads lane 15 - i
  y += dpp_get<0x141>(y);            // row_half_mirror: lane i of 8 reads lane 7 - i
  y += dpp_get<0x4e>(y);             // quad_perm [2,3,0,1]
  y += dpp_get<0xb1>(y);             // quad_perm [1,0,3,2]
  return y;
}

// Field whose total reduce8 leaves in this lane (exact: sums of 0 and a
// single power of two).
__device__ __forceinline__ int reduce8_field(int lane, bool lo8) {
  float tag[8];
#pragma unroll
  for (int f = 0; f < 8; ++f) tag[f] = lane == 0 ? (float)(1 << f) : 0.f;
  const uint32_t bits = (uint32_t)reduce8(tag, lo8);
  return __builtin_ctz(bits | 256u) & 7;
}

// Work queue of the persistent compositing kernels.  head[0] counts the
// positions handed out, head[1] the workgroups that found the queue empty;
// the last of those resets both, so that the next launch starts from zero
// (they start at zero when the workspace is initialised).  Position k is
// tile order[k] of the call (longest lists first, schedule 3) or tile k.
struct TileQueue {
  uint32_t* head;
  const uint32_t* order;
};
constexpr uint32_t kQueueDone = 0xffffffffu;

__device__ __forceinline__ uint32_t queue_next(const TileQueue& q, uint32_t ntiles, uint32_t* s_next) {
  // every thread is done with the previous tile (its LDS and its position)
  __syncthreads();
  if (threadIdx.x == 0) *s_next = atomicAdd(q.head, 1u);
  __syncthreads();
  // uniform across the workgroup: kept in scalar registers, like blockIdx
  const uint32_t k = __builtin_amdgcn_readfirstlane(*s_next);
  if (k >= ntiles) return kQueueDone;
  return q.order ? __builtin_amdgcn_readfirstlane(q.order[k]) : k;
}

__device__ __forceinline__ void queue_exit(const TileQueue& q) {
  if (threadIdx.x == 0) {
    // this workgroup's last atomicAdd on head[0] has returned: once every
    // workgroup has counted itself here, nobody reads head[0] again
    if (atomicAdd(q.head + 1, 1u) == gridDim.x - 1u) {
      atomicExch(q.head, 0u);
      atomicExch(q.head + 1, 0u);
    }
  }
}

// Evaluation of one splat at the pixels of a wavefront's slots, in parts so
// that slots of a column share dx and slots of a row share dy and the
// vertical term: the one place that decides which pixels a splat can reach,
// called by the forward and the adjoint on identical inputs, so that they make
// identical decisions bit for bit.
template <class G>
struct SplatOffsets {
  float dx[G::NX], dy[G::NY], sdy2[G::NY];
  __device__ __forceinline__ void set(float pxc, float pyc, const float4& r0, const float4& r1h) {
#pragma clang fp contract(off)
#pragma unroll
    for (int i = 0; i < G::NX; ++i) dx[i] = (pxc + (float)(i * G::SLW) - r0.x) - r0.z;
#pragma unroll
    for (int k = 0; k < G::NY; ++k) {
      dy[k] = (pyc + (float)(k * G::SLH) - r0.y) - r0.w;
      sdy2[k] = r1h.z * (dy[k] * dy[k]);
    }
  }
  __device__ __forceinline__ SplatGeom power(int q, const float4& r1h) const {
#pragma clang fp contract(off)
    SplatGeom g;
    g.dx = dx[q % G::NX];
    g.dy = dy[q / G::NX];
    g.e = fmaf(r1h.y, g.dy, g.dx);
    g.P = fmaf(r1h.x * g.e, g.e, sdy2[q / G::NX]);
    return g;
  }
};

// m without bit `l`
__device__ __forceinline__ uint64_t clear_bit(uint64_t m, int l) {
  asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(l));
  return m;
}

// n + 1 in the lanes of `mask`: the mask is the carry of an addition of zero
__device__ __forceinline__ uint32_t add_bit(uint32_t n, uint64_t mask) {
  uint64_t carry_out;
  asm("v_addc_co_u32_e64 %0, %1, 0, %0, %2" : "+v"(n), "=s"(carry_out) : "s"(mask));
  return n;
}

// Keeps a staged record's loads where they are written: the compiler would
// move those of the values used late behind the branches in between, one wait
// after another.
__device__ __forceinline__ void keep_loaded(const float4& r1, const float4& r2) {
  asm volatile("" ::"v"(r1.w), "v"(r2.x), "v"(r2.y), "v"(r2.z));
}

struct CompArgs {
  const ViewInfo* views;
  const int32_t* tile_view;
  int32_t tile_begin;
  int32_t ntiles;
  int32_t schedule;
  const uint2* ranges;
  const uint32_t* vals;
  const float4* rec;
  float* img;
  float* T;
  uint32_t* ncontrib;
  uint32_t* last;
  uint16_t* strips;   // per list position, two 16-bit halves: the staged splat's strip bits
  uint32_t cap;
  float bg0, bg1, bg2;
  TileQueue q;
};

// LDS of one compositing workgroup (forward).
template <int BATCH, uint32_t H>
struct FwdShared {
  float4 rec[BATCH * 3];
  uint32_t mask[BATCH * H];
};

// Forward compositing of tile `slot` of the call by the whole workgroup.
template <int TW, int TH, int PPT, int SW, int BATCH>
__device__ __forceinline__ void composite_tile(const CompArgs& a, uint32_t slot,
                                               FwdShared<BATCH, (Geom<TW, TH, PPT, SW>::NWAVES >= 2 ? 2u : 1u)>& sm) {
  using G = Geom<TW, TH, PPT, SW>;
  constexpr uint32_t kHalves = G::NWAVES >= 2 ? 2 : 1;
  constexpr int K = G::SPLATS;
  float4* s_rec = sm.rec;
  uint32_t* s_mask = sm.mask;
  const int t = a.tile_begin + (int)slot;
  const ViewInfo view = a.views[a.tile_view[t]];
  const int local = t - view.tile_base;
  const int ty = local / view.tiles_x, tx = local - ty * view.tiles_x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x0 = tx * TW + (wave % G::WPR) * SW, y0 = ty * TH + (wave / G::WPR) * G::WROWS;
  const int px0 = x0 + lane % G::SLW, py0 = y0 + lane / G::SLW;
  const uint2 rg = clamp_range(a.ranges[t], a.cap);
  const float pxc = (float)px0 + 0.5f, pyc = (float)py0 + 0.5f;
  // the pixels of slot q that still composite, one bit per lane: pixels
  // outside the image never do, and a pixel that stopped keeps its T
  uint64_t live[PPT];
  float T[PPT], c0[PPT], c1[PPT], c2[PPT];
  uint32_t n[PPT], last[PPT];
  uint32_t qlive = 0u;   // bit q: some pixel of slot q still composites
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    live[q] = __ballot(px0 + (q % G::NX) * G::SLW < view.width && py0 + (q / G::NX) * G::SLH < view.height);
    qlive |= live[q] != 0ull ? 1u << q : 0u;
    T[q] = 1.f;
    c0[q] = c1[q] = c2[q] = 0.f;
    n[q] = 0;
    last[q] = rg.x;
  }
  for (uint32_t b0 = rg.x; b0 < rg.y; b0 += BATCH) {
    if (__syncthreads_or(qlive != 0u) == 0) break;
    const uint32_t cnt = min((uint32_t)BATCH, rg.y - b0);
    // two threads per splat share its strip tests (half the wavefronts each)
    for (uint32_t u = threadIdx.x; u < cnt * kHalves; u += G::NT) {
      const uint32_t j = u / kHalves, h = u % kHalves;
      const uint32_t id = a.vals[b0 + j];
      const float4 r0 = a.rec[(size_t)id * 3 + 0], r1 = a.rec[(size_t)id * 3 + 1];
      if (h == 0) {
        s_rec[j * 3 + 0] = r0;
        s_rec[j * 3 + 1] = staged_conic(r1);
        s_rec[j * 3 + 2] = a.rec[(size_t)id * 3 + 2];
      }
      const uint32_t m = splat_strip_mask<G, SW, PPT>(r0, r1, tx * TW, ty * TH, (int)h * G::NWAVES / kHalves,
                                                      ((int)h + 1) * G::NWAVES / kHalves);
      s_mask[u] = m;
      // for the adjoint: each half's bits, shifted to bit 0, in its own 16-bit slot
      a.strips[2 * (b0 + j) + h] = (uint16_t)(m >> (h * G::HALF_BITS));
      if (kHalves == 1) a.strips[2 * (b0 + j) + 1] = 0;
    }
    __syncthreads();
    // 64 splats at a time: lane l reads the strip word of splat base + l, and
    // the wavefront then visits only the splats that touch one of its live
    // strips (all of it uniform: stopped lanes take part with no live bit)
    for (uint32_t base = 0; base < cnt && qlive != 0u; base += 64) {
      const uint32_t jl = base + (uint32_t)lane;
      const uint32_t mw = jl < cnt ? strip_word<kHalves>(s_mask, jl) >> (wave * PPT) & qlive : 0u;
      uint64_t pend = __ballot(mw != 0u);
      while (pend != 0ull) {
        // the next K pending splats (the last visit may hold fewer: qb 0)
        uint32_t j[K], qb[K];
        float4 r1[K], r2[K];
        SplatOffsets<G> so[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const bool have = k == 0 || pend != 0ull;
          const int l = have ? __builtin_ctzll(pend) : 0;
          pend = clear_bit(pend, l);
          j[k] = base + (uint32_t)l;
          qb[k] = have ? (uint32_t)__builtin_amdgcn_readlane((int)mw, l) & qlive : 0u;
          const float4 r0 = s_rec[j[k] * 3];
          r1[k] = s_rec[j[k] * 3 + 1], r2[k] = s_rec[j[k] * 3 + 2];
          so[k].set(pxc, pyc, r0, r1[k]);
        }
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
          // uniform: the splat misses this pixel slot's strip (K > 1 goes with
          // one slot, which every pending splat reaches)
          if (K == 1 && !((qb[0] >> q) & 1u)) continue;
          uint64_t cand[K], any = 0ull;
          float P[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            P[k] = so[k].power(q, r1[k]).P;
            cand[k] = __ballot(P[k] >= kCutoff2) & (k == 0 || qb[k] != 0u ? live[q] : 0ull);
            any |= cand[k];
          }
          if constexpr (K > 1) {
#pragma unroll
            for (int k = 0; k < K; ++k) keep_loaded(r1[k], r2[k]);
          }
          if (any == 0ull) continue;   // uniform: no pixel of this slot is near a splat
          // predicated from here on: no divergent branches in the hot loop
          float al[K];
#pragma unroll
          for (int k = 0; k < K; ++k) al[k] = fminf(splat_opacity(P[k], r1[k].w), kAlphaMax);
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const float Tn = T[q] * (1.f - al[k]);
            // (a pixel that stopped at the visit's previous splat is live no more)
            const uint64_t take = cand[k] & __ballot(al[k] >= kAlphaMin) & (k == 0 ? ~0ull : live[q]);
            const uint64_t stop = take & __ballot(Tn < kTMin);
            const uint64_t comp_m = take & ~stop;
            const bool comp = __builtin_amdgcn_inverse_ballot_w64(comp_m);
            const float w = comp ? al[k] * T[q] : 0.f;
            c0[q] = fmaf(r2[k].x, w, c0[q]);
            c1[q] = fmaf(r2[k].y, w, c1[q]);
            c2[q] = fmaf(r2[k].z, w, c2[q]);
            T[q] = comp ? Tn : T[q];
            n[q] = add_bit(n[q], comp_m);
            last[q] = comp ? b0 + j[k] + 1 : last[q];
            if (stop != 0ull) {   // uniform
              live[q] &= ~stop;
              if (live[q] == 0ull) qlive &= ~(1u << q);
            }
          }
        }
      }
    }
  }
  const int64_t HW = (int64_t)view.width * view.height;
  float* im = a.img + 3 * view.pix_off;
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    const int px = px0 + (q % G::NX) * G::SLW, py = py0 + (q / G::NX) * G::SLH;
    if (px < view.width && py < view.height) {
      const int64_t p = (int64_t)py * view.width + px;
      const float Tf = T[q];
      im[p] = fmaf(Tf, a.bg0, c0[q]);
      im[HW + p] = fmaf(Tf, a.bg1, c1[q]);
      im[2 * HW + p] = fmaf(Tf, a.bg2, c2[q]);
      a.T[view.pix_off + p] = Tf;
      a.ncontrib[view.pix_off + p] = n[q];
      a.last[view.pix_off + p] = last[q];
    }
  }
}

// One workgroup per tile (schedules 0 and 1).  Held to eight wavefronts per
// SIMD: the strip tests would otherwise cost the compiler the few registers
// that take it to seven (nothing is spilled).
template <int TW, int TH, int PPT, int SW, int BATCH>
__global__ __launch_bounds__(TW* TH / PPT) __attribute__((amdgpu_waves_per_eu(8))) void k_composite(CompArgs a) {
  __shared__ FwdShared<BATCH, (Geom<TW, TH, PPT, SW>::NWAVES >= 2 ? 2u : 1u)> sm;
  composite_tile<TW, TH, PPT, SW, BATCH>(a, tile_of_block(blockIdx.x, (uint32_t)a.ntiles, a.schedule), sm);
}

// Persistent (schedules 2 and 3): as many workgroups as fit on the chip at
// once, each taking the call's tiles from the work queue until it is empty.
// Held to eight wavefronts per SIMD like the grid kernel: at four pixels per
// lane the loop around the tile body then spills three to seven registers, and
// still every shape is at least as fast as at seven (1M Gaussians, four views of
// 1280x720, batches of 64: 32x32 tiles at one pixel per lane 792 us instead of
// 1174, at two 452 and 498, at four 388 and 408).
template <int TW, int TH, int PPT, int SW, int BATCH>
__global__ __launch_bounds__(TW* TH / PPT) __attribute__((amdgpu_waves_per_eu(8))) void k_composite_persistent(
    CompArgs a) {
  __shared__ FwdShared<BATCH, (Geom<TW, TH, PPT, SW>::NWAVES >= 2 ? 2u : 1u)> sm;
  __shared__ uint32_t s_next;
  for (;;) {
    const uint32_t slot = queue_next(a.q, (uint32_t)a.ntiles, &s_next);
    if (slot == kQueueDone) break;
    composite_tile<TW, TH, PPT, SW, BATCH>(a, slot, sm);
  }
  queue_exit(a.q);
}

struct BwdArgs {
  const ViewInfo* views;
  const int32_t* tile_view;
  int32_t tile_begin;
  int32_t ntiles;
  int32_t schedule;
  const uint2* ranges;
  const uint32_t* vals;
  const float4* rec;
  const float* img;
  const float* T;
  const uint32_t* last;
  const float* up;
  const uint32_t* strips;   // per list position: the forward's two 16-bit halves of the strip bits
  int mode;
  int loss_mode;
  float* g2;           // field f of pair o at g2[f * g2_plane + o]
  size_t g2_plane;
  float* loss;
  uint32_t cap;
  float bg0, bg1, bg2;
  uint32_t n_gauss;    // Gaussians per view in the value index v * n_gauss + i
  uint32_t n_active;   // Gaussians i < n_active are trainable; the rest are frozen
  TileQueue q;
};

// LDS of one compositing workgroup (adjoint).
template <int BATCH, int NWAVES>
struct BwdShared {
  // splats whose sums are kept at a time: the batch's, over the tile's
  // wavefronts; those of each 64 that a lone wavefront works on, as with 256 it
  // would have 6 instead of 9 workgroups per compute unit (1M Gaussians, four
  // views of 1280x720, batches of 256: 16x16 tiles at four pixels per lane 1367
  // instead of 1642 us, 16x8 at two 1924 and 2293)
  static constexpr int SUMS = NWAVES == 1 && BATCH > 64 ? 64 : BATCH;
  float4 rec[BATCH * 3];
  uint32_t mask[BATCH];
  uint32_t id[BATCH];
  // the splats' sums, field-major; the odd stride puts one splat's fields in
  // different banks.  Zero between batches.
  float g[9 * (SUMS + 1)];
  uint32_t max_last;
};

template <int TW, int TH, int PPT, int SW, int BATCH>
using BwdSharedOf = BwdShared<BATCH, Geom<TW, TH, PPT, SW>::NWAVES>;

// Adjoint of the compositing of one pixel, walked back to front from the
// pixel's last composited splat (Sj = colour arriving from behind splat j,
// background included; T rebuilt from T_final by division):
//   T_j = T_{j+1} / (1 - alpha_j)
//   d out / d col_j   = alpha_j T_j
//   d out / d alpha_j = T_j (col_j - S_j),   S_{j-1} = alpha_j col_j + (1 - alpha_j) S_j
// Only the projection SG_j = S_j . G of S onto the pixel's upstream gradient
// G enters the adjoint, so one scalar per pixel is carried back:
//   d L / d alpha_j = T_j (col_j . G - SG_j),   SG_{j-1} = SG_j + alpha_j (col_j . G - SG_j).
// The division chain runs in FP32 with the hardware reciprocal: each step adds
// at most about 4 units of 2^-24 to T_j's relative error (reciprocal, product,
// and 1 - alpha), which stays inside the same E_p = sum 1/(1 - alpha) bound
// as the forward product's own rounding.
// Adjoint of the compositing of tile `slot` of the call by the whole workgroup.
template <int TW, int TH, int PPT, int SW, int BATCH>
__device__ __forceinline__ void composite_bwd_tile(const BwdArgs& a, uint32_t slot, BwdSharedOf<TW, TH, PPT, SW, BATCH>& sm) {
  using G = Geom<TW, TH, PPT, SW>;
  constexpr int SUMS = BwdSharedOf<TW, TH, PPT, SW, BATCH>::SUMS;
  constexpr int K = G::SPLATS;
  float4* s_rec = sm.rec;
  uint32_t* s_mask = sm.mask;
  uint32_t* s_id = sm.id;
  float* s_g = sm.g;
  uint32_t& s_max = sm.max_last;
  const int t = a.tile_begin + (int)slot;
  const ViewInfo view = a.views[a.tile_view[t]];
  const int local = t - view.tile_base;
  const int ty = local / view.tiles_x, tx = local - ty * view.tiles_x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x0 = tx * TW + (wave % G::WPR) * SW, y0 = ty * TH + (wave / G::WPR) * G::WROWS;
  const int px0 = x0 + lane % G::SLW, py0 = y0 + lane / G::SLW;
  const uint2 rg = clamp_range(a.ranges[t], a.cap);
  const float pxc = (float)px0 + 0.5f, pyc = (float)py0 + 0.5f;
  const int64_t HW = (int64_t)view.width * view.height;
  const float wv = a.loss_mode == 1 ? 1.f / (3.f * (float)HW) : 1.f;
  const bool lo8 = (lane & 8) == 0;
  // the lanes that add a splat's totals into s_g, and the slot each adds to:
  // one lane per 8-lane group for the field reduce8 leaves there, and the
  // last lane of each row for its row's part of the ninth field
  const bool ninth = (lane & 15) == 15;
  const bool writer = (lane & 7) == 0 || ninth;
  const int my_field = reduce8_field(lane, lo8);   // by the whole wavefront
  const int my_slot = (ninth ? 8 : my_field) * (SUMS + 1);
  for (int q = threadIdx.x; q < 9 * (SUMS + 1); q += G::NT) s_g[q] = 0.f;
  if (threadIdx.x == 0) s_max = rg.x;
  __syncthreads();
  float G0[PPT], G1[PPT], G2[PPT], SG[PPT];
  float T[PPT];
  uint32_t last[PPT];
  float lossv = 0.f;
  uint32_t my_max = rg.x;
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    G0[q] = G1[q] = G2[q] = 0.f;
    T[q] = 1.f;
    last[q] = rg.x;
    const int px = px0 + (q % G::NX) * G::SLW, py = py0 + (q / G::NX) * G::SLH;
    if (px < view.width && py < view.height) {
      const int64_t p = (int64_t)py * view.width + px;
      const int64_t ib = 3 * view.pix_off + p;
      if (a.mode == 0) {
        G0[q] = a.up[ib];
        G1[q] = a.up[ib + HW];
        G2[q] = a.up[ib + 2 * HW];
      } else {
        const float d0 = a.img[ib] - a.up[ib];
        const float d1 = a.img[ib + HW] - a.up[ib + HW];
        const float d2 = a.img[ib + 2 * HW] - a.up[ib + 2 * HW];
        G0[q] = wv * (float)((d0 > 0.f) - (d0 < 0.f));
        G1[q] = wv * (float)((d1 > 0.f) - (d1 < 0.f));
        G2[q] = wv * (float)((d2 > 0.f) - (d2 < 0.f));
        lossv += wv * (fabsf(d0) + fabsf(d1) + fabsf(d2));
      }
      T[q] = a.T[view.pix_off + p];
      last[q] = min(max(a.last[view.pix_off + p], rg.x), rg.y);
      my_max = max(my_max, last[q]);
    }
    SG[q] = fmaf(a.bg2, G2[q], fmaf(a.bg1, G1[q], a.bg0 * G0[q]));   // the background behind all splats
  }
  atomicMax(&s_max, my_max);
  // per pixel slot, the wavefront's largest last position: list entries at or
  // past it reach no lane of that slot, so the slot skips them outright
  uint32_t qlast[PPT];
#pragma unroll
  for (int q = 0; q < PPT; ++q) qlast[q] = __builtin_amdgcn_readfirstlane(wave_max_u32(last[q]));
  uint32_t wlast = qlast[0];
#pragma unroll
  for (int q = 1; q < PPT; ++q) wlast = max(wlast, qlast[q]);
  __syncthreads();
  const uint32_t end_all = s_max;
  const bool all_active = a.n_active >= a.n_gauss;
  // `count` splats' totals to the global planes, a wavefront per field (the two
  // of the mean together, as both take the same sums); the LDS slots are left
  // at zero.  Slot e holds splat e of the batch (or `base` - e, see SUMS).
  auto flush = [&](int base, int count) {
    for (int f = wave; f < 8; f += G::NWAVES) {   // uniform
      for (int e = lane; e < count; e += 64) {
        const int j = SUMS == BATCH ? e : base - e;
        float* slot0 = s_g + e;
        float* slot1 = s_g + (f + 1) * (SUMS + 1) + e;
        const float4 r1 = s_rec[j * 3 + 1];   // staged: a and s carry -log2(e)/2
        float* dst = a.g2 + s_id[j];
        const float v = *slot1;
        if (f == 0) {
          const float me = *slot0;
          if (me == 0.f && v == 0.f) continue;
          const float ame = kMinus2Ln2 * r1.x * me;
          atomicAdd(dst, ame);
          atomicAdd(dst + a.g2_plane, fmaf(ame, r1.y, kMinus2Ln2 * r1.z * v));
          *slot0 = 0.f;
        } else {
          if (v == 0.f) continue;
          // d P / d conic = -1/2 dx^2, -dx dy, -1/2 dy^2; dP/do = 1/o per unit of alpha
          atomicAdd(dst + (size_t)(f + 1) * a.g2_plane, f == 4 ? v / r1.w : f == 2 ? -v : f < 4 ? -0.5f * v : v);
        }
        *slot1 = 0.f;
      }
    }
  };
  for (uint32_t b_end = end_all; b_end > rg.x;) {
    const uint32_t b_begin = (b_end - rg.x > (uint32_t)BATCH) ? b_end - BATCH : rg.x;
    const uint32_t cnt = b_end - b_begin;
    // records and the forward's strip bits; flags: the splat's Gaussian is
    // trainable (frozen ones still shape T and S), its alpha may be clamped
    for (uint32_t j = threadIdx.x; j < cnt; j += G::NT) {
      const uint32_t id = a.vals[b_begin + j];
      s_id[j] = id;
      const float4 r1 = a.rec[(size_t)id * 3 + 1];
      s_rec[j * 3 + 0] = a.rec[(size_t)id * 3 + 0];
      s_rec[j * 3 + 1] = staged_conic(r1);
      s_rec[j * 3 + 2] = a.rec[(size_t)id * 3 + 2];
      const uint32_t h2 = a.strips[b_begin + j];
      s_mask[j] = (h2 & 0xffffu) | ((h2 >> 16) << G::HALF_BITS) | (all_active || id % a.n_gauss < a.n_active ? kActiveBit : 0u) |
                  (r1.w >= kMayClamp ? kClampBit : 0u);
    }
    __syncthreads();
    // the wavefront starts at its own last position within the batch
    const int j_hi = wlast > b_begin ? (int)min(cnt, wlast - b_begin) - 1 : -1;
    // 64 splats at a time: lane l reads the strip word of splat base - l, and
    // the wavefront then visits only the splats that touch one of its strips
    // ahead of that slot's largest last position
    for (int base = j_hi; base >= 0; base -= 64) {
      const int jl = base - lane;
      uint32_t mw = 0u;
      if (jl >= 0) {
        const uint32_t word = s_mask[jl];
        uint32_t qm = 0u;
#pragma unroll
        for (int q = 0; q < PPT; ++q) qm |= b_begin + (uint32_t)jl < qlast[q] ? 1u << q : 0u;
        mw = ((word >> (wave * PPT)) & qm) | (word & (kActiveBit | kClampBit));
      }
      uint64_t pend = __ballot((mw & ((1u << PPT) - 1u)) != 0u);
      while (pend != 0ull) {
        // the next K pending splats (the last visit may hold fewer: word 0)
        int j[K];
        uint32_t word[K];
        float4 r1[K], r2[K];
        SplatOffsets<G> so[K];
        // per lane over its slots, with W = dL/dP: sums of W e, W dy, W dx^2,
        // W dx dy, W dy^2, W, and of alpha T G for the three colours; the
        // splat's own factors are applied to the totals at the flush
        float g[K][9];
        uint64_t taken[K];   // lanes that took the splat at one of their pixels
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const bool have = k == 0 || pend != 0ull;
          const int l = have ? __builtin_ctzll(pend) : 0;
          pend = clear_bit(pend, l);
          j[k] = base - l;
          word[k] = have ? (uint32_t)__builtin_amdgcn_readlane((int)mw, l) : 0u;
          const float4 r0 = s_rec[j[k] * 3];
          r1[k] = s_rec[j[k] * 3 + 1], r2[k] = s_rec[j[k] * 3 + 2];
          so[k].set(pxc, pyc, r0, r1[k]);
#pragma unroll
          for (int f = 0; f < 9; ++f) g[k][f] = 0.f;
          taken[k] = 0ull;
        }
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
          // uniform: the splat misses this pixel slot's strip, or lies behind
          // every lane's last composited splat (K > 1 goes with one slot,
          // which every pending splat reaches)
          if (K == 1 && !((word[0] >> q) & 1u)) continue;
          SplatGeom sg[K];
          uint64_t cand[K], any = 0ull;
#pragma unroll
          for (int k = 0; k < K; ++k) {
            sg[k] = so[k].power(q, r1[k]);
            cand[k] = __ballot(sg[k].P >= kCutoff2) & __ballot(b_begin + (uint32_t)j[k] < last[q]);
            if (k > 0 && word[k] == 0u) cand[k] = 0ull;
            any |= cand[k];
          }
          if constexpr (K > 1) {
#pragma unroll
            for (int k = 0; k < K; ++k) keep_loaded(r1[k], r2[k]);
          }
          if (any == 0ull) continue;   // uniform
          float al[K];
          uint64_t clamped[K];
          uint32_t flags = 0u;
#pragma unroll
          for (int k = 0; k < K; ++k) {
            al[k] = splat_opacity(sg[k].P, r1[k].w);
            clamped[k] = 0ull;
            flags |= word[k];
          }
          if (flags & kClampBit) {   // uniform, and rare: kept a branch
            asm volatile("");
#pragma unroll
            for (int k = 0; k < K; ++k) {
              clamped[k] = __ballot(al[k] >= kAlphaMax);
              al[k] = fminf(al[k], kAlphaMax);
            }
          }
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const uint64_t take = cand[k] & __ballot(al[k] >= kAlphaMin);
            taken[k] |= take;
            // predicated from here on: a lane that does not take the splat
            // runs with alpha 0, which leaves its T and S unchanged
            // (1/(1 - 0) is exactly 1) and adds zeros (staged records are
            // finite, so 0 times any product is 0).  A frozen splat runs the
            // same arithmetic (its sums are dropped below): a second,
            // gradient-free copy of this loop costs more registers than the
            // work it would save.
            const float alt = __builtin_amdgcn_inverse_ballot_w64(take) ? al[k] : 0.f;
            T[q] *= __builtin_amdgcn_rcpf(1.f - alt);
            const float at = alt * T[q];
            g[k][6] = fmaf(at, G0[q], g[k][6]);
            g[k][7] = fmaf(at, G1[q], g[k][7]);
            g[k][8] = fmaf(at, G2[q], g[k][8]);
            const float diff = fmaf(r2[k].z, G2[q], fmaf(r2[k].y, G1[q], r2[k].x * G0[q])) - SG[q];
            SG[q] = fmaf(alt, diff, SG[q]);
            // dL/dalpha dalpha/dP; the clamp cuts alpha off from opacity and power.
            // (Selected rather than left to alpha 0: an infinite or NaN upstream
            // gradient at a pixel that does not take the splat is no part of it.)
            const float W = __builtin_amdgcn_inverse_ballot_w64(take & ~clamped[k]) ? at * diff : 0.f;
            g[k][5] += W;
            g[k][0] = fmaf(W, sg[k].e, g[k][0]);
            const float tx_ = W * sg[k].dx, ty_ = W * sg[k].dy;
            g[k][1] += ty_;
            g[k][2] = fmaf(tx_, sg[k].dx, g[k][2]);
            g[k][3] = fmaf(tx_, sg[k].dy, g[k][3]);
            g[k][4] = fmaf(ty_, sg[k].dy, g[k][4]);
          }
        }
        uint64_t any = 0ull;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          if (!(word[k] & kActiveBit)) taken[k] = 0ull;   // frozen: its sums are dropped
          any |= taken[k];
        }
        if (any == 0ull) continue;
        float tot[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const float tot8 = reduce8(g[k], lo8);
          // the ninth field over each row of 16 lanes, its total in the last lane
          float tot9 = dpp_add<0x111, 0xf>(g[k][8]);
          tot9 = dpp_add<0x112, 0xf>(tot9);
          tot9 = dpp_add<0x114, 0xf>(tot9);
          tot9 = dpp_add<0x118, 0xf>(tot9);
          tot[k] = ninth ? tot9 : tot8;
        }
        // LDS float adds: one slot per (splat, field) for all wavefronts
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (taken[k] != 0ull) {   // uniform
            if (writer) atomicAdd(s_g + my_slot + (SUMS == BATCH ? j[k] : base - j[k]), tot[k]);
          }
      }
      if (SUMS < BATCH) {
        __syncthreads();
        flush(base, min(base + 1, 64));
      }
    }
    __syncthreads();
    if (SUMS == BATCH) flush(0, (int)cnt);
    __syncthreads();
    b_end = b_begin;
  }
  if (a.mode == 1) {
    lossv = wave_total_lane63(lossv);
    if (lane == 63 && lossv != 0.f) atomicAdd(a.loss, lossv);
  }
}

// One workgroup per tile (schedules 0 and 1).
template <int TW, int TH, int PPT, int SW, int BATCH>
__global__ __launch_bounds__(TW* TH / PPT) void k_composite_bwd(BwdArgs a) {
  __shared__ BwdSharedOf<TW, TH, PPT, SW, BATCH> sm;
  composite_bwd_tile<TW, TH, PPT, SW, BATCH>(a, tile_of_block(blockIdx.x, (uint32_t)a.ntiles, a.schedule), sm);
}

// Persistent (schedules 2 and 3), as k_composite_persistent.  Held to seven
// wavefronts per SIMD, for the shapes with four pixels per lane: at eight they
// take up to 7% longer (100k Gaussians in two views of 1280x720, 32x32 tiles,
// batches of 64: 265 us at seven, 279 at eight); 32x32 tiles with one pixel per
// lane would gain a quarter (1M Gaussians in four views 2052 and 1557), with
// two 5%.
template <int TW, int TH, int PPT, int SW, int BATCH>
__global__ __launch_bounds__(TW* TH / PPT) __attribute__((amdgpu_waves_per_eu(7))) void k_composite_bwd_persistent(
    BwdArgs a) {
  __shared__ BwdSharedOf<TW, TH, PPT, SW, BATCH> sm;
  __shared__ uint32_t s_next;
  for (;;) {
    const uint32_t slot = queue_next(a.q, (uint32_t)a.ntiles, &s_next);
    if (slot == kQueueDone) break;
    composite_bwd_tile<TW, TH, PPT, SW, BATCH>(a, slot, sm);
  }
  queue_exit(a.q);
}

// ---- dispatch over the built (tile, pixels-per-thread, batch) variants ----
#define GS_RASTER_LIST(X) \
  X(8, 8, 1, 8)           \
  X(16, 8, 1, 16)         \
  X(16, 8, 2, 16)         \
  X(16, 16, 1, 16)        \
  X(16, 16, 2, 16)        \
  X(16, 16, 4, 16)        \
  X(32, 16, 1, 32)        \
  X(32, 16, 2, 32)        \
  X(32, 16, 4, 32)        \
  X(32, 16, 2, 16)        \
  X(32, 16, 4, 16)        \
  X(32, 32, 1, 32)        \
  X(32, 32, 2, 32)        \
  X(32, 32, 4, 32)        \
  X(32, 32, 2, 16)        \
  X(32, 32, 4, 16)

// Workgroups of `kernel` (NT threads) resident on the whole device at once:
// the grid of a persistent launch.  Queried once per kernel.
template <typename K>
hipError_t resident_workgroups(K kernel, int nt, int* out) {
  static int cached = 0;
  if (cached > 0) {
    *out = cached;
    return hipSuccess;
  }
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, nt, 0);
  if (e != hipSuccess) return e;
  cached = (cus > 0 ? cus : 1) * (per_cu > 0 ? per_cu : 1);
  *out = cached;
  return hipSuccess;
}

template <typename K, typename Args>
hipError_t launch_grid_or_persistent(K grid_kernel, K persistent_kernel, int nt, uint32_t ntiles, bool persistent,
                                     hipStream_t st, const Args& a) {
  if (!persistent) {
    hipLaunchKernelGGL(grid_kernel, dim3(ntiles), dim3(nt), 0, st, a);
    return hipGetLastError();
  }
  int res = 0;
  const hipError_t e = resident_workgroups(persistent_kernel, nt, &res);
  if (e != hipSuccess) return e;
  const uint32_t g = ntiles < (uint32_t)res ? ntiles : (uint32_t)res;
  hipLaunchKernelGGL(persistent_kernel, dim3(g), dim3(nt), 0, st, a);
  return hipGetLastError();
}

template <int TW, int TH, int PPT, int SW, typename Args>
hipError_t launch_fwd(int batch, uint32_t ntiles, bool persistent, hipStream_t st, const Args& a) {
  constexpr int NT = TW * TH / PPT;
  switch (batch) {
    case 32:
      return launch_grid_or_persistent(k_composite<TW, TH, PPT, SW, 32>, k_composite_persistent<TW, TH, PPT, SW, 32>,
                                       NT, ntiles, persistent, st, a);
    case 64:
      return launch_grid_or_persistent(k_composite<TW, TH, PPT, SW, 64>, k_composite_persistent<TW, TH, PPT, SW, 64>,
                                       NT, ntiles, persistent, st, a);
    case 128:
      return launch_grid_or_persistent(k_composite<TW, TH, PPT, SW, 128>,
                                       k_composite_persistent<TW, TH, PPT, SW, 128>, NT, ntiles, persistent, st, a);
    case 256:
      return launch_grid_or_persistent(k_composite<TW, TH, PPT, SW, 256>,
                                       k_composite_persistent<TW, TH, PPT, SW, 256>, NT, ntiles, persistent, st, a);
    default: return hipErrorInvalidValue;
  }
}

template <int TW, int TH, int PPT, int SW, typename Args>
hipError_t launch_bwd(int batch, uint32_t ntiles, bool persistent, hipStream_t st, const Args& a) {
  constexpr int NT = TW * TH / PPT;
  switch (batch) {
    case 32:
      return launch_grid_or_persistent(k_composite_bwd<TW, TH, PPT, SW, 32>,
                                       k_composite_bwd_persistent<TW, TH, PPT, SW, 32>, NT, ntiles, persistent, st, a);
    case 64:
      return launch_grid_or_persistent(k_composite_bwd<TW, TH, PPT, SW, 64>,
                                       k_composite_bwd_persistent<TW, TH, PPT, SW, 64>, NT, ntiles, persistent, st, a);
    case 128:
      return launch_grid_or_persistent(k_composite_bwd<TW, TH, PPT, SW, 128>,
                                       k_composite_bwd_persistent<TW, TH, PPT, SW, 128>, NT, ntiles, persistent, st,
                                       a);
    case 256:
      return launch_grid_or_persistent(k_composite_bwd<TW, TH, PPT, SW, 256>,
                                       k_composite_bwd_persistent<TW, TH, PPT, SW, 256>, NT, ntiles, persistent, st,
                                       a);
    default: return hipErrorInvalidValue;
  }
}

// The work queue of a persistent launch (schedules 2 and 3) in the workspace.
TileQueue tile_queue(const Plan& pl, void* ws) {
  TileQueue q;
  q.head = seg<Counters>(ws, pl.ws.counters)->queue;
  q.order = pl.schedule == 3 ? seg<uint32_t>(ws, pl.ws.order) : nullptr;
  return q;
}

void tile_span(const Plan& pl, int v0, int nv, int32_t* tb, int32_t* ntiles) {
  *tb = pl.views[v0].tile_base;
  const int32_t te = (v0 + nv < pl.n_views) ? pl.views[v0 + nv].tile_base : pl.total_tiles;
  *ntiles = te - *tb;
}

}  // namespace

bool raster_variant_built(int tw, int th, int ppt, int sw) {
#define GS_HAS(W, H, P, S) \
  if (tw == W && th == H && ppt == P && sw == S) return true;
  GS_RASTER_LIST(GS_HAS)
#undef GS_HAS
  return false;
}

bool sorted_values_in_b(const Plan& pl, int v0, int nv) {
  const int32_t tb = pl.views[v0].tile_base;
  const int32_t te = (v0 + nv < pl.n_views) ? pl.views[v0 + nv].tile_base : pl.total_tiles;
  int bits = 0;
  while ((1ll << bits) < (int64_t)(te - tb)) ++bits;
  const int passes = bits == 0 ? 1 : (bits + 7) / 8;
  return (passes & 1) != 0;
}

hipError_t launch_composite(const Plan& pl, int v0, int nv, void* ws, float* img, float* T, uint32_t* nc,
                            hipStream_t st) {
  CompArgs a;
  a.views = pl.d_views;
  a.tile_view = pl.d_tile_view;
  a.schedule = pl.schedule;
  int32_t ntiles;
  tile_span(pl, v0, nv, &a.tile_begin, &ntiles);
  a.ntiles = ntiles;
  a.ranges = seg<uint2>(ws, pl.ws.ranges);
  a.vals = seg<uint32_t>(ws, sorted_values_in_b(pl, v0, nv) ? pl.ws.vals_b : pl.ws.vals_a);
  a.rec = seg<float4>(ws, pl.ws.rec);
  a.img = img;
  a.T = T;
  a.ncontrib = nc;
  a.last = seg<uint32_t>(ws, pl.ws.last);
  a.strips = seg<uint16_t>(ws, pl.ws.strips);
  a.cap = (uint32_t)pl.cap;
  a.bg0 = pl.bg[0];
  a.bg1 = pl.bg[1];
  a.bg2 = pl.bg[2];
  a.q = tile_queue(pl, ws);
  if (ntiles <= 0) return hipSuccess;
  const bool persistent = pl.schedule >= 2;
  const int tw = pl.tile_w, th = pl.tile_h, ppt = pl.ppt, sw = pl.wave_w, b = pl.batch_depth;
#define GS_FWD(W, H, P, S) \
  if (tw == W && th == H && ppt == P && sw == S) return launch_fwd<W, H, P, S>(b, (uint32_t)ntiles, persistent, st, a);
  GS_RASTER_LIST(GS_FWD)
#undef GS_FWD
  return hipErrorInvalidValue;
}

hipError_t launch_composite_bwd(const Plan& pl, int v0, int nv, void* ws, const float* img, const float* T,
                                const float* up, int mode, float* loss, int32_t n_active, hipStream_t st) {
  BwdArgs a;
  a.n_gauss = (uint32_t)pl.n;
  a.n_active = (uint32_t)n_active;
  a.views = pl.d_views;
  a.tile_view = pl.d_tile_view;
  a.schedule = pl.schedule;
  int32_t ntiles;
  tile_span(pl, v0, nv, &a.tile_begin, &ntiles);
  a.ntiles = ntiles;
  a.ranges = seg<uint2>(ws, pl.ws.ranges);
  a.vals = seg<uint32_t>(ws, sorted_values_in_b(pl, v0, nv) ? pl.ws.vals_b : pl.ws.vals_a);
  a.rec = seg<float4>(ws, pl.ws.rec);
  a.img = img;
  a.T = T;
  a.last = seg<uint32_t>(ws, pl.ws.last);
  a.up = up;
  a.strips = seg<uint32_t>(ws, pl.ws.strips);
  a.mode = mode;
  a.loss_mode = pl.loss_mode;
  a.g2 = seg<float>(ws, pl.ws.g2);
  a.g2_plane = (size_t)pl.ws.vn;
  a.loss = loss;
  a.cap = (uint32_t)pl.cap;
  a.bg0 = pl.bg[0];
  a.bg1 = pl.bg[1];
  a.bg2 = pl.bg[2];
  a.q = tile_queue(pl, ws);
  if (ntiles <= 0) return hipSuccess;
  const bool persistent = pl.schedule >= 2;
  const int tw = pl.tile_w, th = pl.tile_h, ppt = pl.ppt, sw = pl.wave_w, b = pl.batch_depth;
#define GS_BWD(W, H, P, S) \
  if (tw == W && th == H && ppt == P && sw == S) return launch_bwd<W, H, P, S>(b, (uint32_t)ntiles, persistent, st, a);
  GS_RASTER_LIST(GS_BWD)
#undef GS_BWD
  return hipErrorInvalidValue;
}

}  // namespace gs
