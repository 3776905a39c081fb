// Tile lists: depth pre-sort of the visible pairs (its first pass takes them
// from the dense (view, Gaussian) arrays, compacting as it sorts), key
// emission, radix sort by tile, per-tile ranges.
//
// Order required by the compositing rule: within a tile, splats ascend by
// (FP32 depth bits, Gaussian index).  Instead of sorting one 64-bit
// (tile | depth) key per (tile, Gaussian) pair, the visible (view, Gaussian)
// pairs (a few per Gaussian) are sorted by depth first, keys are emitted in
// that order, and a stable sort on the tile bits alone finishes the job:
// 4 passes over the visible pairs plus ceil(tile bits / 8) passes over the
// keys, instead of ~7 passes over the keys.  Tile ids of up to 16 bits are
// sorted from their high half down: the first pass (fused with the emission)
// leaves the keys in up to 256 buckets, of which only the low byte goes on,
// and the second, inside the buckets, writes values alone and reads the tiles'
// ranges off its digit starts.  From the low digit up, with whole keys, the two
// passes, their counts and the range extraction of 58M keys took 0.82 ms
// instead of 0.59.
//
// All kernels are driven by device-side counts so the stage can be captured
// in a graph: grids are sized for the plan's capacity and idle blocks exit.
#include "internal.h"
#include "list_route.h"

namespace gs {
namespace {

constexpr int B = kSortBlock;
constexpr int NW = B / 64;
static_assert(B >= 256 && B % 256 == 0, "at least one thread per radix digit");

__device__ __forceinline__ uint32_t dev_count(const uint32_t* dcount, int64_t max_count) {
  if (!dcount) return (uint32_t)max_count;
  const uint32_t c = *dcount;
  return c < (uint64_t)max_count ? c : (uint32_t)max_count;
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  return x;
}

// Exclusive scan over the block (W wavefronts); *total receives the block sum.
template <int W = NW>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t* s_wave, uint32_t* total) {
  const uint32_t inc = wave_incl_scan(x);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 63) s_wave[w] = inc;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const uint32_t s = s_wave[k];
    pre += (k < w) ? s : 0u;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return pre + inc - x;
}

__device__ __forceinline__ uint32_t rect_area(uint2 r) {
  // (tx0 | ty0 << 16, tx1 | ty1 << 16): inclusive tile rectangle
  return ((r.y & 0xffffu) - (r.x & 0xffffu) + 1u) * ((r.y >> 16) - (r.x >> 16) + 1u);
}

// Value source of a scan: a[k], (a[k] != 0), a[idx[k]], or the area of
// tile rectangle k (mode 3, a = rectangles as uint2).
struct ScanSrc {
  const uint32_t* a;
  const uint32_t* idx;
  int mode;
  __device__ __forceinline__ uint32_t operator()(uint32_t k) const {
    if (mode == 0) return a[k];
    if (mode == 1) return a[k] != 0u ? 1u : 0u;
    if (mode == 3) return rect_area(reinterpret_cast<const uint2*>(a)[k]);
    return a[idx[k]];
  }
  // Four consecutive values from k (a multiple of 4) with one 16-byte load of
  // the directly indexed array.
  __device__ __forceinline__ void four(uint32_t k, uint32_t v[4]) const {
    if (mode == 3) {
      const uint4 x = *reinterpret_cast<const uint4*>(a + 2 * (size_t)k);
      const uint4 y = *reinterpret_cast<const uint4*>(a + 2 * (size_t)k + 4);
      v[0] = rect_area(make_uint2(x.x, x.y)), v[1] = rect_area(make_uint2(x.z, x.w));
      v[2] = rect_area(make_uint2(y.x, y.y)), v[3] = rect_area(make_uint2(y.z, y.w));
      return;
    }
    const uint4 x = *reinterpret_cast<const uint4*>((mode == 2 ? idx : a) + k);
    if (mode == 0) {
      v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
    } else if (mode == 1) {
      v[0] = x.x != 0u, v[1] = x.y != 0u, v[2] = x.z != 0u, v[3] = x.w != 0u;
    } else {
      v[0] = a[x.x], v[1] = a[x.y], v[2] = a[x.z], v[3] = a[x.w];
    }
  }
  __device__ __forceinline__ bool vec_ok() const {
    return ((reinterpret_cast<uintptr_t>(mode == 2 ? idx : a)) & 15u) == 0;
  }
};

// Chunk layout of the scan kernels: thread t holds elements
//   begin + r * 4B + 4t + c   (round r < kRounds, component c < 4),
// so every round is one coalesced 16-byte load per thread.
constexpr int kRounds = kSortItems / 4;
static_assert(kRounds * 4 * B == kSortChunk, "scan chunk layout");

// The uniform choice between the whole-chunk and the ragged form is taken
// once, outside the rounds, so that the whole-chunk form issues all of its
// loads before waiting for any (chosen per round, the two forms' merged
// registers made every round's load wait for the previous one).
__device__ __forceinline__ void load_chunk(const ScanSrc& src, uint64_t begin, uint32_t n,
                                           uint32_t v[kRounds][4]) {
  if (begin + kSortChunk <= n && src.vec_ok()) {
#pragma unroll
    for (int r = 0; r < kRounds; ++r) src.four((uint32_t)(begin + (uint64_t)r * 4 * B + 4u * threadIdx.x), v[r]);
  } else {
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint64_t k = begin + (uint64_t)r * 4 * B + 4u * threadIdx.x;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[r][c] = k + c < n ? src((uint32_t)(k + c)) : 0u;
    }
  }
}

__global__ __launch_bounds__(B) void k_scan_reduce(ScanSrc src, int64_t max_count, const uint32_t* dcount,
                                                   uint32_t* partial) {
  __shared__ uint32_t s_wave[NW];
  const uint32_t n = dev_count(dcount, max_count);
  const uint64_t begin = (uint64_t)blockIdx.x * kSortChunk;
  if (begin >= n) return;
  uint32_t v[kRounds][4];
  load_chunk(src, begin, n, v);
  uint32_t s = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) s += (v[r][0] + v[r][1]) + (v[r][2] + v[r][3]);
  uint32_t tot;
  block_excl_scan(s, s_wave, &tot);
  if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// Single block: exclusive scan of the per-chunk partial sums in place.
__global__ __launch_bounds__(1024) void k_scan_partials(int64_t max_count, const uint32_t* dcount, uint32_t* partial,
                                                        uint32_t* total) {
  __shared__ uint32_t s_w[16];
  __shared__ uint32_t s_carry;
  const uint32_t n = dev_count(dcount, max_count);
  const uint32_t np = (uint32_t)((n + kSortChunk - 1) / kSortChunk);
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (uint32_t base = 0; base < np; base += 1024) {
    const uint32_t k = base + threadIdx.x;
    const uint32_t x = k < np ? partial[k] : 0u;
    const uint32_t inc = wave_incl_scan(x);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
    for (int q = 0; q < 16; ++q) {
      pre += (q < w) ? s_w[q] : 0u;
      tot += s_w[q];
    }
    const uint32_t carry = s_carry;
    if (k < np) partial[k] = carry + pre + inc - x;
    __syncthreads();
    if (threadIdx.x == 0) s_carry = carry + tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partial[np] = s_carry;
    if (total) *total = s_carry;
  }
}

// With `firsts` (the key-offset scan), element k, whose run of out[k] .. out[k]
// + value - 1 slots it now knows, also records itself as the owner of every
// chunk of kSortChunk slots that starts inside that run: firsts[m] = k for
// m K in [out[k], out[k] + value), m < firsts_len.
// With `direct`, partial holds the chunks' own sums (k_scan_partials has not
// run): each block adds up those before it, and the last block writes the
// total (block 0 writes 0 when there is nothing to scan).
__global__ __launch_bounds__(B) void k_scan_down(ScanSrc src, uint32_t* out, int64_t max_count,
                                                 const uint32_t* dcount, const uint32_t* partial,
                                                 uint32_t* firsts, uint32_t firsts_len, bool direct,
                                                 uint32_t* total) {
  __shared__ uint32_t s_wave[kRounds][NW];
  __shared__ uint32_t s_pre[NW];
  const uint32_t n = dev_count(dcount, max_count);
  const uint64_t begin = (uint64_t)blockIdx.x * kSortChunk;
  if (begin >= n) {
    if (direct && total && blockIdx.x == 0 && threadIdx.x == 0) *total = 0u;
    return;
  }
  uint32_t v[kRounds][4];
  load_chunk(src, begin, n, v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t s[kRounds], inc[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    s[r] = (v[r][0] + v[r][1]) + (v[r][2] + v[r][3]);
    inc[r] = wave_incl_scan(s[r]);
    if (lane == 63) s_wave[r][w] = inc[r];
  }
  __syncthreads();
  uint32_t carry;
  if (direct) {
    uint32_t x = 0;
    for (uint32_t q = threadIdx.x; q < blockIdx.x; q += B) x += partial[q];
    block_excl_scan(x, s_pre, &carry);
  } else {
    carry = partial[blockIdx.x];
  }
  const bool full = begin + kSortChunk <= n && ((reinterpret_cast<uintptr_t>(out)) & 15u) == 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const uint32_t x = s_wave[r][q];
      before += (q < w) ? x : 0u;
      tot += x;
    }
    uint32_t run = carry + before + inc[r] - s[r];
    carry += tot;
    const uint64_t k = begin + (uint64_t)r * 4 * B + 4u * threadIdx.x;
    uint32_t o[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      o[c] = run;
      run += v[r][c];
    }
    if (firsts) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (k + c >= n) continue;
        const uint64_t lo = o[c], hi = lo + v[r][c];
        for (uint64_t m = (lo + kSortChunk - 1) / kSortChunk; m < firsts_len && m * kSortChunk < hi; ++m)
          firsts[m] = (uint32_t)(k + c);
      }
    }
    if (full) {
      *reinterpret_cast<uint4*>(out + k) = make_uint4(o[0], o[1], o[2], o[3]);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (k + c < n) out[k + c] = o[c];
    }
  }
  if (direct && total && begin + kSortChunk >= n && threadIdx.x == 0) *total = carry;
}

__global__ void k_fill_u32(uint32_t* p, uint32_t value, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = value;
}

// ---- radix sort (LSD, digits of up to 8 bits, stable) -----------------------
// Digit counts of one chunk per workgroup; each thread loads its kSortItems
// keys with 16-byte loads (the scan chunk layout) and counts them with LDS
// atomics into one of kHistCopies interleaved copies of its wavefront's
// histogram (copy lane % kHistCopies; the copies of a digit are adjacent
// words, so in different banks).  A skewed digit (the exponent byte of depth
// keys) then meets at most 64 / kHistCopies lanes of one wavefront at each
// address instead of 64.  Counts are stored where hist_at says.
constexpr int kHistCopies = 1024 / B;

// Chunk of workgroup blockIdx.x of a scatter over `chunks` chunks (chunks or more:
// none).  Workgroups are dealt to the eight XCDs in turn; each takes a
// contiguous run of chunks, as the lines where a digit's run of one chunk ends
// and that of the next begins are then completed in one L2 instead of being
// written in parts from two: the depth passes over 16M pairs, 9.6M of them
// visible, take 93 and 62 us instead of 122 and 75.  (Not the emission, whose
// chunks write twice as many runs: 3M Gaussians in four views 390 instead of
// 330 us.)  Grids are multiples of eight (xcd_grid).
__device__ __forceinline__ uint32_t xcd_chunk(uint32_t chunks) {
  const uint32_t xcd = blockIdx.x & 7u, k = blockIdx.x >> 3, each = chunks >> 3, more = chunks & 7u;
  return k < each + (xcd < more ? 1u : 0u) ? xcd * each + min(xcd, more) + k : chunks;
}
inline unsigned xcd_grid(int64_t chunks) { return (unsigned)((chunks + 7) / 8 * 8); }

// Sorts of up to kDirectChunks chunks scan no histogram: it is stored chunk by
// chunk instead of digit by digit, and each scatter workgroup adds up the rows
// of the chunks before its own itself (coalesced, from L2).  The scan costs two
// launches of 4 to 5 us a pass however few chunks there are; the rows cost a
// workgroup about 1 us per 32 chunks.
constexpr int64_t kDirectChunks = 320;

// Where a histogram holds the count of a digit in a chunk: digit by digit
// (digit * nblocks + chunk), as the scan wants it, or chunk by chunk (chunk *
// 256 + digit) where it is read as it is.
__device__ __forceinline__ int64_t hist_at(uint32_t digit, uint32_t chunk, int64_t nblocks, bool direct) {
  return direct ? (int64_t)chunk * 256 + digit : (int64_t)digit * nblocks + chunk;
}

// Global start of digit threadIdx.x's run of chunk `chunk`, from the
// unscanned rows of `chunks` chunks; *all receives the keys of all of them.
__device__ __forceinline__ uint32_t direct_digit_base(const uint32_t* hist, uint32_t chunk, uint32_t chunks,
                                                      uint32_t* s_tmp, uint32_t* all) {
  uint32_t before = 0, total = 0;
  if (threadIdx.x >= 256) chunks = 0;
#pragma unroll 16
  for (uint32_t c = 0; c < chunks; ++c) {
    const uint32_t x = hist[(size_t)c * 256 + threadIdx.x];
    before += c < chunk ? x : 0u;
    total += x;
  }
  return block_excl_scan(total, s_tmp, all) + before;
}

// With `valid` (the first depth pass, reading the dense (view, Gaussian)
// arrays), key k counts only where valid[k] != 0: the pass then compacts the
// visible pairs as it sorts them.
__global__ __launch_bounds__(B) void k_radix_hist(const uint32_t* keys, const uint32_t* valid, int64_t max_count,
                                                  const uint32_t* dcount, int shift, uint32_t dmask, int64_t nblocks,
                                                  uint32_t* hist, bool direct) {
  __shared__ uint32_t h[NW][256][kHistCopies];
#pragma unroll
  for (int q = 0; q < NW * kHistCopies * 256 / B; ++q) (&h[0][0][0])[q * B + threadIdx.x] = 0;
  __syncthreads();
  const uint32_t n = dev_count(dcount, max_count);
  const int w = threadIdx.x >> 6, copy = threadIdx.x & (kHistCopies - 1);
  const int64_t chunk = blockIdx.x;
  const uint64_t begin = (uint64_t)chunk * kSortChunk;
  if (chunk < nblocks && begin < n) {
    uint32_t v[kRounds][4], ok[kRounds][4];
    load_chunk(ScanSrc{keys, nullptr, 0}, begin, n, v);
    if (valid) load_chunk(ScanSrc{valid, nullptr, 1}, begin, n, ok);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (begin + (uint64_t)r * 4 * B + 4u * threadIdx.x + c < n && (!valid || ok[r][c]))
          atomicAdd(&h[w][(v[r][c] >> shift) & dmask][copy], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x >= 256) return;
  uint32_t t = 0;
#pragma unroll
  for (int q = 0; q < NW; ++q)
#pragma unroll
    for (int k = 0; k < kHistCopies; ++k) t += h[q][threadIdx.x][k];
  if (chunk < nblocks) hist[hist_at(threadIdx.x, (uint32_t)chunk, nblocks, direct)] = t;
}

// Scatter of one chunk (kSortChunk keys, split into NW contiguous wavefront
// ranges).  1) Each wavefront ranks its keys stably within (wavefront, digit):
// lanes with equal digits are matched with eight ballots and a per-wavefront
// counter per digit advances by the group size.  2) Per digit, the chunk-local
// start (scan over digits) and the start of each wavefront's group.  3) Keys
// are placed in LDS in digit order (stable), 4) then written out with
// consecutive threads taking consecutive local positions, so each digit's run
// is stored contiguously: global position = scanned histogram of (digit,
// chunk) + position within the digit's run.  With kPay, a 64-bit payload per
// key follows the same permutation through the same LDS space afterwards.
constexpr int kWaveKeys = kSortChunk / NW;
constexpr int kWaveRounds = kWaveKeys / 64;
constexpr int kOutRounds = kSortChunk / B;

// The kernels of a sort hold their chunk in 512 threads of 8 keys: with 256 of
// 16 a sort too short to fill the chip takes a quarter longer (a scatter of one
// chunk per compute unit 12.7 instead of 10.4 us), a long one the same.
// Steps 1-4 of a scatter for the keys a chunk's wavefronts hold (key[r] and
// val[r] of lane l of wavefront w are chunk entry w kWaveKeys + r 64 + l;
// bit r of in_mask says whether it takes part).  s_wc must be zero and
// visible to the whole workgroup on entry.  pos[] (each key's local
// position) and dst[] (with kPay: the global position of local entry
// r B + threadIdx.x) serve a payload that follows the keys; returns the
// number of keys taken.  With kBounded, positions at or past `limit` are not
// written (a safeguard where the digit counts come from another kernel's
// arithmetic rather than from the keys themselves).  kKeyBytes: the keys are
// written whole (4), only their bits below the digit as one byte (1), or not
// at all (0).
template <bool kPay, bool kBounded = false, int kKeyBytes = 4>
__device__ __forceinline__ uint32_t rank_and_write(const uint32_t (&key)[kWaveRounds], const uint32_t (&val)[kWaveRounds],
                                                   uint32_t in_mask, uint32_t digit_base, int shift, uint32_t dmask,
                                                   uint32_t* s_key, uint32_t* s_val, uint32_t (*s_wc)[256],
                                                   uint32_t* s_gbase, uint32_t* s_tmp, uint32_t& s_taken,
                                                   uint32_t* kout, uint32_t* vout, uint32_t (&pos)[kWaveRounds],
                                                   uint32_t (&dst)[kPay ? kOutRounds : 1], uint32_t limit = 0u) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t lr[kWaveRounds];
  // 1. stable ranks within (wavefront, digit)
#pragma unroll
  for (int r = 0; r < kWaveRounds; ++r) {
    const bool taking = (in_mask >> r) & 1u;
    const uint32_t digit = (key[r] >> shift) & dmask;
    // lanes with this lane's digit, bit by bit: with s all ones where the bit
    // is set and zero elsewhere, ~(ballot ^ s) are the lanes that agree
    const uint64_t here = __ballot(taking);
    uint32_t lo = (uint32_t)here, hi = (uint32_t)(here >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      if (b >= 5 && (dmask >> b) == 0u) break;   // uniform: no digit has this bit
      const int32_t s = __builtin_amdgcn_sbfe((int)digit, b, 1);
      const uint64_t bb = __ballot(s != 0);
      lo &= ~((uint32_t)bb ^ (uint32_t)s);
      hi &= ~((uint32_t)(bb >> 32) ^ (uint32_t)s);
    }
    const uint64_t match = ((uint64_t)hi << 32) | lo;
    const uint32_t below = (uint32_t)__popcll(match & lt_mask);
    const uint32_t before = taking ? s_wc[w][digit] : 0u;
    __builtin_amdgcn_wave_barrier();
    lr[r] = before + below;
    if (taking && below == 0) s_wc[w][digit] = before + (uint32_t)__popcll(match);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // 2. chunk-local digit starts and per-wavefront group starts
  {
    const int d = threadIdx.x;
    uint32_t c[NW], tot = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      c[q] = d < 256 ? s_wc[q][d] : 0u;
      tot += c[q];
    }
    uint32_t all;
    const uint32_t lstart = block_excl_scan(tot, s_tmp, &all);
    if (d == 0) s_taken = all;
    if (d < 256) {
      uint32_t run = lstart;
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        s_wc[q][d] = run;
        run += c[q];
      }
      s_gbase[d] = digit_base - lstart;
    }
  }
  __syncthreads();
  // 3. local placement in digit order
#pragma unroll
  for (int r = 0; r < kWaveRounds; ++r) {
    pos[r] = s_wc[w][(key[r] >> shift) & dmask] + lr[r];
    if ((in_mask >> r) & 1u) {
      s_key[pos[r]] = key[r];
      s_val[pos[r]] = val[r];
    }
  }
  __syncthreads();
  // 4. coalesced write-out
  const uint32_t taken = s_taken;
#pragma unroll
  for (int r = 0; r < kOutRounds; ++r) {
    const uint32_t i = (uint32_t)r * B + threadIdx.x;
    if (i < taken) {
      const uint32_t k = s_key[i];
      const uint32_t d = s_gbase[(k >> shift) & dmask] + i;
      if (kBounded && d >= limit) continue;
      if constexpr (kKeyBytes == 4) kout[d] = k;
      if constexpr (kKeyBytes == 1) reinterpret_cast<uint8_t*>(kout)[d] = (uint8_t)(k & ((1u << shift) - 1u));
      vout[d] = s_val[i];
      if constexpr (kPay) dst[r] = d;
    }
  }
  return taken;
}

// kDense (the first depth pass): the input is the dense (view, Gaussian)
// range, key k is taken only where valid[k] != 0, and its value is
// value_base + k (the pair's index), so the pass compacts the visible pairs
// in (view, Gaussian) order as it sorts them.
template <bool kPay, bool kDense = false>
__global__ __launch_bounds__(B) void k_radix_scatter(const uint32_t* kin, const uint32_t* vin, uint32_t* kout,
                                                     uint32_t* vout, const uint2* pin, uint2* pout,
                                                     int64_t max_count, const uint32_t* dcount, int shift,
                                                     uint32_t dmask, int64_t nblocks, const uint32_t* hist, bool direct,
                                                     const uint32_t* valid = nullptr, uint32_t value_base = 0,
                                                     uint32_t* taken_out = nullptr) {
  __shared__ __align__(16) uint32_t s_kv[2 * kSortChunk];   // keys | values, later the payload
  __shared__ uint32_t s_wc[NW][256];
  __shared__ uint32_t s_gbase[256];
  __shared__ uint32_t s_tmp[NW];
  __shared__ uint32_t s_taken;   // keys of the chunk that take part (all but invalid dense entries)
  uint32_t* s_key = s_kv;
  uint32_t* s_val = s_kv + kSortChunk;
  const uint32_t n = dev_count(dcount, max_count);
  const uint32_t chunks = (uint32_t)(((uint64_t)n + kSortChunk - 1) / kSortChunk), chunk = xcd_chunk(chunks);
  if (chunk >= chunks) return;
  const uint64_t begin = (uint64_t)chunk * kSortChunk;
  const uint32_t cnt = (uint32_t)min((uint64_t)kSortChunk, (uint64_t)n - begin);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NW * 256 / B; ++q) (&s_wc[0][0])[q * B + threadIdx.x] = 0;
  uint32_t key[kWaveRounds], val[kWaveRounds];
  uint2 pay[kPay ? kWaveRounds : 1];
  // Each pass reads its input once: streaming loads leave the cache to the
  // histogram, the offsets and the output being assembled.  Every load of
  // the chunk is issued before any result is used (a whole chunk, the common
  // case, loads without conditions; the validity flags of a dense pass are
  // turned into the taken mask only afterwards), and a dense pass loads every
  // entry's key and payload whether or not it takes it: taken and skipped
  // entries share cache lines.
  uint32_t flag[kDense ? kWaveRounds : 1];
  const uint32_t lane0 = (uint32_t)w * kWaveKeys + (uint32_t)lane;
  // this chunk's global start of digit threadIdx.x, needed only after the
  // ranking: loaded with the keys so that its latency overlaps theirs
  uint32_t digit_base = direct || threadIdx.x >= 256 ? 0u : hist[(int64_t)threadIdx.x * nblocks + chunk];
  if (cnt == (uint32_t)kSortChunk) {   // uniform
#pragma unroll
    for (int r = 0; r < kWaveRounds; ++r) {
      const uint64_t k = begin + lane0 + (uint32_t)r * 64u;
      key[r] = __builtin_nontemporal_load(kin + k);
      if constexpr (kDense)
        flag[r] = __builtin_nontemporal_load(valid + k);
      else
        val[r] = __builtin_nontemporal_load(vin + k);
      if constexpr (kPay) {
        const uint32_t* pp = reinterpret_cast<const uint32_t*>(pin + k);
        pay[r] = make_uint2(__builtin_nontemporal_load(pp), __builtin_nontemporal_load(pp + 1));
      }
    }
  } else {
#pragma unroll
    for (int r = 0; r < kWaveRounds; ++r) {
      const uint32_t li = lane0 + (uint32_t)r * 64u;
      const bool here = li < cnt;
      key[r] = here ? __builtin_nontemporal_load(kin + begin + li) : 0u;
      if constexpr (kDense)
        flag[r] = here ? __builtin_nontemporal_load(valid + begin + li) : 0u;
      else
        val[r] = here ? __builtin_nontemporal_load(vin + begin + li) : 0u;
      if constexpr (kPay) {
        if (here) {
          const uint32_t* pp = reinterpret_cast<const uint32_t*>(pin + begin + li);
          pay[r] = make_uint2(__builtin_nontemporal_load(pp), __builtin_nontemporal_load(pp + 1));
        } else {
          pay[r] = make_uint2(0u, 0u);
        }
      }
    }
  }
  uint32_t in_mask = 0;   // bit r: this lane's key of round r takes part
#pragma unroll
  for (int r = 0; r < kWaveRounds; ++r) {
    const uint32_t li = lane0 + (uint32_t)r * 64u;
    bool in = li < cnt;
    if constexpr (kDense) {
      in = in && flag[r] != 0u;
      val[r] = value_base + (uint32_t)(begin + li);
    }
    in_mask |= in ? 1u << r : 0u;
  }
  if (direct) {   // uniform
    uint32_t all;
    digit_base = direct_digit_base(hist, chunk, chunks, s_tmp, &all);
    if (kDense && chunk == 0 && threadIdx.x == 0) *taken_out = all;
  }
  __syncthreads();
  uint32_t pos[kWaveRounds];
  uint32_t dst[kPay ? kOutRounds : 1];
  const uint32_t taken = rank_and_write<kPay>(key, val, in_mask, digit_base, shift, dmask, s_key, s_val, s_wc, s_gbase,
                                              s_tmp, s_taken, kout, vout, pos, dst);
  if constexpr (kPay) {
    uint2* s_pay = reinterpret_cast<uint2*>(s_kv);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kWaveRounds; ++r)
      if ((in_mask >> r) & 1u) s_pay[pos[r]] = pay[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kOutRounds; ++r) {
      const uint32_t i = (uint32_t)r * B + threadIdx.x;
      if (i < taken) pout[dst[r]] = s_pay[i];
    }
  }
}

// ---- key emission in depth order -----------------------------------------
// Workgroup c produces the key slots [c K, (c+1) K) of one chunk of the tile
// sort (K = kSortChunk), twice: k_emit_count counts the digits of the sort's
// first pass over them, and after the scan of those counts k_emit_scatter
// produces them again and performs that first pass, so the keys in slot
// order are never stored.  Its wavefronts take the depth-sorted visible
// pairs from firsts[c], the pair owning slot c K, onwards, 64 consecutive
// pairs at a time, until a group starts past the chunk; a pair that
// straddles a chunk boundary is produced in part by both workgroups.  Within
// a group, lane l produces slot S + l in each round.  The pair owning a slot is found
// without searching: each pair whose first slot falls in the round marks that
// slot, and the marks up to a slot (one ballot and a bit count per lane, added
// to those of the rounds before) count the pairs that started by then.  The
// slot's tile within the pair's rectangle comes from a float-reciprocal
// quotient corrected to the exact integer one.

// One lane's pair of a group of 64 depth-sorted visible pairs: first and
// end key slot, (view, Gaussian) index and tile rectangle as two words
// (x0 | y0 << 16, x1 | y1 << 16); past the last pair, off is 0xffffffff and
// the rest zero.
struct PairIn {
  uint32_t off, end, vi;
  uint2 r;
};

__device__ __forceinline__ PairIn load_pair(const uint32_t* koff, const uint32_t* sorted_vis, const uint2* sorted_rect,
                                            uint32_t k, uint32_t nvis, uint32_t all_keys) {
  PairIn p{0xffffffffu, 0u, 0u, make_uint2(0u, 0u)};
  if (k < nvis) {
    p.off = koff[k];
    p.end = k + 1 < nvis ? koff[k + 1] : all_keys;
    p.vi = sorted_vis[k];
    p.r = sorted_rect[k];
  }
  return p;
}

// Per-wavefront staging of the walk: the current group of 64 pairs.
struct WalkLds {
  // first key slot, (view, Gaussian) index, first key, width | the view's
  // tiles per row << 16 (neither exceeds 2048)
  uint4 pair[NW][64];
  uint32_t mark[NW][64];
};

// The walk over chunk blockIdx.x of the key slots, [S0, S1): every slot is
// produced once, by one lane, which calls emit(slot, key, value).  s_view
// holds each view's (first tile relative to the call's first tile, tiles
// per row) and must be visible to the workgroup on entry.
template <class Emit>
__device__ __forceinline__ void emit_walk(WalkLds& L, const uint32_t* sorted_vis, const uint32_t* koff,
                                          const uint32_t* firsts, uint32_t nvis, uint32_t all_keys,
                                          const uint2* sorted_rect, const int2* s_view, uint32_t ng, uint32_t chunk, uint64_t S0,
                                          uint32_t S1, Emit emit) {
  uint4 (&s_pair)[NW][64] = L.pair;
  uint32_t (&s_mark)[NW][64] = L.mark;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const float inv_ng = 1.f / (float)ng;
  // the wavefront takes every NW-th group of 64 pairs; each group's loads go
  // out together, and before the group in hand is worked through, so that
  // they are in flight meanwhile
  uint32_t g = firsts[chunk] + (uint32_t)w * 64u;
  PairIn nxt = load_pair(koff, sorted_vis, sorted_rect, g + (uint32_t)lane, nvis, all_keys);
  for (; g < nvis; g += NW * 64u) {
    const PairIn cur = nxt;
    if ((uint32_t)__builtin_amdgcn_readfirstlane((int)cur.off) >= S1) break;   // the group starts past the chunk
    const bool valid = g + (uint32_t)lane < nvis;
    const uint32_t off = cur.off, vi = cur.vi;
    // view = vi / n_gauss: a float estimate (off by at most one, as the
    // quotient is below 2^8) corrected to the exact integer quotient (lanes
    // past the last pair stage zeros, which no slot refers to)
    uint32_t v = (uint32_t)((float)vi * inv_ng);
    const uint64_t lv = (uint64_t)v * ng;
    if (lv > vi) v -= 1u;
    else if (lv + ng <= vi) v += 1u;
    const int2 vw = s_view[v];
    const uint32_t rx = cur.r.x & 0xffffu, ry = cur.r.x >> 16, width = (cur.r.y & 0xffffu) - rx + 1u;
    s_pair[w][lane] = make_uint4(off, vi, (uint32_t)(vw.x + (int32_t)(ry * (uint32_t)vw.y + rx)),
                                 width | ((uint32_t)vw.y << 16));
    uint32_t stop = cur.end;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) stop = max(stop, (uint32_t)__shfl_xor((int)stop, d, 64));
    stop = min(stop, S1);
    // every use of this group's loads is above, so the next group's loads
    // stay in flight while the group is worked through
    __builtin_amdgcn_sched_barrier(0);
    nxt = load_pair(koff, sorted_vis, sorted_rect, g + NW * 64u + (uint32_t)lane, nvis, all_keys);
    __builtin_amdgcn_wave_barrier();
    const uint32_t start = max(s_pair[w][0].x, (uint32_t)S0);
    // the last pair of the group that began before `start` (-1: none)
    int carry = (int)__popcll(__ballot(valid && off < start)) - 1;
    for (uint32_t S = start; S < stop; S += 64) {
      s_mark[w][lane] = 0u;
      __builtin_amdgcn_wave_barrier();
      if (valid && off >= S && off - S < 64u) s_mark[w][off - S] = 1u;
      __builtin_amdgcn_wave_barrier();
      // every pair has a key, so starts are distinct: the pairs that start at
      // or before a slot of this round are counted by its lane's bit prefix
      const uint32_t mark = s_mark[w][lane];
      const uint64_t starts = __ballot(mark != 0u);
      const int own = carry + (int)(__builtin_amdgcn_mbcnt_hi((uint32_t)(starts >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)starts, mark)));
      carry += (int)__popcll(starts);
      __builtin_amdgcn_wave_barrier();
      const uint32_t slot = S + (uint32_t)lane;
      if (slot < stop) {
        const uint4 pr = s_pair[w][own];
        const uint32_t m = slot - pr.x, width = pr.w & 0xffffu;
        uint32_t q = (uint32_t)((float)m * __builtin_amdgcn_rcpf((float)width));
        int32_t rem = (int32_t)(m - q * width);
        if (rem < 0) {
          q -= 1u;
          rem += (int32_t)width;
        } else if (rem >= (int32_t)width) {
          q += 1u;
          rem -= (int32_t)width;
        }
        emit(slot, pr.z + q * (pr.w >> 16) + (uint32_t)rem, pr.y);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Digit counts of the tile sort's first pass for every chunk, in the layout
// k_radix_hist writes, without producing the keys: the keys a pair has in one
// tile row of its rectangle are consecutive integers.  Each lane takes one
// pair of the chunk (clipped to the chunk's slots) row by row.
// kMsd (digits key >> low_bits): a row's keys lie in one digit, or in a few
// consecutive ones, each counted with one LDS add.  Otherwise (digits key &
// dmask0): a row adds one to every digit len / (dmask0 + 1) times and to a
// cyclic range of len % (dmask0 + 1) digits once; the ranges go into a
// difference array, whose prefix sums are the counts.
constexpr int kCountBlock = 256;   // (more threads than a chunk's 650 pairs can feed measured slower)
constexpr int kCountWaves = kCountBlock / 64;

template <bool kMsd>
__global__ __launch_bounds__(kCountBlock) void k_emit_count(const uint32_t* sorted_vis, const uint32_t* koff,
                                                            const uint32_t* firsts, const uint32_t* nvis_p,
                                                            const uint32_t* total_keys, const uint2* sorted_rect,
                                                            const ViewInfo* views, int32_t n_views, int64_t n_gauss,
                                                            int32_t tile_begin, uint32_t cap, int64_t nblocks,
                                                            uint32_t dmask0, int low_bits, uint32_t* hist, bool direct,
                                                            Counters* ctr, uint2* ranges, int64_t ntiles) {
  __shared__ int32_t s_diff[257];
  __shared__ uint32_t s_full;
  __shared__ uint32_t s_tmp[kCountWaves];
  __shared__ int2 s_view[kMaxViews];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  s_diff[threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    s_diff[256] = 0;
    s_full = 0u;
  }
  for (int v = threadIdx.x; v < n_views; v += kCountBlock) s_view[v] = make_int2(views[v].tile_base - tile_begin, views[v].tiles_x);
  __syncthreads();
  const uint32_t all_keys = *total_keys;
  // on the side (launches of their own would cost 4 us each): the build's key
  // count and overflow flag, and empty ranges for the tiles
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctr->key_cap = cap;
    if (all_keys > cap) {
      ctr->overflow = 1u;
      ctr->overflow_any = 1u;
    }
  }
  for (int64_t t = (int64_t)blockIdx.x * kCountBlock + threadIdx.x; t < ntiles;
       t += (int64_t)gridDim.x * kCountBlock)
    ranges[t] = make_uint2(0u, 0u);
  const uint32_t n = min(all_keys, cap);
  const uint32_t M = dmask0 + 1u;
  const int bits0 = __popc(dmask0);
  const uint64_t S0 = (uint64_t)blockIdx.x * kSortChunk;
  if (S0 < n) {
    const uint32_t S1 = (uint32_t)min((uint64_t)n, S0 + kSortChunk);
    const uint32_t nvis = *nvis_p;
    const uint32_t ng = (uint32_t)n_gauss;
    const float inv_ng = 1.f / (float)ng;
    // groups of 64 pairs as in the walk, the next group's loads issued
    // before the group in hand is counted
    uint32_t g = firsts[blockIdx.x] + (uint32_t)w * 64u;
    PairIn nxt = load_pair(koff, sorted_vis, sorted_rect, g + (uint32_t)lane, nvis, all_keys);
    for (; g < nvis; g += kCountWaves * 64u) {
      const PairIn cur = nxt;
      if ((uint32_t)__builtin_amdgcn_readfirstlane((int)cur.off) >= S1) break;   // the group starts past the chunk
      const bool valid = g + (uint32_t)lane < nvis;
      const uint32_t off = cur.off, vi = cur.vi;
      const uint32_t lo = max(off, (uint32_t)S0), hi = min(cur.end, S1);
      // everything taken from this group's loads, for every lane (lanes past
      // the last pair or outside the chunk compute values they never use)
      uint32_t v = (uint32_t)((float)vi * inv_ng);   // vi / n_gauss, corrected as in the walk
      const uint64_t lv = (uint64_t)v * ng;
      if (lv > vi) v -= 1u;
      else if (lv + ng <= vi) v += 1u;
      const int2 vw = s_view[v];
      // the rectangle's words pass through an empty asm statement here, so
      // that the compiler does not narrow the next group's rectangle load
      // right where it is issued (which would make the wavefront wait for it)
      uint32_t rw0 = cur.r.x, rw1 = cur.r.y;
      asm volatile("" : "+v"(rw0), "+v"(rw1));
      const uint32_t rx = rw0 & 0xffffu, ry = rw0 >> 16;
      const uint32_t width = (rw1 & 0xffffu) - rx + 1u;
      const uint32_t m0 = lo - off, m1 = hi - off;   // the pair's slots in the chunk, [m0, m1)
      const uint32_t q0 = m0 / width, c0 = m0 - q0 * width;
      const uint32_t q1 = (m1 - 1u) / width, c1 = (m1 - 1u) - q1 * width;
      // so the next group's loads stay in flight while this one is counted
      __builtin_amdgcn_sched_barrier(0);
      nxt = load_pair(koff, sorted_vis, sorted_rect, g + kCountWaves * 64u + (uint32_t)lane, nvis, all_keys);
      if (valid && lo < hi) {
        uint32_t full = 0;
        for (uint32_t q = q0; q <= q1; ++q) {
          const uint32_t cs = q == q0 ? c0 : 0u, ce = q == q1 ? c1 : width - 1u;
          const uint32_t a = (uint32_t)(vw.x + (int32_t)((ry + q) * (uint32_t)vw.y + rx + cs));
          uint32_t len = ce - cs + 1u;
          if constexpr (kMsd) {
            for (uint32_t at = a; len != 0u;) {
              const uint32_t d = at >> low_bits, here = min(len, ((d + 1u) << low_bits) - at);
              atomicAdd(&s_diff[d], (int32_t)here);
              at += here;
              len -= here;
            }
            continue;
          }
          full += len >> bits0;
          const uint32_t rem = len & dmask0;
          if (rem) {
            const uint32_t s = a & dmask0, e = s + rem;
            atomicAdd(&s_diff[s], 1);
            if (e < M) {
              atomicAdd(&s_diff[e], -1);
            } else if (e > M) {
              atomicAdd(&s_diff[0], 1);
              atomicAdd(&s_diff[e - M], -1);
            }
          }
        }
        if (full) atomicAdd(&s_full, full);
      }
    }
  }
  __syncthreads();
  const uint32_t d = threadIdx.x;
  if constexpr (kMsd) {
    hist[hist_at(d, blockIdx.x, nblocks, direct)] = (uint32_t)s_diff[d];
  } else {
    const int32_t x = d < M ? s_diff[d] : 0;
    uint32_t total;
    const uint32_t below = block_excl_scan<kCountWaves>((uint32_t)x, s_tmp, &total);
    hist[hist_at(d, blockIdx.x, nblocks, direct)] = d < M ? below + (uint32_t)x + s_full : 0u;
  }
}

// Buckets of the tile sort: the keys of one value of their high bits, adjacent
// after the first pass.  The second pass takes each bucket's keys in chunks of
// its own (starting at the 16-entry boundary before the bucket's first key, so
// that their bytes can be read 8 at a time): start[b] = first key, start[256] =
// all keys, chunk0[b] = chunks of the buckets before b, chunk0[256] = all chunks.
struct BucketTable {
  uint32_t start[257];
  uint32_t chunk0[257];
};

__device__ __forceinline__ uint32_t bucket_chunks(uint32_t start, uint32_t end) {
  return end > start ? (end - (start & ~15u) + kSortChunk - 1) / kSortChunk : 0u;
}

// The tile sort's first pass fused with the key emission: workgroup c walks
// its chunk's slots again, places each (key, value) at its slot in LDS, and
// then ranks and scatters them as k_radix_scatter does (digits (key >> shift)
// & dmask0, hist the counts of k_emit_count, scanned unless direct), so the
// emitted keys never go through HBM in slot order.  With kKeyBytes 1 or 0 the
// digit is the key's highest bits and the pass splits the keys into buckets,
// whose table the first workgroup writes; of each key only the bits below go
// on (1), or, when there are none, the buckets are the tiles and their ranges
// are written here (0).  Three workgroups of eight wavefronts fit a compute
// unit (45 KB of LDS; the walk's staging shares space with the ranking's
// counters).  Bound by vector instructions: 58M keys of 16 views take 287 us,
// 350 with eight ballots a key, selects of 64-bit masks and a max-scan for the
// owner of a slot.
template <int kKeyBytes>
__global__ __launch_bounds__(B) void k_emit_scatter(const uint32_t* sorted_vis, const uint32_t* koff,
                                                    const uint32_t* firsts, const uint32_t* nvis_p,
                                                    const uint32_t* total_keys, const uint2* sorted_rect,
                                                    const ViewInfo* views, int32_t n_views, int64_t n_gauss,
                                                    int32_t tile_begin, uint32_t cap, int64_t nblocks, uint32_t dmask0,
                                                    int shift, const uint32_t* hist, bool direct, uint32_t* kout,
                                                    uint32_t* vout, BucketTable* buckets, uint2* ranges) {
  __shared__ __align__(16) uint32_t s_kv[2 * kSortChunk];   // keys | values
  __shared__ int2 s_view[kMaxViews];
  __shared__ union {   // the walk's staging, then the ranking's counters
    WalkLds walk;
    struct {
      uint32_t wc[NW][256];
      uint32_t gbase[256];
      uint32_t tmp[NW];
      uint32_t taken;
    } rank;
  } u;
  uint32_t* s_key = s_kv;
  uint32_t* s_val = s_kv + kSortChunk;
  uint32_t* s_scan = s_kv;   // (free until the walk)
  const uint32_t all_keys = *total_keys;
  const uint32_t n = min(all_keys, cap);
  const uint32_t chunks = (uint32_t)(((uint64_t)n + kSortChunk - 1) / kSortChunk), chunk = blockIdx.x;
  const uint64_t S0 = (uint64_t)chunk * kSortChunk;
  if (chunk >= chunks) {
    if (kKeyBytes == 1 && n == 0 && blockIdx.x == 0)   // no keys at all
      for (int q = threadIdx.x; q < 257; q += B) buckets->start[q] = buckets->chunk0[q] = 0u;
    return;
  }
  const uint32_t S1 = (uint32_t)min((uint64_t)n, S0 + kSortChunk);
  const uint32_t cnt = S1 - (uint32_t)S0;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int v = threadIdx.x; v < n_views; v += B) s_view[v] = make_int2(views[v].tile_base - tile_begin, views[v].tiles_x);
  uint32_t digit_base = direct || threadIdx.x >= 256 ? 0u : hist[(int64_t)threadIdx.x * nblocks + chunk];
  if (direct) {   // uniform
    uint32_t all;
    digit_base = direct_digit_base(hist, chunk, chunks, s_scan, &all);
  }
  if (kKeyBytes != 4 && chunk == 0) {
    // the first chunk's digit starts are the buckets'
    const uint32_t d = threadIdx.x;
    if (d < 256) s_scan[NW + d] = digit_base;
    __syncthreads();
    const uint32_t end = d < 255 ? s_scan[NW + d + 1] : n;
    if constexpr (kKeyBytes == 0) {
      if (d < 256 && end > digit_base) ranges[d] = make_uint2(digit_base, end);
    } else {
      uint32_t all;
      const uint32_t c0 = block_excl_scan(d < 256 ? bucket_chunks(digit_base, end) : 0u, s_scan, &all);
      if (d < 256) {
        buckets->start[d] = digit_base;
        buckets->chunk0[d] = c0;
      }
      if (d == 0) {
        buckets->start[256] = n;
        buckets->chunk0[256] = all;
      }
    }
  }
  __syncthreads();
  emit_walk(u.walk, sorted_vis, koff, firsts, *nvis_p, all_keys, sorted_rect, s_view, (uint32_t)n_gauss, chunk, S0, S1,
            [&](uint32_t slot, uint32_t key, uint32_t val) {
              s_key[slot - (uint32_t)S0] = key;
              s_val[slot - (uint32_t)S0] = val;
            });
  __syncthreads();
  uint32_t key[kWaveRounds], val[kWaveRounds];
  uint32_t in_mask = 0;
  const uint32_t lane0 = (uint32_t)w * kWaveKeys + (uint32_t)lane;
#pragma unroll
  for (int r = 0; r < kWaveRounds; ++r) {
    const uint32_t li = lane0 + (uint32_t)r * 64u;
    const bool in = li < cnt;
    key[r] = in ? s_key[li] : 0u;
    val[r] = in ? s_val[li] : 0u;
    in_mask |= in ? 1u << r : 0u;
  }
#pragma unroll
  for (int q = 0; q < NW * 256 / B; ++q) (&u.rank.wc[0][0])[q * B + threadIdx.x] = 0;
  // the ranking places keys into the same LDS space
  __syncthreads();
  uint32_t pos[kWaveRounds];
  uint32_t dst[1];
  rank_and_write<false, true, kKeyBytes>(key, val, in_mask, digit_base, shift, dmask0, s_key, s_val, u.rank.wc,
                                         u.rank.gbase, u.rank.tmp, u.rank.taken, kout, vout, pos, dst, n);
}

// ---- second pass of a tile sort of 9 to 16 bits: inside the buckets ----------
// Bound by memory: per key one byte and the value are read and the value is
// written, and the ranges fall out of the digit starts, 15 bytes a key for the
// whole sort with the first pass; as a second pass over whole 32-bit keys, a
// range extraction after it, it took 32.
struct BucketChunk {
  uint32_t bucket, index, chunks;   // of the chunk; the chunk's index in its bucket; the bucket's chunks
  uint32_t row0;                    // chunks of the buckets before
  uint32_t start, end;              // the bucket's keys
  uint32_t base;                    // first entry of the chunk, a multiple of 16 (entries before start are not its)
};

// Finds chunk blockIdx.x's bucket; false past the last chunk (uniform).
__device__ __forceinline__ bool find_bucket(const BucketTable* t, uint32_t* s_bucket, BucketChunk& c) {
  const uint32_t chunks = t->chunk0[256], me = xcd_chunk(chunks);
  if (me >= chunks) return false;
  if (threadIdx.x < 256 && t->chunk0[threadIdx.x] <= me && me < t->chunk0[threadIdx.x + 1]) *s_bucket = threadIdx.x;
  __syncthreads();
  c.bucket = __builtin_amdgcn_readfirstlane(*s_bucket);
  c.row0 = t->chunk0[c.bucket];
  c.chunks = t->chunk0[c.bucket + 1] - c.row0;
  c.index = me - c.row0;
  c.start = t->start[c.bucket];
  c.end = t->start[c.bucket + 1];
  c.base = (c.start & ~15u) + c.index * (uint32_t)kSortChunk;
  return true;
}

// Digit counts of a bucket's chunks: chunk by chunk (direct), else digit by
// digit within each bucket, so that one scan over all of them gives every
// (bucket, digit, chunk) its place.
__global__ __launch_bounds__(B) void k_bucket_hist(const uint8_t* keys, const BucketTable* table, int low_bits,
                                                   uint32_t* hist, bool direct, uint32_t* rows) {
  __shared__ uint32_t h[NW][256][kHistCopies];
  __shared__ uint32_t s_bucket;
#pragma unroll
  for (int q = 0; q < NW * kHistCopies * 256 / B; ++q) (&h[0][0][0])[q * B + threadIdx.x] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *rows = table->chunk0[256] << low_bits;
  BucketChunk c;
  if (!find_bucket(table, &s_bucket, c)) return;
  constexpr uint32_t kPer = kSortChunk / B;
  static_assert(kPer == 8, "one 8-byte load per thread");
  const uint32_t at = c.base + threadIdx.x * kPer;
  const int w = threadIdx.x >> 6, copy = threadIdx.x & (kHistCopies - 1);
  if (at < c.end) {   // (the key buffers hold whole 8-byte words: their capacity is rounded up)
    const uint2 x = *reinterpret_cast<const uint2*>(keys + at);
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k)
      if (at + k >= c.start && at + k < c.end)
        atomicAdd(&h[w][((k < 4 ? x.x : x.y) >> (8 * (k & 3))) & 255u][copy], 1u);
  }
  __syncthreads();
  const uint32_t d = threadIdx.x, D = 1u << low_bits;
  if (d >= D) return;
  uint32_t t = 0;
#pragma unroll
  for (int q = 0; q < NW; ++q)
#pragma unroll
    for (int k = 0; k < kHistCopies; ++k) t += h[q][d][k];
  hist[direct ? (size_t)(c.row0 + c.index) * D + d : (size_t)c.row0 * D + (size_t)d * c.chunks + c.index] = t;
}

__global__ __launch_bounds__(B) void k_bucket_scatter(const uint8_t* keys, const uint32_t* vin, const BucketTable* table,
                                                      int low_bits, const uint32_t* hist, bool direct, uint32_t* vout,
                                                      uint2* ranges) {
  __shared__ __align__(16) uint32_t s_kv[2 * kSortChunk];
  __shared__ uint32_t s_wc[NW][256];
  __shared__ uint32_t s_gbase[256];
  __shared__ uint32_t s_tmp[NW];
  __shared__ uint32_t s_taken;
  __shared__ uint32_t s_bucket;
  BucketChunk c;
  if (!find_bucket(table, &s_bucket, c)) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t d = threadIdx.x, D = 1u << low_bits;
#pragma unroll
  for (int q = 0; q < NW * 256 / B; ++q) (&s_wc[0][0])[q * B + threadIdx.x] = 0;
  uint32_t digit_base = 0;
  if (!direct && d < D) digit_base = hist[(size_t)c.row0 * D + (size_t)d * c.chunks + c.index];
  uint32_t key[kWaveRounds], val[kWaveRounds];
  uint32_t in_mask = 0;
  const uint32_t at0 = c.base + (uint32_t)w * kWaveKeys + (uint32_t)lane;
#pragma unroll
  for (int r = 0; r < kWaveRounds; ++r) {
    // (keys and values outside the bucket are read, where the buffers hold
    // them, and not taken)
    const uint32_t at = min(at0 + (uint32_t)r * 64u, c.end - 1u);
    key[r] = __builtin_nontemporal_load(keys + at);
    val[r] = __builtin_nontemporal_load(vin + at);
  }
#pragma unroll
  for (int r = 0; r < kWaveRounds; ++r) {
    const uint32_t at = at0 + (uint32_t)r * 64u;
    in_mask |= at >= c.start && at < c.end ? 1u << r : 0u;
  }
  if (direct) {   // uniform
    uint32_t before = 0, total = 0, all;
    if (d < D) {
#pragma unroll 8
      for (uint32_t k = 0; k < c.chunks; ++k) {
        const uint32_t x = hist[(size_t)(c.row0 + k) * D + d];
        before += k < c.index ? x : 0u;
        total += x;
      }
    }
    digit_base = c.start + block_excl_scan(total, s_tmp, &all) + before;
  }
  if (c.index == 0) {   // uniform: the first chunk's digit starts are the tiles'
    if (d < D) s_gbase[d] = digit_base;
    __syncthreads();
    if (d < D) {
      const uint32_t end = d + 1u < D ? s_gbase[d + 1] : c.end;
      if (end > digit_base) ranges[(c.bucket << low_bits) + d] = make_uint2(digit_base, end);
    }
  }
  __syncthreads();
  uint32_t pos[kWaveRounds];
  uint32_t dst[1];
  rank_and_write<false, true, 0>(key, val, in_mask, digit_base, 0, D - 1u, s_kv, s_kv + kSortChunk, s_wc, s_gbase, s_tmp,
                                 s_taken, nullptr, vout, pos, dst, c.end);
}

// Per-tile [start, end) of the sorted keys; thread q looks at keys 4q..4q+3
// (one 16-byte load) and their two outer neighbours.
__global__ __launch_bounds__(256) void k_ranges(const uint32_t* keys, const uint32_t* count_p, uint32_t cap,
                                                int32_t tile_begin, uint2* ranges) {
  constexpr uint32_t kNone = 0xffffffffu;   // no tile id reaches this
  const uint32_t n = min(*count_p, cap);
  const uint32_t nq = (n + 3u) / 4u;
  const bool aligned = (reinterpret_cast<uintptr_t>(keys) & 15u) == 0;
  const uint32_t lane = threadIdx.x & 63u;
  // whole wavefronts go round the loop together (lanes past the last quad
  // hold kNone), so that each quad's outer neighbours, the last key of the
  // quad before and the first of the quad after, come from the lanes beside
  // it
  for (uint32_t qb = blockIdx.x * blockDim.x + (threadIdx.x & ~63u); qb < nq; qb += gridDim.x * blockDim.x) {
    const uint32_t qd = qb + lane;
    const bool here = qd < nq;
    const uint32_t k0 = qd * 4u;
    uint32_t t[6];
    if (here && aligned && k0 + 4u <= n) {
      typedef uint32_t U4 __attribute__((ext_vector_type(4)));
      const U4 x = __builtin_nontemporal_load(reinterpret_cast<const U4*>(keys + k0));
      t[1] = x.x, t[2] = x.y, t[3] = x.z, t[4] = x.w;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) t[1 + c] = here && k0 + c < n ? keys[k0 + c] : kNone;
    }
    // lane 0's key before its quad and lane 63's key after it, in flight
    // together with the quads
    uint32_t before = kNone, after = kNone;
    if (lane == 0u && here && k0 > 0u) before = keys[k0 - 1u];
    if (lane == 63u && here && k0 + 4u < n) after = keys[k0 + 4u];
    t[0] = (uint32_t)__shfl_up((int)t[4], 1, 64);
    t[5] = (uint32_t)__shfl_down((int)t[1], 1, 64);
    if (lane == 0u) t[0] = before;
    if (lane == 63u) t[5] = after;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t k = k0 + c;
      if (here && k < n) {
        if (t[c] != t[c + 1]) ranges[tile_begin + t[c + 1]].x = k;
        if (t[c + 2] != t[c + 1]) ranges[tile_begin + t[c + 1]].y = k + 1u;
      }
    }
  }
}

// ---- longest-first tile order (persistent compositing, schedule 3) ----------
// Tiles are bucketed by the bit length of their list length (0 for an empty
// list), longer buckets first; within a bucket a workgroup's tiles keep
// their row-major neighbourhood.  Only the order in which tiles are handed
// out depends on it, never a result.
constexpr int kOrderBuckets = 33;

__device__ __forceinline__ uint32_t list_bucket(uint2 r) {
  const uint32_t n = r.y > r.x ? r.y - r.x : 0u;
  return 32u - (uint32_t)__clz(n);
}

__global__ __launch_bounds__(256) void k_order_hist(const uint2* ranges, uint32_t ntiles, uint32_t* bkt) {
  __shared__ uint32_t h[kOrderBuckets];
  if (threadIdx.x < kOrderBuckets) h[threadIdx.x] = 0u;
  __syncthreads();
  const uint32_t t = blockIdx.x * 256u + threadIdx.x;
  if (t < ntiles) atomicAdd(&h[list_bucket(ranges[t])], 1u);
  __syncthreads();
  if (threadIdx.x < kOrderBuckets && h[threadIdx.x] != 0u) atomicAdd(&bkt[threadIdx.x], h[threadIdx.x]);
}

// bkt[0..32]: tiles per bucket (complete); bkt[33..65]: cursors, zero at start
__global__ __launch_bounds__(256) void k_order_scatter(const uint2* ranges, uint32_t ntiles, uint32_t* bkt,
                                                       uint32_t* order) {
  __shared__ uint32_t h[kOrderBuckets];
  __shared__ uint32_t base[kOrderBuckets];
  if (threadIdx.x < kOrderBuckets) h[threadIdx.x] = 0u;
  __syncthreads();
  const uint32_t t = blockIdx.x * 256u + threadIdx.x;
  uint32_t b = 0, r = 0;
  if (t < ntiles) {
    b = list_bucket(ranges[t]);
    r = atomicAdd(&h[b], 1u);
  }
  __syncthreads();
  if (threadIdx.x < kOrderBuckets && h[threadIdx.x] != 0u) {
    const uint32_t me = threadIdx.x;
    uint32_t start = 0;
    for (uint32_t q = me + 1; q < (uint32_t)kOrderBuckets; ++q) start += bkt[q];
    base[me] = start + atomicAdd(&bkt[kOrderBuckets + me], h[me]);
  }
  __syncthreads();
  if (t < ntiles) order[base[b] + r] = t;
}

// ---- tile lists of small models ----------------------------------------------
// The sort's launches take 4 to 15 us each however little they hold: 56 us for a
// thousand Gaussians in one small view.  Where every pair can be compared
// with every other of its view and every tile with every pair, three launches
// build the same lists: k_small_rank gives each visible pair its place in its
// view's depth order by counting the pairs before it, k_small_count counts for
// each tile the pairs whose rectangle covers it, and k_small_fill writes them
// in order behind those of the tiles before.
constexpr uint32_t kInvisible = 0xffffffffu;   // above the bits of every depth

// A workgroup ranks 64 pairs of a view, its kRankWaves wavefronts counting an
// equal part of the view's pairs each (one compare and one add of the carry
// per pair): 8 cycles per 64 compares, so a view of 8192 takes 16 wavefronts
// 2 us of each SIMD, where four would leave half of the chip idle for 8 us.
// Ties go by index.
constexpr int kRankWaves = 16;

__global__ __launch_bounds__(64 * kRankWaves) void k_small_rank(const uint32_t* depth, const uint32_t* count, const uint2* rect,
                                                  uint32_t n, uint32_t pair0, uint32_t* sorted_vis, uint2* sorted_rect,
                                                  uint32_t* view_count) {
  __shared__ uint32_t s_key[kRankWaves][64];
  __shared__ uint32_t s_rank[kRankWaves][64];
  __shared__ uint32_t s_valid[kRankWaves];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const size_t v0 = (size_t)blockIdx.y * n;   // the view's first pair
  const uint32_t i = blockIdx.x * 64u + (uint32_t)lane;
  const bool mine = i < n && count[v0 + i] != 0u;
  const uint32_t key = mine ? depth[v0 + i] : kInvisible;
  const uint32_t part = ((n + kRankWaves - 1) / kRankWaves + 63u) & ~63u;
  const uint32_t j0 = (uint32_t)w * part, j1 = min(n, j0 + part);
  uint32_t rank = 0, valid = 0;
  uint32_t nk = kInvisible;
  if (j0 + (uint32_t)lane < j1 && count[v0 + j0 + lane] != 0u) nk = depth[v0 + j0 + lane];
  for (uint32_t j = j0; j < j1; j += 64u) {
    const uint32_t kj = nk;
    nk = kInvisible;
    const uint32_t jn = j + 64u + (uint32_t)lane;   // the next 64, in flight meanwhile
    if (jn < j1 && count[v0 + jn] != 0u) nk = depth[v0 + jn];
    valid += (uint32_t)__popcll(__ballot(kj != kInvisible));
    s_key[w][lane] = kj;
    __builtin_amdgcn_wave_barrier();
    if (j + 64u <= blockIdx.x * 64u) {   // uniform: all before this workgroup's pairs
#pragma unroll
      for (int q = 0; q < 64; ++q) rank += s_key[w][q] <= key ? 1u : 0u;
    } else if (j >= blockIdx.x * 64u + 64u) {
#pragma unroll
      for (int q = 0; q < 64; ++q) rank += s_key[w][q] < key ? 1u : 0u;
    } else {
      for (int q = 0; q < 64; ++q) {
        const uint32_t x = s_key[w][q];
        rank += x < key || (x == key && j + (uint32_t)q < i) ? 1u : 0u;
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  s_rank[w][lane] = rank;
  if (lane == 0) s_valid[w] = valid;
  __syncthreads();
  if (w != 0) return;
  rank = 0;
  valid = 0;
#pragma unroll
  for (int q = 0; q < kRankWaves; ++q) {
    rank += s_rank[q][lane];
    valid += s_valid[q];
  }
  if (blockIdx.x == 0 && lane == 0) view_count[blockIdx.y] = valid;
  if (mine) {
    sorted_vis[v0 + rank] = pair0 + (uint32_t)v0 + i;
    sorted_rect[v0 + rank] = rect[v0 + i];
  }
}

// The part of a tile's pairs that wavefront w looks at, in depth order.
struct SmallTile {
  uint32_t tx, ty;
  size_t first;        // the view's first pair
  uint32_t k0, k1;     // the wavefront's pairs of the view
  __device__ __forceinline__ SmallTile(const ViewInfo* views, const int32_t* tile_view, int32_t tile, int32_t v0,
                                       uint32_t n, const uint32_t* view_count, int w) {
    const int32_t v = tile_view[tile];
    const ViewInfo view = views[v];
    const uint32_t local = (uint32_t)(tile - view.tile_base);
    ty = local / (uint32_t)view.tiles_x;
    tx = local - ty * (uint32_t)view.tiles_x;
    first = (size_t)(v - v0) * n;
    const uint32_t nvis = view_count[v - v0], quarter = ((nvis + NW - 1) / NW + 63u) & ~63u;
    k0 = min(nvis, (uint32_t)w * quarter);
    k1 = min(nvis, k0 + quarter);
  }
  __device__ __forceinline__ bool covers(const uint2* sorted_rect, uint32_t k) const {
    if (k >= k1) return false;
    const uint2 r = sorted_rect[first + k];
    return tx >= (r.x & 0xffffu) && ty >= (r.x >> 16) && tx <= (r.y & 0xffffu) && ty <= (r.y >> 16);
  }
};

// tile_count[t][w]: pairs of tile t among wavefront w's.
__global__ __launch_bounds__(B) void k_small_count(const ViewInfo* views, const int32_t* tile_view, int32_t tile_begin,
                                                   int32_t v0, uint32_t n, const uint32_t* view_count,
                                                   const uint2* sorted_rect, uint32_t* tile_count) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const SmallTile t(views, tile_view, tile_begin + (int32_t)blockIdx.x, v0, n, view_count, w);
  uint32_t c = 0;
#pragma unroll 4
  for (uint32_t k = t.k0; k < t.k1; k += 64u) c += (uint32_t)__popcll(__ballot(t.covers(sorted_rect, k + lane)));
  if (lane == 0) tile_count[blockIdx.x * NW + w] = c;
}

__global__ __launch_bounds__(B) void k_small_fill(const ViewInfo* views, const int32_t* tile_view, int32_t tile_begin,
                                                  int32_t v0, int32_t nv, uint32_t n, const uint32_t* view_count,
                                                  const uint32_t* sorted_vis, const uint2* sorted_rect,
                                                  const uint32_t* tile_count, uint32_t cap, uint32_t* vals,
                                                  uint2* ranges, Counters* ctr) {
  __shared__ uint32_t s_tmp[NW];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t before = 0;
  for (uint32_t q = threadIdx.x; q < blockIdx.x; q += B) {
#pragma unroll
    for (int k = 0; k < NW / 4; ++k) {
      const uint4 c = reinterpret_cast<const uint4*>(tile_count)[q * (NW / 4) + k];
      before += (c.x + c.y) + (c.z + c.w);
    }
  }
  static_assert(NW % 4 == 0, "a tile's counts are read 16 bytes at a time");
  uint32_t base;
  block_excl_scan(before, s_tmp, &base);
  uint32_t cnt[NW], at = base, all = 0;
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    cnt[q] = tile_count[blockIdx.x * NW + q];
    at += q < w ? cnt[q] : 0u;
    all += cnt[q];
  }
  if (threadIdx.x == 0)
    ranges[blockIdx.x] = all ? make_uint2(min(base, cap), min(base + all, cap)) : make_uint2(0u, 0u);
  const SmallTile t(views, tile_view, tile_begin + (int32_t)blockIdx.x, v0, n, view_count, w);
#pragma unroll 4
  for (uint32_t k = t.k0; k < t.k1; k += 64u) {
    const bool in = t.covers(sorted_rect, k + lane);
    const uint64_t m = __ballot(in);
    const uint32_t d = at + (uint32_t)__popcll(m & lt_mask);
    if (in && d < cap) vals[d] = sorted_vis[t.first + k + lane];
    at += (uint32_t)__popcll(m);
  }
  if (blockIdx.x == gridDim.x - 1 && w == 0) {   // the totals
    uint32_t nvis = 0;
    for (int32_t v = lane; v < nv; v += 64) nvis += view_count[v];
    nvis = wave_incl_scan(nvis);
    if (lane == 63) {
      const uint32_t keys = base + all;
      ctr->nvis = nvis;
      ctr->keys = keys;
      ctr->key_cap = cap;
      if (keys > cap) {
        ctr->overflow = 1u;
        ctr->overflow_any = 1u;
      }
    }
  }
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t count, hipStream_t st) {
  if (count > 0) hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)cdiv(count, 256)), dim3(256), 0, st, p, value, count);
  return hipGetLastError();
}

static hipError_t scan_src(ScanSrc src, uint32_t* out, int64_t max_count, const uint32_t* dcount, uint32_t* partial,
                           int64_t partial_len, uint32_t* total, hipStream_t st, uint32_t* firsts = nullptr,
                           uint32_t firsts_len = 0) {
  const int64_t nb = cdiv(max_count, kSortChunk);
  if (nb + 1 > partial_len) return hipErrorInvalidValue;
  // up to kDirectScanBlocks chunks, each down-sweep block adds up the chunk
  // sums before it itself (at most that many reads per block) instead of a
  // single-workgroup scan of them in a launch of its own
  constexpr int64_t kDirectScanBlocks = 4096;
  const bool direct = nb > 0 && nb <= kDirectScanBlocks;
  if (nb > 0) {
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(B), 0, st, src, max_count, dcount, partial);
  }
  if (!direct) hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, st, max_count, dcount, partial, total);
  if (nb > 0) {
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(B), 0, st, src, out, max_count, dcount, partial, firsts,
                       firsts_len, direct, total);
  }
  return hipGetLastError();
}

hipError_t launch_scan(const uint32_t* in, uint32_t* out, int64_t max_count, const uint32_t* dcount, uint32_t* partial,
                       int64_t partial_len, uint32_t* total, hipStream_t st) {
  return scan_src(ScanSrc{in, nullptr, 0}, out, max_count, dcount, partial, partial_len, total, st);
}

// Dense source of a sort's first pass: max_count keys key[k] with payload
// pay[k], taken only where valid[k] != 0, with value value_base + k; the
// number taken is written to *taken, which the later passes read as their
// count.
struct DenseSrc {
  const uint32_t* key;
  const uint32_t* valid;
  const uint2* pay;
  uint32_t value_base;
  uint32_t* taken;
};

// Sorts (key, value) pairs on key bits [0, bits) in ping-pong buffers, the
// first pass on the low first_bits bits and every later one on the next 8;
// returns through *in_b whether the result landed in the second buffer.  With `dense`,
// the first pass reads the dense source instead of (ka, va, pa) and writes
// the taken keys to (ka, va, pa), and the later passes sort *dense->taken of
// them (dcount must then be dense->taken).  With first_done, the caller has
// already performed the first pass into (kb, vb, pb).
static hipError_t radix_sort(const Plan& pl, void* ws, uint32_t* ka, uint32_t* va, uint32_t* kb, uint32_t* vb,
                             uint2* pa, uint2* pb, int64_t max_count, const uint32_t* dcount, int bits, bool* in_b,
                             hipStream_t st, const DenseSrc* dense = nullptr, bool first_done = false,
                             int first_bits = 8) {
  const int64_t nb = cdiv(max_count, kSortChunk);
  uint32_t* hist = seg<uint32_t>(ws, pl.ws.hist);
  uint32_t* partial = seg<uint32_t>(ws, pl.ws.partial);
  if (nb > pl.ws.hist_blocks) return hipErrorInvalidValue;
  if (dense && (!pa || dcount != dense->taken)) return hipErrorInvalidValue;
  bool cur_b = false;   // which buffer holds the data (before a dense first pass: neither)
  for (int shift = 0; shift < bits; shift += (shift == 0 ? first_bits : 8)) {
    const uint32_t dmask = (1u << (shift == 0 ? first_bits : 8)) - 1u;
    const bool from_dense = dense && shift == 0;
    const bool out_b = from_dense ? false : !cur_b;
    const uint32_t* ki = from_dense ? dense->key : cur_b ? kb : ka;
    const uint32_t* vi = from_dense ? nullptr : cur_b ? vb : va;
    const uint2* pi = from_dense ? dense->pay : cur_b ? pb : pa;
    uint32_t* ko = out_b ? kb : ka;
    uint32_t* vo = out_b ? vb : va;
    uint2* po = out_b ? pb : pa;
    if (first_done && shift == 0) {
      cur_b = true;
      continue;
    }
    if (nb > 0) {
      const uint32_t* dc = from_dense ? nullptr : dcount;
      const bool direct = nb <= kDirectChunks;
      hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)nb), dim3(B), 0, st, ki, from_dense ? dense->valid : nullptr,
                         max_count, dc, shift, dmask, nb, hist, direct);
      // a dense pass's digit counts total the taken keys
      hipError_t e = direct ? hipSuccess
                            : scan_src(ScanSrc{hist, nullptr, 0}, hist, 256 * nb, nullptr, partial, pl.ws.partial_len,
                                       from_dense ? dense->taken : nullptr, st);
      if (e != hipSuccess) return e;
      if (from_dense)
        hipLaunchKernelGGL((k_radix_scatter<true, true>), dim3(xcd_grid(nb)), dim3(B), 0, st, ki, vi, ko, vo, pi, po,
                           max_count, dc, shift, dmask, nb, hist, direct, dense->valid, dense->value_base, dense->taken);
      else if (pa)
        hipLaunchKernelGGL((k_radix_scatter<true, false>), dim3(xcd_grid(nb)), dim3(B), 0, st, ki, vi, ko, vo, pi,
                           po, max_count, dc, shift, dmask, nb, hist, direct, nullptr, 0u, nullptr);
      else
        hipLaunchKernelGGL((k_radix_scatter<false, false>), dim3(xcd_grid(nb)), dim3(B), 0, st, ki, vi, ko, vo, pi,
                           po, max_count, dc, shift, dmask, nb, hist, direct, nullptr, 0u, nullptr);
    } else if (from_dense) {
      hipError_t e = launch_fill_u32(dense->taken, 0u, 1, st);
      if (e != hipSuccess) return e;
    }
    cur_b = out_b;
  }
  *in_b = cur_b;
  return hipGetLastError();
}

hipError_t launch_sort_pairs(const Plan& pl, void* ws, uint32_t* ka, uint32_t* va, uint32_t* kb, uint32_t* vb,
                             int64_t count, int bits, bool* in_b, hipStream_t st) {
  return radix_sort(pl, ws, ka, va, kb, vb, nullptr, nullptr, count, nullptr, bits, in_b, st);
}

// Longest-first order of the call's tiles for the persistent compositing kernels.
static hipError_t order_tiles(const Plan& pl, void* ws, int32_t tile_begin, int64_t ntiles, hipStream_t st) {
  if (pl.schedule == 3 && ntiles > 0) {
    const uint2* ranges = seg<uint2>(ws, pl.ws.ranges) + tile_begin;
    uint32_t* bkt = seg<uint32_t>(ws, pl.ws.obucket);
    const hipError_t e = launch_fill_u32(bkt, 0u, 2 * kOrderBuckets, st);
    if (e != hipSuccess) return e;
    const unsigned ob = (unsigned)cdiv(ntiles, 256);
    hipLaunchKernelGGL(k_order_hist, dim3(ob), dim3(256), 0, st, ranges, (uint32_t)ntiles, bkt);
    hipLaunchKernelGGL(k_order_scatter, dim3(ob), dim3(256), 0, st, ranges, (uint32_t)ntiles, bkt,
                       seg<uint32_t>(ws, pl.ws.order));
  }
  return hipGetLastError();
}

// Whether the call's lists are built by comparing everything with everything:
// where that is the faster route, and the tile counts fit the scratch that is
// free then (a few words per tile, short only for a tiny key capacity).
static bool small_lists(const Plan& pl, int nv, int64_t ntiles) {
  return compares_all(pl.n, nv, ntiles) && 4 * NW * ntiles <= (int64_t)(pl.ws.vals_a - pl.ws.vrect_b);
}

hipError_t launch_tile_lists(const Plan& pl, int v0, int nv, void* ws, hipStream_t st) {
  Counters* ctr = seg<Counters>(ws, pl.ws.counters);
  const int64_t N = pl.n;
  const int64_t base = (int64_t)v0 * N, len = (int64_t)nv * N;
  uint32_t* count = seg<uint32_t>(ws, pl.ws.count);
  uint32_t* depth = seg<uint32_t>(ws, pl.ws.depth);
  uint32_t* vis_a = seg<uint32_t>(ws, pl.ws.vis_a);
  uint32_t* vis_b = seg<uint32_t>(ws, pl.ws.vis_b);
  uint32_t* vkey_a = seg<uint32_t>(ws, pl.ws.vkey_a);
  uint32_t* vkey_b = seg<uint32_t>(ws, pl.ws.vkey_b);
  uint32_t* koff = seg<uint32_t>(ws, pl.ws.koff);
  uint2* vrect_a = seg<uint2>(ws, pl.ws.vrect_a);
  uint2* vrect_b = seg<uint2>(ws, pl.ws.vrect_b);
  uint32_t* partial = seg<uint32_t>(ws, pl.ws.partial);
  uint32_t* keys_a = seg<uint32_t>(ws, pl.ws.keys_a);
  uint32_t* keys_b = seg<uint32_t>(ws, pl.ws.keys_b);
  uint32_t* vals_a = seg<uint32_t>(ws, pl.ws.vals_a);
  uint32_t* vals_b = seg<uint32_t>(ws, pl.ws.vals_b);
  uint2* ranges = seg<uint2>(ws, pl.ws.ranges);
  const uint32_t cap = (uint32_t)pl.cap;
  hipError_t e;
  if (len == 0) return hipSuccess;
  const int32_t tile_begin = pl.views[v0].tile_base;
  const int32_t tile_end = (v0 + nv < pl.n_views) ? pl.views[v0 + nv].tile_base : pl.total_tiles;
  const int64_t ntiles = tile_end - tile_begin;
  if (small_lists(pl, nv, ntiles)) {
    uint32_t* view_count = seg<uint32_t>(ws, pl.ws.hist);
    uint32_t* tile_count = reinterpret_cast<uint32_t*>(vrect_b);   // up to the values, all of it free here
    uint32_t* vals = sorted_values_in_b(pl, v0, nv) ? vals_b : vals_a;
    hipLaunchKernelGGL(k_small_rank, dim3((unsigned)cdiv(N, 64), (unsigned)nv), dim3(64 * kRankWaves), 0, st, depth + base,
                       count + base, seg<uint2>(ws, pl.ws.rect) + base, (uint32_t)N, (uint32_t)base, vis_a, vrect_a,
                       view_count);
    hipLaunchKernelGGL(k_small_count, dim3((unsigned)ntiles), dim3(B), 0, st, pl.d_views, pl.d_tile_view, tile_begin,
                       v0, (uint32_t)N, view_count, vrect_a, tile_count);
    hipLaunchKernelGGL(k_small_fill, dim3((unsigned)ntiles), dim3(B), 0, st, pl.d_views, pl.d_tile_view, tile_begin, v0,
                       nv, (uint32_t)N, view_count, vis_a, vrect_a, tile_count, cap, vals, ranges + tile_begin, ctr);
    return order_tiles(pl, ws, tile_begin, ntiles, st);
  }
  // 1-2. stable depth sort of the visible pairs (ties keep (view, Gaussian)
  // order); its first pass reads the dense (view, Gaussian) arrays and takes
  // the visible pairs only, so it also compacts them and counts them into
  // ctr->nvis
  bool in_b = false;
  const DenseSrc dense{depth + base, count + base, seg<uint2>(ws, pl.ws.rect) + base, (uint32_t)base, &ctr->nvis};
  e = radix_sort(pl, ws, vkey_a, vis_a, vkey_b, vis_b, vrect_a, vrect_b, len, &ctr->nvis, 32, &in_b, st, &dense);
  if (e != hipSuccess) return e;
  const uint32_t* sorted_vis = in_b ? vis_b : vis_a;
  const uint2* sorted_rect = in_b ? vrect_b : vrect_a;
  // 3. key offsets in depth order, and the pair owning the first slot of
  // each chunk of the tile sort
  const int64_t key_chunks = cdiv(pl.cap, kSortChunk);
  if (key_chunks > pl.ws.hist_blocks) return hipErrorInvalidValue;
  uint32_t* firsts = seg<uint32_t>(ws, pl.ws.firsts);
  e = scan_src(ScanSrc{reinterpret_cast<const uint32_t*>(sorted_rect), nullptr, 3}, koff, len, &ctr->nvis, partial,
               pl.ws.partial_len, &ctr->keys, st, firsts, (uint32_t)key_chunks);
  if (e != hipSuccess) return e;
  // 4. digit counts of the tile sort's first pass over the (tile, value)
  // pairs in depth order, one sort chunk per workgroup, and their scan
  // tile bits of the call: up to 16 are sorted from the highest bits down, in
  // one pass or two of half the bits each; more, from the lowest up in passes
  // of 8 with the remainder first
  int bits = 0;
  while ((1ll << bits) < ntiles) ++bits;
  if (bits == 0) bits = 1;
  const bool msd = bits <= 16;
  const int low_bits = !msd || bits <= 8 ? 0 : bits / 2;
  const int first_bits = msd ? bits - low_bits : bits - 8 * ((bits - 1) / 8);
  uint32_t* hist = seg<uint32_t>(ws, pl.ws.hist);
  const uint32_t dmask0 = (1u << first_bits) - 1u;
  const bool direct = key_chunks <= kDirectChunks;
  hipLaunchKernelGGL(msd ? k_emit_count<true> : k_emit_count<false>, dim3((unsigned)key_chunks), dim3(kCountBlock), 0,
                     st, sorted_vis, koff, firsts, &ctr->nvis, &ctr->keys, sorted_rect, pl.d_views, pl.n_views, N,
                     tile_begin, cap, key_chunks, dmask0, low_bits, hist, direct, ctr, ranges + tile_begin, ntiles);
  if (!direct) {
    e = scan_src(ScanSrc{hist, nullptr, 0}, hist, 256 * key_chunks, nullptr, partial, pl.ws.partial_len, nullptr, st);
    if (e != hipSuccess) return e;
  }
  // 5. stable sort by tile (relative to the first tile of the call): its
  // first pass fused with the emission, into the second buffers (empty tiles'
  // ranges were written with the digit counts)
  BucketTable* buckets = seg<BucketTable>(ws, pl.ws.buckets);
  auto emit = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)key_chunks), dim3(B), 0, st, sorted_vis, koff, firsts, &ctr->nvis,
                       &ctr->keys, sorted_rect, pl.d_views, pl.n_views, N, tile_begin, cap, key_chunks, dmask0,
                       low_bits, hist, direct, keys_b, vals_b, buckets, ranges + tile_begin);
  };
  if (msd && low_bits == 0) {
    emit(k_emit_scatter<0>);
  } else if (msd) {
    emit(k_emit_scatter<1>);
    const uint8_t* low = reinterpret_cast<const uint8_t*>(keys_b);
    // every bucket's last chunk may be a partial one
    const int64_t chunks = key_chunks + cdiv(ntiles, 1ll << low_bits);
    // (in a workspace word that nothing else holds now)
    uint32_t* rows = firsts;
    hipLaunchKernelGGL(k_bucket_hist, dim3(xcd_grid(chunks)), dim3(B), 0, st, low, buckets, low_bits, hist, direct, rows);
    if (!direct) {
      e = scan_src(ScanSrc{hist, nullptr, 0}, hist, chunks << low_bits, rows, partial, pl.ws.partial_len, nullptr, st);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_bucket_scatter, dim3(xcd_grid(chunks)), dim3(B), 0, st, low, vals_b, buckets, low_bits, hist,
                       direct, vals_a, ranges + tile_begin);
  } else {
    emit(k_emit_scatter<4>);
    e = radix_sort(pl, ws, keys_a, vals_a, keys_b, vals_b, nullptr, nullptr, pl.cap, &ctr->keys, bits, &in_b, st,
                   nullptr, true, first_bits);
    if (e != hipSuccess) return e;
    // 6. ranges
    const uint32_t* sk = in_b ? keys_b : keys_a;
    // one quad of keys per thread (the loop in the kernel covers any size):
    // every wavefront's loads are in flight at once instead of one quad after
    // another per thread
    const int64_t rblocks = cdiv(cdiv(pl.cap, 4), 256) < 0x7fffffffll ? cdiv(cdiv(pl.cap, 4), 256) : 0x7fffffffll;
    hipLaunchKernelGGL(k_ranges, dim3((unsigned)rblocks), dim3(256), 0, st, sk, &ctr->keys, cap, tile_begin, ranges);
  }
  // 7. longest-first order of the call's tiles for the persistent compositing kernels
  return order_tiles(pl, ws, tile_begin, ntiles, st);
}

}  // namespace gs
