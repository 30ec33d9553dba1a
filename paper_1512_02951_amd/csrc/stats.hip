// Security statistics of a protected image against its original (report
// Sec. 6.6 and 6.10, Eqs. (3)-(4), Table 14): byte histograms and uniformity,
// entropies and normalised mutual information from the joint histogram,
// block entropy (h = 8), correlation of adjacent samples, two-dimensional
// correlation, bit difference and PSNR.
//
// Four kernels, every moment an exact integer:
//  * band kernel: one wavefront per band of 8 rows x 32 blocks of a plane;
//    lanes k and k + 32 hold rows 0-3 and 4-7 of block k (8 bytes a row, and
//    the row below).  Pair products with v_dot4_u32_u8 on the words and their
//    neighbours (v_alignbyte_b32 shifts in the next word's first byte):
//    horizontal, vertical and diagonal pairs, sums, squares, the X.Y products
//    and differing bits (v_bcnt).  Pairs that leave the plane multiply a zero;
//    the directional sums of x and y are derived exactly from whole-plane sums
//    minus the border sums the band kernel also gathers.  Block entropy: per-wave
//    LDS byte counters (256 per block, four to a word, ds_add), then the product
//    of every sample's value count; H = 6 - log2(product) / 64.  Per-workgroup
//    partial sums.  It also clears the histogram for the next kernel.  Bound by
//    vector issue (about 990 instructions for a band of both images): 94 -> 60
//    us on 4096^2 RGB since the counters have no bank conflicts, each sample
//    takes 9 instead of 16 instructions, one logarithm serves both images and
//    4 waves share a SIMD (at 4 spilled registers: the next band's rows, loaded
//    ahead for straight-line code, gained nothing by themselves).
//  * joint histogram: a workgroup counts a chunk of samples in 65536 16-bit LDS
//    counters (128 KB; bins b and b + 32768 share a word) and leaves the low
//    bytes of its counts in the workspace; the few counts above 255 go to the
//    global histogram by atomics, as do counters near their limit between
//    parts of the chunk.  32-bit counters of half the bins read the images
//    twice and added every bin by an atomic of its own: 47 us on 4096^2 RGB, 13
//    of them the 8.4 M atomics (about one per L2 channel and clock); now 28, and
//    the rows kernel 13 instead of 8.  A workspace too small for the counts
//    gets all of them by atomics (a call 150 us instead of 110).
//  * rows (256 workgroups) and finalize (one workgroup): reduce the partials
//    and the histogram in fixed orders, then form the histograms, entropies,
//    NMI, chi-square and correlations in FP64.
#include "plain_tile.h"

namespace sf {
namespace {

constexpr int kBandWaves = 4;
constexpr int kBandThreads = 64 * kBandWaves;
constexpr int kBandGrid = 1024;  // the most band workgroups: one partial slot each
constexpr uint32_t kFlushBands = 256;
constexpr int kJointThreads = 1024;
constexpr uint32_t kHalfBins = 32768;
constexpr uint32_t kJointGrid = 256;  // the most joint workgroups: 64 KB of counts each
// 16-bit joint counters: a part of a workgroup's chunk adds at most 16 *
// kJointPart to a counter, which then is below kJointLeast again (spilled)
// before the next part, so none can pass 65535.
constexpr uint64_t kJointPart = 3584;
constexpr uint32_t kJointLeast = 8192;
static_assert(16 * kJointPart + kJointLeast - 1 <= 65535, "joint counters could wrap");
constexpr int kFinThreads = 256;

// Integer moments of one image gathered by the band kernel.
enum : int {
  kT1 = 0, kT2, kSh, kSv, kSd,    // sum x, sum x^2, horizontal / vertical / diagonal products
  kR0S, kR0Q, kRLS, kRLQ,         // first / last row of each plane: sum, sum of squares
  kC0S, kC0Q, kCLS, kCLQ,         // first / last column
  kTLS, kTLQ, kBRS, kBRQ,         // top-left and bottom-right samples
  kImgMoments
};
constexpr int kCrossXY = 2 * kImgMoments;      // sum x y
constexpr int kBitsDiff = kCrossXY + 1;        // differing bits
constexpr int kIntMoments = kBitsDiff + 1;
// Floating partials: per image sum H, sum H^2, min H, max H.
constexpr int kFltMoments = 8;

struct Partial {
  uint64_t m[kIntMoments];
  double f[kFltMoments];
};

struct StatsGeom {
  uint32_t H, W, C, By, Bx;
  uint32_t nbx;     // bands across a plane = ceil(Bx / 32)
  uint32_t nbands;  // C * By * nbx
  UDiv div_nbx, div_by;
};

__device__ __forceinline__ uint32_t udot4(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_udot4(a, b, c, false);
}

__device__ __forceinline__ uint32_t next_bytes(uint32_t w, uint32_t nx) {
  return __builtin_amdgcn_alignbyte(nx, w, 1);  // bytes w1 w2 w3 nx0
}

template <class T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Lane sums of one image over a band (the border sums go straight into the
// wave's record).
enum : int { kLaneMoments = kSd + 1 };
constexpr int kLaneSums = 2 * kLaneMoments + 2;  // X, Y, X.Y, differing bits
__device__ __forceinline__ constexpr int lane_sum_slot(int i) {
  return i < kLaneMoments ? i : i < 2 * kLaneMoments ? kImgMoments + i - kLaneMoments : kCrossXY + i - 2 * kLaneMoments;
}

// The lane's four rows and the row below them: words 2k, 2k + 1 of block k's
// row, and the first byte after them.
struct BandRows {
  uint32_t w[5][2];
  uint32_t nx[5];
};

// One image's moments over one band; adds into acc.  A band adds at most
// 32 * 255^2 = 2 080 800 to a lane's 32-bit sum; the kernel moves the lane
// sums into the wave's 64-bit record every kFlushBands bands (256 * 2 080 800
// < 2^32), so no image shape can wrap them.
__device__ __forceinline__ void band_image_moments(const BandRows &b, uint32_t *acc) {
  uint32_t t1 = 0, t2 = 0, sh = 0, sv = 0, sd = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t w = b.w[r][h], below = b.w[r + 1][h];
      t1 = udot4(w, 0x01010101u, t1);
      t2 = udot4(w, w, t2);
      sh = udot4(w, next_bytes(w, h ? b.nx[r] : b.w[r][1]), sh);
      sv = udot4(w, below, sv);
      sd = udot4(w, next_bytes(below, h ? b.nx[r + 1] : b.w[r + 1][1]), sd);
    }
  acc[kT1] += t1;
  acc[kT2] += t2;
  acc[kSh] += sh;
  acc[kSv] += sv;
  acc[kSd] += sd;
}

// Border sums of one image over one band, added to the wave's record by its
// first lane.  Bands on a border are few, so these cost nothing elsewhere (as
// lane sums they were 24 of the kernel's registers).  Conditions are
// wave-uniform; k_right: block of the plane's last column in this band.
__device__ __forceinline__ void band_border(const BandRows &b, int lane, bool valid, bool top, bool bottom, bool left,
                                            bool right, int k_right, uint64_t *m) {
  auto row = [&](int r, bool mine, int at) {
    uint32_t s = 0, q = 0;
    if (mine && valid) {
      s = udot4(b.w[r][1], 0x01010101u, udot4(b.w[r][0], 0x01010101u, 0u));
      q = udot4(b.w[r][1], b.w[r][1], udot4(b.w[r][0], b.w[r][0], 0u));
    }
    s = wave_sum(s);
    q = wave_sum(q);
    if (lane == 0) {
      m[at] += s;
      m[at + 1] += q;
    }
  };
  auto column = [&](int h, int shift, int k, int at, bool corner, int corner_row, int corner_half, int corner_at) {
    uint32_t s = 0, q = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t v = (b.w[r][h] >> shift) & 0xffu;
      s += v;
      q += v * v;
    }
    const uint32_t c = (b.w[corner_row][h] >> shift) & 0xffu;
    const uint32_t ts = (uint32_t)__builtin_amdgcn_readlane((int)s, k) + (uint32_t)__builtin_amdgcn_readlane((int)s, k + 32);
    const uint32_t tq = (uint32_t)__builtin_amdgcn_readlane((int)q, k) + (uint32_t)__builtin_amdgcn_readlane((int)q, k + 32);
    const uint32_t tc = (uint32_t)__builtin_amdgcn_readlane((int)c, k + 32 * corner_half);
    if (lane == 0) {
      m[at] += ts;
      m[at + 1] += tq;
      if (corner) {
        m[corner_at] += tc;
        m[corner_at + 1] += tc * tc;
      }
    }
  };
  if (top) row(0, lane < 32, kR0S);
  if (bottom) row(3, lane >= 32, kRLS);
  if (left) column(0, 0, 0, kC0S, top, 0, 0, kTLS);
  if (right) column(1, 24, k_right, kCLS, bottom, 3, 1, kBRS);
}

// Block entropy of the lane's half block (lanes k, k + 32 share block k of the
// band): counts in LDS, then the product of the counts of the lane's 32
// samples' values.  sum_i log2(c_i) over the block is log2 of the two lanes'
// products (each count <= 64, so the product is at most 2^384: no overflow in
// FP64, relative error below 64 * 2^-53).
// Counter of value v of block k: byte v % 4 of word 32 (v / 4) + k, so lane k
// only ever touches bank k, and the two lanes of a block are served in
// different halves of an LDS access: no conflicts (with a block's 64 words
// together, a quarter of the band kernel's cycles were bank conflicts).
__device__ __forceinline__ double band_block_count_product(const BandRows &b, uint32_t *cnt, int lane) {
  // zero the wave's 32 x 64 counter words
  uint4 *z = reinterpret_cast<uint4 *>(cnt);
#pragma unroll
  for (int i = 0; i < 8; ++i) z[64 * i + lane] = make_uint4(0, 0, 0, 0);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // one vector instruction each: the counter's address (the value's upper six
  // bits moved to bits 7-12, or-ed with the lane's own bank: the wave's counters
  // are 8 KB aligned), its bit position 8 (v % 4) (low five bits of `low`
  // shifted; the shifts below take no others), the increment
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  const uint32_t own = (uint32_t)(uintptr_t)(lds_u32 *)cnt + 4u * ((uint32_t)lane & 31u);
  auto at = [&](uint32_t w, int i) -> lds_u32 * {
    return (lds_u32 *)(uintptr_t)(((i == 0 ? w << 5 : w >> (8 * i - 5)) & 0x1f80u) | own);
  };
  auto bit = [&](uint32_t low, int i) -> uint32_t { return (i == 0 ? low << 3 : low >> (8 * i - 3)) & 31u; };
  // one row at a time (sched_barrier): all 32 accesses in flight at once
  // would hold twice the registers for no gain
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t w = b.w[r][h];
      uint32_t low = w & 0x03030303u;
      asm volatile("" : "+v"(low));  // masked once a word, not once a sample
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __hip_atomic_fetch_add(at(w, i), 1u << bit(low, i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // products of four counts are exact integers (<= 2^24): multiply those in
  // 32-bit integers, then the eight partial products in FP64
  double p = 1.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t q = 1u, w = b.w[r][h], low;
      asm volatile("" : "+v"(w));  // addresses made again: not 64 values kept from the counting pass
      low = w & 0x03030303u;
      asm volatile("" : "+v"(low));
#pragma unroll
      for (int i = 0; i < 4; ++i) q = __umul24(q, __builtin_amdgcn_ubfe(*at(w, i), bit(low, i), 8u));
      p *= (double)q;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  return p;
}

struct BandArgs {
  StatsGeom g;
  const uint8_t *x;
  const uint8_t *y;
  Partial *partials;  // kBandGrid slots
  float *block_entropy;  // optional: nb values for x, then nb for y
  uint32_t *clear0;      // words set to zero for the kernels that follow
  uint32_t *clear1;
  uint32_t nclear0, nclear1;
};

// A band's place, and this lane's block in it.
struct BandPlace {
  uint32_t plane, by, bandx, bx;
  bool valid;
};

__device__ __forceinline__ BandPlace band_place(const StatsGeom &g, uint32_t band, int lane) {
  BandPlace p;
  const uint32_t rest = udiv(band, g.div_nbx);
  p.bandx = band - rest * g.nbx;
  p.plane = udiv(rest, g.div_by);
  p.by = rest - p.plane * g.By;
  p.bx = p.bandx * 32u + ((uint32_t)lane & 31u);
  p.valid = p.bx < g.Bx;
  return p;
}

// Loads the lane's rows: five 8-byte words (the fifth row is the other half's
// first or the next band's) and the words after them.  img: buffer over the
// image; what lies past the plane takes an offset beyond the buffer, which
// loads zero, so that all loads are unconditional.
constexpr uint32_t kPastImage = 0xfffffff0u;
__device__ __forceinline__ void band_load(__amdgpu_buffer_rsrc_t img, const StatsGeom &g, const BandPlace &p, int lane,
                                          BandRows &b) {
  const uint32_t at = p.plane * g.H * g.W + (p.by * 8u + (lane < 32 ? 0u : 4u)) * g.W + 8u * p.bx;
  const bool below = lane < 32 || p.by + 1u < g.By, after = p.bx + 1u < g.Bx;
  const uint32_t voff = p.valid ? at : kPastImage, voff4 = p.valid && below ? at : kPastImage;
  const uint32_t noff = after ? at + 8u : kPastImage, noff4 = after && below ? at + 8u : kPastImage;
#pragma unroll
  for (int r = 0; r < 5; ++r) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(img, r < 4 ? voff : voff4, (int)(r * g.W), 0);
    b.w[r][0] = v.x;
    b.w[r][1] = v.y;
    b.nx[r] = __builtin_amdgcn_raw_buffer_load_b32(img, r < 4 ? noff : noff4, (int)(r * g.W), 0);
  }
}

__global__ __launch_bounds__(kBandThreads, 4) void stats_band_kernel(BandArgs a) {
  __shared__ __attribute__((aligned(8192))) uint32_t s_cnt[kBandWaves][32 * 64];
  __shared__ Partial s_part[kBandWaves];
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const StatsGeom &g = a.g;
  const __amdgpu_buffer_rsrc_t img_x = buffer_rsrc(a.x, g.C * g.H * g.W), img_y = buffer_rsrc(a.y, g.C * g.H * g.W);
  for (uint32_t i = blockIdx.x * kBandThreads + threadIdx.x; i < a.nclear0; i += gridDim.x * kBandThreads) a.clear0[i] = 0u;
  for (uint32_t i = blockIdx.x * kBandThreads + threadIdx.x; i < a.nclear1; i += gridDim.x * kBandThreads) a.clear1[i] = 0u;
  uint32_t acc[kLaneSums];
#pragma unroll
  for (int i = 0; i < kLaneSums; ++i) acc[i] = 0;
  if (lane == 0)
    for (int i = 0; i < kIntMoments; ++i) s_part[wave].m[i] = 0;
  // lane sums into the wave's 64-bit record, one sum at a time: interleaving
  // all of them holds every partial in registers at once
  auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kLaneSums; ++i) {
      const uint64_t v = wave_sum((uint64_t)acc[i]);
      if (lane == 0) s_part[wave].m[lane_sum_slot(i)] += v;
      acc[i] = 0;
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // block entropies: X in lanes 0-31, Y in lanes 32-63
  double esum = 0.0, esq = 0.0, emin = 1e300, emax = -1e300;
  const uint64_t nb = (uint64_t)g.C * g.By * g.Bx;
  uint32_t since_flush = 0;
  const uint32_t stride = gridDim.x * kBandWaves;
  const int k_right = (int)((g.Bx - 1u) & 31u);
  uint32_t band = blockIdx.x * kBandWaves + wave;
  BandPlace at = band_place(g, min(band, g.nbands - 1u), lane);
  BandRows rows[2];
  band_load(img_x, g, at, lane, rows[0]);
  band_load(img_y, g, at, lane, rows[1]);
  for (; band < g.nbands; band += stride) {
    if (++since_flush > kFlushBands) {
      flush();
      since_flush = 1;
    }
    const BandPlace next = band_place(g, min(band + stride, g.nbands - 1u), lane);
    const bool top = at.by == 0, bottom = at.by + 1u == g.By, left = at.bandx == 0, right = at.bandx + 1u == g.nbx;
#pragma unroll
    for (int im = 0; im < 2; ++im) {
      // lanes past the plane hold zeros and add nothing
      band_image_moments(rows[im], acc + im * kLaneMoments);
      if (top || bottom || left || right)
        band_border(rows[im], lane, at.valid, top, bottom, left, right, k_right, s_part[wave].m + im * kImgMoments);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        acc[2 * kLaneMoments] = udot4(rows[0].w[r][h], rows[1].w[r][h], acc[2 * kLaneMoments]);
        acc[2 * kLaneMoments + 1] += (uint32_t)__builtin_popcount(rows[0].w[r][h] ^ rows[1].w[r][h]);
      }
    // block entropy (every lane takes part in the LDS steps); an image's rows
    // of the next band are loaded as soon as its own are used up
    double prod[2];
    prod[0] = band_block_count_product(rows[0], s_cnt[wave], lane);
    band_load(img_x, g, next, lane, rows[0]);
    prod[1] = band_block_count_product(rows[1], s_cnt[wave], lane);
    band_load(img_y, g, next, lane, rows[1]);
    // lane k takes X's block k (its own half and lane k + 32's), lane k + 32
    // takes Y's: one logarithm for both images
    const double mine = lane < 32 ? prod[0] : prod[1], other = lane < 32 ? prod[1] : prod[0];
    const double h = 6.0 - log2(mine * __shfl_xor(other, 32, 64)) * (1.0 / 64.0);
    if (at.valid) {
      esum += h;
      esq += h * h;
      emin = fmin(emin, h);
      emax = fmax(emax, h);
      if (a.block_entropy)
        a.block_entropy[(lane < 32 ? 0u : nb) + ((uint64_t)at.plane * g.By + at.by) * g.Bx + at.bx] = (float)h;
    }
    at = next;
  }
  // wave, then workgroup reduction into this workgroup's partial slot
  flush();
  // over the 32 lanes of each half
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) {
    esum += __shfl_xor(esum, o, 64);
    esq += __shfl_xor(esq, o, 64);
    emin = fmin(emin, __shfl_xor(emin, o, 64));
    emax = fmax(emax, __shfl_xor(emax, o, 64));
  }
  if ((lane & 31) == 0) {
    double *f = s_part[wave].f + (lane >> 5) * 4;
    f[0] = esum;
    f[1] = esq;
    f[2] = emin;
    f[3] = emax;
  }
  __syncthreads();
  if (threadIdx.x < kIntMoments) {
    uint64_t v = 0;
    for (int w = 0; w < kBandWaves; ++w) v += s_part[w].m[threadIdx.x];
    a.partials[blockIdx.x].m[threadIdx.x] = v;
  } else if (threadIdx.x >= 64 && threadIdx.x < 64 + kFltMoments) {
    const int i = threadIdx.x - 64;
    double v = s_part[0].f[i];
    for (int w = 1; w < kBandWaves; ++w) {
      const double o = s_part[w].f[i];
      v = (i & 3) == 2 ? fmin(v, o) : (i & 3) == 3 ? fmax(v, o) : v + o;
    }
    a.partials[blockIdx.x].f[i] = v;
  }
}

// ---------------------------------------------------------------------------
struct JointArgs {
  const uint4 *x;
  const uint4 *y;
  uint64_t nvec;       // samples / 16
  uint64_t per_chunk;  // vectors per workgroup
  uint32_t *hist;      // 65536 bins, bin = 256 x + y: the counts' parts above 255
  uint8_t *bytes;      // per workgroup, the low bytes of its 65536 counts; or
                       // NULL: no room for them, hist gets whole counts
};

// Counts of both samples of p (bins 256 x + y in its halves).
__device__ __forceinline__ void joint_count2(uint32_t *bins, uint32_t p) {
  uint32_t m = p & 0x80008000u;
  asm volatile("" : "+v"(m));  // one mask for the two samples
  uint8_t *base = reinterpret_cast<uint8_t *>(bins);
  atomicAdd(reinterpret_cast<uint32_t *>(base + ((p << 2) & 0x1fffcu)), 1u << ((m >> 11) & 31u));
  atomicAdd(reinterpret_cast<uint32_t *>(base + ((p >> 14) & 0x1fffcu)), 1u << ((m >> 27) & 31u));
}

// Adds the counters of at least kJointLeast to the global histogram and clears
// them.
__device__ __forceinline__ void joint_spill(uint32_t *bins, uint32_t *hist) {
  for (uint32_t i = threadIdx.x; i < kHalfBins; i += kJointThreads) {
    const uint32_t c = bins[i], lo = c & 0xffffu, hi = c >> 16;
    if (max(lo, hi) < kJointLeast) continue;
    if (lo >= kJointLeast) atomicAdd(&hist[i], lo);
    if (hi >= kJointLeast) atomicAdd(&hist[kHalfBins + i], hi);
    bins[i] = (lo >= kJointLeast ? 0u : lo) | (hi >= kJointLeast ? 0u : c & 0xffff0000u);
  }
}

// The low bytes of four counts as a word; what they have above goes to the
// global histogram.
__device__ __forceinline__ uint32_t joint_bytes(const uint32_t (&c)[4], uint32_t *hist) {
  if ((c[0] | c[1] | c[2] | c[3]) > 255u) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (c[k] > 255u) atomicAdd(&hist[k], c[k] & ~255u);
  }
  return (c[0] & 255u) | ((c[1] & 255u) << 8) | ((c[2] & 255u) << 16) | (c[3] << 24);
}

__global__ __launch_bounds__(kJointThreads) void stats_joint_kernel(JointArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t s_bins[kHalfBins];
  static_assert(__alignof__(s_bins) >= sizeof(uint4), "read 16 bytes at a time below");
  for (uint32_t i = threadIdx.x; i < kHalfBins; i += kJointThreads) s_bins[i] = 0u;
  __syncthreads();
  const uint64_t v0 = (uint64_t)blockIdx.x * a.per_chunk;
  const uint64_t v1 = min(a.nvec, v0 + a.per_chunk);
  for (uint64_t part = v0; part < v1; part += kJointPart) {
    if (part != v0) {
      __syncthreads();
      joint_spill(s_bins, a.hist);
      __syncthreads();
    }
    const uint64_t end = min(v1, part + kJointPart);
    for (uint64_t v = part + threadIdx.x; v < end; v += kJointThreads) {
      typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
      const u32x4 xv = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(&a.x[v]));
      const u32x4 yv = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(&a.y[v]));
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        joint_count2(s_bins, __builtin_amdgcn_perm(xv[k], yv[k], 0x05010400u));
        joint_count2(s_bins, __builtin_amdgcn_perm(xv[k], yv[k], 0x07030602u));
      }
    }
  }
  __syncthreads();
  if (!a.bytes) {
    for (uint32_t i = threadIdx.x; i < kHalfBins; i += kJointThreads) {
      const uint32_t c = s_bins[i];
      if (c & 0xffffu) atomicAdd(&a.hist[i], c & 0xffffu);
      if (c >> 16) atomicAdd(&a.hist[kHalfBins + i], c >> 16);
    }
    return;
  }
  uint32_t *out = reinterpret_cast<uint32_t *>(a.bytes + (size_t)blockIdx.x * 2u * kHalfBins);
  for (uint32_t i = threadIdx.x; i < kHalfBins / 4u; i += kJointThreads) {
    const uint4 c = reinterpret_cast<const uint4 *>(s_bins)[i];
    const uint32_t lo[4] = {c.x & 0xffffu, c.y & 0xffffu, c.z & 0xffffu, c.w & 0xffffu};
    const uint32_t hi[4] = {c.x >> 16, c.y >> 16, c.z >> 16, c.w >> 16};
    out[i] = joint_bytes(lo, a.hist + 4u * i);
    out[kHalfBins / 4u + i] = joint_bytes(hi, a.hist + kHalfBins + 4u * i);
  }
}

// ---------------------------------------------------------------------------
// Reductions after the counting kernels, in the workspace (Reduced):
//  * rows kernel, one workgroup per joint-histogram row j (x = j): the row
//    sum (hist_x[j]), sum c log2 c over the row, and the column sums
//    (hist_y) by 64-bit integer atomics; workgroups j < kIntMoments +
//    kFltMoments also reduce one partial moment over the band workgroups.
//  * finalize, one workgroup: everything else, from 256-entry arrays.  (In the
//    rows kernel's last workgroup instead, the device-scope fences that this
//    takes cost more than the launch: 34 us for both against 8 and 7.)
// All floating sums use fixed trees, so the results do not depend on timing.
struct Reduced {
  uint64_t hx[256];
  uint64_t hy[256];
  double rowlog[256];
  uint64_t m[kIntMoments];
  double f[kFltMoments];
};

struct FinArgs {
  StatsGeom g;
  const Partial *partials;
  uint32_t nparts;
  uint32_t *hist;         // the sums are left here
  const uint8_t *bytes;   // of nbytes workgroups
  uint32_t nbytes;
  Reduced *red;
  sf_security_stats *out;
};

typedef unsigned __int128 u128;
typedef __int128 i128;

// Pearson's r from exact moments; numerator and both variance factors as
// 128-bit integers.
__device__ double pearson(uint64_t n, uint64_t sx, uint64_t sy, uint64_t sxx, uint64_t syy, uint64_t sxy) {
  const i128 num = (i128)((u128)n * sxy) - (i128)((u128)sx * sy);
  const i128 dx = (i128)((u128)n * sxx) - (i128)((u128)sx * sx);
  const i128 dy = (i128)((u128)n * syy) - (i128)((u128)sy * sy);
  if (dx <= 0 || dy <= 0) return 0.0;
  return (double)num / sqrt((double)dx * (double)dy);
}

template <class T, class Op>
__device__ T block_reduce(T v, T *sh, Op op) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = kFinThreads / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] = op(sh[t], sh[t + s]);
    __syncthreads();
  }
  const T r = sh[0];
  __syncthreads();
  return r;
}

__device__ double block_sum(double v, double *sh) {
  return block_reduce(v, sh, [](double a, double b) { return a + b; });
}

__device__ double clog2c(uint64_t c) { return c ? (double)c * log2((double)c) : 0.0; }

// Four sums over the block's threads in one fixed LDS tree (deterministic).
__device__ void block_sum4(double (&v)[4], double (*sh)[kFinThreads]) {
  const int t = threadIdx.x;
#pragma unroll
  for (int q = 0; q < 4; ++q) sh[q][t] = v[q];
  __syncthreads();
  for (int s = kFinThreads / 2; s > 0; s >>= 1) {
    if (t < s)
#pragma unroll
      for (int q = 0; q < 4; ++q) sh[q][t] += sh[q][t + s];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = sh[q][0];
}

// One thread per bin for the histogram sums; the scalar results are then
// spread over threads: 0 entropies, 0-5 one (image, direction) pair
// correlation each, 6 the image-pair figures, 7 the block-entropy summaries.
__global__ __launch_bounds__(kFinThreads) void stats_finalize_kernel(FinArgs a) {
  __shared__ uint64_t s_m[kIntMoments];
  __shared__ double s_f[kFltMoments];
  __shared__ double s_red[4][kFinThreads];
  const int t = threadIdx.x;
  const StatsGeom &g = a.g;
  sf_security_stats *o = a.out;
  const Reduced *rd = a.red;
  if (t < kIntMoments) s_m[t] = rd->m[t];
  else if (t >= 64 && t < 64 + kFltMoments) s_f[t - 64] = rd->f[t - 64];
  const uint64_t hx = rd->hx[t], hy = rd->hy[t];
  o->hist_x[t] = hx;
  o->hist_y[t] = hy;
  const uint64_t N = (uint64_t)g.C * g.H * g.W;
  const double dN = (double)N;
  const double e = dN / 256.0;
  double v[4] = {((double)hy - e) * ((double)hy - e) / e, clog2c(hx), clog2c(hy), rd->rowlog[t]};
  block_sum4(v, s_red);  // its barriers also publish s_m and s_f
  if (t == 0) {
    o->samples = N;
    const double lN = log2(dN);
    const double Hx = lN - v[1] / dN, Hy = lN - v[2] / dN, Hxy = lN - v[3] / dN;
    o->chi2_y = v[0];
    o->entropy_x = Hx;
    o->entropy_y = Hy;
    o->joint_entropy = Hxy;
    o->mutual_information = Hx + Hy - Hxy;
    o->nmi = Hx * Hy > 0.0 ? (Hx + Hy - Hxy) / sqrt(Hx * Hy) : 0.0;
  }
  if (t < 6) {
    // directional pair moments from whole-plane and border sums; h: x drops
    // the last column, y the first; v: rows; d: both
    const int im = t / 3, d = t - 3 * (t / 3);
    const uint64_t C = g.C, H = g.H, W = g.W;
    const uint64_t *m = s_m + im * kImgMoments;
    uint64_t n, sx, sy, qx, qy, pr;
    if (d == 0) {
      n = C * H * (W - 1);
      sx = m[kT1] - m[kCLS];
      sy = m[kT1] - m[kC0S];
      qx = m[kT2] - m[kCLQ];
      qy = m[kT2] - m[kC0Q];
      pr = m[kSh];
    } else if (d == 1) {
      n = C * (H - 1) * W;
      sx = m[kT1] - m[kRLS];
      sy = m[kT1] - m[kR0S];
      qx = m[kT2] - m[kRLQ];
      qy = m[kT2] - m[kR0Q];
      pr = m[kSv];
    } else {
      n = C * (H - 1) * (W - 1);
      sx = m[kT1] - m[kRLS] - m[kCLS] + m[kBRS];
      sy = m[kT1] - m[kR0S] - m[kC0S] + m[kTLS];
      qx = m[kT2] - m[kRLQ] - m[kCLQ] + m[kBRQ];
      qy = m[kT2] - m[kR0Q] - m[kC0Q] + m[kTLQ];
      pr = m[kSd];
    }
    uint64_t *pm = (im == 0 ? o->pair_x : o->pair_y)[d];
    pm[0] = n;
    pm[1] = sx;
    pm[2] = sy;
    pm[3] = qx;
    pm[4] = qy;
    pm[5] = pr;
    (im == 0 ? o->corr_x : o->corr_y)[d] = pearson(n, sx, sy, qx, qy, pr);
  } else if (t == 6) {
    const uint64_t sx = s_m[kT1], sy = s_m[kImgMoments + kT1];
    const uint64_t sxx = s_m[kT2], syy = s_m[kImgMoments + kT2], sxy = s_m[kCrossXY];
    o->cross[0] = N;
    o->cross[1] = sx;
    o->cross[2] = sy;
    o->cross[3] = sxx;
    o->cross[4] = syy;
    o->cross[5] = sxy;
    o->bits_differing = s_m[kBitsDiff];
    o->corr2 = pearson(N, sx, sy, sxx, syy, sxy);
    o->dif = 100.0 * (double)s_m[kBitsDiff] / (8.0 * dN);
    const uint64_t sse = sxx + syy - 2u * sxy;  // sum (x - y)^2, exact
    o->psnr = sse == 0 ? __builtin_huge_val() : 10.0 * log10(65025.0 * dN / (double)sse);
  } else if (t == 7) {
    const double nbk = (double)((uint64_t)g.C * g.By * g.Bx);
    for (int im = 0; im < 2; ++im) {
      double *be = im == 0 ? o->block_entropy_x : o->block_entropy_y;
      const double mean = s_f[4 * im] / nbk;
      const double var = s_f[4 * im + 1] / nbk - mean * mean;
      be[0] = mean;
      be[1] = var > 0.0 ? sqrt(var) : 0.0;
      be[2] = s_f[4 * im + 2];
      be[3] = s_f[4 * im + 3];
    }
  }
}

__global__ __launch_bounds__(kFinThreads) void stats_rows_kernel(FinArgs a) {
  __shared__ double s_d[kFinThreads];
  __shared__ uint64_t s_u[kFinThreads];
  const int t = threadIdx.x;
  const uint32_t j = blockIdx.x;
  // the row's counts: four bins a word, every fourth workgroup's a thread
  // (at most 64 x 255 in a halfword)
  __shared__ __attribute__((aligned(16))) uint32_t s_c[4][256];
  static_assert(__alignof__(s_c) >= sizeof(uint4), "written 16 bytes at a time below");
  uint32_t even = 0, odd = 0;
  const uint32_t *rowp = reinterpret_cast<const uint32_t *>(a.bytes) + 64u * j + (t & 63);
  for (uint32_t p = (uint32_t)t >> 6; p < a.nbytes; p += 64u) {
    uint32_t w[16];  // loads of 16 workgroups' counts in flight
#pragma unroll
    for (uint32_t k = 0; k < 16u; ++k) w[k] = p + 4u * k < a.nbytes ? rowp[(size_t)(p + 4u * k) * 16384u] : 0u;
#pragma unroll
    for (uint32_t k = 0; k < 16u; ++k) {
      even += w[k] & 0x00ff00ffu;
      odd += (w[k] >> 8) & 0x00ff00ffu;
    }
  }
  reinterpret_cast<uint4 *>(s_c[t >> 6])[t & 63] = make_uint4(even & 0xffffu, odd & 0xffffu, even >> 16, odd >> 16);
  __syncthreads();
  const uint32_t c = a.hist[j * 256u + t] + ((s_c[0][t] + s_c[1][t]) + (s_c[2][t] + s_c[3][t]));
  a.hist[j * 256u + t] = c;
  atomicAdd(reinterpret_cast<unsigned long long *>(&a.red->hy[t]), (unsigned long long)c);
  const uint64_t rs = block_reduce<uint64_t>(c, s_u, [](uint64_t x, uint64_t y) { return x + y; });
  const double rl = block_sum(clog2c(c), s_d);
  if (t == 0) {
    a.red->hx[j] = rs;
    a.red->rowlog[j] = rl;
  }
  // one partial moment per workgroup: a fixed split over the threads, then a tree
  if (j < (uint32_t)kIntMoments) {
    uint64_t v = 0;
    for (uint32_t p = t; p < a.nparts; p += kFinThreads) v += a.partials[p].m[j];
    v = block_reduce<uint64_t>(v, s_u, [](uint64_t x, uint64_t y) { return x + y; });
    if (t == 0) a.red->m[j] = v;
  } else if (j < (uint32_t)(kIntMoments + kFltMoments)) {
    const int i = (int)j - kIntMoments;
    const int kind = i & 3;  // 0, 1: sums; 2: min; 3: max
    double v = kind == 2 ? 1e300 : kind == 3 ? -1e300 : 0.0;
    for (uint32_t p = t; p < a.nparts; p += kFinThreads) {
      const double w = a.partials[p].f[i];
      v = kind == 2 ? fmin(v, w) : kind == 3 ? fmax(v, w) : v + w;
    }
    v = block_reduce<double>(v, s_d, [kind](double x, double y) {
      return kind == 2 ? fmin(x, y) : kind == 3 ? fmax(x, y) : x + y;
    });
    if (t == 0) a.red->f[i] = v;
  }
}

StatsGeom stats_geom(uint32_t H, uint32_t W, uint32_t C) {
  StatsGeom g;
  g.H = H;
  g.W = W;
  g.C = C;
  g.By = H / 8;
  g.Bx = W / 8;
  g.nbx = (g.Bx + 31) / 32;
  g.nbands = C * g.By * g.nbx;
  g.div_nbx = udiv_magic(g.nbx);
  g.div_by = udiv_magic(g.By);
  return g;
}

}  // namespace

constexpr size_t kHistBytes = 65536 * sizeof(uint32_t);
constexpr size_t kPartBytes = kBandGrid * sizeof(Partial);
static_assert(kHistBytes % 16 == 0 && kPartBytes % 16 == 0, "workspace parts stay 16-byte aligned");

static_assert(sizeof(Reduced) % 16 == 0, "workspace parts stay 16-byte aligned");

size_t stats_least_workspace_bytes() { return kHistBytes + kPartBytes + sizeof(Reduced); }
size_t stats_workspace_bytes() { return stats_least_workspace_bytes() + kJointGrid * 2u * kHalfBins; }

int launch_security_stats(const DeviceState &ds, const uint8_t *x, const uint8_t *y, uint32_t H, uint32_t W,
                          uint32_t C, void *ws, size_t ws_bytes, sf_security_stats *out, float *block_entropy,
                          hipStream_t stream) {
  const StatsGeom g = stats_geom(H, W, C);
  uint32_t *hist = static_cast<uint32_t *>(ws);
  Partial *parts = reinterpret_cast<Partial *>(static_cast<uint8_t *>(ws) + kHistBytes);
  Reduced *red = reinterpret_cast<Reduced *>(static_cast<uint8_t *>(ws) + kHistBytes + kPartBytes);
  uint8_t *bytes = reinterpret_cast<uint8_t *>(red + 1);
  // the histogram and the column sums start at zero: cleared by the band
  // kernel (not a memset, so the sequence can be captured in a graph)
  BandArgs b{g, x, y, parts, block_entropy, hist, reinterpret_cast<uint32_t *>(red->hy), 65536u,
             (uint32_t)(sizeof(red->hy) / 4u)};
  // one generation of resident workgroups (more would leave a partly empty
  // last generation), at most kBandGrid partial slots
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)&stats_band_kernel, kBandThreads, 0) !=
          hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  const uint32_t need = (g.nbands + kBandWaves - 1) / kBandWaves;
  uint32_t grid = std::min<uint32_t>((uint32_t)ds.num_cu * (uint32_t)per_cu, (uint32_t)kBandGrid);
  grid = std::min(grid, need);
  hipLaunchKernelGGL(stats_band_kernel, dim3(grid), dim3(kBandThreads), 0, stream, b);
  JointArgs j;
  j.x = reinterpret_cast<const uint4 *>(x);
  j.y = reinterpret_cast<const uint4 *>(y);
  j.nvec = (uint64_t)C * H * W / 16u;
  // 128 KB of LDS: one workgroup per CU
  const uint64_t chunks = std::max<uint64_t>(1, std::min<uint64_t>(std::min<uint64_t>((uint64_t)ds.num_cu, kJointGrid), j.nvec / 2048u));
  j.per_chunk = (j.nvec + chunks - 1) / chunks;
  j.hist = hist;
  // a workspace without room for every joint workgroup's counts (sized for
  // the least, which is what it took before there were any) still serves: the
  // joint histogram is then summed by atomics
  const bool room = ws_bytes >= stats_least_workspace_bytes() + chunks * 2u * kHalfBins;
  j.bytes = room ? bytes : nullptr;
  hipLaunchKernelGGL(stats_joint_kernel, dim3((uint32_t)chunks), dim3(kJointThreads), 0, stream, j);
  FinArgs f{g, parts, grid, hist, bytes, room ? (uint32_t)chunks : 0u, red, out};
  hipLaunchKernelGGL(stats_rows_kernel, dim3(256), dim3(kFinThreads), 0, stream, f);
  hipLaunchKernelGGL(stats_finalize_kernel, dim3(1), dim3(kFinThreads), 0, stream, f);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? SF_OK : hip_fail(e, "security statistics launch");
}

}  // namespace sf
