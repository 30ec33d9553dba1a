// Standalone AES-128-CTR over an arbitrary device buffer (encrypt_private).
// Each lane produces one 16-byte keystream block E_K(ctr0 + first + i) from
// the LDS round tables and XORs it into 16 input bytes (coalesced 16-byte
// loads and stores); the trailing partial block is handled byte by byte.
#include "sf_internal.h"

namespace sf {
namespace {

constexpr int kThreads = 256;

struct CtrArgs {
  const uint8_t *in;
  uint8_t *out;
  uint64_t nbytes;
  uint64_t first;
  uint64_t per_group;  // blocks of one workgroup's run (ctr_wide_kernel)
  const uint32_t *aes_t0;
  AesArgs aes;
};

__global__ __launch_bounds__(kThreads) void ctr_kernel(CtrArgs a) {
  __shared__ AesLds s_aes;
  aes_load_tables(s_aes, a.aes_t0, a.aes.key, threadIdx.x, kThreads);
  __syncthreads();
  const uint64_t nblk = (a.nbytes + 15u) / 16u;
  for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < nblk; i += (uint64_t)gridDim.x * kThreads) {
    uint32_t w0, w1, w2, w3;
    aes_counter(a.aes.ctr_hi, a.aes.ctr_lo, a.first + i, w0, w1, w2, w3);
    aes_encrypt(w0, w1, w2, w3, s_aes);
    const uint64_t off = 16u * i;
    if (off + 16u <= a.nbytes) {
      uint4 v = *reinterpret_cast<const uint4 *>(a.in + off);
      v.x ^= w0;
      v.y ^= w1;
      v.z ^= w2;
      v.w ^= w3;
      *reinterpret_cast<uint4 *>(a.out + off) = v;
    } else {
      const uint64_t lo = (uint64_t)w0 | ((uint64_t)w1 << 32), hi = (uint64_t)w2 | ((uint64_t)w3 << 32);
      for (uint64_t j = off; j < a.nbytes; ++j) {
        const uint32_t k = (uint32_t)(j - off);
        const uint8_t ks = (uint8_t)((k < 8u ? lo >> (8u * k) : hi >> (8u * (k - 8u))) & 0xffu);
        a.out[j] = (uint8_t)(a.in[j] ^ ks);
      }
    }
  }
}

// The same for large buffers.  What bounds the kernel above is the LDS: a
// wave's 64 lookups at random table entries pile up on its banks (about 6
// cycles per lookup measured, 2 without conflicts).  Here one workgroup of 16
// waves fills a CU and holds every T-table entry 32 times, once per pair of
// lanes l, l + 32 (the LDS serves a wave 32 lanes at a time), so that lane l
// reads only bank l % 32: T0 | T1 interleaved in one 64 KB half, T2 | T3 in the
// other, entry b of lane l at byte 256 b + 4 (l % 32).  A lookup address is
// then one v_perm_b32 (the state byte next to the lane's byte) and needs no
// rotation of a shared table.  Each workgroup takes one run of consecutive
// counters, whose upper 112 bits seldom change: what they give to the first two
// rounds (14 and 8 of 16 lookups) is kept from block to block and made again
// when they do change.  138 lookups of 2 cycles and about 250 vector
// instructions (1 cycle each over the CU's four SIMDs) are left per 64 blocks,
// so both units are busy.  Measured on 128 MiB in and out: 202 -> 88-93 us (42 ->
// 90-95 G blocks/s).
constexpr int kWideThreads = 1024;
typedef uint32_t WideTables[2][256][64];

struct WideLookup {
  const uint8_t *base;  // LDS
  uint32_t lane;        // 4 (l % 32), and 1 in byte 2 to reach the second half
  // T_K of byte B of s
  template <int K, int B>
  __device__ __forceinline__ uint32_t at(uint32_t s) const {
    constexpr uint32_t sel = 0x0c000000u | ((K & 2) ? 0x00020000u : 0x000c0000u) | ((4u + B) << 8);
    return *reinterpret_cast<const uint32_t *>(base + __builtin_amdgcn_perm(s, lane, sel) + 128 * (K & 1));
  }
  __device__ __forceinline__ uint32_t column(uint32_t s0, uint32_t s1, uint32_t s2, uint32_t s3, uint32_t rk) const {
    return xor3(xor3(at<0, 0>(s0), at<1, 1>(s1), at<2, 2>(s2)), at<3, 3>(s3), rk);
  }
  // last round: S-box byte r sits at byte r of T2, T3, T0, T1 for r = 0..3
  __device__ __forceinline__ uint32_t last(uint32_t s0, uint32_t s1, uint32_t s2, uint32_t s3, uint32_t rk) const {
    const uint32_t lo = __builtin_amdgcn_perm(at<3, 1>(s1), at<2, 0>(s0), 0x0c0c0500u);
    const uint32_t hi = __builtin_amdgcn_perm(at<1, 3>(s3), at<0, 2>(s2), 0x07020c0cu);
    return xor3(lo, hi, rk);
  }
};

__global__ __launch_bounds__(kWideThreads) void ctr_wide_kernel(CtrArgs a) {
  __shared__ __attribute__((aligned(16))) WideTables s_t;
  for (uint32_t c = threadIdx.x; c < sizeof(WideTables) / 16u; c += kWideThreads) {
    const uint32_t k = 2u * (c >> 12) + ((c >> 3) & 1u), v = a.aes_t0[(c >> 4) & 255u];
    const uint32_t r = k ? (v << (8u * k)) | (v >> (32u - 8u * k)) : v;
    reinterpret_cast<uint4 *>(s_t)[c] = make_uint4(r, r, r, r);
  }
  __syncthreads();
  const WideLookup T{reinterpret_cast<const uint8_t *>(s_t), 4u * (threadIdx.x & 31u) | 0x00010000u};
  const uint32_t *rk = a.aes.key.rk;
  const uint64_t nblk = (a.nbytes + 15u) / 16u;
  uint64_t i = (uint64_t)blockIdx.x * a.per_group + threadIdx.x;
  const uint64_t end = min(nblk, (uint64_t)(blockIdx.x + 1) * a.per_group);
  // state after round 1 in columns 2 and 3, and what the upper bits give to
  // columns 0 and 1 of round 1 and to round 2
  uint64_t upper = 0;
  uint32_t k0 = 0, k1 = 0, c0 = 0, c1 = 0, c2 = 0, c3 = 0;
  bool have = false;
  for (; i < end; i += kWideThreads) {
    const uint64_t off = 16u * i;
    const bool whole = off + 16u <= a.nbytes;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (whole) v = *reinterpret_cast<const uint4 *>(a.in + off);
    const uint64_t low = a.aes.ctr_lo + (a.first + i);  // the counter's lower half
    uint32_t s0, s1, s2, s3 = __builtin_bswap32((uint32_t)low) ^ rk[3];
    const uint64_t tag = low >> 16 | (uint64_t)(low < a.aes.ctr_lo) << 48;  // with the carry into the upper half
    if (!have || tag != upper) {
      have = true;
      upper = tag;
      uint32_t w0, w1, w2, w3;
      aes_counter(a.aes.ctr_hi, a.aes.ctr_lo, a.first + i, w0, w1, w2, w3);
      w0 ^= rk[0];
      w1 ^= rk[1];
      w2 ^= rk[2];
      k0 = xor3(T.at<0, 0>(w0), T.at<1, 1>(w1), T.at<2, 2>(w2)) ^ rk[4];
      k1 = xor3(T.at<0, 0>(w1), T.at<1, 1>(w2), T.at<3, 3>(w0)) ^ rk[5];
      const uint32_t k2 = T.column(w2, s3, w0, w1, rk[6]), k3 = T.column(s3, w0, w1, w2, rk[7]);
      c0 = xor3(T.at<2, 2>(k2), T.at<3, 3>(k3), rk[8]);
      c1 = xor3(T.at<1, 1>(k2), T.at<2, 2>(k3), rk[9]);
      c2 = xor3(T.at<0, 0>(k2), T.at<1, 1>(k3), rk[10]);
      c3 = xor3(T.at<0, 0>(k3), T.at<3, 3>(k2), rk[11]);
    }
    const uint32_t f0 = k0 ^ T.at<3, 3>(s3), f1 = k1 ^ T.at<2, 2>(s3);
    s0 = xor3(T.at<0, 0>(f0), T.at<1, 1>(f1), c0);
    s1 = xor3(T.at<0, 0>(f1), T.at<3, 3>(f0), c1);
    s2 = xor3(T.at<2, 2>(f0), T.at<3, 3>(f1), c2);
    s3 = xor3(T.at<1, 1>(f0), T.at<2, 2>(f1), c3);
#pragma unroll
    for (int r = 3; r < 10; ++r) {
      const uint32_t t0 = T.column(s0, s1, s2, s3, rk[4 * r]), t1 = T.column(s1, s2, s3, s0, rk[4 * r + 1]);
      const uint32_t t2 = T.column(s2, s3, s0, s1, rk[4 * r + 2]), t3 = T.column(s3, s0, s1, s2, rk[4 * r + 3]);
      s0 = t0;
      s1 = t1;
      s2 = t2;
      s3 = t3;
    }
    const uint32_t w[4] = {T.last(s0, s1, s2, s3, rk[40]), T.last(s1, s2, s3, s0, rk[41]),
                           T.last(s2, s3, s0, s1, rk[42]), T.last(s3, s0, s1, s2, rk[43])};
    if (whole) {
      v.x ^= w[0];
      v.y ^= w[1];
      v.z ^= w[2];
      v.w ^= w[3];
      *reinterpret_cast<uint4 *>(a.out + off) = v;
    } else {
      for (uint32_t j = 0; off + j < a.nbytes; ++j)
        a.out[off + j] = (uint8_t)(a.in[off + j] ^ (uint8_t)(w[j >> 2] >> (8u * (j & 3u))));
    }
  }
}

// From 4 MiB on the wide kernel: its tables take about 3 us to fill whatever
// the size, and up to 2 MiB both are one launch's latency (8.3 / 8.0 us a call
// in a row of calls at 2 MiB, 9.9 / 8.0 at 4, 16.9 / 9.7 at 8, 53.7 / 26.0 at 32).
constexpr uint64_t kWideMinBlocks = 1u << 18;

}  // namespace

int launch_ctr(const DeviceState &ds, const AesArgs &aes, uint64_t first_block, const uint8_t *in, uint8_t *out,
               size_t nbytes, hipStream_t stream) {
  if (((uintptr_t)in | (uintptr_t)out) & 15u) return fail(SF_EINVAL, "buffers must be 16-byte aligned");
  CtrArgs a;
  a.in = in;
  a.out = out;
  a.nbytes = nbytes;
  a.first = first_block;
  a.per_group = 0;
  a.aes_t0 = ds.d_aes_t0;
  a.aes = aes;
  const uint64_t nblk = (nbytes + 15u) / 16u;
  if (nblk >= kWideMinBlocks && sizeof(WideTables) <= ds.max_lds_per_block) {
    const uint64_t need = (nblk + kWideThreads - 1) / kWideThreads;
    const unsigned wide = (unsigned)(need < (uint64_t)ds.num_cu ? need : (uint64_t)ds.num_cu);
    a.per_group = ((nblk + wide - 1) / wide + 63u) & ~(uint64_t)63u;
    hipLaunchKernelGGL(ctr_wide_kernel, dim3(wide), dim3(kWideThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SF_OK : hip_fail(e, "ctr_wide_kernel launch");
  }
  uint64_t grid = (nblk + kThreads - 1) / kThreads;
  const uint64_t cap = (uint64_t)ds.num_cu * 8u;
  if (grid > cap) grid = cap;
  hipLaunchKernelGGL(ctr_kernel, dim3((unsigned)grid), dim3(kThreads), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "ctr_kernel launch");
  return SF_OK;
}

}  // namespace sf
