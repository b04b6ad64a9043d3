// Benchmark consumers of delivered bytes, shared by the workload kernels: the wrapping
// u64 checksum of little-endian u32 words (a trailing partial word zero-padded), the byte
// histogram, and a block-wide sum. They are not part of the page cache.
#ifndef GFS_CONSUMERS_H
#define GFS_CONSUMERS_H

#include <hip/hip_runtime.h>

#include "gfs_device.h"

namespace gfs_consumers {

// Fold a delivered buffer into the block's consumer state.
// checksum: wrapping u64 sum of LE u32 words, a trailing partial word zero-padded.
__device__ __forceinline__ uint64_t checksum_part(const uint8_t* buf, uint64_t n, uint32_t tid,
                                                  uint32_t nt) {
  uint64_t s = 0;
  const uint64_t n16 = n >> 4;
  const gfsd::gv4u* v = (const gfsd::gv4u*)buf;   /* user buffers are global memory */
  uint64_t i = tid;
  for (; i + 7ull * nt < n16; i += 8ull * nt) {
    gfsd::v4u x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = v[i + (uint64_t)k * nt];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += (uint64_t)x[k].x + x[k].y + x[k].z + x[k].w;
  }
  if (i < n16) {   // the last, partly filled round, its loads in flight together as well
    gfsd::v4u x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      x[k] = gfsd::v4u{0, 0, 0, 0};
      if (i + (uint64_t)k * nt < n16) x[k] = v[i + (uint64_t)k * nt];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) s += (uint64_t)x[k].x + x[k].y + x[k].z + x[k].w;
  }
  // remaining bytes (n not a multiple of 16): whole words, then the zero-padded last word
  const uint64_t rem0 = n16 << 4;
  for (uint64_t w = rem0 + 4ull * tid; w < n; w += 4ull * nt) {
    uint32_t word = 0;
    for (int b = 0; b < 4; ++b)
      if (w + b < n) word |= (uint32_t)buf[w + b] << (8 * b);
    s += word;
  }
  return s;
}

// Byte histogram. The block counts into several copies (columns) of the 256 counters, lane l into
// copy l mod the columns, laid out so that with 32 of them a lane's counters all lie in its own LDS
// bank: no two lanes of half a wave ever wait for each other, whatever the bytes (with one copy, 64
// random bytes met in a bank 4-5 at a time, equal bytes 64 at a time). Eight 16-byte loads a thread
// are in flight; with one, the loop waited a cache round trip for every 16 bytes.
// The rounds go from the last to the first: the buffer's end was delivered last, and its start may
// have left the XCD's L2, and for large reads the last-level cache, before the pass begins.
// 512 MiB of cached 256 KiB pages, gread and histogram: 322 us (one load, one copy), 300 (eight
// loads), 291 (and 32 copies); by now 271 in forward order, 264 in reverse.
//
// Blocks of one and two waves take 4 and 16 columns: a compute unit's registers hold 8 and 4 such
// blocks, which leave 20 and 40 KiB of its LDS to each, 13-14 of them for gread's state. With 32
// columns (32 KiB) only 3 blocks were resident.
__host__ __device__ __forceinline__ constexpr uint32_t hist_column_bits(uint32_t nt) {
  return nt <= 64 ? 2u : nt <= 128 ? 4u : 5u;
}
__host__ __device__ __forceinline__ constexpr uint32_t hist_bytes(uint32_t nt) { return 1024u << hist_column_bits(nt); }

__device__ __forceinline__ void histogram_clear(uint32_t* hist, uint32_t tid, uint32_t nt) {
  for (uint32_t i = tid; i < 256u << hist_column_bits(nt); i += nt) hist[i] = 0;
}

template <bool kSum, uint32_t kOne = 1u>
__device__ __forceinline__ uint64_t count_part(const uint8_t* buf, uint64_t n, uint32_t tid, uint32_t nt,
                                               uint32_t* hist) {
  const uint64_t n16 = n >> 4;
  const gfsd::gv4u* v = (const gfsd::gv4u*)buf;
  const uint32_t cb = hist_column_bits(nt);
  uint32_t* const mine = hist + (tid & ((1u << cb) - 1));
  uint64_t s = 0;
  const auto count = [&](uint32_t w) {
#pragma unroll
    for (int b = 0; b < 4; ++b) atomicAdd(&mine[((w >> (8 * b)) & 0xff) << cb], kOne);
  };
  const auto unit = [&](const gfsd::v4u& x) {
    if (kSum) s += (uint64_t)x.x + x.y + x.z + x.w;
    count(x.x);
    count(x.y);
    count(x.z);
    count(x.w);
  };
  // rounds of eight units a thread; a 64-bit division costs as much as a round
  uint64_t r = n16 >> 32 ? n16 / (8ull * nt) : (uint64_t)((uint32_t)n16 / (8u * nt));
  const uint64_t i = r * 8ull * nt + tid;
  {   // the last, partly filled one
    gfsd::v4u x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (i + (uint64_t)k * nt < n16) x[k] = v[i + (uint64_t)k * nt];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (i + (uint64_t)k * nt < n16) unit(x[k]);
  }
  const gfsd::gv4u* u = v + i;
  while (r-- > 0) {
    gfsd::v4u x[8];
    u -= 8ull * nt;
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = u[(uint64_t)k * nt];
#pragma unroll
    for (int k = 0; k < 8; ++k) unit(x[k]);
  }
  for (uint64_t j = (n16 << 4) + tid; j < n; j += nt) {
    atomicAdd(&mine[(uint32_t)buf[j] << cb], kOne);
    if (kSum) s += (uint64_t)buf[j] << (8 * (j & 3));
  }
  return s;
}
__device__ __forceinline__ void histogram_part(const uint8_t* buf, uint64_t n, uint32_t tid, uint32_t nt,
                                               uint32_t* hist) {
  (void)count_part<false>(buf, n, tid, nt, hist);
}
// checksum_part and histogram_part in one pass over the buffer, which for a large unit no longer
// lies in the XCD's L2. Out of line: its 32 data registers are not the caller's, which keeps values
// across gread. 64 files of 345 MiB: 307 us (two passes), 258 (one), 252 (out of line), 240 (in
// reverse order).
__device__ __attribute__((noinline)) uint64_t checksum_histogram_part(const uint8_t* buf, uint64_t n, uint32_t tid,
                                                                      uint32_t nt, uint32_t* hist) {
  return count_part<true>(buf, n, tid, nt, hist);
}
// Takes a buffer's bytes out of the histogram again; returns the sum to take off.
__device__ __attribute__((noinline)) uint64_t checksum_histogram_undo(const uint8_t* buf, uint64_t n, uint32_t tid,
                                                                      uint32_t nt, uint32_t* hist) {
  return count_part<true, ~0u>(buf, n, tid, nt, hist);
}

// The count of byte value v over all copies (after a barrier); each lane starts at a copy of its own.
__device__ __forceinline__ uint32_t histogram_count(const uint32_t* hist, uint32_t v, uint32_t nt) {
  const uint32_t cb = hist_column_bits(nt);
  uint32_t s = 0;
  for (uint32_t c = 0; c < 1u << cb; ++c) s += hist[(v << cb) + ((c + v) & ((1u << cb) - 1))];
  return s;
}

__device__ __forceinline__ uint64_t block_sum_u64(uint64_t v, uint64_t* red, uint32_t tid, uint32_t nt) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  uint64_t s = 0;
  if (tid == 0)
    for (uint32_t w = 0; w < (nt + 63) / 64; ++w) s += red[w];
  return s;   /* valid in thread 0 */
}

}  // namespace gfs_consumers

#endif  // GFS_CONSUMERS_H
