// Sign bit-packing kernels: logical int8 (+-1, row-major)  <->  device tile layout.
// The layout is described in mdbf_internal.h.
#include "mdbf_internal.h"

namespace mdbf {

// One wave packs the 64 words of a (row tile, block): lane (kg, r) owns row r and the 8-column groups
// f * 32 + kg * 8, f = 0..3, whose entries go to bits 8 (f / 2) + 4 (f % 2) + (e / 2) + 16 (e % 2) of its word.
// Both kernels stream: one byte per sign on one side, one bit on the other, so HBM bounds them.  A lane moves a
// column group at a time, eight bytes (any alignment: the target allows it), 32 bytes of a row per instruction
// and the whole 128-byte line over the four groups; a wave takes kPackBlocks consecutive blocks with all their
// loads in flight, the four waves of a workgroup four consecutive tiles (1 KB of words per block).  Byte by
// byte, 32 loads per word, packing 11008 x 4096 took 91 us and unpacking 82 us; now 14 and
// 17 us (3.6 and 3.0 TB/s; a large copy reaches 5.1 TB/s).  (Sizes are compared as blocks or as differences: a column
// index and a block's end may lie past the largest int.)
constexpr int kPackBlocks = 4;

typedef uint32_t Octet __attribute__((ext_vector_type(2), aligned(1)));   // eight consecutive signs of a row

// sign bits of four bytes (entries e, e + 1, e + 2, e + 3; e = 0 or 4) to bits 0, 16, 1, 17
__device__ __forceinline__ uint32_t gather4(uint32_t d) {
  const uint32_t y = d >> 7;
  return (y & 1u) | ((y & 0x100u) << 8) | ((y & 0x10000u) >> 15) | ((y & 0x1000000u) >> 7);
}
// the inverse: bits 0, 16, 1, 17 to the bytes +1 (0x01) or -1 (0xFF)
__device__ __forceinline__ uint32_t spread4(uint32_t b) {
  const uint32_t y = (b & 1u) | ((b >> 8) & 0x100u) | ((b << 15) & 0x10000u) | ((b << 7) & 0x1000000u);
  return 0x01010101u | (y * 0xFEu);
}

__global__ __launch_bounds__(256) void pack_kernel(const int8_t* __restrict__ signs, int rows, int cols, int64_t ld,
                                                   uint32_t* __restrict__ packed, int KB, int ntiles) {
  const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
  const int tile = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tile >= ntiles) return;
  const int row = tile * kTileRows + r;
  const MDBF_GLOBAL int8_t* src = (const MDBF_GLOBAL int8_t*)signs + (int64_t)min(row, rows - 1) * ld;
  for (int q0 = blockIdx.y * kPackBlocks; q0 < KB; q0 += gridDim.y * kPackBlocks) {
    uint32_t w[kPackBlocks];
    if (q0 + kPackBlocks <= cols / kBlockCols) {              // (uniform) whole blocks: no bounds to respect
      Octet o[kPackBlocks][4];
#pragma unroll
      for (int j = 0; j < kPackBlocks; ++j)
#pragma unroll
        for (int f = 0; f < 4; ++f) o[j][f] = *(const MDBF_GLOBAL Octet*)(src + (q0 + j) * kBlockCols + f * 32 + kg * 8);
#pragma unroll
      for (int j = 0; j < kPackBlocks; ++j) {
        w[j] = 0;
#pragma unroll
        for (int f = 0; f < 4; ++f)
          w[j] |= (gather4(o[j][f].x) | (gather4(o[j][f].y) << 2)) << (8 * (f >> 1) + 4 * (f & 1));
      }
    } else {
#pragma unroll
      for (int j = 0; j < kPackBlocks; ++j) {
        w[j] = 0;
        if (q0 + j >= KB) continue;
#pragma unroll 1
        for (int f = 0; f < 4; ++f) {
          const int c0 = (q0 + j) * kBlockCols + f * 32 + kg * 8;
          uint32_t bits = 0;
          if (c0 <= cols - 8) {
            const Octet o = *(const MDBF_GLOBAL Octet*)(src + c0);
            bits = gather4(o.x) | (gather4(o.y) << 2);
          } else {
            for (int e = 0; e < 8; ++e)
              if (e < cols - c0 && src[c0 + e] < 0) bits |= 1u << ((e >> 1) + 16 * (e & 1));
          }
          w[j] |= bits << (8 * (f >> 1) + 4 * (f & 1));
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kPackBlocks; ++j)
      if (q0 + j < KB)
        ((MDBF_GLOBAL uint32_t*)packed)[word_offset(tile, q0 + j, lane, KB, ntiles)] = row < rows ? w[j] : 0u;
  }
}

__global__ __launch_bounds__(256) void unpack_kernel(const uint32_t* __restrict__ packed, int rows, int cols,
                                                     int8_t* __restrict__ signs, int64_t ld, int KB, int ntiles) {
  const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
  const int tile = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tile >= ntiles) return;
  const int row = tile * kTileRows + r;
  MDBF_GLOBAL int8_t* dst = (MDBF_GLOBAL int8_t*)signs + (int64_t)row * ld;
  for (int q0 = blockIdx.y * kPackBlocks; q0 < KB; q0 += gridDim.y * kPackBlocks) {
    uint32_t w[kPackBlocks];
#pragma unroll
    for (int j = 0; j < kPackBlocks; ++j)
      w[j] = ((const MDBF_GLOBAL uint32_t*)packed)[word_offset(tile, min(q0 + j, KB - 1), lane, KB, ntiles)];
    if (row >= rows) return;
#pragma unroll
    for (int j = 0; j < kPackBlocks; ++j) {
      if (q0 + j >= KB) continue;
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const int c0 = (q0 + j) * kBlockCols + f * 32 + kg * 8;
        const uint32_t bits = w[j] >> (8 * (f >> 1) + 4 * (f & 1));
        Octet o;
        o.x = spread4(bits);
        o.y = spread4(bits >> 2);
        if (c0 <= cols - 8) {
          *(MDBF_GLOBAL Octet*)(dst + c0) = o;
        } else {
          for (int e = 0; e < 8; ++e)
            if (e < cols - c0) dst[c0 + e] = (int8_t)((e < 4 ? o.x >> (8 * e) : o.y >> (8 * e - 32)) & 0xFFu);
        }
      }
    }
  }
}

// (the kernels walk further blocks themselves where the y extent of a grid ends)
static dim3 pack_grid(int KB, int ntiles) {
  const int gy = (KB + kPackBlocks - 1) / kPackBlocks;
  return dim3((unsigned)((ntiles + 3) / 4), (unsigned)(gy < 65535 ? gy : 65535));
}

int launch_pack(const int8_t* signs, int rows, int cols, int64_t ld, uint32_t* packed, hipStream_t s) {
  const int KB = num_blocks(cols), nt = num_tiles(rows);
  hipLaunchKernelGGL(pack_kernel, pack_grid(KB, nt), dim3(256), 0, s, signs, rows, cols, ld, packed, KB, nt);
  return (int)hipGetLastError();
}

int launch_unpack(const uint32_t* packed, int rows, int cols, int8_t* signs, int64_t ld, hipStream_t s) {
  const int KB = num_blocks(cols), nt = num_tiles(rows);
  hipLaunchKernelGGL(unpack_kernel, pack_grid(KB, nt), dim3(256), 0, s, packed, rows, cols, signs, ld, KB, nt);
  return (int)hipGetLastError();
}

// Envelope factor with zero modes appended: dst[r, c] = src[r, c] for c < l, 0 for l <= c < l_to.
// The product is unchanged (the extra modes contribute nothing); ranks 8 and 16 are the ones the matrix-core
// kernels take.  Elements are moved as raw bits: es = bytes per element (2 or 4).
__global__ __launch_bounds__(256) void pad_envelope_kernel(const unsigned char* __restrict__ src, int rows, int l,
                                                           unsigned char* __restrict__ dst, int l_to, int es) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)rows * (size_t)l_to) return;
  const size_t r = i / (size_t)l_to;
  const int c = (int)(i - r * (size_t)l_to);
  if (es == 2) {
    ((MDBF_GLOBAL uint16_t*)dst)[i] = c < l ? ((const MDBF_GLOBAL uint16_t*)src)[r * (size_t)l + c] : (uint16_t)0;
  } else {
    ((MDBF_GLOBAL uint32_t*)dst)[i] = c < l ? ((const MDBF_GLOBAL uint32_t*)src)[r * (size_t)l + c] : 0u;
  }
}

int launch_pad_envelope(const void* src, int rows, int l, void* dst, int l_to, int es, hipStream_t s) {
  const size_t n = (size_t)rows * (size_t)l_to;
  hipLaunchKernelGGL(pad_envelope_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     (const unsigned char*)src, rows, l, (unsigned char*)dst, l_to, es);
  return (int)hipGetLastError();
}

// Plain streaming read: lane t of the launch reads the 16-byte elements t, t + lanes, t + 2 * lanes, ...
// (four independent loads per trip) and XORs them; every wave stores one word.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4_t* __restrict__ src, size_t n16,
                                                          uint32_t* __restrict__ sink) {
  const MDBF_GLOBAL u32x4_t* g = (const MDBF_GLOBAL u32x4_t*)src;
  const size_t lanes = (size_t)gridDim.x * 256;
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  u32x4_t a0 = {0, 0, 0, 0}, a1 = a0, a2 = a0, a3 = a0;
  for (; i + 3 * lanes < n16; i += 4 * lanes) {
    a0 ^= __builtin_nontemporal_load(g + i);
    a1 ^= __builtin_nontemporal_load(g + i + lanes);
    a2 ^= __builtin_nontemporal_load(g + i + 2 * lanes);
    a3 ^= __builtin_nontemporal_load(g + i + 3 * lanes);
  }
  for (; i < n16; i += lanes) a0 ^= __builtin_nontemporal_load(g + i);
  a0 ^= a1 ^ a2 ^ a3;
  uint32_t v = a0.x ^ a0.y ^ a0.z ^ a0.w;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v ^= (uint32_t)__shfl_xor((int)v, d);
  if ((threadIdx.x & 63) == 0) ((MDBF_GLOBAL uint32_t*)sink)[blockIdx.x * 4 + (threadIdx.x >> 6)] = v;
}

int launch_stream_read(const void* src, size_t bytes, uint32_t* sink, int sink_words, hipStream_t s) {
  hipLaunchKernelGGL(stream_read_kernel, dim3((unsigned)(sink_words / 4)), dim3(256), 0, s, (const u32x4_t*)src,
                     bytes / 16, sink);
  return (int)hipGetLastError();
}

}  // namespace mdbf
