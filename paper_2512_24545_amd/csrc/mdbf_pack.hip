// Sign bit-packing kernels: logical int8 (+-1, row-major)  <->  device tile layout.
// The layout is described in mdbf_internal.h.
#include "mdbf_internal.h"

namespace mdbf {

// One wave packs the 64 words of a (row tile, block): lane (kg, r) owns row r and the 8-column groups
// f * 32 + kg * 8, f = 0..3, whose entries go to bits 8 (f / 2) + 4 (f % 2) + (e / 2) + 16 (e % 2) of its word.
// Both kernels stream: one byte per sign on one side, one bit on the other, so HBM bounds them.  A wave takes
// kPackBlocks consecutive blocks with all their loads in flight, the four waves of a workgroup four consecutive tiles
// (1 KB of words per block).  Whole runs of blocks go between memory and the lanes' column groups through LDS: 16 bytes a
// lane at any alignment (the target allows it), 512 consecutive bytes of a row per half wave.  With every lane on its own
// column groups, eight bytes of a row and a quarter of its line per access, packing 11008 x 4096 took 14 us and unpacking 17;
// both together now 19.5 against 28.6 (5.2 TB/s; a large copy reaches 5.1), whichever way the bits are moved (below).  The
// non-temporal hint: 18.9 with it on both sides, 21.4 on the loads alone; left out, the signs may be read again.  Runs
// that the row's end cuts go group by group.  (Sizes are compared as blocks or as differences: a column
// index and a block's end may lie past the largest int.)
constexpr int kPackBlocks = 4;

// Whole runs of kPackBlocks blocks go through LDS, a row's 512 bytes by 32 lanes at a time.
constexpr int kRunBytes = kPackBlocks * kBlockCols;
constexpr int kRunStride = kRunBytes + 16;                                // of a row in LDS
typedef uint32_t Piece __attribute__((ext_vector_type(4), aligned(1)));   // sixteen consecutive signs of a row
typedef uint32_t PieceLds __attribute__((ext_vector_type(4)));
typedef uint32_t OctetLds __attribute__((ext_vector_type(2)));

// a wave's LDS operations execute in order: this keeps the compiler from moving them across
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef uint32_t Octet __attribute__((ext_vector_type(2), aligned(1)));   // eight consecutive signs of a row

// A lane's word from its four column groups, and back.  A dword holds four entries' bytes: entry e of a group's first one
// goes to bit e / 2 + 16 (e % 2) of the group's nibbles, of its second one two bits further.  The sign bits of two groups
// are first put side by side inside each byte (group 0 at bits 0 and 2, group 1 at 4 and 6), then bytes 2 and 3 between
// those of 0 and 1: 21 and 46 vector instructions a word (entry by entry some 90 and 100).
__device__ __forceinline__ uint32_t pack_groups(const Octet (&o)[4]) {
  uint32_t c[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const uint32_t a = ((o[2 * g].x >> 7) & 0x01010101u) | ((o[2 * g].y >> 5) & 0x04040404u) |
                       ((o[2 * g + 1].x >> 3) & 0x10101010u) | ((o[2 * g + 1].y >> 1) & 0x40404040u);
    c[g] = a | (a >> 15);
  }
  return __builtin_amdgcn_perm(c[1], c[0], 0x05010400u);       // bytes: c0.0, c1.0, c0.1, c1.1
}
__device__ __forceinline__ void unpack_groups(uint32_t w, Octet (&o)[4]) {
  // +1 (0x01) or -1 (0xFF) per byte from bit 0 of each: (b << 8) - b has all bits of the bytes whose bit is set
  auto bytes = [](uint32_t b) __attribute__((always_inline)) { return ((b << 8) - b) | 0x01010101u; };
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const uint32_t c = __builtin_amdgcn_perm(0u, w, g == 0 ? 0x0c0c0200u : 0x0c0c0301u);   // bytes g and g + 2
    const uint32_t a = (c & 0x5555u) | ((c & 0xAAAAu) << 15);
    o[2 * g].x = bytes(a & 0x01010101u);
    o[2 * g].y = bytes((a >> 2) & 0x01010101u);
    o[2 * g + 1].x = bytes((a >> 4) & 0x01010101u);
    o[2 * g + 1].y = bytes((a >> 6) & 0x01010101u);
  }
}

// RUNS: rows hold whole runs (narrower ones do without the LDS)
template <bool RUNS>
__global__ __launch_bounds__(256) void pack_kernel(const int8_t* __restrict__ signs, int rows, int cols, int64_t ld,
                                                   uint32_t* __restrict__ packed, int KB, int ntiles) {
  const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
  const int tile = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tile >= ntiles) return;
  const int row = tile * kTileRows + r;
  const MDBF_GLOBAL int8_t* src = (const MDBF_GLOBAL int8_t*)signs + (int64_t)min(row, rows - 1) * ld;
  __shared__ __attribute__((aligned(16))) unsigned char lds[4][RUNS ? kTileRows * kRunStride : 16];
  unsigned char* buf = lds[threadIdx.x >> 6];
  for (int q0 = blockIdx.y * kPackBlocks; q0 < KB; q0 += gridDim.y * kPackBlocks) {
    uint32_t w[kPackBlocks];
    if (RUNS && q0 + kPackBlocks <= cols / kBlockCols) {      // (uniform) whole blocks: no bounds to respect
      Piece v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int rr = min(tile * kTileRows + 2 * i + (lane >> 5), rows - 1);
        v[i] = *(const MDBF_GLOBAL Piece*)((const MDBF_GLOBAL int8_t*)signs + (int64_t)rr * ld + (int64_t)q0 * kBlockCols + (lane & 31) * 16);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<PieceLds*>(buf + (2 * i + (lane >> 5)) * kRunStride + (lane & 31) * 16) = v[i];
      wave_lds_order();
#pragma unroll
      for (int j = 0; j < kPackBlocks; ++j) {
        Octet o[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) o[f] = *reinterpret_cast<const OctetLds*>(buf + r * kRunStride + j * kBlockCols + f * 32 + kg * 8);
        w[j] = pack_groups(o);
      }
      wave_lds_order();
    } else {
#pragma unroll
      for (int j = 0; j < kPackBlocks; ++j) {
        w[j] = 0;
        if (q0 + j >= KB) continue;
        Octet o[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          const int c0 = (q0 + j) * kBlockCols + f * 32 + kg * 8;
          o[f] = Octet{0u, 0u};
          if (c0 <= cols - 8) {
            o[f] = *(const MDBF_GLOBAL Octet*)(src + c0);
          } else {
            for (int e = 0; e < 8; ++e)
              if (e < cols - c0 && src[c0 + e] < 0) {
                if (e < 4) o[f].x |= 0x80u << (8 * e);
                else o[f].y |= 0x80u << (8 * e - 32);
              }
          }
        }
        w[j] = pack_groups(o);
      }
    }
#pragma unroll
    for (int j = 0; j < kPackBlocks; ++j)
      if (q0 + j < KB)
        ((MDBF_GLOBAL uint32_t*)packed)[word_offset(tile, q0 + j, lane, KB, ntiles)] = row < rows ? w[j] : 0u;
  }
}

template <bool RUNS>
__global__ __launch_bounds__(256) void unpack_kernel(const uint32_t* __restrict__ packed, int rows, int cols,
                                                     int8_t* __restrict__ signs, int64_t ld, int KB, int ntiles) {
  const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
  const int tile = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tile >= ntiles) return;
  const int row = tile * kTileRows + r;
  MDBF_GLOBAL int8_t* dst = (MDBF_GLOBAL int8_t*)signs + (int64_t)row * ld;
  __shared__ __attribute__((aligned(16))) unsigned char lds[4][RUNS ? kTileRows * kRunStride : 16];
  unsigned char* buf = lds[threadIdx.x >> 6];
  for (int q0 = blockIdx.y * kPackBlocks; q0 < KB; q0 += gridDim.y * kPackBlocks) {
    uint32_t w[kPackBlocks];
#pragma unroll
    for (int j = 0; j < kPackBlocks; ++j)
      w[j] = ((const MDBF_GLOBAL uint32_t*)packed)[word_offset(tile, min(q0 + j, KB - 1), lane, KB, ntiles)];
    if (RUNS && q0 + kPackBlocks <= cols / kBlockCols) {      // (uniform)
#pragma unroll
      for (int j = 0; j < kPackBlocks; ++j) {
        Octet o[4];
        unpack_groups(w[j], o);
#pragma unroll
        for (int f = 0; f < 4; ++f) *reinterpret_cast<OctetLds*>(buf + r * kRunStride + j * kBlockCols + f * 32 + kg * 8) = o[f];
      }
      wave_lds_order();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int rr = tile * kTileRows + 2 * i + (lane >> 5);
        const PieceLds v = *reinterpret_cast<const PieceLds*>(buf + (2 * i + (lane >> 5)) * kRunStride + (lane & 31) * 16);
        if (rr < rows) *(MDBF_GLOBAL Piece*)((MDBF_GLOBAL int8_t*)signs + (int64_t)rr * ld + (int64_t)q0 * kBlockCols + (lane & 31) * 16) = v;
      }
      wave_lds_order();
      continue;
    }
    if (row >= rows) return;
#pragma unroll
    for (int j = 0; j < kPackBlocks; ++j) {
      if (q0 + j >= KB) continue;
      Octet all[4];
      unpack_groups(w[j], all);
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const int c0 = (q0 + j) * kBlockCols + f * 32 + kg * 8;
        const Octet o = all[f];
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
  if (cols >= kRunBytes) hipLaunchKernelGGL(pack_kernel<true>, pack_grid(KB, nt), dim3(256), 0, s, signs, rows, cols, ld, packed, KB, nt);
  else hipLaunchKernelGGL(pack_kernel<false>, pack_grid(KB, nt), dim3(256), 0, s, signs, rows, cols, ld, packed, KB, nt);
  return (int)hipGetLastError();
}

int launch_unpack(const uint32_t* packed, int rows, int cols, int8_t* signs, int64_t ld, hipStream_t s) {
  const int KB = num_blocks(cols), nt = num_tiles(rows);
  if (cols >= kRunBytes) hipLaunchKernelGGL(unpack_kernel<true>, pack_grid(KB, nt), dim3(256), 0, s, packed, rows, cols, signs, ld, KB, nt);
  else hipLaunchKernelGGL(unpack_kernel<false>, pack_grid(KB, nt), dim3(256), 0, s, packed, rows, cols, signs, ld, KB, nt);
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
