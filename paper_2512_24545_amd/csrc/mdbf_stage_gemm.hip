// Many-token evaluation of one envelope-scaled binary product on gfx950, in reconstruct order.
//
//   out[b, r] = sum_j W[r, j] * vin[b, j],     W[r, j] = S[r, j] * E[r, j],     E = Eout * Ein^T  (rank l)
//
// The same product as the other stage kernels (paper Eq. "me-dbf-basis": the factor is the sign matrix
// modulated by a rank-l envelope), but evaluated as a dense GEMM against the reconstructed factor instead
// of l scaled binary products: (l + T) multiply-adds per sign entry instead of l * T.  Nothing dense ever
// reaches memory: a wave rebuilds its 16 x 128 piece of E with eight small matrix-core products
// (contraction over the l modes), flips signs with the packed bits, rounds to fp16 and holds the piece in
// registers as the B operand of the token product; the activations go through LDS, shared by the waves.
//
//  * workgroup: 4 waves; wave w owns R row tiles (16 rows each); the workgroup owns 16 * TB tokens
//  * per 128-column block: E piece per tile = 2 x v_mfma_f32_16x16x16_f16 per 32 columns.  The products'
//    row index is chosen so that lane (r, g) receives columns 32f + 8g + 0..7 of row r: exactly the columns
//    whose signs sit in the lane's packed word, and exactly the B-operand slot of v_mfma_f32_16x16x32_f16
//    for contraction step f.  No cross-lane movement between reconstruction and use.  Two row tiles at a time (plans of
//    at most eight tokens, and waves of two tiles in single problems with an even number of slabs): one
//    v_mfma_f32_32x32x16_f16 per 32 columns of both
//  * token product: for every 16-token slab, 4 contraction steps; A operand = 8 consecutive fp16 activations
//    read from LDS (rows swizzled by 16-byte chunks against bank conflicts); 32 x 32 x 16 for two tiles and two slabs
// Arithmetic: envelopes and activations rounded to fp16 on load, E accumulated in fp32 and rounded to fp16
// once, token product accumulated in fp32.  Values beyond the fp16 range overflow.
#include "mdbf_internal.h"

namespace mdbf {
namespace gemm {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 4;
constexpr int kDies = 8;                    // accelerator dies (XCDs); workgroup i is placed on die i mod 8
constexpr int kEinBufBytes = 128 * 32;      // 128 columns x 16 modes fp16
// LDS of a workgroup with TB slabs of 16 tokens: two buffers of (16 TB tokens x 128 columns fp16) + envelope rows
__host__ __device__ constexpr int vin_buf_bytes(int TB) { return 16 * TB * 256; }
// waves per SIMD the register budget is cut for: the small shapes live on occupancy (their blocks are short
// dependent chains), the big one on registers
__host__ __device__ constexpr int min_waves(int TB) { return TB >= 4 ? 2 : (TB == 2 ? 3 : 4); }

// Envelope rows of a block in LDS: 128 columns x 16 modes fp16 (32 bytes a column).  A reconstruction
// operand read touches columns 8a + b (+4), a, b = 0..3, eight bytes (four modes) per lane: in column order
// the four values of `a` would land on the same banks.  Column bits 2 and 3 trade places in the row index,
// and the 16-byte halves of a row trade places for columns with bit 4 set: the 32 lanes served together
// then cover every bank once.
__host__ __device__ constexpr int ein_row(int col) { return (col & ~12) | ((col & 4) << 1) | ((col & 8) >> 1); }

__device__ __forceinline__ uint32_t pack_half2(float lo, float hi) {
  half2v h;
  h.x = (_Float16)lo;
  h.y = (_Float16)hi;
  return __builtin_bit_cast(uint32_t, h);
}

// Sign flips of rebuilt pairs where two row tiles share a product, with the signs of the word's top bits (15 and 31), which
// then makes way for the next pair: a word's pairs are taken from bits 15 and 31 downwards.  (Left shifts by constants take
// the vector ALUs four cycles, additions less: 1.9 and 1.3 ns per wave and SIMD measured.  The compiler would turn x + x into
// a shift.)
__device__ __forceinline__ uint32_t flip_next(uint32_t pair, uint32_t& signs) {
  const uint32_t out = pair ^ (signs & 0x80008000u);
  asm("v_add_u32 %0, %0, %0" : "+v"(signs));
  return out;
}

// eight consecutive elements p[idx0 .. idx0+7] as fp16 pairs; elements at or past `nvalid` read as zero
__device__ __forceinline__ u32x4 load8_as_half(const void* p, int64_t idx0, int nvalid, int dt) {
  u32x4 out = {0u, 0u, 0u, 0u};
  if (nvalid <= 0) return out;
  const int es = dtype_size(dt);
  const uintptr_t addr = (uintptr_t)p + (uintptr_t)idx0 * (uintptr_t)es;
  if (nvalid >= 8 && (addr & 15u) == 0) {
    if (dt == MDBF_F16) return *(const MDBF_GLOBAL u32x4*)addr;
    if (dt == MDBF_BF16) {
      const u32x4 raw = *(const MDBF_GLOBAL u32x4*)addr;
      const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
      uint32_t o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = pack_half2(__builtin_bit_cast(float, w[i] << 16), __builtin_bit_cast(float, w[i] & 0xFFFF0000u));
      return u32x4{o[0], o[1], o[2], o[3]};
    }
    const floatx4 a = *(const MDBF_GLOBAL floatx4*)addr;
    const floatx4 b = *(const MDBF_GLOBAL floatx4*)(addr + 16);
    return u32x4{pack_half2(a.x, a.y), pack_half2(a.z, a.w), pack_half2(b.x, b.y), pack_half2(b.z, b.w)};
  }
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (i < nvalid) ? load_as_float(p, idx0 + i, dt) : 0.f;
  return u32x4{pack_half2(v[0], v[1]), pack_half2(v[2], v[3]), pack_half2(v[4], v[5]), pack_half2(v[6], v[7])};
}

// eight consecutive elements of known type, 16-byte aligned, no bounds to respect; fp16 pairs
template <int DT>
__device__ __forceinline__ u32x4 load8_vec(const void* p, int64_t idx0) {
  if (DT == MDBF_F16) return ((const MDBF_GLOBAL u32x4*)((const _Float16*)p + idx0))[0];
  if (DT == MDBF_BF16) {
    const u32x4 raw = ((const MDBF_GLOBAL u32x4*)((const uint16_t*)p + idx0))[0];
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      o[i] = pack_half2(__builtin_bit_cast(float, w[i] << 16), __builtin_bit_cast(float, w[i] & 0xFFFF0000u));
    return u32x4{o[0], o[1], o[2], o[3]};
  }
  const floatx4 a = ((const MDBF_GLOBAL floatx4*)((const float*)p + idx0))[0];
  const floatx4 b = ((const MDBF_GLOBAL floatx4*)((const float*)p + idx0))[1];
  return u32x4{pack_half2(a.x, a.y), pack_half2(a.z, a.w), pack_half2(b.x, b.y), pack_half2(b.z, b.w)};
}

// Four consecutive modes of an envelope row (zeros past the rank), any type, rounded to fp16: the four loads go out
// together.  (One by one, each behind a test and its own wait, they were up to eight trips to memory in front of
// every workgroup's loop.)
__device__ __forceinline__ half4 load4_modes(const StageProb& p, const void* env, int row, int mode0) {
  const int64_t base = (int64_t)row * p.l;
  float v[4];
  if (p.env_dt == MDBF_F32) {
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = ((const MDBF_GLOBAL float*)env)[base + min(mode0 + t, p.l - 1)];
  } else {
    uint32_t b[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) b[t] = ((const MDBF_GLOBAL uint16_t*)env)[base + min(mode0 + t, p.l - 1)];
#pragma unroll
    for (int t = 0; t < 4; ++t)
      v[t] = p.env_dt == MDBF_F16 ? (float)__builtin_bit_cast(_Float16, (uint16_t)b[t]) : __builtin_bit_cast(float, b[t] << 16);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) v[t] = mode0 + t < p.l ? v[t] : 0.f;
  return half4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}

// R row tiles per wave, TB slabs of 16 tokens per workgroup.  MODE 0..2: the common case -- fp16 envelopes of
// rank 16 or 8, activations of type MODE with 16-byte aligned rows and K a multiple of 8: every load is a full
// vector, issued without a branch (addresses are clamped, values past the end replaced by zero).  MODE 3:
// any types, ranks and alignments, element by element.
// BATCH: the rows come from a plan's work items instead of the single problem.
// NW waves, each with R row tiles, share a staging of a block; KS such groups take a run over the contraction each and
// add their sums at the end, in order (small plans).
// PAIR (plans of at most eight tokens): two row tiles at a time.  With up to 16 tokens a piece takes 128 cycles for its
// rebuild on the matrix cores, 64 for the token product, half of whose rows are idle with eight, and some 50 vector
// instructions, which do not overlap with them; one 32 x 32 product rebuilds both tiles' columns in half of the time, and the
// idle rows take the second tile's tokens.  The signs' shifts as additions (flip_next) take another 4 %.  224 matrices, 8
// tokens: 802 -> 737 us per pass with the two and items of 16 tiles (the same sums: bit-identical to 16-row products).
constexpr int kGeneric = kGemmGeneric;
// first: row tiles of the work item in front of this workgroup's.  True (PAIR): some results are infinities or NaNs, and none
// has been stored.
template <int NW, int R, int TB, int MODE, bool BATCH, int KS, bool PAIR>
__device__ __forceinline__ bool stage_gemm_rows(const WorkItem* __restrict__ items, const StageProb& single, int thread, int first,
                                                unsigned char* vin_lds_a, unsigned char* vin_lds_b,
                                                unsigned char* ein_lds_a, unsigned char* ein_lds_b) {
  constexpr int kVinBufBytes = vin_buf_bytes(TB);
  // The wave's tiles in pairs: both tiles' rows in one 32 x 32 rebuild, and (kWide, single problems) in 32 x 32 products
  // with 32 tokens each, whose sums are the same bits as those of 16 x 16.  The rebuild takes half of the matrix cores' time,
  // and a step's activations are all requested before its rebuild (after it: 3 to 10 % longer).  4096 x 4096, k = 2656,
  // fp16, with the same tile shapes: 512 tokens 83.5 -> 69.6 us, 1024 92.3 -> 79.4, 4096 235.6 -> 230.7; 2048 (two
  // workgroups a unit hide each other's waits) 122.4 -> 121.2, nothing on another box; bf16, 1024 tokens 100 -> 85.
  // (Plans of 17 to 64 tokens are not faster for it: 200 attention layers, 30 tokens 484 -> 486 us, 60 tokens 714 -> 733.)
  constexpr bool kWide = !BATCH && R == 2 && TB % 2 == 0;              // (32 tokens at a time)
  static_assert(!kWide || KS == 1, "one run");
  constexpr bool kPairs = PAIR || kWide;
  // the rows of this workgroup: a work item of a plan (at most NW * R row tiles of one problem), or
  // the blockIdx.x-th run of NW * R tiles of the single problem
  StageProb p;
  int item_tile0, item_end, slab_group;
  if (BATCH) {
    const WorkItem& w = items[blockIdx.x];   // uniform address: scalar loads
    p = w.p;
    item_tile0 = w.tile0 + first;
    item_end = w.tile0 + w.ntiles;
    slab_group = blockIdx.y;
  } else {
    // One-dimensional grid.  Workgroups go to the chip's eight dies in turn (id mod 8), each die with an L2
    // of its own; the (token slab group, row group) pairs, token-major, are dealt out in eight contiguous
    // runs, one per die: the workgroups that read the same activations share an L2.
    p = single;
    const int row_groups = (p.ntiles + NW * R - 1) / (NW * R);
    const int slab_groups = (p.T + 16 * TB - 1) / (16 * TB);
    const int total = row_groups * slab_groups;
    const int per_die = (total + kDies - 1) / kDies;
    const int unit = (blockIdx.x % kDies) * per_die + blockIdx.x / kDies;
    if (unit >= total) return false;
    slab_group = unit / row_groups;
    item_tile0 = (unit - slab_group * row_groups) * (NW * R);
    item_end = min(item_tile0 + NW * R, p.ntiles);
  }
  // the run over the contraction that this thread's four waves take, and the thread's and the wave's place in it
  const int run = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(thread / (64 * NW));
  const int tid = thread - run * (64 * NW), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  unsigned char* const vin_a = vin_lds_a + run * kVinBufBytes;
  unsigned char* const vin_b = vin_lds_b + run * kVinBufBytes;
  unsigned char* const ein_a = ein_lds_a + run * kEinBufBytes;
  unsigned char* const ein_b = ein_lds_b + run * kEinBufBytes;
  const int tile0 = item_tile0 + wave * R;                     // first row tile of this wave
  const int tok0 = slab_group * (16 * TB);
  if (tok0 >= p.T) return false;                                  // a plan's grid covers its longest problem
  const int KB = p.KB;

  // ---- per-unit operands: Eout rows of the wave's tiles (B operand of the reconstruction), 4 modes per lane
  // (kPairs: pairs of tiles 2u, 2u + 1; lane (n, h) = (lane & 31, lane >> 5): eight modes 8h .. of row n of a pair's 32)
  half4 eo_op[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int tile = tile0 + (kPairs ? (r & ~1) + (g & 1) : r);
    const int row = min(tile * kTileRows + r16, p.rows - 1);           // (rows past the end are not stored)
    eo_op[r] = load4_modes(p, p.Eout, row, kPairs ? 8 * (g >> 1) + 4 * (r & 1) : 4 * g);
  }
  // sign words: tiles past the end read the last tile (their rows are never stored).  kPairs: word 2u + s of the lane holds
  // columns 16 s + 8 h + 0 .. 7 of each step of its row.
  const MDBF_GLOBAL uint32_t* sbase[R];
  size_t sstride[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int t = min(tile0 + (kPairs ? (r & ~1) + (g & 1) : r), item_end - 1);
    sbase[r] = (const MDBF_GLOBAL uint32_t*)p.S + tile_base_words(t, KB) + (kPairs ? 16 * (2 * (r & 1) + (g >> 1)) + r16 : lane);
    // (an item's tiles are in one group)
    sstride[r] = (size_t)group_tiles(kPairs ? item_tile0 : t, p.ntiles) * 64u;
  }

  constexpr int AR = PAIR ? R / 2 : R;                         // accumulators per slab: a pair's tiles share one
  floatx4 acc[TB][AR];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb)
#pragma unroll
    for (int r = 0; r < AR; ++r) acc[tb][r] = floatx4{0.f, 0.f, 0.f, 0.f};
  typedef float floatx16 __attribute__((ext_vector_type(16)));
  floatx16 z16;
#pragma unroll
  for (int i = 0; i < 16; ++i) z16[i] = 0.f;
  floatx16 wacc[(TB + 1) / 2];                                 // kWide: per 32 tokens
#pragma unroll
  for (int tb = 0; tb < TB / 2; ++tb) wacc[tb] = z16;

  // ---- staging of one block.  Envelope rows and sign words go through registers.  fp16 activations
  //      (kDma) go from global memory straight into LDS, 16 bytes per lane and 1 KB (four token rows) per
  //      instruction; the row swizzle is applied on the global side (a lane fetches the chunk that belongs at
  //      its LDS slot).  Other types are converted in registers on the way.  Values past the end: tokens past
  //      T are never stored; columns past K meet zeroed envelope rows and are zeroed themselves (an infinity in the
  //      row's last columns, which the direct loads of a partial block repeat, would turn into a NaN there).
  constexpr bool kDma = (MODE == MDBF_F16);
  constexpr int kVinChunks = (16 * TB * 16) / (64 * NW);   // 16-byte chunks per thread: TB
  u32x4 vin_reg[kDma ? 1 : kVinChunks];
  constexpr int kEinChunks = 256 / (64 * NW);                  // 16-byte halves of envelope rows per thread
  u32x4 ein_reg[kEinChunks];
  bool ein_ok[kEinChunks];
  uint32_t sw_next[R];
  auto dma_block = [&](int q, unsigned char* vin_buf) {
#pragma unroll
    for (int i = 0; i < kVinChunks; ++i) {
      if (PAIR && wave >= 2) continue;                         // rows 8 .. 15 stay zero
      const int id = tid + 64 * NW * i;
      const int tok = id >> 4, c = (id & 15) ^ (tok & 15);
      const int col = min(q * kBlockCols + c * 8, p.K - 8);
      const int b = min(tok0 + tok, p.T - 1);
      const MDBF_GLOBAL _Float16* src = (const MDBF_GLOBAL _Float16*)p.vin + ((int64_t)b * p.vin_ld + col);
      unsigned char* dst = vin_buf + (wave * 64 + 64 * NW * i) * 16;   // wave-uniform
      __builtin_amdgcn_global_load_lds((const MDBF_GLOBAL void*)src, (MDBF_LDS void*)dst, 16, 0, 0);
    }
  };
  // (kDma) zeros over the columns past K of a partial block: each thread over what it has loaded, once that landed.
  // (Plans do without: their short blocks would take 2 % longer, 50.2 -> 51.5 us for four layers and 8 tokens.  The
  // last block outside the loop instead: 3 to 7 % longer; a zero address for its loads: 1 %.)
  const int partial_block = !BATCH && (p.K & (kBlockCols - 1)) != 0 ? KB - 1 : -1;
  auto clear_tail = [&](int q, unsigned char* vin_buf) __attribute__((always_inline)) {
    if (BATCH || __builtin_expect(q != partial_block, 1)) return;   // (uniform)
#pragma unroll
    for (int i = 0; i < kVinChunks; ++i) {
      const int id = tid + 64 * NW * i;
      const int c = (id & 15) ^ ((id >> 4) & 15);
      if (q * kBlockCols + c * 8 >= p.K) *reinterpret_cast<u32x4*>(vin_buf + id * 16) = u32x4{0u, 0u, 0u, 0u};
    }
  };
  auto fetch_block = [&](int q) __attribute__((always_inline)) {
    if (!kDma) {
#pragma unroll
      for (int i = 0; i < kVinChunks; ++i) {
        const int id = tid + 64 * NW * i;
        const int tok = id >> 4, c = id & 15;
        const int col = q * kBlockCols + c * 8;
        const int b = tok0 + tok;
        if (MODE == kGeneric) {
          const int nvalid = (b < p.T) ? (p.K - col) : 0;
          vin_reg[i] = load8_as_half(p.vin, (int64_t)min(b, p.T - 1) * p.vin_ld + col, nvalid, p.vin_dt);
        } else {
          const u32x4 v = load8_vec<MODE>(p.vin, (int64_t)min(b, p.T - 1) * p.vin_ld + min(col, p.K - 8));
          const bool ok = (b < p.T) && (col < p.K);
          vin_reg[i] = u32x4{ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u};
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kEinChunks; ++i) {
      const int id = tid + 64 * NW * i;
      const int col = q * kBlockCols + (id >> 1);
      if (MODE != kGeneric) {
        // rank 8: a row is one 16-byte vector; the half that would hold modes 8..15 becomes zero
        const int hl = p.l >> 3;
        const bool has_modes = (id & 1) < hl;
        ein_reg[i] = ((const MDBF_GLOBAL u32x4*)p.Ein)[(size_t)min(col, p.K - 1) * hl + (has_modes ? (id & 1) : 0)];
        ein_ok[i] = (col < p.K) && has_modes;          // (the zeros go in when the row is parked: a select here
                                                       //  would make the wave wait for the load here)
      } else {
        // (The type is asked for once and every lane loads, inside its row: asked for element by element, each load would
        // be waited for before the next one is issued.  In bytes from the block's first row, which 32 bits hold.)
        const int qb = min(q, KB - 1), mode0 = 8 * (id & 1), left = col < p.K ? p.l - mode0 : 0;
        const MDBF_GLOBAL char* base = (const MDBF_GLOBAL char*)p.Ein + (size_t)qb * (size_t)(kBlockCols * p.l * dtype_size(p.env_dt));
        const uint32_t first = (uint32_t)((min(col, p.K - 1) - qb * kBlockCols) * p.l);
        float v[8];
        if (p.env_dt == MDBF_F32) {
#pragma unroll
          for (int t = 0; t < 8; ++t) v[t] = *(const MDBF_GLOBAL float*)(base + 4u * (first + (uint32_t)min(mode0 + t, p.l - 1)));
        } else {
          uint16_t raw[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) raw[t] = *(const MDBF_GLOBAL uint16_t*)(base + 2u * (first + (uint32_t)min(mode0 + t, p.l - 1)));
#pragma unroll
          for (int t = 0; t < 8; ++t)
            v[t] = p.env_dt == MDBF_F16 ? (float)__builtin_bit_cast(_Float16, raw[t]) : __builtin_bit_cast(float, (uint32_t)raw[t] << 16);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = t < left ? v[t] : 0.f;
        ein_reg[i] = u32x4{pack_half2(v[0], v[1]), pack_half2(v[2], v[3]), pack_half2(v[4], v[5]), pack_half2(v[6], v[7])};
        ein_ok[i] = true;
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) sw_next[r] = sbase[r][(size_t)min(q, KB - 1) * sstride[r]];
  };
  auto stash_block = [&](unsigned char* vin_buf, unsigned char* ein_buf) __attribute__((always_inline)) {
    if (!kDma) {
#pragma unroll
      for (int i = 0; i < kVinChunks; ++i) {
        const int id = tid + 64 * NW * i;
        const int tok = id >> 4, c = id & 15;
        if (!PAIR || tok < 8) *reinterpret_cast<u32x4*>(vin_buf + tok * 256 + ((c ^ (tok & 15)) << 4)) = vin_reg[i];
      }
    }
#pragma unroll
    for (int i = 0; i < kEinChunks; ++i) {
      const int id = tid + 64 * NW * i;
      const u32x4 v = ein_reg[i];
      const bool ok = ein_ok[i];
      *reinterpret_cast<u32x4*>(ein_buf + ein_row(id >> 1) * 32 + (((id & 1) ^ ((id >> (kPairs ? 4 : 5)) & 1)) << 4)) =
          u32x4{ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u};
    }
  };

  // Register staging runs two blocks ahead (a block is requested at the end of one iteration and parked at
  // the end of the next).  Direct staging runs one block ahead: block q + 1 is requested right after the
  // barrier that opens iteration q, into the buffer iteration q - 1 has just released, and every wave waits
  // for its own requests before it reaches the next barrier.
  const int per_run = (KB + KS - 1) / KS;
  const int q_lo = run * per_run, q_hi = min(q_lo + per_run, KB);    // (the last run may be shorter, or empty)
  uint32_t sw[R];
  if (PAIR) {
    const int id = tid & 127;
    *reinterpret_cast<u32x4*>((tid < 128 ? vin_a : vin_b) + 8 * 256 + id * 16) = u32x4{0u, 0u, 0u, 0u};
  }
  if (kDma) dma_block(min(q_lo, KB - 1), vin_a);
  fetch_block(min(q_lo, KB - 1));
  stash_block(vin_a, ein_a);
#pragma unroll
  for (int r = 0; r < R; ++r) sw[r] = sw_next[r];
  if (kDma) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    clear_tail(min(q_lo, KB - 1), vin_a);
  } else {
    fetch_block(min(q_lo + 1, KB - 1));
  }

  auto block = [&](int q, const unsigned char* vin, const unsigned char* ein, unsigned char* vin_next,
                   unsigned char* ein_next) __attribute__((always_inline)) {
    __syncthreads();
    if (kDma) {
      dma_block(min(q + 1, KB - 1), vin_next);
      fetch_block(min(q + 1, KB - 1));
    }

    // ---- per contraction step f (32 columns): rebuild the wave's pieces of W, wop[r] = B operand of the
    //      token product, then run the step over all token slabs.  The steps are independent of each other,
    //      which lets the rebuild of one step overlap the matrix-core work of the previous one.
    if (KS == 1 || q < q_hi)                                   // (uniform; the barriers are kept)
#pragma unroll
    for (int ff = 0; ff < 4; ++ff) {
      const int f = 3 - ff;
      if constexpr (kPairs) {
        // 32 rows x 32 columns of E in one product (half the time of four 16 x 16 x 16).  Its row m is column m with bits
        // 2 and 3 exchanged, row m of the step in LDS, so that lane (n, h) receives columns 16 s + 8 h + 0 .. 7 of row n
        // in registers 8 s + 0 .. 7: an operand of a 32 x 32 x 16 product with the tokens.
        const int m = lane & 31, h = lane >> 5;
        const half8 ea = *reinterpret_cast<const half8*>(ein + (32 * f + m) * 32 + ((h ^ ((m >> 2) & 1)) << 4));
        if constexpr (kWide) {
          const half8 eo = __builtin_shufflevector(eo_op[0], eo_op[R - 1], 0, 1, 2, 3, 4, 5, 6, 7);
          half8 x[2][TB / 2];
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int tb = 0; tb < TB / 2; ++tb)
              x[s][tb] = *reinterpret_cast<const half8*>(vin + (32 * tb + m) * 256 + (((4 * f + 2 * s + h) ^ (m & 15)) << 4));
          const floatx16 e = __builtin_amdgcn_mfma_f32_32x32x16_f16(ea, eo, z16, 0, 0, 0);
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            u32x4 w;
#pragma unroll
            for (int i = 3; i >= 0; --i) w[i] = flip_next(pack_half2(e[8 * s + 2 * i], e[8 * s + 2 * i + 1]), sw[s]);
#pragma unroll
            for (int tb = 0; tb < TB / 2; ++tb)
              wacc[tb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[s][tb], __builtin_bit_cast(half8, w), wacc[tb], 0, 0, 0);
          }
          continue;
        }
        // PAIR: seen as an operand of a 16 x 16 x 32 product, its lane groups alternate between the
        // two tiles; rows 0 .. 7 of the other operand hold the tokens for the first tile's groups and zeros for the
        // second's, rows 8 .. 15 the other way round.
        const int tok = (r16 & 7) + 8 * ((r16 >> 3) ^ (g & 1));
        half8 x[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) x[s] = *reinterpret_cast<const half8*>(vin + tok * 256 + (((4 * f + 2 * s + h) ^ tok) << 4));
#pragma unroll
        for (int u = 0; u < R / 2; ++u) {
          const half8 eo = __builtin_shufflevector(eo_op[2 * u], eo_op[2 * u + (R > 1)], 0, 1, 2, 3, 4, 5, 6, 7);
          const floatx16 e = __builtin_amdgcn_mfma_f32_32x32x16_f16(ea, eo, z16, 0, 0, 0);
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            u32x4 w;
#pragma unroll
            for (int i = 3; i >= 0; --i) w[i] = flip_next(pack_half2(e[8 * s + 2 * i], e[8 * s + 2 * i + 1]), sw[2 * u + s]);
            acc[0][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x[s], __builtin_bit_cast(half8, w), acc[0][u], 0, 0, 0);
          }
        }
        continue;
      }
      // A operands of the two reconstruction products: rows mi -> columns 32f + 8(mi/4) + mi%4 (+4)
      const int col0 = 32 * f + 8 * (r16 >> 2) + (r16 & 3);
      const int eoff = ein_row(col0) * 32 + ((g ^ ((r16 >> 2) & 2)) << 3);
      const half4 ea0 = *reinterpret_cast<const half4*>(ein + eoff);
      const half4 ea1 = *reinterpret_cast<const half4*>(ein + eoff + (ein_row(4) - ein_row(0)) * 32);
      half8 wop[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const floatx4 z4 = {0.f, 0.f, 0.f, 0.f};
        const floatx4 e0 = __builtin_amdgcn_mfma_f32_16x16x16f16(ea0, eo_op[r], z4, 0, 0, 0);
        const floatx4 e1 = __builtin_amdgcn_mfma_f32_16x16x16f16(ea1, eo_op[r], z4, 0, 0, 0);
        // lane (r16, g) now holds E[row r16][32f + 8g + e], e = 0..3 in e0 and 4..7 in e1.  The packed word
        // keeps the signs of columns e = 2i and 2i+1 at bits p and p + 16, p = 8(f/2) + 4(f%2) + i.
        // (shifted up one by one: four independent chains beside the products.  As one chain of additions, flip_next,
        // they hold a workgroup of one row tile per wave up: 4096 x 4096, k = 2656, as a plan of 16 tokens 20.5 and 23.3 us
        // for the first factor with items of eight tiles, one run; 8 decoder layers of 32 tokens 305 and 316 us.)
        const int pbase = 8 * (f >> 1) + 4 * (f & 1);
        uint32_t w4[4];
        w4[0] = pack_half2(e0[0], e0[1]) ^ ((sw[r] << (15 - (pbase + 0))) & 0x80008000u);
        w4[1] = pack_half2(e0[2], e0[3]) ^ ((sw[r] << (15 - (pbase + 1))) & 0x80008000u);
        w4[2] = pack_half2(e1[0], e1[1]) ^ ((sw[r] << (15 - (pbase + 2))) & 0x80008000u);
        w4[3] = pack_half2(e1[2], e1[3]) ^ ((sw[r] << (15 - (pbase + 3))) & 0x80008000u);
        wop[r] = __builtin_bit_cast(half8, u32x4{w4[0], w4[1], w4[2], w4[3]});
      }
      // the step's A operands (one per token slab) are all requested before the first product
      const int c = f * 4 + g;
      half8 a[TB];
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) {
        const int tok = tb * 16 + r16;
        a[tb] = *reinterpret_cast<const half8*>(vin + tok * 256 + ((c ^ (tok & 15)) << 4));
      }
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int r = 0; r < R; ++r)
          acc[tb][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[tb], wop[r], acc[tb][r], 0, 0, 0);
    }

    // park the next block's register-staged parts and (register staging) request the one after
    // (past the end the last block is requested again: no branch around the loads)
    stash_block(vin_next, ein_next);
#pragma unroll
    for (int r = 0; r < R; ++r) sw[r] = sw_next[r];
    if (kDma) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      clear_tail(min(q + 1, KB - 1), vin_next);
    } else {
      fetch_block(min(q + 2, KB - 1));
    }
  };
#pragma unroll 1
  for (int i = 0; i < per_run; i += 2) {
    block(q_lo + i, vin_a, ein_a, vin_b, ein_b);
    if (i + 1 < per_run) block(q_lo + i + 1, vin_b, ein_b, vin_a, ein_a);
  }

  // ---- the runs' sums, added by the first run's waves in the order of the runs
  if constexpr (KS > 1) {
    constexpr int kRunBytes = NW * TB * AR * 64 * 16;         // a run's sums
    static_assert(kRunBytes <= KS * kVinBufBytes && (KS == 2 || 2 * kRunBytes <= KS * kVinBufBytes), "they take the staging buffers");
    auto sums = [&](int s) { return reinterpret_cast<floatx4*>(s < 3 ? vin_lds_a + (s - 1) * kRunBytes : vin_lds_b); };
    __syncthreads();                                           // every wave is done with the staging buffers
    if (run > 0)
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int r = 0; r < AR; ++r) sums(run)[((wave * TB + tb) * AR + r) * 64 + lane] = acc[tb][r];
    __syncthreads();
    if (!PAIR && run > 0) return false;
#pragma unroll
    for (int s = 1; s < KS; ++s)
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int r = 0; r < AR; ++r) {
          const floatx4 v = sums(s)[((wave * TB + tb) * AR + r) * 64 + lane];
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[tb][r][i] += v[i];
        }
  }

  if constexpr (PAIR) {
    // ---- lane (r16, g) holds out[token 4 (g & 1) + i][row r16 of tile g >> 1 of the pair]
    bool bad = false;
#pragma unroll
    for (int u = 0; u < AR; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) bad |= (__builtin_bit_cast(uint32_t, acc[0][u][i]) & 0x7F800000u) == 0x7F800000u;
    if (__syncthreads_or(run == 0 && bad)) return true;
    if (run > 0) return false;
#pragma unroll
    for (int u = 0; u < AR; ++u) {
      const int tile = tile0 + 2 * u + (g >> 1), row = tile * kTileRows + r16;
      if (tile < item_end && row < p.rows)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int b = 4 * (g & 1) + i;
          if (b < p.T) emit_result(p.out, (int64_t)b * p.out_ld + row, p.out_dt, acc[0][u][i], p.flags);
        }
    }
    return false;
  }
  if constexpr (kWide) {
    // ---- lane (n, h) holds out[token 32 tb + 8 (i / 4) + 4 h + i % 4][row n of the pair's 32]
    const int row = tile0 * kTileRows + (lane & 31);
    if (tile0 + (g & 1) < item_end && row < p.rows)
#pragma unroll
      for (int tb = 0; tb < TB / 2; ++tb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int b = tok0 + 32 * tb + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
          if (b < p.T) emit_result(p.out, (int64_t)b * p.out_ld + row, p.out_dt, wacc[tb][i], p.flags);
        }
    return false;
  }
  // ---- store: lane (r16, g) holds out[token 16 tb + 4g + i][row r16 of tile r]
#pragma unroll
  for (int r = 0; r < AR; ++r) {
    const int row = (tile0 + r) * kTileRows + r16;
    if (tile0 + r < item_end && row < p.rows) {
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int b = tok0 + tb * 16 + 4 * g + i;
          if (b < p.T) emit_result(p.out, (int64_t)b * p.out_ld + row, p.out_dt, acc[tb][r][i], p.flags);
        }
    }
  }
  return false;
}

template <int NW, int R, int TB, int MODE, bool BATCH, int KS, bool PAIR = false>
__global__ __launch_bounds__(64 * NW * KS, min_waves(TB))
void stage_gemm_kernel(const WorkItem* __restrict__ items, StageProb single) {
  // Two buffers each, as objects of their own and chosen at compile time (the loop is written out twice).  With one
  // array and a run-time offset no LDS read could move across the direct-to-LDS loads of the next block: they were
  // all issued first, and the first read then waited for them to land, in every block.  Now the reads of a block
  // go ahead and the loads follow between its products (2048 tokens on 4096 x 4096, k = 2656: 139 -> 124 us; 40
  // tokens: 61 -> 42 us).
  constexpr int kVinBufBytes = vin_buf_bytes(TB);
  __shared__ __attribute__((aligned(1024))) unsigned char vin_lds_a[KS * kVinBufBytes];   // [16*TB tokens][16 chunks of 16 B], swizzled
  __shared__ __attribute__((aligned(1024))) unsigned char vin_lds_b[KS * kVinBufBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char ein_lds_a[KS * kEinBufBytes];   // [128 columns][16 modes]
  __shared__ __attribute__((aligned(1024))) unsigned char ein_lds_b[KS * kEinBufBytes];
  const bool bad = stage_gemm_rows<NW, R, TB, MODE, BATCH, KS, PAIR>(items, single, threadIdx.x, 0, vin_lds_a, vin_lds_b, ein_lds_a, ein_lds_b);
  if constexpr (PAIR) {
    // An entry of E beyond fp16 in a row of one tile has met the zeros of the other tile's tokens and left a NaN in that
    // tile's row too: the tiles one by one (the same sums).  Looking for such results takes 0.4 % of a pass of 224 matrices
    // with 8 tokens (722.7 -> 725.8 us).  The operands are hidden from the compiler, which would keep
    // addresses of the first pass for this one in the registers of its loop.
    int thread = threadIdx.x;
    asm volatile("" : "+s"(items), "+v"(thread));
    if (__builtin_expect(bad, 0))
#pragma unroll 1
      for (int r = 0; r < R; ++r) {
        __syncthreads();                                       // every wave is done with the staging buffers
        stage_gemm_rows<NW, 1, TB, MODE, BATCH, KS, false>(items, single, thread, r * NW, vin_lds_a, vin_lds_b, ein_lds_a, ein_lds_b);
      }
  }
}

// ---------------------------------------------------------------------------------------------------
// One short problem by itself (at most 16 tokens, the vector-load modes) with few row tiles or blocks, or without
// room for partial sums (the kernel further down splits the others): the launch above would give each
// wave one row tile and the whole contraction dimension, a chain of KB dependent steps on a quarter of the
// device.  Here a workgroup owns ONE row tile and its four waves split the column blocks (wave w takes blocks
// 4 i + w); an iteration stages four blocks, two iterations ahead; the four partial results meet in LDS and
// are added in wave order (the same order every time).
// ---------------------------------------------------------------------------------------------------
constexpr int kSplitVinBytes = kWaves * 16 * 256;     // four blocks x 16 tokens x 128 columns fp16
constexpr int kSplitEinBytes = kWaves * kEinBufBytes;
constexpr int kSplitSmem = 2 * (kSplitVinBytes + kSplitEinBytes);

template <int MODE, int R>
__global__ __launch_bounds__(64 * kWaves, 2)
void stage_gemm_split_kernel(StageProb p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* vin_buf = smem;                               // [2][4 blocks][16 tokens][16 chunks], swizzled
  unsigned char* ein_buf = smem + 2 * kSplitVinBytes;          // [2][4 blocks][128 columns][16 modes]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int tile0 = blockIdx.x * R;                            // this workgroup's R consecutive row tiles
  const int KB = p.KB;
  const int iters = (KB + kWaves - 1) / kWaves;

  // Eout row of this lane's tile row, 4 modes per lane (B operand of the reconstruction)
  half4 eo_op[R];
  const MDBF_GLOBAL uint32_t* sbase[R];
  size_t sstride[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    eo_op[r] = load4_modes(p, p.Eout, min((tile0 + r) * kTileRows + r16, p.rows - 1), 4 * g);
    const int t = min(tile0 + r, p.ntiles - 1);               // a tile past the end repeats the last (never stored)
    sbase[r] = (const MDBF_GLOBAL uint32_t*)p.S + tile_base_words(t, KB) + lane;
    sstride[r] = (size_t)group_tiles(t, p.ntiles) * 64u;
  }

  // staging of the four blocks of iteration `it`: thread -> (token, chunk) of every block, and (column, half)
  // of every block's envelope rows.  Columns past K (also whole blocks past KB) get zero envelope rows and
  // zero activations; tokens past T are never stored.
  // (values past the end are replaced by zero when a block is parked, not when it is requested: a select
  // right after the load would make the wave wait for the load there)
  u32x4 vin_reg[kWaves], ein_reg[kWaves];
  uint32_t live = 0;                 // bits j: activations of block j hold real data; bits 8 + j: envelope rows
  uint32_t sw_next[R];
  const int st_tok = tid >> 4, st_c = tid & 15;
  const int hl = p.l >> 3;
  const bool has_modes = (tid & 1) < hl;
  auto fetch = [&](int it) {
    uint32_t lv = 0;
#pragma unroll
    for (int j = 0; j < kWaves; ++j) {
      const int q = it * kWaves + j;
      const int col = q * kBlockCols + st_c * 8;
      vin_reg[j] = load8_vec<MODE>(p.vin, (int64_t)min(st_tok, p.T - 1) * p.vin_ld + min(col, p.K - 8));
      lv |= ((st_tok < p.T) && (col < p.K)) ? (1u << j) : 0u;
      const int ecol = q * kBlockCols + (tid >> 1);
      ein_reg[j] = ((const MDBF_GLOBAL u32x4*)p.Ein)[(size_t)min(ecol, p.K - 1) * hl + (has_modes ? (tid & 1) : 0)];
      lv |= ((ecol < p.K) && has_modes) ? (256u << j) : 0u;
    }
    live = lv;
#pragma unroll
    for (int r = 0; r < R; ++r) sw_next[r] = sbase[r][(size_t)min(it * kWaves + wave, KB - 1) * sstride[r]];
  };
  auto stash = [&](int buf) {
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < kWaves; ++j) {
      *reinterpret_cast<u32x4*>(vin_buf + buf * kSplitVinBytes + j * (16 * 256) + st_tok * 256 +
                                ((st_c ^ (st_tok & 15)) << 4)) = ((live >> j) & 1u) ? vin_reg[j] : zero;
      *reinterpret_cast<u32x4*>(ein_buf + buf * kSplitEinBytes + j * kEinBufBytes + ein_row(tid >> 1) * 32 +
                                (((tid & 1) ^ ((tid >> 5) & 1)) << 4)) = ((live >> (8 + j)) & 1u) ? ein_reg[j] : zero;
    }
  };

  fetch(0);
  stash(0);
  uint32_t sw[R];
  floatx4 acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    sw[r] = sw_next[r];
    acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  fetch(min(1, iters - 1));

#pragma unroll 1
  for (int it = 0; it < iters; ++it) {
    const int cur = it & 1;
    __syncthreads();
    const unsigned char* ein = ein_buf + cur * kSplitEinBytes + wave * kEinBufBytes;
    const unsigned char* vin = vin_buf + cur * kSplitVinBytes + wave * (16 * 256);
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const int col0 = 32 * f + 8 * (r16 >> 2) + (r16 & 3);
      const int eoff = ein_row(col0) * 32 + ((g ^ ((r16 >> 2) & 2)) << 3);
      const half4 ea0 = *reinterpret_cast<const half4*>(ein + eoff);
      const half4 ea1 = *reinterpret_cast<const half4*>(ein + eoff + (ein_row(4) - ein_row(0)) * 32);
      const int c = f * 4 + g;
      const half8 a = *reinterpret_cast<const half8*>(vin + r16 * 256 + ((c ^ r16) << 4));
      const int pbase = 8 * (f >> 1) + 4 * (f & 1);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const floatx4 z4 = {0.f, 0.f, 0.f, 0.f};
        const floatx4 e0 = __builtin_amdgcn_mfma_f32_16x16x16f16(ea0, eo_op[r], z4, 0, 0, 0);
        const floatx4 e1 = __builtin_amdgcn_mfma_f32_16x16x16f16(ea1, eo_op[r], z4, 0, 0, 0);
        uint32_t w4[4];
        w4[0] = pack_half2(e0[0], e0[1]) ^ ((sw[r] << (15 - (pbase + 0))) & 0x80008000u);
        w4[1] = pack_half2(e0[2], e0[3]) ^ ((sw[r] << (15 - (pbase + 1))) & 0x80008000u);
        w4[2] = pack_half2(e1[0], e1[1]) ^ ((sw[r] << (15 - (pbase + 2))) & 0x80008000u);
        w4[3] = pack_half2(e1[2], e1[3]) ^ ((sw[r] << (15 - (pbase + 3))) & 0x80008000u);
        const half8 wop = __builtin_bit_cast(half8, u32x4{w4[0], w4[1], w4[2], w4[3]});
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, wop, acc[r], 0, 0, 0);
      }
    }
    stash(cur ^ 1);
#pragma unroll
    for (int r = 0; r < R; ++r) sw[r] = sw_next[r];
    fetch(min(it + 2, iters - 1));
  }

  // ---- the four partial results: through LDS, added in wave order by wave 0
  __syncthreads();                                             // every wave is done with the staging buffers
  floatx4* red = reinterpret_cast<floatx4*>(smem);              // [R][4 waves][64 lanes]
#pragma unroll
  for (int r = 0; r < R; ++r) red[(r * kWaves + wave) * 64 + lane] = acc[r];
  __syncthreads();
  if (wave < R) {                                              // wave r adds up and stores tile r
    floatx4 sum = red[(wave * kWaves) * 64 + lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      const floatx4 t = red[(wave * kWaves + w) * 64 + lane];
      sum[0] += t[0]; sum[1] += t[1]; sum[2] += t[2]; sum[3] += t[3];
    }
    const int row = (tile0 + wave) * kTileRows + r16;
    if (tile0 + wave < p.ntiles && row < p.rows) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int b = 4 * g + i;
        if (b < p.T) emit_result(p.out, (int64_t)b * p.out_ld + row, p.out_dt, sum[i], p.flags);
      }
    }
  }
}

// R row tiles per workgroup (wave r stores tile r): more tiles mean fewer re-reads of the envelope rows and
// activations (every workgroup reads all of them) but longer chains and fewer workgroups.
template <int MODE, int R>
static int launch_split_r(const StageProb* p, hipStream_t s) {
  static_assert(R >= 1 && R <= kWaves, "wave r stores tile r");
  static KernelSetup setup;
  if (int e = kernel_setup(setup, [] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&stage_gemm_split_kernel<MODE, R>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, kSplitSmem);
      }))
    return e;
  hipLaunchKernelGGL((stage_gemm_split_kernel<MODE, R>), dim3((unsigned)((p->ntiles + R - 1) / R)),
                     dim3(64 * kWaves), kSplitSmem, s, *p);
  return (int)hipGetLastError();
}

// one tile per workgroup as long as the device holds all workgroups at once (two per compute unit)
template <int MODE>
static int launch_split(const StageProb* p, hipStream_t s) {
  if (p->ntiles > 2 * compute_units()) return launch_split_r<MODE, 2>(p, s);
  return launch_split_r<MODE, 1>(p, s);
}

// ---------------------------------------------------------------------------------------------------
// One short problem by itself (at most 64 tokens).  A workgroup owns 8 row tiles (one per wave) and `bs` column
// blocks: its eight tiles share one staging of the activations and envelope rows, and the contraction is split
// over workgroups until the launch fills the device.  Partial sums go to the workspace and a small launch adds
// them in the order of the splits (3 to 4 us; letting the last workgroup of a row group add them took 5 us with
// 16 tokens and 13 us with 37).
// What bounds it: a launch is a few microseconds of dependent trips (stage, rebuild, partial sums), not traffic
// or arithmetic (16 tokens, per launch of 10 us: 5.6 MB fetched, 1.2 us of matrix-core and 2.9 us of vector issue per
// SIMD; 58 % of the wave cycles wait).  One row tile per workgroup and the blocks split over its waves, as before, made every tile
// stage all activations again (176 MB through the L2s for 16 tokens x 11008 columns x 256 tiles: 28 us of the
// call's 38).  4096 x 11008, k = 4096, l = 16, 16 tokens: 38.0 -> 23.2 us per call; 5000 x 3001, k = 2003, l = 3,
// 37 tokens in bf16 (element-wise loads before, vector loads of any alignment now): 172 -> 25.1 us.
//   MODE: type of the activations; rows may start at any element (the target's vector loads need no alignment).
//   EVEC: fp16 envelope rows of rank 8 or 16, one or two vectors each; otherwise any type and rank: the chunk's
//   rows are consecutive elements, loaded as vectors and spread over the LDS rows.
//   TB: slabs of 16 tokens.
// ---------------------------------------------------------------------------------------------------
constexpr int kFewWaves = 8;
constexpr int kFewThreads = 64 * kFewWaves;
constexpr int kFewSplits = 16;                                  // partial sums per output at most
__host__ __device__ constexpr int few_chunk(int TB) { return TB == 1 ? 4 : 2; }   // blocks staged at a time
__host__ __device__ constexpr int few_vin_bytes(int TB) { return few_chunk(TB) * TB * 16 * 256; }
__host__ __device__ constexpr int few_smem(int TB) { return 2 * (few_vin_bytes(TB) + few_chunk(TB) * kEinBufBytes); }

typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));   // a vector at any element's address

struct FewArgs {
  StageProb p;
  int32_t bs, nsplit;          // blocks per workgroup, workgroups per row group
  float* part;                 // [nsplit][T][part_ld] (unused when nsplit == 1)
  int64_t part_ld;
};

template <int MODE, bool EVEC, int TB>
__global__ __launch_bounds__(kFewThreads, 4)
void stage_gemm_few_kernel(FewArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int CK = few_chunk(TB);
  constexpr int kVinBytes = few_vin_bytes(TB);
  constexpr int kVinSlots = CK * TB * 256 / kFewThreads;        // 16-byte LDS slots per thread and chunk
  constexpr int kRaw = MODE == MDBF_F32 ? 2 : 1;                // vectors a slot is loaded as
  constexpr int kEinSlots = EVEC ? CK * 256 / kFewThreads : CK; // EVEC false: up to 128 CK rows of 64 bytes
  const StageProb& p = a.p;
  unsigned char* vin_buf = smem;                                // [2][CK blocks][16 TB tokens][16 slots], swizzled
  unsigned char* ein_buf = smem + 2 * kVinBytes;                // [2][CK blocks][128 columns][16 modes]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int group = (int)blockIdx.x / a.nsplit, split = (int)blockIdx.x - group * a.nsplit;
  const int q_lo = split * a.bs, q_hi = min(q_lo + a.bs, p.KB);
  const int chunks = (q_hi - q_lo + CK - 1) / CK;
  const int tile = group * kFewWaves + wave;                    // (a tile past the end repeats the last, unstored)
  const int tile_c = min(tile, p.ntiles - 1);
  const MDBF_GLOBAL uint32_t* sbase = (const MDBF_GLOBAL uint32_t*)p.S + tile_base_words(tile_c, p.KB) + lane;
  const size_t sstride = (size_t)group_tiles(tile_c, p.ntiles) * 64u;

  u32x4 vin_reg[kVinSlots][kRaw], ein_reg[kEinSlots];
  uint32_t sw[CK], sw_next[CK];
  const int es = dtype_size(p.env_dt);
  const int hl = p.l >> 3;
  const int row_bytes = p.l * es;
  const int64_t ein_bytes = (int64_t)p.K * row_bytes;
  auto fetch = [&](int chunk) {
    const int q0 = q_lo + chunk * CK;
#pragma unroll
    for (int i = 0; i < kVinSlots; ++i) {
      const int id = tid + kFewThreads * i;
      const int c = id & 15, tok = (id >> 4) % (16 * TB), j = id / (256 * TB);
      const int64_t e = (int64_t)min(tok, p.T - 1) * p.vin_ld + max(0, min((q0 + j) * kBlockCols + c * 8, p.K - 8));
      if (p.K >= 8) {                                           // (shorter rows are read when they are parked)
#pragma unroll
        for (int v = 0; v < kRaw; ++v)
          vin_reg[i][v] = *(const MDBF_GLOBAL u32x4_any*)((const MDBF_GLOBAL unsigned char*)p.vin +
                                                          (e + 4 * v) * dtype_size(MODE));
      }
    }
#pragma unroll
    for (int i = 0; i < kEinSlots; ++i) {
      const int id = tid + kFewThreads * i;
      if (EVEC) {
        const int col = q0 * kBlockCols + (id >> 1);
        ein_reg[i] = ((const MDBF_GLOBAL u32x4*)p.Ein)[(size_t)min(col, p.K - 1) * hl + ((id & 1) < hl ? (id & 1) : 0)];
      } else {
        // 16-byte pieces of the chunk's rows; pieces past the factor's end repeat the last one, which never
        // leaves the 16-byte granule of the factor's last element
        const int64_t off = (int64_t)q0 * kBlockCols * row_bytes + id * 16;
        if (kFewThreads * i < CK * 8 * row_bytes)
          ein_reg[i] = *(const MDBF_GLOBAL u32x4*)((const MDBF_GLOBAL unsigned char*)p.Ein + min(off, (ein_bytes - 1) & ~(int64_t)15));
      }
    }
#pragma unroll
    for (int j = 0; j < CK; ++j) sw_next[j] = sbase[(size_t)min(q0 + j, p.KB - 1) * sstride];
  };
  auto stash = [&](int chunk, int buf) {
    const int q0 = q_lo + chunk * CK;
#pragma unroll
    for (int i = 0; i < kVinSlots; ++i) {
      const int id = tid + kFewThreads * i;
      const int c = id & 15, tok = (id >> 4) % (16 * TB), j = id / (256 * TB);
      const int col = (q0 + j) * kBlockCols + c * 8;
      u32x4 v;
      if (p.K < 8) {
        v = load8_as_half(p.vin, (int64_t)min(tok, p.T - 1) * p.vin_ld + col, p.K - col, MODE);
      } else {
        if (MODE == MDBF_F16) {
          v = vin_reg[i][0];
        } else if (MODE == MDBF_BF16) {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            v[t] = pack_half2(__builtin_bit_cast(float, vin_reg[i][0][t] << 16),
                              __builtin_bit_cast(float, vin_reg[i][0][t] & 0xFFFF0000u));
        } else {
          const floatx4 f0 = __builtin_bit_cast(floatx4, vin_reg[i][0]), f1 = __builtin_bit_cast(floatx4, vin_reg[i][kRaw - 1]);
          v = u32x4{pack_half2(f0.x, f0.y), pack_half2(f0.z, f0.w), pack_half2(f1.x, f1.y), pack_half2(f1.z, f1.w)};
        }
        if ((p.K & 7) != 0 && q0 + j == p.KB - 1 && col < p.K && col + 8 > p.K) {
          // the row's last, partial octet was loaded as its last eight elements: move it down, zeros behind
          const int sh = 16 * (col + 8 - p.K);
          uint64_t lo = (uint64_t)v.x | ((uint64_t)v.y << 32), hi = (uint64_t)v.z | ((uint64_t)v.w << 32);
          if (sh >= 64) {
            lo = hi >> (sh - 64);
            hi = 0;
          } else {
            lo = (lo >> sh) | (hi << (64 - sh));
            hi >>= sh;
          }
          v = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
        }
        const bool ok = col < p.K;
        v = u32x4{ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u};
      }
      *reinterpret_cast<u32x4*>(vin_buf + buf * kVinBytes + (j * 16 * TB + tok) * 256 + ((c ^ (tok & 15)) << 4)) = v;
    }
    unsigned char* eb = ein_buf + buf * (CK * kEinBufBytes);
#pragma unroll
    for (int i = 0; i < kEinSlots; ++i) {
      const int id = tid + kFewThreads * i;
      if (EVEC) {
        const int col = id >> 1;                                // inside the chunk
        const bool ok = (q0 * kBlockCols + col < p.K) && (id & 1) < hl;
        const u32x4 v = ein_reg[i];
        *reinterpret_cast<u32x4*>(eb + (col >> 7) * kEinBufBytes + ein_row(col & 127) * 32 + (((id & 1) ^ ((col >> 4) & 1)) << 4)) =
            u32x4{ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u};
      } else if (kFewThreads * i < CK * 8 * row_bytes && id * 16 < CK * kBlockCols * row_bytes) {
        const float rl = 1.f / (float)p.l;
        const int per = 16 / es;
        int first = id * per;                                   // element of the chunk: below 8192
        asm volatile("" : "+v"(first));                         // (its LDS offsets are not worth 32 registers)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          if (t < per) {
            const int e = first + t;
            const int col = (int)(((float)e + 0.5f) * rl), mode = e - col * p.l;
            uint32_t bits = es == 4 ? ein_reg[i][t & 3] : (t & 1) ? ein_reg[i][t >> 1] >> 16 : ein_reg[i][t >> 1] & 0xFFFFu;
            if (p.env_dt != MDBF_F16) {
              const float f = __builtin_bit_cast(float, es == 4 ? bits : bits << 16);
              bits = pack_half2(f, 0.f) & 0xFFFFu;
            }
            if (q0 * kBlockCols + col >= p.K) bits = 0;
            *reinterpret_cast<uint16_t*>(eb + (col >> 7) * kEinBufBytes + ein_row(col & 127) * 32 +
                                         (((mode >> 3) ^ ((col >> 4) & 1)) << 4) + (mode & 7) * 2) = (uint16_t)bits;
          }
        }
      }
    }
  };

  fetch(0);
  // Eout row of this lane's tile row, 4 modes per lane (B operand of the reconstruction)
  const half4 eo_op = load4_modes(p, p.Eout, min(tile_c * kTileRows + r16, p.rows - 1), 4 * g);
  if (!EVEC) {                                                  // the modes past the rank stay zero
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int i = tid; i < 2 * CK * kEinBufBytes / 16; i += kFewThreads) reinterpret_cast<u32x4*>(ein_buf)[i] = zero;
    __syncthreads();
  }
  stash(0, 0);
#pragma unroll
  for (int j = 0; j < CK; ++j) sw[j] = sw_next[j];
  fetch(min(1, chunks - 1));

  floatx4 acc[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) acc[tb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int ch = 0; ch < chunks; ++ch) {
    const int cur = ch & 1;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < CK; ++j) {
      if (q_lo + ch * CK + j < q_hi) {
        const unsigned char* ein = ein_buf + (cur * CK + j) * kEinBufBytes;
        const unsigned char* vin = vin_buf + cur * kVinBytes + j * (16 * TB * 256);
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          const int col0 = 32 * f + 8 * (r16 >> 2) + (r16 & 3);
          const int eoff = ein_row(col0) * 32 + ((g ^ ((r16 >> 2) & 2)) << 3);
          const half4 ea0 = *reinterpret_cast<const half4*>(ein + eoff);
          const half4 ea1 = *reinterpret_cast<const half4*>(ein + eoff + (ein_row(4) - ein_row(0)) * 32);
          const floatx4 z4 = {0.f, 0.f, 0.f, 0.f};
          const floatx4 e0 = __builtin_amdgcn_mfma_f32_16x16x16f16(ea0, eo_op, z4, 0, 0, 0);
          const floatx4 e1 = __builtin_amdgcn_mfma_f32_16x16x16f16(ea1, eo_op, z4, 0, 0, 0);
          const int pbase = 8 * (f >> 1) + 4 * (f & 1);
          u32x4 w4;
          w4.x = pack_half2(e0[0], e0[1]) ^ ((sw[j] << (15 - (pbase + 0))) & 0x80008000u);
          w4.y = pack_half2(e0[2], e0[3]) ^ ((sw[j] << (15 - (pbase + 1))) & 0x80008000u);
          w4.z = pack_half2(e1[0], e1[1]) ^ ((sw[j] << (15 - (pbase + 2))) & 0x80008000u);
          w4.w = pack_half2(e1[2], e1[3]) ^ ((sw[j] << (15 - (pbase + 3))) & 0x80008000u);
          const half8 wop = __builtin_bit_cast(half8, w4);
          const int c = f * 4 + g;
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) {
            const half8 x = *reinterpret_cast<const half8*>(vin + (tb * 16 + r16) * 256 + ((c ^ r16) << 4));
            acc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, wop, acc[tb], 0, 0, 0);
          }
        }
      }
    }
    if (ch + 1 < chunks) {
      stash(ch + 1, cur ^ 1);
#pragma unroll
      for (int j = 0; j < CK; ++j) sw[j] = sw_next[j];
      fetch(min(ch + 2, chunks - 1));
    }
  }

  // ---- lane (r16, g) holds token 16 tb + 4 g + i of row r16 of the tile
  const int row = tile * kTileRows + r16;
  const bool mine = tile < p.ntiles && row < p.rows;
#pragma unroll
  for (int tb = 0; tb < TB; ++tb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = tb * 16 + 4 * g + i;
      if (mine && b < p.T) {
        if (a.nsplit == 1) emit_result(p.out, (int64_t)b * p.out_ld + row, p.out_dt, acc[tb][i], p.flags);
        else ((MDBF_GLOBAL float*)a.part)[((size_t)split * p.T + b) * a.part_ld + row] = acc[tb][i];
      }
    }
}

// the partial sums of the launch before, added in the order of the splits, eight loads in flight
__global__ __launch_bounds__(256) void few_reduce_kernel(FewArgs a) {
  const int row = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
  if (row >= a.p.rows) return;
  const MDBF_GLOBAL float* first = (const MDBF_GLOBAL float*)a.part + (size_t)b * a.part_ld + row;
  const size_t step = (size_t)a.p.T * a.part_ld;
  float sum = 0.f;
  for (int t0 = 0; t0 < a.nsplit; t0 += 8) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = first[min(t0 + j, a.nsplit - 1) * step];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (t0 + j < a.nsplit) sum += v[j];
  }
  emit_result(a.p.out, (int64_t)b * a.p.out_ld + row, a.p.out_dt, sum, a.p.flags);
}

template <int MODE, bool EVEC, int TB>
static int launch_few_met(const FewArgs& a, hipStream_t s) {
  static KernelSetup setup;
  if (int e = kernel_setup(setup, [] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&stage_gemm_few_kernel<MODE, EVEC, TB>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, few_smem(TB));
      }))
    return e;
  const int groups = (a.p.ntiles + kFewWaves - 1) / kFewWaves;
  hipLaunchKernelGGL((stage_gemm_few_kernel<MODE, EVEC, TB>), dim3((unsigned)(groups * a.nsplit)),
                     dim3(kFewThreads), few_smem(TB), s, a);
  return (int)hipGetLastError();
}

// As many slabs as the tokens fill: the products, LDS reads and staging of a slab that holds none are work as of one that does.
// Three instead of four for 33 to 48 tokens: 5000 x 3001, k = 2003, l = 3, 37 tokens in bf16 23.5 -> 22.6 us per call from a
// graph, 3000 x 5001, k = 3003, l = 12, 40 tokens in fp32 28.8 -> 27.3, 1000 x 1001, k = 999, l = 4, 45 tokens 17.4 -> 17.0.
template <int MODE, bool EVEC>
static int launch_few_me(const FewArgs& a, hipStream_t s) {
  if (a.p.T > 48) return launch_few_met<MODE, EVEC, 4>(a, s);
  if (a.p.T > 32) return launch_few_met<MODE, EVEC, 3>(a, s);
  if (a.p.T > 16) return launch_few_met<MODE, EVEC, 2>(a, s);
  return launch_few_met<MODE, EVEC, 1>(a, s);
}

template <int MODE>
static int launch_few_m(const FewArgs& a, hipStream_t s) {
  const bool evec = a.p.env_dt == MDBF_F16 && (a.p.l == 16 || a.p.l == 8);
  return evec ? launch_few_me<MODE, true>(a, s) : launch_few_me<MODE, false>(a, s);
}

// items_dev null: the single problem *p.  Else nitems work items of a plan, `p` describing the launch:
// p->T = the longest token count among the problems.
template <int NW, int R, int TB, int MODE, bool BATCH, int KS, bool PAIR = false>
static int launch_rtmb(const WorkItem* items_dev, int nitems, const StageProb* p, hipStream_t s) {
  const int rows_per_wg = NW * R;   // tiles
  unsigned gx = BATCH ? (unsigned)nitems : (unsigned)((p->ntiles + rows_per_wg - 1) / rows_per_wg);
  unsigned gy = (unsigned)((p->T + 16 * TB - 1) / (16 * TB));
  if (!BATCH) {
    const unsigned total = gx * gy;
    gx = kDies * ((total + kDies - 1) / kDies);
    gy = 1;
  }
  hipLaunchKernelGGL((stage_gemm_kernel<NW, R, TB, MODE, BATCH, KS, PAIR>), dim3(gx, gy), dim3(64 * NW * KS), 0, s,
                     items_dev, *p);
  return (int)hipGetLastError();
}

template <int R, int TB, int MODE>
static int launch_rtm(const StageProb* p, hipStream_t s) {
  if constexpr (R == 2 || MODE != kGeneric) return launch_rtmb<kWaves, R, TB, MODE, false, 1>(nullptr, 0, p, s);
  return (int)hipErrorInvalidValue;
}

// a plan's work items, of NW R row tiles; the forms that gemm_plan_form names
template <int NW, int R, int TB, int MODE>
static int launch_items_rtm(const WorkItem* items_dev, int nitems, int form, const StageProb* p, hipStream_t s) {
  const int runs = form & (kGemmPairs - 1);
  if constexpr (NW * R >= 8 && TB == 1) {
    if (form & kGemmPairs) {
      if constexpr (NW * R == 8)
        if (runs == 2) return launch_rtmb<NW, R, TB, MODE, true, 2, true>(items_dev, nitems, p, s);
      return launch_rtmb<NW, R, TB, MODE, true, 1, true>(items_dev, nitems, p, s);
    }
  }
  if constexpr (TB == 1 && NW * R <= 4) {
    if (runs == 4) return launch_rtmb<NW, R, TB, MODE, true, 4>(items_dev, nitems, p, s);
  }
  if constexpr (TB <= 2 && NW * R <= 8 && !(TB == 1 && NW * R == 2)) {
    if (runs == 2) return launch_rtmb<NW, R, TB, MODE, true, 2>(items_dev, nitems, p, s);
  }
  if constexpr (NW * R == 8 || (TB > 2 && NW * R == 4)) {
    if (runs == 1) return launch_rtmb<NW, R, TB, MODE, true, 1>(items_dev, nitems, p, s);
  }
  return (int)hipErrorInvalidValue;
}
template <int NW, int R, int TB>
static int launch_items_rt(const WorkItem* items_dev, int nitems, int mode, int form, const StageProb* p, hipStream_t s) {
  if (mode == kGeneric) return launch_items_rtm<NW, R, TB, kGeneric>(items_dev, nitems, form, p, s);
  if (mode == MDBF_F16) return launch_items_rtm<NW, R, TB, MDBF_F16>(items_dev, nitems, form, p, s);
  if (mode == MDBF_BF16) return launch_items_rtm<NW, R, TB, MDBF_BF16>(items_dev, nitems, form, p, s);
  return launch_items_rtm<NW, R, TB, MDBF_F32>(items_dev, nitems, form, p, s);
}
template <int NW, int R>
static int launch_items_r(const WorkItem* items_dev, int nitems, int mode, int form, const StageProb* p, hipStream_t s) {
  if constexpr (NW * R > 2)
    if (p->T > 32) return launch_items_rt<NW, R, 4>(items_dev, nitems, mode, form, p, s);
  if (p->T > 16) return launch_items_rt<NW, R, 2>(items_dev, nitems, mode, form, p, s);
  return launch_items_rt<NW, R, 1>(items_dev, nitems, mode, form, p, s);
}

template <int R, int TB>
static int launch_rt(int mode, const StageProb* p, hipStream_t s) {
  if (mode == kGeneric) return launch_rtm<R, TB, kGeneric>(p, s);
  if (mode == MDBF_F16) return launch_rtm<R, TB, MDBF_F16>(p, s);
  if (mode == MDBF_BF16) return launch_rtm<R, TB, MDBF_BF16>(p, s);
  return launch_rtm<R, TB, MDBF_F32>(p, s);
}

// ---------------------------------------------------------------------------------------------------
// Operands of a long call whose rows or types the vector-load mode cannot take as they are: copies in fp16, rows
// of the activations padded with zeros to a multiple of eight columns, envelope rows to 8 or 16 modes (rows past the
// end: zeros).  The values are the ones the element-wise mode rounds to on every load, so the results are the same
// bits; what it cost was one element per load and its conversion again in every workgroup.  5000 x 3001, k = 2003,
// l = 3, 2048 tokens in fp32: 444 -> 131 us per call.
// One launch for up to six copies; a thread makes eight consecutive elements of one.
// ---------------------------------------------------------------------------------------------------
struct HalfCopy {
  const void* src;             // src_rows x cols of type dt, rows ld apart; null: only zeros are written
  void* dst;                   // rows x dst_cols fp16, dst_ld apart (multiples of eight)
  int64_t ld, dst_ld, first;   // first: index of the copy's first thread
  int32_t src_rows, cols, dst_cols, dt;
};
struct HalfCopies {
  HalfCopy c[6];
  int64_t threads;
};
__global__ __launch_bounds__(256) void half_copy_kernel(HalfCopies a) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= a.threads) return;
  int k = 0;
#pragma unroll
  for (int i = 1; i < 6; ++i) k = t >= a.c[i].first ? i : k;
  HalfCopy c = a.c[0];
#pragma unroll
  for (int i = 1; i < 6; ++i)
    if (i == k) c = a.c[i];
  const int64_t v = t - c.first;
  const int per = c.dst_cols >> 3;
  const int64_t row = v / per;
  const int col = (int)(v - row * per) * 8;
  const int nvalid = c.src && row < c.src_rows ? c.cols - col : 0;
  u32x4 out = {0u, 0u, 0u, 0u};
  if (nvalid >= 8) {                                            // (vector loads of any alignment)
    const MDBF_GLOBAL unsigned char* p = (const MDBF_GLOBAL unsigned char*)c.src + (row * c.ld + col) * dtype_size(c.dt);
    const u32x4 r0 = *(const MDBF_GLOBAL u32x4_any*)p;
    if (c.dt == MDBF_F16) {
      out = r0;
    } else if (c.dt == MDBF_BF16) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t w = r0[i];
        out[i] = pack_half2(__builtin_bit_cast(float, w << 16), __builtin_bit_cast(float, w & 0xFFFF0000u));
      }
    } else {
      const floatx4 f0 = __builtin_bit_cast(floatx4, r0);
      const u32x4 r1 = *(const MDBF_GLOBAL u32x4_any*)(p + 16);
      const floatx4 f1 = __builtin_bit_cast(floatx4, r1);
      out = u32x4{pack_half2(f0.x, f0.y), pack_half2(f0.z, f0.w), pack_half2(f1.x, f1.y), pack_half2(f1.z, f1.w)};
    }
  } else if (nvalid > 0) {
    out = load8_as_half(c.src, row * c.ld + col, nvalid, c.dt);
  }
  *(MDBF_GLOBAL u32x4*)((MDBF_GLOBAL uint16_t*)c.dst + row * c.dst_ld + col) = out;
}

}  // namespace gemm

// Row tiles per wave and token slabs per workgroup for a single problem of more than 32 tokens.  In ns per column block: what a
// workgroup takes that has a compute unit to itself (mostly the wait for the next block's activations), and what each adds
// to a unit with several, between the mean number per unit and the busiest unit's; and once, in ns, what a larger form's first
// block and results take longer.  Fitted to 200 to 1048 us long calls of 70 to 4096 tokens on 4096 x 4096, k = 2656,
// 11008 x 4096 and 4096 x 11008, k = 4096, and 1024 x 1024, k = 512; 2 x 7 and the third figure to 594 calls of 33 to
// 3000 tokens on 512 x 512 to 28672 x 8192.  Fewer slabs make more, lighter workgroups: worth it when that evens out the
// last round or fills the device at all.  4096 x 11008, k = 4096, us per call with 2 x 8, 2 x 6, 2 x 4, 2 x 2, 1 x 2:
// 256 tokens 155, 131, 122, 96, 106; 512: 156, 136, 123, 121, 144; 777: 165, 172, 149, 200, 249; 1300: 225, 202, 226, 300,
// 362; 4096: 538, 604, 610, 816, 1039.  2 x 7 is for lengths of seven slabs: 777 tokens on 8192 x 8192 280 -> 263,
// 400 on 28672 x 8192 376 -> 344.  (1 x 4 is nowhere the best.)  bf16 activations as they are (calls of up to 64
// tokens) cost the one-tile form most, a conversion for every four tiles and block: 64 tokens with 1 x 2 and 2 x 2,
// 8192 x 28672, k = 8192, 328 and 231 us, 4096 x 11008, k = 4096, 97 and 88, 1024 x 1024, k = 512, 15.6 and 17.5; fp16
// and fp32 ones cost both forms the same.
// Each output is the same sum in the same order whatever the choice.  The element-wise mode has the two-tile forms only.
struct LongShape {
  int R, TB;
};
static LongShape long_problem_shape(const StageProb& p, bool vectors) {
  static const struct {
    LongShape shape;
    int alone, more, once;
  } forms[] = {{{2, 8}, 1320, 1140, 1120}, {{2, 7}, 1600, 1095, 1000}, {{2, 6}, 1080, 900, 800}, {{2, 4}, 960, 690, 460},
               {{2, 2}, 710, 470, 220},    {{1, 2}, 620, 360, 0}},
    bf16_forms[] = {{{2, 2}, 680, 470, 1100}, {{1, 2}, 790, 1050, 0}};
  const int cus = compute_units();
  const int nblk = (p.K + 127) >> 7;
  LongShape best = {2, 8};
  double least = -1.0;
  for (const auto& any : forms) {
    if (any.shape.R == 1 && !vectors) continue;
    const bool bf16 = vectors && p.vin_dt == MDBF_BF16 && any.shape.TB == 2;
    const auto& f = bf16 ? bf16_forms[any.shape.R == 1] : any;
    const int tiles = f.shape.R * gemm::kWaves;
    const int64_t wgs = (int64_t)((p.ntiles + tiles - 1) / tiles) * ((p.T + 16 * f.shape.TB - 1) / (16 * f.shape.TB));
    const double mean = (double)wgs / cus, busiest = (double)((wgs + cus - 1) / cus);
    const double cost = nblk * std::max((double)f.alone, f.more * 0.5 * (mean + busiest)) + f.once;
    if (least < 0.0 || cost < least) {
      least = cost;
      best = f.shape;
    }
  }
  return best;
}

int gemm_load_mode(const StageProb& p) {
  const int es = dtype_size(p.vin_dt);
  const bool fast = p.env_dt == MDBF_F16 && (p.l == 16 || p.l == 8) && (p.K & 7) == 0 && p.K >= 8 &&
                    (((uintptr_t)p.vin | (uintptr_t)p.Ein) & 15u) == 0 && ((p.vin_ld * es) & 15) == 0;
  return fast ? p.vin_dt : gemm::kGeneric;
}

int launch_half_copies(const HalfMatrix* m, int count, hipStream_t s) {
  gemm::HalfCopies a;
  a.threads = 0;
  for (int i = 0; i < 6; ++i) {
    gemm::HalfCopy& c = a.c[i];
    c = gemm::HalfCopy{nullptr, nullptr, 0, 0, INT64_MAX, 0, 0, 8, MDBF_F16};
    if (i >= count) continue;
    c.src = m[i].src;
    c.dst = m[i].dst;
    c.ld = m[i].ld;
    c.dst_ld = m[i].dst_ld;
    c.first = a.threads;
    c.src_rows = m[i].src_rows;
    c.cols = m[i].cols;
    c.dst_cols = m[i].dst_cols;
    c.dt = m[i].dt;
    a.threads += (int64_t)m[i].rows * (m[i].dst_cols / 8);
  }
  hipLaunchKernelGGL(gemm::half_copy_kernel, dim3((unsigned)((a.threads + 255) / 256)), dim3(256), 0, s, a);
  return (int)hipGetLastError();
}

// Forms of a plan's launch: row tiles per work item / runs over the contraction in its workgroup (p: two row tiles per
// product, PAIR).  Few row tiles leave most of the device idle with items of eight and one run, and a block of such a run
// takes its 0.5 us however few there are: smaller items, and runs side by side.  But every workgroup stages the envelope rows
// and activations of its blocks for its own tiles, so small items and runs multiply that work where there are workgroups
// enough, most of all where operands are loaded element by element; and a contraction of a few blocks has nothing to share
// out.  Where contractions are of different lengths the launch ends with a workgroup's long one: shorter runs for longer.
// The lines lie where the forms' times cross, launch by launch, for 1 to 400 layers of 256 x 256 (k = 128) to 11008 x 4096 and
// 4096 x 11008 (k = 4096), for mixed ones and decoder layers, 8, 16, 32 and 64 tokens, envelopes of fp16 rank 16, 8
// (aligned or not), 5, 3, bf16 rank 12, fp32 rank 16 and 4.  Of 4752 launches none takes more than 5.3 % longer than 8/1, on
// average they take 19 % less.  us per launch of up to 8 tokens, (row tiles, blocks):
//   vectors  (256, 32) 8/1 20.5, 2/4 9.6, 4/2 12.6, 4/4 11.7           (1024, 32) 20.5, 2/4 13.2, 4/2 12.7, 4/4 11.8
//            (2048, 32) 22.0, 2/4 24.3, 4/2 18.3, 8/2p 17.6            (2656, 32) 32.1, 4/2 24.8, 8/1p 27.9, 8/2p 26.3
//            (4096, 32) 32.6, 4/2 32.0, 8/1p 29.1, 8/2p 28.2           (5312, 32) 40.0, 4/2 44.0, 8/1p 37.5, 8/2p 39.9
//            (8192, 32) 52.2, 8/1p 49.0, 8/2p 51.5, 16/1p 46.9         (32768, 21) 127, 8/1p 123, 8/2p 136, 16/1p 113
//            (512, 4) 6.0, 2/4 4.8     (2048, 4) 6.0, 4/2 6.5, 8/1p 6.3, 8/2p 6.8
//            (4096, 8) 12.0, 4/2 13.3, 8/1p 11.2, 8/2p 12.2            (6400, 1) 8.3, 4/2 11.7, 8/1p 8.1, 8/2p 14.0
//            (4296, 21 to 86) 78.2, 4/2 60.5, 8/1p 67.0, 8/2p 68.8     (5728, 21 to 86) 80.1, 4/2 72.9, 8/1p 73.8, 8/2p 70.0
//   without vector loads, bf16 rank 12
//            (1024, 32) 37.1, 2/4 29.0, 4/2 23.1, 4/4 20.3, 8/2p 25.0  (4096, 32) 50.8, 4/2 59.2, 8/1p 47.8, 8/2p 40.1
//            (16384, 32) 128, 4/2 198, 8/1p 127, 8/2p 148, 16/1p 103
//   fp32 rank 16
//            (1024, 32) 55.8, 2/4 78.7, 4/2 44.5, 4/4 45.5, 8/2p 47.3  (2048, 32) 60.0, 4/2 69.7, 8/2p 49.8
//            (4096, 32) 66.2, 4/2 141, 8/1p 65.4, 8/2p 72.8            (16384, 32) 260, 4/2 536, 8/1p 263, 8/2p 281, 16/1p 158
//            (6400, 1) 18.1, 4/2 46.1, 8/2p 32.3, 16/1p 13.3
GemmForm gemm_plan_form(long launch_tiles, long launch_blocks, int max_blocks, int max_tokens, bool generic, bool env32) {
  const long tiles = launch_tiles, blocks = launch_tiles > 0 ? launch_blocks / launch_tiles : 0;   // (on average)
  const bool uneven = 4 * max_blocks > 5 * blocks;
  const int T = max_tokens;
  GemmForm f = {8, 1};
  if (T > 32) {                                    // (one run: two would take the room of a second workgroup)
    if (tiles <= (!generic ? 3072 : !env32 ? 2048 : 1024)) f = {4, 1};
  } else if (!generic) {
    if (tiles <= 512) f = {2, T <= 16 ? 4 : 2};
    else if (tiles <= 1024) f = {4, T <= 16 && blocks >= 16 ? 4 : 2};
    else if (tiles <= 3072) f = blocks >= (tiles > 2048 ? 10 : T <= 16 ? 8 : 4) ? GemmForm{4, 2} : f;
    else if (tiles <= 4096) f = blocks >= (uneven ? 10 : 21) ? GemmForm{8, 2} : f;
    else if (uneven && blocks >= 10)
      f = tiles <= 5504 ? GemmForm{4, 2} : T > 8 || tiles <= 8191 ? GemmForm{8, 2} : tiles > 11008 ? GemmForm{16, 1} : f;
    else if (tiles <= 5504) f = T > 8 && T <= 16 && blocks >= 27 ? GemmForm{8, 2} : f;
    else if (tiles > 11008 && T <= 8) f = {16, 1};
  } else if (!env32) {
    if (tiles <= 1024) f = {4, T <= 16 && blocks >= 8 ? 4 : 2};
    else if (tiles <= 4096) f = blocks >= (tiles <= 2048 ? 4 : 8) ? GemmForm{8, 2} : f;
    else if (uneven && tiles <= (T > 8 && T <= 16 ? 8191 : 11008)) f = blocks >= 10 ? GemmForm{8, 2} : f;
    else if (T <= 8 && tiles > 8191) f = {16, 1};
  } else {
    if (tiles <= 1024) f = blocks >= 4 ? GemmForm{4, T <= 16 && blocks >= 32 ? 4 : 2} : f;
    else if (tiles <= 4096) f = blocks >= (tiles <= 2048 ? 8 : uneven ? 21 : T > 16 ? 32 : 40) ? GemmForm{8, 2} : f;
    else if (T <= 8 && tiles > (uneven ? 8191 : 6144)) f = {16, 1};
  }
  // (8/1 in pairs: up to 7 % slower where a unit has one workgroup; with fp32 envelopes nothing gained)
  if (T <= 8 && f.tiles >= 8 && !(f.tiles == 8 && f.form == 1 && ((generic && env32) || tiles <= 2048))) f.form += kGemmPairs;
  return f;
}
int gemm_plan_max_tokens() { return 64; }   // plans with longer problems launch the single-problem kernel per problem

int launch_stage_gemm(const WorkItem* items_dev, int nitems, int mode, GemmForm form, const StageProb* p, hipStream_t s) {
  if (items_dev) {
    if (form.form == 0)    // a plan built before its header named the runs
      form.form = (p->T > 32 ? 1 : form.tiles == 2 && p->T <= 16 ? 4 : form.tiles < 8 ? 2 : 1) +
                  (p->T <= 8 && form.tiles >= 8 ? kGemmPairs : 0);
    if (form.tiles == 2) return gemm::launch_items_r<2, 1>(items_dev, nitems, mode, form.form, p, s);
    if (form.tiles == 4) return gemm::launch_items_r<4, 1>(items_dev, nitems, mode, form.form, p, s);
    if (form.tiles == 16) return gemm::launch_items_rt<4, 4, 1>(items_dev, nitems, mode, form.form, p, s);
    return gemm::launch_items_r<4, 2>(items_dev, nitems, mode, form.form, p, s);
  }
  mode = gemm_load_mode(*p);
  const bool vectors = mode != gemm::kGeneric;
  if (p->T > kFewMaxTokens || (p->T > 32 && vectors)) {
    const LongShape f = long_problem_shape(*p, vectors);
    if (f.R == 1) return gemm::launch_rt<1, 2>(mode, p, s);
    if (f.TB == 2) return gemm::launch_rt<2, 2>(mode, p, s);
    if (f.TB == 4) return gemm::launch_rt<2, 4>(mode, p, s);
    if (f.TB == 6) return gemm::launch_rt<2, 6>(mode, p, s);
    if (f.TB == 7) return gemm::launch_rt<2, 7>(mode, p, s);
    return gemm::launch_rt<2, 8>(mode, p, s);
  }
  if (p->T > 16 && vectors) return gemm::launch_rt<1, 2>(mode, p, s);
  const SplitGeom one = {p->KB, 1, 0};                          // (no room for partial sums)
  return launch_stage_gemm_few(p, one, nullptr, 0, s);
}

SplitGeom few_geom(int ntiles, int KB, int T, bool vectors, size_t max_splits) {
  // Host arithmetic only (the workspace layout follows from it), for a device of 256 compute units that hold two
  // workgroups each.  In tenths of the time of a chunk, 0.3 us: a workgroup by itself on a unit takes 10 per
  // chunk, two that share one 17 each, further ones queue; partial sums cost 22 for their launch and 4 TB/s.  Measured
  // with 16 tokens: 86 blocks on 32 row groups, 7 or 8 splits of 12 blocks against 11 of 8, 23.8 and 25.6 us per
  // call; 32 blocks on 86 groups, 4 splits of 8 against 3 of 12 (258 workgroups), 24.7 and 27.3 us.
  // Few row tiles or blocks: the kernel with one tile per workgroup needs no partial sums; 4 per iteration of
  // four blocks and 8 KB of staging per tile and block at 10 TB/s (1856 x 2848, k = 128, 11 tokens: 13.8 us
  // against 16.1 split).  Where both cost the same it has one launch less (24 x 4096, k = 24, 2 tokens: 14.3 against
  // 14.5 to 16.2 split).
  // The partial sums are priced for 4 or 32 tokens whatever T is: one split for 2 to 16 tokens and one for 17 to 64,
  // so that a token's result is the same bits in every call of such a range.  Against pricing them for T: 9920 x 640,
  // k = 1790, l = 3, 16 tokens 21.1 -> 19.4 us; 9920 x 896, k = 1792, l = 16, 16 tokens 16.2 -> 16.6 us; 5000 x 3001,
  // k = 2003, l = 3, 17 tokens 20.3 -> 19.8 us; 11008 x 11008, k = 8191, l = 3, 40 tokens 71.8 -> 69.0 us.
  const int64_t tokens = T > 16 ? 32 : 4;
  const int64_t ck = gemm::few_chunk(T > 16 ? 2 : 1);
  SplitGeom best = {KB, 1, (ntiles + gemm::kFewWaves - 1) / gemm::kFewWaves};
  int64_t least = -1;
  for (int64_t bs = ck;; bs += ck) {
    const int64_t nsplit = (KB + bs - 1) / bs, wgs = nsplit * best.ngroup;
    if (nsplit == 1 || (nsplit <= gemm::kFewSplits && (size_t)nsplit <= max_splits)) {
      int64_t cost = (bs < KB ? bs / ck : (KB + ck - 1) / ck) * (wgs <= 256 ? 10 : 17 * ((wgs + 511) / 512));
      if (nsplit > 1) cost += 22 + nsplit * tokens * ntiles * kTileRows * 8 / 1200000;
      if (least < 0 || cost < least) {
        least = cost;
        best.bs = (int)(bs < KB ? bs : KB);
        best.nsplit = (int)nsplit;
      }
    }
    if (nsplit == 1) break;
  }
  if (vectors && T <= 16) {
    const int64_t rounds = ntiles > 512 ? 2 : 1;                // (two tiles per workgroup then)
    if ((KB + 3) / 4 * 4 * rounds + (int64_t)ntiles * KB / 366 <= least) best = SplitGeom{KB, 1, ntiles};
  }
  return best;
}

int launch_stage_gemm_few(const StageProb* p, const SplitGeom& g, float* part, int64_t part_ld, hipStream_t s) {
  if (g.nsplit == 1 && p->T <= 16) {
    const int mode = gemm_load_mode(*p);
    if (mode == MDBF_F16) return gemm::launch_split<MDBF_F16>(p, s);
    if (mode == MDBF_BF16) return gemm::launch_split<MDBF_BF16>(p, s);
    if (mode == MDBF_F32) return gemm::launch_split<MDBF_F32>(p, s);
  }
  gemm::FewArgs a;
  a.p = *p;
  a.bs = g.bs;
  a.nsplit = g.nsplit;
  a.part = part;
  a.part_ld = part_ld;
  int e;
  if (p->vin_dt == MDBF_F16) e = gemm::launch_few_m<MDBF_F16>(a, s);
  else if (p->vin_dt == MDBF_BF16) e = gemm::launch_few_m<MDBF_BF16>(a, s);
  else e = gemm::launch_few_m<MDBF_F32>(a, s);
  if (e || g.nsplit == 1) return e;
  return launch_few_reduce(p, part, g.nsplit, part_ld, s);
}

int launch_few_reduce(const StageProb* p, const float* part, int nsplit, int64_t part_ld, hipStream_t s) {
  gemm::FewArgs a = {};
  a.p = *p;
  a.nsplit = nsplit;
  a.part = const_cast<float*>(part);
  a.part_ld = part_ld;
  hipLaunchKernelGGL(gemm::few_reduce_kernel, dim3((unsigned)((p->rows + 255) / 256), (unsigned)p->T), dim3(256), 0, s, a);
  return (int)hipGetLastError();
}

}  // namespace mdbf
