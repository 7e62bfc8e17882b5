// fp32 vector-ALU evaluation of one envelope-scaled binary product (MDBF_FLAG_PRECISE).
// One wavefront per 16-row tile; lane = (row r, 8-column group kg) as in the packed layout.
// Per lane: acc[c] += (+-1) * Ein[j,c] * vin[j] over its columns, then the four kg lanes of a
// row are summed, and out[r] = sum_c Eout[r,c] * acc[c]   (paper Eq. "me-dbf-expand").
#include <algorithm>

#include "mdbf_internal.h"

namespace mdbf {

__device__ inline int local_col_of_bit_p(int b, int kg) {
  const int h = b >> 4, bb = b & 15;
  const int f = 2 * (bb >> 3) + ((bb >> 2) & 1), i = bb & 3;
  return f * 32 + kg * 8 + 2 * i + h;
}

__global__ __launch_bounds__(64) void stage_precise_kernel(const StageProb* __restrict__ probs,
                                                           const WorkItem* __restrict__ items,
                                                           StageProb single) {
  int tile;
  const StageProb* pp;
  if (probs) {
    // in batch mode every work item is expanded to one block per tile by the launcher
    const WorkItem& it = items[blockIdx.y];
    if ((int)blockIdx.x >= it.ntiles) return;
    pp = &probs[it.prob];
    tile = it.tile0 + blockIdx.x;
  } else {
    pp = &single;
    tile = blockIdx.x;
  }
  const StageProb p = *pp;
  const int lane = threadIdx.x, r = lane & 15, kg = lane >> 4;
  const int row = tile * kTileRows + r;
  for (int b = 0; b < p.T; ++b) {
    float acc[MDBF_MAX_L];
#pragma unroll
    for (int c = 0; c < MDBF_MAX_L; ++c) acc[c] = 0.f;
    for (int q = 0; q < p.KB; ++q) {
      const uint32_t w = ((const MDBF_GLOBAL uint32_t*)p.S)[word_offset(tile, q, lane, p.KB, p.ntiles)];
      for (int bit = 0; bit < 32; ++bit) {
        const int col = q * kBlockCols + local_col_of_bit_p(bit, kg);
        if (col >= p.K) continue;
        const float v = load_as_float(p.vin, (int64_t)b * p.vin_ld + col, p.vin_dt);
        const float sv = ((w >> bit) & 1u) ? -v : v;
#pragma unroll
        for (int c = 0; c < MDBF_MAX_L; ++c)
          if (c < p.l) acc[c] += sv * load_as_float(p.Ein, (int64_t)col * p.l + c, p.env_dt);
      }
    }
    float o = 0.f;
#pragma unroll
    for (int c = 0; c < MDBF_MAX_L; ++c) {
      float a = acc[c];
      a += __shfl_xor(a, 16);
      a += __shfl_xor(a, 32);
      if (c < p.l && row < p.rows) o += a * load_as_float(p.Eout, (int64_t)row * p.l + c, p.env_dt);
    }
    if (kg == 0 && row < p.rows) emit_result(p.out, (int64_t)b * p.out_ld + row, p.out_dt, o, p.flags);
  }
}

int launch_stage_precise(const StageProb* probs_dev, const WorkItem* items_dev, int nitems,
                         const StageProb* single, hipStream_t s) {
  if (probs_dev) {
    // grid.x = upper bound of tiles per item is passed through single->ntiles by the caller
    hipLaunchKernelGGL(stage_precise_kernel, dim3((unsigned)single->ntiles, (unsigned)nitems), dim3(64), 0, s,
                       probs_dev, items_dev, *single);
  } else {
    hipLaunchKernelGGL(stage_precise_kernel, dim3((unsigned)single->ntiles), dim3(64), 0, s,
                       (const StageProb*)nullptr, (const WorkItem*)nullptr, *single);
  }
  return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------
// One-token evaluation of one envelope-scaled binary product by itself, in reconstruct order and fp32.
//
//   out[r] = sum_j S[r, j] * E[r, j] * vin[j],     E = Eout * Ein^T  (rank l)
//
// (paper Eq. "me-dbf-basis" for a single token).  A wave owns R row tiles of 16 rows and walks 128-column blocks:
// the matrix cores rebuild its 16 x 128 piece of E from the envelope rows (fp32 sums of exact products), the vector
// ALUs flip the signs with the packed bits and multiply-add with the activations, all in fp32; the waves of a
// workgroup split the blocks and meet once, in LDS, in wave order.
//
// What bounds it: the launch and the chain load -> rebuild -> sum -> store; from some 20000 (tile, block) pieces on the
// vector ALUs (three instructions per entry: flip, multiply-add, and an addition that doubles the register whose top bit
// is the next sign; 96 of them and 8 products a piece), with fp32 envelopes on the matrix cores.
// Nothing else lies between a wave's loads and its result: no scaled activations are built or shared, no barrier stands
// before the last one, and a row tile's contraction meets in memory only between the two factors, where the reader adds
// the (at most four) partial sums as it loads them, and, for the second one, where few row tiles would leave the device
// idle for long (one_geom_summed).
// Against building block-scaled records of the scaled activations in every workgroup and adding partial sums of both
// factors in memory, per call of one layer again and again from a graph: 4096 x 4096, k = 2656, l = 16 13.1 -> 8.4 us (10.6
// with layers that come from memory); 256 x 256, k = 128, l = 4 in fp32 9.7 -> 5.5 (in one launch 4.7, stage_pair_kernel); 11008 x 4096, k = 4096, l = 16 20.1 ->
// 12.8; two calls of 4096 x 4096, k = 1601, l = 1 25.9 -> 17.9; 3000 x 5000, k = 1777, l = 16 in fp32 19.6 -> 13.5; an empty
// pair of launches is 3 us.  Errors against 64 bits 6e-6 .. 2e-4 -> 2e-7.  Not faster: 1024 x 4096, k = 11008 (second factor
// of 64 row tiles), bf16 rank 16 37.8 -> 40.2, fp32 rank 5 24.5 -> 25.9.
// (Two row tiles per workgroup, which halve the reads of the envelope rows, are slower throughout: 8.7 -> 11.0 us.)
// ---------------------------------------------------------------------------------------------------
namespace one {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bhalf8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));   // a vector at any element's address

constexpr int kMaxWaves = 16;       // waves of a workgroup, each with blocks of its own

constexpr int kOneItemTiles = 8;    // row tiles of a plan's work item, one workgroup each
constexpr int kGridTiles = 1 << 21; // row tiles of a single problem along x: a grid dimension has at most 2^32 - 1 threads

struct OneArgs {
  StageProb p;
  const WorkItem* items;            // a plan's: workgroup (i, t, b) = row tile t of item i, token b; null: p
  int32_t bs, nsplit;               // blocks per workgroup, workgroups per row tile
  int32_t nsplit_in;
  const float* part_in;             // PARTS: vin[j] = sum over s < nsplit_in of part_in[s * part_in_ld + j]
  int64_t part_in_ld;
  float* part_out;                  // [nsplit][part_out_ld] partial sums (unused when nsplit == 1)
  int64_t part_out_ld;
};

// element i of an array whose bytes are addressable with 32 bits
template <class T>
__device__ __forceinline__ T at(const void* base, uint32_t i) {
  return *(const MDBF_GLOBAL T*)((const MDBF_GLOBAL char*)base + i * (uint32_t)sizeof(T));
}

// Envelope rows of a block as operands of the rebuild.  Lane (m, g) = (lane & 15, lane >> 4).  M: modes there is room for.
//   16-bit types: v_mfma_f32_16x16x32, eight consecutive modes of a column per lane.  M = 8: a load is 64 columns, the
//   four lane groups hold four sets of 16; M = 16: 32 columns, two sets, a column's modes on two lane groups.  A product
//   takes the columns of one set: its other operand is zero for the other groups.  All 64 lanes load different data; of
//   rank 8 or 16 a load is 1 KB without a gap.
//   fp32: M / 4 products v_mfma_f32_16x16x4 per set, of M / 4 consecutive modes of a column per lane, one from each.
// In set h of 32-column step f, row m of the product is column 32 f + 8 (m / 4) + 4 h + m % 4, so that lane (r, g) of the
// results holds columns 32 f + 8 g + 0 .. 7 of row r: those of its packed sign word.
//   VEC: rows of exactly M modes.  Other rows are read past their last mode: what is there meets zeros.
template <int ENV, int M>
struct EinBlock {
  static constexpr int kPer = ENV == MDBF_F32 ? M / 4 : 8;          // modes per lane and load
  static constexpr int kLoads = ENV == MDBF_F32 ? 8 : M / 4;        // per block
  uint32_t v[kLoads][ENV == MDBF_F32 ? kPer : 4];
};

// Rows of exactly four fp32 modes come a whole column of set 4 j + g per lane (VEC, below): a lane's entry t of the j-th such
// vector is mode t of column m of set 4 j + g, and has to be mode g of set 4 j + t.  (As one mode per lane and load, sixteen bytes
// apart: stage_pair_kernel on 256 x 256, k = 128 7.5 us per call from a graph instead of 4.7, two launches on 4096 x 4096, k = 512 8.0
// instead of 6.1.)
__device__ __forceinline__ void transpose_modes(uint32_t (&v)[8][1]) {
#pragma unroll
  for (int j = 0; j < 8; j += 4) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    // halves of the wave, then neighbouring sixteens: row r, group g of a 4 x 4 exchange places
    const u32x2 a = __builtin_amdgcn_permlane32_swap(v[j][0], v[j + 2][0], false, false);
    const u32x2 b = __builtin_amdgcn_permlane32_swap(v[j + 1][0], v[j + 3][0], false, false);
    const u32x2 c = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
    const u32x2 d = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
    v[j][0] = c.x;
    v[j + 1][0] = c.y;
    v[j + 2][0] = d.x;
    v[j + 3][0] = d.y;
  }
}

// where the lane's modes of load i of block q begin
template <int ENV, int M>
__device__ __forceinline__ uint32_t ein_first(int K, uint32_t l, int q, int i, int lane) {
  const int m = lane & 15, g = lane >> 4;
  int col = q * kBlockCols + 8 * (m >> 2) + (m & 3);
  if constexpr (ENV == MDBF_F32) col += 32 * (i >> 1) + 4 * (i & 1);
  else if constexpr (M == 8) col += 64 * i + 32 * (g >> 1) + 4 * (g & 1);
  else col += 32 * i + 4 * (g >> 1);
  return (uint32_t)min(col, K - 1) * l + (ENV == MDBF_F32 ? (uint32_t)(g * (M / 4)) : M == 8 ? 0u : 8u * (g & 1));
}

template <int ENV, int M, bool VEC>
__device__ __forceinline__ void load_ein(const StageProb& p, int q, int lane, EinBlock<ENV, M>& e) {
  typedef EinBlock<ENV, M> EB;
  if constexpr (ENV == MDBF_F32 && M == 4 && VEC) {
    const int m = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = q * kBlockCols + 64 * j + 32 * (g >> 1) + 4 * (g & 1) + 8 * (m >> 2) + (m & 3);
      const u32x4 v = at<u32x4>(p.Ein, (uint32_t)min(col, p.K - 1));
#pragma unroll
      for (int t = 0; t < 4; ++t) e.v[4 * j + t][0] = v[t];
    }
    return;
  }
  const uint32_t l = VEC ? (uint32_t)M : (uint32_t)p.l;
  const uint32_t count = (uint32_t)p.K * l;
  constexpr int kWords = sizeof(e.v[0]) / 4;
  typedef uint32_t vec __attribute__((ext_vector_type(kWords), aligned(ENV == MDBF_F32 ? 4 : 2)));
  const bool few = !VEC && count < EB::kPer;                                      // (uniform) no vector fits in:
  const void* from = few ? (const void*)p.S : p.Ein;                              // any will do, ein_tail takes them one by one
#pragma unroll
  for (int i = 0; i < EB::kLoads; ++i) {
    uint32_t first = ein_first<ENV, M>(p.K, l, q, i, lane);
    if (!VEC) first = min(first, few ? 0u : count - EB::kPer);                    // (ein_tail moves the rest)
    const vec v = *(const MDBF_GLOBAL vec*)((const MDBF_GLOBAL char*)from + (uint32_t)dtype_size(ENV) * first);
#pragma unroll
    for (int t = 0; t < kWords; ++t) {
      if constexpr (kWords == 1) e.v[i][t] = v.x;
      else e.v[i][t] = v[t];
    }
  }
}

// Blocks near the end of rows that are read past their last mode: where that would leave the factor, the factor's last
// vector was loaded (of a factor of fewer elements than a vector, none).  What lies behind the end is no number of the
// layer's and would survive its product with a zero mode if it were an infinity or NaN: zeros take its place.
template <int ENV, int M>
__device__ __forceinline__ void ein_tail(const StageProb& p, int q, int lane, EinBlock<ENV, M>& e) {
  typedef EinBlock<ENV, M> EB;
  const int count = p.K * p.l;
  if (count < EB::kPer) {                                               // (uniform)
#pragma unroll
    for (int i = 0; i < EB::kLoads; ++i) {
      const int first = (int)ein_first<ENV, M>(p.K, (uint32_t)p.l, q, i, lane);
      uint32_t x[EB::kPer];
#pragma unroll
      for (int t = 0; t < EB::kPer; ++t) {
        const uint32_t j = (uint32_t)min(first + t, count - 1);
        x[t] = ENV == MDBF_F32 ? at<uint32_t>(p.Ein, j) : (uint32_t)at<uint16_t>(p.Ein, j);
        x[t] = first + t < count ? x[t] : 0u;
      }
#pragma unroll
      for (int t = 0; t < EB::kPer; ++t) {
        if constexpr (ENV == MDBF_F32) e.v[i][t] = x[t];
        else if (t % 2 == 0) e.v[i][t / 2] = x[t] | (x[t + 1] << 16);
      }
      __builtin_amdgcn_sched_barrier(0);                                // (one vector at a time: registers)
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < EB::kLoads; ++i) {
    const int first = (int)ein_first<ENV, M>(p.K, (uint32_t)p.l, q, i, lane);
    const int down = max(0, first - (count - EB::kPer));
    if constexpr (ENV == MDBF_F32) {
#pragma unroll
      for (int t = 0; t < EB::kPer; ++t) {
        uint32_t x = 0;
#pragma unroll
        for (int u = t; u < EB::kPer; ++u) x = t + down == u ? e.v[i][u] : x;
        e.v[i][t] = x;
      }
    } else {
      const int sh = 16 * down;
      uint64_t lo = (uint64_t)e.v[i][0] | ((uint64_t)e.v[i][1] << 32), hi = (uint64_t)e.v[i][2] | ((uint64_t)e.v[i][3] << 32);
      if (sh >= 64) {
        lo = sh >= 128 ? 0 : hi >> (sh - 64);
        hi = 0;
      } else if (sh > 0) {
        lo = (lo >> sh) | (hi << (64 - sh));
        hi >>= sh;
      }
      e.v[i][0] = (uint32_t)lo;
      e.v[i][1] = (uint32_t)(lo >> 32);
      e.v[i][2] = (uint32_t)hi;
      e.v[i][3] = (uint32_t)(hi >> 32);
    }
  }
}

// The other operand: this lane's modes of row `row` times 2^-e, zeros past the rank.
template <int ENV, int M>
struct EoutRow {
  uint32_t v[ENV == MDBF_F32 ? M / 4 : 4];
  int e;
};

template <int ENV, int M, bool VEC>
__device__ __forceinline__ EoutRow<ENV, M> load_eout_bits(const StageProb& p, int row, int g) {
  EoutRow<ENV, M> o;
  constexpr int kN = EinBlock<ENV, M>::kPer;
  const uint32_t l = VEC ? (uint32_t)M : (uint32_t)p.l;
  const uint32_t m0 = ENV == MDBF_F32 ? (uint32_t)(g * kN) : M == 8 ? 0u : 8u * (g & 1);
  const uint32_t first = (uint32_t)row * l;
  o.e = 0;
  if constexpr (VEC && ENV != MDBF_F32) {
    const u32x4 v = at<u32x4>(p.Eout, (first + m0) >> 3);
#pragma unroll
    for (int t = 0; t < 4; ++t) o.v[t] = v[t];
  } else {
    uint32_t b[kN];
#pragma unroll
    for (int t = 0; t < kN; ++t)
      b[t] = ENV == MDBF_F32 ? at<uint32_t>(p.Eout, first + min(m0 + t, l - 1u)) : (uint32_t)at<uint16_t>(p.Eout, first + min(m0 + t, l - 1u));
#pragma unroll
    for (int t = 0; t < kN; ++t) b[t] = m0 + t < l ? b[t] : 0u;
    if constexpr (ENV == MDBF_F32) {
#pragma unroll
      for (int t = 0; t < kN; ++t) o.v[t] = b[t];
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) o.v[t] = b[2 * t] | (b[2 * t + 1] << 16);
    }
  }
  return o;
}

template <int ENV, int M>
__device__ __forceinline__ void scale_eout(EoutRow<ENV, M>& o) {
  if constexpr (ENV != MDBF_F16) {
    constexpr int kN = EinBlock<ENV, M>::kPer;
    // The products of two envelope entries of these types can leave the range of fp32 where entry times activation
    // does not: the row's largest entry goes below 1 / M, so that a sum of M products with entries of any size stays in
    // range (the smallest, 2^-126, keep 19 of their bits with M = 16); the power of two comes back with the result.
    float v[kN];
    float big = 0.f;
#pragma unroll
    for (int t = 0; t < kN; ++t) {
      v[t] = __builtin_bit_cast(float, ENV == MDBF_F32 ? o.v[t] : t & 1 ? o.v[t >> 1] & 0xFFFF0000u : o.v[t >> 1] << 16);
      big = fmaxf(big, fabsf(v[t]));
    }
    big = fmaxf(big, __shfl_xor(big, 16));
    big = fmaxf(big, __shfl_xor(big, 32));
    if (big > 0.f && big < __builtin_huge_valf()) o.e = ilogbf(big) + (M == 4 ? 3 : M == 8 ? 4 : 5);
#pragma unroll
    for (int t = 0; t < kN; ++t) v[t] = ldexpf(v[t], -o.e);
    if constexpr (ENV == MDBF_F32) {
#pragma unroll
      for (int t = 0; t < kN; ++t) o.v[t] = __builtin_bit_cast(uint32_t, v[t]);
    } else {                                              // (still eight significant bits)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        o.v[t] = (__builtin_bit_cast(uint32_t, v[2 * t]) >> 16) | (__builtin_bit_cast(uint32_t, v[2 * t + 1]) & 0xFFFF0000u);
    }
  }
}

template <int ENV, int M, bool VEC>
__device__ __forceinline__ EoutRow<ENV, M> load_eout(const StageProb& p, int row, int g) {
  EoutRow<ENV, M> o = load_eout_bits<ENV, M, VEC>(p, row, g);
  scale_eout<ENV, M>(o);
  return o;
}

template <int ENV>
__device__ __forceinline__ floatx4 rebuild16(u32x4 a, u32x4 b) {
  const floatx4 z = {0.f, 0.f, 0.f, 0.f};
  if constexpr (ENV == MDBF_F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), z, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bhalf8, a), __builtin_bit_cast(bhalf8, b), z, 0, 0, 0);
}

// the lanes of a wave have finished their LDS accesses (which execute in order: this is for the compiler)
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One 16 x 128 piece: acc += its rows' sums over block q, the signs in `sw`, the activations in LDS at `buf`.
template <int ENV, int M, bool VEC>
__device__ __forceinline__ void contract_block(const StageProb& p, int q, int lane, EinBlock<ENV, M>& ein, uint32_t sw,
                                               const EoutRow<ENV, M>& eo, const float* buf, float (&acc)[2]) {
  typedef EinBlock<ENV, M> EB;
  const int g = lane >> 4;
  if constexpr (ENV == MDBF_F32 && M == 4 && VEC) transpose_modes(ein.v);
  // (the block's last row may be read past the factor's end: fewer than sixteen elements lie behind its first)
  if (!VEC && (int64_t)(p.K - (q + 1) * kBlockCols + 1) * p.l < 16) ein_tail<ENV, M>(p, q, lane, ein);
  // the packed word keeps the signs of columns 2 t and 2 t + 1 of step f at bits c and c + 16, c = 8 (f / 2) + 4 (f % 2) + t:
  // they are taken from the top of two registers, which double from entry to entry (a left shift by a constant takes the
  // vector ALUs four cycles, an addition less)
  uint32_t odd = sw, even = sw << 16;
  auto flip = [](float v, uint32_t& signs) __attribute__((always_inline)) {
    const uint32_t out = __builtin_bit_cast(uint32_t, v) ^ (signs & 0x80000000u);
    asm("v_add_u32 %0, %0, %0" : "+v"(signs));
    return __builtin_bit_cast(float, out);
  };
#pragma unroll
  for (int f = 3; f >= 0; --f) {
    const floatx4 xa = *reinterpret_cast<const floatx4*>(buf + 32 * f + 8 * g);
    const floatx4 xb = *reinterpret_cast<const floatx4*>(buf + 32 * f + 8 * g + 4);
    floatx4 d[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (ENV == MDBF_F32) {
        d[h] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < EB::kPer; ++s)
          d[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, ein.v[2 * f + h][s]),
                                                      __builtin_bit_cast(float, eo.v[s]), d[h], 0, 0, 0);
      } else {
        const bool on = M == 8 ? g == 2 * (f & 1) + h : (g >> 1) == h;
        const uint32_t (&x)[4] = ein.v[M == 8 ? f >> 1 : f];
        d[h] = rebuild16<ENV>(u32x4{x[0], x[1], x[2], x[3]},
                              u32x4{on ? eo.v[0] : 0u, on ? eo.v[1] : 0u, on ? eo.v[2] : 0u, on ? eo.v[3] : 0u});
      }
    }
#pragma unroll
    for (int t = 3; t >= 0; --t) {
      const floatx4 e = d[t >> 1], x = t < 2 ? xa : xb;
      acc[0] = fmaf(flip(e[2 * (t & 1)], even), x[2 * (t & 1)], acc[0]);
      acc[1] = fmaf(flip(e[2 * (t & 1) + 1], odd), x[2 * (t & 1) + 1], acc[1]);
    }
    // (a step at a time: without this the products of a block are all made first, in 64 registers)
    asm volatile("" : "+v"(acc[0]), "+v"(acc[1]));
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int ENV, int M, bool VEC, bool PARTS, bool BATCH>
__global__ __launch_bounds__(64 * kMaxWaves) void stage_one_kernel(OneArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef EinBlock<ENV, M> EB;
  int tile = blockIdx.x + blockIdx.z * kGridTiles, split = blockIdx.y, token = 0;
  if constexpr (!BATCH) {
    if (tile >= a.p.ntiles) return;                      // (the last run of kGridTiles)
  } else {
    const WorkItem& w = a.items[blockIdx.x];             // (uniform: scalar loads)
    if ((int)blockIdx.y >= w.ntiles || (int)blockIdx.z >= w.p.T) return;
    tile = w.tile0 + (int)blockIdx.y;
    split = 0;
    token = blockIdx.z;
  }
  const StageProb p = BATCH ? a.items[blockIdx.x].p : a.p;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nwaves = (int)blockDim.x >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  // this wave's blocks: q_lo, q_lo + nwaves, ...
  const int bs = BATCH ? p.KB : a.bs;
  const int q_lo = split * bs + wave, q_hi = min((split + 1) * bs, p.KB);
  const uint32_t x0 = BATCH ? (uint32_t)token * (uint32_t)p.vin_ld : 0u;   // the token's first element
  float* xs = reinterpret_cast<float*>(smem) + wave * (2 * kBlockCols);   // two blocks' activations, this wave's only
  const MDBF_GLOBAL uint32_t* sbase = (const MDBF_GLOBAL uint32_t*)p.S + tile_base_words(tile, p.KB) + lane;
  const size_t sstride = (size_t)group_tiles(tile, p.ntiles) * 64u;

  // What a block needs from memory: columns lane and lane + 64 of the activations (the words they are in, or their
  // parts), envelope rows, signs.
  struct Block {
    uint32_t x[2][PARTS ? kOneMaxSplits : 1];
    EB ein;
    uint32_t sw;
  };
  const uint32_t xshift = p.vin_dt == MDBF_F32 ? 2u : 1u;
  auto fetch = [&](int q, Block& b) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t col = (uint32_t)min(q * kBlockCols + lane + 64 * h, p.K - 1);
      if constexpr (PARTS) {
#pragma unroll
        for (int s = 0; s < kOneMaxSplits; ++s) b.x[h][s] = at<uint32_t>(a.part_in + min(s, a.nsplit_in - 1) * a.part_in_ld, col);
      } else {
        b.x[h][0] = at<uint32_t>(p.vin, ((x0 + col) << xshift) >> 2);   // (the aligned word that holds it)
      }
    }
    load_ein<ENV, M, VEC>(p, q, lane, b.ein);
    b.sw = sbase[(size_t)q * sstride];
  };
  auto park = [&](int q, const Block& b, float* buf) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int col = q * kBlockCols + lane + 64 * h;
      float x;
      if constexpr (PARTS) {
        x = __builtin_bit_cast(float, b.x[h][0]);
#pragma unroll
        for (int s = 1; s < kOneMaxSplits; ++s) x += s < a.nsplit_in ? __builtin_bit_cast(float, b.x[h][s]) : 0.f;
      } else {
        const uint32_t half = ((x0 + min(col, p.K - 1)) & 1u) ? b.x[h][0] >> 16 : b.x[h][0] & 0xFFFFu;
        const float xh = (float)__builtin_bit_cast(_Float16, (uint16_t)half);
        x = p.vin_dt == MDBF_F32 ? __builtin_bit_cast(float, b.x[h][0]) : p.vin_dt == MDBF_F16 ? xh : __builtin_bit_cast(float, half << 16);
      }
      buf[lane + 64 * h] = col < p.K ? x : 0.f;
    }
    wave_lds_order();
  };
  float acc[2] = {0.f, 0.f};
  EoutRow<ENV, M> eo;
  eo.e = 0;
  if (q_lo < q_hi) {
    Block b0, b1;
    fetch(q_lo, b0);
    eo = load_eout<ENV, M, VEC>(p, min(tile * kTileRows + r16, p.rows - 1), g);
    park(q_lo, b0, xs);
    int q = q_lo;
    for (;;) {
      if (q + nwaves < q_hi) fetch(q + nwaves, b1);
      contract_block<ENV, M, VEC>(p, q, lane, b0.ein, b0.sw, eo, xs, acc);
      q += nwaves;
      if (q >= q_hi) break;
      park(q, b1, xs + kBlockCols);
      if (q + nwaves < q_hi) fetch(q + nwaves, b0);
      contract_block<ENV, M, VEC>(p, q, lane, b1.ein, b1.sw, eo, xs + kBlockCols, acc);
      q += nwaves;
      if (q >= q_hi) break;
      park(q, b0, xs);
    }
  }

  // ---- the lane groups' sums, then the waves', in wave order
  float* red = reinterpret_cast<float*>(smem) + nwaves * (2 * kBlockCols);
  float v = acc[0] + acc[1];
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  if constexpr (ENV != MDBF_F16) v = ldexpf(v, eo.e);
  if (lane < kTileRows) red[wave * kTileRows + lane] = v;
  __syncthreads();
  if (tid < kTileRows) {
    float sum = red[tid];
    for (int w = 1; w < nwaves; ++w) sum += red[w * kTileRows + tid];
    const int row = tile * kTileRows + tid;
    if (row < p.rows) {
      if (BATCH || a.nsplit == 1) emit_result(p.out, (int64_t)token * p.out_ld + row, p.out_dt, sum, p.flags);
      else ((MDBF_GLOBAL float*)a.part_out)[split * a.part_out_ld + row] = sum;
    }
  }
}

// ---- Both factors of a small layer in one launch.  Every workgroup works out all of z = V x for itself, in LDS, piece (16 x 128)
// by piece, and then row tiles of its own of U z.  What bounds a call of two launches on such a layer is the launches: 2.7 us each
// on the host.  On the device the second one saved pays for the pieces as long as they are few: pair_pieces.
// us per call, two launches -> one, from a graph, from one of four branches, and one after the other on a stream: 256 x 256, k = 128 (16
// pieces), l = 4 in fp32 5.5 -> 4.8, 7.6 -> 4.1 and 8.8 -> 6.1; l = 16 in fp16 4.8 -> 4.1, 6.5 -> 4.0 and 8.7 -> 6.1; 300 x 384, k = 128 (24)
// 4.9 -> 5.0, 6.6 -> 4.0 and 9.1 -> 6.4; 8190 x 101, k = 383 (24 in each of 256 workgroups) 6.1 -> 5.7, 6.5 -> 4.2 and 9.0 -> 6.4.  A single
// call on operands that come from memory takes what two launches take.
constexpr int kPairPieces = 24;
constexpr int kPairWaves = 8;       // (sixteen, a piece each: no faster, and the element-wise rows spill)

struct PairArgs {
  StageProb p, u;
};

template <int ENV, int M, bool VEC>
__global__ __launch_bounds__(64 * kPairWaves) void stage_pair_kernel(PairArgs a) {
  // the pieces' sums (of the first factor, then of the waves), z, the waves' activations
  __shared__ float red[kPairPieces * kTileRows];
  __shared__ __attribute__((aligned(16))) float z[(kPairPieces * kTileRows + kBlockCols - 1) / kBlockCols * kBlockCols];
  __shared__ __attribute__((aligned(16))) float xs[kPairWaves][kBlockCols];
  const StageProb &p = a.p, &u = a.u;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  struct Piece {
    EinBlock<ENV, M> ein;
    EoutRow<ENV, M> eo;
    uint32_t sw, x[2];
  };
  auto fetch = [&](const StageProb& s, int tile, int q, Piece& b) __attribute__((always_inline)) {
    load_ein<ENV, M, VEC>(s, q, lane, b.ein);
    b.sw = ((const MDBF_GLOBAL uint32_t*)s.S)[word_offset(tile, q, lane, s.KB, s.ntiles)];
    b.eo = load_eout_bits<ENV, M, VEC>(s, min(tile * kTileRows + r16, s.rows - 1), g);
  };
  // a piece's sums, a row on each of the first sixteen lanes
  auto contract = [&](const StageProb& s, int q, Piece& b, const float* x, float* out) __attribute__((always_inline)) {
    float acc[2] = {0.f, 0.f};
    scale_eout<ENV, M>(b.eo);
    contract_block<ENV, M, VEC>(s, q, lane, b.ein, b.sw, b.eo, x, acc);
    float v = acc[0] + acc[1];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if constexpr (ENV != MDBF_F16) v = ldexpf(v, b.eo.e);
    if (lane < kTileRows) out[lane] = v;
  };
  // ---- the first factor: piece i is block i % KB of tile i / KB
  const int pieces = p.ntiles * p.KB;
  const uint32_t xshift = p.vin_dt == MDBF_F32 ? 2u : 1u;
  auto fetch1 = [&](int i, Piece& b) __attribute__((always_inline)) {
    const int q = i % p.KB;
#pragma unroll
    for (int h = 0; h < 2; ++h)                                        // (the aligned word that holds it)
      b.x[h] = at<uint32_t>(p.vin, ((uint32_t)min(q * kBlockCols + lane + 64 * h, p.K - 1) << xshift) >> 2);
    fetch(p, i / p.KB, q, b);
  };
  Piece now, next;
  if (wave < pieces) fetch1(wave, now);
#pragma unroll 1
  for (int i = wave; i < pieces; i += kPairWaves) {
    if (i + kPairWaves < pieces) fetch1(i + kPairWaves, next);
    const int q = i % p.KB;
    wave_lds_order();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int col = q * kBlockCols + lane + 64 * h;
      const uint32_t half = (min(col, p.K - 1) & 1) ? now.x[h] >> 16 : now.x[h] & 0xFFFFu;
      const float xh = (float)__builtin_bit_cast(_Float16, (uint16_t)half);
      const float x = p.vin_dt == MDBF_F32 ? __builtin_bit_cast(float, now.x[h]) : p.vin_dt == MDBF_F16 ? xh : __builtin_bit_cast(float, half << 16);
      xs[wave][lane + 64 * h] = col < p.K ? x : 0.f;
    }
    wave_lds_order();
    contract(p, q, now, xs[wave], red + i * kTileRows);
    now = next;
  }
  // ---- the second one: the waves' slots of a tile each, a block on each of a slot's waves (there are at most three)
  const int slots = kPairWaves / u.KB, slot = wave / u.KB, q2 = wave - slot * u.KB;
  const int tile = (int)blockIdx.x + (int)gridDim.x * slot;
  const bool live = slot < slots && tile < u.ntiles;                   // (uniform in a wave)
  if (live) fetch(u, tile, q2, now);
  __syncthreads();
  for (int r = tid; r < u.KB * kBlockCols; r += 64 * kPairWaves) {     // (zeros past the last row)
    float sum = 0.f;
    if (r < p.rows) {
      const float* part = red + (r >> 4) * p.KB * kTileRows + (r & 15);
      sum = part[0];
      for (int q = 1; q < p.KB; ++q) sum += part[q * kTileRows];
    }
    z[r] = sum;
  }
  __syncthreads();
  if (live) contract(u, q2, now, z + q2 * kBlockCols, red + wave * kTileRows);
  __syncthreads();
  if (live && q2 == 0 && lane < kTileRows) {
    float sum = red[wave * kTileRows + lane];
    for (int q = 1; q < u.KB; ++q) sum += red[(wave + q) * kTileRows + lane];
    const int row = tile * kTileRows + lane;
    if (row < u.rows) emit_result(u.out, row, u.out_dt, sum, u.flags);
  }
}

template <int ENV, int M>
static int launch_pair_em(const PairArgs& a, int grid, hipStream_t s) {
  if (ENV != MDBF_BF16 && a.p.l == M)
    hipLaunchKernelGGL((stage_pair_kernel<ENV, M, ENV != MDBF_BF16>), dim3((unsigned)grid), dim3(64 * kPairWaves), 0, s, a);
  else
    hipLaunchKernelGGL((stage_pair_kernel<ENV, M, false>), dim3((unsigned)grid), dim3(64 * kPairWaves), 0, s, a);
  return (int)hipGetLastError();
}
template <int ENV>
static int launch_pair_e(const PairArgs& a, int grid, hipStream_t s) {
  if constexpr (ENV == MDBF_F32) {
    if (a.p.l <= 4) return launch_pair_em<ENV, 4>(a, grid, s);
  }
  if (a.p.l <= 8) return launch_pair_em<ENV, 8>(a, grid, s);
  return launch_pair_em<ENV, 16>(a, grid, s);
}

template <int ENV, int M, bool VEC>
static int launch_emv(const OneArgs& a, dim3 grid, int waves, hipStream_t s) {
  const dim3 block(64u * (unsigned)waves);
  const size_t smem = (size_t)waves * (2 * kBlockCols + kTileRows) * 4u;
  if (a.items) hipLaunchKernelGGL((stage_one_kernel<ENV, M, VEC, false, true>), grid, block, smem, s, a);
  else if (a.part_in) hipLaunchKernelGGL((stage_one_kernel<ENV, M, VEC, true, false>), grid, block, smem, s, a);
  else hipLaunchKernelGGL((stage_one_kernel<ENV, M, VEC, false, false>), grid, block, smem, s, a);
  return (int)hipGetLastError();
}
template <int ENV, int M>
static int launch_em(const OneArgs& a, dim3 grid, int waves, hipStream_t s) {
  if (ENV != MDBF_BF16 && a.p.l == M) return launch_emv<ENV, M, ENV != MDBF_BF16>(a, grid, waves, s);
  return launch_emv<ENV, M, false>(a, grid, waves, s);
}
template <int ENV>
static int launch_e(const OneArgs& a, dim3 grid, int waves, hipStream_t s) {
  if constexpr (ENV == MDBF_F32) {
    if (a.p.l <= 4) return launch_em<ENV, 4>(a, grid, waves, s);
  }
  if (a.p.l <= 8) return launch_em<ENV, 8>(a, grid, waves, s);
  return launch_em<ENV, 16>(a, grid, waves, s);
}
static int launch(const OneArgs& a, dim3 grid, int waves, hipStream_t s) {
  if (a.p.env_dt == MDBF_F16) return launch_e<MDBF_F16>(a, grid, waves, s);
  if (a.p.env_dt == MDBF_BF16) return launch_e<MDBF_BF16>(a, grid, waves, s);
  return launch_e<MDBF_F32>(a, grid, waves, s);
}

}  // namespace one

// Eight waves; sixteen where a unit has one workgroup of a long contraction, whose loads then hide behind each other
// (4096 x 11008, k = 4096: 13.8 -> 13.1 us; with more workgroups than units eight are better: 11008 x 4096 15.7 -> 13.1).
static OneGeom one_waves(OneGeom g, int ntiles, int KB) {
  g.nsplit = (KB + g.bs - 1) / g.bs;
  while (g.waves < 8 && g.waves < g.bs) g.waves *= 2;
  if (g.bs >= 16 && (int64_t)ntiles * g.nsplit <= 256) g.waves = one::kMaxWaves;
  return g;
}

OneGeom one_geom(int ntiles, int KB, size_t max_splits) {
  // For a device of 256 compute units.  A unit's four SIMDs take four blocks of its workgroups at a time, whichever
  // waves hold them; a partial sum costs its reader a load: 166 row tiles of 32 blocks on three workgroups each leave 22
  // blocks on the busiest unit instead of 32 (8.8 -> 8.4 us per 4096 x 4096 call), 19 tiles of 86 blocks on four
  // 22 (10.4 -> 6.5 us for 200 x 11008, k = 300).
  OneGeom g = {1, KB, 1};
  int64_t least = -1;
  for (int n = 1; n <= kOneMaxSplits && (n == 1 || (size_t)n <= max_splits); ++n) {
    const int bs = (KB + n - 1) / n;
    const int64_t cost = 8 * (((int64_t)ntiles * n + 255) / 256) * ((bs + 3) / 4) + n;
    if (least < 0 || cost < least) {
      least = cost;
      g.bs = bs;
    }
  }
  return one_waves(g, ntiles, KB);
}

OneGeom one_geom_summed(const StageProb& p, size_t max_splits) {
  // Few row tiles of a long contraction leave most of the device idle: up to eight workgroups each, for the 2.4 us that the
  // launch costs which adds their sums up.  ns that a unit takes for the four blocks on its SIMDs: 245 where rows are whole
  // vectors of 16-bit entries, 310 otherwise; fp32 rows of 4, 8, 16 modes 410, 530, 730.  us per call with 1, 2, 4, 8
  // workgroups a row tile, 16 x 128, k = 16000, l = 16 in fp32 28.4, 19.3, 13.9, 10.6, in fp16 12.6, 10.5, 8.8, 7.7;
  // 1000 x 130, k = 8000 (63 row tiles) 18.4, 15.0, 11.6, 11.5 and 9.4, 9.5, 8.6, 8.5; 2000 x 130, k = 8000, l = 8
  // 14.1, 12.7, 12.6, 12.4 and 9.3, 9.7, 9.6, 10.1; 16 x 128, k = 1000 6.3, 7.4, 7.3, 7.2 and 5.2, 6.8, 6.7, 6.7.
  const int modes = p.l <= 4 ? 0 : p.l <= 8 ? 1 : 2;
  static const int fp32_ns[3] = {410, 530, 730};
  const int64_t ns = p.env_dt == MDBF_F32 ? fp32_ns[modes] : p.env_dt == MDBF_F16 && (p.l == 8 || p.l == 16) ? 245 : 310;
  OneGeom g = {1, p.KB, 1};
  int64_t least = -1;
  for (int n = 1; n <= 8 && (n == 1 || (size_t)n <= max_splits); ++n) {
    const int bs = (p.KB + n - 1) / n, used = (p.KB + bs - 1) / bs;
    const int64_t cost = ns * (((int64_t)p.ntiles * used + 255) / 256) * ((bs + 3) / 4) + (used > 1 ? 2400 : 0);
    if (least < 0 || cost < least) {
      least = cost;
      g.bs = bs;
    }
  }
  return one_waves(g, p.ntiles, p.KB);
}

bool stage_is_one(const StageProb& p) {
  const int64_t row = (int64_t)p.l * dtype_size(p.env_dt), most = (int64_t)1 << 32;
  return p.K < (1 << 30) && p.rows < (1 << 30) && p.K * row < most && p.rows * row < most &&
         (p.T == 1 || p.vin_ld < ((int64_t)1 << 30) / p.T);
}

// Pieces of the first factor that one launch may go through in every workgroup: as many as cost about what the launch does on
// the device (the host saves its 2.7 us in any case, and calls beside each other a third of their time).  us per call from a graph of
// different layers one behind the other, two launches and one: rank 16 and 8 in fp16, 16 to 20 pieces 4.8 to 6.0 and 4.1 to 5.4, 21 to 24 (three
// rounds of the eight waves) 4.9 and 5.0 to 5.2, 5.9 and 5.8 (8190 rows): the 2 to 6 % that a graph of nothing else loses there are a
// tenth of what streams and branches gain; fp32 rank 4, 20, 5.7 to 7.3 and 5.4 to 6.6, 24, 5.7 and 5.9; rank 8, 12, 5.6 to 7.0 and 5.2 to 6.0, 16,
// 5.5 and 5.8; other rows, loaded entry by entry or of 16 fp32 modes, 8: 5.4 to 6.9 and 4.4 to 5.6, with 10 to 16 5.8 and 6.5, 5.5 and 6.1.
// And one round of workgroups: 688 row tiles on 344 of them (k = 384) 5.4 and 7.5.
static int pair_pieces(const StageProb& p) {
  if (p.env_dt == MDBF_F16 && (p.l == 16 || p.l == 8)) return one::kPairPieces;
  if (p.env_dt == MDBF_F32 && p.l == 4) return 20;
  return p.env_dt == MDBF_F32 && p.l == 8 ? 12 : 8;
}
// a workgroup for each row tile up to 256 of them, then one for as many as its waves take at once
static int pair_grid(const StageProb& u) {
  const int slots = one::kPairWaves / u.KB;
  return std::max(std::min(u.ntiles, 256), (u.ntiles + slots - 1) / slots);
}

// Do the bytes of the (one token's) activations and of the result meet?  In the one launch workgroups store their rows of Y while
// others still read X; the two launches read all of X before they store anything of Y, so calls in place are theirs.
static bool in_place(const StageProb sp[2]) {
  const uintptr_t x = (uintptr_t)sp[0].vin, y = (uintptr_t)sp[1].out;
  return x < y + (uintptr_t)sp[1].rows * dtype_size(sp[1].out_dt) && y < x + (uintptr_t)sp[0].K * dtype_size(sp[0].vin_dt);
}

bool stage_is_pair(const StageProb sp[2]) {
  return (int64_t)sp[0].ntiles * sp[0].KB <= pair_pieces(sp[0]) && pair_grid(sp[1]) <= 256 && stage_is_one(sp[0]) && stage_is_one(sp[1]) &&
         !in_place(sp);
}

int launch_stage_pair(const StageProb sp[2], hipStream_t s) {
  const one::PairArgs a = {sp[0], sp[1]};
  const int grid = pair_grid(sp[1]);
  if (sp[0].env_dt == MDBF_F16) return one::launch_pair_e<MDBF_F16>(a, grid, s);
  if (sp[0].env_dt == MDBF_BF16) return one::launch_pair_e<MDBF_BF16>(a, grid, s);
  return one::launch_pair_e<MDBF_F32>(a, grid, s);
}

int one_item_tiles() { return one::kOneItemTiles; }

int launch_stage_one(const StageProb* p, const OneGeom& g, const float* part_in, int nsplit_in, int64_t part_in_ld,
                     float* part_out, int64_t part_out_ld, hipStream_t s) {
  one::OneArgs a;
  a.p = *p;
  a.items = nullptr;
  a.bs = g.bs;
  a.nsplit = g.nsplit;
  a.nsplit_in = nsplit_in;
  a.part_in = part_in;
  a.part_in_ld = part_in_ld;
  a.part_out = part_out;
  a.part_out_ld = part_out_ld;
  const int gx = std::min(p->ntiles, one::kGridTiles);
  return one::launch(a, dim3((unsigned)gx, (unsigned)g.nsplit, (unsigned)((p->ntiles + gx - 1) / gx)), g.waves, s);
}

int launch_stage_one_items(const WorkItem* items_dev, int nitems, int env_dt, int rank, int max_tokens, hipStream_t s) {
  one::OneArgs a = {};
  a.p.env_dt = env_dt;
  a.p.l = rank;                  // (chooses the kernel; kOneMixedRanks: room for 16 modes, rows of any length)
  a.items = items_dev;
  const int waves = (int64_t)nitems * one::kOneItemTiles * max_tokens <= 256 ? one::kMaxWaves : 8;
  return one::launch(a, dim3((unsigned)nitems, one::kOneItemTiles, (unsigned)max_tokens), waves, s);
}

}  // namespace mdbf
