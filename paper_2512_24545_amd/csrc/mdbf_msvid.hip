// MSVID_l on the GPU: the projection step of the layer-wise quantizer (paper Sec. 4.2, Eq. "msvid-def"):
//
//   MSVID_l[Z] = sign(Z) o TSVD_l(|Z|),      TSVD_l(|Z|) = A Q^T  (rank l, best in Frobenius norm)
//
// with the singular values split evenly between the factors, A = U_l sqrt(Sigma_l), Q = V_l sqrt(Sigma_l).
// By Theorem 1 (Eq. "rankl-error") the error of the result is the tail of |Z|'s spectrum.
//
// The truncated SVD is taken by block subspace iteration with b = l + oversampling columns and a
// Rayleigh-Ritz step at the end; everything runs on the stream, nothing is read back by the host:
//   V <- caller's start block (cols x b)
//   repeat `iters` times:   B = |Z| V,  orthonormalise;   V = |Z|^T B,  orthonormalise
//   B = |Z| V;   B^T B = W L W^T (Jacobi, fp64);   sigma = sqrt(L);   A = B W_l Sigma_l^(-1/2),   Q = V W_l Sigma_l^(1/2)
// The two products are the whole cost: each reads Z once (HBM-bound, 4 bytes per 2 b multiply-adds), row-major as
// it stands: one kernel, with the roles of rows and columns as a template argument.
// Orthonormalisation is Cholesky-QR: Gram matrix in per-workgroup parts (fp64 sums, stored in fp32) added in fp64, its Cholesky
// factorisation in fp64.  In the first passes the last workgroup of the launch that leaves the parts factorises, and the next
// product applies R^(-1) to the rows of its input block as it stages them; later a workgroup beside the product factorises, and
// R^(-1) is applied to the product's sums.
#include <type_traits>

#include "mdbf_internal.h"

namespace mdbf {
namespace msvid {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx4_any __attribute__((ext_vector_type(4), aligned(4)));    // four elements at any element's address
typedef uint32_t u32_any __attribute__((aligned(1)));

constexpr int kThreads = 256;
constexpr int kOut = 64;              // outputs (columns or rows of Z) per workgroup of the product kernel
constexpr int kChunk = 256;           // contraction entries per workgroup, 64 per wave
constexpr int kSmallThreads = 1024;   // the b x b kernels (a thread per matrix entry, b <= 32) and the chunk reduction
                                      // (few workgroups: many loads in flight in each)
constexpr int kGramRows = 64;         // rows per workgroup of the reduce + Gram kernel

// the signs of the first `count` (at most four) entries
__device__ __forceinline__ void store_signs(floatx4 v, MDBF_GLOBAL int8_t* out, int count) {
  if (count == 4) {
    *(MDBF_GLOBAL u32_any*)out = (v.x < 0.f ? 0xFFu : 1u) | (v.y < 0.f ? 0xFF00u : 0x100u) |
                                 (v.z < 0.f ? 0xFF0000u : 0x10000u) | (v.w < 0.f ? 0xFF000000u : 0x1000000u);
  } else {
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (e < count) out[e] = v[e] < 0.f ? (int8_t)-1 : (int8_t)1;
  }
}

// ---- S = sign(Z) as int8 (+1 / -1, sign(0) = +1: Sec. 2, Notation), four entries per thread, 2^sh threads per row
// (a workgroup takes several rows of a narrow matrix: with one each 10^6 x 24 took 0.5 ms); clears the counter of
// reduce_gram_kernel's launches.  For calls without passes: in others the first product along the columns, which has the
// entries in registers, writes the signs (9.4 us for a pass of its own over 4096 x 2656, 2 us more for that product)
__global__ __launch_bounds__(kThreads) void sign_kernel(const float* __restrict__ Z, int rows, int cols, int64_t ld, int sh,
                                                        int8_t* __restrict__ S, uint32_t* __restrict__ counter) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *counter = 0u;
  const int64_t row = (int64_t)blockIdx.x * (kThreads >> sh) + (threadIdx.x >> sh);
  const int c = (int)((blockIdx.y << sh) + (threadIdx.x & ((1u << sh) - 1u))) * 4;
  if (row >= rows || c >= cols) return;
  const MDBF_GLOBAL float* z = (const MDBF_GLOBAL float*)Z + row * ld + c;
  MDBF_GLOBAL int8_t* out = (MDBF_GLOBAL int8_t*)S + row * cols + c;
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
  if (c + 4 <= cols) {
    v = *(const MDBF_GLOBAL floatx4_any*)z;
  } else {
    for (int e = 0; c + e < cols; ++e) v[e] = z[e];
  }
  store_signs(v, out, min(4, cols - c));
}

// G = sum of the workgroups' parts, in fp64, in a fixed order: a thread adds four neighbouring entries of every
// (THREADS / quads)-th part, sixteen loads in flight, then the groups are added in order.  sums: LDS for a double per entry and
// group.
// COHERENT: the parts were written by other workgroups of the same launch, with device-scope stores
template <int BB, int THREADS>
constexpr int gram_groups() { return THREADS / (BB * BB / 4); }
template <int BB, int THREADS, bool COHERENT>
__device__ void gather_gram(const float* __restrict__ Gp, int nparts, double* __restrict__ sums, double (&G)[BB][BB]) {
  constexpr int kQuads = BB * BB / 4, kGroups = gram_groups<BB, THREADS>();
  static_assert(kGroups >= 1, "a thread per quad");
  const int grp = threadIdx.x / kQuads, qd = threadIdx.x - grp * kQuads;
  if (grp < kGroups) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int w0 = grp; w0 < nparts; w0 += 16 * kGroups) {
      floatx4 v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const MDBF_GLOBAL floatx4* src = (const MDBF_GLOBAL floatx4*)Gp + (size_t)min(w0 + u * kGroups, nparts - 1) * kQuads + qd;
        if constexpr (COHERENT) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint64_t x = __hip_atomic_load((const MDBF_GLOBAL uint64_t*)src + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
            v[u][2 * h] = __builtin_bit_cast(float, lo);
            v[u][2 * h + 1] = __builtin_bit_cast(float, hi);
          }
        } else {
          v[u] = *src;
        }
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (w0 + u * kGroups < nparts) {
#pragma unroll
          for (int e = 0; e < 4; ++e) s[e] += (double)v[u][e];
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) sums[grp * (BB * BB) + 4 * qd + e] = s[e];
  }
  __syncthreads();
  for (int p = threadIdx.x; p < BB * BB; p += THREADS) {
    double sum = sums[p];
#pragma unroll
    for (int w = 1; w < kGroups; ++w) sum += sums[w * (BB * BB) + p];
    G[p / BB][p % BB] = sum;
  }
  __syncthreads();
}

// a double held by lane `src` (a compile-time or wave-uniform index), in every lane
__device__ __forceinline__ double lane_value(double v, int src) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, src);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), src);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// the largest of a non-negative value in this lane and the ones behind it, of the first BB <= 32 lanes (the rest undefined)
template <int BB>
__device__ __forceinline__ float longest_from_here(float v) {
  auto with = [&](auto shift) {
    const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x100 + decltype(shift)::value, 0xF, 0xF, true);   // row_shl
    v = fmaxf(v, __builtin_bit_cast(float, o));
  };
  with(std::integral_constant<int, 1>());
  with(std::integral_constant<int, 2>());
  with(std::integral_constant<int, 4>());
  with(std::integral_constant<int, 8>());
  if constexpr (BB > 16) {
    const float second = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
    v = (threadIdx.x & 16) ? v : fmaxf(v, second);
  }
  return v;
}

// ---- Cholesky-QR: G = R^T R (R upper triangular), Tm = R^(-1): Y Tm has orthonormal columns (Tf: the same in fp32).
// by_length: where a column is shorter than one after it by kTooShort (of the squares) the columns of Y are taken in the order of their
// lengths, longest first (R is triangular in that order, and so do the columns of Y Tm stand).  After a product with |Z| that is the
// order of what they hold of its largest modes, and as each step sorts what the columns in front left, the modes come to stand in
// their order whatever the start block's is (what that is for: run(), below).  The columns of a random start nearly always
// stay where they are (99 of 100 starts of 500 x 500 to 4096 x 2656): their lengths within the bulk of a spectrum differ by less.
// One wave; lane j < 32 holds column j of the matrix in registers (right-looking: after step k the trailing columns
// hold the Schur complement), lane 32 + j column j of the identity, which the same steps turn into column j of
// L^(-1), L D L^T = G, and the roots of the pivots at the end into row j of R^(-1).  Row k is passed round by lane reads: no
// LDS traffic and no barrier inside the b steps, and no substitution after them.
// A column that the earlier ones span (|Z| of lower rank than the block is wide: a member of the format is) has
// a pivot at the level of the Gram matrix's rounding, 1e-6 of its diagonal entry (fp32 partial sums): such a
// column is dropped (its column of Tm is zero, and stays zero through the products that follow).
// What bounds it: instructions of one wave, 8 cycles each (two lane reads and a multiply-add per entry of the trailing
// columns).  The next pivot's entry goes first, so that its reciprocal is worked out between the others' updates:
// 12600 -> 8200 cycles for b = 24 against a root per step and a zero or one per row behind a branch.
constexpr float kTooShort = 16.f;
template <int BB>
__device__ __forceinline__ void cholesky_inverse(const double (&G)[BB][BB], bool by_length, double* Tm, float* Tf) {
  const int j = (int)threadIdx.x & 31;
  const bool inv = (threadIdx.x & 32) != 0;
  const int jc = min(j, BB - 1);                       // lanes past the last column shadow it and store nothing
  const double* column = &G[0][jc];
  int from = jc;                                       // the column at the lane's place
  double a[BB];
#pragma unroll
  for (int i = 0; i < BB; ++i) a[i] = column[i * BB];
  double least = 1e-6 * column[jc * BB];               // of the lane's pivot
  if (by_length) {
    const float length2 = (float)column[jc * BB];
    const bool too_short = longest_from_here<BB>(length2) > kTooShort * length2;
    if (__ballot(!inv && too_short)) {                 // (uniform)
      // ties by index: the keys are all different, whatever the entries are
      const uint32_t key = (__builtin_bit_cast(uint32_t, length2) & ~31u) | (31u - (uint32_t)jc);
      int place = 0;
#pragma unroll 1
      for (int i = 0; i < BB; ++i) place += (uint32_t)__builtin_amdgcn_readlane((int)key, i) > key ? 1 : 0;
      // (lanes without a column of their own send to lanes without a place)
      const int at_place = __builtin_amdgcn_ds_permute(4 * (j < BB && !inv ? place : 32 + j), jc);
      from = __builtin_amdgcn_ds_bpermute(4 * jc, at_place);
      column = &G[0][from];
#pragma unroll
      for (int i = 0; i < BB; ++i) a[i] = column[__builtin_amdgcn_readlane(at_place, i) * BB];
      least = 1e-6 * column[from * BB];
    }
  }
#pragma unroll
  for (int i = 0; i < BB; ++i) {
    asm volatile("" : "+v"(a[i]));                     // (no branch around the loads)
    a[i] = inv ? (i == jc ? 1.0 : 0.0) : a[i];
  }
  double own = 0.0;                                    // the lane's pivot (a dropped column: zero)
  auto keeps = [&](double piv, int k) { const double l = lane_value(least, k); return piv > l && l > 0.0; };
  double piv = lane_value(a[0], 0), r = __builtin_amdgcn_rcp(piv), e = fma(-piv, r, 1.0), t = fma(e, e, e);
  bool keep = keeps(piv, 0);
  r = keep ? fma(r, t, r) : 0.0;                       // (the estimate has 24 bits or more: cubed, all 53)
  own = j == 0 && keep ? piv : own;
#pragma unroll
  for (int k = 0; k + 1 < BB; ++k) {
    const double s = a[k], w = s * r;                  // (a dropped column changes nothing)
    a[k + 1] = fma(-lane_value(s, k + 1), w, a[k + 1]);
    __builtin_amdgcn_sched_barrier(0);
    piv = lane_value(a[k + 1], k + 1);
    r = __builtin_amdgcn_rcp(piv);
    __builtin_amdgcn_sched_barrier(0);
    const int left = BB - (k + 2), per = (left + 3) / 4;
#pragma unroll
    for (int part = 0; part < 4; ++part) {
      double b[(BB + 3) / 4];
#pragma unroll
      for (int u = 0; u < per; ++u)
        if (part * per + u < left) b[u] = lane_value(s, k + 2 + part * per + u);
      __builtin_amdgcn_sched_barrier(0);
      if (part == 0) e = fma(-piv, r, 1.0);
      if (part == 1) t = fma(e, e, e);
      if (part == 2) r = fma(r, t, r);
      if (part == 3) {
        keep = keeps(piv, k + 1);
        r = keep ? r : 0.0;
        own = j == k + 1 && keep ? piv : own;
      }
#pragma unroll
      for (int u = 0; u < per; ++u)
        if (part * per + u < left) a[k + 2 + part * per + u] = fma(-b[u], w, a[k + 2 + part * per + u]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const double root = own > 0.0 ? rsqrt(own) : 0.0;
  if (inv && j < BB) {
#pragma unroll
    for (int i = 0; i < BB; ++i) {
      const double v = a[i] * lane_value(root, i);
      Tm[from * BB + i] = v;
      Tf[from * BB + i] = (float)v;
    }
  }
}

// ---- P[chunk][o][:] = sum over the chunk's contraction entries q of |Z[.]| * X'[q, :],   X' = X T  (SCALED) or X
// SCALED: T (in Tf) is there.  Else, with nparts > 0, workgroup 0 of the launch works it out beside the others' products, from
// the parts of X^T X that the launch before left, and the launch that adds up the partial sums applies it to them:
// |Z| (X T) = (|Z| X) T.
// COLS: outputs are the columns of Z (|Z|^T X, X has a row per row of Z); else its rows (|Z| X).
// Grid: output strips of 64, times contraction chunks of 256.  A wave owns the strip and 64 contraction entries, works out
// its 64 rows of X' and contracts a 64 x 64 piece of Z in four rounds of 16 entries: four 16-byte loads per lane, a
// round ahead, then 4 steps of v_mfma_f32_16x16x4_f32 (fp32 operands and sums) per 16 outputs and 16 columns of X'.
// The four waves meet in LDS in wave order.
// What bounds it: 9 us for one read of Z beside 6 us of matrix-core work and 9 us of launch, staging and partial
// sums, which only partly overlap.  (All of a wave's sixteen loads in flight: no change; X as single elements in
// operand order: 8 us more.)  Lanes that own columns and fused multiply-adds took 24 us per product of 4096 x 2656 and b = 24, and a transposed
// copy of Z for |Z| X another 20 us per call; now 18 to 20 us SCALED, 16 to 19 us not.
template <int BB, bool COLS, bool SCALED>
__global__ __launch_bounds__(kThreads, 4) void abs_mul_kernel(const float* __restrict__ Z, int rows, int cols, int64_t ld,
                                                              const float* __restrict__ X, const float* __restrict__ Gp,
                                                              int nparts, double* __restrict__ Tm, float* __restrict__ Tf,
                                                              float* __restrict__ P, int8_t* __restrict__ S,
                                                              uint32_t* __restrict__ counter) {
  constexpr int NT = (BB + 15) / 16;                   // 16-column tiles of X' (the last may be partly past BB)
  constexpr int RS = BB + 1;                           // floats per output in the waves' sums
  constexpr int kXs = 4 * (64 * BB + 16), kRed = 4 * kOut * RS;
  __shared__ __attribute__((aligned(16))) float buf[kXs > kRed ? kXs : kRed];
  int unit = blockIdx.x;
  if constexpr (!SCALED) {
    if (nparts > 0 && unit-- == 0) {
      constexpr int kEntries = BB * BB;
      static_assert((gram_groups<BB, kThreads>() + 1) * kEntries * 8 <= sizeof(buf), "they take the products' LDS");
      double (&G)[BB][BB] = *reinterpret_cast<double (*)[BB][BB]>(buf);
      gather_gram<BB, kThreads, false>(Gp, nparts, reinterpret_cast<double*>(buf) + kEntries, G);
      if (threadIdx.x < 64) cholesky_inverse<BB>(G, true, Tm, Tf);
      return;
    }
  }
  if (!COLS && counter && blockIdx.x == 0 && threadIdx.x == 0) *counter = 0u;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int nout = COLS ? cols : rows, nin = COLS ? rows : cols;
  const int strips = (nout + kOut - 1) / kOut, chunk = unit / strips;
  const int o0 = (unit - chunk * strips) * kOut, q0 = chunk * kChunk;
  const int qw = q0 + wave * 64;
  // ---- the wave's 64 rows of X, coalesced, and T (requested before Z: a load waits for all before it)
  constexpr int KS = BB / 4;                           // steps of four columns of X
  const MDBF_GLOBAL floatx4* xg = (const MDBF_GLOBAL floatx4*)X;
  floatx4 xr[KS], tr = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < KS; ++i) xr[i] = xg[min((int64_t)qw * KS + lane + 64 * i, (int64_t)nin * KS - 1)];
  if (SCALED && tid < BB * BB / 4) tr = ((const MDBF_GLOBAL floatx4*)Tf)[tid];
  // ---- Z.  COLS: load i of round j covers row qw + 16 j + 4 i + g and columns o0 + 4 n .. + 3: step i contracts its
  // four rows, output tile v holds columns o0 + 4 m + v.  Rows: load i covers row o0 + 16 i + n and columns
  // qw + 16 j + 4 g .. + 3: step v contracts columns qw + 16 j + 4 g' + v, output tile i holds rows o0 + 16 i + m.
  // Entries past the end repeat the last (their X' is zero); outputs past it are not stored.
  const MDBF_GLOBAL float* zb = (const MDBF_GLOBAL float*)Z;
  const bool whole = (COLS ? o0 : qw) + 64 <= cols;    // (uniform) the wave's 64 columns all exist
  auto load = [&](int j, floatx4 (&z)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = COLS ? min(qw + 16 * j + 4 * i + g, rows - 1) : min(o0 + 16 * i + n, rows - 1);
      const int c = COLS ? o0 + 4 * n : qw + 16 * j + 4 * g;
      const MDBF_GLOBAL float* src = zb + (int64_t)r * ld;
      if (whole) {
        z[i] = *(const MDBF_GLOBAL floatx4_any*)(src + c);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) z[i][v] = src[min(c + v, cols - 1)];
      }
    }
  };
  floatx4 z[4], zn[4];
  load(0, zn);
  // ---- X' of the wave's entries in LDS (each wave reads only its own), sixteen rows at a time in the place of X's.
  // (The span is what matters here, fp32 will do; the last block is orthonormalised in fp64 by apply_kernel.)
  float* xs = buf + wave * (64 * BB + 16);
#pragma unroll
  for (int i = 0; i < KS; ++i) {
    const bool ok = qw + (lane + 64 * i) / KS < nin;
    reinterpret_cast<floatx4*>(xs)[lane + 64 * i] = ok ? xr[i] : floatx4{0.f, 0.f, 0.f, 0.f};
  }
  if (lane < 16) xs[64 * BB + lane] = 0.f;             // (read by the partial last tile, never used)
  if constexpr (SCALED) {
    __shared__ __attribute__((aligned(16))) float tms[BB * BB];
    if (tid < BB * BB / 4) reinterpret_cast<floatx4*>(tms)[tid] = tr;
    __syncthreads();
    float tb[KS][NT];
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int u = 0; u < NT; ++u) tb[k][u] = tms[(4 * k + g) * BB + min(n + 16 * u, BB - 1)];   // (past BB: dropped)
#pragma unroll 1
    for (int t = 0; t < 4; ++t) {
      float xa[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) xa[k] = xs[(16 * t + n) * BB + 4 * k + g];
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        floatx4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k) d = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[k], tb[k][u], d, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + 16 * u < BB) xs[(16 * t + 4 * g + i) * BB + n + 16 * u] = d[i];
      }
    }
  }
  __syncthreads();

  floatx4 acc[4][NT];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int u = 0; u < NT; ++u) acc[t][u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = zn[i];
    if (j < 3) load(j + 1, zn);
    if (COLS && SCALED && S) {                         // (uniform) the signs of what is here anyway
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = qw + 16 * j + 4 * i + g, c = o0 + 4 * n;
        if (r < rows) store_signs(z[i], (MDBF_GLOBAL int8_t*)S + (int64_t)r * cols + c, min(4, cols - c));
      }
    }
    const float* xw = xs + (16 * j + (COLS ? g : 4 * g)) * BB + n;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      float b[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) b[u] = xw[(COLS ? 4 * st : st) * BB + 16 * u];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float a = fabsf(COLS ? z[st][t] : z[t][st]);
#pragma unroll
        for (int u = 0; u < NT; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[u], acc[t][u], 0, 0, 0);
      }
    }
  }
  __syncthreads();                                     // every wave is done with X'
  // lane (n, g) holds rows 4 g + i of the tiles, column n + 16 u of X'
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = COLS ? 4 * (4 * g + i) + t : 16 * t + 4 * g + i;
        if (n + 16 * u < BB) buf[(wave * kOut + o) * RS + n + 16 * u] = acc[t][u][i];
      }
  __syncthreads();
  float* out = P + ((size_t)chunk * nout + o0) * BB;
  const int valid = min(kOut, nout - o0) * BB;
#pragma unroll 1
  for (int e = tid; e < valid; e += kThreads) {
    const int o = e / BB, j = e - o * BB;
    const float* r = buf + o * RS + j;
    out[e] = ((r[0] + r[kOut * RS]) + r[2 * kOut * RS]) + r[3 * kOut * RS];
  }
}

// ---- Y = sum over chunks of P (in chunk order), times T where it is given (all in fp64), and this workgroup's part of
// Y^T Y.  Tm (or null): the last workgroup to finish (a counter, which it sets back to zero; nobody waits) adds the parts up
// and leaves Tm = R^(-1) of the Cholesky factorisation (Tf: the same in fp32).  T may be Tm: every workgroup has read it then.
// In launches of their own the sums took 7 us and the factorisation 17; together 15, most of it the chain of b pivots in fp64,
// which the products of later passes work out for themselves: 6 us without it.
template <int BB>
__global__ __launch_bounds__(kSmallThreads) void reduce_gram_kernel(const float* __restrict__ P, int nchunks, int n,
                                                                    float* __restrict__ Y, float* __restrict__ Gp,
                                                                    const double* T, double* Tm, float* Tf, bool by_length,
                                                                    uint32_t* __restrict__ counter) {
  constexpr int NT = (BB + 15) / 16;                   // 16-column tiles (the last may be partly past BB)
  constexpr int RS = BB + 1;                           // entries per row in LDS
  constexpr int kGroups = gram_groups<BB, kSmallThreads>();
  __shared__ float ys[kGramRows * RS];
  __shared__ double yd[kGramRows * RS], ts[BB * BB];
  __shared__ double G[BB][BB];
  __shared__ double sums[kGroups * BB * BB];
  __shared__ uint32_t is_last;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int row0 = blockIdx.x * kGramRows;
  const int nrow = min(kGramRows, n - row0);
  const size_t plane = (size_t)n * BB;
  if (T)
    for (int p = tid; p < BB * BB; p += kSmallThreads) ts[p] = T[p];
  static_assert(kGramRows * BB / 2 <= kSmallThreads && BB % 2 == 0, "a thread per pair");
  if (tid < kGramRows * BB / 2) {                      // two entries, sixteen chunks in flight, added in their order
    const int idx = 2 * tid, r = idx / BB, j = idx - r * BB;
    const size_t e = (size_t)row0 * BB + idx;
    double y[2] = {0.0, 0.0};
    if (r < nrow) {
      for (int c0 = 0; c0 < nchunks; c0 += 16) {
        floatx2 v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = *(const MDBF_GLOBAL floatx2*)((const MDBF_GLOBAL float*)P + (size_t)min(c0 + u, nchunks - 1) * plane + e);
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (c0 + u < nchunks) {
            y[0] += (double)v[u].x;
            y[1] += (double)v[u].y;
          }
      }
      if (!T) *(MDBF_GLOBAL floatx2*)((MDBF_GLOBAL float*)Y + e) = floatx2{(float)y[0], (float)y[1]};
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (T) yd[r * RS + j + i] = y[i];
      else ys[r * RS + j + i] = (float)y[i];
    }
  }
  __syncthreads();
  // Both small products on the matrix cores in fp64: lane (m, g) of an operand holds entry 4 k + g of row (column) m, of the
  // result rows 4 i + g of column m.
  if (T) {
    if (wave < 4 * NT) {                               // 16 rows, 16 columns
      const int t = wave & 3, col = 16 * (wave >> 2) + m;
      doublex4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < BB / 4; ++k)
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(yd[(16 * t + m) * RS + 4 * k + g], ts[(4 * k + g) * BB + min(col, BB - 1)], d, 0, 0, 0);
      if (col < BB) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 16 * t + 4 * i + g;
          ys[r * RS + col] = (float)d[i];
          if (r < nrow) ((MDBF_GLOBAL float*)Y)[(size_t)(row0 + r) * BB + col] = (float)d[i];
        }
      }
    }
    __syncthreads();
  }
  static_assert(4 * NT * NT <= kSmallThreads / 64 && kGroups >= 4, "a wave per tile and quarter of the rows");
  if (wave < 4 * NT * NT) {
    const int q = wave & 3, ci = 16 * ((wave >> 2) % NT) + m, cj = 16 * ((wave >> 2) / NT) + m;
    doublex4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kGramRows / 16; ++k) {
      const float* row = ys + (kGramRows / 4 * q + 4 * k + g) * RS;
      d = __builtin_amdgcn_mfma_f64_16x16x4f64((double)row[min(ci, BB - 1)], (double)row[min(cj, BB - 1)], d, 0, 0, 0);
    }
    if (cj < BB) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (ci - m + 4 * i + g < BB) sums[q * (BB * BB) + (ci - m + 4 * i + g) * BB + cj] = d[i];
    }
  }
  __syncthreads();
  for (int p = tid; p < BB * BB; p += kSmallThreads) {
    const float part = (float)((sums[p] + sums[BB * BB + p]) + (sums[2 * BB * BB + p] + sums[3 * BB * BB + p]));
    __hip_atomic_store((MDBF_GLOBAL float*)Gp + (size_t)blockIdx.x * BB * BB + p, part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!Tm) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's entries are in memory
  __syncthreads();
  if (tid == 0) {
    const uint32_t old = __hip_atomic_fetch_add((MDBF_GLOBAL uint32_t*)counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    is_last = old + 1u == gridDim.x ? 1u : 0u;
  }
  __syncthreads();
  if (!is_last) return;
  if (tid == 0) __hip_atomic_store((MDBF_GLOBAL uint32_t*)counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  gather_gram<BB, kSmallThreads, true>(Gp, gridDim.x, sums, G);
  if (tid >= 64) return;                               // (no barrier below)
  cholesky_inverse<BB>(G, by_length, Tm, Tf);
}

// ---- Rayleigh-Ritz: G = B^T B = W L W^T by cyclic Jacobi in fp64; Ritz values sigma_i = sqrt(L_i), descending.
// MA = W_l Sigma_l^(-1/2) (A = B MA), MQ = W_l Sigma_l^(1/2) (Q = V MQ); both BB x BB row-major, columns >= l zero.
// Cyclic Jacobi with the round-robin ordering: a step rotates the BB / 2 index pairs (2 i, 2 i + 1) at once and moves rows
// and columns on as it writes them (one stays, the others move round a circle), so that the next pairs lie in the same places: BB - 1
// steps bring every two together once, and everything back.  A lane works out the rotation of one column pair and applies it
// to the 2 x 2 block of four rows (with the row pair's, from another lane; rows and columns in one go, into the other of two
// copies) or to two entries of a row of W: one barrier a step, and no more trips to LDS than the entries themselves.
// What bounds it is a step's chain of instructions (8 cycles each for a lone wave of a SIMD), BB - 1 steps in six or seven sweeps.
// The angle comes from fp32 arithmetic, on numbers scaled for it (the next sweep takes out what it leaves, 1e-7 of an entry), its
// cosine and sine from fp64: a rotation to working precision whatever the angle is.  Sweeps end where no entry is above 1e-16 of its
// diagonal ones' mean, in the mean of its two copies: they differ by roundings of that size, and tests of one with rotations by the other
// go on for ever.  As many sweeps as with angles in fp64.
// Moving indices instead of rows, angles in fp64 by one wave and two barriers a step 91 us (every thread for itself 116; every
// wave for itself in fp32 102); now 68.  (Six sweeps, to 1e-13, 64 us: modes 2^-52 of the largest were left as they were.)
constexpr int ritz_block_waves(int BB) { return (BB / 2 + 3) / 4; }   // a row pair, or a row of W, per sixteen lanes
template <int BB>
constexpr int ritz_threads() { return 64 * (ritz_block_waves(BB) + (BB + 3) / 4); }
template <int BB>
__global__ __launch_bounds__(ritz_threads<BB>()) void ritz_kernel(const float* __restrict__ Gp, int nparts, int l,
                                                  double* __restrict__ MA, double* __restrict__ MQ,
                                                  float* __restrict__ sigma) {
  constexpr int H = BB / 2, kThr = ritz_threads<BB>(), RS = BB + 2;   // (rows of 16-byte pairs, spread over the banks)
  __shared__ double g0[BB][BB];
  __shared__ __attribute__((aligned(16))) double lds[4 * BB * RS];    // the matrix, W, and their other copies
  __shared__ int order[BB];
  __shared__ double sums[gram_groups<BB, kThr>() * BB * BB];
  const int t = threadIdx.x, lane = t & 63;
  gather_gram<BB, kThr, false>(Gp, nparts, sums, g0);
  // the largest diagonal entry to [0.5, 1), by a power of two
  double most = 0.0;
  for (int i = 0; i < BB; ++i) most = fmax(most, g0[i][i]);
  int ex = 0;
  if (most > 0.0 && most < __builtin_huge_val()) (void)frexp(most, &ex);
  for (int p = t; p < BB * BB; p += kThr) {
    const int i = p / BB, j = p - i * BB;
    // (row and column i, and BB - 1 - i, at places 2 i and 2 i + 1)
    const int pi = (i & 1) ? BB - 1 - (i >> 1) : i >> 1, pj = (j & 1) ? BB - 1 - (j >> 1) : j >> 1;
    lds[i * RS + j] = ldexp(g0[pi][pj], -ex);
    lds[(BB + i) * RS + j] = i == pj ? 1.0 : 0.0;
  }
  static_assert(BB % 2 == 0 && H >= 3 && H <= 64, "pairs");
  // where a row (column) goes after a step
  auto moved = [](int x) {
    return x == 1 ? 1 : x == 0 ? 3 : x == BB - 1 ? BB - 2 : (x & 1) ? x + 2 : x - 2;
  };
  static_assert(H <= 16 && BB % 4 == 0, "a lane per column pair");
  constexpr int kBlockWaves = ritz_block_waves(BB);
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const bool on_a = wave < kBlockWaves;                // (uniform)
  const int cp = min(lane & 15, H - 1), sub = lane >> 4;              // (lanes past the last pair store nothing)
  const int rp = on_a ? 4 * wave + sub : 0, wrow = on_a ? 0 : 4 * (wave - kBlockWaves) + sub;
  const bool live = (lane & 15) < H && rp < H;
  const int rpc = min(rp, H - 1);
  const int row = on_a ? 2 * rpc : BB + wrow;          // the block's rows (of W: one) and columns
  const int from0 = row * RS + 2 * cp, from1 = from0 + (on_a ? RS : 0);
  const int to_row0 = on_a ? moved(2 * rpc) : BB + wrow, to_row1 = on_a ? moved(2 * rpc + 1) : BB + wrow;
  const int to_col0 = moved(2 * cp), to_col1 = moved(2 * cp + 1);
  const int to00 = to_row0 * RS + to_col0, to01 = to_row0 * RS + to_col1, to10 = to_row1 * RS + to_col0, to11 = to_row1 * RS + to_col1;
  const int diag = 2 * cp * RS + 2 * cp;
  auto cosine = [](float tf) {                         // (the estimate has 22 bits: cubed, all 53)
    const double tt = (double)tf, x = fma(tt, tt, 1.0), c0 = (double)__builtin_amdgcn_rsqf(fmaf(tf, tf, 1.f));
    const double e = fma(-x * c0, c0, 1.0);
    return fma(c0 * e, fma(e, 0.375, 0.5), c0);
  };
  int cur = 0;                                         // the copy that is read: 0 or its distance
  __syncthreads();
  for (int sweep = 0; sweep < 12; ++sweep) {
    bool any = false;                                  // an off-diagonal entry that still has to go
    for (int e = t; e < BB * BB; e += kThr) {
      const int p = e / BB, q = e - p * BB;
      const double apq = 0.5 * (lds[cur + p * RS + q] + lds[cur + q * RS + p]), app = lds[cur + p * RS + p], aqq = lds[cur + q * RS + q];
      any = any || (p < q && fabs(apq) > 1e-150 && apq * apq > 1e-32 * fabs(app * aqq));
    }
    if (!__syncthreads_or(any ? 1 : 0)) break;
#pragma unroll 1
    for (int step = 0; step < BB - 1; ++step) {
      const double* a = lds + cur;
      double* out = lds + (2 * BB * RS - cur);
      const double2 top = *reinterpret_cast<const double2*>(a + diag);
      const double2 bottom = *reinterpret_cast<const double2*>(a + diag + RS);
      const double2 b0 = *reinterpret_cast<const double2*>(a + from0);
      double2 b1 = {0.0, 0.0};
      if (on_a) b1 = *reinterpret_cast<const double2*>(a + from1);
      // the tangent of the smaller of the two rotations, o / (|h| + (h^2 + o^2)^(1/2)) with the sign of h, of both by the larger one's
      // power of two (a branch around that where it is not needed: 7 us more per call)
      const double h = bottom.y - top.x, o = top.y + bottom.x;
      const int larger = __builtin_amdgcn_frexp_exp(fmax(fabs(h), fabs(o)));
      const float hf = (float)ldexp(h, -larger), of = (float)ldexp(o, -larger);
      float tf = of * __builtin_amdgcn_rcpf(fabsf(hf) + __builtin_amdgcn_sqrtf(fmaf(hf, hf, of * of)));
      tf = of == 0.f ? 0.f : fminf(fmaxf(tf, -1.f), 1.f);
      tf = hf >= 0.f ? tf : -tf;
      if (on_a) {
        const float tr = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * rpc, __builtin_bit_cast(int, tf)));
        const double c2 = cosine(tf), s2 = (double)tf * c2, c1 = cosine(tr), s1 = (double)tr * c1;
        const double bpp = c2 * b0.x - s2 * b0.y, bpq = s2 * b0.x + c2 * b0.y;     // columns
        const double bqp = c2 * b1.x - s2 * b1.y, bqq = s2 * b1.x + c2 * b1.y;
        if (live) {
          out[to00] = c1 * bpp - s1 * bqp;                                         // rows
          out[to01] = c1 * bpq - s1 * bqq;
          out[to10] = s1 * bpp + c1 * bqp;
          out[to11] = s1 * bpq + c1 * bqq;
        }
      } else {
        const double c2 = cosine(tf), s2 = (double)tf * c2;
        if (live) {
          out[to00] = c2 * b0.x - s2 * b0.y;
          out[to01] = s2 * b0.x + c2 * b0.y;
        }
      }
      __syncthreads();
      cur = 2 * BB * RS - cur;
    }
  }
  auto eigen = [&](int i) { return ldexp(lds[cur + i * RS + i], ex); };
  if (t < BB) {            // eigenvalues in descending order, ties by index
    // (a NaN, from a NaN or infinity in Z, ranks below everything: `order` is a permutation whatever the entries are)
    const double none = -__builtin_huge_val();
    const double at = eigen(t), mine = at == at ? at : none;
    int rank = 0;
    for (int i = 0; i < BB; ++i) {
      const double ai = eigen(i), e = ai == ai ? ai : none;
      rank += (e > mine || (e == mine && i < t)) ? 1 : 0;
    }
    order[rank] = t;
  }
  __syncthreads();
  if (t < BB) sigma[t] = (float)sqrt(fmax(eigen(order[t]), 0.0));
  for (int p = t; p < BB * BB; p += blockDim.x) {
    const int i = p / BB, j = p - i * BB;
    double ma = 0.0, mq = 0.0;
    if (j < l) {
      const double sg = sqrt(fmax(eigen(order[j]), 0.0));
      const double sg_max = sqrt(fmax(eigen(order[0]), 0.0));
      if (sg > 1e-7 * sg_max) {    // a mode at the level of fp32 rounding of the largest is a null mode of |Z|
        const double rs = sqrt(sg);
        mq = lds[cur + (BB + i) * RS + order[j]] * rs;
        ma = lds[cur + (BB + i) * RS + order[j]] / rs;
      }
    }
    MA[p] = ma;
    MQ[p] = mq;
  }
}

// ---- out (n x lo) = Y (n x BB) . m (BB x BB, its first lo columns), fp64 accumulation; blockIdx.y = 1: the second one
struct Applied {
  const float* Y;
  const double* m;
  float* out;
  int n, lo;
};
template <int BB>
__global__ __launch_bounds__(kThreads) void apply_kernel(Applied first, Applied second) {
  __shared__ double ms[BB * BB];
  const Applied a = blockIdx.y ? second : first;
  for (int p = threadIdx.x; p < BB * BB; p += kThreads) ms[p] = a.m[p];
  __syncthreads();
  const size_t total = (size_t)a.n * a.lo;
  for (size_t e = (size_t)blockIdx.x * kThreads + threadIdx.x; e < total; e += (size_t)gridDim.x * kThreads) {
    const size_t r = e / a.lo;
    const int j = (int)(e - r * a.lo);
    const float* yr = a.Y + r * BB;
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < BB; ++i) s += (double)yr[i] * ms[i * BB + j];
    a.out[e] = (float)s;
  }
}

struct Layout {
  size_t p, yb, yc, v1, gp, tm, ma, mq, tf, ctr, total;
  int nparts_max;
};

template <int BB>
static int run(const float* Z, int rows, int cols, int64_t ld, int l, int iters, const float* X0, int8_t* S, float* A,
               float* Q, float* sigma, unsigned char* ws, const Layout& L, hipStream_t s) {
  float* P = (float*)(ws + L.p);
  float* Yb = (float*)(ws + L.yb);     // rows x BB
  float* Yc = (float*)(ws + L.yc);     // cols x BB
  float* V1 = (float*)(ws + L.v1);     // cols x BB
  float* Gp = (float*)(ws + L.gp);
  double* Tm = (double*)(ws + L.tm);
  float* Tf = (float*)(ws + L.tf);
  double* MA = (double*)(ws + L.ma);
  double* MQ = (double*)(ws + L.mq);
  uint32_t* ctr = (uint32_t*)(ws + L.ctr);
  const dim3 blk(kThreads);
  // (with passes, the first product along the columns writes the signs, and the first one of all clears the counter)
  if (iters == 0) {
    int sh = 0;
    while ((4 << sh) < cols && (1 << sh) < kThreads) ++sh;
    const int rows_per_wg = kThreads >> sh;
    hipLaunchKernelGGL(sign_kernel, dim3((rows + rows_per_wg - 1) / rows_per_wg, (cols + (4 << sh) - 1) / (4 << sh)), blk, 0, s,
                       Z, rows, cols, ld, sh, S, ctr);
  }
  // Y = Yin's sums (nchunks of them), times T, its Gram parts and (Tout) the inverse of its Cholesky factor
  auto reduce = [&](const float* Yin, int nchunks, int n, float* Y, const double* T, double* Tout, bool by_length = false) {
    const int nparts = (n + kGramRows - 1) / kGramRows;
    hipLaunchKernelGGL(reduce_gram_kernel<BB>, dim3(nparts), dim3(kSmallThreads), 0, s, Yin, nchunks, n, Y, Gp, T, Tout, Tf, by_length, ctr);
    return nparts;
  };
  auto product = [&](auto cols_side, auto is_scaled, int nout, int nin, const float* X, int nparts, int step) {
    const int nchunks = (nin + kChunk - 1) / kChunk;
    const int64_t units = (int64_t)((nout + kOut - 1) / kOut) * nchunks + (nparts > 0 ? 1 : 0);
    hipLaunchKernelGGL((abs_mul_kernel<BB, decltype(cols_side)::value, decltype(is_scaled)::value>), dim3((unsigned)units), blk,
                       0, s, Z, rows, cols, ld, X, Gp, nparts, Tm, Tf, P, step == 1 ? S : nullptr, step == 0 ? ctr : nullptr);
    return nchunks;
  };
  // Step 2 i of the iteration is B = |Z| V of pass i, step 2 i + 1 V = |Z|^T B.  X is not orthonormal: T = R^(-1) of X^T X = R^T R
  // is applied to it in front of the product (T from the launch before), or behind it (T from beside it, from the Gram parts):
  // 9 us less of waiting, a product without the 1.6 us of X T.  Behind the product, T also takes out what the leading
  // columns have in common with the others after |Z| has magnified it: with a leading mode sigma_1 / sigma_j = 1 / rho times
  // larger, at an angle theta_i to the first column after i passes, the rounding of those columns grows by at most
  // min(1 / rho, rho^(2 i - 1) tan theta_0) <= (tan theta_0)^(1 / 2 i): 7 after one pass from a random start (tan theta_0 = 50), 2.7 after
  // two, while 38 would be lost at the start of a Gaussian matrix.  So the first two passes apply it in front, and from
  // the second on columns in a bad order are sorted: the first one is then the one with the most of that mode, not the one that the caller
  // put there.  (In the caller's order a first column orthogonal to a mode a hundred times the others cost A Q^T a factor of 25 to 65
  // against R^(-1) in front, 1e-5 of it.  Sorted, over start blocks with one, four or half of the columns orthogonal to the leading modes,
  // lengths from 1e6 to 1e-6 and centred columns, on six kinds of spectra: 0.44 to 1.0 of the errors in front in the mean of a kind, 1.6 at
  // most; over first columns with 1e-7 to 1 of the leading mode 1.33 at most, 2.2 where only columns eight times too short are
  // sorted instead of four times; 3 us more per call of 8 passes.)
  // (Long blocks, of many Gram parts, always: four waves would be too long adding them up.)
  constexpr int kStepsInOrder = 2, kStepsBehind = 4, kMostParts = 256;
  const int row_parts = (rows + kGramRows - 1) / kGramRows, col_parts = (cols + kGramRows - 1) / kGramRows;
  const bool can = row_parts <= kMostParts && col_parts <= kMostParts;
  auto behind = [&](int step) { return can && step >= kStepsBehind; };
  auto step_product = [&](auto cols_side, int step, const float* X, bool last) {
    constexpr bool kCols = decltype(cols_side)::value;
    const int nout = kCols ? cols : rows, nin = kCols ? rows : cols;
    int nchunks;
    if (step == 0 || behind(step))
      nchunks = product(cols_side, std::false_type(), nout, nin, X, step == 0 ? 0 : kCols ? row_parts : col_parts, step);
    else
      nchunks = product(cols_side, std::true_type(), nout, nin, X, 0, step);
    return reduce(P, nchunks, nout, kCols ? Yc : Yb, behind(step) ? Tm : nullptr, last || !behind(step + 1) ? Tm : nullptr, step >= kStepsInOrder);
  };
  const float* X = X0;
  for (int it = 0; it < iters; ++it) {
    step_product(std::false_type(), 2 * it, X, false);
    step_product(std::true_type(), 2 * it + 1, Yb, it + 1 == iters);
    X = Yc;
  }
  // an orthonormal V: Cholesky-QR twice (iters == 0: on the start block itself)
  const int grid_apply = 1024;
  if (iters == 0) reduce(X0, 1, cols, Yc, nullptr, Tm);
  reduce(Yc, 1, cols, V1, Tm, Tm);
  const Applied v = {V1, Tm, Yc, cols, BB}, none = {V1, Tm, Yc, 0, BB};
  hipLaunchKernelGGL(apply_kernel<BB>, dim3(grid_apply), blk, 0, s, v, none);                     // Yc = V, orthonormal
  // Rayleigh-Ritz on B = |Z| V
  const int npb = reduce(P, product(std::false_type(), std::false_type(), rows, cols, Yc, 0, -1), rows, Yb, nullptr, nullptr);
  hipLaunchKernelGGL(ritz_kernel<BB>, dim3(1), dim3(ritz_threads<BB>()), 0, s, Gp, npb, l, MA, MQ, sigma);
  const Applied a = {Yb, MA, A, rows, l}, q = {Yc, MQ, Q, cols, l};
  hipLaunchKernelGGL(apply_kernel<BB>, dim3(grid_apply, 2), blk, 0, s, a, q);
  return (int)hipGetLastError();
}

}  // namespace msvid

int msvid_block(int l) { return l <= 8 ? 16 : 24; }

static msvid::Layout msvid_layout(int rows, int cols, int b) {
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  msvid::Layout L;
  size_t off = 0;
  // The total is what callers have always been asked for: it once held a transposed copy of Z and the sums of
  // 128-entry chunks.  The sums of today's 256-entry chunks lie in the same place.
  const size_t chunks_a = (size_t)(cols + 127) / 128, chunks_b = (size_t)(rows + 127) / 128;
  const size_t pa = chunks_a * (size_t)rows * b * 4u, pb = chunks_b * (size_t)cols * b * 4u;
  L.p = off; off = up(off + (pa > pb ? pa : pb));
  L.yb = off; off = up(off + (size_t)rows * b * 4u);
  L.yc = off; off = up(off + (size_t)cols * b * 4u);
  L.v1 = off; off = up(off + (size_t)cols * b * 4u);
  const int big = rows > cols ? rows : cols;
  L.nparts_max = (big + msvid::kGramRows - 1) / msvid::kGramRows;
  L.gp = off; off = up(off + (size_t)L.nparts_max * b * b * 4u);
  L.tm = off; off = up(off + (size_t)b * b * 8u);
  L.ma = off; off = up(off + (size_t)b * b * 8u);
  L.mq = off; off = up(off + (size_t)b * b * 8u);
  // (in the room of the copy, which held b x b floats and more)
  L.ctr = off;
  L.tf = up(off + 4u);
  const size_t old_total = up(off + (size_t)rows * cols * 4u), used = up(L.tf + (size_t)b * b * 4u);
  L.total = old_total > used ? old_total : used;
  return L;
}

size_t msvid_ws_bytes(int rows, int cols, int l) { return msvid_layout(rows, cols, msvid_block(l)).total; }

int launch_msvid(const float* Z, int rows, int cols, int64_t ld, int l, int iters, const float* X0, int8_t* S, float* A,
                 float* Q, float* sigma, void* ws, hipStream_t s) {
  const int b = msvid_block(l);
  const msvid::Layout L = msvid_layout(rows, cols, b);
  unsigned char* w = (unsigned char*)ws;
  if (b == 16) return msvid::run<16>(Z, rows, cols, ld, l, iters, X0, S, A, Q, sigma, w, L, s);
  return msvid::run<24>(Z, rows, cols, ld, l, iters, X0, S, A, Q, sigma, w, L, s);
}

}  // namespace mdbf
