// Construction of the Acoustic Similarity Groups (Sec. 2.1, Eq. 1) on gfx950: unit vectors in
// bfloat16 (the exact form: fp16), the V x V cosine similarity as an MFMA contraction with fp32 accumulation that
// is thresholded on the fly (the similarity matrix is never stored), per-token member lists
// sorted ascending, identical sets dropped, and the CSR the verification kernels read.  The
// exact form (pcg_asg_build_exact) uses the same contraction as a filter: pairs whose rounded
// similarity is too close to the threshold to decide are settled by the cosine of the
// embeddings themselves in double, so its groups are those of Eq. (1) as written.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "pcg_device.h"
#include "pcg_kernels.h"

namespace pcg {

namespace {

constexpr size_t kAsgAlign = 256;
size_t asg_align(size_t n) { return (n + kAsgAlign - 1) / kAsgAlign * kAsgAlign; }

// ---------------------------------------------------------------------------------------------
// Unit vectors: emb[v] / ||emb[v]|| in double, rounded once to bfloat16 (nearest, ties to even); for the exact form, whose
// filter they are, to fp32, times 2^8 and to fp16, with what is then subnormal set to 0.
// ---------------------------------------------------------------------------------------------

__device__ __forceinline__ uint16_t round_to_bf16(double x) {
  // the two bfloat16 values that bracket x, found from the truncation of its fp32 image
  const double ax = fabs(x);
  uint32_t lo = __float_as_uint((float) ax) & 0xffff0000u;
  if ((double) __uint_as_float(lo) > ax) lo -= 0x10000u;       // the fp32 image rounded up past lo
  uint32_t hi = lo + 0x10000u;
  if ((double) __uint_as_float(hi) < ax) { lo = hi; hi += 0x10000u; }
  const double dlo = ax - (double) __uint_as_float(lo), dhi = (double) __uint_as_float(hi) - ax;
  const uint32_t pick = dlo < dhi ? lo : (dhi < dlo ? hi : (((lo >> 16) & 1u) ? hi : lo));
  // the sign travels as it is: a negative zero stays a negative zero, as in IEEE rounding
  return (uint16_t) ((pick >> 16) | (__double_as_longlong(x) < 0 ? 0x8000u : 0u));
}

// The same for x = e / norm, with inv = 1 / norm: the product is off by less than an fp32 ulp, so its
// fp32 image decides the rounding unless it lies within two ulps of the middle between two bfloat16
// values; only then is the quotient formed.
__device__ __forceinline__ uint16_t quotient_to_bf16(double e, double norm, double inv) {
  const uint32_t u = __float_as_uint((float) (e * inv));
  const uint32_t low = u & 0xffffu;
  if (low - 0x7ffeu <= 4u) return round_to_bf16(e / norm);
  return (uint16_t) ((u + 0x8000u) >> 16);
}

// The exact form's filter works on the unit vectors in fp16, times 2^8: components up to 256, and what would be
// subnormal (below 2^-22 of the unit) is 0.  Three bits more than bf16 at the same MFMA rate narrow the band of
// pairs that have to be settled in double from 3.4e-3 to 5.5e-4 at 65 536 x 1024 (0.7 M pairs to 0.12 M:
// asg_refine_kernel 472 us to 119); the products take 4 % longer for it (the wider multipliers draw
// more power, which is what sets the clock there).
constexpr float kHalfScale = 256.f;

// An element of a unit vector as the products read it, and back.
template <bool EXACT>
__device__ __forceinline__ uint16_t unit_element(double e, double norm, double inv) {
  if constexpr (!EXACT) return quotient_to_bf16(e, norm, inv);
  const float f = (float) (e * inv) * kHalfScale;
  return fabsf(f) < 0x1p-14f ? (uint16_t) 0 : __builtin_bit_cast(uint16_t, (_Float16) f);
}
template <bool EXACT>
__device__ __forceinline__ double unit_value(uint16_t b) {
  if constexpr (!EXACT) return (double) __uint_as_float((uint32_t) b << 16);
  return (double) ((float) __builtin_bit_cast(_Float16, b) * (1.f / kHalfScale));
}

// EXACT: unit vectors in scaled fp16; norms receives ||emb[v]|| in double, and moved[v] how far
// rounding has moved the unit vector; *worst, the largest of them once asg_setup_kernel has run, is
// cleared for it.  (An atomic maximum here, by every wave at once, took 3.4 of 7.2 us at 2048 tokens.)
// One wave per token; its row (up to kRowRegs * 256 elements, d a multiple of 4) stays in registers
// between the norm and the quotients.  Bound by memory: 268 MB of embeddings and 134 MB of unit
// vectors at 65 536 x 1024 take 72 us (175 with 4-byte loads, the row read twice and a
// division in double per element).
template <bool EXACT>
__global__ __launch_bounds__(256) void asg_normalize_kernel(const float *emb, int32_t V, int32_t d,
                                                            uint16_t *unit, double *norms, float *moved,
                                                            float *worst) {
  constexpr int kRowRegs = 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t v = (int64_t) blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
  if (v >= V) return;                       // whole waves leave together
  const float *e = emb + v * d;
  uint16_t *out = unit + v * d;
  double ss = 0.0, err = 0.0;
  const bool wide = d % 4 == 0 && d <= kRowRegs * 4 * kWave && (((uintptr_t) e | (uintptr_t) (2 * (uintptr_t) out)) & 15) == 0;
  if (wide) {                               // uniform over the wave
    float4 x[kRowRegs];
#pragma unroll
    for (int i = 0; i < kRowRegs; ++i) {
      const int32_t k = 4 * (lane + i * kWave);
      x[i] = k < d ? *reinterpret_cast<const float4 *>(e + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < kRowRegs; ++i)
      ss += ((double) x[i].x * (double) x[i].x + (double) x[i].y * (double) x[i].y) +
            ((double) x[i].z * (double) x[i].z + (double) x[i].w * (double) x[i].w);
    const double norm = sqrt(wave_sum(ss)), inv = norm > 0.0 ? 1.0 / norm : 0.0;
    if (EXACT && lane == 0) norms[v] = norm;
#pragma unroll
    for (int i = 0; i < kRowRegs; ++i) {
      const int32_t k = 4 * (lane + i * kWave);
      if (k >= d) continue;
      const float xs[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
      uint16_t q[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        q[j] = norm > 0.0 ? unit_element<EXACT>((double) xs[j], norm, inv) : (uint16_t) 0;
        if constexpr (EXACT) {
          const double off = unit_value<EXACT>(q[j]) - (double) xs[j] * inv;
          err += off * off;
        }
      }
      *reinterpret_cast<uint2 *>(out + k) =
          make_uint2((uint32_t) q[0] | (uint32_t) q[1] << 16, (uint32_t) q[2] | (uint32_t) q[3] << 16);
    }
  } else {
    for (int32_t k = lane; k < d; k += kWave) ss += (double) e[k] * (double) e[k];
    const double norm = sqrt(wave_sum(ss)), inv = norm > 0.0 ? 1.0 / norm : 0.0;
    if (EXACT && lane == 0) norms[v] = norm;
    for (int32_t k = lane; k < d; k += kWave) {
      const uint16_t q = norm > 0.0 ? unit_element<EXACT>((double) e[k], norm, inv) : (uint16_t) 0;
      out[k] = q;
      if constexpr (EXACT) {
        const double off = unit_value<EXACT>(q) - (double) e[k] * inv;
        err += off * off;
      }
    }
  }
  if constexpr (EXACT) {
    // rounded up.  A row with a NaN or an infinity has no cosine above any threshold and must not widen
    // the band.
    const float mine = __double2float_ru(sqrt(wave_sum(err)) * (1.0 + 0x1p-40));
    if (lane == 0) {
      moved[v] = mine < INFINITY ? mine : 0.f;
      if (v == 0) *worst = 0.f;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Similarity + threshold.  A workgroup of four waves owns a 256 x 256 tile of the similarity
// matrix; each wave a 128 x 128 quarter as 4 x 4 MFMA blocks of 32 x 32 (256 accumulators per
// lane; with smaller wave tiles the operand reads alone saturate LDS).  Both operands are rows
// of the same matrix of unit vectors.  They travel global memory -> LDS directly, 32 columns of
// k per stage, four stages resident: while one is used the loads of the next three are in flight,
// and no register is spent on staging.  The matrix is symmetric: only tiles on or above the
// diagonal are computed, and a pair found off the diagonal is recorded for both of its tokens.
//
// A workgroup stays for its share of the tiles, one after the other, and its loads run on into the next
// tile: with one wave a SIMD nothing hides the first loads of a tile, the threshold pass, or the
// atomics that hand out places in the lists (2 to 4 us a round trip between eight XCDs), unless the same
// wave overlaps them.  65 536 x 1024, a workgroup per tile -> this, with fp16 operands: 4.91 -> 4.24 ms; matrix
// cores busy 48 -> 64 % of the cycles, at a clock that falls from 1.7 to 1.6 GHz as they do (2.3 without
// them: the card's power limit).  Of a tile's 51 thousand cycles the products are 33, the threshold pass 6 and
// waits for barriers, loads and LDS 10.  What each part gave, in cycles of the same case (one workgroup a tile:
// 8.5 million): tiles one after the other in one workgroup, places of a tile's pairs used a tile later 8.0;
// threshold pass of 28 instructions a block and loads from scalar bases 7.2; a stage's operands read a
// whole stage ahead 6.6.  Taken out again: 128 x 256 tiles, two workgroups a compute unit (they
// overlap each other, but read half as much again from the L2: 5.1 ms for 4.9).
// ---------------------------------------------------------------------------------------------

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));      // or eight fp16 values, see mfma
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kSimTile = 256;                 // rows and columns of a workgroup's tile
constexpr int kSimK = 32;                     // k columns per LDS stage: rows of 64 bytes
constexpr int kSimBufs = 4;                   // stages resident in LDS
constexpr int kSimThreads = 256;

template <bool EXACT>
__device__ __forceinline__ floatx16 mfma(bf16x8 a, bf16x8 b, floatx16 c) {
  if constexpr (EXACT)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

constexpr int kSimStageBytes = kSimTile * kSimK * 2;      // one operand of one stage: 16 KiB
constexpr int kSimLoads = 2 * kSimTile / 16 / 4;          // direct-to-LDS loads per wave and stage: 8
constexpr int kSimQueue = 2048;               // pairs a wave can hold back in LDS
constexpr int kSimPatchRows = 16;             // rows of tiles walked column by column (sim_tile)

// Makes a wave's LDS writes visible to its own later reads (no other wave shares the data).
__device__ __forceinline__ void wave_handoff() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A member that the rounded similarity could not decide carries this bit until the exact form
// has settled it (token ids stay below 2^31).
constexpr uint32_t kAsgUnsure = 0x80000000u;

// A wave's pairs on their way to the lists: collected in its own slice of LDS (no other wave touches it), so
// that the round trips of the atomics that hand out the places overlap instead of following one another.
// An entry is the pair's row and column inside the wave's part of the tile, kSimUnsure where marked.
constexpr uint32_t kSimUnsure = 0x80000000u;

// The pair of an entry of the part of a tile that begins at (row0, col0).
__device__ __forceinline__ void sim_pair(uint32_t e, int32_t row0, int32_t col0, int32_t &t, int32_t &v) {
  t = row0 + (int32_t) ((e >> 16) & 0x7fffu);
  v = col0 + (int32_t) (e & 0xffffu);
}

// Places for a pair in the lists of both of its tokens, and the pair into them.
struct SimPlaces { int32_t p0, p1; };
__device__ __forceinline__ SimPlaces sim_ask(int32_t t, int32_t v, int32_t cap, int32_t *count) {
  SimPlaces p;
  p.p0 = atomicAdd(&count[t], 1);
  p.p1 = t != v ? atomicAdd(&count[v], 1) : cap;
  return p;
}
__device__ __forceinline__ void sim_put(const SimPlaces &p, int32_t t, int32_t v, uint32_t e, int32_t cap, int32_t *cand) {
  const uint32_t flag = e & kSimUnsure;
  if (p.p0 < cap) cand[(int64_t) t * cap + p.p0] = (int32_t) ((uint32_t) v | flag);
  if (p.p1 < cap) cand[(int64_t) v * cap + p.p1] = (int32_t) ((uint32_t) t | flag);
}

// Entries [from, n) of a wave's queue, all the way.
__device__ __forceinline__ void sim_flush(const uint32_t *q, uint32_t from, uint32_t n, int32_t row0, int32_t col0,
                                          int32_t cap, int32_t *count, int32_t *cand, int lane) {
  wave_handoff();
  for (uint32_t k = from + lane; k < n; k += kWave) {
    int32_t t, v;
    sim_pair(q[k], row0, col0, t, v);
    sim_put(sim_ask(t, v, cap, count), t, v, q[k], cap, cand);
  }
  wave_handoff();
}

// Tile n of those on or above the diagonal of an nt x nt grid: kSimPatchRows rows of tiles at a time,
// column by column from the diagonal on, so that 32 tiles in a row are a patch of 16 x 2 (8 x 4: 5.2 ms for
// 5.0, 4 x 8: 5.7): the 32 workgroups of an XCD find each other's rows in their L2.
__device__ __forceinline__ int sim_tiles(int nt, int first_row) {      // of the rows of tiles from first_row on
  const int h = nt - first_row < kSimPatchRows ? nt - first_row : kSimPatchRows;
  return h * (h + 1) / 2 + (nt - first_row - h) * h;
}
__device__ __forceinline__ void sim_tile(int n, int nt, int &ti, int &tj) {
  int first = 0;
  for (int k = sim_tiles(nt, 0); n >= k; k = sim_tiles(nt, first)) {
    n -= k;
    first += kSimPatchRows;
  }
  const int h = min(kSimPatchRows, nt - first);
  int c = 0;
  while (c < h && n > c) n -= ++c;             // columns of 1, 2 .. h tiles
  if (c == h) {                                // and of h
    c += n / h;
    n %= h;
  }
  ti = first + n;
  tj = first + c;
}

// Clears what the kernels that follow count in.  EXACT: the largest of moved[0 .. V) into *worst, which
// holds 0: one atomic per workgroup (a non-negative float orders as its bits do).
constexpr int kSetupThreads = 256, kSetupTokens = 4 * kSetupThreads;

template <bool EXACT>
__global__ __launch_bounds__(kSetupThreads) void asg_setup_kernel(int32_t V, const float *moved, float *worst,
                                                                  int32_t *count, int64_t *totals) {
  __shared__ float wave_worst[kSetupThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  if (blockIdx.x == 0 && threadIdx.x < 3) totals[threadIdx.x] = 0;
  float mine = 0.f;
#pragma unroll
  for (int i = 0; i < kSetupTokens / kSetupThreads; ++i) {
    const int32_t t = blockIdx.x * kSetupTokens + i * kSetupThreads + threadIdx.x;
    if (t >= V) continue;
    count[t] = 0;
    if constexpr (EXACT) mine = fmaxf(mine, moved[t]);
  }
  if constexpr (EXACT) {
    mine = wave_max(mine);
    if (lane == 0) wave_worst[wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < kSetupThreads / kWave; ++w) mine = fmaxf(mine, wave_worst[w]);
      atomicMax(reinterpret_cast<uint32_t *>(worst), __float_as_uint(mine));
    }
  }
}

// Waits until at most N of this wave's vector-memory operations are still in flight.
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Meets the other waves of the workgroup without the fence of __syncthreads(), which would wait
// for every load still in flight.  The caller has waited for exactly what it needs.
__device__ __forceinline__ void bare_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// How far the fp32-accumulated dot product of two rounded unit vectors can lie from the cosine of
// the vectors they were rounded from, if rounding moved neither by more than e: the exact dot product
// of the rounded ones lies within 2 e + e^2 (Cauchy-Schwarz), and the d additions in fp32 add at most
// d 2^-23 of the vectors' lengths (a rounding, or a truncation, of each partial sum).  2^-20 covers
// the roundings of this expression and of the threshold plus or minus it.
__device__ __forceinline__ float asg_rounding_band(int32_t d, float e) {
  return (2.f * e + e * e) + (float) d * 0x1p-23f * (1.f + e) * (1.f + e) + 0x1p-20f;
}

// EXACT: pairs above theta minus the rounding band are candidates, and those not above theta plus
// the band are marked kAsgUnsure for asg_refine_kernel.
template <bool EXACT>
__global__ __launch_bounds__(kSimThreads, 1) void asg_similarity_kernel(
    const uint16_t *__restrict__ unit, int32_t V, int32_t d, float theta, const float *worst,
    int32_t cap, int32_t ntiles, int32_t run, int32_t *count, int32_t *cand) {
  float theta_hi = theta;
  if constexpr (EXACT) {
    const float band = asg_rounding_band(d, *worst);
    theta_hi = (theta + band) * (kHalfScale * kHalfScale);
    theta = (theta - band) * (kHalfScale * kHalfScale);
  }
  const int nt = (V + kSimTile - 1) / kSimTile;
  // [buffer][operand][row][64 bytes].  A 16-byte LDS read is served 16 lanes at a time, free of
  // conflicts when their addresses differ modulo 256 bytes; the four 16-byte chunks of a row are
  // therefore stored at position chunk ^ ((row >> 2) & 3), which spreads the same chunk of 16
  // consecutive rows over all 16 slots.
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kSimBufs * 2 * kSimStageBytes];
  __shared__ uint32_t queue[kSimThreads / kWave][kSimQueue];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  uint32_t *q = queue[wave];

  // Workgroups go to the 8 XCDs round-robin; the `run` of one XCD take `run` tiles in a row at a time.
  const int step_tiles = 8 * run;
  int n = (blockIdx.x & 7) * run + (int) (blockIdx.x >> 3);
  if (n >= ntiles) return;

  // Direct-to-LDS loads: one instruction of a wave fills 1 KiB = 16 rows, lane i the 16 bytes at
  // row i / 4, position i % 4.  Wave w brings rows 64 w .. 64 w + 63 of both operands.  The loads run ahead
  // of the products by kSimBufs stages, across the tiles: they have a place of their own.
  int ld_n = n, ld_k = 0;
  uint32_t src[kSimLoads];              // byte offsets of this lane's rows and chunk (V d < 2^31 elements)
  auto aim = [&]() {
    int ti, tj;
    sim_tile(ld_n, nt, ti, tj);
    const int r = lane >> 2, p = lane & 3;
    const int c = p ^ ((r >> 2) & 3);                  // the chunk of the row that belongs there
#pragma unroll
    for (int j = 0; j < kSimLoads / 2; ++j) {
      const int row = wave * 64 + j * 16 + r;
      // rows past the end of the matrix re-read the last row; their results are never recorded
      src[j] = 2u * (uint32_t) (min(ti * kSimTile + row, V - 1) * d + c * 8);
      src[kSimLoads / 2 + j] = 2u * (uint32_t) (min(tj * kSimTile + row, V - 1) * d + c * 8);
    }
  };
  aim();
  auto load = [&](int j, unsigned char *stage) {
    unsigned char *dst = stage + (j & 1) * kSimStageBytes + wave * 64 * 64 + (j >> 1) * 1024;
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void *) (reinterpret_cast<const char *>(unit + ld_k) +
                                                          src[(j & 1) * (kSimLoads / 2) + (j >> 1)]),
        (__attribute__((address_space(3))) void *) dst, 16, 0, 0);
  };
  // On to the next stage; past the last tile its stages are repeated: nobody reads what they bring.
  auto advance = [&]() {
    ld_k += kSimK;
    if (ld_k == d) {
      ld_k = 0;
      if (ld_n + step_tiles < ntiles) {
        ld_n += step_tiles;
        aim();
      }
    }
  };

  floatx16 acc[4][4];
  // operand reads of this lane: row lane % 32 of a block, k half lane / 32 of a 16-column step
  const int fr = lane & 31, fh = lane >> 5;
  const int sw = (fr >> 2) & 3;                        // block rows start at multiples of 32
  const int a_row = (wm * 128 + fr) * 64, b_row = (wn * 128 + fr) * 64 + kSimStageBytes;
  const int pos0 = ((0 + fh) ^ sw) * 16, pos1 = ((2 + fh) ^ sw) * 16;

  // Operands of two stages, each of two 16-column steps: one in use, the next on its way from LDS.
  bf16x8 fa[2][2][4], fb[2][2][4];
  auto read = [&](bf16x8 (&a)[2][4], bf16x8 (&b)[2][4], const unsigned char *buf, int k) {      // k: 0 .. 15
    const int pos = k < 8 ? pos0 : pos1, i = k & 3;
    if ((k & 7) < 4) a[k >> 3][i] = *reinterpret_cast<const bf16x8 *>(buf + a_row + pos + i * 32 * 64);
    else b[k >> 3][i] = *reinterpret_cast<const bf16x8 *>(buf + b_row + pos + i * 32 * 64);
  };
  unsigned char *cur = lds, *const end = lds + kSimBufs * 2 * kSimStageBytes;
  // One stage: 32 MFMAs on operand set P.  Behind the first 24 of them, one at a time, the next stage's operands
  // are read from LDS into the other set and the loads of the stage after those on their way are
  // started.  The LDS and memory queues are short: instructions issued in a burst would hold the
  // MFMAs behind them back, and with one wave a SIMD nothing else runs while one waits: the last
  // read has eight MFMAs to come in.  The order is pinned.  FIRST: the sums begin with these products.
  auto stage = [&](auto set, auto first) {
    constexpr int P = decltype(set)::value;
    constexpr bool kFirst = decltype(first)::value;
    unsigned char *nxt = cur + 2 * kSimStageBytes;
    if (nxt == end) nxt = lds;
    // This wave's loads of the next stage have landed once only those of the two stages behind it
    // are out; past the barrier everyone's have, and nobody reads buffer `cur` any more (this stage's
    // operands are in registers).
    wait_vm<(kSimBufs - 2) * kSimLoads>();
    bare_barrier();
#pragma unroll
    for (int m = 0; m < 32; ++m) {
      const int i = (m >> 2) & 3, j = m & 3;
      if (kFirst && m < 16) acc[i][j] = mfma<EXACT>(fa[P][0][i], fb[P][0][j], floatx16{});
      else acc[i][j] = mfma<EXACT>(fa[P][m >> 4][i], fb[P][m >> 4][j], acc[i][j]);
      if (m < 24) {
        __builtin_amdgcn_sched_barrier(0);
        if (m % 3 == 2) load(m / 3, cur);
        else read(fa[1 - P], fb[1 - P], nxt, m / 3 * 2 + m % 3);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    advance();
    cur = nxt;
  };
  constexpr std::integral_constant<int, 0> kEven{};
  constexpr std::integral_constant<int, 1> kOdd{};

#pragma unroll
  for (int s = 0; s < kSimBufs; ++s) {
#pragma unroll
    for (int j = 0; j < kSimLoads; ++j) load(j, lds + s * 2 * kSimStageBytes);
    advance();
  }
  wait_vm<(kSimBufs - 1) * kSimLoads>();    // stage 0 is in; the ones behind it may be on their way
  bare_barrier();
#pragma unroll
  for (int k = 0; k < 16; ++k) read(fa[0], fb[0], lds, k);

  // the last pairs of a tile: their places are asked for at its end and used at the end of the next
  SimPlaces late = {cap, cap};
  int32_t late_t = 0, late_v = 0;
  uint32_t late_e = 0;
  const int nstages = d / kSimK;        // even: d is a multiple of 64
  for (;; n += step_tiles) {
    stage(kEven, std::true_type{});
    stage(kOdd, std::false_type{});
#pragma unroll 1
    for (int s = 2; s < nstages; s += 2) {
      stage(kEven, std::false_type{});
      stage(kOdd, std::false_type{});
    }

    // Threshold (Eq. 1)
    int ti, tj;
    sim_tile(n, nt, ti, tj);
    const int32_t row0 = ti * kSimTile + wm * 128, col0 = tj * kSimTile + wn * 128;
    uint32_t nq = 0;                                   // uniform over the wave
    auto push = [&](bool mine, uint32_t entry) {
      const unsigned long long who = __builtin_amdgcn_ballot_w64(mine);
      if (mine)
        q[nq + __builtin_amdgcn_mbcnt_hi((uint32_t) (who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t) who, 0))] = entry;
      nq += (uint32_t) __popcll(who);
    };
    // Accumulator r of a lane is row 8 (r / 4) + 4 (lane / 32) + r % 4 and column lane % 32 of its 32 x 32
    // block.  Most blocks hold nothing above the threshold: one maximum per lane and a ballot tell.  A queue
    // that cannot take what a block may hold is emptied, and the blocks go on from there.
    int done = 0;
    while (true) {
#pragma unroll
      for (int b = 0; b < 16; ++b) {
        __builtin_amdgcn_sched_barrier(0);             // one block's sums at a time in registers
        if (done != b || nq > (uint32_t) (kSimQueue - 32 * 32)) continue;
        ++done;
        asm volatile("" : "+a"(acc[b >> 2][b & 3]));   // stays where the products left it until here
        const floatx16 a = acc[b >> 2][b & 3];
        float m = fmaxf(a[0], a[1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) m = fmaxf(fmaxf(m, a[r]), a[r + 1]);
        if (__builtin_amdgcn_ballot_w64(m > theta) == 0) continue;
        const int32_t lt = (b >> 2) * 32 + 4 * (lane >> 5), lv = (b & 3) * 32 + (lane & 31);
        const int32_t room = col0 + lv < V ? min(V, col0 + lv) - (row0 + lt) : 0;    // rows below V and the diagonal
        uint32_t hits = 0, sure = 0;                   // bit 15 - r
#pragma unroll
        for (int r = 0; r < 16; ++r) hits = (hits + (a[r] > theta ? 1u : 0u)) + hits;
        if constexpr (EXACT) {
#pragma unroll
          for (int r = 0; r < 16; ++r) sure = (sure + (a[r] > theta_hi ? 1u : 0u)) + sure;
        } else {
          sure = hits;
        }
        while (__builtin_amdgcn_ballot_w64(hits != 0) != 0) {      // every lane its own next one
          const int k = __builtin_ctz(hits | 0x10000u), r = 15 - k, at = 8 * (r >> 2) + (r & 3);
          push(hits != 0 && at < room, (uint32_t) (lt + at) << 16 | (uint32_t) lv | (((sure >> k) & 1u) ? 0u : kSimUnsure));
          hits &= hits - 1;
        }
      }
      if (done == 16) break;
      sim_flush(q, 0, nq, row0, col0, cap, count, cand, lane);
      nq = 0;
    }
    // a token is always a member of its own group, whatever the rounded product says
    if (row0 == col0) {
      if (nq > (uint32_t) (kSimQueue - 128)) {
        sim_flush(q, 0, nq, row0, col0, cap, count, cand, lane);
        nq = 0;
      }
      for (int k = 0; k < 128; k += kWave)
        push(row0 + k + lane < V, (uint32_t) (k + lane) << 16 | (uint32_t) (k + lane));
    }
    sim_flush(q, kWave, nq, row0, col0, cap, count, cand, lane);
    sim_put(late, late_t, late_v, late_e, cap, cand);
    late.p0 = late.p1 = cap;
    if ((uint32_t) lane < nq) {
      late_e = q[lane];
      sim_pair(late_e, row0, col0, late_t, late_v);
      late = sim_ask(late_t, late_v, cap, count);
    }
    if (n + step_tiles >= ntiles) break;
  }
  wait_vm<0>();                         // the loads past the end land while the LDS is still this workgroup's
  sim_put(late, late_t, late_v, late_e, cap, cand);
}

// ---------------------------------------------------------------------------------------------
// Exact form: the pairs marked kAsgUnsure are settled by Eq. (1) itself -- the dot product of the two
// float32 embeddings and their norms, all in double, strict > theta.  A pair stands in both tokens'
// lists; the wave of its smaller token decides it and writes the outcome into both: the plain token
// id, or kAsgRemoved (asg_sort_kernel closes the gaps).  No two waves write the same entry, and a
// wave's own pairs are those with a larger token, whatever has happened to the others it reads.
// The wave's own row stays in registers (up to kRowRegs * 256 elements), the other's comes from
// memory, with its norm and the first 64 entries of its list, while the pair before is summed.  Bound
// by the gather of those rows, 4 d bytes a pair: 65 536 x 1024, 0.12 M undecided pairs, 119 us (with the
// 0.7 M of a filter in bf16 471, and 1711 when both tokens' waves computed each pair and read both rows for
// it).  With few tokens, all of whose waves run at once, it is the longest chain of pairs that counts: 2048 x 128,
// bf16 filter, 5.1 us (5.3 with the list fetched after the sum).
// Lists that did not fit into cap stay undecided: their count stays above cap and the call reports
// PCG_ERR_CAPACITY.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kAsgRemoved = 0xffffffffu;

__global__ __launch_bounds__(256) void asg_refine_kernel(const float *__restrict__ emb,
                                                         const double *__restrict__ norms, int32_t V,
                                                         int32_t d, double theta, int32_t cap,
                                                         const int32_t *__restrict__ count,
                                                         int32_t *cand) {
  constexpr int kRowRegs = 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t t = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
  if (t >= V) return;                       // whole waves leave together
  const int32_t found = count[t];
  if (found > cap) return;
  int32_t *row = cand + (int64_t) t * cap;
  const float *et = emb + (int64_t) t * d;
  const double nt = norms[t];
  float4 own[kRowRegs];                     // d is a multiple of 64
#pragma unroll
  for (int i = 0; i < kRowRegs; ++i) {
    const int32_t k = 4 * (lane + i * kWave);
    own[i] = k < d ? *reinterpret_cast<const float4 *>(et + k) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  auto product = [](const float4 a, const float4 b) {
    return ((double) a.x * (double) b.x + (double) a.y * (double) b.y) +
           ((double) a.z * (double) b.z + (double) a.w * (double) b.w);
  };
  struct Other {
    float4 row[kRowRegs];
    double norm;
    int32_t found;
    uint32_t first;                         // entry `lane` of its list, if it has one there
  };
  // This wave alone writes the entry it looks for in the other's list, so that one fetched early is as
  // good as one fetched late, whatever happens to its neighbours.
  auto fetch = [&](int32_t v, Other &o) {
    const float *ev = emb + (int64_t) v * d;
#pragma unroll
    for (int i = 0; i < kRowRegs; ++i) {
      const int32_t k = 4 * (lane + i * kWave);
      o.row[i] = k < d ? *reinterpret_cast<const float4 *>(ev + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    o.norm = norms[v];
    o.found = count[v];
    o.first = lane < cap ? (uint32_t) cand[(int64_t) v * cap + lane] : 0u;
  };
  for (int32_t c0 = 0; c0 < found; c0 += kWave) {
    const int32_t k = c0 + lane;
    const uint32_t raw = k < found ? (uint32_t) row[k] : 0u;
    const int32_t entry = (int32_t) (raw & ~kAsgUnsure);
    unsigned long long mine = __ballot(raw != kAsgRemoved && (raw & kAsgUnsure) != 0 && entry > t);
    if (mine == 0) continue;                           // uniform over the wave, as everything below
    bool member = false;
    int l = __ffsll((long long) mine) - 1;
    Other o;
    fetch(__builtin_amdgcn_readlane(entry, l), o);
    const unsigned long long all = mine;
    while (true) {
      mine &= mine - 1;
      const int32_t v = __builtin_amdgcn_readlane(entry, l);
      const Other cur = o;
      int ln = 0;
      if (mine) {                                      // the next row is on its way behind this one
        ln = __ffsll((long long) mine) - 1;
        fetch(__builtin_amdgcn_readlane(entry, ln), o);
      }
      double dot = 0.0;
#pragma unroll
      for (int i = 0; i < kRowRegs; ++i) dot += product(own[i], cur.row[i]);
      for (int32_t j = 4 * (lane + kRowRegs * kWave); j < d; j += 4 * kWave)
        dot += product(*reinterpret_cast<const float4 *>(et + j),
                       *reinterpret_cast<const float4 *>(emb + (int64_t) v * d + j));
      dot = wave_sum(dot);
      const double cosine = (nt > 0.0 && cur.norm > 0.0) ? dot / (nt * cur.norm) : 0.0;
      const bool is_member = cosine > theta;
      if (lane == l) member = is_member;
      // the same pair in the other token's list
      const int32_t theirs = min(cur.found, cap);
      int32_t *other = cand + (int64_t) v * cap;
      const uint32_t mark = (uint32_t) t | kAsgUnsure;
      const int32_t outcome = is_member ? t : (int32_t) kAsgRemoved;
      if (lane < theirs && cur.first == mark) other[lane] = outcome;
      for (int32_t j = lane + kWave; j < theirs; j += kWave)
        if ((uint32_t) other[j] == mark) other[j] = outcome;
      if (!mine) break;
      l = ln;
    }
    if ((all >> lane) & 1ull) row[k] = member ? entry : (int32_t) kAsgRemoved;
  }
}

// ---------------------------------------------------------------------------------------------
// Per token: members ascending (bitonic sort in LDS), a hash of the set, its size.
// ---------------------------------------------------------------------------------------------

constexpr int kSortThreads = 256;             // four waves, one token each
constexpr int kAsgMaxCap = PCG_ASG_MAX_CAP;

__device__ __forceinline__ uint64_t mix64(uint64_t x) {   // splitmix64 finaliser
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// One wave per token: its members ascending, an order-independent hash of the set, its size; entries
// marked kAsgRemoved are dropped, what is still marked kAsgUnsure (only where some list did not fit)
// becomes a plain token id again, since the kernels that follow index with it.  Up to 64 members are
// ranked against each other in registers, larger sets go through a bitonic sort in the wave's own
// slice of LDS (153 us for 65 536 sets of 26 members on average, now 41).  cap2 = cap rounded up
// to a power of two, at least 64; the kernel is launched with 4 * cap2 * 4 bytes of dynamic LDS.
__global__ __launch_bounds__(kSortThreads) void asg_sort_kernel(int32_t V, int32_t cap, int32_t cap2,
                                                                const int32_t *count, int32_t *cand,
                                                                int32_t *size, uint64_t *hash) {
  extern __shared__ int32_t sort_lds[];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  const int32_t t = blockIdx.x * (kSortThreads / kWave) + wave;
  if (t >= V) return;                       // whole waves leave together; no workgroup barrier below
  int32_t *key = sort_lds + wave * cap2;
  const int32_t have = min(count[t], cap);
  int32_t *row = cand + (int64_t) t * cap;
  int32_t n = 0;
  if (have <= kWave) {
    // every member's place is the number of members below it (they are distinct)
    const uint32_t raw = lane < have ? (uint32_t) row[lane] : kAsgRemoved;
    const bool valid = raw != kAsgRemoved;
    const int32_t x = valid ? (int32_t) (raw & ~kAsgUnsure) : INT32_MAX;
    n = __popcll(__ballot(valid));
    int32_t rank = 0;
    for (int32_t j = 0; j < have; ++j) rank += __builtin_amdgcn_readlane(x, j) < x;
    if (valid) key[rank] = x;
  } else {
    int32_t n2 = 1;
    while (n2 < have) n2 <<= 1;
    for (int32_t k0 = 0; k0 < n2; k0 += kWave) {
      const int32_t k = k0 + lane;
      const uint32_t raw = k < have ? (uint32_t) row[k] : kAsgRemoved;
      const bool valid = raw != kAsgRemoved;
      key[k] = valid ? (int32_t) (raw & ~kAsgUnsure) : INT32_MAX;
      n += __popcll(__ballot(valid));
    }
    wave_handoff();
    for (int32_t len = 2; len <= n2; len <<= 1)
      for (int32_t step = len >> 1; step > 0; step >>= 1) {
        for (int32_t k = lane; k < n2; k += kWave) {
          const int32_t other = k ^ step;
          if (other > k) {
            const bool up = (k & len) == 0;
            const int32_t x = key[k], y = key[other];
            if ((x > y) == up) { key[k] = y; key[other] = x; }
          }
        }
        wave_handoff();
      }
  }
  wave_handoff();
  uint64_t h = 0;
  for (int32_t k = lane; k < n; k += kWave) {
    row[k] = key[k];
    h += mix64((uint64_t) key[k]);
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) h += __shfl_xor(h, o, kWave);
  if (lane == 0) {
    hash[t] = h;
    size[t] = n;
  }
}

// keep[t] = 0 iff an earlier token has exactly the same set.  Such a token is a member of G(t)
// (every set holds its own token), so only the members below t are looked at.
__global__ __launch_bounds__(256) void asg_dedup_kernel(int32_t V, int32_t cap, const int32_t *cand,
                                                        const int32_t *size, const uint64_t *hash,
                                                        int32_t *keep) {
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t t = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
  if (t >= V) return;
  const int32_t n = size[t];
  const uint64_t h = hash[t];
  const int32_t *mine = cand + (int64_t) t * cap;
  int dup = 0;
  // 64 members at a time, one per lane, are compared by size and hash; a set that agrees in both is
  // then compared member by member
  for (int32_t j0 = 0; j0 < n && !dup; j0 += kWave) {
    const int32_t j = j0 + lane;
    const int32_t m = j < n ? mine[j] : INT32_MAX;
    unsigned long long alike = __ballot(m < t && size[m < t ? m : t] == n && hash[m < t ? m : t] == h);
    while (alike && !dup) {                    // uniform over the wave
      const int32_t other = __builtin_amdgcn_readlane(m, __ffsll((long long) alike) - 1);
      alike &= alike - 1;
      const int32_t *theirs = cand + (int64_t) other * cap;
      bool same = true;
      for (int32_t k = lane; k < n; k += kWave) same = same && mine[k] == theirs[k];
      dup = __all(same);
    }
    if (__ballot(m >= t)) break;               // ascending: no further members below t
  }
  if (lane == 0) keep[t] = !dup;
}

// Exclusive scans over the tokens: gid[t] = kept tokens before t, off[t] = members of kept tokens
// before t; totals[0] = G, totals[1] = nnz, totals[2] = the largest set.  A workgroup per 1024 tokens scans its
// own and needs the sums of those before them: from asg_count_kernel, which leaves every block's, or,
// where that are few tokens, by reading them all (a launch costs more).  (One workgroup walking over
// all tokens took 132 us at V = 65 536; the two take 11.  2048 tokens: 5.4 us, 4.6 in one launch.)
// A token's two counts travel as one double: 1 + 2^11 size; sums over 1024 tokens stay exact.
constexpr int kScanThreads = 1024;
constexpr unsigned kScanAloneBlocks = 8;    // without asg_count_kernel up to 8192 tokens
constexpr double kScanUnit = 2048.0;

__device__ __forceinline__ double scan_item(int32_t t, int32_t V, const int32_t *keep, const int32_t *size) {
  return t < V && keep[t] != 0 ? 1.0 + kScanUnit * (double) size[t] : 0.0;
}

// Sum over the workgroup (fixed order); every thread gets it.
__device__ __forceinline__ double scan_block_sum(double v, double *wave_tot) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  v = wave_sum(v);
  if (lane == 0) wave_tot[wave] = v;
  __syncthreads();
  const double w = wave_sum(lane < kScanThreads / kWave ? wave_tot[lane] : 0.0);
  __syncthreads();
  return w;
}

__global__ __launch_bounds__(kScanThreads) void asg_count_kernel(int32_t V, const int32_t *keep,
                                                                 const int32_t *size, uint64_t *counts) {
  __shared__ double wave_tot[kScanThreads / kWave];
  const double all = scan_block_sum(scan_item(blockIdx.x * kScanThreads + threadIdx.x, V, keep, size), wave_tot);
  if (threadIdx.x == 0) counts[blockIdx.x] = (uint64_t) all;
}

__global__ __launch_bounds__(kScanThreads) void asg_scan_kernel(int32_t V, const int32_t *keep,
                                                                const int32_t *size, const uint64_t *counts,
                                                                const int32_t *count, int32_t cap, int32_t *gid,
                                                                int64_t *off, int64_t *totals) {
  __shared__ int32_t wave_largest[kScanThreads / kWave];
  __shared__ double wave_tot[kScanThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  double g0 = 0.0, n0 = 0.0;                 // of the blocks before this one
  if (counts) {                              // uniform
    for (int32_t k = threadIdx.x; k < (int32_t) blockIdx.x; k += kScanThreads) {
      const uint64_t c = counts[k];
      g0 += (double) (c & 2047);
      n0 += (double) (c >> 11);
    }
  } else {
    for (int32_t k = threadIdx.x; k < (int32_t) blockIdx.x * kScanThreads; k += kScanThreads) {
      g0 += keep[k] != 0 ? 1.0 : 0.0;
      n0 += keep[k] != 0 ? (double) size[k] : 0.0;
    }
  }
  g0 = scan_block_sum(g0, wave_tot);
  n0 = scan_block_sum(n0, wave_tot);
  const int32_t t = blockIdx.x * kScanThreads + threadIdx.x;
  const double mine = scan_item(t, V, keep, size);
  const double inc = wave_scan(mine);
  if (lane == kWave - 1) wave_tot[wave] = inc;
  __syncthreads();
  const double tot = lane < kScanThreads / kWave ? wave_tot[lane] : 0.0;
  const double upto = wave_scan(tot);
  const double before = read_lane(upto, wave) - read_lane(tot, wave) + (inc - mine);
  const uint64_t e = (uint64_t) before;
  if (t < V) {
    gid[t] = (int32_t) ((int64_t) g0 + (int64_t) (e & 2047));
    off[t] = (int64_t) n0 + (int64_t) (e >> 11);
  }
  if (t == V - 1) {
    const uint64_t c = (uint64_t) (before + mine);
    totals[0] = (int64_t) g0 + (int64_t) (c & 2047);
    totals[1] = (int64_t) n0 + (int64_t) (c >> 11);
  }
  // The largest set; where one did not fit, what was found for it.  One atomic per workgroup: one per
  // token, by the kernel that sorts, took 39 of its 42 us at 4096 tokens.
  int32_t largest = 0;
  if (t < V) {
    const int32_t found = count[t];
    largest = found > cap ? found : size[t];
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) largest = max(largest, __shfl_xor(largest, o, kWave));
  if (lane == 0) wave_largest[wave] = largest;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kScanThreads / kWave; ++w) largest = max(largest, wave_largest[w]);
    atomicMax(reinterpret_cast<int32_t *>(totals + 2), largest);
  }
}

// The CSR, and N(t): similarity is symmetric, so the groups that hold t are those of its own members, less the
// dropped ones.  Every wave counts those of its token (an atomic per member on mult[] took 73 us at
// 65 536 tokens of 26 members; this 22).  Writes nothing where a set or the whole did not fit: the host learns of that with
// the sizes, behind this kernel, and so waits once, not twice (2048 x 128: the call 104 -> 87 us, 12 000 x 256 170 -> 156).
__global__ __launch_bounds__(256) void asg_compact_kernel(int32_t V, int32_t cap, const int32_t *cand,
                                                          const int32_t *size, const int32_t *keep,
                                                          const int32_t *gid, const int64_t *off,
                                                          const int64_t *totals, int64_t members_capacity,
                                                          int32_t *row_ptr, int32_t *members, int32_t *mult,
                                                          int32_t *seed_of) {
  if (*reinterpret_cast<const int32_t *>(totals + 2) > cap || totals[1] > members_capacity || totals[1] > INT32_MAX) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t t = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
  if (t >= V) return;
  if (t == 0 && lane == 0) row_ptr[totals[0]] = (int32_t) totals[1];
  const bool kept = keep[t] != 0;
  const int32_t n = size[t], g = gid[t];
  const int64_t o = off[t];
  const int32_t *mine = cand + (int64_t) t * cap;
  int32_t holders = 0;                       // uniform
  for (int32_t k0 = 0; k0 < n; k0 += kWave) {
    const int32_t k = k0 + lane;
    const int32_t m = k < n ? mine[k] : 0;
    if (k < n && kept) members[o + k] = m;
    holders += (int32_t) __popcll(__ballot(k < n && keep[m] != 0));
  }
  if (lane == 0) mult[t] = holders;
  if (!kept) return;
  if (lane == 0) {
    row_ptr[g] = (int32_t) o;
    if (seed_of) seed_of[g] = t;
  }
}

}  // namespace

}  // namespace pcg

using namespace pcg;

namespace {

size_t asg_core_workspace_bytes(size_t v, int32_t cap) {
  return asg_align(v * 4) /* count */ + asg_align(v * (size_t) cap * 4) /* cand */ +
         asg_align(v * 4) /* size */ + asg_align(v * 8) /* hash */ + asg_align(v * 4) /* keep */ +
         asg_align(v * 4) /* gid */ + asg_align(v * 8) /* off */ + asg_align(64) /* totals */;
}

// The groups from the unit vectors; with emb (and norms, workspace of the caller) the exact form.
int asg_build_impl(const float *emb, double *norms, uint16_t *unit_out, const uint16_t *unit_bf16,
                   int32_t V, int32_t d, float theta, int32_t cap, int32_t *row_ptr, int32_t *members,
                   int64_t members_capacity, int32_t *mult, int32_t *seed_of, int32_t *out_G,
                   int64_t *out_nnz, int32_t *out_max_size, char *ws, hipStream_t stream) {
  const size_t v = (size_t) V;
  int32_t *count = (int32_t *) ws; ws += asg_align(v * 4);
  int32_t *cand = (int32_t *) ws; ws += asg_align(v * (size_t) cap * 4);
  int32_t *size = (int32_t *) ws; ws += asg_align(v * 4);
  uint64_t *hash = (uint64_t *) ws; ws += asg_align(v * 8);
  int32_t *keep = (int32_t *) ws; ws += asg_align(v * 4);
  int32_t *gid = (int32_t *) ws; ws += asg_align(v * 4);
  int64_t *off = (int64_t *) ws; ws += asg_align(v * 8);
  int64_t *totals = (int64_t *) ws;          // [0] G, [1] nnz, [2] (as int32) largest set found, [3] worst rounding

  auto fail = [](hipError_t e) { return record_hip_error(e); };
  hipError_t e;
  const unsigned wb = (unsigned) ((v + 3) / 4), ub = (unsigned) ((v + kSetupTokens - 1) / kSetupTokens);
  const int nt = (V + kSimTile - 1) / kSimTile;
  if (nt > 65535) return PCG_ERR_BAD_SHAPE;            // their tiles no longer count in 31 bits
  const int tiles = (int) ((int64_t) nt * (nt + 1) / 2);
  // a workgroup for every compute unit, 32 of an XCD on tiles in a row
  const int run = std::min(32, (tiles + 7) / 8);
  const unsigned sim_grid = (unsigned) (8 * run);
  if (emb) {
    float *worst = (float *) (totals + 3);
    float *moved = (float *) gid;            // read before gid is written
    asg_normalize_kernel<true><<<wb, 256, 0, stream>>>(emb, V, d, unit_out, norms, moved, worst);
    asg_setup_kernel<true><<<ub, kSetupThreads, 0, stream>>>(V, moved, worst, count, totals);
    asg_similarity_kernel<true><<<sim_grid, kSimThreads, 0, stream>>>(
        unit_out, V, d, theta, worst, cap, tiles, run, count, cand);
    asg_refine_kernel<<<wb, 256, 0, stream>>>(emb, norms, V, d, (double) theta, cap, count, cand);
  } else {
    asg_setup_kernel<false><<<ub, kSetupThreads, 0, stream>>>(V, nullptr, nullptr, count, totals);
    asg_similarity_kernel<false><<<sim_grid, kSimThreads, 0, stream>>>(
        unit_bf16, V, d, theta, nullptr, cap, tiles, run, count, cand);
  }
  if ((e = hipGetLastError()) != hipSuccess) return fail(e);
  int32_t cap2 = kWave;
  while (cap2 < cap) cap2 <<= 1;
  asg_sort_kernel<<<wb, kSortThreads, (size_t) (kSortThreads / kWave) * cap2 * sizeof(int32_t), stream>>>(
      V, cap, cap2, count, cand, size, hash);
  asg_dedup_kernel<<<wb, 256, 0, stream>>>(V, cap, cand, size, hash, keep);
  const unsigned sb = (unsigned) ((v + kScanThreads - 1) / kScanThreads);
  uint64_t *counts = sb > kScanAloneBlocks ? hash : nullptr;      // hash: read for the last time by the kernel before
  if (counts) asg_count_kernel<<<sb, kScanThreads, 0, stream>>>(V, keep, size, counts);
  asg_scan_kernel<<<sb, kScanThreads, 0, stream>>>(V, keep, size, counts, count, cap, gid, off, totals);
  if ((e = hipGetLastError()) != hipSuccess) return fail(e);
  asg_compact_kernel<<<wb, 256, 0, stream>>>(V, cap, cand, size, keep, gid, off, totals, members_capacity, row_ptr,
                                             members, mult, seed_of);
  if ((e = hipGetLastError()) != hipSuccess) return fail(e);
  int64_t host_totals[3] = {0, 0, 0};
  if ((e = hipMemcpyAsync(host_totals, totals, sizeof host_totals, hipMemcpyDeviceToHost, stream)) !=
      hipSuccess)
    return fail(e);
  if ((e = hipStreamSynchronize(stream)) != hipSuccess) return fail(e);
  int32_t largest = 0;
  std::memcpy(&largest, &host_totals[2], sizeof largest);
  *out_G = (int32_t) host_totals[0];
  *out_nnz = host_totals[1];
  *out_max_size = largest;
  if (largest > cap) return PCG_ERR_CAPACITY;          // some set did not fit: nothing has been written
  if (host_totals[1] > members_capacity || host_totals[1] > INT32_MAX) return PCG_ERR_CAPACITY;
  return PCG_OK;
}

int asg_check_outputs(int32_t V, int32_t d, float theta, int32_t cap, const int32_t *row_ptr,
                      const int32_t *members, int64_t members_capacity, const int32_t *mult,
                      const void *workspace) {
  if (V < 1 || d < 64 || d % 64 || cap < 1 || cap > kAsgMaxCap || members_capacity < 1 ||
      (int64_t) V * d > INT32_MAX || !std::isfinite(theta))
    return PCG_ERR_BAD_SHAPE;
  if (((uintptr_t) workspace % kAsgAlign) || ((uintptr_t) row_ptr % 4) || ((uintptr_t) members % 4) ||
      ((uintptr_t) mult % 4))
    return PCG_ERR_MISALIGNED;
  return PCG_OK;
}

}  // namespace

extern "C" {

int pcg_asg_normalize(const float *emb, int32_t V, int32_t d, uint16_t *unit_bf16,
                      void *hip_stream) {
  if (!emb || !unit_bf16) return PCG_ERR_NULL_ARG;
  if (V < 1 || d < 1) return PCG_ERR_BAD_SHAPE;
  if (((uintptr_t) emb % 4) || ((uintptr_t) unit_bf16 % 2)) return PCG_ERR_MISALIGNED;
  hipStream_t stream = (hipStream_t) hip_stream;
  asg_normalize_kernel<false><<<(unsigned) ((V + 3) / 4), 256, 0, stream>>>(emb, V, d, unit_bf16, nullptr, nullptr,
                                                                            nullptr);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PCG_OK : record_hip_error(e);
}

size_t pcg_asg_build_workspace_bytes(int32_t V, int32_t cap) {
  if (V < 1 || cap < 1 || cap > kAsgMaxCap) return 0;
  return asg_core_workspace_bytes((size_t) V, cap) + kAsgAlign;
}

int pcg_asg_build(const uint16_t *unit_bf16, int32_t V, int32_t d, float theta, int32_t cap,
                  int32_t *row_ptr, int32_t *members, int64_t members_capacity, int32_t *mult,
                  int32_t *seed_of, int32_t *out_G, int64_t *out_nnz, int32_t *out_max_size,
                  void *workspace, size_t workspace_bytes, void *hip_stream) {
  if (!unit_bf16 || !row_ptr || !members || !mult || !out_G || !out_nnz || !out_max_size ||
      !workspace)
    return PCG_ERR_NULL_ARG;
  if (const int rc = asg_check_outputs(V, d, theta, cap, row_ptr, members, members_capacity, mult, workspace))
    return rc;
  if ((uintptr_t) unit_bf16 % 16) return PCG_ERR_MISALIGNED;
  if (workspace_bytes < pcg_asg_build_workspace_bytes(V, cap)) return PCG_ERR_WORKSPACE_TOO_SMALL;
  return asg_build_impl(nullptr, nullptr, nullptr, unit_bf16, V, d, theta, cap, row_ptr, members,
                        members_capacity, mult, seed_of, out_G, out_nnz, out_max_size,
                        (char *) workspace, (hipStream_t) hip_stream);
}

size_t pcg_asg_build_exact_workspace_bytes(int32_t V, int32_t d, int32_t cap) {
  if (V < 1 || d < 1 || cap < 1 || cap > kAsgMaxCap || (int64_t) V * d > INT32_MAX) return 0;
  const size_t v = (size_t) V;
  return asg_core_workspace_bytes(v, cap) + asg_align(v * (size_t) d * 2) /* unit vectors */ +
         asg_align(v * 8) /* norms */ + kAsgAlign;
}

int pcg_asg_build_exact(const float *emb, int32_t V, int32_t d, float theta, int32_t cap,
                        int32_t *row_ptr, int32_t *members, int64_t members_capacity,
                        int32_t *mult, int32_t *seed_of, int32_t *out_G, int64_t *out_nnz,
                        int32_t *out_max_size, void *workspace, size_t workspace_bytes,
                        void *hip_stream) {
  if (!emb || !row_ptr || !members || !mult || !out_G || !out_nnz || !out_max_size || !workspace)
    return PCG_ERR_NULL_ARG;
  if (const int rc = asg_check_outputs(V, d, theta, cap, row_ptr, members, members_capacity, mult, workspace))
    return rc;
  if ((uintptr_t) emb % 16) return PCG_ERR_MISALIGNED;
  if (workspace_bytes < pcg_asg_build_exact_workspace_bytes(V, d, cap))
    return PCG_ERR_WORKSPACE_TOO_SMALL;
  hipStream_t stream = (hipStream_t) hip_stream;
  const size_t v = (size_t) V;
  char *ws = (char *) workspace;
  uint16_t *unit = (uint16_t *) ws; ws += asg_align(v * (size_t) d * 2);
  double *norms = (double *) ws; ws += asg_align(v * 8);
  return asg_build_impl(emb, norms, unit, unit, V, d, theta, cap, row_ptr, members, members_capacity,
                        mult, seed_of, out_G, out_nnz, out_max_size, ws, stream);
}

}  // extern "C"
