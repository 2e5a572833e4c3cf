// HIP kernels of libpcg for gfx950 (MI355X) and their launchers.
//
// One speculative step (Algorithm 1) runs as four kernels on the caller's stream:
//   row_stats     streams every logits row once: per-wave (max, sum of exponentials)  [HBM-bound];
//                 its leading workgroups also form, for every proposed group, the sums of Eq. (5)
//                 relative to the group's own largest logit (the "probes")
//   accept_delta  per sequence: merges the row statistics, normalises the probes, runs the
//                 accept test of Eq. (7) until the first rejection; then, on the decision row,
//                 the table delta[t] = (q(t) - p(t)) / N(t) (q(t) / N(t) on the bonus row), so
//                 that T[g] - D[g] = sum of delta over G_g
//   gather        the overlap-aware segmented gather-sum of that table over the membership
//                 (Eq. 5, Eq. 8), table tiles staged in LDS, from the prepared layout or the CSR.
//                 Inside pcg_verify no sum leaves the kernel (but see finalize): only fp64 totals of
//                 max(0, .) per run of 16 consecutive groups and per chunk.  pcg_group_probs has every
//                 sum written.
//   finalize      per sequence: the chunk and the run that hold u * total, the run's 16 sums
//                 formed again, the group by inverse CDF, then the token inside it (Eq. 10).
//                 From the CSR with up to 4096 groups the gather writes every sum and the group is
//                 drawn from those (finalize_sums).
// A step that is small, or has many sequences of moderate size, runs as one or two kernels instead
// (small_step, after row_stats where the rows are many): one workgroup per sequence does all of the
// above with everything in LDS.
// pcg_group_probs runs row_weights, statistics and the table q(t) / N(t) by one workgroup a row, or, for few long
// rows, weights_parts and weights, and then the same gather;
// pcg_verify_thinning runs row_stats and accept_thin.  pcg_propose runs one kernel, a workgroup per draft row
// (propose_row), for rows of up to 131 072 logits, row_stats and propose beyond.
#include "pcg_kernels.h"
#include "pcg_layout.h"

#include <float.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

namespace pcg {

// =============================================================================================
// row_stats: one wave per 2048-element part of a row.
// =============================================================================================

constexpr int kPartElems = 2048;      // elements per wave: 32 per lane
constexpr int kStatsWaves = 4;        // waves per workgroup

// Row id of a workgroup: grid.y carries the low part, grid.z the rest (grid.y <= 65535).
constexpr int kRowsPerGridY = 32768;

// A 16-byte load at any element address (the type says so to the compiler, which then relies on
// the unaligned access that the amdhsa target guarantees for global memory: the same instruction
// as an aligned load, at most one cache line more per wave).  Optionally marked as streaming
// (nontemporal): streaming loads reach a higher rate on a pass over logits that are larger than
// the caches, but leave nothing behind for the kernels that follow; STREAM is chosen per entry
// point by how much of the rows those re-read.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
template <bool STREAM>
__device__ __forceinline__ u32x4 load16(const void *p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(p));
  else return *reinterpret_cast<const u32x4_any *>(p);
}

template <bool BF16>
constexpr int kPer16 = BF16 ? 8 : 4;    // logits in 16 bytes

// The 16 bytes of logits that a load16 brought, as floats.
template <bool BF16>
__device__ __forceinline__ void unpack16(const u32x4 w, float *x) {
  const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if constexpr (BF16) {
      x[2 * k] = __uint_as_float(ww[k] << 16);
      x[2 * k + 1] = __uint_as_float(ww[k] & 0xffff0000u);
    } else {
      x[k] = __uint_as_float(ww[k]);
    }
  }
}

// exp((x - M) / temperature) for one element, argument in two pieces so that its error stays
// relative to the result: (x - M) * (c_hi + c_lo) with c_hi + c_lo = log2(e) / temperature.
__device__ __forceinline__ float exp_rel(float x, float M, float c_hi, float c_lo) {
  const float d = x - M;
  // a -inf logit has no mass; (-inf) * c_lo would turn the sum into inf - inf otherwise
  return d == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(fmaf(d, c_hi, d * c_lo));
}

// The probe of target row (b, i), i < K, by one wave: T_i[g] and D_i[g] of the proposed
// group g (Eq. 5), each relative to the group's own largest logit.  A chain of four dependent
// loads (proposal -> group -> members -> logits) that needs no row statistic, which is why it
// rides along with the statistics pass instead of waiting for it.
// GUESS: a trip fewer where the groups are of one size (row_stats of small steps 3.8 -> 3.4 us, of which the
// probes are the longest chain; in the small step, whose other waves have the arithmetic of the statistics
// to do meanwhile, it gives nothing).
template <bool BF16, bool GUESS>
__device__ void probe_row(const RowSet &rs, const ProbeArgs &pa, int64_t b, int32_t i, float c, int lane,
                          Probe *out) {
  const int32_t K = pa.K;
  const int32_t g = pa.prop_groups[b * K + i];
  const bool ok = g >= 0 && g < pa.G;
  double at = 0.0, ad = 0.0;
  float mt = -INFINITY, md = -INFINITY;
  if (ok) {
    const void *trow = target_row(rs, b, i, BF16);
    const void *drow = draft_row(rs, b, i, BF16);
    const int32_t beg = pa.row_ptr[g], end = pa.row_ptr[g + 1];
    // The first 64 members stay in registers; longer groups take a second trip.  Of groups that may be of
    // one size they are asked for before their bounds are known, and again if those are others.
    const float *wts = pa.weights;
    float lt0, ld0, m0, w0;
    auto first_members = [&](int32_t from, int32_t to, uint32_t largest) {
      const bool has = from + lane < to;
      const uint32_t t0 = has ? min((uint32_t) pa.members[from + lane], largest) : 0u;
      lt0 = has ? logit_at<BF16>(trow, t0) : -INFINITY;
      ld0 = has ? logit_at<BF16>(drow, t0) : -INFINITY;
      // the entry's share of its token: 1 / N(t) (Eq. 3), or the caller's weight (Eq. 2)
      m0 = has && !wts ? (float) pa.mult[t0] : 1.f;
      w0 = has && wts ? wts[from + lane] : 1.f;
    };
    const int32_t even = GUESS ? pa.even : 0, guess = g * even;
    // A wrong guess may meet entries that no group holds (nnz above row_ptr[G]): the token ids it finds are
    // kept inside the row, and nothing of it is used.
    if (even > 0) first_members(guess, guess + even, (uint32_t) pa.V - 1);
    if (even == 0 || beg != guess || end != guess + even) first_members(beg, end, UINT32_MAX);   // uniform over the wave
    mt = lt0;
    md = ld0;
    for (int32_t j = beg + lane + kWave; j < end; j += kWave) {
      const int32_t t = pa.members[j];
      mt = fmaxf(mt, logit_at<BF16>(trow, t));
      md = fmaxf(md, logit_at<BF16>(drow, t));
    }
    mt = wave_max(mt);
    md = wave_max(md);
    // masses in the kernels' precision: fp32 exponential and division, fp64 sum
    if (lt0 > -INFINITY) at = (double) (exp_rel(lt0, mt, c, pa.c_lo) * w0 / m0);
    if (ld0 > -INFINITY) ad = (double) (exp_rel(ld0, md, c, pa.c_lo) * w0 / m0);
    for (int32_t j = beg + lane + kWave; j < end; j += kWave) {
      const int32_t t = pa.members[j];
      const float m = wts ? 1.f : (float) pa.mult[t];
      const float w = wts ? wts[j] : 1.f;
      const float lt = logit_at<BF16>(trow, t), ld = logit_at<BF16>(drow, t);
      if (lt > -INFINITY) at += (double) (exp_rel(lt, mt, c, pa.c_lo) * w / m);
      if (ld > -INFINITY) ad += (double) (exp_rel(ld, md, c, pa.c_lo) * w / m);
    }
  }
  at = wave_sum(at);
  ad = wave_sum(ad);
  if (lane == 0) {
    Probe p;
    p.Tp = at; p.Dp = ad; p.Tref = mt; p.Dref = md; p.bad = !ok; p.pad = 0;
    *out = p;
  }
}

// A wave's share of a row on its way: elements e0 .. e0 + kPartElems - 1.
// WIDE: a row holds at least one 16-byte piece (V >= 8 bf16 or 4 fp32 logits).
// 16-byte loads, all issued before the first use; each instruction covers 1 KiB of the row.  Rows
// need no alignment (see load16).  In the last part of a row, pieces that would cross its end are
// read where the row's last 16 bytes lie instead, and what belongs to the piece before (or to no
// piece) is masked: no branch, every load in flight, nothing read past the row.  (Element by element
// such parts took 12.9 us where whole parts take 3.7: V = 20 011, 75 rows.)
template <bool BF16, bool WIDE, bool STREAM>
struct RowPart {
  static constexpr int per = kPer16<BF16>, nv = 32 / per;
  u32x4 w[WIDE ? nv : 1];
  float e[WIDE ? 1 : 32];

  __device__ __forceinline__ void load(const void *rowp, int32_t e0, int32_t V, int lane) {
    if constexpr (WIDE) {
      const char *src = reinterpret_cast<const char *>(rowp);
      constexpr int esz = BF16 ? 2 : 4;
      if (e0 + kPartElems <= V) {
        src += (int64_t) e0 * esz;
#pragma unroll
        for (int j = 0; j < nv; ++j) w[j] = load16<STREAM>(src + (j * kWave + lane) * 16);
      } else {
#pragma unroll
        for (int j = 0; j < nv; ++j)
          w[j] = load16<STREAM>(src + (int64_t) min(e0 + (j * kWave + lane) * per, V - per) * esz);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        const int32_t at = e0 + j * kWave + lane;
        e[j] = (at < V) ? logit_at<BF16>(rowp, at) : -INFINITY;
      }
    }
  }

  __device__ __forceinline__ void get(float (&x)[32], int32_t e0, int32_t V, int lane) const {
    if constexpr (WIDE) {
#pragma unroll
      for (int j = 0; j < nv; ++j) unpack16<BF16>(w[j], x + j * per);
      if (e0 + kPartElems > V) {
#pragma unroll
        for (int j = 0; j < nv; ++j) {
          const int32_t over = e0 + (j * kWave + lane) * per - (V - per);   // elements to mask, if any
#pragma unroll
          for (int k = 0; k < per; ++k)
            if (k < over) x[j * per + k] = -INFINITY;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < 32; ++j) x[j] = e[j];
    }
  }
};

// The statistics of a wave's 32 logits per lane; valid in its last lane.
__device__ __forceinline__ StatPart part_stats(const float (&x)[32], float c) {
  float m0 = fmaxf(x[0], x[1]), m1 = fmaxf(x[2], x[3]);
#pragma unroll
  for (int j = 4; j < 32; j += 4) {
    m0 = fmaxf(fmaxf(m0, x[j]), x[j + 1]);
    m1 = fmaxf(fmaxf(m1, x[j + 2]), x[j + 3]);
  }
  const float m = wave_max(fmaxf(m0, m1));

  // Exponentials relative to the wave's own maximum, in the log2 domain: t = fl(m * c) is the
  // reference, and each term is 2^(x * c - t) with the product exact inside the fused
  // multiply-add, so terms near the maximum carry no argument error.  Whoever merges the parts
  // rescales by 2^(t - M * c) in double; t is an exact float, so nothing is lost.
  const float t = m * c;
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
  for (int j = 0; j < 32; j += 4) {
    s0 += __builtin_amdgcn_exp2f(fmaf(x[j], c, -t));
    s1 += __builtin_amdgcn_exp2f(fmaf(x[j + 1], c, -t));
    s2 += __builtin_amdgcn_exp2f(fmaf(x[j + 2], c, -t));
    s3 += __builtin_amdgcn_exp2f(fmaf(x[j + 3], c, -t));
  }
  double z = (double) ((s0 + s1) + (s2 + s3));
  if (m == -INFINITY) z = 0.0;   // (-inf) - (-inf) is NaN: an all -inf part holds no mass
  StatPart sp;
  sp.z = subwave_sum<64>(z);
  sp.m = m;
  sp.t = t;
  return sp;
}

template <bool BF16, bool WIDE, bool STREAM>
__global__ __launch_bounds__(kStatsWaves *kWave) void row_stats_kernel(RowSet rs, int32_t V,
                                                                       int32_t nparts, int64_t nrows,
                                                                       float c, StatPart *parts,
                                                                       ProbeArgs pa, int64_t probe_slots) {
  const int lane = threadIdx.x & (kWave - 1);
  // everything that selects the data is wave-uniform: keep it in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // grid planes (z) continue the count of y: slot runs over the probe slots, then the rows
  const int64_t slot = (int64_t) blockIdx.z * kRowsPerGridY + blockIdx.y;
  if (slot < probe_slots) {
    // The first probe_slots values (launched only with probes) are not rows of logits: each wave
    // of their workgroups forms the probe of one target row.  They are dealt out first, so the
    // chains of dependent loads behind the probes run while the rest of the grid streams.
    const int64_t prow = (slot * gridDim.x + blockIdx.x) * kStatsWaves + wave;
    if (prow >= rs.nrows0) return;
    int64_t b;
    int32_t i;
    split_row(prow, rs.npos0, rs.magic0, b, i);
    if (i < pa.K) probe_row<BF16, true>(rs, pa, b, i, c, lane, pa.out + b * pa.K + i);   // the bonus row has none
    return;
  }
  const int32_t part = blockIdx.x * kStatsWaves + wave;
  const int64_t row = slot - probe_slots;
  if (part >= nparts || row >= nrows) return;   // whole wave leaves together
  const void *rowp = row_base(rs, row, BF16);
  RowPart<BF16, WIDE, STREAM> raw;
  float x[32];
  raw.load(rowp, part * kPartElems, V, lane);
  raw.get(x, part * kPartElems, V, lane);
  const StatPart sp = part_stats(x, c);
  if (lane == kWave - 1) parts[row * nparts + part] = sp;
}

// Meets the other waves of the workgroup once this wave's LDS accesses are done, without the fence of
// __syncthreads(), which would also wait for every load still in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// What lanes of this wave have written to LDS may be read by its other lanes behind this.
__device__ __forceinline__ void wave_handoff() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// =============================================================================================
// accept: one workgroup per sequence.
// =============================================================================================

constexpr int kTokensPerThread = 8;    // consecutive tokens a thread of the table kernels handles

// The table kernels work on eight consecutive tokens per thread, at any alignment.  A thread whose
// eight would cross the end of the row takes the row's last eight instead (slice_start): it repeats
// what its neighbour does for some of them and stores the same values.  WIDE: V >= 8.
template <bool WIDE>
__device__ __forceinline__ int32_t slice_start(int32_t t, int32_t V) {
  return WIDE ? min(t, V - 8) : t;
}

// Eight consecutive logits of a row as floats: one (bf16) or two (fp32) 16-byte loads.
template <bool BF16, bool WIDE>
__device__ __forceinline__ void load8(const void *row, int32_t t, int32_t V, float *x) {
  if constexpr (WIDE) {
    const char *src = reinterpret_cast<const char *>(row) + (int64_t) t * (BF16 ? 2 : 4);
    unpack16<BF16>(load16<false>(src), x);
    if constexpr (!BF16) unpack16<BF16>(load16<false>(src + 16), x + 4);
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = (t + k < V) ? logit_at<BF16>(row, t + k) : -INFINITY;
  }
}

// Divisors of eight consecutive tokens: their multiplicities, or 1 with mult == NULL (general
// weights: the per-entry weight is applied by the gather instead).
template <bool WIDE>
__device__ __forceinline__ void load8_mult(const int32_t *mult, int32_t t, int32_t V, float *m) {
  if (!mult) {
#pragma unroll
    for (int k = 0; k < 8; ++k) m[k] = 1.f;
  } else if constexpr (WIDE) {
    const u32x4 a = load16<false>(mult + t), b = load16<false>(mult + t + 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) { m[k] = (float) (int32_t) a[k]; m[4 + k] = (float) (int32_t) b[k]; }
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) m[k] = (t + k < V) ? (float) mult[t + k] : 1.f;
  }
}

// Four floats at any float address (a row of the table starts at a multiple of V).
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

template <bool WIDE>
__device__ __forceinline__ void store8(float *out, int32_t t, int32_t V, const float *v) {
  if constexpr (WIDE) {
    f32x4_any a, b;
#pragma unroll
    for (int k = 0; k < 4; ++k) { a[k] = v[k]; b[k] = v[4 + k]; }
    *reinterpret_cast<f32x4_any *>(out + t) = a;
    *reinterpret_cast<f32x4_any *>(out + t + 4) = b;
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (t + k < V) out[t + k] = v[k];
  }
}

constexpr int kAcceptThreads = 1024;   // 16 waves: one per row to merge / per position to probe
constexpr int kAcceptTokens = kAcceptThreads * kTokensPerThread;   // delta tokens per workgroup

// State of one sequence's accept scan, in LDS.
struct AcceptShared {
  RowStat st_t[PCG_MAX_K + 1];                 // statistics of the target rows 0..K
  RowStat st_d[PCG_MAX_K];                     // ... and of the draft rows 0..K-1
  double iz_t[PCG_MAX_K + 1], iz_d[PCG_MAX_K]; // 1 / Z of those rows
  Probe probe[PCG_MAX_K];                      // of the proposed groups
  float uacc[PCG_MAX_K];                       // accept uniforms
  float ugrp[PCG_MAX_K + 1], utok[PCG_MAX_K + 1];   // group and token uniforms (accept_fetch)
  int ptok[PCG_MAX_K], pgrp[PCG_MAX_K];
  int istar;                                   // accept_len of the sequence
};

// Statistics of a row of one part.
__device__ __forceinline__ RowStat one_part(const StatPart &sp, float c) {
  RowStat r;
  r.Z = sp.z > 0.0 ? sp.z * exp2((double) sp.t - (double) sp.m * (double) c) : 0.0;
  r.M = sp.m;
  r.pad = 0.f;
  return r;
}

// Statistics of one row from its parts, by the 16 lanes of one DPP row (sub = lane & 15); four
// rows are merged per wave at once.  Every lane of the 16 returns the result.
__device__ __forceinline__ RowStat merge_row16(const StatPart *rp, int32_t nparts, float c, int sub) {
  // a lane's first two parts stay in registers (rows of up to 65 536 logits: all of them), so
  // that the maximum and the sum need one trip to memory, not two
  constexpr int kKeep = 2;
  StatPart keep[kKeep];
  float M = -INFINITY;
#pragma unroll
  for (int j = 0; j < kKeep; ++j) {
    const int32_t k = sub + 16 * j;
    keep[j].z = 0.0; keep[j].m = -INFINITY; keep[j].t = 0.f;
    if (k < nparts) keep[j] = rp[k];
  }
#pragma unroll
  for (int j = 0; j < kKeep; ++j) M = fmaxf(M, keep[j].m);
  for (int32_t k = sub + 16 * kKeep; k < nparts; k += 16) M = fmaxf(M, rp[k].m);
  M = fmaxf(M, dpp_get<kDppXor1, 0xf>(M, M));
  M = fmaxf(M, dpp_get<kDppXor2, 0xf>(M, M));
  M = fmaxf(M, dpp_get<kDppHalfMirror, 0xf>(M, M));
  M = fmaxf(M, dpp_get<kDppMirror, 0xf>(M, M));
  double Z = 0.0;
#pragma unroll
  for (int j = 0; j < kKeep; ++j)
    if (keep[j].z > 0.0) Z += keep[j].z * exp2((double) keep[j].t - (double) M * (double) c);
  for (int32_t k = sub + 16 * kKeep; k < nparts; k += 16) {
    const StatPart sp = rp[k];
    if (sp.z > 0.0) Z += sp.z * exp2((double) sp.t - (double) M * (double) c);
  }
  RowStat r;
  r.Z = subwave_sum<16>(Z);
  r.M = M;
  r.pad = 0.f;
  return r;
}

// The accept scan of sequence b (Algorithm 1 up to the first rejection) by one workgroup of
// kAcceptThreads, in two halves with a barrier between them.  In the end sh.istar, the statistics and their
// reciprocals are valid for every thread; with `writer` the sequence's outputs and counters are written,
// and its row statistics if a.rowstat is given.  probes: the sequence's K probes; parts_t, parts_d: the
// parts of its target and draft rows.
// Before the barrier one wave also fetches the proposals and draws the uniforms of every position, a
// position per lane: at the decision's own position alone, once that is known, the generator's chain of
// multiplications would stand in every wave's way (16 waves on four SIMDs: 0.7 of the 12.6 us of the small
// step at V = 1024, B = 1, 1.4 of 14.3 at V = 4096, B = 8).
__device__ __forceinline__ void accept_fetch(AcceptShared &sh, const AcceptArgs &a, int b, int lane) {
  for (int i = lane; i < a.K; i += kWave) {
    sh.pgrp[i] = a.prop_groups[(int64_t) b * a.K + i];
    sh.ptok[i] = a.prop_tokens[(int64_t) b * a.K + i];
  }
  for (int i = lane; i <= a.K; i += kWave) {
    const Uniforms u = philox_uniforms(a.seed, a.offset, (uint32_t) b, (uint32_t) i);
    if (i < a.K) sh.uacc[i] = u.acc;
    sh.ugrp[i] = u.grp;
    sh.utok[i] = u.tok;
  }
}

// First half: the probes fetched (NULL: they are in sh), the row statistics merged, all to sh.
__device__ __forceinline__ void accept_merge(AcceptShared &sh, const AcceptArgs &a, int b, bool writer,
                                             const Probe *probes, const StatPart *parts_t, const StatPart *parts_d) {
  const int K = a.K;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  constexpr int nw = kAcceptThreads / kWave;
  // The probes of the proposed groups were formed by the statistics pass; the first wave fetches
  // them (one position per lane), the others merge the row statistics.
  const int nprobe = 1;
  if (wave == 0) {
    if (probes)
      for (int i = lane; i < K; i += kWave) sh.probe[i] = probes[i];
  } else {
    // row statistics of this sequence's 2K+1 rows, four rows per wave at a time
    const int sub = lane & 15;
    for (int r = (wave - nprobe) * 4 + (lane >> 4); r < 2 * K + 1; r += (nw - nprobe) * 4) {
      const bool is_t = r <= K;
      const int i = is_t ? r : r - K - 1;
      const RowStat s = merge_row16((is_t ? parts_t : parts_d) + (int64_t) i * a.nparts, a.nparts, a.c, sub);
      const double iz = 1.0 / s.Z;                  // here once, not by every wave that needs it
      if (sub == 0) {
        if (writer && a.rowstat)
          a.rowstat[is_t ? (int64_t) b * (K + 1) + i : a.rs.nrows0 + (int64_t) b * K + i] = s;
        if (is_t) { sh.st_t[i] = s; sh.iz_t[i] = iz; } else { sh.st_d[i] = s; sh.iz_d[i] = iz; }
      }
    }
  }
}

// Second half, after a barrier.
__device__ __forceinline__ void accept_decide(AcceptShared &sh, const AcceptArgs &a, int b, bool writer) {
  const int K = a.K;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  // Both chains have met.  One wave, one position per lane (K <= 64): normalise the probe,
  // take the accept test, and find the first rejection with a ballot; the draft token stands
  // for its group on accept.  The others wait for nothing but the position: outputs and counters come
  // after the barrier.
  const int i = lane;
  const bool in = i < K;
  double T = 0.0, D = 0.0, u = 0.0;
  bool bad = false;
  unsigned long long rejects = 0;
  if (wave == 0) {
    if (in) {
      const Probe p = sh.probe[i];
      if (p.Tp > 0.0) T = p.Tp * exp2((double) (p.Tref - sh.st_t[i].M) * a.cd) / sh.st_t[i].Z;
      if (p.Dp > 0.0) D = p.Dp * exp2((double) (p.Dref - sh.st_d[i].M) * a.cd) / sh.st_d[i].Z;
      u = (double) sh.uacc[i];
      bad = p.bad != 0;
    }
    rejects = __ballot(in && !(u * D < T));
    if (lane == 0) sh.istar = rejects ? __ffsll((long long) rejects) - 1 : K;
  }
  lds_barrier();
  const int istar = sh.istar;
  if (writer && wave == kAcceptThreads / kWave - 1) {
    int32_t *otok = a.out_tokens + (int64_t) b * (K + 1);
    int32_t *ogrp = a.out_groups + (int64_t) b * (K + 1);
    for (int k = lane; k <= K; k += kWave) {
      // the entry at istar itself is written once the group has been drawn, by another wave
      if (k != istar) {
        otok[k] = k < istar ? sh.ptok[k] : -1;
        ogrp[k] = k < istar ? sh.pgrp[k] : -1;
      }
    }
    if (lane == 0) a.accept_len[b] = istar;
  }
  if (writer && wave == 0 && a.diag) {
    const bool evaluated = in && i <= istar;
    const uint32_t near = __popcll(__ballot(evaluated && fabs(u * D - T) < 1e-6 * D));
    const uint32_t zero_d = __popcll(__ballot(evaluated && !bad && D == 0.0));
    const uint32_t nbad = __popcll(__ballot(evaluated && bad));
    if (lane == 0) {
      if (near) atomicAdd(&a.diag->near_accept, near);
      if (zero_d) atomicAdd(&a.diag->zero_draft_mass, zero_d);
      if (nbad) atomicAdd(&a.diag->bad_proposal, nbad);
      atomicAdd(&a.diag->accepted_total, (uint32_t) istar);
      atomicAdd(&a.diag->sequences, 1u);
    }
  }
}

// The first half on the probes and parts that the statistics pass left in memory.
__device__ __forceinline__ void accept_merge_stored(AcceptShared &sh, const AcceptArgs &a, int b, bool writer) {
  accept_merge(sh, a, b, writer, a.probes + (int64_t) b * a.K, a.parts + (int64_t) b * (a.K + 1) * a.nparts,
               a.parts + (a.rs.nrows0 + (int64_t) b * a.K) * a.nparts);
}

// The whole scan on those, fetch and all.
__device__ __forceinline__ void accept_phase_stored(AcceptShared &sh, const AcceptArgs &a, int b, bool writer) {
  accept_merge_stored(sh, a, b, writer);
  // the last wave has the fewest rows to merge
  if (threadIdx.x >= kAcceptThreads - kWave) accept_fetch(sh, a, b, threadIdx.x & (kWave - 1));
  lds_barrier();
  accept_decide(sh, a, b, writer);
}

// The table entries of eight tokens on a decision row (statistics st; draft sd if it was rejected).
__device__ __forceinline__ void delta8(const float *xt, const float *xd, const float *m, bool rejected,
                                       const RowStat &st, const RowStat &sd, double izt, double izd,
                                       float c, float c_lo, float *v) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float et = exp_rel(xt[k], st.M, c, c_lo);
    // two rounded products and a rounded difference (no fused multiply-add), so that
    // identical target and draft rows give exactly zero
    double diff = __dmul_rn((double) et, izt);
    if (rejected) {
      const float ed = exp_rel(xd[k], sd.M, c, c_lo);
      diff = __dsub_rn(diff, __dmul_rn((double) ed, izd));
    }
    v[k] = (float) diff * __builtin_amdgcn_rcpf(m[k]);   // N(t) is a small integer: 1 ulp, a tenth of a division's cost
  }
}

// accept + delta.  Workgroup (b, s) runs the whole accept scan of sequence b -- every one of
// the sequence's workgroups does, so that none has to wait for another -- and then writes its
// slices of the table the gather sums over, on the decision row i* = accept_len[b]:
//   rejected (i* < K):  delta[t] = (q_{i*}(t) - p_{i*}(t)) / N(t)
//   bonus    (i* = K):  delta[t] =  q_K(t) / N(t)
// Workgroup s = 0 also writes the sequence's outputs, row statistics and counters.
template <bool BF16, bool WIDE>
__global__ __launch_bounds__(kAcceptThreads) void accept_delta_kernel(AcceptArgs a, int32_t nsplit,
                                                                      float c_lo, float *table) {
  __shared__ AcceptShared sh;
  const int b = blockIdx.x / nsplit;
  const int split = blockIdx.x % nsplit;
  const RowSet &rs = a.rs;
  const int32_t V = a.V, K = a.K;
  const float c = a.c;
  const int32_t *mult = a.weights ? nullptr : a.mult;   // with weights delta is q - p as it is
  const int32_t stride = nsplit * kAcceptTokens;
  const int32_t first = split * kAcceptTokens + threadIdx.x * kTokensPerThread;
  // the multiplicities of this thread's first two slices do not depend on the decision row:
  // they are asked for before the accept scan
  float m_a[8], m_b[8];
  if (first < V) load8_mult<WIDE>(mult, slice_start<WIDE>(first, V), V, m_a);
  if (first + stride < V) load8_mult<WIDE>(mult, slice_start<WIDE>(first + stride, V), V, m_b);
  accept_phase_stored(sh, a, b, split == 0);

  // 4. this workgroup's share of the table on the decision row: slices split, split + nsplit, ...
  const int32_t istar = __builtin_amdgcn_readfirstlane(sh.istar);
  const bool rejected = istar < K;
  const void *trow = target_row(rs, b, istar, BF16);
  const void *drow = draft_row(rs, b, rejected ? istar : 0, BF16);
  const RowStat st = sh.st_t[istar];
  const RowStat sd = sh.st_d[rejected ? istar : 0];
  const double izt = sh.iz_t[istar], izd = rejected ? sh.iz_d[istar] : 0.0;
  auto delta = [&](const float *xt, const float *xd, const float *m, float *v) {
    delta8(xt, xd, m, rejected, st, sd, izt, izd, c, c_lo, v);
  };
  float *out = table + (int64_t) b * V;
  // two slices per turn, so that the loads of the second are in flight behind the first
  for (int32_t at = first; at < V; at += 2 * stride) {
    const bool two = at + stride < V;
    const int32_t t = slice_start<WIDE>(at, V), t2 = slice_start<WIDE>(at + stride, V);
    float xt[8], xd[8], m[8], v[8], xt2[8], xd2[8], m2[8];
    load8<BF16, WIDE>(trow, t, V, xt);
    if (rejected) load8<BF16, WIDE>(drow, t, V, xd);
    if (two) {
      load8<BF16, WIDE>(trow, t2, V, xt2);
      if (rejected) load8<BF16, WIDE>(drow, t2, V, xd2);
    }
    if (at == first) {
#pragma unroll
      for (int k = 0; k < 8; ++k) { m[k] = m_a[k]; m2[k] = m_b[k]; }
    } else {
      load8_mult<WIDE>(mult, t, V, m);
      if (two) load8_mult<WIDE>(mult, t2, V, m2);
    }
    delta(xt, xd, m, v);
    store8<WIDE>(out, t, V, v);
    if (two) {
      delta(xt2, xd2, m2, v);
      store8<WIDE>(out, t2, V, v);
    }
  }
}

// =============================================================================================
// accept + thinning: the reject branch drawn the paper's own way (Sec. 2.2 "Residual sampling
// via thinning", Eq. 9), with no enumeration of the groups: y ~ q, one of the groups holding y
// by the weights, accepted with probability [1 - D/T]_+, repeated until one is.  One workgroup
// per sequence; its 16 waves run 16 trials at a time and the first accepted one (in trial
// order) is emitted, so the result is that of running the trials one after the other.
// =============================================================================================

constexpr int kMaxThinParts = 2048;       // parts of a row the token draw can search (V <= 4 Mi)
constexpr int kThinTrialWaves = 16;       // trials a workgroup runs side by side, one per wave

struct WavePick {
  int32_t index;            // first index whose running sum exceeds u * total; -1: nothing has mass
  double total, goal, lo, hi;
};

// Inverse CDF over f(0..n-1) >= 0 by one wave (ascending order; every lane gets the result).
// `total` < 0: the sum of f is formed here first.
template <typename F>
__device__ WavePick wave_inverse_cdf(int32_t n, F f, double u, int lane, double total = -1.0) {
  if (total < 0.0) {
    total = 0.0;
    for (int32_t j = lane; j < n; j += kWave) {
      const double v = f(j);
      if (v > 0.0) total += v;
    }
    total = wave_sum(total);
  }
  WavePick r;
  r.total = total;
  r.goal = u * total;
  r.index = -1;
  r.lo = r.hi = 0.0;
  double base = 0.0;
  int32_t last = -1;
  double last_v = 0.0;
  for (int32_t j0 = 0; j0 < n; j0 += kWave) {
    const int32_t j = j0 + lane;
    double v = j < n ? f(j) : 0.0;
    if (!(v > 0.0)) v = 0.0;
    const double inc = wave_scan(v);
    const unsigned long long pos = __ballot(v > 0.0);
    if (pos) {
      const int hl = 63 - __clzll((long long) pos);
      last = j0 + hl;
      last_v = read_lane(v, hl);
    }
    const unsigned long long hit = __ballot(v > 0.0 && base + inc > r.goal);
    if (hit) {
      const int l = __ffsll((long long) hit) - 1;
      r.index = j0 + l;
      r.hi = base + read_lane(inc, l);
      r.lo = r.hi - read_lane(v, l);
      return r;
    }
    base += read_lane(inc, kWave - 1);
  }
  if (last >= 0) {   // rounding at the top end: the last index that has mass
    r.index = last;
    r.hi = total;
    r.lo = total - last_v;
  }
  return r;
}

__device__ __forceinline__ bool near_edge(const WavePick &p) {
  return (p.lo > 0.0 && p.goal - p.lo < 1e-6 * p.total) ||
         (p.hi < p.total && p.hi - p.goal < 1e-6 * p.total);
}

// Which of the n membership entries of a token (reverse-index positions e0 .. e0+n-1) the
// 24-bit draw picks, K ~ w_{k,x} over k in S(x) (Eq. 6): entry (k24 n) >> 24 under the equal
// split, else the inverse CDF of the entries' weights at k24 / 2^24, by the whole wave.
// *near: that draw is within 1e-6 of an inner edge of the chosen entry's bin.
__device__ __forceinline__ int32_t pick_entry(const float *tok_weights, int32_t e0, int32_t n,
                                              uint32_t k24, int lane, bool *near) {
  *near = false;
  if (!tok_weights) return (int32_t) (((uint64_t) k24 * (uint64_t) max(n, 1)) >> 24);
  const WavePick pk = wave_inverse_cdf(
      n, [&](int32_t e) { return (double) tok_weights[e0 + e]; }, (double) k24 * (1.0 / 16777216.0), lane);
  if (pk.index < 0) return 0;
  *near = near_edge(pk);
  return pk.index;
}

// Masses of up to N parts of one row, as the token draw reads them.
template <int N>
struct PartMasses {
  double Zp[N];     // mass of each part relative to the row maximum, 2^(M c)
  double up[N];     // 2^(M c - t): from the row's units to the part's own
  float tp[N];      // log2-domain reference t of each part
};

// Filled by the calling threads (tid of nthreads) from the statistics of row `rp`; a barrier
// must follow.
template <int N>
__device__ __forceinline__ void fill_part_masses(PartMasses<N> &pm, const StatPart *rp, int32_t nparts,
                                                 float M, float c, int tid, int nthreads) {
  for (int32_t p = tid; p < nparts; p += nthreads) {
    const StatPart sp = rp[p];
    const double e = exp2((double) sp.t - (double) M * (double) c);
    const bool has = sp.z > 0.0 && e > 0.0;
    pm.Zp[p] = has ? sp.z * e : 0.0;
    pm.up[p] = has ? 1.0 / e : 0.0;
    pm.tp[p] = sp.t;
  }
}

struct ThinShared {
  PartMasses<kMaxThinParts> pm;
  uint32_t redo[kThinTrialWaves][32];     // per wave: one lane's 32 logits, spread over the lanes
  int accepted[kThinTrialWaves], group[kThinTrialWaves];
  int token[kThinTrialWaves], near[kThinTrialWaves];
  int done;
};

// 32 consecutive logits of a row as loaded: bf16 stays packed two per register.
template <bool BF16>
struct Logits32 {
  static constexpr int kWords = BF16 ? 16 : 32;
  uint32_t w[kWords];
  __device__ __forceinline__ float get(int k) const {
    if constexpr (BF16) return __uint_as_float((k & 1) ? (w[k >> 1] & 0xffff0000u) : (w[k >> 1] << 16));
    else return __uint_as_float(w[k]);
  }
};

// Tokens e0 .. e0+31 of a row; tokens at or beyond V read as -inf.  A lane wholly inside the row
// uses 16-byte loads at any alignment; one that crosses its end reads element by element, at
// addresses clamped into the row so that its 32 loads are in flight together.
template <bool BF16>
__device__ __forceinline__ void load32(const void *row, int32_t e0, int32_t V, Logits32<BF16> &r) {
  constexpr int nvec = BF16 ? 4 : 8;
  if (e0 + 32 <= V) {
    const char *src = reinterpret_cast<const char *>(row) + (size_t) e0 * (BF16 ? 2 : 4);
#pragma unroll
    for (int i = 0; i < nvec; ++i) {
      const u32x4 q = load16<false>(src + 16 * i);
      r.w[4 * i] = q.x; r.w[4 * i + 1] = q.y; r.w[4 * i + 2] = q.z; r.w[4 * i + 3] = q.w;
    }
  } else {
    const uint32_t ninf = BF16 ? 0xff80u : 0xff800000u;
    uint32_t bits[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const int32_t e = min(e0 + k, V - 1);
      if constexpr (BF16) bits[k] = reinterpret_cast<const uint16_t *>(row)[e];
      else bits[k] = reinterpret_cast<const uint32_t *>(row)[e];
    }
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const uint32_t b = e0 + k < V ? bits[k] : ninf;
      if constexpr (BF16) {
        if (k & 1) r.w[k >> 1] |= b << 16; else r.w[k >> 1] = b;
      } else {
        r.w[k] = b;
      }
    }
  }
}

// y ~ q on the row whose part masses are in pm: the part by its mass, then the lane inside the
// part (each lane sums 32 consecutive tokens), then the token among that lane's 32, which are
// handed to 32 lanes through `redo` (32 words of LDS private to the calling wave).
// *near: the draw is within 1e-6 of an inner edge of the token's bin.
template <bool BF16, int N>
__device__ int32_t draw_token(const PartMasses<N> &pm, uint32_t *redo, const void *trow, int32_t V,
                              int32_t nparts, float c, double u, int lane, bool *near) {
  const WavePick pp = wave_inverse_cdf(nparts, [&](int32_t p) { return pm.Zp[p]; }, u, lane);
  if (pp.index < 0) { *near = false; return 0; }
  const int32_t p = pp.index;
  const float t = pm.tp[p];
  const int32_t e0 = p * kPartElems + lane * 32;
  Logits32<BF16> raw;
  load32<BF16>(trow, e0, V, raw);
  // the same expression row_stats summed; the part has mass, so t is finite and no logit a NaN, and -inf gives 0 without
  // a test (two of its instructions an element: thinning, V = 65 536, 64 sequences 35.8 -> 35.5 us the call)
  auto mass = [&](float x) -> float { return __builtin_amdgcn_exp2f(fmaf(x, c, -t)); };
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 32; k += 2) s += (double) mass(raw.get(k)) + (double) mass(raw.get(k + 1));
  const double inc = wave_scan(s);
  // threshold in the part's own units: masses there are relative to 2^t, in Zp to 2^(M c)
  const double scale = pm.up[p];
  const double goal = (pp.goal - pp.lo) * scale;
  const double part_total = read_lane(inc, kWave - 1);
  const unsigned long long hit = __ballot(s > 0.0 && inc > goal);
  const unsigned long long pos = __ballot(s > 0.0);
  if (!pos) { *near = false; return min(p * kPartElems, V - 1); }   // cannot happen: Zp[p] > 0
  const int l = hit ? __ffsll((long long) hit) - 1 : 63 - __clzll((long long) pos);
  // lane l's 32 tokens, one per lane
  if (lane == l) {
#pragma unroll
    for (int k = 0; k < Logits32<BF16>::kWords; ++k) redo[k] = raw.w[k];
  }
  wave_handoff();
  float x = -INFINITY;
  if (lane < 32) {
    if constexpr (BF16) x = __uint_as_float((uint32_t) reinterpret_cast<const uint16_t *>(redo)[lane] << 16);
    else x = __uint_as_float(redo[lane]);
  }
  const double v = (double) mass(x);
  const double before = read_lane(inc, l) - read_lane(s, l);
  const double cum = before + wave_scan(v);
  const unsigned long long hit2 = __ballot(v > 0.0 && cum > goal);
  const unsigned long long pos2 = __ballot(v > 0.0);
  const int k = hit2 ? __ffsll((long long) hit2) - 1 : 63 - __clzll((long long) pos2);
  const double hi = read_lane(cum, k), lo = hi - read_lane(v, k);
  const int32_t y = p * kPartElems + l * 32 + k;
  const double tot_units = pp.total * scale;
  const bool first_mass = pp.lo <= 0.0 && lo <= 0.0;            // no bin below
  const bool last_mass = pp.hi >= pp.total && hi >= part_total;  // no bin above
  *near = (!first_mass && goal - lo < 1e-6 * tot_units) || (!last_mass && hi - goal < 1e-6 * tot_units);
  return y;
}

template <bool BF16>
__global__ __launch_bounds__(kAcceptThreads) void accept_thin_kernel(
    AcceptArgs a, const int32_t *tok_ptr, const int32_t *tok_groups, const float *tok_weights,
    int32_t *trials, int32_t max_trials) {
  __shared__ AcceptShared sh;
  __shared__ ThinShared th;
  const int b = blockIdx.x;
  accept_phase_stored(sh, a, b, true);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t K = a.K, V = a.V, istar = __builtin_amdgcn_readfirstlane(sh.istar);
  const int32_t pos = sh.istar;          // the same, for the generator: on the vector unit it is the faster chain
  const bool bonus = istar == K;
  const int64_t trow_id = (int64_t) b * (K + 1) + istar;
  const void *trow = target_row(a.rs, b, istar, BF16);
  const void *drow = draft_row(a.rs, b, bonus ? 0 : istar, BF16);
  const RowStat st = sh.st_t[istar];
  const RowStat sd = sh.st_d[bonus ? 0 : istar];
  const float c_lo = (float) (a.cd - (double) a.c);

  fill_part_masses(th.pm, a.parts + trow_id * a.nparts, a.nparts, st.M, a.c, threadIdx.x, kAcceptThreads);
  if (threadIdx.x == 0) th.done = 0;
  __syncthreads();

  // q(t) w and p(t) w of CSR entry j holding token t (w = 1 / N(t) under the equal split), up
  // to the rows' normalisations, in the kernels' precision (fp32)
  const float *wts = a.weights;
  auto wq = [&](int32_t j, int32_t t) -> double {
    const float e = exp_rel(logit_at<BF16>(trow, t), st.M, a.c, c_lo);
    return (double) (wts ? e * wts[j] : e / (float) a.mult[t]);
  };
  auto wp = [&](int32_t j, int32_t t) -> double {
    const float e = exp_rel(logit_at<BF16>(drow, t), sd.M, a.c, c_lo);
    return (double) (wts ? e * wts[j] : e / (float) a.mult[t]);
  };

  // Trials run kThinTrialWaves at a time, one per wave; the other waves only keep the barriers.
  for (int32_t round = 0;; ++round) {
    const int32_t trial = round * kThinTrialWaves + wave;
    const bool active = wave < kThinTrialWaves && (bonus ? trial == 0 : trial < max_trials);
    if (active) {   // uniform over the wave
      const TrialDraws d = philox_trial(a.seed, a.offset, (uint32_t) b, (uint32_t) pos,
                                        (uint32_t) trial);
      bool near_y = false;
      const int32_t y = draw_token<BF16>(th.pm, th.redo[wave], trow, V, a.nparts, a.c,
                                              (double) d.u_y, lane, &near_y);
      const int32_t e0 = tok_ptr[y], n = tok_ptr[y + 1] - e0;
      bool near_e = false;
      const int32_t g = tok_groups[e0 + pick_entry(tok_weights, e0, n, d.k24, lane, &near_e)];
      const int32_t beg = a.row_ptr[g], len = a.row_ptr[g + 1] - beg;
      int accepted = 1, near = near_y || near_e ? 1 : 0;
      int32_t token = y;
      if (!bonus) {
        // the first 64 members stay in registers for the token draw below
        const int32_t t0 = lane < len ? a.members[beg + lane] : -1;
        const double q0 = t0 >= 0 ? wq(beg + lane, t0) : 0.0;
        double at = q0, ad = t0 >= 0 ? wp(beg + lane, t0) : 0.0;
        for (int32_t j = lane + kWave; j < len; j += kWave) {
          const int32_t t = a.members[beg + j];
          at += wq(beg + j, t);
          ad += wp(beg + j, t);
        }
        const double Tn = wave_sum(at), T = Tn / st.Z, D = wave_sum(ad) / sd.Z;
        const double ua = (double) d.u_a;
        accepted = ua * T < T - D;                    // u_a < [1 - D/T]_+
        if (fabs(ua * T - (T - D)) < 1e-6 * T) near |= 1;
        const WavePick pt = wave_inverse_cdf(
            len, [&](int32_t j) { return j < kWave ? q0 : wq(beg + j, a.members[beg + j]); },
            (double) d.u_tok, lane, Tn);
        token = pt.index < 0 ? -1 : (pt.index < kWave ? read_lane(t0, pt.index) : a.members[beg + pt.index]);
        if (pt.index >= 0 && near_edge(pt)) near |= 2;
      }
      if (lane == 0) {
        th.accepted[wave] = accepted; th.group[wave] = g; th.token[wave] = token; th.near[wave] = near;
      }
    } else if (lane == 0 && wave < kThinTrialWaves) {
      th.accepted[wave] = -1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t n_near = 0, n_near_tok = 0;
      int chosen = -1, last_active = -1;
      for (int w = 0; w < kThinTrialWaves && chosen < 0; ++w) {
        if (th.accepted[w] < 0) break;
        last_active = w;
        if (th.near[w] & 1) ++n_near;
        if (th.accepted[w] == 1) chosen = w;
      }
      const bool exhausted = chosen < 0 && (round + 1) * kThinTrialWaves >= max_trials;
      if (exhausted) chosen = last_active;
      if (chosen >= 0) {
        if (th.near[chosen] & 2) ++n_near_tok;
        a.out_groups[(int64_t) b * (K + 1) + istar] = th.group[chosen];
        a.out_tokens[(int64_t) b * (K + 1) + istar] = th.token[chosen];
        trials[b] = bonus ? 0 : round * kThinTrialWaves + chosen + 1;
        th.done = 1;
      }
      if (a.diag) {
        if (n_near) atomicAdd(&a.diag->near_group, n_near);
        if (n_near_tok) atomicAdd(&a.diag->near_token, n_near_tok);
        if (exhausted) atomicAdd(&a.diag->residual_fallback, 1u);
      }
    }
    __syncthreads();
    if (th.done) break;
  }
}

// =============================================================================================
// propose: the draft-side coupling (Sec. 2.2 "Proposal coupling and acceptance", Eq. 6).  One
// wave per draft row: merge the row's part statistics, draw x ~ p through the parts, then one
// of the membership entries of x.
// =============================================================================================

// The uniforms of one row's draw; formed while its first loads are on their way.
__device__ __forceinline__ ProposalDraws propose_uniforms(const RowSet &rs, int64_t row, int32_t K, int32_t pos0,
                                                          uint64_t seed, uint64_t offset) {
  int64_t b;
  int32_t i;
  split_row(row, K, rs.magic0, b, i);
  return philox_proposal(seed, offset, (uint32_t) b, (uint32_t) (pos0 + i));
}

// The draw of one row by one wave, from the masses of its parts.
template <bool BF16, int N>
__device__ __forceinline__ void propose_draw(const PartMasses<N> &pm, uint32_t *redo, const RowSet &rs, int64_t row,
                                             int32_t V, int32_t nparts, float c, const ProposalDraws &d,
                                             const int32_t *tok_ptr, const int32_t *tok_groups,
                                             const float *tok_weights, int32_t *prop_tokens,
                                             int32_t *prop_groups, pcg_diag *diag, int lane) {
  bool near = false;
  const int32_t x = draw_token<BF16>(pm, redo, row_base(rs, row, BF16), V, nparts, c,
                                          (double) d.u_x, lane, &near);
  const int32_t e0 = tok_ptr[x], n = tok_ptr[x + 1] - e0;
  bool near_e = false;
  const int32_t e = pick_entry(tok_weights, e0, n, d.k24, lane, &near_e);
  if (lane == 0) {
    prop_tokens[row] = x;
    prop_groups[row] = tok_groups[e0 + e];
    if (diag) {
      if (near || near_e) atomicAdd(&diag->near_token, 1u);
      atomicAdd(&diag->sequences, 1u);
    }
  }
}

template <bool BF16>
__global__ __launch_bounds__(kWave) void propose_kernel(
    RowSet rs, int32_t V, int32_t K, int32_t pos0, int32_t nparts, float c, const StatPart *parts,
    const int32_t *tok_ptr, const int32_t *tok_groups, const float *tok_weights, uint64_t seed,
    uint64_t offset, int32_t *prop_tokens, int32_t *prop_groups, pcg_diag *diag) {
  __shared__ PartMasses<kMaxThinParts> pm;
  __shared__ uint32_t redo[32];
  const int lane = threadIdx.x;
  const int64_t row = blockIdx.x;
  const StatPart *rp = parts + row * nparts;
  const ProposalDraws d = propose_uniforms(rs, row, K, pos0, seed, offset);
  float M = -INFINITY;
  for (int32_t p = lane; p < nparts; p += kWave) M = fmaxf(M, rp[p].m);
  M = wave_max(M);
  fill_part_masses(pm, rp, nparts, M, c, lane, kWave);
  __syncthreads();
  propose_draw<BF16>(pm, redo, rs, row, V, nparts, c, d, tok_ptr, tok_groups, tok_weights, prop_tokens, prop_groups,
                     diag, lane);
}

// The same in one launch, by one workgroup per row: the row's parts stay in LDS between its statistics
// and the draw, and the rows' draws, chains of dependent loads, run behind other rows' streaming.
// V = 65 536, bf16: 64 rows 8.2 us against 3.6 + 4.5 in two launches, 512 rows 17.5 against 12.4 + 5.2; the
// call, whose launches cost its caller more than that, 14.3 -> 11.3 us for 64 rows.
constexpr int kProposeThreads = 1024;
constexpr int kProposeParts = 64;        // V <= 131 072: beyond, a row is too long for one compute unit

template <bool BF16, bool WIDE>
__global__ __launch_bounds__(kProposeThreads) void propose_row_kernel(
    RowSet rs, int32_t V, int32_t K, int32_t pos0, int32_t nparts, float c, const int32_t *tok_ptr,
    const int32_t *tok_groups, const float *tok_weights, uint64_t seed, uint64_t offset,
    int32_t *prop_tokens, int32_t *prop_groups, pcg_diag *diag) {
  constexpr int kWaves = kProposeThreads / kWave;
  __shared__ StatPart parts[kProposeParts];
  __shared__ PartMasses<kProposeParts> pm;
  __shared__ uint32_t redo[32];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = blockIdx.x;
  const void *rowp = row_base(rs, row, BF16);
  // cached loads: the draw reads a part again; a wave's next part is on its way behind the present one
  RowPart<BF16, WIDE, false> raw;
  if (wave < nparts) raw.load(rowp, wave * kPartElems, V, lane);
  ProposalDraws d = {0.f, 0u};
  if (wave == 0) d = propose_uniforms(rs, row, K, pos0, seed, offset);
  for (int32_t p = wave; p < nparts; p += kWaves) {
    float x[32];
    raw.get(x, p * kPartElems, V, lane);
    if (p + kWaves < nparts) raw.load(rowp, (p + kWaves) * kPartElems, V, lane);
    const StatPart sp = part_stats(x, c);
    if (lane == kWave - 1) parts[p] = sp;
  }
  lds_barrier();
  if (wave > 0) return;
  float M = lane < nparts ? parts[lane].m : -INFINITY;
  M = wave_max(M);
  fill_part_masses(pm, parts, nparts, M, c, lane, kWave);
  wave_handoff();
  propose_draw<BF16>(pm, redo, rs, row, V, nparts, c, d, tok_ptr, tok_groups, tok_weights, prop_tokens, prop_groups,
                     diag, lane);
}

// =============================================================================================
// weights: the per-token table of pcg_group_probs, q(t) / N(t), or q(t) with general weights.
// =============================================================================================

// A row goes in parts of kPartElems tokens, a wave's each: exponentials relative to the part's own maximum, their sum, and
// once the row's total is known the exponentials times the part's scale.  Either a workgroup holds a whole row
// (row_weights_kernel), or a row's parts are spread over the chip twice (weights_parts_kernel, weights_kernel).  Both take every
// step by the functions here, element by element and sum by sum on the same lanes: a row's table is the same to
// the bit whichever kernels form it, so that how many rows come with it does not matter.
constexpr int kTablePieces = kPartElems / (4 * kWave);      // of four tokens a lane, in a part

// First token of piece j of part p in this lane; in the row's last part, pieces that would cross its end are read
// where its last four tokens lie, and the first of those belong to the piece before.
__device__ __forceinline__ int32_t piece_token(int32_t p, int j, int lane) { return p * kPartElems + (j * kWave + lane) * 4; }

// Four consecutive logits as they lie in memory, at any element address.  WIDE: V >= 4.
template <bool BF16>
struct Piece { uint32_t w[BF16 ? 2 : 4]; };

typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
template <bool BF16, bool WIDE, bool STREAM>
__device__ __forceinline__ Piece<BF16> load_piece(const void *row, int32_t t) {
  Piece<BF16> r;
  if constexpr (!WIDE) {                                   // t + k < 0: no token, not read
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (BF16) {
        const uint32_t b = t + k >= 0 ? reinterpret_cast<const uint16_t *>(row)[t + k] : 0u;
        if (k & 1) r.w[k >> 1] |= b << 16; else r.w[k >> 1] = b;
      } else {
        r.w[k] = t + k >= 0 ? reinterpret_cast<const uint32_t *>(row)[t + k] : 0u;
      }
    }
  } else if constexpr (BF16) {
    const u32x2_any *src = reinterpret_cast<const u32x2_any *>(reinterpret_cast<const uint16_t *>(row) + t);
    const u32x2_any q = STREAM ? __builtin_nontemporal_load(src) : *src;
    r.w[0] = q.x; r.w[1] = q.y;
  } else {
    const u32x4 q = load16<STREAM>(reinterpret_cast<const float *>(row) + t);
    r.w[0] = q.x; r.w[1] = q.y; r.w[2] = q.z; r.w[3] = q.w;
  }
  return r;
}

// N pieces of part p from piece j0 on, all asked for at once.  V >= 4.
template <bool BF16, bool STREAM, int N>
__device__ __forceinline__ void load_pieces(Piece<BF16> (&w)[N], const void *row, int32_t p, int j0, int32_t V, int lane) {
  if ((p + 1) * kPartElems <= V) {                         // uniform
    const void *src = elem_ptr(row, piece_token(p, j0, lane), BF16);
#pragma unroll
    for (int j = 0; j < N; ++j) w[j] = load_piece<BF16, true, STREAM>(src, 4 * kWave * j);
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) w[j] = load_piece<BF16, true, STREAM>(row, min(piece_token(p, j0 + j, lane), V - 4));
  }
}

// The logits of N pieces of part p from piece j0 on; -inf for what belongs to the piece before.
template <bool BF16, int N>
__device__ __forceinline__ void piece_logits(const Piece<BF16> (&w)[N], int32_t p, int j0, int32_t V, int lane, float (&x)[4 * N]) {
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (BF16) x[4 * j + k] = __uint_as_float((k & 1) ? (w[j].w[k >> 1] & 0xffff0000u) : (w[j].w[k >> 1] << 16));
      else x[4 * j + k] = __uint_as_float(w[j].w[k]);
    }
  if ((p + 1) * kPartElems > V) {                          // uniform
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int32_t over = piece_token(p, j0 + j, lane) - (V - 4);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < over) x[4 * j + k] = -INFINITY;
    }
  }
}

// The exponential of a logit relative to the maximum of its part: exp_rel; of its test for -inf only the low product is
// left, which for it is an infinity of either sign or, with c_lo = 0, a NaN.  A part without mass has no maximum (its
// -inf - (-inf) would be NaN).
__device__ __forceinline__ float part_exp(float x, float m, float c, float c_lo) {
  const float d = x - (m == -INFINITY ? 0.f : m);
  return __builtin_amdgcn_exp2f(fmaf(d, c, fminf(d * c_lo, FLT_MAX)));
}

// Statistics of a part and, in e, its exponentials.  The maximum is every lane's, the sum the last lane's.
template <bool BF16>
__device__ __forceinline__ double part_exponentials(const Piece<BF16> (&w)[kTablePieces], int32_t p, int32_t V, int lane, float c,
                                                    float c_lo, float (&e)[4 * kTablePieces], float &m) {
  piece_logits<BF16>(w, p, 0, V, lane, e);
  float top = e[0];
#pragma unroll
  for (int k = 1; k < 4 * kTablePieces; ++k) top = fmaxf(top, e[k]);
  m = wave_max(top);
  float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 4 * kTablePieces; ++k) {
    e[k] = part_exp(e[k], m, c, c_lo);
    s[k & 3] += e[k];
  }
  return subwave_sum<64>((double) ((s[0] + s[1]) + (s[2] + s[3])));
}

// N(t) of a piece.
template <bool WIDE>
__device__ __forceinline__ u32x4 load_mult(const int32_t *mult, int32_t at, int32_t V) {
  const int32_t t = min(at, V - 4);
  if constexpr (WIDE) return load16<false>(mult + t);
  u32x4 n;
#pragma unroll
  for (int k = 0; k < 4; ++k) n[k] = t + k >= 0 ? (uint32_t) mult[t + k] : 1u;
  return n;
}

// Four entries of the table from their exponentials: the product with the scale, a double, rounded once (two floats hold
// enough of it); and divided by N(t).
__device__ __forceinline__ f32x4_any scaled(const float *e, double scale) {
  const float f_hi = (float) scale, f_lo = (float) (scale - (double) f_hi);
  f32x4_any v;
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = fmaf(e[k], f_hi, e[k] * f_lo);
  return v;
}
__device__ __forceinline__ f32x4_any divided(f32x4_any v, const u32x4 n) {
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] *= __builtin_amdgcn_rcpf((float) (int32_t) n[k]);
  return v;
}

__device__ __forceinline__ void store_piece(float *out, const f32x4_any v, int32_t at, int32_t V, bool whole) {
  const int32_t t = min(at, V - 4);
  if (whole || at <= V - 4) {
    *reinterpret_cast<f32x4_any *>(out + t) = v;
  } else {
#pragma unroll
    for (int k = 1; k < 4; ++k)
      if (k >= at - t) out[t + k] = v[k];
  }
}

// A row by one workgroup: its exponentials stay in registers until its total is known.  NP: row parts a wave holds (64
// exponentials a lane with two; longer rows take the two kernels below).  A row is read once and its
// exponentials are formed once, where the two kernels read it twice and form them twice.  256 rows of 65 536
// bf16 logits 19.7 us against 7.5 + 20.2, fp32 24.3 against 11.4 + 21.9; what is written (67 MB) and read takes 20 and 27 at
// the rate of a copy.  64 rows, which leave most of the chip to others, take 16.2 against 4.2 + 10.3: a row's instructions on
// one compute unit, of which the exponential and the reciprocal of N(t) take four issue slots each.
constexpr int kRowTableThreads = 1024;
constexpr int kRowTableParts = 2 * kRowTableThreads / kWave;      // V <= 65 536

template <bool BF16, bool WIDE, int NP>
__global__ __launch_bounds__(kRowTableThreads) void row_weights_kernel(RowSet rs, int32_t V, int32_t nparts, float c, float c_lo,
                                                                       double cd, const int32_t *mult, float *table) {
  __shared__ double part_z[kRowTableParts];
  __shared__ float part_m[kRowTableParts];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const void *rowp = row_base(rs, blockIdx.x, BF16);
  float *out = table + (int64_t) blockIdx.x * V;
  Piece<BF16> w[NP][kTablePieces];
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int32_t p = wave * NP + q;
    if (p >= nparts) continue;                           // uniform over the wave
#pragma unroll
    for (int j = 0; j < kTablePieces; ++j) w[q][j] = load_piece<BF16, WIDE, true>(rowp, min(piece_token(p, j, lane), V - 4));
  }
  float e[NP][4 * kTablePieces];
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int32_t p = wave * NP + q;
    if (p >= nparts) continue;
    float m;
    const double z = part_exponentials<BF16>(w[q], p, V, lane, c, c_lo, e[q], m);
    if (lane == kWave - 1) { part_z[p] = z; part_m[p] = m; }
  }
  __syncthreads();
  // every wave: the row's maximum and total, a part per lane
  const float pm = lane < nparts ? part_m[lane] : -INFINITY;
  const double pz = lane < nparts ? part_z[lane] : 0.0;
  const float M = wave_max(pm);
  const double up = exp2((double) (pm - M) * cd);        // from the part's maximum to the row's
  const double iz = 1.0 / wave_sum(pz > 0.0 ? pz * up : 0.0);
  const double scale = up * iz;
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int32_t p = wave * NP + q;
    if (p >= nparts) continue;
    const double f = read_lane(scale, p);
    const bool whole = (p + 1) * kPartElems <= V;
#pragma unroll
    for (int j = 0; j < kTablePieces; ++j) {
      const int32_t at = piece_token(p, j, lane);
      f32x4_any v = scaled(e[q] + 4 * j, f);
      if (mult) v = divided(v, load_mult<WIDE>(mult, at, V));      // uniform
      store_piece(out, v, at, V, whole);
    }
  }
}

// The statistics of every part of every row, a wave each.  V >= 4.
template <bool BF16>
__global__ __launch_bounds__(kStatsWaves *kWave) void weights_parts_kernel(RowSet rs, int32_t V, int32_t nparts, float c,
                                                                           float c_lo, StatPart *parts) {
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t p = blockIdx.x * kStatsWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (p >= nparts) return;                               // whole wave leaves together
  const void *rowp = row_base(rs, blockIdx.y, BF16);
  Piece<BF16> w[kTablePieces];
  load_pieces<BF16, true>(w, rowp, p, 0, V, lane);
  float e[4 * kTablePieces];
  StatPart sp;
  sp.z = part_exponentials<BF16>(w, p, V, lane, c, c_lo, e, sp.m);
  sp.t = 0.f;
  if (lane == kWave - 1) parts[(int64_t) blockIdx.y * nparts + p] = sp;
}

// The table from those, a part by one workgroup.
constexpr int kTableThreads = 256;

template <bool BF16, bool DIVIDE>
__global__ __launch_bounds__(kTableThreads) void weights_kernel(RowSet rs, int32_t V, int32_t nparts, float c, float c_lo,
                                                                double cd, const StatPart *parts, const int32_t *mult,
                                                                float *table) {
  constexpr int kMine = kTablePieces / (kTableThreads / kWave);      // pieces of a wave
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t row = blockIdx.y, p = blockIdx.x;
  const void *rowp = row_base(rs, row, BF16);
  Piece<BF16> w[kMine];
  load_pieces<BF16, false>(w, rowp, p, wave * kMine, V, lane);
  u32x4 n[kMine];
  if constexpr (DIVIDE)
#pragma unroll
    for (int j = 0; j < kMine; ++j) n[j] = load_mult<true>(mult, piece_token(p, wave * kMine + j, lane), V);
  // the row's maximum and total as above; a lane's first part stays in registers (V <= 131 072: all of them)
  const StatPart *rp = parts + (int64_t) row * nparts;
  const float pm = lane < nparts ? rp[lane].m : -INFINITY;
  const double pz = lane < nparts ? rp[lane].z : 0.0;
  float top = pm;
  for (int32_t k = lane + kWave; k < nparts; k += kWave) top = fmaxf(top, rp[k].m);
  const float M = wave_max(top);
  const double up = exp2((double) (pm - M) * cd);
  double z = pz > 0.0 ? pz * up : 0.0;
  for (int32_t k = lane + kWave; k < nparts; k += kWave)
    if (rp[k].z > 0.0) z += rp[k].z * exp2((double) (rp[k].m - M) * cd);
  const double iz = 1.0 / wave_sum(z);
  const bool kept = p < kWave;                           // uniform
  const float m = kept ? __int_as_float(read_lane(__float_as_int(pm), p)) : rp[p].m;
  const double scale = (kept ? read_lane(up, p) : exp2((double) (m - M) * cd)) * iz;
  float *out = table + (int64_t) row * V;
  const bool whole = (p + 1) * kPartElems <= V;
  float e[4 * kMine];
  piece_logits<BF16>(w, p, wave * kMine, V, lane, e);
#pragma unroll
  for (int k = 0; k < 4 * kMine; ++k) e[k] = part_exp(e[k], m, c, c_lo);
#pragma unroll
  for (int j = 0; j < kMine; ++j) {
    f32x4_any v = scaled(e + 4 * j, scale);
    if constexpr (DIVIDE) v = divided(v, n[j]);
    store_piece(out, v, piece_token(p, wave * kMine + j, lane), V, whole);
  }
}

// =============================================================================================
// gather: out[r][g] = sum over members t of G_g of table[r][t], table row staged in LDS.
// =============================================================================================


// Workgroup id -> (row, chunk).  Workgroups are dealt to the 8 XCDs round-robin by id, and each XCD has to bring
// the table rows and the membership of its own workgroups into its own L2.  With row_parts = 2^row_shift, XCD x
// takes the rows that are x % row_parts modulo row_parts and the chunks that are x / row_parts modulo 8 / row_parts.
// (A shift: a division is some 30 dependent instructions ahead of a workgroup's first load, and one is left.)
// False: the workgroup has none.
__device__ __forceinline__ bool gather_place(const GatherMap &m, int32_t nrows, int32_t nchunks, int32_t &row, int32_t &chunk) {
  const uint32_t xcd = blockIdx.x & 7, y = blockIdx.x >> 3, turn = y / (uint32_t) m.chunks_each;
  row = (int32_t) ((xcd & ((1u << m.row_shift) - 1)) + (turn << m.row_shift));
  chunk = (int32_t) ((xcd >> m.row_shift) + ((y - turn * (uint32_t) m.chunks_each) << (3 - m.row_shift)));
  return row < nrows && chunk < nchunks;
}

// One tile of a table row, global memory -> LDS directly: every load of the tile is in flight at once
// and none passes through a register (a wave's instruction fills 64 pieces in lane order, which is
// the table's own order).  16 bytes per lane, or 4 where the row or the tile does not start on 16
// bytes.  The caller waits (vmcnt) and meets the other waves.  tab: 16-byte aligned.
__device__ __forceinline__ void stage_tile(float *tab, const float *src, int32_t tl, int tid) {
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if ((((uintptr_t) src | (uintptr_t) (4 * tl)) & 15) == 0) {        // uniform
    const float4 *s4 = reinterpret_cast<const float4 *>(src);
    const int32_t n4 = tl >> 2;
    for (int32_t k0 = wave * kWave; k0 < n4; k0 += kGatherThreads)
      if (k0 + lane < n4)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void *) (s4 + k0 + lane),
            (__attribute__((address_space(3))) void *) (tab + 4 * k0), 16, 0, 0);
  } else {
    for (int32_t k0 = wave * kWave; k0 < tl; k0 += kGatherThreads)
      if (k0 + lane < tl)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void *) (src + k0 + lane),
            (__attribute__((address_space(3))) void *) (tab + k0), 4, 0, 0);
  }
}

// A workgroup's sums, from LDS to memory: 16 bytes at a time where both sides allow it.
__device__ __forceinline__ void store_sums(float *dst, const float *sums, int32_t ng) {
  if ((((uintptr_t) dst | (uintptr_t) ng) & 15) == 0 && (ng & 3) == 0) {
    for (int32_t i = 4 * threadIdx.x; i < ng; i += 4 * kGatherThreads)
      *reinterpret_cast<float4 *>(dst + i) = *reinterpret_cast<const float4 *>(sums + i);
  } else {
    for (int32_t i = threadIdx.x; i < ng; i += kGatherThreads) dst[i] = sums[i];
  }
}

// Four consecutive entries of a CSR array of nnz, from position j on where they lie inside it.
__device__ __forceinline__ u32x4 csr_load4(const void *p, int32_t j, int32_t nnz) {
  const uint32_t *q = reinterpret_cast<const uint32_t *>(p);
  if (nnz >= 4) return load16<false>(q + min(j, nnz - 4));
  u32x4 r = {0, 0, 0, 0};                           // fewer than four entries in all
  for (int k = 0; k < 4; ++k) {
    const int32_t at = nnz - 4 + k;
    if (at >= 0) r[k] = q[at];
  }
  return r;
}

// What the four entries loaded for position j add to a sum: those from j on, inside the group that ends
// at `end`, and of the tile (added in pairs: a chain of four and then the tree over the lanes would
// round once or twice more).  WHOLE: the tile is the whole row, which every member lies in.
template <bool WEIGHTED, bool WHOLE>
__device__ __forceinline__ float csr_add4(const float *tab, int32_t zero, int32_t t0, int32_t tl, const u32x4 m,
                                          const u32x4 w, int32_t j, int32_t end, int32_t nnz, float acc) {
  const int32_t skip = min(j, nnz - 4) - j;            // below 0 where the load was moved back into the array
  const uint32_t count = (uint32_t) max(end - j, 0);
  float v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int32_t t = WHOLE ? (int32_t) m[k] : (int32_t) m[k] - t0;
    // from j on and inside the group, in one comparison
    const bool mine = (uint32_t) (skip + k) < count && (WHOLE || (uint32_t) t < (uint32_t) tl);
    v[k] = tab[mine ? t : zero];
  }
  if constexpr (WEIGHTED)
    return acc + (fmaf(v[0], __uint_as_float(w[0]), v[1] * __uint_as_float(w[1])) +
                  fmaf(v[2], __uint_as_float(w[2]), v[3] * __uint_as_float(w[3])));
  else
    return acc + ((v[0] + v[1]) + (v[2] + v[3]));
}

// Entries above which a group is left to csr_long_sums: 16 trips of its own W lanes, and far above the mean
// size (where most groups are that large, a few lanes each is the better split).
static int32_t csr_long_size(int64_t nnz, int32_t G, int W) {
  return (int32_t) std::min<int64_t>(INT32_MAX, std::max<int64_t>(64 * W, 4 * (nnz / G)));
}

// Sums over the groups [g_begin, g_end) of the table tile tab[0 .. tl) = tokens [t0, t0 + tl), read
// straight from the CSR by a workgroup of kGatherThreads; sink(g, sum) is called by one lane per
// group.  tab[zero] must read 0.  W lanes share a group, each taking four consecutive entries with
// one 16-byte load (kept inside the nnz entries of the array; what lies outside the group is sent to
// the zero slot); a sub-wave works on kInFlight groups at a time, and while it sums them the
// entries of its next ones and the bounds of those after them are on their way.
// A group of more than long_size entries would keep its few lanes at it, one trip to the L2 after another,
// long after all others are done (one group of 10 000 beside 20 000 of 8, 8 rows: the step took 222 us
// with 8 lanes a group and one entry a lane, 288 with two and four, 137 with this).  Only its first trip
// is added; *has_long (in LDS, false before) tells that csr_long_sums has something to do.
// csr_start asks for the first groups' bounds and entries: ahead of the tile, so that their two trips to memory
// are over when it has come.
constexpr int kCsrInFlight = 4;
template <bool WEIGHTED>
struct CsrGroups {
  int32_t beg[kCsrInFlight], end[kCsrInFlight];     // of the groups that are summed next
  int32_t beg2[kCsrInFlight], end2[kCsrInFlight];   // of those after them
  u32x4 m[kCsrInFlight], w[WEIGHTED ? kCsrInFlight : 1];      // entries of the next ones
};

template <int W>
__device__ __forceinline__ void csr_bounds(int32_t gb, int32_t g_end, const int32_t *row_ptr,
                                           int32_t (&beg)[kCsrInFlight], int32_t (&end)[kCsrInFlight]) {
#pragma unroll
  for (int u = 0; u < kCsrInFlight; ++u) {
    const int32_t g = min(gb + u * (kGatherThreads / W) + (int32_t) threadIdx.x / W, g_end - 1);
    beg[u] = row_ptr[g];
    end[u] = row_ptr[g + 1];
  }
}

template <int W, bool WEIGHTED>
__device__ __forceinline__ void csr_start(CsrGroups<WEIGHTED> &c, int32_t g_begin, int32_t g_end, const int32_t *row_ptr,
                                          const int32_t *members, int32_t nnz, const float *weights) {
  csr_bounds<W>(g_begin, g_end, row_ptr, c.beg, c.end);
  csr_bounds<W>(min(g_begin + kCsrInFlight * (kGatherThreads / W), g_end - 1), g_end, row_ptr, c.beg2, c.end2);
#pragma unroll
  for (int u = 0; u < kCsrInFlight; ++u) {
    const int32_t j = c.beg[u] + 4 * ((int32_t) threadIdx.x % W);
    c.m[u] = csr_load4(members, j, nnz);
    if constexpr (WEIGHTED) c.w[u] = csr_load4(weights, j, nnz);
  }
}

template <int W, bool WEIGHTED, bool WHOLE, typename Sink>
__device__ __forceinline__ void csr_sums(const CsrGroups<WEIGHTED> &start, const float *tab, int32_t zero, int32_t t0,
                                         int32_t tl, int32_t g_begin, int32_t g_end, const int32_t *row_ptr,
                                         const int32_t *members, int32_t nnz, const float *weights, int32_t long_size,
                                         bool *has_long, Sink sink) {
  constexpr int kInFlight = kCsrInFlight;
  constexpr int nsub = kGatherThreads / W;
  constexpr int kPass = nsub * kInFlight;           // groups per turn of the workgroup
  // At the most lanes a group, second trips are the rule: they are asked for together (5 % of the step at
  // sizes of 1 to 128).  With fewer lanes the test alone costs more than it gives (2.5 % of the step at
  // 32 members), and with weights there are no registers for it.
  constexpr bool kAskSecond = W == 16 && !WEIGHTED;
  const int sub = threadIdx.x / W, sl = threadIdx.x % W;
  struct Bounds { int32_t beg[kInFlight], end[kInFlight]; };
  struct Entries { u32x4 m[kInFlight], w[kInFlight]; };
  auto bounds = [&](int32_t gb, Bounds &r) { csr_bounds<W>(gb, g_end, row_ptr, r.beg, r.end); };
  auto load4 = [&](const void *p, int32_t j) { return csr_load4(p, j, nnz); };
  auto entries = [&](const Bounds &r, Entries &e) {
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const int32_t j = r.beg[u] + 4 * sl;
      e.m[u] = load4(members, j);
      if constexpr (WEIGHTED) e.w[u] = load4(weights, j);
    }
  };
  auto add4 = [&](const u32x4 m, const u32x4 w, int32_t j, int32_t end, float acc) {
    return csr_add4<WEIGHTED, WHOLE>(tab, zero, t0, tl, m, w, j, end, nnz, acc);
  };
  Bounds now, after;
  Entries e;
#pragma unroll
  for (int u = 0; u < kInFlight; ++u) {
    now.beg[u] = start.beg[u]; now.end[u] = start.end[u];
    after.beg[u] = start.beg2[u]; after.end[u] = start.end2[u];
    e.m[u] = start.m[u];
    if constexpr (WEIGHTED) e.w[u] = start.w[u];
  }
  for (int32_t gb = g_begin; gb < g_end; gb += kPass) {
    Entries en;
    Bounds later;
    if (gb + kPass < g_end) {                       // uniform over the workgroup
      entries(after, en);
      bounds(min(gb + 2 * kPass, g_end - 1), later);
    }
    u32x4 second[kAskSecond ? kInFlight : 1];
    if constexpr (kAskSecond) {
#pragma unroll
      for (int u = 0; u < kInFlight; ++u)
        if (now.beg[u] + 4 * (sl + W) < now.end[u]) second[u] = load4(members, now.beg[u] + 4 * (sl + W));
    }
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      float acc = add4(e.m[u], e.w[u], now.beg[u] + 4 * sl, now.end[u], 0.f);
      int32_t j = now.beg[u] + 4 * (sl + W);
      if (j < now.end[u]) {                         // longer than one trip
        if (now.end[u] - now.beg[u] > long_size) {
          *has_long = true;
          j = now.end[u];
        } else if constexpr (kAskSecond) {
          acc = add4(second[u], second[u], j, now.end[u], acc);
          j += 4 * W;
        }
        for (; j < now.end[u]; j += 4 * W) {
          const u32x4 m = load4(members, j);
          u32x4 w = m;
          if constexpr (WEIGHTED) w = load4(weights, j);
          acc = add4(m, w, j, now.end[u], acc);
        }
      }
      acc = subwave_sum<W>(acc);
      const int32_t g = gb + u * nsub + sub;
      if (g < g_end && sl == W - 1) sink(g, acc);
    }
    now = after;
    after = later;
    e = en;
  }
}

// The groups that csr_sums left: a wave adds the entries of each beyond its first trip, four loads a lane on
// their way, and hands their sum to more(g, sum).  A barrier lies between csr_sums and this.
template <int W, bool WEIGHTED, bool WHOLE, typename More>
__device__ void csr_long_sums(const float *tab, int32_t zero, int32_t t0, int32_t tl, int32_t g_begin,
                              int32_t g_end, const int32_t *row_ptr, const int32_t *members, int32_t nnz,
                              const float *weights, int32_t long_size, More more) {
  constexpr int kAtOnce = 4;
  const int lane = threadIdx.x & (kWave - 1);
  for (int32_t g0 = g_begin + (threadIdx.x - lane); g0 < g_end; g0 += kGatherThreads) {
    const int32_t g = g0 + lane;
    const int32_t begs = g < g_end ? row_ptr[g] : 0, ends = g < g_end ? row_ptr[g + 1] : 0;
    unsigned long long longs = __ballot(ends - begs > long_size);
    while (longs) {                                 // uniform over the wave, as everything in it
      const int l = __ffsll((long long) longs) - 1;
      longs &= longs - 1;
      const int32_t end = __builtin_amdgcn_readlane(ends, l);
      float sum = 0.f;
      for (int32_t j0 = __builtin_amdgcn_readlane(begs, l) + 4 * W; j0 < end; j0 += kAtOnce * 4 * kWave) {
        u32x4 m[kAtOnce], w[kAtOnce];
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q)
          if (j0 + q * 4 * kWave < end) {
            m[q] = csr_load4(members, j0 + 4 * (q * kWave + lane), nnz);
            if constexpr (WEIGHTED) w[q] = csr_load4(weights, j0 + 4 * (q * kWave + lane), nnz);
          }
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q)
          if (j0 + q * 4 * kWave < end)
            sum = csr_add4<WEIGHTED, WHOLE>(tab, zero, t0, tl, m[q], w[q], j0 + 4 * (q * kWave + lane), end, nnz, sum);
      }
      sum = subwave_sum<64>(sum);
      if (lane == kWave - 1) more(g0 + l, sum);
    }
  }
}

// Totals of max(0, sum) per run of kRunGroups groups (to runs) and over all ng sums of a workgroup
// (to *total), in double and in a fixed order; sums: 16-byte aligned LDS, readable up to the next
// multiple of 4.  Four neighbouring lanes cover one run, four groups each.
__device__ __forceinline__ void run_totals(const float *sums, int32_t ng, double *runs, double *total) {
  __shared__ double wsum[kGatherWaves];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  const float4 *sums4 = reinterpret_cast<const float4 *>(sums);
  double part = 0.0;
#pragma unroll
  for (int j = 0; j < kMaxChunkGroups / (4 * kGatherThreads); ++j) {
    const int32_t i4 = threadIdx.x + j * kGatherThreads;
    const int32_t g = 4 * i4;
    double s = 0.0;
    if (g < ng) {
      const float4 v = sums4[i4];
      s = ((double) fmaxf(v.x, 0.f) + (g + 1 < ng ? (double) fmaxf(v.y, 0.f) : 0.0)) +
          ((g + 2 < ng ? (double) fmaxf(v.z, 0.f) : 0.0) + (g + 3 < ng ? (double) fmaxf(v.w, 0.f) : 0.0));
    }
    s = subwave_sum<4>(s);
    if ((lane & 3) == 0 && g < ng) {
      runs[i4 >> 2] = s;
      part += s;
    }
  }
  part = subwave_sum<64>(part);
  if (lane == kWave - 1) wsum[wave] = part;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kGatherWaves; ++w) t += wsum[w];
    *total = t;
  }
}

// A workgroup sums a chunk of consecutive groups of one row (gather_place).
// LDS holds a tile of the table (tile_len tokens, the zero slot behind it) and the chunk's sums
// (groups_per_chunk, a multiple of 4).  CSUM: only run and chunk totals leave, as from the prepared
// gather; otherwise every sum.
// Bound by the L2, which hands every row its own copy of the members (4 bytes an entry, once per
// tile).  One entry per lane and load, with every pass waiting for its bounds, then its entries, took
// 28.3 us at V = 16 384, 32 members, 32 rows, and 13.2 us to scan the sums; this takes 12.6, and 6.4 to
// locate the draw (V = 65 536, 64 rows: 450 us and 51 us before, 189 and 9 now).  Behind the L2 it is the vector
// instructions of an entry that count: without the test for the tile where there is one only (WHOLE) and
// with one comparison for both ends of a group 14.0 -> 12.6 us, V = 32 768, 64 rows 71.8 -> 67.4; with weights
// 16.0 -> 14.8, V = 65 536, 64 rows 234 -> 223.  The first groups' bounds and entries asked for ahead of the tile: 12.2 -> 11.9
// there; whole calls V = 65 536, 64 rows 218 -> 212, fp32, V = 32 768, 1 to 128 members, 128 rows 450 -> 440, one sequence of
// V = 1024 (small step) 10.7 -> 10.2, eight of V = 4096 17.1 -> 16.3.
template <int W, bool CSUM, bool WEIGHTED, bool WHOLE>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(
    int32_t V, int32_t G, int32_t nrows, GatherMap map, int32_t nchunks, int32_t groups_per_chunk, int32_t ntiles,
    int32_t tile_len, int32_t nnz, int32_t long_size, const int32_t *row_ptr, const int32_t *members,
    const float *weights, const float *table, float *out, double *csum, int64_t csum_stride, double *runs) {
  __shared__ __attribute__((aligned(16))) float lds[kTileMax];
  __shared__ bool has_long;
  float *sums = lds, *tab = lds + groups_per_chunk;
  int32_t r, chunk;
  if (!gather_place(map, nrows, nchunks, r, chunk)) return;   // whole workgroup leaves together, before any barrier
  const float *src = table + (int64_t) r * V;
  const int32_t g_begin = chunk * groups_per_chunk;
  const int32_t ng = min(groups_per_chunk, G - g_begin);
  CsrGroups<WEIGHTED> groups;
  for (int tile = 0; tile < (WHOLE ? 1 : ntiles); ++tile) {
    const int32_t t0 = tile * tile_len;
    const int32_t tl = min(tile_len, V - t0);
    if (tl <= 0) break;                             // uniform: no tile starts past the row
    // With weights the compiler must not know that the groups are the same in every tile: it would keep the
    // addresses of the first ones' bounds from one tile to the next, 16 registers that this form does not
    // have (3 went to scratch: V = 65 536, 32 members, one sequence 74.5 us instead of 65.8).
    int32_t first = g_begin;
    if constexpr (WEIGHTED && !WHOLE) asm volatile("" : "+s"(first));
    // Where there is one turn of the workgroup and registers to spare, the entries of its groups are kept for the
    // next tile (V = 65 536, 32 members, one row: the call 27.0 -> 26.4 us).
    constexpr bool kKeep = W <= 8 && !WEIGHTED;
    if (WHOLE || !kKeep || tile == 0 || ng > kCsrInFlight * (kGatherThreads / W))
      csr_start<W>(groups, first, first + ng, row_ptr, members, nnz, weights);
    stage_tile(tab, src + t0, tl, threadIdx.x);
    if (threadIdx.x == 0) {
      tab[tile_len] = 0.f;
      if (tile == 0) has_long = false;              // the same groups are long in every tile
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);             // vmcnt(0): this wave's part of the tile has landed
    __syncthreads();
    csr_sums<W, WEIGHTED, WHOLE>(groups, tab, tile_len, t0, tl, first, first + ng, row_ptr, members, nnz, weights,
                          long_size, &has_long, [&](int32_t g, float a) {
                            // the same lane in every tile: no other touches this sum meanwhile
                            sums[g - g_begin] = tile > 0 ? sums[g - g_begin] + a : a;
                          });
    __syncthreads();                                // everyone is done with the tile
    if (has_long) {                                 // uniform
      csr_long_sums<W, WEIGHTED, WHOLE>(tab, tile_len, t0, tl, g_begin, g_begin + ng, row_ptr, members, nnz, weights,
                                 long_size, [&](int32_t g, float a) { sums[g - g_begin] += a; });
      __syncthreads();
    }
  }
  if constexpr (CSUM) {
    run_totals(sums, ng, runs + ((int64_t) r * nchunks + chunk) * (groups_per_chunk / kRunGroups),
               csum + r * csum_stride + chunk);
  } else {
    store_sums(out + (int64_t) r * G + g_begin, sums, ng);
  }
}

// =============================================================================================
// finalize: group from the residual by inverse CDF, then the token inside it (Eq. 10).
// =============================================================================================

constexpr int kFinalThreads = 512;
constexpr int32_t kScanGroups = 4096;    // sums of a row that finalize reads and scans whole

struct CdfPick {
  int32_t index;    // first index whose running sum exceeds the threshold; -1 if nothing has mass
  double total, lo, hi;   // total mass; running sum before / after the chosen bin
};

// Inverse CDF over f(0..n-1) >= 0 by a whole workgroup of NT threads.  Each thread owns a
// contiguous run, so the running sum is the ascending one up to fp64 rounding.  All threads get
// the result.  The threshold is u * total.
template <int NT, int kRegRun = 32, typename F>   // kRegRun: runs up to this length are held in registers
__device__ CdfPick block_inverse_cdf(int32_t n, F f, double u) {
  __shared__ double wave_tot[NT / kWave];
  __shared__ int first_thread, last_pos;
  __shared__ CdfPick res;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int32_t run = (n + NT - 1) / NT;
  const int32_t lo_i = min(n, tid * run), hi_i = min(n, lo_i + run);
  const bool in_regs = run <= kRegRun;           // uniform
  if (tid == 0) { first_thread = INT_MAX; last_pos = -1; }
  double mine = 0.0;
  double vals[kRegRun];
  if (in_regs) {
    // all loads of the run are issued before the first is used
#pragma unroll
    for (int j = 0; j < kRegRun; ++j) vals[j] = (lo_i + j < hi_i) ? f(lo_i + j) : 0.0;
#pragma unroll
    for (int j = 0; j < kRegRun; ++j)
      if (vals[j] > 0.0) mine += vals[j];
  } else {
    for (int32_t k = lo_i; k < hi_i; ++k) {
      const double v = f(k);
      if (v > 0.0) mine += v;
    }
  }
  // inclusive scan inside the wave, then across waves
  const double inc = wave_scan(mine);
  if (lane == kWave - 1) wave_tot[wave] = inc;
  __syncthreads();
  double before = 0.0, total = 0.0;
  for (int w = 0; w < NT / kWave; ++w) {
    if (w < wave) before += wave_tot[w];
    total += wave_tot[w];
  }
  const double excl = before + (inc - mine);
  const double goal = u * total;
  // the first thread whose run carries the running sum past the threshold: first lane of each
  // wave by ballot, then one LDS atomic per wave
  const unsigned long long hit = __ballot(mine > 0.0 && excl + mine > goal);
  if (hit != 0 && lane == __ffsll((long long) hit) - 1) atomicMin(&first_thread, tid);
  __syncthreads();
  const int ft = __builtin_amdgcn_readfirstlane(first_thread);   // the same in every lane
  if (in_regs && ft != INT_MAX) {
    // The crossing lies inside thread ft's run: its wave looks at the run's bins side by side, one
    // per lane (a run held in registers is at most 32 long), instead of thread ft walking them
    // one after the other.
    static_assert(kRegRun <= kWave, "one lane per bin of a run");
    if (wave == (ft >> 6)) {                     // uniform over the wave
      const int fl = ft & (kWave - 1);
      const double base = read_lane(excl, fl);
      const int32_t lo = read_lane(lo_i, fl), hi = read_lane(hi_i, fl);
      const int32_t k = lo + lane;
      double v = k < hi ? (double) f(k) : 0.0;
      if (!(v > 0.0)) v = 0.0;
      const double run_inc = wave_scan(v);
      const unsigned long long pos = __ballot(v > 0.0);
      const unsigned long long cross = __ballot(v > 0.0 && base + run_inc > goal);
      // the first bin that carries the sum past the threshold; rounding may leave none (the sum
      // of the run was taken in another order): then the last bin that has mass
      const int l = cross ? __ffsll((long long) cross) - 1 : 63 - __clzll((long long) pos);
      const double top = base + read_lane(run_inc, l), width = read_lane(v, l);
      if (lane == 0) {
        res.index = lo + l; res.hi = top; res.lo = top - width; res.total = total;
      }
    }
  } else if (ft == tid) {
    double cum = excl;
    int32_t last = lo_i;
    bool done = false;
    for (int32_t k = lo_i; k < hi_i && !done; ++k) {
      const double v = f(k);
      if (!(v > 0.0)) continue;
      const double nxt = cum + v;
      if (nxt > goal) { res.index = k; res.lo = cum; res.hi = nxt; done = true; }
      else { last = k; cum = nxt; }
    }
    if (!done) {   // summation order: excl + mine > goal, yet the walk stayed below: last bin
      const double v = (double) f(last);
      res.index = last; res.lo = cum - v; res.hi = cum;
    }
    res.total = total;
  }
  if (ft == INT_MAX) {
    // rounding at the top end (or no mass at all): the last index that has mass
    int32_t my_last = -1;
    for (int32_t k = lo_i; k < hi_i; ++k)
      if (f(k) > 0.0) my_last = k;
    if (my_last >= 0) atomicMax(&last_pos, my_last);
    __syncthreads();
    if (tid == 0) {
      res.index = last_pos; res.total = total; res.lo = total; res.hi = total;
      if (last_pos >= 0) res.lo = total - f(last_pos);
    }
  }
  __syncthreads();
  CdfPick out = res;
  __syncthreads();   // res / first_thread may be reused by the next call
  return out;
}

__device__ __forceinline__ bool near_edge(const CdfPick &p, double u) {
  const double goal = u * p.total;
  const bool near_lo = p.lo > 0.0 && (goal - p.lo) < 1e-6 * p.total;
  const bool near_hi = p.hi < p.total && (p.hi - goal) < 1e-6 * p.total;
  return near_lo || near_hi;
}

// The token inside the chosen group (Eq. 10) and the sequence's last outputs, by one whole workgroup
// of NT threads; pg: the group draw (total mass <= 0: the fallback to T of this row).
template <bool BF16, int NT>
__device__ void finish_sequence(const FinalizeArgs &fa, int32_t G, int b, int32_t istar, const void *trow,
                                const RowStat &st, const Uniforms &u, CdfPick pg) {
  const int32_t K = fa.K;
  const int32_t *row_ptr = fa.row_ptr, *members = fa.members, *mult = fa.mult;
  const float *wts = fa.weights;
  const double cd = fa.cd;

  // q(t) w_{k,t} of CSR entry j on the decision row (q(t) / N(t) under the equal split), in double
  auto weight = [&](int32_t j) -> double {
    const int32_t t = members[j];
    const double e = exp2((double) (logit_at<BF16>(trow, t) - st.M) * cd);
    return wts ? e * (double) wts[j] / st.Z : e / (st.Z * (double) mult[t]);
  };

  bool fallback = false;
  if (!(pg.total > 0.0) || pg.index < 0) {
    // Residual total <= 0 (cannot happen in exact arithmetic): draw from T of this row instead.
    fallback = true;
    float *Rb = fa.R + (int64_t) b * G;
    for (int32_t g = threadIdx.x; g < G; g += NT) {
      double s = 0.0;
      for (int32_t j = row_ptr[g]; j < row_ptr[g + 1]; ++j) s += weight(j);
      Rb[g] = (float) s;
    }
    __syncthreads();
    pg = block_inverse_cdf<NT>(G, [&](int32_t g) { return (double) Rb[g]; }, (double) u.grp);
  }
  const int32_t gs = pg.index < 0 ? 0 : pg.index;

  const int32_t beg = row_ptr[gs], end = row_ptr[gs + 1];
  CdfPick pt;
  constexpr int kTokRounds = 4;          // entries per lane the one-wave path keeps in registers
  if (end - beg <= kTokRounds * kWave) {
    // The token inside the group (Eq. 10) by the first wave alone: every entry's mass is loaded
    // once, all loads in flight together, and kept in registers for the total and for the scan.
    if (threadIdx.x < kWave) {
      const int lane = threadIdx.x;
      const int32_t n = end - beg;
      double w[kTokRounds];
#pragma unroll
      for (int c = 0; c < kTokRounds; ++c) {
        const int32_t j = c * kWave + lane;
        w[c] = j < n ? weight(beg + j) : 0.0;
        if (!(w[c] > 0.0)) w[c] = 0.0;
      }
      double total = 0.0;
#pragma unroll
      for (int c = 0; c < kTokRounds; ++c)
        if (c * kWave < n) total += wave_sum(w[c]);                      // ascending, 64 at a time
      pt.index = -1; pt.total = total; pt.lo = pt.hi = 0.0;
      const double goal = (double) u.tok * total;
      double base = 0.0, last_v = 0.0;
      int32_t last = -1;
      bool done = false;
#pragma unroll
      for (int c = 0; c < kTokRounds; ++c) {
        if (done || c * kWave >= n) continue;                            // uniform
        const double inc = wave_scan(w[c]);
        const unsigned long long pos = __ballot(w[c] > 0.0);
        if (pos) {
          const int hl = 63 - __clzll((long long) pos);
          last = c * kWave + hl;
          last_v = read_lane(w[c], hl);
        }
        const unsigned long long hit = __ballot(w[c] > 0.0 && base + inc > goal);
        if (hit) {
          const int l = __ffsll((long long) hit) - 1;
          pt.index = c * kWave + l;
          pt.hi = base + read_lane(inc, l);
          pt.lo = pt.hi - read_lane(w[c], l);
          done = true;
        } else {
          base += read_lane(inc, kWave - 1);
        }
      }
      if (!done && last >= 0) {          // rounding at the top end: the last entry that has mass
        pt.index = last; pt.hi = total; pt.lo = total - last_v;
      }
    }
  } else {
    pt = block_inverse_cdf<NT>(end - beg, [&](int32_t j) { return weight(beg + j); }, (double) u.tok);
  }
  if (threadIdx.x == 0) {
    fa.out_groups[(int64_t) b * (K + 1) + istar] = gs;
    fa.out_tokens[(int64_t) b * (K + 1) + istar] = pt.index < 0 ? -1 : members[beg + pt.index];
    if (fa.diag) {
      if (pg.index >= 0 && near_edge(pg, (double) u.grp)) atomicAdd(&fa.diag->near_group, 1u);
      if (pt.index >= 0 && near_edge(pt, (double) u.tok)) atomicAdd(&fa.diag->near_token, 1u);
      if (fallback) atomicAdd(&fa.diag->residual_fallback, 1u);
    }
  }
}

// Inverse CDF over the run totals rp[0 .. n) >= 0, n <= 2 NT, by a workgroup of NT threads, two neighbouring
// runs each: the first whose running sum exceeds `goal`; index -1 if nothing has mass.  All threads get
// the result.  (Two barriers; block_inverse_cdf, which takes any function and any number, has four.)
template <int NT>
__device__ __forceinline__ CdfPick pick_run(const double *rp, int32_t n, double goal) {
  constexpr int kWaves = NT / kWave;
  __shared__ double wave_tot[kWaves];
  __shared__ CdfPick res;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t k = 2 * tid;
  double r0 = 0.0, r1 = 0.0;
  if (k < n) r0 = fmax(rp[k], 0.0);
  if (k + 1 < n) r1 = fmax(rp[k + 1], 0.0);
  const double mine = r0 + r1, inc = wave_scan(mine);
  if (lane == kWave - 1) wave_tot[wave] = inc;
  lds_barrier();
  const double tot = lane < kWaves ? wave_tot[lane] : 0.0, upto = wave_scan(tot);
  const unsigned long long pos = __ballot(tot > 0.0), hit = __ballot(tot > 0.0 && upto > goal);
  // the wave that holds the crossing; rounding at the top end may leave none: the last that has mass
  const int at = !pos ? 0 : hit ? __ffsll((long long) hit) - 1 : 63 - __clzll((long long) pos);
  if (wave == at) {                                   // uniform over the wave
    const double before = read_lane(upto, at) - read_lane(tot, at), total = read_lane(upto, kWave - 1);
    const unsigned long long has = __ballot(mine > 0.0);
    const unsigned long long over = hit ? __ballot(mine > 0.0 && before + inc > goal) : 0;
    const int l = !has ? 0 : over ? __ffsll((long long) over) - 1 : 63 - __clzll((long long) has);
    if (lane == l) {
      const double lo = before + (inc - mine);
      const bool second = r0 <= 0.0 || (r1 > 0.0 && lo + r0 <= goal);
      res.index = !pos ? -1 : k + (second ? 1 : 0);
      res.total = total;
      res.lo = second ? lo + r0 : lo;
      res.hi = second ? lo + mine : lo + r0;
    }
  }
  lds_barrier();
  return res;
}

// The last step of a sequence, by one whole workgroup of NT threads.  The gather left no sums, only
// the totals of max(0, T[g] - D[g]) (T[g] on a bonus row) over chunks of chunk_groups consecutive
// groups and over runs of kRunGroups: the chunk and the run that hold the draw are located from
// them, and the run's sums are formed again here: 32 lanes a group, OWN entries a lane that stay in registers,
// so that the token of a group of up to 32 OWN is drawn without a second look at memory.  OWN = 4 where
// the mean group has more than 32 entries: V = 16 384, 1 to 128 members, 32 rows 11.6 us instead of 13.8,
// V = 32 768, 100 members, 16 rows 13.8 instead of 14.8; else one, since four cost 0.8 of 9.7 us at 32 members.
template <bool BF16, int NT, int OWN>
__device__ void finalize_sequence(const FinalizeArgs &fa, int32_t V, int32_t G, int b,
                                  const double *csum, int64_t csum_stride, const double *runs,
                                  int32_t nchunks, int32_t chunk_groups) {
  const int32_t K = fa.K;
  // asked for before anything waits for the accept length
  const double *cs = csum + b * csum_stride;
  const int ln = threadIdx.x & (kWave - 1);
  const double cs_any = cs[min(ln, nchunks - 1)];
  const int32_t istar = fa.accept_len[b];
  const bool rejected = istar < K;
  const int64_t trow_id = (int64_t) b * (K + 1) + istar;
  const void *trow = target_row(fa.rs, b, istar, BF16);
  const void *drow = draft_row(fa.rs, b, rejected ? istar : 0, BF16);
  const RowStat st = fa.rowstat[trow_id];
  const RowStat sd = fa.rowstat[fa.rs.nrows0 + (int64_t) b * K + (rejected ? istar : 0)];
  const Uniforms u = philox_uniforms(fa.seed, fa.offset, (uint32_t) b, (uint32_t) istar);
  const int32_t *row_ptr = fa.row_ptr, *members = fa.members, *mult = fa.mult;
  const float *wts = fa.weights;
  const double cd = fa.cd;

  // residual total and the chunk that holds u * total, from the per-chunk sums (ascending), 64 side by
  // side; every wave does the same
  CdfPick pg;
  {
    const double cs0 = ln < nchunks ? cs_any : 0.0;
    double S = wave_sum(cs0);
    for (int32_t c0 = kWave; c0 < nchunks; c0 += kWave) S += wave_sum(c0 + ln < nchunks ? cs[c0 + ln] : 0.0);
    const double goal = (double) u.grp * S;
    double cum = 0.0, base = 0.0;
    int32_t cstar = -1;
    for (int32_t c0 = 0; c0 < nchunks; c0 += kWave) {
      const double v = c0 == 0 ? cs0 : (c0 + ln < nchunks ? cs[c0 + ln] : 0.0);
      const double inc = wave_scan(v);
      const unsigned long long pos = __ballot(v > 0.0), hit = __ballot(v > 0.0 && cum + inc > goal);
      if (pos) {
        const int l = hit ? __ffsll((long long) hit) - 1 : 63 - __clzll((long long) pos);
        cstar = c0 + l;
        base = cum + (read_lane(inc, l) - read_lane(v, l));
      }
      if (hit) break;
      cum += read_lane(inc, kWave - 1);
    }
    pg.index = -1; pg.total = S; pg.lo = pg.hi = 0.0;
    if (S > 0.0 && cstar >= 0) {
      const int32_t g0 = cstar * chunk_groups, ng = min(chunk_groups, G - g0);
      {
        // The gather left no sums, only the totals of runs of kRunGroups groups: find the run
        // that holds the crossing, form its groups' sums again -- 32 lanes per group, the table
        // kernel's arithmetic for every entry (Eq. 8 on the decision row) -- and walk them.
        static_assert(NT == kRunGroups * 32, "one half-wave per group of a run");
        constexpr int kOwnEntries = 32 * OWN;
        // Above this a group is summed by the whole workgroup: a half-wave alone would make a chain of trips
        // to memory (V = 65 536, 8 members, 100 groups of 1000, 8 rows: 53 us; now 18).
        constexpr int32_t kLongGroup = 256;
        __shared__ float run_r[kRunGroups];
        const int32_t nruns = (ng + kRunGroups - 1) / kRunGroups;
        const double *rp = runs + ((int64_t) b * nchunks + cstar) * (chunk_groups / kRunGroups);
        static_assert(kMaxChunkGroups / kRunGroups <= 2 * NT, "two runs per thread at most");
        const CdfPick pr = pick_run<NT>(rp, nruns, goal - base);
        if (pr.index >= 0) {
          __shared__ int32_t run_n[kRunGroups], run_beg[kRunGroups];
          __shared__ bool run_has[kRunGroups];          // some entry of the group adds to it
          const double izt = 1.0 / st.Z, izd = rejected ? 1.0 / sd.Z : 0.0;
          const int32_t gr0 = g0 + pr.index * kRunGroups;
          const int k = threadIdx.x >> 5, l = threadIdx.x & 31;
          const int32_t g = gr0 + k;
          float acc = 0.f;
          bool adds = false;
          // adds an entry, with the table kernel's arithmetic; share: w_{k,t}, or N(t)
          auto add = [&](float lt, float ld, float share) {
            double diff = __dmul_rn((double) exp_rel(lt, st.M, fa.c, fa.c_lo), izt);
            if (rejected) diff = __dsub_rn(diff, __dmul_rn((double) exp_rel(ld, sd.M, fa.c, fa.c_lo), izd));
            acc = wts ? fmaf((float) diff, share, acc)
                      : acc + (float) diff * __builtin_amdgcn_rcpf(share);
            adds = adds || (diff > 0.0 && share > 0.f);
          };
          auto add_entry = [&](int32_t j) {
            const int32_t t = members[j];
            add(logit_at<BF16>(trow, t), rejected ? logit_at<BF16>(drow, t) : 0.f,
                wts ? wts[j] : (float) mult[t]);
          };
          int32_t beg = 0, n_g = 0;
          if (g < g0 + ng) { beg = row_ptr[g]; n_g = row_ptr[g + 1] - beg; }
          int32_t own_t[OWN];
          float own_lt[OWN], own_ld[OWN], own_share[OWN];
#pragma unroll
          for (int e = 0; e < OWN; ++e) {
            const int32_t at = l + 32 * e;
            own_t[e] = at < n_g ? members[beg + at] : -1;
          }
#pragma unroll
          for (int e = 0; e < OWN; ++e) {
            own_lt[e] = own_ld[e] = -INFINITY;
            own_share[e] = 1.f;
            if (own_t[e] >= 0) {
              own_lt[e] = logit_at<BF16>(trow, own_t[e]);
              if (rejected) own_ld[e] = logit_at<BF16>(drow, own_t[e]);
              own_share[e] = wts ? wts[beg + l + 32 * e] : (float) mult[own_t[e]];
            }
          }
          if (n_g <= kLongGroup) {
#pragma unroll
            for (int e = 0; e < OWN; ++e)
              if (own_t[e] >= 0) add(own_lt[e], own_ld[e], own_share[e]);
            for (int32_t at = l + kOwnEntries; at < n_g; at += 32) add_entry(beg + at);
          }
          acc = subwave_sum<32>(acc);                   // total in the last lane of each 32
          const bool has = (__ballot(adds) >> (threadIdx.x & 32) & 0xffffffffull) != 0;   // of this half-wave
          if (l == 31) { run_r[k] = fmaxf(acc, 0.f); run_n[k] = n_g; run_has[k] = has; run_beg[k] = beg; }
          __syncthreads();
          const int ln0 = threadIdx.x & (kRunGroups - 1);
          if (__any(run_n[ln0] > kLongGroup)) {         // the same in every thread
            __shared__ float part_r[kRunGroups][NT / kWave];
            __shared__ bool part_has[kRunGroups][NT / kWave];
            for (int k2 = 0; k2 < kRunGroups; ++k2) {
              const int32_t n = run_n[k2], b2 = run_beg[k2];
              if (n <= kLongGroup) continue;
              acc = 0.f;
              adds = false;
              for (int32_t at = threadIdx.x; at < n; at += NT) add_entry(b2 + at);
              acc = subwave_sum<64>(acc);
              const bool any = __any(adds);
              if ((threadIdx.x & (kWave - 1)) == kWave - 1) {
                part_r[k2][threadIdx.x >> 6] = acc;
                part_has[k2][threadIdx.x >> 6] = any;
              }
            }
            __syncthreads();
            if (threadIdx.x < kRunGroups && run_n[threadIdx.x] > kLongGroup) {
              float sum = 0.f;
              bool any = false;
              for (int w = 0; w < NT / kWave; ++w) {
                sum += part_r[threadIdx.x][w];
                any = any || part_has[threadIdx.x][w];
              }
              run_r[threadIdx.x] = fmaxf(sum, 0.f);
              run_has[threadIdx.x] = any;
            }
            __syncthreads();
          }
          double cum = base + pr.lo, last_v = 0.0;
          int pick = -1, last = -1;
#pragma unroll
          for (int k2 = 0; k2 < kRunGroups; ++k2) {
            const double v = (double) run_r[k2];
            if (pick < 0 && v > 0.0) {
              if (cum + v > goal) { pick = k2; pg.lo = cum; pg.hi = cum + v; }
              else { last = k2; last_v = v; cum += v; }
            }
          }
          if (pick < 0) {
            // rounding (the run's total was summed in another order): the last group of the run that has
            // mass.  Where sums that cancel gave the run its total and none of them comes out positive
            // here, a group that has entries with q > p: any group with a positive sum had one.
            pick = last;
            for (int k2 = kRunGroups - 1; k2 >= 0 && last < 0; --k2)
              if (run_has[k2]) pick = k2;
            pg.hi = cum; pg.lo = cum - last_v;
          }
          if (pick >= 0) pg.index = gr0 + pick;         // none (cannot happen): the fallback below
          if (pick >= 0 && run_n[pick] <= kOwnEntries) {        // uniform over the workgroup
            // The token inside the group (Eq. 10) by the half-wave that formed the group's sum.
            const int wv = __builtin_amdgcn_readfirstlane(pick >> 1);
            if ((int) (threadIdx.x >> 6) == wv) {
              const int lane = threadIdx.x & (kWave - 1);
              double w[OWN];
              CdfPick pt;
              pt.index = -1; pt.total = 0.0; pt.lo = pt.hi = 0.0;
#pragma unroll
              for (int e = 0; e < OWN; ++e) {
                w[e] = 0.0;
                if (k == pick && own_t[e] >= 0) {
                  const double x = exp2((double) (own_lt[e] - st.M) * cd);
                  w[e] = wts ? x * (double) own_share[e] / st.Z : x / (st.Z * (double) own_share[e]);
                  if (!(w[e] > 0.0)) w[e] = 0.0;
                }
                pt.total += wave_sum(w[e]);             // ascending, 32 entries at a time
              }
              const double goal_t = (double) u.tok * pt.total;
              int32_t tok = -1;
              double upto = 0.0;
              bool done = false;
#pragma unroll
              for (int e = 0; e < OWN; ++e) {
                const double inc = wave_scan(w[e]);
                const unsigned long long pos = __ballot(w[e] > 0.0);
                const unsigned long long hit = __ballot(w[e] > 0.0 && upto + inc > goal_t);
                if (!done && pos) {                     // uniform; without a hit the last entry that has mass
                  const int src = hit ? __ffsll((long long) hit) - 1 : 63 - __clzll((long long) pos);
                  pt.index = 32 * e + (src & 31);
                  pt.hi = hit ? upto + read_lane(inc, src) : pt.total;
                  pt.lo = pt.hi - read_lane(w[e], src);
                  tok = read_lane(own_t[e], src);
                  done = hit != 0;
                }
                upto += read_lane(inc, kWave - 1);
              }
              if (lane == 0) {
                fa.out_groups[(int64_t) b * (K + 1) + istar] = pg.index;
                fa.out_tokens[(int64_t) b * (K + 1) + istar] = tok;
                if (fa.diag) {
                  if (near_edge(pg, (double) u.grp)) atomicAdd(&fa.diag->near_group, 1u);
                  if (pt.index >= 0 && near_edge(pt, (double) u.tok)) atomicAdd(&fa.diag->near_token, 1u);
                }
              }
            }
            return;                                     // the whole workgroup, together
          }
        }
      }
    }
  }
  finish_sequence<BF16, NT>(fa, G, b, istar, trow, st, u, pg);
}

// One workgroup per sequence.  csum, runs, nchunks, chunk_groups: the totals as the gather wrote them.
template <bool BF16, int OWN>
__global__ __launch_bounds__(kFinalThreads) void finalize_kernel(FinalizeArgs fa, int32_t V,
                                                                 int32_t G, const double *csum,
                                                                 int64_t csum_stride,
                                                                 const double *runs,
                                                                 int32_t nchunks,
                                                                 int32_t chunk_groups) {
  finalize_sequence<BF16, kFinalThreads, OWN>(fa, V, G, blockIdx.x, csum, csum_stride, runs, nchunks, chunk_groups);
}

// The last step from the sums themselves: few enough that all of them are read and scanned sooner than
// totals of them, a run and its sums formed again.  V = 4096, CSR, 8 rows: 100 members 7.0 us here, 9.3 from
// the totals; 48 members 6.6 and 8.5.
template <bool BF16>
__global__ __launch_bounds__(kFinalThreads) void finalize_sums_kernel(FinalizeArgs fa, int32_t G) {
  const int b = blockIdx.x;
  const int32_t istar = fa.accept_len[b];
  const int64_t trow_id = (int64_t) b * (fa.K + 1) + istar;
  const Uniforms u = philox_uniforms(fa.seed, fa.offset, (uint32_t) b, (uint32_t) istar);
  const float *sums = fa.R + (int64_t) b * G;
  const CdfPick pg = block_inverse_cdf<kFinalThreads, kScanGroups / kFinalThreads>(
      G, [&](int32_t g) { return (double) sums[g]; }, (double) u.grp);
  finish_sequence<BF16, kFinalThreads>(fa, G, b, istar, target_row(fa.rs, b, istar, BF16), fa.rowstat[trow_id], u, pg);
}

// ---------------------------------------------------------------------------------------------
// The same sum read from the prepared layout (pcg_prepared): no cross-lane reduction and no
// address arithmetic beyond a shift.  A workgroup owns one chunk of consecutive groups of one
// table row.  Wave w owns the blocks block_of(q, w), q = 0..3, of the chunk and walks them one
// after the other; lane l handles each block's 4 groups r*64 + l -- the same 16 groups in every
// tile pass, so their running sums stay in registers.  One 16-byte load per lane brings 2 slots for
// each of a block's 4 groups.  Results are put back into group order through LDS.  Without CSUM
// they leave with coalesced stores; with CSUM (the residual of pcg_verify, Eq. 8) only totals of
// max(0, .) leave, in double and summed in a fixed order: one per run of kRunGroups consecutive
// groups and one for the chunk.
// ---------------------------------------------------------------------------------------------

// One step of a block: 8 slots per lane, two for each of its 4 groups.  All eight reads are issued
// before the first sum waits for one (left to itself the compiler, short of registers, lets each
// addition wait for its own read).
__device__ __forceinline__ void gather_step(const float *tab, const uint4 w, float *acc) {
  const float a0 = tab[w.x & 0xffffu], a1 = tab[w.y & 0xffffu], a2 = tab[w.z & 0xffffu], a3 = tab[w.w & 0xffffu];
  const float b0 = tab[w.x >> 16], b1 = tab[w.y >> 16], b2 = tab[w.z >> 16], b3 = tab[w.w >> 16];
  __builtin_amdgcn_sched_barrier(0);
  acc[0] += a0; acc[1] += a1; acc[2] += a2; acc[3] += a3;
  acc[0] += b0; acc[1] += b1; acc[2] += b2; acc[3] += b3;
}

// The same with general weights (Eq. 4): every slot comes with its w_{k,t}, 8 floats per lane
// and step next to the 8 slots.
__device__ __forceinline__ void gather_step_w(const float *tab, const uint4 s, const float4 wa,
                                              const float4 wb, float *acc) {
  const float a0 = tab[s.x & 0xffffu], a1 = tab[s.y & 0xffffu], a2 = tab[s.z & 0xffffu], a3 = tab[s.w & 0xffffu];
  const float b0 = tab[s.x >> 16], b1 = tab[s.y >> 16], b2 = tab[s.z >> 16], b3 = tab[s.w >> 16];
  __builtin_amdgcn_sched_barrier(0);
  acc[0] = fmaf(a0, wa.x, acc[0]); acc[1] = fmaf(a1, wa.z, acc[1]);
  acc[2] = fmaf(a2, wb.x, acc[2]); acc[3] = fmaf(a3, wb.z, acc[3]);
  acc[0] = fmaf(b0, wa.y, acc[0]); acc[1] = fmaf(b1, wa.w, acc[1]);
  acc[2] = fmaf(b2, wb.y, acc[2]); acc[3] = fmaf(b3, wb.w, acc[3]);
}

// One step of one block as it comes from memory: 8 slots and, with weights, their 8 weights.
template <bool WEIGHTED>
struct GatherStep;
template <>
struct GatherStep<false> {
  uint4 s;
  __device__ __forceinline__ void load(const uint4 *__restrict__ data, const float4 *, int lane) {
    s = data[lane];
  }
  __device__ __forceinline__ void apply(const float *tab, float *acc) const { gather_step(tab, s, acc); }
};
template <>
struct GatherStep<true> {
  uint4 s;
  float4 w0, w1;
  __device__ __forceinline__ void load(const uint4 *__restrict__ data,
                                       const float4 *__restrict__ wdata, int lane) {
    s = data[lane];
    w0 = wdata[2 * lane];
    w1 = wdata[2 * lane + 1];
  }
  __device__ __forceinline__ void apply(const float *tab, float *acc) const {
    gather_step_w(tab, s, w0, w1, acc);
  }
};

// The prepared layout as the kernels see it.
struct PreparedView {
  const uint32_t *desc;
  const uint16_t *perm;
  const uint4 *data;
  const float4 *wdata;
  int32_t nchunks, chunk_groups, ntiles, tile_len, blocks_per_chunk;
};

// First unit and number of steps of a wave's blocks in one tile of one chunk (dsc; NULL: none).
__device__ __forceinline__ void load_desc(const uint32_t *dsc, int bpc, int wave,
                                          uint32_t (&steps)[kMaxBlocksPerWave],
                                          uint32_t (&offs)[kMaxBlocksPerWave]) {
#pragma unroll
  for (int q = 0; q < kMaxBlocksPerWave; ++q) {
    const int bl = block_of(q, wave);
    steps[q] = 0;
    offs[q] = 0;
    if (dsc && bl < bpc) {                            // uniform over the wave: scalar registers
      steps[q] = __builtin_amdgcn_readfirstlane(dsc[2 * bl + 1]);
      offs[q] = __builtin_amdgcn_readfirstlane(dsc[2 * bl]);
    }
  }
}

// A wave's way through its blocks, one after the other.  The steps come through a ring of registers
// that is always kRing steps ahead: slot i takes the steps i, i + kRing, ... of a block, and once the
// block has none left, step i of the wave's next block (in the last block of a tile: of the next
// tile's first), so that the stream never waits at a block's or a tile's end.
template <bool WEIGHTED>
struct SlotStream {
  // Steps in flight per wave.  A wave used to keep one step of each of its blocks in flight, so
  // one left with a single long block (or none beside it) waited for the L2 on every step: 17.0 us
  // at B = 1, V = 65 536 against 13.4 with this ring, 57.5 against 46.3 at B = 128, V = 32 768 with
  // groups of 1 to 128, 27.4 against 25.2 at B = 64, V = 65 536.  Six steps spill with weights and
  // change nothing without; eight spill (27.8 us).
  static constexpr int kRing = WEIGHTED ? 2 : 4;
  GatherStep<WEIGHTED> ring[kRing];
  bool filled = false;                                // the ring holds the first steps of the coming tile
  uint32_t steps[kMaxBlocksPerWave], offs[kMaxBlocksPerWave];             // this tile's blocks
  uint32_t succ_off[kMaxBlocksPerWave], succ_last[kMaxBlocksPerWave];     // what follows each of them

  // a scalar base and the lane as the only vector part: no address arithmetic per load
  __device__ __forceinline__ void load(int i, uint32_t unit, const uint4 *data, const float4 *wdata, int lane) {
    const uint32_t u = __builtin_amdgcn_readfirstlane(unit);
    ring[i].load(data + u, wdata + 2 * (size_t) u, lane);
  }

  // Before a tile (steps, offs set): finds what follows each block, nsteps / noffs being the next
  // tile's, and fills the ring unless the tile before has done so.
  __device__ __forceinline__ void begin(const uint32_t (&nsteps)[kMaxBlocksPerWave],
                                        const uint32_t (&noffs)[kMaxBlocksPerWave], const uint4 *data,
                                        const float4 *wdata, int lane) {
    uint32_t so = 0, sn = 0, first_off = 0, first_steps = 0;
#pragma unroll
    for (int q = kMaxBlocksPerWave - 1; q >= 0; --q)
      if (nsteps[q] > 0) { so = noffs[q]; sn = nsteps[q]; }
    const bool follows = sn > 0;
#pragma unroll
    for (int q = kMaxBlocksPerWave - 1; q >= 0; --q) {
      // nothing follows: the block's own first steps are read again, and not used
      succ_off[q] = sn > 0 ? so : offs[q];
      succ_last[q] = (sn > 0 ? sn : max(steps[q], 1u)) - 1;
      if (steps[q] > 0) { so = first_off = offs[q]; sn = first_steps = steps[q]; }
    }
    if (!filled && first_steps > 0) {
#pragma unroll
      for (int i = 0; i < kRing; ++i)
        load(i, first_off + min((uint32_t) i, first_steps - 1) * kWave, data, wdata, lane);
    }
    if (first_steps > 0) filled = follows;
  }

  // Adds the tile's entries to the wave's sums.
  __device__ __forceinline__ void walk(const float *tab, const uint4 *data, const float4 *wdata, int lane,
                                       float *acc) {
#pragma unroll
    for (int q = 0; q < kMaxBlocksPerWave; ++q) {
      const uint32_t n = steps[q];                    // uniform over the wave, as everything below
      float *a = acc + q * kLaneGroups;
      auto next = [&](int i) { return succ_off[q] + min((uint32_t) i, succ_last[q]) * kWave; };
      if (n >= (uint32_t) kRing) {
        uint32_t t = 0;
        for (; t + kRing <= n; t += kRing) {
#pragma unroll
          for (int i = 0; i < kRing; ++i) {
            ring[i].apply(tab, a);
            const uint32_t k = t + i + kRing;
            load(i, k < n ? offs[q] + k * kWave : next(i), data, wdata, lane);
          }
        }
#pragma unroll
        for (int i = 0; i < kRing - 1; ++i) {
          if (t + i < n) {
            ring[i].apply(tab, a);
            load(i, next(i), data, wdata, lane);
          }
        }
      } else if (n > 0) {
        // a short block: the slots it has no step for pass to its successor first
#pragma unroll
        for (int i = 1; i < kRing; ++i)
          if ((uint32_t) i >= n) load(i, next(i), data, wdata, lane);
#pragma unroll
        for (int i = 0; i < kRing - 1; ++i) {
          if ((uint32_t) i < n) {
            ring[i].apply(tab, a);
            load(i, next(i), data, wdata, lane);
          }
        }
      }
    }
  }
};

template <bool CSUM, bool WEIGHTED>
__global__ __launch_bounds__(kGatherThreads) void gather_prepared_kernel(
    int32_t V, int32_t G, int32_t nrows, GatherMap map, PreparedView p, const float *__restrict__ table,
    float *__restrict__ out, double *__restrict__ csum, double *__restrict__ runs) {
  const int32_t nchunks = p.nchunks, chunk_groups = p.chunk_groups, ntiles = p.ntiles, tile_len = p.tile_len;
  const int32_t bpc = p.blocks_per_chunk;
  const uint4 *__restrict__ data = p.data;
  const float4 *__restrict__ wdata = p.wdata;
  const uint16_t *__restrict__ perm = p.perm;
  __shared__ __attribute__((aligned(16))) float tab[kTileMax];
  int32_t r, chunk;
  if (!gather_place(map, nrows, nchunks, r, chunk)) return;   // whole workgroup leaves together, before any barrier
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t g0 = chunk * chunk_groups;
  const int32_t ng = min(chunk_groups, G - g0);
  const float *src = table + (int64_t) r * V;

  float acc[kMaxAcc];
  uint16_t where[kMaxAcc];     // group (inside the chunk) behind each running sum; loaded now,
                               // needed only when the sums are put back into group order
#pragma unroll
  for (int q = 0; q < kMaxBlocksPerWave; ++q) {
    const int bl = block_of(q, wave);
#pragma unroll
    for (int rr = 0; rr < kLaneGroups; ++rr) {
      acc[q * kLaneGroups + rr] = 0.f;
      where[q * kLaneGroups + rr] =
          bl < bpc ? perm[((size_t) chunk * bpc + bl) * kBlockGroups + rr * kWave + lane]
                   : (uint16_t) 0xFFFFu;
    }
  }

  const uint32_t *dsc = p.desc + (size_t) chunk * ntiles * bpc * 2;
  uint32_t nsteps[kMaxBlocksPerWave], noffs[kMaxBlocksPerWave];      // the next tile's blocks
  SlotStream<WEIGHTED> stream;
  load_desc(dsc, bpc, wave, stream.steps, stream.offs);

  for (int h = 0; h < ntiles; ++h) {
    const int32_t t0 = h * tile_len;
    const int32_t tl = min(tile_len, V - t0);
    if (h > 0) lds_barrier();                         // everyone is done reading the old tile
    stage_tile(tab, src + t0, tl, threadIdx.x);
    if (threadIdx.x < kBanks) tab[tile_len + threadIdx.x] = 0.f;   // the padding slots
    // The next tile's descriptors and, in the first tile, the first steps are asked for while the
    // tile is still on its way into LDS.
    load_desc(h + 1 < ntiles ? dsc + (size_t) (h + 1) * bpc * 2 : nullptr, bpc, wave, nsteps, noffs);
    stream.begin(nsteps, noffs, data, wdata, lane);
    __builtin_amdgcn_s_waitcnt(0x0f70);               // vmcnt(0): this wave's part of the tile has landed
    __syncthreads();
    stream.walk(tab, data, wdata, lane, acc);
#pragma unroll
    for (int q = 0; q < kMaxBlocksPerWave; ++q) { stream.steps[q] = nsteps[q]; stream.offs[q] = noffs[q]; }
  }

  // back into group order through LDS, then coalesced stores
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kMaxAcc; ++j)
    if (where[j] != 0xFFFFu) tab[where[j]] = acc[j];
  __syncthreads();
  if constexpr (!CSUM) {
    store_sums(out + (int64_t) r * G + g0, tab, ng);
  } else {
    // The caller draws one group by inverse CDF over max(0, sum).  It does not need the sums
    // themselves for that, only where the running total crosses its threshold: the totals of runs of
    // kRunGroups consecutive groups and the chunk's; the few sums of the run that holds the
    // crossing are formed again by the caller.
    run_totals(tab, ng, runs + ((int64_t) r * nchunks + chunk) * (chunk_groups / kRunGroups),
               csum + (int64_t) r * nchunks + chunk);
  }
}

// =============================================================================================
// small step: one workgroup runs a sequence's whole step, the statistics of its 2K + 1 rows, the
// accept scan, the table, the sums of all groups and the draws, without leaving the compute unit.
// Four launches cost about 5 us each whatever the size (the launch, a trip to memory for what the
// kernel before has written, a drain); here the parts, the probes, the table and the sums pass
// through LDS, and what is left is the chain of loads proposal -> members -> logits and group ->
// members -> logits.  Bound by latency, and by one compute unit's arithmetic in the statistics (34
// parts and 8 probes of V = 4096, K = 8: 6.5 us), which a launch of their own spreads over the chip where
// there are more than a few.  At V = 1024, K = 4: statistics and probes 4.4 us, accept scan 0.9, table 1.2, sums
// 1.6, group 1.4, token 1.3.  The whole call: V = 1024, K = 4, B = 1 10.7 us (one launch; four take 22.8);
// V = 4096, K = 8, B = 8 14.2 (two; four 23.8).  With 16 waves on four SIMDs an instruction that every wave
// repeats costs four: what is the same for all of them is computed once, ahead of the decision where it can
// be, or on the scalar unit (12.9 -> 10.7 and 17.4 -> 14.2 us).
// =============================================================================================

constexpr int kSmallTokens = 16384;    // table entries in LDS: 64 KB
constexpr int kSmallGroups = 16384;    // sums in LDS: 64 KB
constexpr int kSmallParts = 512;       // row parts (2048 logits each) of a sequence: 8 KB

constexpr int kSmallCsrWidth = 4;      // lanes per group, from the CSR

// Where the sums come from.
constexpr int kSumsPrepared = 0, kSumsPreparedWeighted = 1, kSumsCsr = 2, kSumsCsrWeighted = 3;

// Inverse CDF over max(0, sums[0 .. n)) (LDS, 16-byte aligned, n <= kSmallGroups) by a workgroup of
// 1024 threads, four neighbouring groups a thread and turn: first index whose running sum exceeds
// u * total.  All threads get the result.
__device__ CdfPick pick_group(const float *sums, int32_t n, double u) {
  constexpr int kTurns = kSmallGroups / (4 * kGatherThreads);
  static_assert(kTurns * kGatherWaves <= kWave, "one lane per total");
  __shared__ double wtot[kTurns * kGatherWaves];
  __shared__ CdfPick res;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int turns = (n + 4 * kGatherThreads - 1) / (4 * kGatherThreads);     // uniform
  double mine[kTurns], inc[kTurns];
#pragma unroll
  for (int k = 0; k < kTurns; ++k) {
    mine[k] = inc[k] = 0.0;
    if (k < turns) {
      const int32_t g = 4 * (k * kGatherThreads + tid);
      if (g < n) {
        const float4 v = *reinterpret_cast<const float4 *>(sums + g);
        mine[k] = ((double) fmaxf(v.x, 0.f) + (g + 1 < n ? (double) fmaxf(v.y, 0.f) : 0.0)) +
                  ((g + 2 < n ? (double) fmaxf(v.z, 0.f) : 0.0) + (g + 3 < n ? (double) fmaxf(v.w, 0.f) : 0.0));
      }
      inc[k] = wave_scan(mine[k]);
    }
    if (lane == kWave - 1) wtot[k * kGatherWaves + wave] = inc[k];
  }
  __syncthreads();
  // every wave finds the wave and turn that hold the crossing; rounding at the top end may leave
  // none: the last that has mass
  const double tot = lane < kTurns * kGatherWaves ? wtot[lane] : 0.0;
  const double upto = wave_scan(tot);
  const double total = read_lane(upto, kWave - 1), goal = u * total;
  const unsigned long long pos = __ballot(tot > 0.0), hit = __ballot(tot > 0.0 && upto > goal);
  if (!pos) {
    CdfPick r;
    r.index = -1; r.total = total; r.lo = r.hi = 0.0;
    return r;                                       // the same in every thread
  }
  const int at = hit ? __ffsll((long long) hit) - 1 : 63 - __clzll((long long) pos);
  if (wave == at % kGatherWaves) {                  // uniform over the wave
    const double before = read_lane(upto, at) - read_lane(tot, at);
    double my_mine = 0.0, my_inc = 0.0;
#pragma unroll
    for (int k = 0; k < kTurns; ++k)
      if (k == at / kGatherWaves) { my_mine = mine[k]; my_inc = inc[k]; }
    const unsigned long long has = __ballot(my_mine > 0.0);
    const unsigned long long over = hit ? __ballot(my_mine > 0.0 && before + my_inc > goal) : 0;
    const int l = over ? __ffsll((long long) over) - 1 : 63 - __clzll((long long) has);
    if (lane == l) {                                // walks its four groups
      const int32_t g0 = 4 * (at / kGatherWaves * kGatherThreads + tid);
      double cum = before + (my_inc - my_mine), last_v = 0.0;
      int32_t pick = -1;
      bool done = false;
      for (int j = 0; j < 4; ++j) {
        const double v = g0 + j < n ? (double) fmaxf(sums[g0 + j], 0.f) : 0.0;
        if (!done && v > 0.0) {
          pick = g0 + j;
          last_v = v;
          cum += v;
          done = cum > goal;
        }
      }
      res.index = pick;
      res.total = total;
      res.hi = hit ? cum : total;
      res.lo = res.hi - last_v;
    }
  }
  __syncthreads();
  return res;
}

// STATS: the row parts and probes are formed here; otherwise row_stats has left them in memory.
template <bool BF16, int SUMS, bool STATS>
__global__ __launch_bounds__(kAcceptThreads) void small_step_kernel(AcceptArgs a, FinalizeArgs fa, ProbeArgs pa,
                                                                    PreparedView p, int32_t nnz, int32_t long_size) {
  static_assert(kAcceptThreads == kGatherThreads, "one workgroup plays both parts");
  __shared__ AcceptShared sh;
  __shared__ StatPart parts[STATS ? kSmallParts : 1];
  __shared__ __attribute__((aligned(16))) float tab[kSmallTokens + kBanks];
  __shared__ __attribute__((aligned(16))) float sums[kSmallGroups];
  constexpr bool kWeighted = SUMS == kSumsPreparedWeighted || SUMS == kSumsCsrWeighted;
  const int b = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowSet &rs = a.rs;
  const int32_t V = a.V, G = a.G, K = a.K;

  // the first multiplicities do not depend on any row
  const int32_t first = threadIdx.x * kTokensPerThread;
  float m[8];
  auto load_m = [&]() {
    if (first < V) load8_mult<true>(kWeighted ? nullptr : a.mult, slice_start<true>(first, V), V, m);
  };
  const bool whole_rows = a.nparts == 1;              // a part is a row: nothing to merge
  if constexpr (STATS) {
    // Row parts, dealt to the waves in turn, and probes, one each for the first waves.  Everything starts
    // with a trip to memory, so a wave asks for its first two parts before anything else and keeps two
    // on their way: they come in behind the probes' chains of loads.  (Handed out one by one to
    // whichever wave was free, a part at a time ahead, 34 parts and 8 probes took 7.4 us instead of 6.5, of which
    // their arithmetic on one compute unit is 5.6.)
    const int32_t nparts_all = (2 * K + 1) * a.nparts;
    RowPart<BF16, true, false> raw[2];    // cached: the decision rows are read again
    auto ask = [&](RowPart<BF16, true, false> &to, int32_t it) {
      const int32_t r = whole_rows ? it : it / a.nparts, part = whole_rows ? 0 : it % a.nparts;
      to.load(r <= K ? target_row(rs, b, r, BF16) : draft_row(rs, b, r - K - 1, BF16), part * kPartElems, V, lane);
    };
    if (wave < nparts_all) ask(raw[0], wave);
    if (wave + kGatherWaves < nparts_all) ask(raw[1], wave + kGatherWaves);
    load_m();
    if (wave == kGatherWaves - 1) accept_fetch(sh, a, b, lane);
    for (int32_t i = wave; i < K; i += kGatherWaves) probe_row<BF16, false>(rs, pa, b, i, a.c, lane, sh.probe + i);
    auto reduce = [&](RowPart<BF16, true, false> &from, int32_t it) {
      float x[32];
      from.get(x, whole_rows ? 0 : (it % a.nparts) * kPartElems, V, lane);
      if (it + 2 * kGatherWaves < nparts_all) ask(from, it + 2 * kGatherWaves);
      const StatPart sp = part_stats(x, a.c);
      if (lane == kWave - 1) parts[it] = sp;
    };
    for (int32_t it = wave; it < nparts_all; it += 2 * kGatherWaves) {
      reduce(raw[0], it);
      if (it + kGatherWaves < nparts_all) reduce(raw[1], it + kGatherWaves);
    }
    wave_handoff();                                   // parts, from the lane that has a sum to the lane of its row
    const int32_t r = wave + kGatherWaves * lane;     // the wave's own rows, one per lane
    if (whole_rows && r < nparts_all) {
      const RowStat s = one_part(parts[r], a.c);
      const double iz = 1.0 / s.Z;
      if (r <= K) { sh.st_t[r] = s; sh.iz_t[r] = iz; } else { sh.st_d[r - K - 1] = s; sh.iz_d[r - K - 1] = iz; }
    }
  } else {
    accept_merge_stored(sh, a, b, true);
    load_m();
    if (wave == kGatherWaves - 1) accept_fetch(sh, a, b, lane);
  }
  SlotStream<kWeighted> stream;
  if constexpr (SUMS <= kSumsPreparedWeighted) load_desc(p.desc, p.blocks_per_chunk, wave, stream.steps, stream.offs);
  // the first chunk's slots and the places of its sums: on their way through the accept scan
  uint32_t nsteps[kMaxBlocksPerWave], noffs[kMaxBlocksPerWave];
  uint16_t where[kMaxAcc];
  auto ask_chunk = [&](int32_t chunk) {
    load_desc(chunk + 1 < p.nchunks ? p.desc + (size_t) (chunk + 1) * p.blocks_per_chunk * 2 : nullptr,
              p.blocks_per_chunk, wave, nsteps, noffs);
    stream.begin(nsteps, noffs, p.data, p.wdata, lane);
#pragma unroll
    for (int j = 0; j < kMaxAcc; ++j) {
      const int bl = block_of(j / kLaneGroups, wave);
      where[j] = bl < p.blocks_per_chunk
                     ? p.perm[((size_t) chunk * p.blocks_per_chunk + bl) * kBlockGroups + (j % kLaneGroups) * kWave + lane]
                     : (uint16_t) 0xFFFFu;
    }
  };
  CsrGroups<SUMS == kSumsCsrWeighted> groups;
  if constexpr (SUMS <= kSumsPreparedWeighted) ask_chunk(0);
  else csr_start<kSmallCsrWidth>(groups, 0, G, a.row_ptr, a.members, nnz, a.weights);
  lds_barrier();
  if constexpr (STATS) {
    if (!whole_rows) {
      accept_merge(sh, a, b, true, nullptr, parts, parts + (K + 1) * a.nparts);
      lds_barrier();
    }
  }
  accept_decide(sh, a, b, true);

  // the table on the decision row, straight into LDS
  const int32_t istar = __builtin_amdgcn_readfirstlane(sh.istar);
  const bool rejected = istar < K;
  const void *trow = target_row(rs, b, istar, BF16);
  const void *drow = draft_row(rs, b, rejected ? istar : 0, BF16);
  const RowStat st = sh.st_t[istar];
  const RowStat sd = sh.st_d[rejected ? istar : 0];
  const double izt = sh.iz_t[istar], izd = rejected ? sh.iz_d[istar] : 0.0;
  for (int32_t at = first; at < V; at += kAcceptTokens) {
    const int32_t t = slice_start<true>(at, V);
    float xt[8], xd[8], v[8];
    load8<BF16, true>(trow, t, V, xt);
    if (rejected) load8<BF16, true>(drow, t, V, xd);
    if (at != first) load8_mult<true>(kWeighted ? nullptr : a.mult, t, V, m);
    delta8(xt, xd, m, rejected, st, sd, izt, izd, a.c, fa.c_lo, v);
    if ((t & 3) == 0) {
      *reinterpret_cast<float4 *>(tab + t) = make_float4(v[0], v[1], v[2], v[3]);
      *reinterpret_cast<float4 *>(tab + t + 4) = make_float4(v[4], v[5], v[6], v[7]);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) tab[t + k] = v[k];
    }
  }

  // the sums of all groups
  if constexpr (SUMS <= kSumsPreparedWeighted) {
    if (threadIdx.x < kBanks) tab[p.tile_len + threadIdx.x] = 0.f;
    lds_barrier();                                  // the table is complete
    for (int32_t chunk = 0; chunk < p.nchunks; ++chunk) {
      float acc[kMaxAcc];
#pragma unroll
      for (int j = 0; j < kMaxAcc; ++j) acc[j] = 0.f;
      if (chunk > 0) {
#pragma unroll
        for (int q = 0; q < kMaxBlocksPerWave; ++q) { stream.steps[q] = nsteps[q]; stream.offs[q] = noffs[q]; }
        ask_chunk(chunk);
      }
      stream.walk(tab, p.data, p.wdata, lane, acc);
#pragma unroll
      for (int j = 0; j < kMaxAcc; ++j)
        if (where[j] != 0xFFFFu) sums[chunk * p.chunk_groups + where[j]] = acc[j];
    }
  } else {
    __shared__ bool has_long;
    if (threadIdx.x == 0) { tab[V] = 0.f; has_long = false; }
    lds_barrier();
    csr_sums<kSmallCsrWidth, kWeighted, true>(groups, tab, V, 0, V, 0, G, a.row_ptr, a.members, nnz, a.weights, long_size, &has_long,
                           [&](int32_t g, float s) { sums[g] = s; });
    lds_barrier();
    if (has_long)                                   // uniform
      csr_long_sums<kSmallCsrWidth, kWeighted, true>(tab, V, 0, V, 0, G, a.row_ptr, a.members, nnz, a.weights, long_size,
                                  [&](int32_t g, float s) { sums[g] += s; });
  }
  lds_barrier();

  Uniforms u;
  u.acc = 0.f;
  u.grp = sh.ugrp[istar];
  u.tok = sh.utok[istar];
  const CdfPick pg = pick_group(sums, G, (double) u.grp);
  finish_sequence<BF16, kAcceptThreads>(fa, G, b, istar, trow, st, u, pg);
}

// =============================================================================================
// Launchers.
// =============================================================================================

int32_t even_size(const pcg_groups &g) { return g.nnz % g.G == 0 ? (int32_t) (g.nnz / g.G) : 0; }

int32_t stats_nparts(int32_t V) { return (V + kPartElems - 1) / kPartElems; }

hipError_t launch_row_stats(const RowSet &rs, bool bf16, int32_t V, int64_t nrows, float c,
                            bool streaming, StatPart *parts, hipStream_t stream,
                            const ProbeArgs *probes) {
  const int32_t nparts = stats_nparts(V);
  if (nrows == 0) return hipSuccess;
  ProbeArgs pa{};
  if (probes) pa = *probes;
  // With probes, the grid starts with a few rows of workgroups that form them, one target row per
  // wave; the rows of logits follow (the first grid plane holds fewer of them by that much).
  const unsigned gx = (unsigned) ((nparts + kStatsWaves - 1) / kStatsWaves);
  const int64_t probe_y =
      probes ? (rs.nrows0 + (int64_t) gx * kStatsWaves - 1) / ((int64_t) gx * kStatsWaves) : 0;
  const int64_t slots = nrows + probe_y;                    // values of (z, y) the grid must hold
  const unsigned gz = (unsigned) ((slots + kRowsPerGridY - 1) / kRowsPerGridY);
  const dim3 grid(gx, (unsigned) std::min<int64_t>(slots, kRowsPerGridY), gz), block(kStatsWaves * kWave);
  const bool wide = V >= (bf16 ? kPer16<true> : kPer16<false>);
  auto launch = [&](auto kernel) {
    kernel<<<grid, block, 0, stream>>>(rs, V, nparts, nrows, c, parts, pa, probe_y);
  };
  if (bf16) {
    if (!wide) launch(row_stats_kernel<true, false, false>);
    else if (streaming) launch(row_stats_kernel<true, true, true>);
    else launch(row_stats_kernel<true, true, false>);
  } else {
    if (!wide) launch(row_stats_kernel<false, false, false>);
    else if (streaming) launch(row_stats_kernel<false, true, true>);
    else launch(row_stats_kernel<false, true, false>);
  }
  return hipGetLastError();
}

// Workgroups per sequence in the accept + delta kernel: enough to give every compute unit one,
// never more than there are slices of the table.
int32_t accept_nsplit(int32_t V, int32_t B) {
  const int32_t slices = (V + kAcceptTokens - 1) / kAcceptTokens;
  return std::max(1, std::min(slices, (256 + B - 1) / B));
}

hipError_t launch_accept_delta(const AcceptArgs &a, bool bf16, int32_t B, float c_lo, float *table,
                               hipStream_t stream) {
  const int32_t nsplit = accept_nsplit(a.V, B);
  const dim3 grid((unsigned) ((int64_t) B * nsplit));
  const bool vec = a.V >= 8;
#define PCG_LAUNCH_AD(BF, VE) \
  accept_delta_kernel<BF, VE><<<grid, kAcceptThreads, 0, stream>>>(a, nsplit, c_lo, table)
  if (bf16) { if (vec) PCG_LAUNCH_AD(true, true); else PCG_LAUNCH_AD(true, false); }
  else { if (vec) PCG_LAUNCH_AD(false, true); else PCG_LAUNCH_AD(false, false); }
#undef PCG_LAUNCH_AD
  return hipGetLastError();
}

hipError_t launch_accept_thin(const AcceptArgs &a, bool bf16, int32_t B, const int32_t *tok_ptr,
                              const int32_t *tok_groups, const float *tok_weights, int32_t *trials,
                              int32_t max_trials, hipStream_t stream) {
  auto launch = [&](auto kernel) {
    kernel<<<B, kAcceptThreads, 0, stream>>>(a, tok_ptr, tok_groups, tok_weights, trials, max_trials);
  };
  if (bf16) launch(accept_thin_kernel<true>); else launch(accept_thin_kernel<false>);
  return hipGetLastError();
}

int32_t thin_max_parts() { return kMaxThinParts; }

bool propose_in_rows(int32_t V) { return stats_nparts(V) <= kProposeParts; }

hipError_t launch_propose(const RowSet &rs, bool bf16, int32_t V, int32_t K, int32_t pos0, float c,
                          const StatPart *parts, const int32_t *tok_ptr, const int32_t *tok_groups,
                          const float *tok_weights, uint64_t seed, uint64_t offset,
                          int32_t *prop_tokens, int32_t *prop_groups, pcg_diag *diag,
                          hipStream_t stream) {
  const int32_t nparts = stats_nparts(V);
  const unsigned grid = (unsigned) rs.nrows0;
  if (!parts) {
    auto launch = [&](auto kernel) {
      kernel<<<grid, kProposeThreads, 0, stream>>>(rs, V, K, pos0, nparts, c, tok_ptr, tok_groups, tok_weights,
                                                   seed, offset, prop_tokens, prop_groups, diag);
    };
    if (bf16) { if (V >= kPer16<true>) launch(propose_row_kernel<true, true>); else launch(propose_row_kernel<true, false>); }
    else { if (V >= kPer16<false>) launch(propose_row_kernel<false, true>); else launch(propose_row_kernel<false, false>); }
    return hipGetLastError();
  }
  auto launch = [&](auto kernel) {
    kernel<<<grid, kWave, 0, stream>>>(rs, V, K, pos0, nparts, c, parts, tok_ptr, tok_groups, tok_weights,
                                       seed, offset, prop_tokens, prop_groups, diag);
  };
  if (bf16) launch(propose_kernel<true>); else launch(propose_kernel<false>);
  return hipGetLastError();
}

hipError_t launch_weights_parts(const RowSet &rs, bool bf16, int32_t V, int32_t nrows, float c, float c_lo, StatPart *parts,
                                hipStream_t stream) {
  const int32_t nparts = stats_nparts(V);
  const dim3 grid((unsigned) ((nparts + kStatsWaves - 1) / kStatsWaves), (unsigned) nrows);
  auto launch = [&](auto kernel) { kernel<<<grid, kStatsWaves * kWave, 0, stream>>>(rs, V, nparts, c, c_lo, parts); };
  if (bf16) launch(weights_parts_kernel<true>); else launch(weights_parts_kernel<false>);
  return hipGetLastError();
}

hipError_t launch_weights(const RowSet &rs, bool bf16, const pcg_groups &g, int32_t nrows, float c, float c_lo, double cd,
                          const StatPart *parts, float *table, hipStream_t stream) {
  const int32_t nparts = stats_nparts(g.V);
  // with general weights the table is the plain probability: the gather applies the weights
  const int32_t *mult = g.weights ? nullptr : g.mult;
  auto launch = [&](auto kernel) {
    kernel<<<dim3((unsigned) nparts, (unsigned) nrows), kTableThreads, 0, stream>>>(rs, g.V, nparts, c, c_lo, cd, parts, mult, table);
  };
  if (bf16) { if (mult) launch(weights_kernel<true, true>); else launch(weights_kernel<true, false>); }
  else { if (mult) launch(weights_kernel<false, true>); else launch(weights_kernel<false, false>); }
  return hipGetLastError();
}

// One compute unit a row, and a launch less, or the row's parts spread over the chip twice.  The call by
// weights_parts and weights, and by rows, in us (V, members, rows; bf16 unless stated):
//   up to 8 parts:   1000, 8, 18: 11.9 and 10.1;  4096, 8, 32: 12.5 and 11.2, 1152: 45.4 and 37.9;  12 000, 8, 2: 12.9 and
//                    10.5;  16 384, 8, 128: 19.7 and 16.4, 1152: 89.0 and 79.0
//   up to 16 parts:  32 768, 32, 2: 12.8 and 13.8, 16: 15.8 and 16.9, fp32 8: 14.7 and 16.3;  30 000, 32, 64: 24.7 and 22.8,
//                    128: 33.8 and 31.9;  32 768, 32, 128, fp32: 35.6 and 32.7
//   beyond:          40 000, 32, 64: 28.3 and 31.3, 96: 41.8 and 44.1, 128: 50.2 and 50.2;  65 536, 32, 64: 37.9 and 41.5, 96:
//                    59.4 and 59.7, 128: 65.4 and 64.4;  fp32, 96: 57.2 and 57.7 at 50 000
bool weights_by_rows(int32_t V, int32_t nrows) {
  const int32_t nparts = stats_nparts(V);
  return nparts <= kRowTableParts && nrows >= (nparts <= 8 ? 1 : nparts <= 16 ? 64 : 128);
}

hipError_t launch_row_weights(const RowSet &rs, bool bf16, const pcg_groups &g, int32_t nrows, float c, float c_lo, double cd,
                              float *table, hipStream_t stream) {
  const int32_t nparts = stats_nparts(g.V);
  const int32_t *mult = g.weights ? nullptr : g.mult;
  auto launch = [&](auto kernel, int np) {
    const unsigned waves = (unsigned) ((nparts + np - 1) / np);
    kernel<<<(unsigned) nrows, waves * kWave, 0, stream>>>(rs, g.V, nparts, c, c_lo, cd, mult, table);
  };
  if (g.V < 4) { if (bf16) launch(row_weights_kernel<true, false, 1>, 1); else launch(row_weights_kernel<false, false, 1>, 1); }
  else if (nparts * 2 <= kRowTableParts) { if (bf16) launch(row_weights_kernel<true, true, 1>, 1); else launch(row_weights_kernel<false, true, 1>, 1); }
  else { if (bf16) launch(row_weights_kernel<true, true, 2>, 2); else launch(row_weights_kernel<false, true, 2>, 2); }
  return hipGetLastError();
}

// The most chunks of nrows rows that all run at once, on the 32 compute units of each XCD, by some split of rows
// and chunks over the XCDs (as many as there are compute units in all, rounded up, left the last few for
// a second turn: the call at V = 20 000, 32 members, 12 rows 30.8 us, now 24.8; 24 rows with weights 41.7, now 31.5).
static int64_t csr_chunks_at_once(int64_t nrows) {
  int64_t most = 1;
  for (int64_t rp = 8; rp >= 1; rp /= 2) most = std::max(most, 8 / rp * (32 / ((nrows + rp - 1) / rp)));
  return most;
}

CsrShape csr_shape(int32_t V, int32_t G, int64_t nnz, int64_t nrows, int64_t max_chunks) {
  CsrShape p;
  // Lanes per group: enough for a group of mean size in one trip of four entries a lane, 2 to 16
  // (fewer lanes leave long groups to one lane's loop, more leave lanes idle).
  const double mean = (double) nnz / (double) G;
  p.width = 2;
  while (p.width < 16 && 4 * p.width < mean) p.width *= 2;
  // More lanes for long groups only where G times an XCD's rows is one pass of its 32 compute units: there they were
  // never behind.  Calls with 16 lanes and with 32 (V, members, rows): 4096, 100, 1: 21.1 and 19.8;  2048, 1 to 128 with weights,
  // 2: 19.1 and 17.9;  4096, 40, 1: 18.4 and 18.4.  Beyond, gains (20 000, 100, 1: 24.7 and 24.1;  8192, 100, 1: 24.5 and 23.1) and
  // losses (16 384, 40, 16: 27.9 and 33.2;  30 000, 40 with weights, 4: 25.3 and 28.8;  65 536, 140, 2: 57.4 and 64.3) mix: of 640
  // shapes 148 gain more than 2 %, 382 lose as much.
  const int64_t rows_per_xcd = (nrows + 7) / 8;
  if (mean > 32 && (int64_t) G * rows_per_xcd <= 32 * 4 * (kGatherThreads / 32)) p.width = 32;
  // Chunks per row: a workgroup for every compute unit, each with at least one pass of groups, at most
  // kMaxChunkGroups and, where that allows it, at most max_chunks.
  const int64_t pass = 4 * (kGatherThreads / p.width);
  auto cut = [&](int64_t want) {
    CsrShape c = p;
    int64_t nchunks = std::min<int64_t>({want, max_chunks, (G + pass - 1) / pass});
    nchunks = std::max<int64_t>(nchunks, ((int64_t) G + kMaxChunkGroups - 1) / kMaxChunkGroups);
    int64_t gpc = (G + nchunks - 1) / nchunks;
    gpc = (gpc + kRunGroups - 1) / kRunGroups * kRunGroups;
    c.chunk_groups = (int32_t) gpc;
    c.nchunks = (int32_t) ((G + gpc - 1) / gpc);
    // LDS: the chunk's sums, then as much of the table row as fits (a tile and its zero slot)
    const int32_t room = (kTileMax - c.chunk_groups - 64) / 64 * 64;
    c.ntiles = (V + room - 1) / room;
    c.tile_len = std::min(room, ((V + c.ntiles - 1) / c.ntiles + 63) / 64 * 64);
    return c;
  };
  // As many chunks as all run at once, or a few more of them, the last in a second turn, where those leave room for a larger
  // tile: every tile walks all entries of a chunk.  A workgroup's walks, and in us (V, members, rows; at once and more):
  //   two tiles and one:    30 592, 68, 70: 2 x G / 3 and 2 turns of G / 4: 249 and 164;  33 720, 133, 55: 2 x G / 4 and 2 of G / 5:
  //                         323 and 248;  31 736, 1 to 128, 84: 2 x G / 2 and 2 of G / 4: 361 and 163;  29 706, 4, 127: 47.5 and 35.7
  //   three tiles and two:  57 588, 1 to 128, 49: 3 x G / 4 and 2 x 2 of G / 6: 523 and 475;  48 918, 64, 75: 3 x G / 3 and 2 x 2 of G / 4: 382
  //                         and 382;  60 411, 32, 44: 3 x G / 5 and 2 x 2 of G / 6: 160 and 178
  const int64_t at_once = csr_chunks_at_once(nrows);
  auto walks = [&](const CsrShape &c) { return (int64_t) c.ntiles * c.chunk_groups * (c.nchunks > at_once ? 2 : 1); };
  const CsrShape one = cut(at_once), two = cut((256 + nrows - 1) / nrows);
  return two.ntiles < one.ntiles && walks(two) < walks(one) ? two : one;
}

CsrShape step_csr_shape(const pcg_groups &g, int32_t B, int32_t K) {
  return csr_shape(g.V, g.G, g.nnz, B, std::max(csum_room(g.G), csum_room_in_parts(g.V, K)));
}

// How the XCDs share rows and chunks.  All chunks of a row on one XCD, unless another split saves each of them half a MiB
// to bring in, a whole one from the CSR (the rows, which everything waits for, counted four times, twice beside a prepared stream
// with weights), and, where not all workgroups run at once, from the prepared layout leaves no more of them to the last turn.  Whole
// calls, or the gather alone, in us, all on one and split (V, members, rows):
//   prepared:  65 536, 32, 8: call 34.0 and 32.8;  16: 37.1 and 35.7;  weights, 16: 47.5 and 40.8, 64: 88.3 and 87.3 (gather 46.8 and
//              44.9);  64 (no saving): gather 25.4 and 27.0;  32 768, 1 to 128, 128 (none): 47.6 and 51.9;  59 549, 64, 18: 31.8 and 33.6
//              (over two XCDs 32.3)
//   turns:     50 945, 1 to 128 with weights, 49 (3 in a second turn, or 18): 121 and 151;  50 464, 94, 33 (3 or 7): 65.0 and 76.5;
//              35 648, 117, 54 (18 or 34): 69.2 and 79.4;  51 092, 128, 19 (21 or 9): 50.5 and 43.0;  65 507, 1 to 64, 17 (16 either way):
//              64.4 and 53.6
//   CSR:       65 536, 32, 1: call 54.7 and 25.6;  30 000, 100, 8: 48.5 and 37.8;  16 384, 32, 32 (0.5 MiB): gather 12.6 and
//              12.2, but finalize, which finds a row's totals in its own XCD's L2 if they were formed there, 6.2 and 6.5;  rows 14 987, 1 to 15 with weights, 1 (0.8): 12.3 and 13.1;
//              turns: 28 456, 111 with weights, 86 (6 in a second turn, or 44): 300 and 288;  32 524, 72 with weights, 56 (24 or 40): 192 and 187
GatherMap gather_map(int32_t nrows, int32_t nchunks, int64_t row_bytes, int64_t chunk_bytes, bool csr, bool weights) {
  const int64_t row_cost = !csr && weights ? 2 : 4, saving = (int64_t) 1 << (csr ? 20 : 19);
  struct Split { int64_t turns, late, bytes; } best{}, one{};
  GatherMap map{3, nchunks};
  for (int32_t shift = 3; shift >= 0; --shift) {
    const int32_t rp = 1 << shift, cp = 8 / rp, rows = (nrows + rp - 1) / rp, chunks = (nchunks + cp - 1) / cp;
    Split s;
    s.turns = ((int64_t) rows * chunks + 31) / 32;         // of an XCD's compute units
    s.late = 0;                                            // workgroups in the last of several
    for (int32_t x = 0; x < 8 && s.turns > 1 && !csr; ++x) {
      const int64_t mine = (int64_t) ((nrows - (x & (rp - 1)) + rp - 1) / rp) * ((nchunks - (x >> shift) + cp - 1) / cp);
      s.late += std::max<int64_t>(0, mine - 32 * (s.turns - 1));
    }
    s.bytes = row_cost * rows * row_bytes + chunks * chunk_bytes + (rp < 8 ? saving : 0);
    if (shift == 3) { best = one = s; continue; }
    if (s.turns > one.turns || (s.turns == one.turns && s.late > one.late)) continue;
    if (s.turns < best.turns || (s.turns == best.turns && s.bytes < best.bytes)) {
      best = s;
      map = GatherMap{shift, chunks};
    }
  }
  return map;
}
static unsigned gather_grid(const GatherMap &m, int32_t nrows) {
  return 8u * (((unsigned) nrows + (1u << m.row_shift) - 1) >> m.row_shift) * (unsigned) m.chunks_each;
}

// Few rows leave most of the chip to chunks of at least 4096 groups, and those who have one wait for their slots from
// memory; from the CSR a row is cut as fine as there are compute units.  Whole calls, prepared and CSR, in us
// (V, members, sequences of pcg_verify or rows of pcg_group_probs; turns: of the CSR's workgroups):
//   one tile, one turn:   verify 12 000, 8, 3: 21.6 and 20.9;  20 000, 32, 1: 23.4 and 21.3;  100, 1: 31.8 and 26.2;  40 000, 32, 2: 25.0
//                         and 22.7;  rows 4100, 4, 1: 10.3 and 9.8, 16, 36: 12.3 and 11.0, 100, 5: 26.8 and 11.6;  14 000, 13, 9: 12.4 and 10.7
//   two:                  with 8 lanes a group and one size, verify 20 011, 20, 12: 25.1 and 24.5, rows 8192, 24, 18: 13.0 and 12.4;
//                         with 16, verify 12 000, 100, 8: 32.4 and 28.7, 30 000, 1 to 128, 3: 29.7 and 29.0;  but rows 10 000, 10, 48:
//                         11.9 and 12.8;  verify 20 000, 8, 32: 26.5 and 27.5;  1 to 40, 5: 26.1 and 27.0
//   three:                verify 14 000, 33, 9: 25.2 and 25.8, 64: 28.7 and 27.0 at 30 000, 5;  7000, 1 to 200, 18: 35.6 and 37.3
//   weights, 8 lanes:     a turn takes as long for 17 members as for 32.  Two turns: rows 17 000, 20, 9: 15.0 and 14.3, 1 to 50, 36: 14.1
//                         and 15.0 at 4500, up to 32 members, half of them 32: 13.9 and 12.3;  three: rows 7000, 18, 48: 12.9 and
//                         14.2, 5000, 28, 64: 14.4 and 14.0, 20 to 40, verify 14 000, 18: 29.1 and 32.2;  four: rows 7000, 20, 64: 13.2
//                         and 15.6, 28: 14.6 and 15.6, verify 20 011, 32, 24: 34.1 and 32.1
//   weights, 16 lanes:    four: rows 20 011, 33, 12: 19.2 and 19.0, verify 17 000, 1 to 128, 12: 41.7 and 39.7;  five: verify 26 000, 56, 9: 37.2
//                         and 33.7, but rows 14 000, 33, 18: 16.7 and 18.7, 4100, 1 to 128, 64: 21.9 and 24.3
//   two tiles, one turn:  verify 65 536, 32, 1: 27.1 and 25.7;  24, 2: 26.8 and 26.3;  up to 32 members, half of them 32: 25.7 and 24.5 at
//                         45 000, but 1 to 40: 27.4 and 29.1;  140, 1: 41.9 and 45.0 at 50 000;  12, 2: rows 17.1 and 17.8
static int32_t csr_turns(const CsrShape &p) {
  const int32_t turn = kCsrInFlight * (kGatherThreads / p.width);
  return (p.chunk_groups + turn - 1) / turn;
}
bool csr_is_faster(const pcg_groups &g, const CsrShape &p) {
  const int32_t turns = csr_turns(p);
  if (g.G <= kScanGroups) return false;                // one chunk, whose totals finalize reads at once
  if (p.ntiles == 2) return p.width == 8 && !g.weights && turns == 1;
  const bool even = even_size(g) > 0;
  const double mean = (double) g.nnz / (double) g.G;
  int32_t most = 1;
  if (p.width >= 16) most = !g.weights ? 2 : even && mean > 44 ? 5 : 4;
  else if (p.width == 8 && g.weights) most = !even ? 2 : mean > 28 ? 4 : mean > 24 ? 3 : 2;
  else if (p.width == 8 && even) most = 2;
  return p.ntiles == 1 && turns <= most;
}

hipError_t launch_gather(const pcg_groups &g, const CsrShape &p, int32_t nrows, const float *table, float *out,
                         double *csum, int64_t csum_stride, double *runs, hipStream_t stream) {
  if (nrows == 0) return hipSuccess;
  const GatherMap map = gather_map(nrows, p.nchunks, (int64_t) g.V * 4, g.nnz * (g.weights ? 8 : 4) / p.nchunks, true, g.weights);
  const dim3 grid(gather_grid(map, nrows));
  auto launch = [&](auto kernel) {
    kernel<<<grid, kGatherThreads, 0, stream>>>(g.V, g.G, nrows, map, p.nchunks, p.chunk_groups, p.ntiles, p.tile_len,
                                                (int32_t) g.nnz, csr_long_size(g.nnz, g.G, p.width), g.row_ptr,
                                                g.members, g.weights, table, out, csum, csum_stride, runs);
  };
  auto pick = [&](auto width) {
    constexpr int W = decltype(width)::value;
    auto form = [&](auto whole) {
      constexpr bool O = decltype(whole)::value;
      if (g.weights) { if (csum) launch(gather_kernel<W, true, true, O>); else launch(gather_kernel<W, false, true, O>); }
      else { if (csum) launch(gather_kernel<W, true, false, O>); else launch(gather_kernel<W, false, false, O>); }
    };
    if (p.ntiles == 1) form(std::true_type{}); else form(std::false_type{});
  };
  switch (p.width) {
    case 2: pick(std::integral_constant<int, 2>{}); break;
    case 4: pick(std::integral_constant<int, 4>{}); break;
    case 8: pick(std::integral_constant<int, 8>{}); break;
    case 16: pick(std::integral_constant<int, 16>{}); break;
    default: pick(std::integral_constant<int, 32>{}); break;
  }
  return hipGetLastError();
}

// Bytes of slots (and weights) that a gather over the prepared layout reads for a row.
static int64_t prepared_slot_bytes(const pcg_groups &g) {
  const pcg_prepared &p = *g.prepared_info;
  const int64_t slots = (p.off_weights ? p.off_weights : p.bytes) - p.off_data;
  return g.weights ? 3 * slots : slots;
}

static PreparedView prepared_view(const pcg_groups &g) {
  const pcg_prepared &p = *g.prepared_info;
  const char *blob = reinterpret_cast<const char *>(g.prepared);
  PreparedView v;
  v.desc = reinterpret_cast<const uint32_t *>(blob + p.off_desc);
  v.perm = reinterpret_cast<const uint16_t *>(blob + p.off_perm);
  v.data = reinterpret_cast<const uint4 *>(blob + p.off_data);
  // general weights are read from the blob (the caller's checks made sure it holds them)
  v.wdata = g.weights ? reinterpret_cast<const float4 *>(blob + p.off_weights) : nullptr;
  v.nchunks = p.nchunks;
  v.chunk_groups = p.chunk_groups;
  v.ntiles = p.ntiles;
  v.tile_len = p.tile_len;
  v.blocks_per_chunk = p.blocks_per_chunk;
  return v;
}

hipError_t launch_gather_prepared(const pcg_groups &g, int32_t nrows, const float *table, float *out,
                                  double *csum, double *runs, hipStream_t stream) {
  if (nrows == 0) return hipSuccess;
  const PreparedView p = prepared_view(g);
  const GatherMap map = gather_map(nrows, p.nchunks, (int64_t) g.V * 4, prepared_slot_bytes(g) / p.nchunks, false, g.weights);
  const dim3 grid(gather_grid(map, nrows));
  auto launch = [&](auto kernel) {
    kernel<<<grid, kGatherThreads, 0, stream>>>(g.V, g.G, nrows, map, p, table, out, csum, runs);
  };
  if (g.weights) {
    if (csum) launch(gather_prepared_kernel<true, true>);
    else launch(gather_prepared_kernel<false, true>);
  } else {
    if (csum) launch(gather_prepared_kernel<true, false>);
    else launch(gather_prepared_kernel<false, false>);
  }
  return hipGetLastError();
}

StepShape step_shape(const pcg_groups &g, int32_t B, int32_t K) {
  // what the small step's LDS and its row loads can take
  const int64_t row_parts = (2 * (int64_t) K + 1) * stats_nparts(g.V);
  if (g.V < 8 || g.V > kSmallTokens || g.G > kSmallGroups || B > 256) return StepShape::kFour;
  if (g.prepared && (g.prepared_info->ntiles != 1 || g.prepared_info->tile_len > kSmallTokens))
    return StepShape::kFour;
  // The statistics by the same workgroup, if that is at most two items a wave (V = 1024, K = 4: 13.0
  // against 13.7 us; V = 4096, K = 8: 19.0 against 16.7) or there is a sequence for every compute unit
  // (B = 256: V = 4096 22.1 against 25.3, 16 384 52.8 against 56.3).
  const bool one = row_parts <= kSmallParts && (K + row_parts <= 2 * kGatherWaves || B > 128);
  const StepShape small = one ? StepShape::kOne : StepShape::kTwo;
  // One compute unit per sequence for all that follows the statistics, or four kernels that spread a
  // sequence over the chip but pay for three more boundaries.  Whole calls in us, four launches and this,
  // bf16, K = 8 unless stated (V, members, B).
  // From 129 sequences on not even two workgroups each of the four kernels run at once, and this wins at
  // any size: 16 384, 32, 130, K = 3: 55 and 37, from the CSR 8192, 4, 130, K = 3: 33 and 27, 16 384, 40, 130, K = 3:
  // 157 and 90, 16 384, 4, 160: 60 and 57, 16 384, 128 with weights, 224: 316 and 295.
  if (B > 128) return small;
  if (g.prepared) {
    // What counts here is the table (tokens) and the slots, padding and all, that one unit reads, three times as many
    // bytes each with weights: the load.
    // With one chunk of groups a sequence's gather from the prepared layout is one workgroup in any case, and this wins
    // over that throughout: 8192, 64, 64: 36.1 and 27.2, 16 384, 100, 64: 64.9 and 56.3, with weights 126.5 and 116.8.  But few
    // sequences are gathered from the CSR by four launches (csr_is_faster), which takes longer by its turns:
    //   one turn:   load 144: 16 384, 4, 1: 19.8 and 18.3;  160: 16 384, 8, 1: 19.9 and 19.7;  172: 16 000, 6 with weights, 1: 21.5
    //               and 19.3;  187: 12 000, 32, 1: 20.2 and 23.2;  192: 8192, 64, 8: 22.1 and 24.6, 16 384, 16, 1: 20.0 and 22.2,
    //               16 384, 8 with weights, 1: 19.8 and 20.4;  528: 16 384, 100, 1: 23.6 and 48.1, with weights (928) 25.4 and 126.6
    //   more:       three, load 142: 6000, 32 with weights, 64: 27.0 and 24.6;  four, 236: 4500, 1 to 128 with weights, 48: 36.6 and
    //               31.8;  two, 281: 12 000, 64, 8: 24.5 and 30.6
    // Several chunks are walked one after the other here, and side by side there.
    //   B < 128:  load 128: 8192, 32, 1: 19.1 and 20.3, 64: 25.7 and 22.5;  116: 12 000, 8, 1: 19.2 and 20.8, 64: 27.1 and
    //             25.6;  140: 12 000, 16, 1: 19.3 and 22.2, 64: 28.0 and 27.2;  144: 16 384, 4, 1: 19.6 and 23.3, 64: 27.9 and 29.5;
    //             192: 8192, 32 with weights, 1: 20.5 and 24.4, 64: 30.7 and 30.3;  320: 8192, 64 with weights, 64: 40.8 and 46.9
    //   B = 128:  load 256: 16 384, 16 with weights: 44.2 and 43.3, 8192, 48 with weights: 43.3 and 43.7;  192:
    //             8192, 64: 37.0 and 35.0;  320: 8192, 64 with weights: 48.3 and 51.0
    const pcg_prepared &p = *g.prepared_info;
    const int64_t slots = ((p.off_weights ? p.off_weights : p.bytes) - p.off_data) / 2;
    const int64_t load = g.V / 128 + slots / (g.weights ? 2048 : 4096);
    if (p.nchunks > 1) return load <= (B == 128 ? 256 : 130) ? small : StepShape::kFour;
    const CsrShape cut = step_csr_shape(g, B, K);
    return !csr_is_faster(g, cut) || load <= 176 + 30 * (csr_turns(cut) - 1) ? small : StepShape::kFour;
  }
  // The CSR is read by 256 sub-waves of four lanes: a turn takes 1024 groups, and a trip in it 16 entries of each (as many
  // trips as the mean group needs; four parts of a load of five for one).  The four kernels spread them over the chip, the less
  // of it the more sequences there are.
  //   load, B <= 64:   17: 1000, 64, 1: 16.0 and 14.7, 16: 17.4 and 15.2;  18: 2048, 24, 16: 17.2 and 15.7, with weights, 1: 16.2 and
  //                    16.4;  20: 4096, 16, 16: 18.8 and 16.2, with weights, 1: 17.7 and 17.4;  25: 5000, 16, 1: 18.5 and 18.0, with weights,
  //                    1: 18.7 and 19.4, K = 1, 64: 22.6 and 18.5;  27: 3000, 32, 1: 16.5 and 18.3, 64: 20.6 and 19.7;  29: 1000, 100, 1:
  //                    17.1 and 18.4;  30: 6000, 8, 1: 19.1 and 19.3
  //   65 to 96:        26: 2048, 48, 80: 21.3 and 17.8;  27: 3072, 32 with weights, 80: 21.8 and 22.0;  30: 6144, 12, 80: 23.1 and 21.0,
  //                    4 with weights, 80: 22.0 and 23.2;  35: 7168, 4 with weights, 80: 25.1 and 26.1
  //   97 to 128:       34: 2048, 64, 128: 23.9 and 19.8;  36: 4096, 32, 128: 26.7 and 24.2, with weights 29.0 and 28.6;  39: 3072, 48, 128:
  //                    28.5 and 25.4;  40: 8192, 4, 128: 27.6 and 27.9, with weights 28.4 and 31.9;  45: 5120, 32 with weights, 128:
  //                    32.7 and 34.8
  // Groups far above the mean are not in it: 1130 tokens, 416 groups of 75 and some of 1000, weights, 64: 20.9 and 23.7.
  const int64_t turns = (g.G + 1023) / 1024, per_turn = (g.nnz + 16 * (int64_t) g.G - 1) / (16 * (int64_t) g.G);
  const int64_t load = turns * (4 * per_turn + 1);
  const bool few = load <= (B <= 64 ? (g.weights && !one ? 21 : 25) : B <= 96 ? (g.weights ? 29 : 30) : (g.weights ? 36 : 39));
  return few ? small : StepShape::kFour;
}

hipError_t launch_small_step(const AcceptArgs &a, const FinalizeArgs &fa, const ProbeArgs &pa,
                             const pcg_groups &g, bool bf16, bool stats, int32_t B, hipStream_t stream) {
  const PreparedView p = g.prepared ? prepared_view(g) : PreparedView{};
  auto launch = [&](auto kernel) {
    kernel<<<B, kAcceptThreads, 0, stream>>>(a, fa, pa, p, (int32_t) g.nnz, csr_long_size(g.nnz, g.G, kSmallCsrWidth));
  };
  auto pick = [&](auto is_bf16, auto with_stats) {
    constexpr bool BF = decltype(is_bf16)::value, ST = decltype(with_stats)::value;
    if (g.prepared) { if (g.weights) launch(small_step_kernel<BF, kSumsPreparedWeighted, ST>); else launch(small_step_kernel<BF, kSumsPrepared, ST>); }
    else { if (g.weights) launch(small_step_kernel<BF, kSumsCsrWeighted, ST>); else launch(small_step_kernel<BF, kSumsCsr, ST>); }
  };
  if (bf16) { if (stats) pick(std::true_type{}, std::true_type{}); else pick(std::true_type{}, std::false_type{}); }
  else { if (stats) pick(std::false_type{}, std::true_type{}); else pick(std::false_type{}, std::false_type{}); }
  return hipGetLastError();
}

bool finalize_scans(int32_t G) { return G <= kScanGroups; }

hipError_t launch_finalize_sums(const FinalizeArgs &fa, bool bf16, const pcg_groups &g, int32_t B, hipStream_t stream) {
  if (bf16) finalize_sums_kernel<true><<<B, kFinalThreads, 0, stream>>>(fa, g.G);
  else finalize_sums_kernel<false><<<B, kFinalThreads, 0, stream>>>(fa, g.G);
  return hipGetLastError();
}

hipError_t launch_finalize(const FinalizeArgs &fa, bool bf16, const pcg_groups &g, int32_t B,
                           const double *csum, int64_t csum_stride, const double *runs, int32_t nchunks,
                           int32_t chunk_groups, hipStream_t stream) {
  auto launch = [&](auto kernel) {
    kernel<<<B, kFinalThreads, 0, stream>>>(fa, g.V, g.G, csum, csum_stride, runs, nchunks, chunk_groups);
  };
  if (g.nnz > 32 * (int64_t) g.G) { if (bf16) launch(finalize_kernel<true, 4>); else launch(finalize_kernel<false, 4>); }
  else { if (bf16) launch(finalize_kernel<true, 1>); else launch(finalize_kernel<false, 1>); }
  return hipGetLastError();
}

}  // namespace pcg
