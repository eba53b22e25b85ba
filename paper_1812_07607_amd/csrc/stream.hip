// stream.hip -- candidate pass of the eps-join for operand rows of up to 512
// bytes (d <= 256 in 16-bit formats, d <= 512 in E4M3): R stationary in
// registers, S streamed through LDS.
//
// Paper: section "Query Processing" (Nested Loop Join over all pairs) with
// the Euclidean predicate of section "Derived Data", recast as the product
// of the two operand copies on the matrix cores.
//
// What bounds a short-row pass is not the matrix cores but what feeds them:
// a 256 x 256 tile of d = 128 bf16 rows is two K-steps of work, for which
// both operand tiles go through LDS (128 KiB in, 384 KiB out) and every wave
// meets a barrier and an epilogue.  Here each wave keeps its rows of R as
// operand fragments in 128 registers for as long as its workgroup works on
// them, so only S moves: a strip of 32 S rows is read from LDS once per wave
// and meets all of the wave's 128 (or 64) R rows, a quarter of the LDS reads
// per product and an eighth of the operand traffic of the tile form.
//
// Layout: 512 threads = 8 waves.  WR of them along R, each with
// 16 * kNB rows of its own, times 8 / WR along S (the strips of a stage are
// dealt to them); WR is small when R is, so that a few rows still use every
// wave.  v_mfma_f32_16x16x32 (E4M3: 16x16x128): the strip's two 16-row blocks
// are the A operand, the wave's R rows the B operand, so the outputs a lane
// holds of one R block belong to one R row (lane % 16), and the candidate test
// is a minimum over registers and one compare with one threshold register per
// block.  The R fragments carry flipped signs: the accumulator starts at h_j
// and holds h_j - a.b = -P~ (exactly, each rounding being symmetric), which is
// compared with -thr_i.  The 16x16 form, not the 32x32 one: on random operands
// the matrix cores run into the board's power limit, and per product the
// 16x16x32 instruction moves half the accumulator bits (a loop of them on
// register operands of unit-vector values: 2.05 PFLOP/s at 2.0 GHz, of
// 32x32x16 ones 1.80; on constants both reach 2.45).
//
// S moves in stages of 24 or 32 KiB into a ring of four (global_load_lds,
// one 1 KiB transfer per 8 rows x 128 bytes, pieces swizzled as in the tile
// form).  One barrier per stage; at it every transfer but the one issued
// next has landed (three stages are in LDS or on the way), so a wave reads
// fragments ahead across stages, and a wave that stages candidates falls
// behind its SIMD partner, not behind the barrier.
//
// Work is counted in units of (block of WR * 16 kNB rows of R, stage of S),
// R-major; each workgroup takes one contiguous, equal share of the units, so
// no last round is part empty and R changes only a few times per workgroup.
// (Workgroups of one XCD walking S in step, so that its L2 serves them all,
// gained 1% on the 10^6-row join and lost the even shares: S is read once for
// each block of 1,024 rows of R, 250 GB there, 1.5 to 1.6 TB/s, which HBM gives.)
//
// Measured (one MI355X): the 10^6 x 10^6, d = 128, bf16 pass 158 to 169 ms on the
// cards seen (1.62 to 1.52 PFLOP/s) against the tile form's 238 ms; a loop of the
// same matrix instructions and LDS reads alone, on such operands, runs at 1.94
// PFLOP/s.  The matrix cores are busy 68% of the time at 2.13 GHz (168 ms); what
// idles them is not what bounds the pass: letting the two waves of a SIMD test in
// turns, or meeting a barrier every second stage only, changed nothing (the clock
// gives what the stalls no longer take).
#include <algorithm>
#include <type_traits>

#include "cand_device.hpp"

namespace dl {

hipError_t launch_zero_ranges(uint32_t*, int64_t, uint32_t*, int64_t, uint32_t*, int64_t, uint32_t*, int64_t,
                              hipStream_t, int);

template <int kPrec, int kKB>
struct StreamGeom {
  static constexpr int kSteps = kKB / 64;                   // 16-byte pieces per lane and 16 rows
  static constexpr int kUnit = kPrec == DL_FP8 ? 2 : 1;     // pieces per matrix instruction
  static constexpr int kUnits = kSteps / kUnit;
  // A fragments held: two units; E4M3, whose units are twice as large, holds
  // one and takes its two 16-row blocks in turn (each is read again while the
  // other is multiplied)
  static constexpr bool kTurns = kPrec == DL_FP8;
  static constexpr int kWindow = kTurns ? 1 : 2;
  static constexpr int kNB = kKB <= 256 ? 8 : 4;            // 16-row blocks of R per wave
  static constexpr int kWaveRows = 16 * kNB;
  static constexpr int kStageRows = kKB == 128 ? 256 : kKB == 256 ? 128 : 64;
  static constexpr int kStrips = kStageRows / 32;
  static constexpr int kStageBytes = kStageRows * kKB;
  static constexpr int kDma = kStageBytes / 1024 / 8;       // transfers per wave and stage
  static constexpr int kRowGroups = kStageRows / 8;
  static constexpr int kRecords = kPrec == DL_FP8 && kKB == 128 ? 96 : 128;  // staged per wave: what LDS has left
};
constexpr int kStreamStages = 4;

// c = c0 + x.y over one fragment unit (16-bit: 16x16x32; E4M3: 16x16x128 with
// the row scales sx and byte kByte of sy)
template <int kPrec, int kByte>
__device__ inline void stream_mac(f32x4& c, const f32x4& c0, const uint4* x, const uint4* y, int sx, int sy) {
  if constexpr (kPrec == DL_BF16) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[0]), __builtin_bit_cast(bf16x8, y[0]), c0,
                                                0, 0, 0);
  } else if constexpr (kPrec == DL_FP16) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, x[0]), __builtin_bit_cast(f16x8, y[0]), c0, 0,
                                               0, 0);
  } else {
    const i32x8 a{(int)x[0].x, (int)x[0].y, (int)x[0].z, (int)x[0].w, (int)x[1].x, (int)x[1].y, (int)x[1].z, (int)x[1].w};
    const i32x8 b{(int)y[0].x, (int)y[0].y, (int)y[0].z, (int)y[0].w, (int)y[1].x, (int)y[1].y, (int)y[1].z, (int)y[1].w};
    c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c0, 0, 0, 0, sx, kByte, sy);
  }
}

__device__ inline float min3(float a, float b, float c) {
  return __builtin_elementwise_minimum(__builtin_elementwise_minimum(a, b), c);
}

constexpr int kCmpOLE = 5;  // ordered <= (false for NaN)
__device__ inline uint64_t mask_le(float a, float b) { return __builtin_amdgcn_fcmpf(a, b, kCmpOLE); }

// A unit's place: R block and S stage, from its index.
struct UnitAt {
  int rb, st;
};
__device__ inline int stream_first(const StreamParams& p, int rb) { return p.c.self_join ? rb * p.stages_per_block : 0; }
__device__ inline int64_t stream_prefix(const StreamParams& p, int64_t rb) {
  return rb * p.nst - (p.c.self_join ? (int64_t)p.stages_per_block * (rb * (rb - 1) / 2) : 0);
}
__device__ inline UnitAt stream_unit(const StreamParams& p, int64_t L) {
  int lo = 0, hi = p.nrb - 1;
  while (lo < hi) {  // largest rb with prefix(rb) <= L
    const int mid = (lo + hi + 1) >> 1;
    if (stream_prefix(p, mid) <= L) lo = mid; else hi = mid - 1;
  }
  return {lo, stream_first(p, lo) + (int)(L - stream_prefix(p, lo))};
}

// Max mode: the first of the eight rows of S that octet o of the sample's strip
// t holds.  Octets lie evenly over S.  Consecutive ones fall into different
// slots (and the four of a strip into the four quarters of S), so that near rows
// that lie together in S spread over many groups: with the groups runs of S
// instead, a neighbourhood of consecutive rows fell into a few of them, and the
// k-th largest group maximum lay outside it (300,000 rows in order of their 100
// centres, top-10: 3,100 rows of S at or above a row's bound on average, against
// 270; in random order 90 either way).  A strip past the sample repeats row 0
// on (its outputs are dropped).
__device__ inline uint32_t sample_row(const StreamParams& p, uint32_t t, uint32_t o) {
  if (t >= (uint32_t)p.strips) return 0;
  const uint32_t q = udiv32(t, p.dv_slot_m, p.dv_slot_s1, p.dv_slot_s2);
  const uint32_t n = o * (uint32_t)p.strips + (t - q * (uint32_t)p.slot_strips) * (uint32_t)p.nslots + q;
  return 8 * (n * (uint32_t)(p.step >> 32) + __umulhi(n, (uint32_t)p.step));
}

// kStreamEps: candidates (P~ >= thr_i) to the global list.  kStreamBand: top-k
// band entries (P~ >= the row's threshold of p.gkey) to the row's buffer.
// kStreamMax: per row and group of S rows the largest P~ (p.gmax), from which
// the band's thresholds come.
enum : int { kStreamEps = 0, kStreamBand = 1, kStreamMax = 2 };

// A wave's staged outputs.  A record is one lane's four outputs of a 16 x 16
// block of which at least one passes: its row i, its first column j and the
// outputs (-P~).  Staging whole records costs one compaction per block, where
// compacting hit by hit costs eight compares and branches and fifteen
// instructions a hit; what each record holds is sorted out 64 records at a
// time, when the queue is full: the outputs against the row's threshold, the
// columns against the end of S and the diagonal.  Against hits staged one by
// one: 60,001 rows, d = 100, fp16, 0.58M candidates 463 -> 416 us of pass; top-10
// of 200,000 x 200,000 9.4 -> 9.0 ms of passes; of 37 x 4M 325 -> 287 us; 20,000 x 1M, d = 256, E4M3 6.1 -> 5.6 ms; 195M candidates in E4M3 9.5
// -> 4.7 ms (half of that by the list's parts).
// Bit r: output r of the record is a hit.
template <int kMode>
__device__ inline uint32_t record_hits(const StreamParams& p, const f32x4& v, const uint2& ij, float nthr) {
  uint32_t hits = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t j = ij.y + r;
    const bool in = v[r] <= nthr && j < (uint32_t)p.c.nS &&
                    (kMode == kStreamEps ? !p.c.self_join || j > ij.x : !p.c.exclude_self || j != ij.x + p.first_row);
    hits |= in ? 1u << r : 0u;
  }
  return hits;
}

// The hits of nq records, in their order, lo to hi - 1 of them to the candidate
// list from slot base on; returns their number.
template <bool kStageP, bool kWrite>
__device__ inline int spill_eps(const StreamParams& p, const f32x4* qv, const uint2* qij, const float* thr,
                                uint32_t row0, int nq, int64_t base, int lo, int hi) {
  const int lane = fresh_lane();
  int n = 0;
#pragma unroll 1
  for (int s0 = 0; s0 < nq; s0 += 64) {
    const int s = s0 + lane;
    uint32_t hits = 0;
    f32x4 v{};
    uint2 ij = make_uint2(0, 0);
    if (s < nq) {
      v = qv[s];
      ij = qij[s];
      hits = record_hits<kStreamEps>(p, v, ij, thr[ij.x - row0]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint64_t m = __ballot(hits >> r & 1);
      if (kWrite && (hits >> r & 1)) {
        const int at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        if (at >= lo && at < hi) {
          p.c.cand[base + (at - lo)] = make_uint2(ij.x, ij.y + r);
          if (kStageP && p.c.candp) p.c.candp[base + (at - lo)] = -v[r];
        }
      }
      n += __popcll(m);
    }
  }
  return n;
}
// All of them, to the workgroup's part of the list and, should it be full, the
// parts after it (past the last one hits are only counted: the caller retries
// with room).  Returns their number.
template <bool kStageP>
__device__ inline int flush_eps_records(const StreamParams& p, const f32x4* qv, const uint2* qij, const float* thr,
                                        uint32_t row0, int nq) {
  const int n = spill_eps<kStageP, false>(p, qv, qij, thr, row0, nq, 0, 0, 0);
  int lo = 0;
#pragma unroll 1
  for (int t = 0; t < kSegments && lo < n; ++t) {
    const int s = p.c.seg ? (blockIdx.x + t) & (kSegments - 1) : 0;
    unsigned long long at = 0;
    if (fresh_lane() == 0) at = atomicAdd(p.c.seg ? p.c.seg + s * kSegWords : p.c.ccount, (unsigned long long)(n - lo));
    const int64_t pos = uniform64((int64_t)at) + (p.c.seg ? segment_first(p.c.ccap, s) : 0);
    const int64_t room = (p.c.seg ? segment_end(p.c.ccap, s) : p.c.ccap) - pos;
    if (room > 0) {
      const int hi = room < n - lo ? lo + (int)room : n;
      spill_eps<kStageP, true>(p, qv, qij, thr, row0, nq, pos, lo, hi);
      lo = hi;
    }
    if (!p.c.seg) break;
  }
  return n;
}

// The hits of nq records to their rows' buffers, one atomic per record on the
// row's counter (two in flight per lane); entries past the buffer are counted
// and flagged.
__device__ inline void flush_rows(const StreamParams& p, const f32x4* qv, const uint2* qij, const float* thr,
                                  uint32_t row0, int nq) {
  const int lane = fresh_lane();
  uint32_t hits[2], at[2];
  f32x4 v[2];
  uint2 ij[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int s = 64 * h + lane;
    hits[h] = 0;
    if (s < nq) {
      v[h] = qv[s];
      ij[h] = qij[s];
      hits[h] = record_hits<kStreamBand>(p, v[h], ij[h], thr[ij[h].x - row0]);
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (hits[h]) at[h] = (uint32_t)atomicAdd(p.c.bcount + ij[h].x, __popc(hits[h]));
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (!hits[h]) continue;
    uint2* const row = p.c.band + (int64_t)ij[h].x * p.c.cap;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (!(hits[h] >> r & 1)) continue;
      if (at[h] < (uint32_t)p.c.cap) row[at[h]] = make_uint2(__float_as_uint(-v[h][r]), ij[h].y + r);
      else *p.c.overflow = 1;
      ++at[h];
    }
  }
}

template <int kPrec, int kKB, int kMode>
__global__ __launch_bounds__(kThreads, 1) void stream_kernel(StreamParams p) {
  using G = StreamGeom<kPrec, kKB>;
  constexpr bool kFp8 = kPrec == DL_FP8;
  constexpr int kNB = G::kNB, kUnits = G::kUnits, kW = G::kWindow, kU = G::kUnit;
  __shared__ __attribute__((aligned(1024))) uint8_t ring[kStreamStages][G::kStageBytes];
  __shared__ __attribute__((aligned(16))) float side_h[kStreamStages][G::kStageRows];
  __shared__ __attribute__((aligned(16))) int side_s[kFp8 ? kStreamStages : 1][kFp8 ? G::kStageRows : 4];
  constexpr bool kMax = kMode == kStreamMax;
  constexpr int kRecords = G::kRecords;
  __shared__ __attribute__((aligned(16))) f32x4 qv_lds[kMax ? 1 : kThreads / 64][kMax ? 1 : kRecords];
  __shared__ __attribute__((aligned(16))) uint2 qij_lds[kMax ? 1 : kThreads / 64][kMax ? 1 : kRecords];
  __shared__ float thr_lds[kMax ? 1 : kThreads / 64][kMax ? 1 : G::kWaveRows];  // nthr, by row
  constexpr bool kStageP = kMode == kStreamEps && !kFp8;  // (E4M3 candidates need no P~: it is never exact)

  if (p.c.gate && __builtin_amdgcn_readfirstlane(*p.c.gate)) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  // this workgroup's share of the units; consecutive shares on one XCD
  const int ng = gridDim.x;
  const int share = (blockIdx.x & 7) * (ng >> 3) + (blockIdx.x >> 3);
  const int64_t u0 = uniform64(p.units * share / ng), u1 = uniform64(p.units * (share + 1) / ng);
  const int nu = (int)(u1 - u0);
  if (nu <= 0) return;
  const int wr = p.wr, ws = 8 / wr;
  const int rw = wave & (wr - 1), grp = wave / wr;  // rows and strips of this wave
  const int per = G::kStrips / ws;                  // strips of a stage this wave takes

  UnitAt at = stream_unit(p, u0);
  int rb = __builtin_amdgcn_readfirstlane(at.rb), st = __builtin_amdgcn_readfirstlane(at.st);
  int lrb = rb, lst = st;  // of the loader's next unit
  int lu = 0;
  // One stage: every wave moves kDma blocks of 8 rows x 128 bytes.  A block is
  // kept as two 64-byte K-steps of 8 rows x 4 pieces; rows 4..7 of each 16
  // have the pieces exchanged by 1, 8..11 by 2, 12..15 by 3, so that one
  // piece of 16 rows touches all 64 banks.
  auto issue = [&]() {
    const int buf = lu & (kStreamStages - 1);
    const int64_t j0 = (int64_t)lst * G::kStageRows;
    const uint32_t t0 = (uint32_t)lst * G::kStrips;  // first strip
    const int l = fresh_lane();
    const uint8_t* src = p.c.qb + (kMax ? 0 : j0 * kKB);
    const uint32_t dst = lds_addr(&ring[buf][0]) + wave * G::kDma * 1024;
#pragma unroll
    for (int t = 0; t < G::kDma; ++t) {
      const int q = wave * G::kDma + t;
      const int c = q / G::kRowGroups, r8 = q % G::kRowGroups;
      const int row = r8 * 8 + ((l >> 2) & 7);
      const int piece = 4 * (l >> 5) + ((l ^ (row >> 2)) & 3);
      if constexpr (kMax)
        lds_dma16_at(src + (int64_t)sample_row(p, t0 + (r8 >> 2), r8 & 3) * kKB +
                         (uint32_t)((row & 7) * kKB + c * 128 + piece * 16),
                     dst + t * 1024);
      else
        lds_dma16_at(src + (uint32_t)(row * kKB + c * 128 + piece * 16), dst + t * 1024);
    }
    auto four = [&]() {  // the first of the lane's four rows
      return kMax ? (int64_t)sample_row(p, t0 + (l >> 3), (l >> 1) & 3) + 4 * (l & 1) : j0 + 4 * l;
    };
    if (wave == 7 && l < G::kStageRows / 4) lds_dma16(p.c.hb + four(), side_h[buf]);
    if constexpr (kFp8)
      if (wave == 6 && l < G::kStageRows / 4) lds_dma16(p.c.sexb + four(), side_s[buf]);
    ++lu;
    if (++lst == p.nst) {
      ++lrb;
      lst = stream_first(p, lrb);
    }
  };
#pragma unroll
  for (int s = 0; s < kStreamStages - 1; ++s)
    if (lu < nu) issue();

  uint4 rf[kNB][G::kSteps];  // the wave's R rows, signs flipped
  // of row lane % 16 of each block: -thr_i; max mode: the smallest output so
  // far of the lane's S rows of the current group
  float nthr[kNB];
  int rsc[kFp8 ? kNB / 4 : 1];  // E4M3: the rows' scales, four blocks to a register
  f32x4 acc[kNB][2];
  uint4 a[kW][2][kU];        // A fragments of the coming units, both 16-row blocks
  f32x4 ini[2];
  int ssc[2] = {0, 0};
  int nq = 0;
  // row numbers fit 32 bits (relations are shorter than 2^31 rows)
  uint32_t row0 = 0;  // first R row of this wave
  uint32_t pj = 0;    // first S row of the strip whose outputs await their test (max mode: the strip)
  int64_t hits = 0;  // flushed so far (eps)
  auto flush = [&]() {
    if constexpr (kMode == kStreamEps)
      hits += flush_eps_records<kStageP>(p, qv_lds[wave], qij_lds[wave], thr_lds[wave], row0, nq);
    if constexpr (kMode == kStreamBand) flush_rows(p, qv_lds[wave], qij_lds[wave], thr_lds[wave], row0, nq);
    nq = 0;
  };
  auto load_r = [&]() {
    if constexpr (!kMax)
      if (nq) flush();  // (the records' thresholds are the leaving rows')
    row0 = (uint32_t)(rb * wr + rw) * G::kWaveRows;
    const uint32_t flip = kFp8 ? 0x80808080u : 0x80008000u;
    // rows past the padded relation repeat its last row and never hit
    const int left = (int)(p.npad_r - (int64_t)row0 < G::kWaveRows ? p.npad_r - (int64_t)row0 : G::kWaveRows);
    const uint32_t i0 = left > 0 ? row0 : (uint32_t)p.npad_r - 1;
    const uint8_t* const src = p.c.qa + (int64_t)i0 * kKB;
#pragma unroll
    for (int b = 0; b < kNB; ++b) {
      const int l = fresh_lane();
      const int want = b * 16 + (l & 15);
      const uint32_t i = want < left ? want : (left > 0 ? left - 1 : 0);
      const uint32_t off = i * kKB + (l >> 4) * 16;
#pragma unroll
      for (int f = 0; f < G::kSteps; ++f) {
        uint4 v = *reinterpret_cast<const uint4*>(src + (off + f * 64));
        v.x ^= flip; v.y ^= flip; v.z ^= flip; v.w ^= flip;
        rf[b][f] = v;
      }
      if constexpr (kMode == kStreamEps) nthr[b] = want < left ? -p.c.thr[i0 + i] : -INFINITY;
      // (rows of the padding have no key: they never hit)
      if constexpr (kMode == kStreamBand)
        nthr[b] = (int64_t)row0 + want < p.c.nR ? -key_float(p.c.gkey[i0 + i]) : -INFINITY;
      if constexpr (kMax) nthr[b] = INFINITY;
      else if (l < 16) thr_lds[wave][want] = nthr[b];
      if constexpr (kFp8) {
        const int e = (p.c.sexa[i0 + i] + 127) << (8 * (b & 3));
        rsc[b / 4] = (b & 3) ? rsc[b / 4] | e : e;
      }
    }
  };
  // One block's outputs v (strip pj, threshold nt): the lanes of its two 16 x
  // 16 blocks that pass.
  auto passing = [&](const f32x4 (&v)[2], float nt, uint64_t (&m)[2]) {
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
      m[sb] = mask_le(__builtin_elementwise_minimum(min3(v[sb][0], v[sb][1], v[sb][2]), v[sb][3]), nt);
  };
  auto stage = [&](const f32x4& v, uint64_t m, uint32_t i, uint32_t j) {
    if (__builtin_amdgcn_inverse_ballot_w64(m)) {
      const int s = nq + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
      qv_lds[wave][s] = v;
      qij_lds[wave][s] = make_uint2(i, j);
    }
    nq += __popcll(m);
  };
  // The candidate test of a strip's outputs: four minimum instructions and a
  // compare per block, one branch for all.  A strip with few hits stages its
  // records straight from the accumulators; one with many takes its blocks
  // through one copy of the code that checks the queue's room (a copy each
  // would overflow the instruction cache).
  auto test = [&]() {
    uint64_t any = 0, h[kNB];
#pragma unroll
    for (int b = 0; b < kNB; ++b) {
      const f32x4 &v = acc[b][0], &w = acc[b][1];
      h[b] = mask_le(min3(min3(v[0], v[1], v[2]), min3(v[3], w[0], w[1]), __builtin_elementwise_minimum(w[2], w[3])),
                     nthr[b]);
      any |= h[b];
    }
    if (!any) return;
    int most = 0;  // records of the strip, at most
#pragma unroll
    for (int b = 0; b < kNB; ++b) most += 2 * __popcll(h[b]);
    if (nq + most > kRecords && nq > 0) flush();
    if (most <= kRecords) {
      const int l = fresh_lane();
      const uint32_t i0 = row0 + (l & 15), j0 = pj + 4 * (l >> 4);
#pragma unroll
      for (int b = 0; b < kNB; ++b) {
        if (!h[b]) continue;
        uint64_t m[2];
        passing(acc[b], nthr[b], m);
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) stage(acc[b][sb], m[sb], i0 + b * 16, j0 + 16 * sb);
      }
      return;
    }
    uint32_t hb = 0;
#pragma unroll
    for (int b = 0; b < kNB; ++b) hb |= (h[b] ? 1u : 0u) << b;
#pragma unroll 1
    while (hb) {
      const int b = __builtin_ctz(hb);
      hb &= hb - 1;
      f32x4 v[2];
      float nt = 0.0f;
#pragma unroll
      for (int c = 0; c < kNB; ++c)
        if (b == c) {
          v[0] = acc[c][0];
          v[1] = acc[c][1];
          nt = nthr[c];
          // a uniform jump to eight moves, not a chain of selects
          asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(nt));
        }
      uint64_t m[2];
      passing(v, nt, m);
#pragma unroll 1
      for (int sb = 0; sb < 2; ++sb) {  // (64 records at most each)
        if (nq + __popcll(m[0]) > kRecords) flush();
        const int l = fresh_lane();
        stage(v[0], m[0], row0 + b * 16 + (l & 15), pj + 16 * sb + 4 * (l >> 4));
        v[0] = v[1];
        m[0] = m[1];
      }
    }
  };
  // Max mode: the strip's outputs into the running minima (all of its rows are
  // rows of S; the row itself, in a self-join, is not left out: the caller takes
  // the (k + 1)-th largest).
  bool fresh_acc = false;  // the accumulators hold a strip's outputs
  auto fold = [&]() {
    if (!fresh_acc || pj >= (uint32_t)p.strips) return;
#pragma unroll
    for (int b = 0; b < kNB; ++b) {
      const f32x4 &v = acc[b][0], &w = acc[b][1];
      nthr[b] = min3(min3(nthr[b], v[0], v[1]), min3(v[2], v[3], w[0]), min3(w[1], w[2], w[3]));
    }
  };
  // the running minima to group `slot` (of every lane quarter), and restart
  auto put_max = [&](uint32_t slot) {
    if (slot >= (uint32_t)p.nslots) return;  // strips past the sample
    const int l = fresh_lane();
    uint32_t* const g = p.gmax + (int64_t)slot * 4 * p.c.nR;
#pragma unroll
    for (int b = 0; b < kNB; ++b) {
      const int64_t i = (int64_t)row0 + b * 16 + (l & 15);
      if (i < p.c.nR) atomicMax(g + (l >> 4) * p.c.nR + i, order_key(-nthr[b]));
      nthr[b] = INFINITY;
    }
  };

  // the lane's LDS offset of its piece of K-step 0 of 16 rows; the K-step and
  // the 16-row block are immediate offsets (formed anew for each strip: kept
  // over the test it would be spilled, and a reload waits for every transfer
  // issued before it)
  int lo0;
  auto piece_offset = [&]() {
    const int l = fresh_lane();
    const int r16 = l & 15;
    lo0 = (r16 >> 3) * 1024 + (r16 & 7) * 64 + (((l >> 4) ^ (r16 >> 2)) << 4);
  };
  auto load_a1 = [&](const uint8_t* strip, int u, int sb) {
#pragma unroll
    for (int q = 0; q < kU; ++q) {
      const int f = u * kU + q;
      a[u % kW][sb][q] = *reinterpret_cast<const uint4*>(strip + lo0 + (sb * 2048 + (f >> 1) * (G::kStageRows * 128) +
                                                                        (f & 1) * 512));
    }
  };
  auto load_a = [&](const uint8_t* strip, int u) {
    load_a1(strip, u, 0);
    load_a1(strip, u, 1);
  };
  auto load_ini = [&](int buf, int strip) {
    const int l = fresh_lane();
    const float* h = &side_h[buf][strip * 32 + 4 * (l >> 4)];
    ini[0] = *reinterpret_cast<const f32x4*>(h);
    ini[1] = *reinterpret_cast<const f32x4*>(h + 16);
  };
  // the E4M3 scales of the strip's 16-row block sb (used by every unit)
  auto load_scale = [&](int buf, int strip, int sb) {
    if constexpr (kFp8) ssc[sb] = side_s[buf][strip * 32 + sb * 16 + (fresh_lane() & 15)] + 127;
  };
  // unit u of the current strip for blocks b0 .. b0 + 3 and S blocks s0 ..
  // s1 - 1 (kFirst: from the initial values)
  auto mac4 = [&](auto first, int u, int b0, int s0, int s1) {
    constexpr bool kFirst = decltype(first)::value;
#define DL_STREAM_MAC(B)                                                                                       \
  _Pragma("unroll") for (int sb = s0; sb < s1; ++sb)                                                           \
      stream_mac<kPrec, B>(acc[b0 + B][sb], kFirst ? ini[sb] : acc[b0 + B][sb], a[u % kW][sb],                 \
                           &rf[b0 + B][u * kU], ssc[sb], kFp8 ? rsc[b0 / 4] : 0);
    DL_STREAM_MAC(0)
    DL_STREAM_MAC(1)
    DL_STREAM_MAC(2)
    DL_STREAM_MAC(3)
#undef DL_STREAM_MAC
  };
  using True = std::true_type;
  using False = std::false_type;

  load_r();
#pragma unroll
  for (int b = 0; b < kNB; ++b) acc[b][0] = acc[b][1] = f32x4{NAN, NAN, NAN, NAN};  // no outputs yet
  int u = 0, t = 0, buf = 0;
  bool fresh_r = false;  // the next strip meets a new block of R
  // max mode: the run of strips being folded, and where it ends
  uint32_t slot = 0, slot_end = 0;
  for (;;) {  // one strip per pass; the last pass only tests
    if (t == 0 && u < nu) {
      // the stages up to the next one have landed (this wave's transfers by
      // the wait, the others' by the barrier), and the stage before this one
      // is free
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0x0070);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      buf = u & (kStreamStages - 1);
      if (lu < nu) issue();
      if (u == 0) {
        piece_offset();
#pragma unroll
        for (int f = 0; f < kW; ++f) load_a(ring[buf] + grp * 4096, f);
        load_ini(buf, grp);
        load_scale(buf, grp, 0);
        load_scale(buf, grp, 1);
      }
    }
    // the last strip's outputs are tested just before this strip's first
    // products replace them
    const int strip = t * ws + grp;
    if constexpr (kMax) {
      fold();
      const uint32_t s = (uint32_t)(st * G::kStrips + strip);
      if (!fresh_acc || fresh_r || u == nu || s >= slot_end) {
        if (fresh_acc) put_max(slot);
        slot = s / (uint32_t)p.slot_strips;
        slot_end = (slot + 1) * (uint32_t)p.slot_strips;
      }
      fresh_acc = true;
    } else {
      test();
    }
    if (u == nu) break;
    if (fresh_r) {
      load_r();
      fresh_r = false;
    }
    piece_offset();
    const bool last = t + 1 == per;
    const int nbuf = last ? (buf + 1) & (kStreamStages - 1) : buf;
    const int nstrip = last ? grp : strip + ws;
    const uint8_t* cur = ring[buf] + strip * 4096;
    const uint8_t* nxt = ring[nbuf] + nstrip * 4096;
    // the products stay behind the test's branch (moved above it they would
    // need a second set of accumulators), and fragments are read into the
    // registers just used, not beside them
    asm volatile("" : "+v"(ini[0]), "+v"(ini[1]));
    if constexpr (G::kTurns) {
#pragma unroll
      for (int f = 0; f < kUnits; ++f) {
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
#pragma unroll
          for (int b = 0; b < kNB; b += 4)
            if (f == 0) mac4(True{}, f, b, sb, sb + 1); else mac4(False{}, f, b, sb, sb + 1);
          __builtin_amdgcn_sched_barrier(0);
          if (f == 0 && sb == 1) load_ini(nbuf, nstrip);
          load_a1(f + 1 < kUnits ? cur : nxt, f + 1 < kUnits ? f + 1 : 0, sb);
          if (f + 1 == kUnits) load_scale(nbuf, nstrip, sb);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
#pragma unroll
      for (int f = 0; f < kUnits; ++f) {
#pragma unroll
        for (int b = 0; b < kNB; b += 4)
          if (f == 0) mac4(True{}, f, b, 0, 2); else mac4(False{}, f, b, 0, 2);
        __builtin_amdgcn_sched_barrier(0);
        if (f == 0) load_ini(nbuf, nstrip);
        load_a(f + kW < kUnits ? cur : nxt, f + kW < kUnits ? f + kW : f + kW - kUnits);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    pj = kMax ? (uint32_t)(st * G::kStrips + strip) : (uint32_t)st * G::kStageRows + strip * 32;
    if (++t == per) {
      t = 0;
      ++u;
      if (++st == p.nst) {
        ++rb;
        st = stream_first(p, rb);
        fresh_r = true;
      }
    }
  }
  if constexpr (kMode == kStreamEps) {
    if (nq) flush();
    if (p.c.seg) {
      // the workgroup's total; the words lie in a stage no wave reads any more
      int64_t* const s_hits = reinterpret_cast<int64_t*>(ring[nu & (kStreamStages - 1)]);
      if (lane == 0) s_hits[wave] = hits;
      __syncthreads();
      if (threadIdx.x == 0) {
        unsigned long long all = 0;
        for (int w = 0; w < kThreads / 64; ++w) all += (unsigned long long)s_hits[w];
        if (all) atomicAdd(p.c.ccount, all);
      }
    }
  } else if constexpr (kMode == kStreamBand) {
    if (nq) flush();
  }
}

// The k-th largest of each row's ngroups group maxima (order keys, group-major,
// zero where a group is empty), minus the row's margin, as the row's band
// threshold.  The groups partition a subset of S, so at least k rows of S have
// a P~ at or above it: the band P~ >= v - E_i keeps every one of the k
// nearest, as in the tile form's tightening.  kPer lanes share a row, each
// with kKeys of its keys in registers, 64 / kPer rows side by side in a wave.
// Many rows: 64 keys a lane.  Few: the rows' latency is the kernel's time, so
// their keys are spread over as many lanes as leave eight each (37 rows of 64
// keys: 26 -> 8 us).
constexpr int kKeys = 64, kFewKeys = 8;
template <int kPer, int kKeys>
__global__ __launch_bounds__(64) void band_key_kernel(const uint32_t* __restrict__ gmax, int ngroups, int64_t nR, int k,
                                                      const float* __restrict__ marg, uint32_t* __restrict__ gkey) {
  constexpr int kRows = 64 / kPer;
  const int part = threadIdx.x / kRows;
  const int64_t i = (int64_t)blockIdx.x * kRows + threadIdx.x % kRows;
  uint32_t key[kKeys];
#pragma unroll
  for (int t = 0; t < kKeys; ++t) {
    const int g = t * kPer + part;
    key[t] = g < ngroups && i < nR ? gmax[(int64_t)g * nR + i] : 0u;
  }
  uint32_t v = 0;  // largest key with at least k group maxima at or above it
  for (int b = 31; b >= 0; --b) {
    const uint32_t cand = v | (1u << b);
    int c = 0;
#pragma unroll
    for (int t = 0; t < kKeys; ++t) c += key[t] >= cand;
#pragma unroll
    for (int o = kRows; o < 64; o <<= 1) c += __shfl_xor(c, o, 64);
    if (c >= k) v = cand;
  }
  // (fewer than k groups: no bound)
  if (part == 0 && i < nR && v > order_key(-INFINITY))
    gkey[i] = max(gkey[i], order_key(f32_down((double)key_float(v) - (double)marg[i])));
}

// Whether the pass takes rows of qld operand bytes: as many R fragments as
// registers hold.  float32 candidates stay with the tile form (its rate is the
// matrix cores' own there).  The unit count of a workgroup is 32-bit.
bool stream_applies(dl_prec prec, int64_t qld, int64_t nR, int64_t nS) {
  return prec != DL_FP32 && (qld == 128 || qld == 256 || qld == 384 || qld == 512) &&
         (double)nR * (double)nS < 0x1p51;
}

// Whether an eps-join's pass is left to the tile form, having few tiles of 256 x
// 256: where every tile has a CU of its own that form is a load of two tiles and
// one epilogue, and the streaming pass has its R fragments to load and its ring
// to fill first (12.5 us of pass against 24.4 at 3,000 x 3,000, d = 256, no
// candidates).  Call time, tile form over streaming, d = 128, bf16, no pairs and 5
// a row: 2,560 x 2,560 (100 tiles) 0.84 and 0.97, 4,000 x 4,000 (256) 0.83 and
// 0.96, 300 x 30,000 (236) 0.82 and 0.92.  With more tiles than CUs the pairs make
// up for it: 6,000 x 6,000 (576) 0.91 and 1.01.  So they do where the form leaves
// CUs idle over the candidates' staging, with few tiles (1,100 x 1,100, 25: 0.91
// and 1.04; 2,600 to itself, 66: 0.91 and 1.03), or with an R much longer than S,
// whose candidates sit in few columns (20,000 x 300: 0.90 and 1.05), and earlier in
// self-joins, half of whose diagonal tiles is dropped (4,000, 136: 0.90 and 0.98;
// 5,500, 253: 0.87 and 0.99, E4M3 1.08).
bool few_tiles(int64_t nR, int64_t nS, bool self, int cu_count) {
  const int64_t tr = (nR + kTile - 1) / kTile, ts = (nS + kTile - 1) / kTile;
  const int64_t tiles = self ? tr * (tr + 1) / 2 : tr * ts;
  return tiles > cu_count * 3 / 8 && tiles <= (self ? cu_count * 5 / 8 : cu_count) && tr <= 4 * ts;
}

template <int kPrec, int kKB, int kMode>
static hipError_t launch_stream_kb(StreamParams p, int64_t npad_r, hipStream_t st, int cu_count) {
  using G = StreamGeom<kPrec, kKB>;
  p.npad_r = npad_r;
  p.nst = kMode == kStreamMax ? (p.strips + G::kStrips - 1) / G::kStrips
                              : (int)((p.c.nS + G::kStageRows - 1) / G::kStageRows);
  // waves along R: as many as R fills, fewer while there are fewer than four
  // units per workgroup (a stage has to hold a strip for every wave along S,
  // and a self-join's block at least a stage)
  int wr = 8;
  const int wr_min = 8 / (G::kStrips < 8 ? G::kStrips : 8);
  const bool tri = p.c.self_join;
  auto units_of = [&](int w) {
    const int64_t rows = (int64_t)w * G::kWaveRows, nrb = (p.c.nR + rows - 1) / rows;
    const int64_t spb = rows / G::kStageRows;
    return nrb * p.nst - (tri ? spb * (nrb * (nrb - 1) / 2) : 0);
  };
  while (wr > wr_min && (!tri || wr / 2 * G::kWaveRows >= G::kStageRows) &&
         (p.c.nR <= (int64_t)(wr / 2) * G::kWaveRows || units_of(wr) < 4 * (int64_t)cu_count))
    wr /= 2;
  p.wr = wr;
  const int64_t rows = (int64_t)wr * G::kWaveRows;
  p.nrb = (int)((p.c.nR + rows - 1) / rows);
  p.stages_per_block = (int)(rows / G::kStageRows);
  p.units = units_of(wr);
  int64_t g = cu_count / 8 * 8;
  if (g > (p.units + 7) / 8 * 8) g = (p.units + 7) / 8 * 8;
  hipLaunchKernelGGL((stream_kernel<kPrec, kKB, kMode>), dim3((unsigned)g), dim3(kThreads), 0, st, p);
  return hipGetLastError();
}

template <int kMode, int kPrec>
static hipError_t launch_stream_prec(const StreamParams& p, int64_t npad_r, hipStream_t st, int cu_count) {
  switch (p.c.qld) {
    case 128: return launch_stream_kb<kPrec, 128, kMode>(p, npad_r, st, cu_count);
    case 256: return launch_stream_kb<kPrec, 256, kMode>(p, npad_r, st, cu_count);
    case 384: return launch_stream_kb<kPrec, 384, kMode>(p, npad_r, st, cu_count);
    case 512: return launch_stream_kb<kPrec, 512, kMode>(p, npad_r, st, cu_count);
  }
  return hipErrorInvalidValue;
}

template <int kMode>
static hipError_t launch_stream(dl_prec prec, const StreamParams& p, int64_t npad_r, hipStream_t st, int cu_count) {
  if (p.c.nR == 0 || p.c.nS == 0) return hipSuccess;
  switch (prec) {
    case DL_BF16: return launch_stream_prec<kMode, DL_BF16>(p, npad_r, st, cu_count);
    case DL_FP16: return launch_stream_prec<kMode, DL_FP16>(p, npad_r, st, cu_count);
    case DL_FP8: return launch_stream_prec<kMode, DL_FP8>(p, npad_r, st, cu_count);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_stream_eps(dl_prec prec, const CandParams& c, int64_t npad_r, hipStream_t st, int cu_count) {
  StreamParams p{};
  p.c = c;
  return launch_stream<kStreamEps>(prec, p, npad_r, st, cu_count);
}

// Groups of S rows whose maxima bound a row's k-th largest P~: a few times k,
// so that the k largest rarely share one (ngroups / 4 slots of sampled strips,
// each split over the four lane quarters).
int stream_groups(int k) {
  const int g = (4 * k + 63) / 64 * 64;
  return g < 64 ? 64 : g;
}

// Whether the streaming top-k's thresholds exist (enough groups of S rows) or
// are not needed (all of S fits a row's buffer, of at least kAllRows entries).
constexpr int64_t kAllRows = 512;
bool stream_band_applies(int64_t nS, int k) { return nS >= 16 * (int64_t)k || nS <= kAllRows; }

// One row in how many of S the sample takes.  The sample costs 1 / stride
// of a pass and leaves about stride times the rows of the band itself to be
// staged and selected from.  Few rows wait for what they stage: the sum is
// smallest where stride^2 is nS / 100 (k + 90) or so (37 x 4M, top-10: 20, 285
// us of passes; 36, 299).  Many hide it behind the matrix cores: nS / (240 k +
// 600) (200,000 x 200,000, top-10, passes: stride 4 9.08 ms, 5 8.87, 6 8.80, 8
// 8.69; 178,455 x 247,864, top-50: 4 11.7, 5 11.8, 6 12.0), up to 8, or what few
// rows would take where that is more.  E4M3 takes at most 8: its margin is as
// wide as the spread of near rows, so its bands grow faster as the threshold
// loosens (50,000 queries x 4M rows, d = 256, top-32: stride 9 takes 64 ms of
// call time, 4 takes 70, 18 overflows buffers).
static int sample_stride(dl_prec prec, int64_t nR, int64_t nS, int k) {
  int few = 1, many = 1;
  while ((int64_t)(few + 1) * (few + 1) * 100 * (k + 90) <= nS) ++few;
  while (many < 8 && (int64_t)(many + 1) * (many + 1) * (240 * k + 600) <= nS) ++many;
  const int s = nR >= 1024 && many > few ? many : few;
  return prec == DL_FP8 && s > 8 ? 8 : s;
}

// Room for a row's entries: with less the rows of R are to go in blocks.  The
// k-th largest of the group maxima is about the 1.15 k stride-th largest P~, up
// to twice that for the worst of many rows, and the margin lets a few times as
// many in where the rows of S are dense about the k-th; of rows that lie
// together in S near ones share groups, so that up to 4 k stride of them can be
// above the bound.  The fullest of 1,024 rows, random mixtures (d = 128, bf16):
// k = 10, stride 8: 255 entries; 50, 4: 550; 100, 3: 507; 256, 2: 845; 10, 28
// (8M rows): 1,272; S in order of its centres: 10, 8: 587; 50, 4: 1,059; 256, 2:
// 2,105.  E4M3's margin holds a row's whole neighbourhood (980 entries at d = 256, k
// = 32, 1,000 rows a centre; 2,960 at d = 128 and 3,000): room for a thirty-second of
// S, up to 4,096 (65,536 x 4,000, k = 10: 0.59 ms; in blocks 0.87).  A sample of every
// row leaves less: buffers of 1,024 held k = 100 to 127 of 65,536 x 2,100 to 20,000
// rows (16 bits, d = 64 and 256, 3 to 1,000 centres, in order and not), where two
// blocks cost 5% (k = 100 of 65,536 x 4,000: 1.85 ms, 1.95).
int64_t stream_band_room(dl_prec prec, int64_t nR, int64_t nS, int k) {
  const int stride = sample_stride(prec, nR, nS, k);
  const int64_t margin = prec == DL_FP8 ? std::clamp<int64_t>(nS / 32, 512, 4096) : 512;
  const int64_t room = (stride == 1 ? 4 : 6) * (int64_t)k * stride + margin;
  return room < nS ? room : nS;
}

template <int kKeysOf>
static hipError_t launch_band_key_of(int per, const uint32_t* gmax, int ng, int64_t nR, int k, const float* marg,
                                     uint32_t* gkey, hipStream_t st) {
  const dim3 grid((unsigned)((nR + 64 / per - 1) / (64 / per))), block(64);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, st, gmax, ng, nR, k, marg, gkey); };
  switch (per) {
    case 1: go(band_key_kernel<1, kKeysOf>); break;
    case 2: go(band_key_kernel<2, kKeysOf>); break;
    case 4: go(band_key_kernel<4, kKeysOf>); break;
    case 8: go(band_key_kernel<8, kKeysOf>); break;
    case 16: go(band_key_kernel<16, kKeysOf>); break;
    default: go(band_key_kernel<32, kKeysOf>); break;
  }
  return hipGetLastError();
}
static hipError_t launch_band_key(const uint32_t* gmax, int ng, int64_t nR, int k, const float* marg, uint32_t* gkey,
                                  hipStream_t st, int cu_count) {
  int per = 1, few = 8;
  while (per * kKeys < ng) per *= 2;
  while (few * kFewKeys < ng) few *= 2;
  if (few <= 32 && nR * few <= (int64_t)cu_count * 4 * 64)  // a wave per SIMD at most
    return launch_band_key_of<kFewKeys>(few, gmax, ng, nR, k, marg, gkey, st);
  return launch_band_key_of<kKeys>(per, gmax, ng, nR, k, marg, gkey, st);
}

// The sample: as many strips as S has octets for at this stride, cut to whole
// slots (of at most nslots, the number that drops the fewest strips; S of 16 k
// rows and more leaves at least 2 k groups), its octets spread over all of S.
static void plan_sample(StreamParams& p, int64_t nS, int ngroups) {
  const int64_t octets = nS / 8, strips = (octets + p.stride - 1) / p.stride / 4;
  int best = 1;
  int64_t left = strips;
  for (int n = ngroups / 4 < strips ? ngroups / 4 : (int)strips; 8 * n >= ngroups || (n > 0 && n == strips); --n)
    if (strips % n < left) {
      best = n;
      left = strips % n;
    }
  p.nslots = best;
  p.slot_strips = (int)(strips / best);
  p.strips = p.nslots * p.slot_strips;
  div_magic((uint32_t)p.slot_strips, p.dv_slot_m, p.dv_slot_s1, p.dv_slot_s2);
  p.step = p.strips ? ((uint64_t)octets << 32) / (4 * (uint64_t)p.strips) : 0;
}

// Thresholds of the top-k band of every row of R: its k-th largest group maximum
// over a sample of S.  gmax: scratch of stream_groups(k) * nR words.  c.gkey holds
// what bounds are known (order keys).
hipError_t launch_stream_keys(dl_prec prec, const CandParams& c, int64_t npad_r, int k, uint32_t* gmax, hipStream_t st,
                              int cu_count) {
  if (c.nR == 0 || c.nS <= kAllRows) return hipSuccess;
  StreamParams p{};
  p.c = c;
  p.c.self_join = 0;
  p.stride = sample_stride(prec, c.nR, c.nS, k);
  plan_sample(p, c.nS, stream_groups(k));
  const int ng = 4 * p.nslots;
  p.gmax = gmax;
  hipError_t e = launch_zero_ranges(gmax, ng * c.nR, nullptr, 0, nullptr, 0, nullptr, 0, st, cu_count);
  if (e != hipSuccess) return e;
  if ((e = launch_stream<kStreamMax>(prec, p, npad_r, st, cu_count)) != hipSuccess) return e;
  return launch_band_key(gmax, ng, c.nR, k, c.marg, c.gkey, st, cu_count);
}

// Top-k band of rows of R whose thresholds are known: the pass over all of S
// stages what reaches them.  c.bcount: zeros; c's row 0 is R's row first_row.
//
// Measured (one MI355X): top-10 of 200,000 x 200,000, d = 128, bf16: sample
// 0.85 ms, thresholds 0.05, pass 7.9, against 21.4 ms for the tile form, whose
// bands are tightened row by row inside the pass.
hipError_t launch_stream_band(dl_prec prec, const CandParams& c, int64_t npad_r, int64_t first_row, hipStream_t st,
                              int cu_count) {
  StreamParams p{};
  p.c = c;
  p.c.self_join = 0;
  p.first_row = (uint32_t)first_row;
  return launch_stream<kStreamBand>(prec, p, npad_r, st, cu_count);
}

}  // namespace dl
