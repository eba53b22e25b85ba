// join_params.hpp -- launch parameters shared by the join kernels and the
// C ABI layer.
#pragma once

#include "dl_internal.hpp"

namespace dl {

// Device-side counters of one call (cleared by a kernel, so the sequence can
// be captured in a graph).
struct Counters {
  unsigned long long cand;   // candidates appended
  unsigned long long out;    // pairs confirmed
  unsigned long long ties;   // float64 decisions
  int bad_index;
  int overflow;
  int too_many;
  int invalid;  // an input relation has a non-finite value or a row norm >= 2^62
  int pad[6];
};
static_assert(sizeof(Counters) == 64, "counter block size");

// Counts of the top-k selection, spread over cache lines of their own (summed
// by the host).
struct SelectCount {
  unsigned long long band;  // entries in the exact band
  unsigned long long ties;  // entries ordered in float64
  unsigned long long pad[6];
};
constexpr int kSelectCounts = 32;

// What a join call clears at its start and sends to the host at its end, in
// one piece.
struct CallState {
  Counters c;
  RelStats r, s;  // the relations' maxima
  SelectCount sel[kSelectCounts];
};
constexpr int kStateWords = (sizeof(Counters) + 2 * sizeof(RelStats)) / 8;  // 64-bit words without the counts
static_assert(sizeof(CallState) == 8 * kStateWords + sizeof(SelectCount) * kSelectCounts, "one piece");

// One relation of a prep launch.
struct PrepJob {
  const float* X;
  int64_t n, ld;
  Prep P;
  RelStats* rs;
  const uint32_t* perm;  // nullable: operand row r holds row perm[r] of X
};
struct PrepPair {
  PrepJob j[2];  // the second may be empty (P.npad 0)
};

// A candidate list in parts: part s holds the slots from segment_first(cap, s)
// to the next part's first.  A pass that finds many candidates is bound by the
// list's counter (17 ns an atomic on one address, whoever sends it: 195M
// candidates in flushes of 128 took 26 ms of counter); eight count side by
// side.  A flush that its part has no room for goes on in the next one, so the
// list holds as many candidates as one part of its size would.
constexpr int kSegments = 8;
constexpr int kSegWords = 16;  // 64-bit words between counters: lines of their own
__host__ __device__ inline int64_t segment_first(int64_t cap, int s) { return cap / kSegments * s; }
__host__ __device__ inline int64_t segment_end(int64_t cap, int s) {
  return s + 1 == kSegments ? cap : segment_first(cap, s + 1);
}

// Division of a 32-bit block-uniform n by an invariant d through a
// multiply-high and shifts (Granlund and Montgomery, "Division by Invariant
// Integers using Multiplication", PLDI 1994): q = (t + ((n - t) >> s1)) >> s2
// with t = mulhi(m, n); m, s1, s2 come from the host (div_magic).
__device__ inline uint32_t udiv32(uint32_t n, uint32_t m, uint32_t s1, uint32_t s2) {
  const uint32_t t = __umulhi(n, m);
  return (t + ((n - t) >> s1)) >> s2;
}
inline void div_magic(uint32_t d, uint32_t& m, uint32_t& s1, uint32_t& s2) {
  uint32_t l = 0;
  while (l < 32 && (1ull << l) < d) ++l;
  m = (uint32_t)(((((1ull << l) - d) << 32) / d) + 1);
  s1 = l < 1 ? l : 1;
  s2 = l > 1 ? l - 1 : 0;
}

// Candidate pass on the matrix cores (join_mfma.hip).
struct CandParams {
  const uint8_t* qa;   // R operand rows (qld bytes each, npad rows)
  const uint8_t* qb;   // S operand rows
  int64_t qld;         // bytes per operand row (multiple of kChunkBytes)
  int nchunks;         // qld / kChunkBytes
  const float* hb;     // S accumulator init h_j (npadS)
  const int* sexa;     // FP8 row scales of R / S
  const int* sexb;
  int64_t nR, nS;      // real rows
  int64_t nTR, nTS;    // tiles
  int self_join;       // eps: keep j > i only; band: exclude j == i when excl
  int exclude_self;
  // tile order (eps mode)
  int GM;              // row tiles per group
  int64_t ngroups;
  int64_t nlogical;    // logical tiles incl. skipped ones
  // 32-bit division by the tile-order divisors (valid when small32): the
  // group size GM * nTS, GM, and the last group's height
  int small32;
  uint32_t dv_grp_m, dv_grp_s1, dv_grp_s2;
  uint32_t dv_gm_m, dv_gm_s1, dv_gm_s2;
  uint32_t dv_gl_m, dv_gl_s1, dv_gl_s2;
  // eps mode
  const float* thr;    // per R row (npadR)
  unsigned long long* ccount;  // candidate counter
  uint2* cand;         // (i, j) records
  float* candp;        // P~ of each record (null: not kept)
  int64_t ccap;
  // streaming pass (nullable): counters of the list's kSegments parts, each on
  // lines of its own; ccount then gets every workgroup's total once
  unsigned long long* seg;
  // band mode
  int P;               // S splits
  int64_t tps;         // S tiles per split
  int k;
  int cap;             // band entries per (row, split)
  int retight;         // entries appended to a row between tightenings
  int limit;           // highest trigger; a count reaching it forces a round
  int batch;           // queued rows that start a tightening round
  uint32_t* gkey;      // per row: largest band threshold of any split (order key)
  int flood;           // 1: every threshold starts at -inf (else from gkey)
  const float* marg;   // E_i per R row
  uint2* band;         // (P~ bits, j): [(row * P + split) * cap + slot]
  int* bcount;         // [row * P + split]
  int* overflow;       // set when a band exceeds cap - 256
  // band mode over the tiles of an index (nullable): bit tj of row tile
  // ti's words surv[ti * sw ..] set when (ti, tj) may hold a row's top-k
  // neighbour (other tiles are skipped); jmap[j] = the index in S that band
  // entries carry for column j of the ordered S
  const uint32_t* surv;
  int64_t sw;
  const uint32_t* jmap;
  const int* gate;     // nonzero: invalid input, the kernel does nothing
  // eps mode over a tile list (index-pruned join): (ti, tj) entries and the
  // device-side count; null = every tile
  const uint2* tiles;
  const unsigned long long* ntiles;
  int64_t list_all;    // nonzero: walk the list only if 2 * *ntiles < list_all, else the full grid
  // mark mode: bit (tile tj, row i) at mark[tj * mark_words + i / 32]
  uint32_t* mark;
  int64_t mark_words;
  // nearest mode: per row, the maximum of (order key of P~ << 32 | ~column)
  unsigned long long* argkey;
  // eps mode (nullable, at most 64 K-steps): per tile of each operand, bit s
  // set when some row of the tile has a nonzero byte in K-step s.  A step
  // that is zero in every row of either tile adds only zero products and is
  // skipped.
  const uint64_t* kmaskA;
  const uint64_t* kmaskB;
};

// Candidate pass over units of (R block, S stage) (stream.hip).
struct StreamParams {
  CandParams c;
  int64_t npad_r;        // rows of the R operand copy
  int64_t units;
  int nst, nrb;          // stages of S, blocks of R
  int stages_per_block;  // self-join: block rb starts at stage rb * stages_per_block
  int wr;                // waves along R (8 / wr along S)
  uint32_t first_row;    // R's number of the first row (band mode)
  // max mode: a sample of S in strips of four octets (8 rows each), nslots
  // slots of slot_strips strips; the largest P~ per row, slot and lane quarter
  // go to gmax[(4 slot + quarter) * nR + row] (order keys).  strips = nslots *
  // slot_strips; step: octets of S per octet of the sample, in 2^-32.
  int stride, nslots, slot_strips, strips;
  uint32_t dv_slot_m, dv_slot_s1, dv_slot_s2;  // division by slot_strips
  uint64_t step;
  uint32_t* gmax;
};

// eps-join recheck (recheck.hip).
struct RecheckParams {
  const float* R; int64_t ldr;
  const float* S; int64_t lds;
  int d;
  const uint2* cand; const unsigned long long* ccount; int64_t ccap;
  const unsigned long long* seg;  // the parts' counters, or null: one list of *ccount
  const float* candp;   // P~ of each candidate, or null
  const int* pexR;      // per R row: the candidate pass computed P~ exactly
  const double* nrm2R;  // |a|^2 per R row (float64)
  const float* xnR; const int* mlR;
  const float* xnS; const int* mlS;
  double T;
  const double* Trow;  // per-row thresholds (device) or null for T
  int bj;  // bits of j in the output key
  unsigned long long* keys; float* dist; unsigned long long* ocount;
  unsigned long long* nties;
  uint32_t* rowcnt;  // pairs written per row of R (zero before)
  // index-pruned join: candidates are rows of the permuted operand copies;
  // permR / permS give each one's row in R / S (null: no permutation), and
  // swap orders a self-join's pair as (min, max)
  const uint32_t* permR; const uint32_t* permS;
  int swap;
};

// top-k exact selection (recheck.hip).
struct SelectParams {
  const float* R; int64_t ldr;
  const float* S; int64_t lds;
  int d; int64_t nR;
  uint2* band; const int* bcount; int P; int cap; int k;
  const float* marg;
  const double* nrm2R;  // |a|^2 per R row (float64)
  const float* xnR; const int* mlR;
  const RelStats* sS;  // S maxima: xnorm_max, mlsb_min
  uint32_t* out_j; float* out_dist;
  SelectCount* counts; int* too_many;
  const int* gate;  // nonzero: invalid input, every row is written as padding
  // per row (nullable): rstate 1 once a selection over memory has replaced
  // the row's band P~ by float32 d2; wide 1 when the row had more near-tie
  // contenders than the selection holds (the wide selection takes it)
  int* rstate;
  int* wide;
};

}  // namespace dl
