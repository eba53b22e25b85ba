// recheck.hip -- exact decisions for the candidates of the matrix-core pass.
//
// Every candidate pair gets d2_32 = sum_k (a_k - b_k)^2 in float32 (direct
// form, from the float32 rows).  Its distance to the canonical float64 value
// d2_64 is at most beta = 2 gamma_{d+2} d2_32 + (d+2) 2^-148 +
// (d+4) 2^-52 (|a| + |b|)^2, and beta = 0 when both rows lie on a binary grid
// fine enough that every operation is exact (lowest-set-bit certificate).
//   eps-join: in if d2_32 + beta <= T, out if d2_32 - beta > T, otherwise a
//             boundary tie, decided by d2_64 <= T in float64.
//   top-k:    entries whose [d2_32 - beta, d2_32 + beta] overlaps another
//             contender's interval are ordered by d2_64; the rest are ordered
//             by d2_32, which cannot disagree with d2_64 for them.
// d2_64 is the canonical definition (subtract, square, add in increasing k,
// each rounded separately), so every decision equals the float64 reference.
//
// Paper: Nested Loop Join semantics (section "Query Processing") with the
// Euclidean threshold predicate (section "Derived Data") and the closest-image
// query q1 (section "Queries").
#include <type_traits>

#include "join_params.hpp"

namespace dl {

__device__ inline int wave_sumi(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Direct-form bound and exactness certificate (see file comment).
__device__ inline bool exact32(int mlsb, double xsum) {
  // x rows on the grid 2^m: differences are multiples of 2^m below
  // 2^(m+12) <= 2^(m+24) and squares / sums multiples of 2^(2m) below
  // 2^(2m+24): all exact in float32 while 2m >= -126 (no subnormals).
  if (mlsb >= kLsbNone) return true;  // both rows zero
  return 2 * mlsb >= -126 && xsum * xsum <= ldexp(1.0, 2 * mlsb + 24);
}
__device__ inline double beta32(double d2, int d, double xsum) {
  return 2.0 * gamma_n((double)d + 2.0, 0x1p-24) * d2 + ((double)d + 2.0) * 0x1p-148 +
         ((double)d + 4.0) * 0x1p-52 * xsum * xsum;
}

// float32 direct-form d2 of rows a and b, summed by one lane in increasing
// k (any order stays within the bound beta).  vec4: both rows 16-byte
// aligned.
__device__ inline float lane_d2(const float* a, const float* b, int d, bool vec4) {
  float acc = 0.0f;
  int q = 0;
  if (vec4) {
    // unrolled so that several row loads are in flight per lane; the sum is
    // still one chain in index order
#pragma unroll 8
    for (; q + 4 <= d; q += 4) {
      const float4 x = *reinterpret_cast<const float4*>(a + q);
      const float4 y = *reinterpret_cast<const float4*>(b + q);
      float u = x.x - y.x;
      acc = fmaf(u, u, acc);
      u = x.y - y.y;
      acc = fmaf(u, u, acc);
      u = x.z - y.z;
      acc = fmaf(u, u, acc);
      u = x.w - y.w;
      acc = fmaf(u, u, acc);
    }
  }
  for (; q < d; ++q) {
    const float u = a[q] - b[q];
    acc = fmaf(u, u, acc);
  }
  return acc;
}

// Sum over a group of kPairLanes neighbouring lanes, the same in each (a fixed
// order).
template <int kCtrl>
__device__ inline float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}
template <int kPairLanes>
__device__ inline float group_sum(float v) {
  static_assert(kPairLanes == 2 || kPairLanes == 4 || kPairLanes == 8, "lane exchanges below");
  v = dpp_add<0xb1>(v);                               // lanes 1 0 3 2 of each four
  if constexpr (kPairLanes >= 4) v = dpp_add<0x4e>(v);  // lanes 2 3 0 1
  if constexpr (kPairLanes >= 8) v = dpp_add<0x141>(v); // each eight reversed: the other four's sum
  return v;
}

// float32 direct-form d2 of kN row pairs (a[u], b[u]) by the lanes of a group
// (sub = the lane's place in it): each lane sums four consecutive elements of
// every 4 kPairLanes in increasing k (vec4: with 16-byte loads, the rows being
// aligned), then the lanes' sums are added.  The value depends on the pair
// alone.
template <int kPairLanes, int kN>
__device__ inline void group_d2(const float* const (&a)[kN], const float* const (&b)[kN], int d, bool vec4, int sub,
                                float (&out)[kN]) {
  float acc[kN];
#pragma unroll
  for (int u = 0; u < kN; ++u) acc[u] = 0.0f;
  const int d4 = d & ~3;
  auto add = [&](int u, float x, float y) {
    const float t = x - y;
    acc[u] = fmaf(t, t, acc[u]);
  };
  if (vec4) {
#pragma unroll 4
    for (int q = 4 * sub; q < d4; q += 4 * kPairLanes) {
#pragma unroll
      for (int u = 0; u < kN; ++u) {
        const float4 x = *reinterpret_cast<const float4*>(a[u] + q);
        const float4 y = *reinterpret_cast<const float4*>(b[u] + q);
        add(u, x.x, y.x);
        add(u, x.y, y.y);
        add(u, x.z, y.z);
        add(u, x.w, y.w);
      }
    }
  } else {
#pragma unroll 2
    for (int q = 4 * sub; q < d4; q += 4 * kPairLanes) {
#pragma unroll
      for (int u = 0; u < kN; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) add(u, a[u][q + e], b[u][q + e]);
    }
  }
#pragma unroll 1
  for (int q = d4 + sub; q < d; q += kPairLanes) {  // up to three elements past the last four
#pragma unroll
    for (int u = 0; u < kN; ++u) add(u, a[u][q], b[u][q]);
  }
#pragma unroll
  for (int u = 0; u < kN; ++u) out[u] = group_sum<kPairLanes>(acc[u]);
}

// ------------------------------------------------------------ eps recheck

// A wave takes 64 candidates at a time, one per lane; each four lanes compute
// the float32 distances of their four candidates in turn, then the wave
// classifies the 64 lane-parallel.  The confirmed ones of a workgroup's four
// waves, one or kRecheckChunks such batches each, are appended with one atomic
// (one counter serves the whole grid: at about 10 ns apiece, an atomic per
// wave and batch was most of the time for 0.5M candidates).  A candidate whose
// P~ the matrix-core pass computed exactly (pexR) and whose float32 form is
// exact (the lowest-set-bit certificate) needs no row reads: then
// d2 = |a|^2 - 2 P~ exactly (P~ = a.b - |b|^2/2), evaluated in float64
// without rounding.
//
// Bound by the gather of the rows.  Four lanes a candidate read 64 bytes of a
// row at a time; with fewer a load touches more rows, with more the
// per-candidate work (addresses, the sum across lanes) weighs more.
// Microseconds with two / four / eight lanes: 23k candidates, d = 64: 16.5 /
// 15.5 / 18.5; 0.58M, d = 100: 79 / 82 / 98; 5M, d = 128: 870 / 748 / 741;
// 195M, d = 100: 20,800 / 17,600 / 19,400; 0.1M, d = 512: 101 / 97 / 96.
constexpr int kRecheckChunks = 4;  // 64-candidate batches of a wave per output atomic, at most
constexpr int kRecheckLanes = 4;   // lanes that share a candidate's rows

__global__ __launch_bounds__(256) void recheck_eps_kernel(RecheckParams p) {
  __shared__ unsigned long long s_pos;
  __shared__ int s_in[4];
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63, sub = lane & (kRecheckLanes - 1);
  // the candidates of the list's part `lane` (one part without seg: its counter
  // shares a line with the output's, on which this kernel's atomics queue, so it
  // is read once a wave through the scalar cache; by the lanes, 0.5M candidates
  // take 170 us instead of 81)
  int64_t mine_n = 0;
  if (p.seg) {
    if (lane < kSegments)
      mine_n = min((int64_t)p.seg[lane * kSegWords], segment_end(p.ccap, lane) - segment_first(p.ccap, lane));
  } else {
    const int64_t all = min((int64_t)*p.ccount, p.ccap);
    if (lane == 0) mine_n = all;
  }
  auto part = [&](int s) {  // of part s
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)mine_n, s);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)mine_n >> 32), s);
    return (int64_t)((uint64_t)hi << 32 | lo);
  };
  int64_t n = 0, some = 0;
  for (int s = 0; s < kSegments; ++s) {
    const int64_t len = part(s);
    n += len;
    if (len) some = segment_first(p.ccap, s);
  }
  const uint64_t lt = __lanemask_lt();
  // 16-byte row loads when every row is aligned
  const bool vec4 = ((reinterpret_cast<uintptr_t>(p.S) | reinterpret_cast<uintptr_t>(p.R)) & 15) == 0 &&
                    ((p.lds | p.ldr) & 3) == 0;
  // Several batches per atomic once the workgroups they make fill the CUs
  // (0.5M candidates without row reads: 31 us with one batch, 20 with four),
  // and, where rows are gathered, fill them several times over (0.58M, d = 100:
  // 82 us with one, 99 with four).
  const bool gathers = !(p.candp && n > 0 && p.pexR[p.cand[some].x]);
  const int64_t fill = (int64_t)gridDim.x / 16 * 256 * kRecheckChunks;  // the grid is 16 per CU
  const int chunks = n >= fill * (gathers ? 8 : 1) ? kRecheckChunks : 1;
  const int64_t span = 64 * chunks;  // of a wave
  const int span_log = chunks == 1 ? 8 : 10;  // of a workgroup
  static_assert(kRecheckChunks == 4, "span_log");
  // (at most a span per part more than n fills; without candidates nothing is
  // looked for: 9.6 -> 5 us.  A return before the counters are read costs the
  // kernel 16 registers and its fifth wave per SIMD.)
  const int64_t spans = n ? (n >> span_log) + kSegments + 1 : 0;
  for (int64_t block = blockIdx.x; block < spans; block += gridDim.x) {
    // the part this workgroup's next spans lie in, and where
    int64_t block0 = -1, end = 0, left = block;
    for (int s = 0; s < kSegments; ++s) {
      const int64_t len = part(s), blocks = (len + span * 4 - 1) >> span_log;
      if (left < blocks) {
        block0 = segment_first(p.ccap, s) + left * span * 4;
        end = segment_first(p.ccap, s) + len;
        break;
      }
      left -= blocks;
    }
    if (block0 < 0) break;
    const int64_t base0 = block0 + wave * span;
    bool in[kRecheckChunks], tie[kRecheckChunks];
    float dist[kRecheckChunks];
    uint2 mine[kRecheckChunks];
#pragma unroll
    for (int c = 0; c < kRecheckChunks; ++c) {
      in[c] = false;
      tie[c] = false;
      dist[c] = 0.0f;
      mine[c] = make_uint2(0, 0);
      const int64_t base = base0 + c * 64;
      const int cnt = (int)max((int64_t)0, min((int64_t)64, end - base));
      if (c >= chunks || cnt == 0) continue;
      if (lane < cnt) mine[c] = p.cand[base + lane];
      float mys = 0.0f;
      bool quick = lane >= cnt;  // d2 from P~ (see above), or no candidate
      if (lane < cnt && p.candp && p.pexR[mine[c].x]) {
        const double xs = (double)p.xnR[mine[c].x] + (double)p.xnS[mine[c].y];
        if (exact32(min(p.mlR[mine[c].x], p.mlS[mine[c].y]), xs)) {
          quick = true;
          mys = (float)(p.nrm2R[mine[c].x] - 2.0 * (double)p.candp[base + lane]);
        }
      }
      // the candidate's rows of R and S (through the permutations of an
      // index-pruned join; statistics stay indexed by the operand row)
      const uint32_t oi = lane < cnt && p.permR ? p.permR[mine[c].x] : mine[c].x;
      const uint32_t oj = lane < cnt && p.permS ? p.permS[mine[c].y] : mine[c].y;
      if (__ballot(!quick)) {
        // (a quick or absent candidate's rows are read too: rows 0 if absent)
#pragma unroll 1
        for (int r = 0; r < kRecheckLanes; ++r) {
          const int l0 = (lane & ~(kRecheckLanes - 1)) + r;
          const float* const a[1] = {p.R + (int64_t)__shfl(oi, l0, 64) * p.ldr};
          const float* const b[1] = {p.S + (int64_t)__shfl(oj, l0, 64) * p.lds};
          float d2[1];
          group_d2<kRecheckLanes, 1>(a, b, p.d, vec4, sub, d2);
          if (!quick && sub == r) mys = d2[0];
        }
      }
      if (lane < cnt) {
        const double d2 = mys;
        const double xsum = (double)p.xnR[mine[c].x] + (double)p.xnS[mine[c].y];
        const bool ex = exact32(min(p.mlR[mine[c].x], p.mlS[mine[c].y]), xsum);
        const double bt = ex ? 0.0 : beta32(d2, p.d, xsum);
        const double hi = ex ? d2 : (d2 + bt) * (1.0 + 0x1p-50);
        const double lo = ex ? d2 : (d2 - bt) * (1.0 - 0x1p-50);
        const double T = p.Trow ? p.Trow[mine[c].x] : p.T;
        in[c] = hi <= T;
        dist[c] = sqrtf(mys);
        if (!in[c] && !(lo > T)) {  // boundary tie: the canonical float64 value decides
          tie[c] = true;
          const double d64 = canonical_d2(p.R + (int64_t)oi * p.ldr, p.S + (int64_t)oj * p.lds, p.d);
          in[c] = d64 <= T;
          dist[c] = (float)sqrt(d64);
        }
      }
      // the output names the pair by its rows of R and S (a self-join's
      // smaller row first)
      mine[c] = p.swap && oi > oj ? make_uint2(oj, oi) : make_uint2(oi, oj);
    }
    // one atomic for the whole span
    uint64_t mi[kRecheckChunks];
    int total = 0, nt = 0;
#pragma unroll
    for (int c = 0; c < kRecheckChunks; ++c) {
      mi[c] = __ballot(in[c]);
      total += __popcll(mi[c]);
      nt += __popcll(__ballot(tie[c]));
    }
    // one atomic for the workgroup's spans
    if (lane == 0) {
      s_in[wave] = total;
      if (nt) atomicAdd(p.nties, (unsigned long long)nt);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const int all = s_in[0] + s_in[1] + s_in[2] + s_in[3];
      s_pos = all ? atomicAdd(p.ocount, (unsigned long long)all) : 0ull;
    }
    __syncthreads();
    unsigned long long pos = s_pos;
    for (int w = 0; w < wave; ++w) pos += s_in[w];
#pragma unroll
    for (int c = 0; c < kRecheckChunks; ++c) {
      const unsigned long long at = pos + __popcll(mi[c] & lt);
      if (in[c] && at < (unsigned long long)p.ccap) {
        p.keys[at] = ((unsigned long long)mine[c].x << p.bj) | mine[c].y;
        p.dist[at] = dist[c];
      }
      // the row counts of the ordering, one atomic per run of equal rows
      if (mi[c]) {
        const uint32_t prev = __shfl_up(mine[c].x, 1, 64);
        const bool head = lane == 0 || prev != mine[c].x;
        const uint64_t later = __ballot(head) & ~lt & ~(1ull << lane);
        const uint64_t run = mi[c] & ~lt & (later ? (later & -later) - 1 : ~0ull);
        if (head && run) atomicAdd(p.rowcnt + mine[c].x, (uint32_t)__popcll(run));
      }
      pos += __popcll(mi[c]);
    }
    __syncthreads();
  }
}

hipError_t launch_recheck_eps(const RecheckParams& p, hipStream_t st, int cu_count) {
  hipLaunchKernelGGL(recheck_eps_kernel, dim3(cu_count * 16), dim3(256), 0, st, p);
  return hipGetLastError();
}

// ------------------------------------------------------------ pair d2
__global__ __launch_bounds__(256) void pair_d2_kernel(const float* R, int64_t ldr, int64_t nR, const float* S,
                                                      int64_t lds, int64_t nS, int d, const uint32_t* pi,
                                                      const uint32_t* pj, int64_t m, double* out, int* bad) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m; t += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t i = pi[t], j = pj[t];
    if (i >= nR || j >= nS) {
      out[t] = __longlong_as_double(0x7ff8000000000000ll);
      *reinterpret_cast<volatile int*>(bad) = 1;
      continue;
    }
    out[t] = canonical_d2(R + (int64_t)i * ldr, S + (int64_t)j * lds, d);
  }
}

hipError_t launch_pair_d2(const float* R, int64_t ldr, int64_t nR, const float* S, int64_t lds, int64_t nS, int d,
                          const uint32_t* pi, const uint32_t* pj, int64_t m, double* out, int* bad,
                          hipStream_t st, int cu_count) {
  if (m == 0) return hipSuccess;
  int64_t blocks = (m + 255) / 256;
  if (blocks > (int64_t)cu_count * 16) blocks = (int64_t)cu_count * 16;
  hipLaunchKernelGGL(pair_d2_kernel, dim3((unsigned)blocks), dim3(256), 0, st, R, ldr, nR, S, lds, nS, d, pi, pj, m,
                     out, bad);
  return hipGetLastError();
}

// ------------------------------------------------------------ top-k select
// Contenders per row held in LDS: kSelSmall for k <= 128 (smaller LDS
// buffers, more waves per CU), kSelLarge otherwise and whenever a row of
// the small launch had more (the host then runs the select again).
constexpr int kSelSmall = 256;
constexpr int kSelLarge = 512;
constexpr int kSelWaves = 4;
// Entries per lane held in registers: unions and refined bands of up to 512,
// or, for E4M3, 1,024 (its refined bands hold several hundred entries: 600 on
// average in the 20,000 x 1M, d = 256, top-32 join, where longer ones take the
// path over memory, 5.4 ms).
constexpr int kSelRegsNarrow = 8, kSelRegsWide = 16;
constexpr int kSelLanes = 8;  // lanes that share an entry's row

__device__ inline uint32_t ord_f(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Entries in a row's buffer (the streaming pass counts past its end).
__device__ inline int band_count(const SelectParams& p, int64_t at) { return min(p.bcount[at], p.cap); }

// One wave per row.  Counting over the row's band entries uses ballots
// (scalar popcounts, no shuffle chains); distances are computed by groups of
// eight lanes, four entries of a group at a time; the k nearest are emitted by
// rank, since the (key, j) pairs of a row are distinct.
//
// The band is refined before most distances are taken: the k entries of
// largest P~ give, exactly, an upper bound D of the row's k-th distance, and
// an entry whose P~ puts its d2 above D by more than the margin cannot be
// among the k nearest.  That bound has the margin once where the band's has it
// twice (P~_(k) may itself be off by it).  20,000 rows x 1M, d = 256, top-32,
// E4M3: bands of about 970 entries refined to about 600, the selection 2.7 ms
// (7.9 with every distance taken, one lane each), of which the rows' gather is
// 12 GB; 200,000 x 200,000, d = 128, top-10, bf16: 2.6 -> 0.9 ms.
//
// LDS per wave: first the staged entries (64 * kSelRegs of 8 bytes); then the
// list of entries whose distances are taken (j and float32 d2); then the
// contenders' j, float32 d2 and float64 key.
template <int kSelMax, int kSelRegs>
__global__ __launch_bounds__(64 * kSelWaves, kSelMax == kSelSmall && kSelRegs == kSelRegsNarrow ? 5 : 4) void topk_select_kernel(SelectParams p) {
  constexpr int kList = 64 * kSelRegs;
  constexpr int kBytes = 16 * kSelMax > 8 * kList ? 16 * kSelMax : 8 * kList;
  __shared__ __attribute__((aligned(16))) uint8_t s_buf[kSelWaves][kBytes];
  const int lane = threadIdx.x & 63, sub = lane & (kSelLanes - 1), grp = lane / kSelLanes;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = p.k;
  const uint64_t lt = __lanemask_lt();
  // The waves' band and tie counts go to one of kSelectCounts counters once a
  // workgroup: whichever wave is done last adds them.  (Atomics on one address
  // queue at tens of ns each: with a single counter, 200,000 rows spent 1.8 of
  // 2.0 ms on them.)
  __shared__ int s_cnt[3];  // band entries, ties, waves done
  if (threadIdx.x < 3) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  auto leave = [&](int nb, int nt) {
    if (lane) return;
    if (nb) atomicAdd(&s_cnt[0], nb);
    if (nt) atomicAdd(&s_cnt[1], nt);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    if (atomicAdd(&s_cnt[2], 1) != kSelWaves - 1) return;
    const int b = atomicAdd(&s_cnt[0], 0), t = atomicAdd(&s_cnt[1], 0);
    SelectCount* const c = p.counts + blockIdx.x % kSelectCounts;
    if (b) atomicAdd(&c->band, (unsigned long long)b);
    if (t) atomicAdd(&c->ties, (unsigned long long)t);
  };
  const int64_t i = (int64_t)blockIdx.x * kSelWaves + wave;
  if (i >= p.nR) return leave(0, 0);
  const float* a = p.R + i * p.ldr;
  if (p.gate && __builtin_amdgcn_readfirstlane(*p.gate)) {
    // invalid input: the candidate pass did no work and the band counts are
    // not set; the call reports the error, the rows hold padding
    for (int t = lane; t < k; t += 64) {
      p.out_j[i * k + t] = 0xffffffffu;
      p.out_dist[i * k + t] = INFINITY;
    }
    return leave(0, 0);
  }
  int total = 0;
  for (int s = 0; s < p.P; ++s) total += band_count(p, i * p.P + s);
  const double xsum = (double)p.xnR[i] + (double)p.sS->xnorm_max;
  const bool ex = exact32(min(p.mlR[i], p.sS->mlsb_min), xsum);
  const double c1 = ex ? 0.0 : 2.0 * gamma_n((double)p.d + 2.0, 0x1p-24);
  const double c0 = ex ? 0.0 : ((double)p.d + 2.0) * 0x1p-148 + ((double)p.d + 4.0) * 0x1p-52 * xsum * xsum;
  const bool vec4 = ((reinterpret_cast<uintptr_t>(p.S) | reinterpret_cast<uintptr_t>(a)) & 15) == 0 &&
                    (p.lds & 3) == 0;
  int nc = 0, nb = 0;
  // entries with d2 - beta > D_k + beta(D_k) cannot be among the k nearest
  auto cut_of = [&](uint64_t dk) {
    const double Dk = dk >= 0x7f800000ull ? INFINITY : (double)__uint_as_float((uint32_t)dk);
    return isinf(Dk) ? INFINITY : (Dk * (1.0 + c1) + 2.0 * c0) / (1.0 - c1) * (1.0 + 0x1p-50);
  };
  auto fence = [&]() {
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
  };
  // Stage into LDS, compactly, the union's entries with P~ >= floor (up to
  // kList of them); returns how many there are.
  uint2* st = reinterpret_cast<uint2*>(s_buf[wave]);
  // every entry of the union, 64 at a time (four loads in flight): f(entry, real)
  auto scan = [&](auto f) {
    for (int s = 0; s < p.P; ++s) {
      const uint2* e = p.band + (i * p.P + s) * (int64_t)p.cap;
      const int n = band_count(p, i * p.P + s);
      for (int base = 0; base < n; base += 256) {
        uint2 w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = base + 64 * u + lane;
          w[u] = t < n ? e[t] : make_uint2(0, 0);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (base + 64 * u < n) f(w[u], base + 64 * u + lane < n);
      }
    }
  };
  auto stage = [&](float floor) {
    int g = 0;
    scan([&](uint2 w, bool real) {
      const bool in = real && __uint_as_float(w.x) >= floor;
      const uint64_t m = __ballot(in);
      const int pos = g + __popcll(m & lt);
      if (in && pos < kList) st[pos] = w;
      g += __popcll(m);
    });
    fence();
    return g;
  };
  uint32_t key[kSelRegs], jv[kSelRegs];
  auto load_keys = [&](int cnt) {
#pragma unroll
    for (int r = 0; r < kSelRegs; ++r) {
      const int gi = r * 64 + lane;
      const uint2 v = gi < cnt ? st[gi] : make_uint2(0xff800000u, 0xffffffffu);
      key[r] = gi < cnt ? ord_f(__uint_as_float(v.x)) : 0u;
      jv[r] = v.y;
    }
  };
  // k-th largest of the first cnt keys (0 if there are fewer than k), by
  // ballot counts over registers
  auto kth_of = [&](int cnt) {
    if (cnt < k) return 0u;
    const int nr = (cnt + 63) / 64;
    // the bits all keys share need no counting
    uint32_t hi = 0, lo = 0xffffffffu;
#pragma unroll
    for (int r = 0; r < kSelRegs; ++r)
      if (r * 64 + lane < cnt) {
        hi = max(hi, key[r]);
        lo = min(lo, key[r]);
      }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
      lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
    }
    hi = __builtin_amdgcn_readfirstlane(hi);
    lo = __builtin_amdgcn_readfirstlane(lo);
    const int top = hi == lo ? 0 : 32 - __builtin_clz(hi ^ lo);  // bits that differ
    uint32_t t = top >= 32 ? 0u : hi & ~((1u << top) - 1u);
    auto count = [&](auto regs) {  // (the registers in use, so that a step has no branches)
      for (int b = top - 1; b >= 0; --b) {
        const uint32_t cand = t | (1u << b);
        int c = 0;
#pragma unroll
        for (int r = 0; r < decltype(regs)::value; ++r) c += __popcll(mask_ge(key[r], cand));
        if (c >= k) t = cand;
      }
    };
    if (nr <= 2) count(std::integral_constant<int, 2>{});
    else if (nr <= 4) count(std::integral_constant<int, 4>{});
    else if (nr <= 8) count(std::integral_constant<int, 8>{});
    else count(std::integral_constant<int, kSelRegs>{});
    return t;
  };
  // A row whose buffers an earlier selection over memory rewrote holds d2
  // (not P~) in its entries: it goes to the memory path with the band known.
  const bool in_d2 = p.rstate && __builtin_amdgcn_readfirstlane(p.rstate[i]);
  // (1) The k-th largest P~ of the union, v: from registers if the union fits
  // them; else the k-th largest of its first entries bounds v from below, and
  // the entries at or above that bound hold the k largest (a few rounds, while
  // they are too many).
  int kept = in_d2 ? kList + 1 : stage(-INFINITY);
  const bool whole = kept <= kList;  // st holds the whole union
  uint32_t v = 0;
  if (!in_d2) {
    load_keys(min(kept, kList));
    v = kth_of(min(kept, kList));
    for (int t = 0; t < 4 && kept > kList; ++t) {
      kept = stage(v ? key_float(v) : -INFINITY);
      load_keys(min(kept, kList));
      v = max(v, kth_of(min(kept, kList)));
    }
  }
  uint32_t* cj = reinterpret_cast<uint32_t*>(s_buf[wave]);
  float* cd = reinterpret_cast<float*>(s_buf[wave] + 4 * kList);
  // d2 of list entries lo .. hi - 1
  auto distances = [&](int lo, int hi) {
    fence();
    for (int base = lo; base < hi; base += 4 * kSelLanes) {
      const float* const ra[4] = {a, a, a, a};
      float d2[4];
      auto row = [&](int u) { return p.S + (int64_t)cj[min(base + 8 * u + grp, hi - 1)] * p.lds; };
      const float* const rb[4] = {row(0), row(1), row(2), row(3)};
      group_d2<kSelLanes, 4>(ra, rb, p.d, vec4, sub, d2);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (sub == u && base + 8 * u + grp < hi) cd[base + 8 * u + grp] = d2[u];
    }
    fence();
  };
  bool listed = kept <= kList, done = false;
  if (listed) {
    // (2) the band P~ >= bt, and the list: first the entries at or above v
    const float bt = v ? f32_down((double)key_float(v) - (double)p.marg[i]) : -INFINITY;
    fence();
    int nl = 0;
#pragma unroll
    for (int r = 0; r < kSelRegs; ++r)
      if (r * 64 < kept) {
        const uint64_t m = __ballot(r * 64 + lane < kept && key[r] >= v);
        if (m & (1ull << lane)) cj[nl + __popcll(m & lt)] = jv[r];
        nl += __popcll(m);
      }
    const int na = nl;
    float th = bt;
    if (v) {
      // their largest d2 bounds the k-th distance: D, rounded up
      distances(0, na);
      float dmax = 0.0f;
      for (int t = lane; t < na; t += 64) dmax = fmaxf(dmax, cd[t]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) dmax = fmaxf(dmax, __shfl_xor(dmax, o, 64));
      const double D = ((double)dmax * (1.0 + c1) + c0) * (1.0 + 0x1p-50), a2 = p.nrm2R[i], E = p.marg[i];
      th = fmaxf(th, f32_down(0.5 * (a2 - D - E) - 0x1p-50 * (fabs(a2) + D + E)));
    }
    // (3) then the others the refined band keeps
    if (whole) {
#pragma unroll
      for (int r = 0; r < kSelRegs; ++r)
        if (r * 64 < kept) {
          const bool real = r * 64 + lane < kept;
          const float P = key_float(key[r]);
          nb += __popcll(__ballot(real && P >= bt));
          const uint64_t m = __ballot(real && key[r] < v && P >= th);
          if (m & (1ull << lane)) cj[nl + __popcll(m & lt)] = jv[r];
          nl += __popcll(m);
        }
    } else {
      scan([&](uint2 w, bool real) {
        const float P = __uint_as_float(w.x);
        nb += __popcll(__ballot(real && P >= bt));
        const uint64_t m = __ballot(real && ord_f(P) < v && P >= th);
        const int pos = nl + __popcll(m & lt);
        if ((m & (1ull << lane)) && pos < kList) cj[pos] = w.y;
        nl += __popcll(m);
      });
    }
    listed = nl <= kList;  // (else the list is too long: over memory, below)
    if (listed) distances(v ? na : 0, nl);
    if (nl <= 64) {
      // (4) a list of at most 64, one entry a lane: each one's rank by d2
      // (non-negative floats order as integers).  With all d2 distinct and no
      // two contenders' intervals overlapping (which neighbours in rank would
      // show, the intervals growing with d2), the ranks are the answer.
      const bool real = lane < nl;
      const uint32_t db = real ? __float_as_uint(cd[lane]) : 0xffffffffu;
      const uint32_t j = real ? cj[lane] : 0u;
      int below = 0, upto = 0;
      for (int u = 0; u < nl; ++u) {
        const uint32_t o = __builtin_amdgcn_readlane(db, u);
        below += o < db;
        upto += o <= db;
      }
      const uint64_t at = __ballot(real && below < k && upto >= k);  // D_k's lanes
      const double cut = cut_of(at ? (uint64_t)__builtin_amdgcn_readlane(db, __builtin_ctzll(at)) : 0x7f800000ull);
      const float d2 = __uint_as_float(db);
      const bool keep = real && !isinf(d2) && (double)d2 <= cut;
      nc = __popcll(__ballot(keep));
      const bool dup = __ballot(real && upto != below + 1) != 0;
      fence();  // the list is in registers; the contenders take its place
      uint32_t* const oj = reinterpret_cast<uint32_t*>(s_buf[wave]);
      float* const od = reinterpret_cast<float*>(s_buf[wave] + 4 * kSelMax);
      const int slot = dup ? __popcll(__ballot(keep) & lt) : below;
      if (keep) {
        od[slot] = d2;
        oj[slot] = j;
      }
      fence();
      bool tie = dup;
      if (!dup && keep && slot + 1 < nc) {
        const double x = d2, y = od[slot + 1];
        tie = !((x + (c1 * x + c0)) * (1.0 + 0x1p-50) < (y - (c1 * y + c0)) * (1.0 - 0x1p-50));
      }
      if (!__ballot(tie)) {
        if (keep && slot < k) {
          p.out_j[i * k + slot] = j;
          p.out_dist[i * k + slot] = sqrtf(d2);
        }
        for (int r = nc + lane; r < k; r += 64) {
          p.out_j[i * k + r] = 0xffffffffu;
          p.out_dist[i * k + r] = INFINITY;
        }
        done = true;
      }
    } else if (listed) {
      // a longer list: D_k = k-th smallest d2 by counting (all-ones bits, which no count below includes, past the list)
      uint32_t d2b[kSelRegs];
#pragma unroll
      for (int r = 0; r < kSelRegs; ++r) {
        const bool real = r * 64 + lane < nl;
        d2b[r] = real ? __float_as_uint(cd[r * 64 + lane]) : 0xffffffffu;
        jv[r] = real ? cj[r * 64 + lane] : 0u;
      }
      const int nr = (nl + 63) / 64;  // register slots in use (wave-uniform)
      uint64_t dk = 0;
      for (int b = 31; b >= 0; --b) {
        const uint64_t lim = dk + (1ull << b);
        int c = 0;
#pragma unroll
        for (int r = 0; r < kSelRegs; ++r)
          if (r < nr) c += __popcll(mask_lt((uint64_t)d2b[r], lim));
        if (c < k) dk = lim;
      }
      const double cut = cut_of(dk);
      fence();  // the list is in registers; the contenders take its place
      uint32_t* const oj = reinterpret_cast<uint32_t*>(s_buf[wave]);
      float* const od = reinterpret_cast<float*>(s_buf[wave] + 4 * kSelMax);
#pragma unroll
      for (int r = 0; r < kSelRegs; ++r) {
        if (r < nr) {
          const float d2 = __uint_as_float(d2b[r]);
          const bool keep = r * 64 + lane < nl && !isinf(d2) && (double)d2 <= cut;
          const uint64_t m = __ballot(keep);
          const int pos = nc + __popcll(m & lt);
          if (keep && pos < kSelMax) {
            od[pos] = d2;
            oj[pos] = jv[r];
          }
          nc += __popcll(m);
        }
      }
    } else {
      nb = -1;  // (the thresholds found are left in LDS)
      fence();
      if (lane == 0) {
        reinterpret_cast<float*>(s_buf[wave])[0] = bt;
        reinterpret_cast<float*>(s_buf[wave])[1] = th;
      }
      fence();
    }
  }
  cd = reinterpret_cast<float*>(s_buf[wave] + 4 * kSelMax);
  double* ck = reinterpret_cast<double*>(s_buf[wave] + 8 * kSelMax);
  if (!listed) {
    // a union or list too large for the above: the same steps over the split
    // buffers in memory, with the band refined where its k-th largest P~ was found
    auto count = [&](auto pred) {
      int c = 0;
      for (int s = 0; s < p.P; ++s) {
        const uint2* e = p.band + (i * p.P + s) * (int64_t)p.cap;
        const int n = band_count(p, i * p.P + s);
        for (int base = 0; base < n; base += 64) {
          const int t = base + lane;
          c += __popcll(__ballot(t < n && pred(e[t].x)));
        }
      }
      return c;
    };
    if (!in_d2) {
      float bt = -INFINITY, th = -INFINITY;
      if (nb < 0) {
        bt = reinterpret_cast<const float*>(s_buf[wave])[0];
        th = reinterpret_cast<const float*>(s_buf[wave])[1];
        nb = 0;
      } else if (total >= k) {
        uint32_t t = 0;
        for (int b = 31; b >= 0; --b) {
          const uint32_t cand = t | (1u << b);
          if (count([&](uint32_t w) { return ord_f(__uint_as_float(w)) >= cand; }) >= k) t = cand;
        }
        const float pk = __uint_as_float((t & 0x80000000u) ? (t & 0x7fffffffu) : ~t);
        bt = th = f32_down((double)pk - (double)p.marg[i]);
      }
      // each entry's P~ is replaced by its float32 d2 (+inf outside the band, and
      // what no d2 reaches in the band but not the refined one): the steps below,
      // and any later selection of the row, read that
      for (int s = 0; s < p.P; ++s) {
        uint2* e = p.band + (i * p.P + s) * (int64_t)p.cap;
        const int n = band_count(p, i * p.P + s);
        for (int base = 0; base < n; base += 64) {
          const int t = base + lane;
          const uint2 v = t < n ? e[t] : make_uint2(0, 0);
          const bool inband = t < n && __uint_as_float(v.x) >= bt;
          float d2 = inband ? 0x1.fffffep127f : INFINITY;
          if (inband && __uint_as_float(v.x) >= th) d2 = lane_d2(a, p.S + (int64_t)v.y * p.lds, p.d, vec4);
          if (t < n) e[t].x = __float_as_uint(d2);
          nb += __popcll(__ballot(inband));
        }
      }
      __builtin_amdgcn_s_waitcnt(0);
      if (p.rstate && lane == 0) p.rstate[i] = 1;
    } else {
      nb = count([](uint32_t w) { return w < 0x7f800000u; });
    }
    uint64_t dk = 0;
    for (int b = 31; b >= 0; --b) {
      const uint64_t lim = dk + (1ull << b);
      if (count([&](uint32_t w) { return (uint64_t)w < lim; }) < k) dk = lim;
    }
    const double cut = cut_of(dk);
    for (int s = 0; s < p.P; ++s) {
      const uint2* e = p.band + (i * p.P + s) * (int64_t)p.cap;
      const int n = band_count(p, i * p.P + s);
      for (int base = 0; base < n; base += 64) {
        const int t = base + lane;
        uint2 v = make_uint2(0x7f800000u, 0);
        if (t < n) v = e[t];
        const float d2 = __uint_as_float(v.x);
        const bool keep = t < n && !isinf(d2) && (double)d2 <= cut;
        const uint64_t m = __ballot(keep);
        const int pos = nc + __popcll(m & lt);
        if (keep && pos < kSelMax) {
          cd[pos] = d2;
          cj[pos] = v.y;
        }
        nc += __popcll(m);
      }
    }
  }
  if (done) return leave(nb, 0);
  if (nc > kSelMax) {
    if (lane == 0) {
      atomicOr(p.too_many, 1);
      if (p.wide) p.wide[i] = 1;
    }
    for (int t = lane; t < k; t += 64) {
      p.out_j[i * k + t] = 0xffffffffu;
      p.out_dist[i * k + t] = INFINITY;
    }
    return leave(nb, 0);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();

  // (5) overlapping intervals -> float64 keys
  int nt = 0;
  for (int t = lane; t < nc; t += 64) {
    const double dx = cd[t];
    const double lox = dx - (c1 * dx + c0), hix = dx + (c1 * dx + c0);
    bool tie = false;
    for (int u = 0; u < nc && !tie; ++u) {
      if (u == t) continue;
      const double dy = cd[u];
      const double loy = dy - (c1 * dy + c0), hiy = dy + (c1 * dy + c0);
      tie = !(hix * (1.0 + 0x1p-50) < loy * (1.0 - 0x1p-50) || hiy * (1.0 + 0x1p-50) < lox * (1.0 - 0x1p-50));
    }
    double key = dx;
    if (tie && !ex) {
      key = canonical_d2(a, p.S + (int64_t)cj[t] * p.lds, p.d);
      ++nt;
    }
    ck[t] = key;
  }
  nt = wave_sumi(nt);
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();

  // (6) each contender's rank in (key, j) order is its output slot
  for (int t = lane; t < nc; t += 64) {
    const double kt = ck[t];
    const uint32_t jt = cj[t];
    int rank = 0;
    for (int u = 0; u < nc; ++u) {
      const double ku = ck[u];
      rank += ku < kt || (ku == kt && cj[u] < jt);
    }
    if (rank < k) {
      p.out_j[i * k + rank] = jt;
      p.out_dist[i * k + rank] = kt == (double)cd[t] ? sqrtf(cd[t]) : (float)sqrt(kt);
    }
  }
  for (int r = nc + lane; r < k; r += 64) {
    p.out_j[i * k + r] = 0xffffffffu;
    p.out_dist[i * k + r] = INFINITY;
  }
  leave(nb, nt);
}

// Rows with more near-tie contenders than the selection's LDS holds (p.wide
// set): one wave per such row works on the row's band buffers in memory.
// Every contender (float32 d2 within the cut) gets its float64 canonical key,
// recomputed wherever it is needed instead of stored; the k-th smallest
// (key, j) is found bit by bit over the 96-bit pair (64 key bits, then 32
// index bits), counting the contenders below each trial value, and the k
// contenders at or below it are ranked in LDS.  Slow (96 counting passes,
// each d float64 operations per contender) but bounded by the row's band,
// so a row of many exact duplicates still gets its exact answer.
__global__ __launch_bounds__(64 * kSelWaves) void topk_select_wide_kernel(SelectParams p) {
  __shared__ double s_key[kSelWaves][256];
  __shared__ uint32_t s_j[kSelWaves][256];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = (int64_t)blockIdx.x * kSelWaves + wave;
  if (i >= p.nR || !__builtin_amdgcn_readfirstlane(p.wide[i])) return;
  const float* a = p.R + i * p.ldr;
  const int k = p.k;
  const uint64_t lt = __lanemask_lt();
  const bool vec4 = ((reinterpret_cast<uintptr_t>(p.S) | reinterpret_cast<uintptr_t>(a)) & 15) == 0 &&
                    (p.lds & 3) == 0;
  int total = 0;
  for (int s = 0; s < p.P; ++s) total += band_count(p, i * p.P + s);
  auto count = [&](auto pred) {
    int c = 0;
    for (int s = 0; s < p.P; ++s) {
      const uint2* e = p.band + (i * p.P + s) * (int64_t)p.cap;
      const int n = band_count(p, i * p.P + s);
      for (int base = 0; base < n; base += 64) {
        const int t = base + lane;
        c += __popcll(__ballot(t < n && pred(e[t])));
      }
    }
    return c;
  };
  // (1) the row's entries as float32 d2 (+inf outside the band)
  if (!__builtin_amdgcn_readfirstlane(p.rstate[i])) {
    float bt = -INFINITY;
    if (total >= k) {
      uint32_t t = 0;
      for (int b = 31; b >= 0; --b) {
        const uint32_t cand = t | (1u << b);
        if (count([&](uint2 v) { return ord_f(__uint_as_float(v.x)) >= cand; }) >= k) t = cand;
      }
      const float pk = __uint_as_float((t & 0x80000000u) ? (t & 0x7fffffffu) : ~t);
      bt = f32_down((double)pk - (double)p.marg[i]);
    }
    for (int s = 0; s < p.P; ++s) {
      uint2* e = p.band + (i * p.P + s) * (int64_t)p.cap;
      const int n = band_count(p, i * p.P + s);
      for (int base = 0; base < n; base += 64) {
        const int t = base + lane;
        const uint2 v = t < n ? e[t] : make_uint2(0, 0);
        float d2 = INFINITY;
        if (t < n && __uint_as_float(v.x) >= bt) d2 = lane_d2(a, p.S + (int64_t)v.y * p.lds, p.d, vec4);
        if (t < n) e[t].x = __float_as_uint(d2);
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    if (lane == 0) p.rstate[i] = 1;
  }
  // (2) D_k and the cut, as in the selection
  const double xsum = (double)p.xnR[i] + (double)p.sS->xnorm_max;
  const bool ex = exact32(min(p.mlR[i], p.sS->mlsb_min), xsum);
  const double c1 = ex ? 0.0 : 2.0 * gamma_n((double)p.d + 2.0, 0x1p-24);
  const double c0 = ex ? 0.0 : ((double)p.d + 2.0) * 0x1p-148 + ((double)p.d + 4.0) * 0x1p-52 * xsum * xsum;
  uint64_t dk = 0;
  for (int b = 31; b >= 0; --b) {
    const uint64_t lim = dk + (1ull << b);
    if (count([&](uint2 v) { return (uint64_t)v.x < lim; }) < k) dk = lim;
  }
  const double Dk = dk >= 0x7f800000ull ? INFINITY : (double)__uint_as_float((uint32_t)dk);
  const double cut = isinf(Dk) ? INFINITY : (Dk * (1.0 + c1) + 2.0 * c0) / (1.0 - c1) * (1.0 + 0x1p-50);
  auto contender = [&](uint2 v) {
    const float d2 = __uint_as_float(v.x);
    return !isinf(d2) && (double)d2 <= cut;
  };
  auto key_of = [&](uint2 v) { return canonical_d2(a, p.S + (int64_t)v.y * p.lds, p.d); };
  const int nc = count(contender);
  const int want = nc < k ? nc : k;
  // (3) the want-th smallest (key, j): largest (K, J) with fewer than want
  // contenders below it
  uint64_t K = 0;
  uint32_t J = 0;
  if (want > 0) {
    for (int b = 63; b >= 0; --b) {
      const uint64_t cand = K | (1ull << b);
      const int c = count([&](uint2 v) {
        return contender(v) && (uint64_t)__double_as_longlong(key_of(v)) < cand;
      });
      if (c < want) K = cand;
    }
    for (int b = 31; b >= 0; --b) {
      const uint32_t cand = J | (1u << b);
      const int c = count([&](uint2 v) {
        if (!contender(v)) return false;
        const uint64_t kv = (uint64_t)__double_as_longlong(key_of(v));
        return kv < K || (kv == K && v.y < cand);
      });
      if (c < want) J = cand;
    }
  }
  // (4) the want contenders at or below (K, J) into LDS, then ranked
  int g = 0;
  for (int s = 0; s < p.P; ++s) {
    const uint2* e = p.band + (i * p.P + s) * (int64_t)p.cap;
    const int n = band_count(p, i * p.P + s);
    for (int base = 0; base < n; base += 64) {
      const int t = base + lane;
      const uint2 v = t < n ? e[t] : make_uint2(0x7f800000u, 0);
      double kd = 0.0;
      bool in = false;
      if (t < n && contender(v)) {
        kd = key_of(v);
        const uint64_t kv = (uint64_t)__double_as_longlong(kd);
        in = kv < K || (kv == K && v.y <= J);
      }
      const uint64_t m = __ballot(in);
      const int pos = g + __popcll(m & lt);
      if (in && pos < want) {
        s_key[wave][pos] = kd;
        s_j[wave][pos] = v.y;
      }
      g += __popcll(m);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
  for (int t = lane; t < want; t += 64) {
    const double kt = s_key[wave][t];
    const uint32_t jt = s_j[wave][t];
    int rank = 0;
    for (int u = 0; u < want; ++u) {
      const double ku = s_key[wave][u];
      rank += ku < kt || (ku == kt && s_j[wave][u] < jt);
    }
    p.out_j[i * k + rank] = jt;
    p.out_dist[i * k + rank] = (float)sqrt(kt);
  }
  for (int r = want + lane; r < k; r += 64) {
    p.out_j[i * k + r] = 0xffffffffu;
    p.out_dist[i * k + r] = INFINITY;
  }
  const int nt = want;
  if (lane == 0) {
    atomicAdd(&p.counts[blockIdx.x % kSelectCounts].ties, (unsigned long long)nt);
    p.wide[i] = 0;
  }
}

hipError_t launch_topk_select_wide(const SelectParams& p, hipStream_t st) {
  if (p.nR == 0 || !p.wide || !p.rstate) return hipSuccess;
  const dim3 grid((unsigned)((p.nR + kSelWaves - 1) / kSelWaves)), block(64 * kSelWaves);
  hipLaunchKernelGGL(topk_select_wide_kernel, grid, block, 0, st, p);
  return hipGetLastError();
}

// wide_band: E4M3 candidates (kSelRegsWide)
hipError_t launch_topk_select(const SelectParams& p, bool small, bool wide_band, hipStream_t st) {
  if (p.nR == 0) return hipSuccess;
  const dim3 grid((unsigned)((p.nR + kSelWaves - 1) / kSelWaves)), block(64 * kSelWaves);
  if (small && wide_band) hipLaunchKernelGGL((topk_select_kernel<kSelSmall, kSelRegsWide>), grid, block, 0, st, p);
  else if (small) hipLaunchKernelGGL((topk_select_kernel<kSelSmall, kSelRegsNarrow>), grid, block, 0, st, p);
  else if (wide_band) hipLaunchKernelGGL((topk_select_kernel<kSelLarge, kSelRegsWide>), grid, block, 0, st, p);
  else hipLaunchKernelGGL((topk_select_kernel<kSelLarge, kSelRegsNarrow>), grid, block, 0, st, p);
  return hipGetLastError();
}
bool topk_select_small(int k) { return k <= 128; }

}  // namespace dl
