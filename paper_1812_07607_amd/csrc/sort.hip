// sort.hip -- canonical (i, j) order for the eps-join output.
//
// The confirmed pairs (keys i << bj | j with a float distance) are bucketed
// by row with a count, an exclusive scan and an atomic placement, then each
// row's segment is ordered by j.  Deterministic: the output depends only on
// the set of pairs, not on the order the candidate kernel produced them in.
#include "join_params.hpp"

namespace dl {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanChunk = kScanThreads * kScanItems;  // 4096

// --------------------------------------------------------------- scan
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t* lds_w, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds_w[wave] = x;
  __syncthreads();
  const int nw = blockDim.x >> 6;
  uint32_t off = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    const uint32_t s = lds_w[w];
    if (w < wave) off += s;
    tot += s;
  }
  __syncthreads();
  total = tot;
  return off + x - v;
}

__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(const uint32_t* in, int64_t n, uint32_t* sums) {
  __shared__ uint32_t lw[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk;
  uint32_t s = 0;
  for (int t = 0; t < kScanItems; ++t) {
    const int64_t idx = base + (int64_t)t * kScanThreads + threadIdx.x;
    if (idx < n) s += in[idx];
  }
  uint32_t tot;
  block_exclusive_scan(s, lw, tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// single workgroup: exclusive scan of nb chunk sums in place (nb <= 2^20)
__global__ __launch_bounds__(1024) void scan_top_kernel(uint32_t* sums, int64_t nb) {
  __shared__ uint32_t lw[16];
  uint32_t carry = 0;
  for (int64_t base = 0; base < nb; base += 1024) {
    const int64_t idx = base + threadIdx.x;
    const uint32_t v = idx < nb ? sums[idx] : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(v, lw, tot);
    if (idx < nb) sums[idx] = carry + ex;
    carry += tot;
    __syncthreads();
  }
}

// Each thread owns kScanItems consecutive entries of the chunk.  What lies
// before the chunk: its entry of sums (scanned), the plain sums of the chunks
// before it (sums given), or their entries, added up by the workgroup.
__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(const uint32_t* in, int64_t n, const uint32_t* sums,
                                                                  bool scanned, uint32_t* out,
                                                                  const unsigned long long* some) {
  __shared__ uint32_t lw[kScanThreads / 64];
  if (some && *some == 0) return;
  uint32_t before = 0;
  if (scanned) {
    before = sums[blockIdx.x];
  } else if (!sums) {
    uint32_t x = 0;
    for (int c = 0; c < (int)blockIdx.x; ++c)
#pragma unroll
      for (int t = 0; t < kScanItems; ++t) x += in[c * kScanChunk + t * kScanThreads + threadIdx.x];
    block_exclusive_scan(x, lw, before);
  } else if (blockIdx.x > 0) {
    uint32_t x = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kScanThreads) x += sums[t];
    block_exclusive_scan(x, lw, before);
  }
  const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  uint32_t s = 0;
#pragma unroll
  for (int t = 0; t < kScanItems; ++t) {
    v[t] = base + t < n ? in[base + t] : 0u;
    s += v[t];
  }
  uint32_t tot;
  uint32_t run = block_exclusive_scan(s, lw, tot) + before;
#pragma unroll
  for (int t = 0; t < kScanItems; ++t) {
    if (base + t < n) out[base + t] = run;
    run += v[t];
  }
}

int64_t scan_scratch_words(int64_t n) { return (n + kScanChunk - 1) / kScanChunk; }

// One launch for up to kScanSelf chunks, whose entries a workgroup adds up for
// itself, and two up to kScanFlat, whose sums it adds up (a few loads a thread,
// where a launch costs about 5 us: 5,000 rows 10.8 us in two, 7.0 in one); three
// beyond, where that would grow quadratically.  some (nullable): a scan of one
// launch does nothing where it holds zero (the wait for it costs each launch of a
// longer one a microsecond).
constexpr int64_t kScanSelf = 4, kScanFlat = 4096;
hipError_t launch_exclusive_scan(const uint32_t* in, int64_t n, uint32_t* out, uint32_t* sums, hipStream_t st,
                                 const unsigned long long* some) {
  if (n == 0) return hipSuccess;
  const int64_t nb = (n + kScanChunk - 1) / kScanChunk;
  const bool one = nb <= kScanSelf;
  if (!one) hipLaunchKernelGGL(scan_reduce_kernel, dim3((unsigned)nb), dim3(kScanThreads), 0, st, in, n, sums);
  if (nb > kScanFlat) hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(1024), 0, st, sums, nb);
  hipLaunchKernelGGL(scan_apply_kernel, dim3((unsigned)nb), dim3(kScanThreads), 0, st, in, n, one ? nullptr : sums,
                     nb > kScanFlat, out, one ? some : nullptr);
  return hipGetLastError();
}

// --------------------------------------------------------------- rows
// Canonical (i, j) order by rows: the recheck has counted the pairs of each
// row; scan the counts into row offsets, place every pair in its row's segment (in any
// order), then order each segment by j, one wave per row.  A pair's output
// slot is the number of the row's pairs with a smaller j (the (i, j) pairs
// are distinct, so the result does not depend on the order of placement):
// rows of at most 64 pairs rank in registers, rows of at most 256 against
// their j values staged in LDS; longer rows set one bit per pair in an LDS
// bitmap over a window of j, take a prefix count of the bitmap words, and
// read each pair's rank from it, window by window (windows that hold no
// pair are skipped), unless its pairs are few for the range of j they span:
// then buckets of j, ranked within a bucket.  The number of
// pairs is read on the device: the launches are queued before the host knows it.
__device__ inline int64_t ordered_pairs(const Counters* c, int64_t cap) {
  return (int64_t)c->cand > cap ? 0 : (int64_t)c->out;  // none if candidates were lost: the call fails
}

// The confirmed pairs arrive in runs of equal i (the candidate pass emits
// them tile by tile), so the row counters take one atomic per run of equal
// rows inside a wave rather than one per pair.  For the pair of lane l:
// head = the lane that starts its run, len = the run's length.
struct RowRun {
  uint64_t i;
  int head, len;
  bool valid;
};

__device__ inline RowRun row_run(const unsigned long long* keys, int64_t t, int64_t m, int bj) {
  const int lane = threadIdx.x & 63;
  RowRun r;
  r.valid = t < m;
  r.i = r.valid ? keys[t] >> bj : ~0ull;
  const uint64_t prev = __shfl_up(r.i, 1, 64);
  const bool start = r.valid && (lane == 0 || prev != r.i);
  const uint64_t heads = __ballot(start);
  const uint64_t ends = heads | ~__ballot(r.valid);  // a run also ends at the first lane past m
  r.head = 63 - __clzll(heads & (~0ull >> (63 - lane)));
  const uint64_t after = ends & ~(~0ull >> (63 - r.head));
  r.len = (after ? __ffsll((long long)after) - 1 : 64) - r.head;
  return r;
}

// cnt holds each row's pair count on entry and zero on exit: each run takes
// len of its row's slots by one atomic decrement.
__global__ void place_rows_kernel(const unsigned long long* __restrict__ keys, const float* __restrict__ vals,
                                  const Counters* __restrict__ c, int64_t cap, int bj,
                                  const uint32_t* __restrict__ off, uint32_t* __restrict__ cnt,
                                  unsigned long long* __restrict__ pk, float* __restrict__ pv) {
  const int64_t m = ordered_pairs(c, cap);
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63); t0 < m; t0 += stride) {
    const int64_t t = t0 + lane;
    const RowRun r = row_run(keys, t, m, bj);
    uint32_t first = 0;
    if (r.valid && r.head == lane) first = off[r.i] + atomicSub(&cnt[r.i], (uint32_t)r.len) - (uint32_t)r.len;
    first = __shfl(first, r.head, 64);
    if (r.valid) {
      const uint32_t pos = first + (uint32_t)(lane - r.head);
      pk[pos] = keys[t];
      pv[pos] = vals[t];
    }
  }
}

constexpr int kRowWaves = 4;
constexpr int kWinWords = 1024;             // bitmap words per wave
constexpr int kWinBits = 32 * kWinWords;    // j values per window
constexpr int kWordsPerLane = kWinWords / 64;
constexpr int kQuadRow = 256;               // longest row ranked pair against pair
constexpr int kOrderGroup = 8;              // lanes per short row, where rows are many
constexpr int kOrderFill = 64;              // ... (this many per CU)
constexpr uint32_t kFewWindows = 4;         // windows of j that cost no more than buckets
constexpr uint32_t kBucketMost = 64;        // pairs of a bucket, ranked pair against pair

__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
}

// Orders one row's pairs [b, e) by a whole wave (bm, pre: kWinWords of LDS).
__device__ inline void order_row(const unsigned long long* __restrict__ pk, const float* __restrict__ pv, int64_t i,
                                 int64_t b, int64_t e, uint32_t* __restrict__ js, int bj, int64_t w,
                                 uint32_t* __restrict__ oi, uint32_t* __restrict__ oj, float* __restrict__ od,
                                 uint32_t* bm, uint32_t* pre) {
  const int lane = threadIdx.x & 63;
  const unsigned long long mask = (1ull << bj) - 1;
  auto emit = [&](int64_t at, int64_t t, uint32_t j) {
    if (at < w) {
      oi[at] = (uint32_t)i;
      oj[at] = j;
      od[at] = pv[t];
    }
  };
  if (e - b <= 64) {
    const int64_t t = b + lane;
    const uint32_t j = t < e ? (uint32_t)(pk[t] & mask) : 0xffffffffu;
    int rank = 0;
    for (int u = 0; u < (int)(e - b); ++u) rank += __shfl(j, u, 64) < j;
    if (t < e) emit(b + rank, t, j);
    return;
  }
  if (e - b <= kQuadRow) {
    // rank against the row's j values staged in LDS (broadcast reads)
    for (int64_t t = b + lane; t < e; t += 64) bm[t - b] = (uint32_t)(pk[t] & mask);
    wave_lds_sync();
    const int len = (int)(e - b);
    uint32_t jq[kQuadRow / 64];
    int rk[kQuadRow / 64];
#pragma unroll
    for (int q = 0; q < kQuadRow / 64; ++q) {
      jq[q] = lane + 64 * q < len ? bm[lane + 64 * q] : 0u;
      rk[q] = 0;
    }
    for (int u = 0; u < len; ++u) {
      const uint32_t v = bm[u];
#pragma unroll
      for (int q = 0; q < kQuadRow / 64; ++q) rk[q] += v < jq[q];
    }
#pragma unroll
    for (int q = 0; q < kQuadRow / 64; ++q)
      if (lane + 64 * q < len) emit(b + rk[q], b + lane + 64 * q, jq[q]);
    return;
  }
  uint32_t jlo = 0xffffffffu, jhi = 0;
  for (int64_t t = b + lane; t < e; t += 64) {
    const uint32_t j = (uint32_t)(pk[t] & mask);
    jlo = j < jlo ? j : jlo;
    jhi = j > jhi ? j : jhi;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const uint32_t a = __shfl_xor(jlo, o, 64), z = __shfl_xor(jhi, o, 64);
    jlo = a < jlo ? a : jlo;
    jhi = z > jhi ? z : jhi;
  }
  // Few pairs over a wide range of j: 1,024 buckets of equal width instead of
  // windows (900 queries of a few hundred pairs each among 2M rows: a window
  // holds 32,768 j, so a row walked 61 of them; the ordering 196 -> 30 us).
  if (jhi - jlo >= kFewWindows * kWinBits) {
    const int sh = 22 - __clz(jhi - jlo);  // (jhi - jlo) >> sh < kWinWords
    const int len = (int)(e - b);
#pragma unroll
    for (int q = 0; q < kWordsPerLane; ++q) bm[lane + 64 * q] = 0;
    wave_lds_sync();
    for (int t = lane; t < len; t += 64) atomicAdd(&bm[((uint32_t)(pk[b + t] & mask) - jlo) >> sh], 1u);
    wave_lds_sync();
    uint32_t c[kWordsPerLane], run = 0, most = 0;
#pragma unroll
    for (int q = 0; q < kWordsPerLane; ++q) {
      const uint32_t n = bm[lane * kWordsPerLane + q];
      most = n > most ? n : most;
      c[q] = run;
      run += n;
    }
    uint32_t x = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (!__ballot(most > kBucketMost)) {
#pragma unroll
      for (int q = 0; q < kWordsPerLane; ++q) bm[lane * kWordsPerLane + q] = x - run + c[q];
      wave_lds_sync();
      // the j values bucket by bucket (in any order within one), in LDS or
      // behind it in memory; bm ends up holding the buckets' ends
      const bool fits = len <= kWinWords;
      for (int t = lane; t < len; t += 64) {
        const uint32_t j = (uint32_t)(pk[b + t] & mask);
        const uint32_t at = atomicAdd(&bm[(j - jlo) >> sh], 1u);
        if (fits) pre[at] = j;
        else js[b + at] = j;
      }
      __threadfence_block();
      wave_lds_sync();
      for (int t = lane; t < len; t += 64) {
        const uint32_t j = (uint32_t)(pk[b + t] & mask);
        const uint32_t k = (j - jlo) >> sh;
        const uint32_t u0 = k ? bm[k - 1] : 0u, u1 = bm[k];
        uint32_t rank = u0;
        if (fits)
          for (uint32_t u = u0; u < u1; ++u) rank += pre[u] < j;
        else
          for (uint32_t u = u0; u < u1; ++u) rank += js[b + u] < j;
        emit(b + rank, b + t, j);
      }
      return;
    }
    wave_lds_sync();
  }
  int64_t below = 0;  // pairs of the row in earlier windows
  uint64_t lo = jlo;
  while (lo <= jhi) {
#pragma unroll
    for (int q = 0; q < kWordsPerLane; ++q) bm[lane * kWordsPerLane + q] = 0;
    wave_lds_sync();
    for (int64_t t = b + lane; t < e; t += 64) {
      const uint64_t r = (pk[t] & mask) - lo;
      if (r < (uint64_t)kWinBits) atomicOr(&bm[r >> 5], 1u << (r & 31));
    }
    wave_lds_sync();
    uint32_t c[kWordsPerLane], run = 0;
#pragma unroll
    for (int q = 0; q < kWordsPerLane; ++q) {
      c[q] = run;
      run += __popc(bm[lane * kWordsPerLane + q]);
    }
    uint32_t x = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    const uint32_t base = x - run, total = __shfl(x, 63, 64);
#pragma unroll
    for (int q = 0; q < kWordsPerLane; ++q) pre[lane * kWordsPerLane + q] = base + c[q];
    wave_lds_sync();
    uint32_t nxt = 0xffffffffu;  // smallest j past this window: the next window starts there
    for (int64_t t = b + lane; t < e; t += 64) {
      const uint64_t j = pk[t] & mask;
      const uint64_t r = j - lo;
      if (r < (uint64_t)kWinBits) {
        const uint32_t wd = (uint32_t)(r >> 5);
        const uint32_t rank = pre[wd] + __popc(bm[wd] & ((1u << (r & 31)) - 1u));
        emit(b + below + rank, t, (uint32_t)j);
      } else if (j > lo && j < nxt) {
        nxt = (uint32_t)j;
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const uint32_t a = __shfl_xor(nxt, o, 64);
      nxt = a < nxt ? a : nxt;
    }
    below += total;
    lo = nxt;
    wave_lds_sync();
  }
}

// kGroup lanes per row of at most kGroup pairs, and the wave for the longer
// ones, one after the other; few rows take a wave each.  Bound by the rows, not
// their bytes, where they are short: 1M rows of about one pair took 443 us with
// a wave each (the whole ordering), 305 / 159 / 101 with 32 / 16 / 8 lanes; 1M
// of about 17 pairs 1321, 1016 / 981 / 982; 60,000 of 25 165, 151 / 149 / 154.
template <int kGroup>
__global__ __launch_bounds__(64 * kRowWaves) void order_rows_kernel(const unsigned long long* __restrict__ pk,
                                                                   const float* __restrict__ pv, int64_t nR,
                                                                   uint32_t* __restrict__ js,
                                                                   const uint32_t* __restrict__ off,
                                                                   const Counters* __restrict__ c, int64_t cap,
                                                                   int bj, int64_t w, uint32_t* __restrict__ oi,
                                                                   uint32_t* __restrict__ oj, float* __restrict__ od) {
  __shared__ uint32_t bits_lds[kRowWaves][kWinWords];
  __shared__ uint32_t pre_lds[kRowWaves][kWinWords];
  if (ordered_pairs(c, cap) == 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i0 = ((int64_t)blockIdx.x * kRowWaves + wave) * (64 / kGroup);
  if (kGroup == 64) {
    if (i0 < nR)
      order_row(pk, pv, i0, off[i0], off[i0 + 1], js, bj, w, oi, oj, od, bits_lds[wave], pre_lds[wave]);
    return;
  }
  const int64_t i = i0 + lane / kGroup;
  const uint32_t b = i < nR ? off[i] : 0u, e = i < nR ? off[i + 1] : 0u;
  const uint32_t t = b + (lane & (kGroup - 1));
  const bool in = e - b <= kGroup && t < e;
  const uint32_t j = in ? (uint32_t)(pk[t] & ((1ull << bj) - 1)) : 0xffffffffu;
  uint32_t at = b;
#pragma unroll
  for (int u = 0; u < kGroup; ++u) at += __shfl(j, (lane & ~(kGroup - 1)) + u, 64) < j;
  if (in && at < w) {
    oi[at] = (uint32_t)i;
    oj[at] = j;
    od[at] = pv[t];
  }
  uint64_t longer = __ballot(e - b > kGroup && (lane & (kGroup - 1)) == 0);
  while (longer) {
    const int l = __ffsll((long long)longer) - 1;
    longer &= longer - 1;
    order_row(pk, pv, i0 + l / kGroup, __shfl(b, l, 64), __shfl(e, l, 64), js, bj, w, oi, oj, od, bits_lds[wave],
              pre_lds[wave]);
    wave_lds_sync();
  }
}

int64_t row_sort_words(int64_t nR) { return 2 * (nR + 1) + scan_scratch_words(nR + 1) + 1; }

// Scratch layout: the row counts (nR + 1 words, the last 0), the row offsets
// and the scan's sums.
// keys/vals: the confirmed pairs (key i << bj | j) of a recheck that counted
// them into words (overwritten); c, cap: its counters and candidate capacity; pk/pv: cap
// entries of scratch.  Writes the first w pairs in (i, j) order to oi/oj/od.
hipError_t row_sort_pairs(unsigned long long* keys, const float* vals, const Counters* c, int64_t cap, int64_t nR,
                          int bj, unsigned long long* pk, float* pv, uint32_t* words, int64_t w, uint32_t* oi,
                          uint32_t* oj, float* od, hipStream_t st, int cu_count) {
  uint32_t* cnt = words;
  uint32_t* off = words + (nR + 1);
  uint32_t* sums = words + 2 * (nR + 1);
  uint32_t* js = reinterpret_cast<uint32_t*>(keys);  // free once the pairs are placed
  const int64_t gm = (cap + 255) / 256 < (int64_t)cu_count * 8 ? (cap + 255) / 256 : (int64_t)cu_count * 8;
  hipError_t e = launch_exclusive_scan(cnt, nR + 1, off, sums, st, &c->out);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(place_rows_kernel, dim3((unsigned)gm), dim3(256), 0, st, keys, vals, c, cap, bj, off, cnt, pk, pv);
  auto order = [&](auto kernel, int rows) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((nR + rows - 1) / rows)), dim3(64 * kRowWaves), 0, st, pk, pv, nR, js,
                       off, c, cap, bj, w, oi, oj, od);
  };
  if (nR >= (int64_t)cu_count * kOrderFill) order(order_rows_kernel<kOrderGroup>, kRowWaves * (64 / kOrderGroup));
  else order(order_rows_kernel<64>, kRowWaves);
  return hipGetLastError();
}

}  // namespace dl
