// featurize.hip -- colour-histogram transformer over uint8 RGB patches.
//
// Paper: section "Visual ETL", Transformers (colour histogram features for
// image matching); the patches are crops of frames given by bounding boxes
// (section "Iterator API for Patches": a patch refers to a region of an
// image), either already cut out (n patches of h x w pixels) or as boxes over
// full frames.  One wavefront builds the histogram of one patch in a
// wave-private LDS array, so the waves of a workgroup never wait for one
// another (wave-level LDS ordering only); boxes that are few, and large patches
// no 16-byte load fits, take a workgroup of two or four waves.  The only global
// traffic is one read of the pixels and one coalesced write of the normalised
// bins.  HBM-bound: algorithmic bytes per patch are h*w*3 read plus bins^3*4
// written.
//
// The fused kernel (materialise into a store, section "Visual ETL") hands
// each bin straight from LDS to the operand prep of the join (operand copy
// and row statistics), so the float32 histograms are written once and never
// read back.
#include "prep_row.hpp"

namespace dl {

constexpr int kHistWaves = 4;  // patches (waves) per workgroup

// This wave's LDS operations are complete and every lane has reached this
// point (the histogram is private to the wave).  Only the LDS counter is
// waited for (s_waitcnt lgkmcnt(0); vmcnt and expcnt at their no-wait
// values): the wave's global stores of the previous patch need not land
// before it clears and counts the next one.
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_wave_barrier();
}

// Counts of one 16-pixel group (48 bytes = 12 dwords) into the wave's bins.
// Neighbouring pixels often share a bin, so a run of equal bins is added
// with one LDS atomic (fewer atomics, and fewer lanes colliding on the
// same bin in one instruction; measured 0.157 -> 0.127 ms on 100,000
// palette patches).
__device__ inline void count16(uint32_t* __restrict__ hist, const uint32_t w[12], int shift, int bins) {
  uint32_t prev = 0xffffffffu, run = 0;
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int b0 = 3 * p, b1 = 3 * p + 1, b2 = 3 * p + 2;
    uint32_t r = (w[b0 >> 2] >> ((b0 & 3) * 8)) & 0xffu;
    uint32_t g = (w[b1 >> 2] >> ((b1 & 3) * 8)) & 0xffu;
    uint32_t b = (w[b2 >> 2] >> ((b2 & 3) * 8)) & 0xffu;
    uint32_t bin = (((r >> shift) * bins) + (g >> shift)) * bins + (b >> shift);
    if (bin == prev) {
      ++run;
    } else {
      if (run) atomicAdd(&hist[prev], run);
      prev = bin;
      run = 1;
    }
  }
  atomicAdd(&hist[prev], run);
}

// Counts of `rows` runs of cw pixels, pitch bytes apart, into the bins, by
// kThreads threads (t of them).  A thread takes four neighbouring pixels at a
// time, 12 bytes in one (unaligned) load; a run's last four overlap the ones
// before, whose pixels it leaves out, so no byte beside the run is read.
// kUnits such groups are in flight per thread.
constexpr int kUnits = 4;
struct __attribute__((packed)) Bytes12 {
  uint32_t w[3];
};
template <int kThreads>
__device__ inline void count_runs(uint32_t* __restrict__ hist, const uint8_t* __restrict__ base, int64_t pitch, int cw,
                                  int rows, int shift, int bins, int t) {
  const int width = 8 - shift;
  auto field = [&](uint32_t w, int off) { return __builtin_amdgcn_ubfe(w, off + shift, width); };
  auto bin_of = [&](uint32_t r, uint32_t g, uint32_t b) { return __umul24(__umul24(r, bins) + g, bins) + b; };
  // pixels of a run (narrow ones, and all of them at most one per thread), or
  // groups of four
  const bool single = cw < 4 || cw * rows <= kThreads;
  const int per = single ? cw : (cw + 3) / 4;
  const int units = per * rows;
  // run of a unit by a float reciprocal, then one correction step each way
  // (units < 2^24, so the estimate is off by at most one)
  const float rper = 1.0f / (float)per;
  auto run_of = [&](int q, int& x) {
    int y = (int)((float)q * rper);
    x = q - y * per;
    if (x < 0) {
      --y;
      x += per;
    } else if (x >= per) {
      ++y;
      x -= per;
    }
    return base + y * pitch;
  };
  if (single) {
    for (int q = t; q < units; q += kThreads) {
      int x;
      const uint8_t* px = run_of(q, x) + 3 * x;
      atomicAdd(&hist[bin_of(px[0] >> shift, px[1] >> shift, px[2] >> shift)], 1u);
    }
    return;
  }
  for (int q0 = 0; q0 < units; q0 += kThreads * kUnits) {
    Bytes12 v[kUnits];
    int skip[kUnits];
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      if (q0 + kThreads * u >= units) break;
      const int q = q0 + kThreads * u + t;
      skip[u] = 4;
      if (q < units) {
        int x;
        const uint8_t* run = run_of(q, x);
        const int at = min(4 * x, cw - 4);
        skip[u] = 4 * x - at;
        v[u] = *reinterpret_cast<const Bytes12*>(run + 3 * at);
      }
    }
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      if (q0 + kThreads * u >= units) break;
      const uint32_t w0 = v[u].w[0], w1 = v[u].w[1], w2 = v[u].w[2];
      const uint32_t b[4] = {bin_of(field(w0, 0), field(w0, 8), field(w0, 16)),
                             bin_of(field(w0, 24), field(w1, 0), field(w1, 8)),
                             bin_of(field(w1, 16), field(w1, 24), field(w2, 0)),
                             bin_of(field(w2, 8), field(w2, 16), field(w2, 24))};
      // equal neighbours add up to one count
      uint32_t run = 0;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        run += p >= skip[u];
        if (p < 3 && b[p] == b[p + 1]) continue;
        if (run) atomicAdd(&hist[b[p]], run);
        run = 0;
      }
    }
  }
}

// Pixel sources.  kSrcPatch48: contiguous patches whose pixel count is a
// multiple of 16, 16-byte aligned (three 16-byte loads per 16 pixels);
// kSrcPatch: any contiguous patches; kSrcCrop: boxes over frames.
enum : int { kSrcPatch48 = 0, kSrcPatch = 1, kSrcCrop = 2 };

struct PixelSource {
  const uint8_t* pix;      // patches (n x h x w x 3) or frames (nframes x h x w x 3)
  int32_t h, w;            // patch size, or frame size for crops
  const dl_box* boxes;     // crops: one box per patch
  int64_t nframes;
  int* bad_box;            // crops: set when a box is not inside its frame
};

// The pixels of a box or of a contiguous patch: `rows` runs of cw pixels (none
// for a box that is not inside its frame).
struct Runs {
  const uint8_t* base;
  int64_t pitch;
  int cw, rows;
  bool bad;
};
template <int kSrc>
__device__ inline Runs runs_of(const PixelSource& src, int64_t p) {
  if constexpr (kSrc == kSrcCrop) {
    const dl_box bx = src.boxes[p];
    if (bx.frame >= 0 && bx.frame < src.nframes && bx.x0 >= 0 && bx.x0 < bx.x1 && bx.x1 <= src.w && bx.y0 >= 0 &&
        bx.y0 < bx.y1 && bx.y1 <= src.h)
      return {src.pix + (((int64_t)bx.frame * src.h + bx.y0) * src.w + bx.x0) * 3, (int64_t)src.w * 3, bx.x1 - bx.x0,
              bx.y1 - bx.y0, false};
    return {nullptr, 0, 0, 0, true};
  } else {
    const int npx = src.h * src.w;
    return {src.pix + p * (int64_t)npx * 3, 0, npx, 1, false};
  }
}

// Counts the pixels of patch p into the wave's bins; returns the pixel count
// (0 for an invalid box, which contributes nothing).
template <int kSrc>
__device__ inline int count_patch(const PixelSource& src, int64_t p, uint32_t* __restrict__ hist, int shift,
                                  int bins, int lane) {
  if constexpr (kSrc == kSrcPatch48) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const int npx = src.h * src.w;
    const u32x4* v = reinterpret_cast<const u32x4*>(src.pix + p * (int64_t)npx * 3);
    const int groups = npx / 16;  // 16 pixels = 48 bytes = 3 x 16 bytes
    for (int c = lane; c < groups; c += 64) {
      const u32x4 x0 = __builtin_nontemporal_load(v + 3 * c + 0);
      const u32x4 x1 = __builtin_nontemporal_load(v + 3 * c + 1);
      const u32x4 x2 = __builtin_nontemporal_load(v + 3 * c + 2);
      uint32_t w[12] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w, x2.x, x2.y, x2.z, x2.w};
      count16(hist, w, shift, bins);
    }
    return npx;
  } else {
    const Runs r = runs_of<kSrc>(src, p);
    if (r.bad && lane == 0) atomicOr(src.bad_box, 1);
    if (r.rows) count_runs<64>(hist, r.base, r.pitch, r.cw, r.rows, shift, bins, lane);
    return r.cw * r.rows;
  }
}

static int bin_shift(int bins) {
  int shift = 0;
  while ((256 >> shift) > bins) ++shift;
  return shift;
}

// Histograms only: bin / pixel count, rounded once (IEEE division).  A wave per
// patch: aligned patches, others of at most kWaveArea pixels (a workgroup of two
// waves each: 200,000 of 5 x 7, 8 / 4 bins, 141 / 78 us against 93 / 26; 60,000 of 31
// x 33 60 against 53), and boxes that are many.  Not with more than kWaveBins bins a
// channel, unless the loads are aligned: LDS holds eight histograms of 16 KiB a CU so,
// ten workgroups the other way (16 bins: 200,000 of 5 x 7 605 us against 775, 60,000 of
// 31 x 33 203 against 278).
constexpr int kWaveArea = 1024, kWaveBins = 8;
template <int kSrc>
__global__ __launch_bounds__(64 * kHistWaves) void hist_patch_kernel(PixelSource src, int64_t n, int32_t bins,
                                                                   int32_t shift, float* __restrict__ out) {
  extern __shared__ uint32_t lds_hist[];
  const int nb = bins * bins * bins;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t* hist = lds_hist + wave * nb;
  const int64_t ngroups = (n + kHistWaves - 1) / kHistWaves;
  for (int64_t g = blockIdx.x; g < ngroups; g += gridDim.x) {
    const int64_t p = g * kHistWaves + wave;
    if (p >= n) break;
    for (int b = lane; b < nb; b += 64) hist[b] = 0u;
    wave_lds_fence();
    const int npx = count_patch<kSrc>(src, p, hist, shift, bins, lane);
    wave_lds_fence();
    const float fnpx = (float)(npx > 0 ? npx : 1);  // exact: npx < 2^24
    float* dst = out + p * (int64_t)nb;
    for (int b = lane; b < nb; b += 64) dst[b] = (float)hist[b] / fnpx;  // IEEE division
    wave_lds_fence();  // the bins are read before the next patch clears them
  }
}

// Boxes and larger unaligned patches: a workgroup each.
template <int kSrc, int kThreads>
__global__ __launch_bounds__(kThreads) void hist_runs_kernel(PixelSource src, int32_t bins, int32_t shift,
                                                             float* __restrict__ out) {
  extern __shared__ uint32_t lds_hist[];
  const int nb = bins * bins * bins;
  const int64_t p = blockIdx.x;
  for (int b = threadIdx.x; b < nb; b += kThreads) lds_hist[b] = 0u;
  __syncthreads();
  const Runs r = runs_of<kSrc>(src, p);
  if (r.bad && threadIdx.x == 0) atomicOr(src.bad_box, 1);
  if (r.rows) count_runs<kThreads>(lds_hist, r.base, r.pitch, r.cw, r.rows, shift, bins, threadIdx.x);
  __syncthreads();
  const float fnpx = (float)(r.rows ? r.cw * r.rows : 1);
  float* dst = out + p * (int64_t)nb;
  for (int b = threadIdx.x; b < nb; b += kThreads) dst[b] = (float)lds_hist[b] / fnpx;
}

template <int kSrc>
static hipError_t launch_hist_patches(const PixelSource& src, int64_t n, int32_t bins, float* out, hipStream_t st,
                                      int cu_count) {
  const int64_t groups = (n + kHistWaves - 1) / kHistWaves, most = (int64_t)cu_count * 64;
  const size_t lds = (size_t)kHistWaves * bins * bins * bins * sizeof(uint32_t);
  hipLaunchKernelGGL(hist_patch_kernel<kSrc>, dim3((unsigned)(groups < most ? groups : most)), dim3(64 * kHistWaves),
                     lds, st, src, n, bins, bin_shift(bins), out);
  return hipGetLastError();
}

// A box's size varies and is known on the device alone.  A wave by itself is
// bound by its loads' latency round after round (200 boxes of up to 200 x 200: 38
// us with a wave each, 20 / 12 with two / four), many workgroups by their
// launches and barriers.  So four waves a box while every box is resident at
// once, two up to 160 boxes per CU, a wave each beyond: call time with two waves /
// one, sides of up to 8, 96 and 200 pixels: 20,000 boxes 35 / 33 us, 48 / 54; 40,000
// 46 / 41, 68 / 73, 117 / 143; 45,000 50 / 41, 106 / 111, 274 / 314; 300,000 of up to
// 8 265 / 187, 16 270 / 194, 96 535 / 567.
template <int kSrc>
static hipError_t launch_hist_runs(const PixelSource& src, int64_t n, int32_t bins, float* out, hipStream_t st,
                                   int cu_count) {
  if (n > (int64_t)cu_count * 160 && (bins <= kWaveBins || n > (1 << 24)))  // (a launch holds 2^32 threads)
    return launch_hist_patches<kSrc>(src, n, bins, out, st, cu_count);
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(threads), bins * bins * bins * sizeof(uint32_t), st, src, bins,
                       bin_shift(bins), out);
    return hipGetLastError();
  };
  return n <= (int64_t)cu_count * 8 ? go(hist_runs_kernel<kSrc, 256>, 256) : go(hist_runs_kernel<kSrc, 128>, 128);
}

// Histograms plus the join's operand prep of each histogram row (rows n..npad
// of the operand copy are zero padding, as the prep kernel writes them).
template <int kSrc, int kPrec>
__global__ __launch_bounds__(64 * kHistWaves) void hist_prep_kernel(PixelSource src, int64_t n, int32_t bins,
                                                                    int32_t shift, float* __restrict__ out,
                                                                    int64_t dpad, Prep P, RelStats* rs) {
  extern __shared__ uint32_t lds_hist[];
  const int nb = bins * bins * bins;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t* hist = lds_hist + wave * nb;
  const int64_t ngroups = (P.npad + kHistWaves - 1) / kHistWaves;
  for (int64_t g = blockIdx.x; g < ngroups; g += gridDim.x) {
    const int64_t p = g * kHistWaves + wave;
    if (p >= P.npad) break;
    const bool real = p < n;
    int npx = 0;
    if (real) {
      for (int b = lane; b < nb; b += 64) hist[b] = 0u;
      wave_lds_fence();
      npx = count_patch<kSrc>(src, p, hist, shift, bins, lane);
      wave_lds_fence();
    }
    const float fnpx = (float)(npx > 0 ? npx : 1);
    int sexp = 0;
    if (kPrec == DL_FP8 && real) {
      // the largest bin, divided as the bins are (rounding is monotone)
      uint32_t cmax = 0;
      for (int b = lane; b < nb; b += 64) cmax = max(cmax, hist[b]);
      sexp = e4m3_row_scale(wave_max((float)cmax / fnpx));
    }
    RowPrep<kPrec> rp(P, p, sexp);
    float* dst = out + p * (int64_t)nb;
    for (int64_t k = lane; k < dpad; k += 64) {
      float v = 0.0f;
      if (real && k < nb) {
        v = (float)hist[k] / fnpx;  // IEEE division
        dst[k] = v;
      }
      rp.element(v, k);
    }
    rp.finish(P, p, dpad, real, rs, lane);
    wave_lds_fence();
  }
}

// Host launchers; arguments validated by the caller.
hipError_t launch_hist_rgb8(const uint8_t* patches, int64_t n, int32_t h, int32_t w, int32_t bins,
                            float* out, hipStream_t st, int cu_count) {
  if (n == 0) return hipSuccess;
  const int32_t npx = h * w;
  const PixelSource src{patches, h, w, nullptr, 0, nullptr};
  if (npx % 16 == 0 && (reinterpret_cast<uintptr_t>(patches) & 15) == 0)
    return launch_hist_patches<kSrcPatch48>(src, n, bins, out, st, cu_count);
  if (npx <= kWaveArea && bins <= kWaveBins) return launch_hist_patches<kSrcPatch>(src, n, bins, out, st, cu_count);
  return launch_hist_runs<kSrcPatch>(src, n, bins, out, st, cu_count);
}

hipError_t launch_hist_crops(const uint8_t* frames, int64_t nframes, int32_t height, int32_t width,
                             const dl_box* boxes, int64_t n, int32_t bins, float* out, int* bad_box, hipStream_t st,
                             int cu_count) {
  if (n == 0) return hipSuccess;
  return launch_hist_runs<kSrcCrop>(PixelSource{frames, height, width, boxes, nframes, bad_box}, n, bins, out, st, cu_count);
}

template <int kSrc>
static void launch_hist_prep_src(const PixelSource& src, int64_t n, int32_t bins, float* out, dl_prec prec,
                                 const Prep& P, RelStats* rs, dim3 grid, size_t lds, hipStream_t st) {
  const int64_t dpad = dpad_of(bins * bins * bins, prec);
  const int shift = bin_shift(bins);
  switch (prec) {
    case DL_FP32:
      hipLaunchKernelGGL((hist_prep_kernel<kSrc, DL_FP32>), grid, dim3(64 * kHistWaves), lds, st, src, n, bins, shift,
                         out, dpad, P, rs);
      break;
    case DL_BF16:
      hipLaunchKernelGGL((hist_prep_kernel<kSrc, DL_BF16>), grid, dim3(64 * kHistWaves), lds, st, src, n, bins, shift,
                         out, dpad, P, rs);
      break;
    case DL_FP16:
      hipLaunchKernelGGL((hist_prep_kernel<kSrc, DL_FP16>), grid, dim3(64 * kHistWaves), lds, st, src, n, bins, shift,
                         out, dpad, P, rs);
      break;
    case DL_FP8:
      hipLaunchKernelGGL((hist_prep_kernel<kSrc, DL_FP8>), grid, dim3(64 * kHistWaves), lds, st, src, n, bins, shift,
                         out, dpad, P, rs);
      break;
  }
}

// Fused featurise + prep into P (npad rows); the caller runs the statistics
// reduction after it.  frames/boxes null: patches of h x w.
hipError_t launch_hist_prep(const uint8_t* pix, int64_t nframes, int32_t h, int32_t w, const dl_box* boxes, int64_t n,
                            int32_t bins, float* out, int* bad_box, dl_prec prec, const Prep& P, RelStats* rs,
                            hipStream_t st, int cu_count) {
  const int nb = bins * bins * bins;
  const size_t lds = (size_t)kHistWaves * nb * sizeof(uint32_t);
  const int64_t ngroups = (P.npad + kHistWaves - 1) / kHistWaves;
  const dim3 grid((unsigned)(ngroups < (int64_t)cu_count * 64 ? ngroups : (int64_t)cu_count * 64));
  if (boxes) {
    launch_hist_prep_src<kSrcCrop>(PixelSource{pix, h, w, boxes, nframes, bad_box}, n, bins, out, prec, P, rs, grid,
                                   lds, st);
  } else {
    const PixelSource src{pix, h, w, nullptr, 0, nullptr};
    if (((int64_t)h * w) % 16 == 0 && (reinterpret_cast<uintptr_t>(pix) & 15) == 0)
      launch_hist_prep_src<kSrcPatch48>(src, n, bins, out, prec, P, rs, grid, lds, st);
    else
      launch_hist_prep_src<kSrcPatch>(src, n, bins, out, prec, P, rs, grid, lds, st);
  }
  return hipGetLastError();
}

}  // namespace dl
