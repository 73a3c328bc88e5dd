// Gray-scale transformations (Sec. 2.2.6): the zscale display range of a
// frame, point maps (linear, logarithmic, exponential, power law) over a
// value range, and histogram equalization (pixel counts per gray level,
// their cumulative distribution, and an interpolating map onto it).
//
// zscale follows the display-range estimate of SAOimage DS9 and IRAF:
// sort a grid sample of the frame, fit a straight line to the sorted values
// against their index with iterative rejection of outlying samples (each
// rejection widened to its neighbours), and evaluate the line, with its
// slope divided by a contrast factor, at the ends of the index range
// through the median.
#include "ipp_internal.h"
#include "kernels.h"

namespace ipp {

namespace {

// Frame of a flat row index, given each frame's first row (ascending).
__device__ __forceinline__ int gray_frame_of(const GrayFrame* fr, int n,
                                             int row) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (fr[mid].row0 <= row) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Rows [r0, r1) of the batch handled by this block: contiguous ranges, so
// that a block meets few frame changes.
__device__ __forceinline__ void block_rows(int total_rows, int* r0, int* r1) {
  const int per = (total_rows + gridDim.x - 1) / gridDim.x;
  *r0 = min(total_rows, (int)blockIdx.x * per);
  *r1 = min(total_rows, *r0 + per);
}

// ln(1 + u) for u >= 0 in binary32, from w = fl(1 + u): ln(w) u / (w - 1)
// (Goldberg, "What every computer scientist should know about
// floating-point arithmetic", 1991, Thm. 4), with the hardware log2.
__device__ __forceinline__ float log1p_g(float u) {
  const float w = 1.0f + u;
  if (w == 1.0f) return u;
  return 0.69314718f * __builtin_amdgcn_logf(w) * (u / (w - 1.0f));
}

// e^t - 1 in binary32 from u = fl(e^t): (u - 1) t / ln(u) (W. Kahan's
// identity), with the hardware exp2 and log2.
__device__ __forceinline__ float expm1_k(float t) {
  const float u = __builtin_amdgcn_exp2f(t * 1.44269504f);
  if (u == 1.0f) return t;
  const float lu = 0.69314718f * __builtin_amdgcn_logf(u);
  return (u - 1.0f) * (t / lu);
}

struct MapConst {
  int kind;
  float a;          // the map's parameter
  float c;          // LOG: 1 / ln(1 + a); EXP: 1 / (a - 1)
  float lna;        // EXP: ln a
};

// Gray level of one pixel: x = (v - lo) / (hi - lo) in binary64, clipped
// to [0, 1], then the map in binary32.
__device__ __forceinline__ float map_pixel(float v, double lo, double inv,
                                           bool step, const MapConst& m) {
  if (!isfinite(v)) return __builtin_nanf("");
  double xd = step ? ((double)v <= lo ? 0.0 : 1.0) : ((double)v - lo) * inv;
  xd = fmin(fmax(xd, 0.0), 1.0);
  const float x = (float)xd;
  switch (m.kind) {
    case IPP_MAP_LOG:
      return log1p_g(m.a * x) * m.c;
    case IPP_MAP_EXP:
      return expm1_k(x * m.lna) * m.c;
    case IPP_MAP_POWER: {
      if (xd <= 0.0) return 0.0f;
      // log2 of the binary64 x through its exponent (x may be below the
      // binary32 normal range)
      int e;
      const double mant = frexp(xd, &e);              // [0.5, 1)
      const float l2 = (float)e + __builtin_amdgcn_logf((float)mant);
      return __builtin_amdgcn_exp2f(m.a * l2);
    }
    default:
      return x;
  }
}

// Four consecutive values of a row of any alignment: one load or store (a
// vector access to global memory needs only its elements' alignment).  Four
// 4095 x 4093 frames, map and equalization: 380 us, 660 a value at a time.
typedef float Float4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ Float4 load4(const float* a) {
  return *(const __attribute__((address_space(1))) Float4*)a;
}
__device__ __forceinline__ void store4(float* a, Float4 v) {
  *(__attribute__((address_space(1))) Float4*)a = v;
}

// Row y of frame F: fn(v, out_row, x) with v a Float4 of columns x..x+3, or a
// float of column x for the last w % 4.  Two groups per thread are loaded
// before either is used, so that both loads are in flight together.
template <typename Fn>
__device__ __forceinline__ void row_elements(const GrayFrame& F, int y,
                                             Fn fn) {
  const float* in = F.pix + (int64_t)y * F.pitch;
  float* out = F.out ? F.out + (int64_t)y * F.w : nullptr;
  const int n4 = F.w >> 2;
  int i = threadIdx.x;
  for (; i + kBlock < n4; i += 2 * kBlock) {
    const Float4 a = load4(in + 4 * i), b = load4(in + 4 * (i + kBlock));
    fn(a, out, 4 * i);
    fn(b, out, 4 * (i + kBlock));
  }
  if (i < n4) fn(load4(in + 4 * i), out, 4 * i);
  // the row's end (by the last threads instead: 392 against 380 us)
  const int xt = (n4 << 2) + (int)threadIdx.x;
  if (xt < F.w) fn(gld(in + xt), out, xt);
}

}  // namespace

// ---------------------------------------------------------------------
// zscale: one workgroup per frame; sample e belongs to thread e % kBlock.
// One workgroup's chain of dependent steps, so what counts is their number:
// the sample's loads are in flight together, the sort needs a barrier only
// around its stages that cross the waves' quarters, a fit's four sums share
// one, and a rejection's neighbours are bits of ballots.  Four 4096^2
// frames: 24 us (48 with a barrier at each of the 55 stages and at every
// sum, and loops over the neighbours).
// ---------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_zscale(const GrayFrame* frames,
                                                   double contrast,
                                                   double krej, int max_iter,
                                                   double* z1z2,
                                                   double* info) {
  constexpr int kPer = kZMax / kBlock;
  constexpr int kQuarter = kZMax / kWaves;
  static_assert(kPer == 4 && kWaves == 4, "four samples a thread");
  __shared__ float sv[kZMax];
  __shared__ uint64_t rej[kZMax / kWave + 1];
  __shared__ double redd[2][4][kWaves];
  __shared__ int redi[kWaves];
  const int f = blockIdx.x;
  const GrayFrame F = frames[f];
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(t / kWave);
  const int ns = F.sy * F.sx;          // <= kZMax, checked on the host
  // ---- the grid sample; non-finite values and padding sort last --------
  float v[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = min(t + k * kBlock, ns - 1);
    const int i = e / F.sx, j = e - (e / F.sx) * F.sx;
    v[k] = F.pix[(int64_t)i * F.s * F.pitch + (int64_t)j * F.s];
  }
  int nfin = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const bool ok = t + k * kBlock < ns && isfinite(v[k]);
    nfin += ok;
    sv[t + k * kBlock] = ok ? v[k] : __builtin_inff();
  }
  const int n = block_sum(nfin, redi);
  // ---- bitonic sort, ascending -------------------------------------------
  // Pair e of a stage with stride j <= kQuarter / 2 lies in the quarter of
  // the wave that takes it.
  bool crossed = true;                 // other waves' values are due
  for (int k = 2; k <= kZMax; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      const bool cross = j > kQuarter / 2;
      if (cross || crossed) __syncthreads();
      else __builtin_amdgcn_wave_barrier();
      crossed = cross;
#pragma unroll
      for (int i = 0; i < kPer / 2; ++i) {
        const int e = wv * (kQuarter / 2) + i * kWave + lane;
        const int lo = 2 * e - (e & (j - 1));        // index bit of j clear
        const int hi = lo + j;
        const bool up = (lo & k) == 0;
        const float a = sv[lo], b = sv[hi];
        sv[lo] = (a > b) == up ? b : a;
        sv[hi] = (a > b) == up ? a : b;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
  __syncthreads();
  if (n == 0) {
    if (t == 0) {
      z1z2[2 * f] = 0.0;
      z1z2[2 * f + 1] = 0.0;
      if (info) {
        info[4 * f] = 0.0;
        info[4 * f + 1] = 0.0;
        info[4 * f + 2] = 0.0;
        info[4 * f + 3] = 0.0;
      }
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) v[k] = sv[t + k * kBlock];
  // the block sums of N values, one barrier (two buffers in turn)
  int buf = 0;
  auto sums = [&](auto& s) {
    constexpr int N = sizeof(s) / sizeof(double);
#pragma unroll
    for (int q = 0; q < N; ++q) {
      s[q] = wave_sum(s[q]);
      if (lane == 0) redd[buf][q][wv] = s[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const double* r = redd[buf][q];
      s[q] = (r[0] + r[1]) + (r[2] + r[3]);
    }
    buf ^= 1;
  };
  // median of the sorted sample (Eq. 1)
  const double med = (n & 1) ? (double)sv[(n - 1) / 2]
                             : ((double)sv[n / 2 - 1] + (double)sv[n / 2]) /
                                   2.0;
  const int minpix = max(5, n / 2);
  const int half = max(1, n / 100) / 2;                 // at most 5
  bool live[kPer];                     // in range and not rejected
#pragma unroll
  for (int k = 0; k < kPer; ++k) live[k] = t + k * kBlock < n;
  int kept = n, last = n + 1, fits = 0;
  double b = 0.0;
  while (fits < max_iter && kept < last && kept >= minpix) {
    // ---- least-squares line over the kept samples ---------------------
    double s[4] = {0.0, 0.0, 0.0, 0.0};          // i, i^2, v, i v
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (!live[k]) continue;
      const double i = (double)(t + k * kBlock), y = (double)v[k];
      s[0] += i;
      s[1] += i * i;
      s[2] += y;
      s[3] += i * y;
    }
    sums(s);
    const double nk = (double)kept;
    const double den = nk * s[1] - s[0] * s[0];
    b = den != 0.0 ? (nk * s[3] - s[0] * s[2]) / den : 0.0;
    const double a = (s[2] - b * s[0]) / nk;
    ++fits;
    // ---- scale: ddof-0 deviation of the kept residuals ----------------
    double res[kPer];
    double s1[1] = {0.0};
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      res[k] = (double)v[k] - (a + b * (double)(t + k * kBlock));
      if (live[k]) s1[0] += res[k];
    }
    sums(s1);
    const double mu = s1[0] / nk;
    double s2[1] = {0.0};
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const double d = res[k] - mu;
      if (live[k]) s2[0] += d * d;
    }
    sums(s2);
    const double thr = krej * sqrt(s2[0] / nk);
    // ---- reject, widen each rejection, count --------------------------
    // bit e of rej: sample e, rejected before or not, lies outside
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint64_t m = ballot(t + k * kBlock < n && fabs(res[k]) > thr);
      if (lane == 0) rej[k * kWaves + wv] = m;
    }
    if (t == 0) rej[kZMax / kWave] = 0;
    __syncthreads();
    double nk2[1] = {0.0};
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      // the bits of samples max(e - half, 0) .. e + half
      const int e = t + k * kBlock;
      const int j0 = max(0, e - half), len = e + half - j0 + 1;
      const int q = j0 >> 6, o = j0 & 63;
      uint64_t w = rej[q] >> o;
      if (o) w |= rej[q + 1] << (64 - o);
      if (w & ((1ull << len) - 1)) live[k] = false;
      nk2[0] += live[k] ? 1.0 : 0.0;
    }
    last = kept;
    sums(nk2);
    kept = (int)nk2[0];
  }
  if (t == 0) {
    double z1 = (double)sv[0], z2 = (double)sv[n - 1];
    if (kept >= minpix) {
      const double slope = contrast > 0.0 ? b / contrast : b;
      const int c = (n - 1) / 2;
      z1 = fmax(z1, med - (double)c * slope);
      z2 = fmin(z2, med + (double)(n - 1 - c) * slope);
    }
    z1z2[2 * f] = z1;
    z1z2[2 * f + 1] = z2;
    if (info) {
      info[4 * f] = (double)n;
      info[4 * f + 1] = (double)kept;
      info[4 * f + 2] = (double)fits;
      info[4 * f + 3] = b;
    }
  }
}

// ---------------------------------------------------------------------
// Point map of every frame over [lohi[2f], lohi[2f+1]].
// ---------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_gray_map(
    const GrayFrame* frames, int nframes, int total_rows, int kind, float a,
    float c, float lna, const double* lohi) {
  const MapConst m = {kind, a, c, lna};
  for (int row = blockIdx.x; row < total_rows; row += gridDim.x) {
    const int f = gray_frame_of(frames, nframes, row);
    const GrayFrame F = frames[f];
    const int y = row - F.row0;
    const double lo = lohi[2 * f], hi = lohi[2 * f + 1];
    const bool step = !(hi > lo);
    const double inv = step ? 0.0 : 1.0 / (hi - lo);
    row_elements(F, y, [&](auto v, float* out, int x) {
      if constexpr (sizeof(v) == sizeof(Float4)) {
        Float4 o;
        o.x = map_pixel(v.x, lo, inv, step, m);
        o.y = map_pixel(v.y, lo, inv, step, m);
        o.z = map_pixel(v.z, lo, inv, step, m);
        o.w = map_pixel(v.w, lo, inv, step, m);
        store4(out + x, o);
      } else {
        gst(out + x, map_pixel(v, lo, inv, step, m));
      }
    });
  }
}

// ---------------------------------------------------------------------
// Histogram equalization.
// ---------------------------------------------------------------------
// The value ranges and counts of n frames cleared, in one launch (a kernel,
// not a memset: the call may be captured into a graph).
__global__ __launch_bounds__(kBlock) void k_eq_clear(uint32_t* mm, int n,
                                                     uint32_t* counts,
                                                     int64_t nc) {
  for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < nc;
       i += (int64_t)gridDim.x * kBlock) {
    counts[i] = 0;
    if (i < n) {
      mm[i] = 0xFFFFFFFFu;
      mm[n + i] = 0u;
    }
  }
}

// Smallest and largest finite value of every frame, as ordered keys in
// mm[f] (min, starts at ~0) and mm[nframes + f] (max, starts at 0).
// One workgroup's range joins its frame's: most workgroups find it already
// inside and leave without an atomic operation (all of a frame's go to the
// same two words).
__device__ __forceinline__ void take_range(uint32_t* lo, uint32_t* hi,
                                           uint32_t bmin, uint32_t bmax) {
  if (bmin > bmax) return;                      // no finite value
  if (bmin < __hip_atomic_load(lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMin(lo, bmin);
  if (bmax > __hip_atomic_load(hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(hi, bmax);
}

__global__ __launch_bounds__(kBlock) void k_eq_minmax(const GrayFrame* frames,
                                                      int nframes,
                                                      int total_rows,
                                                      uint32_t* mm) {
  __shared__ uint32_t red[kWaves];
  int r0, r1;
  block_rows(total_rows, &r0, &r1);
  if (r0 >= r1) return;
  int f = gray_frame_of(frames, nframes, r0);
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  for (int row = r0; row < r1; ++row) {
    while (f + 1 < nframes && frames[f + 1].row0 <= row) {
      // frame change: flush this frame's partial range
      const uint32_t bmin = block_min(kmin, red);
      const uint32_t bmax = block_max(kmax, red);
      if (threadIdx.x == 0) take_range(&mm[f], &mm[nframes + f], bmin, bmax);
      kmin = 0xFFFFFFFFu;
      kmax = 0u;
      ++f;
    }
    const GrayFrame F = frames[f];
    auto take = [&](float v) {
      if (isfinite(v)) {
        const uint32_t k = f2key(v + 0.0f);
        kmin = min(kmin, k);
        kmax = max(kmax, k);
      }
    };
    row_elements(F, row - F.row0, [&](auto v, float*, int) {
      if constexpr (sizeof(v) == sizeof(Float4)) {
        take(v.x); take(v.y); take(v.z); take(v.w);
      } else {
        take(v);
      }
    });
  }
  const uint32_t bmin = block_min(kmin, red);
  const uint32_t bmax = block_max(kmax, red);
  if (threadIdx.x == 0) take_range(&mm[f], &mm[nframes + f], bmin, bmax);
}

// Bin of a finite value: floor(((v - lo) / (hi - lo)) * nbins), the top
// value in the last bin (binary64, division as written).  t = (v - lo) *
// (nbins / (hi - lo)) is within a few units in the last place (< 4e-12 for
// t <= 4096) of the value the written form floors, so where t is more than
// 1e-9 from an integer its floor is the bin; values nearer a bin edge take
// the division.
__device__ __forceinline__ int eq_bin(float v, double lo, double range,
                                      double scale, int nbins) {
  const double d = (double)v - lo;
  const double t = d * scale;
  const double ft = floor(t);
  const double fr = t - ft;
  int k = (int)ft;
  if (fr < 1e-9 || fr > 1.0 - 1e-9)
    k = (int)floor((d / range) * (double)nbins);
  return min(k, nbins - 1);
}

// Per-block LDS histograms in two copies (lane parity picks the copy, the
// copies of a bin sit in adjacent banks), so that the many lanes whose sky
// values fall in the same few bins collide half as often; each lane merges
// equal bins among its four values before adding.
__global__ __launch_bounds__(kBlock) void k_eq_hist(const GrayFrame* frames,
                                                    int nframes,
                                                    int total_rows, int nbins,
                                                    const uint32_t* mm,
                                                    uint32_t* counts) {
  __shared__ uint32_t h[2 * kMaxBins];
  int r0, r1;
  block_rows(total_rows, &r0, &r1);
  if (r0 >= r1) return;
  const uint32_t rep = threadIdx.x & 1u;
  for (int i = threadIdx.x; i < 2 * nbins; i += kBlock) h[i] = 0;
  __syncthreads();
  int f = gray_frame_of(frames, nframes, r0);
  auto flush = [&](int fr) {
    __syncthreads();
    for (int i = threadIdx.x; i < nbins; i += kBlock) {
      const uint32_t c = h[2 * i] + h[2 * i + 1];
      if (c) atomicAdd(&counts[(size_t)fr * nbins + i], c);
      h[2 * i] = 0;
      h[2 * i + 1] = 0;
    }
    __syncthreads();
  };
  int64_t held = 0;                        // pixels counted since a flush
  for (int row = r0; row < r1; ++row) {
    while (f + 1 < nframes && frames[f + 1].row0 <= row) {
      flush(f);
      held = 0;
      ++f;
    }
    const GrayFrame F = frames[f];
    if (held + F.w > (int64_t)1 << 31) {     // keep the 32-bit counters exact
      flush(f);
      held = 0;
    }
    held += F.w;
    const uint32_t kl = mm[f], kh = mm[nframes + f];
    if (kl > kh) continue;                 // no finite value in the frame
    const double lo = (double)key2f(kl), hi = (double)key2f(kh);
    const double range = hi - lo;
    const double scale = range > 0.0 ? (double)nbins / range : 0.0;
    auto bin = [&](float v) -> int {       // -1: not finite
      if (!isfinite(v)) return -1;
      return range > 0.0 ? eq_bin(v, lo, range, scale, nbins) : 0;
    };
    auto add = [&](int k, uint32_t c) {
      if (k >= 0) atomicAdd(&h[2 * k + rep], c);
    };
    row_elements(F, row - F.row0, [&](auto v, float*, int) {
      if constexpr (sizeof(v) == sizeof(Float4)) {
        const int k0 = bin(v.x), k1 = bin(v.y);
        const int k2 = bin(v.z), k3 = bin(v.w);
        // runs of equal bins among the four
        uint32_t c = 1;
        if (k1 == k0) ++c; else { add(k0, c); c = 1; }
        if (k2 == k1) ++c; else { add(k1, c); c = 1; }
        if (k3 == k2) ++c; else { add(k2, c); c = 1; }
        add(k3, c);
      } else {
        add(bin(v), 1u);
      }
    });
  }
  flush(f);
}

// y = the interpolation of (centre_k, cdf_k) at v, held at the ends, with
// cdf_k = (pixels of the frame in bins 0..k) / (its finite pixels).  Each
// block maps a contiguous range of rows; it forms the cdf of the frame being
// mapped itself, from the counts, and holds it in LDS in binary32 (values in
// [0, 1]: 6e-8 absolute).  The position of v among the centres,
// t = (v - lo) / w - 1/2, is taken in binary64 (v - lo exactly) and clamped
// to the centres; the interpolation is continuous, so the interval a value
// on a centre falls in does not change y.
// Bound by memory: enough workgroups that their loads are in flight together,
// and no branches between them and the stores.  Four 4096^2 frames: 98 us,
// 5.5 TB/s (167 with branches and half as many workgroups, and 8 for the cdf
// as a kernel of its own).
__global__ __launch_bounds__(kBlock) void k_eq_map(const GrayFrame* frames,
                                                   int nframes,
                                                   int total_rows, int nbins,
                                                   const uint32_t* mm,
                                                   const uint32_t* counts) {
  __shared__ float T[kMaxBins + 1];
  __shared__ int red[kWaves];
  constexpr int kPer = kMaxBins / kBlock;
  int r0, r1;
  block_rows(total_rows, &r0, &r1);
  if (r0 >= r1) return;
  int f = -1;
  double lo = 0.0, inv_w = 0.0;
  bool span = false;
  for (int row = r0; row < r1; ++row) {
    int nf = f < 0 ? gray_frame_of(frames, nframes, row) : f;
    while (nf + 1 < nframes && frames[nf + 1].row0 <= row) ++nf;
    if (nf != f) {
      // a new frame: its value range and cdf
      f = nf;
      const uint32_t kl = mm[f], kh = mm[nframes + f];
      const double l = kl <= kh ? (double)key2f(kl) : 0.0;
      const double h = kl <= kh ? (double)key2f(kh) : 0.0;
      lo = l;
      span = h > l;
      inv_w = span ? (double)nbins / (h - l) : 0.0;
      __syncthreads();
      if (span) {
        const uint32_t* c = counts + (size_t)f * nbins;
        const int b0 = threadIdx.x * kPer;
        int own[kPer];
        int sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i)
          own[i] = b0 + i < nbins ? (int)c[b0 + i] : 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) sum += own[i];
        int total;
        int run = block_exclusive_scan(sum, red, &total);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
          run += own[i];
          if (b0 + i < nbins) T[b0 + i] = (float)((double)run / (double)total);
        }
        // the last centre holds: its neighbour in the table is itself
        if (threadIdx.x == 0) T[nbins] = 1.0f;
      }
      __syncthreads();
    }
    const GrayFrame F = frames[f];
    auto eq = [&](float vf) -> float {
      const double t = ((double)vf - lo) * inv_w - 0.5;
      const double tc = fmin(fmax(t, 0.0), (double)(nbins - 1));
      const int j = (int)tc;
      const float fr = (float)(tc - (double)j);
      const float y0 = T[j];
      const float y = y0 + (T[j + 1] - y0) * fr;
      return !isfinite(vf) ? __builtin_nanf("") : span ? y : 1.0f;
    };
    row_elements(F, row - F.row0, [&](auto v, float* out, int x) {
      if constexpr (sizeof(v) == sizeof(Float4)) {
        Float4 o;
        o.x = eq(v.x); o.y = eq(v.y); o.z = eq(v.z); o.w = eq(v.w);
        store4(out + x, o);
      } else {
        gst(out + x, eq(v));
      }
    });
  }
}

}  // namespace ipp
