// asinh gray-scale stretch y = b * asinh(v / a) and its backward
// (Sec. 2.2.6: per-pixel gray-scale maps ahead of neural networks).
// Element-wise and HBM-bound: 8 B/px forward (read v, write y), 12 B/px
// backward (read v and dL/dy, write dL/dv).  The parameter gradients are
// binary64 block partials reduced in a fixed order by one workgroup.
#include <mutex>

#include <type_traits>

#include "ipp_internal.h"
#include "kernels.h"

namespace ipp {

// Scratch of the allocation-free backward: the binary64 block partials of
// the two parameter gradients.  One copy per GPU, held until the process
// ends.  In host code `scratch` names a host-side stand-in, never the
// device memory: kernels are given the address from asinh_scratch().
static __device__ __align__(256) double scratch[2 * kAsinhMaxBlocks];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t asinh_scratch(int device, double** ptr) {
  *ptr = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) hipSetDevice(cur);
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = (double*)p;
  }
  *ptr = g_scratch_ptr[device];
  return hipSuccess;
}

// Elements i (float4 groups when every pointer is 16-byte aligned), two
// groups per thread and step, so that several loads are in flight.
template <typename Fn>
__device__ __forceinline__ void for_elements(int64_t n, bool vec, Fn fn) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  const int64_t i0 = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  int64_t done = 0;
  if (vec) {
    const int64_t n4 = n >> 2;
    for (int64_t i = i0; i < n4; i += 2 * stride) {
      fn(i, true);
      if (i + stride < n4) fn(i + stride, true);
    }
    done = n4 << 2;
  }
  for (int64_t i = done + i0; i < n; i += stride) fn(i, false);
}

// b * asinh(t) in binary32: for |t| < 1/4 the Maclaurin series of asinh
// through t^11 (the first term left out is below 3e-10 relative),
// otherwise ln 2 * log2(|t| + sqrt(t^2 + 1)) with the hardware base-2
// logarithm (its argument is then above 1.28, so the result keeps a
// relative error of a few 1e-7), and log2|t| + 1 where t^2 would overflow.
__device__ __forceinline__ float stretch(float x, float inv_a, float b) {
  const float t = x * inv_a;
  const float at = fabsf(t);
  const float t2 = at * at;
  float p = -63.0f / 2816.0f;
  p = fmaf(p, t2, 35.0f / 1152.0f);
  p = fmaf(p, t2, -5.0f / 112.0f);
  p = fmaf(p, t2, 3.0f / 40.0f);
  p = fmaf(p, t2, -1.0f / 6.0f);
  const float ser = fmaf(at * t2, p, at);
  const float u = at + sqrtf(fmaf(at, at, 1.0f));
  const float lg = at > 1e18f ? __builtin_amdgcn_logf(at) + 1.0f
                              : __builtin_amdgcn_logf(u);
  const float big = 0.693147180559945f * lg;
  return b * copysignf(at < 0.25f ? ser : big, t);
}

// Parameters read on the device: (a, b) = ab[0..1].  A non-positive or
// non-finite a, or a non-finite b, makes every output NaN (the host cannot
// check values it never sees).
__device__ __forceinline__ bool device_params(const double* ab, double* a,
                                              double* b) {
  *a = ab[0];
  *b = ab[1];
  return *a > 0.0 && isfinite(*a) && isfinite(*b);
}

__global__ __launch_bounds__(kBlock) void k_asinh_fwd(const float* v,
                                                      float* y, int64_t n,
                                                      float inv_a, float b,
                                                      const double* ab) {
  if (ab) {
    double ad, bd;
    const bool ok = device_params(ab, &ad, &bd);
    inv_a = ok ? (float)(1.0 / ad) : __builtin_nanf("");
    b = ok ? (float)bd : __builtin_nanf("");
  }
  const bool vec = (((uintptr_t)v | (uintptr_t)y) & 15) == 0;
  for_elements(n, vec, [&](int64_t i, bool four) {
    if (four) {
      float4 x = ((const float4*)v)[i];
      x.x = stretch(x.x, inv_a, b);
      x.y = stretch(x.y, inv_a, b);
      x.z = stretch(x.z, inv_a, b);
      x.w = stretch(x.w, inv_a, b);
      ((float4*)y)[i] = x;
    } else {
      y[i] = stretch(v[i], inv_a, b);
    }
  });
}

// ln(1 + y) for y >= 0 in binary64: 1 + y = m 2^e with m in [1, 2), and
// ln(1 + y) = e ln 2 - ln c + ln(1 + x) with c near 1 / m from a table over
// the first seven bits of m and x = m c - 1, |x| < 2^-7 (for e = 0 formed
// as y c + (c - 1), and c = 1 in the first interval, so that small y keep
// every digit): the Maclaurin series through x^8 (the first term left out
// is below 2e-18 relative).
// ln 2 is split in two parts (Cody and Waite's argument-reduction split: a
// 30-bit leading part, so that e times it is exact, and the remainder).
constexpr int kLogBits = 7;
struct LogEntry {
  double c, t;                             // c and -ln c
};
__device__ __forceinline__ LogEntry log_entry(int i) {
  LogEntry e;
  e.c = i == 0 ? 1.0 : 1.0 / (1.0 + ((double)i + 0.5) / (1 << kLogBits));
  e.t = -log(e.c);
  return e;
}
__device__ __forceinline__ double log1p_pos(double y, const LogEntry* tab) {
  const double u = 1.0 + y;
  const uint32_t hi = (uint32_t)__double2hiint(u);
  const int e = (int)(hi >> 20) - 1023;    // u >= 1 (NaN: masked below)
  const int i = (int)(hi >> (20 - kLogBits)) & ((1 << kLogBits) - 1);
  const double m =
      __hiloint2double((int)((hi & 0xFFFFFu) | 0x3FF00000u), __double2loint(u));
  const LogEntry q = tab[i];
  const double x = fma(e == 0 ? y : m, q.c, (e == 0 ? q.c : 0.0) - 1.0);
  double p = -1.0 / 8.0;
  p = fma(p, x, 1.0 / 7.0);
  p = fma(p, x, -1.0 / 6.0);
  p = fma(p, x, 1.0 / 5.0);
  p = fma(p, x, -1.0 / 4.0);
  p = fma(p, x, 1.0 / 3.0);
  p = fma(p, x, -1.0 / 2.0);
  const double l = fma(x * x, p, x);       // ln(1 + x)
  const double ed = (double)e;
  const double ln2_hi = 6.93147180369123816490e-01;   // 30 leading bits
  const double ln2_lo = 1.90821492927058770002e-10;   // ln 2 - ln2_hi
  const double r = fma(ed, ln2_hi, q.t + fma(ed, ln2_lo, l));
  return fma(y, 0.0, r);                   // NaN for y infinite or NaN
}

// One element of the backward.  With r = sqrt(a^2 + v^2) and y = 1 / r,
// both from one reciprocal square root (no division, no square root):
//   dy/dv = b y,
//   dy/da = -(b / a) v y, summed as v y (the factor at the end),
//   asinh(v / a) = sign(v) log1p((|v| + (r - a)) / a),
// where r - a is corrected by the remainder v^2 - (r - a)(r + a), so that it
// keeps its digits for |v| far below a.
template <bool TINY>
__device__ __forceinline__ void asinh_bwd_one(float x, float g, double a,
                                              double a2, double inv_a,
                                              double b, bool want_ab,
                                              const LogEntry* tab, float* dv,
                                              double& pa, double& pb) {
  if (!want_ab) {
    const float af = (float)a, bf = (float)b;
    *dv = g * (bf / sqrtf(af * af + x * x));
    return;
  }
  if (TINY && x == 0.0f) {           // a^2 is zero, but 1 / r is 1 / a
    *dv = g * (float)(b * inv_a);
    return;
  }
  const double xd = (double)x, gd = (double)g;
  const double s = fma(xd, xd, a2);
  // the hardware's reciprocal square root, two Newton steps, then r and y
  // corrected by their own remainders
  double y = __builtin_amdgcn_rsq(s);
  y = fma(0.5 * y, fma(-s * y, y, 1.0), y);
  y = fma(0.5 * y, fma(-s * y, y, 1.0), y);
  double r = s * y;
  r = fma(fma(-r, r, s), 0.5 * y, r);
  y = fma(fma(-r, y, 1.0), y, y);
  *dv = g * (float)(b * y);
  pa = fma(gd, xd * y, pa);
  const double d = r - a;
  const double w = fma(fma(-d, r + a, xd * xd), 0.5 * y, d);
  const double as = log1p_pos((fabs(xd) + w) * inv_a, tab);
  pb = fma(gd, copysign(as, xd), pb);
}

// HBM traffic of 12 B per element (read v and dL/dy, write dL/dv); with a
// division, a square root and a logarithm's division per element in binary64
// it was bound by their issue (293 us for 67.1 million elements); 67 vector
// instructions per element now fill 114 of its 187 us (4.3 TB/s).  Loading
// the next group before working on one changes nothing (190 us).
__global__ __launch_bounds__(kBlock) void k_asinh_bwd(const float* v,
                                                      const float* dy,
                                                      float* dv, int64_t n,
                                                      double a, double b,
                                                      const double* ab,
                                                      double* partial) {
  __shared__ double red[kWaves];
  if (ab && !device_params(ab, &a, &b)) a = b = __builtin_nan("");
  const double inv_a = 1.0 / a, a2 = a * a;
  const bool want_ab = partial != nullptr;
  __shared__ LogEntry tab[1 << kLogBits];
  if (want_ab) {
    for (int i = threadIdx.x; i < (1 << kLogBits); i += kBlock)
      tab[i] = log_entry(i);
    __syncthreads();
  }
  double pa = 0.0, pb = 0.0;
  const bool vec =
      (((uintptr_t)v | (uintptr_t)dy | (uintptr_t)dv) & 15) == 0;
  auto element = [&](auto tiny, float x, float g, float* o) {
    asinh_bwd_one<tiny.value>(x, g, a, a2, inv_a, b, want_ab, tab, o, pa, pb);
  };
  auto walk = [&](auto tiny) {
    for_elements(n, vec, [&](int64_t i, bool four) {
      if (four) {
        const float4 x = ((const float4*)v)[i];
        const float4 g = ((const float4*)dy)[i];
        float4 o;
        element(tiny, x.x, g.x, &o.x);
        element(tiny, x.y, g.y, &o.y);
        element(tiny, x.z, g.z, &o.z);
        element(tiny, x.w, g.w, &o.w);
        if (dv) ((float4*)dv)[i] = o;
      } else {
        float o;
        element(tiny, v[i], dy[i], &o);
        if (dv) dv[i] = o;
      }
    });
  };
  // a below 1.5e-162: a loop of its own (the test in every element's way:
  // 289 against 285 us forward and backward)
  if (a2 == 0.0) walk(std::true_type{});
  else walk(std::false_type{});
  if (!want_ab) return;
  pa = block_sum(pa, red) * (-b * inv_a);
  pb = block_sum(pb, red);
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = pa;
    partial[2 * blockIdx.x + 1] = pb;
  }
}

__global__ __launch_bounds__(kBlock) void k_asinh_bwd_final(
    const double* partial, int nb, double* out) {
  __shared__ double red[kWaves];
  double pa = 0.0, pb = 0.0;
  for (int i = threadIdx.x; i < nb; i += kBlock) {
    pa += partial[2 * i];
    pb += partial[2 * i + 1];
  }
  pa = block_sum(pa, red);
  pb = block_sum(pb, red);
  if (threadIdx.x == 0) {
    out[0] = pa;
    out[1] = pb;
  }
}

}  // namespace ipp
