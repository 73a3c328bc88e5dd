// Stamp convolution and image subtraction (Sec. 2.2.4, Eq. 8-10): the
// template R is convolved with a spatially varying kernel
//   K(u, v) = sum_n a_n(x, y) exp(-(u^2 + v^2) / (2 sigma_k^2)) u^i v^j
// and the difference D = (I + B) - R (x) K is written.  As in the paper's
// GPU design, the image is cut into stamps (21 x 21 by default); here one
// wavefront handles one stamp, or a workgroup a larger one: the stamp's kernel (a_n and B evaluated at
// the stamp centre) is built in binary64 and kept in LDS as binary32, the
// template tile with its (2 hw)-pixel margin is staged in LDS (zero outside
// the frame), and each output pixel sums its (2hw+1)^2 products in binary32
// per kernel column, the columns in binary64: the error stays below
// (2hw + 2) 2^-24 of sum |K| |R|.  One HBM read of I and R and one write
// of D per pixel (12 B/px); the tile re-reads its margin from L2.
#include "ipp_internal.h"
#include "kernels.h"

namespace ipp {

namespace {
__device__ __forceinline__ double norm_c(double x, int n) {
  return n > 1 ? (2.0 * x - (double)(n - 1)) / (double)(n - 1) : 0.0;
}

// sum c_pq xn^p yn^q over p = 0..d, q = 0..d-p, in that order
__device__ double poly2(const double* c, int d, double xn, double yn) {
  double tot = 0.0;
  int k = 0;
  double xp = 1.0;
  for (int p = 0; p <= d; ++p) {
    double yq = 1.0;
    for (int q = 0; q <= d - p; ++q) {
      tot += c[k++] * xp * yq;
      yq *= yn;
    }
    xp *= xn;
  }
  return tot;
}

// Orders the wave's own LDS accesses.
__device__ __forceinline__ void sub_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
}  // namespace

// LDS (dynamic, laid out by sub_layout): per workgroup the one-dimensional
// basis factors E[g][k][d] = exp(-d^2 / (2 sigma_g^2)) d^k of every Gaussian
// g and power k (the same table serves u and v); per wavefront the stamp's
// kernel in columns (column u: its taps v, padded to whole float4s), and one
// region that holds first a_n and the row factors T[g][i][v] =
// sum_j a_gij E[g][j][v] and then the template tile with its margin.
constexpr int kSubRows = 7;          // outputs per thread, in one column (R)
constexpr int kSubFine = 4;          // the same where a workgroup has a stamp
constexpr int kSubStamp = 21;        // stamps up to this size: narrow tile
struct SubLayout {
  int nw;              // wavefronts per workgroup
  int ne;              // (g, k) pairs
  int wave_off;        // bytes of the workgroup's tables
  int ker_bytes;       // bytes of a wavefront's kernel
  int wave_bytes;      // bytes of a wavefront's slice
};
__host__ __device__ inline int sub_groups(int stamp, int R) {
  return (stamp + R - 1) / R;
}
// Row stride of the template tile, and the offset of tile row r: 22 words
// between groups of kSubRows rows, so that with the default 21-pixel stamps
// and 21 x 21 kernels the row groups of a wavefront start 21 banks apart
// and its 63 threads meet different banks.
constexpr int kSubGap = 22;
constexpr int kSubMaxRows = kSubMaxGauss * (kSubMaxOrder + 1);
__host__ __device__ constexpr int sub_tstride(int hw, int stamp) {
  return (2 * hw + (stamp <= kSubStamp ? kSubStamp : kSubMaxStamp)) | 1;
}
__host__ __device__ constexpr int sub_tile_at(int r, int stride, int R) {
  return r * stride + (r / R) * kSubGap;
}
static SubLayout sub_layout(const SubBasis& bs, int R) {
  SubLayout l;
  const int kw = 2 * bs.hw + 1;
  l.ne = 0;
  for (int g = 0; g < bs.ngauss; ++g) l.ne += bs.order[g] + 1;
  l.wave_off = kSubMaxRows * (int)sizeof(int4) +
               ((l.ne * kw * (int)sizeof(double) + 15) & ~15);
  l.ker_bytes = kw * ((kw + 3) & ~3) * (int)sizeof(float);
  const int head = ((bs.nbasis + 1) + l.ne * kw) * (int)sizeof(double);
  // whole groups of R output rows
  const int tile = sub_tile_at(R * sub_groups(bs.stamp, R) + 2 * bs.hw,
                               sub_tstride(bs.hw, bs.stamp), R) *
                   (int)sizeof(float);
  l.wave_bytes = l.ker_bytes + (((head > tile ? head : tile) + 15) & ~15);
  l.nw = (65536 - l.wave_off) / l.wave_bytes;
  l.nw = l.nw > kWaves ? kWaves : l.nw;
  return l;
}

// One wavefront per stamp, up to four stamps side by side in a workgroup,
// no workgroup barrier after the tables.  A thread computes kSubRows outputs
// of one column: for a 21-pixel stamp 21 x 3 threads, 63 of 64 lanes and no
// idle output.  Per kernel column it reads its kSubRows + 2 HW template
// values (neighbouring lanes read neighbouring words) and the column's taps
// (a broadcast) from LDS for kSubRows (2 HW + 1) FMAs; four adjacent outputs
// of a row per thread needed twice the LDS words per FMA and left 13 % of
// the outputs idle.  Each output sums half a kernel column's products at a
// time in binary32, taps in order, and the columns in binary64.  The kernel
// is built from its separable factors: 15 products per tap for the default
// 49 terms instead of 49, and no exponential per tap.
// Bound by VALU issue (5,290 vector instructions per stamp, 3,087 of them
// the convolution's FMAs; issuing them takes over 90 % of the time): 344 -> 219 us
// for the 10.3 Mpx of two frame pairs of 2047 x 3001 and 2048 x 2048 (26 -> 41
// TFLOP/s of the 78.6 that unpacked FP32 FMAs reach).  Stamps up to 21 pixels
// take the narrow tile (7 KB: four wavefronts per SIMD fit the LDS), larger
// ones the wide one (16 KB).
// SHARED: a workgroup of one wavefront per 64 threads' outputs takes a stamp
// (see launch_subtract), each step split over its threads; the sums are the
// same.
template <int HW, int STAMP, bool SHARED, int R>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(HW <= 10 ? 4 : 2))) void k_subtract_t(
    const SubFrame* frames, int nframes, SubBasis bs, SubLayout l,
    int64_t total_stamps) {
  constexpr int KW = 2 * HW + 1;
  constexpr int KR = (KW + 3) / 4;            // float4s of a kernel column
  constexpr int KS = 4 * KR;
  constexpr int NRV = R + 2 * HW;      // template values per column
  extern __shared__ __align__(16) unsigned char sub_lds[];
  constexpr int TS = sub_tstride(HW, STAMP);
  int4* rows = (int4*)sub_lds;                // of each (g, i): a0, e0, count
  double* E = (double*)(rows + kSubMaxRows);  // [g, k][d + HW]
  // this thread of the N that share a stamp; the stamp's slot in the workgroup
  const int N = SHARED ? (int)blockDim.x : kWave;
  const int lane = SHARED ? (int)threadIdx.x : (int)threadIdx.x & (kWave - 1);
  const int wv =
      SHARED ? 0
             : __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  auto sync = [] {
    if constexpr (SHARED) __syncthreads();
    else sub_sync();
  };
  unsigned char* mine = sub_lds + l.wave_off + wv * l.wave_bytes;
  float* ker = (float*)mine;                  // [u][v]
  double* a_s = (double*)(mine + l.ker_bytes);
  double* T = a_s + bs.nbasis + 1;            // [g, i][v]
  float* tile = (float*)(mine + l.ker_bytes);

  for (int e = threadIdx.x; e < l.ne * KW; e += blockDim.x) {
    int gk = e / KW, g = 0;
    const double d = (double)(e - gk * KW - HW);
    while (gk > bs.order[g]) gk -= bs.order[g++] + 1;
    double v = exp(-(d * d) / (2.0 * bs.sigma[g] * bs.sigma[g]));
    for (int k = 0; k < gk; ++k) v *= d;
    E[e] = v;
  }
  if ((int)threadIdx.x < l.ne) {
    int i = threadIdx.x, g = 0, a0 = 0, e0 = 0;  // a0, e0: first of Gaussian g
    while (i > bs.order[g]) {
      const int o = bs.order[g++] + 1;
      i -= o;
      e0 += o;
      a0 += o * (o + 1) / 2;
    }
    const int o = bs.order[g];
    rows[threadIdx.x] = make_int4(a0 + i * (o + 1) - i * (i - 1) / 2, e0,
                                  o - i + 1, 0);
  }
  __syncthreads();

  const int S = bs.stamp;
  const int64_t nwv = (int64_t)gridDim.x * l.nw;
  for (int64_t st = (int64_t)blockIdx.x * l.nw + wv; st < total_stamps;
       st += nwv) {
    int f = 0, hi = nframes - 1;              // frame of this stamp
    while (f < hi) {
      const int mid = (f + hi + 1) >> 1;
      if (frames[mid].stamp0 <= st) f = mid; else hi = mid - 1;
    }
    const SubFrame fr = frames[f];
    const int64_t ls = st - fr.stamp0;
    const int sy = (int)(ls / fr.nsx), sx = (int)(ls - (int64_t)sy * fr.nsx);
    const int x0 = sx * S, y0 = sy * S;
    const int x1 = min(x0 + S, fr.w), y1 = min(y0 + S, fr.h);
    const double xc = (double)(x0 + x1 - 1) / 2.0;
    const double yc = (double)(y0 + y1 - 1) / 2.0;
    const double xn = norm_c(xc, fr.w), yn = norm_c(yc, fr.h);
    const int ns = (bs.spatial_order + 1) * (bs.spatial_order + 2) / 2;
    for (int n = lane; n <= bs.nbasis; n += N)
      a_s[n] = poly2(fr.coef + (int64_t)n * ns,
                     n < bs.nbasis ? bs.spatial_order : bs.bkg_order, xn, yn);
    sync();
    const double B = a_s[bs.nbasis];
    // row factors T[g, i][v]
    for (int e = lane; e < l.ne * KW; e += N) {
      const int row = e / KW, vv = e - row * KW;
      const int4 d = rows[row];
      double t = 0.0;
      for (int j = 0; j < d.z; ++j)
        t = fma(a_s[d.x + j], E[(d.y + j) * KW + vv], t);
      T[e] = t;
    }
    sync();
    // the kernel in binary64, kept as binary32 (column padding 0)
    for (int e = lane; e < KW * KS; e += N) {
      const int uu = e / KS, vv = e - uu * KS;
      double k = 0.0;
      if (vv < KW)
#pragma unroll 5
        for (int r = 0; r < l.ne; ++r)
          k = fma(E[r * KW + uu], T[r * KW + vv], k);
      ker[e] = (float)k;
    }
    sync();                            // T is read, the tile takes its place
    // template tile with its margin, zero outside the frame; the loads of
    // eight rounds are issued before the first is stored (32-bit byte
    // offsets from the tile's first in-frame row)
    {
      const int tw = S + 2 * HW, tn = tw * tw;
      const int dr = N / tw, dc = N - (N / tw) * tw;
      const int gy0 = y0 - HW, gx0 = x0 - HW, ry0 = max(gy0, 0);
      const char* rp =
          uniform_ptr((const char*)(fr.R + (int64_t)ry0 * fr.pitchR));
      const uint32_t pitchB = (uint32_t)fr.pitchR * 4u;
      const bool inside =
          gy0 >= 0 && gx0 >= 0 && gy0 + tw <= fr.h && gx0 + tw <= fr.w;
      int ty = lane / tw, tx = lane - (lane / tw) * tw;
      for (int e0 = 0; e0 < tn; e0 += 8 * N) {
        float r[8];
        int at[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          // a lane past the tile's end repeats a pixel of its last row
          const int wy = min(ty, tw - 1);
          const int gx = gx0 + tx;
          if (inside) {
            r[c] = gld((const float*)(
                rp + ((uint32_t)wy * pitchB + (uint32_t)gx * 4u)));
          } else {
            const int gy = gy0 + wy;
            const bool in =
                (gy >= 0) & (gy < fr.h) & (gx >= 0) & (gx < fr.w);
            const uint32_t o = (uint32_t)(gy - ry0) * pitchB + (uint32_t)gx * 4u;
            const float v = gld((const float*)(rp + (in ? o : 0u)));
            r[c] = in ? v : 0.0f;
          }
          // wy / R for wy < 64
          static_assert(R == 7 || R == 4, "37 / 256 divides by 7");
          at[c] = wy * TS + tx + (R == 7 ? (wy * 37) >> 8 : wy >> 2) * kSubGap;
          ty += dr;
          tx += dc;
          if (tx >= tw) {
            tx -= tw;
            ++ty;
          }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) tile[at[c]] = r[c];
      }
    }
    sync();
    const int ow = x1 - x0, oh = y1 - y0;
    const int items = S * sub_groups(S, R);
    for (int e0 = 0; e0 < items; e0 += N) {
      const int e = min(e0 + lane, items - 1);
      const int g = e / S, lx = e - g * S;
      double acc[R];
#pragma unroll
      for (int i = 0; i < R; ++i) acc[i] = 0.0;
      // R(x - u, y - v) = tile[ly + 2HW - vv][lx + 2HW - uu]
      const float* tcol = tile + g * sub_tile_at(R, TS, R) + lx + 2 * HW;
#pragma unroll 3
      for (int uu = 0; uu < KW; ++uu) {          // uu = u + HW
        float r[NRV], kr[4 * KR];
#pragma unroll
        for (int k = 0; k < NRV; ++k) r[k] = tcol[sub_tile_at(k, TS, R) - uu];
        const float4* kcol = (const float4*)(ker + uu * KS);
#pragma unroll
        for (int q = 0; q < KR; ++q) {
          const float4 a = kcol[q];
          kr[4 * q] = a.x; kr[4 * q + 1] = a.y;
          kr[4 * q + 2] = a.z; kr[4 * q + 3] = a.w;
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
          // two partial sums of half a column each
          float ra = 0.0f, rb = 0.0f;
#pragma unroll
          for (int vv = 0; vv < HW; ++vv)        // vv = v + HW
            ra = fmaf(kr[vv], r[i + 2 * HW - vv], ra);
#pragma unroll
          for (int vv = HW; vv < KW; ++vv)
            rb = fmaf(kr[vv], r[i + 2 * HW - vv], rb);
          acc[i] += (double)(ra + rb);
        }
      }
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int ly = R * g + i;
        if (e0 + lane < items && lx < ow && ly < oh) {
          const int64_t gy = y0 + ly, gx = x0 + lx;
          const double I = (double)gld(fr.I + gy * fr.pitchI + gx);
          gst(fr.D + gy * fr.w + gx, (float)((I + B) - acc[i]));
        }
      }
    }
    sync();                            // the slice is reused
  }
}

hipError_t launch_subtract(const SubFrame* frames, int nframes,
                           const SubBasis& bs, int64_t stamps,
                           hipStream_t s) {
  // Stamps over 21 pixels have outputs for several wavefronts, and their slices
  // leave few wavefronts a compute unit: a workgroup takes one, with four
  // outputs a thread while the stamps are few or the column's last group would
  // be short (28 of 35 rows), but a wavefront each where kernels are small and
  // stamps many.  Stamps of 32, half-width 15, 49 and 16,000 of them: 27 and
  // 515 us (84 and 1013 as a wavefront each, 36 and 671 with seven outputs a
  // thread); of 25, half-width 10, 26,240: 402 (506; 446 with four outputs);
  // of 25, half-width 5, 1,440 and 26,240: 24 and 179 (26 and 153); of 28,
  // half-width 7, 5,328 and 21,021: 67 and 206 (78 and 202).
  const bool wide = bs.stamp > kSubStamp;
  const bool shared =
      wide && (bs.hw > 7 || stamps < (bs.hw > 5 ? 8192 : 2048));
  const bool fine = shared && (stamps < 1024 || bs.stamp > 4 * kSubRows);
  const int R = fine ? kSubFine : kSubRows;
  SubLayout l = sub_layout(bs, R);
  // Two stamps per wavefront: the basis table is shared by eight stamps and
  // the last round of workgroups stays short.  Few stamps are spread over the
  // compute units instead, a wavefront each (half-width 5, 110 stamps: 34
  // against 19 us; half-width 10, 2,496 stamps of 1000 x 1100: 57 before the
  // wavefront per stamp, 43).
  int per = 2;
  if (stamps < 1024 * l.nw) per = 1;
  while (l.nw > 1 && stamps < 512 * l.nw) l.nw /= 2;
  const int items = bs.stamp * sub_groups(bs.stamp, R);
  int64_t nb = (stamps + per * l.nw - 1) / (per * l.nw);
  int threads = l.nw * kWave;
  if (shared) {
    l.nw = 1;
    nb = stamps;
    threads = (items + kWave - 1) / kWave * kWave;
  }
  const dim3 g((unsigned)(nb < (1 << 20) ? nb : (1 << 20)));
  const dim3 b(threads);
  const size_t lds = (size_t)l.wave_off + (size_t)l.nw * l.wave_bytes;
  switch (bs.hw) {
#define IPP_SUB_LAUNCH(H, STAMP, SHARED, ROWS)                            \
  hipLaunchKernelGGL((k_subtract_t<H, STAMP, SHARED, ROWS>), g, b, lds, s, \
                     frames, nframes, bs, l, stamps)
#define IPP_SUB_CASE(H)                                                   \
  case H:                                                                 \
    if (!wide)                                                            \
      IPP_SUB_LAUNCH(H, kSubStamp, false, kSubRows);                      \
    else if (!shared)                                                     \
      IPP_SUB_LAUNCH(H, kSubMaxStamp, false, kSubRows);                   \
    else if (!fine)                                                       \
      IPP_SUB_LAUNCH(H, kSubMaxStamp, true, kSubRows);                    \
    else                                                                  \
      IPP_SUB_LAUNCH(H, kSubMaxStamp, true, kSubFine);                    \
    break;
    IPP_SUB_CASE(1) IPP_SUB_CASE(2) IPP_SUB_CASE(3) IPP_SUB_CASE(4)
    IPP_SUB_CASE(5) IPP_SUB_CASE(6) IPP_SUB_CASE(7) IPP_SUB_CASE(8)
    IPP_SUB_CASE(9) IPP_SUB_CASE(10) IPP_SUB_CASE(11) IPP_SUB_CASE(12)
    IPP_SUB_CASE(13) IPP_SUB_CASE(14) IPP_SUB_CASE(15)
#undef IPP_SUB_CASE
#undef IPP_SUB_LAUNCH
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ipp
