// AUTO (Kron) photometry (Sec. 2.2.5 lists auto photometry among the
// per-object measurements; Sec. 3.3 compares its magnitudes).
//
// One wavefront per object, in a workgroup of its own.  The object's
// second moments (x2, y2, xy), regularised by the variance 1/12 of a
// uniform unit pixel on each axis, give the quadratic form
//   q(dx, dy) = (Y dx^2 + X dy^2 - 2 xy dx dy) / det,  det = X Y - xy^2,
// (q = 1 on the one-sigma ellipse).  Pass 1: over the pixel centres with
// q <= search^2, r1 = sum sqrt(q) v / sum v (v = I - B32); the Kron radius
// is R = max(k r1, R_min), or R_min when the sums are unusable.  Pass 2:
// over the pixels of the ellipse q <= R^2, the AUTO flux sum w v and area
// sum w, w the exact pixel overlap: u = L d (L the upper Cholesky factor
// of the form / R^2) maps the ellipse onto the unit disk and the pixel
// onto a parallelogram, whose intersection with the disk is summed edge by
// edge (a triangle where an edge piece lies inside the disk, a circular
// sector where it lies outside), then divided by det L.  A pixel whose
// four corners lie inside the ellipse (q <= R^2 with a relative margin of
// 1e-12) is wholly inside it, its area exactly 1; only the other member
// pixels are listed (LDS) and then computed, every lane busy.  A window of
// more than kKronBigPx pixels (wide moments, or a large R where the first
// moment's weights nearly cancel: up to the whole frame) would hold one
// wavefront for hundreds or thousands of rounds: such a pass (with its pass 1
// when the search window is the large one) is cut into parts of kKronPart
// pixels that the whole grid shares, and the parts' sums are added in a
// fixed order.
//
// The membership tests (q against search^2, the frame bounds) use the
// same binary64 operations as the oracle; the sums are taken over the
// wavefront in a fixed order (deterministic, equal to the oracle's
// sequential sums to rounding).
#include "ipp_internal.h"
#include "kernels.h"
#include "phot_geom.h"

namespace ipp {

namespace {

__device__ __forceinline__ double qform(double X, double Y, double xy,
                                        double det, double dx, double dy) {
  return (Y * dx * dx + X * dy * dy - 2.0 * xy * dx * dy) / det;
}

// Smallest q over the square [x0, x1] x [y0, y1] of offsets: 0 when the
// centre lies in it, else the smallest edge minimum (the stationary point
// of q along the edge, clamped to it).
__device__ double min_q(double X, double Y, double xy, double det, double x0,
                        double x1, double y0, double y1) {
  if (x0 <= 0.0 && 0.0 <= x1 && y0 <= 0.0 && 0.0 <= y1) return 0.0;
  double best = __builtin_inf();
  const double xs[2] = {x0, x1}, ys[2] = {y0, y1};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double dx = xs[k];
    const double dy = fmin(fmax(xy * dx / X, y0), y1);
    best = fmin(best, qform(X, Y, xy, det, dx, dy));
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double dy = ys[k];
    const double dx = fmin(fmax(xy * dy / Y, x0), x1);
    best = fmin(best, qform(X, Y, xy, det, dx, dy));
  }
  return best;
}

// Area of the unit disk inside the triangle (0, a, b): the edge is cut at
// its crossings with the circle; the piece between them lies inside the
// disk and adds its triangle to tri, the others turn (re, im) by their
// sectors' angles, or with ONE unset add those angles to ang (from the atan
// series table coef).
template <bool ONE>
__device__ __forceinline__ void disk_tri(double ax, double ay, double bx,
                                         double by, AtanCoef coef,
                                         double& tri, double& re, double& im,
                                         double& ang) {
#pragma clang fp contract(fast)
  const double dx = bx - ax, dy = by - ay;
  const double A = dx * dx + dy * dy;
  const double B = ax * dx + ay * dy;
  const double C = ax * ax + ay * ay - 1.0;
  const double disc = B * B - A * C;
  if (A == 0.0) return;
  const bool cross = disc > 0.0;
  const double s = sqrt(cross ? disc : 0.0);
  const double i = 1.0 / A;
  // the crossings, clamped to the edge (none: one piece, outside)
  const double t0 = cross ? fmin(fmax((-B - s) * i, 0.0), 1.0) : 1.0;
  const double t1 = cross ? fmin(fmax((-B + s) * i, 0.0), 1.0) : 1.0;
  const double px = ax + t0 * dx, py = ay + t0 * dy;
  const double qx = ax + t1 * dx, qy = ay + t1 * dy;
  auto sector = [&](bool some, double gx, double gy, double hx, double hy) {
    if constexpr (ONE) {
      const double c = some ? gx * hx + gy * hy : 1.0;
      const double n = some ? gx * hy - hx * gy : 0.0;
      const double nre = re * c - im * n;
      im = re * n + im * c;
      re = nre;
    } else if (some) {
      ang += angle_of(gx * hx + gy * hy, gx * hy - hx * gy, coef);
    }
  };
  sector(t0 > 0.0, ax, ay, px, py);
  tri += t1 > t0 ? px * qy - qx * py : 0.0;
  sector(t1 < 1.0, qx, qy, bx, by);
}

struct Ell {
  double l11, l12, l22, inv_det;   // unit-disk map and 1 / det L
  bool one;      // an ellipse's arc inside one pixel is below half of it
};

__device__ __forceinline__ Ell ell_map(double X, double Y, double xy,
                                       double det, double R) {
  const double s = det * R * R;
  const double a = Y / s, b = -xy / s, c = X / s;
  Ell e;
  e.l11 = sqrt(a);
  e.l12 = b / e.l11;
  e.l22 = sqrt(c - e.l12 * e.l12);
  e.inv_det = 1.0 / (e.l11 * e.l22);
  // an arc of half the ellipse or more holds two antipodal points, at least
  // twice the minor semi-axis apart: more than a pixel's diagonal once that
  // exceeds 3/4 (lambda_min R^2 > 9/16, lambda_min = det / lambda_max and
  // lambda_max at most the trace)
  e.one = det * R * R > 0.5625 * (X + Y);
  return e;
}

// Exact area of pixel (px, py) inside the ellipse centred at (cx, cy).
__device__ double ell_overlap(const Ell& e, double cx, double cy, int px,
                              int py, AtanCoef coef) {
  const double x0 = (double)px - 0.5 - cx, x1 = (double)px + 0.5 - cx;
  const double y0 = (double)py - 0.5 - cy, y1 = (double)py + 0.5 - cy;
  // corners in counter-clockwise order for x right, y up: a positive sum
  const double ux[4] = {e.l11 * x0 + e.l12 * y0, e.l11 * x1 + e.l12 * y0,
                        e.l11 * x1 + e.l12 * y1, e.l11 * x0 + e.l12 * y1};
  const double uy[4] = {e.l22 * y0, e.l22 * y0, e.l22 * y1, e.l22 * y1};
  // The sectors' angles sum to the ellipse's arc inside the pixel; below
  // half a turn they are composed as one rotation and one angle returns the
  // sum (each edge has up to two sectors, and a lane's wave takes them all:
  // eight angle evaluations otherwise).
  double tri = 0.0, re = 1.0, im = 0.0, ang = 0.0;
  if (e.one) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      disk_tri<true>(ux[k], uy[k], ux[(k + 1) & 3], uy[(k + 1) & 3], coef,
                     tri, re, im, ang);
    ang = rotor_angle(re, im, coef);
  } else {
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
      // corners k and k + 1, selected (no indexed registers)
      const double ax = k < 2 ? (k == 0 ? ux[0] : ux[1])
                              : (k == 2 ? ux[2] : ux[3]);
      const double bx = k < 2 ? (k == 0 ? ux[1] : ux[2])
                              : (k == 2 ? ux[3] : ux[0]);
      disk_tri<false>(ax, k < 2 ? uy[0] : uy[2], bx,
                      k == 0 || k == 3 ? uy[0] : uy[2], coef, tri, re, im,
                      ang);
    }
  }
  return 0.5 * (tri + ang) * e.inv_det;
}

constexpr int kCut = 1024;     // listed pixels per flush (a multiple of 64)
constexpr int kChunk = 4;      // rounds whose loads are issued together

__device__ __forceinline__ int lo_px(double v, int a) {
  return (int)fmax(ceil(v), (double)a);
}
__device__ __forceinline__ int hi_px(double v, int b) {
  return (int)fmin(floor(v), (double)b);
}

// A row's inputs: frame, centre and the moments regularised by the
// variance 1/12 of a uniform unit pixel; ok = all usable.
struct KronRow {
  int f;
  double cx, cy, X, Y, xy, det;
  bool ok;
};

__device__ __forceinline__ KronRow kron_row(const Work& wk,
                                            const ipp_sources& src,
                                            const double* mom,
                                            long long row) {
  KronRow r;
  r.f = src.frame[row];
  r.cx = src.x[row];
  r.cy = src.y[row];
  r.X = mom[6 * row] + 1.0 / 12.0;
  r.Y = mom[6 * row + 1] + 1.0 / 12.0;
  r.xy = mom[6 * row + 2];
  r.det = r.X * r.Y - r.xy * r.xy;
  r.ok = r.f >= 0 && r.f < wk.nframes && isfinite(r.X) && isfinite(r.Y) &&
         isfinite(r.xy) && r.det > 0.0 && isfinite(r.cx) && isfinite(r.cy) &&
         fabs(r.cx) < 1e9 && fabs(r.cy) < 1e9;
  return r;
}

// Pass-2 window: the Kron ellipse's bounding box within the frame and a
// ring of one pixel around it (an ellipse centred in the frame that reaches
// outside meets the ring: it is convex).
struct KronWin {
  int xa, ya, nwx, npx;
};

__device__ __forceinline__ KronWin kron_window(const FrameDev& fr,
                                               const KronRow& r, double R) {
  const double gx = R * sqrt(r.X), gy = R * sqrt(r.Y);
  const int xa = lo_px(r.cx - gx - 0.5, -1), xb = hi_px(r.cx + gx + 0.5, fr.w);
  const int ya = lo_px(r.cy - gy - 0.5, -1), yb = hi_px(r.cy + gy + 0.5, fr.h);
  KronWin k;
  k.xa = xa;
  k.ya = ya;
  k.nwx = max(xb - xa + 1, 0);
  k.npx = yb >= ya ? k.nwx * (yb - ya + 1) : 0;
  return k;
}

// Pass-1 window: the search ellipse's box within the frame.
__device__ __forceinline__ KronWin search_window(const FrameDev& fr,
                                                 const KronRow& r,
                                                 double search) {
  // bounds clamped in binary64 before the conversion to int
  const double hx = search * sqrt(r.X), hy = search * sqrt(r.Y);
  const int xa = lo_px(r.cx - hx - 0.5, 0), xb = hi_px(r.cx + hx + 0.5, fr.w - 1);
  const int ya = lo_px(r.cy - hy - 0.5, 0), yb = hi_px(r.cy + hy + 0.5, fr.h - 1);
  KronWin k;
  k.xa = xa;
  k.ya = ya;
  k.nwx = xb >= xa ? xb - xa + 1 : 0;
  k.npx = (xb >= xa && yb >= ya) ? k.nwx * (yb - ya + 1) : 0;
  return k;
}

// Pass 1 over search-window pixels [e_begin, e_end) (raster order): the
// sums sqrt(q) v and v over the pixel centres with q <= search^2 and a
// finite I; each lane sums its pixels in window order, the loads of kChunk
// rounds issued before any is used.
__device__ void kron_pass1(const FrameDev& fr, const KronRow& r,
                           double search, const KronWin& kw, int e_begin,
                           int e_end, int lane, double& num, double& den) {
  const int nwx = kw.nwx;
  if (nwx <= 0 || e_end <= e_begin) return;
  const double s2 = search * search;
  const int dwr = kWave / nwx, dwc = kWave - dwr * nwx;
  const int el0 = e_begin + lane;
  int wr = el0 / nwx, wc = el0 - (el0 / nwx) * nwx;
  for (int e0 = e_begin; e0 < e_end; e0 += kChunk * kWave) {
    float Iv[kChunk], Bv[kChunk];
    int pxs[kChunk], pys[kChunk];
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      const bool live = e0 + c * kWave + lane < e_end;
      pxs[c] = live ? kw.xa + wc : -1;
      pys[c] = kw.ya + wr;
      const int qx = live ? kw.xa + wc : kw.xa, qy = live ? kw.ya + wr : kw.ya;
      Iv[c] = fr.pix[(int64_t)qy * fr.pitch + qx];
      Bv[c] = fr.bkg[(int64_t)qy * fr.w + qx];
      wr += dwr;
      wc += dwc;
      if (wc >= nwx) {
        wc -= nwx;
        ++wr;
      }
    }
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      if (pxs[c] < 0) continue;
      const double q = qform(r.X, r.Y, r.xy, r.det, (double)pxs[c] - r.cx,
                             (double)pys[c] - r.cy);
      if (!(q <= s2)) continue;
      if (!isfinite(Iv[c])) continue;
      const double v = (double)Iv[c] - (double)Bv[c];
      num += sqrt(q) * v;
      den += v;
    }
  }
}

// The Kron radius from the first-moment sums (flag 2: R_min used).
__device__ __forceinline__ double kron_radius(double num, double den,
                                              double kfac, double rmin,
                                              uint32_t* fl) {
  const double r1 = den > 0.0 ? num / den : __builtin_nan("");
  if (den > 0.0 && isfinite(r1)) {
    const double R = kfac * r1;
    return R > rmin ? R : rmin;
  }
  *fl |= 2u;
  return rmin;
}

// Pass 2 over window pixels [e_begin, e_end) (raster order): members of
// the open ellipse whose four corners lie inside it add v and area 1, the
// other members are listed and add w v and w, w the exact overlap; a
// member off the frame or not finite sets edge.  Membership is the exact
// predicate min_q < R^2, but most pixels are settled by their centre
// without it: min_q <= q(centre), and sqrt(min_q) >= sqrt(q(centre)) - m
// with m the largest sqrt(q) of a half-pixel corner offset, so a centre
// with q below R^2 (1 - 1e-9) is a member and one above (R + m)^2
// (1 + 1e-9) is not (margins no rounding here can cross); the pixels in
// between (a band along the boundary) are listed and tested exactly, all
// lanes busy.  Per chunk of kCut / 2 window pixels the band is listed
// from the back of `cut`, the cut members from its front.  Each lane
// accumulates the settled members in window order, then the band's, then
// the cut ones; the pixel loads of kChunk rounds are issued before any is
// used (clamped into the frame; only members use them).
__device__ void kron_pass2(const FrameDev& fr, const KronRow& r,
                           const Ell& el, double R, const KronWin& kw,
                           int e_begin, int e_end, int lane, int* cut,
                           double& fs, double& as, bool& edge) {
  const double X = r.X, Y = r.Y, xy = r.xy, det = r.det;
  const double cx = r.cx, cy = r.cy;
  const double R2 = R * R;
  // corners inside: q det <= R^2 det (1 - 1e-12), no division
  const double lim = R2 * det * (1.0 - 1e-12);
  const double m = sqrt(0.25 * (X + Y + 2.0 * fabs(xy)) / det);
  const double lim_in = R2 * det * (1.0 - 1e-9);
  const double lim_out = (R + m) * (R + m) * det * (1.0 + 1e-9);
  auto qd = [&](double dx, double dy) {
    return Y * dx * dx + X * dy * dy - 2.0 * xy * dx * dy;
  };
  // a member pixel with its loaded values: edge, a whole pixel, or listed
  auto member = [&](int px, int py, float I, float B, int pos, bool* listed,
                    int* lpos) {
    const bool in = px >= 0 && px < fr.w && py >= 0 && py < fr.h;
    if (!in || !isfinite(I)) {
      edge = true;
      return;
    }
    const double x0 = (double)px - 0.5 - cx, x1 = (double)px + 0.5 - cx;
    const double y0 = (double)py - 0.5 - cy, y1 = (double)py + 0.5 - cy;
    if (qd(x0, y0) <= lim && qd(x1, y0) <= lim && qd(x0, y1) <= lim &&
        qd(x1, y1) <= lim) {
      fs += (double)I - (double)B;
      as += 1.0;
    } else {
      *listed = true;
      *lpos = pos;
    }
  };
  const int nwx = kw.nwx;
  if (nwx <= 0 || e_end <= e_begin) return;
  // window positions stepped round by round without division
  const int dwr = kWave / nwx, dwc = kWave - dwr * nwx;
  const int el0 = e_begin + lane;
  int sy = el0 / nwx, sx = el0 - (el0 / nwx) * nwx;
  constexpr int kPart = kCut / 2;      // window pixels per chunk
  for (int e0 = e_begin; e0 < e_end; e0 += kPart) {
    int ncut = 0, nband = 0;
    const int e1 = min(e_end, e0 + kPart);
    for (int eb = e0; eb < e1; eb += kChunk * kWave) {
      float Iv[kChunk], Bv[kChunk];
      int wys[kChunk], wxs[kChunk];
#pragma unroll
      for (int c = 0; c < kChunk; ++c) {
        if (eb + c * kWave >= e1) break;             // wave-uniform
        wys[c] = sy;
        wxs[c] = sx;
        const int qx = min(max(kw.xa + sx, 0), fr.w - 1);
        const int qy = min(max(kw.ya + sy, 0), fr.h - 1);
        Iv[c] = fr.pix[(int64_t)qy * fr.pitch + qx];
        Bv[c] = fr.bkg[(int64_t)qy * fr.w + qx];
        sy += dwr;
        sx += dwc;
        if (sx >= nwx) {
          sx -= nwx;
          ++sy;
        }
      }
#pragma unroll
      for (int c = 0; c < kChunk; ++c) {
        if (eb + c * kWave >= e1) break;             // wave-uniform
        const int e = eb + c * kWave + lane;
        bool listed = false, band = false;
        int pos = 0;
        if (e < e1) {
          const int wy = wys[c], wx = wxs[c];
          const int py = kw.ya + wy, px = kw.xa + wx;
          pos = (wy << 16) | wx;
          const double qc = qd((double)px - cx, (double)py - cy);
          if (qc <= lim_in) {
            int lp = 0;
            member(px, py, Iv[c], Bv[c], pos, &listed, &lp);
          } else {
            band = !(qc >= lim_out);
          }
        }
        const uint64_t bb = ballot(band);
        if (band) cut[kCut - 1 - (nband + lanes_before(bb))] = pos;
        nband += __popcll(bb);
        const uint64_t b = ballot(listed);
        if (listed) cut[ncut + lanes_before(b)] = pos;
        ncut += __popcll(b);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // the band: the exact predicate, then as any member
    for (int j0 = 0; j0 < nband; j0 += kWave) {
      const int j = j0 + lane;
      bool listed = false;
      int pos = 0;
      if (j < nband) {
        const int t = cut[kCut - 1 - j];
        const int wx = t & 0xFFFF, wy = t >> 16;
        const int px = kw.xa + wx, py = kw.ya + wy;
        const double x0 = (double)px - 0.5 - cx, x1 = (double)px + 0.5 - cx;
        const double y0 = (double)py - 0.5 - cy, y1 = (double)py + 0.5 - cy;
        if (min_q(X, Y, xy, det, x0, x1, y0, y1) < R2) {
          const bool in = px >= 0 && px < fr.w && py >= 0 && py < fr.h;
          float I = 0.0f, B = 0.0f;
          if (in) {
            I = fr.pix[(int64_t)py * fr.pitch + px];
            B = fr.bkg[(int64_t)py * fr.w + px];
          }
          member(px, py, I, B, t, &listed, &pos);
        }
      }
      const uint64_t b = ballot(listed);
      if (listed) cut[ncut + lanes_before(b)] = pos;
      ncut += __popcll(b);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int j = lane; j < ncut; j += kWave) {
      const AtanCoef coef = atan_table();
      const int t = cut[j];
      const int px = kw.xa + (t & 0xFFFF), py = kw.ya + (t >> 16);
      const double w = ell_overlap(el, cx, cy, px, py, coef);
      const double v = (double)fr.pix[(int64_t)py * fr.pitch + px] -
                       (double)fr.bkg[(int64_t)py * fr.w + px];
      fs += w * v;
      as += w;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

}  // namespace

// Parts of the windows left to the whole grid: per pass a count of parts,
// and per part its row, its number within the row and its sums (KronPart).
// A row's parts are consecutive; the first one's `done` counts the parts that
// are summed (and notes a member off the frame).  A row that finds the table
// full carries a bit in its flags until it is finished.
namespace {
constexpr int kPartEdge = 1 << 30;                   // in done
constexpr uint32_t kKronLeft1 = 1u << 31, kKronLeft2 = 1u << 30;

__device__ __forceinline__ int kron_parts(int npx) {
  return (npx + kKronPart - 1) / kKronPart;
}

// A part's sum stored and loaded where every XCD sees it.
__device__ __forceinline__ void part_store(double* p, double v) {
  __hip_atomic_store((long long*)p, __double_as_longlong(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double part_load(const double* p) {
  return __longlong_as_double(__hip_atomic_load(
      (const long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Reserves and fills the part entries of a row; wave-uniform result.
__device__ __forceinline__ bool kron_reserve(const KronTable& tb,
                                             long long row, int np,
                                             int lane) {
  long long base = 0;
  if (lane == 0)
    base = (long long)atomicAdd((unsigned long long*)tb.count,
                                (unsigned long long)np);
  base = __shfl(base, 0, kWave);
  if (base + np > tb.cap) {
    // entries that would fit stay marked empty
    for (long long i = base + lane; i < tb.cap && i < base + np; i += kWave)
      tb.part[i].row = -1;
    return false;
  }
  for (int i = lane; i < np; i += kWave) {
    tb.part[base + i].row = row;
    tb.part[base + i].k = i;
    tb.part[base + i].done = 0;
  }
  return true;
}

// The sums of part k of a row's pass PASS window, by one wave: pass 1 sum
// sqrt(q) v and sum v, pass 2 sum w v, sum w and the edge flag.
template <int PASS>
__device__ __forceinline__ void kron_part(const FrameDev& fr,
                                          const KronRow& r, double R,
                                          double search, const KronWin& kw,
                                          int k, int lane, int* cut,
                                          double& s0, double& s1,
                                          bool& edge) {
  const int eb = k * kKronPart, ee = min(kw.npx, eb + kKronPart);
  s0 = s1 = 0.0;
  edge = false;
  if constexpr (PASS == 1) {
    kron_pass1(fr, r, search, kw, eb, ee, lane, s0, s1);
  } else {
    const Ell el = ell_map(r.X, r.Y, r.xy, r.det, R);
    kron_pass2(fr, r, el, R, kw, eb, ee, lane, cut, s0, s1, edge);
  }
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  edge = ballot(edge) != 0;
}
}  // namespace

// Three wavefronts a SIMD: at four the registers spill (362 against 308 us
// for the candidates of four 4096^2 frames).
__global__ __launch_bounds__(kRowThreads)
__attribute__((amdgpu_waves_per_eu(3))) void k_kron(Work wk, ipp_sources src,
                                                 const double* mom,
                                                 double kfac, double rmin,
                                                 double search, KronTable t1,
                                                 KronTable t2, double* kron,
                                                 double* flux, double* area,
                                                 uint32_t* flags) {
  // pixels of the Kron ellipse cut by its boundary: py << 16 | px offsets
  // from the window corner, per wave
  __shared__ int cut_lds[kRowWaves][kCut];
  int* cut = cut_lds[threadIdx.x / kWave];
  const int lane = threadIdx.x & (kWave - 1);
  long long nrows = src.capacity;
  if (src.n_total && *src.n_total < nrows) nrows = *src.n_total;
  const long long wid =
      blockIdx.x * (long long)kRowWaves +
      __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const long long nw = (long long)gridDim.x * kRowWaves;
  for (long long row = wid; row < nrows; row += nw) {
    const KronRow r = kron_row(wk, src, mom, row);
    if (!r.ok) {
      if (lane == 0) {
        kron[row] = __builtin_nan("");
        flux[row] = __builtin_nan("");
        area[row] = 0.0;
        flags[row] = 1u;                               // bad shape
      }
      continue;
    }
    const double cx = r.cx, cy = r.cy, X = r.X, Y = r.Y, xy = r.xy;
    const double det = r.det;
    const FrameDev fr = wk.frames[r.f];
    uint32_t fl = 0;
    // ---- pass 1: first moment over the search ellipse ------------------
    const KronWin sw = search_window(fr, r, search);
    if (sw.npx > kKronBigPx) {             // both passes in parts
      const bool listed = kron_reserve(t1, row, kron_parts(sw.npx), lane);
      if (lane == 0) flags[row] = listed ? 0u : kKronLeft1;
      continue;
    }
    double num = 0.0, den = 0.0;
    kron_pass1(fr, r, search, sw, 0, sw.npx, lane, num, den);
    num = wave_sum(num);
    den = wave_sum(den);
    const double R = kron_radius(num, den, kfac, rmin, &fl);
    // ---- pass 2: exact overlaps with the Kron ellipse -------------------
    // (one centred outside the frame is flagged outright)
    if (!(cx >= -0.5 && cx <= (double)fr.w - 0.5 && cy >= -0.5 &&
          cy <= (double)fr.h - 0.5))
      fl |= 4u;
    const KronWin kw = kron_window(fr, r, R);
    if (kw.npx > kKronBigPx) {             // pass 2 in parts
      const bool listed = kron_reserve(t2, row, kron_parts(kw.npx), lane);
      if (lane == 0) {
        kron[row] = R;
        flags[row] = listed ? fl : fl | kKronLeft2;
      }
      continue;
    }
    const Ell el = ell_map(X, Y, xy, det, R);
    double fs = 0.0, as = 0.0;
    bool edge = false;
    kron_pass2(fr, r, el, R, kw, 0, kw.npx, lane, cut, fs, as, edge);
    fs = wave_sum(fs);
    as = wave_sum(as);
    if (__builtin_amdgcn_ballot_w64(edge)) fl |= 4u;    // off the frame
    if (lane == 0) {
      kron[row] = R;
      flux[row] = fs;
      area[row] = as;
      flags[row] = fl;
    }
  }
}

// The listed parts of one pass, a wave each; the wave that sums the last of a
// row's parts finishes the row: its lane l adds the parts l, l + 64, .. in
// order, then the lanes are added.  Pass 1 gives the Kron radius and lists the
// row's pass-2 parts, pass 2 flux and area.  Rows that found the table full
// (there are none unless the count exceeds it) take a workgroup each, its waves
// summing the parts in turn; the additions are the same.  (1000 rows of
// windows of 4,489 and 12,100 pixels, with room and without: 193 and
// 208 us; up to 512 rows one after the other in a workgroup: 24,970.)
// A launch is bound by the longest part: with 2048 pixels pass 2 of four
// 4096 x 4096 frames takes 34 us and pass 1 21, with 4096 pixels the longer
// took nearly twice that (59 against 32, before it finished the rows).
// Windows over 4096 pixels go in parts; one wavefront takes about 20 us for
// such a window.  Finishing the
// rows in two kernels of their own cost every call two launches more (20 rows
// of a 256 x 256 frame: 38 against 33.5 us) and read every row's windows again
// (13 us on the four frames; 5 here).  Pass 1 takes 84 registers: at eight
// wavefronts a SIMD it spills (33 against 30 us, both with the release).
template <int PASS>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(PASS == 2 ? 3 : 4))) void k_kron_parts(
    Work wk, ipp_sources src, const double* mom, double kfac, double rmin,
    double search, KronTable tb, KronTable next, double* kron, double* flux,
    double* area, uint32_t* flags) {
  __shared__ int cut_lds[kWaves][PASS == 2 ? kCut : 1];
  __shared__ double part[2][kWave];
  __shared__ int pedge;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int lane = threadIdx.x & (kWave - 1);
  const long long count = *tb.count;
  // row's result from the sums over its parts (one wave)
  auto finish = [&](long long row, const KronRow& r, const FrameDev& fr,
                    double s0, double s1, bool edge) {
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    if constexpr (PASS == 1) {
      uint32_t fl = 0;
      const double R = kron_radius(s0, s1, kfac, rmin, &fl);
      if (!(r.cx >= -0.5 && r.cx <= (double)fr.w - 0.5 && r.cy >= -0.5 &&
            r.cy <= (double)fr.h - 0.5))
        fl |= 4u;
      const int np = kron_parts(kron_window(fr, r, R).npx);
      const bool listed = np == 0 || kron_reserve(next, row, np, lane);
      if (lane == 0) {
        kron[row] = R;
        flags[row] = listed ? fl : fl | kKronLeft2;
        if (np == 0) flux[row] = area[row] = 0.0;   // nothing left to sum
      }
    } else if (lane == 0) {
      flux[row] = s0;
      area[row] = s1;
      flags[row] = (flags[row] & ~kKronLeft2) | (edge ? 4u : 0u);  // off frame
    }
  };
  const long long n = count < tb.cap ? count : tb.cap;
  for (long long i = blockIdx.x * (long long)kWaves + wv; i < n;
       i += (long long)gridDim.x * kWaves) {
    const long long row = tb.part[i].row;
    if (row < 0) continue;
    const KronRow r = kron_row(wk, src, mom, row);
    const FrameDev fr = wk.frames[r.f];
    const double R = PASS == 2 ? kron[row] : 0.0;
    const KronWin kw =
        PASS == 1 ? search_window(fr, r, search) : kron_window(fr, r, R);
    const int k = tb.part[i].k, np = kron_parts(kw.npx);
    KronPart* first = tb.part + (i - k);
    double s0, s1;
    bool edge;
    kron_part<PASS>(fr, r, R, search, kw, k, lane, cut_lds[wv], s0, s1, edge);
    int before = 0;
    if (lane == 0) {
      // The sums are performed (stores past the L2, and a wait for them)
      // before the part is counted, and those of a full count are loaded past
      // the caches after it: the parts of a row may be summed on several
      // XCDs.  (A device-scope release in their place writes the L2 back,
      // once a part: 30 against 21 us for pass 1 of four 4096^2 frames.)
      part_store(&tb.part[i].s0, s0);
      part_store(&tb.part[i].s1, s1);
      if (edge)
        __hip_atomic_fetch_or(&first->done, kPartEdge, __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_s_waitcnt(0);
      before = __hip_atomic_fetch_add(&first->done, 1, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    }
    before = __builtin_amdgcn_readfirstlane(before);
    if ((before & (kPartEdge - 1)) != np - 1) continue;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    s0 = s1 = 0.0;
    for (int q = lane; q < np; q += kWave) {
      s0 += part_load(&first[q].s0);
      s1 += part_load(&first[q].s1);
    }
    finish(row, r, fr, s0, s1, (before & kPartEdge) != 0);
  }
  if (count <= tb.cap) return;
  // ---- rows that found the table full -----------------------------------
  long long nrows = src.capacity;
  if (src.n_total && *src.n_total < nrows) nrows = *src.n_total;
  for (long long row = blockIdx.x; row < nrows; row += gridDim.x) {
    // (the bit is this workgroup's to clear, after all its waves have read it)
    if (!(flags[row] & (PASS == 1 ? kKronLeft1 : kKronLeft2))) continue;
    const KronRow r = kron_row(wk, src, mom, row);
    const FrameDev fr = wk.frames[r.f];
    const double R = PASS == 2 ? kron[row] : 0.0;
    const KronWin kw =
        PASS == 1 ? search_window(fr, r, search) : kron_window(fr, r, R);
    const int np = kron_parts(kw.npx);
    double t0 = 0.0, t1 = 0.0;
    if (threadIdx.x == 0) pedge = 0;
    for (int k0 = 0; k0 < np; k0 += kWave) {
      __syncthreads();
      for (int k = k0 + wv; k < min(np, k0 + kWave); k += kWaves) {
        double s0, s1;
        bool edge;
        kron_part<PASS>(fr, r, R, search, kw, k, lane, cut_lds[wv], s0, s1,
                        edge);
        if (lane == 0) {
          part[0][k - k0] = s0;
          part[1][k - k0] = s1;
          if (edge) atomicOr(&pedge, 1);
        }
      }
      __syncthreads();
      if (k0 + lane < np) {
        t0 += part[0][lane];
        t1 += part[1][lane];
      }
    }
    __syncthreads();
    if (wv == 0) finish(row, r, fr, t0, t1, pedge != 0);
    __syncthreads();
  }
}

template __global__ void k_kron_parts<1>(Work, ipp_sources, const double*,
                                         double, double, double, KronTable,
                                         KronTable, double*, double*, double*,
                                         uint32_t*);
template __global__ void k_kron_parts<2>(Work, ipp_sources, const double*,
                                         double, double, double, KronTable,
                                         KronTable, double*, double*, double*,
                                         uint32_t*);

}  // namespace ipp
