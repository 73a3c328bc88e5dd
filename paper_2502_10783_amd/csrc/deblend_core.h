// Records and helpers of multi-threshold deblending and cleaning
// (Sec. 2.2.5: deblending and cleaning phases), shared by the kernels in
// k_deblend.hip.
//
// Readings (the paper states the phases, not their formulas):
//  levels   t0 = nsigma R32(peak pixel); q = (peak / t0)^(1/N) by log2(N)
//           square roots; t_i = t_{i-1} q for i = 1 .. N-1 (binary64).
//  tree     at level i the candidate's pixels with v > t_i form components
//           (the detection's connectivity), each inside one component of
//           level i-1; the candidate is the root (level 0).
//  contrast a node is significant iff its intensity above its level,
//           fl(S 2^-28) - n t_i with S the exact sum of the fixed-point
//           weights, exceeds mincont times the candidate's flux.
//  pruning  bottom up: a leaf is one object; a node with >= 2 significant
//           children stands for their objects; with one, for that child's
//           objects if it has >= 2, else for itself; with none, itself.
//  seeds    the pixels of the object nodes, numbered in raster order of
//           their first pixels; the other pixels go to the seed whose
//           Moffat (index 2) model F s2 / (s2 + d^2)^2 is largest there
//           (F, barycentre and s2 = x2 + y2 + 1/6 from the seed's exact
//           moments), ties to the lower index.
//  cleaning an object whose mean value minus the modelled light of the
//           brighter objects at its seed barycentre, k_c F s2 /
//           (pi (s2 + d^2)^2) summed in index order, falls below t0 is
//           merged into the brightest such contributor.
//
// Tree representation: chains.  A node with exactly one child at the next
// level and that child carry the same objects unless the child's own
// subtree splits, and the intensity can only grow towards the root, so a
// run of single-child nodes is kept as one chain record (its top node's
// intensity, and whether every node below the top is significant).  The
// records are made from the highest level down (build_tree): a chain starts
// where a pixel of a level meets no component of the level above, or where
// components of the level above meet, and ends (its top node known) where it
// meets another; so children come before their parents.  There are at most
// twice as many chains as leaves, and at most as many leaves as pixels.
//
// Exact sums: every sum of fixed-point weights is an integer sum, kept as
// 64-bit sums of 32-bit limbs (a term T = sum_j L_j 2^(32 j), L_0..L_2 in
// [0, 2^32), L_3 = T >> 96) so that they can be added in any order, by any
// thread, and rebuilt exactly as a 128-bit integer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ipp {
namespace db {

constexpr int kMaxLevels = 64;      // nthresh: a power of two in [2, 64]

struct Chain {
  double F_top;              // intensity above its level of the top node
  int64_t nobj_sum;          // objects of the significant child chains
  int32_t parent;            // chain of the parent node (-1: the root)
  int16_t last, top;         // levels of the chain's highest and top node
  int32_t nsig;              // significant child chains
  int32_t one;               // a significant child chain (nsig == 1)
  int32_t nobj;              // objects this chain stands for
  int32_t mode;              // 0 the top node is the object, 1 children's
  int32_t bmode;             // 1 all significant children, 2 the one
  int32_t allsig;            // the highest node (then every node below the
                             // top: intensities grow downwards) significant
  int32_t reached, objof;    // on the object path; object chain (or -1)
  int32_t slot;              // seed index of an object chain
  int32_t first;             // first pixel of an object chain's seed
};

// the scratch of a candidate that ipp.h states
static_assert(sizeof(Chain) == 64 && kMaxLevels <= 0x7FFF, "a chain record");

// One seed / object.  m[s][j]: limb j of the seed sums S = sum d,
// Sx = sum d dx, Sy = sum d dy, Sxx = sum d dx^2, Syy = sum d dy^2 (dx, dy
// about the seed's corner); fin: limbs 0 and 1 of the final pixels' sum
// (d = hi 2^32 + lo, hi the signed part), nfin their count.
struct Obj {
  int64_t m[5][4];
  int64_t fin[2];
  int64_t nfin;
  double F, xc, yc, s2;
  int32_t xmin, ymin, first, target;
  int32_t final_obj, idx;    // object after merges; survivor number
};
static_assert(sizeof(Obj) == 240, "an object record");

__host__ __device__ inline size_t align16(size_t b) { return (b + 15) & ~(size_t)15; }

// Per-candidate scratch in the pool; A = bounding-box pixels, m =
// candidate pixels.  The arrays after asg serve boxes too large for the
// kernels' LDS (the live roots and their chains then lie in the objects'
// place, which is not in use before the seeds).
struct Pool {
  double* val;      // [A] v of members, -inf elsewhere
  int32_t* asg;     // [A] out: object index of members, -1 elsewhere
  int32_t* par;     // [A] union-find parent (also the seed marks)
  int32_t* ch;      // [A] chain of each pixel's node
  int64_t* accL;    // [A] per root: low limb sums
  int64_t* accH;    // [A] per root: high (signed) limb sums
  int32_t* accN;    // [A] per root: pixel counts and flags
  int32_t* list;    // [A] member pixels by level, highest first
  int32_t* chn;     // [A] per root: its chain at this level
  Chain* chains;    // [2 m + 2]
  Obj* objs;        // [m + 1]
  int32_t chain_cap, obj_cap;
};

__host__ __device__ inline size_t pool_bytes(int64_t A, int64_t m) {
  return 3 * align16(8 * (size_t)A) + 6 * align16(4 * (size_t)A) +
         align16(sizeof(Chain) * (size_t)(2 * m + 2)) +
         align16(sizeof(Obj) * (size_t)(m + 1));
}

__host__ __device__ inline Pool carve(char* b, int64_t A, int64_t m) {
  Pool s;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* r = b + o;
    o += align16(bytes);
    return r;
  };
  s.val = (double*)take(8 * (size_t)A);
  s.accL = (int64_t*)take(8 * (size_t)A);
  s.accH = (int64_t*)take(8 * (size_t)A);
  s.par = (int32_t*)take(4 * (size_t)A);
  s.ch = (int32_t*)take(4 * (size_t)A);
  s.asg = (int32_t*)take(4 * (size_t)A);
  s.accN = (int32_t*)take(4 * (size_t)A);
  s.list = (int32_t*)take(4 * (size_t)A);
  s.chn = (int32_t*)take(4 * (size_t)A);
  s.chains = (Chain*)take(sizeof(Chain) * (size_t)(2 * m + 2));
  s.objs = (Obj*)take(sizeof(Obj) * (size_t)(m + 1));
  s.chain_cap = (int32_t)(2 * m + 2);
  s.obj_cap = (int32_t)(m + 1);
  return s;
}

// Correctly rounded (nearest, ties to even) binary64 value of an int128.
__host__ __device__ inline double to_f64(__int128 v) {
  const bool neg = v < 0;
  unsigned __int128 u = neg ? (unsigned __int128)0 - (unsigned __int128)v
                            : (unsigned __int128)v;
  if (u == 0) return 0.0;
  const uint64_t hi = (uint64_t)(u >> 64), lo = (uint64_t)u;
  const int top = hi ? 127 - __builtin_clzll(hi) : 63 - __builtin_clzll(lo);
  double r;
  if (top < 53) {
    r = (double)(uint64_t)u;
  } else {
    const int sh = top - 52;
    uint64_t mant = (uint64_t)(u >> sh);
    const unsigned __int128 rem = u & ((((unsigned __int128)1) << sh) - 1);
    const unsigned __int128 half = ((unsigned __int128)1) << (sh - 1);
    if (rem > half || (rem == half && (mant & 1))) mant += 1;
    r = ldexp((double)mant, sh);
  }
  return neg ? -r : r;
}

// Fixed-point weight of a value: round(v 2^28), clamped to +-(2^62 - 1)
// (binary64 comparison with 2^62 is exact: see the source table).
__host__ __device__ inline int64_t fixed_d(double v) {
  const double s = rint(v * 268435456.0);
  const int64_t dmax = (int64_t)(((uint64_t)1 << 62) - 1);
  if (s >= 0x1p62) return dmax;
  if (s <= -0x1p62) return -dmax;
  return (int64_t)s;
}

// The 128-bit value of four limb sums (see the header).
__host__ __device__ inline __int128 from_limbs4(const int64_t* l) {
  return (__int128)l[0] + ((__int128)l[1] << 32) + ((__int128)l[2] << 64) +
         ((__int128)l[3] << 96);
}

// The 128-bit value of a low (unsigned 32-bit terms) and a high (signed)
// limb sum.
__host__ __device__ inline __int128 from_limbs2(int64_t lo, int64_t hi) {
  return (__int128)lo + ((__int128)hi << 32);
}

__host__ __device__ inline int high_bit(uint64_t v) {
  return 63 - __builtin_clzll(v);
}

// What the tree knows of a chain when it starts (F_top, parent and top
// follow when it ends), and the fields that the pruning fills.
__host__ __device__ inline void chain_start(Chain& c, int level, bool sig) {
  c.last = (int16_t)level;
  c.allsig = sig ? 1 : 0;
}
__host__ __device__ inline void chain_clear(Chain& c) {
  c.nobj_sum = 0;
  c.nsig = 0;
  c.one = -1;
  c.nobj = 1;
  c.mode = 0;
  c.bmode = 0;
  c.reached = 0;
  c.objof = -1;
  c.slot = -1;
  c.first = 0x7FFFFFFF;
}

// Root of x in the union-find of M (par words: -1 outside the level's mask).
// Every word points to a smaller index of the same component (linking puts
// the larger root under the smaller), so a component's root is its first
// pixel and every walk ends.  The find halves the path it walks: a word is
// overwritten with its grandparent, which keeps both properties; a link
// that such a write replaces belongs to a union whose atomic found its
// target already linked, and that union joins the target's new root itself
// before it returns.
template <class M>
__host__ __device__ inline int uf_find(M& m, int x) {
  while (true) {
    const int px = m.par(x);
    if (px == x) return x;
    const int gp = m.par(px);
    if (gp == px) return px;
    m.set_par(x, gp);
    x = gp;
  }
}
template <class M>
__host__ __device__ inline void uf_unite(M& m, int a, int b) {
  while (true) {
    a = uf_find(m, a);
    b = uf_find(m, b);
    if (a == b) return;
    if (a > b) {
      const int t = a;
      a = b;
      b = t;
    }
    const int old = m.min_par(b, a);
    if (old == b) return;
    b = old;       // b was linked meanwhile: join a with b's new parent
  }
}

// The chain records of a candidate, from its highest level down: each level
// adds its own pixels (list[start[lv]] .. of them cnt[lv]) to the union-find
// of the levels above, so that a pixel is worked on once, not at every level
// below its value.  Called by every thread of the group G; levels: the levels
// with pixels (bit lv, 1 <= lv < 64); T[lv]: their thresholds; M: the arrays.
// Before the call par and chf are -1 (chf: negative) everywhere and every
// listed pixel's sum holds its own weight.  Afterwards chf holds the chain of the highest node of every
// listed pixel and *root the chain of the candidate.  Returns the number of
// chains (0: no level has a pixel), -1 if they exceed cap.
template <class G, class M, class Row>
__host__ __device__ inline int build_tree(const G& g, M& m, int conn, int bw,
                                          int A, Row row_of, const double* T,
                                          const int* start, const int* cnt,
                                          uint64_t levels, double froot,
                                          double fmin, Chain* chains, int cap,
                                          int* root) {
  constexpr int Tn = G::T;
  constexpr int kOne = 1 << 30;             // a component above lies inside
  constexpr int kTwo = (int)0x80000000u;    // two or more do
  constexpr int kCount = kOne - 1;
  auto intensity = [&](int r, int lv) {
    return m.sum(r) * 0x1p-28 - (double)(m.num(r) & kCount) * T[lv];
  };
  int nr = 0, nch = 0;                      // live components, chains
  while (levels) {
    const int lv = high_bit(levels);
    levels &= ~(1ull << lv);
    const int a = start[lv], b = a + cnt[lv];
    // this thread's first pixel and first live component stay in registers,
    // with their roots once the level's unions are done
    const int k1 = a + Tn;
    int p1 = 0, o1 = 0, c1 = 0, pr1 = 0, or1 = 0;
    if (a + g.tid < b) p1 = m.list(a + g.tid);
    if (g.tid < nr) {
      o1 = m.root(g.tid);
      c1 = m.root_chain(g.tid);
    }
    auto pixel = [&](int k) { return k < k1 ? p1 : m.list(k); };
    auto pixel_root = [&](int k, int p) { return k < k1 ? pr1 : m.par(p); };
    auto comp = [&](int j) { return j < Tn ? o1 : m.root(j); };
    auto comp_root = [&](int j, int o) { return j < Tn ? or1 : uf_find(m, o); };
    auto comp_chain = [&](int j) { return j < Tn ? c1 : m.root_chain(j); };
    for (int k = a + g.tid; k < b; k += Tn) {
      const int p = pixel(k);
      m.set_num(p, 1);
      m.set_par(p, p);
    }
    g.msync();
    for (int k = a + g.tid; k < b; k += Tn) {
      const int p = pixel(k);
      const int y = row_of(p), x = p - y * bw;
      // neighbours around p: up, up right, right, .. up left
      const bool l = x > 0, r = x + 1 < bw, u = p >= bw, d = p + bw < A;
      const int in = (int)u | (int)(u && r) << 1 | (int)r << 2 |
                     (int)(d && r) << 3 | (int)d << 4 | (int)(d && l) << 5 |
                     (int)l << 6 | (int)(u && l) << 7;
      auto at = [&](int i) {                  // neighbour i
        const int row = i < 2 || i == 7 ? -bw : (i > 2 && i < 6 ? bw : 0);
        const int col = i > 0 && i < 4 ? 1 : (i > 4 ? -1 : 0);
        return p + row + col;
      };
      int act = 0, old = 0;                   // in the mask; of levels above
      int pv[8], cv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {           // all requested, then used
        const int q = (in >> i) & 1 ? at(i) : p;
        pv[i] = m.par(q);
        cv[i] = m.chf(q);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        act |= (int)(pv[i] >= 0) << i;
        old |= (int)(cv[i] >= 0) << i;
      }
      act &= in;
      old &= act;
      // Neighbours of levels above that touch each other are joined already:
      // one link per run of them around p.  Pixels of this level: the four
      // (two) before p in raster order, the others link to p themselves.
      const int back1 = ((old << 1) | (old >> 7)) & 0xFF;
      const int back2 = ((old << 2) | (old >> 6)) & 0xFF;
      int link = conn == 8 ? old & ~back1 : old & 0x55 & ~(back1 & back2);
      if (old == 0xFF) link = 1;
      link |= act & ~old & (conn == 8 ? 0xC3 : 0x41);
      while (link) {
        uf_unite(m, p, at(__builtin_ctz(link)));
        link &= link - 1;
      }
    }
    g.msync();
    // the new pixels point at their roots; each root learns how many of the
    // components above it holds
    for (int k = a + g.tid; k < b; k += Tn) {
      const int p = pixel(k);
      const int r = uf_find(m, p);
      if (r != p) m.set_par(p, r);
      if (k < k1) pr1 = r;
    }
    for (int j = g.tid; j < nr; j += Tn) {
      const int r = uf_find(m, comp(j));
      if (m.or_num(r, kOne) & kOne) m.or_num(r, kTwo);
      if (j < Tn) or1 = r;
    }
    g.msync();
    // components that met end their chains at the level above; a root that
    // holds none or several of them gets a new chain
    for (int j0 = 0; j0 < nr; j0 += Tn) {
      const int j = j0 + g.tid;
      bool fresh = false;
      int o = 0;
      if (j < nr) {
        o = comp(j);
        const int r = comp_root(j, o), c = comp_chain(j);
        if (m.num(r) & kTwo) {
          chains[c].F_top = intensity(o, lv + 1);
          chains[c].top = (int16_t)(lv + 1);
          fresh = r == o;
        } else {
          m.set_chn(r, c);
        }
      }
      int tot;
      const int id = nch + g.rank(fresh, &tot);
      if (fresh) m.set_chn(o, id);
      nch += tot;
    }
    for (int k0 = a; k0 < b; k0 += Tn) {
      const int k = k0 + g.tid;
      bool fresh = false;
      int p = 0;
      if (k < b) {
        p = pixel(k);
        if (pixel_root(k, p) == p) {
          const int f = m.num(p);
          fresh = !(f & kOne) || (f & kTwo);
        }
      }
      int tot;
      const int id = nch + g.rank(fresh, &tot);
      if (fresh) m.set_chn(p, id);
      nch += tot;
    }
    if (nch > cap) return -1;
    g.msync();
    // the ended chains' parents, the roots' sums, the new pixels' chains
    for (int j = g.tid; j < nr; j += Tn) {
      const int o = comp(j), r = comp_root(j, o);
      if (m.num(r) & kTwo) chains[comp_chain(j)].parent = m.chn(r);
      if (r != o) {
        m.add_sum(r, o);
        m.add_num(r, m.num(o) & kCount);
      }
    }
    for (int k = a + g.tid; k < b; k += Tn) {
      const int p = pixel(k), r = pixel_root(k, p);
      m.set_chf(p, m.chn(r));
      if (r != p) {
        m.add_sum(r, p);
        m.add_num(r, 1);
      }
    }
    g.msync();
    // the new chains and the list of live components
    int w = 0;
    for (int j0 = 0; j0 < nr; j0 += Tn) {
      const int j = j0 + g.tid;
      int o = 0, c = 0;
      bool keep = false;
      if (j < nr) {
        o = comp(j);
        keep = comp_root(j, o) == o;
        if (keep) {
          c = m.chn(o);
          const int f = m.num(o);
          if (f & kTwo) chain_start(chains[c], lv, intensity(o, lv) > fmin);
          m.set_num(o, f & kCount);
        }
      }
      int tot;
      const int at = w + g.rank(keep, &tot);
      if (keep) m.set_root(at, o, c);
      w += tot;
    }
    for (int k0 = a; k0 < b; k0 += Tn) {
      const int k = k0 + g.tid;
      int p = 0, c = 0;
      bool keep = false;
      if (k < b) {
        p = pixel(k);
        keep = pixel_root(k, p) == p;
        if (keep) {
          c = m.chn(p);
          const int f = m.num(p);
          if (!(f & kOne) || (f & kTwo))
            chain_start(chains[c], lv, intensity(p, lv) > fmin);
          m.set_num(p, f & kCount);
        }
      }
      int tot;
      const int at = w + g.rank(keep, &tot);
      if (keep) m.set_root(at, p, c);
      w += tot;
    }
    nr = w;
    g.msync();
  }
  if (nr == 0) return 0;
  if (nr == 1) {
    *root = m.root_chain(0);
    if (g.tid == 0) {
      Chain& c = chains[*root];
      c.F_top = froot;
      c.top = 0;
      c.parent = -1;
    }
  } else {
    *root = nch;
    if (nch + 1 > cap) return -1;
    for (int j = g.tid; j < nr; j += Tn) {
      Chain& c = chains[m.root_chain(j)];
      c.F_top = intensity(m.root(j), 1);
      c.top = 1;
      c.parent = nch;
    }
    if (g.tid == 0) {
      Chain& c = chains[nch];
      chain_start(c, 0, true);
      c.F_top = froot;
      c.top = 0;
      c.parent = -1;
    }
    ++nch;
  }
  return nch;
}

// Pruning, children before parents (chains are numbered that way), then the
// object path, parents before children; one thread, on records cleared by
// chain_clear.
__host__ __device__ inline void prune_tree(Chain* chains, int nch, int root,
                                           double fmin) {
  for (int k = 0; k < nch; ++k) {
    Chain& C = chains[k];
    int bmode = 0;
    int64_t nb = 1;
    if (C.nsig >= 2) {
      bmode = 1;
      nb = C.nobj_sum;
    } else if (C.nsig == 1 && chains[C.one].nobj >= 2) {
      bmode = 2;
      nb = chains[C.one].nobj;
    }
    C.bmode = bmode;
    if (bmode != 0 && (C.allsig || C.top == C.last)) {
      C.mode = 1;
      C.nobj = (int32_t)nb;
    } else {
      C.mode = 0;
      C.nobj = 1;
    }
    if (C.parent >= 0 && C.F_top > fmin) {
      Chain& P = chains[C.parent];
      P.nsig += 1;
      P.nobj_sum += C.nobj;
      P.one = k;
    }
  }
  if (chains[root].nobj < 2) return;
  for (int k = nch - 1; k >= 0; --k) {
    Chain& C = chains[k];
    int up = -1;
    if (C.parent < 0) {
      C.reached = 1;
    } else {
      const Chain& P = chains[C.parent];
      C.reached = P.reached && P.mode == 1 &&
                  ((P.bmode == 1 && C.F_top > fmin) ||
                   (P.bmode == 2 && P.one == k));
      up = P.objof;
    }
    C.objof = C.reached && C.mode == 0 ? k : up;
  }
}

// The same on the records' few fields that it needs, for chains held in LDS:
// sig lists the significant chains (F_top > fmin), ascending, and the root.
// Only those can add to a parent or be reached, so one thread walks them
// alone; the objof of the others is their nearest listed ancestor's.
struct Node {
  int32_t parent, nobj, nobj_sum, one, objof;
  int16_t nsig, flags;       // kNode*
};
constexpr int kNodeSig = 1, kNodeKeep = 2, kNodeMode = 4, kNodeB1 = 8,
              kNodeB2 = 16, kNodeReached = 32;
__host__ __device__ inline void node_init(Node& n, const Chain& c,
                                          double fmin) {
  n.parent = c.parent;
  n.nobj = 1;
  n.nobj_sum = 0;
  n.one = -1;
  n.objof = -1;
  n.nsig = 0;
  n.flags = (int16_t)((c.F_top > fmin ? kNodeSig : 0) |
                      (c.allsig || c.top == c.last ? kNodeKeep : 0));
}
__host__ __device__ inline void prune_nodes(Node* nodes, const uint16_t* sig,
                                            int nsig, int root) {
  for (int i = 0; i < nsig; ++i) {
    const int k = sig[i];
    Node& C = nodes[k];
    int b = 0, nb = 1;
    if (C.nsig >= 2) {
      b = kNodeB1;
      nb = C.nobj_sum;
    } else if (C.nsig == 1 && nodes[C.one].nobj >= 2) {
      b = kNodeB2;
      nb = nodes[C.one].nobj;
    }
    const bool mode = b != 0 && (C.flags & kNodeKeep);
    C.flags = (int16_t)(C.flags | b | (mode ? kNodeMode : 0));
    C.nobj = mode ? nb : 1;
    if (C.parent >= 0 && (C.flags & kNodeSig)) {
      Node& P = nodes[C.parent];
      P.nsig += 1;
      P.nobj_sum += C.nobj;
      P.one = k;
    }
  }
  if (nodes[root].nobj < 2) return;
  for (int i = nsig - 1; i >= 0; --i) {
    const int k = sig[i];
    Node& C = nodes[k];
    bool reached = true;
    int up = -1;
    if (C.parent >= 0) {
      const Node& P = nodes[C.parent];
      const int f = P.flags;
      reached = (f & kNodeReached) && (f & kNodeMode) &&
                ((f & kNodeB1) || ((f & kNodeB2) && P.one == k));
      int a = C.parent;
      while (!(nodes[a].flags & kNodeSig) && nodes[a].parent >= 0)
        a = nodes[a].parent;
      up = nodes[a].objof;
    }
    if (reached) C.flags = (int16_t)(C.flags | kNodeReached);
    C.objof = reached && !(C.flags & kNodeMode) ? k : up;
  }
}

}  // namespace db
}  // namespace ipp
