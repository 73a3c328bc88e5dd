// Deblending and cleaning of detection candidates (Sec. 2.2.5), a
// wavefront or a workgroup per candidate, and the object maps and table
// that follow from them.
//
//   k_db_need    scratch bytes of each candidate (256-byte units)
//   k_scan64_*   exclusive scans (scratch offsets, then object offsets)
//   k_db_large   boxes over kDbMidBox pixels and candidates whose sums need
//                more than 64 bits, a workgroup of eight wavefronts each
//   k_db_mid     boxes over kDbSmallBox pixels, a workgroup of four each
//   k_db_small   the other candidates, a wavefront each
//   k_db_all     the three in one launch, for tables of up to 2048 rows
//   k_db_write   a wavefront per candidate: object ids into the object
//                maps, the objects' rows (frame, label, parent, pixel
//                count, box)
//   k_db_offsets per-frame object offsets and count
//   k_db_flags   BLENDED on the objects of split candidates (after the
//                pre-analysis kernel has filled the rows)
#include "deblend_core.h"
#include "ipp_internal.h"
#include "kernels.h"

namespace ipp {

namespace {
__device__ __forceinline__ long long table_rows(const ipp_sources& t) {
  long long n = t.capacity;
  if (t.n_total && *t.n_total < n) n = *t.n_total;
  return n;
}

__device__ __forceinline__ int64_t block_scan64(int64_t v, int64_t* red,
                                                int64_t* total) {
  const int lane = threadIdx.x & (kWave - 1);
  const int w = threadIdx.x / kWave;
  int64_t x = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int64_t u = __shfl_up(x, o, kWave);
    if (lane >= o) x += u;
  }
  __syncthreads();
  if (lane == kWave - 1) red[w] = x;
  __syncthreads();
  int64_t off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    off += i < w ? red[i] : 0;
    tot += red[i];
  }
  *total = tot;
  return off + x - v;
}

// The class of a candidate: 0 for a wavefront, 1 and 2 for a workgroup (2:
// the larger boxes, and every candidate whose sums need more than 64 bits).
__device__ __forceinline__ int db_class(int64_t A, double peak, int m) {
  if (!(peak * (double)m < 0x1p62 / 268435456.0)) return 2;
  return A <= kDbSmallBox ? 0 : (A <= kDbMidBox ? 1 : 2);
}
}  // namespace

__global__ __launch_bounds__(kBlock) void k_db_need(ipp_sources cand,
                                                    int64_t* need,
                                                    int32_t* big,
                                                    int64_t* nbig,
                                                    int64_t* queue) {
  const long long n = table_rows(cand);
  const long long rows = cand.capacity + 1;
  const int nq = db_queues(cand.capacity);
  for (long long r = blockIdx.x * (long long)kBlock + threadIdx.x;
       r <= cand.capacity; r += (long long)gridDim.x * kBlock) {
    int64_t u = 0;
    if (r < n && cand.npix[r] >= 2) {
      const int64_t A = (int64_t)(cand.xmax[r] - cand.xmin[r] + 1) *
                        (cand.ymax[r] - cand.ymin[r] + 1);
      u = (int64_t)((db::pool_bytes(A, cand.npix[r]) + 255) / 256);
      // the workgroup kernels' rows (the two ends of one list of `rows`
      // entries cannot meet)
      const int cls = db_class(A, cand.peak[r], cand.npix[r]);
      if (cls == 2) {
        const long long k =
            (long long)atomicAdd((unsigned long long*)&nbig[0], 1ull);
        big[k] = (int32_t)r;
      } else if (cls == 1) {
        const long long k =
            (long long)atomicAdd((unsigned long long*)&nbig[1], 1ull);
        big[rows - 1 - k] = (int32_t)r;
      }
    }
    need[r] = u;
    if (nq > 1 && r < nq * kDbQueueStep) queue[r] = 0;
  }
}

// Exclusive scan of n int64 values: block sums of 1024 values, a scan of
// the block sums by one workgroup (chunks of 1024 with a carry), and the
// scan inside each block.
__global__ __launch_bounds__(kBlock) void k_scan64_blocks(const int64_t* in,
                                                          int64_t* blocks,
                                                          int64_t n) {
  __shared__ int64_t red[kWaves];
  const int64_t b0 = blockIdx.x * (int64_t)1024;
  int64_t s = 0;
  for (int i = 0; i < 4; ++i) {
    const int64_t j = b0 + threadIdx.x * 4 + i;
    if (j < n) s += in[j];
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) blocks[blockIdx.x] = s;
}

__global__ __launch_bounds__(kBlock) void k_scan64_top(int64_t* blocks,
                                                       int64_t nblocks,
                                                       int64_t* total) {
  __shared__ int64_t red[kWaves];
  int64_t carry = 0;
  for (int64_t c0 = 0; c0 < nblocks; c0 += 1024) {
    int64_t v[4];
    int64_t s = 0;
    for (int i = 0; i < 4; ++i) {
      const int64_t j = c0 + threadIdx.x * 4 + i;
      v[i] = j < nblocks ? blocks[j] : 0;
      s += v[i];
    }
    int64_t tot;
    int64_t ex = block_scan64(s, red, &tot) + carry;
    for (int i = 0; i < 4; ++i) {
      const int64_t j = c0 + threadIdx.x * 4 + i;
      if (j < nblocks) blocks[j] = ex;
      ex += v[i];
    }
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = carry;
}

__global__ __launch_bounds__(kBlock) void k_scan64_apply(const int64_t* in,
                                                         const int64_t* blocks,
                                                         int64_t* out,
                                                         int64_t n) {
  __shared__ int64_t red[kWaves];
  const int64_t b0 = blockIdx.x * (int64_t)1024;
  int64_t v[4];
  int64_t s = 0;
  for (int i = 0; i < 4; ++i) {
    const int64_t j = b0 + threadIdx.x * 4 + i;
    v[i] = j < n ? in[j] : 0;
    s += v[i];
  }
  int64_t tot;
  int64_t ex = block_scan64(s, red, &tot) + blocks[blockIdx.x];
  for (int i = 0; i < 4; ++i) {
    const int64_t j = b0 + threadIdx.x * 4 + i;
    if (j < n) out[j] = ex;
    ex += v[i];
  }
}

// ---------------------------------------------------------------------------
// Deblending of one candidate by a group of NW wavefronts: the pixels' values
// and levels, the pixels listed by level, the chain records from the highest
// level down (build_tree), the pruning, and for a candidate that splits the
// seeds, the assignment of the other pixels and the cleaning.  The tree's
// arrays sit in LDS for boxes of up to CAP pixels whose sums fit 64 bits, and
// in the candidate's pool scratch otherwise.
// ---------------------------------------------------------------------------

namespace {

template <int NW, bool POOL = false>
struct Grp {
  static constexpr int T = kWave * NW;
  int tid, lane, wave;
  int* red;          // LDS, NW ints
  int64_t* red64;    // LDS, 2 NW int64

  __device__ __forceinline__ void sync() const {
    if constexpr (NW == 1) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
      __syncthreads();
    }
  }
  // A step between two phases on the tree's arrays.  In LDS it orders LDS
  // accesses only (stores of chain records need not complete); in the pool
  // every access of the group so far has been performed.
  __device__ __forceinline__ void msync() const {
    if constexpr (POOL) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_s_waitcnt(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      if constexpr (NW == 1) __builtin_amdgcn_wave_barrier();
      else __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
  }
  __device__ __forceinline__ bool any(bool f) const {
    if constexpr (NW == 1) return ballot(f) != 0;
    else return __syncthreads_or(f ? 1 : 0) != 0;
  }
  // Rank of a set flag among the group's threads (thread order) and the
  // number of set flags; called by every thread of the group.
  __device__ __forceinline__ int rank(bool f, int* total) const {
    const uint64_t b = ballot(f);
    const int below = lanes_before(b);
    if constexpr (NW == 1) {
      *total = __popcll(b);
      return below;
    } else {
      __syncthreads();
      if (lane == 0) red[wave] = __popcll(b);
      __syncthreads();
      int off = 0, tot = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const int c = red[i];
        off += i < wave ? c : 0;
        tot += c;
      }
      *total = tot;
      return off + below;
    }
  }
  // Group sums of two int64 values, returned to every thread.
  __device__ __forceinline__ void sum2(int64_t& a, int64_t& b) const {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
      a += __shfl_xor(a, o, kWave);
      b += __shfl_xor(b, o, kWave);
    }
    if constexpr (NW > 1) {
      __syncthreads();
      if (lane == 0) {
        red64[2 * wave] = a;
        red64[2 * wave + 1] = b;
      }
      __syncthreads();
      a = 0;
      b = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        a += red64[2 * i];
        b += red64[2 * i + 1];
      }
    }
  }
};


constexpr int kNone16 = 0xFFFE;      // this and above: no chain, no object

// LDS of one group.
template <int NW, int CAP>
struct DbLds {
  int64_t S[CAP];                    // per root: sum of weights
  int par[CAP], num[CAP];
  uint16_t chn[CAP], chf[CAP], list[CAP];
  uint16_t root[CAP / 2 + 2], rch[CAP / 2 + 2];
  double T[db::kMaxLevels + 1];
  int start[db::kMaxLevels], cnt[db::kMaxLevels], put[db::kMaxLevels];
  int red[NW];
  int64_t red64[2 * NW];
};

// Accesses of words that other threads of the group update atomically.
__device__ __forceinline__ int ld_at(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int64_t ld_at(const int64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_at(int64_t* p, int64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_at(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void add_at(int64_t* p, int64_t v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void add_at(int* p, int v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void min_at(int* p, int v) {
  __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}


// The tree's arrays in LDS (boxes of up to 65534 pixels, 64-bit sums).
template <int NW, int CAP>
struct TreeLds {
  static constexpr bool kLds = true;
  DbLds<NW, CAP>& L;
  static __device__ __forceinline__ int ld(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ int par(int p) const { return ld(&L.par[p]); }
  __device__ void set_par(int p, int v) {
    __hip_atomic_store(&L.par[p], v, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ int min_par(int p, int v) {
    return __hip_atomic_fetch_min(&L.par[p], v, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ void set_weight(int p, int64_t d) { L.S[p] = d; }
  __device__ double sum(int r) const {
    return (double)__hip_atomic_load(&L.S[r], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ void add_sum(int r, int o) {
    __hip_atomic_fetch_add(&L.S[r], L.S[o], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ int num(int r) const { return ld(&L.num[r]); }
  __device__ void set_num(int r, int v) { L.num[r] = v; }
  __device__ int or_num(int r, int v) {
    return __hip_atomic_fetch_or(&L.num[r], v, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ void add_num(int r, int v) {
    __hip_atomic_fetch_add(&L.num[r], v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ int chn(int r) const { return L.chn[r]; }
  __device__ void set_chn(int r, int c) { L.chn[r] = (uint16_t)c; }
  __device__ int chf(int p) const {
    const int c = L.chf[p];
    return c >= kNone16 ? -1 : c;
  }
  __device__ void set_chf(int p, int c) { L.chf[p] = (uint16_t)c; }
  __device__ int list(int k) const { return L.list[k]; }
  __device__ void set_list(int k, int p) { L.list[k] = (uint16_t)p; }
  __device__ int root(int j) const { return L.root[j]; }
  __device__ int root_chain(int j) const { return L.rch[j]; }
  __device__ void set_root(int j, int o, int c) {
    L.root[j] = (uint16_t)o;
    L.rch[j] = (uint16_t)c;
  }
};

// The same in the pool: sums of 32-bit limbs, every access past the L1.
struct TreePool {
  static constexpr bool kLds = false;
  const db::Pool& s;
  int* roots;            // root and chain pairs
  __device__ int par(int p) const { return ld_at(s.par + p); }
  __device__ void set_par(int p, int v) { st_at(s.par + p, v); }
  __device__ int min_par(int p, int v) {
    return __hip_atomic_fetch_min(s.par + p, v, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ void set_weight(int p, int64_t d) {
    st_at(s.accL + p, (int64_t)(uint32_t)d);
    st_at(s.accH + p, d >> 32);
  }
  __device__ double sum(int r) const {
    return db::to_f64(
        db::from_limbs2(ld_at(s.accL + r), ld_at(s.accH + r)));
  }
  __device__ void add_sum(int r, int o) {
    add_at(s.accL + r, ld_at(s.accL + o));
    add_at(s.accH + r, ld_at(s.accH + o));
  }
  __device__ int num(int r) const { return ld_at(s.accN + r); }
  __device__ void set_num(int r, int v) { st_at(s.accN + r, v); }
  __device__ int or_num(int r, int v) {
    return __hip_atomic_fetch_or(s.accN + r, v, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ void add_num(int r, int v) { add_at(s.accN + r, v); }
  __device__ int chn(int r) const { return ld_at(s.chn + r); }
  __device__ void set_chn(int r, int c) { st_at(s.chn + r, c); }
  __device__ int chf(int p) const { return ld_at(s.ch + p); }
  __device__ void set_chf(int p, int c) { st_at(s.ch + p, c); }
  __device__ int list(int k) const { return ld_at(s.list + k); }
  __device__ void set_list(int k, int p) { st_at(s.list + k, p); }
  __device__ int root(int j) const { return ld_at(roots + 2 * j); }
  __device__ int root_chain(int j) const { return ld_at(roots + 2 * j + 1); }
  __device__ void set_root(int j, int o, int c) {
    st_at(roots + 2 * j, o);
    st_at(roots + 2 * j + 1, c);
  }
};

// Adds NV int64 values of each active lane to the accumulators of its key
// (op(key, j, sum)): the wavefront first sums the values of equal keys,
// one lane per distinct key then adds them.
template <int NV, class Op>
__device__ __forceinline__ void keyed_add(bool act, int key,
                                          const int64_t* v, int lane,
                                          Op&& op) {
  uint64_t left = ballot(act);
  while (left) {
    const int lead = __ffsll((unsigned long long)left) - 1;
    const int k0 = __builtin_amdgcn_readlane(key, lead);
    const bool in = act && key == k0;
    left &= ~ballot(in);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      int64_t s = in ? v[j] : 0;
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
      if (lane == lead) op(k0, j, s);
    }
    act = act && !in;
  }
}
// The same with the minimum of one int per key (op(key, min)).
template <class Op>
__device__ __forceinline__ void keyed_min(bool act, int key, int v, int lane,
                                          Op&& op) {
  uint64_t left = ballot(act);
  while (left) {
    const int lead = __ffsll((unsigned long long)left) - 1;
    const int k0 = __builtin_amdgcn_readlane(key, lead);
    const bool in = act && key == k0;
    left &= ~ballot(in);
    int s = in ? v : 0x7FFFFFFF;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) s = min(s, __shfl_xor(s, o, kWave));
    if (lane == lead) op(k0, s);
    act = act && !in;
  }
}

__device__ __forceinline__ void limbs4(__int128 t, int64_t* l) {
  const unsigned __int128 u = (unsigned __int128)t;
  l[0] = (int64_t)(uint32_t)u;
  l[1] = (int64_t)(uint32_t)(u >> 32);
  l[2] = (int64_t)(uint32_t)(u >> 64);
  l[3] = (int64_t)(t >> 96);
}


struct DbCand {
  int lab, x0, y0, bw, bh, m;
  double t0, peak;
};

// The objects of a split candidate whose tree lies in LDS (chn: the object
// chain of every chain): seeds, assignment and cleaning with every sum, minimum and object
// record in LDS, in the place of the tree's sums (16 words per object).
// Returns the object count with s.asg set, or -1, nothing written, when the
// objects are too many for that place or a second moment's term may exceed
// 62 bits.
template <int NW, int CAP, class Row>
__device__ int finish_lds(const Grp<NW>& g, DbLds<NW, CAP>& L,
                          const DbCand& c, int A, int bw, Row row_of, int nch,
                          int root, int clean, double kc, db::Pool& s) {
  constexpr int T = Grp<NW>::T;
  constexpr int W = 16, kMaxObj = CAP / W;
  // words of an object: 0..9 low and high limb sums of d, d dx, d dy, d dx^2,
  // d dy^2 (later 0..3: F, xc, yc, s2), 10..12 final limbs and count, 13 the
  // seed's first pixel, 14 its xmin
  int64_t* acc = L.S;
  const double side = (double)max(bw, c.bh);
  if (nch > CAP || !(c.peak * side * side < 0x1p62 / 268435456.0)) return -1;
  auto add = [&](int64_t* p, int64_t v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto low = [&](int* p, int v) {
    __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // per chain: its object chain (chn), then the object's first pixel and slot
  for (int j = g.tid; j < nch; j += T) L.num[j] = 0x7FFFFFFF;
  for (int e = g.tid; e < W * kMaxObj; e += T) acc[e] = 0;
  g.sync();
  // per pixel (list): its object chain, kNone16 outside the seeds, kNone16 + 1
  // outside the candidate
  for (int p = g.tid; p < A; p += T) {
    int o = kNone16 + 1;
    if (s.asg[p] >= 0) {
      const int f = L.chf[p];
      o = L.chn[f >= kNone16 ? root : f];
    }
    L.list[p] = (uint16_t)o;
    L.par[p] = -1;
    if (o < kNone16) low(&L.num[o], p);
  }
  g.sync();
  for (int j = g.tid; j < nch; j += T)
    if (L.chn[j] == j && L.num[j] != 0x7FFFFFFF) L.par[L.num[j]] = j;
  g.sync();
  // slots in raster order of the seeds' first pixels
  int K = 0;
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    const int j = p < A ? L.par[p] : -1;
    int tot;
    const int k = K + g.rank(j >= 0, &tot);
    if (j >= 0) {
      L.num[j] = k;
      if (k < kMaxObj) {
        acc[W * k + 13] = p;
        *(int*)&acc[W * k + 14] = 0x7FFFFFFF;
      }
    }
    K += tot;
  }
  if (K > kMaxObj) return -1;
  g.sync();
  for (int p = g.tid; p < A; p += T) {
    const int o = L.list[p];
    if (o < kNone16) {
      const int k = L.num[o];
      L.list[p] = (uint16_t)k;
      low((int*)&acc[W * k + 14], p - row_of(p) * bw);
    }
  }
  g.sync();
  // seed moments about each seed's corner
  for (int p = g.tid; p < A; p += T) {
    const int k = L.list[p];
    if (k >= kNone16) continue;
    int64_t* b = acc + W * k;
    const int y = row_of(p), x = p - y * bw;
    const int64_t d = db::fixed_d(s.val[p]);
    const int64_t dx = x - *(const int*)&b[14];
    const int64_t dy = y - row_of((int)b[13]);
    const int64_t v[5] = {d, d * dx, d * dy, d * dx * dx, d * dy * dy};
#pragma unroll
    for (int a = 0; a < 5; ++a) {
      add(b + 2 * a, (int64_t)(uint32_t)v[a]);
      add(b + 2 * a + 1, v[a] >> 32);
    }
  }
  g.sync();
  for (int k = g.tid; k < K; k += T) {
    int64_t* b = acc + W * k;
    auto val = [&](int a) {
      return db::to_f64(db::from_limbs2(b[2 * a], b[2 * a + 1]));
    };
    const double fS = val(0);
    const double mx = val(1) / fS;
    const double my = val(2) / fS;
    const double x2 = val(3) / fS - mx * mx;
    const double y2 = val(4) / fS - my * my;
    double* o = (double*)b;
    const int xmin = *(const int*)&b[14];
    o[0] = fS * 0x1p-28;
    o[1] = (double)(c.x0 + xmin) + mx;
    o[2] = (double)(c.y0 + row_of((int)b[13])) + my;
    o[3] = (x2 + y2) + 1.0 / 6.0;
  }
  g.sync();
  const double* obj = (const double*)acc;
  // the other pixels: the brightest model
  for (int p = g.tid; p < A; p += T) {
    if (L.list[p] != kNone16) continue;
    const int py = row_of(p);
    const double x = (double)(c.x0 + p - py * bw);
    const double y = (double)(c.y0 + py);
    double best = -1.0;
    int bk = 0;
    for (int k = 0; k < K; ++k) {
      const double* b = obj + W * k;
      const double dx = x - b[1];
      const double dy = y - b[2];
      const double d2 = dx * dx + dy * dy;
      const double den = b[3] + d2;
      const double sc = (b[0] * b[3]) / (den * den);
      if (sc > best) {
        best = sc;
        bk = k;
      }
    }
    L.list[p] = (uint16_t)bk;
  }
  g.sync();
  if (!clean) {
    for (int p = g.tid; p < A; p += T)
      if (L.list[p] < kNone16) s.asg[p] = L.list[p];
    g.sync();
    return K;
  }
  // cleaning
  for (int p = g.tid; p < A; p += T) {
    const int k = L.list[p];
    if (k >= kNone16) continue;
    const int64_t d = db::fixed_d(s.val[p]);
    add(acc + W * k + 10, (int64_t)(uint32_t)d);
    add(acc + W * k + 11, d >> 32);
    add(acc + W * k + 12, 1);
  }
  g.sync();
  const double pi = 3.14159265358979311600;   // binary64 nearest to pi
  for (int o = g.tid; o < K; o += T) {
    const double* b = obj + W * o;
    const int64_t* n = acc + W * o;
    const double mu = db::to_f64(db::from_limbs2(n[10], n[11])) * 0x1p-28 /
                      (double)n[12];
    double tot = 0.0, best = -1.0;
    int bm = -1;
    for (int q = 0; q < K; ++q) {
      if (q == o) continue;
      const double* e = obj + W * q;
      const bool brighter = e[0] > b[0] || (e[0] == b[0] && q < o);
      if (!brighter) continue;
      const double dx = b[1] - e[1];
      const double dy = b[2] - e[2];
      const double d2 = dx * dx + dy * dy;
      double den = e[3] + d2;
      den = den * den;
      den = pi * den;
      const double cm = kc * ((e[0] * e[3]) / den);
      tot += cm;
      if (cm > best) {
        best = cm;
        bm = q;
      }
    }
    L.root[o] = (uint16_t)((bm >= 0 && mu - tot < c.t0) ? bm : o);
  }
  g.sync();
  // follow merges to an object that stays; number the survivors in order
  int nk = 0;
  for (int o0 = 0; o0 < K; o0 += T) {
    const int o = o0 + g.tid;
    const bool surv = o < K && L.root[o] == o;
    int tot;
    const int r = nk + g.rank(surv, &tot);
    if (surv) L.rch[o] = (uint16_t)r;
    nk += tot;
  }
  g.sync();
  for (int p = g.tid; p < A; p += T) {
    int k = L.list[p];
    if (k >= kNone16) continue;
    while (L.root[k] != k) k = L.root[k];
    s.asg[p] = L.rch[k];
  }
  g.sync();
  return nk;
}

// Deblends one candidate; returns the object count (every thread of the
// group gets it) with s.asg set for every member of a candidate that splits,
// or -1 when the chain records would exceed the scratch (not reachable with
// the bounds of pool_bytes).  Every thread of the group calls it.
template <bool ONE_WAVE, int NW, int CAP, class M>
__device__ int deblend_group(const Grp<NW, !M::kLds>& g, DbLds<NW, CAP>& L,
                             M m,
                             const FrameDev& fr, const DbCand& c, int conn,
                             int nthresh, int clean, double mincont,
                             double kc, db::Pool& s) {
  constexpr int T = Grp<NW>::T;
  const int A = c.bw * c.bh;
  const int bw = c.bw;
  if (!(c.t0 > 0.0) || c.m < 2 || !(c.peak > c.t0)) return 1;
  const double inv_bw = 1.0 / (double)bw;
  auto row_of = [&](int p) {
    int y = (int)((double)p * inv_bw);
    if (y * bw > p) --y;
    else if ((y + 1) * bw <= p) ++y;
    return y;
  };
  const double ninf = -__builtin_inf();
  // thresholds of the levels (products in order), no pixel above the last
  {
    double q = c.peak / c.t0;
    for (int k = nthresh; k > 1; k >>= 1) q = sqrt(q);
    double t = c.t0;
    for (int i = 1; i < nthresh; ++i) {
      t = t * q;
      if (g.tid == 0) L.T[i] = t;
    }
    for (int i = g.tid; i < db::kMaxLevels; i += T) L.cnt[i] = 0;
  }
  g.sync();

  // members' values, weights and levels, the candidate's flux
  int64_t fl = 0, fh = 0;
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    if (p < A) {
      const int y = row_of(p), x = p - y * bw;
      const int64_t row = c.y0 + y;
      const int64_t q = row * fr.w + c.x0 + x;
      const bool mem = fr.labels[q] == c.lab;
      const double v =
          (double)fr.pix[row * fr.pitch + c.x0 + x] - (double)fr.bkg[q];
      s.val[p] = mem ? v : ninf;
      s.asg[p] = mem ? 0 : -1;
      m.set_par(p, -1);
      m.set_chf(p, -1);
      int lev = 0;
      if (mem) {
        const int64_t d = db::fixed_d(v);
        fl += (int64_t)(uint32_t)d;
        fh += d >> 32;
        m.set_weight(p, d);
        // the number of thresholds below v (they do not decrease)
        int hi = nthresh - 1;
        while (lev < hi) {
          const int mid = (lev + hi + 1) >> 1;
          if (v > L.T[mid]) lev = mid; else hi = mid - 1;
        }
        if (lev > 0)
          __hip_atomic_fetch_add(&L.cnt[lev], 1, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      m.set_num(p, lev);
    }
  }
  g.sum2(fl, fh);
  g.sync();
  const double froot = db::to_f64(db::from_limbs2(fl, fh)) * 0x1p-28;
  const double fmin = mincont * froot;
  // the levels' places in the list, highest first
  uint64_t levels;
  {
    const int lv = db::kMaxLevels - 1 - g.lane;      // lane 0: level 63
    const int n = L.cnt[lv];
    int at = n;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int u = __shfl_up(at, o, kWave);
      if (g.lane >= o) at += u;
    }
    at -= n;
    levels = __builtin_bitreverse64(ballot(n > 0));
    if (g.wave == 0) {
      L.start[lv] = at;
      L.put[lv] = at;
    }
  }
  g.msync();
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    const int lev = p < A ? m.num(p) : 0;
    if (lev > 0) {
      const int k = __hip_atomic_fetch_add(&L.put[lev], 1, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
      m.set_list(k, p);
    }
  }
  // A leaf of the tree is a plateau of one level without a neighbour of a
  // higher one; its first pixel has no neighbour of its own level before it
  // either.  A candidate with at most one such pixel does not split.
  {
    int tops = 0;
    for (int c0 = 0; c0 < A && tops < 2; c0 += T) {
      const int p = c0 + g.tid;
      bool top = false;
      if (p < A) {
        const int lev = m.num(p);
        const int y = row_of(p), x = p - y * bw;
        const bool l = x > 0, r = x + 1 < bw, u = p >= bw, d = p + bw < A;
        top = lev > 0;
        auto before = [&](bool in, int q) {
          if (in) top = top && m.num(q) < lev;
        };
        auto after = [&](bool in, int q) {
          if (in) top = top && m.num(q) <= lev;
        };
        before(l, p - 1);
        before(u, p - bw);
        after(r, p + 1);
        after(d, p + bw);
        if (conn == 8) {
          before(l && u, p - bw - 1);
          before(r && u, p - bw + 1);
          after(l && d, p + bw - 1);
          after(r && d, p + bw + 1);
        }
      }
      int n;
      g.rank(top, &n);
      tops += n;
    }
    if (tops < 2) return 1;
  }
  g.msync();
  int root = 0, nch = 0;
  if constexpr (ONE_WAVE) {
    // a level adds a few tens of pixels: one wavefront builds the tree, its
    // phases ordered without the workgroup's barriers
    if (g.wave == 0) {
      const Grp<1> g1 = {g.lane, g.lane, 0, nullptr, nullptr};
      nch = db::build_tree(g1, m, conn, bw, A, row_of, L.T, L.start, L.cnt,
                           levels, froot, fmin, s.chains, s.chain_cap, &root);
      if (g.lane == 0) {
        L.put[0] = nch;
        L.put[1] = root;
      }
    }
    g.sync();
    nch = L.put[0];
    root = L.put[1];
    g.sync();
  } else {
    nch = db::build_tree(g, m, conn, bw, A, row_of, L.T, L.start, L.cnt,
                         levels, froot, fmin, s.chains, s.chain_cap, &root);
  }
  if (nch < 0) return -1;
  if (nch < 2) return 1;
  g.sync();
  if constexpr (M::kLds) {
    // nodes in the place of the sums, their list in that of the levels'
    db::Node* nodes = (db::Node*)L.S;
    if (nch <= (int)(sizeof(L.S) / sizeof(db::Node))) {
      int nsig = 0;
      for (int k0 = 0; k0 < nch; k0 += T) {
        const int k = k0 + g.tid;
        bool in = false;
        if (k < nch) {
          db::Node n;
          db::node_init(n, s.chains[k], fmin);
          nodes[k] = n;
          in = (n.flags & db::kNodeSig) || k == root;
        }
        int tot;
        const int at = nsig + g.rank(in, &tot);
        if (in) L.list[at] = (uint16_t)k;
        nsig += tot;
      }
      g.sync();
      if (g.tid == 0) db::prune_nodes(nodes, L.list, nsig, root);
      g.sync();
      if (nodes[root].nobj < 2) return 1;
      // each chain's object chain
      for (int k = g.tid; k < nch; k += T) {
        int a = k;
        while (!(nodes[a].flags & db::kNodeSig) && a != root)
          a = nodes[a].parent;
        const int o = nodes[a].objof;
        L.chn[k] = (uint16_t)(o < 0 ? kNone16 : o);
      }
      g.sync();
      const int k = finish_lds(g, L, c, A, bw, row_of, nch, root, clean, kc, s);
      if (k >= 0) return k;
    }
  }
  for (int k = g.tid; k < nch; k += T) db::chain_clear(s.chains[k]);
  g.sync();
  if (g.tid == 0) db::prune_tree(s.chains, nch, root, fmin);
  g.sync();
  if (ld_at(&s.chains[root].nobj) < 2) return 1;
  auto chain_of = [&](int p) {
    const int k = m.chf(p);
    return k < 0 ? root : k;
  };

  // seeds: the first pixel of each object chain (par reused for marks)
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    int o = -1;
    if (p < A) {
      m.set_par(p, -1);
      if (s.asg[p] >= 0) {
        o = s.chains[chain_of(p)].objof;
        if (o < 0) s.asg[p] = -2;          // not in a seed
      }
    }
    keyed_min(o >= 0, o, p, g.lane,
              [&](int k, int v) { min_at(&s.chains[k].first, v); });
  }
  g.sync();
  for (int j = g.tid; j < nch; j += T) {
    if (s.chains[j].objof == j) {
      const int f = ld_at(&s.chains[j].first);
      if (f != 0x7FFFFFFF) m.set_par(f, j);
    }
  }
  g.sync();
  // object slots in raster order of the first pixels
  int K = 0;
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    const int j = p < A ? m.par(p) : -1;
    int tot;
    const int k = K + g.rank(j >= 0, &tot);
    if (j >= 0 && k < s.obj_cap) {
      s.chains[j].slot = k;
      db::Obj& b = s.objs[k];
      for (int a = 0; a < 5; ++a)
        for (int l = 0; l < 4; ++l) b.m[a][l] = 0;
      b.fin[0] = 0;
      b.fin[1] = 0;
      b.nfin = 0;
      b.first = p;
      b.xmin = 0x7FFFFFFF;
      b.ymin = row_of(p);
      b.target = -1;
    }
    K += tot;
  }
  if (K > s.obj_cap) return -1;
  g.sync();
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    int k = -1, x = 0;
    if (p < A && s.asg[p] >= 0) {
      k = s.chains[s.chains[chain_of(p)].objof].slot;
      s.asg[p] = k;
      x = p - row_of(p) * bw;
    }
    keyed_min(k >= 0, k, x, g.lane,
              [&](int kk, int v) { min_at(&s.objs[kk].xmin, v); });
  }
  g.sync();
  // seed moments about each seed's corner, one sum at a time
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    int k = -1;
    int64_t d = 0, dx = 0, dy = 0;
    if (p < A) {
      k = s.asg[p];
      if (k >= 0) {
        const db::Obj& b = s.objs[k];
        const int y = row_of(p), x = p - y * bw;
        d = db::fixed_d(s.val[p]);
        dx = x - ld_at(&b.xmin);
        dy = y - b.ymin;
      }
    }
    for (int a = 0; a < 5; ++a) {
      const int64_t f = a == 0   ? 1
                        : a == 1 ? dx
                        : a == 2 ? dy
                        : a == 3 ? dx * dx
                                 : dy * dy;
      int64_t v[4];
      limbs4((__int128)d * f, v);
      keyed_add<4>(k >= 0, k, v, g.lane, [&](int kk, int j, int64_t sum) {
        add_at(&s.objs[kk].m[a][j], sum);
      });
    }
  }
  g.sync();
  for (int k = g.tid; k < K; k += T) {
    db::Obj& b = s.objs[k];
    int64_t l[5][4];
    for (int a = 0; a < 5; ++a)
      for (int j = 0; j < 4; ++j) l[a][j] = ld_at(&b.m[a][j]);
    const double fS = db::to_f64(db::from_limbs4(l[0]));
    const double mx = db::to_f64(db::from_limbs4(l[1])) / fS;
    const double my = db::to_f64(db::from_limbs4(l[2])) / fS;
    const double x2 = db::to_f64(db::from_limbs4(l[3])) / fS - mx * mx;
    const double y2 = db::to_f64(db::from_limbs4(l[4])) / fS - my * my;
    const int xmin = ld_at(&b.xmin);
    b.F = fS * 0x1p-28;
    b.xc = (double)(c.x0 + xmin) + mx;
    b.yc = (double)(c.y0 + b.ymin) + my;
    b.s2 = (x2 + y2) + 1.0 / 6.0;
  }
  g.sync();
  // the other pixels: the brightest model
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    if (p < A && s.asg[p] == -2) {
      const int py = row_of(p);
      const double x = (double)(c.x0 + p - py * bw);
      const double y = (double)(c.y0 + py);
      double best = -1.0;
      int bk = 0;
      for (int k = 0; k < K; ++k) {
        const db::Obj& b = s.objs[k];
        const double dx = x - b.xc;
        const double dy = y - b.yc;
        const double d2 = dx * dx + dy * dy;
        const double den = b.s2 + d2;
        const double sc = (b.F * b.s2) / (den * den);
        if (sc > best) {
          best = sc;
          bk = k;
        }
      }
      s.asg[p] = bk;
    }
  }
  g.sync();
  if (!clean) return K;

  // cleaning
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    int k = -1;
    int64_t v[3] = {0, 0, 0};
    if (p < A) {
      k = s.asg[p];
      if (k >= 0) {
        const int64_t d = db::fixed_d(s.val[p]);
        v[0] = (int64_t)(uint32_t)d;
        v[1] = d >> 32;
        v[2] = 1;
      }
    }
    keyed_add<3>(k >= 0, k, v, g.lane, [&](int kk, int j, int64_t sum) {
      if (j < 2) add_at(&s.objs[kk].fin[j], sum);
      else add_at(&s.objs[kk].nfin, sum);
    });
  }
  g.sync();
  const double pi = 3.14159265358979311600;   // binary64 nearest to pi
  for (int o = g.tid; o < K; o += T) {
    db::Obj& b = s.objs[o];
    const double mu =
        db::to_f64(db::from_limbs2(ld_at(&b.fin[0]), ld_at(&b.fin[1]))) *
        0x1p-28 / (double)ld_at(&b.nfin);
    double tot = 0.0, best = -1.0;
    int bm = -1;
    for (int m = 0; m < K; ++m) {
      if (m == o) continue;
      const db::Obj& n = s.objs[m];
      const bool brighter = n.F > b.F || (n.F == b.F && m < o);
      if (!brighter) continue;
      const double dx = b.xc - n.xc;
      const double dy = b.yc - n.yc;
      const double d2 = dx * dx + dy * dy;
      double den = n.s2 + d2;
      den = den * den;
      den = pi * den;
      const double cm = kc * ((n.F * n.s2) / den);
      tot += cm;
      if (cm > best) {
        best = cm;
        bm = m;
      }
    }
    b.target = (bm >= 0 && mu - tot < c.t0) ? bm : o;
  }
  g.sync();
  // follow merges to an object that stays; number the survivors in order
  for (int o = g.tid; o < K; o += T) {
    int k = o;
    while (s.objs[k].target != k) k = s.objs[k].target;
    s.objs[o].final_obj = k;
  }
  g.sync();
  int nk = 0;
  for (int o0 = 0; o0 < K; o0 += T) {
    const int o = o0 + g.tid;
    const bool surv = o < K && s.objs[o].final_obj == o;
    int tot;
    const int r = nk + g.rank(surv, &tot);
    if (o < K) s.objs[o].idx = surv ? r : -1;
    nk += tot;
  }
  g.sync();
  for (int c0 = 0; c0 < A; c0 += T) {
    const int p = c0 + g.tid;
    if (p < A) {
      const int k = s.asg[p];
      if (k >= 0) s.asg[p] = s.objs[s.objs[k].final_obj].idx;
    }
  }
  g.sync();
  return nk;
}

// One candidate: its tree in LDS if the box fits and its sums fit 64 bits
// (every weight counted at a level is positive and at most the peak's), else
// in the pool.
template <int NW, int CAP, bool POOL>
__device__ __forceinline__ int deblend_row(
    const Grp<NW>& g, DbLds<NW, CAP>& L, const FrameDev& fr, const DbCand& c,
    int conn, int nthresh, int clean, double mincont, double kc,
    db::Pool& s) {
  const int64_t A = (int64_t)c.bw * c.bh;
  const bool fits =
      A <= CAP && c.peak * (double)c.m < 0x1p62 / 268435456.0;
  if (!POOL || fits) {
    return deblend_group<(NW > 1), NW, CAP>(g, L, TreeLds<NW, CAP>{L}, fr, c,
                                            conn, nthresh, clean, mincont,
                                            kc, s);
  } else {
    const Grp<NW, true> gp = {g.tid, g.lane, g.wave, g.red, g.red64};
    return deblend_group<false, NW, CAP>(gp, L, TreePool{s, (int*)s.objs}, fr,
                                         c, conn, nthresh, clean, mincont, kc,
                                         s);
  }
}

// Candidates of class CLS, one per group, taken from the queue counter: class
// 0 in row order, the others from k_db_need's list (class 2 from its front,
// class 1 from its back).  The group is number gi of ng.
template <int NW, int CAP, int CLS>
__device__ __forceinline__ void db_groups(
    const Work& wk, const ipp_sources& cand, const int64_t* off,
    const int64_t* tot, char* pool, int64_t pool_units, double nsigma,
    int conn, int nthresh, int clean, double mincont, double kc, int64_t* cnt,
    int64_t* queue, const int32_t* big, const int64_t* nbig,
    DbLds<NW, CAP>& lds, int gi, int ng) {
  Grp<NW> g;
  g.tid = threadIdx.x % Grp<NW>::T;
  g.lane = threadIdx.x & (kWave - 1);
  g.wave = g.tid / kWave;
  g.red = lds.red;
  g.red64 = lds.red64;
  const long long n = table_rows(cand);
  const bool fits = *tot <= pool_units;
  if (CLS == 0) {
    // the counts of the rows that need no deblending (beyond the table: 0;
    // single pixels, or every row when the pool is too small: 1)
    for (long long r = gi * (long long)Grp<NW>::T + g.tid; r <= cand.capacity;
         r += (long long)ng * Grp<NW>::T) {
      if (r >= n) cnt[r] = 0;
      else if (cand.npix[r] < 2 || !fits) cnt[r] = 1;
    }
  }
  if (!fits) return;
  const long long nlist = CLS == 0 ? n : (CLS == 2 ? nbig[0] : nbig[1]);
  // class 0 takes its rows from several counters, a group from one of them
  // (thousands of short candidates queue up at one address: 12 ns each)
  const int nq = CLS == 0 ? db_queues(cand.capacity) : 1;
  const int qi = CLS == 0 ? gi % nq : 0;
  while (true) {
    long long r = 0;
    if (g.tid == 0)
      r = (long long)atomicAdd(
          (unsigned long long*)queue + qi * kDbQueueStep, 1ull);
    if constexpr (NW == 1) {
      r = __shfl(r, 0, kWave);
    } else {
      if (g.tid == 0) lds.red64[0] = r;
      __syncthreads();
      r = lds.red64[0];
      __syncthreads();
    }
    if (CLS == 0) r = r * nq + qi;
    if (r >= nlist) break;
    if (CLS == 2) r = big[r];
    if (CLS == 1) r = big[cand.capacity - r];
    const int m = cand.npix[r];
    DbCand c;
    c.x0 = cand.xmin[r];
    c.y0 = cand.ymin[r];
    c.bw = cand.xmax[r] - c.x0 + 1;
    c.bh = cand.ymax[r] - c.y0 + 1;
    c.peak = cand.peak[r];
    const int64_t A = (int64_t)c.bw * c.bh;
    if (CLS == 0 && (m < 2 || db_class(A, c.peak, m) != 0)) continue;
    const int f = cand.frame[r];
    const FrameDev fr = wk.frames[f];
    c.lab = cand.label[r];
    c.m = m;
    c.t0 = nsigma * (double)fr.rms[(int64_t)cand.peak_y[r] * fr.w +
                                   cand.peak_x[r]];
    db::Pool s = db::carve(pool + off[r] * 256, A, m);
    int k = deblend_row<NW, CAP, CLS == 2>(g, lds, fr, c, conn, nthresh,
                                           clean, mincont, kc, s);
    if (k < 0) {
      if (g.tid == 0)
        atomicOr((unsigned long long*)&wk.counters[2], 2ull);
      k = 1;
    }
    if (g.tid == 0) cnt[r] = k;
    g.sync();
  }
}

}  // namespace

#define IPP_DB_KERNEL(NAME, NW, CAP, CLS)                                    \
  __global__ __launch_bounds__(NW * kWave) void NAME(                        \
      Work wk, ipp_sources cand, const int64_t* off, const int64_t* tot,     \
      char* pool, int64_t pool_units, double nsigma, int conn, int nthresh,  \
      int clean, double mincont, double kc, int64_t* cnt, int64_t* queue,    \
      const int32_t* big, const int64_t* nbig) {                             \
    __shared__ DbLds<NW, CAP> lds;                                           \
    db_groups<NW, CAP, CLS>(wk, cand, off, tot, pool, pool_units, nsigma,    \
                            conn, nthresh, clean, mincont, kc, cnt, queue,   \
                            big, nbig, lds, blockIdx.x, gridDim.x);          \
  }
// Boxes of up to 512 pixels: a wavefront per candidate (13 KB of LDS each);
// of up to 2048: a workgroup of four (51 KB); larger ones, in LDS up to 6144
// pixels (149 KB) and in the pool beyond: a workgroup of eight.  24 bytes of
// LDS per box pixel bound the candidates in flight, and each is a chain of
// dependent LDS accesses (some four hundred instructions per level, half of
// the time waiting).  On the 18,676 candidates of four 2048 x 2048 frames the
// three take 457, 498 and 305 us one after the other; working through every pixel of the box at
// every level, as a wavefront and a workgroup kernel, took 1573 and 3741.
IPP_DB_KERNEL(k_db_small, 1, kDbSmallBox, 0)
IPP_DB_KERNEL(k_db_mid, 4, kDbMidBox, 1)
IPP_DB_KERNEL(k_db_large, 8, kDbBigBox, 2)
#undef IPP_DB_KERNEL

// Everything in one launch, for tables of at most kDbAllRows rows: a workgroup
// of eight wavefronts takes the candidates of the larger classes, then each of
// its wavefronts small ones (2048 in flight on the device, so none waits).
// Three launches, one of them forked to a side stream and joined, cost the
// host more than a few candidates' work: 16 candidates of a 128 x 128 frame,
// two levels, 226 us a call, 175 so (204 with two kernels on one stream); 218
// of 300 x 300, 32 levels, 501 and 342.  Longer tables gain as well while their
// large candidates are few (682 of 512 x 512 in a table of 5120: 487 and 317)
// and lose where they are many (4,700 of a crowded 2048^2 frame: 639 and
// 730), which only the device knows.
__global__ __launch_bounds__(8 * kWave) void k_db_all(
    Work wk, ipp_sources cand, const int64_t* off, const int64_t* tot,
    char* pool, int64_t pool_units, double nsigma, int conn, int nthresh,
    int clean, double mincont, double kc, int64_t* cnt, int64_t* queue2,
    int64_t* queue1, int64_t* queue0, const int32_t* big,
    const int64_t* nbig) {
  __shared__ union {
    DbLds<8, kDbBigBox> group;
    DbLds<1, kDbSmallBox> wave[8];
  } lds;
  db_groups<8, kDbBigBox, 2>(wk, cand, off, tot, pool, pool_units, nsigma,
                             conn, nthresh, clean, mincont, kc, cnt, queue2,
                             big, nbig, lds.group, blockIdx.x, gridDim.x);
  db_groups<8, kDbBigBox, 1>(wk, cand, off, tot, pool, pool_units, nsigma,
                             conn, nthresh, clean, mincont, kc, cnt, queue1,
                             big, nbig, lds.group, blockIdx.x, gridDim.x);
  __syncthreads();                     // the group's LDS is the waves' now
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  db_groups<1, kDbSmallBox, 0>(wk, cand, off, tot, pool, pool_units, nsigma,
                               conn, nthresh, clean, mincont, kc, cnt, queue0,
                               big, nbig, lds.wave[wv], blockIdx.x * 8 + wv,
                               gridDim.x * 8);
}

__global__ __launch_bounds__(kBlock) void k_db_zero(Work wk) {
  for (int f = blockIdx.y; f < wk.nframes; f += gridDim.y) {
    const FrameDev fr = wk.frames[f];
    const int64_t np = (int64_t)fr.h * fr.w;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < np;
         i += (int64_t)gridDim.x * kBlock)
      fr.objects[i] = 0;
  }
}

// The box pixels [eb, ee) of one candidate, a wavefront: the ids into the
// object map and, for a split candidate (asg: each pixel's object), each
// object's pixel count and box, added to its row with atomics (integer sums,
// minima and maxima: the same whatever the order).  Up to kDbWriteObj objects
// are accumulated in LDS, every pixel with its own LDS atomics, and added
// once at the end, an object a lane; more of them are reduced over the wave
// round by round.  Four rounds' loads are in flight together.
namespace {
struct DbWrite {
  const FrameDev* fr;
  const int32_t* asg;                  // nullptr: not split
  int lab, id0, x0, y0, bw, k;         // k: objects
  int64_t base;
};
constexpr int kDbWriteObj = 64;
struct DbWriteLds {
  int npix[kDbWriteObj], xmin[kDbWriteObj], xmax[kDbWriteObj];
  int ymin[kDbWriteObj], ymax[kDbWriteObj];
};

__device__ __forceinline__ void db_add(const ipp_sources& obj, int64_t o,
                                       int n, int xn, int xm, int yn, int ym,
                                       int lane) {
#pragma unroll
  for (int s = kWave / 2; s > 0; s >>= 1) {
    xn = min(xn, __shfl_xor(xn, s, kWave));
    xm = max(xm, __shfl_xor(xm, s, kWave));
    yn = min(yn, __shfl_xor(yn, s, kWave));
    ym = max(ym, __shfl_xor(ym, s, kWave));
  }
  if (lane == 0) {
    atomicAdd(&obj.npix[o], n);
    atomicMin(&obj.xmin[o], xn);
    atomicMax(&obj.xmax[o], xm);
    atomicMin(&obj.ymin[o], yn);
    atomicMax(&obj.ymax[o], ym);
  }
}

__device__ __forceinline__ void db_write_part(const DbWrite& c,
                                              const ipp_sources& obj,
                                              int64_t eb, int64_t ee,
                                              DbWriteLds& L, int lane) {
  constexpr int kAhead = 4, kFar = 0x7FFFFFFF;
  const bool table = c.asg && c.k <= kDbWriteObj;
  const int fw = c.fr->w;
  const int dy = kWave / c.bw, dx = kWave - (kWave / c.bw) * c.bw;
  int y = (int)((eb + lane) / c.bw);
  int x = (int)(eb + lane - (int64_t)y * c.bw);
  if (table) {
    L.npix[lane] = 0;
    L.xmin[lane] = L.ymin[lane] = kFar;
    L.xmax[lane] = L.ymax[lane] = -1;
    __builtin_amdgcn_wave_barrier();   // the wave's LDS operations in order
  }
  for (int64_t e0 = eb; e0 < ee; e0 += kAhead * kWave) {
    int a[kAhead], px[kAhead], py[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (e0 + k * kWave >= ee) break;               // wave-uniform
      const int64_t e = e0 + k * kWave + lane;
      px[k] = c.x0 + x;
      py[k] = c.y0 + y;
      a[k] = -1;
      if (e < ee) {
        if (c.asg) a[k] = c.asg[e];
        else if (c.fr->labels[(int64_t)py[k] * fw + px[k]] == c.lab) a[k] = 0;
      }
      y += dy;
      x += dx;
      if (x >= c.bw) {
        x -= c.bw;
        ++y;
      }
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (e0 + k * kWave >= ee) break;
      if (a[k] >= 0)
        c.fr->objects[(int64_t)py[k] * fw + px[k]] = c.id0 + a[k];
    }
    if (!c.asg) continue;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (e0 + k * kWave >= ee) break;
      const bool act = a[k] >= 0 && c.base + a[k] < obj.capacity;
      if (table) {
        if (act) {
          atomicAdd(&L.npix[a[k]], 1);
          atomicMin(&L.xmin[a[k]], px[k]);
          atomicMax(&L.xmax[a[k]], px[k]);
          atomicMin(&L.ymin[a[k]], py[k]);
          atomicMax(&L.ymax[a[k]], py[k]);
        }
        continue;
      }
      uint64_t left = ballot(act);
      while (left) {
        const int k0 =
            __builtin_amdgcn_readlane(a[k], __builtin_ctzll(left));
        const bool in = act && a[k] == k0;
        const uint64_t mk = ballot(in);
        left &= ~mk;
        db_add(obj, c.base + k0, (int)__popcll(mk), in ? px[k] : kFar,
               in ? px[k] : -1, in ? py[k] : kFar, in ? py[k] : -1, lane);
      }
    }
  }
  if (!table) return;
  __builtin_amdgcn_wave_barrier();
  if (lane < c.k && L.npix[lane] > 0) {
    const int64_t o = c.base + lane;
    atomicAdd(&obj.npix[o], L.npix[lane]);
    atomicMin(&obj.xmin[o], L.xmin[lane]);
    atomicMax(&obj.xmax[o], L.xmax[lane]);
    atomicMin(&obj.ymin[o], L.ymin[lane]);
    atomicMax(&obj.ymax[o], L.ymax[lane]);
  }
  __builtin_amdgcn_wave_barrier();     // the table is free again
}
}  // namespace

// A wavefront per candidate: its objects' rows (lane-parallel), then its
// bounding box.  Boxes over kDbWritePart pixels are left for the workgroup's
// wavefronts together, in parts of that size.  Bound by latency and by the
// last workgroups' large boxes: 18,676 candidates of four 2048 x 2048 frames
// 60 us (102 with sixteen wavefronts a workgroup; 155 with a wavefront for
// every box and each object of a round reduced by shuffles).
constexpr int64_t kDbWritePart = 1024;

__global__ __launch_bounds__(kDbWriteThreads) void k_db_write(
    Work wk, ipp_sources cand, const int64_t* off, const int64_t* tot,
    const char* pool, int64_t pool_units, const int64_t* cnt,
    const int64_t* ooff, ipp_sources obj, int32_t* parent) {
  constexpr int NW = kDbWriteThreads / kWave;
  __shared__ long long large[NW];
  __shared__ int nlarge;
  __shared__ DbWriteLds tables[NW];
  const long long n = table_rows(cand);
  const bool fits = *tot <= pool_units;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  auto describe = [&](long long r, int64_t* A) {
    DbWrite c;
    const int f = cand.frame[r];
    c.fr = &wk.frames[f];
    c.lab = cand.label[r];
    c.base = ooff[r];
    c.id0 = (int32_t)(c.base - ooff[cand.frame_offsets[f]] + 1);
    c.x0 = cand.xmin[r];
    c.y0 = cand.ymin[r];
    c.bw = cand.xmax[r] - c.x0 + 1;
    *A = (int64_t)c.bw * (cand.ymax[r] - c.y0 + 1);
    c.asg = nullptr;
    c.k = (int)cnt[r];
    const int m = cand.npix[r];
    if (c.k != 1 && fits && m >= 2)
      c.asg = db::carve((char*)pool + off[r] * 256, *A, m).asg;
    return c;
  };
  for (long long r0 = blockIdx.x * (long long)NW; r0 < n;
       r0 += (long long)gridDim.x * NW) {
    if (threadIdx.x == 0) nlarge = 0;
    __syncthreads();
    const long long r = r0 + wv;
    if (r < n) {
      int64_t A;
      const DbWrite c = describe(r, &A);
      const int k = c.k;
      for (int j = lane; j < k; j += kWave) {
        const int64_t o = c.base + j;
        if (o >= obj.capacity) break;
        obj.frame[o] = cand.frame[r];
        obj.label[o] = c.id0 + j;
        parent[o] = c.lab;
        if (k == 1) {
          obj.npix[o] = cand.npix[r];
          obj.xmin[o] = c.x0;
          obj.xmax[o] = cand.xmax[r];
          obj.ymin[o] = c.y0;
          obj.ymax[o] = cand.ymax[r];
        } else {
          obj.npix[o] = 0;
          obj.xmin[o] = 0x7FFFFFFF;
          obj.xmax[o] = -1;
          obj.ymin[o] = 0x7FFFFFFF;
          obj.ymax[o] = -1;
        }
      }
      if (A > kDbWritePart) {
        if (lane == 0) large[atomicAdd(&nlarge, 1)] = r;
      } else {
        // the rows' initial values are in memory before the atomics (this
        // wave's stores completed; the atomics are performed in the same
        // L2): a workgroup-scope release, which waits for them without the
        // device-scope cache write-back
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        db_write_part(c, obj, 0, A, tables[wv], lane);
      }
    }
    __syncthreads();                   // (the same release, to the workgroup)
    const int nl = nlarge;
    int next = wv;                     // this wave's next part, of all of them
    for (int i = 0; i < nl; ++i) {
      int64_t A;
      const DbWrite c = describe(large[i], &A);
      const int parts = (int)((A + kDbWritePart - 1) / kDbWritePart);
      for (; next < parts; next += NW) {
        const int64_t eb = next * kDbWritePart;
        db_write_part(c, obj, eb, min(A, eb + kDbWritePart), tables[wv], lane);
      }
      next -= parts;
    }
    __syncthreads();                   // the list is free again
  }
}

__global__ void k_db_offsets(Work wk, ipp_sources cand, const int64_t* ooff,
                             const int64_t* total, ipp_sources obj) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f <= wk.nframes)
    obj.frame_offsets[f] =
        f < wk.nframes ? ooff[cand.frame_offsets[f]] : *total;
  if (f == 0) {
    if (obj.n_total) *obj.n_total = *total;
    wk.counters[3] = *total;
  }
}

__global__ __launch_bounds__(kBlock) void k_db_flags(
    ipp_sources cand, const int64_t* cnt, const int64_t* total,
    ipp_sources obj, const int32_t* parent) {
  long long n = *total;
  if (n > obj.capacity) n = obj.capacity;
  for (long long o = blockIdx.x * (long long)kBlock + threadIdx.x; o < n;
       o += (long long)gridDim.x * kBlock) {
    const int64_t cr = cand.frame_offsets[obj.frame[o]] + parent[o] - 1;
    if (cnt[cr] > 1) obj.flags[o] |= IPP_SRC_BLENDED;
  }
}

}  // namespace ipp

namespace ipp {
__global__ void k_db_diag(const int64_t* tot, int64_t pool_units,
                          const int64_t* counters, int64_t* diag) {
  if (threadIdx.x == 0) {
    diag[0] = tot[0] * 256;
    diag[1] = pool_units * 256;
    diag[2] = (tot[0] > pool_units ? 1 : 0) | counters[2];
    diag[3] = tot[1];
  }
}
}  // namespace ipp
