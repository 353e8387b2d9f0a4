// lt_tree.hip -- tree kernels and the C ABI of the adaptation cycle.
//
// Keys stay sorted throughout: every kernel that changes the leaf set counts
// its outputs per input leaf, takes an exclusive scan of the counts with
// decoupled look-back, and writes its outputs in input order, which is
// Morton order.  No sort, no linearisation pass and no atomics decide any
// output position, so results are deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "tree.hpp"

using lt::KeyGeom;

namespace lt {

namespace {
thread_local std::string g_err;
}

void set_error(const std::string& msg) { g_err = msg; }

lt_status fail(lt_status s, const std::string& msg) {
  g_err = msg;
  return s;
}

namespace {
std::mutex g_alloc_mu;
Alloc g_alloc;  // registered by lt_set_allocator; empty: hipMalloc / hipFree
}  // namespace

Alloc registered_alloc() {
  std::lock_guard<std::mutex> lk(g_alloc_mu);
  return g_alloc;
}

void register_alloc(const Alloc& A) {
  std::lock_guard<std::mutex> lk(g_alloc_mu);
  g_alloc = A;
}

hipError_t dev_malloc(const Alloc& A, void** p, size_t bytes) {
  *p = nullptr;
  if (!A.alloc) return hipMalloc(p, bytes);
  *p = A.alloc(bytes, nullptr, A.ctx);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}

hipError_t dev_free(const Alloc& A, void* p) {
  if (!p) return hipSuccess;
  if (!A.free_) return hipFree(p);
  const hipError_t e = hipDeviceSynchronize();
  A.free_(p, nullptr, A.ctx);
  return e;
}

}  // namespace lt

#define LT_HIP(expr)                                                                   \
  do {                                                                                 \
    hipError_t e_ = (expr);                                                            \
    if (e_ != hipSuccess)                                                              \
      return lt::fail(LT_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

#define LT_TRY(expr)                \
  do {                              \
    lt_status s_ = (expr);          \
    if (s_ != LT_OK) return s_;     \
  } while (0)

namespace lt {
namespace {


int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ------------------------------------------------------------------ kernels
// Zero the look-back words and counters before a scan.
__global__ void k_clear_scan(uint64_t* status, int64_t ntiles, DevCtr* ctr, int clear_err, int clear_list) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < ntiles) status[i] = 0;
  if (i == 0) {
    if (clear_list) {  // the lists adapt and balance refinement build for the next pass
      ctr->nexam[0] = 0;
      ctr->nfused = 0;
    }
    ctr->ticket = 0;
    ctr->total = 0;
    ctr->nmarked = 0;
    ctr->nfgroups = 0;
    if (clear_err) ctr->err = 0;
  }
}

// The same done by a kernel that runs ahead of the scan anyway (a launch less:
// without seven of them a captured 3D cycle of 37 000 leaves takes 312 us instead
// of 336).  ctr null: nothing.
struct ScanClear {
  uint64_t* status;
  int64_t ntiles;
  DevCtr* ctr;
  int64_t* nexam;  // the examine list the scan appends to
  int64_t* cnt_dst;
  const int64_t* cnt_src;
};

// Every thread of a launch of `threads` calls; tid: its index there.
__device__ inline void scan_clear(const ScanClear& c, int64_t tid, int64_t threads) {
  if (!c.ctr) return;
  for (int64_t i = tid; i < c.ntiles; i += threads) c.status[i] = 0;
  if (tid == 0) {
    if (c.nexam) *c.nexam = 0;
    if (c.cnt_dst) *c.cnt_dst = *c.cnt_src;
    c.ctr->ticket = 0;
    c.ctr->total = 0;
    c.ctr->nmarked = 0;
    c.ctr->nfgroups = 0;
  }
}

// Start of a captured cycle: words from pinned host memory, everything cleared
// for adapt's scan, the count before the cycle kept.
__global__ void k_cycle_start(const uint32_t* __restrict__ host, uint32_t* __restrict__ p, int n, ScanClear c) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = host[i];
  scan_clear(c, i, int64_t(gridDim.x) * blockDim.x);
  if (i == 0) {
    c.ctr->err = 0;
    c.ctr->conv = 0;
    c.ctr->nfused = 0;
    c.ctr->nexam[0] = 0;
    c.ctr->nexam[1] = 0;
  }
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Uniform tree: leaf i of depth D has Morton index i * span(D).
__global__ void k_uniform(KeyGeom g, int depth, int64_t n, uint64_t* keys) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) keys[i] = make_key(g, uint64_t(i) << (g.dim * (g.dmax - depth)), depth);
}

// Ensemble of uniform trees: mesh m holds 2^(dim*depth_m) leaves starting at offs[m].
__global__ void k_uniform_batch(KeyGeom g, const int64_t* __restrict__ offs,
                                const int8_t* __restrict__ depth, int nmesh, int64_t n,
                                uint64_t* __restrict__ keys) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int lo = 0, hi = nmesh - 1;
  while (lo < hi) {  // last mesh whose first leaf is <= i
    const int mid = (lo + hi + 1) >> 1;
    if (offs[mid] <= i)
      lo = mid;
    else
      hi = mid - 1;
  }
  const int d = depth[lo];
  keys[i] = (uint64_t(lo) << g.mesh_shift) |
            make_key(g, uint64_t(i - offs[lo]) << (g.dim * (g.dmax - d)), d);
}

// First leaf of every mesh (offs[nmesh] = n).
__global__ void k_mesh_offsets(KeyGeom g, const uint64_t* __restrict__ keys, int64_t n, int nmesh,
                               int64_t* __restrict__ offs) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m > nmesh) return;
  offs[m] = m == nmesh ? n : lower_bound(keys, n, uint64_t(m) << g.mesh_shift);
}

// Complete linear tree check: each key valid, and the Morton range of leaf i
// ends exactly where leaf i+1 starts (so keys ascend, tile, and do not overlap).
__global__ void k_validate(KeyGeom g, const uint64_t* __restrict__ keys, int64_t n, unsigned* err) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t k = keys[i];
  const int d = key_depth(g, k);
  const uint64_t m = key_m(g, k);
  bool ok = d <= g.dmax;
  if (ok) {
    if ((m & (span(g, d) - 1)) != 0) ok = false;                      // padding bits
    if (g.dim * g.dmax < 64 && (m >> (g.dim * g.dmax)) != 0) ok = false;  // outside the domain
  }
  if (ok) {
    const uint64_t end = m + span(g, d);
    if (i + 1 < n) {
      const uint64_t kn = keys[i + 1];
      if (key_depth(g, kn) > g.dmax || key_m(g, kn) != end) ok = false;
    } else {
      const uint64_t full = g.dim * g.dmax >= 64 ? 0 : (uint64_t(1) << (g.dim * g.dmax));
      if (end != full) ok = false;
    }
    if (i == 0 && m != 0) ok = false;
  }
  if (!ok) atomicOr(err, ERR_INVALID_TREE);
}

// Adaptation (Section 4.1).  Per leaf: +1 -> 2^dim children, first leaf of a
// complete all -1 family -> parent, other members of such a family -> nothing,
// everything else -> itself.
// Balance marks written by adapt (see the marking pass): the children of a
// refined leaf are to be examined, a fused parent is to be checked against
// finer neighbours; every other leaf is balanced with its neighbours already.
constexpr uint32_t kMarkExamine = 4u;
// Workgroups of a marking pass over the examine list (it strides over the
// list, whose length is on the device).
constexpr int64_t kMarkGrid = 2048;
constexpr uint32_t kMarkFused = 16u;

// An append to a device-side list.  A captured cycle whose output outgrows
// its capacity keeps running (the host discards the result), so appends past
// the list's capacity are dropped rather than written.
__device__ inline void list_put(int32_t* __restrict__ l, int64_t i, int64_t cap, int32_t v) {
  if (i < cap) l[i] = v;
}

// What a tile of leaves emits, from one mask per wave and round: a lane's
// output offset is the tile's prefix, plus its wave's, plus the outputs of the
// wave's earlier rounds and of the lower lanes of its own, all of them
// population counts.
struct WaveOut {
  int base;  // outputs of the block's earlier waves
  int all;   // of the whole block
};

// Exclusive scans over the block's waves of two small counts (their sums over
// a block below 2^31), every thread calling with its wave's.
__device__ inline void block_waves(int a, int b, WaveOut* A, WaveOut* B) {
  constexpr int kWaves = kScanBig / 64;
  __shared__ int wa[kWaves], wb[kWaves];
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    wa[w] = a;
    wb[w] = b;
  }
  __syncthreads();
  int ea = 0, eb = 0, ta = 0, tb = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    ea += i < w ? wa[i] : 0;
    eb += i < w ? wb[i] : 0;
    ta += wa[i];
    tb += wb[i];
  }
  __syncthreads();
  *A = WaveOut{ea, ta};
  *B = WaveOut{eb, tb};
}

// Reserves `all` entries of a device-side list for the block (one atomic);
// returns where they start.
__device__ inline int64_t block_append(int all, int64_t* count) {
  __shared__ int64_t s_at;
  if (threadIdx.x == 0)
    s_at = all > 0 ? int64_t(atomicAdd(reinterpret_cast<unsigned long long*>(count), (unsigned long long)all)) : 0;
  __syncthreads();
  const int64_t at = s_at;
  __syncthreads();
  return at;
}

__device__ inline uint64_t lanes_below() { return (uint64_t(1) << (threadIdx.x & 63)) - 1; }

// R rounds of 64 consecutive leaves per wave.  Bound: latency (the ticket, the
// leaves, a flagged leaf's family, the look-back, the stores), so a tile's
// loads and stores are whole rows of consecutive leaves and its counts are
// ballots.  With eight consecutive leaves per thread and 64-bit scans of their
// counts adapt took 36 us at 37 000 leaves and 44 at 1.9M, a refinement pass 18
// and 40; in this form 12 and 32, 8 and 19.
template <int R>
__global__ __launch_bounds__(kScanBig) void k_adapt(KeyGeom g, const uint64_t* __restrict__ in,
                                                  const int8_t* __restrict__ flags,
                                                  uint64_t* __restrict__ out, int64_t cap,
                                                  ScanState st, uint32_t* __restrict__ marks,
                                                  int32_t* __restrict__ elist, int64_t* nexam,
                                                  int64_t ecap, int32_t* __restrict__ flist,
                                                  int64_t* nflist, int64_t fcap) {
  const int64_t tile = take_ticket(st);
  if (tile >= scan_tiles(st)) return;
  const int64_t n = st.items.get();
  const int lane = threadIdx.x & 63;
  const int64_t base = tile * (int64_t(kScanBig) * R) + int64_t(threadIdx.x >> 6) * (64 * R) + lane;
  const int nc = g.nchild();
  uint64_t key[R];
  uint64_t one[R], ref[R], par[R];  // lanes that emit themselves or their parent; their children; their parent
  int n_one = 0, n_ref = 0, n_par = 0;
  unsigned err = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t i = base + 64 * k;
    int a = 3;  // 0 keep, 1 refine, 2 emit parent, 3 drop
    key[k] = 0;
    if (i < n) {
      const uint64_t kk = in[i];
      key[k] = kk;
      int f = flags[i];
      if (f < -1 || f > 1) {
        err |= ERR_BAD_FLAG;
        f = 0;
      }
      const int d = key_depth(g, kk);
      int lo, hi;
      depth_limits(g, kk, &lo, &hi);
      if (f == 1 && d >= hi) f = 0;
      if (f == -1 && d <= lo) f = 0;
      a = 0;
      if (f == 1) {
        a = 1;
      } else if (f == -1) {
        // The family is complete iff the 2^dim keys around i are exactly the
        // siblings (consecutive, same depth, raw IDs incrementing by one).
        const uint64_t m = key_m(g, kk);
        const int c = child_index(g, m, d);
        const int64_t h = i - c;
        const uint64_t step = uint64_t(1) << (g.dim * (g.dmax - d) + g.mb);
        const uint64_t k0 = kk - uint64_t(c) * step;
        bool all = h >= 0 && h + nc <= n;
        if (all) {
          // every sibling's key and flag loaded before any is compared: one
          // round trip instead of a chain of 2^dim dependent ones
          uint64_t sk[8];
          int sf[8];
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (j < nc) {
              sk[j] = in[h + j];
              sf[j] = flags[h + j];
            }
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (j < nc) all = all && sk[j] == k0 + uint64_t(j) * step && sf[j] == -1;
        }
        if (all) a = c == 0 ? 2 : 3;
      }
    }
    ref[k] = __ballot(a == 1);
    par[k] = __ballot(a == 2);
    one[k] = __ballot(a == 0) | par[k];
    n_one += __popcll(one[k]);
    n_ref += __popcll(ref[k]);
    n_par += __popcll(par[k]);
  }
  // new children go on the list of leaves the first balance pass examines,
  // fused parents on the list it probes around
  WaveOut wr, wp;
  block_waves(n_ref * nc, n_par, &wr, &wp);
  WaveOut wo, unused;
  block_waves(n_one, 0, &wo, &unused);
  int64_t eo = elist ? block_append(wr.all, nexam) + wr.base : 0;
  int64_t fo = flist ? block_append(wp.all, nflist) + wp.base : 0;
  int64_t o = tile_prefix(st, tile, int64_t(wr.all) + wo.all) + wr.base + wo.base;
  const uint64_t below = lanes_below();
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int rb = __popcll(ref[k] & below);
    const int64_t q = o + int64_t(rb) * nc + __popcll(one[k] & below);
    const int64_t eq = eo + int64_t(rb) * nc, fq = fo + __popcll(par[k] & below);
    o += int64_t(__popcll(ref[k])) * nc + __popcll(one[k]);
    eo += int64_t(__popcll(ref[k])) * nc;
    fo += __popcll(par[k]);
    const bool is_ref = (ref[k] >> lane) & 1, is_par = (par[k] >> lane) & 1;
    if (!is_ref && !((one[k] >> lane) & 1)) continue;
    const int cnt = is_ref ? nc : 1;
    const uint64_t kk = key[k];
    if (q + cnt > cap) {
      err |= ERR_CAPACITY;
      // the slots below the capacity still get a valid key: the kernels after
      // this one in a captured cycle read them before the result is discarded
      for (int64_t t = q; t < cap && t < q + cnt; ++t) {
        out[t] = kk;
        if (marks) marks[t] = 0u;
      }
      if (elist && is_ref)
        for (int c = 0; c < nc; ++c) list_put(elist, eq + c, ecap, -1);
      if (flist && is_par) list_put(flist, fq, fcap, -1);
      continue;
    }
    const int d = key_depth(g, kk);
    if (!is_ref) {
      out[q] = is_par ? make_key(g, key_m(g, kk), d - 1) : kk;
      if (marks) marks[q] = is_par ? kMarkFused : 0u;
      if (flist && is_par) list_put(flist, fq, fcap, int32_t(q));
    } else {
      const uint64_t m = key_m(g, kk);
      for (int c = 0; c < nc; ++c) {
        out[q + c] = child_key(g, m, d, c);
        if (marks) marks[q + c] = kMarkExamine;
        if (elist) list_put(elist, eq + c, ecap, int32_t(q + c));
      }
    }
  }
  if (err) atomicOr(st.err, err);
}

// Radix directory of a sorted key array (see KeyDir): leaf i owns the
// buckets c with keys[i] <= c << shift < keys[i + 1].  A wave fills those of 64
// consecutive leaves (lane = leaf i with its key and the next leaf's; every
// lane calls): spans of up to 64 buckets each by its own lane, longer ones (very
// coarse leaves) by the whole wave in turn, four stores to a turn of its loop.
// Bound: the issue of those loops where a few waves hold the coarse leaves.  At
// 37 000 leaves 5.9 us (8.4 with one store to a turn), on trees of 1M points
// (0.6M leaves) 12 us (15).  One search per bucket instead, 64 to a wave, takes
// 5.7 and 12 us there but 6.8 against 3.6 on an ensemble of finer meshes.
__device__ inline void dir_fill(int64_t i, int64_t n, uint64_t key, uint64_t next, int shift, int64_t nb,
                                int32_t* __restrict__ d) {
  const int lane = threadIdx.x & 63;
  auto ceil_sh = [shift](uint64_t k) -> int64_t {
    const uint64_t mask = (uint64_t(1) << shift) - 1;
    return int64_t(k >> shift) + ((k & mask) ? 1 : 0);
  };
  int c0 = 0, c1 = 0;
  if (i < n) {
    const int64_t b = i + 1 < n ? ceil_sh(next) : nb + 1;
    c1 = int(b < nb + 1 ? b : nb + 1);
    const int64_t a = ceil_sh(key);
    c0 = int(a < c1 ? a : c1);
    if (i == 0)
      for (int c = 0; c < c0; ++c) d[c] = -1;
  }
  const bool big = c1 - c0 > 64;
  if (!big)
    for (int c = c0; c < c1; ++c) d[c] = int32_t(i);
  for (uint64_t bm = __ballot(big); bm; bm &= bm - 1) {
    const int l = __ffsll((unsigned long long)bm) - 1;
    const int a = __builtin_amdgcn_readlane(c0, l), b = __builtin_amdgcn_readlane(c1, l);
    const int32_t v = int32_t(i) - lane + l;
    int c = a + lane;
    for (; c - lane + 256 <= b; c += 256) {
      d[c] = v;
      d[c + 64] = v;
      d[c + 128] = v;
      d[c + 192] = v;
    }
    for (; c < b; c += 64) d[c] = v;
  }
}

__global__ __launch_bounds__(256) void k_build_dir(const uint64_t* __restrict__ keys, Count cn,
                                                   int shift, int64_t nb, int32_t* __restrict__ d,
                                                   const unsigned* conv, ScanClear clear) {
  scan_clear(clear, int64_t(blockIdx.x) * blockDim.x + threadIdx.x, int64_t(gridDim.x) * blockDim.x);
  if (conv && *conv) return;  // captured cycles: keys unchanged since the last build
  const int64_t n = cn.get();
  const int lane = threadIdx.x & 63;
  for (int64_t wb = int64_t(blockIdx.x) * blockDim.x + (threadIdx.x & ~63); wb < n;
       wb += int64_t(gridDim.x) * blockDim.x) {
    const int64_t i = wb + lane;
    dir_fill(i, n, i < n ? keys[i] : 0, i + 1 < n ? keys[i + 1] : 0, shift, nb, d);
  }
}

// Orders one wave's LDS writes before its later reads by other lanes.
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 2:1 balance after adaptation, fused parents.  A parent P (depth D) that
// replaced 2^dim balanced leaves can touch leaves of depth D+2 (never deeper,
// never coarser than D-1 -- the leaves it replaced were balanced).  Such a leaf
// sits in a depth-(D+1) octant touching P, and any such octant that is
// subdivided has a child touching P: one lane per (parent, depth-(D+1) cell of
// the shell around it) -- per the balance kind, cells across faces only, or
// also edges, or also corners -- looks whether its cell is subdivided, and marks
// P for splitting then.  Adapt lists the fused parents (any order, count
// ctr->nfused).  The check runs beside the marking in one launch: both wait for
// reads, and one after the other they took 8 to 10 us more of a captured cycle
// (333 -> 325 us at 37 000 leaves, 635 -> 622 for the mixed-degree ensemble).
constexpr int kShellW = 4;  // cells per axis around P: -1 .. 2 in units of a depth-(D+1) cell

// Search key of shell cell cidx around the fused parent; false for a cell the
// balance kind leaves out, outside a non-periodic domain, or of a parent too
// deep to touch a leaf two levels finer.
template <int DIM>
__device__ inline bool shell_probe(const KeyGeom& g, uint64_t key, int cidx, int limit, uint64_t* probe) {
  constexpr int W = kShellW;
  const int off[3] = {cidx % W - 1, (cidx / W) % W - 1, DIM == 3 ? cidx / (W * W) - 1 : 0};
  int outside = 0;
#pragma unroll
  for (int a = 0; a < DIM; ++a) outside += (off[a] < 0 || off[a] > 1) ? 1 : 0;
  const int d = key_depth(g, key);
  if (outside == 0 || outside > limit || d + 2 > g.dmax) return false;
  uint64_t m = key_morton(g, key);
  const int half = DIM * (g.dmax - d - 1);  // a cell is 2^(dmax - d - 1) wide
  bool ok = true;
#pragma unroll
  for (int a = 0; a < DIM; ++a)
    if (off[a] != 0) ok = ok && shift_morton(g, &m, a, off[a] > 0, half + (off[a] == 2 ? DIM : 0));
  *probe = point_key(g, m | (key_mesh_bits(g, key) >> g.mb));
  return ok;
}

// Thread tid of `threads` that share the listed parents' cells.
template <int DIM>
__device__ inline void fused_probe(const KeyGeom& g, const uint64_t* __restrict__ keys, int64_t n, const KeyDir& D,
                                   const int32_t* __restrict__ list, uint32_t* mark, DevCtr* ctr, int64_t tid,
                                   int64_t threads) {
  constexpr int NCELL = DIM == 3 ? kShellW * kShellW * kShellW : kShellW * kShellW;
  const int64_t work = int64_t(ctr->nfused) * NCELL;
  const int limit = g.balance == 0 ? 1 : (g.balance == 1 ? 2 : 3);
  for (int64_t t = tid; t < work; t += threads) {
    const int64_t i = list[t / NCELL];
    if (i < 0 || i >= n) continue;
    const uint64_t key = keys[i];
    uint64_t probe;
    if (!shell_probe<DIM>(g, key, int(t % NCELL), limit, &probe)) continue;
    const int64_t j = dir_last_le(keys, n, D, probe);
    if (j >= 0 && key_depth(g, keys[j]) >= key_depth(g, key) + 2) {
      const uint32_t was = atomicOr(&mark[i], 1u);
      if (!(was & 1u)) atomicAdd(&ctr->nmarked, 1ull);
    }
  }
}

// 2:1 balance, marking pass.  For a leaf L of depth D with parent P, the
// leaves that touch L and are two or more levels coarser are exactly the
// leaves strictly containing one of the 2^dim - 1 depth-(D-1) neighbours of P
// around the vertex L shares with P (the searching keys of Section 3.2),
// restricted to face / face+edge neighbours for the weaker balance kinds.
// Such a leaf gets bit 0 (split); L gets bit 1 (check again next pass).
// Only leaves with bit 2 (new or re-checked) are examined unless check_all.
//
// Not every searching key is searched:
//  - a neighbour of P with P's own parent is a sibling of P, so no leaf
//    strictly contains it;
//  - siblings of L that share the face (edge) of P ask for the same neighbour;
//    the first of them in Morton order asks for all (child index within the
//    key's axes).  Where that sibling is itself subdivided, its leaf at the
//    same corner asks for a smaller octant inside that neighbour, which the
//    same coarse leaf contains.
// That leaves 19 of 56 searches per family in 3D on average.  A wave lists its
// PER leaves' searches in LDS and takes them 64 at a time, so that lanes
// without one cost nothing: 64 leaves where every leaf is examined (about three
// rounds of searches), 16 of a list, which is short enough that one round each
// on more waves ends sooner.
// Bound: latency of the directory and key reads.  The passes of a tree built
// from 1M points (five, the first over every leaf) take 200 us (75 the first)
// against 552 with a lane per leaf and key, searched or not.  340 of them were
// left while every wave added its marks to the counter and every search marked
// for itself: atomics to one address queue up, so a workgroup adds once, runs of
// lanes that found the same leaf mark it once, and a leaf's violations are
// gathered in LDS.

// Bit sub set: the neighbour of the key's parent across the axes of `sub` is
// searched (see above); limit: the most axes (balance kind).
template <int DIM>
__device__ inline unsigned balance_searches(const KeyGeom& g, uint64_t key, int limit) {
  constexpr int NC = 1 << DIM;
  const int d = key_depth(g, key);
  if (d < 2) return 0;
  const uint64_t m = key_m(g, key);
  const unsigned c = child_index(g, m, d), cp = child_index(g, m, d - 1);
  const unsigned cross = ~(c ^ cp);  // axes on which P's neighbour leaves P's parent
  unsigned need = 0;
#pragma unroll
  for (unsigned sub = 1; sub < unsigned(NC); ++sub)
    if (__popc(sub) <= limit && (c & sub) == c && (sub & cross) != 0) need |= 1u << sub;
  return need;
}

// Search key of that neighbour; false outside a non-periodic domain.
template <int DIM>
__device__ inline bool balance_probe(const KeyGeom& g, uint64_t key, int sub, uint64_t* probe) {
  const int child = DIM * (g.dmax - key_depth(g, key)), parent = child + DIM;
  uint64_t m = key_morton(g, key);
  const unsigned c = unsigned(m >> child);  // low bits: the child index
  m = (m >> parent) << parent;              // the parent's anchor
  bool ok = true;
#pragma unroll
  for (int a = 0; a < DIM; ++a)
    if ((sub >> a) & 1) ok = ok && shift_morton(g, &m, a, (c >> a) & 1u, parent);
  *probe = point_key(g, m | (key_mesh_bits(g, key) >> g.mb));
  return ok;
}

template <int DIM, int PER, bool PROBE>
__global__ __launch_bounds__(kBlock) void k_balance_mark(KeyGeom g, const uint64_t* __restrict__ keys,
                                                         Count cn, KeyDir D, uint32_t* mark,
                                                         int check_all, DevCtr* ctr,
                                                         const unsigned* conv,
                                                         const int32_t* __restrict__ elist,
                                                         const int64_t* nexam, int64_t ecap,
                                                         const int32_t* __restrict__ flist, unsigned mblocks) {
  // waves stride over the leaves: every one (check_all), or the listed ones
  // (elist: *nexam entries, the leaves holding bit 2).  `conv` (captured
  // cycles): the fixpoint was already reached, nothing to examine.
  if (conv && *conv) return;
  // PROBE (the first pass after an adaptation): the workgroups from mblocks on
  // take the fused parents beside the marking
  if constexpr (PROBE)
    if (blockIdx.x >= mblocks) {
      fused_probe<DIM>(g, keys, cn.get(), D, flist, mark, ctr,
                       int64_t(blockIdx.x - mblocks) * kBlock + threadIdx.x, int64_t(gridDim.x - mblocks) * kBlock);
      return;
    }
  constexpr int NC = 1 << DIM, kWaves = kBlock / 64;
  __shared__ uint64_t s_key[kWaves][PER];
  __shared__ uint16_t s_task[kWaves][PER * (NC - 1)];
  __shared__ uint8_t s_viol[kWaves][PER];
  __shared__ unsigned long long s_fresh[kWaves];
  const int64_t n = cn.get();
  const int64_t items = elist ? min(*nexam, ecap) : n;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int limit = g.balance == 0 ? 1 : (g.balance == 1 ? 2 : 3);
  unsigned long long nfresh = 0;
  for (int64_t wb = (int64_t(blockIdx.x) * kWaves + wv) * PER; wb < items; wb += int64_t(mblocks) * kWaves * PER) {
    const int64_t it = lane < PER ? wb + lane : items;
    const int64_t i = it < items ? (elist ? int64_t(elist[it]) : it) : -1;
    unsigned need = 0;
    uint64_t key = 0;
    if (i >= 0 && i < n && (check_all || (mark[i] & 4u))) {
      key = keys[i];
      need = balance_searches<DIM>(g, key, limit);
    }
    if (lane < PER) {
      s_key[wv][lane] = key;
      s_viol[wv][lane] = 0;
    }
    // the wave's searches, listed by lane
    int at = __popc(need), total = at;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(total, o, 64);
      if (lane >= o) total += y;
    }
    at = total - at;
    total = __shfl(total, 63);
#pragma unroll
    for (unsigned sub = 1; sub < unsigned(NC); ++sub)
      if ((need >> sub) & 1u) s_task[wv][at++] = uint16_t(lane * NC + sub);
    wave_lds_fence();
    for (int t = lane; t < ((total + 63) & ~63); t += 64) {
      int32_t hit = -1;  // the leaf to split
      if (t < total) {
        const int w = s_task[wv][t];
        const int l = w / NC, sub = w % NC;
        const uint64_t k = s_key[wv][l];
        uint64_t probe;
        if (balance_probe<DIM>(g, k, sub, &probe)) {
          const int64_t j = dir_last_le(keys, n, D, probe);
          if (j >= 0 && key_depth(g, keys[j]) < key_depth(g, k) - 1) {
            hit = int32_t(j);
            s_viol[wv][l] = 1;
          }
        }
      }
      // runs of lanes that found the same leaf mark it once
      const int32_t before = __shfl_up(hit, 1, 64);
      bool fresh = hit >= 0 && (lane == 0 || before != hit);
      if (fresh) fresh = !(atomicOr(&mark[hit], 1u) & 1u);
      nfresh += __popcll(__ballot(fresh));
    }
    wave_lds_fence();  // the lists are read before the next leaves overwrite them
    if (lane < PER && s_viol[wv][lane]) atomicOr(&mark[i], 2u);
  }
  // one addition for the workgroup: thousands to one address queue up
  if (lane == 0) s_fresh[wv] = nfresh;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long all = 0;
    for (int w = 0; w < kWaves; ++w) all += s_fresh[w];
    if (all) atomicAdd(&ctr->nmarked, all);
  }
}

constexpr int kMarkList = 16;  // listed leaves a wave takes at a time

// A marking pass over every leaf (elist null) or the listed ones, and with flist
// the fused parents' check; `leaves` bounds their number.
void launch_balance_mark(const KeyGeom& g, const uint64_t* keys, Count cn, int64_t leaves, const KeyDir& D,
                         uint32_t* mark, DevCtr* ctr, const unsigned* conv, const int32_t* elist,
                         const int64_t* nexam, int64_t ecap, const int32_t* flist, hipStream_t s) {
  const int per = (elist ? kMarkList : 64) * (kBlock / 64);  // leaves a block takes at a time
  const int64_t full = ceil_div(leaves, per);
  const unsigned blocks = unsigned(elist ? std::min<int64_t>(full, kMarkGrid) : full);
  // the fused parents' number is on the device: up to a workgroup per 64 leaves
  const unsigned probes = elist && flist ? unsigned(std::max<int64_t>(1, std::min<int64_t>(1024, leaves / 64))) : 0;
#define LT_MARK(DIM, PER, PROBE, ALL)                                                                    \
  k_balance_mark<DIM, PER, PROBE><<<blocks + probes, kBlock, 0, s>>>(g, keys, cn, D, mark, ALL, ctr, conv, \
                                                                   elist, nexam, ecap, flist, blocks)
#define LT_MARK_DIM(DIM)                          \
  do {                                            \
    if (!elist) LT_MARK(DIM, 64, false, 1);       \
    else if (flist) LT_MARK(DIM, kMarkList, true, 0); \
    else LT_MARK(DIM, kMarkList, false, 0);       \
  } while (0)
  if (g.dim == 3)
    LT_MARK_DIM(3);
  else
    LT_MARK_DIM(2);
#undef LT_MARK_DIM
#undef LT_MARK
}

// Balance of a small tree in one workgroup: keys and marks in LDS, where
// neighbours are found by bisection, all passes in one launch.  Up to
// kSmallLeaves leaves (a wave holds kSmallRounds rounds of 64), the result
// included.  marks: adapt's, or null to examine every leaf.  Writes the error
// word, the number of balanced leaves to ctr->total, their keys if any leaf was
// split, and their directory.  Keys that do not fit `out` raise ERR_CAPACITY
// with their number, a tree that outgrows the workgroup with 0, and leave
// everything else as it was.
// Bound: one CU's issue rate and the latency of the LDS searches: 11 000 leaves
// of a 2D tree, six passes: 85 us (22 the first marking pass, about 6 us of
// counting, refinement and marking each later one); 800 leaves, three passes:
// 21 us.  The multi-workgroup passes take 15 to 20 us of kernels and 25 us of
// host readback each; with them a cycle of those trees took 328 and 254 us, with
// this 269 and 212.  The limit is the LDS (8 bytes a leaf and its mark).
constexpr int kSmallRounds = 14;
constexpr int kSmallLeaves = kScanBig * kSmallRounds;

template <int DIM>
__global__ __launch_bounds__(kScanBig) void k_balance_small(KeyGeom g, const uint64_t* in, int n,
                                                          const uint32_t* __restrict__ marks,
                                                          uint64_t* out, int64_t cap, int shift, int64_t nb,
                                                          int32_t* __restrict__ dir, DevCtr* ctr) {
  constexpr int NC = 1 << DIM, kWaves = kScanBig / 64, R = kSmallRounds;
  constexpr int NCELL = DIM == 3 ? kShellW * kShellW * kShellW : kShellW * kShellW;
  constexpr int kTasks = 64 + 64 * (NC - 1);  // a wave's pending searches
  __shared__ uint64_t K[kSmallLeaves];
  __shared__ uint32_t M[kSmallLeaves / 4];  // a byte per leaf, bits as the marks'
  __shared__ uint32_t s_task[kWaves][kTasks];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // rounds: as few as the leaves take, so that small trees use every wave
  int rounds = (n + kScanBig - 1) / kScanBig, first = wv * (64 * rounds) + lane;
  const int limit = g.balance == 0 ? 1 : (g.balance == 1 ? 2 : 3);
  uint8_t* Mb = reinterpret_cast<uint8_t*>(M);
  auto mark_bits = [&](int i, unsigned bits) { atomicOr(&M[i >> 2], bits << (8 * (i & 3))); };
  for (int r = 0; r < rounds; ++r) {
    const int i = first + 64 * r;
    if (i < n) K[i] = in[i];
    Mb[i] = i < n ? uint8_t(marks ? marks[i] : 4u) : 0;
  }
  __syncthreads();
  auto find = [&](uint64_t probe) {  // last key <= probe
    // four ways a step: three reads at once instead of two in a row
    int lo = 0;
    for (int step = 1 << ((31 - __clz(n)) & ~1); step > 0; step >>= 2) {
      const int t1 = lo + step, t2 = t1 + step, t3 = t2 + step;
      const uint64_t k1 = K[min(t1, n) - 1], k2 = K[min(t2, n) - 1], k3 = K[min(t3, n) - 1];
      lo += (t1 <= n && k1 <= probe) ? step : 0;
      lo += (t2 <= n && k2 <= probe) ? step : 0;
      lo += (t3 <= n && k3 <= probe) ? step : 0;
    }
    return lo - 1;
  };
  auto search = [&](uint32_t task) {
    const int i = int(task >> 3);
    const uint64_t k = K[i];
    uint64_t probe;
    if (!balance_probe<DIM>(g, k, int(task & 7u), &probe)) return;
    const int j = find(probe);
    if (j >= 0 && key_depth(g, K[j]) < key_depth(g, k) - 1) {
      mark_bits(j, 1u);
      mark_bits(i, 2u);
    }
  };
  bool grown = false, full = false;
  for (;;) {
    // marking: the waves take 64 leaves in turn (leaves to examine come in
    // runs), and their searches 64 at a time
    int pend = 0;
    for (int w = wv * 64; w < n; w += kScanBig) {
      const int i = w + lane;
      const unsigned m = i < n ? Mb[i] : 0;
      unsigned need = (m & 4u) ? balance_searches<DIM>(g, K[i], limit) : 0;
      if (__ballot(need != 0)) {
        int at = __popc(need), upto = at;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(upto, o, 64);
          if (lane >= o) upto += y;
        }
        at = pend + upto - at;
        pend += __shfl(upto, 63);
        for (; need; need &= need - 1) s_task[wv][at++] = uint32_t(i) << 3 | uint32_t(__ffs(need) - 1);
        wave_lds_fence();
        for (; pend >= 64; pend -= 64) search(s_task[wv][pend - 64 + lane]);
        wave_lds_fence();
      }
      // fused parents (first pass): NCELL lanes each, lane = shell cell
      for (uint64_t fm = __ballot(m & kMarkFused); fm;) {
        int f = -1;
#pragma unroll
        for (int q = 0; q < 64 / NCELL; ++q) {
          if (fm && lane / NCELL == q) f = i - lane + __ffsll((unsigned long long)fm) - 1;
          fm &= fm - 1;
        }
        uint64_t probe;
        if (f >= 0 && shell_probe<DIM>(g, K[f], lane % NCELL, limit, &probe)) {
          const int j = find(probe);
          if (j >= 0 && key_depth(g, K[j]) >= key_depth(g, K[f]) + 2) mark_bits(f, 1u);
        }
      }
    }
    if (lane < pend) search(s_task[wv][lane]);
    __syncthreads();
    // refinement, in place: every leaf to registers before any is written
    uint64_t key[R], one[R], ref[R], chk[R];
    int n_one = 0, n_ref = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      key[r] = ref[r] = one[r] = chk[r] = 0;
      if (r >= rounds) continue;
      const int i = first + 64 * r;
      const unsigned m = i < n ? Mb[i] : 0;
      key[r] = i < n ? K[i] : 0;
      ref[r] = __ballot(m & 1u);
      one[r] = __ballot(i < n && !(m & 1u));
      chk[r] = __ballot((m & 3u) == 2u);
      n_one += __popcll(one[r]);
      n_ref += __popcll(ref[r]);
    }
    WaveOut wo, wr;
    block_waves(n_ref * NC + n_one, n_ref, &wo, &wr);
    if (wr.all == 0) break;
    grown = true;
    if (wo.all > kSmallLeaves) {
      n = wo.all;
      full = true;
      break;
    }
    int o = wo.base;
    const uint64_t below = lanes_below();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r >= rounds) continue;
      const int q = o + __popcll(ref[r] & below) * NC + __popcll(one[r] & below);
      o += __popcll(ref[r]) * NC + __popcll(one[r]);
      if ((ref[r] >> lane) & 1) {
        const uint64_t m = key_m(g, key[r]);
        const int d = key_depth(g, key[r]);
        for (int c = 0; c < NC; ++c) {
          K[q + c] = child_key(g, m, d, c);
          Mb[q + c] = 4;
        }
      } else if ((one[r] >> lane) & 1) {
        K[q] = key[r];
        Mb[q] = (chk[r] >> lane) & 1 ? 4 : 0;
      }
    }
    n = wo.all;
    rounds = (n + kScanBig - 1) / kScanBig;
    first = wv * (64 * rounds) + lane;
    __syncthreads();
  }
  full = full || (grown && n > cap);
  if (threadIdx.x == 0) {
    ctr->err = full ? ERR_CAPACITY : 0;
    ctr->total = n <= kSmallLeaves ? n : 0;
  }
  if (full) return;
  for (int r = 0; r < rounds; ++r) {
    const int i = first + 64 * r;
    const uint64_t k = i < n ? K[i] : 0;
    if (grown && i < n) out[i] = k;
    dir_fill(i, n, k, i + 1 < n ? K[i + 1] : 0, shift, nb, dir);
  }
}

void launch_balance_small(const KeyGeom& g, const uint64_t* in, int n, const uint32_t* marks, uint64_t* out,
                          int64_t cap, int shift, int64_t nb, int32_t* dir, DevCtr* ctr, hipStream_t s) {
  if (g.dim == 3)
    k_balance_small<3><<<1, kScanBig, 0, s>>>(g, in, n, marks, out, cap, shift, nb, dir, ctr);
  else
    k_balance_small<2><<<1, kScanBig, 0, s>>>(g, in, n, marks, out, cap, shift, nb, dir, ctr);
}

// 2:1 balance, refinement pass: split bit-0 leaves one level, in order.  The
// new mark array holds bit 2 for leaves to examine next pass: the children of
// split leaves and the leaves that found a violation.
template <int R>
__global__ __launch_bounds__(kScanBig) void k_balance_refine(KeyGeom g, const uint64_t* __restrict__ in,
                                                           const uint32_t* __restrict__ mark,
                                                           uint64_t* __restrict__ out,
                                                           uint32_t* __restrict__ mark_out, int64_t cap,
                                                           ScanState st, DevCtr* cyc,
                                                           int32_t* __restrict__ elist, int64_t* nexam,
                                                           int64_t ecap) {
  constexpr int64_t kTile = int64_t(kScanBig) * R;
  if (cyc && (cyc->conv || cyc->nmarked == 0)) {
    // captured cycles at the fixpoint (no marks: noted for the passes after
    // this one) or past it: the pass is the identity, a plain copy
    if (blockIdx.x == 0 && threadIdx.x == 0) cyc->conv = 1;
    const int64_t n = st.items.get();
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int64_t i = int64_t(blockIdx.x) * kTile + int64_t(k) * kScanBig + threadIdx.x;
      if (i < n) {
        out[i] = in[i];
        mark_out[i] = 0u;
      }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) publish_total(st, n);
    return;
  }
  const int64_t tile = take_ticket(st);
  if (tile >= scan_tiles(st)) return;
  const int64_t n = st.items.get();
  const int lane = threadIdx.x & 63;
  const int64_t base = tile * kTile + int64_t(threadIdx.x >> 6) * (64 * R) + lane;
  const int nc = g.nchild();
  uint64_t key[R];  // read with the marks, ahead of the look-back
  uint64_t one[R], ref[R], chk[R];  // lanes kept, split, and kept but to be examined again
  int n_one = 0, n_ref = 0, n_chk = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t i = base + 64 * k;
    const uint32_t w = i < n ? mark[i] : 0u;
    key[k] = i < n ? in[i] : 0;
    ref[k] = __ballot(w & 1u);
    one[k] = __ballot(i < n && !(w & 1u));
    chk[k] = __ballot((w & 3u) == 2u);
    n_one += __popcll(one[k]);
    n_ref += __popcll(ref[k]);
    n_chk += __popcll(chk[k]);
  }
  // leaves the next pass examines (bit 2): the children of split leaves and
  // the leaves that found a violation, also put on the examine list
  WaveOut wr, we;
  block_waves(n_ref * nc + n_one, n_ref * nc + n_chk, &wr, &we);
  int64_t eo = block_append(we.all, nexam) + we.base;
  int64_t o = tile_prefix(st, tile, wr.all) + wr.base;
  const uint64_t below = lanes_below();
  unsigned err = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int rb = __popcll(ref[k] & below);
    const int64_t q = o + int64_t(rb) * nc + __popcll(one[k] & below);
    const int64_t eq = eo + int64_t(rb) * nc + __popcll(chk[k] & below);
    o += int64_t(__popcll(ref[k])) * nc + __popcll(one[k]);
    eo += int64_t(__popcll(ref[k])) * nc + __popcll(chk[k]);
    const bool is_ref = (ref[k] >> lane) & 1, is_chk = (chk[k] >> lane) & 1;
    if (!is_ref && !((one[k] >> lane) & 1)) continue;
    const int cnt = is_ref ? nc : 1;
    const uint64_t kk = key[k];
    if (q + cnt > cap) {
      err |= ERR_CAPACITY;
      for (int64_t t = q; t < cap && t < q + cnt; ++t) {  // valid keys below the capacity
        out[t] = kk;
        mark_out[t] = 0u;
      }
      for (int c = 0; c < (is_ref ? nc : (is_chk ? 1 : 0)); ++c) list_put(elist, eq + c, ecap, -1);
      continue;
    }
    if (is_ref) {
      const uint64_t m = key_m(g, kk);
      const int d = key_depth(g, kk);
      for (int c = 0; c < nc; ++c) {
        out[q + c] = child_key(g, m, d, c);
        mark_out[q + c] = 4u;
        list_put(elist, eq + c, ecap, int32_t(q + c));
      }
    } else {
      out[q] = kk;
      mark_out[q] = is_chk ? 4u : 0u;
      if (is_chk) list_put(elist, eq, ecap, int32_t(q));
    }
  }
  if (err) atomicOr(st.err, err);
}

// Launches over the look-back tiles of st (prepared with tile_of(count)).
void launch_adapt(const KeyGeom& g, const uint64_t* in, const int8_t* flags, uint64_t* out, int64_t cap,
                  const ScanState& st, uint32_t* marks, int32_t* elist, int64_t* nexam, int64_t ecap,
                  int32_t* flist, int64_t* nflist, int64_t fcap, hipStream_t s) {
  if (st.tile == kScanBig)
    k_adapt<1><<<grid_tiles(st), kScanBig, 0, s>>>(g, in, flags, out, cap, st, marks, elist, nexam, ecap,
                                                   flist, nflist, fcap);
  else
    k_adapt<kRounds><<<grid_tiles(st), kScanBig, 0, s>>>(g, in, flags, out, cap, st, marks, elist, nexam,
                                                         ecap, flist, nflist, fcap);
}

void launch_balance_refine(const KeyGeom& g, const uint64_t* in, const uint32_t* mark, uint64_t* out,
                           uint32_t* mark_out, int64_t cap, const ScanState& st, DevCtr* cyc,
                           int32_t* elist, int64_t* nexam, int64_t ecap, hipStream_t s) {
  if (st.tile == kScanBig)
    k_balance_refine<1><<<grid_tiles(st), kScanBig, 0, s>>>(g, in, mark, out, mark_out, cap, st, cyc, elist,
                                                            nexam, ecap);
  else
    k_balance_refine<kRounds><<<grid_tiles(st), kScanBig, 0, s>>>(g, in, mark, out, mark_out, cap, st, cyc,
                                                                  elist, nexam, ecap);
}

// Face connectivity (Section 3.3).  For face f = 2a + side the same-size box
// across the face is located by the leaf that holds its anchor: depth <= D
// means that leaf holds the whole box; deeper means the box is subdivided and
// e is the coarse side of a hanging face, whose 2^(dim-1) fine leaves are the
// box's children on the side facing e.
//
// Pass 1: one lane per (leaf, face), 2^DIM lanes per leaf (2D: 4, 3D: 8, two
// idle); nbr rows are written coalesced and each leaf's hanging faces become
// a bit mask.
template <int DIM>
__global__ __launch_bounds__(256) void k_connect_faces(KeyGeom g, const uint64_t* __restrict__ keys,
                                                       Count cn, KeyDir D, int32_t* __restrict__ nbr,
                                                       uint8_t* __restrict__ hmask, ScanClear clear) {
  // for the scan of the rows, which follows
  const int64_t gt = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  scan_clear(clear, gt, int64_t(gridDim.x) * blockDim.x);
  if (clear.ctr && gt == 0) clear.ctr->err = 0;
  constexpr int SL = 1 << DIM, NF = 2 * DIM;
  const int64_t n = cn.get();
  const int64_t lanes = n * SL;
  const int lane = threadIdx.x & 63;
  for (int64_t wb = int64_t(blockIdx.x) * blockDim.x + (threadIdx.x & ~63); wb < lanes;
       wb += int64_t(gridDim.x) * blockDim.x) {
    const int64_t tid = wb + lane;
    const int64_t e = tid / SL;
    const int f = int(tid % SL);
    bool hanging = false;
    if (e < n && f < NF) {
      const uint64_t key = keys[e];
      const int d = key_depth(g, key);
      uint64_t m = key_morton(g, key);
      int32_t v;
      if (!shift_morton(g, &m, f >> 1, f & 1, DIM * (g.dmax - d))) {
        v = -2;
      } else {
        const int64_t j = dir_last_le(keys, n, D, point_key(g, m | (key_mesh_bits(g, key) >> g.mb)));
        if (j < 0) {
          v = -2;  // unreachable for a complete tree (keys[0] has anchor 0)
        } else if (key_depth(g, keys[j]) <= d) {
          v = int32_t(j);
        } else {
          v = -1;
          hanging = true;
        }
      }
      nbr[e * NF + f] = v;
    }
    const uint64_t hb = __ballot(hanging);
    if (f == 0 && e < n) hmask[e] = uint8_t((hb >> lane) & ((1u << SL) - 1));
  }
}

// Pass 2: hanging-face rows in (leaf, face) order: count from the masks,
// decoupled look-back scan, then each row's leaf and face.
__global__ __launch_bounds__(kScanSmall) void k_connect_rows(const uint8_t* __restrict__ hmask, int dim,
                                                         int32_t* __restrict__ hang, int64_t cap_rows,
                                                         ScanState st) {
  const int64_t tile = take_ticket(st);
  if (tile >= scan_tiles(st)) return;
  const int64_t n = st.items.get();
  const int64_t base = tile * kTileMin + int64_t(threadIdx.x) * kItems;
  const int nf = 2 * dim;
  const int width = 2 + (1 << (dim - 1));
  uint64_t hm8 = 0;  // kItems masks, one byte each
  if (base + kItems <= n) {
    hm8 = *reinterpret_cast<const uint64_t*>(hmask + base);
  } else {
    for (int k = 0; k < kItems; ++k)
      if (base + k < n) hm8 |= uint64_t(hmask[base + k]) << (8 * k);
  }
  int64_t blk;
  const int64_t thr = block_exclusive<kScanSmall>(__popcll(hm8), &blk);
  int64_t o = tile_prefix(st, tile, blk) + thr;
  for (int k = 0; k < kItems && hm8; ++k) {
    const unsigned hm = unsigned(hm8 >> (8 * k)) & 0xffu;
    for (int f = 0; f < nf; ++f) {
      if (!((hm >> f) & 1u)) continue;
      if (o < cap_rows) {  // else the host grows the table and runs this pass again
        hang[o * width] = int32_t(base + k);
        hang[o * width + 1] = f;
      }
      o++;
    }
  }
}

// Pass 3: one lane per (row, slot): the fine leaf of the hanging face.  Slot
// bits are the tangential child bits in axis order, lower axis first; the
// fine leaves are the children of the same-size box on the side facing e.
__global__ __launch_bounds__(256) void k_connect_fine(KeyGeom g, const uint64_t* __restrict__ keys,
                                                      Count cn, KeyDir D, int32_t* __restrict__ hang,
                                                      const int64_t* total, int64_t cap_rows,
                                                      unsigned* err) {
  const int64_t n = cn.get();
  const int nh = 1 << (g.dim - 1);
  const int width = 2 + nh;
  const int64_t tid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t r = tid / nh;
  const int slot = int(tid % nh);
  const int64_t rows = *total < cap_rows ? *total : cap_rows;  // rows the table holds
  if (r >= rows) return;
  int32_t* row = hang + r * width;
  const int64_t e = row[0];
  const int f = row[1];
  if (e < 0 || e >= n || f < 0 || f >= 2 * g.dim) {
    atomicOr(err, ERR_UNBALANCED);
    row[2 + slot] = -1;
    return;
  }
  const uint64_t key = keys[e];
  const int d = key_depth(g, key);
  uint64_t m = key_morton(g, key);
  const int a = f >> 1, side = f & 1;
  shift_morton(g, &m, a, side, g.dim * (g.dmax - d));  // a hanging face has a neighbour
  int c = (1 - side) << a, j = 0;
  for (int t = 0; t < g.dim; ++t) {
    if (t == a) continue;
    c |= ((slot >> j) & 1) << t;
    ++j;
  }
  const uint64_t ck = child_key(g, m | (key_mesh_bits(g, key) >> g.mb), d, c);
  const int64_t idx = dir_last_le(keys, n, D, ck);
  if (idx < 0 || keys[idx] != ck) {
    atomicOr(err, ERR_UNBALANCED);
    row[2 + slot] = -1;
  } else {
    row[2 + slot] = int32_t(idx);
  }
}

// Old -> new mapping (Section 4.2): lower bound B of each new key in the old
// tree, then the case it falls in.  old(i) reads old key i.
template <class Old>
__device__ inline void map_case(KeyGeom g, const Old& old, int64_t n_old, uint64_t key, int64_t B,
                                int64_t j, int32_t* __restrict__ src, int8_t* __restrict__ kind,
                                unsigned* err) {
  const int d = key_depth(g, key);
  if (B < n_old && old(B) == key) {
    src[j] = int32_t(B);
    kind[j] = 0;
    return;
  }
  if (B > 0 && d > 0) {
    const uint64_t pk = old(B - 1);
    const uint64_t m = key_m(g, key);
    const uint64_t pm = key_m(g, pk);
    if (key_depth(g, pk) == d - 1 && (m & ~(span(g, d - 1) - 1)) == pm) {
      src[j] = int32_t(B - 1);
      kind[j] = int8_t(1 + child_index(g, m, d));
      return;
    }
  }
  const int nc = g.nchild();
  if (B + nc <= n_old && old(B) == key + 1 && d < g.dmax) {
    const uint64_t last = child_key(g, key_m(g, key), d, nc - 1);
    if (old(B + nc - 1) == last) {
      src[j] = int32_t(B);
      kind[j] = -1;
      return;
    }
  }
  // fits none of the three cases (the old tree was not balanced): report it;
  // the entry stays a valid index so that a captured transfer reads in bounds
  src[j] = 0;
  kind[j] = 0;
  atomicOr(err, ERR_MAP);
}

// First indices of keys[0, n) >= pa and >= pb, found by the whole wave
// together (every lane passes the same two probes): each half of the wave
// probes 32 evenly spaced keys of its remaining range per round and keeps the
// one gap its probe falls in -- one memory round trip per round for both
// searches (five at 1.6M keys) instead of one per halving.
__device__ inline void wave_lower_bound2(const uint64_t* __restrict__ keys, int64_t n, uint64_t pa,
                                         uint64_t pb, int64_t* ra, int64_t* rb) {
  const int lane = threadIdx.x & 63, half = lane >> 5, hl = lane & 31;
  const uint64_t probe = half ? pb : pa;
  int64_t lo = 0, hi = n;  // this half's bound lies in [lo, hi]
  for (;;) {
    const bool wide = hi - lo > 32;
    if (__ballot(wide) == 0) break;  // both halves narrow: the loop is left by the whole wave
    const int64_t step = wide ? (hi - lo + 31) / 32 : 1;
    const int64_t p = lo + int64_t(hl) * step;
    // the probes below the bound are a prefix of the half's lanes (the keys ascend)
    const uint64_t m = __ballot(p < hi && keys[p] < probe);
    const int c = __popc(unsigned(half ? (m >> 32) : m));
    if (wide) {
      if (c == 0) {
        hi = lo;
      } else {
        const int64_t nlo = lo + int64_t(c - 1) * step + 1;
        hi = std::min(hi, lo + int64_t(c) * step);
        lo = nlo;
      }
    }
  }
  const int64_t p = lo + hl;
  const uint64_t m = __ballot(p < hi && keys[p] < probe);
  const int64_t r = lo + __popc(unsigned(half ? (m >> 32) : m));
  *ra = __shfl(r, 0);
  *rb = __shfl(r, 32);
}

// A wave maps 64 consecutive new keys.  Their lower bounds lie between those
// of the wave's first and last key, found by one cooperative search; the
// old keys around that range (the case checks read B - 1 and B + 2^d - 1) go
// to the wave's LDS window in one coalesced load, and each lane bisects its
// own bound there.  A range wider than the window is bisected in memory.
constexpr int kMapWin = 640;
__global__ __launch_bounds__(kBlock) void k_map(KeyGeom g, const uint64_t* __restrict__ old_keys,
                                                Count cn_old, const uint64_t* __restrict__ keys,
                                                Count cn, int32_t* __restrict__ src,
                                                int8_t* __restrict__ kind, unsigned* err, DevCtr* cyc) {
  // captured cycles: marks left by the last marking pass mean that the fixed
  // balance passes did not reach the fixpoint; the transfer's lists count from 0
  if (cyc && blockIdx.x == 0 && threadIdx.x == 0) {
    if (cyc->nmarked != 0) atomicOr(err, ERR_BALANCE_PASSES);
    scan_clear(ScanClear{nullptr, 0, cyc, nullptr, nullptr, nullptr}, 0, 1);
  }
  __shared__ uint64_t win[kBlock / 64][kMapWin];
  const int64_t n_old = cn_old.get(), n = cn.get();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int nc = g.nchild();
  uint64_t* W = win[wv];
  for (int64_t wb = int64_t(blockIdx.x) * blockDim.x + (threadIdx.x & ~63); wb < n;
       wb += int64_t(gridDim.x) * blockDim.x) {
    const int64_t j = wb + lane;
    const bool live = j < n;
    const uint64_t key = keys[live ? j : n - 1];  // lanes past the end repeat the last key
    int64_t bf, bl;
    wave_lower_bound2(old_keys, n_old, __shfl(key, 0), __shfl(key, 63), &bf, &bl);
    const int64_t w0 = bf > 0 ? bf - 1 : 0;
    const int64_t w1 = std::min(bl + nc, n_old);
    if (w1 - w0 <= kMapWin) {
      for (int64_t q = w0 + lane; q < w1; q += 64) W[q - w0] = old_keys[q];
      wave_lds_fence();
      int64_t lo = bf, hi = bl;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (W[mid - w0] < key)
          lo = mid + 1;
        else
          hi = mid;
      }
      if (live) map_case(g, [&](int64_t i) { return W[i - w0]; }, n_old, key, lo, j, src, kind, err);
      wave_lds_fence();  // every lane done with the window before the next one overwrites it
    } else {
      int64_t lo = bf, hi = bl;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (old_keys[mid] < key)
          lo = mid + 1;
        else
          hi = mid;
      }
      if (live) map_case(g, [&](int64_t i) { return old_keys[i]; }, n_old, key, lo, j, src, kind, err);
    }
  }
}


// ------------------------------------------------------------------ host helpers
}  // namespace

void dir_params(const KeyGeom& g, int64_t n, int* shift, int64_t* nb) {
  int kb = g.mesh_shift;
  if (g.nmesh > 1) {
    int mbits = 0;
    while ((int64_t(1) << mbits) < g.nmesh) ++mbits;
    kb += mbits;
  }
  kb = std::min(kb, 64);
  int L = 0;
  while (L < 62 && (int64_t(1) << L) < n) ++L;
  L = std::max(10, std::min(24, L - 1));
  L = std::min(L, kb);
  *shift = kb - L;
  // The buckets end with the last mesh's key range (nmesh << mesh_shift),
  // not at the next power of two of the mesh count: otherwise the last leaf
  // would own every bucket of the empty mesh slots.
  const int ms = g.mesh_shift;
  const int64_t nm = std::max(1, g.nmesh);
  if (*shift <= ms)
    *nb = nm << (ms - *shift);
  else
    *nb = (nm + (int64_t(1) << (*shift - ms)) - 1) >> (*shift - ms);
}

// A scan over n_items whose words and counters an earlier kernel clears (clear).
lt_status plan_scan(const Alloc& A, uint64_t** status, int64_t* status_cap, DevCtr* ctr, int64_t n_items,
                    int64_t tile, ScanState* st, ScanClear* clear) {
  const int64_t ntiles = std::max<int64_t>(1, ceil_div(n_items, tile));
  LT_TRY(grow(A, status, status_cap, ntiles));
  *st = ScanState{*status, &ctr->ticket, &ctr->err, &ctr->total, Count{n_items, nullptr}, tile, nullptr, 0};
  *clear = ScanClear{*status, ntiles, ctr, nullptr, nullptr, nullptr};
  return LT_OK;
}

namespace {
lt_status prep_scan_on(const Alloc& A, uint64_t** status, int64_t* status_cap, DevCtr* ctr,
                       int64_t n_items, int64_t tile, hipStream_t stream, int flags, ScanState* st) {
  ScanClear c;
  LT_TRY(plan_scan(A, status, status_cap, ctr, n_items, tile, st, &c));
  k_clear_scan<<<unsigned(ceil_div(c.ntiles, 256)), 256, 0, stream>>>(c.status, c.ntiles, ctr, flags & 1,
                                                                     (flags >> 1) & 1);
  LT_HIP(hipGetLastError());
  return LT_OK;
}
}  // namespace

lt_status prep_scan(lt_tree t, int64_t n_items, int64_t tile, hipStream_t stream, int flags, ScanState* st) {
  return prep_scan_on(t->A, &t->status, &t->status_cap, t->dctr, n_items, tile, stream, flags, st);
}

lt_status prep_scan_conn(lt_tree t, int64_t n_items, hipStream_t stream, int flags, ScanState* st) {
  return prep_scan_on(t->A, &t->cstatus, &t->cstatus_cap, t->cctr, n_items, kTileMin, stream, flags,
                      st);
}

// Counters to pinned host memory: a kernel of one wave writes them and then the
// readback's number, which the host watches.  Everything before it on the stream
// has ended when it runs, as after a synchronization of the stream.  A copy
// command and that synchronization take about 10 us more of the host's time:
// cycles of 800 and 11 000 2D leaves, four readbacks each, take 169 us instead of
// 209 and 226 instead of 265.
constexpr int kCtrWords = int(sizeof(DevCtr) / 8);
static_assert(sizeof(DevCtr) % 8 == 0 && kCtrWords <= 32, "counters are published by 32 lanes");
static_assert(offsetof(HostCtr, r.seq) == kCtrWords * 8, "the number follows the counters");

__global__ void k_publish(DevCtr* ctr, uint64_t* host, const int64_t* more, int64_t* more_host, int words) {
  const int lane = threadIdx.x;
  const uint64_t seq = ctr->reads + 1;
  if (lane < kCtrWords)
    __hip_atomic_store(&host[lane], reinterpret_cast<const uint64_t*>(ctr)[lane], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  if (lane >= 32 && lane - 32 < words)
    __hip_atomic_store(&more_host[lane - 32], more[lane - 32], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();  // one wave: every lane's words before the number
  if (lane == 0) {
    ctr->reads = seq;
    __hip_atomic_store(&host[kCtrWords], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

lt_status publish(DevCtr* dev, HostCtr* host, hipStream_t stream, const int64_t* more, int64_t* more_host,
                  int words) {
  k_publish<<<1, 64, 0, stream>>>(dev, reinterpret_cast<uint64_t*>(host), more, more_host, words);
  LT_HIP(hipGetLastError());
  return LT_OK;
}

lt_status await_read(HostCtr* host, ReadTicket ticket, hipStream_t stream) {
  hipError_t e = hipSuccess;
  const ReadEnd end = read_await(&host->r, ticket, std::chrono::milliseconds(1), [&] {
    e = hipStreamSynchronize(stream);
    return e == hipSuccess;
  });
  if (end == ReadEnd::failed) return fail(LT_ERR_HIP, std::string("readback: ") + hipGetErrorString(e));
  if (end == ReadEnd::missing) return fail(LT_ERR_INTERNAL, "a readback did not arrive");
  return LT_OK;
}

lt_status read_back(DevCtr* dev, HostCtr* host, hipStream_t stream) {
  const ReadTicket ticket = read_expect(&host->r);
  LT_TRY(publish(dev, host, stream));
  return await_read(host, ticket, stream);
}

// Pinned memory of the trees' mirrors.  Allocating and freeing a block takes 20
// to 25 us each (with a device-wide wait for what is in flight), so up to
// kPinnedKept blocks of destroyed trees wait here for the next ones: a tree from
// 1M points, balanced and destroyed, takes 887 us instead of 993.
constexpr int kPinnedKept = 16;
struct PinnedPool {
  std::mutex mu;
  void* kept[kPinnedKept] = {};
  int n = 0;
};
// Nothing to construct or destroy at run time, so that it outlives every tree
// and no call on it can throw.
static_assert(std::is_trivially_destructible<PinnedPool>::value, "lives until the process ends");
static PinnedPool g_pinned;

hipError_t pinned_get(HostCtr** two) {
  void* q = nullptr;
  {
    std::lock_guard<std::mutex> l(g_pinned.mu);
    if (g_pinned.n > 0) q = g_pinned.kept[--g_pinned.n];
  }
  hipError_t e = hipSuccess;
  if (!q) e = hipHostMalloc(&q, 2 * sizeof(HostCtr), kPinnedFlags);
  if (e == hipSuccess) std::memset(q, 0, 2 * sizeof(HostCtr));
  *two = e == hipSuccess ? static_cast<HostCtr*>(q) : nullptr;
  return e;
}

// After the last work that may write it.
void pinned_put(HostCtr* two) {
  if (!two) return;
  {
    std::lock_guard<std::mutex> l(g_pinned.mu);
    if (g_pinned.n < kPinnedKept) {
      g_pinned.kept[g_pinned.n++] = two;
      return;
    }
  }
  (void)hipHostFree(two);
}

lt_status read_ctr(lt_tree t, hipStream_t stream) {
  return read_back(t->dctr, t->hctr, stream);
}

void launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t stream) {
  if (n > 0) k_fill_u32<<<unsigned(ceil_div(n, 256)), 256, 0, stream>>>(p, n, v);
}

lt_status clear_counters(DevCtr* ctr, hipStream_t stream) {
  k_clear_scan<<<1, 64, 0, stream>>>(nullptr, 0, ctr, 0, 0);
  LT_HIP(hipGetLastError());
  return LT_OK;
}

lt_status clear_err(lt_tree t, hipStream_t stream) {
  k_clear_scan<<<1, 64, 0, stream>>>(t->status, 0, t->dctr, 1, 0);
  LT_HIP(hipGetLastError());
  return LT_OK;
}

namespace {

lt_status check_geom(const lt_geom* g) {
  if (!g) return fail(LT_ERR_ARG, "geom is NULL");
  if (g->dim != 2 && g->dim != 3) return fail(LT_ERR_ARG, "dim must be 2 or 3");
  if (g->d_max < 1 || g->d_min < 0 || g->d_min > g->d_max)
    return fail(LT_ERR_DEPTH, "need 0 <= d_min <= d_max and d_max >= 1");
  int mb = 0;
  while ((g->d_max >> mb) != 0) ++mb;
  if (g->dim * g->d_max + mb > 64) return fail(LT_ERR_DEPTH, "dim*d_max + bitlength(d_max) > 64");
  if (g->dim == 3 && g->d_max > 21) return fail(LT_ERR_DEPTH, "3D d_max above 21");
  if (g->balance < 0 || g->balance > 2) return fail(LT_ERR_ARG, "balance must be 0, 1 or 2");
  return LT_OK;
}

lt_status new_tree(const lt_geom* geom, hipStream_t s, lt_tree* out) {
  LT_TRY(check_geom(geom));
  if (!out) return fail(LT_ERR_ARG, "out is NULL");
  lt_tree t = new lt_tree_s;
  int mb = 0;
  while ((geom->d_max >> mb) != 0) ++mb;
  t->g.dim = geom->dim;
  t->g.dmax = geom->d_max;
  t->g.dmin = geom->d_min;
  t->g.mb = mb;
  t->g.periodic = geom->periodic_mask & ((1u << geom->dim) - 1);
  t->g.balance = geom->balance;
  t->g.mesh_shift = mb + geom->dim * geom->d_max;
  t->g.nmesh = 1;
  t->g.lim = nullptr;
  t->A = registered_alloc();
  hipError_t e = hipGetDevice(&t->device);
  if (e == hipSuccess) e = dev_malloc(t->A, reinterpret_cast<void**>(&t->dctr), 2 * sizeof(DevCtr));
  if (e == hipSuccess) e = pinned_get(&t->hctr);
  if (e != hipSuccess) {
    lt_destroy(t);
    return fail(e == hipErrorOutOfMemory ? LT_ERR_OOM : LT_ERR_HIP,
                std::string("tree setup: ") + hipGetErrorString(e));
  }
  t->cctr = t->dctr + 1;
  t->hcctr = t->hctr + 1;
  const int words = int(2 * sizeof(DevCtr) / 4);
  k_fill_u32<<<1, unsigned(words), 0, s>>>(reinterpret_cast<uint32_t*>(t->dctr), words, 0u);
  e = hipGetLastError();
  if (e != hipSuccess) {
    lt_destroy(t);
    return fail(LT_ERR_HIP, std::string("tree setup: ") + hipGetErrorString(e));
  }
  *out = t;
  return LT_OK;
}

void invalidate(lt_tree t) {
  t->dir_valid = false;
  t->conn_valid = false;
  t->n_hang = -1;
  t->map_valid = false;
}

// Radix directory of the current keys (see KeyDir): about one bucket per
// two leaves (2^10 .. 2^24 buckets) over the range the keys can take.
lt_status ensure_dir(lt_tree t, hipStream_t s, KeyDir* D) {
  const int64_t n = t->n_cur;
  if (!t->dir_valid) {
    dir_params(t->g, n, &t->dir_shift, &t->dir_nb);
    LT_TRY(grow(t->A, &t->dir, &t->dir_cap, t->dir_nb + 1));
    if (n > 0) {
      k_build_dir<<<unsigned(ceil_div(n, 256)), 256, 0, s>>>(t->kbuf[t->cur], Count{n, nullptr},
                                                             t->dir_shift, t->dir_nb, t->dir, nullptr, ScanClear{});
      LT_HIP(hipGetLastError());
    }
    t->dir_valid = true;
  }
  D->d = t->dir;
  D->shift = t->dir_shift;
  D->nb = t->dir_nb;
  return LT_OK;
}

lt_status do_map(lt_tree t, hipStream_t stream) {
  if (!t->has_old) return fail(LT_ERR_STATE, "lt_map needs a prior lt_adapt");
  LT_TRY(grow(t->A, &t->map_src, &t->map_cap, t->n_cur));
  LT_TRY(grow(t->A, &t->map_kind, &t->kind_cap, t->n_cur));
  LT_TRY(clear_err(t, stream));
  if (t->n_cur > 0)
    k_map<<<unsigned(ceil_div(t->n_cur, kBlock)), kBlock, 0, stream>>>(
        t->g, t->kbuf[t->old], Count{t->n_old, nullptr}, t->kbuf[t->cur], Count{t->n_cur, nullptr},
        t->map_src, t->map_kind, &t->dctr->err, nullptr);
  LT_HIP(hipGetLastError());
  LT_TRY(read_ctr(t, stream));
  if (t->hctr->c.err & ERR_MAP)
    return fail(LT_ERR_UNBALANCED,
                "a new leaf is neither an old leaf, a child of one, nor a parent of 2^dim old leaves");
  if (t->hctr->c.err) return fail(LT_ERR_INTERNAL, "device check failed in lt_map");
  t->map_valid = true;
  return LT_OK;
}

// ---------------------------------------------------------- captured cycles
// Also folds connectivity's error word (its branch ran on a side stream)
// into the cycle's.
__global__ void k_copy_keys(const uint64_t* __restrict__ src, uint64_t* __restrict__ dst, Count cn,
                            unsigned* err, const unsigned* cerr) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const unsigned ce = *cerr;
  if (i == 0 && ce != 0) atomicOr(err, ce);
  if ((*err | ce) != 0) return;  // keep the pre-cycle keys for the host's recovery
  if (i < cn.get()) dst[i] = src[i];
}

}  // namespace

lt_status record_cycle(lt_tree_s* t, const CycleRec& r, hipStream_t s) {
  const KeyGeom& g = t->g;
  const int64_t C = r.cap;
  int64_t* S = r.dsz;
  uint64_t* K0 = t->kbuf[0];
  uint64_t* K[2] = {t->kbuf[1], t->kbuf[2]};
  const unsigned nb256 = unsigned(ceil_div(C, 256));
  // the search kernels stride over their work: a bounded grid, whatever the capacity
  constexpr int64_t kStrideGrid = 4096;
  const unsigned nlanes = unsigned(std::min<int64_t>(ceil_div(C * g.nchild(), 256), kStrideGrid));
  const unsigned nleaf = unsigned(std::min<int64_t>(ceil_div(C, 256), kStrideGrid));
  const unsigned* conv = &t->dctr->conv;
  unsigned* err = &t->dctr->err;
  int8_t* F = t->map_kind;  // the flags live in the kind array until the mapping overwrites it
  // flags (parameters from the device table, fetched from the host's)
  ScanState st;
  ScanClear sc;
  LT_TRY(plan_scan(t->A, &t->status, &t->status_cap, t->dctr, C, tile_of(C), &st, &sc));
  sc.cnt_dst = &S[1];  // leaves before the cycle
  sc.cnt_src = &S[0];
  const int fw = int(flag_args_size() * size_t(r.nmesh) / 4);
  k_cycle_start<<<unsigned(ceil_div(fw, 256)), 256, 0, s>>>(static_cast<const uint32_t*>(r.flag_host),
                                                          static_cast<uint32_t*>(t->flag_tab), fw, sc);
  LT_HIP(hipGetLastError());
  LT_TRY(launch_flag_table(g, r.tmpl, r.nmesh, t->flag_tab, K0, Count{C, &S[0]}, F, s));
  if (r.mlp)  // learned flags, the geometric ones as the fallback below conf_min
    LT_TRY(launch_mlp_flag(t, r.mlp, Count{C, &S[0]}, r.uo, r.ld, r.conf_min, F, nullptr, s));
  // adapt K0 -> K[0]
  st.items.p = &S[1];
  st.commit = &S[0];
  st.commit_cap = C;
  launch_adapt(g, K0, F, K[0], C, st, t->mbuf[0], t->elist, &t->dctr->nexam[0], t->elist_cap, t->fused,
               &t->dctr->nfused, t->fused_cap, s);
  LT_HIP(hipGetLastError());
  // balance: fixed passes, then a check
  // (the tree entering the cycle is balanced, so adapt's marks restrict the
  // first pass to new children and fused parents)
  const KeyDir D{t->dir, r.dir_shift, r.dir_nb};
  int ki = 0, mi = 0;
  for (int pass = 0; pass <= r.passes; ++pass) {
    // The directory build also clears for the pass's refinement and copies its
    // input count to S[3], where it reads it: the last tile commits the new count
    // to S[0] while workgroups of the capacity-sized grid may still be taking
    // tickets, and each must see the count the scan started from.
    LT_TRY(plan_scan(t->A, &t->status, &t->status_cap, t->dctr, C, tile_of(C), &st, &sc));
    sc.nexam = &t->dctr->nexam[1 - (pass & 1)];
    sc.cnt_dst = &S[3];
    sc.cnt_src = &S[0];
    k_build_dir<<<nleaf, 256, 0, s>>>(K[ki], Count{C, &S[0]}, r.dir_shift, r.dir_nb, t->dir, conv, sc);
    launch_balance_mark(g, K[ki], Count{C, &S[0]}, C, D, t->mbuf[mi], t->dctr, conv, t->elist,
                        &t->dctr->nexam[pass & 1], t->elist_cap, pass == 0 ? t->fused : nullptr, s);
    LT_HIP(hipGetLastError());
    if (pass == r.passes) break;
    st.items.p = &S[3];
    st.commit = &S[0];
    st.commit_cap = C;
    launch_balance_refine(g, K[ki], t->mbuf[mi], K[1 - ki], t->mbuf[1 - mi], C, st, t->dctr, t->elist, sc.nexam,
                          t->elist_cap, s);
    LT_HIP(hipGetLastError());
    ki = 1 - ki;
    mi = 1 - mi;
  }
  if (ki != 0) return fail(LT_ERR_ARG, "balance passes of a captured cycle must be even");
  // map
  k_map<<<nleaf, kBlock, 0, s>>>(g, K0, Count{C, &S[1]}, K[0], Count{C, &S[0]}, t->map_src,
                                  t->map_kind, err, t->dctr);
  LT_HIP(hipGetLastError());
  // connect on the side stream (the directory of K[0] was built by the check
  // pass); it reads the new keys only, and its scan words and counters are its
  // own, so it runs beside the transfer (forked after the mapping, which runs
  // alone: beside connectivity's searches it took three times as long)
  hipStream_t cs = r.side;
  LT_HIP(hipEventRecord(r.fork, s));
  LT_HIP(hipStreamWaitEvent(cs, r.fork, 0));
  ScanState cst;
  ScanClear cc;
  LT_TRY(plan_scan(t->A, &t->cstatus, &t->cstatus_cap, t->cctr, C, kTileMin, &cst, &cc));
  const unsigned cgrid = t->conn_grid > 0 ? std::min<unsigned>(nlanes, unsigned(t->conn_grid)) : nlanes;
  if (g.dim == 3)
    k_connect_faces<3><<<cgrid, 256, 0, cs>>>(g, K[0], Count{C, &S[0]}, D, t->nbr, t->hmask, cc);
  else
    k_connect_faces<2><<<cgrid, 256, 0, cs>>>(g, K[0], Count{C, &S[0]}, D, t->nbr, t->hmask, cc);
  cst.items.p = &S[0];
  cst.commit = &S[2];  // rows past the table's capacity raise ERR_CAPACITY
  cst.commit_cap = r.hang_rows;
  k_connect_rows<<<grid_tiles(cst), kScanSmall, 0, cs>>>(t->hmask, g.dim, t->hang, r.hang_rows, cst);
  const int nh = 1 << (g.dim - 1);
  k_connect_fine<<<unsigned(ceil_div(r.hang_rows * nh, 256)), 256, 0, cs>>>(
      g, K[0], Count{C, &S[0]}, D, t->hang, &t->cctr->total, r.hang_rows, &t->cctr->err);
  LT_HIP(hipGetLastError());
  LT_HIP(hipEventRecord(r.join, cs));
  // transfer
  if (r.precision == 1) {
    LT_TRY(launch_split_transfer(t, Count{C, &S[0]}, r.p, r.nvar, r.uo, r.ld, r.un, r.ld, s));
  } else if (r.p < 0) {  // per-mesh degrees
    LT_TRY(launch_transfer_mixed(t, K[0], Count{C, &S[0]}, r.nvar, r.uo, r.ld, r.un, r.ld, s));
  } else {
    LT_TRY(launch_transfer(t, Count{C, &S[0], t->n_cur}, r.p, r.ops, r.nvar, r.uo, r.ld, r.un, r.ld, s));
  }
  // the new keys become the next cycle's input, once connectivity is done
  LT_HIP(hipStreamWaitEvent(s, r.join, 0));
  k_copy_keys<<<nb256, 256, 0, s>>>(K[0], K0, Count{C, &S[0]}, err, &t->cctr->err);
  LT_HIP(hipGetLastError());
  return publish(t->dctr, t->hctr, s, S, r.hsz, 3);
}

namespace {

}  // namespace
// A new tree with no leaves yet (geometry checked, allocator and counters set
// up), for the translation units that build trees of their own.
lt_status create_tree(const lt_geom* geom, hipStream_t s, lt_tree* out) { return new_tree(geom, s, out); }

}  // namespace lt

using namespace lt;

// =================================================================== C ABI
extern "C" {

const char* lt_last_error(void) { return lt::g_err.c_str(); }

lt_status lt_set_allocator(void* (*alloc)(size_t bytes, void* stream, void* ctx),
                           void (*free_)(void* ptr, void* stream, void* ctx), void* ctx) {
  if ((alloc == nullptr) != (free_ == nullptr))
    return fail(LT_ERR_ARG, "alloc and free must both be set or both be NULL");
  Alloc A;
  A.alloc = alloc;
  A.free_ = free_;
  A.ctx = alloc ? ctx : nullptr;
  register_alloc(A);
  return LT_OK;
}

lt_status lt_build_uniform(const lt_geom* geom, int depth, void* stream, lt_tree* out) {
  lt_tree t = nullptr;
  LT_TRY(new_tree(geom, static_cast<hipStream_t>(stream), &t));
  if (depth < 0 || depth > geom->d_max) {
    lt_destroy(t);
    return fail(LT_ERR_DEPTH, "uniform depth outside [0, d_max]");
  }
  if (geom->dim * depth > 40) {
    lt_destroy(t);
    return fail(LT_ERR_ARG, "uniform tree too large");
  }
  const int64_t n = int64_t(1) << (geom->dim * depth);
  hipStream_t s = static_cast<hipStream_t>(stream);
  lt_status st = grow(t->A, &t->kbuf[t->cur], &t->kcap[t->cur], n);
  if (st != LT_OK) {
    lt_destroy(t);
    return st;
  }
  k_uniform<<<unsigned(ceil_div(n, kBlock)), kBlock, 0, s>>>(t->g, depth, n, t->kbuf[t->cur]);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    lt_destroy(t);
    return fail(LT_ERR_HIP, std::string("uniform build: ") + hipGetErrorString(e));
  }
  t->n_cur = n;
  t->balanced = true;  // uniform per mesh
  *out = t;
  return LT_OK;
}

lt_status lt_build(const lt_geom* geom, const uint64_t* keys, int64_t n, void* stream, lt_tree* out) {
  if (!keys || n < 1) return fail(LT_ERR_ARG, "keys must be a non-empty device array");
  lt_tree t = nullptr;
  LT_TRY(new_tree(geom, static_cast<hipStream_t>(stream), &t));
  hipStream_t s = static_cast<hipStream_t>(stream);
  lt_status st = grow(t->A, &t->kbuf[t->cur], &t->kcap[t->cur], n);
  if (st != LT_OK) {
    lt_destroy(t);
    return st;
  }
  hipError_t e = hipMemcpyAsync(t->kbuf[t->cur], keys, size_t(n) * 8, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess) {
    k_validate<<<unsigned(ceil_div(n, kBlock)), kBlock, 0, s>>>(t->g, t->kbuf[t->cur], n,
                                                                 &t->dctr->err);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&t->hctr->c, t->dctr, sizeof(DevCtr), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    lt_destroy(t);
    return fail(LT_ERR_HIP, std::string("build: ") + hipGetErrorString(e));
  }
  if (t->hctr->c.err) {
    lt_destroy(t);
    return fail(LT_ERR_INVALID_TREE, "keys are not the ascending IDs of a complete linear tree");
  }
  t->n_cur = n;
  *out = t;
  return LT_OK;
}

lt_status lt_build_batch(const lt_geom* geom, int nmesh, const int* d_min, const int* d_max,
                         const int* depth, void* stream, lt_tree* out) {
  if (!geom || !d_min || !d_max || !depth || !out || nmesh < 1)
    return fail(LT_ERR_ARG, "NULL argument or no mesh");
  lt_geom g0 = *geom;
  g0.d_min = 0;
  LT_TRY(check_geom(&g0));
  int mb = 0;
  while ((geom->d_max >> mb) != 0) ++mb;
  int mesh_bits = 0;
  while (((nmesh - 1) >> mesh_bits) != 0) ++mesh_bits;
  if (mb + geom->dim * geom->d_max + mesh_bits > 64)
    return fail(LT_ERR_DEPTH, "mesh index does not fit above the Morton bits");
  std::vector<int8_t> lim(2 * size_t(nmesh)), dep(nmesh);
  std::vector<int64_t> offs(size_t(nmesh) + 1, 0);
  for (int m = 0; m < nmesh; ++m) {
    if (d_min[m] < 0 || d_min[m] > d_max[m] || d_max[m] > geom->d_max || depth[m] < 0 ||
        depth[m] > geom->d_max)
      return fail(LT_ERR_DEPTH, "mesh " + std::to_string(m) + ": need 0 <= d_min <= d_max <= finest");
    if (geom->dim * depth[m] > 36) return fail(LT_ERR_ARG, "uniform mesh too large");
    lim[2 * m] = int8_t(d_min[m]);
    lim[2 * m + 1] = int8_t(d_max[m]);
    dep[m] = int8_t(depth[m]);
    offs[m + 1] = offs[m] + (int64_t(1) << (geom->dim * depth[m]));
  }
  const int64_t n = offs[nmesh];
  lt_tree t = nullptr;
  LT_TRY(new_tree(&g0, static_cast<hipStream_t>(stream), &t));
  hipStream_t s = static_cast<hipStream_t>(stream);
  int8_t* dep_dev = nullptr;
  lt_status st = grow(t->A, &t->kbuf[t->cur], &t->kcap[t->cur], n);
  hipError_t e = hipSuccess;
  if (st == LT_OK) {
    e = dev_malloc(t->A, reinterpret_cast<void**>(&t->lim), lim.size());
    if (e == hipSuccess)
      e = dev_malloc(t->A, reinterpret_cast<void**>(&t->mesh_offs), sizeof(int64_t) * (nmesh + 1));
    if (e == hipSuccess) e = dev_malloc(t->A, reinterpret_cast<void**>(&dep_dev), dep.size());
    if (e == hipSuccess) e = dev_malloc(t->A, &t->flag_tab, flag_args_size() * nmesh);
    if (e == hipSuccess)
      e = hipMemcpy(t->lim, lim.data(), lim.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(dep_dev, dep.data(), dep.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess)
      e = hipMemcpy(t->mesh_offs, offs.data(), sizeof(int64_t) * (nmesh + 1), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
      t->g.nmesh = nmesh;
      t->g.lim = t->lim;
      k_uniform_batch<<<unsigned(ceil_div(n, kBlock)), kBlock, 0, s>>>(t->g, t->mesh_offs, dep_dev,
                                                                        nmesh, n, t->kbuf[t->cur]);
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess)
      st = fail(e == hipErrorOutOfMemory ? LT_ERR_OOM : LT_ERR_HIP,
                std::string("batch build: ") + hipGetErrorString(e));
  }
  (void)dev_free(t->A, dep_dev);
  if (st != LT_OK) {
    lt_destroy(t);
    return st;
  }
  t->n_cur = n;
  t->balanced = true;  // uniform per mesh
  *out = t;
  return LT_OK;
}

lt_status lt_flag_batch(lt_tree t, const lt_flag_params* per_mesh, int nmesh, int8_t* flags,
                        void* stream) {
  if (!t || !per_mesh || !flags) return fail(LT_ERR_ARG, "NULL argument");
  if (nmesh != t->g.nmesh || !t->flag_tab)
    return fail(LT_ERR_ARG, "nmesh must equal the ensemble's mesh count");
  return launch_flag_batch(t->g, per_mesh, nmesh, t->flag_tab, t->kbuf[t->cur], t->n_cur, flags,
                           static_cast<hipStream_t>(stream));
}

lt_status lt_mesh_offsets(lt_tree t, int64_t* offsets, void* stream) {
  if (!t || !offsets) return fail(LT_ERR_ARG, "NULL argument");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nm = t->g.nmesh;
  if (!t->mesh_offs)
    if (dev_malloc(t->A, reinterpret_cast<void**>(&t->mesh_offs), sizeof(int64_t) * (nm + 1)) != hipSuccess)
      return fail(LT_ERR_OOM, "mesh offsets");
  k_mesh_offsets<<<unsigned(ceil_div(nm + 1, 64)), 64, 0, s>>>(t->g, t->kbuf[t->cur], t->n_cur, nm,
                                                                 t->mesh_offs);
  LT_HIP(hipGetLastError());
  LT_HIP(hipMemcpyAsync(offsets, t->mesh_offs, sizeof(int64_t) * (nm + 1), hipMemcpyDeviceToHost, s));
  LT_HIP(hipStreamSynchronize(s));
  return LT_OK;
}

lt_status lt_flag(lt_tree t, const lt_flag_params* fp, int8_t* flags, void* stream) {
  if (!t || !fp || !flags) return fail(LT_ERR_ARG, "NULL argument");
  if (t->g.nmesh > 1) return fail(LT_ERR_ARG, "an ensemble takes lt_flag_batch");
  return launch_flag(t->g, fp, t->kbuf[t->cur], t->n_cur, flags, static_cast<hipStream_t>(stream));
}

lt_status lt_adapt(lt_tree t, const int8_t* flags, void* stream) {
  if (!t || !flags) return fail(LT_ERR_ARG, "NULL argument");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t n = t->n_cur;
  // Output bound: every leaf refined.  The output goes to whichever of the
  // two free key buffers already holds the bound: the buffers rotate roles
  // from cycle to cycle, and growing a small one costs a device-wide free and
  // allocation.  The old snapshot is left alone until the call has succeeded.
  const int64_t need = n * t->g.nchild();
  int out = t->tmp, spare = t->aux;
  if (t->kcap[out] < need && t->kcap[spare] >= need) std::swap(out, spare);
  if (t->kcap[out] < need) {
    // growing: grow the other free buffer with it, so that from now on one of
    // the free buffers holds the bound and steady cycles allocate nothing
    LT_TRY(grow(t->A, &t->kbuf[out], &t->kcap[out], need));
    LT_TRY(grow(t->A, &t->kbuf[spare], &t->kcap[spare], need));
  }
  // From a balanced tree, adapt also writes the first balance pass's marks.
  const bool marks = t->balanced;
  int64_t cap = t->kcap[out];
  if (marks) {
    LT_TRY(grow(t->A, &t->mbuf[0], &t->mcap[0], need));
    LT_TRY(grow(t->A, &t->elist, &t->elist_cap, need));
    LT_TRY(grow(t->A, &t->fused, &t->fused_cap, need));
    cap = std::min(cap, std::min(t->mcap[0], std::min(t->elist_cap, t->fused_cap)));
  }
  ScanState st;
  LT_TRY(prep_scan(t, n, tile_of(n), s, 1 | 2, &st));
  launch_adapt(t->g, t->kbuf[t->cur], flags, t->kbuf[out], cap, st, marks ? t->mbuf[0] : nullptr,
               marks ? t->elist : nullptr, &t->dctr->nexam[0], t->elist_cap, marks ? t->fused : nullptr,
               &t->dctr->nfused, t->fused_cap, s);
  LT_HIP(hipGetLastError());
  LT_TRY(read_ctr(t, s));
  if (t->hctr->c.err & ERR_BAD_FLAG) return fail(LT_ERR_ARG, "flags must be -1, 0 or 1");
  if (t->hctr->c.err) return fail(LT_ERR_INTERNAL, "device check failed in lt_adapt");
  // old <- cur, cur <- the output, the other free buffer and the superseded
  // snapshot become the free ones
  const int prev_old = t->old;
  t->old = t->cur;
  t->cur = out;
  t->tmp = spare;
  t->aux = prev_old;
  t->n_old = n;
  t->n_cur = t->hctr->c.total;
  t->has_old = true;
  invalidate(t);
  t->balanced = false;
  t->adapt_marks = marks;
  return LT_OK;
}

}  // extern "C"

namespace {
// The balance fixpoint from the leaves in kbuf[t->cur].  Each refinement pass
// reads the current buffer and writes into one of the two free ones (tmp and
// aux in turn), then makes its output current; the buffer that held the
// leaves on entry is never written, so the caller can restore it.
lt_status balance_passes(lt_tree t, hipStream_t s) {
  // One host readback per pass (the number of leaves to split).  The refine
  // pass's own consistency checks land in the error word and are read with
  // the next pass's count.
  // The first pass examines every leaf, or -- right after adapt of a
  // balanced tree -- only the new children and the fused parents.
  int mi = 0;
  const bool restricted = t->adapt_marks && t->mcap[0] >= t->n_cur;
  t->adapt_marks = false;
  // A tree that fits one workgroup with room to grow: every pass in one launch
  // and one readback (another launch where the output buffer is too small).  One
  // that outgrows it goes through the passes below, which find everything as it
  // was.
  if (t->n_cur > 0 && t->n_cur <= kSmallLeaves - kScanBig) {
    const int out = t->cur == t->tmp ? t->aux : t->tmp;
    if (!t->dir_valid) {
      dir_params(t->g, t->n_cur, &t->dir_shift, &t->dir_nb);
      LT_TRY(grow(t->A, &t->dir, &t->dir_cap, t->dir_nb + 1));
    }
    t->dir_valid = false;
    for (;;) {
      launch_balance_small(t->g, t->kbuf[t->cur], int(t->n_cur), restricted ? t->mbuf[0] : nullptr, t->kbuf[out],
                           t->kcap[out], t->dir_shift, t->dir_nb, t->dir, t->dctr, s);
      LT_HIP(hipGetLastError());
      LT_TRY(read_ctr(t, s));
      if (!t->hctr->c.err || !t->hctr->c.total) break;
      LT_TRY(grow(t->A, &t->kbuf[out], &t->kcap[out], t->hctr->c.total));
    }
    if (!t->hctr->c.err) {
      if (t->hctr->c.total != t->n_cur) {
        t->cur = out;
        t->n_cur = t->hctr->c.total;
        invalidate(t);
      }
      t->dir_valid = true;
      return LT_OK;
    }
    LT_TRY(clear_err(t, s));
  }
  if (!restricted) {
    LT_TRY(grow(t->A, &t->mbuf[mi], &t->mcap[mi], t->n_cur));
    k_fill_u32<<<unsigned(ceil_div(t->n_cur, 256)), 256, 0, s>>>(t->mbuf[mi], t->n_cur, 0u);
    LT_HIP(hipGetLastError());
  }
  // Right after a successful adapt the error word, the mark count and the
  // fused-parent count are already zero (adapt's scan preparation cleared
  // them and adapt read the error word back), and the examine list must
  // survive: only other entries need the counters cleared.
  if (!restricted) LT_TRY(clear_err(t, s));
  const int max_pass = 4 * t->g.dmax + 16;
  int64_t expect_total = -1;
  for (int pass = 0;; ++pass) {
    if (pass > max_pass) return fail(LT_ERR_INTERNAL, "balance did not converge");
    KeyDir D;
    LT_TRY(ensure_dir(t, s, &D));
    if (t->n_cur > 0) {
      const bool all = pass == 0 && !restricted;
      const int32_t* el = all ? nullptr : t->elist;
      const Count cn{t->n_cur, nullptr};
      // adapt listed the fused parents (the list is sized for its output)
      const int32_t* fl = pass == 0 && restricted ? t->fused : nullptr;
      launch_balance_mark(t->g, t->kbuf[t->cur], cn, t->n_cur, D, t->mbuf[mi], t->dctr, nullptr, el,
                          &t->dctr->nexam[0], t->elist_cap, fl, s);
      LT_HIP(hipGetLastError());
    }
    LT_TRY(read_ctr(t, s));
    if (t->hctr->c.err) return fail(LT_ERR_INTERNAL, "device check failed in lt_balance");
    if (expect_total >= 0 && t->hctr->c.total != expect_total)
      return fail(LT_ERR_INTERNAL, "balance refinement size mismatch");
    const int64_t marked = int64_t(t->hctr->c.nmarked);
    if (marked == 0) break;
    const int64_t n_new = t->n_cur + marked * (t->g.nchild() - 1);
    const int out = t->cur == t->tmp ? t->aux : t->tmp;
    LT_TRY(grow(t->A, &t->kbuf[out], &t->kcap[out], n_new));
    LT_TRY(grow(t->A, &t->mbuf[1 - mi], &t->mcap[1 - mi], n_new));
    LT_TRY(grow(t->A, &t->elist, &t->elist_cap, n_new));
    ScanState st;
    // also zeroes the mark count and the examine list for the next pass
    LT_TRY(prep_scan(t, t->n_cur, tile_of(t->n_cur), s, 2, &st));
    const int64_t cap = std::min(std::min(t->kcap[out], t->mcap[1 - mi]), t->elist_cap);
    launch_balance_refine(t->g, t->kbuf[t->cur], t->mbuf[mi], t->kbuf[out], t->mbuf[1 - mi], cap, st,
                          nullptr, t->elist, &t->dctr->nexam[0], t->elist_cap, s);
    LT_HIP(hipGetLastError());
    expect_total = n_new;
    t->cur = out;
    t->n_cur = n_new;
    mi = 1 - mi;
    invalidate(t);
  }
  return LT_OK;
}
}  // namespace

extern "C" {

lt_status lt_balance(lt_tree t, void* stream) {
  if (!t) return fail(LT_ERR_ARG, "NULL tree");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int cur0 = t->cur;
  const int64_t n0 = t->n_cur;
  const bool conn0 = t->conn_valid, map0 = t->map_valid;
  const int64_t hang0 = t->n_hang;
  const lt_status st = balance_passes(t, s);
  if (st != LT_OK) {
    // strong guarantee: the leaves before the call are still in kbuf[cur0];
    // connectivity and mapping arrays were not touched by the passes
    t->cur = cur0;
    t->n_cur = n0;
    t->conn_valid = conn0;
    t->map_valid = map0;
    t->n_hang = hang0;
    t->dir_valid = false;     // the directory may describe intermediate leaves
    t->adapt_marks = false;   // the first pass's marks were consumed
    return st;
  }
  if (t->cur != cur0) {  // cur0 and the free buffer the passes did not end in are free
    if (t->cur == t->tmp)
      t->tmp = cur0;
    else
      t->aux = cur0;
  }
  t->balanced = true;
  return LT_OK;
}


lt_status lt_connect(lt_tree t, void* stream) {
  if (!t) return fail(LT_ERR_ARG, "NULL tree");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t n = t->n_cur;
  const int nf = 2 * t->g.dim;
  const int width = 2 + (1 << (t->g.dim - 1));
  LT_TRY(grow(t->A, &t->nbr, &t->nbr_cap, n * nf));
  LT_TRY(grow(t->A, &t->hmask, &t->hmask_cap, n + kItems));
  // initial table: one row per 16 leaves, as a captured cycle reserves (the
  // hanging faces sit on the refinement fronts: one per 90 leaves in the
  // 1.7M-leaf workload, more than one per 64 at 9M leaves)
  LT_TRY(grow(t->A, &t->hang, &t->hang_cap, std::max<int64_t>(1024, n / 16) * width));
  KeyDir D;
  LT_TRY(ensure_dir(t, s, &D));
  ScanState st;
  ScanClear clear;
  LT_TRY(plan_scan(t->A, &t->cstatus, &t->cstatus_cap, t->cctr, n, kTileMin, &st, &clear));
  if (n > 0) {
    const int64_t lanes = ceil_div(n * t->g.nchild(), 256);
    const unsigned blocks = unsigned(t->conn_grid > 0 ? std::min<int64_t>(lanes, t->conn_grid) : lanes);
    if (t->g.dim == 3)
      k_connect_faces<3><<<blocks, 256, 0, s>>>(t->g, t->kbuf[t->cur], Count{n, nullptr}, D, t->nbr,
                                                t->hmask, clear);
    else
      k_connect_faces<2><<<blocks, 256, 0, s>>>(t->g, t->kbuf[t->cur], Count{n, nullptr}, D, t->nbr,
                                                t->hmask, clear);
    LT_HIP(hipGetLastError());
  }
  const int nh = 1 << (t->g.dim - 1);
  int64_t rows = -1;
  for (int attempt = 0; attempt < 2 && rows < 0; ++attempt) {
    const int64_t cap_rows = t->hang_cap / width;
    if (attempt > 0 || n == 0) LT_TRY(prep_scan_conn(t, n, s, 1, &st));
    k_connect_rows<<<grid_tiles(st), kScanSmall, 0, s>>>(t->hmask, t->g.dim, t->hang, cap_rows, st);
    LT_HIP(hipGetLastError());
    // fine leaves of the rows the table holds (the row count stays on the device)
    k_connect_fine<<<unsigned(ceil_div(cap_rows * nh, 256)), 256, 0, s>>>(
        t->g, t->kbuf[t->cur], Count{n, nullptr}, D, t->hang, &t->cctr->total, cap_rows,
        &t->cctr->err);
    LT_HIP(hipGetLastError());
    LT_TRY(read_back(t->cctr, t->hcctr, s));
    if (t->hcctr->c.err & ERR_UNBALANCED)
      return fail(LT_ERR_UNBALANCED, "tree is not 2:1 balanced across a face");
    if (t->hcctr->c.err) return fail(LT_ERR_INTERNAL, "device check failed in lt_connect");
    if (t->hcctr->c.total <= cap_rows)
      rows = t->hcctr->c.total;
    else  // the hanging-face table overflowed: grow it (with room for the next
          // cycles: a regrowth frees memory, which waits for the whole device)
          // and emit the rows again
      LT_TRY(grow(t->A, &t->hang, &t->hang_cap, 2 * t->hcctr->c.total * width));
  }
  if (rows < 0) return fail(LT_ERR_INTERNAL, "hanging-face table overflowed twice");
  t->n_hang = rows;
  t->conn_valid = true;
  return LT_OK;
}

lt_status lt_set_connect_grid(lt_tree t, int blocks) {
  if (!t) return fail(LT_ERR_ARG, "NULL tree");
  if (blocks < 0) return fail(LT_ERR_ARG, "the connectivity grid cap must be >= 0");
  t->conn_grid = blocks;
  return LT_OK;
}

lt_status lt_map(lt_tree t, void* stream) {
  if (!t) return fail(LT_ERR_ARG, "NULL tree");
  return do_map(t, static_cast<hipStream_t>(stream));
}

lt_status lt_transfer(lt_tree t, int p, int nvar, const double* u_old, int64_t ld_old, double* u_new,
                      int64_t ld_new, int precision, void* stream) {
  if (!t || !u_old || !u_new) return fail(LT_ERR_ARG, "NULL argument");
  if (precision != 0 && precision != 1) return fail(LT_ERR_ARG, "precision must be 0 or 1");
  if (nvar < 1) return fail(LT_ERR_ARG, "nvar must be positive");
  if (p < 1 || p > (t->g.dim == 3 ? 3 : LT_MAX_DEGREE))
    return fail(LT_ERR_ARG, "unsupported polynomial degree for this dimension");
  if (!t->has_old) return fail(LT_ERR_STATE, "lt_transfer needs a prior lt_adapt");
  if (ld_old < t->n_old || ld_new < t->n_cur) return fail(LT_ERR_ARG, "leading dimension too small");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!t->map_valid) LT_TRY(lt_map(t, stream));
  if (precision == 1) return launch_split_transfer(t, p, nvar, u_old, ld_old, u_new, ld_new, s);
  LT_TRY(build_transfer_ops(t->A, p, &t->ops[p], s));
  return launch_transfer(t, p, t->ops[p], nvar, u_old, ld_old, u_new, ld_new, s);
}

lt_status lt_size(lt_tree t, int64_t* n_cur, int64_t* n_old, int64_t* n_hang) {
  if (!t) return fail(LT_ERR_ARG, "NULL tree");
  if (n_cur) *n_cur = t->n_cur;
  if (n_old) *n_old = t->has_old ? t->n_old : -1;
  if (n_hang) *n_hang = t->conn_valid ? t->n_hang : -1;
  return LT_OK;
}

static lt_status field_info(lt_tree t, lt_field what, const void** ptr, int64_t* count, size_t* elem) {
  const int nf = 2 * t->g.dim, width = 2 + (1 << (t->g.dim - 1));
  switch (what) {
    case LT_KEYS: *ptr = t->kbuf[t->cur]; *count = t->n_cur; *elem = 8; break;
    case LT_OLD_KEYS:
      *ptr = t->has_old ? t->kbuf[t->old] : nullptr; *count = t->has_old ? t->n_old : 0; *elem = 8; break;
    case LT_NBR:
      *ptr = t->conn_valid ? t->nbr : nullptr; *count = t->conn_valid ? t->n_cur * nf : 0; *elem = 4; break;
    case LT_HANG:
      *ptr = t->conn_valid ? t->hang : nullptr; *count = t->conn_valid ? t->n_hang * width : 0; *elem = 4; break;
    case LT_MAP_SRC:
      *ptr = t->map_valid ? t->map_src : nullptr; *count = t->map_valid ? t->n_cur : 0; *elem = 4; break;
    case LT_MAP_KIND:
      *ptr = t->map_valid ? t->map_kind : nullptr; *count = t->map_valid ? t->n_cur : 0; *elem = 1; break;
    default: return fail(LT_ERR_ARG, "unknown field");
  }
  return LT_OK;
}

lt_status lt_view(lt_tree t, lt_field what, const void** ptr, int64_t* count) {
  if (!t || !ptr || !count) return fail(LT_ERR_ARG, "NULL argument");
  size_t elem;
  return field_info(t, what, ptr, count, &elem);
}

lt_status lt_export(lt_tree t, lt_field what, void* dst, int64_t capacity, void* stream) {
  if (!t) return fail(LT_ERR_ARG, "NULL tree");
  const void* p;
  int64_t count;
  size_t elem;
  LT_TRY(field_info(t, what, &p, &count, &elem));
  if (!p && count > 0) return fail(LT_ERR_STATE, "field not computed");
  if (capacity < count) return fail(LT_ERR_ARG, "destination too small");
  if (count > 0 && !dst) return fail(LT_ERR_ARG, "NULL destination");
  if (count > 0)
    LT_HIP(hipMemcpyAsync(dst, p, size_t(count) * elem, hipMemcpyDeviceToDevice,
                          static_cast<hipStream_t>(stream)));
  return LT_OK;
}

void lt_destroy(lt_tree t) {
  if (!t) return;
  (void)hipDeviceSynchronize();
  const Alloc A = t->A;
  auto fr = [&](void* p) { (void)dev_free(A, p); };
  for (auto& b : t->kbuf) fr(b);
  for (auto& b : t->mbuf) fr(b);
  for (void* b : {(void*)t->nbr, (void*)t->hmask, (void*)t->fused, (void*)t->dir, (void*)t->hang,
                  (void*)t->map_src, (void*)t->map_kind, (void*)t->status, (void*)t->lim,
                  (void*)t->flag_tab, (void*)t->mesh_offs, (void*)t->dctr, (void*)t->cstatus,
                  (void*)t->elist, t->split_frags, (void*)t->split_vec,
                  (void*)t->split_R, (void*)t->split_F, (void*)t->copy_delta, (void*)t->grp_list})
    fr(b);
  for (auto& o : t->ops) fr(o);
  for (auto& o : t->fr_tab) fr(o);
  fr(t->mesh_np);
  fr(t->chunk_np);
  fr(t->fr_u1);
  fr(t->fr_hb);
  fr(t->fr_code);
  fr(t->fr_hm);
  pinned_put(t->hctr);
  if (t->xs) (void)hipStreamDestroy(t->xs);
  for (hipEvent_t e : t->xev)
    if (e) (void)hipEventDestroy(e);
  delete t;
}

}  // extern "C"
