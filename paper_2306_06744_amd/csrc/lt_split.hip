// lt_split.hip -- split-precision solution transfer on BF16 MFMA.
//
// The same operators as the FP64 transfer of Section 4.2 (interpolation of
// the parent polynomial on refinement, L2 projection on coarsening), applied
// as dense (p+1)^d x (p+1)^d products on the matrix cores:
//   * every operator entry and every FP64 solution value is split into three
//     BF16 terms, x ~ x0 + x1 + x2 (each the BF16 rounding of the remainder);
//   * the six products a0b0, a0b1, a1b0, a0b2, a1b1, a2b0 are accumulated in
//     FP32 by v_mfma_f32_16x16x32_bf16 (smallest first);
//   * the result is shifted per element so that its cell mean (the
//     Gauss-Legendre quadrature mean) equals the FP64 cell mean: for a refined
//     child the mean of the parent polynomial over the child, for a fused
//     parent the average of its children's means (the projection conserves
//     the integral).
// Supported: 64 points per element (3D p = 3, 2D p = 7).  Copies are copies.
// Work lists (first child of each refined family, each fused parent) are
// built on the device, so the call never synchronises.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "tree.hpp"

namespace lt {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kNP = 64;        // points per element
constexpr int kMT = kNP / 16;  // 16-row tiles of an operator
constexpr int kKS = kNP / 32;  // 32-deep K steps
constexpr int kTC = 16;        // columns (families / fused parents) per tile

__device__ inline void split3(double x, __bf16& b0, __bf16& b1, __bf16& b2) {
  b0 = __bf16(float(x));
  const double r1 = x - double(float(b0));
  b1 = __bf16(float(r1));
  const double r2 = r1 - double(float(b1));
  b2 = __bf16(float(r2));
}

// Dense operator entry: op 0 interpolation I_c, op 1 projection P_c, from the
// 1D factors (A_0, A_1, P_0, P_1 row-major n1 x n1) by tensor product.
__device__ inline double dense_entry(const double* ops1d, int n1, int dim, int op, int c, int row,
                                     int k) {
  double v = 1.0;
  for (int a = 0; a < dim; ++a) {
    const int b = (c >> a) & 1;
    const double* M = ops1d + (2 * op + b) * n1 * n1;
    v *= M[(row % n1) * n1 + (k % n1)];
    row /= n1;
    k /= n1;
  }
  return v;
}

// A-operand fragments for v_mfma_f32_16x16x32_bf16: lane l of tile (mt, ks)
// holds rows mt*16 + (l % 16), columns ks*32 + 8*(l / 16) + t, t = 0..7.
// Layout: frags[((((op*nc + c)*3 + s)*kMT + mt)*kKS + ks)*64 + lane].
__global__ void k_build_split(const double* __restrict__ ops1d, int n1, int dim, int nc,
                              bf16x8* __restrict__ frags) {
  const int total = 2 * nc * kMT * kKS * 64;
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= total) return;
  const int lane = id % 64, ks = (id / 64) % kKS, mt = (id / (64 * kKS)) % kMT;
  const int c = (id / (64 * kKS * kMT)) % nc, op = id / (64 * kKS * kMT * nc);
  bf16x8 f0, f1, f2;
  for (int t = 0; t < 8; ++t) {
    const int row = mt * 16 + (lane % 16), k = ks * 32 + 8 * (lane / 16) + t;
    __bf16 x0, x1, x2;
    split3(dense_entry(ops1d, n1, dim, op, c, row, k), x0, x1, x2);
    f0[t] = x0;
    f1[t] = x1;
    f2[t] = x2;
  }
  const int base = (op * nc + c) * 3;
  frags[(((base + 0) * kMT + mt) * kKS + ks) * 64 + lane] = f0;
  frags[(((base + 1) * kMT + mt) * kKS + ks) * 64 + lane] = f1;
  frags[(((base + 2) * kMT + mt) * kKS + ks) * 64 + lane] = f2;
}

// FP64 mean weights: Wn[i] = quadrature weight / element volume (sums to 1),
// and g_c[k] = sum_i Wn[i] I_c[i][k] (mean over child c of parent basis k).
__global__ void k_build_split_vec(const double* __restrict__ ops1d, int n1, int dim, int nc,
                                  double* __restrict__ vec) {
  const double* w = ops1d + 4 * n1 * n1;
  for (int i = threadIdx.x; i < kNP; i += blockDim.x) {
    double W = 1.0;
    int r = i;
    for (int a = 0; a < dim; ++a) {
      W *= 0.5 * w[r % n1];
      r /= n1;
    }
    vec[i] = W;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nc * kNP; q += blockDim.x) {
    const int c = q / kNP, k = q % kNP;
    double s = 0.0;
    for (int i = 0; i < kNP; ++i) s += vec[i] * dense_entry(ops1d, n1, dim, 0, c, i, k);
    vec[kNP + q] = s;
  }
}

// Work lists from the mapping: R = first child of each refined family (kind
// 1) whose nc children all lie among the leaves, F = each fused parent (kind
// -1).  (The refinement stores a family whole.  Only a captured cycle that
// outgrew its capacity holds a family cut off at the end; its result is
// discarded, but nothing may be stored past its leaves.)  Waves take rounds of 64 leaves and
// count by ballots; a workgroup appends its entries, in leaf order, by one
// atomic per list (the workgroups' order is arbitrary: every family and every
// parent is computed on its own).
__global__ __launch_bounds__(kBlock) void k_split_lists(const int8_t* __restrict__ kind, Count cn,
                                                        int nc, int32_t* __restrict__ R, int64_t* nR,
                                                        int32_t* __restrict__ F, int64_t* nF) {
  constexpr int kWaves = kBlock / 64;
  __shared__ int cr[kWaves], cf[kWaves];
  __shared__ int64_t at[2];
  const int64_t n = cn.get();
  if (int64_t(blockIdx.x) * kTileMin >= n) return;  // launches sized for a capacity
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = int64_t(blockIdx.x) * kTileMin + w * (64 * kItems) + lane;
  int kd[kItems];
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int64_t j = base + 64 * k;
    kd[k] = j < n ? int(kind[j]) : 0;
    if (kd[k] == 1 && j + nc > n) kd[k] = 0;
  }
  int r = 0, f = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    r += __popcll(__ballot(kd[k] == 1));
    f += __popcll(__ballot(kd[k] == -1));
  }
  if (lane == 0) {
    cr[w] = r;
    cf[w] = f;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int* c = threadIdx.x == 0 ? cr : cf;
    int all = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) all += c[i];
    unsigned long long* count = reinterpret_cast<unsigned long long*>(threadIdx.x == 0 ? nR : nF);
    at[threadIdx.x] = all ? int64_t(atomicAdd(count, (unsigned long long)all)) : 0;
  }
  __syncthreads();
  int64_t ro = at[0], fo = at[1];
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    ro += i < w ? cr[i] : 0;
    fo += i < w ? cf[i] : 0;
  }
  const uint64_t below = (uint64_t(1) << lane) - 1;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const uint64_t mr = __ballot(kd[k] == 1), mf = __ballot(kd[k] == -1);
    if (kd[k] == 1) R[ro + __popcll(mr & below)] = int32_t(base + 64 * k);
    if (kd[k] == -1) F[fo + __popcll(mf & below)] = int32_t(base + 64 * k);
    ro += __popcll(mr);
    fo += __popcll(mf);
  }
}

__device__ inline f32x4 mma6(const bf16x8& a0, const bf16x8& a1, const bf16x8& a2, const bf16x8& b0,
                             const bf16x8& b1, const bf16x8& b2, f32x4 acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2, b0, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b2, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b0, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b1, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b0, acc, 0, 0, 0);
  return acc;
}

// Refinement.  A persistent block of NC waves takes (tile of 16 refined
// families, variable) items; wave c computes child c of all 16, I_c staying in
// its registers over all of the block's items (24 KB a wave: read for each
// item, the operators were most of the bytes), the shared parent tile split
// once into LDS.  The D fragment of lane l holds rows 4*(l/16) + r of a 16-row
// tile, column l % 16.  The item list is read three items ahead, the sources
// two and the parents' values one, so that no load is waited for where it is
// issued.  Two barriers an item: the values' LDS is rewritten after the second
// barrier, when every wave has read it, and the outputs' after the next first
// one, when every wave has stored from it.  Bound where refined families lie
// alone between copies: their 64-byte row segments reach memory as partial
// lines (10 000 scattered families, 5 variables: 154 us alone, 87 with the same
// bytes stored densely).  One item per block and five barriers took 276 us
// beside the copy pass, this form 197.
template <int NC>
__global__ __launch_bounds__(64 * NC) void k_split_refine(
    const bf16x8* __restrict__ fragI, const double* __restrict__ vec, const int32_t* __restrict__ R,
    const int64_t* __restrict__ count, int nvar, const int32_t* __restrict__ src,
    const double* __restrict__ uo, int64_t ldo, double* __restrict__ un, int64_t ldn) {
  constexpr int kThreads = 64 * NC;
  constexpr int kVals = kNP * kTC / kThreads;  // parent values a thread splits
  __shared__ double Bd[kNP][kTC];
  __shared__ __attribute__((aligned(16))) __bf16 Bf[3][kKS][64][8];
  __shared__ double Out[kNP][kTC * NC];
  __shared__ int32_t s_j0[kTC];
  const int lane = threadIdx.x & 63, c = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int cc = threadIdx.x % kTC, k0 = threadIdx.x / kTC;  // this thread's column and first point
  const int64_t nR = *count;
  const uint32_t ntile = uint32_t((nR + kTC - 1) / kTC);
  const uint32_t items = ntile * uint32_t(nvar);
  if (blockIdx.x >= items) return;
  bf16x8 a[3][kMT][kKS];
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) a[s][mt][ks] = fragI[(((c * 3 + s) * kMT + mt) * kKS + ks) * 64 + lane];
  const double* Wn = vec;
  const double* g = vec + kNP + c * kNP;
  // items run variable by variable, so that a variable's rows stay near each
  // other; past the end the last item again (never used), and columns past the
  // last family repeat it (same values, same address), so that every lane
  // loads and stores
  const uint32_t G = gridDim.x;
  auto clamped = [&](uint32_t it) { return it < items ? it : items - 1; };
  auto var_of = [&](uint32_t it) { return int64_t(clamped(it) / ntile); };
  auto family = [&](uint32_t it) -> int32_t {  // first child of this thread's column
    const int64_t r = int64_t(clamped(it) % ntile) * kTC + cc;
    return R[r < nR ? r : nR - 1];
  };
  auto values = [&](uint32_t it, int32_t sp, double* x) {
    const double* U = uo + var_of(it) * kNP * ldo + sp;
#pragma unroll
    for (int h = 0; h < kVals; ++h) x[h] = U[int64_t(k0 + h * (kThreads / kTC)) * ldo];
  };
  uint32_t it = blockIdx.x;
  int32_t j_0 = family(it), j_1 = family(it + G), j_2 = family(it + 2 * G);
  int32_t p_1 = src[j_1];
  double x[kVals];
  values(it, src[j_0], x);
  for (; it < items; it += G) {
    // this item's values, split, and its columns' first children
#pragma unroll
    for (int h = 0; h < kVals; ++h) {
      const int k = k0 + h * (kThreads / kTC);
      Bd[k][cc] = x[h];
      __bf16 x0, x1, x2;
      split3(x[h], x0, x1, x2);
      const int ks = k >> 5, l = ((k & 31) >> 3) * 16 + cc, t = k & 7;
      Bf[0][ks][l][t] = x0;
      Bf[1][ks][l][t] = x1;
      Bf[2][ks][l][t] = x2;
    }
    if (threadIdx.x < kTC) s_j0[threadIdx.x] = j_0;
    // the next items' loads, in flight over this item's products
    values(it + G, p_1, x);
    const int32_t p_2 = src[j_2];
    const int32_t j_3 = family(it + 3 * G);
    __syncthreads();
    f32x4 acc[kMT];
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) {
      const bf16x8 b0 = *reinterpret_cast<const bf16x8*>(Bf[0][ks][lane]);
      const bf16x8 b1 = *reinterpret_cast<const bf16x8*>(Bf[1][ks][lane]);
      const bf16x8 b2 = *reinterpret_cast<const bf16x8*>(Bf[2][ks][lane]);
#pragma unroll
      for (int mt = 0; mt < kMT; ++mt)
        acc[mt] = mma6(a[0][mt][ks], a[1][mt][ks], a[2][mt][ks], b0, b1, b2, acc[mt]);
    }
    // cell-mean correction in FP64
    double ms = 0.0, mf = 0.0;
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) ms += Wn[mt * 16 + 4 * grp + r] * double(acc[mt][r]);
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) mf += g[16 * grp + kk] * Bd[16 * grp + kk][col];
    ms += __shfl_xor(ms, 16, 64);
    ms += __shfl_xor(ms, 32, 64);
    mf += __shfl_xor(mf, 16, 64);
    mf += __shfl_xor(mf, 32, 64);
    const double delta = mf - ms;
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) Out[mt * 16 + 4 * grp + r][col * NC + c] = double(acc[mt][r]) + delta;
    const int32_t jo = s_j0[(threadIdx.x % (kTC * NC)) / NC];  // read before the next item's are written
    __syncthreads();
    const int q = threadIdx.x % (kTC * NC), r0 = threadIdx.x / (kTC * NC);
    double* O = un + var_of(it) * kNP * ldn + jo + (q % NC);
    constexpr int kStep = kThreads / (kTC * NC);  // rows a block stores at once
#pragma unroll
    for (int i = 0; i < kNP / kStep; ++i) O[int64_t(r0 + i * kStep) * ldn] = Out[r0 + i * kStep][q];
    j_0 = j_1;
    j_1 = j_2;
    j_2 = j_3;
    p_1 = p_2;
  }
}

// Coarsening.  A persistent block of NC waves takes (tile of 16 fused parents,
// variable) items; wave c multiplies P_c by the values of child c (split in
// registers); the partial results are summed over the children through LDS.
// Lists, sources and values are read ahead as in the refinement.
template <int NC>
__global__ __launch_bounds__(64 * NC) void k_split_fuse(
    const bf16x8* __restrict__ fragP, const double* __restrict__ vec, const int32_t* __restrict__ F,
    const int64_t* __restrict__ count, int nvar, const int32_t* __restrict__ src,
    const double* __restrict__ uo, int64_t ldo, double* __restrict__ un, int64_t ldn) {
  constexpr int kThreads = 64 * NC;
  constexpr int kVals = kNP * kTC / kThreads;
  __shared__ float Part[NC][kNP][kTC];
  __shared__ double Mc[NC][kTC];
  __shared__ double Ms[NC][kTC];
  const int lane = threadIdx.x & 63, c = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int64_t nF = *count;
  const uint32_t ntile = uint32_t((nF + kTC - 1) / kTC);
  const uint32_t items = ntile * uint32_t(nvar);
  if (blockIdx.x >= items) return;
  bf16x8 a[3][kMT][kKS];
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) a[s][mt][ks] = fragP[(((c * 3 + s) * kMT + mt) * kKS + ks) * 64 + lane];
  const double* Wn = vec;
  const uint32_t G = gridDim.x;
  auto clamped = [&](uint32_t it) { return it < items ? it : items - 1; };
  auto var_of = [&](uint32_t it) { return int64_t(clamped(it) / ntile); };
  auto parent = [&](uint32_t it) -> int32_t {  // the lane's column; past the last parent that one again
    const int64_t r = int64_t(clamped(it) % ntile) * kTC + col;
    return F[r < nF ? r : nF - 1];
  };
  // rows 32*ks + 8*grp + t of child c
  auto values = [&](uint32_t it, int32_t sp, double* x) {
    const double* U = uo + (var_of(it) * kNP + 8 * grp) * ldo + sp + c;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
      for (int t = 0; t < 8; ++t) x[8 * ks + t] = U[int64_t(ks * 32 + t) * ldo];
  };
  uint32_t it = blockIdx.x;
  int32_t j_0 = parent(it), j_1 = parent(it + G), j_2 = parent(it + 2 * G);
  int32_t p_1 = src[j_1];
  double x[8 * kKS];
  values(it, src[j_0], x);
  for (; it < items; it += G) {
    double mpart = 0.0;
    f32x4 acc[kMT];
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) {
      bf16x8 b0, b1, b2;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const double xr = x[8 * ks + t];
        mpart += Wn[ks * 32 + 8 * grp + t] * xr;
        __bf16 x0, x1, x2;
        split3(xr, x0, x1, x2);
        b0[t] = x0;
        b1[t] = x1;
        b2[t] = x2;
      }
#pragma unroll
      for (int mt = 0; mt < kMT; ++mt)
        acc[mt] = mma6(a[0][mt][ks], a[1][mt][ks], a[2][mt][ks], b0, b1, b2, acc[mt]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the next items' loads, in flight over the sums below
    values(it + G, p_1, x);
    const int32_t p_2 = src[j_2];
    const int32_t j_3 = parent(it + 3 * G);
    mpart += __shfl_xor(mpart, 16, 64);
    mpart += __shfl_xor(mpart, 32, 64);
    if (grp == 0) Mc[c][col] = mpart;
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) Part[c][mt * 16 + 4 * grp + r][col] = acc[mt][r];
    __syncthreads();
    // sums over the children, one column and kVals rows a thread, and their
    // means: over the wave's rows, then over the waves
    const int cc = threadIdx.x % kTC;
    double sum[kVals], ms = 0.0;
#pragma unroll
    for (int h = 0; h < kVals; ++h) {
      const int row = threadIdx.x / kTC + h * (kThreads / kTC);
      sum[h] = 0.0;
#pragma unroll
      for (int ch = 0; ch < NC; ++ch) sum[h] += double(Part[ch][row][cc]);
      ms += Wn[row] * sum[h];
    }
    ms += __shfl_xor(ms, 16, 64);
    ms += __shfl_xor(ms, 32, 64);
    if (grp == 0) Ms[c][col] = ms;
    __syncthreads();
    double mf = 0.0, mt = 0.0;
#pragma unroll
    for (int ch = 0; ch < NC; ++ch) {
      mf += Mc[ch][cc];
      mt += Ms[ch][cc];
    }
    const double shift = mf / NC - mt;
    // this thread's column is its lane's: its parent is j_0
    double* O = un + var_of(it) * kNP * ldn + j_0;
#pragma unroll
    for (int h = 0; h < kVals; ++h)
      O[int64_t(threadIdx.x / kTC + h * (kThreads / kTC)) * ldn] = sum[h] + shift;
    __syncthreads();  // the sums' LDS is read before the next item writes it
    j_0 = j_1;
    j_1 = j_2;
    j_2 = j_3;
    p_1 = p_2;
  }
}

}  // namespace

lt_status prepare_split(lt_tree_s* t, int p, hipStream_t s) {
  const int dim = t->g.dim;
  if (!((dim == 3 && p == 3) || (dim == 2 && p == 7)))
    return fail(LT_ERR_ARG, "split precision needs 64 points per element (3D p=3 or 2D p=7)");
  const int nc = 1 << dim, n1 = p + 1;
  LT_TRY_STATUS(build_transfer_ops(t->A, p, &t->ops[p], s));
  if (!t->split_frags) {
    const size_t nfr = size_t(2) * nc * 3 * kMT * kKS * 64;
    void* q = nullptr;
    if (dev_malloc(t->A, &q, nfr * sizeof(bf16x8)) != hipSuccess) return fail(LT_ERR_OOM, "split operators");
    void* qv = nullptr;
    if (dev_malloc(t->A, &qv, sizeof(double) * (kNP + nc * kNP)) != hipSuccess) {
      (void)dev_free(t->A, q);
      return fail(LT_ERR_OOM, "split operators");
    }
    k_build_split<<<unsigned((nfr / 3 + 255) / 256), 256, 0, s>>>(t->ops[p], n1, dim, nc,
                                                                  static_cast<bf16x8*>(q));
    k_build_split_vec<<<1, 256, 0, s>>>(t->ops[p], n1, dim, nc, static_cast<double*>(qv));
    if (hipGetLastError() != hipSuccess) {
      (void)dev_free(t->A, q);
      (void)dev_free(t->A, qv);
      return fail(LT_ERR_HIP, "split operator build failed to launch");
    }
    t->split_frags = q;
    t->split_vec = static_cast<double*>(qv);
  }
  return LT_OK;
}

lt_status launch_split_transfer(lt_tree_s* t, int p, int nvar, const double* u_old, int64_t ld_old,
                                double* u_new, int64_t ld_new, hipStream_t s) {
  return launch_split_transfer(t, Count{t->n_cur, nullptr}, p, nvar, u_old, ld_old, u_new, ld_new, s);
}

lt_status launch_split_transfer(lt_tree_s* t, Count cn, int p, int nvar, const double* u_old,
                                int64_t ld_old, double* u_new, int64_t ld_new, hipStream_t s) {
  const int dim = t->g.dim;
  if (nvar < 1 || int64_t(nvar) * kNP > 65535) return fail(LT_ERR_ARG, "nvar * 64 must be in [1, 65535]");
  LT_TRY_STATUS(prepare_split(t, p, s));
  const int nc = 1 << dim;
  const int64_t n = cn.n;  // leaves, or the capacity of a launch whose count lives on the device
  if (n == 0) return LT_OK;
  LT_TRY_STATUS(grow(t->A, &t->split_R, &t->split_R_cap, n));
  LT_TRY_STATUS(grow(t->A, &t->split_F, &t->split_F_cap, n));
  const bf16x8* fr = static_cast<const bf16x8*>(t->split_frags);
  const bf16x8* fI = fr;
  const bf16x8* fP = fr + size_t(nc) * 3 * kMT * kKS * 64;
  // The copy pass writes only copies and the refinement and fusion passes
  // only refined and fused elements: the latter run on the tree's second
  // stream beside the copy pass, forked before it is enqueued and joined back;
  // the work lists before the fork or after it (lists_first).
  hipStream_t side = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  LT_TRY_STATUS(transfer_side(t, &side, &fork, &join));
  int64_t *nR = &t->dctr->total, *nF = &t->dctr->nfgroups;
  auto lists = [&](hipStream_t q) -> lt_status {
    if (!cn.p) LT_TRY_STATUS(clear_counters(t->dctr, q));  // a captured cycle's mapping cleared them
    k_split_lists<<<unsigned((n + kTileMin - 1) / kTileMin), kBlock, 0, q>>>(t->map_kind, cn, nc, t->split_R,
                                                                           nR, t->split_F, nF);
    return LT_OK;
  };
  if (lists_first(n)) LT_TRY_STATUS(lists(s));
  hipError_t ef = hipEventRecord(fork, s);
  if (ef != hipSuccess) return fail(LT_ERR_HIP, std::string("split transfer fork: ") + hipGetErrorString(ef));
  lt_status r = launch_copy(t, cn, int64_t(nvar) * kNP, u_old, ld_old, u_new, ld_new, s);
  ef = hipStreamWaitEvent(side, fork, 0);
  if (r == LT_OK && ef == hipSuccess && !lists_first(n)) r = lists(side);
  if (r == LT_OK && ef == hipSuccess) {
    const int64_t max_ref = ((n / nc + kTC - 1) / kTC + 1) * nvar;
    const int64_t max_fuse = ((n + kTC - 1) / kTC + 1) * nvar;
    // persistent: one workgroup of 8 waves per compute unit (the operator
    // takes 96 registers a wave), or two of 4
    const int64_t slots = nc == 8 ? 256 : 512;
    const unsigned gr = unsigned(std::min(max_ref, slots)), gf = unsigned(std::min(max_fuse, slots));
    // a short copy pass ends before the refinement: the fusion follows it
    hipStream_t fs = lists_first(n) ? s : side;
    if (nc == 8) {
      k_split_refine<8><<<gr, 512, 0, side>>>(fI, t->split_vec, t->split_R, nR, nvar, t->map_src, u_old,
                                              ld_old, u_new, ld_new);
      k_split_fuse<8><<<gf, 512, 0, fs>>>(fP, t->split_vec, t->split_F, nF, nvar, t->map_src, u_old,
                                            ld_old, u_new, ld_new);
    } else {
      k_split_refine<4><<<gr, 256, 0, side>>>(fI, t->split_vec, t->split_R, nR, nvar, t->map_src, u_old,
                                              ld_old, u_new, ld_new);
      k_split_fuse<4><<<gf, 256, 0, fs>>>(fP, t->split_vec, t->split_F, nF, nvar, t->map_src, u_old,
                                            ld_old, u_new, ld_new);
    }
  }
  // the join on every path that forked, so that a capture in progress stays whole
  const hipError_t ej = hipEventRecord(join, side);
  const hipError_t ew = ej == hipSuccess ? hipStreamWaitEvent(s, join, 0) : ej;
  if (r != LT_OK) return r;
  if (ef != hipSuccess) return fail(LT_ERR_HIP, std::string("split transfer fork: ") + hipGetErrorString(ef));
  if (ew != hipSuccess) return fail(LT_ERR_HIP, std::string("split transfer join: ") + hipGetErrorString(ew));
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(LT_ERR_HIP, std::string("split transfer launch: ") + hipGetErrorString(e));
  return LT_OK;
}

}  // namespace lt
