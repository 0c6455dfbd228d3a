// Whole-matrix RMSE over the loaded ratings (Algorithm 1's termination
// test): sqrt((1/nnz) sum (x - u_i.v_j)^2), dot products in fp32, squares
// summed in fp64.  Reads the wave-major records.  With the row-block's U
// rows in LDS (k_rmse_lds) a workgroup covers one row-block; otherwise
// (k_rmse_partial) a workgroup covers one row-block and a group of
// column-blocks, its wave w every fourth of them from w.  A group of lanes
// shares one rating and loads 16-byte slices of u_i and v_j.  Per-wave sums
// are combined in a fixed order by a second kernel, so the result does not
// depend on scheduling.
#include <algorithm>
#include <type_traits>

#include "bgmf_internal.h"

namespace bgmfk {
namespace {

// Column-blocks per workgroup of k_rmse_partial.  Workgroups are numbered
// group-major (all row-blocks of column-blocks 0..63, then 64..127, ...), so
// the workgroups resident at one time read the V rows of about 64
// column-blocks, which stay in the caches, instead of all of V.
constexpr int kRmseColGroup = 64;

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// Lanes per rating: from k = 32 up, each lane holds four float4 slices of
// u_i and of v_j (KP/16 lanes per rating), which keeps the cross-lane levels
// and the per-rating index work per wave step low; at k = 16 four lanes
// hold one slice each.  Twice or half as many lanes are slower (100M ratings,
// k = 64: 1.58 and 1.56 ms against 1.34).
template <int KP>
constexpr int rmse_lanes() { return KP >= 32 ? KP / 16 : KP / 4; }
// Wave steps whose loads are in flight together, without U in LDS.  From
// KP = 64 up a second step costs waves per SIMD (about 100 registers a lane
// instead of 60: four or five waves instead of eight), and the launch decides:
// one of at most few_waves waits for its loads and takes two steps, a larger
// one gains more from the waves.  In-core pass of 10M ratings, one step
// against two: k = 64, p = 64 (256 waves) 1.34 and 0.92 ms, p = 400 (11,200)
// 282 and 266 us, p = 512 (16,384) 342 and 322 (other shapes 415 and 454,
// 501 and 521), p = 640 (25,600) 322 and 376; k = 128, p = 64 2.52 and 1.80
// ms, p = 512 712 and 574 us, p = 768 (36,864) 733 and 689, p = 1024 (65,536)
// 728 and 891.
template <int KP>
constexpr int64_t few_waves() { return KP == 64 ? 16384 : 40960; }
template <int KP>
constexpr int rmse_unroll(bool few) { return KP >= 64 ? (few ? 2 : 1) : KP >= 32 ? 2 : 8; }
// With U in LDS one workgroup of 16 waves fills a CU, which leaves a lane 128
// registers.  A width that fills its lanes takes three steps (two and one:
// 1.30, 1.34, 1.31 ms at 100M ratings, k = 64).  A masked width, whose
// slices have offsets of their own, spills with three; one step is fastest
// (three, two, one: k = 48 294, 266, 250 us; k = 80 536, 486, 462; k = 144
// 1042, 943, 880, each 20M ratings).  At k = 16 two of one slice (eight,
// four, two, one: 58, 57, 54, 72 us at 10M ratings).
template <int KP, bool FULL>
constexpr int rmse_unroll_lds() { return KP < 32 ? 2 : FULL ? 3 : 1; }

// Ratings of a block are counted in 32 bits without a sign: there are fewer
// than 2^31, and a position at most kAhead past the last one (the loops' step
// and the records fetched ahead) does not wrap.
constexpr uint32_t kAhead = 4096;
static_assert(0x7FFFFFFFu + kAhead > 0x7FFFFFFFu, "positions past the end compare as such");

// Factor rows are addressed in bytes: a 64-bit base plus row * rowbytes is
// one multiply-add.
__device__ __forceinline__ const char *row_ptr(const float *base, uint32_t row, uint32_t rowbytes) {
  return reinterpret_cast<const char *>(base) + (uint64_t)row * rowbytes;
}

// The lane's share of the dot product of u_i and v_j: its float4 slices
// q = gl, gl + L, ... of both rows.  FULL: k = KP.  Otherwise a slice past k
// reads slice 0 (so no load needs a branch) and counts as zero.
template <int KP, bool FULL>
struct Dot {
  static constexpr int L = rmse_lanes<KP>();  // lanes per rating
  static constexpr int QL = KP / 4 / L;       // slices per lane
  uint32_t off[FULL ? 1 : QL];                // byte offset of each slice in a row
  bool in[FULL ? 1 : QL];
  __device__ __forceinline__ Dot(int gl, int32_t k) {
    if constexpr (FULL) {
      off[0] = (uint32_t)gl * 16u;
    } else {
#pragma unroll
      for (int i = 0; i < QL; ++i) {
        in[i] = 4 * (gl + i * L) < k;
        off[i] = in[i] ? (uint32_t)(gl + i * L) * 16u : 0u;
      }
    }
  }
  __device__ __forceinline__ uint32_t at(int i) const {
    if constexpr (FULL) return off[0] + (uint32_t)(i * L) * 16u;
    else return off[i];
  }
  __device__ __forceinline__ void load(float4 (&x)[QL], const char *row) const {
#pragma unroll
    for (int i = 0; i < QL; ++i) x[i] = *reinterpret_cast<const float4 *>(row + at(i));
  }
  // x - u.v, in every lane of the rating's group
  __device__ __forceinline__ float error(float x, const float4 (&a)[QL], const float4 (&c)[QL]) const {
    float part = 0.0f;
#pragma unroll
    for (int i = 0; i < QL; ++i) {
      float t = part;
      t = fmaf(a[i].x, c[i].x, t);
      t = fmaf(a[i].y, c[i].y, t);
      t = fmaf(a[i].z, c[i].z, t);
      t = fmaf(a[i].w, c[i].w, t);
      if constexpr (FULL) part = t;
      else part = in[i] ? t : part;
    }
    part += dpp_mov<0xB1>(part);
    if constexpr (L > 2) part += dpp_mov<0x4E>(part);
    if constexpr (L > 4) part += dpp_mov<0x141>(part);
    if constexpr (L > 8) part += dpp_mov<0x140>(part);
    return x - part;
  }
};

// Every lane of a group adds the group's squares, so the wave's total is L
// times the sum (an exact scaling).
template <int L>
__device__ __forceinline__ double wave_sum(double acc) {
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  return acc * (1.0 / L);
}

// Keeps a wave step's loads ahead of the arithmetic that follows.  Left to
// itself the compiler sinks them to their uses, to save registers, and a wave
// then waits for one or two rows at a time.
__device__ __forceinline__ void loads_issued() { __builtin_amdgcn_sched_barrier(0); }

// KP: k rounded up to a power of two.  FEW: at most few_waves waves
// (only from KP = 64 up).
//
// The loads are fenced except in the widest kernels of a large launch, whose
// other waves fill the gaps (k = 128, p = 2048: 2.15 ms without, 2.22 with).
// Without the fence: 10M ratings, k = 16, p = 32 1.30 against 0.63 ms, p =
// 256 217 against 161 us; k = 32, p = 64 945 against 562 us; k = 48, p = 512
// 446 against 397.
template <int KP, bool FULL, bool FEW>
__global__ void __launch_bounds__(256)
k_rmse_partial(const uint2 *__restrict__ rec, const int64_t *__restrict__ wblock_ptr,
               const float *__restrict__ U, const float *__restrict__ V, Grid G, int32_t k,
               double *__restrict__ partials) {
  using Dt = Dot<KP, FULL>;
  constexpr int L = Dt::L, QL = Dt::QL;
  constexpr int RPS = 64 / L;             // ratings per wave step
  constexpr int UNR = rmse_unroll<KP>(FEW);  // wave steps whose loads are in flight together
  constexpr bool kFence = KP <= 64 || FEW;
  const int32_t p = G.p;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane / L;
  const Dt dot(lane % L, k);
  const uint32_t rowbytes = (uint32_t)k * 4u;
  const int b = blockIdx.x % p;    // row-block
  const int cg = blockIdx.x / p;   // group of column-blocks
  const int c_end = min(p, (cg + 1) * kRmseColGroup);
  const float *Ub = U + G.row_start(b) * k;
  const uint32_t rmax = (uint32_t)(G.row_start(b + 1) - G.row_start(b)) - 1u;
  double acc = 0.0;
  for (int c = cg * kRmseColGroup + wave; c < c_end; c += kWavesPerGroup) {
    const int s = (c - b + p) % p;  // block (b, c) is in stratum s
    const int64_t beg = wblock_ptr[(int64_t)b * p + s];
    const int64_t end = wblock_ptr[(int64_t)b * p + s + 1];
    if (beg == end) continue;
    const float *Vb = V + G.col_start(c) * k;
    const uint32_t cmax = (uint32_t)(G.col_start(c + 1) - G.col_start(c)) - 1u;
    const uint32_t len = (uint32_t)(end - beg);
    static_assert((2 * UNR + 1) * RPS <= kAhead, "positions do not wrap");
    const uint2 *rb = rec + beg;
    // records of the next iteration are loaded one iteration ahead, so the
    // factor-row loads never wait for a record load
    uint2 rn[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const uint32_t t = u * RPS + grp;
      rn[u] = rb[t < len ? t : 0];
    }
    for (uint32_t t0 = 0; t0 < len; t0 += RPS * UNR) {
      float4 ua[UNR][QL], va[UNR][QL];
      float x[UNR];
      uint2 r[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        r[u] = rn[u];
        const uint32_t t = t0 + (UNR + u) * RPS + grp;
        rn[u] = rb[t < len ? t : 0];
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        x[u] = __uint_as_float(r[u].y);
        dot.load(ua[u], row_ptr(Ub, min(r[u].x & kRowMask, rmax), rowbytes));
        dot.load(va[u], row_ptr(Vb, min((r[u].x >> kColShift) & kColMask, cmax), rowbytes));
      }
      if constexpr (kFence) loads_issued();
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        float d = dot.error(x[u], ua[u], va[u]);
        d = t0 + u * RPS + grp < len ? d : 0.0f;
        acc = fma((double)d, (double)d, acc);
      }
    }
  }
  acc = wave_sum<L>(acc);
  if (lane == 0) partials[(int64_t)blockIdx.x * kWavesPerGroup + wave] = acc;
}

// Out-of-core RMSE over the strata [s0, s1) held in one device slot: the
// wave of row-block b and grid row y adds the squared errors of blocks
// (b, s), s = s0 + y, s0 + y + gridDim.y, ..., to partials[y p + b] (each
// partial is owned by one wave per launch, and launches are ordered on the
// stream).  A record and the rows it names are read in the same step.
//
// Steps in flight as in k_rmse_partial, FEW from other measurements (ratings
// streamed, one step and no fence against two fenced: 10M, p = 64, k = 64 4.3
// and 2.5 ms, k = 128 7.3 and 5.1; p = 1024, k = 128 1.45 and 1.42; 20M, p =
// 1024, k = 64 2.30 and 2.28; p = 2048, k = 128 2.76 and 3.11; p = 4096, k =
// 64 3.1 and 4.9).  At k = 16 a fence would hold back the next records' loads
// (p = 32: 2.8 against 1.8 ms); at k = 32 it pays (1.53 against 1.64).
constexpr int64_t kStratumFewWaves = 16384;  // 16 p waves in a full launch

template <int KP, bool FULL, bool FEW>
__global__ void __launch_bounds__(256)
k_rmse_stratum(const uint2 *__restrict__ rec, int64_t rec_origin,
               const int64_t *__restrict__ block_ptr, int32_t s0, int32_t s1,
               const float *__restrict__ U, const float *__restrict__ V, Grid G, int32_t k,
               double *__restrict__ partials) {
  using Dt = Dot<KP, FULL>;
  constexpr int L = Dt::L, QL = Dt::QL;
  constexpr int RPS = 64 / L;
  constexpr int UNR = rmse_unroll<KP>(FEW);
  constexpr bool kFence = KP == 32 || (KP >= 64 && FEW);
  const int32_t p = G.p;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane / L;
  const Dt dot(lane % L, k);
  const uint32_t rowbytes = (uint32_t)k * 4u;
  const int b = blockIdx.x * kWavesPerGroup + wave;
  if (b >= p) return;
  const float *Ub = U + G.row_start(b) * k;
  const uint32_t rmax = (uint32_t)(G.row_start(b + 1) - G.row_start(b)) - 1u;
  double acc = 0.0;
  for (int32_t s = s0 + (int32_t)blockIdx.y; s < s1; s += (int32_t)gridDim.y) {
    const int64_t beg = block_ptr[(int64_t)s * p + b];
    const uint32_t len = (uint32_t)(block_ptr[(int64_t)s * p + b + 1] - beg);
    static_assert((UNR + 1) * RPS <= kAhead, "positions do not wrap");
    const uint2 *rb = rec + (beg - rec_origin);
    const int C = (b + s) % p;
    const float *Vb = V + G.col_start(C) * k;
    const uint32_t cmax = (uint32_t)(G.col_start(C + 1) - G.col_start(C)) - 1u;
    for (uint32_t t0 = 0; t0 < len; t0 += RPS * UNR) {
      float4 ua[UNR][QL], va[UNR][QL];
      float x[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const uint32_t t = t0 + u * RPS + grp;
        const uint2 r = rb[t < len ? t : 0];
        x[u] = __uint_as_float(r.y);
        dot.load(ua[u], row_ptr(Ub, min(r.x & kRowMask, rmax), rowbytes));
        dot.load(va[u], row_ptr(Vb, min((r.x >> kColShift) & kColMask, cmax), rowbytes));
      }
      if constexpr (kFence) loads_issued();
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        float d = dot.error(x[u], ua[u], va[u]);
        d = t0 + u * RPS + grp < len ? d : 0.0f;
        acc = fma((double)d, (double)d, acc);
      }
    }
  }
  acc = wave_sum<L>(acc);
  if (lane == 0) partials[(int64_t)blockIdx.y * p + b] += acc;
}

// RMSE over caller-given COO ratings (for example a held-out split): the
// same dot products and fp64 squares, with a lane group per rating taken
// from a fixed grid-stride order, and one partial per wave.  A rating whose
// row or column lies outside the matrix, or whose value is not finite, adds
// nothing and sets a bit of *bad (1: index, 2: value); row 0 is read in the
// place of a row that does not exist.
//
// The rows of U and V are random reads, so the kernel is bound by how many
// of them are in flight: a wave has the rows of kCooUnroll steps outstanding
// and reads the indices of the steps after them meanwhile (10M ratings,
// k = 64: 474 us with one step and its indices in turn, 449 with indices
// ahead, 430 with two steps).  Two steps also at k = 16: eight take 130
// registers, with which only three quarters of the fixed grid (four waves
// per SIMD) fit the chip at once, and cost small calls 43.4 us against 40.1
// (100K ratings; 222 us either way at 10M).
constexpr int kCooUnroll = 2;

template <int KP, bool FULL>
__global__ void __launch_bounds__(256)
k_rmse_coo(const int32_t *__restrict__ rows, const int32_t *__restrict__ cols,
           const float *__restrict__ vals, int64_t nnz, const float *__restrict__ U,
           const float *__restrict__ V, int32_t k, int64_t n, int64_t m,
           double *__restrict__ partials, int32_t *bad) {
  using Dt = Dot<KP, FULL>;
  constexpr int L = Dt::L, QL = Dt::QL;
  constexpr int RPS = 64 / L;
  constexpr int UNR = kCooUnroll;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gl = lane % L, grp = lane / L;
  const Dt dot(gl, k);
  const uint32_t rowbytes = (uint32_t)k * 4u;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerGroup + wave;
  const int64_t stride = (int64_t)gridDim.x * kWavesPerGroup * RPS;
  double acc = 0.0;
  int32_t ri[UNR], rj[UNR];
  float rx[UNR];
  auto fetch = [&](int64_t t0) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int64_t t = t0 + u * stride + grp;
      const int64_t e = t < nnz ? t : 0;
      ri[u] = rows[e];
      rj[u] = cols[e];
      rx[u] = vals[e];
    }
  };
  int64_t t0 = gw * RPS;
  if (t0 < nnz) fetch(t0);
  for (; t0 < nnz; t0 += UNR * stride) {
    float4 ua[UNR][QL], va[UNR][QL];
    float x[UNR];
    bool ok[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const bool live = t0 + u * stride + grp < nnz;
      const bool in = ri[u] >= 0 && ri[u] < n && rj[u] >= 0 && rj[u] < m;
      const bool fin = __builtin_isfinite(rx[u]);
      if (live && gl == 0 && !(in && fin)) atomicOr(bad, (in ? 0 : 1) | (fin ? 0 : 2));
      ok[u] = live && in && fin;
      x[u] = rx[u];
      dot.load(ua[u], row_ptr(U, in ? (uint32_t)ri[u] : 0u, rowbytes));
      dot.load(va[u], row_ptr(V, in ? (uint32_t)rj[u] : 0u, rowbytes));
    }
    fetch(t0 + UNR * stride);
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      float d = dot.error(x[u], ua[u], va[u]);
      d = ok[u] ? d : 0.0f;
      acc = fma((double)d, (double)d, acc);
    }
  }
  acc = wave_sum<L>(acc);
  if (lane == 0) partials[gw] = acc;
}

__global__ void k_zero_i32(int32_t *x) { *x = 0; }

__global__ void k_zero(double *x, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = 0.0;
}

// Variant with the row-block's U rows staged in LDS: one workgroup of 16
// waves per row-block, u_i read from LDS, v_j from global memory.  The
// row-block's records of all strata are contiguous (wave-major), so each
// wave sums one contiguous sixteenth of them as a single stream; a table of
// block starts and column-blocks in LDS gives the block of each rating (a
// lane group steps its block forward as its ratings cross block starts), so
// no block boundary waits for memory.  Used when the rows and the tables
// fit in LDS.  100M ratings, k = 64: 1.27 ms.  The vector cache's data return
// is busy for 83% of all CU cycles, as long as the CUs are (the v rows alone,
// 256 bytes per rating at 64 bytes per cycle, take 0.72 ms); its address unit
// for 79%, LDS for 51% (36% bank conflicts: the rating groups of a wave read
// the same 64-byte piece of their rows together), the vector ALUs for 38%.
// Without the v loads 0.92 of 1.30 ms remained, so the units share the time:
// with one workgroup on a CU their work overlaps only in part.
constexpr int kLdsWaves = 16;

template <int KP, bool FULL>
__global__ void __launch_bounds__(1024)
k_rmse_lds(const uint2 *__restrict__ rec, const int64_t *__restrict__ wblock_ptr,
           const float *__restrict__ U, const float *__restrict__ V, Grid G, int32_t k,
           double *__restrict__ partials) {
  using Dt = Dot<KP, FULL>;
  constexpr int L = Dt::L, QL = Dt::QL;
  constexpr int RPS = 64 / L;
  constexpr int UNR = rmse_unroll_lds<KP, FULL>();
  const int32_t p = G.p;
  extern __shared__ float4 us[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = lane / L;
  const Dt dot(lane % L, k);
  const uint32_t rowbytes = (uint32_t)k * 4u;
  const int b = blockIdx.x;
  const int64_t r0 = G.row_start(b);
  const uint32_t rows_b = (uint32_t)(G.row_start(b + 1) - r0);
  const uint32_t rmax = rows_b - 1u;
  const int kq = k / 4;
  // after the rows: the start of block (b, s) relative to the row-block's
  // first record (p + 1 entries), then per stratum its column-block's first
  // column and widest local column
  int32_t *bnd = reinterpret_cast<int32_t *>(us + rows_b * (uint32_t)kq);
  int2 *ctab = reinterpret_cast<int2 *>(bnd + ((p + 2) & ~1));
  const int64_t W0 = wblock_ptr[(int64_t)b * p];
  {  // the row-block's rows are contiguous in U
    const float4 *src = reinterpret_cast<const float4 *>(U + r0 * k);
    const uint32_t total = rows_b * (uint32_t)kq;
    for (uint32_t i = threadIdx.x; i < total; i += blockDim.x) us[i] = src[i];
    for (int s = threadIdx.x; s <= p; s += blockDim.x)
      bnd[s] = (int32_t)(wblock_ptr[(int64_t)b * p + s] - W0);
    for (int s = threadIdx.x; s < p; s += blockDim.x) {
      const int C = (b + s) % p;
      const int64_t c0 = G.col_start(C);
      ctab[s] = make_int2((int32_t)c0, (int32_t)(G.col_start(C + 1) - c0 - 1));
    }
  }
  __syncthreads();
  // The wave's ratings are [tb, tb + cnt) of the row-block's; t below is
  // relative to tb (at most 2^31 / 16 ratings, so 32 bits hold every t).
  const int32_t T = __builtin_amdgcn_readfirstlane(bnd[p]);
  const int32_t tb = (int32_t)((int64_t)T * wave / kLdsWaves);
  const int32_t cnt = (int32_t)((int64_t)T * (wave + 1) / kLdsWaves) - tb;
  double acc = 0.0;
  if (cnt > 0) {
    // block of the wave's first rating: the last s with bnd[s] <= tb
    int32_t lo = 0, hi = p - 1;
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (bnd[mid] <= tb) lo = mid;
      else hi = mid - 1;
    }
    int32_t sg = lo;           // block of the lane group's current rating
    int32_t nb = bnd[sg + 1] - tb;  // start of the block after it
    int2 ct = ctab[sg];
    const uint2 *rb = rec + W0 + tb;
    // The records of an iteration are loaded two iterations ahead and turned
    // into row addresses one iteration ahead, while the rows of the current
    // one are on their way, so no load waits for another.
    uint2 rn[UNR];
    const char *vp[UNR];
    uint32_t uo[UNR];
    float xn[UNR];
    auto fetch = [&](int32_t t0) {
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int32_t t = t0 + u * RPS + grp;
        rn[u] = rb[t < cnt ? t : 0];
      }
    };
    auto decode = [&](int32_t t0) {
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int32_t t = t0 + u * RPS + grp;
        // step to the block of rating t (past empty blocks); tb + cnt <= bnd[p]
        if (t < cnt && t >= nb) {
          do {
            ++sg;
            nb = bnd[sg + 1] - tb;
          } while (t >= nb);
          ct = ctab[sg];
        }
        xn[u] = __uint_as_float(rn[u].y);
        uo[u] = min(rn[u].x & kRowMask, rmax) * rowbytes;
        vp[u] = row_ptr(V, (uint32_t)ct.x + min((rn[u].x >> kColShift) & kColMask, (uint32_t)ct.y),
                        rowbytes);
      }
    };
    fetch(0);
    decode(0);
    fetch(RPS * UNR);
    for (int32_t t0 = 0; t0 < cnt; t0 += RPS * UNR) {
      float4 ua[UNR][QL], va[UNR][QL];
      float x[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        dot.load(va[u], vp[u]);
        dot.load(ua[u], reinterpret_cast<const char *>(us) + uo[u]);
        x[u] = xn[u];
      }
      decode(t0 + RPS * UNR);
      fetch(t0 + 2 * RPS * UNR);
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        float d = dot.error(x[u], ua[u], va[u]);
        d = t0 + u * RPS + grp < cnt ? d : 0.0f;
        acc = fma((double)d, (double)d, acc);
      }
    }
  }
  acc = wave_sum<L>(acc);
  if (lane == 0) partials[(int64_t)b * kLdsWaves + wave] = acc;
}

// Sum of the partials in a fixed order (the result does not depend on
// scheduling): thread t adds partials t, t + 256, ... into eight sums by
// index (eight loads in flight instead of one), combined pairwise, then a
// tree over the threads.
__global__ void __launch_bounds__(256)
k_rmse_final(const double *__restrict__ partials, int64_t count, int64_t nnz, double *out) {
  __shared__ double sh[256];
  constexpr int A = 8;
  double a[A];
#pragma unroll
  for (int u = 0; u < A; ++u) a[u] = 0.0;
  int64_t i = threadIdx.x;
  for (; i + (A - 1) * 256 < count; i += A * 256) {
#pragma unroll
    for (int u = 0; u < A; ++u) a[u] += partials[i + u * 256];
  }
  for (; i < count; i += 256) a[0] += partials[i];
  sh[threadIdx.x] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = nnz > 0 ? sqrt(sh[0] / (double)nnz) : 0.0;
}

}  // namespace

size_t rmse_partials_count(int32_t p) {
  const int64_t groups = ((int64_t)p + kRmseColGroup - 1) / kRmseColGroup;
  return (size_t)p * (size_t)std::max<int64_t>(groups * kWavesPerGroup, kLdsWaves);
}

namespace {
template <int KP, bool FULL>
hipError_t launch_rmse_kp(const uint2 *rec, const int64_t *wblock_ptr, const float *U,
                          const float *V, const Grid &G, int64_t rows_max, int32_t k,
                          double *partials, size_t lds_limit, int64_t *count,
                          hipStream_t stream) {
  const int32_t p = G.p;
  const size_t lds = (size_t)rows_max * (size_t)k * sizeof(float) +
                     (size_t)((p + 2) & ~1) * sizeof(int32_t) + (size_t)p * sizeof(int2);
  if (lds <= lds_limit) {
    static bool attr_set = false;
    if (!attr_set) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_rmse_lds<KP, FULL>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)lds_limit);
      if (e != hipSuccess) return e;
      attr_set = true;
    }
    hipLaunchKernelGGL((k_rmse_lds<KP, FULL>), dim3((unsigned)p), dim3(64 * kLdsWaves), lds, stream,
                       rec, wblock_ptr, U, V, G, k, partials);
    *count = (int64_t)p * kLdsWaves;
  } else {
    const int64_t groups = (int64_t)p * ((p + kRmseColGroup - 1) / kRmseColGroup);
    constexpr bool kByWaves = KP >= 64;  // narrower rows: one variant
    auto f = kByWaves && groups * kWavesPerGroup <= few_waves<KP>()
                 ? k_rmse_partial<KP, FULL, kByWaves>
                 : k_rmse_partial<KP, FULL, false>;
    hipLaunchKernelGGL(f, dim3((unsigned)groups), dim3(256), 0, stream, rec, wblock_ptr, U, V, G,
                       k, partials);
    *count = groups * kWavesPerGroup;
  }
  return hipGetLastError();
}

// Calls f with the kernels' template arguments for width k.
template <class F>
hipError_t with_width(int32_t k, F &&f) {
  int kp = 16;
  while (kp < k) kp <<= 1;
  auto full = [&](auto w) {
    constexpr int KP = decltype(w)::value;
    return k == KP ? f(w, std::true_type{}) : f(w, std::false_type{});
  };
  switch (kp) {
    case 16: return f(std::integral_constant<int, 16>{}, std::true_type{});
    case 32: return f(std::integral_constant<int, 32>{}, std::true_type{});
    case 64: return full(std::integral_constant<int, 64>{});
    case 128: return full(std::integral_constant<int, 128>{});
    case 256: return full(std::integral_constant<int, 256>{});
    default: return hipErrorInvalidValue;
  }
}
}  // namespace

hipError_t rmse_stratum_begin(double *partials, int32_t p, hipStream_t stream) {
  const int64_t count = (int64_t)kRmseStrataGroups * p;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, partials,
                     count);
  return hipGetLastError();
}

hipError_t rmse_stratum_add(const uint2 *rec, int64_t rec_origin, const int64_t *block_ptr,
                            int32_t s0, int32_t s1, const float *U, const float *V,
                            const Grid &G, int32_t k, double *partials, hipStream_t stream) {
  const int32_t p = G.p;
  const dim3 grid((unsigned)((p + kWavesPerGroup - 1) / kWavesPerGroup),
                  (unsigned)std::min(kRmseStrataGroups, s1 - s0));
  return with_width(k, [&](auto w, auto full) {
    constexpr int KP = decltype(w)::value;
    constexpr bool FULL = decltype(full)::value;
    const int64_t waves = (int64_t)grid.x * grid.y * kWavesPerGroup;
    constexpr bool kByWaves = KP >= 64;
    auto f = kByWaves && waves <= kStratumFewWaves ? k_rmse_stratum<KP, FULL, kByWaves>
                                            : k_rmse_stratum<KP, FULL, false>;
    hipLaunchKernelGGL(f, grid, dim3(256), 0, stream, rec, rec_origin, block_ptr, s0, s1, U, V, G,
                       k, partials);
    return hipGetLastError();
  });
}

hipError_t rmse_stratum_end(const double *partials, int32_t p, int64_t nnz, double *out,
                            hipStream_t stream) {
  hipLaunchKernelGGL(k_rmse_final, dim3(1), dim3(256), 0, stream, partials,
                     (int64_t)kRmseStrataGroups * p, nnz, out);
  return hipGetLastError();
}

size_t rmse_coo_partials_count() { return (size_t)kRmseCooGroups * kWavesPerGroup; }

hipError_t launch_rmse_coo(const int32_t *rows, const int32_t *cols, const float *vals,
                           int64_t nnz, const float *U, const float *V, int32_t k, int64_t n,
                           int64_t m, double *partials, double *out, int32_t *bad,
                           hipStream_t stream) {
  hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(1), 0, stream, bad);
  hipError_t e = with_width(k, [&](auto w, auto full) {
    hipLaunchKernelGGL((k_rmse_coo<decltype(w)::value, decltype(full)::value>),
                       dim3(kRmseCooGroups), dim3(64 * kWavesPerGroup), 0, stream, rows, cols, vals,
                       nnz, U, V, k, n, m, partials, bad);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_rmse_final, dim3(1), dim3(256), 0, stream, partials,
                     (int64_t)rmse_coo_partials_count(), nnz, out);
  return hipGetLastError();
}

hipError_t launch_rmse(const uint2 *rec, const int64_t *wblock_ptr, const float *U,
                       const float *V, const Grid &G, int64_t rows_max, int32_t k, int64_t nnz,
                       double *partials, double *out, size_t lds_limit, hipStream_t stream) {
  int64_t count = 0;
  hipError_t e = with_width(k, [&](auto w, auto full) {
    return launch_rmse_kp<decltype(w)::value, decltype(full)::value>(
        rec, wblock_ptr, U, V, G, rows_max, k, partials, lds_limit, &count, stream);
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_rmse_final, dim3(1), dim3(256), 0, stream, partials, count, nnz, out);
  return hipGetLastError();
}

}  // namespace bgmfk
