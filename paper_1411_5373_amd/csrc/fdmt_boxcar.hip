// Boxcar search over FDMT output planes: for every row (trial delay) and
// width w = 2^j, the causal running sum b_w[t] = y[t] + ... + y[t - w + 1]
// (zero before the record), its largest value with the first time it occurs,
// and the mean and standard deviation of b_w over the record. A pulse
// profile shared by all frequencies commutes with the transform (Sec. 4.2,
// pulse profile), so one transform serves every width.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "fdmt_boxcar.h"

// Device scratch of the allocation-free boxcar search: the per-(row, tile,
// width) partials, for callers that cannot allocate (see
// boxcar_static_scratch). Each GPU the library runs on holds its own copy
// until the process ends. Host code must not pass this name to a kernel: on
// the host it stands for a host-side shadow, not the device address, which
// boxcar_static_scratch looks up per device.
static __device__ __align__(256) unsigned char scratch[fdmt::kBoxScratchBytes];

namespace fdmt {

namespace {

constexpr int kBoxThreads = 64;  // one wave: its LDS steps need no workgroup barrier to wait on other waves

// Peak order: larger value first, then earlier time.
__device__ __forceinline__ bool better(float v, int t, float bv, int bt) { return v > bv || (v == bv && t < bt); }

template <typename T>
__device__ __forceinline__ T xor_lane(T x, int mask) {
  return __shfl_xor(x, mask, 64);
}

// ---------------------------------------------------------------------------
// Boxcar search of a row, one wave per `span` consecutive tiles of kBoxTile
// samples. Width 2w comes from width w as b_2w[t] = b_w[t] + b_w[t - w], which
// sums each window in a fixed tree.
//
// A tile lives in registers: chunk c of 256 samples, 4 consecutive ones per
// lane, so loads are coalesced and an addition per sample and width is all the
// doubling costs. b_w[t - w] is a lane's own sample or its neighbour's for
// w = 1 and 2 (one DPP move into lane i from lane i - 1, lane 0's from the
// chunk before), and for w >= 4 one 16-byte LDS write and one aligned 16-byte
// read per chunk. The last w values of each width are kept for the next tile;
// a wave's first tile takes them from a run over the samples before it.
//
// What bounds it: the vector ALU. Per sample and width there is the addition,
// the conversion, sum and sum of squares in FP64 and half a v_max3. The peak
// keeps only values: its first time is looked up once per tile and width, and
// the FP64 sums are reduced across the wave once per span (a tile's own are
// never used). With every width in LDS, a peak test per sample and a reduction
// per tile and width, widths 1..256 over 2048 x 65536 took 0.62 ms; this takes
// 0.30-0.33 ms at 76% of the vector ALU's issue rate (reading the plane takes 0.1 ms).
constexpr int kBoxChunks = kBoxTile / 256;

typedef float Float4 __attribute__((ext_vector_type(4)));
typedef float Float4u __attribute__((ext_vector_type(4), aligned(4)));  // a row starts at any sample

// x of the lane before; lane 0 takes `first`.
__device__ __forceinline__ float lane_before(float first, float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, first), __builtin_bit_cast(int, x),
                                                               0x138, 0xf, 0xf, false));  // wave_shr:1
}
// Rotated by one lane: lane 0 has lane 63's x.
__device__ __forceinline__ float rotated(float x) {
  const int i = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, 0x13c, 0xf, 0xf, false));  // wave_ror:1
}

// Largest value over the wave (NaN never wins), the same for every lane.
__device__ __forceinline__ float wave_max(float x) {
#define FDMT_MAX_STEP(CTRL, ROWS)                                                                              \
  {                                                                                                            \
    const int i = __builtin_bit_cast(int, x);                                                                  \
    x = __builtin_fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, CTRL, ROWS, 0xf, false))); \
  }
  FDMT_MAX_STEP(0x111, 0xf)  // row_shr:1, 2, 4, 8: lane 15 of each row has the row's
  FDMT_MAX_STEP(0x112, 0xf)
  FDMT_MAX_STEP(0x114, 0xf)
  FDMT_MAX_STEP(0x118, 0xf)
  FDMT_MAX_STEP(0x142, 0xa)  // row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3
  FDMT_MAX_STEP(0x143, 0xc)
#undef FDMT_MAX_STEP
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}

// LDS accesses of one wave run in program order; the compiler must not move
// them past each other on the grounds that one lane's addresses differ.
__device__ __forceinline__ void lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// What a tile needs of the one before: the last w values of each width w.
struct BoxHistory {
  float one = 0.0f, two[2] = {0.0f, 0.0f};  // widths 1 and 2, in lane 0
  float *lds;                               // width w >= 4: lds[w .. 2w - 1]
};

// v: values of width 2^J, C chunks; becomes width 2^(J + 1). buf: 256 C samples.
template <int J, int C>
__device__ __forceinline__ void box_double(Float4 (&v)[C], BoxHistory &h, float *buf, int lane) {
  if constexpr (J == 0) {
    float first = h.one;
    h.one = rotated(v[C - 1][3]);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const Float4 x = v[c];
      v[c] = x + Float4{lane_before(first, x[3]), x[0], x[1], x[2]};
      if (c + 1 < C) first = rotated(x[3]);
    }
  } else if constexpr (J == 1) {
    float f0 = h.two[0], f1 = h.two[1];
    h.two[0] = rotated(v[C - 1][2]);
    h.two[1] = rotated(v[C - 1][3]);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const Float4 x = v[c];
      v[c] = x + Float4{lane_before(f0, x[2]), lane_before(f1, x[3]), x[0], x[1]};
      if (c + 1 < C) {
        f0 = rotated(x[2]);
        f1 = rotated(x[3]);
      }
    }
  } else {
    constexpr int w = 1 << J;
    constexpr int kPast = w > 256 ? w / 256 : 1;  // chunks whose earlier samples reach before the tile
    static_assert(kPast <= C, "a tile holds the widest history");
    float *hist = h.lds + w;
    lds_order();
#pragma unroll
    for (int c = 0; c < C; ++c) *reinterpret_cast<Float4 *>(buf + 256 * c + 4 * lane) = v[c];
    lds_order();
    Float4 past[kPast];
    if constexpr (w >= 256) {
#pragma unroll
      for (int c = 0; c < kPast; ++c) past[c] = *reinterpret_cast<const Float4 *>(hist + 256 * c + 4 * lane);
    } else {
      past[0] = *reinterpret_cast<const Float4 *>(4 * lane < w ? hist + 4 * lane : buf + 4 * lane - w);
    }
    lds_order();
    if constexpr (w >= 256) {
#pragma unroll
      for (int c = 0; c < kPast; ++c) *reinterpret_cast<Float4 *>(hist + 256 * c + 4 * lane) = v[C - kPast + c];
    } else {
      if (4 * lane >= 256 - w) *reinterpret_cast<Float4 *>(hist + 4 * lane - (256 - w)) = v[C - 1];
    }
#pragma unroll
    for (int c = kPast; c < C; ++c) v[c] = v[c] + *reinterpret_cast<const Float4 *>(buf + 256 * c + 4 * lane - w);
#pragma unroll
    for (int c = 0; c < kPast; ++c) v[c] = v[c] + past[c];
  }
}

// Statistics of one width over a tile of C chunks: FP64 sums of the lane's
// samples, and the wave's peak with its first sample (INT32_MAX: no peak, every
// value a NaN). FULL: every sample counts; else those below nvalid.
template <bool FULL, int C>
__device__ __forceinline__ void box_stats(const Float4 (&v)[C], int nvalid, int lane, double &s, double &q,
                                          float &peak, int &at) {
  float top[C];
  double s1 = 0.0, q1 = 0.0;
  float best = -__builtin_inff();
#pragma unroll
  for (int c = 0; c < C; ++c) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double x = static_cast<double>(v[c][i]);
      if (!FULL) x = 256 * c + 4 * lane + i < nvalid ? x : 0.0;
      if (c & 1) {
        s1 += x;
        q1 = __builtin_fma(x, x, q1);
      } else {
        s += x;
        q = __builtin_fma(x, x, q);
      }
    }
    if (FULL) {
      top[c] = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(v[c][0], v[c][1]), v[c][2]), v[c][3]);
    } else {
      top[c] = __builtin_nanf("");  // stays one, equal to no peak, without a valid sample that is a number
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (256 * c + 4 * lane + i < nvalid) top[c] = __builtin_fmaxf(top[c], v[c][i]);
    }
    best = __builtin_fmaxf(best, top[c]);
  }
  s += s1;
  q += q1;
  // the sums are done here: left to the scheduler they move past the branches
  // below, with every width's samples kept for them (1.3 KB of scratch)
  asm volatile("" : "+v"(s), "+v"(q));
  peak = wave_max(best);
  at = INT32_MAX;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    if (at != INT32_MAX) continue;
    const bool here = top[c] == peak;
    const uint64_t lanes = __builtin_amdgcn_ballot_w64(here);
    if (lanes) {
      int i = 3;
      if (v[c][2] == peak) i = 2;
      if (v[c][1] == peak) i = 1;
      if (v[c][0] == peak) i = 0;
      const int l = __builtin_ctzll(lanes);
      at = 256 * c + 4 * l + __builtin_amdgcn_readlane(i, l);
    }
  }
}

// Sums of the widths of a span, per lane, and the step over a tile's widths.
template <int M>
struct BoxSums {
  double s[M + 1] = {}, q[M + 1] = {};
};

template <int M, int J, bool FULL, int C>
__device__ __forceinline__ void box_widths(Float4 (&v)[C], BoxHistory &h, float *buf, int lane, int nvalid,
                                           BoxSums<M> &sums, BoxPartial *p, int64_t width_stride, int32_t t0) {
  float peak;
  int at;
  box_stats<FULL>(v, nvalid, lane, sums.s[J], sums.q[J], peak, at);
  if (lane == 0) {
    // a tile without a peak keeps INT32_MAX: the kernels below know it by that
    p[J * width_stride] = BoxPartial{0.0, 0.0, peak, at == INT32_MAX ? INT32_MAX : t0 + at};
  }
  if constexpr (J < M) {
    // keep the widths apart: mixed by the scheduler, their values are all live
    // at once (362 VGPRs at M = 8)
    __builtin_amdgcn_sched_barrier(0);
    box_double<J>(v, h, buf, lane);
    __builtin_amdgcn_sched_barrier(0);
    box_widths<M, J + 1, FULL>(v, h, buf, lane, nvalid, sums, p, width_stride, t0);
  }
}

template <int M, int J, int C>
__device__ __forceinline__ void box_warm(Float4 (&v)[C], BoxHistory &h, float *buf, int lane) {
  if constexpr (J < M) {
    box_double<J>(v, h, buf, lane);
    box_warm<M, J + 1>(v, h, buf, lane);
  }
}

// A row's last tile of nvalid samples, at most C chunks (nothing follows that
// would need its history).
template <int M, int C>
__device__ __forceinline__ void box_last_tile(const float *y, BoxHistory &h, float *buf, int lane, int nvalid,
                                              BoxSums<M> &sums, BoxPartial *p, int64_t width_stride, int32_t t0) {
  Float4 v[C];
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = 256 * c + 4 * lane + i;
      v[c][i] = u < nvalid ? y[u] : 0.0f;
    }
  box_widths<M, 0, false>(v, h, buf, lane, nvalid, sums, p, width_stride, t0);
}

// Rows of kBoxFew chunks or fewer (SHORT) do no more than those chunks: 50000
// rows of 50 samples with widths 1..32 took 163 us with every width in LDS, 221
// us as whole tiles and now 113 us. Other rows' last tiles are whole ones: with a
// form for few chunks beside, the search of long rows was 3% slower.
constexpr int kBoxFew = 2;  // the widest history, 512 samples, takes as many

// Three waves per SIMD: at four (128 VGPRs) the widest searches spill, 0.36 ms.
template <int M, bool SHORT>
__global__ __launch_bounds__(kBoxThreads, 3) void boxcar_tile_kernel(const float *__restrict__ plane,
                                                                  BoxPartial *__restrict__ part, int64_t nt,
                                                                  int32_t nd, int32_t ntiles, int32_t span) {
  __shared__ __align__(16) float buf[kBoxTile];
  __shared__ __align__(16) float hist[1 << (M > 2 ? M : 2)];
  const int row = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
  const int first = blockIdx.x * span;
  const int last = first + span < ntiles ? first + span : ntiles;
  const float *y = plane + (static_cast<int64_t>(b) * nd + row) * nt;
  const int64_t width_stride = static_cast<int64_t>(nd) * ntiles;
  BoxPartial *p = part + (static_cast<int64_t>(b) * (M + 1) * nd + row) * ntiles;
  BoxHistory h;
  h.lds = hist;
  for (int i = lane; i < (1 << (M > 2 ? M : 2)); i += kBoxThreads) hist[i] = 0.0f;
  if (first > 0 && M > 0) {
    // the widest window reaches 2^M - 1 samples back
    constexpr int C = M > 8 ? 1 << (M - 8) : 1;
    Float4 v[C];
    const float *x = y + (static_cast<int64_t>(first) * kBoxTile - 256 * C);
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = *reinterpret_cast<const Float4u *>(x + 256 * c + 4 * lane);
    box_warm<M, 0>(v, h, buf, lane);
  }
  BoxSums<M> sums;
  for (int tile = first; tile < last; ++tile) {
    const int64_t t0 = static_cast<int64_t>(tile) * kBoxTile;
    const int64_t left = nt - t0;
    if (SHORT) {
      box_last_tile<M, kBoxFew>(y + t0, h, buf, lane, static_cast<int>(left), sums, p + tile, width_stride,
                                static_cast<int32_t>(t0));
    } else if (left >= kBoxTile) {
      Float4 v[kBoxChunks];
#pragma unroll
      for (int c = 0; c < kBoxChunks; ++c) v[c] = *reinterpret_cast<const Float4u *>(y + t0 + 256 * c + 4 * lane);
      box_widths<M, 0, true>(v, h, buf, lane, kBoxTile, sums, p + tile, width_stride, static_cast<int32_t>(t0));
    } else {
      box_last_tile<M, kBoxChunks>(y + t0, h, buf, lane, static_cast<int>(left), sums, p + tile, width_stride,
                                   static_cast<int32_t>(t0));
    }
  }
  // the span's sums go to its first tile's partials
#pragma unroll
  for (int j = 0; j <= M; ++j) {
    double s = sums.s[j], q = sums.q[j];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      s += xor_lane(s, m);
      q += xor_lane(q, m);
    }
    if (lane == 0) {
      p[j * width_stride + first].sum = s;
      p[j * width_stride + first].sumsq = q;
    }
  }
}

// Windows that straddle the start of tile k >= 1 (their first samples lie in
// tile k - 1), for a search whose tile partials cover only the windows
// inside each tile (the search fused into the last forward pass). One wave
// per (tile start, row, beam) loads the 2^max_log2 - 1 samples before the
// start and as many from it, builds the widths with the same doubling tree,
// and for width w folds b_w at t = start .. start + w - 2 into the tile's
// partial: its sums, and its peak when not smaller than the tile's (these
// times come first).
__global__ __launch_bounds__(kBoxThreads) void boxcar_edge_kernel(const float *__restrict__ plane,
                                                                  BoxPartial *__restrict__ part, int64_t nt,
                                                                  int32_t nd, int32_t ntiles, int32_t max_log2) {
  extern __shared__ float ebuf[];  // 2 * (2^max_log2 - 1) samples
  const int tile = blockIdx.x + 1, row = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  const int halo = (1 << max_log2) - 1;
  const int64_t start = static_cast<int64_t>(tile) * kBoxTile;
  const int64_t left = nt - start;
  const int after = left < halo ? static_cast<int>(left) : halo;  // samples of the tile the edge windows end at
  const int n = halo + after;
  const float *y = plane + (static_cast<int64_t>(b) * nd + row) * nt;
  // local index i holds time start - halo + i (start - halo >= 0 since tile >= 1)
  for (int i = tid; i < n; i += kBoxThreads) ebuf[i] = y[start - halo + i];
  __syncthreads();
  for (int j = 0; j <= max_log2; ++j) {
    const int w = 1 << j;
    if (j > 0) {
      // width w from width w/2, in place from the top down: a group of 64
      // reads all its old values before writing, and reads only below its top
      const int hw = w >> 1;
      for (int top = n - 1; top >= hw; top -= kBoxThreads) {
        const int i = top - tid;
        float nv = 0.0f;
        if (i >= hw) nv = ebuf[i] + ebuf[i - hw];
        if (i >= hw) ebuf[i] = nv;
      }
      __syncthreads();
    }
    // times start .. start + min(w - 1, after) - 1: local index halo + u
    const int cnt = w - 1 < after ? w - 1 : after;
    double s = 0.0, q = 0.0;
    float best = -__builtin_inff();
    int best_t = INT32_MAX;
    for (int u = tid; u < cnt; u += kBoxThreads) {
      const float v = ebuf[halo + u];
      s += static_cast<double>(v);
      q += static_cast<double>(v) * static_cast<double>(v);
      if (v > best || (v == best && u < best_t)) {
        best = v;
        best_t = u;
      }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      s += xor_lane(s, m);
      q += xor_lane(q, m);
      const float ov = xor_lane(best, m);
      const int ot = xor_lane(best_t, m);
      if (better(ov, ot, best, best_t)) {
        best = ov;
        best_t = ot;
      }
    }
    if (tid == 0 && cnt > 0) {
      BoxPartial &p = part[((static_cast<int64_t>(b) * (max_log2 + 1) + j) * nd + row) * ntiles + tile];
      p.sum += s;
      p.sumsq += q;
      // an edge time precedes every time of the tile's own partial
      if (best_t != INT32_MAX && (best >= p.peak || p.t == INT32_MAX)) {
        p.peak = best;
        p.t = static_cast<int32_t>(start) + best_t;
      }
    }
    __syncthreads();
  }
}

// kCombineLanes lanes per (beam, width, row), which take the tiles' partials in
// turn. mean_sd (optional) receives the float64 mean and standard deviation,
// found (optional) is the candidate count, cleared for the kernel after this.
// One thread per row walked 32 partials one after another: 14 us for 9 widths
// of 2048 rows, now 6 us.
// A launch takes fewer than 2^32 threads, so more than kCombineBlocks blocks'
// worth of results go round the grid.
constexpr int kCombineLanes = 16;
constexpr int64_t kCombineBlocks = 1 << 20;
__global__ __launch_bounds__(256) void boxcar_combine_kernel(const BoxPartial *__restrict__ part,
                                                             fdmt_boxcar_t *__restrict__ out, int64_t nt,
                                                             int32_t ntiles, int64_t count,
                                                             double2 *__restrict__ mean_sd,
                                                             int32_t *__restrict__ found) {
  const int64_t id = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (found && id == 0) *found = 0;
  const int lane = static_cast<int>(id % kCombineLanes);
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x / kCombineLanes;
  for (int64_t k = id / kCombineLanes; k < count; k += stride) {  // the same for a whole group of lanes
    const BoxPartial *p = part + k * ntiles;
    double s = 0.0, q = 0.0;
    float best = -__builtin_inff();
    int best_t = INT32_MAX;
    for (int i = lane; i < ntiles; i += kCombineLanes) {
      const BoxPartial x = p[i];
      s += x.sum;
      q += x.sumsq;
      if (better(x.peak, x.t, best, best_t)) {
        best = x.peak;
        best_t = x.t;
      }
    }
#pragma unroll
    for (int m = kCombineLanes / 2; m >= 1; m >>= 1) {
      s += __shfl_xor(s, m, kCombineLanes);
      q += __shfl_xor(q, m, kCombineLanes);
      const float ov = __shfl_xor(best, m, kCombineLanes);
      const int ot = __shfl_xor(best_t, m, kCombineLanes);
      if (better(ov, ot, best, best_t)) {
        best = ov;
        best_t = ot;
      }
    }
    if (lane != 0) continue;
    const double mean = s / static_cast<double>(nt);
    const double var = q / static_cast<double>(nt) - mean * mean;
    const double sd = var > 0.0 ? sqrt(var) : 0.0;
    fdmt_boxcar_t r;
    r.peak = best;
    r.t = best_t;
    r.mean = static_cast<float>(mean);
    r.stdev = static_cast<float>(sd);
    r.snr = sd > 0.0 ? static_cast<float>((static_cast<double>(best) - mean) / sd) : 0.0f;
    out[k] = r;
    if (mean_sd) mean_sd[k] = make_double2(mean, sd);
  }
}

// One thread per (beam, width, row, tile): the tile's peak is a candidate
// when its S/N against the row's float64 statistics reaches the threshold.
__global__ __launch_bounds__(256) void boxcar_candidate_kernel(const BoxPartial *__restrict__ part,
                                                               const double2 *__restrict__ mean_sd, int32_t nd,
                                                               int32_t ntiles, int32_t max_log2, int64_t count,
                                                               float threshold, fdmt_candidate_t *__restrict__ cand,
                                                               int32_t cap, int32_t *__restrict__ found) {
  const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= count) return;
  const BoxPartial p = part[k];
  if (p.t == INT32_MAX) return;  // a tile without a peak (every value NaN)
  const int64_t r = k / ntiles;  // (beam, width, row)
  const double2 ms = mean_sd[r];
  const double snr = ms.y > 0.0 ? (static_cast<double>(p.peak) - ms.x) / ms.y : 0.0;
  if (!(snr >= static_cast<double>(threshold))) return;
  const int32_t row = static_cast<int32_t>(r % nd);
  const int32_t j = static_cast<int32_t>((r / nd) % (max_log2 + 1));
  const int32_t b = static_cast<int32_t>(r / nd / (max_log2 + 1));
  const int32_t slot = atomicAdd(found, 1);
  if (slot < cap) {
    fdmt_candidate_t c;
    c.beam = b;
    c.dt = row;
    c.t = p.t;
    c.width_log2 = j;
    c.peak = p.peak;
    c.snr = static_cast<float>(snr);
    cand[slot] = c;
  }
}

} // namespace

size_t boxcar_workspace_bytes(int32_t batch, int32_t nd, int64_t nt, int32_t max_log2) {
  const int64_t ntiles = (nt + kBoxTile - 1) / kBoxTile;
  return static_cast<size_t>(batch) * (max_log2 + 1) * nd * ntiles * sizeof(BoxPartial);
}

hipError_t boxcar_static_scratch(int device, void **ptr) {
  // device addresses of `scratch`, looked up once per device with that device current
  static std::mutex lock;
  static void *addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> guard(lock);
  if (!addr[device]) {
    int current = -1;
    hipError_t e = hipGetDevice(&current);
    if (e != hipSuccess) return e;
    if (current != device) return hipErrorInvalidDevice;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[device] = p;
  }
  *ptr = addr[device];
  return hipSuccess;
}

hipError_t launch_boxcar_tiles(const float *plane, int32_t batch, int32_t nd, int64_t nt, int32_t max_log2,
                               BoxPartial *part, hipStream_t stream) {
  const int64_t ntiles = (nt + kBoxTile - 1) / kBoxTile;
  // four tiles per wave while that leaves each of the 1024 SIMDs four waves:
  // the sums are reduced, and the samples before a span read again, per wave
  int32_t span = 4;
  while (span > 1 && (ntiles + span - 1) / span * nd * batch < 4096) span /= 2;
  const dim3 grid(static_cast<unsigned>((ntiles + span - 1) / span), nd, batch);
#define FDMT_BOX(MM)                                                                                             \
  case MM:                                                                                                       \
    if (nt <= 256 * kBoxFew)                                                                                     \
      hipLaunchKernelGGL((boxcar_tile_kernel<MM, true>), grid, dim3(kBoxThreads), 0, stream, plane, part, nt, nd, \
                         static_cast<int32_t>(ntiles), span);                                                    \
    else                                                                                                         \
      hipLaunchKernelGGL((boxcar_tile_kernel<MM, false>), grid, dim3(kBoxThreads), 0, stream, plane, part, nt,    \
                         nd, static_cast<int32_t>(ntiles), span);                                                \
    break;
  switch (max_log2) {
    FDMT_BOX(0) FDMT_BOX(1) FDMT_BOX(2) FDMT_BOX(3) FDMT_BOX(4) FDMT_BOX(5)
    FDMT_BOX(6) FDMT_BOX(7) FDMT_BOX(8) FDMT_BOX(9) FDMT_BOX(10)
    default: return hipErrorInvalidValue;
  }
#undef FDMT_BOX
  return hipGetLastError();
}

hipError_t launch_boxcar_edges(const float *plane, int32_t batch, int32_t nd, int64_t nt, int32_t max_log2,
                               BoxPartial *part, hipStream_t stream) {
  const int64_t ntiles = (nt + kBoxTile - 1) / kBoxTile;
  if (ntiles < 2 || max_log2 == 0) return hipSuccess;  // no window straddles a tile start
  const size_t lds = 2 * ((1 << max_log2) - 1) * sizeof(float);
  hipLaunchKernelGGL(boxcar_edge_kernel, dim3(static_cast<unsigned>(ntiles - 1), nd, batch), dim3(kBoxThreads),
                     lds, stream, plane, part, nt, nd, static_cast<int32_t>(ntiles), max_log2);
  return hipGetLastError();
}

hipError_t launch_boxcar_combine(const BoxPartial *part, int32_t batch, int32_t nd, int64_t nt, int32_t max_log2,
                                 fdmt_boxcar_t *out, double2 *mean_sd, int32_t *found, hipStream_t stream) {
  const int64_t ntiles = (nt + kBoxTile - 1) / kBoxTile;
  const int64_t count = static_cast<int64_t>(batch) * (max_log2 + 1) * nd;
  const int64_t blocks = (count * kCombineLanes + 255) / 256;
  hipLaunchKernelGGL(boxcar_combine_kernel, dim3(static_cast<unsigned>(blocks < kCombineBlocks ? blocks : kCombineBlocks)),
                     dim3(256), 0, stream, part, out, nt, static_cast<int32_t>(ntiles), count, mean_sd, found);
  return hipGetLastError();
}

hipError_t launch_boxcar_candidates(const BoxPartial *part, const double2 *mean_sd, int32_t batch, int32_t nd,
                                    int64_t nt, int32_t max_log2, float threshold, fdmt_candidate_t *cand,
                                    int32_t cap, int32_t *found, hipStream_t stream) {
  const int64_t ntiles = (nt + kBoxTile - 1) / kBoxTile;
  const int64_t count = static_cast<int64_t>(batch) * (max_log2 + 1) * nd * ntiles;
  hipLaunchKernelGGL(boxcar_candidate_kernel, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0,
                     stream, part, mean_sd, nd, static_cast<int32_t>(ntiles), max_log2, count, threshold, cand, cap,
                     found);
  return hipGetLastError();
}

hipError_t launch_boxcar(const float *plane, int32_t batch, int32_t nd, int64_t nt, int32_t max_log2,
                         fdmt_boxcar_t *out, void *ws, hipStream_t stream) {
  BoxPartial *part = static_cast<BoxPartial *>(ws);
  hipError_t e = launch_boxcar_tiles(plane, batch, nd, nt, max_log2, part, stream);
  if (e != hipSuccess) return e;
  return launch_boxcar_combine(part, batch, nd, nt, max_log2, out, nullptr, nullptr, stream);
}

} // namespace fdmt
