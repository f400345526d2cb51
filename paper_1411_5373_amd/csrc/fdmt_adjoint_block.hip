// Block passes of the adjoint transform: up to four iterations per launch, the
// first two gathered through the caches into LDS, the others from LDS.
//
// Why: a register gather of k iterations reads about 2^k leaves per output, so
// three iterations per pass (four passes at Nf = 4096) was the best it gave,
// waiting on its loads. The rows of plane m are shared by the 2^(k - k1)
// sub-bands below them: four iterations cost 4-4.5 loads and about 4 LDS reads
// per output, and planes cross HBM once per four iterations.
//
// Split: ranges of 28 rows of plane m with the few more their outputs reach,
// 64 VGPRs. A row in LDS is a window of plane l_hi, moved by the range's own
// shift, and an output row is tiled from its own offset, rounded to 128-byte
// lines: tiles that share a line write it from two workgroups, and loads and
// stores together then took twice the sum of either alone (47 and 53 us, 105 us
// both). A window of 512 samples pays for the rounding and halves the scalar
// work per sample.
//
// Measured (one MI355X, register gathers -> block passes): Nf=4096, Nt=65536,
// Nd=2048 1.33 -> 1.05 ms (3.7 TB/s of plane traffic); batch 16 of Nf=1024,
// Nt=16384, Nd=1024 2.51 -> 1.79 ms; Nf=2048, Nt=30003, Nd=1500 0.59 -> 0.35 ms;
// Nf=1000, Nt=40001, Nd=900 0.41 -> 0.28 ms. Bound by latency and issue: with
// neither loads nor stores the passes take 0.55 of their time.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fdmt_launch.h"
#include "fdmt_schedule.h"

namespace fdmt {

namespace {

// Workgroup size of a window of 256 Q samples.
constexpr int adj_threads(int q) { return 512 * q; }

struct AdjBlockArgs {
  const void *leaves1;  // AdjBlockLeaf records of the pass
  const void *places1;  // uniform batches: the same as byte offsets, branch depth in the low two bits
  const void *mids, *outs, *leaves2, *heads;
  int32_t nt, nblocks, tile;
  int32_t streaming;  // output not read again by this call: non-temporal stores
  int64_t src_stride, src_bstride, dst_stride, dst_bstride;
};

// Running sums of one row, one accumulator per tree depth, 4 Q samples: a leaf
// whose path branches off the one before at depth b closes the nodes deeper
// than b, deepest first, which is the order of the level-by-level transpose.
template <typename Tacc, int D, int Q>
struct NestedSum {
  typedef Tacc V __attribute__((ext_vector_type(4)));
  V acc[D][Q];
  __device__ __forceinline__ NestedSum() {
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[d][q] = V(0);
  }
  __device__ __forceinline__ void close(int b) {
#pragma unroll
    for (int d = D - 1; d >= 1; --d)
      if (d > b) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          acc[d - 1][q] = acc[d - 1][q] + acc[d][q];
          acc[d][q] = V(0);
        }
      }
  }
  __device__ __forceinline__ void add(const V (&v)[Q], int b) {
    close(b);
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[D - 1][q] = acc[D - 1][q] + v[q];
  }
};

// Calls f(first, count constant) over [x0, x1), B at a time and then the rest
// at once: within a call every load is issued before the first is used.
template <int B, typename F>
__device__ __forceinline__ void in_batches(int x0, int x1, F &&f) {
  int x = x0;
  for (; x + B <= x1; x += B) f(x, std::integral_constant<int, B>());
  const int rest = x1 - x;
  if constexpr (B > 3)
    if (rest == 3) f(x, std::integral_constant<int, 3>());
  if constexpr (B > 2)
    if (rest == 2) f(x, std::integral_constant<int, 2>());
  if (rest == 1) f(x, std::integral_constant<int, 1>());
}

template <typename Tacc, int D1, int D2, int Q, bool RAGGED, bool TURN>
__global__ __launch_bounds__(adj_threads(Q), 8) void adjoint_block_kernel(const Tacc *__restrict__ src,
                                                                            Tacc *__restrict__ dst, AdjBlockArgs a,
                                                                            RaggedMap rg) {
  constexpr int kWaves = adj_threads(Q) / 64;
  constexpr int kPitch = 256 * Q;
  constexpr int kBatch = 4 / Q;  // leaves at a time
  typedef Tacc V __attribute__((ext_vector_type(4)));
  typedef Tacc Vu __attribute__((ext_vector_type(4), aligned(4)));
  extern __shared__ __align__(16) unsigned char lds_raw[];
  Tacc *area = reinterpret_cast<Tacc *>(lds_raw);
  const int wave = uniform(threadIdx.x / 64), lane = threadIdx.x % 64;
  int place = blockIdx.x;
  if constexpr (TURN) {
    const int even = a.nblocks & -a.nblocks, mask = (even < 8 ? even : 8) - 1;  // even: largest power of two in it
    const int slot = place + static_cast<int>((blockIdx.y + gridDim.y * blockIdx.z) >> 4);
    place = (place & ~mask) | (slot & mask);
  }
  const int block = xcd_local_order(place, a.nblocks);
  BeamSpan bs = beam_span<RAGGED>(rg, a.nt, a.src_stride, a.src_bstride, a.dst_stride, a.dst_bstride);
  if (!RAGGED && rg.reverse) bs.tile = static_cast<int>(gridDim.y) - 1 - bs.tile;
  const int nt = bs.nt;
  const int t0 = bs.tile * a.tile;
  const Const<int32_t> head = as_const<int32_t>(a.heads) + static_cast<int64_t>(block) * kAdjBlockHeader;
  if (t0 >= nt + head[5]) return;  // past the end of every output row
  const Const<int32_t> mids = as_const<int32_t>(a.mids) + head[0];
  const Const<Int2> leaves1 = as_const<Int2>(a.leaves1);
  const Const<Int2> places1 = as_const<Int2>(a.places1);
  const Tacc *base = src + bs.src_off;
  // Stage 1: a wave per row of plane m, 4 consecutive samples per lane.
  const bool inside = t0 + kPitch + head[4] <= nt;  // every sample of every leaf inside the record
  for (int r = wave; r < head[1]; r += kWaves) {
    NestedSum<Tacc, D1, Q> sum;
    const int x0 = mids[r], x1 = mids[r + 1];
    if (inside) {
      in_batches<kBatch>(x0, x1, [&](int x, auto count) {
        constexpr int N = decltype(count)::value;
        int branch[N];
        V v[N][Q];
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const Tacc *p;  // wave-uniform
          if constexpr (RAGGED) {
            const Int2 e = leaves1[x + j];
            branch[j] = e.y & 3;
            p = base + row_offset(e.x, bs.src_stride) + (t0 + (e.y >> 2));
          } else {
            const Int2 e = places1[x + j];
            branch[j] = e.x & 3;
            const uint64_t at = static_cast<uint64_t>(static_cast<uint32_t>(e.y)) << 32 | static_cast<uint32_t>(e.x & ~3);
            p = reinterpret_cast<const Tacc *>(reinterpret_cast<const char *>(base + t0) + at);
          }
#pragma unroll
          for (int q = 0; q < Q; ++q) v[j][q] = *reinterpret_cast<const Vu *>(p + 256 * q + 4 * lane);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) sum.add(v[j], branch[j]);
      });
    } else {
      for (int x = x0; x < x1; ++x) {
        const Int2 e = leaves1[x];
        const Tacc *p = base + row_offset(e.x, bs.src_stride);
        const int ts = t0 + 4 * lane + (e.y >> 2);
        V v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int t = ts + 256 * q + i;
            const Tacc z = p[t < nt ? t : nt - 1];
            v[q][i] = t < nt ? z : Tacc(0);
          }
        sum.add(v, e.y & 3);
      }
    }
    sum.close(0);
#pragma unroll
    for (int q = 0; q < Q; ++q) *reinterpret_cast<V *>(area + r * kPitch + 256 * q + 4 * lane) = sum.acc[0][q];
  }
  __syncthreads();
  // Stage 2: a wave per output row, columns lane, lane + 64, ...
  const Const<Int4> outs = as_const<Int4>(a.outs) + head[2];
  const Const<int32_t> leaves2 = as_const<int32_t>(a.leaves2);
  for (int r = wave; r < head[3]; r += kWaves) {
    const Int4 o = outs[r];  // {first leaf, last, row, offset}
    NestedSum<Tacc, D2, Q> sum;
    in_batches<kBatch>(o.x, o.y, [&](int x, auto count) {
      constexpr int N = decltype(count)::value;
      int branch[N];
      V v[N][Q];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const int e = leaves2[x + j];
        branch[j] = e & 3;
        const Tacc *p = reinterpret_cast<const Tacc *>(lds_raw + (e & ~3)) + lane;
#pragma unroll
        for (int c = 0; c < 4 * Q; ++c) v[j][c / 4][c % 4] = p[64 * c];
      }
#pragma unroll
      for (int j = 0; j < N; ++j) sum.add(v[j], branch[j]);
    });
    sum.close(0);
    const int ts = t0 - o.w;  // first sample of the window in this row
    const int from = ts < 0 ? -ts : 0;
    const int to = nt - ts < a.tile ? nt - ts : a.tile;
    Tacc *d = dst + bs.dst_off + o.z * bs.dst_stride + ts;
#pragma unroll
    for (int c = 0; c < 4 * Q; ++c) {
      const int col = 64 * c + lane;
      if (col >= from && col < to) {
        if (a.streaming)
          __builtin_nontemporal_store(sum.acc[0][c / 4][c % 4], d + col);
        else
          d[col] = sum.acc[0][c / 4][c % 4];
      }
    }
  }
}

} // namespace

size_t adjoint_block_lds_bytes(const AdjPass &ps) {
  // an output's columns past the tile are read from up to 128 samples past the last row
  return static_cast<size_t>(ps.rows_mid) * ps.pitch * 4 + 512;
}

template <typename Tacc>
hipError_t launch_adjoint_block(const AdjBlockLaunch &g, const Tacc *src, Tacc *dst) {
  const AdjPass &ps = *g.pass;
  // Blocks are unequal work, and a few of them whose number shares a factor with
  // the 8 XCDs would run on the same XCDs in every tile: they change places every
  // 16 tiles (64 beams of Nf=100, Nt=700, Nd=100 87 -> 55 us, 200 of Nf=50,
  // Nt=1000, Nd=100 145 -> 127 us, Nf=64, Nt=100000, Nd=200 174 -> 149 us). With
  // more blocks an XCD has several, and handing them on gained nothing or cost
  // up to 8%; the test for it in the code cost 1% of short windows.
  const bool turn = ps.nblocks <= 32 && ps.nblocks % 2 == 0 && g.grid.y * g.grid.z >= 128;
  AdjBlockArgs a{g.leaves1, g.places1, g.mids, g.outs, g.leaves2, g.heads, g.nt, ps.nblocks, ps.tile, g.streaming,
                 g.src_stride, g.src_bstride, g.dst_stride, g.dst_bstride};
  const size_t lds = adjoint_block_lds_bytes(ps);
#define FDMT_ADJ_LAUNCH(A, B, QQ, R, T)                                                                           \
  hipLaunchKernelGGL((adjoint_block_kernel<Tacc, A, B, QQ, R, T>), g.grid, dim3(adj_threads(QQ)), lds, g.stream,  \
                     src, dst, a, g.rg)
#define FDMT_ADJ_BLOCK(A, B, QQ)                                                                                  \
  if (ps.k1 == A && ps.depth2 == B && ps.pitch == 256 * QQ) {                                                     \
    if (g.ragged && turn)                                                                                         \
      FDMT_ADJ_LAUNCH(A, B, QQ, true, true);                                                                      \
    else if (g.ragged)                                                                                            \
      FDMT_ADJ_LAUNCH(A, B, QQ, true, false);                                                                     \
    else if (turn)                                                                                                \
      FDMT_ADJ_LAUNCH(A, B, QQ, false, true);                                                                     \
    else                                                                                                          \
      FDMT_ADJ_LAUNCH(A, B, QQ, false, false);                                                                    \
    return hipGetLastError();                                                                                     \
  }
#define FDMT_ADJ_BLOCKS(F) F(1, 1, 1) F(1, 2, 1) F(2, 1, 1) F(2, 2, 1) F(2, 3, 1) F(1, 1, 2) F(1, 2, 2) F(2, 1, 2) F(2, 2, 2) F(2, 3, 2)
  FDMT_ADJ_BLOCKS(FDMT_ADJ_BLOCK)
#undef FDMT_ADJ_BLOCK
#undef FDMT_ADJ_LAUNCH
  return hipErrorInvalidValue;
}

hipError_t prepare_adjoint_blocks() {
  const int lds = kAdjBlockRows * 512 * 4 + 512;
#define FDMT_ADJ_KERNEL(...) reinterpret_cast<const void *>(&adjoint_block_kernel<__VA_ARGS__>),
#define FDMT_ADJ_FN(A, B, QQ)                                                                                     \
  FDMT_ADJ_KERNEL(float, A, B, QQ, false, false) FDMT_ADJ_KERNEL(float, A, B, QQ, false, true)                    \
  FDMT_ADJ_KERNEL(float, A, B, QQ, true, false) FDMT_ADJ_KERNEL(float, A, B, QQ, true, true)                      \
  FDMT_ADJ_KERNEL(int32_t, A, B, QQ, false, false) FDMT_ADJ_KERNEL(int32_t, A, B, QQ, false, true)                \
  FDMT_ADJ_KERNEL(int32_t, A, B, QQ, true, false) FDMT_ADJ_KERNEL(int32_t, A, B, QQ, true, true)
  const void *fns[] = {FDMT_ADJ_BLOCKS(FDMT_ADJ_FN)};
#undef FDMT_ADJ_FN
#undef FDMT_ADJ_KERNEL
#undef FDMT_ADJ_BLOCKS
  for (const void *f : fns) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template hipError_t launch_adjoint_block<float>(const AdjBlockLaunch &, const float *, float *);
template hipError_t launch_adjoint_block<int32_t>(const AdjBlockLaunch &, const int32_t *, int32_t *);

} // namespace fdmt
