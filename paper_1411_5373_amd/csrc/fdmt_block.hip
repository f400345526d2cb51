// Block passes of the forward transform: up to six iterations per launch, the
// first two loaded through the caches, the others from LDS.
//
// Why: a register gather of k iterations loads 2^k terms per output sample, so
// the address unit, not HBM, bounds it, and three iterations per pass (four
// passes at Nf = 4096) was the best it gave. A block of 16 rows shares its
// tree: six iterations need 31 rows of 4 loads (7.75 loads per output, as many
// as three iterations of a register gather), then two rounds of four LDS reads.
// Planes cross HBM once per five or six iterations instead of three.
//
// Split: rows of at most 16 (six iterations: 52 KiB of LDS, three workgroups
// per CU) or 18 (24-26 KiB, four); a tile of 224 samples, 256 less the spread
// of the block's shifts rounded to whole 128-byte lines (tiles rounded to 4
// samples were 4-6% slower); 64 VGPRs for eight waves per SIMD, so two rows'
// loads at a time (four rows' were 5-70% slower). From the input a workgroup
// runs two tiles, its tables then in the scalar cache (7-10% faster; planes
// are no faster, and four or eight tiles slower).
//
// Measured (one MI355X, register gathers -> block passes): Nf=4096, Nt=65536,
// Nd=2048 uint8 0.776 -> 0.53-0.57 ms, FP32 1.238 -> 0.85-0.90 ms; batch 16 of
// Nf=1024, Nt=16384, Nd=1024 FP32 2.120 -> 1.23 ms (3.5 TB/s of plane
// traffic); Nf=1000, Nt=40001, Nd=900 uint8 0.240 -> 0.096 ms; Nf=64, Nt=1024,
// Nd=64 FP32 0.023 -> 0.007 ms (one launch). What bounds a pass now is its
// instruction stream and the latency between its stages: without loads and
// stores a six-iteration pass of the first workload still takes 0.18 ms, its
// loads and stores add 0.1 ms each.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fdmt_launch.h"

namespace fdmt {

namespace {

constexpr int kBlockThreads = 512;
constexpr int kBlockWaves = kBlockThreads / 64;

template <typename T>
using Acc4 = T __attribute__((ext_vector_type(4)));

// The value of x in the lane before (lane 0: its own, not used) and in the
// lane after (lane 63: its own, not used).
template <typename T>
__device__ __forceinline__ T lane_before(T x) {
  const int i = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(i, i, 0x138, 0xf, 0xf, false));  // wave_shr:1
}
template <typename T>
__device__ __forceinline__ T lane_after(T x) {
  const int i = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(i, i, 0x130, 0xf, 0xf, false));  // wave_shl:1
}

// Four consecutive samples per lane from a wave-uniform address. Types
// narrower than a word come as the aligned words that hold a lane's samples;
// the samples past them are the next lane's, so the last kBlockTail columns
// of a row are not used.
template <typename T>
struct Quad {  // 4-byte types
  typedef T Raw __attribute__((ext_vector_type(4), aligned(4)));
  static __device__ __forceinline__ Raw load(const T *p, int lane) { return *reinterpret_cast<const Raw *>(p + 4 * lane); }
  template <typename Tacc>
  static __device__ __forceinline__ Acc4<Tacc> expand(Raw r, const T *) {
    return __builtin_convertvector(r, Acc4<Tacc>);
  }
};
template <typename T>
struct QuadHalf {  // 2-byte types
  typedef uint32_t Raw __attribute__((ext_vector_type(2), aligned(4)));
  static __device__ __forceinline__ Raw load(const T *p, int lane) {
    const char *q = reinterpret_cast<const char *>(p) - (reinterpret_cast<uintptr_t>(p) & 3);
    return *reinterpret_cast<const Raw *>(q + 8 * lane);
  }
  template <typename Tacc>
  static __device__ __forceinline__ Acc4<Tacc> expand(Raw r, const T *p) {
    const uint32_t mis = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p)) & 3;
    const uint32_t x[2] = {__builtin_amdgcn_alignbyte(r[1], r[0], mis),
                           __builtin_amdgcn_alignbyte(lane_after(r[0]), r[1], mis)};
    Acc4<Tacc> v;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      v[i] = widen<Tacc>(__builtin_bit_cast(T, static_cast<uint16_t>(i & 1 ? x[i / 2] >> 16 : x[i / 2] & 0xffffu)));
    return v;
  }
};
template <>
struct Quad<uint16_t> : QuadHalf<uint16_t> {};
template <>
struct Quad<_Float16> : QuadHalf<_Float16> {};
template <>
struct Quad<uint8_t> {
  typedef uint32_t Raw;
  static __device__ __forceinline__ Raw load(const uint8_t *p, int lane) {
    const uint8_t *q = p - (reinterpret_cast<uintptr_t>(p) & 3);
    return *reinterpret_cast<const Raw *>(q + 4 * lane);
  }
  // the four bytes in a word
  static __device__ __forceinline__ uint32_t word(Raw r, const uint8_t *p) {
    return __builtin_amdgcn_alignbyte(lane_after(r), r, static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p)) & 3);
  }
  template <typename Tacc>
  static __device__ __forceinline__ Acc4<Tacc> expand(Raw r, const uint8_t *p) {
    const uint32_t x = word(r, p);
    return Acc4<Tacc>{static_cast<Tacc>(x & 0xffu), static_cast<Tacc>((x >> 8) & 0xffu),
                      static_cast<Tacc>((x >> 16) & 0xffu), static_cast<Tacc>(x >> 24)};
  }
};

struct BlockArgs {
  const void *terms;   // Term (from a plane) or InTerm (from the input) records of the pass
  const void *places;  // uniform batches: the same records, {row, shift} as the byte offset of the term's place
  const int32_t *offs, *heads;
  int32_t nt, nblocks, tile, rows_a;
  int32_t tiles_per_wg;  // consecutive time tiles of a workgroup
  int32_t streaming;  // output not read again by this call: non-temporal stores
  int32_t turn;       // uniform: see xcd_turned_order(); ragged: blocks that change places, less 1
  int64_t src_stride, src_bstride, dst_stride, dst_bstride;
};

// Sums v[0..N-1] into v[0] as the recursion does: sibling pairs first, then
// pairs of pairs, lower half before upper half.
template <int N, typename V>
__device__ __forceinline__ void tree_sum(V (&v)[N]) {
#pragma unroll
  for (int span = 1; span < N; span *= 2)
#pragma unroll
    for (int j = 0; j < N; j += 2 * span) v[j] = v[j] + v[j + span];
}

// Calls f(row, batch size constant) for the wave's rows wave, wave + 8, ...
// below `rows`: batches of B rows kBlockWaves apart while a whole one is left,
// then of half as many. A batch has no conditions inside, so all its loads are
// issued before the first is waited for.
template <int B, typename F>
__device__ __forceinline__ void row_batches(int wave, int rows, F &&f) {
  int r = wave;
  for (; r + (B - 1) * kBlockWaves < rows; r += B * kBlockWaves) f(r, std::integral_constant<int, B>());
  if constexpr (B > 2)
    if (r + (B / 2 - 1) * kBlockWaves < rows) {
      f(r, std::integral_constant<int, B / 2>());
      r += B / 2 * kBlockWaves;
    }
  if constexpr (B > 1)
    for (; r < rows; r += kBlockWaves) f(r, std::integral_constant<int, 1>());
}

// Rows r, r + kBlockWaves, ... (RU of them) as tree sums of 2^K rows of an LDS
// area; a lane takes columns lane, lane + 64, lane + 128 and lane + 192.
template <typename Tacc, int K, int RU>
__device__ __forceinline__ void lds_rows(Acc4<Tacc> (&out)[RU], const Tacc *area, Const<int32_t> off, int r, int lane) {
  constexpr int N = 1 << K;
  int o[RU][N];
#pragma unroll
  for (int u = 0; u < RU; ++u)
#pragma unroll
    for (int j = 0; j < N; ++j) o[u][j] = off[(r + u * kBlockWaves) * N + j];
  Acc4<Tacc> v[RU][N];
#pragma unroll
  for (int u = 0; u < RU; ++u)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const Tacc *p = area + o[u][j] + lane;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[u][j][c] = p[64 * c];
    }
#pragma unroll
  for (int u = 0; u < RU; ++u) {
    tree_sum(v[u]);
    out[u] = v[u][0];
  }
}

template <typename Tsrc, typename Tacc, typename Tdst, bool FROM_INPUT, int K1, int K2, int K3, bool RAGGED>
__global__ __launch_bounds__(kBlockThreads, 8) void block_pass_kernel(const Tsrc *__restrict__ src,
                                                                   Tdst *__restrict__ dst, BlockArgs a,
                                                                   RaggedMap rg) {
  typedef Acc4<Tacc> V;
  typedef Quad<Tsrc> Q;
  typedef typename std::conditional<FROM_INPUT, Int4, Int2>::type Rec;  // {row, shift} or {channel, shift, chain}
  constexpr int N1 = 1 << K1;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  Tacc *area_a = reinterpret_cast<Tacc *>(lds_raw);
  Tacc *area_b = area_a + a.rows_a * kBlockPitch;
  const int wave = uniform(threadIdx.x / 64), lane = threadIdx.x % 64;
  int place = blockIdx.x;
  if constexpr (RAGGED) place = (place & ~a.turn) | ((place + static_cast<int>(blockIdx.y >> 4)) & a.turn);
  const int block = FROM_INPUT && !RAGGED ? xcd_turned_order(place, a.nblocks, a.turn)
                                          : xcd_local_order(place, a.nblocks);
  BeamSpan bs = beam_span<RAGGED>(rg, a.nt, a.src_stride, a.src_bstride, a.dst_stride, a.dst_bstride);
  if (!RAGGED && rg.reverse) bs.tile = static_cast<int>(gridDim.y) - 1 - bs.tile;
  const int nt = bs.nt;
  const Const<int32_t> head = as_const<int32_t>(a.heads) + static_cast<int64_t>(block) * kBlockHeader;
  const Const<int32_t> offs = as_const<int32_t>(a.offs);
  const Tsrc *base = src + bs.src_off;
  const Const<Rec> terms = as_const<Rec>(a.terms) + head[0];
  const Const<Rec> places = as_const<Rec>(a.places) + head[0];
  // Option-1 chain of a term from its four samples: the samples before them
  // are the neighbour lane's (lane 0 has none: the first kBlockLead columns of
  // a row are not used).
  const auto add_chain = [](V &v, int chain) {
    if (chain > 0) {
      const V u = v;
      V prev;
#pragma unroll
      for (int i = 0; i < 4; ++i) prev[i] = lane_before(u[i]);
      v = u + V{prev[3], u[0], u[1], u[2]};
      if (chain > 1) v = v + V{prev[2], prev[3], u[0], u[1]};
      if (chain > 2) v = v + V{prev[1], prev[2], prev[3], u[0]};
      if (chain > 3) v = v + prev;
    }
  };
  // Stage 1: a wave per row of area A, 4 consecutive samples per lane. The
  // aligned words of a narrow type may start 3 bytes before a term's samples:
  // in a buffer that is not word-aligned, those have to be the row's.
  const int room = sizeof(Tsrc) < 4 && (reinterpret_cast<uintptr_t>(src) & 3) != 0 ? 4 : 0;
  const int tiles = FROM_INPUT ? a.tiles_per_wg : 1;
  int t0 = bs.tile * tiles * a.tile;
  for (int tile = 0; tile < tiles && t0 < nt; ++tile, t0 += a.tile) {
  if (K2 == 0 && tile > 0) __syncthreads();  // stage 3 of the tile before has read area A
  // rows of which every sample of every term lies inside the record
  const int fast = t0 - room >= head[7] && t0 + kBlockPitch <= nt ? head[8] : 0;
  if (fast > 0) {
    row_batches<8 / N1>(wave, fast, [&](int r, auto batch) {
      constexpr int RU = decltype(batch)::value;
      const Tsrc *p[RU][N1];  // wave-uniform
      int chain[RU][N1];
#pragma unroll
      for (int u = 0; u < RU; ++u)
#pragma unroll
        for (int j = 0; j < N1; ++j) {
          const int i = (r + u * kBlockWaves) * N1 + j;
          if constexpr (RAGGED) {
            const Rec e = terms[i];
            p[u][j] = base + row_offset(e.x, bs.src_stride) + (t0 - e.y);
            if constexpr (FROM_INPUT) chain[u][j] = e.z;
          } else {
            const Rec e = places[i];
            const uint64_t at = static_cast<uint64_t>(static_cast<uint32_t>(e.y)) << 32 | static_cast<uint32_t>(e.x);
            p[u][j] = reinterpret_cast<const Tsrc *>(reinterpret_cast<const char *>(base + t0) + static_cast<int64_t>(at));
            if constexpr (FROM_INPUT) chain[u][j] = e.z;
          }
        }
      typename Q::Raw x[RU][N1];
#pragma unroll
      for (int u = 0; u < RU; ++u)
#pragma unroll
        for (int j = 0; j < N1; ++j) x[u][j] = Q::load(p[u][j], lane);
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        V sum;
        if constexpr (FROM_INPUT && std::is_same<Tsrc, uint8_t>::value && std::is_same<Tacc, int32_t>::value) {
          // integer sums of bytes in any order: two 16-bit sums per word
          // (at most 2^K1 = 4 chains of 5 bytes), samples 0 and 2, and 1 and 3
          uint32_t even = 0, odd = 0;
#pragma unroll
          for (int j = 0; j < N1; ++j) {
            const uint32_t w = Q::word(x[u][j], p[u][j]);
            even += w & 0x00ff00ffu;
            odd += (w >> 8) & 0x00ff00ffu;
            if (chain[u][j] > 0) {
              const uint32_t before = lane_before(w);
              for (int d = 1; d <= chain[u][j]; ++d) {
                const uint32_t y = d < 4 ? __builtin_amdgcn_alignbyte(w, before, 4 - d) : before;
                even += y & 0x00ff00ffu;
                odd += (y >> 8) & 0x00ff00ffu;
              }
            }
          }
          sum = V{static_cast<Tacc>(even & 0xffffu), static_cast<Tacc>(odd & 0xffffu), static_cast<Tacc>(even >> 16),
                  static_cast<Tacc>(odd >> 16)};
        } else {
          V v[N1];
#pragma unroll
          for (int j = 0; j < N1; ++j) {
            v[j] = Q::template expand<Tacc>(x[u][j], p[u][j]);
            if constexpr (FROM_INPUT) add_chain(v[j], chain[u][j]);
          }
          tree_sum(v);
          sum = v[0];
        }
        *reinterpret_cast<V *>(area_a + (r + u * kBlockWaves) * kBlockPitch + 4 * lane) = sum;
      }
    });
  }
  {
    // record edges and rows with missing channels: each sample from its clamped
    // place, zero before the record (past it the value does not matter: no sample
    // before nt sums it)
    for (int r = fast + wave; r < head[1]; r += kBlockWaves) {
      V v[N1];
#pragma unroll
      for (int j = 0; j < N1; ++j) {
        const Rec e = terms[r * N1 + j];
        const Tsrc *p = base + row_offset(e.x, bs.src_stride);
        const int ts = t0 - e.y + 4 * lane;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = ts + i < 0 ? 0 : ts + i < nt ? ts + i : nt - 1;
          const Tacc x = widen<Tacc>(p[t]);
          v[j][i] = ts + i >= 0 ? x : Tacc(0);
        }
        if constexpr (FROM_INPUT) add_chain(v[j], e.z);
      }
      tree_sum(v);
      *reinterpret_cast<V *>(area_a + r * kBlockPitch + 4 * lane) = v[0];
    }
  }
  __syncthreads();
  const Tacc *last = area_a;
  if constexpr (K2 > 0) {
    row_batches<1>(wave, head[3], [&](int r, auto batch) {
      constexpr int RU = decltype(batch)::value;
      V v[RU];
      lds_rows<Tacc, K2>(v, area_a, offs + head[2], r, lane);
#pragma unroll
      for (int u = 0; u < RU; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) area_b[(r + u * kBlockWaves) * kBlockPitch + 64 * c + lane] = v[u][c];
    });
    __syncthreads();
    last = area_b;
  }
  Tdst *out = dst + bs.dst_off + head[6] * bs.dst_stride + t0;
  const int valid = nt - t0 < a.tile ? nt - t0 : a.tile;
  row_batches<1>(wave, head[5], [&](int r, auto batch) {
    constexpr int RU = decltype(batch)::value;
    V v[RU];
    lds_rows<Tacc, K3>(v, last, offs + head[4], r, lane);
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      Tdst *o = out + (r + u * kBlockWaves) * bs.dst_stride;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (64 * c + lane < valid) {
          const Tdst x = static_cast<Tdst>(v[u][c]);
          if (a.streaming)
            __builtin_nontemporal_store(x, o + 64 * c + lane);
          else
            o[64 * c + lane] = x;
        }
      }
    }
  });
  }
}

// The same for a first pass from uint8 input whose sums all stay below 2^16:
// LDS holds two samples per word (no half carries into the other), a row is 512
// samples, and one addition, LDS access and store serves two, for a kernel that
// its instructions bound. A lane loads 8 samples. A stage-2 or -3 term at an odd
// column takes each word's halves from two words, so five iterations go through
// LDS twice (eight such terms at a time were 14% slower). Measured: the first
// pass of Nf=4096, Nt=65536, Nd=2048 0.287 -> 0.219 ms, of four beams of Nf=128,
// Nt=50000 40 -> 28 us, of Nf=1000, Nt=40001 55 -> 50 us.
template <int K>
__device__ __forceinline__ void packed_terms(uint32_t (&out)[4], const uint32_t *area, Const<int32_t> off, int lane) {
  constexpr int N = 1 << K;
  int o[N];
  uint32_t v[N][4], w[N][4];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    o[j] = off[j];
    const uint32_t *p = area + (o[j] >> 1) + lane;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[j][c] = p[64 * c];
  }
#pragma unroll
  for (int j = 0; j < N; ++j)
    if (o[j] & 1) {
      const uint32_t *p = area + (o[j] >> 1) + 1 + lane;
#pragma unroll
      for (int c = 0; c < 4; ++c) w[j][c] = p[64 * c];
    }
#pragma unroll
  for (int c = 0; c < 4; ++c) out[c] = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if (o[j] & 1) {
#pragma unroll
      for (int c = 0; c < 4; ++c) v[j][c] = __builtin_amdgcn_alignbyte(w[j][c], v[j][c], 2);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) out[c] += v[j][c];
  }
}

template <typename Tdst, int K1, int K2, int K3, bool RAGGED>
__global__ __launch_bounds__(kBlockThreads, 8) void packed_block_kernel(const uint8_t *__restrict__ src,
                                                                     Tdst *__restrict__ dst, BlockArgs a,
                                                                     RaggedMap rg) {
  constexpr int N1 = 1 << K1;
  constexpr int kPitch = 2 * kBlockPitch, kWords = kBlockPitch;  // samples and words per LDS row
  typedef uint32_t Words2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef uint32_t Words4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) unsigned char lds_raw[];
  uint32_t *area_a = reinterpret_cast<uint32_t *>(lds_raw);
  uint32_t *area_b = area_a + a.rows_a * kWords;
  const int wave = uniform(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int block = xcd_local_order(blockIdx.x, a.nblocks);
  BeamSpan bs = beam_span<RAGGED>(rg, a.nt, a.src_stride, a.src_bstride, a.dst_stride, a.dst_bstride);
  if (!RAGGED && rg.reverse) bs.tile = static_cast<int>(gridDim.y) - 1 - bs.tile;
  const int nt = bs.nt;
  const Const<int32_t> head = as_const<int32_t>(a.heads) + static_cast<int64_t>(block) * kBlockHeader;
  const Const<int32_t> offs = as_const<int32_t>(a.offs);
  const uint8_t *base = src + bs.src_off;
  const Const<Int4> terms = as_const<Int4>(a.terms) + head[0];
  const Const<Int4> places = as_const<Int4>(a.places) + head[0];
  // Adds a term's chain: w0 and w1 hold a lane's samples 0-3 and 4-7, the four
  // before them are the neighbour lane's. even: samples 0, 2 and 4, 6; odd the
  // others, one per half word.
  const auto add_chain = [](uint32_t (&even)[2], uint32_t (&odd)[2], uint32_t w0, uint32_t w1, int chain) {
    even[0] += w0 & 0x00ff00ffu;
    odd[0] += (w0 >> 8) & 0x00ff00ffu;
    even[1] += w1 & 0x00ff00ffu;
    odd[1] += (w1 >> 8) & 0x00ff00ffu;
    if (chain > 0) {
      const uint32_t before = lane_before(w1);
      for (int d = 1; d <= chain; ++d) {
        const uint32_t y0 = d < 4 ? __builtin_amdgcn_alignbyte(w0, before, 4 - d) : before;
        const uint32_t y1 = d < 4 ? __builtin_amdgcn_alignbyte(w1, w0, 4 - d) : w0;
        even[0] += y0 & 0x00ff00ffu;
        odd[0] += (y0 >> 8) & 0x00ff00ffu;
        even[1] += y1 & 0x00ff00ffu;
        odd[1] += (y1 >> 8) & 0x00ff00ffu;
      }
    }
  };
  const auto put_row = [&](int r, const uint32_t (&even)[2], const uint32_t (&odd)[2]) {
    *reinterpret_cast<Words4 *>(area_a + r * kWords + 4 * lane) =
        Words4{__builtin_amdgcn_perm(odd[0], even[0], 0x05040100u), __builtin_amdgcn_perm(odd[0], even[0], 0x07060302u),
               __builtin_amdgcn_perm(odd[1], even[1], 0x05040100u), __builtin_amdgcn_perm(odd[1], even[1], 0x07060302u)};
  };
  // the aligned words may start 3 bytes before a term's samples: see block_pass_kernel
  const int room = (reinterpret_cast<uintptr_t>(src) & 3) != 0 ? 4 : 0;
  int t0 = bs.tile * a.tiles_per_wg * a.tile;
  for (int tile = 0; tile < a.tiles_per_wg && t0 < nt; ++tile, t0 += a.tile) {
    if (K2 == 0 && tile > 0) __syncthreads();
    const int fast = t0 - room >= head[7] && t0 + kPitch <= nt ? head[8] : 0;
    if (fast > 0) {
      row_batches<8 / N1>(wave, fast, [&](int r, auto batch) {
        constexpr int RU = decltype(batch)::value;
        int mis[RU][N1], chain[RU][N1];
        Words2 x[RU][N1];
#pragma unroll
        for (int u = 0; u < RU; ++u)
#pragma unroll
          for (int j = 0; j < N1; ++j) {
            const int i = (r + u * kBlockWaves) * N1 + j;
            const uint8_t *p;  // wave-uniform
            if constexpr (RAGGED) {
              const Int4 e = terms[i];
              p = base + row_offset(e.x, bs.src_stride) + (t0 - e.y);
              chain[u][j] = e.z;
            } else {
              const Int4 e = places[i];
              const uint64_t at = static_cast<uint64_t>(static_cast<uint32_t>(e.y)) << 32 | static_cast<uint32_t>(e.x);
              p = base + t0 + static_cast<int64_t>(at);
              chain[u][j] = e.z;
            }
            mis[u][j] = static_cast<int>(reinterpret_cast<uintptr_t>(p) & 3);
            x[u][j] = *reinterpret_cast<const Words2 *>(p - mis[u][j] + 8 * lane);
          }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          uint32_t even[2] = {0, 0}, odd[2] = {0, 0};
#pragma unroll
          for (int j = 0; j < N1; ++j) {
            const uint32_t m = static_cast<uint32_t>(mis[u][j]);
            add_chain(even, odd, __builtin_amdgcn_alignbyte(x[u][j][1], x[u][j][0], m),
                      __builtin_amdgcn_alignbyte(lane_after(x[u][j][0]), x[u][j][1], m), chain[u][j]);
          }
          put_row(r + u * kBlockWaves, even, odd);
        }
      });
    }
    {
      for (int r = fast + wave; r < head[1]; r += kBlockWaves) {
        uint32_t even[2] = {0, 0}, odd[2] = {0, 0};
        for (int j = 0; j < N1; ++j) {
          const Int4 e = terms[r * N1 + j];
          const uint8_t *p = base + row_offset(e.x, bs.src_stride);
          const int ts = t0 - e.y + 8 * lane;
          uint32_t w[2] = {0, 0};
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int t = ts + i < 0 ? 0 : ts + i < nt ? ts + i : nt - 1;
            const uint32_t z = p[t];
            w[i / 4] |= (ts + i >= 0 ? z : 0u) << (8 * (i % 4));
          }
          add_chain(even, odd, w[0], w[1], e.z);
        }
        put_row(r, even, odd);
      }
    }
    __syncthreads();
    const uint32_t *last = area_a;
    if constexpr (K2 > 0) {
      for (int r = wave; r < head[3]; r += kBlockWaves) {
        uint32_t v[4];
        packed_terms<K2>(v, area_a, offs + head[2] + r * (1 << K2), lane);
#pragma unroll
        for (int c = 0; c < 4; ++c) area_b[r * kWords + 64 * c + lane] = v[c];
      }
      __syncthreads();
      last = area_b;
    }
    const int valid = nt - t0 < a.tile ? nt - t0 : a.tile;
    for (int r = wave; r < head[5]; r += kBlockWaves) {
      uint32_t v[4];
      packed_terms<K3>(v, last, offs + head[4] + r * (1 << K3), lane);
      Tdst *o = dst + bs.dst_off + (head[6] + r) * bs.dst_stride + t0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int col = 128 * c + 2 * lane;
        if (col + 1 < valid) {
          if constexpr (sizeof(Tdst) == 2) {
            *reinterpret_cast<uint32_t *>(o + col) = v[c];  // plane rows and tiles start on words
          } else {
            typedef Tdst D2 __attribute__((ext_vector_type(2), aligned(4)));
            const D2 d = {static_cast<Tdst>(v[c] & 0xffffu), static_cast<Tdst>(v[c] >> 16)};
            __builtin_nontemporal_store(d, reinterpret_cast<D2 *>(o + col));
          }
        } else if (col < valid) {
          o[col] = static_cast<Tdst>(v[c] & 0xffffu);
        }
      }
    }
  }
}

} // namespace

size_t block_lds_bytes(const Pass &ps) {
  // a row's columns past its width are computed from up to kBlockPitch samples past the area
  return static_cast<size_t>(ps.rows_a + ps.rows_b + 1) * kBlockPitch * 4;
}

template <typename Tsrc, typename Tacc, typename Tdst, bool FROM_INPUT>
hipError_t launch_block(const BlockLaunch &g, const Tsrc *src, Tdst *dst) {
  const Pass &ps = *g.pass;
  BlockArgs a{};
  a.terms = g.terms;
  a.places = g.places;
  a.offs = g.offs;
  a.heads = g.heads;
  a.nt = g.nt;
  a.nblocks = ps.nblocks;
  a.tile = ps.tile;
  a.tiles_per_wg = ps.tiles_per_wg;
  // Uniform batches from the input, where blocks of many sub-bands run over many
  // tiles, move on every 16 tiles: Nf=4096, Nt=65536 FP32 0.468 -> 0.447 ms, batch
  // 16 of Nf=1024, Nt=16384 0.652 -> 0.619 ms. Every tile or every 4 loses the
  // L2's overlap of neighbouring tiles (0.466, 0.450 ms). A pass from a plane
  // reads most of it again in the next tile and got slower (up to 8%, with the
  // test alone in its code 5%), packed and ragged passes gained nothing.
  // Ragged batches of a few blocks whose number shares a factor with the 8 XCDs
  // hand them on too: 500 beams of 30 to 800 samples, Nf=256, Nd=128 FP32 301 -> 258 us,
  // 60 of 500 to 5000, Nf=1024, Nd=300 355 -> 317 us.
  const int even = ps.nblocks & -ps.nblocks;  // largest power of two in it
  if (g.ragged) a.turn = !ps.packed && ps.nblocks <= 32 ? (even < 8 ? even : 8) - 1 : 0;
  else
    a.turn = FROM_INPUT && !ps.packed && ps.nblocks % 8 == 0 && ps.nblocks >= 64 && g.grid.y * g.grid.z >= 128 ? 4 : 0;
  a.rows_a = ps.rows_a;
  a.streaming = g.streaming;
  a.src_stride = g.src_stride;
  a.src_bstride = g.src_bstride;
  a.dst_stride = g.dst_stride;
  a.dst_bstride = g.dst_bstride;
  const size_t lds = block_lds_bytes(ps);
  if (lds > 64 * 1024) return hipErrorInvalidValue;
  // uint8 input into integer sums that all fit 16 bits
  constexpr bool kBytes = FROM_INPUT && std::is_same<Tsrc, uint8_t>::value && std::is_same<Tacc, int32_t>::value;
  if (ps.packed) {
    if constexpr (kBytes) {
#define FDMT_PACKED(A, B, C)                                                                                       \
  if (ps.k1 == A && ps.k2 == B && ps.k3 == C) {                                                                    \
    if (g.ragged)                                                                                                  \
      hipLaunchKernelGGL((packed_block_kernel<Tdst, A, B, C, true>), g.grid, dim3(kBlockThreads), lds, g.stream,   \
                         src, dst, a, g.rg);                                                                       \
    else                                                                                                           \
      hipLaunchKernelGGL((packed_block_kernel<Tdst, A, B, C, false>), g.grid, dim3(kBlockThreads), lds, g.stream,  \
                         src, dst, a, g.rg);                                                                       \
    return hipGetLastError();                                                                                      \
  }
      FDMT_PACKED(1, 0, 2)
      FDMT_PACKED(2, 0, 2)
      FDMT_PACKED(2, 1, 2)
      FDMT_PACKED(2, 2, 2)
#undef FDMT_PACKED
    }
    return hipErrorInvalidValue;
  }
#define FDMT_BLOCK(A, B, C)                                                                                        \
  if (ps.k1 == A && ps.k2 == B && ps.k3 == C) {                                                                    \
    if (g.ragged)                                                                                                  \
      hipLaunchKernelGGL((block_pass_kernel<Tsrc, Tacc, Tdst, FROM_INPUT, A, B, C, true>), g.grid,                 \
                         dim3(kBlockThreads), lds, g.stream, src, dst, a, g.rg);                                   \
    else                                                                                                           \
      hipLaunchKernelGGL((block_pass_kernel<Tsrc, Tacc, Tdst, FROM_INPUT, A, B, C, false>), g.grid,                \
                         dim3(kBlockThreads), lds, g.stream, src, dst, a, g.rg);                                   \
    return hipGetLastError();                                                                                      \
  }
  FDMT_BLOCK(1, 0, 2)
  FDMT_BLOCK(2, 0, 2)
  FDMT_BLOCK(2, 0, 3)
  FDMT_BLOCK(2, 2, 2)
#undef FDMT_BLOCK
  return hipErrorInvalidValue;
}

#define FDMT_BLOCK_INST(TS, TA, TD, IN) \
  template hipError_t launch_block<TS, TA, TD, IN>(const BlockLaunch &, const TS *, TD *);
FDMT_BLOCK_INST(float, float, float, true)
FDMT_BLOCK_INST(_Float16, float, float, true)
FDMT_BLOCK_INST(uint8_t, int32_t, uint16_t, true)
FDMT_BLOCK_INST(uint8_t, int32_t, float, true)
FDMT_BLOCK_INST(uint8_t, int32_t, int32_t, true)
FDMT_BLOCK_INST(uint8_t, float, float, true)
FDMT_BLOCK_INST(int32_t, int32_t, int32_t, true)
FDMT_BLOCK_INST(float, float, float, false)
FDMT_BLOCK_INST(int32_t, int32_t, int32_t, false)
FDMT_BLOCK_INST(uint16_t, int32_t, uint16_t, false)
FDMT_BLOCK_INST(uint16_t, int32_t, float, false)
FDMT_BLOCK_INST(uint16_t, int32_t, int32_t, false)
#undef FDMT_BLOCK_INST

} // namespace fdmt
