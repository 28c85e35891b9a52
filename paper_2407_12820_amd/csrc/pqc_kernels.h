// Kernels of libpqcache (gfx950).  Grid layout: blockIdx.y = unit (sequence b, KV
// head g); blockIdx.x = workgroup inside the unit (query head for finalize_kernel).
//
// Decode path (pqc_decode), three launches, two for short caches (From::kCount, From::kShort), every dependency at a kernel boundary:
//   hist_kernel      table -> scan codes -> histogram of scores over kNB bins, and every
//                    token's bin number left behind for the next kernel
//   select_kernel    threshold bin from the histogram -> tokens whose stored bin lies
//                    above it (and the two windows) are listed in ascending order
//                    without atomics and attended at once; tokens inside the bin
//                    ("candidates") are recorded with their logits and V row
//   finalize_kernel  one to four workgroups per query head rank the candidates and fold the
//                    admitted ones and all partial softmax states into the output;
//                    copy workgroups beside them write the indices and zero the unit's
//                    histogram and record counter again, which nothing reads after the
//                    select kernel: every call leaves them as it found them
//
// Codes are read 16 bytes at a time (P = 16/M tokens).  A unit's codes start at byte
// u*N*M, which need not be 16-byte aligned: chunks are laid over the aligned-down
// address, so chunk 0 may begin with up to P-1 "phantom" tokens of the previous unit
// and the last chunk may end with phantoms; both are masked by the token range check.
#pragma once
#include "pqc_device.h"

namespace pqc {

constexpr int kMaxVecA = 4;   // 16-byte code chunks per thread, histogram kernel

// ------------------------------------------------------------------ sources
// Where a kernel takes its scores from: PQ codes through the LDS table (the decode
// path) or a score array in global memory (the stand-alone top-k stage).

// The upper bytes of 16, from byte `n` on (0 <= n <= 16), moved down to the first; zeros behind them.
__device__ __forceinline__ u32x4_t bytes_from(const u32x4_t& r, int n) {
  unsigned long long lo = r[0] | ((unsigned long long)r[1] << 32), hi = r[2] | ((unsigned long long)r[3] << 32);
  lo = n & 8 ? hi : lo;
  hi = n >= 8 ? 0ull : hi;
  const int sh = 8 * (n & 7);
  lo = (lo >> sh) | ((hi << 1) << (63 - sh));
  hi >>= sh;
  lo = n < 16 ? lo : 0ull;
  return u32x4_t{(unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32)};
}

template <int M_>
struct CodeChunks {
  static constexpr int M = M_;
  static constexpr int P = 16 / M_;  // tokens per chunk
  static constexpr bool kFromCodes = true;
  using Raw = u32x4_t;
  const uint8_t* all;       // whole code tensor
  long long total_bytes;    // its size
  long long unit_byte0;     // aligned-down byte offset of this unit's codes
  int lead;                 // phantom tokens before token 0
  const float* lut;         // LDS
  const uint8_t* spare;     // 16 readable bytes of any content
  __device__ __forceinline__ void init(const void* ptr, int u, int N, int units, const float* lut_, const void* spare16) {
    all = static_cast<const uint8_t*>(ptr);
    spare = static_cast<const uint8_t*>(spare16);
    total_bytes = (long long)units * N * M;
    const long long ob = (long long)u * N * M;
    unit_byte0 = ob & ~15ll;
    lead = (int)((ob - unit_byte0) / M);
    lut = lut_;
  }
  // Unconditional 16-byte load (straight-line code keeps many loads in flight, and lets the
  // compiler count them when it waits for earlier ones): a chunk that reaches beyond the tensor is
  // redirected to the tensor's last 16 bytes (to the spare bytes if it has fewer; global loads take any
  // address), and fix_tail() moves the bytes of the one chunk that holds the tensor's ragged end into place
  // afterwards.  (Loaded byte by byte instead they are a chain of memory round trips in the last workgroup: 7 units
  // of 20009 tokens, 4x64, 22.9 us per layer, now 21.7, which is what 20008 tokens take; 9 of 7595 19.0, now 17.7.)
  __device__ __forceinline__ Raw load(int chunk) const {
    long long off = unit_byte0 + 16ll * chunk;
    off = off < total_bytes - 16 ? off : total_bytes - 16;
    off = off > 0 ? off : 0;
    Raw r;
    __builtin_memcpy(&r, total_bytes < 16 ? spare : all + off, 16);
    return r;
  }
  // Whether the last of a unit's chunks is that one (uniform).
  __device__ __forceinline__ bool ragged(int chunks) const { return unit_byte0 + 16ll * chunks > total_bytes; }
  __device__ __forceinline__ void fix_tail(Raw& r, int chunk) const {
    const long long off = unit_byte0 + 16ll * chunk;
    if (off + 16 > total_bytes && off < total_bytes) {  // at most one chunk in the whole tensor
      if (total_bytes >= 16) {
        r = bytes_from(r, (int)(off + 16 - total_bytes));
      } else {
        r = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll 1
        for (int b = (int)total_bytes - 1; b >= 0; --b) {  // the bytes enter at the bottom and move up
          r = u32x4_t{r[0] << 8, __builtin_amdgcn_alignbit(r[1], r[0], 24), __builtin_amdgcn_alignbit(r[2], r[1], 24), __builtin_amdgcn_alignbit(r[3], r[2], 24)};
          r[0] |= (unsigned)all[b];
        }
      }
    }
  }
  __device__ __forceinline__ float score(const Raw& r, int i) const { return score_from_word<M>(chunk_word<M>(r, i), lut); }
  // one token: the load (issue early) and the table look-up (after the table is ready)
  using One = typename CodeWord<M>::type;
  __device__ __forceinline__ One load_one(int t, int u, int N) const {
    return (reinterpret_cast<const One*>(all) + (size_t)u * N)[(unsigned)t];  // (the tensor is 16-byte aligned)
  }
  __device__ __forceinline__ float score_one(One w) const { return score_from_word<M>(w, lut); }
  __device__ __forceinline__ float score_of_token(int t, int u, int N) const { return score_one(load_one(t, u, N)); }
};

struct ScoreChunks {
  static constexpr int M = 0;
  static constexpr int P = 4;
  static constexpr bool kFromCodes = false;
  struct Raw {
    float f[4];
  };
  const float* scores;  // this unit's [N] scores
  int n;
  int lead;
  __device__ __forceinline__ void init(const void* ptr, int u, int N, int, const float*, const void*) {
    scores = static_cast<const float*>(ptr) + (size_t)u * N;
    n = N;
    lead = 0;
  }
  __device__ __forceinline__ Raw load(int chunk) const {
    Raw r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      long long t = (long long)chunk * 4 + i;
      t = t < n ? t : n - 1;  // clamped: straight-line loads; tokens >= n are masked by the caller
      r.f[i] = scores[t];
    }
    return r;
  }
  __device__ __forceinline__ float score(const Raw& r, int i) const { return r.f[i]; }
  using One = float;
  __device__ __forceinline__ One load_one(int t, int, int) const { return scores[t]; }
  __device__ __forceinline__ float score_one(One w) const { return w; }
  __device__ __forceinline__ float score_of_token(int t, int, int) const { return scores[t]; }
};

// ------------------------------------------------------------------ utilities
// Workgroups are handed to the 8 XCDs round-robin in launch order (x fastest).  The workgroups of a unit that all read its centroids
// (and codes) share an XCD and its L2: eight units at a time are interleaved.
__device__ __forceinline__ void unit_of_workgroup(int units, int nx /* workgroups per unit */, int& u, int& bx) {
  const int lin = blockIdx.y * nx + blockIdx.x;
  if (lin < (units & ~7) * nx) {
    const int i = lin % (8 * nx);
    u = (lin / (8 * nx)) * 8 + (i & 7);
    bx = i >> 3;
  }
}

// Stand-alone table (pqc_lut).
template <typename T, int M>
__global__ __launch_bounds__(256) void lut_kernel(Shape s, const T* __restrict__ q, const float* __restrict__ cent,
                                                  float* __restrict__ table) {
  __shared__ float lut[M * kLutRow];
  __shared__ float qs[kD];
  __shared__ float red[32];
  __shared__ float tile[lut_tile_floats(256, M, 256)];
  const int u = blockIdx.y, b = u / s.Hkv, g = u % s.Hkv;
  build_lut<T, 256, M>(q + ((size_t)b * s.Hq + (size_t)g * s.G) * kD, cent + (size_t)u * M * s.C * (kD / M), s.G, s.C, lut,
                       qs, red, tile, [](int) {}, []() {});
  for (int e = threadIdx.x; e < M * s.C; e += 256) table[(size_t)u * M * s.C + e] = lut[(e / s.C) * kLutRow + (e % s.C)];
}

// Stand-alone scan (pqc_scan): scores[N], -inf inside the two windows.
template <int M>
__global__ __launch_bounds__(256) void scan_kernel(Shape s, const float* __restrict__ table,
                                                   const uint8_t* __restrict__ codes, float* __restrict__ scores) {
  __shared__ float lut[M * kLutRow];
  const int u = blockIdx.y;
  for (int e = threadIdx.x; e < M * s.C; e += 256) lut[(e / s.C) * kLutRow + (e % s.C)] = table[(size_t)u * M * s.C + e];
  __syncthreads();
  using W = typename CodeWord<M>::type;
  const W* cw = reinterpret_cast<const W*>(codes) + (size_t)u * s.cap;
  const int t0 = blockIdx.x * 2048;
  for (int t = t0 + threadIdx.x; t < min(t0 + 2048, s.N); t += 256) {
    const bool mid = t >= s.I && t < s.N - s.L;
    scores[(size_t)u * s.N + t] = mid ? score_from_word<M>(cw[t], lut) : -INFINITY;
  }
}

// ------------------------------------------------------------- 1. histogram
// SRC = CodeChunks<M>: builds the unit's table first; score bounds come from the table.
// SRC = ScoreChunks: bounds come from score_range_kernel.  Every workgroup of a unit
// then derives the same bin layout from the same sampled tokens (workgroup 0 publishes
// the table for the select kernel) and counts its own tokens.  Workgroups of a
// unit spread their counts over histCopies replicas.
// VW: 16-byte pieces of the centroid tensor per thread (1024 * 4 * VW floats cover the unit's M*C*Dm);
// VA: 16-byte chunks of codes (or scores) per thread (1024 * VA chunks cover the workgroup's tokA tokens).
// Both are template parameters so that no thread issues loads it does not need: the loads of a workgroup's
// sixteen waves go through one address unit, 64 bytes per clock, and redundant ones cost as much as real ones.
template <typename T, class SRC, int VW, int VA>
__global__ __launch_bounds__(1024) void hist_kernel(Shape s, Workspace ws, const T* __restrict__ q,
                                                    const float* __restrict__ cent, const void* __restrict__ src_ptr) {
  constexpr int NT = 1024, P = SRC::P;
  static_assert(VA >= 1 && VA <= kMaxVecA, "chunks per thread");
  constexpr int LM = SRC::kFromCodes ? SRC::M : 1;
  __shared__ float lut[LM * kLutRow];
  __shared__ __attribute__((aligned(16))) float qs[kD];
  __shared__ float red[32];
  extern __shared__ __attribute__((aligned(16))) float tile[];  // lut_tile_floats(NT, LM, C) floats when the source is codes
  __shared__ unsigned hist[kNB];
  __shared__ int scan_sm[2 * (NT / 64) + 1 + 2];
  const int tid = threadIdx.x, units = s.B * s.Hkv;
  int u = blockIdx.y, bx = blockIdx.x;
  unit_of_workgroup(units, s.nblkA, u, bx);
  PQC_MARK(ws, 0, 0);
#ifdef PQC_TRACE
  PQC_NOTE(ws, 0, 15, (__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15) | (u << 8));  // XCC_ID[3:0], unit
#endif
  SRC src;
  const int src_stride = SRC::kFromCodes ? s.cap : s.N;  // tokens between units: code tensor, or dense score array
  src.init(src_ptr, u, src_stride, units, lut, ws.hist);
  // this workgroup's chunks and this thread's sample: the loads are issued before anything else,
  // except that a table build puts its centroid loads in front of them
  const int chunks = s.tokA / P, chunk0 = bx * chunks;
  typename SRC::Raw raw[VA];
  typename SRC::One sample;
  auto issue_loads = [&]() {
#pragma unroll
    for (int v = 0; v < VA; ++v) raw[v] = src.load(chunk0 + min(v * NT + tid, chunks - 1));
    sample = src.load_one(sample_token(s, min(tid, s.sampleN - 1)), u, src_stride);
  };
  float2 bounds;
  if constexpr (SRC::kFromCodes) {
    const int b = u / s.Hkv, g = u % s.Hkv;
    for (int i = tid; i < kNB; i += NT) hist[i] = 0u;
    auto mark = [&](int slot) { PQC_MARK(ws, 0, slot); };
    bounds = build_lut<T, NT, LM, decltype(mark), decltype(issue_loads), VW>(
        q + ((size_t)b * s.Hq + (size_t)g * s.G) * kD, cent + (size_t)u * LM * s.C * (kD / LM), s.G, s.C, lut, qs, red, tile,
        mark, issue_loads);
    if (bx == 0)
      for (int e = tid; e < LM * s.C; e += NT) ws.lut[(size_t)u * LM * s.C + e] = lut[(e / s.C) * kLutRow + (e % s.C)];
  } else {
    issue_loads();
    PQC_LOADS_ISSUED();
    for (int i = tid; i < kNB; i += NT) hist[i] = 0u;
    bounds = ws.range[u];
    __syncthreads();
  }
  PQC_MARK(ws, 0, 1);
  const float sample_score[1] = {src.score_one(sample)};
  const BinMap map = sample_window<NT, 1>(bounds.x, bounds.y, sample_score, s.sampleN, s.rankHi, s.rankLo, hist, scan_sm);
  if constexpr (SRC::kFromCodes) {
    const int all = (s.N + src.lead + P - 1) / P;  // chunks of the unit
    if (src.ragged(all) && chunk0 + chunks >= all) {  // uniform (behind the window: in front of it every step takes 0.2 us longer)
#pragma unroll
      for (int v = 0; v < VA; ++v)
        if (chunk0 + v * NT + tid == all - 1) src.fix_tail(raw[v], all - 1);
    }
  }
  PQC_MARK(ws, 0, 2);
  // most tokens score below the window and are not counted, the rest go to their LDS bin (an LDS atomic costs in proportion
  // to the lanes that take part)
  unsigned short* bins_u = ws.bins + (size_t)u * s.binStride;
#pragma unroll
  for (int v = 0; v < VA; ++v) {
    if (v * NT + tid < chunks) {
      const int t0 = (chunk0 + v * NT + tid) * P - src.lead;
      unsigned st[P];  // what the select kernel will read back: bin, or the window mark
      if (t0 >= s.I && t0 + P <= s.N - s.L) {  // all P tokens are middle tokens (all but the chunks at the two ends)
#pragma unroll
        for (int i = 0; i < P; ++i) st[i] = score_bin(src.score(raw[v], i), map);
#pragma unroll
        for (int i = 0; i < P; ++i)
          if (st[i]) atomicAdd(&hist[st[i]], 1u);
      } else {
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const int t = t0 + i;
          const bool mid = t >= s.I && t < s.N - s.L;
          const unsigned bin = score_bin(src.score(raw[v], i), map);
          if (mid && bin) atomicAdd(&hist[bin], 1u);
          st[i] = mid ? bin : kBinWindow;
        }
      }
      if (src.lead == 0 && t0 + P <= s.N) {  // the usual case: aligned, all P tokens exist
        if constexpr (P == 1) {
          bins_u[t0] = (unsigned short)st[0];
        } else {
          unsigned pw[P / 2];
#pragma unroll
          for (int i = 0; i < P / 2; ++i) pw[i] = st[2 * i] | (st[2 * i + 1] << 16);
          if constexpr (P == 2) *reinterpret_cast<unsigned*>(bins_u + t0) = pw[0];
          if constexpr (P == 4) *reinterpret_cast<uint2*>(bins_u + t0) = make_uint2(pw[0], pw[1]);
          if constexpr (P >= 8) {
#pragma unroll
            for (int i = 0; i < P / 8; ++i)
              reinterpret_cast<uint4*>(bins_u + t0)[i] = make_uint4(pw[4 * i], pw[4 * i + 1], pw[4 * i + 2], pw[4 * i + 3]);
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < P; ++i)
          if (t0 + i >= 0 && t0 + i < s.N) bins_u[t0 + i] = (unsigned short)st[i];
      }
    }
  }
  __syncthreads();
  PQC_MARK(ws, 0, 3);
  unsigned* gh = ws.hist + ((size_t)u * s.histCopies + (bx % s.histCopies)) * kNB;
  for (int i = tid; i < kNB; i += NT)
    if (hist[i]) atomicAdd(&gh[i], hist[i]);
  PQC_MARK(ws, 0, 4);
}

// ---------------------------------------------------- 2. select (+ attention)
// One workgroup owns tokens [blockIdx.x*tokC, +tokC) of its unit, each of its waves a contiguous share.  The histogram kernel
// left every token's bin behind, so a token is classified by comparing that number with the threshold bin.  Per wave, lanes hold
// 8 consecutive tokens and counts are prefix-summed across lanes and waves; then the selected tokens (ascending) are written to the
// front of one list in LDS and the boundary-bin candidates to its end.  SRC is only used to score the few candidates exactly.
// (A list per wave took a search over the waves' counts at every look-up; 131072 tokens x 8 heads, a layer: 35.8 us, now 35.2.)

// Where the threshold comes from.  kBins: from the histogram kernel in front.  The other forms have no histogram kernel: every workgroup
// builds the table itself and finds the threshold without the others.
//   kPairs  (M = 2, up to 64 centroids) from code-pair counts of the caller's (pair_classes); tokens above it are those with a higher
//           exact score, its own are the candidates.  kPairsMany: the same in workgroups of 256 threads, two of them per compute unit (the
//           list lies over the counts, so that both fit its LDS), for grids that one workgroup per compute unit leaves uneven.
//   kCount  (M = 2, up to 64 centroids) from code-pair counts that the workgroup takes of all tokens of its unit while the table is built:
//           the pairs' scores go to the bins that the histogram kernel would have put the tokens into, and the tokens of the threshold's
//           bin are the candidates, whichever of its pairs they carry.
//   kShort  (M = 2 or 4) scores all tokens of its unit.
// In the last two the launch of the histogram kernel, its table and what it leaves in memory are saved, against work in each workgroup that
// grows with the unit: one LDS addition per token (kCount), or M look-ups and a bin (kShort); see short_cache(), and pairs_form().  A workgroup of 512
// threads per compute unit (the table and the waves' tiles share its LDS) keeps as many rows in flight as two of 256, and does
// what does not depend on its own tokens once instead of twice.
enum class From { kBins, kPairs, kPairsMany, kCount, kShort };
template <From FROM>
constexpr int select_threads() { return FROM == From::kBins || FROM == From::kPairsMany ? 256 : 512; }
constexpr int kShortChunks = 4;  // 16-byte code chunks per thread and step, the next step's in flight
// kCount: while two waves build the table the other six count, kCountEarly chunks per thread (about as long as the table takes), requested
// in front of the wait for the centroids; then all count the rest, kCountChunks per thread under way (together 33792 tokens).
constexpr int kCountEarly = 3;
constexpr int kCountChunks = 6;
constexpr int max_tokens_per_select(From f) { return f == From::kPairs ? 16384 : 8192; }
// Of the two the one with counted pairs wherever there are few enough pairs, kShort and kCount, 2x64, us per layer, bf16, 4 query heads per
// unit, a tenth retrieved: 8 units of 2048 tokens 15.6, 15.7, of 8192 16.9, 16.4, of 16384 19.1, 17.7, of 24576 21.7, 19.3; 1 unit of 4096 15.3, 15.3.
inline bool counts_pairs(const Shape& s) { return s.M == 2 && s.C <= kPairC; }
template <From FROM>
constexpr size_t list_bytes(int tokC) { return ((size_t)tokC + select_threads<FROM>()) * sizeof(unsigned short); }
template <From FROM>
constexpr int tiles_bytes(bool mfma) { return mfma ? select_threads<FROM>() / 64 * kVTileBytes : 16; }
template <From FROM>
constexpr int states_bytes(int G) { return select_threads<FROM>() / 64 * G * (kD + 2) * (int)sizeof(float); }
// Dynamic LDS of the forms with a table of their own: the centroid tile, then (over it) V tiles, the waves' states, the list and the
// own tokens' bins (kShort).
template <From FROM>
constexpr size_t table_form_lds_bytes(const Shape& s, bool mfma) {
  const size_t tile = (size_t)lut_tile_floats(512 /* the whole table */, s.M, s.C) * sizeof(float);
  const size_t work = tiles_bytes<FROM>(mfma) + states_bytes<FROM>(s.G) + (FROM == From::kPairsMany ? 0 : list_bytes<FROM>(s.tokC)) + (FROM == From::kShort ? (size_t)s.tokC * 2 : 0);
  return tile > work ? tile : work;
}

// The workgroup's own tokens [lo, hi): what is known of each is kept in LDS, two bytes a token.
struct OwnTokens {
  unsigned short* at;
  int lo, hi;
};
template <int P>
__device__ __forceinline__ void keep_own(const OwnTokens& own, int lead, int t0, const unsigned (&v)[P]) {
  if (t0 + P > own.lo && t0 < own.hi) {
    if (lead == 0) {  // uniform; then a chunk is the workgroup's as a whole (tokC is a multiple of P)
      unsigned short* dst = own.at + (t0 - own.lo);
      unsigned pw[P / 2];
#pragma unroll
      for (int i = 0; i < P / 2; ++i) pw[i] = v[2 * i] | (v[2 * i + 1] << 16);
      if constexpr (P == 4) *reinterpret_cast<uint2*>(dst) = make_uint2(pw[0], pw[1]);
      if constexpr (P == 8) *reinterpret_cast<uint4*>(dst) = make_uint4(pw[0], pw[1], pw[2], pw[3]);
    } else {
#pragma unroll
      for (int i = 0; i < P; ++i)
        if (t0 + i >= own.lo && t0 + i < own.hi) own.at[t0 + i - own.lo] = (unsigned short)v[i];
    }
  }
}
// kCount: the chunks that hold middle tokens only, and the middle tokens beside them (fewer than eight at each end).
struct MiddleChunks {
  int n;               // chunks
  int head, head_end;  // tokens in front
  int tail, tail_end;  // tokens behind
  const uint8_t* base;
  __device__ __forceinline__ MiddleChunks(const CodeChunks<2>& src, int mid_lo, int mid_hi) {
    const int first = (mid_lo + src.lead + 7) / 8;
    n = max(0, (mid_hi + src.lead) / 8 - first);
    head = mid_lo;
    head_end = min(first * 8 - src.lead, mid_hi);
    tail = max((first + n) * 8 - src.lead, head_end);
    tail_end = mid_hi;
    base = n > 0 ? src.all + src.unit_byte0 + 16ll * first : src.spare;
  }
  // (the chunk nearest to c; all of them lie inside the tensor)
  __device__ __forceinline__ u32x4_t load(int c) const {
    return *reinterpret_cast<const u32x4_t*>(base + 16u * (unsigned)max(min(c, n - 1), 0));
  }
};
struct Absent {
  template <class... A>
  __device__ __forceinline__ Absent(const A&...) {}
};
// Counts the pairs of the chunks from `begin` on below `end`, NT threads (`t`: this one) in turns of one chunk each, U of a thread under
// way: its first U have been requested, and a chunk's registers take the next one as soon as it has been read.  One addition per token,
// bound by LDS: 64 lanes in 64 random places of 4096 take 9 clocks (32768 tokens 2.0 us).  The code is kept small: that of a step's
// kernels lives in 64 KB of instruction cache.  Chunks whose lanes meet in one address (padding, a repeated token: they add one after the
// other, two clocks each) are read again in a part of its own.
template <int NT, int U>
__device__ __forceinline__ void count_pairs(u32x4_t (&code)[U], const MiddleChunks& m, int begin, int end, int t, unsigned* cnt) {
  const int lane = threadIdx.x & 63;
  for (int c0 = begin; c0 < end; c0 += U * NT) {
    unsigned crowded = 0u;  // wave-uniform: turns with such chunks
#pragma unroll
    for (int v = 0; v < U; ++v) {
      if (c0 + v * NT < end) {  // uniform
        const int c = c0 + v * NT + t;
        unsigned slot[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) pair_slots(code[v][k], slot[2 * k], slot[2 * k + 1]);
        if (c0 + (U + v) * NT < end) code[v] = m.load(c + U * NT);  // uniform
        if (__popcll(__ballot(c < end && slot[0] == (unsigned)__builtin_amdgcn_readfirstlane((int)slot[0]))) >= 32) {
          crowded |= 1u << v;
        } else if (c < end) {
#pragma unroll
          for (int i = 0; i < 8; ++i) atomicAdd(&cnt[slot[i]], 1u);
        }
      }
    }
    while (crowded) {  // wave-uniform
      const int c = c0 + (__ffs((int)crowded) - 1) * NT + t;
      crowded &= crowded - 1u;
      if (c < end) {
        const u32x4_t r = m.load(c);
#pragma unroll 1
        for (int i = 0; i < 8; ++i) {
          unsigned s0, s1;
          pair_slots(i < 2 ? r[0] : i < 4 ? r[1] : i < 6 ? r[2] : r[3], s0, s1);
          const unsigned slot = i & 1 ? s1 : s0, first = (unsigned)__builtin_amdgcn_readfirstlane((int)slot);
          const unsigned long long same = __ballot(slot == first);  // counted in one go
          if (slot != first) atomicAdd(&cnt[slot], 1u);
          else if (lane == __ffsll((long long)same) - 1) atomicAdd(&cnt[first], (unsigned)__popcll(same));
        }
      }
    }
  }
}
// Codes of the eight tokens from t on, two partitions.  (A unit's tokens need not begin at a multiple of 16 bytes; global loads take
// any address.)  A load that would reach beyond the tensor is moved back, and its bytes into place by fix.
struct OwnCodes {
  const uint8_t* base;  // of the unit
  int room;             // bytes from there to the tensor's end, or more than any token's place
  __device__ __forceinline__ OwnCodes(const CodeChunks<2>& src, int u, int cap) {
    const long long at = (long long)u * cap * 2, left = src.total_bytes - at;
    room = (int)min(left, 1ll << 24);
    base = left < 16 ? src.spare : src.all + at;
  }
  __device__ __forceinline__ u32x4_t load(int t) const {
    u32x4_t r;
    __builtin_memcpy(&r, base + (unsigned)max(min(2 * t, room - 16), 0), 16);
    return r;
  }
  __device__ __forceinline__ void fix(const CodeChunks<2>& src, int u, int cap, int t, u32x4_t& r) const {
    const int beyond = 2 * t + 16 - room;
    if (__any(beyond > 0)) {  // wave-uniform, the last tokens of the tensor
      if (room >= 16) {  // uniform
        r = bytes_from(r, max(0, min(beyond, 16)));
      } else {
        r = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll 1
        for (int i = 7; i >= 0; --i) {  // tokens enter at the bottom and move up
          r = u32x4_t{r[0] << 16, __builtin_amdgcn_alignbit(r[1], r[0], 16), __builtin_amdgcn_alignbit(r[2], r[1], 16), __builtin_amdgcn_alignbit(r[3], r[2], 16)};
          if (2 * (t + i) + 2 <= room) r[0] |= src.load_one(t + i, u, cap);
        }
      }
    }
  }
};
// kShort: middle tokens per score bin, and the stored bins of the workgroup's own tokens.
template <int NT, int U, class SRC>
__device__ __forceinline__ void bin_scores(const SRC& src, typename SRC::Raw (&code)[U], int chunks, int mid_lo, int mid_hi, const OwnTokens& own,
                                           const BinMap& map, unsigned* hist /* [kNB + 64] */) {
  constexpr int P = SRC::P;
  const int tid = threadIdx.x, lane = tid & 63;
  const bool ragged = src.ragged(chunks);
  for (int c0 = 0; c0 < chunks; c0 += U * NT) {
    if (ragged && c0 + U * NT >= chunks) {  // uniform, and apart from the loop below, whose code is kept short
#pragma unroll
      for (int v = 0; v < U; ++v)
        if (c0 + v * NT + tid == chunks - 1) src.fix_tail(code[v], chunks - 1);
    }
#pragma unroll
    for (int v = 0; v < U; ++v) {
      const int c = c0 + v * NT + tid;
      if (c < chunks) {
        const int t0 = c * P - src.lead;
        unsigned st[P], hb[P];
#pragma unroll
        for (int i = 0; i < P; ++i) hb[i] = st[i] = score_bin(src.score(code[v], i), map);
        if (t0 < mid_lo || t0 + P > mid_hi) {
#pragma unroll
          for (int i = 0; i < P; ++i) {
            const bool mid = t0 + i >= mid_lo && t0 + i < mid_hi;
            st[i] = mid ? st[i] : kBinWindow;
            hb[i] = mid ? hb[i] : 0u;
          }
        }
#pragma unroll
        for (int i = 0; i < P; ++i) atomicAdd(&hist[hb[i] ? hb[i] : kNB + lane], 1u);
        keep_own<P>(own, src.lead, t0, st);
      }
      if (c0 + (U + v) * NT < chunks) code[v] = src.load(min(c + U * NT, chunks - 1));  // uniform
    }
  }
}

template <typename T, int G, class SRC, bool ATTN, From FROM = From::kBins, int VW = 1 /* 16-byte pieces of the centroids per thread, for the table */>
__global__ __launch_bounds__(select_threads<FROM>(), 2) void select_kernel(Shape s, Workspace ws, const T* __restrict__ q,
                                                     const T* __restrict__ kc, const T* __restrict__ vc,
                                                     const void* __restrict__ src_ptr,
                                                     const float* __restrict__ cent = nullptr,
                                                     const unsigned* __restrict__ pair_counts = nullptr,
                                                     int uncounted = -1 /* kPairs: a window token not in the counts yet */) {
  constexpr bool PAIRS = FROM == From::kPairs || FROM == From::kPairsMany, COUNT = FROM == From::kCount, SHORT = FROM == From::kShort;
  constexpr bool TABLE = FROM != From::kBins;
  constexpr int NT = select_threads<FROM>(), NW = NT / 64;
  constexpr bool kMfma = ATTN && sizeof(T) == 2 && kMatrixCoreAttention;
  static_assert(!(PAIRS || COUNT) || (SRC::kFromCodes && SRC::M == 2), "pair counts exist for two partitions only");
  static_assert(!TABLE || (SRC::kFromCodes && ATTN && (SRC::P == 4 || SRC::P == 8)), "the forms with a table are those of the decode step with two or four partitions");
  constexpr int LM = SRC::kFromCodes ? SRC::M : 1;
  constexpr int GV = max_tokens_per_select(FROM) / (8 * NT);  // 8-token groups per lane, at most
  extern __shared__ __attribute__((aligned(16))) unsigned char select_lds[];
  constexpr int kList = TABLE ? tiles_bytes<FROM>(kMfma) + states_bytes<FROM>(G) : 0;
  __shared__ std::conditional_t<PAIRS || COUNT, PairLds, int> pl;
  unsigned short* list = reinterpret_cast<unsigned short*>(select_lds + kList);  // [tokC] token offsets from the workgroup's first token, [NT] see below
  if constexpr (FROM == From::kPairsMany) {
    static_assert(sizeof(pl.cnt) >= list_bytes<FROM>(max_tokens_per_select(FROM)), "the list lies over the counts");
    list = reinterpret_cast<unsigned short*>(pl.cnt);
  }
  __shared__ int scan_sm[2 * NW + 1 + 4];
  __shared__ int wcnt[NW];
  __shared__ float red_own[ATTN && !TABLE ? states_bytes<FROM>(G) / 4 : 1];
  __shared__ float qlds[ATTN ? G * kD : 1];
  __shared__ __attribute__((aligned(16))) unsigned char vtile_own[TABLE ? 16 : tiles_bytes<FROM>(kMfma)];
  __shared__ __attribute__((aligned(16))) float lut[TABLE ? LM * kLutRow : 1];
  __shared__ __attribute__((aligned(16))) unsigned hist[TABLE ? kNB + 64 : 4];  // behind the bins: a place per lane for what is not counted
  unsigned char* vtile = TABLE ? select_lds : vtile_own;
  float* red = TABLE ? reinterpret_cast<float*>(select_lds + tiles_bytes<FROM>(kMfma)) : red_own;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if constexpr (TABLE)  // the arguments that the first loads wait for, in one go
    asm volatile("" ::"s"(s.Hkv), "s"(s.B), "s"(s.N), "s"(s.C), "s"(s.I), "s"(s.L), "s"(s.cap), "s"(s.tokC), "s"(s.nblkC), "s"(q), "s"(src_ptr), "s"(cent));
  int u = blockIdx.y, bx = blockIdx.x;
  if constexpr (TABLE) unit_of_workgroup(s.B * s.Hkv, s.nblkC, u, bx);
  const int b = u / s.Hkv, g = u % s.Hkv;
  PQC_MARK(ws, 1, 0);
  const int tpw = s.tokC / NW;           // tokens per wave, in groups of 8 per lane
  const int gpw = (tpw + 511) / 512;     // groups per lane: 1, 2 or 4 (the last lanes idle when tpw < 512)
  const int wave_t0 = bx * s.tokC + w * tpw;
  u32x4_t raw[GV];
  Threshold th{0, 0, 0, 0};
  unsigned short* own = nullptr;  // kShort: [tokC] stored bins
  if constexpr (TABLE) {
    own = reinterpret_cast<unsigned short*>(select_lds + kList + list_bytes<FROM>(s.tokC));
    __shared__ __attribute__((aligned(16))) float qs[kD];
    [[maybe_unused]] __shared__ float lut_red[32];
    SRC src;
    src.init(src_ptr, u, s.cap, s.B * s.Hkv, lut, ws.hist);
    const int chunks = (s.N + src.lead + SRC::P - 1) / SRC::P;  // of the unit
    [[maybe_unused]] const std::conditional_t<COUNT, MiddleChunks, Absent> mids(src, s.I, s.N - s.L);
    [[maybe_unused]] int n_early = 0;  // kCount: chunks counted while the table is built
    if constexpr (COUNT) n_early = min(mids.n, kCountEarly * (NT - 128));
    [[maybe_unused]] unsigned short edge = 0;  // kCount: the code word of a token beside those chunks
    constexpr int U = PAIRS ? 1 : COUNT ? kCountChunks : kShortChunks;
    typename SRC::Raw code[U];
    [[maybe_unused]] u32x4_t early[kCountEarly];
    constexpr int PS = 1024 / NT, QN = (G * kD + NT - 1) / NT;
    typename SRC::One sample[PS];
    constexpr int PER = kPairPer<NT>;
    u32x4_t given[PER / 4];  // kPairs: the counts of this thread's slots
    unsigned short wcode = 0;  // kPairs: this thread's first window token (the usual case: I + L <= NT)
    [[maybe_unused]] const std::conditional_t<PAIRS || COUNT, OwnCodes, Absent> own_codes(src, u, s.cap);
    auto own_token = [&](int v) -> int { return min(wave_t0 + min((v * 64 + lane) * 8, tpw - 8), s.N - 1); };
    auto issue_early = [&]() {
      if constexpr (COUNT) {
#pragma unroll
        for (int v = 0; v < kCountEarly; ++v) early[v] = mids.load(v * (NT - 128) + tid - 128);
      }
      PQC_LOADS_ISSUED();
      if constexpr (PAIRS || COUNT) {
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) reinterpret_cast<uint4*>(pl.cnt)[i * NT + tid] = make_uint4(0u, 0u, 0u, 0u);
        if (tid < kSampleBins / 4) reinterpret_cast<uint4*>(pl.samples)[tid] = make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int i = 0; i < kNB / (4 * NT); ++i) reinterpret_cast<uint4*>(hist)[i * NT + tid] = make_uint4(0u, 0u, 0u, 0u);
    };
    auto issue_loads = [&]() {
      if constexpr (PAIRS) {
        const unsigned* pc = pair_counts + (size_t)u * s.C * s.C;
        const int c0 = (tid * PER) & 63, c1 = (tid * PER) >> 6;
        if (s.C == kPairC) {  // uniform
#pragma unroll
          for (int i = 0; i < PER / 4; ++i) given[i] = reinterpret_cast<const u32x4_t*>(pc)[PER / 4 * tid + i];
        } else {
#pragma unroll
          for (int i = 0; i < PER; ++i) given[i / 4][i % 4] = pc[min(c1, s.C - 1) * s.C + min(c0 + i, s.C - 1)];
        }
        const int wt = min(max(tid - 128, 0), max(s.I + s.L - 1, 0)), t = wt < s.I ? wt : s.N - s.L + (wt - s.I);
        wcode = src.load_one(min(max(t, 0), s.N - 1), u, s.cap);
      } else if constexpr (COUNT) {
#pragma unroll
        for (int x = 0; x < PS; ++x) sample[x] = src.load_one(sample_token(s, min(x * NT + tid, s.sampleN - 1)), u, s.cap);
        edge = src.load_one(min(max((tid & 8 ? mids.tail : mids.head) + (tid & 7), 0), s.N - 1), u, s.cap);
#pragma unroll
        for (int v = 0; v < U; ++v)
          if (n_early + v * NT < mids.n) code[v] = mids.load(n_early + v * NT + tid);  // uniform
      } else {
#pragma unroll
        for (int x = 0; x < PS; ++x) sample[x] = src.load_one(sample_token(s, min(x * NT + tid, s.sampleN - 1)), u, s.cap);
#pragma unroll
        for (int v = 0; v < U; ++v)
          if (v * NT < chunks) code[v] = src.load(min(v * NT + tid, chunks - 1));  // uniform
      }
      if constexpr (PAIRS || COUNT) {
#pragma unroll
        for (int v = 0; v < GV; ++v)
          if (v < gpw) raw[v] = own_codes.load(own_token(v));  // uniform
      }
    };
    static_assert(kNB % (4 * NT) == 0 && (FROM != From::kShort || kNB == 4 * NT), "whole 16-byte pieces per thread; one in kShort");
    const T* qu = q + ((size_t)b * s.Hq + (size_t)g * G) * kD;
    const float* cu = cent + (size_t)u * LM * s.C * (kD / LM);
    float* tile = reinterpret_cast<float*>(select_lds);
    float qv[QN];
#pragma unroll
    for (int x = 0; x < QN; ++x) qv[x] = load_as_float<T>(qu, min(x * NT + tid, G * kD - 1));
    auto mark = [&](int slot) {};
    auto store_query = [&]() {
#pragma unroll
      for (int x = 0; x < QN; ++x)
        if (x * NT + tid < G * kD) qlds[x * NT + tid] = qv[x];
    };
    if constexpr (PAIRS || COUNT) {
      lut_stage<T, NT, LM, VW>(qu, cu, G, s.C, qs, tile, mark, issue_early, issue_loads);
      store_query();
      __syncthreads();
      PQC_MARK(ws, 1, 11);
#pragma unroll
      for (int v = 0; v < GV; ++v)
        if (v < gpw) own_codes.fix(src, u, s.cap, own_token(v), raw[v]);
      if (w < 2) {
        float lo, hi;
        pair_table<PAIRS>(tile, qs, s.C, w, lut, lo, hi);
        if (lane == 0) {
          pl.bounds[2 * w] = lo;
          pl.bounds[2 * w + 1] = hi;
        }
      } else if constexpr (PAIRS) {  // the window tokens among the counted ones
        for (int wt = tid - 128; wt < s.I + s.L; wt += NT - 128) {
          const int t = wt < s.I ? wt : s.N - s.L + (wt - s.I);
          unsigned cw = wcode;
          if (wt >= NT - 128) cw = src.load_one(t, u, s.cap);
          // (a code outside [0, C) was never counted)
          if ((cw & 0xffu) < (unsigned)s.C && (cw >> 8) < (unsigned)s.C && t != uncounted) atomicAdd(&pl.cnt[(cw & 0xffu) + kPairC * (cw >> 8)], 1u);
        }
      } else {
        count_pairs<NT - 128, kCountEarly>(early, mids, 0, n_early, tid - 128, pl.cnt);
      }
      __syncthreads();
      PQC_MARK(ws, 1, 12);
      const float lo = __fadd_rn(pl.bounds[0], pl.bounds[2]), hi = __fadd_rn(pl.bounds[1], pl.bounds[3]);  // added like a score, so that lo <= score <= hi in fp32
      if constexpr (COUNT) {
        const float inv_u = sample_scale(lo, hi);
#pragma unroll
        for (int x = 0; x < PS; ++x)
          if (x * NT + tid < s.sampleN) atomicAdd(&pl.samples[sample_bin(src.score_one(sample[x]), lo, inv_u)], 1u);
        if (tid < 16 && (tid & 8 ? mids.tail + (tid & 7) < mids.tail_end : mids.head + (tid & 7) < mids.head_end)) {
          unsigned s0, s1;
          pair_slots(edge, s0, s1);
          atomicAdd(&pl.cnt[s0], 1u);
        }
        count_pairs<NT, U>(code, mids, n_early, mids.n, tid, pl.cnt);
        __syncthreads();
      }
      PQC_MARK(ws, 1, 9);
      unsigned count[PER];
#pragma unroll
      for (int i = 0; i < PER; i += 4) {
        const uint4 x = *reinterpret_cast<const uint4*>(&pl.cnt[tid * PER + i]);
        count[i] = x.x; count[i + 1] = x.y; count[i + 2] = x.z; count[i + 3] = x.w;
      }
      if constexpr (PAIRS) {
        const int c0 = (tid * PER) & 63, c1 = (tid * PER) >> 6;
#pragma unroll
        for (int i = 0; i < PER; ++i) count[i] = c1 < s.C && c0 + i < s.C ? given[i / 4][i % 4] - count[i] : 0u;
        pair_classes<NT>(s, lut, lo, hi, count, pl, hist, scan_sm);
        th.bstar = 1;
        __syncthreads();
      } else {
        int b_hi, b_lo;  // (every wave walks the samples by itself)
        walk_samples<false>(pl.samples, s.rankHi, s.rankLo, b_hi, b_lo);
        const BinMap map = window_bins(lo, hi, b_hi, b_lo);
        float sc[PER];
        unsigned bin[PER];
        pair_scores(lut, sc);
#pragma unroll
        for (int i = 0; i < PER; ++i) bin[i] = score_bin(sc[i], map);
        store_classes(pl.cls, bin);
#pragma unroll
        for (int i = 0; i < PER; ++i)
          if (bin[i] && count[i]) atomicAdd(&hist[bin[i]], count[i]);
      }
    } else {
      reinterpret_cast<uint4*>(hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
      const float2 bounds = build_lut<T, NT, LM, decltype(mark), decltype(issue_loads), VW>(qu, cu, G, s.C, lut, qs, lut_red, tile, mark, issue_loads);
      store_query();
      float sample_score[PS];
#pragma unroll
      for (int x = 0; x < PS; ++x) sample_score[x] = src.score_one(sample[x]);
      const BinMap map = sample_window<NT, PS>(bounds.x, bounds.y, sample_score, s.sampleN, s.rankHi, s.rankLo, hist, scan_sm);
      PQC_MARK(ws, 1, 9);
      const OwnTokens mine{own, bx * s.tokC, bx * s.tokC + s.tokC};
      bin_scores<NT, U>(src, code, chunks, s.I, s.N - s.L, mine, map, hist);
    }
    if constexpr (!PAIRS) {
      __syncthreads();
      PQC_MARK(ws, 1, 10);
      ThresholdSearch<NT> ts;
      ts.load(hist, 1);
      th = ts.resolve(s.K, s.N - s.I - s.L, scan_sm);
    }
  } else {
    // this wave's stored bins, the query and the histogram: all requested up front
    const unsigned short* bins_u = ws.bins + (size_t)u * s.binStride;
#pragma unroll
    for (int v = 0; v < GV; ++v)
      raw[v] = *reinterpret_cast<const u32x4_t*>(bins_u + min(wave_t0 + min((v * 64 + lane) * 8, tpw - 8), s.binStride - 8));
    constexpr int QV = ATTN ? (G * kD + NT - 1) / NT : 1;  // query elements per thread
    float qreg[QV];
    if constexpr (ATTN) {
#pragma unroll
      for (int x = 0; x < QV; ++x)
        qreg[x] = load_as_float<T>(q + ((size_t)b * s.Hq + (size_t)g * G) * kD, min(x * NT + tid, G * kD - 1));
    }
    ThresholdSearch<NT> ts;
    ts.load(ws.hist + (size_t)u * s.histCopies * kNB, s.histCopies);
    PQC_LOADS_ISSUED();
    if constexpr (ATTN) {
#pragma unroll
      for (int x = 0; x < QV; ++x)
        if (x * NT + tid < G * kD) qlds[x * NT + tid] = qreg[x];
    }
    th = ts.resolve(s.K, s.N - s.I - s.L, scan_sm);  // syncs: qlds ready
  }
  PQC_MARK(ws, 1, 1);

  const int wg_t0 = bx * s.tokC;
  int place[GV];   // (selected, candidates << 16) of the wave in front of the group
  int count = 0;   // the same, of the wave
  const unsigned thr = (unsigned)th.bstar;
#pragma unroll
  for (int v = 0; v < GV; ++v) {
    if (v < gpw) {  // uniform
      if constexpr (SHORT) raw[v] = *reinterpret_cast<const u32x4_t*>(own + w * tpw + min((v * 64 + lane) * 8, tpw - 8));
      const int t0 = wave_t0 + (v * 64 + lane) * 8;
      unsigned wv[4] = {raw[v].x, raw[v].y, raw[v].z, raw[v].w};  // two tokens each, in stored form: selected above thr, candidates at thr
      if constexpr (PAIRS || COUNT) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          unsigned s0, s1;
          pair_slots(wv[k], s0, s1);
          wv[k] = pl.cls[s0] | ((unsigned)pl.cls[s1] << 16);
        }
        if (__any(t0 < s.I || t0 + 8 > s.N - s.L)) {  // uniform, rare
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
              const int t = t0 + 2 * k + y;
              if (t < s.I || t >= s.N - s.L) wv[k] |= kBinWindow << (16 * y);
            }
        }
      }
      const int nreal = (v * 64 + lane) * 8 < tpw ? min(8, max(0, s.N - t0)) : 0;  // tokens of this group that exist
      if (__any(nreal < 8)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) wv[k] = 2 * k + 1 < nreal ? wv[k] : 2 * k < nreal ? wv[k] & 0xffffu : 0u;
      }
      // counts of the group, two tokens at a time: (0 or 1) for each half of a word
      unsigned above2 = 0u, other2 = 0u;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        above2 += pk_min_u16(pk_sub_sat_u16(wv[k], thr * 0x10001u), 0x10001u);
        other2 += pk_min_u16(wv[k] ^ (thr * 0x10001u), 0x10001u);
      }
      const int n_abv = (int)((above2 & 0xffffu) + (above2 >> 16));
      int n_cnd = 8 - (int)((other2 & 0xffffu) + (other2 >> 16));
      if (thr == 0u) n_cnd = max(0, n_cnd - (8 - nreal));  // uniform, rare: tokens that do not exist look like candidates then
      const int cnt = n_abv | (n_cnd << 16);
      const int inc = wave_inclusive_scan(cnt);
      place[v] = count + inc - cnt;
      count += wave_last(inc);
      raw[v] = u32x4_t{wv[0], wv[1], wv[2], wv[3]};
    }
  }
  PQC_MARK(ws, 1, 8);
  if (lane == 0) wcnt[w] = count;
  __syncthreads();
  int before = 0, total = 0;  // of the waves in front of this one, and of all
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int c = wcnt[i];
    before += i < w ? c : 0;
    total += c;
  }
  const int tot_sel = total & 0xffff, tot_cand = total >> 16;
#pragma unroll
  for (int v = 0; v < GV; ++v) {
    if (v < gpw) {  // uniform
      const unsigned wv[4] = {raw[v].x, raw[v].y, raw[v].z, raw[v].w};
      const int off0 = (wave_t0 - wg_t0) + (v * 64 + lane) * 8;
      int ps = (before + place[v]) & 0xffff;
      // every token is stored, those not selected in a place of the thread's own behind the list: eight stores under conditions of
      // their own are eight branches, and few waves are there to hide them
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const bool sel = ((wv[i >> 1] >> (16 * (i & 1))) & 0xffffu) > thr;
        list[sel ? ps : s.tokC + tid] = (unsigned short)(off0 + i);
        ps += sel ? 1 : 0;
      }
      if (count >> 16) {  // uniform: the wave has candidates; they go to the list's end, backwards
        int pc = (before + place[v]) >> 16;
        const int nreal = off0 < (w + 1) * tpw ? min(8, max(0, s.N - wg_t0 - off0)) : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (i < nreal && ((wv[i >> 1] >> (16 * (i & 1))) & 0xffffu) == thr) list[s.tokC - 1 - (pc++)] = (unsigned short)(off0 + i);
      }
    }
  }
  __syncthreads();
  PQC_MARK(ws, 1, 2);
  // record slots for this workgroup's candidates: requested now, needed only after the
  // attention below, which hides the round trip of the returning atomic
  int rec_base;  // set and read by thread 0 only; no initialiser, or the merge with it would wait for the atomic here
  if (tid == 0 && tot_cand > 0) rec_base = (int)atomicAdd(&ws.cand_count[u], (unsigned)tot_cand);
  // A candidate's exact score comes from its codes and the unit's table (same evaluation order
  // as everywhere), or from the score array of the stand-alone top-k.
  struct CandKey {
    unsigned cb[SRC::kFromCodes ? SRC::M : 1];
    float sc;
  };
  auto cand_token = [&](int c) -> int { return wg_t0 + list[s.tokC - 1 - c]; };
  auto cand_key_load = [&](int t) -> CandKey {
    CandKey k;
    k.sc = 0.0f;
    if constexpr (SRC::kFromCodes) {
      const uint8_t* cp = static_cast<const uint8_t*>(src_ptr) + ((size_t)u * s.cap + t) * SRC::M;
#pragma unroll
      for (int j = 0; j < SRC::M; ++j) k.cb[j] = cp[j];
    } else {
      k.cb[0] = 0u;
      k.sc = static_cast<const float*>(src_ptr)[(size_t)u * s.N + t];
    }
    return k;
  };
  auto cand_score = [&](const CandKey& k) -> float {
    if constexpr (TABLE) {
      float sc = lut[k.cb[0]];
#pragma unroll
      for (int j = 1; j < SRC::M; ++j) sc = __fadd_rn(sc, lut[j * kLutRow + k.cb[j]]);
      return sc;
    } else if constexpr (SRC::kFromCodes) {
      const float* tb = ws.lut + (size_t)u * SRC::M * s.C;
      float sc = tb[k.cb[0]];
#pragma unroll
      for (int j = 1; j < SRC::M; ++j) sc = __fadd_rn(sc, tb[j * s.C + k.cb[j]]);
      return sc;
    } else {
      return k.sc;
    }
  };
  auto sel_at = [&](int p) -> int { return wg_t0 + list[p]; };

  // selected list for the finalize kernel's index output
  unsigned long long* stage = ws.stage + ((size_t)u * s.nblkC + bx) * s.stageStride;
  int* stage32 = reinterpret_cast<int*>(stage);
  PQC_MARK(ws, 1, 3);

  const T* kbase = kc + (size_t)u * s.cap * kD;
  const T* vbase = vc + (size_t)u * s.cap * kD;
  // The first candidates (one per 16-lane group): their codes and K/V rows are requested now, so that
  // after the attention only the table look-up, arithmetic and the record write remain.
  const int sub = lane & 15, grp = tid >> 4;
  int c0_t = 0;
  CandKey c0_key;
  RowRaw<T> c0_k, c0_v;
  c0_key.sc = 0.0f;
#pragma unroll
  for (int j = 0; j < (SRC::kFromCodes ? SRC::M : 1); ++j) c0_key.cb[j] = 0u;
  c0_k.zero();
  c0_v.zero();
  if (grp < tot_cand) {
    c0_t = cand_token(grp);
    c0_key = cand_key_load(c0_t);
    if constexpr (ATTN) {
      c0_k.load(kbase, c0_t, sub);
      c0_v.load(vbase, c0_t, sub);
    }
  }
  // Rows this workgroup attends: its own tokens above the threshold bin, and, instead of the
  // window tokens it happens to hold (the list's first nI and last nL entries), every
  // nblkC-th token of the two windows, so that the window rows are spread over the unit's
  // workgroups.
  const int tok_lo = bx * s.tokC, tok_hi = min(s.N, (bx + 1) * s.tokC);
  const int nI = max(0, min(s.I, tok_hi) - tok_lo), nL = max(0, tok_hi - max(s.N - s.L, tok_lo));
  const int n_own = tot_sel - nI - nL;
  const int n_win = bx < s.I + s.L ? (s.I + s.L - bx + s.nblkC - 1) / s.nblkC : 0;
  const int n_att = n_own + n_win;
  auto att_at = [&](int p) -> int {
    if (p < n_own) return sel_at(p + nI);
    const int wt = bx + (p - n_own) * s.nblkC;
    return wt < s.I ? wt : s.N - s.L + (wt - s.I);
  };
  if constexpr (ATTN) {
    if constexpr (kMfma) {
      bf16x8_t qf[4];
      load_q_frags(reinterpret_cast<const bf16_t*>(q) + ((size_t)b * s.Hq + (size_t)g * G) * kD, G, qf);
      MfmaState st;
      st.init();
      mfma_attend(reinterpret_cast<const bf16_t*>(kbase), reinterpret_cast<const bf16_t*>(vbase), s.N, att_at, n_att,
                  w * 16 * kMfmaTiles, NW * 16 * kMfmaTiles, s.scale_log2e, qf, vtile + w * kVTileBytes, st);
      PQC_MARK(ws, 1, 4);
      mfma_stash_wave_state<G>(st, red);
    } else {
      float qr[G][8];
      load_query<T, G>(q + ((size_t)b * s.Hq + (size_t)g * G) * kD, s.scale_log2e, qr);
      AttnState<G> st;
      st.init();
      constexpr int R = (G >= 8 || sizeof(T) == 4) ? 2 : 4;
      attend_rows<T, G, R>(kbase, vbase, s.N, att_at, n_att, w * 4 * R, NW * 4 * R, qr, st);
      PQC_MARK(ws, 1, 4);
      stash_wave_state<T, G>(st, red);
    }
    __syncthreads();
    // this workgroup's partial state: the accumulators as 128 floats per head ([j][h][kD] over the unit's workgroups j),
    // the (m, l) pairs in a dense array per head behind all accumulators ([units][h][j]); see finalize_kernel
    float* pacc = ws.partials + (((size_t)u * s.npart + bx) * G) * kD;
    float2* pml = reinterpret_cast<float2*>(ws.partials + (size_t)s.B * s.Hkv * s.npart * G * kD) + (size_t)u * G * s.npart + bx;
    for (int o = tid; o < G * kD; o += NT) {
      const int h = o / kD, d = o % kD;
      float m, l, acc;
      combine_waves<G, NW>(red, h, d, m, l, acc);
      pacc[h * kD + d] = acc;
      if (d == 0) pml[(size_t)h * s.npart] = make_float2(m, l);
    }
  }
  // (written after the attention: stores issued while the K/V loads of the co-resident workgroup
  // fill the memory pipeline would only delay this workgroup's own first loads)
  for (int p = tid; p < tot_sel; p += NT) stage32[p] = sel_at(p);
  if (tid == 0) ws.stage_cnt[(size_t)u * s.nblkC + bx] = make_int2(tot_sel, tot_cand);
  PQC_MARK(ws, 1, 5);
  PQC_NOTE(ws, 1, 14, tot_sel);
  PQC_NOTE(ws, 1, 15, tot_cand);

  // candidates (few): composite for the generic path, and a full record while slots last
  if (tot_cand > 0) {  // workgroup-uniform
    if (tid == 0) scan_sm[0] = rec_base;
    __syncthreads();
    const int base = scan_sm[0];
    for (int c = grp; c < tot_cand; c += NT / 16) {
      int t = c0_t;
      CandKey key = c0_key;
      RowRaw<T> kr = c0_k, vr = c0_v;
      if (c >= NT / 16) {  // beyond the candidates whose loads went out before the attention
        t = cand_token(c);
        key = cand_key_load(t);
        if constexpr (ATTN) {
          kr.load(kbase, t, sub);
          vr.load(vbase, t, sub);
        }
      }
      const unsigned long long comp = make_composite(cand_score(key), t);
      if (sub == 0) stage[s.tokC - 1 - c] = comp;
      if (base + c < kCandRec) {
        const CandView cv = cand_view(ws.cand_rec + (size_t)u * ws.rec_stride, ATTN ? G : 1);
        if (sub == 0) cv.composite[base + c] = comp;
        if constexpr (ATTN) {
          float kf[8];
          kr.unpack(kf);
#pragma unroll
          for (int h = 0; h < G; ++h) {
            float d = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) d = fmaf(qlds[h * kD + owned_dim<T>(sub, e)], kf[e], d);
            d = group16_sum(d);
            if (sub == 0) cv.logit[h * kCandRec + base + c] = d;
          }
          vr.store(cv.v + (size_t)(base + c) * kD * sizeof(T), sub);
        }
      }
    }
  }
}

// ------------------------------------------------------------- 3. finalize
// Grid (heads * SL + s.copyWgs, units), 512 threads; heads = the group's query heads, SL = Shape::slices (one
// head, one slice for the stand-alone top-k).
//   blockIdx.x <  heads * SL  slice blockIdx.x % SL of head blockIdx.x / SL: ranks the candidates and
//                        folds the admitted ones and all partial softmax states into kD / SL dimensions
//                        of this head's output; workgroup 0 also writes the admitted candidates'
//                        indices (best first)
//   blockIdx.x >= heads * SL  copy workgroups: concatenate the staged lists into out_idx; the
//                        first one also zeroes the unit's histogram and record counter
// The staged "selected" lists already hold the two windows: in workgroup order they read
//   [0..I) , tokens above the threshold bin (ascending) , [N-L..N).
// Fast path (at most kCandRec candidates): all a head needs is in the candidate records,
// which sit densely in order of arrival.  That order differs from run to run, so every
// sum over candidates is taken in rank order.  Generic path: candidates are the
// composites staged per select workgroup; admitted rows are gathered from the K/V cache.
template <int NT>
__device__ __forceinline__ float block_max(float v, float* sm /* [NT/64] */) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = sm[0];
#pragma unroll
  for (int i = 1; i < NT / 64; ++i) r = fmaxf(r, sm[i]);
  __syncthreads();
  return r;
}
template <int NT>
__device__ __forceinline__ float block_sum(float v, float* sm /* [NT/64] */) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = sm[0];
#pragma unroll
  for (int i = 1; i < NT / 64; ++i) r += sm[i];
  __syncthreads();
  return r;
}

// 512 threads: a head's work is a chain of short steps, alone on its compute unit with nothing to hide their latency, and what a thread
// does of each is half of what it is with 256 (from the first workgroup's start to the last one's end, 8 x 131072 tokens, 2x64: 5.4 us, now
// 4.5; 8 x 32768: 4.7, now 3.9; 64 x 32768, 4x256: 5.0 both, bound by what it reads).
constexpr int kFinalThreads = 512;
constexpr int kHdrPerThread = kCandRec / kFinalThreads;  // candidate record headers per thread
constexpr int kAccPer = 4;                     // partial states a thread keeps in flight at once
constexpr int kVPer = 6;                       // candidate records per thread whose V values are requested before the ranking knows which are admitted (96 records
                                               // with sixteen threads per dimension: tie classes of two-partition tables reach 70 tokens at 128K)
constexpr int kVPerFew = 4;                    // the same without large tie classes, or with fewer threads per dimension (many units)
constexpr int kManyCand = 4096;                // candidates whose composites the path for large tie classes keeps in LDS
constexpr int kRankStep = 8;                    // composites read per step of the ranking loop
constexpr int kFoldRanks = 96;                 // admitted rows whose terms meet in LDS by rank (beyond: fetched by rank from the records)
constexpr int kMaxSlices = 4;                  // workgroups per query head, at most (32 output dimensions each)
constexpr int kIdxLists = 4;                   // staged index lists a wave copies with loads issued up front

// dynamic LDS of finalize_kernel
inline size_t finalize_lds_bytes(const Shape& s, bool attn) {
  const size_t terms = attn ? (size_t)(kFoldRanks + 1) * (kD / s.slices) * sizeof(float) : 0;  // and a spare row
  const size_t many = (size_t)kManyCand * (sizeof(unsigned long long) + sizeof(int));  // the same region, when a unit has more than kCandRec candidates
  return (size_t)(4 * s.nblkC + 2) * sizeof(int) + (terms > many ? terms : many);
}

// The code of one appended token per unit (Section 3.1: nearest centroid of each partition): nothing in the
// step depends on it, so one more workgroup per unit of the finalize kernel computes it beside the others.
struct AppendArgs {
  const void* key;    // [units][kD] in the cache's element type, or null: nothing to append
  const float* cent;  // [units][M][C][Dm]
  uint8_t* codes;     // the code tensor; written at `position` of every unit
  int position;
  unsigned* pair_counts;  // two partitions: [units][C*C] counts that gain the token's code pair, or null
};

// acc += sum_x w_j a_x, l += sum_x w_j l_j over the states j = first, first + step, ... below n, with w_j = exp2(m_j - m*).
template <int U>
__device__ __forceinline__ void fold_states(const float* pm, const float* pl, float mstar, int first, int step, int n, const float (&a)[U], float& acc,
                                            float& lsum) {
  float m[U], l[U];
#pragma unroll
  for (int x = 0; x < U; ++x) {
    const int j = min(first + step * x, n - 1);
    m[x] = pm[j];
    l[x] = pl[j];
  }
#pragma unroll
  for (int x = 0; x < U; ++x) {
    const float w = __builtin_amdgcn_exp2f(m[x] - mstar), na = fmaf(w, a[x], acc), nl = fmaf(w, l[x], lsum);
    acc = first + step * x < n ? na : acc;  // (a state that is not there may hold infinities)
    lsum = first + step * x < n ? nl : lsum;
  }
}

// WIDE: four workgroups per head (sixteen threads per output dimension) and large tie classes; they request more candidate records up front.
// (Four waves per SIMD, so that two workgroups share a compute unit: fp32 would take 129 to 131 registers instead of 128, and then a
// compute unit holds one.  200 units of 2056 tokens, 2x64, fp32, two query heads: 13.5 us, now 9.1.)
template <typename T, int G, bool ATTN, bool WIDE = false>
__global__ __launch_bounds__(kFinalThreads, ATTN && sizeof(T) == 4 ? 4 : 2) void finalize_kernel(Shape s, Workspace ws, const T* __restrict__ q,
                                                       const T* __restrict__ kc, const T* __restrict__ vc,
                                                       int* __restrict__ out_idx, float* __restrict__ out_attn, AppendArgs ap) {
  constexpr int NT = kFinalThreads, NW = NT / 64;
  constexpr int heads = ATTN ? G : 1;
  constexpr int VPER = WIDE ? kVPer : kVPerFew;
  const int SL = ATTN ? s.slices : 1;  // head workgroups per head
  if ((int)blockIdx.x == heads * SL + s.copyWgs) {
    // -------------------------------------------------------------- append workgroup
    // one thread per centroid, the distance chain of pq_round_vector_kernel, the smallest (distance, centroid) pair
    // of each partition through a 64-bit LDS minimum
    __shared__ float ax[kD];
    __shared__ unsigned long long abest[8];
    const int u = blockIdx.y, c = threadIdx.x;
    if (c < kD) ax[c] = load_as_float<T>(static_cast<const T*>(ap.key), (size_t)u * kD + c);
    if (c < 8) abest[c] = ~0ull;
    __syncthreads();
    if (c < s.C) {
      for (int j = 0; j < s.M; ++j) {
        const float* cr = ap.cent + (((size_t)u * s.M + j) * s.C + c) * s.Dm;
        const float* xj = ax + j * s.Dm;
        float d2 = 0.0f;
        for (int e = 0; e < s.Dm; e += 4) {  // Dm is a multiple of 4
          const float4 cv = *reinterpret_cast<const float4*>(cr + e);
          float df = xj[e] - cv.x;
          d2 = fmaf(df, df, d2);
          df = xj[e + 1] - cv.y;
          d2 = fmaf(df, df, d2);
          df = xj[e + 2] - cv.z;
          d2 = fmaf(df, df, d2);
          df = xj[e + 3] - cv.w;
          d2 = fmaf(df, df, d2);
        }
        atomicMin(&abest[j], ((unsigned long long)__float_as_uint(d2) << 32) | (unsigned)c);  // d2 >= 0: bits order like values
      }
    }
    __syncthreads();
    if (c < s.M) ap.codes[((size_t)u * s.cap + ap.position) * s.M + c] = (uint8_t)(abest[c] & 0xffu);
    if (c == 0 && ap.pair_counts) ap.pair_counts[(size_t)u * s.C * s.C + (abest[0] & 0xffu) + s.C * (abest[1] & 0xffu)] += 1u;
    return;
  }
  extern __shared__ int dyn[];  // pre_sel[nblkC+1], pre_cand[nblkC+1], pm[nblkC], pl[nblkC], then terms[kFoldRanks][kD/slices] or, with
                                // more than kCandRec candidates, their composites and the admitted tokens (finalize_lds_bytes)
  __shared__ int scan_sm[2 * NW + 1];
  __shared__ float fsm[NW];
  __shared__ int ism[2 * NW];
  __shared__ unsigned long long comp[kCandRec + kRankStep];  // candidate composites, in record order
  __shared__ float lgk[kCandRec];                // by rank: logit, then softmax weight of the admitted ones
  __shared__ unsigned short ordv[kCandRec];      // by rank: record
  __shared__ unsigned short rankv[kCandRec];     // by record: rank
  __shared__ unsigned mkey;                      // order-preserving key of the largest logit (states and admitted rows)
  __shared__ unsigned rhist[256];
  __shared__ int digit_sm[2];
  __shared__ int rows_sm[NT];
  __shared__ float red[ATTN ? NW * (kD + 2) : 1];
  __shared__ float part_acc[ATTN ? NT : 1];
  __shared__ float slice_sm[ATTN ? NT : 1];  // [threads per dimension][dimensions of the workgroup]
  __shared__ float lsm[NW];
  const int u = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int b = u / s.Hkv, g = u % s.Hkv;
  int* pre_sel = dyn;
  int* pre_cand = dyn + (s.nblkC + 1);
  float* pm = reinterpret_cast<float*>(dyn + 2 * (s.nblkC + 1));
  float* pl = pm + s.nblkC;
  float* terms = pl + s.nblkC;  // [kFoldRanks + 1][dimensions of the workgroup]: weighted V values of the admitted rows, by rank
  const int2* cnt = ws.stage_cnt + (size_t)u * s.nblkC;
  const unsigned long long* stage_u = ws.stage + (size_t)u * s.nblkC * s.stageStride;
  int* out = out_idx + (size_t)u * s.Ktot;
  PQC_MARK(ws, 2, 0);

  // exclusive prefix sums of the per-workgroup list sizes (into LDS); returns the totals
  auto scan_counts = [&](const int2 cnt0, int& n_list, int& n_cand) {
    int carry_s = 0, carry_c = 0;
    for (int j0 = 0; j0 < s.nblkC; j0 += NT) {
      const int j = j0 + tid;
      const int2 c = j < s.nblkC ? (j0 == 0 ? cnt0 : cnt[j]) : make_int2(0, 0);
      int ts, tc;
      const int ps = block_exclusive_scan<NT>(c.x, &ts, scan_sm);
      const int pc = block_exclusive_scan<NT>(c.y, &tc, scan_sm);
      if (j < s.nblkC) {
        pre_sel[j] = carry_s + ps;
        pre_cand[j] = carry_c + pc;
      }
      carry_s += ts;
      carry_c += tc;
    }
    if (tid == 0) {
      pre_sel[s.nblkC] = carry_s;
      pre_cand[s.nblkC] = carry_c;
    }
    __syncthreads();
    n_list = carry_s;
    n_cand = carry_c;
  };

  if ((int)blockIdx.x >= heads * SL) {
    // ---------------------------------------------------------------- copy workgroup
    // a wave copies 256 entries of a list at a time, coalesced; with fewer lists than waves several waves share a list, with more a wave
    // takes every so manieth list as a whole.  The local window moves behind the admitted candidates.
    const int cw = blockIdx.x - heads * SL, waves = s.copyWgs * NW, wid = cw * NW + w;
    const int shares = max(1, waves / s.nblkC);              // waves per list
    const int j_first = wid / shares, share = wid % shares;  // this wave's (first) list, and which of its waves it is
    const int j_step = shares > 1 ? s.nblkC : waves;
    const int2 cnt0 = cnt[min(tid, s.nblkC - 1)];
    int ix[kIdxLists][4];  // its first 256 * kIdxLists entries, or those 256 of its first kIdxLists lists
    auto list_at = [&](int j) { return reinterpret_cast<const int*>(stage_u + (size_t)min(j, s.nblkC - 1) * s.stageStride); };
#pragma unroll
    for (int x = 0; x < kIdxLists; ++x) {
      const int* src = list_at(shares > 1 ? j_first : j_first + x * j_step);
      const int p0 = shares > 1 ? (share + x * shares) * 256 : 0;
#pragma unroll
      for (int y = 0; y < 4; ++y) ix[x][y] = src[min(p0 + y * 64 + lane, 2 * s.tokC - 1)];
    }
    PQC_LOADS_ISSUED();
    int n_list, n_cand;
    scan_counts(cnt0, n_list, n_cand);
    const int n_above = max(0, n_list - s.I - s.L);
    const int need = max(0, min(s.K - n_above, n_cand));
    PQC_MARK(ws, 2, 1);
    int x = 0;  // of the pieces requested above
    for (int j = j_first; j < s.nblkC; j += j_step) {
      const int base = pre_sel[j], n = pre_sel[j + 1] - base;
      const int* src = list_at(j);
      for (int p0 = share * 256; p0 < n; p0 += shares * 256) {
        int v[4];
        if (x < kIdxLists && (shares > 1 || p0 == 0)) {
#pragma unroll
          for (int y = 0; y < 4; ++y) v[y] = x == 0 ? ix[0][y] : x == 1 ? ix[1][y] : x == 2 ? ix[2][y] : ix[3][y];
        } else {
#pragma unroll
          for (int y = 0; y < 4; ++y)
            if (p0 + y * 64 + lane < n) v[y] = src[p0 + y * 64 + lane];
        }
        if (shares > 1) ++x;
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          const int pos = base + p0 + y * 64 + lane;
          // (the bound only matters when the caller's pair counts do not belong to the codes: then n_above can exceed K)
          const int dst = pos < s.I + n_above ? pos : pos + need;
          if (p0 + y * 64 + lane < n && dst < s.Ktot) out[dst] = v[y];
        }
      }
      if (shares == 1) ++x;
    }
    PQC_MARK(ws, 2, 4);
    if (cw == 0) {  // the select kernel was their last reader: zero histogram and record counter for the next call
      unsigned* gh = ws.hist + (size_t)u * s.histCopies * kNB;
      for (int i = tid; i < s.histCopies * kNB; i += NT) gh[i] = 0u;
      if (tid == 0) ws.cand_count[u] = 0u;
    }
    PQC_MARK(ws, 2, 5);
    return;
  }

  // ------------------------------------------------------------------ head workgroup
  // One of SL workgroups of query head hq: it produces output dimensions [dims*sl, dims*sl + dims), dims = kD / SL.
  // A compute unit reads what other compute units wrote at a small fraction of the chip's bandwidth (about a hundred
  // cache lines per microsecond), so with few units the partial states of a head are spread over several workgroups,
  // each reading only its dimensions of every state, and everything a workgroup reads of the candidates is dense.
  const int hq = (int)blockIdx.x / SL, sl = (int)blockIdx.x % SL;
  const int dims = kD / SL, nps = NT / dims;   // output dimensions of this workgroup; threads per dimension (4, 8 or 16)
  const int dl = tid & (dims - 1), ps = tid / dims;  // dimension inside the slice; which share of the states and admitted rows
  const int d = dims * sl + dl;
  const int units = s.B * s.Hkv;
  // ---- everything whose address is known up front is requested first
  const CandView cv = cand_view(ws.cand_rec + (size_t)u * ws.rec_stride, heads);
  unsigned long long rc[kHdrPerThread];  // candidate x*NT + tid; the first 256 are requested up front
  float rl[kHdrPerThread];
  rc[0] = cv.composite[tid & 255];
  rl[0] = ATTN ? cv.logit[hq * kCandRec + (tid & 255)] : 0.0f;
  const float* pacc = ws.partials + (size_t)u * s.npart * G * kD;                                   // [j][h][kD]
  const float2* pml = reinterpret_cast<const float2*>(ws.partials + (size_t)units * s.npart * G * kD) +
                      ((size_t)u * G + hq) * s.npart;                                                // [j] of this head
  const int jc = min(tid, s.nblkC - 1);
  const int2 cnt0 = cnt[jc];  // list sizes of the first NT select workgroups
  float2 ml0 = make_float2(kNegBig, 0.0f);
  float a0[kAccPer];  // this thread's first states: ps, ps + nps, ...
  float vv0[VPER];    // V values of the candidate records ps, ps + nps, ... (this thread's dimension)
  if constexpr (ATTN) {
    ml0 = pml[jc];
#pragma unroll
    for (int x = 0; x < kAccPer; ++x)  // states that do not exist re-read the first one (a cache hit, no extra traffic)
      a0[x] = pacc[((size_t)(ps + nps * x < s.nblkC ? ps + nps * x : 0) * G + hq) * kD + d];
    // the V values of the first candidates (in order of arrival), this workgroup's dimensions: which of them are
    // admitted is known only after the ranking, but requested now they are here by then
#pragma unroll
    for (int x = 0; x < VPER; ++x)
      vv0[x] = load_as_float<T>(reinterpret_cast<const T*>(cv.v) + (size_t)(ps + nps * x) * kD, d);
  }
  PQC_LOADS_ISSUED();
  float mpart = kNegBig;  // largest maximum of the partial states
  if constexpr (ATTN) {
    if (tid < s.nblkC) {
      pm[tid] = ml0.x;
      pl[tid] = ml0.y;
      mpart = ml0.x;
    }
    for (int j = NT + tid; j < s.nblkC; j += NT) {  // beyond the first NT lists (very long contexts)
      const float2 v = pml[j];
      pm[j] = v.x;
      pl[j] = v.y;
      mpart = fmaxf(mpart, v.x);
    }
  }
  // totals of the per-workgroup list sizes, and that maximum (one barrier)
  int n_list, n_cand;
  {
    int ss = tid < s.nblkC ? cnt0.x : 0, sc = tid < s.nblkC ? cnt0.y : 0;
    for (int j = NT + tid; j < s.nblkC; j += NT) {
      const int2 c = cnt[j];
      ss += c.x;
      sc += c.y;
    }
    ss = wave_last(wave_inclusive_scan(ss));
    sc = wave_last(wave_inclusive_scan(sc));
    mpart = wave_max(mpart);
    if (lane == 0) {
      ism[w] = ss;
      ism[NW + w] = sc;
      fsm[w] = mpart;
    }
    __syncthreads();  // also: pm, pl visible
    n_list = 0;
    n_cand = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      n_list += ism[i];
      n_cand += ism[NW + i];
      mpart = fmaxf(mpart, fsm[i]);
    }
  }
  const int n_above = max(0, n_list - s.I - s.L);  // n_list = I + (tokens above the bin) + L
  const int need = max(0, min(s.K - n_above, n_cand));
  PQC_MARK(ws, 2, 1);

  if (n_cand <= kCandRec) {
    // rank every candidate (count of larger composites); the admitted ones are the `need` best
    const bool meet = ATTN && need <= kFoldRanks;  // the admitted rows' terms meet in LDS, by rank
    if (need > 0) {
#pragma unroll
      for (int x = 0; x < kHdrPerThread; ++x) {
        if (x > 0) {
          rc[x] = 0ull;
          rl[x] = 0.0f;
        }
        if (x * NT + tid < n_cand && (x > 0 || tid >= 256)) {  // rare: more than 256 candidates
          rc[x] = cv.composite[x * NT + tid];
          rl[x] = ATTN ? cv.logit[hq * kCandRec + x * NT + tid] : 0.0f;
        }
      }
      // (entries up to the next multiple of kRankStep are zero, which ranks behind everything: the loop below reads
      // kRankStep composites at a time, because one LDS read per step is a chain of latencies)
#pragma unroll
      for (int x = 0; x < kHdrPerThread; ++x)
        if (x * NT + tid < n_cand + kRankStep) comp[x * NT + tid] = x * NT + tid < n_cand ? rc[x] : 0ull;
      if (tid == 0) mkey = score_key(mpart);
      __syncthreads();
#pragma unroll
      for (int x = 0; x < kHdrPerThread; ++x) {
        const int k = x * NT + tid;
        if (k < n_cand) {
          const unsigned long long mine = rc[x];
          int rank = 0;
          for (int j0 = 0; j0 < n_cand; j0 += kRankStep) {
            unsigned long long c[kRankStep];
#pragma unroll
            for (int y = 0; y < kRankStep; ++y) c[y] = comp[j0 + y];
#pragma unroll
            for (int y = 0; y < kRankStep; ++y) rank += c[y] > mine ? 1 : 0;
          }
          rankv[k] = (unsigned short)rank;
          if (rank < need) {
            if (blockIdx.x == 0 && s.I + n_above + rank < s.Ktot) out[s.I + n_above + rank] = composite_token(mine);  // best first
            const float lg = rl[x] * s.scale_log2e;
            lgk[rank] = lg;
            ordv[rank] = (unsigned short)k;
            if constexpr (ATTN) atomicMax(&mkey, score_key(lg));
          }
        }
      }
      __syncthreads();
    }
    if constexpr (ATTN) {
      // out[d] = (sum_j w_j acc_j[d] + sum_r p_r V_r[d]) / l with w_j = exp2(m_j - m*), p_r = exp2(logit_r - m*):
      // nps threads per dimension, thread ps taking the states j = ps (mod nps) and the admitted rows r = ps (mod nps),
      // each in ascending order; the nps sums are added in order.  m* is the larger of the states' maximum (it came
      // with the totals above) and the admitted logits' maximum (an LDS maximum taken while ranking); the threads of
      // dimension 0 sum l alongside.
      const float mstar = need > 0 ? key_score(mkey) : mpart;
      if (meet && need > 0) {
        // the V values requested up front belong to the records ps + nps x in order of arrival; each admitted one's
        // term goes to the row of its rank, so that the sums below run in rank order whatever the order of arrival
        for (int k0 = 0; k0 < n_cand; k0 += nps * VPER) {
          if (k0 > 0) {  // rare: more candidates than the up-front loads cover
#pragma unroll
            for (int x = 0; x < VPER; ++x)
              vv0[x] = load_as_float<T>(reinterpret_cast<const T*>(cv.v) + (size_t)min(k0 + ps + nps * x, kCandRec - 1) * kD, d);
          }
          // (half of them at a time, all look-ups of a kind before the first of the next: one after the other they are a chain of LDS
          // latencies; records that are not admitted go to a spare row)
          constexpr int H = VPER / 2;
#pragma unroll
          for (int x0 = 0; x0 < VPER; x0 += H) {
            if (k0 + nps * x0 >= n_cand) break;  // uniform
            int r[H];
            float lg[H];
#pragma unroll
            for (int x = 0; x < H; ++x) r[x] = rankv[min(k0 + ps + nps * (x0 + x), kCandRec - 1)];
#pragma unroll
            for (int x = 0; x < H; ++x) {
              r[x] = k0 + ps + nps * (x0 + x) < n_cand && r[x] < need ? r[x] : kFoldRanks;
              lg[x] = lgk[min(r[x], need - 1)];
            }
#pragma unroll
            for (int x = 0; x < H; ++x) terms[r[x] * dims + dl] = __builtin_amdgcn_exp2f(lg[x] - mstar) * vv0[x0 + x];
          }
        }
      }
      float acc = 0.0f, lsum = 0.0f;
      fold_states<kAccPer>(pm, pl, mstar, ps, nps, s.nblkC, a0, acc, lsum);
      for (int j0 = nps * kAccPer + ps; j0 < s.nblkC; j0 += nps * kAccPer) {
        float a[kAccPer];
#pragma unroll
        for (int x = 0; x < kAccPer; ++x) a[x] = pacc[((size_t)min(j0 + nps * x, s.nblkC - 1) * G + hq) * kD + d];
        fold_states<kAccPer>(pm, pl, mstar, j0, nps, s.nblkC, a, acc, lsum);
      }
      if (meet) {
        if (need > 0) __syncthreads();  // (need is uniform over the workgroup)
        for (int r0 = ps; r0 < need; r0 += nps * 4) {
          float t[4], lg[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const int r = min(r0 + nps * x, need - 1);
            t[x] = terms[r * dims + dl];
            lg[x] = lgk[r];
          }
#pragma unroll
          for (int x = 0; x < 4; ++x)
            if (r0 + nps * x < need) {
              acc += t[x];
              lsum += __builtin_amdgcn_exp2f(lg[x] - mstar);
            }
        }
      } else {
        // more admitted rows than the LDS rows hold (a large tie class at the threshold): fetched by rank
        for (int r0 = ps; r0 < need; r0 += nps * kAccPer) {
          float vv[kAccPer];
#pragma unroll
          for (int x = 0; x < kAccPer; ++x)
            vv[x] = load_as_float<T>(reinterpret_cast<const T*>(cv.v) + (size_t)ordv[min(r0 + nps * x, need - 1)] * kD, d);
#pragma unroll
          for (int x = 0; x < kAccPer; ++x) {
            const int r = r0 + nps * x;
            if (r < need) {
              acc += __builtin_amdgcn_exp2f(lgk[r] - mstar) * vv[x];
              lsum += __builtin_amdgcn_exp2f(lgk[r] - mstar);
            }
          }
        }
      }
      // waves that hold two shares of 32 dimensions add them up first: then there are eight shares, or four of 128 dimensions
      if (dims == 32) {  // uniform
        acc += __shfl_xor(acc, 32);
        lsum += __shfl_xor(lsum, 32);
      }
      const int shares = dims == kD ? NT / kD : NW, share = dims == kD ? ps : w;
      if (dims > 32 || lane < 32) slice_sm[share * dims + dl] = acc;
      if (dl == 0) lsm[share] = lsum;
      __syncthreads();
      PQC_MARK(ws, 2, 2);
      if (tid < dims) {
        float ts[NW], ls[NW];
#pragma unroll
        for (int x = 0; x < NW; ++x) {
          ts[x] = slice_sm[min(x, shares - 1) * dims + tid];
          ls[x] = lsm[min(x, shares - 1)];
        }
        float tot = ts[0], lstar = ls[0];
#pragma unroll
        for (int x = 1; x < NW; ++x)
          if (x < shares) {
            tot += ts[x];
            lstar += ls[x];
          }
        out_attn[((size_t)b * s.Hq + (size_t)g * G + hq) * kD + dims * sl + tid] = tot / lstar;
      }
      PQC_MARK(ws, 2, 3);
    }
  } else if (sl == 0) {
    // generic path (one workgroup per head does all 128 dimensions): radix select of the need-th largest staged
    // composite, 8 bits per pass
    const int d128 = tid & (kD - 1), part = tid / kD;
    {
      int nl, nc;
      scan_counts(cnt0, nl, nc);
    }
    auto owner = [&](int p) -> int {  // largest j with pre_cand[j] <= p
      int lo = 0, hi = s.nblkC - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre_cand[mid] <= p) lo = mid; else hi = mid - 1;
      }
      return lo;
    };
    auto cand_global = [&](int i) -> unsigned long long {
      const int j = owner(i);
      return stage_u[(size_t)j * s.stageStride + s.tokC - 1 - (i - pre_cand[j])];
    };
    // Up to kManyCand composites are fetched once into LDS (every pass over them would otherwise be a chain of
    // memory round trips); the bytes that all of them share (the whole score, when the candidates are one tie
    // class) need no radix pass.
    unsigned long long* gcomp = reinterpret_cast<unsigned long long*>(terms);  // [kManyCand]
    int* gtok = reinterpret_cast<int*>(gcomp + kManyCand);                     // [kManyCand] admitted tokens, in candidate order
    const bool cached = n_cand <= kManyCand;
    unsigned long long varying = ~0ull, common = 0ull;
    if (cached && need > 0) {
      unsigned long long a_and = ~0ull, a_or = 0ull;
      for (int i0 = 0; i0 < n_cand; i0 += 4 * NT) {
        unsigned long long c[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) c[x] = cand_global(min(i0 + x * NT + tid, n_cand - 1));
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int i = i0 + x * NT + tid;
          if (i < n_cand) {
            gcomp[i] = c[x];
            a_and &= c[x];
            a_or |= c[x];
          }
        }
      }
      if (tid < 4) rhist[tid] = tid < 2 ? 0xffffffffu : 0u;
      __syncthreads();
      atomicAnd(&rhist[0], (unsigned)a_and);
      atomicAnd(&rhist[1], (unsigned)(a_and >> 32));
      atomicOr(&rhist[2], (unsigned)a_or);
      atomicOr(&rhist[3], (unsigned)(a_or >> 32));
      __syncthreads();
      common = ((unsigned long long)rhist[1] << 32) | rhist[0];
      varying = common ^ (((unsigned long long)rhist[3] << 32) | rhist[2]);
      __syncthreads();
    }
    auto cand_at = [&](int i) -> unsigned long long { return cached ? gcomp[i] : cand_global(i); };
    unsigned long long thr = ~0ull;
    if (need > 0) {
      unsigned long long prefix = 0;
      int want = need;
      for (int shift = 56; shift >= 0; shift -= 8) {
        if (((varying >> shift) & 0xffull) == 0) {  // uniform: every candidate has this byte
          prefix |= common & (0xffull << shift);
          continue;
        }
        if (tid < 256) rhist[tid] = 0u;
        __syncthreads();
        for (int i = tid; i < n_cand; i += NT) {
          const unsigned long long c = cand_at(i);
          if (shift == 56 || (c >> (shift + 8)) == (prefix >> (shift + 8))) atomicAdd(&rhist[(unsigned)(c >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (tid == 0) {
          int cum = 0, dg = 255;
          for (; dg > 0; --dg) {
            if (cum + (int)rhist[dg] >= want) break;
            cum += (int)rhist[dg];
          }
          digit_sm[0] = dg;
          digit_sm[1] = want - cum;
        }
        __syncthreads();
        prefix |= (unsigned long long)digit_sm[0] << shift;
        want = digit_sm[1];
        __syncthreads();
      }
      thr = prefix;
    }
    // admitted candidates in token order: indices out, rows attended (all at once when they fit the LDS list, else
    // NT candidates per round)
    AttnState<1> st;
    st.init();
    float qr[1][8];
    if constexpr (ATTN) load_query<T, 1>(q + ((size_t)b * s.Hq + (size_t)g * G + hq) * kD, s.scale_log2e, qr);
    int carry = 0;
    for (int i0 = 0; i0 < (need > 0 ? n_cand : 0); i0 += NT) {
      const int i = i0 + tid;
      unsigned long long c = 0;
      if (i < n_cand) c = cand_at(i);
      const int flag = (i < n_cand && c >= thr) ? 1 : 0;
      int tot;
      const int pos = block_exclusive_scan<NT>(flag, &tot, scan_sm);
      if (flag) {
        if (cached) gtok[carry + pos] = composite_token(c); else rows_sm[pos] = composite_token(c);
        if (hq == 0 && s.I + n_above + carry + pos < s.Ktot) out[s.I + n_above + carry + pos] = composite_token(c);
      }
      if (!cached) {
        __syncthreads();
        if constexpr (ATTN) {
          auto row_at = [&](int p) -> int { return rows_sm[p]; };
          attend_rows<T, 1, 4>(kc + (size_t)u * s.cap * kD, vc + (size_t)u * s.cap * kD, s.N, row_at, tot, w * 16, NW * 16, qr, st);
        }
        __syncthreads();
      }
      carry += tot;
    }
    if (cached) {
      __syncthreads();
      if constexpr (ATTN) {
        auto row_at = [&](int p) -> int { return gtok[p]; };
        attend_rows<T, 1, 4>(kc + (size_t)u * s.cap * kD, vc + (size_t)u * s.cap * kD, s.N, row_at, carry, w * 16, NW * 16, qr, st);
      }
    }
    if constexpr (ATTN) {
      stash_wave_state<T, 1>(st, red);
      __syncthreads();
      float m_own, l_own, acc;
      combine_waves<1, NW>(red, 0, d128, m_own, l_own, acc);
      float mx = m_own;
      for (int j = tid; j < s.nblkC; j += NT) mx = fmaxf(mx, pm[j]);
      const float mstar = block_max<NT>(mx, fsm);
      float lsum = 0.0f;
      for (int j = tid; j < s.nblkC; j += NT) {
        const float wj = __builtin_amdgcn_exp2f(pm[j] - mstar);
        pm[j] = wj;
        lsum = fmaf(wj, pl[j], lsum);
      }
      const float f_own = __builtin_amdgcn_exp2f(m_own - mstar);
      const float lstar = block_sum<NT>(lsum, fsm) + l_own * f_own;
      acc = part == 0 ? acc * f_own : 0.0f;
      for (int j = part; j < s.nblkC; j += NT / kD) acc = fmaf(pm[j], pacc[((size_t)j * G + hq) * kD + d128], acc);
      part_acc[tid] = acc;
      __syncthreads();
      if (part == 0) {
#pragma unroll
        for (int x = 1; x < NT / kD; ++x) acc += part_acc[x * kD + d128];
        out_attn[((size_t)b * s.Hq + (size_t)g * G + hq) * kD + d128] = acc / lstar;
      }
    }
  }
  PQC_NOTE(ws, 2, 13, n_above);
  PQC_NOTE(ws, 2, 14, n_cand);
  PQC_NOTE(ws, 2, 15, need);
}

// ---------------------------------------------- stand-alone attention over a list
// pqc_gather_attn: workgroup x of unit u attends list positions [x*rowsP, +rowsP).
template <typename T, int G>
__global__ __launch_bounds__(256) void attn_list_kernel(Shape s, Workspace ws, const T* __restrict__ q,
                                                        const T* __restrict__ kc, const T* __restrict__ vc,
                                                        const int* __restrict__ idx) {
  constexpr int NT = 256, NW = 4;
  constexpr bool kMfma = sizeof(T) == 2 && kMatrixCoreAttention;
  __shared__ float red[NW * G * (kD + 2)];
  __shared__ __attribute__((aligned(16))) unsigned char vtile[kMfma ? NW * kVTileBytes : 16];
  const int u = blockIdx.y, tid = threadIdx.x, w = tid >> 6;
  const int b = u / s.Hkv, g = u % s.Hkv;
  const int p0 = blockIdx.x * s.rowsP;
  const int count = min(s.rowsP, s.Ktot - p0);
  // this workgroup's slice of the list goes to LDS first: one coalesced load instead of a
  // dependent global load in front of every stage of row loads
  extern __shared__ int lst[];  // [rowsP]
  for (int p = tid; p < count; p += NT) lst[p] = idx[(size_t)u * s.Ktot + p0 + p];
  __syncthreads();
  auto row_at = [&](int p) -> int { return lst[p]; };
  const T* kbase = kc + (size_t)u * s.cap * kD;
  const T* vbase = vc + (size_t)u * s.cap * kD;
  if constexpr (kMfma) {
    bf16x8_t qf[4];
    load_q_frags(reinterpret_cast<const bf16_t*>(q) + ((size_t)b * s.Hq + (size_t)g * G) * kD, G, qf);
    MfmaState st;
    st.init();
    mfma_attend(reinterpret_cast<const bf16_t*>(kbase), reinterpret_cast<const bf16_t*>(vbase), s.N, row_at, count,
                w * 16 * kMfmaTiles, NW * 16 * kMfmaTiles, s.scale_log2e, qf, vtile + w * kVTileBytes, st);
    mfma_stash_wave_state<G>(st, red);
  } else {
    float qr[G][8];
    load_query<T, G>(q + ((size_t)b * s.Hq + (size_t)g * G) * kD, s.scale_log2e, qr);
    AttnState<G> st;
    st.init();
    constexpr int R = G >= 8 ? 2 : 4;
    attend_rows<T, G, R>(kbase, vbase, s.N, row_at, count, w * 4 * R, NW * 4 * R, qr, st);
    stash_wave_state<T, G>(st, red);
  }
  __syncthreads();
  float* part = ws.partials + ((size_t)u * s.npart + blockIdx.x) * G * (kD + 2);
  for (int o = tid; o < G * kD; o += NT) {
    const int h = o / kD, d = o % kD;
    float m, l, acc;
    combine_waves<G, NW>(red, h, d, m, l, acc);
    part[h * (kD + 2) + 2 + d] = acc;
    if (d == 0) {
      part[h * (kD + 2)] = m;
      part[h * (kD + 2) + 1] = l;
    }
  }
}

// Folds the partial softmax states of a unit into the outputs: grid (G, units), one
// workgroup per query head, two threads per output dimension.
template <int G>
__global__ __launch_bounds__(256) void merge_kernel(Shape s, Workspace ws, int nparts, float* __restrict__ out_attn) {
  constexpr int NT = 256, NW = 4, kBatch = 16;
  extern __shared__ float wsm[];  // [nparts] weights
  __shared__ float fsm[NW];
  __shared__ float half_acc[kD];
  const int u = blockIdx.y, hq = blockIdx.x, b = u / s.Hkv, g = u % s.Hkv, tid = threadIdx.x;
  const int d = tid & (kD - 1), half = tid >> 7;
  const float* parts = ws.partials + ((size_t)u * s.npart * G + hq) * (kD + 2);
  const size_t stride = (size_t)G * (kD + 2);
  float mx = kNegBig;
  for (int j = tid; j < nparts; j += NT) {
    const float m = parts[j * stride];
    wsm[j] = m;
    mx = fmaxf(mx, m);
  }
  const float mstar = block_max<NT>(mx, fsm);  // its barriers make wsm visible
  float lsum = 0.0f;
  for (int j = tid; j < nparts; j += NT) {
    const float wj = __builtin_amdgcn_exp2f(wsm[j] - mstar);
    wsm[j] = wj;
    lsum = fmaf(wj, parts[j * stride + 1], lsum);
  }
  const float lstar = block_sum<NT>(lsum, fsm);
  float acc = 0.0f;
  for (int j0 = half; j0 < nparts; j0 += 2 * kBatch) {
    float a[kBatch];
#pragma unroll
    for (int x = 0; x < kBatch; ++x) a[x] = parts[(size_t)min(j0 + 2 * x, nparts - 1) * stride + 2 + d];
#pragma unroll
    for (int x = 0; x < kBatch; ++x) acc = fmaf(j0 + 2 * x < nparts ? wsm[j0 + 2 * x] : 0.0f, a[x], acc);
  }
  if (half == 1) half_acc[d] = acc;
  __syncthreads();
  if (half == 0) out_attn[((size_t)b * s.Hq + (size_t)g * G + hq) * kD + d] = (acc + half_acc[d]) / lstar;
}

// Select kernels without a histogram kernel in front (pqc_short.hip): of a decode step (kCount or kShort), and with given pair counts.
void launch_pairs_select(bool bf16, const Shape& s, const Workspace& ws, const void* q, const float* cent, const uint8_t* codes,
                         const unsigned* pair_counts, int uncounted, const void* k, const void* v, hipStream_t st);
void launch_short_select(bool bf16, const Shape& s, const Workspace& ws, const void* q, const float* cent, const uint8_t* codes, const void* k,
                         const void* v, hipStream_t st);

}  // namespace pqc
