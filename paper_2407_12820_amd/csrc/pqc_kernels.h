// Kernels of libpqcache (gfx950).  The workgroups of a unit (sequence b, KV head g) are placed by place_workgroup.
//
// Decode path (pqc_decode), two launches:
//   hist_kernel      table -> scan codes -> histogram of scores over kNB bins, and every token's bin number left behind
//                    for the next kernel
//   select_kernel    threshold bin from the histogram -> tokens whose stored bin lies above it (and the two windows)
//                    are listed in ascending order without atomics, written to the index output at their final place
//                    and attended at once; tokens inside the bin ("candidates") are recorded with their logits and V
//                    row.  The workgroup of a unit that finishes last ranks the candidates, folds the admitted ones
//                    and all partial softmax states into the output, and zeroes the unit's histogram and counters
//                    again: every call leaves them as it found them.  No workgroup waits for another.
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
template <int M_>
struct CodeChunks {
  static constexpr int M = M_;
  static constexpr int P = 16 / M_;  // tokens per chunk
  static constexpr bool kFromCodes = true;
  using Raw = uint4;
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
  // compiler count them when it waits for earlier ones): a chunk at or beyond the tensor's last
  // full 16 bytes is redirected to that last full chunk (to the spare bytes if the tensor has
  // none), and fix_tail() patches the one chunk that holds the tensor's ragged end afterwards.
  __device__ __forceinline__ Raw load(int chunk) const {
    const long long last_full = (total_bytes & ~15ll) - 16;  // < 0 for tensors under 16 bytes
    long long off = unit_byte0 + 16ll * chunk;
    off = off < last_full ? off : last_full;
    off = off > 0 ? off : 0;
    const uint8_t* p = total_bytes < 16 ? spare : all + off;
    return *reinterpret_cast<const uint4*>(p);
  }
  __device__ __forceinline__ void fix_tail(Raw& r, int chunk) const {
    const long long off = unit_byte0 + 16ll * chunk;
    if (off + 16 > total_bytes && off < total_bytes) {  // at most one chunk in the whole tensor
      unsigned w[4] = {0u, 0u, 0u, 0u};
      for (int b = 0; b < 16; ++b)
        if (off + b < total_bytes) w[b >> 2] |= (unsigned)all[off + b] << (8 * (b & 3));
      r = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
  __device__ __forceinline__ float score(const Raw& r, int i) const { return score_from_word<M>(chunk_word<M>(r, i), lut); }
  // one token: the load (issue early) and the table look-up (after the table is ready)
  using One = typename CodeWord<M>::type;
  __device__ __forceinline__ One load_one(int t, int u, int N) const {
    const uint8_t* p = all + ((long long)u * N + t) * M;
    One w = 0;
#pragma unroll
    for (int j = 0; j < M; ++j) w |= (One)p[j] << (8 * j);
    return w;
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
  __device__ __forceinline__ void fix_tail(Raw&, int) const {}
  __device__ __forceinline__ float score(const Raw& r, int i) const { return r.f[i]; }
  using One = float;
  __device__ __forceinline__ One load_one(int t, int, int) const { return scores[t]; }
  __device__ __forceinline__ float score_one(One w) const { return w; }
  __device__ __forceinline__ float score_of_token(int t, int, int) const { return scores[t]; }
};

// ------------------------------------------------------------------ utilities
__global__ void reset_kernel(unsigned* a, size_t na) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < na) a[i] = 0u;
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

// Score range of the middle tokens of a score array (stand-alone top-k only).
__global__ __launch_bounds__(1024) void score_range_kernel(Shape s, const float* __restrict__ scores,
                                                           float2* __restrict__ range) {
  __shared__ float smn[16], smx[16];
  const int u = blockIdx.y;
  float mn = INFINITY, mx = -INFINITY;
  for (int t = s.I + threadIdx.x; t < s.N - s.L; t += 1024) {
    const float v = scores[(size_t)u * s.N + t];
    mn = fminf(mn, v);
    mx = fmaxf(mx, v);
  }
  mn = wave_min(mn);
  mx = wave_max(mx);
  if ((threadIdx.x & 63) == 0) {
    smn[threadIdx.x >> 6] = mn;
    smx[threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) {
      mn = fminf(mn, smn[w]);
      mx = fmaxf(mx, smx[w]);
    }
    range[u] = make_float2(mn, mx);
  }
}

// ------------------------------------------------------------- 1. histogram
// SRC = CodeChunks<M>: builds the unit's table first; score bounds come from the table.
// SRC = ScoreChunks: bounds come from score_range_kernel.  Every workgroup of a unit
// then derives the same bin layout from the same sampled tokens (workgroup 0 publishes
// table and layout for the select kernel) and counts its own tokens.  Workgroups of a
// unit spread their counts over histCopies replicas.
// VW: 16-byte pieces of the centroid tensor per thread (1024 * 4 * VW floats cover the unit's M*C*Dm);
// VA: 16-byte chunks of codes (or scores) per thread (1024 * VA chunks cover the workgroup's tok tokens).
// Both are template parameters so that no thread issues loads it does not need: the loads of a workgroup's
// sixteen waves go through one address unit, 64 bytes per clock, and redundant ones cost as much as real ones.
// Workgroups are handed to the 8 XCDs round-robin in launch order (x fastest).  The workgroups of a unit all read that
// unit's centroids, histogram and stored bins, so eight units at a time are interleaved: the workgroups of one unit then
// share an XCD and its L2, the same one in both kernels.
__device__ __forceinline__ void place_workgroup(int units, int& u, int& bx) {
  u = blockIdx.y;
  bx = blockIdx.x;
  const int nx = gridDim.x, lin = blockIdx.y * nx + blockIdx.x;
  if (lin < (units & ~7) * nx) {
    const int i = lin % (8 * nx);
    u = (lin / (8 * nx)) * 8 + (i & 7);
    bx = i >> 3;
  }
}

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
  int u, bx;
  place_workgroup(units, u, bx);
  PQC_MARK(ws, 0, 0);
#ifdef PQC_TRACE
  PQC_NOTE(ws, 0, 15, (__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15) | (u << 8));  // XCC_ID[3:0], unit
#endif
  SRC src;
  const int src_stride = SRC::kFromCodes ? s.cap : s.N;  // tokens between units: code tensor, or dense score array
  src.init(src_ptr, u, src_stride, units, lut, ws.hist);
  // this workgroup's chunks and this thread's sample: the loads are issued before anything else,
  // except that a table build puts its centroid loads in front of them
  const int chunks = s.tok / P, chunk0 = bx * chunks;
  // Chunks that do not lie among the middle tokens as a whole (at the two ends of the unit, and behind its last token) are left
  // to a loop over single tokens, a thread each: taken by the threads that hold them, the two ways through the scan add up.
  const int front = min(max((s.I + src.lead + P - 1) / P - chunk0, 0), chunks);                    // such chunks at this workgroup's start
  const int back0 = max(min(max((s.N - s.L + src.lead) / P - chunk0, 0), chunks), front);           // and from here on at its end
  const int n_edge = (front + chunks - back0) * P;
  auto edge_pos = [&](int e) -> int { return (e < front * P ? e : e - front * P + back0 * P) + chunk0 * P; };
  typename SRC::Raw raw[VA];
  typename SRC::One sample, edge;
  const bool have_sample = tid < s.sampleN;
  auto issue_loads = [&]() {
#pragma unroll
    for (int v = 0; v < VA; ++v) raw[v] = src.load(chunk0 + min(v * NT + tid, chunks - 1));
    const int sample_i = min(tid, s.sampleN - 1);
    sample = src.load_one(min(s.N - 1, s.I + (int)(((long long)sample_i * max(0, s.N - s.I - s.L)) / s.sampleN)), u, src_stride);
    if (n_edge > 0) edge = src.load_one(min(max(edge_pos(min(tid, n_edge - 1)) - src.lead, 0), s.N - 1), u, src_stride);  // uniform
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
#pragma unroll
  for (int v = 0; v < VA; ++v) src.fix_tail(raw[v], chunk0 + min(v * NT + tid, chunks - 1));
  const BinParams bp =
      sample_window<NT>(bounds.x, bounds.y, src.score_one(sample), have_sample, s.rankHi, s.rankLo, hist, scan_sm);
  if (bx == 0 && tid == 0) ws.ctl[u] = bp;
  const float b_c0 = bp.c0, b_c1 = bp.c1, b_ic = bp.inv_c, b_ihi = bp.inv_hi;
  PQC_MARK(ws, 0, 2);
  // most tokens score below the window: they are counted in a register (bin 0), the rest
  // go to their LDS bin (an LDS atomic costs in proportion to the lanes that take part)
  int n_low = 0;
  unsigned short* bins_u = ws.bins + (size_t)u * s.nblk * s.tok;
#pragma unroll
  for (int v = 0; v < VA; ++v) {
    if (v * NT + tid >= front && v * NT + tid < back0) {
      unsigned st[P];  // what the select kernel will read back: bin + 1, or the window mark
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const float sc = src.score(raw[v], i);
        const int bin = score_bin(sc, b_c0, b_c1, b_ic, b_ihi);
        if (!(sc < b_c0)) atomicAdd(&hist[bin], 1u);
        n_low += sc < b_c0 ? 1 : 0;
        st[i] = (unsigned)bin + 1u;
      }
      // stored by chunk, the unit's phantom tokens included, so that every store is aligned
      unsigned short* dst = bins_u + (size_t)(chunk0 + v * NT + tid) * P;
      unsigned pw[P / 2];
#pragma unroll
      for (int i = 0; i < P / 2; ++i) pw[i] = st[2 * i] | (st[2 * i + 1] << 16);
      if constexpr (P == 2) *reinterpret_cast<unsigned*>(dst) = pw[0];
      if constexpr (P == 4) *reinterpret_cast<uint2*>(dst) = make_uint2(pw[0], pw[1]);
      if constexpr (P >= 8) {
#pragma unroll
        for (int i = 0; i < P / 8; ++i)
          reinterpret_cast<uint4*>(dst)[i] = make_uint4(pw[4 * i], pw[4 * i + 1], pw[4 * i + 2], pw[4 * i + 3]);
      }
    }
  }
  for (int e = tid; e < n_edge; e += NT) {
    const int pos = edge_pos(e), t = pos - src.lead;
    unsigned st = t >= 0 && t < s.N ? kBinWindow : 0u;
    if (t >= s.I && t < s.N - s.L) {
      const float sc = src.score_one(e == tid ? edge : src.load_one(t, u, src_stride));
      const int bin = score_bin(sc, b_c0, b_c1, b_ic, b_ihi);
      if (!(sc < b_c0)) atomicAdd(&hist[bin], 1u);
      n_low += sc < b_c0 ? 1 : 0;
      st = (unsigned)bin + 1u;
    }
    bins_u[pos] = (unsigned short)st;
  }
  n_low = wave_last(wave_inclusive_scan(n_low));
  if ((tid & 63) == 0 && n_low) atomicAdd(&hist[0], (unsigned)n_low);
  __syncthreads();
  PQC_MARK(ws, 0, 3);
  unsigned* gh = ws.hist + ((size_t)u * s.histCopies + (bx % s.histCopies)) * kNB;
  for (int i = tid; i < kNB; i += NT)
    if (hist[i]) atomicAdd(&gh[i], hist[i]);
  PQC_MARK(ws, 0, 4);
}

// ---------------------------------------------------- 2. select (+ attention)
// One workgroup owns the positions [bx*tok, +tok) of its unit (position = token + phantom tokens in front of token 0);
// its 8 waves each classify a contiguous eighth of them.  The histogram kernel left every token's bin behind, so a token
// is classified by comparing that number with the threshold bin.  Per wave, lanes hold 8 consecutive tokens, counts are
// prefix-summed across lanes and waves, and the workgroup's LDS list receives the selected tokens (ascending) from the
// front, the boundary-bin candidates from the back.  SRC is only used to score the few candidates exactly.
constexpr int kSelThreads = 512, kSelWaves = kSelThreads / 64;
constexpr int kMaxVecC = 4;        // 8-token groups per lane (tok <= 16384)
constexpr int kManyCand = 4096;    // candidates whose composites the path for large tie classes keeps in LDS
constexpr int kRankStep = 8;       // composites read per step of the ranking loop
constexpr int kRowStep = 8;        // admitted rows read per step of the fold

// What a workgroup publishes when it has classified its tokens: how many it selects (low half), its candidates (bits 32..47) and
// that the word is there.  The workgroups behind it read these words after their attention, many microseconds later, to
// place their lists in the index output; a workgroup that does not find all of them yet leaves its list to the unit's last one.
constexpr unsigned long long kCountsHere = 1ull << 63, kListLate = 1ull << 62;
__device__ __forceinline__ int count_selected(unsigned long long c) { return (int)(unsigned)c; }
__device__ __forceinline__ int count_candidates(unsigned long long c) { return (int)((c >> 32) & 0x3fffffffull); }

enum SelectMode {
  kFromHist,   // threshold from the histogram kernel, tokens classified by their stored bins
  kFromPairs,  // M = 2: threshold from the code-pair counts (pair_threshold), tokens classified by their exact score keys
};

// The code of one appended token per unit (Section 3.1: nearest centroid of each partition): nothing in the step depends
// on it, so it is computed beside the step.
struct AppendArgs {
  const void* key;    // [units][kD] in the cache's element type, or null: nothing to append
  const float* cent;  // [units][M][C][Dm]
  uint8_t* codes;     // the code tensor; written at `position` of every unit
  int position;
  unsigned* pair_counts;  // two partitions: [units][C*C] counts that gain the token's code pair, or null
};

// LDS of select_kernel beyond its few static words: one block, laid out once for the selection and the attention and once
// for the unit's last workgroup (the two do not overlap in time).
struct SelectLds {
  int red, qlds, vtile, pairs, list;                          // selection, attention
  int ml, slice, lg, lgr, comp, order, rows, many_tok;        // last workgroup (red is shared)
  int bytes;
};
__host__ __device__ inline SelectLds select_lds(int G, int elem_bytes, bool attn, bool mfma, bool pairs, int tok, int nblk) {
  SelectLds o;
  int a = 0;
  auto take = [](int& at, int n) {
    const int r = at;
    at += (n + 15) / 16 * 16;
    return r;
  };
  o.red = take(a, attn ? kSelWaves * G * (kD + 2) * 4 : 0);
  int b = a;
  o.qlds = take(a, attn ? G * kD * 4 : 0);
  o.vtile = take(a, mfma ? kSelWaves * kVTileBytes : 0);
  o.pairs = take(a, pairs ? (int)sizeof(PairLds) : 0);
  o.list = take(a, tok * 2);
  o.ml = take(b, attn ? G * nblk * 8 : 0);
  o.slice = take(b, attn ? kSelThreads * 8 : 0);
  o.lg = take(b, attn ? G * kCandRows * 4 : 0);
  o.lgr = take(b, attn ? G * (kCandRows + kRowStep) * 4 : 0);
  o.comp = take(b, (kCandRec + kRankStep) * 8);
  o.order = take(b, kCandRec * 4);
  const int rows = attn ? kCandRows * kD * elem_bytes : 0, many = kManyCand * 12;
  o.rows = take(b, rows > many ? rows : many);
  o.many_tok = o.rows + kManyCand * 8;
  o.bytes = a > b ? a : b;
  return o;
}

// The code of the appended token: one thread per centroid, the distance chain of pq_encode_kernel, the smallest
// (distance, centroid) pair of each partition through a 64-bit LDS minimum.
template <typename T>
__device__ __forceinline__ void append_code(const Shape& s, const AppendArgs& ap, int u, float* ax /* [kD] */,
                                            unsigned long long* abest /* [8] */) {
  const int c = threadIdx.x;
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
}

// ------------------------------------------------ 3. the unit's last workgroup
// Every workgroup of a unit draws a ticket when all it hands over has been written (put32 / put64, then a wait for the
// stores); the one that draws the last ticket comes here.  It ranks the candidates by counting larger composites, admits the
// `need` best, and folds them and the partial softmax states into the output:
//   out[d] = (sum_j w_j acc_j[d] + sum_r p_r V_r[d]) / l      w_j = exp2(m_j - m*), p_r = exp2(logit_r - m*)
// with states in workgroup order and admitted rows in rank order, whatever the order of arrival.
// All a compute unit reads here was written by other compute units, a round trip of more than a microsecond, so everything
// is requested at once: a thread owns two output dimensions of a head (and every SLC-th state when the heads leave threads
// over) and keeps up to kAccPer states in flight.  Up to kCandRows candidates travel as records (composite, logits, V row);
// with more, the admitted rows are attended from the cache, in rank order up to kCandRec candidates, beyond that (large tie
// classes: slow, always correct) in token order behind an 8-bit radix select of the composites.
constexpr int kAccPer = 16;
template <typename T, int G, class SRC, bool ATTN, int MODE>
__device__ __forceinline__ void finish_unit(const Shape& s, const Workspace& ws, const T* __restrict__ q, const T* __restrict__ kc,
                                            const T* __restrict__ vc, const void* __restrict__ src_ptr, int* __restrict__ out_idx,
                                            float* __restrict__ out_attn, int u, int lead, int n_cand, int n_above, bool any_late,
                                            unsigned char* dyn, const SelectLds& o, int* scan_sm, int* sm2) {
  constexpr int NT = kSelThreads, NW = kSelWaves;
  constexpr int PR = G * (kD / 2), SLC = NT / PR;  // pairs of output dimensions; threads per pair
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int b = u / s.Hkv, g = u % s.Hkv, units = s.B * s.Hkv;
  const int h = (tid % PR) / (kD / 2), d = 2 * (tid % (kD / 2)), sl = tid / PR;
  float* red = reinterpret_cast<float*>(dyn + o.red);
  float2* ml = reinterpret_cast<float2*>(dyn + o.ml);       // [G][nblk]
  float2* slice = reinterpret_cast<float2*>(dyn + o.slice); // [SLC][PR]
  float* lg = reinterpret_cast<float*>(dyn + o.lg);         // [G][kCandRows], by record
  float* lgr = reinterpret_cast<float*>(dyn + o.lgr);       // [G][kCandRows + kRowStep], by rank, in the log2 domain
  unsigned long long* comp = reinterpret_cast<unsigned long long*>(dyn + o.comp);
  int* order = reinterpret_cast<int*>(dyn + o.order);       // by rank: record, or token
  T* rows = reinterpret_cast<T*>(dyn + o.rows);             // [kCandRows][kD], by record
  unsigned long long* cnt = ws.counts + (size_t)u * s.nblk;
  int* out = out_idx + (size_t)u * s.Ktot;
  const CandView cv = cand_view(ws.cand_rec + (size_t)u * ws.rec_stride, ATTN ? G : 1);
  const float* pacc = ws.partials + (size_t)u * s.npart * G * kD;                                       // [j][h][kD]
  const float* pml = ws.partials + (size_t)units * s.npart * G * kD + (size_t)u * G * s.npart * 2;      // [h][j](m, l)
  __shared__ float mpart_sm[8], lpart_sm[8];  // per head: largest maximum of the states, sum of their weighted l
  __shared__ unsigned mcand_sm[8];            // per head: key of the largest admitted logit
  __shared__ float lslice_sm[8];              // [SLC][G]

  if (MODE == kFromPairs || any_late) {  // uniform
    // the totals (with code pairs), and the place of every list that is still to be copied
    int* pre = order;  // [nblk]
    int carry_s = 0, carry_c = 0;
    for (int j0 = 0; j0 < s.nblk; j0 += NT) {
      const int j = j0 + tid;
      const unsigned long long c = j < s.nblk ? get64(cnt + j) : 0ull;
      int ts, tc;
      const int ps = block_exclusive_scan<NT>(count_selected(c), &ts, scan_sm);
      block_exclusive_scan<NT>(count_candidates(c), &tc, scan_sm);
      if (j < s.nblk) pre[j] = (carry_s + ps) | ((c & kListLate) ? (int)0x80000000 : 0);
      carry_s += ts;
      carry_c += tc;
    }
    __syncthreads();
    n_cand = carry_c;
    n_above = max(0, carry_s - s.I - s.L);
    if (any_late) {
      const int need = max(0, min(s.K - n_above, n_cand));
      for (int j = w; j < s.nblk; j += NW) {  // a wave per list
        if (pre[j] >= 0) continue;
        const int base = pre[j] & 0x7fffffff, n = (j + 1 < s.nblk ? pre[j + 1] & 0x7fffffff : carry_s) - base;
        const unsigned short* src = ws.bins + ((size_t)u * s.nblk + j) * s.tok;
        for (int p = lane; p < n; p += 64) {
          const int pos = base + p, dst = pos < s.I + n_above ? pos : pos + need;
          const unsigned v = get32(src + (p & ~1));
          if (dst < s.Ktot) out[dst] = j * s.tok - lead + (int)((v >> (16 * (p & 1))) & 0xffffu);
        }
      }
      __syncthreads();
    }
  }
  const int need = max(0, min(s.K - n_above, n_cand));
  const bool recorded = n_cand <= kCandRows;  // uniform
  PQC_NOTE(ws, 1, 14, n_cand);
  PQC_NOTE(ws, 1, 15, need);

  // ---- everything is requested: candidates and (m, l) pairs first, which are needed first, then this thread's states
  const bool ranked = n_cand <= kCandRec;
  const int n_comp = need > 0 && ranked ? n_cand : 0;
  unsigned long long c0 = 0ull, c1 = 0ull;  // composites tid and NT + tid
  if (tid < n_comp) c0 = get64(cv.composite + tid);
  if (NT + tid < n_comp) c1 = get64(cv.composite + NT + tid);
  constexpr int VP = kD * (int)sizeof(T) / 8;  // 8-byte pieces of a V row
  unsigned long long vraw[4];
  unsigned lraw[G];
  const int n_rec = ATTN && need > 0 && recorded ? n_cand : 0;
  const int mh = tid / (NT / G), mj = tid % (NT / G);  // whose (m, l) pair this thread fetches
  unsigned long long m0 = 0ull;
  unsigned long long a0[ATTN ? kAccPer : 1];
  if constexpr (ATTN) {
    const unsigned long long* vsrc = reinterpret_cast<const unsigned long long*>(cv.v);
    if (tid < n_rec) {
#pragma unroll
      for (int hh = 0; hh < G; ++hh) lraw[hh] = get32(cv.logit + hh * kCandRows + tid);
    }
    if (mj < s.nblk) m0 = get64(pml + ((size_t)mh * s.npart + mj) * 2);
    if (n_rec > 0) {
#pragma unroll
      for (int x = 0; x < 4; ++x) vraw[x] = get64(vsrc + min(x * NT + tid, n_rec * VP - 1));
    }
#pragma unroll
    for (int x = 0; x < kAccPer; ++x)
      a0[x] = SLC * x < s.nblk ? get64(pacc + ((size_t)min(sl + SLC * x, s.nblk - 1) * G + h) * kD + d) : 0ull;  // uniform
    PQC_LOADS_ISSUED();
    unsigned long long* vdst = reinterpret_cast<unsigned long long*>(rows);
    if (tid < n_rec) {
#pragma unroll
      for (int hh = 0; hh < G; ++hh) lg[hh * kCandRows + tid] = __uint_as_float(lraw[hh]);
    }
    if (mj < s.nblk) ml[mh * s.nblk + mj] = unpack2(m0);
    for (int j = mj + NT / G; j < s.nblk; j += NT / G) ml[mh * s.nblk + j] = unpack2(get64(pml + ((size_t)mh * s.npart + j) * 2));
    if (n_rec > 0) {
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (x * NT + tid < n_rec * VP) vdst[x * NT + tid] = vraw[x];
      for (int i = 4 * NT + tid; i < n_rec * VP; i += NT) vdst[i] = get64(vsrc + i);  // (more candidates than is usual)
    }
    if (tid < 8) mcand_sm[tid] = 0u;
  }
  if (n_comp > 0) {
    // (entries up to the next multiple of kRankStep are zero, which ranks behind everything)
    if (tid < n_comp + kRankStep) comp[tid] = c0;
    if (NT + tid < n_comp + kRankStep) comp[NT + tid] = c1;
    if (tid < kRankStep) comp[kCandRec + tid] = 0ull;
  }
  __syncthreads();
  PQC_MARK(ws, 1, 9);

  // ---- which candidates are admitted; beside it, by one wave per head, the weights of the states among themselves
  // (they replace the maxima in ml.x)
  bool attended = false;  // admitted rows were attended from the cache: their state is in red
  if constexpr (ATTN) {
    if (w >= NW - G) {
      const int hh = w - (NW - G);
      float mx = kNegBig, l = 0.0f;
      for (int j = lane; j < s.nblk; j += 64) mx = fmaxf(mx, ml[hh * s.nblk + j].x);
      mx = wave_max(mx);
      for (int j = lane; j < s.nblk; j += 64) {
        const float2 v = ml[hh * s.nblk + j];
        const float e = __builtin_amdgcn_exp2f(v.x - mx);
        ml[hh * s.nblk + j].x = e;
        l = fmaf(e, v.y, l);
      }
      l = wave_sum(l);
      if (lane == 0) {
        mpart_sm[hh] = mx;
        lpart_sm[hh] = l;
      }
    }
  }
  if (need > 0) {
    if (ranked) {
      // four lanes per candidate share the counting (with up to kCandRows candidates one round of the workgroup)
      for (int k0 = 0; k0 < n_cand; k0 += NT / 4) {
        const int k = k0 + (tid >> 2);
        const unsigned long long mine = comp[min(k, kCandRec)];
        int rank = 0;
        for (int j0 = (tid & 3) * kRankStep; j0 < n_cand; j0 += 4 * kRankStep) {
          unsigned long long c[kRankStep];
#pragma unroll
          for (int y = 0; y < kRankStep; ++y) c[y] = comp[j0 + y];
#pragma unroll
          for (int y = 0; y < kRankStep; ++y) rank += c[y] > mine ? 1 : 0;
        }
        rank += dpp_i<0xB1>(0, rank);
        rank += dpp_i<0x4E>(0, rank);
        if (k >= n_cand || (tid & 3) != 0) continue;
        if (rank < need) {
          const int t = composite_token(mine);
          if (s.I + n_above + rank < s.Ktot) out[s.I + n_above + rank] = t;  // best first
          order[rank] = recorded ? k : t;
          if constexpr (ATTN) {
            if (recorded) {
#pragma unroll
              for (int hh = 0; hh < G; ++hh) {
                const float v = lg[hh * kCandRows + k] * s.scale_log2e;
                lgr[hh * (kCandRows + kRowStep) + rank] = v;
                atomicMax(&mcand_sm[hh], score_key(v));
              }
            }
          }
        }
      }
      if constexpr (ATTN) {
        if (recorded && tid < G * kRowStep) {  // rows behind the last one weigh nothing
          lgr[(tid / kRowStep) * (kCandRows + kRowStep) + need + tid % kRowStep] = kNegBig;
          if (tid < kRowStep) order[need + tid] = 0;
        }
      }
      __syncthreads();
      if constexpr (ATTN) {
        if (!recorded) {
          attended = true;
          float qr[G][8];
          load_query<T, G>(q + ((size_t)b * s.Hq + (size_t)g * G) * kD, s.scale_log2e, qr);
          AttnState<G> st;
          st.init();
          constexpr int R = G >= 8 ? 2 : 4;
          auto row_at = [&](int p) -> int { return order[p]; };
          attend_rows<T, G, R>(kc + (size_t)u * s.cap * kD, vc + (size_t)u * s.cap * kD, s.N, row_at, need, w * 4 * R, NW * 4 * R, qr, st);
          stash_wave_state<T, G>(st, red);
          __syncthreads();
        }
      }
    } else {
      // Large tie class.  Candidates as (score, token) composites made from their codes again, in workgroup order, which is
      // token order; up to kManyCand of them kept in LDS (every pass over them would otherwise be a chain of memory round
      // trips); the bytes that all of them share (the whole score, when they are one tie class) need no radix pass.
      attended = ATTN;
      __shared__ unsigned rhist[256];
      int* pre = order;  // [nblk]: candidates before each workgroup's
      const int* ctok = ws.cand_tok + (size_t)u * s.nblk * s.tok;
      {
        int carry = 0;
        for (int j0 = 0; j0 < s.nblk; j0 += NT) {
          const int j = j0 + tid;
          int tot;
          const int ps = block_exclusive_scan<NT>(j < s.nblk ? count_candidates(get64(cnt + j)) : 0, &tot, scan_sm);
          if (j < s.nblk) pre[j] = carry + ps;
          carry += tot;
        }
        __syncthreads();
      }
      auto cand_global = [&](int i) -> unsigned long long {
        int lo = 0, hi = s.nblk - 1;  // largest j with pre[j] <= i
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (pre[mid] <= i) lo = mid; else hi = mid - 1;
        }
        const int t = (int)get32(ctok + (size_t)lo * s.tok + (i - pre[lo]));
        float sc = 0.0f;  // (code pairs: the candidates share one score)
        if constexpr (MODE == kFromPairs) {
        } else if constexpr (SRC::kFromCodes) {
          const uint8_t* cp = static_cast<const uint8_t*>(src_ptr) + ((size_t)u * s.cap + t) * SRC::M;
          const float* tb = ws.lut + (size_t)u * SRC::M * s.C;
          sc = tb[cp[0]];
#pragma unroll
          for (int j = 1; j < SRC::M; ++j) sc = __fadd_rn(sc, tb[j * s.C + cp[j]]);
        } else {
          sc = static_cast<const float*>(src_ptr)[(size_t)u * s.N + t];
        }
        return make_composite(sc, t);
      };
      unsigned long long* gcomp = reinterpret_cast<unsigned long long*>(dyn + o.rows);  // [kManyCand]
      int* gtok = reinterpret_cast<int*>(dyn + o.many_tok);                             // [kManyCand] admitted tokens
      const bool cached = n_cand <= kManyCand;
      unsigned long long varying = ~0ull, common = 0ull;
      if (cached) {
        unsigned long long a_and = ~0ull, a_or = 0ull;
        for (int i = tid; i < n_cand; i += NT) {
          const unsigned long long c = cand_global(i);
          gcomp[i] = c;
          a_and &= c;
          a_or |= c;
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
      unsigned long long thr = 0ull;
      int want = need;
      for (int shift = 56; shift >= 0; shift -= 8) {
        if (((varying >> shift) & 0xffull) == 0) {  // uniform: every candidate has this byte
          thr |= common & (0xffull << shift);
          continue;
        }
        if (tid < 256) rhist[tid] = 0u;
        __syncthreads();
        for (int i = tid; i < n_cand; i += NT) {
          const unsigned long long c = cand_at(i);
          if (shift == 56 || (c >> (shift + 8)) == (thr >> (shift + 8))) atomicAdd(&rhist[(unsigned)(c >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (tid == 0) {
          int cum = 0, dg = 255;
          for (; dg > 0; --dg) {
            if (cum + (int)rhist[dg] >= want) break;
            cum += (int)rhist[dg];
          }
          sm2[0] = dg;
          sm2[1] = want - cum;
        }
        __syncthreads();
        thr |= (unsigned long long)sm2[0] << shift;
        want = sm2[1];
        __syncthreads();
      }
      // admitted candidates in token order: indices out, rows attended (all at once when they fit the LDS list, else NT
      // candidates per round)
      AttnState<G> st;
      float qr[G][8];
      constexpr int R = G >= 8 ? 2 : 4;
      auto row_at = [&](int p) -> int { return gtok[p]; };
      if constexpr (ATTN) {
        st.init();
        load_query<T, G>(q + ((size_t)b * s.Hq + (size_t)g * G) * kD, s.scale_log2e, qr);
      }
      int carry = 0;
      for (int i0 = 0; i0 < n_cand; i0 += NT) {
        const int i = i0 + tid;
        unsigned long long c = 0ull;
        if (i < n_cand) c = cand_at(i);
        const int flag = (i < n_cand && c >= thr) ? 1 : 0;
        int tot;
        const int pos = block_exclusive_scan<NT>(flag, &tot, scan_sm);
        if (flag) {
          gtok[(cached ? carry : 0) + pos] = composite_token(c);
          if (s.I + n_above + carry + pos < s.Ktot) out[s.I + n_above + carry + pos] = composite_token(c);
        }
        if (!cached) {
          __syncthreads();
          if constexpr (ATTN)
            attend_rows<T, G, R>(kc + (size_t)u * s.cap * kD, vc + (size_t)u * s.cap * kD, s.N, row_at, tot, w * 4 * R, NW * 4 * R, qr, st);
          __syncthreads();
        }
        carry += tot;
      }
      if constexpr (ATTN) {
        if (cached) {
          __syncthreads();
          attend_rows<T, G, R>(kc + (size_t)u * s.cap * kD, vc + (size_t)u * s.cap * kD, s.N, row_at, carry, w * 4 * R, NW * 4 * R, qr, st);
        }
        stash_wave_state<T, G>(st, red);
        __syncthreads();
      }
    }
  }

  if constexpr (ATTN) {
    if (need == 0) __syncthreads();  // (every other way here has passed a barrier since the weights)
    PQC_MARK(ws, 1, 10);
    // ---- fold
    const int nrow = attended ? 0 : need;
    float mstar = mpart_sm[h];
    if (nrow > 0) mstar = fmaxf(mstar, key_score(mcand_sm[h]));
    if (attended)
      for (int x = 0; x < NW; ++x) mstar = fmaxf(mstar, red[((size_t)x * G + h) * (kD + 2)]);
    float ax = 0.0f, ay = 0.0f;
    float e0[kAccPer];
#pragma unroll
    for (int x = 0; x < kAccPer; ++x) e0[x] = ml[h * s.nblk + min(sl + SLC * x, s.nblk - 1)].x;
#pragma unroll
    for (int x = 0; x < kAccPer; ++x) {
      const float e = sl + SLC * x < s.nblk ? e0[x] : 0.0f;
      const float2 v = unpack2(a0[x]);
      ax = fmaf(e, v.x, ax);
      ay = fmaf(e, v.y, ay);
    }
    for (int j0 = sl + SLC * kAccPer; j0 < s.nblk; j0 += SLC * kAccPer) {
      unsigned long long a[kAccPer];
#pragma unroll
      for (int x = 0; x < kAccPer; ++x) a[x] = get64(pacc + ((size_t)min(j0 + SLC * x, s.nblk - 1) * G + h) * kD + d);
#pragma unroll
      for (int x = 0; x < kAccPer; ++x) {
        const int j = j0 + SLC * x;
        const float e = j < s.nblk ? ml[h * s.nblk + min(j, s.nblk - 1)].x : 0.0f;
        const float2 v = unpack2(a[x]);
        ax = fmaf(e, v.x, ax);
        ay = fmaf(e, v.y, ay);
      }
    }
    const float f = __builtin_amdgcn_exp2f(mpart_sm[h] - mstar);
    ax *= f;
    ay *= f;
    float l = 0.0f;  // of this slice's rows
    for (int r0 = sl * kRowStep; r0 < nrow; r0 += SLC * kRowStep) {
      float e[kRowStep];
      float2 v[kRowStep];
#pragma unroll
      for (int y = 0; y < kRowStep; ++y) {
        e[y] = __builtin_amdgcn_exp2f(lgr[h * (kCandRows + kRowStep) + r0 + y] - mstar);
        v[y] = load_pair(rows + (size_t)order[r0 + y] * kD + d);
      }
#pragma unroll
      for (int y = 0; y < kRowStep; ++y) {
        l += e[y];
        ax = fmaf(e[y], v[y].x, ax);
        ay = fmaf(e[y], v[y].y, ay);
      }
    }
    if (sl == 0) l += f * lpart_sm[h];
    if (attended && sl == 0) {
      for (int x = 0; x < NW; ++x) {
        const float* st = red + ((size_t)x * G + h) * (kD + 2);
        const float e = __builtin_amdgcn_exp2f(st[0] - mstar);
        l = fmaf(st[1], e, l);
        ax = fmaf(e, st[2 + d], ax);
        ay = fmaf(e, st[3 + d], ay);
      }
    }
    if constexpr (SLC > 1) {
      slice[tid] = make_float2(ax, ay);
      if (d == 0) lslice_sm[sl * G + h] = l;
      __syncthreads();
      if (sl == 0) {
#pragma unroll
        for (int x = 1; x < SLC; ++x) {
          const float2 v = slice[x * PR + tid];
          ax += v.x;
          ay += v.y;
          l += lslice_sm[x * G + h];
        }
      }
    }
    if (sl == 0) {
      *reinterpret_cast<float2*>(out_attn + ((size_t)b * s.Hq + (size_t)g * G + h) * kD + d) = make_float2(ax / l, ay / l);
    }
  }
  // ---- the next call finds histogram and counters zero
  if constexpr (MODE == kFromHist) {
    uint4* gh = reinterpret_cast<uint4*>(ws.hist + (size_t)u * s.histCopies * kNB);
    for (int i = tid; i < s.histCopies * kNB / 4; i += NT) gh[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  for (int j = tid; j < s.nblk; j += NT) cnt[j] = 0ull;
  if (tid == 0) {
    ws.ticket[u] = 0u;
    ws.cand_count[u] = 0u;
  }
}

template <typename T, int G, class SRC, bool ATTN, int MODE>
__global__ __launch_bounds__(kSelThreads, 2) void select_kernel(Shape s, Workspace ws, const T* __restrict__ q,
                                                                const T* __restrict__ kc, const T* __restrict__ vc,
                                                                const void* __restrict__ src_ptr, const float* __restrict__ cent,
                                                                const unsigned* pair_counts, int* __restrict__ out_idx,
                                                                float* __restrict__ out_attn, AppendArgs ap) {
  constexpr int NT = kSelThreads, NW = kSelWaves;
  constexpr bool kMfma = ATTN && sizeof(T) == 2 && kMatrixCoreAttention;
  constexpr bool PAIRS = MODE == kFromPairs;
  static_assert(!PAIRS || (SRC::kFromCodes && SRC::M == 2), "pair counts exist for two partitions only");
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ int scan_sm[2 * NW + 1 + 4];
  __shared__ int wcnt[2 * NW];
  __shared__ int sm2[4];
  __shared__ int late_sm;  // some workgroup before this one had not published its counts
  const SelectLds o = select_lds(G, sizeof(T), ATTN, kMfma, PAIRS, s.tok, s.nblk);
  float* red = reinterpret_cast<float*>(dyn + o.red);
  float* qlds = reinterpret_cast<float*>(dyn + o.qlds);
  unsigned char* vtile = dyn + o.vtile;
  unsigned short* list = reinterpret_cast<unsigned short*>(dyn + o.list);  // [tok] offsets from the workgroup's first position
  PairLds& pl = *reinterpret_cast<PairLds*>(dyn + o.pairs);
  int u, bx;
  place_workgroup(s.B * s.Hkv, u, bx);
  if (bx == s.nblk) {  // one more workgroup per unit (not with code-pair counts, which this launch reads)
    append_code<T>(s, ap, u, reinterpret_cast<float*>(dyn), reinterpret_cast<unsigned long long*>(dyn + kD * 4));
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int b = u / s.Hkv, g = u % s.Hkv;
  PQC_MARK(ws, 1, 0);
  // this wave's stored bins, the query and the histogram: all requested up front
  const int tpw = s.tok / NW;            // positions per wave, in groups of 8 per lane
  const int gpw = (tpw + 511) / 512;     // groups per lane: 1 to 4 (the last lanes idle when tpw is no multiple of 512)
  const int lead = SRC::kFromCodes ? (int)((((long long)u * s.cap * (SRC::M ? SRC::M : 1)) & 15) / (SRC::M ? SRC::M : 1)) : 0;
  const int wg_p0 = bx * s.tok, wave_p0 = wg_p0 + w * tpw;  // positions
  const int wg_t0 = wg_p0 - lead;                           // token of the workgroup's first position
  // 16 bytes per group of 8 tokens: their stored bins, or (PAIRS) their codes (the capacity is a multiple of 8 there: lead is 0)
  const unsigned short* bins_u =
      PAIRS ? reinterpret_cast<const unsigned short*>(static_cast<const uint8_t*>(src_ptr) + (size_t)u * s.cap * 2)
            : ws.bins + (size_t)u * s.nblk * s.tok;
  const int last_group = PAIRS ? s.cap - 8 : s.nblk * s.tok - 8;
  uint4 raw[kMaxVecC];
#pragma unroll
  for (int v = 0; v < kMaxVecC; ++v)
    raw[v] = *reinterpret_cast<const uint4*>(bins_u + min(wave_p0 + min((v * 64 + lane) * 8, tpw - 8), last_group));
  constexpr int QV = ATTN ? (G * kD + NT - 1) / NT : 1;  // query elements per thread
  float qreg[QV];
  if constexpr (ATTN) {
#pragma unroll
    for (int x = 0; x < QV; ++x)
      qreg[x] = load_as_float<T>(q + ((size_t)b * s.Hq + (size_t)g * G) * kD, min(x * NT + tid, G * kD - 1));
  }
  Threshold th{0, 0, 0, 0};
  PairThreshold pth{0u, true};
  if constexpr (PAIRS) {
    PQC_LOADS_ISSUED();
    if constexpr (ATTN) {
#pragma unroll
      for (int x = 0; x < QV; ++x)
        if (x * NT + tid < G * kD) qlds[x * NT + tid] = qreg[x];
    }
    pth = pair_threshold<T, NT>(s, q + ((size_t)b * s.Hq + (size_t)g * G) * kD, cent + (size_t)u * 2 * s.C * (kD / 2),
                                pair_counts + (size_t)u * s.C * s.C, static_cast<const uint8_t*>(src_ptr) + (size_t)u * s.cap * 2,
                                pl, scan_sm, [&](int slot) { PQC_MARK(ws, 1, slot); },
                                ap.key ? ap.position : -1 /* a window token the counts do not hold yet */);  // syncs: qlds ready
  } else {
    ThresholdSearch<NT> ts;
    ts.load(ws.hist + (size_t)u * s.histCopies * kNB, s.histCopies);
    PQC_LOADS_ISSUED();
    if constexpr (ATTN) {
#pragma unroll
      for (int x = 0; x < QV; ++x)
        if (x * NT + tid < G * kD) qlds[x * NT + tid] = qreg[x];
    }
    th = ts.resolve(s.K, scan_sm);  // syncs: qlds ready
  }
  PQC_MARK(ws, 1, 1);
  unsigned selm[kMaxVecC], candm[kMaxVecC];
  int place[kMaxVecC];  // selected (low half) and candidates (high half) of the wave in front of this lane's group
  int wave_cnt = 0;
  const unsigned thr = (unsigned)th.bstar + 1u;  // in stored form
#pragma unroll
  for (int v = 0; v < kMaxVecC; ++v) {
    selm[v] = 0u;
    candm[v] = 0u;
    place[v] = 0;
    if (v < gpw) {  // uniform
      const unsigned wv[4] = {raw[v].x, raw[v].y, raw[v].z, raw[v].w};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const unsigned st = (wv[i >> 1] >> (16 * (i & 1))) & 0xffffu;
        if constexpr (PAIRS) {
          const int t = wave_p0 + (v * 64 + lane) * 8 + i;
          const bool window = t < s.I || t >= s.N - s.L;
          const unsigned key =
              score_key(__fadd_rn(pl.lut[min(st & 0xffu, (unsigned)kPairC - 1)], pl.lut[kPairC + min(st >> 8, (unsigned)kPairC - 1)]));
          selm[v] |= ((window || (!pth.none && key > pth.key)) ? 1u : 0u) << i;
          candm[v] |= ((!window && !pth.none && key == pth.key) ? 1u : 0u) << i;
        } else {
          selm[v] |= (st > thr ? 1u : 0u) << i;
          candm[v] |= (st == thr ? 1u : 0u) << i;
        }
      }
      int nreal = (v * 64 + lane) * 8 < tpw ? 8 : 0;  // tokens of this group that exist (the stored bins say so themselves)
      if constexpr (PAIRS) nreal = min(nreal, max(0, s.N - (wave_p0 + (v * 64 + lane) * 8)));
      selm[v] &= (1u << nreal) - 1u;
      candm[v] &= (1u << nreal) - 1u;
      const int cnt = __popc(selm[v]) | (__popc(candm[v]) << 16);
      const int inc = wave_inclusive_scan(cnt);
      place[v] = wave_cnt + inc - cnt;
      wave_cnt += wave_last(inc);
    }
  }
  PQC_MARK(ws, 1, 8);
  if (lane == 0) wcnt[w] = wave_cnt;
  __syncthreads();
  int tot_sel = 0, tot_cand = 0, base_sel = 0, base_cand = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int c = wcnt[i];
    base_sel += i < w ? c & 0xffff : 0;
    base_cand += i < w ? c >> 16 : 0;
    tot_sel += c & 0xffff;
    tot_cand += c >> 16;
  }
#pragma unroll
  for (int v = 0; v < kMaxVecC; ++v) {
    if (v < gpw) {  // uniform
      int ps = base_sel + (place[v] & 0xffff), pc = base_cand + (place[v] >> 16);
      const int off = w * tpw + (v * 64 + lane) * 8;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (selm[v] & (1u << i)) list[ps++] = (unsigned short)(off + i);
        if (candm[v] & (1u << i)) list[s.tok - 1 - (pc++)] = (unsigned short)(off + i);
      }
    }
  }
  // published for the workgroups behind this one; and record slots for the candidates, requested now and needed only after the
  // attention below, which hides the round trip of the returning atomic
  int rec_asked;  // set and read by thread 0 only; no initialiser, or the merge with it would wait for the atomic here
  unsigned long long* cnt = ws.counts + (size_t)u * s.nblk;
  const unsigned long long mine = kCountsHere | ((unsigned long long)(unsigned)tot_cand << 32) | (unsigned)tot_sel;
  if (tid == 0) {
    late_sm = 0;
    put64(cnt + bx, mine);
    if (tot_cand > 0) rec_asked = (int)atomicAdd(&ws.cand_count[u], (unsigned)tot_cand);
  }
  __syncthreads();
  PQC_MARK(ws, 1, 2);
  // A candidate's exact score comes from its codes and the unit's table (same evaluation order as everywhere), or from the
  // score array of the stand-alone top-k.
  struct CandKey {
    unsigned cb[SRC::kFromCodes ? SRC::M : 1];
    float te[SRC::kFromCodes ? SRC::M : 1];
  };
  auto cand_token = [&](int c) -> int { return wg_t0 + list[s.tok - 1 - c]; };
  auto cand_key_load = [&](int t) -> CandKey {
    CandKey k;
    if constexpr (SRC::kFromCodes) {
      const uint8_t* cp = static_cast<const uint8_t*>(src_ptr) + ((size_t)u * s.cap + t) * SRC::M;
#pragma unroll
      for (int j = 0; j < SRC::M; ++j) k.cb[j] = cp[j];
    } else {
      k.cb[0] = 0u;
      k.te[0] = static_cast<const float*>(src_ptr)[(size_t)u * s.N + t];
    }
    return k;
  };
  auto cand_table = [&](CandKey k) -> CandKey {  // the table entries its codes name
    if constexpr (PAIRS) {
      k.te[0] = pl.lut[min(k.cb[0], (unsigned)kPairC - 1)];
      k.te[1] = pl.lut[kPairC + min(k.cb[1], (unsigned)kPairC - 1)];
    } else if constexpr (SRC::kFromCodes) {
      const float* tb = ws.lut + (size_t)u * SRC::M * s.C;
#pragma unroll
      for (int j = 0; j < SRC::M; ++j) k.te[j] = tb[j * s.C + k.cb[j]];
    }
    return k;
  };
  auto cand_score = [&](const CandKey& k) -> float {
    float sc = k.te[0];
#pragma unroll
    for (int j = 1; j < (SRC::kFromCodes ? SRC::M : 1); ++j) sc = __fadd_rn(sc, k.te[j]);
    return sc;
  };
  PQC_MARK(ws, 1, 3);

  const T* kbase = kc + (size_t)u * s.cap * kD;
  const T* vbase = vc + (size_t)u * s.cap * kD;
  // The first candidates (one per 16-lane group): their codes and K/V rows are requested now, so that after the attention
  // only the table look-up, arithmetic and the record write remain.
  const int sub = lane & 15, grp = tid >> 4;
  int c0_t = 0;
  CandKey c0_key;
  RowRaw<T> c0_k, c0_v;
#pragma unroll
  for (int j = 0; j < (SRC::kFromCodes ? SRC::M : 1); ++j) {
    c0_key.cb[j] = 0u;
    c0_key.te[j] = 0.0f;
  }
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
  // Rows this workgroup attends: its own tokens above the threshold bin, and, instead of the window tokens it happens to hold
  // (the list's first nI and last nL entries), every nblk-th token of the two windows, so that the window rows are spread over
  // the unit's workgroups.
  const int tok_lo = max(0, wg_t0), tok_hi = min(s.N, wg_t0 + s.tok);
  const int nI = max(0, min(s.I, tok_hi) - tok_lo), nL = max(0, tok_hi - max(s.N - s.L, tok_lo));
  const int n_own = tot_sel - nI - nL;
  const CandView cv = cand_view(ws.cand_rec + (size_t)u * ws.rec_stride, ATTN ? G : 1);
  float c0_logit[ATTN ? G : 1];
  auto cand_logits = [&](const RowRaw<T>& kr, float (&lg)[ATTN ? G : 1]) {
    float kf[8];
    kr.unpack(kf);
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float d = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) d = fmaf(qlds[h * kD + owned_dim<T>(sub, e)], kf[e], d);
      lg[h] = group16_sum(d);
    }
  };
  // Requested when a wave has attended its first rows, used after the workgroup's partial state is on its way: what the workgroups
  // before this one have published (the first 64 of them; the place of the list in the index output follows from it) and the
  // table entries of the first candidates.
  unsigned long long seen = kCountsHere;
  auto ask = [&]() {
    if (lane < bx) seen = get64(cnt + lane);
    if (grp < tot_cand) c0_key = cand_table(c0_key);
  };
  if constexpr (ATTN) {
    const int n_win = bx < s.I + s.L ? (s.I + s.L - bx + s.nblk - 1) / s.nblk : 0;
    const int n_att = n_own + n_win;
    // every wave attends an equal, contiguous share of the rows (shares of whole stages would leave some waves a stage more)
    const int share = (n_att + NW - 1) / NW, att0 = w * share, att1 = min(n_att, att0 + share);
    auto att_at = [&](int p) -> int {
      if (p < n_own) return wg_t0 + list[p + nI];
      const int wt = bx + (p - n_own) * s.nblk;
      return wt < s.I ? wt : s.N - s.L + (wt - s.I);
    };
    if constexpr (kMfma) {
      bf16x8_t qf[4];
      load_q_frags(reinterpret_cast<const bf16_t*>(q) + ((size_t)b * s.Hq + (size_t)g * G) * kD, G, qf);
      MfmaState st;
      st.init();
      mfma_attend(reinterpret_cast<const bf16_t*>(kbase), reinterpret_cast<const bf16_t*>(vbase), s.N, att_at, att1, att0,
                  16 * kMfmaTiles, s.scale_log2e, qf, vtile + w * kVTileBytes, st, ask);
      PQC_MARK(ws, 1, 4);
      mfma_stash_wave_state<G>(st, red);
    } else {
      float qr[G][8];
      load_query<T, G>(q + ((size_t)b * s.Hq + (size_t)g * G) * kD, s.scale_log2e, qr);
      AttnState<G> st;
      st.init();
      constexpr int R = (G >= 8 || sizeof(T) == 4) ? 2 : 4;
      attend_rows<T, G, R>(kbase, vbase, s.N, att_at, att1, att0, 4 * R, qr, st, ask);
      PQC_MARK(ws, 1, 4);
      stash_wave_state<T, G>(st, red);
    }
    if (grp < tot_cand) cand_logits(c0_k, c0_logit);
    if (tid == 0 && tot_cand > 0) sm2[2] = rec_asked;
    __syncthreads();
    PQC_MARK(ws, 1, 12);
    // this workgroup's partial state: the accumulators as 128 floats per head ([j][h][kD] over the unit's workgroups j), the
    // (m, l) pairs in a dense array per head behind all accumulators ([units][h][j])
    float* pacc = ws.partials + (((size_t)u * s.npart + bx) * G) * kD;
    float* pml = ws.partials + (size_t)s.B * s.Hkv * s.npart * G * kD + ((size_t)u * G * s.npart + bx) * 2;
    for (int i = tid; i < G * kD / 2; i += NT) {
      const int h = i / (kD / 2), d = 2 * (i % (kD / 2));
      float m[NW], l[NW];
      float2 a[NW];
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        const float* src = red + ((size_t)x * G + h) * (kD + 2);
        m[x] = src[0];
        l[x] = src[1];
        a[x] = *reinterpret_cast<const float2*>(src + 2 + d);
      }
      float mx = m[0], ls = 0.0f, ax = 0.0f, ay = 0.0f;
#pragma unroll
      for (int x = 1; x < NW; ++x) mx = fmaxf(mx, m[x]);
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        const float e = __builtin_amdgcn_exp2f(m[x] - mx);
        ls = fmaf(l[x], e, ls);
        ax = fmaf(a[x].x, e, ax);
        ay = fmaf(a[x].y, e, ay);
      }
      put64(pacc + h * kD + d, pack2(ax, ay));
      if (d == 0) put64(pml + (size_t)h * s.npart * 2, pack2(mx, ls));
    }
  } else {
    ask();
    if (tid == 0 && tot_cand > 0) sm2[2] = rec_asked;
    __syncthreads();
  }
  // candidates (few): tokens for the path of large tie classes, and full records while slots last
  for (int c = grp; c < tot_cand; c += NT / 16) {
    int t = c0_t;
    RowRaw<T> vr = c0_v;
    if (c >= NT / 16) {  // beyond the candidates whose loads went out before the attention
      t = cand_token(c);
      c0_key = cand_table(cand_key_load(t));
      if constexpr (ATTN) {
        RowRaw<T> kr;
        kr.load(kbase, t, sub);
        vr.load(vbase, t, sub);
        cand_logits(kr, c0_logit);
      }
    }
    const int slot = sm2[2] + c;
    if (sub == 0) {
      put32(&ws.cand_tok[((size_t)u * s.nblk + bx) * s.tok + c], (unsigned)t);
      if (slot < kCandRec) put64(cv.composite + slot, make_composite(cand_score(c0_key), t));
    }
    if constexpr (ATTN) {
      if (slot < kCandRows) {
        if (sub == 0) {
#pragma unroll
          for (int h = 0; h < G; ++h) put32(cv.logit + h * kCandRows + slot, __float_as_uint(c0_logit[h]));
        }
        vr.put(cv.v + (size_t)slot * kD * sizeof(T), sub);
      }
    }
  }
  // tokens that the workgroups before this one select, initial window aside (every wave adds them up for itself)
  bool late = __ballot(!(seen & kCountsHere)) != 0ull;
  int before = wave_last(wave_inclusive_scan(count_selected(seen))) - min(s.I, max(0, wg_t0));
  for (int j0 = 64; j0 < bx; j0 += 64) {  // (long contexts)
    const unsigned long long c = j0 + lane < bx ? get64(cnt + j0 + lane) : kCountsHere;
    late |= __ballot(!(c & kCountsHere)) != 0ull;
    before += wave_last(wave_inclusive_scan(count_selected(c)));
  }
#ifdef PQC_TRACE
  late |= s.forceLate != 0;
#endif
  if (late && lane == 0) late_sm = 1;
  PQC_MARK(ws, 1, 5);
  // every store above has arrived before this workgroup counts itself as done
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  late = late_sm != 0;
  if (late) {  // (rare) the list waits where the bins were, which nobody reads any more, for the unit's last workgroup
    unsigned short* dst = ws.bins + ((size_t)u * s.nblk + bx) * s.tok;
    for (int p = 2 * tid; p < tot_sel; p += 2 * NT) put32(dst + p, (unsigned)list[p] | ((unsigned)list[min(p + 1, s.tok - 1)] << 16));
    if (tid == 0) put64(cnt + bx, mine | kListLate);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
  PQC_MARK(ws, 1, 6);
  const unsigned draw = late ? 0x10001u : 1u;  // done workgroups, and those with a late list in the upper half
  if (tid == 0) sm2[3] = (int)(draw + __hip_atomic_fetch_add(&ws.ticket[u], draw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  // the list at its place in the index output, while the ticket is on its way
  if (!late) {
    int* out = out_idx + (size_t)u * s.Ktot;
    for (int p = tid; p < tot_sel; p += NT) {
      const int t = wg_t0 + list[p];
      const int dst = t < s.I ? t : t >= s.N - s.L ? s.I + s.K + (t - (s.N - s.L)) : s.I + before + (p - nI);
      // (the bound only matters when the caller's pair counts do not belong to the codes: then more than K tokens may be listed)
      if (dst < s.Ktot) out[dst] = t;
    }
  }
  __syncthreads();
  if ((sm2[3] & 0xffff) != s.nblk) return;
  PQC_MARK(ws, 1, 7);
  finish_unit<T, G, SRC, ATTN, MODE>(s, ws, q, kc, vc, src_ptr, out_idx, out_attn, u, lead, th.bstar < kNB ? th.n_cand : 0, th.n_above,
                                     (sm2[3] >> 16) != 0, dyn, o, scan_sm, sm2);
  if constexpr (PAIRS) {
    if (ap.key) {  // the counts have been read by every workgroup of the unit
      __syncthreads();
      append_code<T>(s, ap, u, reinterpret_cast<float*>(dyn), reinterpret_cast<unsigned long long*>(dyn + kD * 4));
    }
  }
  PQC_MARK(ws, 1, 11);
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

}  // namespace pqc
