// Device-side building blocks of libpqcache (gfx950, wave64).
//
// Everything here is a __device__ template; the kernels that use them live in
// pqc_kernels.h.  Citations are to the paper's sections (PQ search: Section 2.2 and
// Section 3.1 step 4; top-k: Section 3.1 steps 4-5 and Section 3.2; selective
// attention: Section 2.1 and Section 3.1 step 6).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace pqc {

constexpr int kNB = 2048;        // score bins of the one-pass threshold search
constexpr int kHistCopies = 4;   // histogram replica slots per unit; Shape::histCopies of them are in use
constexpr int kD = 128;          // head dimension
constexpr int kLutRow = 256;     // LDS stride of one partition's table (max centroids)
constexpr int kCandRec = 1024;   // boundary-bin candidate records per unit (ranked inside LDS by the finalize kernel)
constexpr float kNegBig = -1.0e30f;

struct bf16_t {
  uint16_t bits;
};

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;

// Geometry of one decode step, passed by value to every kernel.
struct Shape {
  int B, Hq, Hkv, G, N, M, C, Dm, K, I, L, Ktot;
  int cap;          // tokens the K/V caches and the code tensor hold per unit (>= N): their stride between units
  int tokA, nblkA;  // histogram kernel: tokens per workgroup, workgroups per unit
  int tokC, nblkC;  // select kernel: tokens per workgroup, workgroups per unit
  int rowsP, nblkP; // list-attention kernel: rows per workgroup, workgroups per unit
  int npart;        // partial slots per unit
  int slices;       // finalize kernel: workgroups per query head (1, 2 or 4), each producing kD/slices output dimensions
  bool pairsMany;   // step with given pair counts: in two workgroups of 256 threads per compute unit (From::kPairsMany)
  int copyWgs;      // finalize kernel: workgroups per unit that copy the index lists
  int binStride;    // stored bins per unit (nblkC * tokC)
  int stageStride;  // 8-byte words between the staging slots of consecutive select workgroups: tokC plus a pad, so that
                    // the slots do not all start on the same memory channels
  int histCopies;   // histogram replicas in use (1, 2 or 4): spreads the flush atomics of units with many workgroups
  int sampleN;      // tokens sampled per unit to place the fine bins (<= 1024)
  int rankHi, rankLo;  // sample ranks (from the top) that bracket the K-th largest score
  float scale_log2e;
};

// What a select workgroup leaves behind for every boundary-bin candidate, enough for the finalize kernel to rank it
// and, if admitted, to add it to the attention output without touching the K/V cache again.  Per unit, as arrays
// over the candidates in order of arrival (at most kCandRec), so that what a finalize workgroup reads of them is dense:
//   composite  [kCandRec]      uint64   (score key, ~token): larger ranks first
//   logit      [G][kCandRec]   float    q_h . k for the group's heads (raw, unscaled)
//   v          [kCandRec][kD]  T        the V row
struct CandView {
  unsigned long long* composite;
  float* logit;
  unsigned char* v;
};
__host__ __device__ constexpr size_t cand_unit_bytes(int G, int elem_bytes) {
  return ((size_t)kCandRec * 8 + (size_t)G * kCandRec * 4 + (size_t)kCandRec * kD * elem_bytes + 255) / 256 * 256;
}
__device__ __forceinline__ CandView cand_view(unsigned char* unit_base, int G) {
  CandView c;
  c.composite = reinterpret_cast<unsigned long long*>(unit_base);
  c.logit = reinterpret_cast<float*>(unit_base + (size_t)kCandRec * 8);
  c.v = unit_base + (size_t)kCandRec * 8 + (size_t)G * kCandRec * 4;
  return c;
}

// Device pointers carved out of the caller's workspace.
struct Workspace {
  float* lut;                  // [units][M][C]
  float2* range;               // [units]                       (min, max) score, stand-alone top-k only
  unsigned* hist;              // [2][units][histCopies][kNB]   zero between uses (room for kHistCopies replicas)
  unsigned* cand_count;        // [2][units]   records handed out so far (directly behind hist, zeroed with it)
  unsigned short* bins;        // [units][binStride]  per token: its bin, or kBinWindow inside the two windows
  unsigned char* cand_rec;     // [units] blocks of rec_stride bytes: the candidates' composites, logits and V rows (CandView)
  unsigned long long* stage;   // [units][nblkC][stageStride]: selected ids (front, int32) / candidate composites (ending at word tokC)
  int2* stage_cnt;             // [units][nblkC]     (selected, candidates)
  float* partials;             // [units][npart][G][kD+2]
  int rec_stride;
#ifdef PQC_TRACE
  unsigned long long* trace;   // [3 kernels][kTraceWgs][kTraceSlots] time stamps (debug builds only)
#endif
};

// Phase time stamps for debug builds (-DPQC_TRACE); compiled out otherwise.
#ifdef PQC_TRACE
constexpr int kTraceWgs = 4096, kTraceSlots = 16;
#define PQC_MARK(ws, kid, slot)                                                                              \
  do {                                                                                                       \
    if (threadIdx.x == 0) {                                                                                  \
      const size_t wg_ = (size_t)blockIdx.y * gridDim.x + blockIdx.x;                                        \
      if (wg_ < (size_t)kTraceWgs) (ws).trace[((size_t)(kid)*kTraceWgs + wg_) * kTraceSlots + (slot)] = wall_clock64(); \
    }                                                                                                        \
  } while (0)
#define PQC_NOTE(ws, kid, slot, val)                                                                         \
  do {                                                                                                       \
    if (threadIdx.x == 0) {                                                                                  \
      const size_t wg_ = (size_t)blockIdx.y * gridDim.x + blockIdx.x;                                        \
      if (wg_ < (size_t)kTraceWgs) (ws).trace[((size_t)(kid)*kTraceWgs + wg_) * kTraceSlots + (slot)] = (unsigned long long)(val); \
    }                                                                                                        \
  } while (0)
#else
#define PQC_MARK(ws, kid, slot) \
  do {                          \
  } while (0)
#define PQC_NOTE(ws, kid, slot, val) \
  do {                               \
  } while (0)
#endif

// Marks the end of a group of independent loads: the instruction scheduler may not move
// anything across this point, so the loads above are all issued before their first use
// (left alone it tends to interleave load and use to save registers, which turns one
// memory round trip into many).
#define PQC_LOADS_ISSUED() __builtin_amdgcn_sched_barrier(0)

// ---------------------------------------------------------------- small helpers
__device__ __forceinline__ unsigned score_key(float f) {
  // order-preserving map float -> unsigned (larger score, larger key); -0 == +0
  f += 0.0f;
  unsigned u = __float_as_uint(f);
  return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}

__device__ __forceinline__ float key_score(unsigned k) {  // inverse of score_key
  return __uint_as_float(k ^ ((k >> 31) ? 0x80000000u : 0xffffffffu));
}

__device__ __forceinline__ unsigned long long make_composite(float score, int token) {
  // larger composite = ranks first: higher score, then lower token index
  return ((unsigned long long)score_key(score) << 32) | (unsigned long long)(0xffffffffu - (unsigned)token);
}

__device__ __forceinline__ int composite_token(unsigned long long c) {
  return (int)(0xffffffffu - (unsigned)(c & 0xffffffffull));
}

// Monotone map score -> bin.  Bin 0 takes every score below c0 and is not counted (it holds the middle tokens that no other
// bin does), kFineBins fine bins cover [c0, c1], kHighBins coarse bins lie above c1.  Inside a piece, subtraction, multiplication
// by a non-negative constant and rounding down preserve order.  Only the number of boundary-bin candidates depends on how well
// [c0, c1] brackets the K-th largest score; which tokens are selected never does.  (Should the K-th largest score lie below c0,
// every token of bin 0 becomes a candidate: slow, still exact.)  The order of the retrieved tokens does depend on the edges of the
// threshold bin (its members come last, best first), and so on how (s - c0) * ic rounds: another form of the map (a fused
// multiply-add s * ic + b, for one, which is four instructions instead of eleven) selects the same tokens and puts some in another
// place.  A layer of 8 heads x 32768 tokens, 2x64: 26.7 us, 26.4 with the fused form; 8 x 131072 35.8 and 35.6; 32 x 131072, 4x256, 76.6
// both.
constexpr int kHighBins = 256;
constexpr unsigned kBinWindow = 0xffffu;  // stored bin of a window token: above every threshold
constexpr int kFineBins = kNB - 1 - kHighBins;
struct BinMap {
  float c0, ic, c1, nih;  // start and slope of the fine piece, start and slope (negated) of the coarse piece
};
// Both pieces are computed and added, each clamped to its own bins, without comparisons and selections: a score above c1 fills the
// fine piece, one up to c1 adds nothing of the coarse one.
__device__ __forceinline__ unsigned score_bin(float s, const BinMap& m) {
  const float y = (s - m.c0) * m.ic, down = m.c1 - s, z = down * m.nih;
  int fine;
  unsigned high;  // (these conversions saturate; in C++ they would be undefined for values out of range and NaN)
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(fine) : "v"(y));  // rounds down: negative below c0
  asm("v_cvt_u32_f32 %0, %1" : "=v"(high) : "v"(z));      // truncates; negative values and NaN give 0
  fine = max(-1, min(fine, kFineBins - 1));
  high = min(high, (unsigned)(kHighBins - 1));
  return (unsigned)fine + high + 1u + (__float_as_uint(down) >> 31);  // the last: 1 above c1
}
// Bin layout from bounds lo <= score <= hi and a window [q_lo, q_hi] expected to hold
// the K-th largest score.
__device__ __forceinline__ BinMap make_bins(float lo, float hi, float q_lo, float q_hi) {
  BinMap m;
  m.c0 = fmaxf(lo, q_lo);
  m.c1 = fminf(hi, q_hi);
  if (!(m.c1 > m.c0)) {  // degenerate window: the fine piece over everything
    m.c0 = lo;
    m.c1 = hi;
  }
  // Where a bound is infinite (or the spread is below 1e-28) one of the pieces is a single bin.  For the fine one the slope is not a
  // number: then all products are none, infinite scores' among them, and whatever the conversion makes of that is the same for all.
  const float wc = m.c1 - m.c0, wh = hi - m.c1;
  m.ic = (wc > 1e-30f && wc < 3e38f) ? (float)kFineBins / wc : __builtin_nanf("");
  m.nih = (wh > 1e-30f && wh < 3e38f) ? -((float)kHighBins / wh) : 0.0f;
  return m;
}

// ------------------------------------------------------------ cross-lane helpers
// DPP moves: a lane whose source is outside its row (or masked out) keeps `identity`.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ int dpp_i(int identity, int x) {
  return __builtin_amdgcn_update_dpp(identity, x, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_f(float identity, float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(identity), __float_as_int(x), CTRL, ROW_MASK, 0xf, false));
}
// row_shr:1,2,4,8 then row_bcast:15 (rows 1,3) and row_bcast:31 (rows 2,3)
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += dpp_i<0x111>(0, v);
  v += dpp_i<0x112>(0, v);
  v += dpp_i<0x114>(0, v);
  v += dpp_i<0x118>(0, v);
  v += dpp_i<0x142, 0xa>(0, v);
  v += dpp_i<0x143, 0xc>(0, v);
  return v;
}
__device__ __forceinline__ int wave_last(int v) { return __builtin_amdgcn_readlane(v, 63); }
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f<0x111>(0.0f, v);
  v += dpp_f<0x112>(0.0f, v);
  v += dpp_f<0x114>(0.0f, v);
  v += dpp_f<0x118>(0.0f, v);
  v += dpp_f<0x142, 0xa>(0.0f, v);
  v += dpp_f<0x143, 0xc>(0.0f, v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f<0x111>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x112>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x114>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x118>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x142, 0xa>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x143, 0xc>(-INFINITY, v));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_min(float v) { return -wave_max(-v); }
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
  v = max(v, (unsigned)dpp_i<0x111>(0, (int)v));
  v = max(v, (unsigned)dpp_i<0x112>(0, (int)v));
  v = max(v, (unsigned)dpp_i<0x114>(0, (int)v));
  v = max(v, (unsigned)dpp_i<0x118>(0, (int)v));
  v = max(v, (unsigned)dpp_i<0x142, 0xa>(0, (int)v));
  v = max(v, (unsigned)dpp_i<0x143, 0xc>(0, (int)v));
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// Sum over the 16 lanes of a DPP row; every lane of the row receives the total.
__device__ __forceinline__ float group16_sum(float x) {
  x += dpp_f<0xB1>(0.0f, x);   // quad_perm [1,0,3,2]: neighbour in the pair
  x += dpp_f<0x4E>(0.0f, x);   // quad_perm [2,3,0,1]: other pair of the quad
  x += dpp_f<0x141>(0.0f, x);  // row_half_mirror: other quad of the half row
  x += dpp_f<0x140>(0.0f, x);  // row_mirror: other half of the row
  return x;
}

// Two 16-bit values at a time: a - b (0 where b is larger), and the smaller of a and b.
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2_t;
__device__ __forceinline__ unsigned pk_sub_sat_u16(unsigned a, unsigned b) {
  return __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}
__device__ __forceinline__ unsigned pk_min_u16(unsigned a, unsigned b) {
  return __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}

// Exclusive prefix sum over the threads of a workgroup (NT threads, multiple of 64).
template <int NT>
__device__ __forceinline__ int block_exclusive_scan(int v, int* total, int* sm /* [2*(NT/64)+1] */) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int inc = wave_inclusive_scan(v);
  if (lane == 63) sm[w] = inc;
  __syncthreads();
  if (w == 0) {
    const int s = lane < NW ? sm[lane] : 0;
    const int si = wave_inclusive_scan(s);
    if (lane < NW) sm[NW + lane] = si - s;
    if (lane == NW - 1) sm[2 * NW] = si;
  }
  __syncthreads();
  const int res = inc - v + sm[NW + w];
  *total = sm[2 * NW];
  __syncthreads();
  return res;
}

// --------------------------------------------------------------- look-up table
// Section 2.2 (search) / Section 3.1 step 4: table[j][c] = qs[j*Dm..] . cent[j][c][..]
// with qs the sum of the group's query heads.  Fixed fp32 order: head order for
// the sum, one fused multiply-add chain per entry.  Also derives the score -> bin map
// from bounds on every possible score (lo = sum_j min_c table[j][c], hi likewise with
// max, added in the same order as a score, so that lo <= score <= hi holds in fp32)
// and from the mean and spread the scores would have under uniform code usage.
template <typename T>
__device__ __forceinline__ float load_as_float(const T* p, int i);
template <>
__device__ __forceinline__ float load_as_float<float>(const float* p, int i) {
  return p[i];
}
template <>
__device__ __forceinline__ float load_as_float<bf16_t>(const bf16_t* p, int i) {
  return __uint_as_float((unsigned)p[i].bits << 16);
}

// Centroids travel global -> registers (coalesced, all loads in flight at once) -> a
// padded LDS tile -> one thread per table entry runs the chain.  With 512 threads and more the
// tile holds the whole table (C*(kD+M) floats, up to 136 KB of the CU's 160 KB) and there
// is a single pass over the centroids; with fewer threads the table goes through a tile of kLutTileFloats
// floats piece by piece.
constexpr int kLutTileFloats = 8192;
// Row stride of the whole-table tile.  Long rows (one or two partitions: few entries, few busy
// waves) are padded by four floats and read 128 bits at a time; short rows keep every thread busy
// and measured faster with an odd stride and 32-bit accesses.
__host__ __device__ constexpr int lut_row_stride(int M) { return M <= 2 ? kD / M + 4 : kD / M + 1; }
__host__ __device__ constexpr int lut_tile_floats(int nt, int M, int C) {
  return nt >= 512 ? M * C * lut_row_stride(M) : kLutTileFloats + kLutTileFloats / (kD / M);
}
// The group's query heads: all loads first (clamped, straight-line), the caller's `issue_first` behind them, then the sum in head order.
template <typename T, class FirstFn, class IssueFn>
__device__ __forceinline__ void sum_query(const T* __restrict__ q, int G, float* qs, FirstFn issue_first, IssueFn issue_more) {
  const int dq = threadIdx.x & (kD - 1);
  T qr[8];  // (as they are in memory: a conversion here would be waited for in front of the loads that follow)
#pragma unroll
  for (int h = 0; h < 8; ++h) qr[h] = q[min(h, G - 1) * kD + dq];
  PQC_LOADS_ISSUED();
  issue_first();
  // Loads return in issue order: whatever the caller streams from HBM goes behind the table's
  // (mostly L2-resident) centroids, so that the table is built while that stream arrives.
  PQC_LOADS_ISSUED();
  issue_more();
  PQC_LOADS_ISSUED();
  float qv[8];
#pragma unroll
  for (int h = 0; h < 8; ++h) qv[h] = load_as_float<T>(&qr[h], 0);
  float a = qv[0];
#pragma unroll
  for (int h = 1; h < 8; ++h) {
    const float t = __fadd_rn(a, qv[h]);
    a = h < G ? t : a;  // select, not branch: keeps the eight loads above in flight together
  }
  qs[dq] = a;  // every thread (tid and tid + kD hold the same sum): a branch here would split the block, and the
               // compiler would then move the centroid loads above down to their use, behind this wait
}

// The first half of it in whole-table mode: the group's query heads summed into qs and the centroids in the tile, visible behind a
// barrier of the caller's.  VWP: 16-byte pieces of the table per thread; VWP * NT * 4 floats must cover M*C*Dm.
template <typename T, int NT, int M, int VWP, class MarkFn, class EarlyFn, class IssueFn>
__device__ __forceinline__ void lut_stage(const T* __restrict__ q /* [G][kD] of this unit */, const float* __restrict__ cent /* [M][C][Dm] */,
                                          int G, int C, float* qs, float* tile /* [lut_tile_floats(NT, M, C)] */, MarkFn mark,
                                          EarlyFn issue_early /* the caller's loads that go right behind the thread's centroid loads, always as
                                                                 many: the wait for the centroids counts them */,
                                          IssueFn issue_more /* and those behind its tile stores */) {
  constexpr int Dm = kD / M, RS = lut_row_stride(M);
  const int tid = threadIdx.x, total = M * C * Dm;  // floats, a multiple of 4
  // (a native vector type: a float4 struct copied from global memory to LDS is turned into one 16-byte copy at
  // the place of the store, which puts every load behind the waits in front of it, one round trip after the other)
  const f32x4_t* centv = reinterpret_cast<const f32x4_t*>(cent);
  f32x4_t vw[VWP];
  auto load_centroids = [&]() {
#pragma unroll
    for (int x = 0; x < VWP; ++x) vw[x] = centv[min(x * NT + tid, total / 4 - 1)];
  };
  // With 512 threads the query goes in front of the centroids, many per thread: behind them its sum waits for nearly all of them, and
  // left alone the compiler takes either order (8 units of 1000 tokens, two query heads, us per layer: 4x256 17.7 and 17.4, 2x256 17.4, 17.1; the
  // histogram kernel's 1024 threads have few: 1 of 106444, 4x64, 23.2 behind them, 23.4 in front).
  if constexpr (NT >= 1024) load_centroids();
  sum_query<T>(q, G, qs, [&]() {
    if constexpr (NT < 1024) load_centroids();
  }, issue_early);
  mark(8);
#pragma unroll
  for (int x = 0; x < VWP; ++x) {
    // No branch around the store: a thread beyond the table holds the table's last float4 (its load was clamped)
    // and writes it to that float4's place once more.  With a branch here the compiler moves each load down into
    // its branch and waits for it there, one memory round trip after the other.
    const int fl = min((x * NT + tid) * 4, total - 4);  // float index inside the table
    const int row = fl / Dm, col = fl % Dm;             // Dm is a multiple of 4: one row per float4
    float* dst = tile + row * RS + col;
    if constexpr (RS % 4 == 0) {
      *reinterpret_cast<f32x4_t*>(dst) = vw[x];
    } else {
      dst[0] = vw[x][0]; dst[1] = vw[x][1]; dst[2] = vw[x][2]; dst[3] = vw[x][3];
    }
  }
  // the caller's stream from HBM is requested now, behind every wave's centroid loads (a compute unit's loads
  // pass through one address unit): the table is built while that stream arrives
  issue_more();
  PQC_LOADS_ISSUED();
  mark(10);
}

template <typename T, int NT, int M, class MarkFn, class IssueFn, int VWP = (256 * kD) / (4 * NT)>
__device__ __forceinline__ float2 build_lut(const T* __restrict__ q, const float* __restrict__ cent, int G, int C, float* lut, float* qs,
                                            float* red /* [4*8] */, float* tile, MarkFn mark, IssueFn issue_more) {
  constexpr int Dm = kD / M, RS = lut_row_stride(M);
  constexpr bool kWhole = NT >= 512;
  constexpr int VPG = kLutTileFloats / (4 * NT);      // float4 per thread per tile (piecewise mode)
  constexpr int NG = (256 * kD) / kLutTileFloats;      // tiles at the largest C (piecewise mode)
  const int tid = threadIdx.x;
  const int total = M * C * Dm;                        // floats, a multiple of 4
  const float4* cent4 = reinterpret_cast<const float4*>(cent);
  if constexpr (kWhole) {
    lut_stage<T, NT, M, VWP>(q, cent, G, C, qs, tile, mark, []() {}, issue_more);
    unsigned* mm = reinterpret_cast<unsigned*>(red);  // [0..8): smallest entry of a partition, [8..16): largest, as score keys
    if (tid < 16) mm[tid] = tid < 8 ? 0xffffffffu : 0u;
    __syncthreads();  // tile, qs and mm visible
    mark(11);
    for (int e0 = 0; e0 + (tid & ~63) < M * C; e0 += NT) {  // per wave: the wave-wide reductions below need every lane
      const int e = e0 + tid;
      const bool valid = e < M * C;
      const int ec = valid ? e : 0;
      const int j = ec / C, c = ec - j * C;
      const float* qj = qs + j * Dm;
      const float* cr = tile + ec * RS;
      float p = 0.0f;
      if constexpr (RS % 4 == 0) {
        // Few entries, so few busy waves and nothing to hide the LDS latency behind: the operands are read two
        // stages of four 16-byte pieces ahead of the chain (left alone the compiler reads one piece ahead and the
        // chain waits for LDS at every fourth step).
        constexpr int kStages = Dm / 16;
        const f32x4_t* qv4 = reinterpret_cast<const f32x4_t*>(qj);
        const f32x4_t* cv4 = reinterpret_cast<const f32x4_t*>(cr);
        f32x4_t qa[2][4], ca[2][4];
#pragma unroll
        for (int st = 0; st < 2 && st < kStages; ++st)
#pragma unroll
          for (int y = 0; y < 4; ++y) {
            qa[st][y] = qv4[st * 4 + y];
            ca[st][y] = cv4[st * 4 + y];
          }
#pragma unroll
        for (int st = 0; st < kStages; ++st) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int y = 0; y < 4; ++y) {
            p = __fmaf_rn(qa[st & 1][y][0], ca[st & 1][y][0], p);
            p = __fmaf_rn(qa[st & 1][y][1], ca[st & 1][y][1], p);
            p = __fmaf_rn(qa[st & 1][y][2], ca[st & 1][y][2], p);
            p = __fmaf_rn(qa[st & 1][y][3], ca[st & 1][y][3], p);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (st + 2 < kStages) {
#pragma unroll
            for (int y = 0; y < 4; ++y) {
              qa[st & 1][y] = qv4[(st + 2) * 4 + y];
              ca[st & 1][y] = cv4[(st + 2) * 4 + y];
            }
          }
        }
      } else {
#pragma unroll
        for (int x = 0; x < Dm / 4; ++x) {  // the query four at a time (one address per wave: a broadcast)
          const float4 qq = reinterpret_cast<const float4*>(qj)[x];
          p = __fmaf_rn(qq.x, cr[4 * x + 0], p);
          p = __fmaf_rn(qq.y, cr[4 * x + 1], p);
          p = __fmaf_rn(qq.z, cr[4 * x + 2], p);
          p = __fmaf_rn(qq.w, cr[4 * x + 3], p);
        }
      }
      if (valid) lut[j * kLutRow + c] = p;
      // the partition's smallest and largest entry (as order-preserving keys): one pair of LDS atomics per wave
      // when the wave's 64 entries lie in one partition, else one pair per entry
      if ((C & 63) == 0) {  // uniform
        const float pmin = wave_min(valid ? p : INFINITY), pmax = wave_max(valid ? p : -INFINITY);
        if ((tid & 63) == 0 && valid) {  // the wave's first entry is valid whenever any is
          atomicMin(&mm[j], score_key(pmin));
          atomicMax(&mm[8 + j], score_key(pmax));
        }
      } else if (valid) {
        atomicMin(&mm[j], score_key(p));
        atomicMax(&mm[8 + j], score_key(p));
      }
    }
    mark(9);
  } else {
    sum_query<T>(q, G, qs, []() {}, issue_more);
    mark(8);
    float4 v[VPG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (g * kLutTileFloats < total) {  // uniform
#pragma unroll
        for (int x = 0; x < VPG; ++x) {
          const int f = g * (kLutTileFloats / 4) + x * NT + tid;
          v[x] = cent4[min(f, total / 4 - 1)];
        }
        if (g > 0) __syncthreads();  // previous tile fully consumed
#pragma unroll
        for (int x = 0; x < VPG; ++x) {
          const int fl = (x * NT + tid) * 4;  // float index inside the tile
          if (g * kLutTileFloats + fl < total) {
            const int row = fl / Dm, col = fl % Dm;
            float* dst = tile + row * (Dm + 1) + col;
            dst[0] = v[x].x; dst[1] = v[x].y; dst[2] = v[x].z; dst[3] = v[x].w;
          }
        }
        __syncthreads();  // tile (and, first time round, qs) visible
        const int rows = min(kLutTileFloats, total - g * kLutTileFloats) / Dm;
        for (int r = tid; r < rows; r += NT) {
          const int e = g * (kLutTileFloats / Dm) + r;
          const int j = e / C, c = e - j * C;
          const float* qj = qs + j * Dm;
          const float* cr = tile + r * (Dm + 1);
          float p = 0.0f;
#pragma unroll
          for (int x = 0; x < Dm; ++x) p = __fmaf_rn(qj[x], cr[x], p);
          lut[j * kLutRow + c] = p;
        }
      }
    }
  }
  __syncthreads();
  mark(13);
  if constexpr (kWhole) {
    // bounds are added in the same order as a score, so lo <= score <= hi holds in fp32
    const unsigned* mm = reinterpret_cast<const unsigned*>(red);
    float lo = key_score(mm[0]), hi = key_score(mm[8]);
    for (int j = 1; j < M; ++j) {
      lo = __fadd_rn(lo, key_score(mm[j]));
      hi = __fadd_rn(hi, key_score(mm[8 + j]));
    }
    return make_float2(lo, hi);
  }
  // per table: min and max (one wave per table)
  const int lane = tid & 63, w = tid >> 6;
  for (int j = w; j < M; j += NT / 64) {
    float mn = INFINITY, mx = -INFINITY;
    for (int c = lane; c < C; c += 64) {
      const float x = lut[j * kLutRow + c];
      mn = fminf(mn, x);
      mx = fmaxf(mx, x);
    }
    mn = wave_min(mn);
    mx = wave_max(mx);
    if (lane == 0) {
      red[j] = mn;
      red[8 + j] = mx;
    }
  }
  __syncthreads();
  // bounds are added in the same order as a score, so lo <= score <= hi holds in fp32
  float lo = red[0], hi = red[8];
  for (int j = 1; j < M; ++j) {
    lo = __fadd_rn(lo, red[j]);
    hi = __fadd_rn(hi, red[8 + j]);
  }
  return make_float2(lo, hi);
}

// The token of sample i of n, spread evenly over the nmid middle tokens: i * nmid / n with n = 1024 or, with fewer tokens, n = nmid
// (there are at most 2^22 tokens).
__device__ __forceinline__ int sample_token(const Shape& s, int i) {
  const unsigned step = s.sampleN == 1024 ? (unsigned)max(0, s.N - s.I - s.L) : 1024u;
  return min(s.N - 1, s.I + (int)(((unsigned)i * step) >> 10));
}

// Where the fine bins go: every workgroup of a unit scores the same `n` sampled tokens,
// histograms them over kSampleBins uniform bins of [lo, hi] and takes the bins that hold the
// sample's rank_hi-th and rank_lo-th largest scores as the window.  The ranks bracket
// the K-th largest of all tokens by several standard errors of the sample quantile, so
// the window almost always holds it (and when it does not, only speed is lost).
constexpr int kSampleBins = 256;
__device__ __forceinline__ float sample_scale(float lo, float hi) {
  const float width = hi - lo;
  return (width > 1e-30f && width < 3e38f) ? (float)kSampleBins / width : 0.0f;
}
__device__ __forceinline__ int sample_bin(float score, float lo, float inv_u) {
  return max(0, min(kSampleBins - 1, __float2int_rz((score - lo) * inv_u)));
}
// One wave walks the histogram (four bins per lane, a wave-wide prefix sum) and, on demand, clears it again; b_hi and b_lo: the bins
// of the two ranks, or -1.
template <bool CLEAR>
__device__ __forceinline__ void walk_samples(unsigned* hist, int rank_hi, int rank_lo, int& b_hi, int& b_lo) {
  constexpr int NBS = kSampleBins, PER = NBS / 64;
  static_assert(PER == 4, "one 16-byte access per lane");
  const int lane = threadIdx.x & 63;
  // lane l owns bins [NBS - (l+1)*PER, NBS - l*PER): the lanes run from the top bin down
  uint4* mine = reinterpret_cast<uint4*>(hist + NBS - (lane + 1) * PER);
  const uint4 x = *mine;
  if constexpr (CLEAR) *mine = make_uint4(0u, 0u, 0u, 0u);
  const int h[PER] = {(int)x.x, (int)x.y, (int)x.z, (int)x.w};
  const int sum = h[0] + h[1] + h[2] + h[3];
  int cum = wave_inclusive_scan(sum) - sum;  // samples in the bins above this lane's
  int r0 = -1, r1 = -1;
#pragma unroll
  for (int e = PER - 1; e >= 0; --e) {  // this lane's bins, from its top one down
    const int b = NBS - (lane + 1) * PER + e;
    if (rank_hi >= 1 && cum < rank_hi && cum + h[e] >= rank_hi) r0 = b;
    if (rank_lo >= 1 && cum < rank_lo && cum + h[e] >= rank_lo) r1 = b;
    cum += h[e];
  }
  // at most one lane finds each of the two bins: its number from that lane
  const unsigned long long m0 = __ballot(r0 >= 0), m1 = __ballot(r1 >= 0);
  b_hi = m0 ? __builtin_amdgcn_readlane(r0, __ffsll((long long)m0) - 1) : -1;
  b_lo = m1 ? __builtin_amdgcn_readlane(r1, __ffsll((long long)m1) - 1) : -1;
}
__device__ __forceinline__ BinMap window_bins(float lo, float hi, int b_hi, int b_lo) {
  const float wu = (hi - lo) * (1.0f / (float)kSampleBins);
  const float q_hi = b_hi >= 0 ? fmaf((float)(b_hi + 1), wu, lo) : hi;
  const float q_lo = b_lo >= 0 ? fmaf((float)b_lo, wu, lo) : lo;
  return make_bins(lo, hi, q_lo, q_hi);
}
// Two barriers: the samples are counted, then the first wave alone walks the histogram.
//   hist  LDS [>= kSampleBins], zero on entry, zero again on return      sm  LDS [2]
// PS samples per thread: thread t holds the samples t, t + NT, ... below n.
template <int NT, int PS>
__device__ __forceinline__ BinMap sample_window(float lo, float hi, const float (&my_score)[PS], int n, int rank_hi, int rank_lo,
                                                unsigned* hist, int* sm) {
  const int tid = threadIdx.x;
  const float inv_u = sample_scale(lo, hi);
#pragma unroll
  for (int x = 0; x < PS; ++x)
    if (x * NT + tid < n) atomicAdd(&hist[sample_bin(my_score[x], lo, inv_u)], 1u);
  __syncthreads();
  if (tid < 64) {
    int b_hi, b_lo;
    walk_samples<true>(hist, rank_hi, rank_lo, b_hi, b_lo);
    if (tid == 0) {
      sm[0] = b_hi;
      sm[1] = b_lo;
    }
  }
  __syncthreads();
  return window_bins(lo, hi, sm[0], sm[1]);
}

// ------------------------------------------------------------------- code scan
// Section 3.1 step 4: a token's score is the sum over partitions of the table entry
// its code names, added left to right.
template <int M>
struct CodeWord;
template <>
struct CodeWord<1> {
  using type = uint8_t;
};
template <>
struct CodeWord<2> {
  using type = uint16_t;
};
template <>
struct CodeWord<4> {
  using type = uint32_t;
};
template <>
struct CodeWord<8> {
  using type = uint64_t;
};

template <int M>
__device__ __forceinline__ float score_from_word(typename CodeWord<M>::type w, const float* lut) {
  float s = lut[(unsigned)(w & 0xff)];
#pragma unroll
  for (int j = 1; j < M; ++j) s = __fadd_rn(s, lut[j * kLutRow + (unsigned)((w >> (8 * j)) & 0xff)]);
  return s;
}

// 16 bytes of codes = P = 16/M consecutive tokens; word i of the chunk.
template <int M>
__device__ __forceinline__ typename CodeWord<M>::type chunk_word(const u32x4_t& raw, int i) {
  const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
  if constexpr (M == 8) {
    return ((unsigned long long)w[2 * i + 1] << 32) | w[2 * i];
  } else if constexpr (M == 4) {
    return w[i];
  } else if constexpr (M == 2) {
    return (uint16_t)(w[i >> 1] >> (16 * (i & 1)));
  } else {
    return (uint8_t)(w[i >> 2] >> (8 * (i & 3)));
  }
}

// ------------------------------------------------------------ threshold search
// Section 3.2 (k-th largest score).  The unit's histogram over kNB monotone score
// bins fixes the bin b* that holds the K-th largest score: bins above it are taken
// whole, bins below dropped, and only b*'s members ("candidates") need ranking.
struct Threshold {
  int bstar;    // kNB when K == 0
  int n_above;  // tokens in bins above bstar
  int need;     // candidates to admit = K - n_above
  int n_cand;   // tokens in bin bstar
};

// Two steps so that a kernel can issue the histogram loads together with its other
// loads: load() only reads (ghist: the unit's kHistCopies replicas), resolve() sums the
// replicas and searches.  Thread tid owns bins [kNB - (tid+1)*PER, kNB - tid*PER).
template <int NT>
struct ThresholdSearch {
  static constexpr int PER = kNB / NT;
  static_assert(PER % 4 == 0, "bins per thread must allow 16-byte loads");
  uint4 x[kHistCopies][PER / 4];
  __device__ __forceinline__ void load(const unsigned* __restrict__ ghist, int copies) {
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) {
      const uint4* src = reinterpret_cast<const uint4*>(ghist + c * kNB + kNB - (threadIdx.x + 1) * PER);
#pragma unroll
      for (int v = 0; v < PER / 4; ++v) x[c][v] = c < copies ? src[v] : make_uint4(0u, 0u, 0u, 0u);  // uniform
    }
  }
  // Two barriers; a barrier of the caller's lies between the last use of sm in front of the call and the first one behind it.
  __device__ __forceinline__ Threshold resolve(int K, int n_mid /* middle tokens of the unit; negative: bin 0 is counted like the others */, int* sm /* [2*(NT/64)+1+4] */) const {
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    unsigned h[PER];  // descending bins: h[e] is bin kNB-1-(tid*PER+e)
#pragma unroll
    for (int e = 0; e < PER; ++e) h[e] = 0u;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c)
#pragma unroll
      for (int v = 0; v < PER / 4; ++v) {
        h[PER - 1 - (4 * v + 0)] += x[c][v].x;
        h[PER - 1 - (4 * v + 1)] += x[c][v].y;
        h[PER - 1 - (4 * v + 2)] += x[c][v].z;
        h[PER - 1 - (4 * v + 3)] += x[c][v].w;
      }
    int sum = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) sum += (int)h[e];
    const int inc = wave_inclusive_scan(sum);
    int* res = sm + 2 * NW + 1;
    if (lane == 63) sm[w] = inc;
    if (tid == 0) {
      res[0] = kNB;
      res[1] = 0;
      res[2] = 0;
      res[3] = 0;
    }
    __syncthreads();
    int cum = inc - sum, total = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int v = sm[i];
      cum += i < w ? v : 0;
      total += v;
    }
    if (n_mid >= 0 && tid == NT - 1) h[PER - 1] = (unsigned)(n_mid - total);  // bin 0 is not counted: it holds the rest
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (K > 0 && cum < K && cum + (int)h[e] >= K) {
        res[0] = kNB - 1 - (tid * PER + e);
        res[1] = cum;
        res[2] = K - cum;
        res[3] = (int)h[e];
      }
      cum += (int)h[e];
    }
    __syncthreads();
    return Threshold{res[0], res[1], res[2], res[3]};
  }
};

// ------------------------------------------------- threshold from code-pair counts
// With M = 2 and C <= 64 a token's score takes one of C*C values, one per pair of codes: given how many middle tokens carry each
// pair, the threshold follows from the table without a pass over the tokens, and a token is classified by one look-up.  A pair has
// the slot c0 + 64 * c1 whatever C is, and a thread of NT the kPairPer<NT> slots from kPairPer<NT> * thread on: they share c1, and have
// whole 16-byte pieces of every array to themselves.
constexpr int kPairSlots = 4096;
constexpr int kPairC = 64;        // largest C
template <int NT>
constexpr int kPairPer = kPairSlots / NT;  // slots per thread: eight or sixteen
constexpr int kPairList = 256;    // pairs resolved by direct ranking; more fall back to a radix search
struct PairLds {
  unsigned cnt[kPairSlots + 128];            // tokens per pair: the middle tokens, or the window tokens that the given counts hold besides
                                             // (kPairsMany: afterwards the list of up to 8192 tokens, and 256 places behind it)
  unsigned short cls[kPairSlots];            // what a token of the pair is, in stored form
  unsigned long long lst[kPairList];         // (key << 32) | count of the pairs in the threshold bin
  int res[4];
  unsigned samples[kSampleBins];             // sampled tokens per coarse bin
  float bounds[4];                           // smallest and largest table entry of either partition
};
// Slots of two tokens whose codes lie in one word (codes beyond 63, which name no centroid, are taken modulo 64).
__device__ __forceinline__ void pair_slots(unsigned word, unsigned& s0, unsigned& s1) {
  const unsigned w = word & 0x3f3f3f3fu;
  s0 = __builtin_amdgcn_udot4(w, 0x00004001u, 0u, false);
  s1 = __builtin_amdgcn_udot4(w, 0x40010000u, 0u, false);
}
// One partition's table of two, up to 64 centroids, by one wave: a lane has one entry.  lo, hi: the smallest and the largest one; BY_KEY:
// in the order of score keys, in which an entry that is not a number is an end of the range like an infinite one (else it is left out).
template <bool BY_KEY>
__device__ __forceinline__ void pair_table(const float* tile, const float* qs, int C, int j, float* lut, float& lo, float& hi) {
  constexpr int Dm = kD / 2, RS = lut_row_stride(2), kStages = Dm / 16;
  const int lane = threadIdx.x & 63;
  const f32x4_t* cv = reinterpret_cast<const f32x4_t*>(tile + (j * C + min(lane, C - 1)) * RS);
  const f32x4_t* qv = reinterpret_cast<const f32x4_t*>(qs + j * Dm);
  float p = 0.0f;
  f32x4_t qa[2][4], ca[2][4];  // two stages of four 16-byte pieces: read ahead of the chain
  auto read = [&](int st) {
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      qa[st & 1][y] = qv[st * 4 + y];
      ca[st & 1][y] = cv[st * 4 + y];
    }
  };
  read(0);
  read(1);
#pragma unroll
  for (int st = 0; st < kStages; ++st) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
      for (int e = 0; e < 4; ++e) p = __fmaf_rn(qa[st & 1][y][e], ca[st & 1][y][e], p);
    __builtin_amdgcn_sched_barrier(0);
    if (st + 2 < kStages) read(st + 2);
  }
  if (lane < C) lut[j * kLutRow + lane] = p;
  if (!BY_KEY && C == 64) {  // uniform
    lo = key_score(score_key(wave_min(p)));
    hi = key_score(score_key(wave_max(p)));
  } else {
    const unsigned key = score_key(p);
    lo = key_score(~wave_max_u32(lane < C ? ~key : 0u));
    hi = key_score(wave_max_u32(lane < C ? key : 0u));
  }
}
// The scores of this thread's slots (entries of centroids that do not exist hold anything).
template <int PER>
__device__ __forceinline__ void pair_scores(const float* lut, float (&sc)[PER]) {
  const int c0 = (int)(threadIdx.x * PER) & 63, c1 = (int)(threadIdx.x * PER) >> 6;
  f32x4_t a[PER / 4];
#pragma unroll
  for (int i = 0; i < PER / 4; ++i) a[i] = *reinterpret_cast<const f32x4_t*>(&lut[c0 + 4 * i]);
  const float y = lut[kLutRow + c1];
#pragma unroll
  for (int i = 0; i < PER; ++i) sc[i] = __fadd_rn(a[i / 4][i % 4], y);
}
template <int PER>
__device__ __forceinline__ void store_classes(unsigned short* cls, const unsigned (&v)[PER]) {
#pragma unroll
  for (int i = 0; i < PER; i += 8)
    *reinterpret_cast<uint4*>(&cls[threadIdx.x * PER + i]) =
        make_uint4(v[i] | (v[i + 1] << 16), v[i + 2] | (v[i + 3] << 16), v[i + 4] | (v[i + 5] << 16), v[i + 6] | (v[i + 7] << 16));
}

// The classes of all pairs by exact score keys: 0 below the K-th largest score, 1 at it, 2 above; visible behind a barrier of the
// caller's.  `count`: middle tokens of this thread's slots; `hist` is zero on entry.
// The pair scores, weighted by their counts, are counted into uniform bins; the few pairs of the bin that holds the K-th largest
// are then ranked.  Scores use the same fp32 order as everywhere.  lo and hi bound them in the order of keys: where one is infinite or
// not a number there is a single bin, and the keys decide.
template <int NT>
__device__ __forceinline__ void pair_classes(const Shape& s, const float* lut, float lo, float hi, const unsigned (&count)[kPairPer<NT>], PairLds& L,
                                             unsigned* hist, int* scan_sm) {
  constexpr int PER = kPairPer<NT>;
  static_assert(PER == 8 || PER == 16, "512 or 256 threads");
  const int tid = threadIdx.x;
  const float width = hi - lo;
  const float inv = (width > 1e-30f && width < 3e38f) ? (float)kNB / width : 0.0f;
  float sc[PER];
  unsigned key[PER];
  int bin[PER];
  pair_scores(lut, sc);
  if (tid == 0) L.res[0] = L.res[1] = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    key[i] = score_key(sc[i]);
    bin[i] = max(0, min(kNB - 1, __float2int_rz((sc[i] - lo) * inv)));
    if (count[i]) atomicAdd(&hist[bin[i]], count[i]);
  }
  __syncthreads();
  ThresholdSearch<NT> ts;
  ts.load(hist, 1);
  const Threshold th = ts.resolve(s.K, -1, scan_sm);
  unsigned kth = 0u;
  if (th.bstar < kNB) {  // uniform
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (count[i] && bin[i] == th.bstar) {
        const int slot = atomicAdd(&L.res[0], 1);
        if (slot < kPairList) L.lst[slot] = ((unsigned long long)key[i] << 32) | count[i];
      }
    __syncthreads();
    const int n_in = L.res[0];
    if (n_in <= 64) {  // uniform; the usual case: every wave ranks them by itself, a pair per lane
      const int lane = tid & 63;
      const unsigned long long mine = L.lst[min(lane, n_in - 1)];
      const unsigned mk = (unsigned)(mine >> 32);
      unsigned above = 0u, same = 0u;
      for (int j0 = 0; j0 < n_in; j0 += 4) {  // four independent LDS reads per round
        unsigned long long o[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = L.lst[min(j0 + x, n_in - 1)];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const unsigned ok = (unsigned)(o[x] >> 32), oc = j0 + x < n_in ? (unsigned)o[x] : 0u;
          above += ok > mk ? oc : 0u;
          same += ok == mk ? oc : 0u;
        }
      }
      const unsigned long long hit = __ballot((int)above < th.need && th.need <= (int)(above + same));
      kth = hit ? (unsigned)__builtin_amdgcn_readlane((int)mk, __ffsll((long long)hit) - 1) : 0u;
    } else if (n_in <= kPairList) {
      if (tid < n_in) {
        const unsigned long long mine = L.lst[tid];
        const unsigned mk = (unsigned)(mine >> 32);
        long long above = 0, same = 0;
        for (int j = 0; j < n_in; ++j) {
          const unsigned long long o = L.lst[j];
          above += (unsigned)(o >> 32) > mk ? (unsigned)o : 0u;
          same += (unsigned)(o >> 32) == mk ? (unsigned)o : 0u;
        }
        if (above < th.need && th.need <= above + same) L.res[1] = (int)mk;
      }
      __syncthreads();
      kth = (unsigned)L.res[1];
    } else {
      // many pairs share the bin (nearly equal scores): 8-bit radix search over their keys
      long long want = th.need;
      for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) hist[tid] = 0u;  // digits
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i)
          if (count[i] && bin[i] == th.bstar && (shift == 24 || (key[i] >> (shift + 8)) == (kth >> (shift + 8))))
            atomicAdd(&hist[(key[i] >> shift) & 255u], count[i]);
        __syncthreads();
        if (tid == 0) {
          long long c2 = 0;
          int dg = 255;
          for (; dg > 0; --dg) {
            if (c2 + (long long)hist[dg] >= want) break;
            c2 += hist[dg];
          }
          L.res[2] = dg;
          L.res[3] = (int)(want - c2);
        }
        __syncthreads();
        kth |= (unsigned)L.res[2] << shift;
        want = L.res[3];
        __syncthreads();
      }
    }
  }
  // No score has the lowest key, so that the K-th largest's is at least 1; nothing lies above the highest.
  const unsigned base = th.bstar < kNB ? max(kth, 1u) - 1u : 0xffffffffu;
  unsigned c[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) c[i] = min(__builtin_elementwise_sub_sat(key[i], base), 2u);
  store_classes(L.cls, c);
}

// ------------------------------------------------------- attention, vector ALU
// Section 2.1 restricted to listed tokens (Section 3.1 step 6).  Lane layout inside
// a wave: sub = lane & 15 owns 8 of the 128 dimensions of a row, slot = lane >> 4
// picks one of 4 rows handled at once; a 16-lane group reads one contiguous row.
// Logits are kept in the log2 domain (q is pre-multiplied by scale*log2(e)).
// Used for fp32 caches, for candidate logits and for the rare slow finalize path.
template <typename T>
struct RowRaw;
template <>
struct RowRaw<bf16_t> {
  uint4 a;
  __device__ __forceinline__ void load(const bf16_t* base, int t, int sub) {
    a = *reinterpret_cast<const uint4*>(base + (size_t)t * kD + sub * 8);
  }
  __device__ __forceinline__ void load_row(const void* row, int sub) {
    a = *reinterpret_cast<const uint4*>(static_cast<const unsigned char*>(row) + sub * 16);
  }
  __device__ __forceinline__ void zero() { a = make_uint4(0, 0, 0, 0); }
  __device__ __forceinline__ void unpack(float (&f)[8]) const {
    f[0] = __uint_as_float(a.x << 16);
    f[1] = __uint_as_float(a.x & 0xffff0000u);
    f[2] = __uint_as_float(a.y << 16);
    f[3] = __uint_as_float(a.y & 0xffff0000u);
    f[4] = __uint_as_float(a.z << 16);
    f[5] = __uint_as_float(a.z & 0xffff0000u);
    f[6] = __uint_as_float(a.w << 16);
    f[7] = __uint_as_float(a.w & 0xffff0000u);
  }
  __device__ __forceinline__ void store(unsigned char* dst, int sub) const { *reinterpret_cast<uint4*>(dst + sub * 16) = a; }
};
template <>
struct RowRaw<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* base, int t, int sub) {
    a = *reinterpret_cast<const float4*>(base + (size_t)t * kD + sub * 4);
    b = *reinterpret_cast<const float4*>(base + (size_t)t * kD + 64 + sub * 4);
  }
  __device__ __forceinline__ void load_row(const void* row, int sub) {
    a = *reinterpret_cast<const float4*>(static_cast<const unsigned char*>(row) + sub * 16);
    b = *reinterpret_cast<const float4*>(static_cast<const unsigned char*>(row) + 256 + sub * 16);
  }
  __device__ __forceinline__ void zero() {
    a = make_float4(0, 0, 0, 0);
    b = a;
  }
  __device__ __forceinline__ void unpack(float (&f)[8]) const {
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
  __device__ __forceinline__ void store(unsigned char* dst, int sub) const {
    *reinterpret_cast<float4*>(dst + sub * 16) = a;
    *reinterpret_cast<float4*>(dst + 256 + sub * 16) = b;
  }
};

// Dimension held in register e of lane-group member `sub`.
template <typename T>
__device__ __forceinline__ int owned_dim(int sub, int e);
template <>
__device__ __forceinline__ int owned_dim<bf16_t>(int sub, int e) {
  return sub * 8 + e;
}
template <>
__device__ __forceinline__ int owned_dim<float>(int sub, int e) {
  return e < 4 ? sub * 4 + e : 64 + sub * 4 + (e - 4);
}

template <int G>
struct AttnState {
  float m[G], l[G], acc[G][8];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      m[h] = kNegBig;
      l[h] = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[h][e] = 0.0f;
    }
  }
};

template <typename T, int G>
__device__ __forceinline__ void load_query(const T* __restrict__ q /* [G][kD] */, float factor, float (&qr)[G][8]) {
  const int sub = threadIdx.x & 15;
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) qr[h][e] = load_as_float<T>(q, h * kD + owned_dim<T>(sub, e)) * factor;
}

// Attend the rows list(p), p in [first, count) stepping by `stride`, where every
// wave-iteration covers 4*R consecutive list positions.  list(p) must be valid
// for p < count; tokens are clamped into [0, N).
template <typename T, int G, int R, class ListFn>
__device__ __forceinline__ void attend_rows(const T* __restrict__ kbase, const T* __restrict__ vbase, int N,
                                            ListFn list, int count, int first, int stride,
                                            const float (&qr)[G][8], AttnState<G>& st) {
  const int lane = threadIdx.x & 63;
  const int sub = lane & 15, slot = lane >> 4;
  for (int base = first; base < count; base += stride) {
    RowRaw<T> kr[R], vr[R];
    bool ok[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int p = base + r * 4 + slot;
      ok[r] = p < count;
      if (ok[r]) {
        int t = list(p);
        t = max(0, min(N - 1, t));
        kr[r].load(kbase, t, sub);
        vr[r].load(vbase, t, sub);
      } else {
        kr[r].zero();
        vr[r].zero();
      }
    }
    PQC_LOADS_ISSUED();
    float s[R][G];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float kf[8];
      kr[r].unpack(kf);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float d = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) d = fmaf(qr[h][e], kf[e], d);
        s[r][h] = group16_sum(d);
      }
    }
    float pw[R][G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float mb = st.m[h];
#pragma unroll
      for (int r = 0; r < R; ++r) mb = ok[r] ? fmaxf(mb, s[r][h]) : mb;
      const float corr = __builtin_amdgcn_exp2f(st.m[h] - mb);
      float lsum = 0.0f;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        pw[r][h] = ok[r] ? __builtin_amdgcn_exp2f(s[r][h] - mb) : 0.0f;
        lsum += pw[r][h];
      }
      st.l[h] = st.l[h] * corr + lsum;
      st.m[h] = mb;
#pragma unroll
      for (int e = 0; e < 8; ++e) st.acc[h][e] *= corr;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float vf[8];
      vr[r].unpack(vf);
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) st.acc[h][e] = fmaf(pw[r][h], vf[e], st.acc[h][e]);
    }
  }
}

// Merge the 4 row slots of a wave (all lanes end with the merged state).
template <int G>
__device__ __forceinline__ void merge_slots(AttnState<G>& st) {
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float mo = __shfl_xor(st.m[h], o), lo = __shfl_xor(st.l[h], o);
      const float mn = fmaxf(st.m[h], mo);
      const float a = __builtin_amdgcn_exp2f(st.m[h] - mn), b = __builtin_amdgcn_exp2f(mo - mn);
      st.l[h] = st.l[h] * a + lo * b;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float ao = __shfl_xor(st.acc[h][e], o);
        st.acc[h][e] = st.acc[h][e] * a + ao * b;
      }
      st.m[h] = mn;
    }
  }
}

// Per-wave softmax state in LDS: red[w][h] = { m, l, acc[kD] }.
template <typename T, int G>
__device__ __forceinline__ void stash_wave_state(AttnState<G>& st, float* red) {
  merge_slots<G>(st);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane < 16) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float* dst = red + ((size_t)w * G + h) * (kD + 2);
#pragma unroll
      for (int e = 0; e < 8; ++e) dst[2 + owned_dim<T>(lane, e)] = st.acc[h][e];
      if (lane == 0) {
        dst[0] = st.m[h];
        dst[1] = st.l[h];
      }
    }
  }
}

template <int G, int NW>
__device__ __forceinline__ void combine_waves(const float* red, int h, int d, float& m, float& l, float& acc) {
  m = kNegBig;
#pragma unroll
  for (int w = 0; w < NW; ++w) m = fmaxf(m, red[((size_t)w * G + h) * (kD + 2)]);
  l = 0.0f;
  acc = 0.0f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float* src = red + ((size_t)w * G + h) * (kD + 2);
    const float f = __builtin_amdgcn_exp2f(src[0] - m);
    l = fmaf(src[1], f, l);
    acc = fmaf(src[2 + d], f, acc);
  }
}

// Build switch for the record of why the matrix cores are used: with -DPQC_VECTOR_ATTENTION bf16 caches take the
// vector-ALU attention above, like fp32 caches (a compile-time choice, there is no run-time dispatch between the two).
#ifdef PQC_VECTOR_ATTENTION
constexpr bool kMatrixCoreAttention = false;
#else
constexpr bool kMatrixCoreAttention = true;
#endif

// ------------------------------------------------------ attention, matrix cores
// bf16 caches.  Per wave and per tile of 16 listed rows:
//   S[token][head] = K_tile[16 x 128] . Q^T[128 x 16]     4 x v_mfma_f32_16x16x32_bf16
//   O[head][dim]  += P[head][token]  . V_tile[16 x 128]   8 x 2 x v_mfma_f32_16x16x16_bf16
// Operand layouts (lane l, quad = l / 16, col = l % 16):
//   16x16x32: A[m=col][k=8*quad+e], B[k=8*quad+e][n=col], D[m=4*quad+i][n=col]
//   16x16x16: A[m=col][k=4*quad+e], B[k=4*quad+e][n=col], D[m=4*quad+i][n=col]
// so the QK output (tokens 4*quad+i of head col) is, lane for lane, the A operand of
// the PV product.  Heads G..15 are zero padding.  K rows feed the matrix core straight
// from global memory (lane: row col, 16 bytes at dims 32*kk + 8*quad); V rows are
// transposed through a wave-private LDS tile (row stride 264 bytes: the four quads of
// a transposed read land in different banks).  P is split into two bf16 terms
// (p = hi + lo, error 2^-17) because one bf16 term alone would cost 2^-9 of the result.
//
// Softmax: a wave first computes the logits of a stage of up to kMfmaTiles tiles,
// takes its maximum per head, rescales O once if the maximum grew, then accumulates.
constexpr int kMfmaTiles = 2;          // tiles (of 16 rows) per stage and wave
constexpr int kVTileStride = 264;      // bytes per V row in the LDS transpose tile
constexpr int kVTileBytes = 16 * kVTileStride;

struct MfmaState {
  f32x4_t o[8];  // O[head 4*quad+i][dim 16*j + col]
  float m, l;    // head col, over this lane's tokens (log2 domain); merged across quads at the end
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    m = kNegBig;
    l = 0.0f;
  }
};

// Q^T fragments (B operand of the QK product) for this lane; heads >= G are zero.
__device__ __forceinline__ void load_q_frags(const bf16_t* __restrict__ q /* [G][kD] */, int G, bf16x8_t (&qf)[4]) {
  const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    uint4 raw = make_uint4(0, 0, 0, 0);
    if (col < G) raw = *reinterpret_cast<const uint4*>(q + (size_t)col * kD + 32 * kk + 8 * quad);
    __builtin_memcpy(&qf[kk], &raw, 16);
  }
}

__device__ __forceinline__ unsigned bf16_round_bits(float f) {  // round to nearest even, finite inputs
  const unsigned u = __float_as_uint(f);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// One stage = kMfmaTiles tiles.  Two stages are kept in registers: while one is being
// consumed the loads of the next are in flight, so a wave never sits without outstanding
// memory requests until its rows run out.  Loads are unconditional (positions past the
// end of the list re-read its last row, which the caches hold); masking happens on the
// logits.
struct MfmaStage {
  uint4 kr[kMfmaTiles][4], vr[kMfmaTiles][4];
};

template <class ListFn>
__device__ __forceinline__ void mfma_issue(const bf16_t* __restrict__ kbase, const bf16_t* __restrict__ vbase, int N,
                                           ListFn list, int count, int base, MfmaStage& g) {
  const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
#pragma unroll
  for (int tl = 0; tl < kMfmaTiles; ++tl) {
    int t = list(min(base + tl * 16 + col, count - 1));
    t = max(0, min(N - 1, t));
    const uint4* kp = reinterpret_cast<const uint4*>(kbase + (size_t)t * kD + 8 * quad);
    const uint4* vp = reinterpret_cast<const uint4*>(vbase + (size_t)t * kD + 8 * quad);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      g.kr[tl][kk] = kp[4 * kk];  // dims 32*kk + 8*quad .. +7
      g.vr[tl][kk] = vp[4 * kk];
    }
  }
}

__device__ __forceinline__ void mfma_consume(const MfmaStage& g, int count, int base, float scale_log2e,
                                             const bf16x8_t (&qf)[4], unsigned char* vt, MfmaState& st) {
  const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
  // logits of the stage
  f32x4_t s[kMfmaTiles];
  float mx = kNegBig;
#pragma unroll
  for (int tl = 0; tl < kMfmaTiles; ++tl) {
    s[tl] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (base + tl * 16 < count) {  // wave-uniform
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        bf16x8_t a;
        __builtin_memcpy(&a, &g.kr[tl][kk], 16);
        s[tl] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[kk], s[tl], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool ok = base + tl * 16 + 4 * quad + i < count;
        s[tl][i] = ok ? s[tl][i] * scale_log2e : kNegBig;
        mx = fmaxf(mx, s[tl][i]);
      }
    }
  }
  // the stage's maximum per head (over the four quads: row_ror 16 and 32 of the wave), and the
  // one-off rescale of O
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  const float mnew = fmaxf(st.m, mx);
  const float corr = __builtin_amdgcn_exp2f(st.m - mnew);
  st.l *= corr;
  st.m = mnew;
  if (__any(corr != 1.0f)) {
    float cr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) cr[i] = __shfl(corr, 4 * quad + i);  // corr of head 4*quad+i lives in lane col == that head
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) st.o[j][i] *= cr[i];
  }
  // accumulate
#pragma unroll
  for (int tl = 0; tl < kMfmaTiles; ++tl) {
    if (base + tl * 16 < count) {
      // V tile -> LDS, row `col`, bytes 64*kk + 16*quad (two 8-byte stores: rows are 8-byte aligned)
      unsigned char* vrow = vt + col * kVTileStride + 16 * quad;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        *reinterpret_cast<uint2*>(vrow + 64 * kk) = make_uint2(g.vr[tl][kk].x, g.vr[tl][kk].y);
        *reinterpret_cast<uint2*>(vrow + 64 * kk + 8) = make_uint2(g.vr[tl][kk].z, g.vr[tl][kk].w);
      }
      // P = exp2(S - m), as hi + lo bf16 terms (masked rows hold kNegBig: P = 0)
      unsigned hi[4], lo[4];
      float psum = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = __builtin_amdgcn_exp2f(s[tl][i] - mnew);
        psum += p;
        hi[i] = bf16_round_bits(p);
        lo[i] = bf16_round_bits(p - __uint_as_float(hi[i] << 16));
      }
      st.l += psum;
      s16x4_t pa_hi, pa_lo;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        pa_hi[i] = (short)hi[i];
        pa_lo[i] = (short)lo[i];
      }
      // the wave's LDS stores must land before its lanes read each other's rows
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const unsigned short* vt16 = reinterpret_cast<const unsigned short*>(vt);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        s16x4_t vb;  // B[k = token 4*quad+e][n = dim 16*j + col]
#pragma unroll
        for (int e = 0; e < 4; ++e) vb[e] = (short)vt16[(4 * quad + e) * (kVTileStride / 2) + 16 * j + col];
        st.o[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa_hi, vb, st.o[j], 0, 0, 0);
        st.o[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa_lo, vb, st.o[j], 0, 0, 0);
      }
      // tile fully read before the next tile overwrites it
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
}

// Rows list(first), list(first+1), ... in stages of 16*kMfmaTiles positions, `stride` apart.
template <class ListFn>
__device__ __forceinline__ void mfma_attend(const bf16_t* __restrict__ kbase, const bf16_t* __restrict__ vbase, int N,
                                            ListFn list, int count, int first, int stride, float scale_log2e,
                                            const bf16x8_t (&qf)[4], unsigned char* vt /* wave-private LDS [kVTileBytes] */,
                                            MfmaState& st) {
  if (first >= count) return;  // wave-uniform
  MfmaStage ga, gb;
  int base = first;
  mfma_issue(kbase, vbase, N, list, count, base, ga);
  for (;;) {
    mfma_issue(kbase, vbase, N, list, count, base + stride, gb);
    PQC_LOADS_ISSUED();
    mfma_consume(ga, count, base, scale_log2e, qf, vt, st);
    base += stride;
    if (base >= count) break;
    mfma_issue(kbase, vbase, N, list, count, base + stride, ga);
    PQC_LOADS_ISSUED();
    mfma_consume(gb, count, base, scale_log2e, qf, vt, st);
    base += stride;
    if (base >= count) break;
  }
}

// Per-wave state -> red[w][h] = { m, l, acc[kD] } (same slots as the vector path).
template <int G>
__device__ __forceinline__ void mfma_stash_wave_state(MfmaState& st, float* red) {
  const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4, w = threadIdx.x >> 6;
  // the four quads of head `col` hold partial sums under one shared maximum
  float l = st.l;
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (quad == 0 && col < G) {
    float* dst = red + ((size_t)w * G + col) * (kD + 2);
    dst[0] = st.m;
    dst[1] = l;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int h = 4 * quad + i;
    if (h < G) {
      float* dst = red + ((size_t)w * G + h) * (kD + 2) + 2;
#pragma unroll
      for (int j = 0; j < 8; ++j) dst[16 * j + col] = st.o[j][i];
    }
  }
}

}  // namespace pqc
