// PQ construction on the GPU (paper, Section 2.2 "index construction" and Section 3.1
// step 2): per (sequence, KV head, partition) Lloyd K-Means over the keys' sub-vectors,
// and the nearest-centroid code of a token that leaves the local window (Section 3.1,
// last paragraph; Algorithm 2 "PQArgNearest").
//
// Distances are compared in fp32; the lowest centroid index wins ties.  Centroid sums
// are accumulated in 64-bit fixed point (2^-20 resolution), which makes the update
// independent of summation order and therefore reproducible; an empty cluster keeps its
// centroid.
#pragma once
#include <type_traits>

#include "pqc_device.h"

namespace pqc {

constexpr int kFixShift = 20;

struct BuildShape {
  int units, N, M, C, Dm;
  int cap;  // tokens the key and code tensors hold per unit (>= N): their stride between units
};

// centroids[u][j][c][:] = keys[u][init_idx[u][j][c]][j*Dm : (j+1)*Dm]; member sums and counts cleared, so many sets of them
template <typename T>
__global__ __launch_bounds__(256) void pq_init_kernel(BuildShape s, const T* __restrict__ keys,
                                                      const int* __restrict__ init_idx, float* __restrict__ cent,
                                                      unsigned long long* __restrict__ sums, unsigned* __restrict__ counts, int sets) {
  const int uj = blockIdx.y, u = uj / s.M, j = uj % s.M;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= s.C * s.Dm) return;
  const int c = i / s.Dm, e = i % s.Dm;
  int t = init_idx[(size_t)uj * s.C + c];
  t = max(0, min(s.N - 1, t));
  cent[(size_t)uj * s.C * s.Dm + i] = load_as_float<T>(keys, ((size_t)u * s.cap + t) * kD + j * s.Dm + e);
  if (!sums) return;  // no round adds to them
  for (int x = 0; x < sets; ++x) {
    const size_t set = (size_t)x * s.units * s.M + uj;
    sums[set * s.C * s.Dm + i] = 0ull;
    if (e == 0) counts[set * s.C + c] = 0u;
  }
}

// One token per unit (the code of an appended token): one thread per centroid, the same distance chain
// as pq_round_vector_kernel, the smallest (distance, centroid) pair through a 64-bit LDS minimum.
template <typename T>
__global__ __launch_bounds__(256) void pq_encode_kernel(BuildShape s, const T* __restrict__ key /* [units][kD] */, int position,
                                                        const float* __restrict__ cent, uint8_t* __restrict__ codes) {
  __shared__ float x[kD];
  __shared__ unsigned long long best;
  const int uj = blockIdx.x, u = uj / s.M, j = uj % s.M, c = threadIdx.x;
  if (c < s.Dm) x[c] = load_as_float<T>(key, (size_t)u * kD + j * s.Dm + c);
  if (c == 0) best = ~0ull;
  __syncthreads();
  if (c < s.C) {
    const float* cr = cent + ((size_t)uj * s.C + c) * s.Dm;
    float d2 = 0.0f;
    for (int e = 0; e < s.Dm; e += 4) {  // Dm is a multiple of 4
      const float4 cv = *reinterpret_cast<const float4*>(cr + e);
      float df = x[e] - cv.x;
      d2 = fmaf(df, df, d2);
      df = x[e + 1] - cv.y;
      d2 = fmaf(df, df, d2);
      df = x[e + 2] - cv.z;
      d2 = fmaf(df, df, d2);
      df = x[e + 3] - cv.w;
      d2 = fmaf(df, df, d2);
    }
    atomicMin(&best, ((unsigned long long)__float_as_uint(d2) << 32) | (unsigned)c);  // d2 >= 0: its bits order like its value
  }
  __syncthreads();
  if (c == 0) codes[((size_t)u * s.cap + position) * s.M + j] = (uint8_t)(best & 0xffu);
}

// ------------------------------------------------------------- one K-Means round
// Assignment of every token to its nearest centroid and, in the same pass over the keys, the sums of the new
// centroids' members.  A workgroup owns one range of tokens of one (unit, partition): it stages the centroids in LDS
// once, streams its keys through registers, and adds each key to an LDS accumulator of its centroid; at the end the
// accumulators are added to the sums of the (unit, partition) in the workspace with atomics (integers: whatever the order).
// The means are taken by the launch behind, by each of its workgroups when it stages the centroids (RoundLink), so that a
// round is one launch; the sums take turns in three places, as one is read, one added to and one cleared at a time.
// With ACCUM = false the kernel is the assignment alone and writes codes.
//
// Why so for every number of ranges: a launch of the means costs about 6 us a round with its gap, taking them here about 1.5 and
// the additions of all workgroups at about the same time up to 4.  Against a launch that adds up a set of sums per range (up to 16
// ranges) or takes the means of a shared one, eight rounds: 2048 tokens of one head, 2x64, 108 -> 86 us; 8 heads 129 -> 105; 131072
// tokens x 8 heads 717 -> 665; 2048 tokens x 4 heads, 4x256, 185 -> 132.  About even where 4 to 16 ranges of one batch each end together
// with 256 centroids: 8192 tokens x 8 heads 259 -> 258, 32768 x 4 347 -> 353; one shared set with a launch for the means is slower there
// too, 277 and 365 us.
//
// Sums are 64-bit integers of the values in fixed point (2^-20, round to nearest even), so the result does not depend
// on the order of tokens, waves or workgroups.  The conversion is one addition in double precision: x + 1.5 * 2^32 has
// its last bit at 2^-20, so its bit pattern is the pattern of 1.5 * 2^32 plus the fixed-point integer; the constant is
// taken out again count times when the accumulators are written.  (|x| >= 2^30 takes a conversion of its own.)
struct RoundGrid {
  int ranges;   // token ranges per (unit, partition)
  int tokens;   // tokens per range, a multiple of 16
  int staged;   // centroids staged at a time (all of them when they fit; always all with ACCUM)
};
// What a launch takes over from the round in front of it.  sums null: nothing, the centroids it is given are the ones to use.
struct RoundLink {
  const unsigned long long* sums;  // of that round's members, complete
  const unsigned* counts;
  float* cent;                     // where the means go; not where this launch reads the centroids of the round in front
  unsigned long long* next_sums;   // cleared for the round behind this one, or null
  unsigned* next_counts;
};
constexpr double kFixBias = 6442450944.0;  // 1.5 * 2^32
constexpr long long kFixBiasBits = 0x41f8000000000000ll;
__device__ __forceinline__ unsigned long long fix_biased(float x) { return (unsigned long long)__double_as_longlong((double)x + kFixBias); }
__device__ __forceinline__ unsigned long long fix_biased_large(float x) {
  return (unsigned long long)__float2ll_rn(x * (float)(1 << kFixShift)) + (unsigned long long)kFixBiasBits;
}

// LDS of a round: the staged centroids, then the accumulators and the member counts.  Rows of Dm + 1 sums
// (an odd row length spreads the rows of the centroids that a wave adds to over the banks), or, matrix-core kernel with 64 and
// 128 dimensions, rows of Dm sums, so that the bank of a sum depends on its dimension alone, in the order of sum_place: every
// second 32 dimensions are turned by 16, which lets the sixteen lanes of a quad add to sixteen different sums modulo 32.
__host__ __device__ constexpr int sum_place(int e) { return e ^ ((e >> 1) & 16); }
__host__ __device__ constexpr size_t round_sum_bytes(int C, int Dm) { return (size_t)C * (Dm + 1) * 8 + ((size_t)C * 4 + 15) / 16 * 16; }
__host__ __device__ constexpr int mfma_term_stride(int Dm) { return Dm + 8; }  // bf16 values; 16 bytes of padding
__host__ __device__ constexpr size_t mfma_stage_bytes(int staged, int Dm) {
  return (size_t)((staged + 15) / 16 * 16) * (3 * mfma_term_stride(Dm) * 2 + 4);
}
__host__ __device__ constexpr size_t vector_stage_bytes(int staged, int Dm) { return (size_t)staged * (Dm + 4) * 4; }

// Workgroups go to the eight XCDs round-robin.  The M partitions of a token range read interleaved pieces of the same
// rows (64 or 128 bytes each), so they are placed on one XCD, next to each other, and share the lines in its L2.
__device__ __forceinline__ void round_place(const BuildShape& s, int ranges, int& u, int& j, int& p) {
  const int items = s.units * ranges, lin = blockIdx.x, full = items / 8 * 8;
  int item;
  if (lin < full * s.M) {
    const int i = lin % (8 * s.M);
    item = lin / (8 * s.M) * 8 + (i & 7);
    j = i >> 3;
  } else {
    const int i = lin - full * s.M, left = items - full;
    item = full + i % left;
    j = i / left;
  }
  u = item / ranges;
  p = item % ranges;
}

// One division serves the values of a centroid; the quotient is corrected by its remainder.
__device__ __forceinline__ float fixed_mean(unsigned long long sum, unsigned count) {
  const double n = (double)count, inv = 1.0 / n, v = (double)(long long)sum * (1.0 / (double)(1 << kFixShift)), q = v * inv;
  return (float)fma(fma(-q, n, v), inv, q);
}

enum class SumRow { kOdd, kPlain, kPlaced };  // rows of Dm + 1 sums; of Dm sums; of Dm sums in the order of sum_place
template <SumRow ROW, int DM>
__device__ __forceinline__ int sum_index(int c, int e) {
  return ROW == SumRow::kOdd ? c * (DM + 1) + e : c * DM + (ROW == SumRow::kPlaced ? sum_place(e) : e);
}

// The means of the round in front, handed to put(first of four values, the values) one by one over the workgroup; an empty
// cluster keeps its centroid.  The first range of a (unit, partition) writes them out for the launch behind, and every range
// clears its share of the sums that launch adds to.
template <int DM, int NT, class Put>
__device__ __forceinline__ void linked_means(const BuildShape& s, const RoundGrid& r, const RoundLink& k, int uj, int p,
                                             const float* cent, Put put) {
  constexpr int B = 2;  // groups of four values in flight per thread
  const int n = s.C * DM, n4 = n / 4;
  const ulonglong2* sp = reinterpret_cast<const ulonglong2*>(k.sums + (size_t)uj * n);
  const f32x4_t* op = reinterpret_cast<const f32x4_t*>(cent + (size_t)uj * n);
  f32x4_t* out = reinterpret_cast<f32x4_t*>(k.cent + (size_t)uj * n);
  for (int i0 = threadIdx.x; i0 < n4; i0 += B * NT) {
    ulonglong2 a[B], b[B];
    unsigned m[B];
#pragma unroll
    for (int x = 0; x < B; ++x) {
      const int i = min(i0 + x * NT, n4 - 1);
      a[x] = sp[2 * i];
      b[x] = sp[2 * i + 1];
      m[x] = k.counts[(size_t)uj * s.C + i / (DM / 4)];
    }
    PQC_LOADS_ISSUED();
#pragma unroll
    for (int x = 0; x < B; ++x) {
      const int i = i0 + x * NT;
      if (i < n4) {
        f32x4_t v;
        if (m[x])
          v = f32x4_t{fixed_mean(a[x].x, m[x]), fixed_mean(a[x].y, m[x]), fixed_mean(b[x].x, m[x]), fixed_mean(b[x].y, m[x])};
        else
          v = op[i];
        put(4 * i, v);
        if (p == 0) out[i] = v;
      }
    }
  }
  if (k.next_sums) {
    const int end = (int)((long long)n * (p + 1) / r.ranges), cend = (int)((long long)s.C * (p + 1) / r.ranges);
    for (int i = (int)((long long)n * p / r.ranges) + threadIdx.x; i < end; i += NT) k.next_sums[(size_t)uj * n + i] = 0ull;
    for (int i = (int)((long long)s.C * p / r.ranges) + threadIdx.x; i < cend; i += NT) k.next_counts[(size_t)uj * s.C + i] = 0u;
  }
}

// The accumulators to the workspace; a workgroup that owns all tokens of its (unit, partition) writes the new centroids
// itself (nobody else reads them in this launch, and it has staged the old ones).
template <SumRow ROW, int DM>
__device__ __forceinline__ void round_flush(const BuildShape& s, const RoundGrid& r, int uj, int p, const unsigned long long* sums,
                                            const unsigned* cnt, float* __restrict__ cent, unsigned long long* __restrict__ part_sums,
                                            unsigned* __restrict__ part_counts) {
  const int n = s.C * DM;
  // ranges start at different places of the sums they share: they finish at about the same time
  const int first = (int)((long long)n * p / r.ranges) & ~63;
  int tid = threadIdx.x;
  asm("" : "+v"(tid));  // (else places of the flush are kept in registers across the whole round)
  for (int i0 = tid; i0 < n; i0 += blockDim.x) {
    const int i = i0 + first < n ? i0 + first : i0 + first - n;
    const int c = i / DM, e = i % DM;
    const unsigned long long v = sums[sum_index<ROW, DM>(c, e)] - (unsigned long long)cnt[c] * (unsigned long long)kFixBiasBits;
    if (!cnt[c]) continue;
    if (r.ranges == 1)
      cent[(size_t)uj * n + i] = fixed_mean(v, cnt[c]);
    else
      atomicAdd(&part_sums[(size_t)uj * n + i], v);
  }
  if (r.ranges > 1)
    for (int i = tid; i < s.C; i += blockDim.x)
      if (cnt[i]) atomicAdd(&part_counts[(size_t)uj * s.C + i], cnt[i]);
}

// Eight bf16 values turned: value e becomes the one that was value (e + n) modulo 8, n < 8.
__device__ __forceinline__ void turn_left(unsigned (&v)[4], int n) {
  const unsigned a[4] = {n & 2 ? v[1] : v[0], n & 2 ? v[2] : v[1], n & 2 ? v[3] : v[2], n & 2 ? v[0] : v[3]};
  const unsigned b[4] = {n & 4 ? a[2] : a[0], n & 4 ? a[3] : a[1], n & 4 ? a[0] : a[2], n & 4 ? a[1] : a[3]};
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_alignbit(b[(i + 1) & 3], b[i], (n & 1) * 16);
}

// if (low < best) { best = low; index = c; kept = v; }
// Moves under a narrowed execution mask; selections by VCC that follow one another take longer (pq_round_mfma_kernel: KEEP).
__device__ __forceinline__ void keep_lower(float& best, int& index, f32x4_t& kept, float low, int c, const f32x4_t& v) {
  unsigned long long mask;
  float k0 = kept[0], k1 = kept[1], k2 = kept[2], k3 = kept[3];
  asm("v_cmp_lt_f32_e32 vcc, %[low], %[best]\n\t"
      "s_and_saveexec_b64 %[mask], vcc\n\t"
      "v_mov_b32_e32 %[best], %[low]\n\t"
      "v_mov_b32_e32 %[index], %[c]\n\t"
      "v_mov_b32_e32 %[k0], %[v0]\n\t"
      "v_mov_b32_e32 %[k1], %[v1]\n\t"
      "v_mov_b32_e32 %[k2], %[v2]\n\t"
      "v_mov_b32_e32 %[k3], %[v3]\n\t"
      "s_mov_b64 exec, %[mask]"
      : [best] "+v"(best), [index] "+v"(index), [k0] "+v"(k0), [k1] "+v"(k1), [k2] "+v"(k2), [k3] "+v"(k3), [mask] "=&s"(mask)
      : [low] "v"(low), [c] "v"(c), [v0] "v"(v[0]), [v1] "v"(v[1]), [v2] "v"(v[2]), [v3] "v"(v[3])
      : "vcc", "scc");
  kept = f32x4_t{k0, k1, k2, k3};
}

// bf16 keys and sub-vectors of 32, 64 or 128 dimensions: the assignment is a dense contraction (tokens x dimensions by
// dimensions x centroids) and runs on the matrix cores.  The nearest centroid minimises |c|^2 - 2 x.c.  Keys are bf16
// already; an fp32 centroid is split into three bf16 terms that add up to it exactly, so the products are exact and
// only the fp32 accumulation rounds.  With 64 and 128 dimensions the terms are those of -2c and the accumulation starts from |c|^2;
// with 32 the finished product is taken from |c|^2 / 2.  Why the line lies there: with one product per term, starting from |c|^2
// rounds three times at that size instead of twice, with more it takes the partial sums down instead of up.  Sum over all
// tokens and partitions of (squared distance of the assigned centroid - that of the nearest), 64-bit, 8 heads x 131072 tokens
// ~N(0,1) + N(0,4) per channel, ten draws, 256 centroids, taken from the finished product against started from |c|^2: 32
// dimensions 2.60e-2 and 2.77e-2; 64 dimensions 7.6e-2 and 4.7e-2; 128 dimensions 2.1e-1 and 9.7e-2.
// Per wave: TT tiles of 16 tokens as the B operand (kept in registers), 16-centroid
// tiles as the A operand (from LDS), D[centroid 4*quad+i][token col]: a lane keeps the best of its four centroid rows
// for one token per tile, so that the index costs one register per tile and only the four quads are merged at the end
// (with the operands the other way round, sixteen columns of four tokens each had to be merged).
template <int DM, int TT, bool ACCUM>
__global__ __launch_bounds__(1024) void pq_round_mfma_kernel(BuildShape s, RoundGrid r, RoundLink link, const bf16_t* __restrict__ keys,
                                                             float* cent, uint8_t* __restrict__ codes,
                                                             unsigned long long* __restrict__ part_sums,
                                                             unsigned* __restrict__ part_counts) {
  constexpr int NT = 1024, NW = NT / 64, KK = DM / 32, RS = mfma_term_stride(DM);
  // With short sub-vectors the comparisons take about as long as the matrix products and do not hide behind them: the four scores
  // of the best tile are kept (9 instructions for four scores instead of 12) and which of them it was is found at the end.  64 heads
  // x 32768 tokens, 4x256, assignment: 395 us, 419 with selections by VCC.  With longer sub-vectors the registers hold keys.
  constexpr bool KEEP = DM == 32;
  constexpr bool FROM_NORM = DM > 32;
  // The form for short ranges has few waves and is bound by latency: the products of its two tiles are under way together (4 heads x
  // 8564 tokens, 4x64, twenty rounds: 229 us, 233 with one tile after the other; 5000 tokens, 4x256, eight: 170 and 172).
  constexpr bool SHORT = TT == 2;
  constexpr int GANG = SHORT ? 2 : 1;
  // 64 and 128 dimensions: sums turned (see sum_place; 131072 tokens x 8 heads, 2x64, eight rounds 900 -> 770 us).  With 32 the
  // turning costs more than the banks give back, as the matrix products and comparisons take longer than the additions.
  constexpr bool TURNED = KK > 1;
  constexpr int SR = TURNED ? DM : DM + 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char round_lds[];
  const int rows = (r.staged + 15) / 16 * 16;
  unsigned short* ct = reinterpret_cast<unsigned short*>(round_lds);  // [3][rows * RS]: hi, mid, lo terms
  float* cn = reinterpret_cast<float*>(round_lds + (size_t)rows * RS * 6);
  unsigned long long* sums = reinterpret_cast<unsigned long long*>(round_lds + mfma_stage_bytes(r.staged, DM));
  unsigned* cnt = reinterpret_cast<unsigned*>(sums + s.C * SR);
  int u, j, p;
  round_place(s, r.ranges, u, j, p);
  const int uj = u * s.M + j, tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6, col = lane & 15, quad = lane >> 4;
  const int t_begin = p * r.tokens, t_end = min(s.N, t_begin + r.tokens);
  const bool one_group = DM <= 64 || s.C <= r.staged;  // then the centroids are staged once (256 of 64 dimensions fit)
  // four values of a staged centroid (FROM_NORM: times -2) as three bf16 terms that add up to each exactly, and its squared norm (or
  // half of it) from the DM / 4 lanes that hold its values
  auto put = [&](int i, const f32x4_t& v) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
    const int row = i / DM, e = i % DM;
    f32x4_t left = FROM_NORM ? -2.0f * v : v;
#pragma unroll
    for (int term = 0; term < 3; ++term) {
      const bf16x4_t b = __builtin_convertvector(left, bf16x4_t);
      left -= __builtin_convertvector(b, f32x4_t);
      __builtin_memcpy(&ct[(term * rows + row) * RS + e], &b, 8);
    }
    float n2 = fmaf(v[3], v[3], fmaf(v[2], v[2], fmaf(v[1], v[1], v[0] * v[0])));
    if constexpr (DM == 32) {  // eight values in one chain, the sums of the chains in pairs
      const float before = dpp_f<0x111>(0.0f, n2);
      n2 = fmaf(v[3], v[3], fmaf(v[2], v[2], fmaf(v[1], v[1], fmaf(v[0], v[0], before))));  // (in every second lane)
      n2 += dpp_f<0x112>(0.0f, n2);
      n2 += dpp_f<0x114>(0.0f, n2);
      if (e == DM - 4) cn[row] = 0.5f * n2;
    } else {
      n2 += dpp_f<0xB1>(0.0f, n2);
      n2 += dpp_f<0x4E>(0.0f, n2);
      n2 += dpp_f<0x141>(0.0f, n2);
      n2 += dpp_f<0x140>(0.0f, n2);
      if constexpr (DM >= 128) n2 += __shfl_xor(n2, 16);
      if (e == 0) cn[row] = n2;
    }
  };
  auto pad = [&](int nc) {  // rows that hold no centroid lose always (and zero, so that no stale bits of LDS reach the products)
    for (int i = tid; i < (rows - nc) * DM; i += NT) {
      const int o = (nc + i / DM) * RS + (i % DM);
      ct[o] = ct[rows * RS + o] = ct[2 * rows * RS + o] = 0;
    }
    for (int i = nc + tid; i < rows; i += NT) cn[i] = INFINITY;
  };
  auto stage = [&](int c0) {
    const int nc = min(r.staged, s.C - c0), n4 = nc * (DM / 4);
    const f32x4_t* src = reinterpret_cast<const f32x4_t*>(cent + ((size_t)uj * s.C + c0) * DM);
    for (int i0 = tid; i0 < n4; i0 += 2 * NT) {
      const f32x4_t v0 = src[i0], v1 = src[min(i0 + NT, n4 - 1)];
      put(4 * i0, v0);
      if (i0 + NT < n4) put(4 * (i0 + NT), v1);
    }
    pad(nc);
  };
  const int turn = col & 7;      // where a lane starts in the eight dimensions it holds, so that the lanes of a quad spread
  const bool upper = col >= 8;
  if (link.sums) {  // (all centroids are staged at once)
    linked_means<DM, NT>(s, r, link, uj, p, cent, put);
    pad(s.C);
  } else if (one_group) {
    stage(0);
  }
  if constexpr (ACCUM) {
    for (int i = tid; i < s.C * SR; i += NT) sums[i] = 0ull;
    for (int i = tid; i < s.C; i += NT) cnt[i] = 0u;
  }
  if (one_group) __syncthreads();
  for (int b0 = t_begin; b0 < t_end; b0 += NW * 16 * TT) {  // workgroup-uniform
    const int tok0 = b0 + w * 16 * TT;
    const bool live = tok0 < t_end;  // wave-uniform
    bf16x8_t x[TT][KK];              // tile tt: token col, dims 32*kk + 8*quad .. +7
    float best[TT];    // smallest score of this lane's centroid rows for the token
    f32x4_t kept[TT];  // KEEP: the four scores of the tile of centroids that holds it
    int bidx[TT];      // its centroid (KEEP: the first of those four)
    if (live) {
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        const int t = min(tok0 + tt * 16 + col, s.N - 1);
        const uint4* kp = reinterpret_cast<const uint4*>(keys + ((size_t)u * s.cap + t) * kD + j * DM + 8 * quad);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const uint4 raw = kp[4 * kk];
          __builtin_memcpy(&x[tt][kk], &raw, 16);
        }
      }
    }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      best[tt] = INFINITY;
      kept[tt] = f32x4_t{INFINITY, INFINITY, INFINITY, INFINITY};
      bidx[tt] = 0;
    }
    for (int c0 = 0; c0 < s.C; c0 += r.staged) {
      if (!one_group) {
        __syncthreads();
        stage(c0);
        __syncthreads();
      }
      if (!live) continue;
      const int nc = min(r.staged, s.C - c0);
      for (int nt = 0; nt * 16 < nc; ++nt) {
        bf16x8_t a[3][KK];  // centroid row nt*16 + col
#pragma unroll
        for (int term = 0; term < 3; ++term)
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            const uint4 raw = *reinterpret_cast<const uint4*>(&ct[(term * rows + nt * 16 + col) * RS + 32 * kk + 8 * quad]);
            __builtin_memcpy(&a[term][kk], &raw, 16);
          }
        const f32x4_t cnv = *reinterpret_cast<const f32x4_t*>(&cn[nt * 16 + 4 * quad]);
        const int c = c0 + nt * 16 + 4 * quad;
        if constexpr (SHORT) PQC_LOADS_ISSUED();
#pragma unroll
        for (int t0 = 0; t0 < TT; t0 += GANG) {
          f32x4_t acc[GANG];
#pragma unroll
          for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int term = 2; term >= 0; --term)  // small terms first: from zero they add up among themselves
#pragma unroll
              for (int g = 0; g < GANG; ++g)
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[term][kk], x[t0 + g][kk],
                                                                  kk || term < 2 ? acc[g] : FROM_NORM ? cnv : f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          if constexpr (!FROM_NORM)
#pragma unroll
            for (int g = 0; g < GANG; ++g)
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[g][i] = cnv[i] - acc[g][i];
          // strict comparisons: an earlier (lower) centroid of this lane keeps a tie
#pragma unroll
          for (int g = 0; g < GANG; ++g) {
            const int tt = t0 + g;
            if constexpr (KEEP) {
              const float low = fminf(fminf(fminf(fminf(best[tt], acc[g][0]), acc[g][1]), acc[g][2]), acc[g][3]);
              keep_lower(best[tt], bidx[tt], kept[tt], low, c, acc[g]);
            } else {
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const bool lower = acc[g][i] < best[tt];
                best[tt] = lower ? acc[g][i] : best[tt];
                bidx[tt] = lower ? c + i : bidx[tt];
              }
            }
          }
        }
      }
    }
    if (!live) continue;
    // merge the four quads; equal values: lower centroid index
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      if constexpr (KEEP) bidx[tt] += kept[tt][0] == best[tt] ? 0 : kept[tt][1] == best[tt] ? 1 : kept[tt][2] == best[tt] ? 2 : 3;
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float ov = __shfl_xor(best[tt], o);
        const int oi = __shfl_xor(bidx[tt], o);
        const bool take = ov < best[tt] || (ov == best[tt] && oi < bidx[tt]);
        best[tt] = take ? ov : best[tt];
        bidx[tt] = take ? oi : bidx[tt];
      }
    }
    if constexpr (ACCUM) {
      auto add_tiles = [&](auto crowd) {
        constexpr bool CROWDED = decltype(crowd)::value, TURN = TURNED || CROWDED;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          if (tok0 + tt * 16 + col < t_end) {
            unsigned long long* row = sums + bidx[tt] * SR;
            if constexpr (CROWDED) {  // the first token's centroid counts its members of the tile in one go
              const int first = __builtin_amdgcn_readfirstlane(bidx[tt]);
              const int same = __popcll(__ballot(bidx[tt] == first));  // four lanes per token
              if (quad == 0) {
                if (bidx[tt] != first)
                  atomicAdd(&cnt[bidx[tt]], 1u);
                else if (col == 0)
                  atomicAdd(&cnt[first], (unsigned)same / 4);
              }
            } else {
              if (quad == 0) atomicAdd(&cnt[bidx[tt]], 1u);
            }
#pragma unroll
            for (int k0 = 0; k0 < KK; k0 += 2) {
              unsigned rw[2][4];
              __builtin_memcpy(rw[0], &x[tt][k0], 16);
              __builtin_memcpy(rw[1], &x[tt][k0 + 1 < KK ? k0 + 1 : k0], 16);
              if constexpr (KK > 1) {  // the upper eight lanes of a quad take the other 32 dimensions first
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const unsigned lo = rw[0][i];
                  rw[0][i] = upper ? rw[1][i] : lo;
                  rw[1][i] = upper ? lo : rw[1][i];
                }
              }
#pragma unroll
              for (int h = 0; h < (KK > 1 ? 2 : 1); ++h) {
                // dimensions of 32 * kk + 8 * quad + {turn, turn + 1, ... modulo 8}
                unsigned long long* part = row + 32 * k0 + (KK > 1 && (h == 1) != upper ? sum_place(32 + 8 * quad) : 8 * quad);
                float f[8], top = 0.0f;
                int by = turn;
                if constexpr (CROWDED) asm("" : "+v"(by));  // (the places of eight additions are not worth eight registers)
                if constexpr (TURN) turn_left(rw[h], by);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  f[2 * e] = __uint_as_float(rw[h][e] << 16);
                  f[2 * e + 1] = __uint_as_float(rw[h][e] & 0xffff0000u);
                  top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(f[2 * e]), fabsf(f[2 * e + 1])), top);  // NaN stays
                }
                if (__builtin_expect(!(top < 1073741824.0f), 0)) {
#pragma unroll
                  for (int e = 0; e < 8; ++e) atomicAdd(&part[TURN ? (by + e) & 7 : e], fix_biased_large(f[e]));
                } else {
#pragma unroll
                  for (int e = 0; e < 8; ++e) atomicAdd(&part[TURN ? (by + e) & 7 : e], fix_biased(f[e]));
                }
              }
            }
          }
        }
      };
      // Lanes that meet in one address add one after the other.  With 32 dimensions, where half of the wave's first tile shares a
      // centroid, additions are turned too and members counted together (131072 equal tokens x 8 heads, 4x16, three rounds:
      // 1446 -> 294 us; 20000 of one head 67 -> 33 us; keys that spread take the plain additions).
      if constexpr (TURNED) {
        add_tiles(std::false_type{});
      } else if (__popcll(__ballot(bidx[0] == __builtin_amdgcn_readfirstlane(bidx[0]))) >= 32) {  // wave-uniform
        add_tiles(std::true_type{});
      } else {
        add_tiles(std::false_type{});
      }
    } else {
      // lane (quad, col) writes the code of token col of tile 4*k + quad: one store for four tiles
      uint8_t* cp = codes + ((size_t)u * s.cap) * s.M + j;
#pragma unroll
      for (int k = 0; k < TT; k += 4) {
        int code = bidx[k];
#pragma unroll
        for (int y = 1; y < 4; ++y)
          if (k + y < TT) code = quad == y ? bidx[k + y < TT ? k + y : 0] : code;
        const int t = tok0 + (k + quad) * 16 + col;
        if (k + quad < TT && t < t_end) cp[(size_t)t * s.M] = (uint8_t)code;
      }
    }
  }
  if constexpr (ACCUM) {
    __syncthreads();
    round_flush<TURNED ? SumRow::kPlaced : SumRow::kOdd, DM>(s, r, uj, p, sums, cnt, cent, part_sums, part_counts);
  }
}

// Values turned: value e becomes the one that was value (e + n) modulo N, n < 64.  (Bit masks instead of selections,
// which the compiler turns into indexed registers.)
template <int N>
__device__ __forceinline__ void turn_values(float (&x)[N], int n) {
#pragma unroll
  for (int b = 1; b < N && b < 64; b <<= 1) {
    unsigned y[N];
    const unsigned mask = n & b ? ~0u : 0u;
#pragma unroll
    for (int e = 0; e < N; ++e) y[e] = (__float_as_uint(x[(e + b) % N]) & mask) | (__float_as_uint(x[e]) & ~mask);
#pragma unroll
    for (int e = 0; e < N; ++e) x[e] = __uint_as_float(y[e]);
  }
}

// fp32 keys, and sub-vectors of 16 dimensions: on the vector ALU, distances as sum_e (x_e - c_e)^2, e ascending.  Bound by the
// vector ALU: two instructions per dimension and centroid.
// LANES = 1: a lane owns TT tokens and runs all their chains.  LANES = 4: four lanes share a token (lane = 16*quad + token):
// quad q runs the chains of centroids q, q+4, ..., so that short caches still occupy the chip (a single fp32 head of 10007
// tokens is 157 waves at one token per lane), and adds the dimensions q, q+4, ... of the key to the sums.
template <typename T, int DM, int NT, int LANES, int TT, bool ACCUM>
__global__ __launch_bounds__(NT) void pq_round_vector_kernel(BuildShape s, RoundGrid r, RoundLink link, const T* __restrict__ keys, float* cent,
                                                             uint8_t* __restrict__ codes, unsigned long long* __restrict__ part_sums,
                                                             unsigned* __restrict__ part_counts) {
  static_assert(DM % 8 == 0 && (LANES == 1 || (LANES == 4 && TT == 1)), "several tokens per lane, or several lanes per token");
  constexpr int NW = NT / 64, RS = DM + 4;
  constexpr int TS = 64 / LANES;  // tokens side by side in a wave
  // Sixteen waves are all that fit a compute unit beside the sums, so that a wave needs several chains of its own: CC centroids of
  // TT tokens, four differences of each ahead of the additions that wait for them, the next four values of the centroids read
  // from LDS meanwhile.  (Assignment of 64 x 32768 tokens, one chain per wave and each difference right before its addition:
  // 3670 us with 2x256 and 1290 with 1x64; so 2850 and 770.)
  constexpr int CC = DM >= 128 ? 4 : 2;
  // LANES = 1: a lane starts its additions at the dimension of its own number, and rows of DM sums make the bank of a sum depend
  // on its dimension alone (DM a multiple of 32), so that lanes meet in few addresses whatever their centroids are (131072 equal
  // tokens x 8 heads, bf16, 8x16, three rounds: 1900 us with the lanes of a wave in one address, 500 so).
  constexpr bool TURNED = LANES == 1;
  constexpr int SR = TURNED ? DM : DM + 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char round_lds[];
  float* cs = reinterpret_cast<float*>(round_lds);  // [C][RS]
  unsigned long long* sums = reinterpret_cast<unsigned long long*>(round_lds + vector_stage_bytes(s.C, DM));
  unsigned* cnt = reinterpret_cast<unsigned*>(sums + s.C * SR);
  int u, j, p;
  round_place(s, r.ranges, u, j, p);
  const int uj = u * s.M + j, tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6, col = lane % TS, quad = lane / TS;
  const int t_begin = p * r.tokens, t_end = min(s.N, t_begin + r.tokens);
  if (link.sums) {
    linked_means<DM, NT>(s, r, link, uj, p, cent,
                         [&](int i, const f32x4_t& v) { *reinterpret_cast<f32x4_t*>(&cs[(i / DM) * RS + (i % DM)]) = v; });
  } else {
    const f32x4_t* src = reinterpret_cast<const f32x4_t*>(cent + (size_t)uj * s.C * DM);
    for (int i = tid; i < s.C * (DM / 4); i += NT) *reinterpret_cast<f32x4_t*>(&cs[(i / (DM / 4)) * RS + 4 * (i % (DM / 4))]) = src[i];
  }
  if constexpr (ACCUM) {
    for (int i = tid; i < s.C * SR; i += NT) sums[i] = 0ull;
    for (int i = tid; i < s.C; i += NT) cnt[i] = 0u;
  }
  __syncthreads();
  for (int tok0 = t_begin + w * TS * TT; tok0 < t_end; tok0 += NW * TS * TT) {  // wave-uniform
    float x[TT][DM];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const T* kp = keys + ((size_t)u * s.cap + min(tok0 + tt * TS + col, s.N - 1)) * kD + j * DM;
      constexpr int EPV = 16 / (int)sizeof(T);
#pragma unroll
      for (int v = 0; v < DM / EPV; ++v) {
        const uint4 raw = reinterpret_cast<const uint4*>(kp)[v];
        const unsigned rw[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (sizeof(T) == 2) {
            x[tt][v * EPV + 2 * e] = __uint_as_float(rw[e] << 16);
            x[tt][v * EPV + 2 * e + 1] = __uint_as_float(rw[e] & 0xffff0000u);
          } else {
            x[tt][v * EPV + e] = __uint_as_float(rw[e]);
          }
        }
      }
    }
    float best[TT];
    int arg[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      best[tt] = INFINITY;
      arg[tt] = 0;
    }
    f32x4_t cv[2][CC];  // four values of each centroid, and the next four on their way
    auto centroid = [&](int c0, int k) { return min(c0 + k * LANES, s.C - 1); };  // (the last one again: not nearer than itself)
    auto read = [&](f32x4_t (&v)[CC], int c0, int e) {
#pragma unroll
      for (int k = 0; k < CC; ++k) v[k] = *reinterpret_cast<const f32x4_t*>(&cs[centroid(c0, k) * RS + 4 * e]);
    };
    const int c_first = LANES == 1 ? 0 : quad;
    read(cv[0], c_first, 0);
    for (int c0 = c_first; c0 < s.C; c0 += LANES * CC) {
      float d2[CC][TT];
#pragma unroll
      for (int k = 0; k < CC; ++k)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) d2[k][tt] = 0.0f;
#pragma unroll
      for (int e = 0; e < DM / 4; ++e) {
        if (e + 1 < DM / 4)
          read(cv[(e + 1) & 1], c0, e + 1);
        else
          read(cv[0], c0 + LANES * CC, 0);
        __builtin_amdgcn_sched_barrier(0);
        float df[CC][TT][4];
#pragma unroll
        for (int k = 0; k < CC; ++k)
#pragma unroll
          for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int y = 0; y < 4; ++y) df[k][tt][y] = x[tt][4 * e + y] - cv[e & 1][k][y];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
          for (int k = 0; k < CC; ++k)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) d2[k][tt] = fmaf(df[k][tt][y], df[k][tt][y], d2[k][tt]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int k = 0; k < CC; ++k)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          const bool lower = d2[k][tt] < best[tt];
          best[tt] = lower ? d2[k][tt] : best[tt];
          arg[tt] = lower ? centroid(c0, k) : arg[tt];
        }
    }
    if constexpr (LANES == 4) {
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {  // equal values: lower centroid index
        const float ov = __shfl_xor(best[0], o);
        const int oi = __shfl_xor(arg[0], o);
        const bool take = ov < best[0] || (ov == best[0] && oi < arg[0]);
        best[0] = take ? ov : best[0];
        arg[0] = take ? oi : arg[0];
      }
    }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int t = tok0 + tt * TS + col;
      if constexpr (!ACCUM) {
        if (quad == 0 && t < t_end) codes[((size_t)u * s.cap + t) * s.M + j] = (uint8_t)arg[tt];
      } else if constexpr (LANES == 4) {
        if (t < t_end) {
          unsigned long long* row = sums + arg[0] * SR + quad;
          if (quad == 0) atomicAdd(&cnt[arg[0]], 1u);
#pragma unroll
          for (int e = 0; e < DM / 4; ++e) {
            const float v = quad == 0 ? x[0][4 * e] : quad == 1 ? x[0][4 * e + 1] : quad == 2 ? x[0][4 * e + 2] : x[0][4 * e + 3];
            atomicAdd(&row[4 * e], __builtin_expect(!(fabsf(v) < 1073741824.0f), 0) ? fix_biased_large(v) : fix_biased(v));
          }
        }
      } else {
        int turn = lane;
        asm("" : "+v"(turn));  // (else the places of all additions are kept in registers across the loop)
        turn_values(x[tt], turn);
        if (t < t_end) {
          // the members of the first lane's centroid are counted in one go: lanes that meet in one address add one by one
          const int first = __builtin_amdgcn_readfirstlane(arg[tt]);
          const unsigned long long same = __ballot(arg[tt] == first);
          if (arg[tt] != first)
            atomicAdd(&cnt[arg[tt]], 1u);
          else if (lane == 0)
            atomicAdd(&cnt[first], (unsigned)__popcll(same));
          unsigned long long* row = sums + arg[tt] * SR;
#pragma unroll
          for (int e0 = 0; e0 < DM; e0 += 8) {
            float top = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) top = __builtin_elementwise_maximum(fabsf(x[tt][e0 + e]), top);  // NaN stays
            if (__builtin_expect(!(top < 1073741824.0f), 0)) {
#pragma unroll
              for (int e = 0; e < 8; ++e) atomicAdd(&row[(turn + e0 + e) & (DM - 1)], fix_biased_large(x[tt][e0 + e]));
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e) atomicAdd(&row[(turn + e0 + e) & (DM - 1)], fix_biased(x[tt][e0 + e]));
            }
          }
        }
      }
    }
  }
  if constexpr (ACCUM) {
    __syncthreads();
    round_flush<TURNED ? SumRow::kPlain : SumRow::kOdd, DM>(s, r, uj, p, sums, cnt, cent, part_sums, part_counts);
  }
}

// sums[u][j][c][e] += fix(keys[u][t][j*Dm+e]) for every token t with code c; counts[u][j][c] += 1.  For sums that do not fit
// into LDS (64 dimensions and more, many centroids).
// A workgroup first sorts its tokens by code (a counting sort in LDS: one 32-bit atomic per token), then each wave
// takes centroids in turn and sums the centroid's members in registers: a lane loads 16 bytes of a member's
// sub-vector (8 bf16 or 4 fp32 values), a group of Dm*sizeof(T)/16 lanes covers one member and a wave several
// members per load; the lane groups' partial sums meet in a wave-private LDS tile.
// Sums are 64-bit integers of the values in fixed point (2^-20), so the result does not depend on the order of
// the members, of the waves or of the workgroups.
__host__ __device__ constexpr int accum_tokens_per_wg(int C) { return 32 * C < 2048 ? 2048 : (32 * C > 8192 ? 8192 : 32 * C); }
template <typename T, int DM>
__global__ __launch_bounds__(256) void pq_accum_kernel(BuildShape s, const T* __restrict__ keys,
                                                       const uint8_t* __restrict__ codes,
                                                       unsigned long long* __restrict__ sums,
                                                       unsigned* __restrict__ counts) {
  constexpr int EPV = 16 / (int)sizeof(T);  // values per lane
  constexpr int LPT = DM / EPV;             // lanes per member
  constexpr int MPW = 64 / LPT;             // members a wave loads at a time
  constexpr int U = 4;                      // such loads in flight
  constexpr int NW = 4;
  static_assert(DM % EPV == 0 && LPT >= 1 && LPT <= 64, "a sub-vector is a whole number of 16-byte pieces");
  extern __shared__ unsigned short order[];  // [tokens per workgroup] token offsets, sorted by code
  __shared__ unsigned cnt[256];
  __shared__ int start[257];
  __shared__ int scan_sm[2 * NW + 1];
  __shared__ long long part[NW][MPW * DM];   // per wave: [member slot][dimension]
  const int uj = blockIdx.y, u = uj / s.M, j = uj % s.M, tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6, sub = lane % LPT, slot = lane / LPT;
  const int tpw = accum_tokens_per_wg(s.C);
  const int t0 = blockIdx.x * tpw, nt = min(tpw, s.N - t0);
  const uint8_t* cp = codes + ((size_t)u * s.cap + t0) * s.M + j;
  // ---- counting sort of the workgroup's tokens by code
  cnt[tid] = 0u;
  __syncthreads();
  for (int t = tid; t < nt; t += 256) {
    const unsigned c = cp[(size_t)t * s.M];
    if (c < (unsigned)s.C) atomicAdd(&cnt[c], 1u);  // (a code that names no centroid is left out)
  }
  __syncthreads();
  {
    const int mine = (int)cnt[tid];
    int total;
    const int ex = block_exclusive_scan<256>(mine, &total, scan_sm);
    start[tid] = ex;
    if (tid == 255) start[256] = total;
    cnt[tid] = (unsigned)ex;  // now the bucket's fill position
  }
  __syncthreads();
  for (int t = tid; t < nt; t += 256) {
    const unsigned c = cp[(size_t)t * s.M];
    if (c < (unsigned)s.C) order[atomicAdd(&cnt[c], 1u)] = (unsigned short)t;
  }
  __syncthreads();
  // ---- one centroid at a time per wave
  const T* kbase = keys + ((size_t)u * s.cap + t0) * kD + j * DM + sub * EPV;
  long long* mypart = part[w];
  for (int c = w; c < s.C; c += NW) {
    const int base = start[c], n = start[c + 1] - base;  // wave-uniform
    if (n == 0) continue;
    long long acc[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] = 0;
    for (int m0 = 0; m0 < n; m0 += MPW * U) {
      uint4 raw[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int t = order[base + min(m0 + k * MPW + slot, n - 1)];  // clamped: straight-line loads, masked below
        raw[k] = *reinterpret_cast<const uint4*>(kbase + (size_t)t * kD);
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        if (m0 + k * MPW + slot < n) {
          const unsigned rw[4] = {raw[k].x, raw[k].y, raw[k].z, raw[k].w};
          float x[EPV];
          if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              x[2 * e] = __uint_as_float(rw[e] << 16);
              x[2 * e + 1] = __uint_as_float(rw[e] & 0xffff0000u);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(rw[e]);
          }
#pragma unroll
          for (int e = 0; e < EPV; ++e) {
            const float xs = x[e] * (float)(1 << kFixShift);
            // the usual case in 32-bit arithmetic (a 64-bit conversion is a long instruction sequence)
            long long fx = (long long)__float2int_rn(xs);
            if (__builtin_expect(!(fabsf(xs) < 2147483520.0f), 0)) fx = __float2ll_rn(xs);  // |x| >= 2048, or not a number
            acc[e] += fx;
          }
        }
      }
    }
    // the lane groups' sums meet in the wave's tile; then one lane per dimension adds them up
#pragma unroll
    for (int e = 0; e < EPV; ++e) mypart[slot * DM + sub * EPV + e] = acc[e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int used = min(MPW, n);  // slots beyond the members hold zeros; skipping them is only quicker
    for (int d = lane; d < DM; d += 64) {
      long long tot = 0;
      for (int sl = 0; sl < used; ++sl) tot += mypart[sl * DM + d];
      if (tot) atomicAdd(&sums[((size_t)uj * s.C + c) * DM + d], (unsigned long long)tot);
    }
    if (lane == 0) atomicAdd(&counts[(size_t)uj * s.C + c], (unsigned)n);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// cent = sums / counts where counts > 0, else the centroid as it was; the sums are cleared for the next round.  A workgroup's 256
// sums are those of whole centroids (sub-vectors have 16, 32, 64 or 128 dimensions), so that it alone reads the counts that it clears.
__global__ __launch_bounds__(256) void pq_mean_kernel(BuildShape s, unsigned long long* __restrict__ sums, unsigned* __restrict__ counts,
                                                      const float* old /* may be cent */, float* cent) {
  const int n = s.C * s.Dm, i = blockIdx.x * 256 + threadIdx.x, c = i / s.Dm;
  const size_t uj = blockIdx.y;
  const bool live = i < n;
  const unsigned k = live ? counts[uj * s.C + c] : 0u;
  const unsigned long long v = live ? sums[uj * n + i] : 0ull;
  const float o = live ? old[uj * n + i] : 0.0f;
  __syncthreads();
  if (!live) return;
  cent[uj * n + i] = k ? fixed_mean(v, k) : o;
  if (k) {
    sums[uj * n + i] = 0ull;
    if (i % s.Dm == 0) counts[uj * s.C + c] = 0u;
  }
}

// ------------------------------------------------------------ block statistics
// Section 3.4: the block-level cache is refreshed with the k_cache blocks that hold the
// most retrieved tokens.  One workgroup per unit: counts per block, a histogram of the
// count values (a count never exceeds the block size when the listed tokens are distinct),
// the cut c* and the number of blocks to admit at the cut, then the blocks in the order in
// which the cache refresh serves them: fullest first, the lower block number first among
// equal counts.
//
// What bounds it: latency (13175 listed tokens of a unit are 52 KB).  The list is read eight
// entries per thread at a time; lists are mostly ascending, so the entries of a block sit in
// neighbouring lanes and only the first lane of a run of equal blocks adds, the run's length:
// an LDS atomic takes about a clock per lane when the lanes meet in one address.  With
// LDS_COUNTS (up to kLdsBlocks blocks) the counts live in LDS; beyond that they are counted in
// the output array with global atomics and read back through the L2, as was done for every
// size before: 120 us at 131072 tokens in blocks of 128, 13175 listed (8 units), against
// 8.2 us now.
// The blocks above the cut are few (fewer than k_cache): up to kRankBlocks of them are ranked by
// counting larger (count, lower block number) keys; beyond that a block's place is (blocks with
// a larger count) + (blocks before it with the same count), the second term coming from a counter
// per count value that the waves of a chunk of 1024 blocks advance one after the other, lanes
// with equal counts being ranked inside a wave by ballots (quadratic ranking would take longer).
constexpr int kCountBins = 2048;
constexpr int kLdsBlocks = 16384;  // 64 KB of counts beside the 25 KB the selection needs
constexpr int kRankBlocks = 256;   // four keys per step and wave: 64 steps
constexpr int kBlockShift = 40;    // token / block size as a product: exact for tokens < 2^22 and block sizes < 2^11
template <bool LDS_COUNTS>
__global__ __launch_bounds__(1024) void block_stats_kernel(const int* __restrict__ idx, long long n_idx, int N,
                                                           unsigned long long inv_bt /* ceil(2^kBlockShift / block size) */,
                                                           int nb, int k_cache, int* __restrict__ counts,
                                                           int* __restrict__ blocks) {
  constexpr int NT = 1024, NW = NT / 64, U = 8;
  extern __shared__ int lcnt[];  // [nb] with LDS_COUNTS
  __shared__ unsigned hist[kCountBins];
  __shared__ int above[kCountBins];  // blocks with a larger count
  __shared__ int run[kCountBins];    // blocks with this count placed so far
  __shared__ unsigned long long keys[kRankBlocks];  // (count, inverted block number): larger is served first
  __shared__ int scan_sm[2 * NW + 1];
  __shared__ int res[3];
  __shared__ int any_sm;
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int* cu = counts + (size_t)u * nb;
  int* cnt = LDS_COUNTS ? lcnt : cu;
  for (int i = tid; i < nb; i += NT) cnt[i] = 0;
  for (int i = tid; i < kCountBins; i += NT) {
    hist[i] = 0u;
    run[i] = 0;
  }
  if (tid == 0) {
    res[0] = kCountBins;  // cut (no block reaches it when k_cache == 0)
    res[1] = 0;           // blocks above the cut
    res[2] = 0;           // of them collected so far
  }
  if constexpr (!LDS_COUNTS) __threadfence();
  __syncthreads();
  const int* lst = idx + (size_t)u * n_idx;
  for (long long i0 = 0; i0 < n_idx; i0 += (long long)U * NT) {
    int t[U];
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const long long i = i0 + x * NT + tid;
      t[x] = lst[i < n_idx ? i : n_idx - 1];
    }
    PQC_LOADS_ISSUED();
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const bool ok = i0 + x * NT + tid < n_idx && t[x] >= 0 && t[x] < N;
      const int blk = ok ? (int)(((unsigned long long)(unsigned)t[x] * inv_bt) >> kBlockShift) : -1;
      const int prev = dpp_i<0x138>(-2, blk);  // the lane below (wave_shr:1)
      const unsigned long long heads = __ballot(blk != prev);
      if (blk >= 0 && blk != prev) {
        const unsigned long long next = (heads >> lane) >> 1;
        atomicAdd(&cnt[blk], next ? __ffsll((long long)next) : 64 - lane);
      }
    }
  }
  if constexpr (!LDS_COUNTS) __threadfence();
  __syncthreads();
  auto count_of = [&](int i) -> int { return LDS_COUNTS ? lcnt[i] : atomicAdd(&cu[i], 0); };
  for (int i = tid; i < nb; i += NT) {
    const int c = count_of(i);
    if constexpr (LDS_COUNTS) cu[i] = c;
    if (k_cache > 0) atomicAdd(&hist[min(c, kCountBins - 1)], 1u);
  }
  if (k_cache == 0) return;  // uniform
  __syncthreads();
  // thread tid owns count values kCountBins-1-2*tid and kCountBins-2-2*tid (descending)
  const int h0 = (int)hist[kCountBins - 1 - 2 * tid], h1 = (int)hist[kCountBins - 2 - 2 * tid];
  int total;
  int cum = block_exclusive_scan<NT>(h0 + h1, &total, scan_sm);
  above[kCountBins - 1 - 2 * tid] = cum;
  above[kCountBins - 2 - 2 * tid] = cum + h0;
  if (cum < k_cache && cum + h0 >= k_cache) {
    res[0] = kCountBins - 1 - 2 * tid;
    res[1] = cum;
  } else if (cum + h0 < k_cache && cum + h0 + h1 >= k_cache) {
    res[0] = kCountBins - 2 - 2 * tid;
    res[1] = cum + h0;
  }
  __syncthreads();
  const int cut = res[0], n_above = res[1], need = k_cache - n_above;
  const bool ranked = n_above <= kRankBlocks;  // uniform
  int* out = blocks + (size_t)u * k_cache;
  int carry_t = 0;
  for (int i0 = 0; i0 < nb; i0 += NT) {
    const int i = i0 + tid;
    const int c = i < nb ? min(count_of(i), kCountBins - 1) : -1;
    const bool a = c > cut;
    // blocks at the cut: the lowest-numbered `need` of them, behind all blocks above the cut
    if (carry_t < need) {  // uniform
      int tt;
      const int pt = block_exclusive_scan<NT>(c == cut ? 1 : 0, &tt, scan_sm);
      if (c == cut && carry_t + pt < need) out[n_above + carry_t + pt] = i;
      carry_t += tt;
    }
    if (ranked) {
      if (a) keys[atomicAdd(&res[2], 1)] = ((unsigned long long)c << 32) | (0xffffffffu - (unsigned)i);
      continue;
    }
    // blocks above the cut (chunks without any skip the ordered part)
    if (tid == 0) any_sm = 0;
    __syncthreads();
    if (a) any_sm = 1;
    __syncthreads();
    if (any_sm) {  // uniform
      // rank among the wave's lanes with the same count (lanes ascend with the block number), one count value per round
      int rank_w = 0, cnt_w = 0;
      bool leader = false;
      unsigned long long todo = __ballot(a);
      while (todo) {  // wave-uniform
        const int src = __ffsll((long long)todo) - 1;
        const int k0 = __shfl(c, src);
        const unsigned long long m = __ballot(a && c == k0);
        if (a && c == k0) {
          rank_w = __popcll(m & ((1ull << lane) - 1ull));
          cnt_w = __popcll(m);
          leader = lane == src;
        }
        todo &= ~m;
      }
      // the waves advance the per-count counters one after the other (a wave's LDS accesses stay in program order:
      // every lane has read the counter before the leader of its count value moves it on)
      int base = 0;
      for (int ww = 0; ww < NW; ++ww) {
        if (w == ww && a) {
          base = run[c];
          if (leader) run[c] = base + cnt_w;
        }
        __syncthreads();
      }
      if (a) out[above[c] + base + rank_w] = i;
    }
  }
  if (ranked) {
    __syncthreads();
    if (tid < n_above) {
      const unsigned long long mine = keys[tid];
      int rank = 0;
      for (int j0 = 0; j0 < n_above; j0 += 4) {
        unsigned long long o[4];
#pragma unroll
        for (int y = 0; y < 4; ++y) o[y] = keys[min(j0 + y, n_above - 1)];
#pragma unroll
        for (int y = 0; y < 4; ++y) rank += (j0 + y < n_above && o[y] > mine) ? 1 : 0;
      }
      out[rank] = (int)(0xffffffffu - (unsigned)mine);
    }
  }
}

// ------------------------------------------------------------ block cache refresh
// Section 3.4: the block-level cache is looked up with this step's retrieved tokens, then refreshed
// with the step's requested blocks under an LRU or LFU policy.  One workgroup per unit.  Sequentially,
// each absent block would take the lowest empty slot or else the policy's victim among the slots not
// requested in this step; since the order of those slots (empty ones by index, then by (uses,) last
// use, slot) does not change while the step is served, the i-th absent block simply takes the slot of
// rank i in that order, which is found by counting.
constexpr int kCacheSlots = 1024;  // most slots, and most requested blocks, per unit
__global__ __launch_bounds__(256) void block_cache_kernel(int nb, int n_slots, int k_cache, int lfu, int step,
                                                          const int* __restrict__ counts, const int* __restrict__ blocks,
                                                          int* __restrict__ slot_block, int* __restrict__ slot_stamp,
                                                          int* __restrict__ slot_uses, int* __restrict__ stats) {
  constexpr int NT = 256, NW = NT / 64;
  __shared__ int blk[kCacheSlots], stamp[kCacheSlots], uses[kCacheSlots];
  __shared__ int req[kCacheSlots], req_slot[kCacheSlots], miss_rank[kCacheSlots];
  __shared__ int by_rank[kCacheSlots];                 // slot of rank r among the slots not requested in this step
  __shared__ unsigned long long key[kCacheSlots];      // ordering key of a slot; ~0 = requested in this step
  __shared__ int scan_sm[2 * NW + 1];
  __shared__ int red[4];
  const int u = blockIdx.x, tid = threadIdx.x;
  int* sb = slot_block + (size_t)u * n_slots;
  int* ss = slot_stamp + (size_t)u * n_slots;
  int* su = slot_uses + (size_t)u * n_slots;
  const int* cu = counts + (size_t)u * nb;
  if (tid < 4) red[tid] = 0;
  for (int s = tid; s < n_slots; s += NT) {
    blk[s] = sb[s];
    stamp[s] = ss[s];
    uses[s] = su[s];
  }
  for (int i = tid; i < k_cache; i += NT) req[i] = blocks[(size_t)u * k_cache + i];
  __syncthreads();
  // look-up against the cache as it stands: retrieved tokens inside resident blocks
  int ht = 0;
  for (int s = tid; s < n_slots; s += NT)
    if (blk[s] >= 0 && blk[s] < nb) ht += cu[blk[s]];
  if (ht) atomicAdd(&red[0], ht);
  // requested blocks that are resident: mark them used
  int hb = 0;
  for (int i = tid; i < k_cache; i += NT) {
    int found = -1;
    for (int s = 0; s < n_slots; ++s) found = blk[s] == req[i] ? s : found;
    if (req[i] < 0 || req[i] >= nb) found = -2;  // not a block: neither a hit nor a request
    req_slot[i] = found;
    hb += found >= 0;
  }
  if (hb) atomicAdd(&red[1], hb);
  __syncthreads();
  for (int s = tid; s < n_slots; s += NT) {
    const unsigned long long st = (unsigned)stamp[s] ^ 0x80000000u;  // signed order as unsigned order
    const unsigned long long k1 = lfu ? ((unsigned long long)(unsigned)uses[s] << 32) | st : st;
    key[s] = blk[s] < 0 ? 0ull : (1ull << 63) | k1;
  }
  __syncthreads();
  for (int i = tid; i < k_cache; i += NT) {
    const int s = req_slot[i];
    if (s >= 0) {
      key[s] = ~0ull;
      stamp[s] = step;
      atomicAdd(&uses[s], 1);
    }
  }
  __syncthreads();
  // rank of every other slot in victim order
  int n_free_local = 0;
  for (int s = tid; s < n_slots; s += NT) {
    const unsigned long long ks = key[s];
    if (ks == ~0ull) continue;
    int r = 0;
    for (int t = 0; t < n_slots; ++t) {
      const unsigned long long kt = key[t];
      r += (kt != ~0ull) && (kt < ks || (kt == ks && t < s));
    }
    by_rank[r] = s;
    ++n_free_local;
  }
  if (n_free_local) atomicAdd(&red[2], n_free_local);
  // absent requests, numbered in request order
  int carry = 0;
  for (int i0 = 0; i0 < k_cache; i0 += NT) {
    const int i = i0 + tid;
    const int miss = i < k_cache && req_slot[i] == -1;
    int total;
    const int pos = block_exclusive_scan<NT>(miss, &total, scan_sm);
    if (i < k_cache) miss_rank[i] = miss ? carry + pos : -1;
    carry += total;
  }
  __syncthreads();
  const int n_free = red[2], n_ins = min(carry, n_free);
  int evicted = 0;
  for (int i = tid; i < k_cache; i += NT) {
    const int r = miss_rank[i];
    if (r >= 0 && r < n_ins) {
      const int s = by_rank[r];
      evicted += blk[s] >= 0;
      blk[s] = req[i];
      stamp[s] = step;
      uses[s] = 1;
    }
  }
  if (evicted) atomicAdd(&red[3], evicted);
  __syncthreads();
  for (int s = tid; s < n_slots; s += NT) {
    sb[s] = blk[s];
    ss[s] = stamp[s];
    su[s] = uses[s];
  }
  if (tid == 0) {
    int* o = stats + (size_t)u * 4;
    o[0] = red[0];
    o[1] = red[1];
    o[2] = n_ins;
    o[3] = red[3];
  }
}

// -------------------------------------------------------------- code-pair counts
// M = 2: how many tokens of a unit carry each pair of codes (c0 + C*c1), over all N tokens.
// A statistic of the codes alone; pqc_decode_indexed takes its threshold from it.
constexpr int kPairTok = 8192;  // tokens per workgroup
__global__ __launch_bounds__(256) void pair_count_kernel(const uint8_t* __restrict__ codes, int N, int cap, int C,
                                                         unsigned* __restrict__ counts) {
  __shared__ unsigned h[4096];
  const int u = blockIdx.y, tid = threadIdx.x, np = C * C;
  for (int i = tid; i < np; i += 256) h[i] = 0u;
  __syncthreads();
  const unsigned short* cu = reinterpret_cast<const unsigned short*>(codes) + (size_t)u * cap;
  const int t1 = min(N, ((int)blockIdx.x + 1) * kPairTok);
  for (int t = blockIdx.x * kPairTok + tid; t < t1; t += 256) {
    const unsigned cw = cu[t];
    const int c0 = (int)(cw & 0xffu), c1 = (int)(cw >> 8);
    if (c0 < C && c1 < C) atomicAdd(&h[c0 + C * c1], 1u);  // a code outside [0, C) names no pair: not counted
  }
  __syncthreads();
  for (int i = tid; i < np; i += 256)
    if (h[i]) atomicAdd(&counts[(size_t)u * np + i], h[i]);
}

// one appended token per unit: its pair gains a token
__global__ void pair_count_add_kernel(const uint8_t* __restrict__ codes, int cap, int C, int units, int position,
                                      unsigned* __restrict__ counts) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= units) return;
  const uint8_t* cp = codes + ((size_t)u * cap + position) * 2;
  const int c0 = (int)cp[0], c1 = (int)cp[1];
  if (c0 < C && c1 < C) counts[(size_t)u * C * C + c0 + C * c1] += 1u;
}

}  // namespace pqc
