// Host side of libpqcache: the C ABI of include/pqcache.h, configuration checks,
// workspace carving and kernel dispatch.  No device memory is allocated here and
// nothing synchronises the host: every entry point only enqueues kernels.
#include "../../include/pqcache.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

#include "pqc_build_kernels.h"
#include "pqc_kernels.h"

namespace pqc {

__global__ void reset_kernel(unsigned* a, size_t na) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < na) a[i] = 0u;
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

}  // namespace pqc

namespace {

using namespace pqc;

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Plan {
  Shape s;
  bool short_form;  // the decode step's threshold is found by the select kernel itself (From::kCount, kShort), no histogram kernel
  size_t off_lut, off_range, off_hist, off_bins, off_crec, off_stage, off_cnt, off_part, off_trace, total;
  int rec_stride;
};

// Launch-shape overrides from the environment, for sweeps: debug builds (-DPQC_TRACE) only.  The shipped library
// reads no environment variable.
int env_int(const char* name, int fallback) {
#ifdef PQC_TRACE
  const char* v = std::getenv(name);
  if (!v || !*v) return fallback;
  const int x = std::atoi(v);
  return x > 0 ? x : fallback;
#else
  (void)name;
  return fallback;
#endif
}

// Offsets of the workspace regions for the given per-unit sizes.
void lay_out(Plan* p, size_t bins_per_unit, size_t stage_words_per_unit, size_t counts_per_unit, size_t partials_per_unit) {
  const Shape& s = p->s;
  const size_t units = (size_t)s.B * s.Hkv;
  size_t off = 0;
  p->off_lut = off;   off = align_up(off + sizeof(float) * units * s.M * s.C);
  p->off_range = off; off = align_up(off + sizeof(float2) * units);
  p->off_hist = off;  off = align_up(off + sizeof(unsigned) * units * (kHistCopies * kNB + 1));  // + record counters
#ifdef PQC_TRACE  // in front of what depends on the length, so that it lies in one place for every plan of a context
  p->off_trace = off; off = align_up(off + sizeof(unsigned long long) * 3 * kTraceWgs * kTraceSlots);
#endif
  p->off_bins = off;  off = align_up(off + sizeof(unsigned short) * units * bins_per_unit);
  p->off_crec = off;  off = align_up(off + (size_t)p->rec_stride * units);
  p->off_stage = off; off = align_up(off + sizeof(unsigned long long) * units * stage_words_per_unit);
  p->off_cnt = off;   off = align_up(off + sizeof(int2) * units * counts_per_unit);
  p->off_part = off;  off = align_up(off + sizeof(float) * units * partials_per_unit * s.G * (kD + 2));
  p->total = off;
}

// Whether a step of this shape is quicker without the histogram kernel (From::kCount, kShort in pqc_kernels.h): a launch, the table's
// second build and the stored bins saved, against work over all N tokens in every workgroup.  Measured on layers of their own K/V,
// centroids and codes in turn (4 to 32 of them, over 1.5 GB), us per layer with and without the histogram kernel, bf16, 4 query heads
// per unit, a tenth retrieved:
//   kCount tokens 2048         8192         16384        24576        32768        49152        57344        65536      (2x64)
//   1 unit        18.3, 15.4   18.5, 15.5   18.9, 16.3   19.1, 17.0   19.5, 17.9   21.0, 20.8   21.2, 21.4   21.8, 22.5
//   8 units       19.5, 15.7   20.1, 16.4   20.7, 17.7   22.0, 19.3   22.9, 21.0   25.4, 24.2   26.4, 25.9   27.0, 27.1
//   32 units                   22.8, 18.7   25.8, 22.4   29.7, 25.9   30.2, 28.2   40.8, 37.7                46.3, 43.8
//   64 units                   25.8, 21.3   30.7, 27.6   40.3, 35.8   45.2, 41.3
// A fifth retrieved, 1 unit of 49152 21.7, 21.6, 8 units of 53248 31.7, 31.4, of 57344 31.7, 31.9; one query head and a twentieth, 1 unit
// of 49152 19.4, 19.3; 16 units of 57344 31.3, 30.2, of 65536 32.1, 32.2.
//   kShort tokens 8192         12288        16384
//   1 unit        19.1, 17.3   19.2, 18.7   19.3, 19.7   (4x64)
//   8 units       20.3, 18.0   20.5, 19.7   20.9, 20.9
//   1 unit        20.7, 19.7   20.8, 21.0   21.1, 22.0   (4x256)
//   8 units       22.1, 20.5   22.8, 22.5   23.0, 23.6
// 7 units of 12288 (4x64), one query head, a twentieth 18.3, 18.5.  Beyond one workgroup per compute unit those of a unit go over it one
// after the other: 128 units of 24000 (2x64) 66.9, 71.5.  With as many workgroups as compute units and much to attend, two smaller ones
// per unit hide each other's latency: a fifth retrieved, 240 units of 8192 77.1, 79.9, 128 of 12288 64.3, 65.0, but of 16384 71.2, 69.9,
// 64 of 32768 66.3, 63.9; a tenth retrieved, 240 of 8192 53.7, 51.0, 128 of 12288 43.9, 40.3.
bool short_cache(const Shape& s) {
  if (s.M != 2 && s.M != 4) return false;
  const long long units = (long long)s.B * s.Hkv, blocks = units * ((s.N + 8191) / 8192);
  if (s.N > 8192 && blocks > 256) return false;
  const bool roomy = s.N < 8192 || blocks < 208 || 6ll * s.K < s.N;
  if (counts_pairs(s)) return s.N <= (units < 8 ? 49152 : units < 16 ? 53248 : units < 32 ? 57344 : 65536) && (roomy || s.N >= 16384);
  return (long long)s.N * s.M <= (s.C > 64 ? 32768 : units < 8 ? 45056 : 49152) && roomy;
}

// Tokens per workgroup of the select kernel: twice as many until `resident` workgroups per compute unit hold all of them, or a unit is one
// workgroup's.  (Without the second condition more than `resident` * 256 units always took the largest, of which one wave then held every token
// of a short unit: 264 units of 2048 tokens, 2x64, 4 query heads, a tenth retrieved, us per layer, given pair counts 54.3, now 45.7, without
// 48.3, now 45.4.)
int select_tokens(const Shape& s, int resident, int most) {
  const long long units = (long long)s.B * s.Hkv;
  int tok = 512;
  while (tok < most && tok < s.N && units * ((s.N + tok - 1) / tok) > 256ll * resident) tok *= 2;
  return tok;
}

// The select kernel of a step with given pair counts.  One workgroup of 512 threads per compute unit and up to 16384 tokens is the
// quickest while a unit's tokens divide well among the compute units; where they don't (more units than compute units, or a round of
// workgroups that is nearly empty), two smaller workgroups per compute unit are: of 256 threads (From::kPairsMany), or of 512 where their
// registers leave room for two (fp32, up to two query heads).  Compared by the tokens that the busiest compute unit goes through and what its
// workgroups pay for their start, in tokens: 2400 for one, 1600 for each of two.  us per layer, 2x64, a tenth retrieved, bf16, one and two:
//   8 units of 4096 tokens, 4 query heads 16.1, 17.4; 64 of 16384, one 24.6, 26.5; 100 of 9000, one 30.0, 26.1; 100 of 28000, one 46.7, 49.4;
//   130 of 20000, two 83.1, 51.6; 256 of 17000, two 94.1, 88.0; 264 of 2048, four 45.7, 38.8; 1024 of 2048, two 99.5, 81.8.
// fp32, one workgroup of 512 threads, two of them, and two of 256: 100 of 20000, one query head 62.2, 53.4, 55.6; 130 of 28000, two 125.7, 104.9,
// 122.3; 400 of 9000, two 112.7, 123.3, 132.1; two of 512 and two of 256, 600 of 2048, two query heads 68.9, 75.7.
struct PairsForm {
  From from;
  int tokens;
};
PairsForm pairs_form(const Shape& s, bool f32) {
  const long long units = (long long)s.B * s.Hkv;
  auto rounds = [&](int tok) { return (units * ((s.N + tok - 1) / tok) + 255) / 256; };
  const int one = select_tokens(s, 1, max_tokens_per_select(From::kPairs)), two = select_tokens(s, 2, max_tokens_per_select(From::kPairsMany));
  const long long cost_one = rounds(one) * (std::min(one, s.N) + 2400);
  const long long cost_two = rounds(two) * std::min(two, s.N) + std::max(rounds(two), 2ll) * 1600;
  if (cost_one <= cost_two) return {From::kPairs, one};
  return {f32 && s.G <= 2 ? From::kPairs : From::kPairsMany, two};
}

// Tokens that share all their codes share a score: with few distinct code words the tie class at the threshold is large (131072 tokens
// over 64 x 64 code pairs: up to 70 candidates), and the finalize kernel requests more records up front.
bool large_tie_classes(const Shape& s, double tokens_per_word = 16.0) {
  double words = 1.0;
  for (int j = 0; j < s.M; ++j) words *= s.C;
  return s.N >= tokens_per_word * words;
}

// Workgroups per unit of the finalize kernel that copy the lists, beside `heads` others: fewer where there are many units (64 of 20000,
// 4x256: four 47.7, two 46.7; 12 of 20011 fp32: two 24.2, four 23.6, six 23.1), and where fewer keep the grid within one workgroup per compute
// unit (20011 tokens, 4x64, a tenth retrieved: 12 units of 4 heads six 22.7, four 22.3, 24 units of 8 heads four 26.6, two 25.7; a grid that is
// beyond it either way takes four, 32 units of 8 heads, 4x256, 131072 tokens: two 76.7, four 75.7; and with large tie classes there is more to copy,
// 2x64, 131072 tokens, a fifth retrieved: 8 units of 8 heads two 45.6, four 41.8).
int copy_workgroups(long long units, int heads, bool large_ties) {
  const int n = units > 32 ? 2 : units > 16 || units < 4 ? 4 : 6;
  auto fits = [&](int m) { return units * (heads + m) <= 256; };
  if (n == 2 || fits(n)) return n;
  return !fits(4) && fits(2) && !large_ties ? 2 : 4;
}

// What a launch plan is for: the decode step, the step with given pair counts, or any other call.
enum class For { kOther, kDecode, kPairs };
int make_plan(const pqc_config* c, Plan* p, For call = For::kOther) {
  if (!c) return PQC_EINVAL;
  if (c->batch < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->head_dim < 1 || c->n_tokens < 1 || c->pq_m < 1 ||
      c->pq_centroids < 1 || c->topk < 0 || c->n_init < 0 || c->n_local < 0)
    return PQC_EINVAL;
  if (c->n_q_heads % c->n_kv_heads || c->head_dim % c->pq_m) return PQC_EINVAL;
  if ((long long)c->n_init + c->topk + c->n_local > c->n_tokens || c->n_init + c->topk + c->n_local < 1) return PQC_EINVAL;
  if (c->kv_dtype != PQC_F32 && c->kv_dtype != PQC_BF16) return PQC_EINVAL;
  if (!(c->softmax_scale == c->softmax_scale) || std::isinf(c->softmax_scale)) return PQC_EINVAL;
  const int G = c->n_q_heads / c->n_kv_heads;
  if (c->head_dim != kD) return PQC_EUNSUPPORTED;
  if (c->pq_m != 1 && c->pq_m != 2 && c->pq_m != 4 && c->pq_m != 8) return PQC_EUNSUPPORTED;
  if (c->pq_centroids > 256) return PQC_EUNSUPPORTED;
  if (G != 1 && G != 2 && G != 4 && G != 8) return PQC_EUNSUPPORTED;
  if (c->n_capacity < 0 || (c->n_capacity && c->n_capacity < c->n_tokens)) return PQC_EINVAL;
  if (c->n_tokens > (1 << 22) || c->n_capacity > (1 << 22)) return PQC_EUNSUPPORTED;
  if ((long long)c->batch * c->n_kv_heads > 65535) return PQC_EUNSUPPORTED;

  Shape& s = p->s;
  s.B = c->batch; s.Hq = c->n_q_heads; s.Hkv = c->n_kv_heads; s.G = G; s.N = c->n_tokens;
  s.cap = c->n_capacity ? c->n_capacity : c->n_tokens;
  s.M = c->pq_m; s.C = c->pq_centroids; s.Dm = c->head_dim / c->pq_m;
  s.K = c->topk; s.I = c->n_init; s.L = c->n_local; s.Ktot = s.I + s.K + s.L;
  const float scale = c->softmax_scale > 0.0f ? c->softmax_scale : 1.0f / std::sqrt((float)c->head_dim);
  s.scale_log2e = scale * 1.4426950408889634f;
  const long long units = (long long)s.B * s.Hkv;

  // A unit's codes start at byte u*cap*M; when that is not always 16-byte aligned the first
  // chunk of a unit begins with up to 15 phantom tokens that the grids must cover as well.
  const int lead = ((long long)s.cap * s.M) % 16 == 0 ? 0 : 15;
  // histogram kernel: about one 1024-thread workgroup per compute unit over all units
  const int maxA = 4096 * (16 / s.M) < 16384 ? 4096 * (16 / s.M) : 16384;  // kMaxVecA chunks per thread
  int tokA = env_int("PQC_TOK_A", 0);
  if (!tokA) {
    // every workgroup builds the unit's whole table first, so few, large workgroups: 4096 tokens measured best
    // from 32K to 128K tokens per unit (at 32K: 27.6 us per step against 28.3 with 1024)
    tokA = 4096;
    while (tokA < maxA && units * ((s.N + lead + tokA - 1) / tokA) > 320) tokA *= 2;
  }
  if (tokA % 1024 || tokA > maxA) return PQC_EINVAL;
  s.tokA = tokA; s.nblkA = (s.N + lead + tokA - 1) / tokA;
  s.histCopies = s.nblkA <= 32 ? 1 : s.nblkA <= 64 ? 2 : kHistCopies;
  // select kernel: two workgroups of 256 threads per compute unit, or one of 512 where there is no histogram kernel
  p->short_form = call == For::kDecode && short_cache(s);
  const PairsForm pairs = call == For::kPairs ? pairs_form(s, c->kv_dtype == PQC_F32) : PairsForm{From::kBins, 0};
  const From form = p->short_form ? From::kShort : pairs.from;
  s.pairsMany = form == From::kPairsMany;
  int tokC = env_int("PQC_TOK_C", 0);
  if (!tokC) tokC = call == For::kPairs ? pairs.tokens : select_tokens(s, p->short_form ? 1 : 2, max_tokens_per_select(form));
  if (tokC < 512 || tokC > max_tokens_per_select(form) || (tokC & (tokC - 1))) return PQC_EINVAL;
  s.tokC = tokC; s.nblkC = (s.N + tokC - 1) / tokC;
  s.binStride = s.nblkC * s.tokC;
  s.stageStride = s.tokC + 40;
  s.rowsP = env_int("PQC_ROWS_P", 256);
  s.nblkP = (s.Ktot + s.rowsP - 1) / s.rowsP;
  s.npart = s.nblkC > s.nblkP ? s.nblkC : s.nblkP;
  p->rec_stride = (int)cand_unit_bytes(G, c->kv_dtype == PQC_F32 ? 4 : 2);
  // finalize kernel: as many workgroups per query head (each with its share of the output dimensions) as keep the
  // grid within about one workgroup per compute unit (16 units of 8 heads, 4096 tokens, us per layer: two per head, 320 workgroups, 17.8, one
  // 17.1), or two with large tie classes, whose many admitted rows are spread over them (one partition of 256 centroids, 40000 tokens: 24 units of 4
  // heads 47.3, two 39.4, 14 of 8 heads 45.7, 39.0; 2x64, 131072 tokens: 24 units of 4 heads 60.7, 58.7).  With given pair counts only one pair's
  // tokens are candidates, not those of all pairs in a bin (24 units of 4 heads: 2x16, 20000 tokens 29.7, 27.4, fp32; 8 units of 8 heads, 2x64, 72000
  // tokens 51.0, 52.9).
  const bool ties = large_tie_classes(s, call == For::kPairs ? 64.0 : 16.0);
  s.slices = 1;
  while (s.slices < kMaxSlices && units * (2 * s.slices * G + 4) <= (ties ? 512 : 256)) s.slices *= 2;
  s.copyWgs = copy_workgroups(units, s.slices * G, ties);
  // sample ranks that bracket the K-th largest score by 5 standard errors (+2)
  const int nmid = s.N - s.I - s.L;
  s.sampleN = nmid < 1024 ? (nmid > 0 ? nmid : 1) : 1024;
  {
    const double pr = nmid > 0 ? (double)s.K / (double)nmid : 0.0;
    const double centre = pr * s.sampleN, hw = 5.0 * std::sqrt(s.sampleN * pr * (1.0 - pr)) + 2.0;
    s.rankHi = (int)std::floor(centre - hw);                       // < 1: the window reaches the upper bound
    s.rankLo = (int)std::ceil(centre + hw);
    if (s.rankLo > s.sampleN) s.rankLo = 0;                        // 0: the window reaches the lower bound
    if (s.rankHi < 1) s.rankHi = 0;
  }

  lay_out(p, (size_t)s.binStride, (size_t)s.nblkC * s.stageStride, (size_t)s.nblkC, (size_t)s.npart);
  return PQC_OK;
}

// Whether the step with given pair counts takes this configuration.
bool pairs_supported(const pqc_config* c) {
  return c->pq_m == 2 && c->pq_centroids <= kPairC && (c->n_capacity ? c->n_capacity : c->n_tokens) % 8 == 0;
}

// Workspace needed by any context of this configuration whose length is changed later
// (pqc_set_length) to anything up to the capacity: every size that depends on the length,
// replaced by a bound over all lengths.
size_t workspace_bound(const pqc_config* c) {
  Plan p;
  if (make_plan(c, &p) != PQC_OK) return 0;
  const Shape& s = p.s;
  if (s.cap == s.N) {
    size_t most = p.total;
    for (For call : {For::kDecode, For::kPairs}) {
      Plan d;
      if (call == For::kPairs && !pairs_supported(c)) continue;
      make_plan(c, &d, call);
      most = std::max(most, d.total);
    }
    return most;
  }
  const size_t units = (size_t)s.B * s.Hkv, cap = (size_t)s.cap;
  // select kernel grid: tokens per workgroup double until the grid has at most 512 workgroups or
  // they reach 8192, or 16384 with given pair counts (an override by environment may pin them as low as 512)
  const size_t tok_min = env_int("PQC_TOK_C", 0) ? (size_t)env_int("PQC_TOK_C", 0) : 8192;
  size_t nb = 512 / units;
  if (nb < (cap + tok_min - 1) / tok_min) nb = (cap + tok_min - 1) / tok_min;
  if (nb < 1) nb = 1;
  size_t npart = (cap + s.rowsP - 1) / s.rowsP;
  if (npart < nb) npart = nb;
  const size_t last = max_tokens_per_select(pairs_supported(c) ? From::kPairs : From::kBins);  // what the last workgroup may hold beyond the length
  lay_out(&p, cap + last, cap + last + 40 * nb, nb, npart);
  return p.total;
}

}  // namespace

struct pqc_ctx {
  pqc_config cfg;
  Plan plan;           // of every call but the decode step
  Plan decode_plan;    // of the decode step: `plan`, or its short form
  Plan pairs_plan;     // of the step with given pair counts
  Workspace ws;        // views of `plan`
  Workspace decode_ws; // views of `decode_plan`; histograms and record counters lie in the same place in all three
  Workspace pairs_ws;  // views of `pairs_plan`
  AppendArgs append;       // set for the duration of a pqc_decode_append call
  char* workspace;         // the caller's device memory
  size_t workspace_bytes;
  bool hist_clean;  // the histogram is known to be all zero
  int next_phase;   // pqc_decode_phase: the phase that continues the step begun on this context (0: none begun)
  int last_hip;
};

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_launch(pqc_ctx* ctx) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    ctx->last_hip = (int)e;
    ctx->hist_clean = false;
    return PQC_EHIP;
  }
  return PQC_OK;
}

// Histograms and record counters must be zero when a call starts; finalize_kernel leaves them
// so, which makes a completed call stateless (and a captured one replayable).
int ensure_clean_hist(pqc_ctx* ctx, hipStream_t st) {
  if (ctx->next_phase != 0) {  // a step begun phase by phase (pqc_decode_phase) was left unfinished: its histogram is stale
    ctx->hist_clean = false;
    ctx->next_phase = 0;
  }
  if (ctx->hist_clean) return PQC_OK;
  const Shape& s = ctx->plan.s;
  const size_t na = (size_t)s.B * s.Hkv * (kHistCopies * kNB + 1);  // histograms and the record counters behind them
  hipLaunchKernelGGL(reset_kernel, dim3((unsigned)((na + 255) / 256)), dim3(256), 0, st, ctx->ws.hist, na);
  return check_launch(ctx);
}

// ---- template dispatch -------------------------------------------------------
// The histogram kernel is compiled for the number of 16-byte loads a thread needs: of the centroids (VW: the
// unit's M*C*Dm floats over 1024 threads) and of the codes or scores (VA: the workgroup's tokA tokens).
template <typename T, class SRC, int VW>
void launch_hist_w(const Shape& s, const Workspace& ws, const T* q, const float* cent, const void* src, size_t lds, hipStream_t st) {
  const dim3 grid(s.nblkA, (unsigned)(s.B * s.Hkv));
  const int chunks = s.tokA / SRC::P, va = (chunks + 1023) / 1024;
  if (va <= 1)
    hipLaunchKernelGGL((hist_kernel<T, SRC, VW, 1>), grid, dim3(1024), lds, st, s, ws, q, cent, src);
  else if (va <= 2)
    hipLaunchKernelGGL((hist_kernel<T, SRC, VW, 2>), grid, dim3(1024), lds, st, s, ws, q, cent, src);
  else
    hipLaunchKernelGGL((hist_kernel<T, SRC, VW, 4>), grid, dim3(1024), lds, st, s, ws, q, cent, src);
}
template <typename T, class SRC>
void launch_hist(const Shape& s, const Workspace& ws, const T* q, const float* cent, const void* src, size_t lds, hipStream_t st) {
  if constexpr (!SRC::kFromCodes) {
    launch_hist_w<T, SRC, 1>(s, ws, q, cent, src, lds, st);
  } else {
    const int vw = (s.M * s.C * s.Dm + 4095) / 4096;
    if (vw <= 1) launch_hist_w<T, SRC, 1>(s, ws, q, cent, src, lds, st);
    else if (vw <= 2) launch_hist_w<T, SRC, 2>(s, ws, q, cent, src, lds, st);
    else if (vw <= 4) launch_hist_w<T, SRC, 4>(s, ws, q, cent, src, lds, st);
    else launch_hist_w<T, SRC, 8>(s, ws, q, cent, src, lds, st);
  }
}

template <typename T, int G>
void launch_finalize(pqc_ctx* ctx, const Shape& s, const Workspace& ws, const T* qt, const T* kt, const T* vt, int32_t* out_idx,
                     float* out_attn, hipStream_t st) {
  const dim3 grid(G * s.slices + s.copyWgs + (ctx->append.key ? 1 : 0), (unsigned)(s.B * s.Hkv));
  if (s.slices == kMaxSlices && large_tie_classes(s))
    hipLaunchKernelGGL((finalize_kernel<T, G, true, true>), grid, dim3(kFinalThreads), finalize_lds_bytes(s, true), st, s, ws, qt, kt, vt,
                       out_idx, out_attn, ctx->append);
  else
    hipLaunchKernelGGL((finalize_kernel<T, G, true, false>), grid, dim3(kFinalThreads), finalize_lds_bytes(s, true), st, s, ws, qt, kt, vt,
                       out_idx, out_attn, ctx->append);
}

// phases: bit k set = launch kernel k of the decode path (0 histogram, 1 select + attention, 2 finalize); the short form has no
// kernel 0
template <typename T, int G, int M>
void launch_decode_tgm(pqc_ctx* ctx, const void* q, const float* cent, const uint8_t* codes, const void* k,
                       const void* v, int32_t* out_idx, float* out_attn, hipStream_t st, unsigned phases) {
  const Shape& s = ctx->decode_plan.s;
  const Workspace& ws = ctx->decode_ws;
  const unsigned units = (unsigned)(s.B * s.Hkv);
  const T* qt = static_cast<const T*>(q);
  const T* kt = static_cast<const T*>(k);
  const T* vt = static_cast<const T*>(v);
  if (ctx->decode_plan.short_form) {
    if (phases & 2u) launch_short_select(sizeof(T) == 2, s, ws, q, cent, codes, k, v, st);
  } else {
    if (phases & 1u) launch_hist<T, CodeChunks<M>>(s, ws, qt, cent, static_cast<const void*>(codes), sizeof(float) * lut_tile_floats(1024, M, s.C), st);
    if (phases & 2u)
      hipLaunchKernelGGL((select_kernel<T, G, CodeChunks<M>, true>), dim3(s.nblkC, units), dim3(256), list_bytes<From::kBins>(s.tokC), st, s, ws, qt, kt, vt, static_cast<const void*>(codes));
  }
  if (phases & 4u)
    launch_finalize<T, G>(ctx, s, ws, qt, kt, vt, out_idx, out_attn, st);
}

template <typename T, int G>
void launch_decode_tg(pqc_ctx* ctx, const void* q, const float* cent, const uint8_t* codes, const void* k, const void* v,
                      int32_t* out_idx, float* out_attn, hipStream_t st, unsigned phases) {
  switch (ctx->plan.s.M) {
    case 1: launch_decode_tgm<T, G, 1>(ctx, q, cent, codes, k, v, out_idx, out_attn, st, phases); break;
    case 2: launch_decode_tgm<T, G, 2>(ctx, q, cent, codes, k, v, out_idx, out_attn, st, phases); break;
    case 4: launch_decode_tgm<T, G, 4>(ctx, q, cent, codes, k, v, out_idx, out_attn, st, phases); break;
    default: launch_decode_tgm<T, G, 8>(ctx, q, cent, codes, k, v, out_idx, out_attn, st, phases); break;
  }
}

template <typename T>
void launch_decode_t(pqc_ctx* ctx, const void* q, const float* cent, const uint8_t* codes, const void* k, const void* v,
                     int32_t* out_idx, float* out_attn, hipStream_t st, unsigned phases) {
  switch (ctx->plan.s.G) {
    case 1: launch_decode_tg<T, 1>(ctx, q, cent, codes, k, v, out_idx, out_attn, st, phases); break;
    case 2: launch_decode_tg<T, 2>(ctx, q, cent, codes, k, v, out_idx, out_attn, st, phases); break;
    case 4: launch_decode_tg<T, 4>(ctx, q, cent, codes, k, v, out_idx, out_attn, st, phases); break;
    default: launch_decode_tg<T, 8>(ctx, q, cent, codes, k, v, out_idx, out_attn, st, phases); break;
  }
}

// decode with the threshold taken from code-pair counts (M = 2): select + finalize, no histogram kernel
template <typename T>
void launch_indexed_t(pqc_ctx* ctx, const void* q, const float* cent, const uint8_t* codes, const unsigned* pair_counts,
                      const void* k, const void* v, int32_t* out_idx, float* out_attn, hipStream_t st) {
  const Shape& s = ctx->pairs_plan.s;
  const Workspace& ws = ctx->pairs_ws;
  const T* qt = static_cast<const T*>(q);
  const T* kt = static_cast<const T*>(k);
  const T* vt = static_cast<const T*>(v);
  launch_pairs_select(sizeof(T) == 2, s, ws, q, cent, codes, pair_counts, ctx->append.key ? ctx->append.position : -1, k, v, st);
  switch (s.G) {
    case 1: launch_finalize<T, 1>(ctx, s, ws, qt, kt, vt, out_idx, out_attn, st); break;
    case 2: launch_finalize<T, 2>(ctx, s, ws, qt, kt, vt, out_idx, out_attn, st); break;
    case 4: launch_finalize<T, 4>(ctx, s, ws, qt, kt, vt, out_idx, out_attn, st); break;
    default: launch_finalize<T, 8>(ctx, s, ws, qt, kt, vt, out_idx, out_attn, st); break;
  }
}

template <typename T, int G>
void launch_attn_tg(pqc_ctx* ctx, const void* q, const void* k, const void* v, const int32_t* idx, float* out,
                    hipStream_t st) {
  const Shape& s = ctx->plan.s;
  const unsigned units = (unsigned)(s.B * s.Hkv);
  hipLaunchKernelGGL((attn_list_kernel<T, G>), dim3(s.nblkP, units), dim3(256), sizeof(int) * s.rowsP, st, s, ctx->ws,
                     static_cast<const T*>(q), static_cast<const T*>(k), static_cast<const T*>(v), idx);
  hipLaunchKernelGGL((merge_kernel<G>), dim3(G, units), dim3(256), sizeof(float) * s.nblkP, st, s, ctx->ws, s.nblkP, out);
}

template <typename T>
void launch_attn_t(pqc_ctx* ctx, const void* q, const void* k, const void* v, const int32_t* idx, float* out,
                   hipStream_t st) {
  switch (ctx->plan.s.G) {
    case 1: launch_attn_tg<T, 1>(ctx, q, k, v, idx, out, st); break;
    case 2: launch_attn_tg<T, 2>(ctx, q, k, v, idx, out, st); break;
    case 4: launch_attn_tg<T, 4>(ctx, q, k, v, idx, out, st); break;
    default: launch_attn_tg<T, 8>(ctx, q, k, v, idx, out, st); break;
  }
}

template <typename T>
void launch_lut_t(const Shape& s, const T* q, const float* cent, float* table, hipStream_t st) {
  const dim3 grid(1, (unsigned)(s.B * s.Hkv));
  switch (s.M) {
    case 1: hipLaunchKernelGGL((lut_kernel<T, 1>), grid, dim3(256), 0, st, s, q, cent, table); break;
    case 2: hipLaunchKernelGGL((lut_kernel<T, 2>), grid, dim3(256), 0, st, s, q, cent, table); break;
    case 4: hipLaunchKernelGGL((lut_kernel<T, 4>), grid, dim3(256), 0, st, s, q, cent, table); break;
    default: hipLaunchKernelGGL((lut_kernel<T, 8>), grid, dim3(256), 0, st, s, q, cent, table); break;
  }
}

template <int M>
void launch_scan_m(pqc_ctx* ctx, const float* table, const uint8_t* codes, float* scores, hipStream_t st) {
  const Shape& s = ctx->plan.s;
  hipLaunchKernelGGL((scan_kernel<M>), dim3((s.N + 2047) / 2048, (unsigned)(s.B * s.Hkv)), dim3(256), 0, st, s, table,
                     codes, scores);
}

}  // namespace

extern "C" {

int pqc_version(void) { return 200; }

const char* pqc_strerror(int status) {
  switch (status) {
    case PQC_OK: return "ok";
    case PQC_EINVAL: return "invalid argument or configuration";
    case PQC_EUNSUPPORTED: return "configuration outside the supported shapes";
    case PQC_EWORKSPACE: return "workspace missing, misaligned or too small";
    case PQC_EHIP: return "HIP call failed";
    case PQC_ESCRATCH: return "shape needs more than the static scratch of pqc_decode_static (use pqc_decode with a workspace)";
    default: return "unknown status";
  }
}

#ifdef PQC_TRACE
size_t pqc_debug_trace_offset(const pqc_config* cfg) {
  Plan p;
  if (make_plan(cfg, &p) != PQC_OK) return 0;
  return p.off_trace;
}
#endif

size_t pqc_workspace_bytes(const pqc_config* cfg) { return workspace_bound(cfg); }

namespace {
// Views of the regions of a plan.
Workspace views(char* base, const Plan& p) {
  Workspace ws;
  ws.lut = reinterpret_cast<float*>(base + p.off_lut);
  ws.hist = reinterpret_cast<unsigned*>(base + p.off_hist);
  ws.cand_count = ws.hist + (size_t)p.s.B * p.s.Hkv * kHistCopies * kNB;
  ws.range = reinterpret_cast<float2*>(base + p.off_range);
  ws.bins = reinterpret_cast<unsigned short*>(base + p.off_bins);
  ws.cand_rec = reinterpret_cast<unsigned char*>(base + p.off_crec);
  ws.rec_stride = p.rec_stride;
  ws.stage = reinterpret_cast<unsigned long long*>(base + p.off_stage);
  ws.stage_cnt = reinterpret_cast<int2*>(base + p.off_cnt);
  ws.partials = reinterpret_cast<float*>(base + p.off_part);
#ifdef PQC_TRACE
  ws.trace = reinterpret_cast<unsigned long long*>(base + p.off_trace);
#endif
  return ws;
}

// The context's plans of its configuration (`p`: the general one), and their views.  A workspace that holds the general plan but
// not a step's own takes the general one for it.
void bind_plans(pqc_ctx* ctx, const Plan& p) {
  ctx->plan = p;
  if (make_plan(&ctx->cfg, &ctx->decode_plan, For::kDecode) != PQC_OK || ctx->decode_plan.total > ctx->workspace_bytes) ctx->decode_plan = p;
  if (make_plan(&ctx->cfg, &ctx->pairs_plan, For::kPairs) != PQC_OK || ctx->pairs_plan.total > ctx->workspace_bytes) ctx->pairs_plan = p;
  ctx->ws = views(ctx->workspace, ctx->plan);
  ctx->decode_ws = views(ctx->workspace, ctx->decode_plan);
  ctx->pairs_ws = views(ctx->workspace, ctx->pairs_plan);
}
}  // namespace

int pqc_create(pqc_ctx** out, const pqc_config* cfg, void* workspace, size_t workspace_bytes) {
  if (!out) return PQC_EINVAL;
  *out = nullptr;
  Plan p;
  const int rc = make_plan(cfg, &p);
  if (rc != PQC_OK) return rc;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign) || workspace_bytes < p.total) return PQC_EWORKSPACE;
  pqc_ctx* ctx = new (std::nothrow) pqc_ctx;
  if (!ctx) return PQC_EINVAL;
  ctx->cfg = *cfg;
  ctx->cfg.n_capacity = p.s.cap;
  ctx->workspace = static_cast<char*>(workspace);
  ctx->workspace_bytes = workspace_bytes;
  bind_plans(ctx, p);
  ctx->hist_clean = false;
  ctx->next_phase = 0;
  ctx->last_hip = 0;
  ctx->append = AppendArgs{nullptr, nullptr, nullptr, 0, nullptr};
  *out = ctx;
  return PQC_OK;
}

int pqc_set_length(pqc_ctx* ctx, int32_t n_tokens, int32_t topk) {
  if (!ctx) return PQC_EINVAL;
  pqc_config c = ctx->cfg;
  c.n_tokens = n_tokens;
  c.topk = topk;
  Plan p;
  const int rc = make_plan(&c, &p);  // rejects a length beyond the capacity
  if (rc != PQC_OK) return rc;
  if (p.total > ctx->workspace_bytes) return PQC_EWORKSPACE;
  // The histogram region does not move and a clean one is all zero, whatever the length: it stays clean.
  ctx->cfg = c;
  bind_plans(ctx, p);
  return PQC_OK;
}

void pqc_destroy(pqc_ctx* ctx) { delete ctx; }

int pqc_last_hip_error(const pqc_ctx* ctx) { return ctx ? ctx->last_hip : 0; }

static int decode_impl(pqc_ctx* ctx, const void* q, const float* centroids, const uint8_t* codes, const void* k_cache,
                       const void* v_cache, int32_t* out_idx, float* out_attn, void* stream, unsigned phases) {
  if (!ctx || !q || !centroids || !codes || !k_cache || !v_cache || !out_idx || !out_attn) return PQC_EINVAL;
  if (!aligned16(q) || !aligned16(centroids) || !aligned16(codes) || !aligned16(k_cache) || !aligned16(v_cache) ||
      !aligned16(out_idx) || !aligned16(out_attn))
    return PQC_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  int rc = PQC_OK;
  if (phases & 1u) {
    rc = ensure_clean_hist(ctx, st);
    if (rc != PQC_OK) return rc;
    ctx->hist_clean = false;
  }
  if (ctx->cfg.kv_dtype == PQC_F32)
    launch_decode_t<float>(ctx, q, centroids, codes, k_cache, v_cache, out_idx, out_attn, st, phases);
  else
    launch_decode_t<bf16_t>(ctx, q, centroids, codes, k_cache, v_cache, out_idx, out_attn, st, phases);
  rc = check_launch(ctx);
  if (rc == PQC_OK && (phases & 4u)) {
    ctx->hist_clean = true;  // finalize_kernel zeroed them again
  }
  return rc;
}

int pqc_decode(pqc_ctx* ctx, const void* q, const float* centroids, const uint8_t* codes, const void* k_cache,
               const void* v_cache, int32_t* out_idx, float* out_attn, void* stream) {
  return decode_impl(ctx, q, centroids, codes, k_cache, v_cache, out_idx, out_attn, stream, 7u);
}

int pqc_decode_append(pqc_ctx* ctx, const void* q, const float* centroids, uint8_t* codes, const void* k_cache,
                      const void* v_cache, const void* new_key, int32_t position, int32_t* out_idx, float* out_attn,
                      void* stream) {
  if (!ctx || !new_key || !aligned16(new_key)) return PQC_EINVAL;
  const Shape& s = ctx->plan.s;
  // only a position whose code this call does not read: inside a window, or beyond the tokens in use
  if (position < 0 || position >= s.cap || (position >= s.I && position < s.N - s.L)) return PQC_EINVAL;
  ctx->append = AppendArgs{new_key, centroids, codes, (int)position, nullptr};
  const int rc = decode_impl(ctx, q, centroids, codes, k_cache, v_cache, out_idx, out_attn, stream, 7u);
  ctx->append = AppendArgs{nullptr, nullptr, nullptr, 0, nullptr};
  return rc;
}

static int indexed_impl(pqc_ctx* ctx, const void* q, const float* centroids, const uint8_t* codes,
                        const uint32_t* pair_counts, const void* k_cache, const void* v_cache, int32_t* out_idx,
                        float* out_attn, void* stream) {
  if (!ctx || !q || !centroids || !codes || !pair_counts || !k_cache || !v_cache || !out_idx || !out_attn) return PQC_EINVAL;
  if (!aligned16(q) || !aligned16(centroids) || !aligned16(codes) || !aligned16(pair_counts) || !aligned16(k_cache) ||
      !aligned16(v_cache) || !aligned16(out_idx) || !aligned16(out_attn))
    return PQC_EINVAL;
  if (!pairs_supported(&ctx->cfg)) return PQC_EUNSUPPORTED;
  hipStream_t st = static_cast<hipStream_t>(stream);
  int rc = ensure_clean_hist(ctx, st);  // the record counters live with the histograms
  if (rc != PQC_OK) return rc;
  ctx->hist_clean = false;
  if (ctx->cfg.kv_dtype == PQC_F32)
    launch_indexed_t<float>(ctx, q, centroids, codes, pair_counts, k_cache, v_cache, out_idx, out_attn, st);
  else
    launch_indexed_t<bf16_t>(ctx, q, centroids, codes, pair_counts, k_cache, v_cache, out_idx, out_attn, st);
  rc = check_launch(ctx);
  if (rc == PQC_OK) {
    ctx->hist_clean = true;
  }
  return rc;
}

int pqc_decode_indexed(pqc_ctx* ctx, const void* q, const float* centroids, const uint8_t* codes,
                       const uint32_t* pair_counts, const void* k_cache, const void* v_cache, int32_t* out_idx,
                       float* out_attn, void* stream) {
  return indexed_impl(ctx, q, centroids, codes, pair_counts, k_cache, v_cache, out_idx, out_attn, stream);
}

int pqc_decode_indexed_append(pqc_ctx* ctx, const void* q, const float* centroids, uint8_t* codes, uint32_t* pair_counts,
                              const void* k_cache, const void* v_cache, const void* new_key, int32_t position,
                              int32_t* out_idx, float* out_attn, void* stream) {
  if (!ctx || !new_key || !aligned16(new_key)) return PQC_EINVAL;
  const Shape& s = ctx->plan.s;
  if (position < 0 || position >= s.cap || (position >= s.I && position < s.N - s.L)) return PQC_EINVAL;
  ctx->append = AppendArgs{new_key, centroids, codes, (int)position, pair_counts};
  const int rc = indexed_impl(ctx, q, centroids, codes, pair_counts, k_cache, v_cache, out_idx, out_attn, stream);
  ctx->append = AppendArgs{nullptr, nullptr, nullptr, 0, nullptr};
  return rc;
}

int pqc_pair_counts(const pqc_config* cfg, const uint8_t* codes, uint32_t* pair_counts, void* stream) {
  Plan p;
  const int rc = make_plan(cfg, &p);
  if (rc != PQC_OK) return rc;
  if (!codes || !pair_counts) return PQC_EINVAL;
  if (cfg->pq_m != 2 || cfg->pq_centroids > kPairC) return PQC_EUNSUPPORTED;
  const Shape& s = p.s;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const size_t n = (size_t)s.B * s.Hkv * s.C * s.C;
  hipLaunchKernelGGL(reset_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, pair_counts, n);
  hipLaunchKernelGGL(pair_count_kernel, dim3((unsigned)((s.N + kPairTok - 1) / kPairTok), (unsigned)(s.B * s.Hkv)), dim3(256), 0,
                     st, codes, s.N, s.cap, s.C, pair_counts);
  return hipGetLastError() == hipSuccess ? PQC_OK : PQC_EHIP;
}

int pqc_pair_counts_add(const pqc_config* cfg, const uint8_t* codes, int32_t position, uint32_t* pair_counts, void* stream) {
  Plan p;
  const int rc = make_plan(cfg, &p);
  if (rc != PQC_OK) return rc;
  if (!codes || !pair_counts || position < 0 || position >= p.s.cap) return PQC_EINVAL;
  if (cfg->pq_m != 2 || cfg->pq_centroids > kPairC) return PQC_EUNSUPPORTED;
  const int units = p.s.B * p.s.Hkv;
  hipLaunchKernelGGL(pair_count_add_kernel, dim3((unsigned)((units + 63) / 64)), dim3(64), 0, static_cast<hipStream_t>(stream),
                     codes, p.s.cap, p.s.C, units, (int)position, pair_counts);
  return hipGetLastError() == hipSuccess ? PQC_OK : PQC_EHIP;
}

int pqc_decode_phase(pqc_ctx* ctx, int phase, const void* q, const float* centroids, const uint8_t* codes,
                     const void* k_cache, const void* v_cache, int32_t* out_idx, float* out_attn, void* stream) {
  if (!ctx || phase < 0 || phase >= PQC_DECODE_KERNELS) return PQC_EINVAL;
  if (phase != ctx->next_phase) return PQC_EINVAL;  // a phase out of turn would count a histogram twice or read a stale one
  const int rc = decode_impl(ctx, q, centroids, codes, k_cache, v_cache, out_idx, out_attn, stream, 1u << phase);
  if (rc == PQC_OK) ctx->next_phase = (phase + 1) % PQC_DECODE_KERNELS;
  return rc;
}

int pqc_lut(pqc_ctx* ctx, const void* q, const float* centroids, float* table, void* stream) {
  if (!ctx || !q || !centroids || !table) return PQC_EINVAL;
  if (!aligned16(q) || !aligned16(centroids) || !aligned16(table)) return PQC_EINVAL;
  const Shape& s = ctx->plan.s;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (ctx->cfg.kv_dtype == PQC_F32)
    launch_lut_t<float>(s, static_cast<const float*>(q), centroids, table, st);
  else
    launch_lut_t<bf16_t>(s, static_cast<const bf16_t*>(q), centroids, table, st);
  return check_launch(ctx);
}

int pqc_scan(pqc_ctx* ctx, const float* table, const uint8_t* codes, float* scores, void* stream) {
  if (!ctx || !table || !codes || !scores) return PQC_EINVAL;
  if (!aligned16(table) || !aligned16(codes) || !aligned16(scores)) return PQC_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  switch (ctx->plan.s.M) {
    case 1: launch_scan_m<1>(ctx, table, codes, scores, st); break;
    case 2: launch_scan_m<2>(ctx, table, codes, scores, st); break;
    case 4: launch_scan_m<4>(ctx, table, codes, scores, st); break;
    default: launch_scan_m<8>(ctx, table, codes, scores, st); break;
  }
  return check_launch(ctx);
}

int pqc_topk(pqc_ctx* ctx, const float* scores, int32_t* out_idx, void* stream) {
  if (!ctx || !scores || !out_idx) return PQC_EINVAL;
  if (!aligned16(scores) || !aligned16(out_idx)) return PQC_EINVAL;
  Shape s = ctx->plan.s;
  hipStream_t st = static_cast<hipStream_t>(stream);
  int rc = ensure_clean_hist(ctx, st);
  if (rc != PQC_OK) return rc;
  ctx->hist_clean = false;
  const unsigned units = (unsigned)(s.B * s.Hkv);
  s.copyWgs = copy_workgroups(units, 1, false);
  const float* nof = nullptr;
  hipLaunchKernelGGL(score_range_kernel, dim3(1, units), dim3(1024), 0, st, s, scores, ctx->ws.range);
  launch_hist<float, ScoreChunks>(s, ctx->ws, nof, nof, static_cast<const void*>(scores), 0, st);
  hipLaunchKernelGGL((select_kernel<float, 1, ScoreChunks, false>), dim3(s.nblkC, units), dim3(256), list_bytes<From::kBins>(s.tokC), st,
                     s, ctx->ws, nof, nof, nof, static_cast<const void*>(scores));
  hipLaunchKernelGGL((finalize_kernel<float, 1, false>), dim3(1 + s.copyWgs, units), dim3(kFinalThreads), finalize_lds_bytes(s, false), st, s,
                     ctx->ws, nof, nof, nof, out_idx, static_cast<float*>(nullptr), AppendArgs{nullptr, nullptr, nullptr, 0, nullptr});
  rc = check_launch(ctx);
  if (rc == PQC_OK) {
    ctx->hist_clean = true;
  }
  return rc;
}

int pqc_gather_attn(pqc_ctx* ctx, const void* q, const void* k_cache, const void* v_cache, const int32_t* idx,
                    float* out_attn, void* stream) {
  if (!ctx || !q || !k_cache || !v_cache || !idx || !out_attn) return PQC_EINVAL;
  if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(idx) || !aligned16(out_attn)) return PQC_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (ctx->cfg.kv_dtype == PQC_F32)
    launch_attn_t<float>(ctx, q, k_cache, v_cache, idx, out_attn, st);
  else
    launch_attn_t<bf16_t>(ctx, q, k_cache, v_cache, idx, out_attn, st);
  return check_launch(ctx);
}


}  // extern "C"

/* ------------------------------------------------- decode without an allocation */
// For callers that can neither allocate device memory nor hold a workspace of their own (code under HIP graph
// capture, serving loops, harnesses that forbid hipMalloc): the workspace of the step is a file-scope device
// array.  Host code never uses the array's name as an address: its device address is looked up once per device.
namespace {

constexpr size_t kStaticScratchBytes = (size_t)24 << 20;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices];  // per device: where that device holds its copy of `scratch`

// Device address of the current device's scratch array (looked up on the first call on that device).
int static_scratch(unsigned char** out, int* hip_code) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    *hip_code = (int)e;
    return PQC_EHIP;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      *hip_code = (int)e;
      return PQC_EHIP;
    }
    g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
  }
  *out = g_scratch_ptr[dev];
  return PQC_OK;
}

}  // namespace

extern "C" {

size_t pqc_static_scratch_bytes(void) { return kStaticScratchBytes; }

int pqc_decode_static(const pqc_config* cfg, const void* q, const float* centroids, const uint8_t* codes, const void* k_cache,
                      const void* v_cache, int32_t* out_idx, float* out_attn, void* stream) {
  pqc_ctx ctx;  // on the stack: nothing is allocated, on the host either
  Plan p;
  const int rc = make_plan(cfg, &p);
  if (rc != PQC_OK) return rc;
  if (p.total > kStaticScratchBytes) return PQC_ESCRATCH;
  unsigned char* base = nullptr;
  int hip_code = 0;
  const int rs = static_scratch(&base, &hip_code);
  if (rs != PQC_OK) return rs;
  ctx.cfg = *cfg;
  ctx.cfg.n_capacity = p.s.cap;
  ctx.workspace = reinterpret_cast<char*>(base);
  ctx.workspace_bytes = kStaticScratchBytes;
  bind_plans(&ctx, p);
  ctx.next_phase = 0;
  ctx.hist_clean = false;  // the array keeps what the last call (of any shape) left: the step's counters are cleared first,
                           // by a fill kernel, so that the call can be recorded into a graph
  ctx.last_hip = 0;
  ctx.append = AppendArgs{nullptr, nullptr, nullptr, 0, nullptr};
  return decode_impl(&ctx, q, centroids, codes, k_cache, v_cache, out_idx, out_attn, stream, 7u);
}

}  // extern "C"

/* ------------------------------------------------------------ PQ construction */
namespace {

struct BuildPlan {
  BuildShape s;
  int staged;  // centroids staged at a time
  bool fused;  // the accumulators of a round fit into LDS beside the centroids
};

constexpr size_t kRoundLds = 156 * 1024;  // of the compute unit's 160 KB

// Token ranges per (unit, partition), up to 256 of them (one unit with one partition then has a workgroup on every compute
// unit).  One workgroup fills a compute unit, so the time of a launch is that of its rounds of 256 workgroups; each pays for
// staging the centroids and writing the sums what about 1024 tokens cost.
// (A search of up to 256 steps: for calls that launch such a grid.)
RoundGrid round_grid(const BuildPlan& bp) {
  const BuildShape& s = bp.s;
  RoundGrid r{1, (s.N + 15) / 16 * 16, bp.staged};
  double best = 1e30;
  const double least = (double)s.units * s.M * s.N / 256.0;  // all compute units busy
  for (int p = 1; p <= 256; ++p) {
    const int tokens = ((s.N + p - 1) / p + 15) / 16 * 16;
    const int ranges = (s.N + tokens - 1) / tokens;
    const double rounds = std::ceil((double)s.units * s.M * ranges / 256.0);
    if (least + rounds * 1024.0 >= best) break;  // (no cut that takes more rounds can cost less)
    const double cost = rounds * (tokens + 1024.0);
    if (cost < best * 0.999) {
      best = cost;
      r.ranges = ranges;
      r.tokens = tokens;
    }
  }
  return r;
}

int make_build_plan(const pqc_config* cfg, BuildPlan* bp) {
  Plan p;
  const int rc = make_plan(cfg, &p);
  if (rc != PQC_OK) return rc;
  BuildShape& s = bp->s;
  s.units = p.s.B * p.s.Hkv;
  s.N = p.s.N; s.M = p.s.M; s.C = p.s.C; s.Dm = p.s.Dm; s.cap = p.s.cap;
  const bool mfma = cfg->kv_dtype == PQC_BF16 && s.Dm >= 32;
  auto stage_bytes = [&](int n) { return mfma ? mfma_stage_bytes(n, s.Dm) : vector_stage_bytes(n, s.Dm); };
  bp->staged = s.C;
  while (stage_bytes(bp->staged) > kRoundLds) bp->staged = (bp->staged / 2 + 15) / 16 * 16;
  bp->fused = stage_bytes(s.C) + round_sum_bytes(s.C, s.Dm) <= kRoundLds;
  return PQC_OK;
}

// The workspace holds sets of sums and counts, one sum per centroid value.  Neither the least a build runs in (one set) nor what it
// makes use of depends on n_tokens, so that one workspace serves every length of a cache.
struct BuildWorkspace {
  size_t off_counts, off_cent, total;
};
constexpr int kLinkedSets = 3;  // of the round in front, of the round itself, and cleared meanwhile for the round behind
BuildWorkspace build_workspace(const BuildShape& s, bool linked) {
  const size_t n = (size_t)s.units * s.M * s.C, sets = linked ? kLinkedSets : 1;
  BuildWorkspace b;
  b.off_counts = align_up(sizeof(unsigned long long) * n * s.Dm * sets);
  b.off_cent = align_up(b.off_counts + sizeof(unsigned) * n * sets);
  b.total = linked ? align_up(b.off_cent + sizeof(float) * n * s.Dm) : b.off_cent;
  return b;
}

// One launch over all token ranges: with sums a K-Means round, without it the assignment (codes written).
template <typename T, int DM, bool ACCUM>
void launch_round_d(const BuildShape& s, const RoundGrid& r, const RoundLink& link, const T* keys, float* cent, uint8_t* codes, unsigned long long* sums,
                    unsigned* counts, hipStream_t st) {
  const dim3 grid((unsigned)(s.units * s.M * r.ranges));
  const size_t acc = ACCUM ? round_sum_bytes(s.C, s.Dm) : 0;
  if constexpr (sizeof(T) == 2 && DM >= 32) {
    static_assert(DM > 64 || mfma_stage_bytes(256, DM) <= kRoundLds, "all centroids are staged at once, which the kernel knows");
    const size_t lds = mfma_stage_bytes(r.staged, DM) + acc;
    // eight tiles per wave read each staged centroid once for 128 tokens (as many as the registers of four waves per SIMD hold
    // with longer sub-vectors: six of 64 dimensions spill and take 1197 us for the eight rounds that five do in 770 us, four in
    // 777 us); short ranges take two, so that more than a few of the sixteen waves have tokens
    constexpr int kTiles = DM >= 128 ? 3 : DM == 64 ? 5 : 8;
    if (r.tokens >= 16 * 16 * kTiles)
      hipLaunchKernelGGL((pq_round_mfma_kernel<DM, kTiles, ACCUM>), grid, dim3(1024), lds, st, s, r, link, keys, cent, codes, sums, counts);
    else
      hipLaunchKernelGGL((pq_round_mfma_kernel<DM, 2, ACCUM>), grid, dim3(1024), lds, st, s, r, link, keys, cent, codes, sums, counts);
  } else {
    static_assert(vector_stage_bytes(256, DM) <= kRoundLds, "all centroids are staged at once");
    // one lane per token and two tokens per lane as soon as every wave has that many (8192 tokens x 8 heads, fp32, 4x256, which is
    // 1024 tokens per workgroup: assignment 105 us with four lanes per token, 97 us with one)
    constexpr int NT = DM >= 128 ? 512 : 1024, TT = DM <= 32 ? 2 : 1;
    const size_t lds = vector_stage_bytes(s.C, DM) + acc;
    if (r.tokens < NT) {
      hipLaunchKernelGGL((pq_round_vector_kernel<T, DM, NT, 4, 1, ACCUM>), grid, dim3(NT), lds, st, s, r, link, keys, cent, codes, sums, counts);
    } else if constexpr (ACCUM || DM >= 128) {
      if (r.tokens >= NT * TT)
        hipLaunchKernelGGL((pq_round_vector_kernel<T, DM, NT, 1, TT, ACCUM>), grid, dim3(NT), lds, st, s, r, link, keys, cent, codes, sums, counts);
      else if constexpr (TT > 1)
        hipLaunchKernelGGL((pq_round_vector_kernel<T, DM, NT, 1, 1, ACCUM>), grid, dim3(NT), lds, st, s, r, link, keys, cent, codes, sums, counts);
    } else {
      // The assignment alone needs no room for sums, so that small workgroups share a compute unit, and they are many: a last
      // one that is nearly empty holds nobody up (50001 tokens x 24 heads, fp32, 4x256: 1655 us with the ranges of a round,
      // 1490 us so; with 128 dimensions a compute unit holds one workgroup either way).  Two batches per workgroup where
      // there are enough of them; the number of workgroups has a limit.
      constexpr int kSmall = DM >= 64 ? 512 : 256;
      const bool wide = r.tokens >= NT * TT;
      int tokens = kSmall * (wide ? TT : 1) * (DM <= 32 && r.tokens >= 2 * NT * TT ? 2 : 1);
      while ((long long)s.units * s.M * ((s.N + tokens - 1) / tokens) > (1 << 20)) tokens *= 2;
      const RoundGrid a{(s.N + tokens - 1) / tokens, tokens, s.C};
      const dim3 agrid((unsigned)(s.units * s.M * a.ranges));
      if (wide)
        hipLaunchKernelGGL((pq_round_vector_kernel<T, DM, kSmall, 1, TT, false>), agrid, dim3(kSmall), lds, st, s, a, link, keys, cent, codes, sums, counts);
      else if constexpr (TT > 1)
        hipLaunchKernelGGL((pq_round_vector_kernel<T, DM, kSmall, 1, 1, false>), agrid, dim3(kSmall), lds, st, s, a, link, keys, cent, codes, sums, counts);
    }
  }
}
template <typename T, bool ACCUM>
void launch_round(const BuildShape& s, const RoundGrid& r, const RoundLink& link, const T* keys, float* cent, uint8_t* codes, unsigned long long* sums,
                  unsigned* counts, hipStream_t st) {
  switch (s.Dm) {
    case 16: launch_round_d<T, 16, ACCUM>(s, r, link, keys, cent, codes, sums, counts, st); break;
    case 32: launch_round_d<T, 32, ACCUM>(s, r, link, keys, cent, codes, sums, counts, st); break;
    case 64: launch_round_d<T, 64, ACCUM>(s, r, link, keys, cent, codes, sums, counts, st); break;
    default: launch_round_d<T, 128, ACCUM>(s, r, link, keys, cent, codes, sums, counts, st); break;
  }
}
constexpr RoundLink kNoLink{nullptr, nullptr, nullptr, nullptr, nullptr};
template <typename T>
void launch_assign(const BuildShape& s, const RoundGrid& r, const RoundLink& link, const T* keys, const float* cent, uint8_t* codes, hipStream_t st) {
  launch_round<T, false>(s, r, link, keys, const_cast<float*>(cent), codes, nullptr, nullptr, st);  // read only without sums
}

// Whether a build's rounds are linked: a round takes the means of the round in front when it stages its centroids, instead of a
// launch of their own in between.  Where one workgroup owns all tokens it writes the means itself, and where a round is two
// launches (sums that do not fit LDS) there is one that takes them anyway.
bool linked_rounds(const BuildPlan& bp, const RoundGrid& r) { return bp.fused && r.ranges > 1; }
// The assignment on the vector ALU runs in small workgroups when ranges are long, too many for each to read the sums.
template <typename T>
bool linked_assignment(const BuildShape& s, const RoundGrid& r) {
  return (sizeof(T) == 2 && s.Dm >= 32) || r.tokens < (s.Dm >= 128 ? 512 : 1024);
}

template <typename T>
int pq_build_t(const BuildPlan& bp, const RoundGrid& r, bool linked, const T* keys, const int32_t* init_idx, int iters, float* cent, uint8_t* codes,
               char* wsp, hipStream_t st) {
  const BuildShape& s = bp.s;
  const BuildWorkspace b = build_workspace(s, linked);
  const unsigned uj = (unsigned)(s.units * s.M);
  const size_t n_cent = (size_t)uj * s.C, n_val = n_cent * s.Dm;
  unsigned long long* const sums = reinterpret_cast<unsigned long long*>(wsp);
  unsigned* const counts = reinterpret_cast<unsigned*>(wsp + b.off_counts);
  const dim3 per_cent((unsigned)((s.C * s.Dm + 255) / 256), uj);
  const bool means = !bp.fused || r.ranges > 1;  // else a round writes them itself
  // linked: two places for the centroids in turn, the last ones to the caller's
  auto place = [&](int it) { return linked && ((iters - it) & 1) ? reinterpret_cast<float*>(wsp + b.off_cent) : cent; };
  auto link_of = [&](int it) {  // what launch `it` takes over from round it - 1; the last launch is the assignment
    if (!linked || it == 0) return kNoLink;
    const int prev = (it - 1) % kLinkedSets, next = (it + 1) % kLinkedSets;
    const bool more = it + 1 < iters;
    return RoundLink{sums + prev * n_val, counts + prev * n_cent, place(it), more ? sums + next * n_val : nullptr,
                     more ? counts + next * n_cent : nullptr};
  };
  hipLaunchKernelGGL((pq_init_kernel<T>), per_cent, dim3(256), 0, st, s, keys, init_idx, place(0), means && iters > 0 ? sums : nullptr,
                     counts, linked ? std::min(iters, 2) : 1);
  for (int it = 0; it < iters; ++it) {
    if (bp.fused) {
      const int set = linked ? it % kLinkedSets : 0;
      launch_round<T, true>(s, r, link_of(it), keys, place(std::max(it - 1, 0)), codes, sums + set * n_val, counts + set * n_cent, st);
    } else {  // the accumulators are too large for LDS: codes first, then the sums of the members of each code
      static_assert(mfma_stage_bytes(256, 32) + round_sum_bytes(256, 32) <= kRoundLds, "and 16 and 32 dimensions always fit");
      static_assert(vector_stage_bytes(256, 32) + round_sum_bytes(256, 32) <= kRoundLds, "and 16 and 32 dimensions always fit");
      launch_assign<T>(s, r, kNoLink, keys, cent, codes, st);
      const int tpw = accum_tokens_per_wg(s.C);
      const dim3 grid((s.N + tpw - 1) / tpw, uj);
      const size_t lds = (size_t)tpw * sizeof(unsigned short);
      switch (s.Dm) {
        case 64: hipLaunchKernelGGL((pq_accum_kernel<T, 64>), grid, dim3(256), lds, st, s, keys, codes, sums, counts); break;
        default: hipLaunchKernelGGL((pq_accum_kernel<T, 128>), grid, dim3(256), lds, st, s, keys, codes, sums, counts); break;
      }
    }
    if (means && !linked) hipLaunchKernelGGL(pq_mean_kernel, per_cent, dim3(256), 0, st, s, sums, counts, cent, cent);
  }
  if (linked && iters > 0 && linked_assignment<T>(s, r)) {
    launch_assign<T>(s, r, link_of(iters), keys, place(iters - 1), codes, st);
  } else {
    if (linked && iters > 0) {
      const int last = (iters - 1) % kLinkedSets;
      hipLaunchKernelGGL(pq_mean_kernel, per_cent, dim3(256), 0, st, s, sums + last * n_val, counts + last * n_cent, place(iters - 1), cent);
    }
    launch_assign<T>(s, r, kNoLink, keys, cent, codes, st);
  }
  return hipGetLastError() == hipSuccess ? PQC_OK : PQC_EHIP;
}

}  // namespace

extern "C" {

size_t pqc_pq_build_workspace_bytes(const pqc_config* cfg) {
  BuildPlan bp;
  if (make_build_plan(cfg, &bp) != PQC_OK) return 0;
  return build_workspace(bp.s, bp.fused).total;
}

int pqc_pq_build(const pqc_config* cfg, const void* keys, const int32_t* init_idx, int32_t iters, float* centroids,
                 uint8_t* codes, void* workspace, size_t workspace_bytes, void* stream) {
  BuildPlan bp;
  const int rc = make_build_plan(cfg, &bp);
  if (rc != PQC_OK) return rc;
  if (!keys || !init_idx || !centroids || !codes || iters < 0) return PQC_EINVAL;
  if (!aligned16(keys) || !aligned16(init_idx) || !aligned16(centroids) || !aligned16(codes)) return PQC_EINVAL;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign) || workspace_bytes < build_workspace(bp.s, false).total)
    return PQC_EWORKSPACE;
  const RoundGrid r = round_grid(bp);
  const bool linked = linked_rounds(bp, r) && workspace_bytes >= build_workspace(bp.s, true).total;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* wsp = static_cast<char*>(workspace);
  if (cfg->kv_dtype == PQC_F32) return pq_build_t<float>(bp, r, linked, static_cast<const float*>(keys), init_idx, iters, centroids, codes, wsp, st);
  return pq_build_t<bf16_t>(bp, r, linked, static_cast<const bf16_t*>(keys), init_idx, iters, centroids, codes, wsp, st);
}

int pqc_pq_assign(const pqc_config* cfg, const void* keys, const float* centroids, uint8_t* codes, void* stream) {
  BuildPlan bp;
  const int rc = make_build_plan(cfg, &bp);
  if (rc != PQC_OK) return rc;
  if (!keys || !centroids || !codes) return PQC_EINVAL;
  if (!aligned16(keys) || !aligned16(centroids) || !aligned16(codes)) return PQC_EINVAL;
  const RoundGrid r = round_grid(bp);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (cfg->kv_dtype == PQC_F32)
    launch_assign<float>(bp.s, r, kNoLink, static_cast<const float*>(keys), centroids, codes, st);
  else
    launch_assign<bf16_t>(bp.s, r, kNoLink, static_cast<const bf16_t*>(keys), centroids, codes, st);
  return hipGetLastError() == hipSuccess ? PQC_OK : PQC_EHIP;
}

int pqc_pq_encode_token(const pqc_config* cfg, const void* key, const float* centroids, uint8_t* codes, int32_t position,
                        void* stream) {
  BuildPlan bp;
  const int rc = make_build_plan(cfg, &bp);
  if (rc != PQC_OK) return rc;
  if (!key || !centroids || !codes || position < 0 || position >= bp.s.cap) return PQC_EINVAL;
  if (!aligned16(key) || !aligned16(centroids) || !aligned16(codes)) return PQC_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const BuildShape& s = bp.s;
  const dim3 grid((unsigned)(s.units * s.M));
  if (cfg->kv_dtype == PQC_F32)
    hipLaunchKernelGGL(pq_encode_kernel<float>, grid, dim3(256), 0, st, s, static_cast<const float*>(key), (int)position, centroids,
                       codes);
  else
    hipLaunchKernelGGL(pq_encode_kernel<bf16_t>, grid, dim3(256), 0, st, s, static_cast<const bf16_t*>(key), (int)position,
                       centroids, codes);
  return hipGetLastError() == hipSuccess ? PQC_OK : PQC_EHIP;
}

int pqc_block_stats(const pqc_config* cfg, const int32_t* idx, int64_t n_idx, int32_t block_tokens, int32_t k_cache,
                    int32_t* counts, int32_t* blocks, void* stream) {
  Plan p;
  int rc = make_plan(cfg, &p);
  if (rc != PQC_OK) return rc;
  if (!idx || !counts || n_idx < 0 || block_tokens < 1 || block_tokens >= kCountBins) return PQC_EINVAL;
  const int nb = (p.s.N + block_tokens - 1) / block_tokens;
  if (k_cache < 0 || k_cache > nb || (k_cache > 0 && !blocks)) return PQC_EINVAL;
  const unsigned long long inv_bt = ((1ull << kBlockShift) + (unsigned)block_tokens - 1) / (unsigned)block_tokens;
  const dim3 grid((unsigned)(p.s.B * p.s.Hkv));
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (nb <= kLdsBlocks)
    hipLaunchKernelGGL(block_stats_kernel<true>, grid, dim3(1024), (size_t)nb * sizeof(int), st, idx, (long long)n_idx, p.s.N, inv_bt, nb,
                       (int)k_cache, counts, blocks);
  else
    hipLaunchKernelGGL(block_stats_kernel<false>, grid, dim3(1024), 0, st, idx, (long long)n_idx, p.s.N, inv_bt, nb, (int)k_cache, counts,
                       blocks);
  return hipGetLastError() == hipSuccess ? PQC_OK : PQC_EHIP;
}

int pqc_block_cache_update(const pqc_config* cfg, int32_t block_tokens, int32_t n_slots, int32_t policy, int32_t step,
                           const int32_t* counts, const int32_t* blocks, int32_t k_cache, int32_t* slot_block,
                           int32_t* slot_stamp, int32_t* slot_uses, int32_t* stats, void* stream) {
  Plan p;
  const int rc = make_plan(cfg, &p);
  if (rc != PQC_OK) return rc;
  if (!counts || !slot_block || !slot_stamp || !slot_uses || !stats || block_tokens < 1) return PQC_EINVAL;
  if (n_slots < 1 || n_slots > kCacheSlots || k_cache < 0 || k_cache > kCacheSlots || (k_cache > 0 && !blocks)) return PQC_EINVAL;
  if (policy != PQC_CACHE_LRU && policy != PQC_CACHE_LFU) return PQC_EINVAL;
  const int nb = (p.s.N + block_tokens - 1) / block_tokens;
  hipLaunchKernelGGL(block_cache_kernel, dim3((unsigned)(p.s.B * p.s.Hkv)), dim3(256), 0, static_cast<hipStream_t>(stream), nb,
                     (int)n_slots, (int)k_cache, policy == PQC_CACHE_LFU ? 1 : 0, (int)step, counts, blocks, slot_block, slot_stamp,
                     slot_uses, stats);
  return hipGetLastError() == hipSuccess ? PQC_OK : PQC_EHIP;
}

}  // extern "C"
