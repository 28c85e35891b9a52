// The select kernels that have no histogram kernel in front (From::kCount, kShort, kPairs and kPairsMany), instantiated in a file of their own: it
// compiles beside pqc_api.hip.
#include "pqc_kernels.h"

namespace pqc {
namespace {

struct Args {
  const Shape& s;
  const Workspace& ws;
  const void* q;
  const float* cent;
  const uint8_t* codes;
  const unsigned* pair_counts;
  int uncounted;
  const void *k, *v;
  hipStream_t st;
};

template <typename T, int G, int M, From FROM, int VW>
void launch(const Args& a) {
  hipLaunchKernelGGL((select_kernel<T, G, CodeChunks<M>, true, FROM, VW>), dim3(a.s.nblkC, (unsigned)(a.s.B * a.s.Hkv)), dim3(select_threads<FROM>()),
                     table_form_lds_bytes<FROM>(a.s, sizeof(T) == 2 && kMatrixCoreAttention), a.st, a.s, a.ws, static_cast<const T*>(a.q),
                     static_cast<const T*>(a.k), static_cast<const T*>(a.v), static_cast<const void*>(a.codes), a.cent, a.pair_counts, a.uncounted);
}

template <typename T, int G>
void launch_form(const Args& a) {
  if (a.pair_counts && a.s.pairsMany)
    launch<T, G, 2, From::kPairsMany, 8>(a);
  else if (a.pair_counts)
    launch<T, G, 2, From::kPairs, 4>(a);
  else if (counts_pairs(a.s))
    launch<T, G, 2, From::kCount, 4>(a);
  else if (a.s.M == 2)
    launch<T, G, 2, From::kShort, 16>(a);
  else if (a.s.C <= 64)
    launch<T, G, 4, From::kShort, 4>(a);
  else
    launch<T, G, 4, From::kShort, 16>(a);
}

template <typename T>
void launch_g(const Args& a) {
  switch (a.s.G) {
    case 1: launch_form<T, 1>(a); break;
    case 2: launch_form<T, 2>(a); break;
    case 4: launch_form<T, 4>(a); break;
    default: launch_form<T, 8>(a); break;
  }
}

}  // namespace

void launch_pairs_select(bool bf16, const Shape& s, const Workspace& ws, const void* q, const float* cent, const uint8_t* codes,
                         const unsigned* pair_counts, int uncounted, const void* k, const void* v, hipStream_t st) {
  const Args a{s, ws, q, cent, codes, pair_counts, uncounted, k, v, st};
  if (bf16)
    launch_g<bf16_t>(a);
  else
    launch_g<float>(a);
}

void launch_short_select(bool bf16, const Shape& s, const Workspace& ws, const void* q, const float* cent, const uint8_t* codes, const void* k,
                         const void* v, hipStream_t st) {
  launch_pairs_select(bf16, s, ws, q, cent, codes, nullptr, -1, k, v, st);
}

}  // namespace pqc
