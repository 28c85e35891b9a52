// The select kernel of short caches (From::kShort), instantiated in a file of its own: it compiles beside pqc_api.hip.
#include "pqc_kernels.h"

namespace pqc {
namespace {

template <typename T, int G, int M>
void launch(const Shape& s, const Workspace& ws, const void* q, const float* cent, const uint8_t* codes, const void* k, const void* v,
            hipStream_t st) {
  const dim3 grid(s.nblkC, (unsigned)(s.B * s.Hkv)), block(select_threads<From::kShort>());
  const size_t lds = short_lds_bytes(s, sizeof(T) == 2 && kMatrixCoreAttention);
  const T *qt = static_cast<const T*>(q), *kt = static_cast<const T*>(k), *vt = static_cast<const T*>(v);
  const void* src = codes;
  if (s.C <= 64)
    hipLaunchKernelGGL((select_kernel<T, G, CodeChunks<M>, true, From::kShort, 4>), grid, block, lds, st, s, ws, qt, kt, vt, src, cent,
                       static_cast<const unsigned*>(nullptr), -1);
  else
    hipLaunchKernelGGL((select_kernel<T, G, CodeChunks<M>, true, From::kShort, 16>), grid, block, lds, st, s, ws, qt, kt, vt, src, cent,
                       static_cast<const unsigned*>(nullptr), -1);
}

template <typename T, int G>
void launch_m(const Shape& s, const Workspace& ws, const void* q, const float* cent, const uint8_t* codes, const void* k, const void* v,
              hipStream_t st) {
  if (s.M == 2)
    launch<T, G, 2>(s, ws, q, cent, codes, k, v, st);
  else
    launch<T, G, 4>(s, ws, q, cent, codes, k, v, st);
}

template <typename T>
void launch_g(const Shape& s, const Workspace& ws, const void* q, const float* cent, const uint8_t* codes, const void* k, const void* v,
              hipStream_t st) {
  switch (s.G) {
    case 1: launch_m<T, 1>(s, ws, q, cent, codes, k, v, st); break;
    case 2: launch_m<T, 2>(s, ws, q, cent, codes, k, v, st); break;
    case 4: launch_m<T, 4>(s, ws, q, cent, codes, k, v, st); break;
    default: launch_m<T, 8>(s, ws, q, cent, codes, k, v, st); break;
  }
}

}  // namespace

void launch_short_select(bool bf16, const Shape& s, const Workspace& ws, const void* q, const float* cent, const uint8_t* codes, const void* k,
                         const void* v, hipStream_t st) {
  if (bf16)
    launch_g<bf16_t>(s, ws, q, cent, codes, k, v, st);
  else
    launch_g<float>(s, ws, q, cent, codes, k, v, st);
}

}  // namespace pqc
