// Instances of the decode kernels for one width of the state: compiled once with each BEAM_KST, the
// number of matrix steps over e (bf16, beam_kernel: 1, 2, 3, 4 or 8 steps of 32; float32,
// decode_lds_kernel: 16 or 32 steps of 4; for other widths the next larger one).
#include "beam_args.h"

#include <type_traits>

#ifndef BEAM_KST
#error "BEAM_KST is not set"
#endif
#define BEAM_CAT2(a, b) a##b
#define BEAM_CAT(a, b) BEAM_CAT2(a, b)

namespace nezha {
namespace {
#include "device_common.h"
#include "beam_common.h"
#if BEAM_KST <= 8
#include "beam_level.h"
#else
#include "decode_lds.h"
#endif

template <class Kernel>
int launch(Kernel kern, const BeamArgs& a, int B, size_t lds, hipStream_t stream) {
  if (lds > 64 * 1024)
    NEZHA_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kern, dim3((unsigned)B), dim3(kBeamThreads), lds, stream, a);
  NEZHA_HIP_CHECK(hipGetLastError());
  return NEZHA_OK;
}
}  // namespace

#if BEAM_KST <= 8
int BEAM_CAT(launch_beam_, BEAM_KST)(const BeamArgs& a, int B, int row_tiles, size_t lds,
                                     hipStream_t stream) {
  switch (row_tiles) {
    case 1: return launch(beam_kernel<BEAM_KST, 1>, a, B, lds, stream);
    case 2: return launch(beam_kernel<BEAM_KST, 2>, a, B, lds, stream);
    case 3: return launch(beam_kernel<BEAM_KST, 3>, a, B, lds, stream);
    case 4: return launch(beam_kernel<BEAM_KST, 4>, a, B, lds, stream);
    case 5: return launch(beam_kernel<BEAM_KST, 5>, a, B, lds, stream);
    case 6: return launch(beam_kernel<BEAM_KST, 6>, a, B, lds, stream);
    case 7: return launch(beam_kernel<BEAM_KST, 7>, a, B, lds, stream);
    default: return launch(beam_kernel<BEAM_KST, 8>, a, B, lds, stream);
  }
}
#else
int BEAM_CAT(launch_decode_lds_, BEAM_KST)(const BeamArgs& a, int B, int row_tiles, size_t lds,
                                           hipStream_t stream) {
  if (row_tiles == 1) return launch(decode_lds_kernel<BEAM_KST, 1>, a, B, lds, stream);
  if (row_tiles == 2) return launch(decode_lds_kernel<BEAM_KST, 2>, a, B, lds, stream);
#if BEAM_KST <= 16
  if (row_tiles <= 4) return launch(decode_lds_kernel<BEAM_KST, 4>, a, B, lds, stream);
#endif
  return NEZHA_EINVAL;
}
#endif
#if BEAM_KST == 4
size_t beam_shared_bytes() { return sizeof(BeamShared); }
#endif
#if BEAM_KST == 16
size_t decode_shared_bytes() { return sizeof(DecodeShared); }
#endif
}  // namespace nezha
