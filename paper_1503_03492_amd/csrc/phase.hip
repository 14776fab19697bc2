// phase.hip -- the sweep kernel's instances.  Built once per image / increment
// type and region side (SMRE_TX, SMRE_TQ, SMRE_KAHAN, SMRE_R), in parallel: an
// instance holds the unrolled code of every side and takes long to compile.
#include "sparse.hpp"

namespace smre {

template <typename TX, typename TQ, int R, int SMAX, bool KAHAN>
void launch_phase(int grid, const PhaseArgs& p, bool stream, hipStream_t s) {
  if (stream)
    hipLaunchKernelGGL((stream_batch<TX, TQ, R, SMAX, KAHAN>), dim3(grid), dim3(128), 0, s,
                       p.imgs, p.items, p);
  else
    hipLaunchKernelGGL((region_phase<TX, TQ, R, SMAX, KAHAN>), dim3(grid), dim3(kPhaseThreads), 0,
                       s, p.imgs, p.items, p);
}

template <typename TX, typename TQ, int R, int SMAX, bool KAHAN>
void launch_stream(const ImageDesc& a, int cy, int cx, int ncx, int grid, const PhaseArgs& p,
                   hipStream_t s) {
  hipLaunchKernelGGL((stream_phase<TX, TQ, R, SMAX, KAHAN>), dim3(grid), dim3(128), 0, s, a, cy, cx,
                     ncx, p.done, p.abort, p.q);
}

template <typename TX, typename TQ, int R, int SMAX, bool KAHAN> hipError_t phase_blocks(int* n, bool stream) {
  if (stream)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(
        n, (const void*)stream_batch<TX, TQ, R, SMAX, KAHAN>, 128, 0);
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(
      n, (const void*)region_phase<TX, TQ, R, SMAX, KAHAN>, kPhaseThreads, 0);
}

#define SMRE_INSTANCE(smax)                                                              \
  template void launch_phase<SMRE_TX, SMRE_TQ, SMRE_R, smax, SMRE_KAHAN>(                \
      int, const PhaseArgs&, bool, hipStream_t);                                         \
  template void launch_stream<SMRE_TX, SMRE_TQ, SMRE_R, smax, SMRE_KAHAN>(               \
      const ImageDesc&, int, int, int, int, const PhaseArgs&, hipStream_t);              \
  template hipError_t phase_blocks<SMRE_TX, SMRE_TQ, SMRE_R, smax, SMRE_KAHAN>(int*, bool);
#if SMRE_R == 16
SMRE_INSTANCE(9)
#endif
#if SMRE_R == 8
SMRE_INSTANCE(9)
#elif SMRE_R == 16
SMRE_INSTANCE(17)
#else
SMRE_INSTANCE(33)
#endif

}  // namespace smre
