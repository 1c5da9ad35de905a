// GRAPE kernels of d = 2, 4, 8 (see small_grape.h).
#define GRAPE_KERNELS
#include "small_grape.h"

namespace redo {

template <>
hipError_t grape_fused<2>(const TView& tv, const SmallGrapeArgs& a, hipStream_t st) {
    return launch_fused_kind<2>(tv, a, st);
}
template <>
hipError_t grape_fused<4>(const TView& tv, const SmallGrapeArgs& a, hipStream_t st) {
    return launch_fused_kind<4>(tv, a, st);
}
template <>
hipError_t grape_fused<8>(const TView& tv, const SmallGrapeArgs& a, hipStream_t st) {
    return launch_fused_kind<8>(tv, a, st);
}
template <>
hipError_t grape_scan<8>(const TView& tv, const ScanArgs& a, hipStream_t st) {
    return launch_scan<8>(tv, a, st);
}
template <>
hipError_t grape_traces<8>(const TView& tv, const TraceArgs& a, hipStream_t st) {
    return launch_trace_kind<8>(tv, a, st);
}

}  // namespace redo
