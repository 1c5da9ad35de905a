// GRAPE kernels of d = 64 (see small_grape.h).
#define GRAPE_KERNELS
#include "small_grape.h"

namespace redo {

template <>
hipError_t grape_fused<64>(const TView& tv, const SmallGrapeArgs& a, hipStream_t st) {
    return launch_fused_kind<64>(tv, a, st);
}
template <>
hipError_t grape_scan<64>(const TView& tv, const ScanArgs& a, hipStream_t st) {
    return launch_scan<64>(tv, a, st);
}
template <>
hipError_t grape_traces<64>(const TView& tv, const TraceArgs& a, hipStream_t st) {
    return launch_trace_kind<64>(tv, a, st);
}

}  // namespace redo
