// GRAPE kernels of d = 32 (see small_grape.h).
#define GRAPE_KERNELS
#include "small_grape.h"

namespace redo {

template <>
hipError_t grape_fused<32>(const TView& tv, const SmallGrapeArgs& a, hipStream_t st) {
    return launch_fused_kind<32>(tv, a, st);
}
template <>
hipError_t grape_scan<32>(const TView& tv, const ScanArgs& a, hipStream_t st) {
    return launch_scan<32>(tv, a, st);
}
template <>
hipError_t grape_traces<32>(const TView& tv, const TraceArgs& a, hipStream_t st) {
    return launch_trace_kind<32>(tv, a, st);
}

}  // namespace redo
