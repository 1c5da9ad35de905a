// GRAPE at d = 2 .. 64: choice of the form, its workspace, and the sequence of launches
// (kernels in small_grape.h).
#include "small_grape.h"

namespace redo {
namespace {

// a step is one factor between diagonal scalings: the scans walk the factors
bool one_factor(const TView& tv) { return tv.d >= 32 && tv.cache && tv.K == 1 && step_kind(tv) <= 1; }

// workspace of the side-by-side form for bc instances at a time
struct ScanWS {
    int* codes;
    double* phi;
    double *tr, *d0, *nu, *fpart;
    double2* ov;
    float2 *Up, *X, *LH;
    size_t bytes;
    ScanWS(const redo_table_s* t, long long bc, long long N, void* base) {
        const size_t mat = (size_t)t->entry_elems, K = t->desc.K;
        const bool one = one_factor(view_of(t));
        Carve c(base);
        codes = c.take<int>(bc * N * K);
        phi = c.take<double>(t->desc.phased ? bc * N * K : 0);
        tr = c.take<double>(bc * N * K * 6);
        d0 = c.take<double>(bc * K * 2);
        nu = c.take<double>(bc);
        ov = c.take<double2>(bc);
        fpart = c.take<double>(fidelity_partial_doubles((int)bc));
        Up = c.take<float2>(one ? 0 : mat * bc * N);
        X = c.take<float2>(mat * bc * N);
        LH = c.take<float2>(mat * bc * (N + 1));
        if (one) Up = nullptr;
        bytes = c.used;
    }
};

// instances taken at a time: all, or as many as the limit holds (0: not one)
long long scan_chunk(const redo_table_s* t, long long B, long long N, size_t limit) {
    if (ScanWS(t, B, N, nullptr).bytes <= limit) return B;
    long long lo = 0, hi = B;
    while (lo + 1 < hi) {
        const long long mid = (lo + hi) / 2;
        (ScanWS(t, mid, N, nullptr).bytes <= limit ? lo : hi) = mid;
    }
    return lo;
}
size_t scan_limit(long long requested) { return requested > 0 ? SMALL_SCAN_CHECKPOINTED_MAX : SMALL_SCAN_MAX; }

}  // namespace

size_t small_grape_workspace_bytes(int d, int K, long long B, long long N_max, long long C) {
    const long long nck = (N_max + C - 1) / C;
    const size_t mats = sizeof(float2) * (size_t)d * d * (size_t)B * (size_t)(nck + C);
    return ((mats + 255) & ~size_t(255)) + sizeof(double) * (size_t)B * K * 6;
}

size_t small_grape_scan_bytes(const redo_table_s* t, long long B, long long N_max, long long requested) {
    // d = 8: a batch that fills the chip walks its factors with the states in registers, and needs
    // neither the propagators nor LH in memory
    if (t->desc.d < 8 || (t->desc.d == 8 && B > SMALL_SCAN_D8_BATCH)) return 0;
    const long long bc = scan_chunk(t, B, N_max, scan_limit(requested));
    return bc < 1 ? 0 : ScanWS(t, bc, N_max, nullptr).bytes;
}

hipError_t small_grape(const redo_table_s* t, const SmallGrapeArgs& a, hipStream_t st) {
    const TView tv = view_of(t);
    switch (tv.d) {
        case 2: return grape_fused<2>(tv, a, st);
        case 4: return grape_fused<4>(tv, a, st);
        case 8: return grape_fused<8>(tv, a, st);
        case 16: return grape_fused<16>(tv, a, st);
        case 32: return grape_fused<32>(tv, a, st);
        case 64: return grape_fused<64>(tv, a, st);
        default: return hipErrorInvalidValue;
    }
}

redo_status small_grape_scan(const redo_table_s* t, const float* u, const int* n_steps, int B, int N, const float2* U_target,
                             long long requested, double* fidelity, double2* overlap, float* grad, void* workspace,
                             hipStream_t st) {
    const TView tv = view_of(t);
    const int d = tv.d, K = tv.K, KK = tv.phased ? 2 : 1;
    const long long mat = tv.ent, bc = scan_chunk(t, B, N, scan_limit(requested));
    const ScanWS w(t, bc, N, workspace);
    for (long long b0 = 0; b0 < B; b0 += bc) {
        const int cnt = (int)std::min<long long>(bc, B - b0);
        const float* uc = u + b0 * N * K * KK;
        const int* ns = n_steps ? n_steps + b0 : nullptr;
        REDO_HIP(quantise_all(t, uc, cnt, N, w.codes, w.phi, st));
        if (w.Up) {
            SmallChainArgs c{};
            c.u = uc;
            c.n_steps = ns;
            c.B = cnt;
            c.N_max = N;
            c.compose = 1;
            c.drift0 = (int)(b0 % tv.n_drift);
            c.X_out = w.Up;
            c.quiet = 1;   // quantise_all has reported the controls
            REDO_HIP(small_chain(t, c, st));
        }
        ScanArgs s{};
        s.n_steps = ns;
        s.B = cnt;
        s.N_max = N;
        s.U_target = U_target + b0 * mat;
        s.Up = w.Up;
        s.u = uc;
        s.drift0 = (int)(b0 % tv.n_drift);
        s.X = w.X;
        s.LH = w.LH;
        TraceArgs tr{};
        tr.u = uc;
        tr.n_steps = ns;
        tr.B = cnt;
        tr.N_max = N;
        tr.drift0 = s.drift0;
        tr.X = w.X;
        tr.LH = w.LH;
        tr.tr = w.tr;
        switch (d) {
            case 8: REDO_HIP(grape_scan<8>(tv, s, st)); break;
            case 16: REDO_HIP(grape_scan<16>(tv, s, st)); break;
            case 32: REDO_HIP(grape_scan<32>(tv, s, st)); break;
            default: REDO_HIP(grape_scan<64>(tv, s, st));
        }
        REDO_HIP(unitary_fidelity_sliced(d, cnt, s.U_target, mat, w.X + (size_t)(N - 1) * mat, mat * N, w.ov, fidelity + b0,
                                         w.nu, w.fpart, st));
        if (overlap)
            REDO_HIP(hipMemcpyAsync(overlap + b0, w.ov, sizeof(double2) * cnt, hipMemcpyDeviceToDevice, st));
        switch (d) {
            case 8: REDO_HIP(grape_traces<8>(tv, tr, st)); break;
            case 16: REDO_HIP(grape_traces<16>(tv, tr, st)); break;
            case 32: REDO_HIP(grape_traces<32>(tv, tr, st)); break;
            default: REDO_HIP(grape_traces<64>(tv, tr, st));
        }
        REDO_HIP(d0_traces(d, cnt, K, tv.phased, w.LH, mat * (N + 1), tv.g, w.d0, st, 1));
        REDO_HIP(grad_assemble(cnt, N, K, tv.phased, tv.eps, tv.dt, w.codes, tv.phased ? w.phi : nullptr, w.tr, w.d0, w.ov,
                               w.nu, ns, grad + b0 * N * K * KK, 0, st));
    }
    return REDO_OK;
}

}  // namespace redo
