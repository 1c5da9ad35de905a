// Kernels of the GRAPE objective and gradient at d = 2 .. 64 (Sec. III), on the register-resident
// steps of reg_step.h.
//
// With the forward states X_n = U_n .. U_1 and the conjugate-transposed backward factors
// LH_n = L_n^dag, L_N = U_f^dag, L_{n-1} = L_n U_n (so LH_{n-1} = U_n^dag LH_n: both chains
// are left products), the gradient needs traces of Y_n = X_n L_n, one more product per step.
//   * d = 8 .. 64, every state kept: the two chains run at the same time in one launch, each
//     walking precomposed step propagators (or the factors, when a step is one of them), then
//     one launch takes the traces of every (instance, step) in parallel.  The dependent depth
//     is one product per step.
//   * d = 2, 4, large batches at d = 8, and any d in a small workspace: one launch; a wave
//     walks its instances forward, keeping every state or every C-th, and back, forming the
//     traces of each step beside the adjoint product.
// d = 16, 256 instances x 500 steps: 1.23 ms (scans 0.84, traces 0.22, composition 0.17) against 5.6
// for one workgroup per instance with states in LDS; d = 32, 64 x 1500 ragged with five channels:
// 3.7 ms (2.2, 0.6, 0.9) against 29.4; d = 4, 65,536 x 200, fused: 2.9 ms against 5.2.  The order
// of every sum is that of the scalar complex product: gradients at small phased amplitudes
// amplify rounding (errors to 2e-3 of the largest entry), and a layout that summed in another
// order gave other digits there.
#pragma once
#include "large_path.h"
#include "reg_step.h"

namespace redo {

struct ScanArgs {
    const int* n_steps;
    int B, N_max;
    const float2* U_target;
    const float2* Up;    // [B][N_max][d][d] step propagators (precomposed form)
    const float* u;      // controls (factor form)
    int drift0;
    float2* X;           // [B][N_max][d][d]: X_1 .. X_N (X_N also in the last place when shorter)
    float2* LH;          // [B][N_max + 1][d][d]: LH_0 .. LH_N
};

struct TraceArgs {
    const float* u;
    const int* n_steps;
    int B, N_max, drift0;
    const float2* X;
    const float2* LH;
    double* tr;   // [B][N_max][K][6]: traces of Y_{s+1}
};

// by dimension, one source file each
template <int D>
hipError_t grape_fused(const TView& tv, const SmallGrapeArgs& a, hipStream_t st);
template <int D>
hipError_t grape_scan(const TView& tv, const ScanArgs& a, hipStream_t st);
template <int D>
hipError_t grape_traces(const TView& tv, const TraceArgs& a, hipStream_t st);

#ifdef GRAPE_KERNELS
namespace {

constexpr size_t SV_LDS_MAX = 40 * 1024;   // generator values kept in LDS up to this

// ---------------------------------------------------------------- the traces of one step
// Y_n is formed in the state's layout (lane = column a) and parked in LDS by columns; thread
// (a, part) of an instance then weighs the entries Y_ja that the generators' row a meets,
// every PARTS-th of them.
template <int D>
struct TraceShape {
    static constexpr int NT = RC<D>::COL ? D : 64 * RC<D>::W;   // threads per instance
    static constexpr int PARTS = NT / D;
};

// the generators' row pattern: columns [d][w] and values [K][d][w] in LDS, or (sv null) in
// global memory; w = 0: no pattern, every entry of the FP32 generators
struct TraceView {
    const TView& tv;
    const double2* sv;
    const int* sc;
    int drift;
};

// exp(-i psi (g_a - g_j)) for the channel's phase: hp = exp(i psi / 2) with half-integer
// generators, (psi, 0) otherwise
template <int PH>
__device__ __forceinline__ double2 trace_phase(const TView& tv, int k, int D, int a, int j, double2 hp) {
    if constexpr (PH == 1) {
        const int m = tv.g2[k * D + a] - tv.g2[k * D + j];
        return zpowx(zconj(hp), m);
    } else {
        return expmi(hp.x * (tv.g[k * D + a] - tv.g[k * D + j]));
    }
}

// y = conj of rows of LH (in the layout of a right operand) from LDS: L = LH^dag
template <int D>
__device__ __forceinline__ void load_l_lds(float2 (&y)[RC<D>::NR], const float2* Ll, int lane, int wave) {
    const int col = reg_col<D>(lane, wave);
    if constexpr (RC<D>::COL && D > 2) {
#pragma unroll
        for (int r = 0; r < D; r += 2) {
            const float4 w = *reinterpret_cast<const float4*>(Ll + col * RC<D>::LD + r);
            y[r] = make_float2(w.x, -w.y);
            y[r + 1] = make_float2(w.z, -w.w);
        }
    } else {
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) y[r] = cconj(Ll[col * RC<D>::LD + reg_row<D>(r, lane)]);
    }
}

// Y (this lane's part, its column col) into LDS by columns
template <int D>
__device__ __forceinline__ void park_y(const float2 (&y)[RC<D>::NR], float2* Yl, int lane, int wave) {
    const int col = reg_col<D>(lane, wave);
    if constexpr (RC<D>::COL && D > 2) {
#pragma unroll
        for (int r = 0; r < D; r += 2)
            *reinterpret_cast<float4*>(Yl + col * RC<D>::LD + r) = make_float4(y[r].x, y[r].y, y[r + 1].x, y[r + 1].y);
    } else {
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) Yl[col * RC<D>::LD + reg_row<D>(r, lane)] = y[r];
    }
}

// Traces T1 = Tr(S^psi Y), T2 = Tr(S^{pi/2} Y) (phased channels at the origin) and
// D = Tr(G Y) of every channel in FP64, this thread's share: emit(k, origin, v6) gets T1, T2, D.
template <int D, int PH, class Code, class Phase, class Emit>
__device__ __forceinline__ void trace_step(const TraceView& v, const float2* Yl, int li, Code code, Phase phase,
                                           Emit emit) {
    using C = RC<D>;
    constexpr int PARTS = TraceShape<D>::PARTS;
    constexpr bool PHASED = kind_phased(PH);
    const TView& tv = v.tv;
    const double2 hq = PH == 1 ? make_double2(0.70710678118654752, 0.70710678118654752)
                               : make_double2(1.5707963267948966, 0.0);
    const int a = li % D, part = li / D, sw = tv.spw, ne = sw ? sw : D;
    const float2* ya = Yl + a * C::LD;
    for (int k = 0; k < tv.K; ++k) {
        double o[6] = {0, 0, 0, 0, 0, 0};
        const bool origin = PHASED && code(k) == 0;
        const double2 hp = PHASED ? phase(k) : make_double2(1.0, 0.0);
        for (int e = part; e < ne; e += PARTS) {
            double2 s;
            int j;
            if (sw) {
                const int at = (k * D + a) * sw + e;
                s = v.sv ? v.sv[at] : tv.spv[at];
                j = v.sv ? v.sc[a * sw + e] : tv.spc[a * sw + e];
            } else {
                const float2 s32 = tv.S[((long long)k * D + a) * D + e];
                s = make_double2(s32.x, s32.y);
                j = e;
            }
            if (s.x == 0.0 && s.y == 0.0) continue;
            const float2 y = ya[j];
            const double yr = y.x, yi = y.y;
            if (tv.strang) s = zmulx(expmi(0.5 * tv.dt * (tv.h[v.drift * D + a] - tv.h[v.drift * D + j])), s);
            double2 w = s;
            if constexpr (PHASED) {
                if (!origin) w = zmulx(trace_phase<PH>(tv, k, D, a, j, hp), s);
            }
            o[0] = fma(w.x, yr, fma(-w.y, yi, o[0]));
            o[1] = fma(w.x, yi, fma(w.y, yr, o[1]));
            if constexpr (PHASED) {
                if (origin) {
                    w = zmulx(trace_phase<PH>(tv, k, D, a, j, hq), s);
                    o[2] = fma(w.x, yr, fma(-w.y, yi, o[2]));
                    o[3] = fma(w.x, yi, fma(w.y, yr, o[3]));
                }
            }
        }
        if constexpr (PHASED) {
            if (part == 0) {
                const double ga = tv.g[k * D + a];
                o[4] = ga * ya[a].x;
                o[5] = ga * ya[a].y;
            }
        }
        emit(k, origin, o);
    }
}

// cos and sin of the channel's phase from what Steps keeps of it
template <int PH>
__device__ __forceinline__ double2 cos_sin(double2 ro) {
    if constexpr (PH == 1) return make_double2(ro.x * ro.x - ro.y * ro.y, 2.0 * ro.x * ro.y);
    return make_double2(cos(ro.x), sin(ro.x));
}

// ---------------------------------------------------------------- one launch for everything
struct Pending {   // the traces of a step whose gradient waits for D of the earlier state
    double t1r, t1i, t2r, t2i, dr, di, c, s, om;
};

template <int D, int PH>
struct GrapeLds {   // byte offsets of the dynamic LDS of a workgroup
    size_t steps, x, l, pend, sum, sv, sc, total;
    bool sv_lds;
    __host__ __device__ GrapeLds(int K, int rep, int spw) {
        using C = RC<D>;
        const size_t mat = (size_t)C::IPW * D * C::LD * sizeof(float2);
        steps = 0;
        x = (C::W * Steps<D, PH>::lds_bytes(K, rep) + 15) & ~size_t(15);
        l = x + mat;
        pend = (l + mat + 15) & ~size_t(15);
        sum = pend + (size_t)C::IPW / rep * K * sizeof(Pending);
        sv = (sum + (size_t)C::IPW / rep * K * 6 * C::W * sizeof(double) + 15) & ~size_t(15);
        const size_t svb = (size_t)K * D * spw * sizeof(double2);
        sv_lds = spw && RC<D>::COL && svb <= SV_LDS_MAX;
        sc = sv + (sv_lds ? svb : 0);
        total = sc + (sv_lds ? (size_t)D * spw * sizeof(int) : 0);
    }
};

// a lane's part of a state in the scan's own order (d <= 16: columns, 16-byte words)
template <int D>
__device__ __forceinline__ void keep_state(const float2 (&x)[RC<D>::NR], float2* dst, int lane) {
    if constexpr (RC<D>::COL) {
        float4* p = reinterpret_cast<float4*>(dst + lane % D * D);
#pragma unroll
        for (int r = 0; r < D; r += 2) p[r / 2] = make_float4(x[r].x, x[r].y, x[r + 1].x, x[r + 1].y);
    } else {
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) dst[r * RC<D>::THREADS + threadIdx.x] = x[r];
    }
}
template <int D>
__device__ __forceinline__ void fetch_state(float2 (&x)[RC<D>::NR], const float2* src, int lane) {
    if constexpr (RC<D>::COL) {
#pragma unroll
        for (int r = 0; r < D; r += 2) {
            const float4 w = gld4(src + lane % D * D + r);
            x[r] = make_float2(w.x, w.y);
            x[r + 1] = make_float2(w.z, w.w);
        }
    } else {
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) x[r] = gld2(src + r * RC<D>::THREADS + threadIdx.x);
    }
}

template <int D, int PH, int SC>
__global__ __launch_bounds__(RC<D>::THREADS, RC<D>::COL ? 2 : 1) void grape_kernel(TView tv_in, SmallGrapeArgs a, int rep) {
    using C = RC<D>;
    constexpr bool PHASED = kind_phased(PH);
    constexpr int KK = PHASED ? 2 : 1;
    constexpr int UG = D <= 4 ? 2 : 1, SU = SC <= UG ? SC : 0;   // ring of the scans
    TView tv = tv_in;
    tv.phased = PHASED;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ double red[C::W];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane / C::LPI, ipw = C::IPW / rep, inst = grp % ipw;
    const int b = blockIdx.x * ipw + inst;
    const bool valid = b < a.B, first = valid && grp < ipw;
    const int len = valid ? (a.n_steps ? a.n_steps[b] : a.N_max) : 0;
    int N = len;
    if constexpr (RC<D>::COL) {
#pragma unroll
        for (int off = 32; off >= C::LPI; off >>= 1) N = max(N, __shfl_xor(N, off, 64));
    }
    N = __builtin_amdgcn_readfirstlane(N);
    const bool ragged = RC<D>::COL && a.n_steps;
    const GrapeLds<D, PH> lay(tv.K, rep, tv.spw);
    float2* Xl = reinterpret_cast<float2*>(lds + lay.x) + grp * D * C::LD;
    float2* Ll = reinterpret_cast<float2*>(lds + lay.l) + grp * D * C::LD;
    Pending* pend = reinterpret_cast<Pending*>(lds + lay.pend) + inst * tv.K;
    double* sums = reinterpret_cast<double*>(lds + lay.sum) + inst * tv.K * 6 * C::W;   // [k][6][W]
    double2* svl = reinterpret_cast<double2*>(lds + lay.sv);
    int* scl = reinterpret_cast<int*>(lds + lay.sc);
    if (lay.sv_lds) {
        for (int e = threadIdx.x; e < tv.K * D * tv.spw; e += C::THREADS) svl[e] = tv.spv[e];
        for (int e = threadIdx.x; e < D * tv.spw; e += C::THREADS) scl[e] = tv.spc[e];
        __syncthreads();
    }
    const int bs = valid ? b : 0, drift = (a.drift0 + bs) % tv.n_drift;
    const long long ustride = (long long)tv.K * KK;
    // threads of the instance: those of one lane group (d <= 8), or all
    const int li = RC<D>::COL ? lane % D : (int)threadIdx.x;
    Steps<D, PH> st(tv, lds + wave * Steps<D, PH>::lds_bytes(tv.K, rep), a.u + (long long)bs * a.N_max * ustride, len,
                    drift, lane, inst, grp / ipw * C::LPI + lane % C::LPI, rep, wave == 0);
    float2 dph[C::NR];
    if constexpr (!PHASED) drift_rows<D>(tv, drift, lane, dph);
    const int Cn = a.checkpoint_every;
    const bool whole = Cn >= a.N_max;   // one segment holds every state: nothing is recomputed
    auto kept = [&](float2* base, int n) __attribute__((always_inline)) {
        return base + ((long long)n * a.B + bs) * D * D;
    };

    // ---- forward
    float2 x[C::NR];
    identity_state<D>(x, lane, wave);
    walk<D, PH, 1, UG, SU>(
        x, st, 0, N, drift, ragged, dph,
        [&](int n) __attribute__((always_inline)) {
            if (!whole && n % Cn == 0 && first && n < len) keep_state<D>(x, kept(a.ckpt, n / Cn), lane);
        },
        [&](int n) __attribute__((always_inline)) {
            if (whole && first && n < len) keep_state<D>(x, kept(a.seg, n), lane);
        });
    st.report = false;
    // ---- overlap g = Tr(U_f^dag X_N) / Tr(U_f^dag U_f)
    const float2* Uf = a.U_target + (long long)bs * D * D;
    float2 l[C::NR];
    load_state<D>(l, Uf, D, lane, wave);
    double gr = 0.0, gi = 0.0, nu = 0.0;
#pragma unroll
    for (int r = 0; r < C::NR; ++r) {
        gr += (double)l[r].x * x[r].x + (double)l[r].y * x[r].y;
        gi += (double)l[r].x * x[r].y - (double)l[r].y * x[r].x;
        nu += (double)l[r].x * l[r].x + (double)l[r].y * l[r].y;
    }
    gr = inst_sum<D>(gr, red);
    gi = inst_sum<D>(gi, red);
    nu = inst_sum<D>(nu, red);
    gr /= nu;
    gi /= nu;
    if (first && st.lt == 0 && wave == 0) {
        a.fidelity[b] = gr * gr + gi * gi;
        if (a.overlap) a.overlap[b] = make_double2(gr, gi);
    }
    const double scale = 2.0 / nu;   // dF = 2 Re(conj(g) dg) with the 1/nu of g folded in
    float* gb = a.grad + (long long)bs * a.N_max * ustride;
    if (first)   // steps past this instance's length
        for (long long e = (long long)len * ustride + li; e < (long long)a.N_max * ustride; e += TraceShape<D>::NT)
            gb[e] = 0.f;
    auto im_gc = [&](double zr, double zi) { return gr * zi - gi * zr; };   // Im(conj(g) z)
    // gradient of channel k of step s from its traces and D of the earlier state
    auto finalize = [&](int s, int k, const Pending& p, double Dr, double Di) {
        float* o = gb + (long long)s * ustride + KK * k;
        const double dFo = scale * tv.dt * im_gc(p.t1r, p.t1i);
        if constexpr (!PHASED) {
            o[0] = (float)dFo;
        } else if (p.om == 0.0) {
            o[0] = (float)dFo;
            o[1] = (float)(scale * tv.dt * im_gc(p.t2r, p.t2i));
        } else {
            const double dFp = scale * im_gc(p.dr - Dr, p.di - Di);
            o[0] = (float)(p.c * dFo - p.s * dFp / p.om);
            o[1] = (float)(p.s * dFo + p.c * dFp / p.om);
        }
    };
    // ---- backward
    const TraceView tview{tv, lay.sv_lds ? svl : nullptr, scl, drift};
    const int nseg = whole ? 1 : (N + Cn - 1) / Cn;
    for (int sg = nseg - 1; sg >= 0; --sg) {
        const int s0 = whole ? 0 : sg * Cn, s1 = whole ? N : min(N, s0 + Cn);
        if (!whole) {
            if (valid && s0 < len) fetch_state<D>(x, kept(a.ckpt, sg), lane);
            walk<D, PH, 1, UG, SU>(
                x, st, s0, s1, drift, ragged, dph, [](int) {},
                [&](int n) __attribute__((always_inline)) {
                    if (first && n < len) keep_state<D>(x, kept(a.seg, n - s0), lane);
                });
        }
        // what this instance has kept is read by its own lanes, and by those of the other lane
        // groups and waves that hold it
        if (rep > 1) __threadfence();
        float2 xs[C::NR];
        fetch_state<D>(xs, kept(a.seg, min(s1, max(len, s0 + 1)) - 1 - s0), lane);
        walk<D, PH, -1, UG, SU>(
            l, st, s0, s1, drift, ragged, dph,
            [&](int s) __attribute__((always_inline)) {
                const bool active = valid && s < len;
                inst_sync<D>();
                store_state<D>(xs, Xl, C::LD, lane, wave);
                store_state<D>(l, Ll, C::LD, lane, wave);
                inst_sync<D>();
                if (s > s0 && s <= len) fetch_state<D>(xs, kept(a.seg, s - 1 - s0), lane);
                Frag<D> xf[C::NP];
                float2 y[C::NR];
#pragma unroll
                for (int p = 0; p < C::NP; ++p) load_piece_lds<D>(xf[p], Xl, p, lane);
                load_l_lds<D>(y, Ll, lane, wave);
                mul_full<D>(y, xf, 1.f);
                inst_sync<D>();
                park_y<D>(y, Xl, lane, wave);
                inst_sync<D>();
                trace_step<D, PH>(
                    tview, Xl, li, [&](int k) { return st.code(s, k); }, [&](int k) { return st.phase(s, k); },
                    [&](int k, bool origin, double (&v)[6]) __attribute__((always_inline)) {
                        const bool t2 = PHASED && __any(origin);
#pragma unroll
                        for (int j = 0; j < 6; ++j) {
                            if ((!PHASED && j >= 2) || ((j == 2 || j == 3) && !t2)) continue;
                            v[j] = lane_sum<D>(v[j]);
                        }
                        if (lane % C::LPI == 0)
#pragma unroll
                            for (int j = 0; j < 6; ++j) sums[(k * 6 + j) * C::W + wave] = v[j];
                    });
                inst_sync<D>();
                if (active) {
                    for (int k = li; k < tv.K; k += TraceShape<D>::NT) {
                        double v[6];
#pragma unroll
                        for (int j = 0; j < 6; ++j) {
                            v[j] = sums[(k * 6 + j) * C::W];
#pragma unroll
                            for (int w = 1; w < C::W; ++w) v[j] += sums[(k * 6 + j) * C::W + w];
                        }
                        if (s + 1 < len && first) finalize(s + 1, k, pend[k], v[4], v[5]);
                        Pending p;
                        p.t1r = v[0], p.t1i = v[1], p.t2r = v[2], p.t2i = v[3], p.dr = v[4], p.di = v[5];
                        p.c = p.s = p.om = 0.0;
                        if constexpr (PHASED) {
                            const double2 cs = cos_sin<PH>(st.phase(s, k));
                            p.c = cs.x;
                            p.s = cs.y;
                            p.om = st.code(s, k) * tv.eps;
                        }
                        pend[k] = p;
                    }
                }
            },
            [](int) {});
    }
    // D_0 = Tr(G Y_0), Y_0 = X_0 L_0 = L_0
    inst_sync<D>();
    for (int k = 0; k < tv.K; ++k) {
        double dr = 0.0, di = 0.0;
        if constexpr (PHASED) {
            const int col = reg_col<D>(lane, wave);
            const double ga = tv.g[k * D + col];
#pragma unroll
            for (int r = 0; r < C::NR; ++r)
                if (reg_row<D>(r, lane) == col) {
                    dr += ga * l[r].x;
                    di -= ga * l[r].y;
                }
            dr = inst_sum<D>(dr, red);
            di = inst_sum<D>(di, red);
        }
        if (first && len > 0 && li == k % TraceShape<D>::NT) finalize(0, k, pend[k], dr, di);
    }
}

// ---------------------------------------------------------------- the two chains side by side
// steps in flight ahead of the current product: their propagators come from HBM or the
// memory-side cache, and a product takes 64 to 256 matrix-core instructions
template <int D>
constexpr int scan_ring() {
    return D == 8 ? 4 : D <= 32 ? 2 : 1;
}

// N: the longest instance of the wave; len, out: this lane's instance
template <int D, int DIR>
__device__ __forceinline__ void scan_products(float2 (&x)[RC<D>::NR], const float2* Up, int len, int N, float2* out,
                                              bool store, int lane, int wave) {
    constexpr int U = scan_ring<D>();
    constexpr bool ADJ = DIR < 0;
    const int mat = D * D;
    Ahead<D, U> a;
    auto slot = [&](int i) __attribute__((always_inline)) {   // i-th step in the order of travel
        const int n = ADJ ? max(len - 1 - i, 0) : min(i, max(len - 1, 0));
        return Slot{Up + (long long)n * mat, ADJ ? -1.f : 1.f, i < len, ADJ};
    };
#pragma unroll
    for (int i = 0; i < U; ++i) fetch_slot<D, U>(a, i, slot(i), lane);
    for (int i0 = 0; i0 < N; i0 += U) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (i0 + i < N) {
                apply_slot<D, U, ADJ>(x, a, i, slot(i0 + i + U), lane);
                const int n = ADJ ? len - 1 - i0 - i : i0 + i;   // LH_n, or X_{n+1}
                if (store && i0 + i < len) store_state<D>(x, out + (long long)n * mat, D, lane, wave);
            }
        }
    }
}

// blockIdx.y 0: X_{n+1} = U_n X_n from the identity; 1: LH_n = U_n^dag LH_{n+1} from U_f.
// rep: lane groups per instance (d <= 16)
template <int D>
__global__ __launch_bounds__(RC<D>::THREADS, 1) void scan_kernel(ScanArgs a, int rep) {
    using C = RC<D>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane / C::LPI, ipw = C::IPW / rep;
    const int bi = blockIdx.x * ipw + grp % ipw, b = min(bi, a.B - 1);
    const bool store = bi < a.B && grp < ipw;
    const int len = a.n_steps ? a.n_steps[b] : a.N_max;
    int N = len;
    if constexpr (C::COL) {
#pragma unroll
        for (int off = 32; off >= C::LPI; off >>= 1) N = max(N, __shfl_xor(N, off, 64));
    }
    N = __builtin_amdgcn_readfirstlane(N);
    const long long mat = D * D;
    const float2* Up = a.Up + (long long)b * a.N_max * mat;
    float2 x[C::NR];
    if (blockIdx.y == 0) {
        float2* X = a.X + (long long)b * a.N_max * mat;
        identity_state<D>(x, lane, wave);
        scan_products<D, 1>(x, Up, len, N, X, store, lane, wave);
        if (store && len < a.N_max) store_state<D>(x, X + (a.N_max - 1) * mat, D, lane, wave);
    } else {
        float2* LH = a.LH + (long long)b * (a.N_max + 1) * mat;
        load_state<D>(x, a.U_target + b * mat, D, lane, wave);
        if (store) store_state<D>(x, LH + len * mat, D, lane, wave);
        scan_products<D, -1>(x, Up, len, N, LH, store, lane, wave);
    }
}

// the same on the factors: steps of one factor each need no composition
// (d = 32, 64: one instance per workgroup)
template <int D, int PH>
__global__ __launch_bounds__(RC<D>::THREADS, 1) void scan_factor_kernel(TView tv_in, ScanArgs a) {
    using C = RC<D>;
    constexpr int KK = kind_phased(PH) ? 2 : 1;
    TView tv = tv_in;
    tv.phased = kind_phased(PH);
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, b = blockIdx.x;
    const int len = a.n_steps ? a.n_steps[b] : a.N_max;
    const long long mat = D * D;
    const int drift = (a.drift0 + b) % tv.n_drift;
    Steps<D, PH> st(tv, lds + wave * Steps<D, PH>::lds_bytes(tv.K, 1), a.u + (long long)b * a.N_max * tv.K * KK, len,
                    drift, lane, 0, lane, 1, false);
    float2 x[C::NR], dph[C::NR];
    if constexpr (!kind_phased(PH)) drift_rows<D>(tv, drift, lane, dph);
    if (blockIdx.y == 0) {
        float2* X = a.X + (long long)b * a.N_max * mat;
        identity_state<D>(x, lane, wave);
        walk<D, PH, 1, C::U, 1>(x, st, 0, len, drift, false, dph, [](int) {},
                                [&](int n) __attribute__((always_inline)) {
                                    store_state<D>(x, X + n * mat, D, lane, wave);
                                });
        if (len < a.N_max) store_state<D>(x, X + (a.N_max - 1) * mat, D, lane, wave);
    } else {
        float2* LH = a.LH + (long long)b * (a.N_max + 1) * mat;
        load_state<D>(x, a.U_target + b * mat, D, lane, wave);
        store_state<D>(x, LH + len * mat, D, lane, wave);
        walk<D, PH, -1, C::U, 1>(x, st, 0, len, drift, false, dph, [](int) {},
                                 [&](int n) __attribute__((always_inline)) {
                                     store_state<D>(x, LH + n * mat, D, lane, wave);
                                 });
    }
}

// ---------------------------------------------------------------- traces of every step
constexpr int TRACE_STEPS = 8;   // steps a workgroup takes, the next one's states on their way

template <int D>
struct TraceLds {
    size_t x, l, sum, sv, sc, total;
    bool sv_lds;
    __host__ __device__ TraceLds(int K, int spw) {
        using C = RC<D>;
        const size_t mat = (size_t)C::IPW * D * C::LD * sizeof(float2);
        x = 0;
        l = x + mat;
        sum = (l + (C::COL ? 0 : mat) + 15) & ~size_t(15);
        sv = (sum + (size_t)C::IPW * K * 6 * C::W * sizeof(double) + 15) & ~size_t(15);
        const size_t svb = (size_t)K * D * spw * sizeof(double2);
        sv_lds = spw && svb <= SV_LDS_MAX;
        sc = sv + (sv_lds ? svb : 0);
        total = sc + (sv_lds ? (size_t)D * spw * sizeof(int) : 0);
    }
};

// d <= 16: a wave takes IPW consecutive steps of one instance at a time, one per lane group, and
// their operands come straight from memory (rows of X as the left operand, rows of LH as the
// columns of L); d = 32, 64: one step at a time, both through LDS.
template <int D, int PH>
__global__ __launch_bounds__(RC<D>::THREADS, 1) void trace_kernel(TView tv_in, TraceArgs a) {
    using C = RC<D>;
    constexpr bool PHASED = kind_phased(PH);
    constexpr int KK = PHASED ? 2 : 1, G = C::COL ? C::IPW : 1;   // steps at a time
    TView tv = tv_in;
    tv.phased = PHASED;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ int hq[G * KMAX];
    __shared__ double2 hr[G * KMAX];
    const TraceLds<D> lay(tv.K, tv.spw);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.y;
    const int grp = C::COL ? lane / C::LPI : 0, li = C::COL ? lane % C::LPI : tid;
    float2* Xl = reinterpret_cast<float2*>(lds + lay.x) + grp * D * C::LD;
    float2* Ll = reinterpret_cast<float2*>(lds + lay.l);
    double* sums = reinterpret_cast<double*>(lds + lay.sum) + grp * tv.K * 6 * C::W;
    double2* svl = reinterpret_cast<double2*>(lds + lay.sv);
    int* scl = reinterpret_cast<int*>(lds + lay.sc);
    const int len = a.n_steps ? a.n_steps[b] : a.N_max;
    const int s0 = blockIdx.x * TRACE_STEPS * G, s1 = min(len, s0 + TRACE_STEPS * G);
    if (s0 >= s1) return;
    if (lay.sv_lds) {
        for (int e = tid; e < tv.K * D * tv.spw; e += C::THREADS) svl[e] = tv.spv[e];
        for (int e = tid; e < D * tv.spw; e += C::THREADS) scl[e] = tv.spc[e];
        __syncthreads();
    }
    const TraceView tview{tv, lay.sv_lds ? svl : nullptr, scl, (a.drift0 + b) % tv.n_drift};
    const long long mat = D * D;
    const float2* X = a.X + (long long)b * a.N_max * mat;
    const float2* LH = a.LH + (long long)b * (a.N_max + 1) * mat;
    constexpr int NV = C::COL ? 1 : D * D / 2 / C::THREADS;   // 16-byte words of a state per thread
    float4 xv[NV], lv[NV];
    Frag<D> xf[C::NP];
    float2 y[C::NR];
    auto fetch = [&](int sb) __attribute__((always_inline)) {
        if constexpr (C::COL) {
            const int s = min(sb + grp, s1 - 1);
            load_piece<D>(xf[0], X + s * mat, false, 0, lane);
#pragma unroll
            for (int r = 0; r < D; r += 2) {
                const float4 w = gld4(LH + (s + 1) * mat + li * D + r);
                y[r] = make_float2(w.x, -w.y);
                y[r + 1] = make_float2(w.z, -w.w);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                xv[i] = gld4(X + sb * mat + 2 * (tid + C::THREADS * i));
                lv[i] = gld4(LH + (sb + 1) * mat + 2 * (tid + C::THREADS * i));
            }
        }
    };
    fetch(s0);
    for (int sb = s0; sb < s1; sb += G) {
        const int s = sb + grp;
        const bool live = s < s1;
        if constexpr (!C::COL) {
            inst_sync<D>();
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int e = 2 * (tid + C::THREADS * i), at = e / D * C::LD + e % D;
                Xl[at] = make_float2(xv[i].x, xv[i].y);
                Xl[at + 1] = make_float2(xv[i].z, xv[i].w);
                Ll[at] = make_float2(lv[i].x, lv[i].y);
                Ll[at + 1] = make_float2(lv[i].z, lv[i].w);
            }
        }
        if constexpr (PHASED) {
            for (int e = tid; e < G * tv.K; e += C::THREADS) {   // codes and phases of these steps
                const int sg = min(sb + e / tv.K, s1 - 1), k = e % tv.K;
                const float* up = a.u + (((long long)b * a.N_max + sg) * tv.K + k) * KK;
                double2 ro;
                hq[e] = quantise_reg<PH>((double)up[0], (double)up[1], tv.eps, tv.qmax, ro, nullptr);
                hr[e] = ro;
            }
        }
        inst_sync<D>();
        if constexpr (!C::COL) {
#pragma unroll
            for (int p = 0; p < C::NP; ++p) load_piece_lds<D>(xf[p], Xl, p, lane);
            load_l_lds<D>(y, Ll, lane, wave);
        }
        float2 yy[C::NR];
#pragma unroll
        for (int r = 0; r < C::NR; ++r) yy[r] = y[r];
        mul_full<D>(yy, xf, 1.f);
        inst_sync<D>();
        park_y<D>(yy, Xl, lane, wave);
        inst_sync<D>();
        if (sb + G < s1) fetch(sb + G);
        trace_step<D, PH>(
            tview, Xl, li, [&](int k) { return hq[grp * tv.K + k]; }, [&](int k) { return hr[grp * tv.K + k]; },
            [&](int k, bool origin, double (&v)[6]) __attribute__((always_inline)) {
                const bool t2 = PHASED && __any(origin);
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    if ((!PHASED && j >= 2) || ((j == 2 || j == 3) && !t2)) continue;
                    v[j] = lane_sum<D>(v[j]);
                }
                if (lane % C::LPI == 0)
#pragma unroll
                    for (int j = 0; j < 6; ++j) sums[(k * 6 + j) * C::W + wave] = v[j];
            });
        inst_sync<D>();
        if (live) {
            double* out = a.tr + ((long long)b * a.N_max + s) * tv.K * 6;
            for (int e = li; e < tv.K * 6; e += TraceShape<D>::NT) {
                double t = sums[e * C::W];
#pragma unroll
                for (int w = 1; w < C::W; ++w) t += sums[e * C::W + w];
                out[e] = t;
            }
        }
    }
}

// ---------------------------------------------------------------- launches
template <int D>
int grape_lane_groups(int B) {   // as the chain's
    int rep = 1;
    if constexpr (RC<D>::COL)
        while (2 * rep <= RC<D>::IPW && (long long)B * 2 * rep <= 1024LL * RC<D>::IPW) rep *= 2;
    return rep;
}

template <int D, int PH, int SC>
hipError_t launch_fused(const TView& tv, const SmallGrapeArgs& a, hipStream_t st) {
    using C = RC<D>;
    const int rep = grape_lane_groups<D>(a.B);
    const GrapeLds<D, PH> lay(tv.K, rep, tv.spw);
    const void* k = (const void*)grape_kernel<D, PH, SC>;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lay.total);
    if (e != hipSuccess) return e;
    const int ipw = C::IPW / rep;
    hipLaunchKernelGGL((grape_kernel<D, PH, SC>), dim3((a.B + ipw - 1) / ipw), dim3(C::THREADS), lay.total, st, tv, a, rep);
    return hipGetLastError();
}
template <int D, int PH>
hipError_t launch_fused_slots(const TView& tv, const SmallGrapeArgs& a, hipStream_t st) {
    if constexpr (D == 4 && PH <= 1) {
        if (tv.cache && tv.K == 1) return launch_fused<D, PH, 1>(tv, a, st);
        if (tv.cache && tv.K == 2) return launch_fused<D, PH, 2>(tv, a, st);
    }
    if constexpr (D == 8 && PH <= 1) {
        if (tv.cache && tv.K == 1) return launch_fused<D, PH, 1>(tv, a, st);
    }
    return launch_fused<D, PH, 0>(tv, a, st);
}
template <int D>
hipError_t launch_fused_kind(const TView& tv, const SmallGrapeArgs& a, hipStream_t st) {
    switch (step_kind(tv)) {
        case 0: return launch_fused_slots<D, 0>(tv, a, st);
        case 1: return launch_fused_slots<D, 1>(tv, a, st);
        case 2: return launch_fused_slots<D, 2>(tv, a, st);
        default: return launch_fused_slots<D, 3>(tv, a, st);
    }
}

template <int D, int PH>
hipError_t launch_trace(const TView& tv, const TraceArgs& a, hipStream_t st) {
    constexpr int G = TRACE_STEPS * (RC<D>::COL ? RC<D>::IPW : 1);
    const TraceLds<D> lay(tv.K, tv.spw);
    const void* k = (const void*)trace_kernel<D, PH>;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lay.total);
    if (e != hipSuccess) return e;
    for (int b0 = 0; b0 < a.B; b0 += 65535) {   // grid.y
        TraceArgs p = a;
        p.B = std::min(a.B - b0, 65535);
        p.drift0 = (a.drift0 + b0) % tv.n_drift;
        p.u += (long long)b0 * a.N_max * tv.K * (tv.phased ? 2 : 1);
        if (a.n_steps) p.n_steps += b0;
        p.X += (long long)b0 * a.N_max * D * D;
        p.LH += (long long)b0 * (a.N_max + 1) * D * D;
        p.tr += (long long)b0 * a.N_max * tv.K * 6;
        hipLaunchKernelGGL((trace_kernel<D, PH>), dim3((a.N_max + G - 1) / G, p.B), dim3(RC<D>::THREADS), lay.total, st, tv,
                           p);
    }
    return hipGetLastError();
}
template <int D>
hipError_t launch_trace_kind(const TView& tv, const TraceArgs& a, hipStream_t st) {
    switch (step_kind(tv)) {
        case 0: return launch_trace<D, 0>(tv, a, st);
        case 1: return launch_trace<D, 1>(tv, a, st);
        case 2: return launch_trace<D, 2>(tv, a, st);
        default: return launch_trace<D, 3>(tv, a, st);
    }
}

template <int D, int PH>
hipError_t launch_scan_factor(const TView& tv, const ScanArgs& a, hipStream_t st) {
    const size_t bytes = RC<D>::W * Steps<D, PH>::lds_bytes(tv.K, 1);
    const void* k = (const void*)scan_factor_kernel<D, PH>;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((scan_factor_kernel<D, PH>), dim3(a.B, 2), dim3(RC<D>::THREADS), bytes, st, tv, a);
    return hipGetLastError();
}
template <int D>
hipError_t launch_scan(const TView& tv, const ScanArgs& a, hipStream_t st) {
    if constexpr (!RC<D>::COL) {
        if (!a.Up) return tv.phased ? launch_scan_factor<D, 1>(tv, a, st) : launch_scan_factor<D, 0>(tv, a, st);
    }
    const int rep = grape_lane_groups<D>(2 * a.B), ipw = RC<D>::IPW / rep;
    hipLaunchKernelGGL(scan_kernel<D>, dim3((a.B + ipw - 1) / ipw, 2), dim3(RC<D>::THREADS), 0, st, a, rep);
    return hipGetLastError();
}

}  // namespace
#endif
}  // namespace redo
