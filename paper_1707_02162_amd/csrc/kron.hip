// Structure-aware chain (a competitor of the dense REDO factors, not the paper's
// method): when d = 2^n and every control generator is a sum of single-spin
// terms, S_k = sum_q s_kq, the factors of one step factorise over the spins,
//     exp(-i theta S_k) = (x)_q exp(-i theta s_kq),
// and the step of Sec. III (Eq. propUn, split form U_n = Z (prod_k R_k) Z^dag V)
// becomes a row scaling, one 2 x 2 unitary per spin, and a row scaling:
//     U_n X = post (.) [ (x)_q g_q ] (pre (.) X),   g_q = prod_k exp(-i theta_k s_kq),
// with pre = Z^dag V and post = Z (Strang: pre = Z^dag V(dt/2), post = V(dt/2) Z).
// theta_k = dt times the REDO-quantised amplitude (Sec. II, Eq. cgrain) or the
// amplitude as given.  Cost per step and instance O(n d^2) instead of O(d^3).
#include "large_path.h"
#include "redo_internal.h"

namespace redo {
namespace {

constexpr int KRON_NT = 512;
constexpr int KRON_VB = 4;                  // row bits held in registers per round
constexpr int KRON_VALS = 1 << KRON_VB;     // values per thread

// per instance and step: the spins' 2 x 2 factors in FP64 (rounded once to FP32) and
// the two diagonal row scalings
struct KronPlanArgs {
    const double2* s;     // [K][n][4] single-spin generators
    const double* h;      // [n_drift][d] diagonal drifts
    const double* g;      // [K][d] phase generators (phased) or null
    const int* codes;     // [B][N][K] (quantised) or null
    const double* phi;    // [B][N][K] (quantised, phased) or null
    const float* u;       // amplitudes (unquantised) or null
    const int* n_steps;
    float2* gates;        // [B][n][4]
    float2* pre;          // [B][d]
    float2* post;         // [B][d]
    double eps, dt;
    int n, d, K, N, n_drift, phased, strang, step;
};

// exp(-i theta s) for a Hermitian 2 x 2 s = a0 I + ax X + ay Y + az Z:
// e^{-i theta a0} (cos(theta r) I - i sin(theta r) (a . sigma) / r), r = |a|
__device__ inline void exp2x2(const double2* s, double theta, double2 (&e)[4]) {
    const double a0 = 0.5 * (s[0].x + s[3].x), az = 0.5 * (s[0].x - s[3].x);
    const double ax = s[1].x, ay = -s[1].y;
    const double r = sqrt(ax * ax + ay * ay + az * az);
    double c, sn;
    sincos(theta * r, &sn, &c);
    const double f = r > 0.0 ? sn / r : theta;   // sin(theta r) / r
    const double2 ph = expmi(theta * a0);
    // M = c I - i f (a . sigma);  a . sigma = [[az, ax - i ay], [ax + i ay, -az]]
    const double2 m00 = make_double2(c, -f * az), m11 = make_double2(c, f * az);
    const double2 m01 = make_double2(-f * ay, -f * ax), m10 = make_double2(f * ay, -f * ax);
    e[0] = zmul(ph, m00);
    e[1] = zmul(ph, m01);
    e[2] = zmul(ph, m10);
    e[3] = zmul(ph, m11);
}

// channel amplitudes of one instance and step by the first K threads: theta_k = dt Omega_k (signed
// for unphased channels), phases phi_k
__device__ inline void kron_channels(const KronPlanArgs& a, long long ci, double* th, double* ph) {
    if ((int)threadIdx.x < a.K) {
        const int k = threadIdx.x;
        double om, p = 0.0;
        if (a.codes) {
            om = a.codes[ci + k] * a.eps;   // negative codes carry the sign (unphased)
            if (a.phased) p = a.phi[ci + k];
        } else if (a.phased) {
            const double ux = a.u[(ci + k) * 2], uy = a.u[(ci + k) * 2 + 1];
            om = sqrt(ux * ux + uy * uy);
            p = atan2(uy, ux);
        } else {
            om = a.u[ci + k];
        }
        th[k] = om * a.dt;
        ph[k] = p;
    }
}

// the factor of spin q, channel 0 first
__device__ inline void kron_spin_factor(const KronPlanArgs& a, int q, const double* th, double2 (&acc)[4]) {
    acc[0] = acc[3] = make_double2(1, 0);
    acc[1] = acc[2] = make_double2(0, 0);
    for (int k = 0; k < a.K; ++k) {
        double2 e[4];
        exp2x2(a.s + ((long long)k * a.n + q) * 4, th[k], e);
        const double2 n00 = zadd(zmul(e[0], acc[0]), zmul(e[1], acc[2]));
        const double2 n01 = zadd(zmul(e[0], acc[1]), zmul(e[1], acc[3]));
        const double2 n10 = zadd(zmul(e[2], acc[0]), zmul(e[3], acc[2]));
        const double2 n11 = zadd(zmul(e[2], acc[1]), zmul(e[3], acc[3]));
        acc[0] = n00, acc[1] = n01, acc[2] = n10, acc[3] = n11;
    }
}

// the row scalings before (p) and after (q) the spin factors
__device__ inline void kron_row_scalings(const KronPlanArgs& a, int b, int r, const double* ph, double2& p, double2& q) {
    double tz = 0.0;   // Z = diag(e^{-i tz})
    if (a.phased)
        for (int k = 0; k < a.K; ++k) tz += ph[k] * a.g[(long long)k * a.d + r];
    const double hd = a.dt * a.h[(long long)(b % a.n_drift) * a.d + r];
    if (a.strang) {
        p = expmi(0.5 * hd - tz);
        q = expmi(0.5 * hd + tz);
    } else {
        p = expmi(hd - tz);
        q = a.phased ? expmi(tz) : make_double2(1.0, 0.0);
    }
}

__global__ __launch_bounds__(256) void kron_plan_kernel(KronPlanArgs a) {
    const int b = blockIdx.x;
    if (a.n_steps && a.step >= a.n_steps[b]) return;
    const long long ci = ((long long)b * a.N + a.step) * a.K;
    __shared__ double th[16], ph[16];
    kron_channels(a, ci, th, ph);
    __syncthreads();
    if ((int)threadIdx.x < a.n) {
        const int q = threadIdx.x;
        double2 acc[4];
        kron_spin_factor(a, q, th, acc);
        float2* o = a.gates + ((long long)b * a.n + q) * 4;
        for (int e = 0; e < 4; ++e) o[e] = make_float2((float)acc[e].x, (float)acc[e].y);
    }
    for (int r = threadIdx.x; r < a.d; r += blockDim.x) {
        double2 p, q;
        kron_row_scalings(a, b, r, ph, p, q);
        a.pre[(long long)b * a.d + r] = make_float2((float)p.x, (float)p.y);
        a.post[(long long)b * a.d + r] = make_float2((float)q.x, (float)q.y);
    }
}

__device__ inline long long kron_xcd(long long bid, long long nb) {
    return (nb % 8 == 0) ? (bid % 8) * (nb / 8) + bid / 8 : bid;
}

// LDS row swizzle: the low KRON_VB row bits XOR the next KRON_VB (a bijection), so that
// the rows one instruction touches in any round fall into different banks
__device__ inline int kron_lds(int a, int c, int sw) { return (a ^ ((a >> KRON_VB) & (KRON_VALS - 1))) * sw + c; }

template <int D>
struct KronShape {
    static constexpr int n = D == 128 ? 7 : D == 256 ? 8 : D == 512 ? 9 : D == 1024 ? 10 : D == 2048 ? 11 : 12;
    static constexpr int SW = KRON_NT * KRON_VALS / D;   // columns per workgroup (8192 values in LDS)
    static constexpr int rounds = (n + KRON_VB - 1) / KRON_VB;
    static_assert(rounds >= 2 && rounds <= 3, "two or three register rounds");
};

// row of register value i and thread part `rest` in a round whose register bits start at lo
__device__ inline int kron_row(int rest, int i, int lo) {
    return (rest & ((1 << lo) - 1)) | (i << lo) | ((rest >> lo) << (lo + KRON_VB));
}

template <int J>
__device__ inline void kron_gate_bit(float2 (&v)[KRON_VALS], const float2* gq) {
    const float2 g00 = gq[0], g01 = gq[1], g10 = gq[2], g11 = gq[3];
#pragma unroll
    for (int i = 0; i < KRON_VALS; ++i) {
        if (i & (1 << J)) continue;
        const int i1 = i | (1 << J);
        const float2 x = v[i], y = v[i1];
        float2 r0 = make_float2(0.f, 0.f), r1 = make_float2(0.f, 0.f);
        cfma(r0, g00, x);
        cfma(r0, g01, y);
        cfma(r1, g10, x);
        cfma(r1, g11, y);
        v[i] = r0;
        v[i1] = r1;
    }
}

// register bits of round R start at row bit lo(R); round R applies spins VB R .. VB R + VB - 1
template <int D, int R>
struct KronRound {
    static constexpr int n = KronShape<D>::n, VB = KRON_VB;
    static constexpr int lo = VB * R < n - VB ? VB * R : n - VB;
    static constexpr int q0 = VB * R, q1 = VB * R + VB < n ? VB * R + VB : n;
};

template <int D, int R, int Q>
__device__ inline void kron_round_gate(float2 (&v)[KRON_VALS], const float2* gl) {
    using RR = KronRound<D, R>;
    if constexpr (RR::q0 + Q < RR::q1) kron_gate_bit<RR::q0 + Q - RR::lo>(v, gl + (RR::q0 + Q) * 4);
}

template <int D, int R>
__device__ inline void kron_round_gates(float2 (&v)[KRON_VALS], const float2* gl) {
    static_assert(KRON_VB == 4, "one call per register bit");
    kron_round_gate<D, R, 0>(v, gl);
    kron_round_gate<D, R, 1>(v, gl);
    kron_round_gate<D, R, 2>(v, gl);
    kron_round_gate<D, R, 3>(v, gl);
}

// hand the strip from the register layout of round R - 1 to that of round R through LDS
template <int D, int R>
__device__ inline void kron_exchange(float2 (&v)[KRON_VALS], float2* buf, int rest, int c) {
    constexpr int SW = KronShape<D>::SW;
#pragma unroll
    for (int i = 0; i < KRON_VALS; ++i) buf[kron_lds(kron_row(rest, i, KronRound<D, R - 1>::lo), c, SW)] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KRON_VALS; ++i) v[i] = buf[kron_lds(kron_row(rest, i, KronRound<D, R>::lo), c, SW)];
    __syncthreads();
}

// One step for every instance: workgroup = (instance, strip of SW columns).  Pass 0
// reads the strip from HBM with register bits = row bits 0..VB-1, applies the pre
// scaling and spins 0..VB-1, and parks the strip in LDS; pass r takes row bits
// lo_r .. lo_r + VB - 1 (lo_r = min(VB r, n - VB)) and applies spins VB r .. VB r + VB - 1;
// the last pass applies the post scaling and writes the strip back in place.
// 64 KiB of LDS per workgroup: two workgroups (four waves per SIMD) per CU.
template <int D>
__global__ __launch_bounds__(KRON_NT, 4) void kron_step_kernel(float2* X0, float2* X1, const int* loc,
                                                               long long xstride, const float2* __restrict__ gates,
                                                               const float2* __restrict__ pre,
                                                               const float2* __restrict__ post, const int* n_steps,
                                                               int step) {
    using S = KronShape<D>;
    constexpr int n = S::n, SW = S::SW, NSTRIP = D / SW;
    __shared__ float2 buf[KRON_NT * KRON_VALS];
    __shared__ float2 gl[n * 4];
    const long long bid = kron_xcd(blockIdx.x, gridDim.x);
    const int b = (int)(bid / NSTRIP), strip = (int)(bid % NSTRIP);
    if (n_steps && step >= n_steps[b]) return;   // uniform over the workgroup
    float2* X = ((loc && loc[b]) ? X1 : X0) + (long long)b * xstride + strip * SW;
    const int t = threadIdx.x, c = t % SW, rest = t / SW;
    if (t < n * 4) gl[t] = gates[(long long)b * n * 4 + t];
    const float2* pb = pre + (long long)b * D;
    const float2* qb = post + (long long)b * D;
    float2 v[KRON_VALS];
#pragma unroll
    for (int i = 0; i < KRON_VALS; ++i) {
        const int a = kron_row(rest, i, 0);
        v[i] = cmul(pb[a], X[(long long)a * D + c]);
    }
    __syncthreads();   // gates in LDS
    kron_round_gates<D, 0>(v, gl);
    kron_exchange<D, 1>(v, buf, rest, c);
    kron_round_gates<D, 1>(v, gl);
    if constexpr (S::rounds > 2) {
        kron_exchange<D, 2>(v, buf, rest, c);
        kron_round_gates<D, 2>(v, gl);
    }
    constexpr int flo = KronRound<D, S::rounds - 1>::lo;
#pragma unroll
    for (int i = 0; i < KRON_VALS; ++i) {
        const int a = kron_row(rest, i, flo);
        X[(long long)a * D + c] = cmul(qb[a], v[i]);
    }
}

// kron_step_kernel<1024> followed, in the same workgroup, by the observable in the right
// Walsh frame on the strip it has just written, while the strip is still in registers: the
// strip goes to the exchange buffer in the layout of the one-pass observable (16-byte
// chunks swizzled by row, mx8_off), each pair of lanes forms (M W)_aj for a row and four
// columns from the packed lists and adds D_j Re(conj(W_aj) (M W)_aj) (FP32 within a row,
// FP64 across rows); the workgroup's sum goes to partial[b][strip].  The observable's own
// read of every state disappears.
template <int WP>
__global__ __launch_bounds__(KRON_NT, 4) void kron_step_obs_kernel(float2* X0, float2* X1, const int* loc,
                                                                   long long xstride,
                                                                   const float2* __restrict__ gates,
                                                                   const float2* __restrict__ pre,
                                                                   const float2* __restrict__ post,
                                                                   const int* n_steps, int step,
                                                                   const int* __restrict__ cols,
                                                                   const float2* __restrict__ vals,
                                                                   const double* __restrict__ spec,
                                                                   double* __restrict__ partial) {
    constexpr int D = 1024;
    using S = KronShape<D>;
    constexpr int n = S::n, SW = S::SW, NSTRIP = D / SW;
    static_assert(SW == 8 && S::rounds > 2, "8-column strips, the buffer free after the last exchange");
    __shared__ float2 buf[KRON_NT * KRON_VALS];
    __shared__ float2 gl[n * 4];
    __shared__ double red[KRON_NT / 64];
    const long long bid = kron_xcd(blockIdx.x, gridDim.x);
    const int b = (int)(bid / NSTRIP), strip = (int)(bid % NSTRIP);
    if (n_steps && step >= n_steps[b]) return;   // uniform over the workgroup
    float2* X = ((loc && loc[b]) ? X1 : X0) + (long long)b * xstride + strip * SW;
    const int t = threadIdx.x, c = t % SW, rest = t / SW;
    if (t < n * 4) gl[t] = gates[(long long)b * n * 4 + t];
    const float2* pb = pre + (long long)b * D;
    const float2* qb = post + (long long)b * D;
    float2 v[KRON_VALS];
#pragma unroll
    for (int i = 0; i < KRON_VALS; ++i) {
        const int a = kron_row(rest, i, 0);
        v[i] = cmul(pb[a], X[(long long)a * D + c]);
    }
    __syncthreads();   // gates in LDS
    kron_round_gates<D, 0>(v, gl);
    kron_exchange<D, 1>(v, buf, rest, c);
    kron_round_gates<D, 1>(v, gl);
    kron_exchange<D, 2>(v, buf, rest, c);
    kron_round_gates<D, 2>(v, gl);
    constexpr int flo = KronRound<D, S::rounds - 1>::lo;
    // the last exchange ended with a barrier after its reads: the buffer is free
#pragma unroll
    for (int i = 0; i < KRON_VALS; ++i) {
        const int a = kron_row(rest, i, flo);
        const float2 y = cmul(qb[a], v[i]);
        X[(long long)a * D + c] = y;
        buf[mx8_off(a, c)] = y;
    }
    __syncthreads();
    asm volatile("" ::: "memory");   // the observable's mask loads stay below the step (register pressure)
    constexpr int LPR = 2, CPL = SW / LPR, NCH = CPL / 2, RPP = KRON_NT / LPR;
    const float4* strip4 = reinterpret_cast<const float4*>(buf);
    const int lr = t % LPR;
    float dj[CPL];
#pragma unroll
    for (int u = 0; u < CPL; ++u) dj[u] = (float)spec[strip * SW + lr * CPL + u];
    // M_ac = f(a XOR c) (the frame needs it): row a's list is row 0's with every column XORed
    // by a, so the masks and values are read once (one address for every lane), zeros skipped
    int mk[WP];
    float2 fv[WP];
    obs_list<WP>(cols, vals, 0, mk, fv);
    double sum = 0.0;
    for (int a = t / LPR; a < D; a += RPP) {
        float2 acc[CPL];
#pragma unroll
        for (int u = 0; u < CPL; ++u) acc[u] = make_float2(0.f, 0.f);
#pragma unroll
        for (int e = 0; e < WP; ++e) {
            if (fv[e].x == 0.f && fv[e].y == 0.f) continue;   // the same for every lane
            const int c = a ^ mk[e];
#pragma unroll
            for (int j = 0; j < NCH; ++j) {
                const int ch = lr * NCH + j;
                const float4 x = strip4[c * 4 + ((ch ^ (c >> 2)) & 3)];
                cfma(acc[2 * j], fv[e], make_float2(x.x, x.y));
                cfma(acc[2 * j + 1], fv[e], make_float2(x.z, x.w));
            }
            asm volatile("" ::: "memory");   // one mask's gathers at a time (register pressure)
        }
        float row = 0.f;
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const int ch = lr * NCH + j;
            const float4 wv = strip4[a * 4 + ((ch ^ (a >> 2)) & 3)];
            row += dj[2 * j] * (wv.x * acc[2 * j].x + wv.y * acc[2 * j].y) +
                   dj[2 * j + 1] * (wv.z * acc[2 * j + 1].x + wv.w * acc[2 * j + 1].y);
        }
        sum += (double)row;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if ((t & 63) == 0) red[t >> 6] = sum;
    __syncthreads();
    if (t == 0) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < KRON_NT / 64; ++w) s += red[w];
        partial[(long long)b * NSTRIP + strip] = s;
    }
}

template <int WP>
hipError_t launch_kron_step_obs(int B, float2* X0, float2* X1, const int* loc, long long xstride, const float2* gates,
                                const float2* pre, const float2* post, const int* n_steps, int step, const int* pc,
                                const float2* pv, const double* spec, double* partial, hipStream_t st) {
    constexpr int NSTRIP = 1024 / KronShape<1024>::SW;
    void* tok = nullptr;
    const bool prof = profiling_on();
    if (prof) profile_begin(st, &tok, 1);
    hipLaunchKernelGGL(kron_step_obs_kernel<WP>, dim3((unsigned)((long long)B * NSTRIP)), dim3(KRON_NT), 0, st, X0, X1,
                       loc, xstride, gates, pre, post, n_steps, step, pc, pv, spec, partial);
    if (prof) profile_end(st, tok);
    return hipGetLastError();
}

// the step and the Walsh-frame observable in one launch (d = 1024), then the per-instance sums
hipError_t kron_step_observable(int B, float2* X0, float2* X1, const int* loc, long long xstride,
                                const float2* gates, const float2* pre, const float2* post, const int* n_steps,
                                int step, int w, const int* pc, const float2* pv, const float2* vals,
                                const double* spec, double* partial, double* out, long long out_stride,
                                hipStream_t st) {
    hipError_t e;
    switch ((w + 3) / 4 * 4) {
        case 4: e = launch_kron_step_obs<4>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, pc, pv, spec, partial, st); break;
        case 8: e = launch_kron_step_obs<8>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, pc, pv, spec, partial, st); break;
        case 12: e = launch_kron_step_obs<12>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, pc, pv, spec, partial, st); break;
        default: e = launch_kron_step_obs<16>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, pc, pv, spec, partial, st);
    }
    if (e != hipSuccess) return e;
    return observable_final(1024 / KronShape<1024>::SW, B, partial, vals, 1024 * w, n_steps, step, out, out_stride, st);
}

template <int D>
hipError_t launch_kron_step(int B, float2* X0, float2* X1, const int* loc, long long xstride, const float2* gates,
                            const float2* pre, const float2* post, const int* n_steps, int step, hipStream_t st) {
    constexpr int NSTRIP = D / KronShape<D>::SW;
    void* tok = nullptr;
    const bool prof = profiling_on();
    if (prof) profile_begin(st, &tok, 1);
    hipLaunchKernelGGL(kron_step_kernel<D>, dim3((unsigned)((long long)B * NSTRIP)), dim3(KRON_NT), 0, st, X0, X1, loc,
                       xstride, gates, pre, post, n_steps, step);
    if (prof) profile_end(st, tok);
    return hipGetLastError();
}

hipError_t kron_step(int d, int B, float2* X0, float2* X1, const int* loc, long long xstride, const float2* gates,
                     const float2* pre, const float2* post, const int* n_steps, int step, hipStream_t st) {
    switch (d) {
        case 128: return launch_kron_step<128>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, st);
        case 256: return launch_kron_step<256>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, st);
        case 512: return launch_kron_step<512>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, st);
        case 1024: return launch_kron_step<1024>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, st);
        case 2048: return launch_kron_step<2048>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, st);
        case 4096: return launch_kron_step<4096>(B, X0, X1, loc, xstride, gates, pre, post, n_steps, step, st);
        default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------- several steps per launch
// d = 128 .. 1024: the step acts on the columns of X one by one, so a workgroup keeps its strip of
// columns on chip for a chunk of steps and HBM sees one read and one write of the states per
// chunk.  Every spin factor is split into diagonal phases and a real rotation,
//     g = diag(p0, p1) [[c, -s], [s, c]] diag(1, r1),
// the phases of all spins and max(c, s) going into the step's two row scalings (FP64, rounded
// once).  A rotation with s > c is one by 90 degrees less, followed by the quarter turn
// (x, y) -> (-y, x): a flip of the spin's row bit, which the next exchange's address takes, and a
// sign, which the row scaling takes.  What is left of a factor is (x - t y, y + t x) with
// |t| <= 1: 4 FMAs per pair and spin instead of 16 operations.  256 threads hold 32 values each: row bits 0..4 in
// registers (layout A) for spins 0..4, bits n-5..n-1 (layout B) for the others, one exchange
// through LDS from A to B and one back per step.  Bound: vector FP32, 2 n d^2 instructions
// per instance-step for the rotations, 8 d^2 for the scalings, n d^2 for the magnetisation.
// 512 instances at d = 1024 with the magnetisation: 0.75 ms per step (0.5 ms is the issue time of
// the vector instructions), against 2.8 ms for one launch per step; 1.02 ms with (c, s) rotations.
constexpr int KM_NT = 256, KM_V = 32, KM_STEPS = 16;   // threads, values per thread, steps per launch

template <int N>
struct KMShape {
    static constexpr int D = 1 << N, SW = KM_NT * KM_V / D, NSTRIP = D / SW, HB = N - 5;
    static_assert(N >= 7 && N <= 10, "two register layouts cover the row bits");
};

struct KronMultiPlan {
    KronPlanArgs p;        // p.step: the first step of the chunk
    float* rot;            // [B][T][16]: t per spin; [15] the flipped row bits (int)
    float2* pre;           // [B][T][d], by rows
    float2* post;          // [B][T][d], by rows before the flip of bits 5.., in layout B
    int T;
};

__global__ __launch_bounds__(256) void kron_multi_plan_kernel(KronMultiPlan m) {
    const KronPlanArgs& a = m.p;
    const int b = blockIdx.x, t = blockIdx.y, step = a.step + t, n = a.n, d = a.d;
    if (a.n_steps && step >= a.n_steps[b]) return;
    const long long ci = ((long long)b * a.N + step) * a.K;
    __shared__ double th[16], ph[16];
    __shared__ double mx[16];
    __shared__ int turned[16];
    __shared__ double2 p0[16], p1[16], r1[16], lowP[32], lowR[32], highP[32], highR[32];
    kron_channels(a, ci, th, ph);
    __syncthreads();
    if ((int)threadIdx.x < n) {
        const int q = threadIdx.x;
        double2 g[4];
        kron_spin_factor(a, q, th, g);
        // g00 = p0 c, g10 = p1 s, g01 = -p0 s r1, g11 = p1 c r1
        const double c = sqrt(g[0].x * g[0].x + g[0].y * g[0].y), s = sqrt(g[2].x * g[2].x + g[2].y * g[2].y);
        const double2 one = make_double2(1.0, 0.0);
        const double2 u0 = c > 0.0 ? make_double2(g[0].x / c, g[0].y / c) : one;
        const double2 u1 = s > 0.0 ? make_double2(g[2].x / s, g[2].y / s) : one;
        // the larger of c, s gives r1
        double2 r = c >= s ? zmul(g[3], zconj(u1)) : zmul(make_double2(-g[1].x, -g[1].y), zconj(u0));
        const double l = sqrt(r.x * r.x + r.y * r.y);
        r = make_double2(r.x / l, r.y / l);
        p0[q] = u0;
        p1[q] = u1;
        r1[q] = r;
        turned[q] = s > c;
        mx[q] = s > c ? s : c;
        m.rot[((long long)b * m.T + t) * 16 + q] = s > c ? (float)(-c / s) : (float)(s / c);
    }
    __syncthreads();
    if (threadIdx.x < 64) {   // products over the low five spins and over the others
        const bool hi = threadIdx.x >= 32;
        const int r = threadIdx.x & 31, q0 = hi ? 5 : 0, q1 = hi ? n : 5;
        double2 P = make_double2(1.0, 0.0), Rr = P;
        for (int q = q0; q < q1; ++q) {
            const bool bit = (r >> (q - q0)) & 1;
            P = zmul(P, bit ? p1[q] : p0[q]);
            const double f = turned[q] && !bit ? -mx[q] : mx[q];
            P = make_double2(P.x * f, P.y * f);
            if (bit) Rr = zmul(Rr, r1[q]);
        }
        (hi ? highP : lowP)[r] = P;
        (hi ? highR : lowR)[r] = Rr;
    }
    __syncthreads();
    const int hb = n - 5;
    int flip = 0;
    for (int q = 0; q < n; ++q) flip |= turned[q] << q;
    if (threadIdx.x == 0) m.rot[((long long)b * m.T + t) * 16 + 15] = __int_as_float(flip);
    const int up = flip & ~31;
    float2* pre = m.pre + ((long long)b * m.T + t) * d;
    float2* post = m.post + ((long long)b * m.T + t) * d;
    for (int r = threadIdx.x; r < d; r += blockDim.x) {
        double2 p, q;
        kron_row_scalings(a, b, r, ph, p, q);
        p = zmul(p, zmul(lowR[r & 31], highR[r >> 5]));
        q = zmul(q, zmul(lowP[r & 31], highP[r >> 5]));
        pre[r] = make_float2((float)p.x, (float)p.y);
        const int o = r ^ up;
        post[(o & ((1 << hb) - 1)) * 32 + (o >> hb)] = make_float2((float)q.x, (float)q.y);
    }
}

template <int J>
__device__ inline void km_rotate(float2 (&v)[KM_V], float t) {
#pragma unroll
    for (int i = 0; i < KM_V; ++i) {
        if (i & (1 << J)) continue;
        const float2 x = v[i], y = v[i | (1 << J)];
        v[i] = make_float2(fmaf(-t, y.x, x.x), fmaf(-t, y.y, x.y));
        v[i | (1 << J)] = make_float2(fmaf(t, x.x, y.x), fmaf(t, x.y, y.y));
    }
}

// Re sum over the pairs of register bit J of conj(v_i) v_j
template <int J>
__device__ inline float km_pairs(const float2 (&v)[KM_V]) {
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < KM_V; ++i) {
        if (i & (1 << J)) continue;
        const float2 x = v[i], y = v[i | (1 << J)];
        a = fmaf(x.x, y.x, fmaf(x.y, y.y, a));
    }
    return a;
}

__device__ inline void km_scale(float2 (&v)[KM_V], const float2* __restrict__ s) {
    const float4* p = reinterpret_cast<const float4*>(s);
#pragma unroll
    for (int i = 0; i < KM_V; i += 2) {
        const float4 w = p[i / 2];
        v[i] = cmul(make_float2(w.x, w.y), v[i]);
        v[i + 1] = cmul(make_float2(w.z, w.w), v[i + 1]);
    }
}

// per spin 2 f of an observable M_ij = sum_q f_q [i XOR j = 2^q], by value
struct KronBits {
    float f[10];
};

template <int N, bool OBS>
__global__ __launch_bounds__(KM_NT, 2) void kron_multi_kernel(float2* X0, float2* X1, const int* loc, long long xstride,
                                                              const float* __restrict__ rot,
                                                              const float2* __restrict__ pre,
                                                              const float2* __restrict__ post, const int* n_steps,
                                                              int step0, int T, int chunk, KronBits ob,
                                                              const double* __restrict__ spec,
                                                              double* __restrict__ partial) {
    using S = KMShape<N>;
    constexpr int D = S::D, SW = S::SW, NSTRIP = S::NSTRIP, HB = S::HB;
    __shared__ float2 buf[KM_NT * KM_V];
    const long long bid = kron_xcd(blockIdx.x, gridDim.x);
    const int b = (int)(bid / NSTRIP), strip = (int)(bid % NSTRIP);
    const int steps = n_steps ? min(T, n_steps[b] - step0) : T;
    if (steps <= 0) return;   // uniform over the workgroup
    float2* X = ((loc && loc[b]) ? X1 : X0) + (long long)b * xstride + strip * SW;
    const int t = threadIdx.x, c = t % SW, rest = t / SW;
    // LDS place of (row, column): the low row bits XOR the high ones, so that the rows of one
    // access fall into different banks in both layouts.  The place of a XOR of rows is the XOR
    // of the places; the bases are kept opaque, or 64 addresses would be held in registers.
    auto lin = [](int row) { return (row ^ (row >> 5)) * SW * 8; };   // bytes
    auto lds = [&](int o) -> float2& { return *reinterpret_cast<float2*>(reinterpret_cast<char*>(buf) + o); };
    int la = lin(rest << 5) + c * 8, lb = lin(rest) + c * 8;
    float2 v[KM_V];
#pragma unroll
    for (int i = 0; i < KM_V; ++i) v[i] = X[(long long)(i | rest << 5) * D + c];
    double dj = 0.0;
    if constexpr (OBS) dj = spec[strip * SW + c];
    const long long pb = (long long)b * chunk;
    for (int k = 0; k < steps; ++k) {
        const float* g = rot + (pb + k) * 16;
        const int flip = __float_as_int(g[15]);
        asm volatile("" : "+v"(la), "+v"(lb));
        const int wa = la ^ lin(flip & 31), wb = lb ^ lin(flip & ~31);
        km_scale(v, pre + (pb + k) * D + rest * 32);
        km_rotate<0>(v, g[0]);
        km_rotate<1>(v, g[1]);
        km_rotate<2>(v, g[2]);
        km_rotate<3>(v, g[3]);
        km_rotate<4>(v, g[4]);
#pragma unroll
        for (int i = 0; i < KM_V; ++i) lds(wa ^ lin(i)) = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < KM_V; ++i) v[i] = lds(lb ^ lin(i << HB));
        __syncthreads();
        km_rotate<5 - HB>(v, g[5]);
        km_rotate<6 - HB>(v, g[6]);
        if constexpr (N > 7) km_rotate<7 - HB>(v, g[7]);
        if constexpr (N > 8) km_rotate<8 - HB>(v, g[8]);
        if constexpr (N > 9) km_rotate<9 - HB>(v, g[9]);
        km_scale(v, post + (pb + k) * D + rest * 32);
        float acc = 0.f;
        if constexpr (OBS) {
            acc = fmaf(ob.f[5], km_pairs<5 - HB>(v), acc);
            acc = fmaf(ob.f[6], km_pairs<6 - HB>(v), acc);
            if constexpr (N > 7) acc = fmaf(ob.f[7], km_pairs<7 - HB>(v), acc);
            if constexpr (N > 8) acc = fmaf(ob.f[8], km_pairs<8 - HB>(v), acc);
            if constexpr (N > 9) acc = fmaf(ob.f[9], km_pairs<9 - HB>(v), acc);
        }
#pragma unroll
        for (int i = 0; i < KM_V; ++i) lds(wb ^ lin(i << HB)) = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < KM_V; ++i) v[i] = lds(la ^ lin(i));
        __syncthreads();
        if constexpr (OBS) {
            acc = fmaf(ob.f[0], km_pairs<0>(v), acc);
            acc = fmaf(ob.f[1], km_pairs<1>(v), acc);
            acc = fmaf(ob.f[2], km_pairs<2>(v), acc);
            acc = fmaf(ob.f[3], km_pairs<3>(v), acc);
            acc = fmaf(ob.f[4], km_pairs<4>(v), acc);
            double s = dj * (double)acc;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
            if ((t & 63) == 0) partial[((pb + k) * NSTRIP + strip) * (KM_NT / 64) + (t >> 6)] = s;
        }
    }
#pragma unroll
    for (int i = 0; i < KM_V; ++i) X[(long long)(i | rest << 5) * D + c] = v[i];
}

// out[b][step0 + k] = sum of the parts / Tr(M M); one wave per (instance, step)
__global__ __launch_bounds__(64) void kron_multi_final_kernel(int nparts, int chunk, int T, const double* partial,
                                                              double norm, const int* n_steps, int step0, double* out,
                                                              long long out_stride) {
    const int b = blockIdx.x, k = blockIdx.y;
    if (k >= T || (n_steps && step0 + k >= n_steps[b])) return;
    const double* p = partial + ((long long)b * chunk + k) * nparts;
    double s = 0.0;
    for (int e = threadIdx.x; e < nparts; e += 64) s += p[e];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (threadIdx.x == 0) out[(long long)b * out_stride + k] = s / norm;
}

// several steps per launch where two register layouts cover the rows.  At d = 2048 and 4096 a row
// no longer fits (a third layout, strips of 4 and 2 columns), and an observable that is not a sum
// over single spins needs every state in memory after its step: these take kron_step_kernel
bool kron_multi(int d) { return d >= 128 && d <= 1024; }

template <int N>
hipError_t launch_kron_multi(int B, float2* X0, float2* X1, const int* loc, long long xstride, const float* rot,
                             const float2* pre, const float2* post, const int* n_steps, int step0, int T, int chunk,
                             const KronBits* ob, const double* spec, double* partial, hipStream_t st) {
    void* tok = nullptr;
    const bool prof = profiling_on();
    if (prof) profile_begin(st, &tok, 1);
    const dim3 grid((unsigned)((long long)B * KMShape<N>::NSTRIP));
    if (ob)
        hipLaunchKernelGGL((kron_multi_kernel<N, true>), grid, dim3(KM_NT), 0, st, X0, X1, loc, xstride, rot, pre, post,
                           n_steps, step0, T, chunk, *ob, spec, partial);
    else
        hipLaunchKernelGGL((kron_multi_kernel<N, false>), grid, dim3(KM_NT), 0, st, X0, X1, loc, xstride, rot, pre, post,
                           n_steps, step0, T, chunk, KronBits{}, spec, partial);
    if (prof) profile_end(st, tok);
    return hipGetLastError();
}

struct KronWS {
    int* codes;
    double* phi;
    float2* W1;
    float2* gates;
    float2 *pre, *post;
    GemmDesc* descs;
    float2* E;   // re-projection scratch: E = (I - X^dag X) / 2 of a chunk
    double* obs_partial;
    int* loc;
    int* plain;
    float2* obsT;
    int chunk;               // steps per launch (kron_multi), else 1
    float* rot;              // [B][chunk][16] rotations (kron_multi)
    double* parts;           // [B][chunk][strips][waves] observable sums (kron_multi)
    size_t bytes;
    KronWS(const redo_table_s* t, int B, int N, void* base) {
        const int d = t->desc.d, K = t->desc.K;
        const size_t mat = (size_t)d * d;
        Carve c(base);
        codes = c.take<int>((size_t)B * N * K);
        phi = c.take<double>((size_t)B * N * K);
        W1 = c.take<float2>(mat * B);
        gates = c.take<float2>((size_t)B * 16 * 4);
        const bool multi = kron_multi(d);
        chunk = multi ? std::min(N, KM_STEPS) : 1;
        pre = c.take<float2>((size_t)B * chunk * d);
        post = c.take<float2>((size_t)B * chunk * d);
        rot = c.take<float>(multi ? (size_t)B * chunk * 16 : 0);
        parts = c.take<double>(multi ? (size_t)B * chunk * ((size_t)d * d / (KM_NT * KM_V)) * (KM_NT / 64) : 0);
        descs = c.take<GemmDesc>((size_t)2 * B);
        E = c.take<float2>(mat * std::min(B, REPROJECT_CHUNK));
        obs_partial = c.take<double>(observable_partial_doubles(d, B));
        loc = c.take<int>(B);
        plain = c.take<int>(B);
        obsT = c.take<float2>(mat * std::min(B, OBS_CHUNK));
        bytes = c.used;
    }
};

}  // namespace

bool kron_supported(const redo_table_s* t) {
    const int d = t->desc.d;
    return t->kron_n > 0 && t->desc.drift_is_diag && d >= 128 && d <= 4096 && (d & (d - 1)) == 0;
}

size_t kron_workspace_bytes(const redo_table_s* t, int B, int N) { return KronWS(t, B, N, nullptr).bytes; }

redo_status kron_chain(redo_table_s* t, int quantised, const float* u, const int* n_steps, int B, int N,
                       int step_offset, int reproject_every, const float* X0, float* U_total, const int* obs_cols,
                       const float* obs_vals, int obs_width, double* obs_out, void* workspace, size_t workspace_bytes,
                       hipStream_t st, bool walsh_frame, const double* walsh, const double* bits) {
    KronWS need(t, B, N, nullptr);
    if (!workspace || workspace_bytes < need.bytes)
        return fail(REDO_ERR_WORKSPACE, "structure-aware chain workspace needs " + std::to_string(need.bytes) + " bytes");
    KronWS w(t, B, N, workspace);
    const int d = t->desc.d;
    const long long mat = (long long)d * d;
    float2* X[2] = {reinterpret_cast<float2*>(U_total), w.W1};
    if (quantised) REDO_HIP(quantise_all(t, u, B, N, w.codes, w.phi, st));
    if (!X0)
        REDO_HIP(walsh_frame ? walsh_fill(d, B, X[0], mat, st) : fill_identity(d, B, X[0], mat, st));
    else if (X0 != U_total)
        REDO_HIP(hipMemcpyAsync(X[0], X0, sizeof(float2) * mat * B, hipMemcpyDeviceToDevice, st));
    StepProducts gram{1, 1, nullptr, nullptr};
    if (reproject_every > 0) REDO_HIP(chain_products(t, B, 1, X[0], X0 != nullptr, w.plain, &gram, st));
    REDO_HIP(fill_int(w.loc, B, 0, st));
    KronPlanArgs pa{};
    pa.s = t->kron_s;
    pa.h = t->h64;
    pa.g = t->desc.phased ? t->g64 : nullptr;
    pa.n_steps = n_steps;
    pa.gates = w.gates;
    pa.pre = w.pre;
    pa.post = w.post;
    pa.eps = t->desc.eps;
    pa.dt = t->desc.dt;
    pa.n = t->kron_n;
    pa.d = d;
    pa.K = t->desc.K;
    pa.N = N;
    pa.n_drift = t->desc.n_drift;
    pa.phased = t->desc.phased;
    pa.strang = t->desc.splitting;
    if (quantised) {
        pa.codes = w.codes;
        pa.phi = t->desc.phased ? w.phi : nullptr;
    } else {
        pa.u = u;
    }
    // in the Walsh frame at d = 1024 the observable rides on the step kernel (steps without
    // a re-projection: there it must see the re-projected state)
    const bool fuse = walsh_frame && obs_out && d == 1024;
    int* pc = nullptr;
    float2* pv = nullptr;
    if (fuse) {
        REDO_HIP(obs_pack_lists(d, B, obs_width, obs_cols, reinterpret_cast<const float2*>(obs_vals), w.obs_partial, st));
        obs_packed_lists(d, B, w.obs_partial, &pc, &pv);
    }
    // several steps per launch, up to the next re-projection (whose step the observable sees
    // re-projected) or the end of the chunk
    const bool bits_obs = walsh_frame && obs_out && bits;
    if (kron_multi(d) && (!obs_out || bits_obs)) {
        KronBits kb{};
        double norm = 0.0;
        for (int q = 0; bits_obs && q < pa.n; ++q) {
            kb.f[q] = (float)(2.0 * bits[q]);
            norm += bits[q] * bits[q] * d;
        }
        const int parts = (int)((size_t)d * d / (KM_NT * KM_V)) * (KM_NT / 64);
        int n = 0;
        while (n < N) {
            int T = std::min(w.chunk, N - n);
            bool reproj = false;
            if (reproject_every > 0) {
                const long long left = reproject_every - ((long long)step_offset + n) % reproject_every;
                if (left <= T) {
                    T = (int)left;
                    reproj = true;
                }
            }
            KronMultiPlan m{};
            m.p = pa;
            m.p.step = n;
            m.rot = w.rot;
            m.pre = w.pre;
            m.post = w.post;
            m.T = w.chunk;
            hipLaunchKernelGGL(kron_multi_plan_kernel, dim3(B, T), dim3(256), 0, st, m);
            REDO_HIP(hipGetLastError());
            const KronBits* ob = bits_obs ? &kb : nullptr;
#define REDO_KM(NN)                                                                                                    \
    REDO_HIP(launch_kron_multi<NN>(B, X[0], X[1], w.loc, mat, w.rot, w.pre, w.post, n_steps, n, T, w.chunk, ob, walsh, \
                                   w.parts, st))
            switch (pa.n) {
                case 7: REDO_KM(7); break;
                case 8: REDO_KM(8); break;
                case 9: REDO_KM(9); break;
                default: REDO_KM(10);
            }
#undef REDO_KM
            const int Tf = reproj ? T - 1 : T;
            if (ob && Tf > 0) {
                hipLaunchKernelGGL(kron_multi_final_kernel, dim3(B, Tf), dim3(64), 0, st, parts, w.chunk, Tf, w.parts, norm,
                                   n_steps, n, obs_out + n, (long long)N);
                REDO_HIP(hipGetLastError());
            }
            if (reproj) {   // X <- X (3I - X^dag X) / 2 into the other buffer
                REDO_HIP(reproject_states(d, B, X[0], X[1], mat, w.E, w.descs, w.loc, n_steps, n + T - 1, gram, t->flags, st));
                if (ob)
                    REDO_HIP(observable_walsh(d, B, X[0], X[1], w.loc, mat, obs_cols, reinterpret_cast<const float2*>(obs_vals),
                                              obs_width, walsh, n_steps, n + T - 1, w.obs_partial, obs_out + n + T - 1, N, st));
            }
            n += T;
        }
        REDO_HIP(gather_back(d, B, X[0], X[1], mat, w.loc, st));
        return REDO_OK;
    }
    for (int n = 0; n < N; ++n) {
        pa.step = n;
        hipLaunchKernelGGL(kron_plan_kernel, dim3(B), dim3(256), 0, st, pa);
        REDO_HIP(hipGetLastError());
        const bool reproj = reproject_every > 0 && ((long long)step_offset + n + 1) % reproject_every == 0;
        if (fuse && !reproj) {
            REDO_HIP(kron_step_observable(B, X[0], X[1], w.loc, mat, w.gates, w.pre, w.post, n_steps, n, obs_width, pc,
                                          pv, reinterpret_cast<const float2*>(obs_vals), walsh, w.obs_partial,
                                          obs_out + n, N, st));
            continue;
        }
        REDO_HIP(kron_step(d, B, X[0], X[1], w.loc, mat, w.gates, w.pre, w.post, n_steps, n, st));
        if (reproj)   // X <- X (3I - X^dag X) / 2 into the other buffer
            REDO_HIP(reproject_states(d, B, X[0], X[1], mat, w.E, w.descs, w.loc, n_steps, n, gram, t->flags, st));
        if (obs_out)
            REDO_HIP(walsh_frame ? observable_walsh(d, B, X[0], X[1], w.loc, mat, obs_cols,
                                             reinterpret_cast<const float2*>(obs_vals), obs_width, walsh, n_steps,
                                             n, w.obs_partial, obs_out + n, N, st)
                           : observable(d, B, X[0], X[1], w.loc, mat, obs_cols,
                                        reinterpret_cast<const float2*>(obs_vals), obs_width, n_steps, n,
                                        w.obs_partial, obs_out + n, N, w.obsT, OBS_CHUNK, st));
    }
    REDO_HIP(gather_back(d, B, X[0], X[1], mat, w.loc, st));
    return REDO_OK;
}

}  // namespace redo
