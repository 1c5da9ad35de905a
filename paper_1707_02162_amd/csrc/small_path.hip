// Small-dimension REDO path (d = 2 .. 64): a chain runs whole in one launch with its state
// in registers (reg_step.h).  Each step quantises its amplitudes (Sec. II, Eq. cgrain),
// multiplies the state by the table factors that the digits select (processes 1 and 2,
// Eqs. redoform and exp2prod), or by one composed level per channel when the cache holds
// every level (process 3), between the drift and phase scalings of the split step (Sec.
// III, Eqs. vn and vnd), and chains the result (Sec. III, Eq. propUn).
#include "reg_step.h"

namespace redo {
namespace {

// Newton-Schulz polar step x <- x (3I - x^dag x) / 2; the watchdog counts an instance whose
// ||x^dag x - I||_F / sqrt(D) exceeds UNITARITY_WARN.  The state goes through LDS here (it is
// needed by rows): once per re-projection, not per step.
// scale: 1, or 1 / d for a state kept as X H (below), whose Gram matrix is d I.
template <int D>
__device__ __forceinline__ void reproject(float2 (&x)[RC<D>::NR], float2* Xs, float scale, bool active, int lane, int wave, double* red,
                          DeviceFlags* flags, bool leader) {
    using C = RC<D>;
    constexpr int NR = C::NR;
    inst_sync<D>();
    store_state<D>(x, Xs, C::LD, lane, wave);
    inst_sync<D>();
    const int col = reg_col<D>(lane, wave);
    float2 z[NR];
    Frag<D> f[C::NP];
    // row i of X^T: column i of the state
    if constexpr (D == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[0].v[e] = Xs[e % 2 * C::LD + e / 2];
    } else if constexpr (C::COL) {
#pragma unroll
        for (int k = 0; k < D; ++k) f[0].v[k] = x[k];
    } else {
#pragma unroll
        for (int p = 0; p < C::NP; ++p)
#pragma unroll
            for (int r = 0; r < NR; ++r) f[p].v[r] = Xs[reg_row<D>(r, lane) * C::LD + 16 * p + tile_row<D>(lane)];
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) z[r] = x[r];
    mul_full<D>(z, f, -1.f);   // conj(X^T) X
    double dev2 = 0.0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const bool dg = reg_row<D>(r, lane) == col;
        z[r].x *= scale;   // a power of two
        z[r].y *= scale;
        const double er = (double)z[r].x - (dg ? 1.0 : 0.0), ei = z[r].y;
        dev2 += er * er + ei * ei;
        z[r] = make_float2((dg ? 1.5f : 0.f) - 0.5f * z[r].x, -0.5f * z[r].y);
    }
    dev2 = inst_sum<D>(dev2, red);
    if (active && leader) report_drift(flags, sqrt(dev2 / D));
#pragma unroll
    for (int p = 0; p < C::NP; ++p) load_piece_lds<D>(f[p], Xs, p, lane);
    mul_full<D>(z, f, 1.f);
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (active) x[r] = z[r];
}

// ---------------------------------------------------------------- the observable
// Tr(X M X^dag M) / Tr(M M) from row lists (Sec. IV).  General M: the state is parked in LDS
// and gathered by the lists.  d = 4, 8 and M_ac = f(a XOR c) with f real (the collective
// transverse magnetisation is one; a Hermitian M of that form has f real): the chain carries
// W = X H, H the Sylvester-Hadamard matrix (entries +-1, so nothing is rounded on the way in),
// which evolves by the same left products, and with D = H f
//     Tr(X M X^dag M) = (1/d) sum_j D_j w_j^dag M w_j:
// a lane has the whole column w_j in registers, so no element leaves its lane; X = W H / d at
// the end.
__device__ __forceinline__ float dpp_xor(float v, int bit) {
    const int b = __float_as_int(v);
    int r;
    if (bit == 1) {
        r = __builtin_amdgcn_update_dpp(0, b, 0xB1, 0xf, 0xf, true);
    } else if (bit == 2) {
        r = __builtin_amdgcn_update_dpp(0, b, 0x4E, 0xf, 0xf, true);
    } else if (bit == 4) {   // mirror within eight lanes (xor 7), then within four (xor 3)
        r = __builtin_amdgcn_update_dpp(0, b, 0x141, 0xf, 0xf, true);
        r = __builtin_amdgcn_update_dpp(0, r, 0x1B, 0xf, 0xf, true);
    } else {   // 8: mirror within sixteen (xor 15), then within eight
        r = __builtin_amdgcn_update_dpp(0, b, 0x140, 0xf, 0xf, true);
        r = __builtin_amdgcn_update_dpp(0, r, 0x141, 0xf, 0xf, true);
    }
    return __int_as_float(r);
}

// x <- x H over the columns (lanes) of an instance, d = 2 .. 16
template <int D>
__device__ __forceinline__ void hadamard_lanes(float2 (&x)[RC<D>::NR], int lane) {
#pragma unroll
    for (int bit = 1; bit < D; bit <<= 1) {
        const float sgn = (lane & bit) ? -1.f : 1.f;
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) {
            x[r].x = fmaf(sgn, x[r].x, dpp_xor(x[r].x, bit));
            x[r].y = fmaf(sgn, x[r].y, dpp_xor(x[r].y, bit));
        }
    }
}

__device__ __forceinline__ double uniform_double(double v) {   // the same in every lane: to scalar registers
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | lo);
}

template <int D>
struct Observable {
    using C = RC<D>;
    static constexpr bool XOR = D == 4 || D == 8;
    double f[XOR ? D : 1];   // by XOR mask
    int w;
    bool masks;              // M_ac = f(a XOR c), f real: the chain carries W
    double norm, dj;

    // the row lists into LDS and their form; every thread of the workgroup takes part
    __device__ __forceinline__ void setup(const SmallChainArgs& a, float2* vs, int* cs, double* fm, int* flag, int lane, int wave) {
        w = a.obs_width;
        masks = false;
        for (int e = threadIdx.x; e < D * w; e += C::THREADS) {
            vs[e] = a.obs_vals[e];
            cs[e] = a.obs_cols[e];
        }
        if constexpr (XOR) {
            if (threadIdx.x == 0) *flag = 1;
            if (threadIdx.x < D) fm[threadIdx.x] = 0.0;
        }
        __syncthreads();
        double s = 0.0;
        for (int e = 0; e < D * w; ++e) {
            const float2 v = vs[e];
            s += (double)v.x * v.x + (double)v.y * v.y;
        }
        norm = uniform_double(s);   // Tr(M M) = sum |M_ab|^2 (M Hermitian)
        dj = 0.0;
        if constexpr (XOR) {
            // row ra's list is row 0's with its columns XORed by ra: no duplicates, real values
            if (threadIdx.x < D) {
                const int ra = threadIdx.x;
                int cnt = 0, cnt0 = 0;
                bool ok = true;
                for (int e = 0; e < w; ++e) {
                    const float2 v0 = vs[e];
                    if (v0.x != 0.f || v0.y != 0.f) ++cnt0;
                    const float2 v = vs[ra * w + e];
                    if (v.x == 0.f && v.y == 0.f) continue;
                    ++cnt;
                    ok = ok && v.y == 0.f;
                    const int c = cs[ra * w + e];
                    bool found = false;
                    for (int e0 = 0; e0 < w; ++e0) {
                        const float2 u0 = vs[e0];
                        if ((u0.x != 0.f || u0.y != 0.f) && cs[e0] == (c ^ ra) && u0.x == v.x && u0.y == v.y) found = true;
                    }
                    for (int e2 = 0; e2 < e; ++e2) {
                        const float2 u2 = vs[ra * w + e2];
                        if ((u2.x != 0.f || u2.y != 0.f) && cs[ra * w + e2] == c) ok = false;
                    }
                    ok = ok && found && c >= 0 && c < D;
                }
                if (!ok || cnt != cnt0) atomicAnd(flag, 0);
            }
            __syncthreads();
            masks = __builtin_amdgcn_readfirstlane(*flag) != 0;
            if (masks) {
                if (threadIdx.x == 0)
                    for (int e = 0; e < w; ++e)
                        if (vs[e].x != 0.f) fm[cs[e]] = vs[e].x;
                __syncthreads();
                const int j = reg_col<D>(lane, wave);
#pragma unroll
                for (int m = 0; m < D; ++m) {
                    f[m] = uniform_double(fm[m]);
                    dj += (__popc(m & j) & 1) ? -f[m] : f[m];
                }
                dj /= D * norm;
            }
        }
    }
    // every lane of the instance gets the value
    __device__ __forceinline__ double value(const float2 (&x)[C::NR], float2* Xs, const float2* ovs, const int* ocs, int lane, int wave,
                            double* red) const {
        double acc = 0.0;
        if constexpr (XOR) {
            if (masks) {
#pragma unroll
                for (int m = 0; m < D; ++m) {
                    if (f[m] == 0.0) continue;   // the same for every lane
                    double s = 0.0;
#pragma unroll
                    for (int r = 0; r < D; ++r)
                        if (m == 0 || r < (r ^ m))
                            s = fma((double)x[r].x, (double)x[r ^ m].x, fma((double)x[r].y, (double)x[r ^ m].y, s));
                    acc = fma(m == 0 ? f[m] : 2.0 * f[m], s, acc);
                }
                return inst_sum<D>(acc * dj, red);
            }
        }
        inst_sync<D>();
        store_state<D>(x, Xs, C::LD, lane, wave);
        inst_sync<D>();
        const int cb = reg_col<D>(lane, wave);
#pragma unroll
        for (int r = 0; r < C::NR; ++r) {
            const int ra = reg_row<D>(r, lane);
            float2 xm = make_float2(0.f, 0.f), mx = make_float2(0.f, 0.f);
            for (int t = 0; t < w; ++t) {
                cfma(xm, Xs[ra * C::LD + ocs[cb * w + t]], cconj(ovs[cb * w + t]));
                cfma(mx, ovs[ra * w + t], Xs[ocs[ra * w + t] * C::LD + cb]);
            }
            acc += (double)xm.x * mx.x + (double)xm.y * mx.y;
        }
        return inst_sum<D>(acc, red) / norm;
    }
};

template <int D, int PH>
struct ChainLds {   // byte offsets of the dynamic LDS of a workgroup
    size_t steps, mat, obs_f, obs_v, obs_c, total;
    __host__ __device__ ChainLds(int K, int rep, bool needs_mat, int obs_width) {
        using C = RC<D>;
        steps = 0;
        mat = C::W * Steps<D, PH>::lds_bytes(K, rep);
        obs_f = mat + (needs_mat ? (size_t)C::IPW * D * C::LD * sizeof(float2) : 0);
        obs_v = obs_f + (obs_width ? 16 * sizeof(double) : 0);
        obs_c = obs_v + (size_t)D * obs_width * sizeof(float2);
        total = obs_c + (size_t)D * obs_width * sizeof(int);
    }
};

// PH: the table's phased flag at compile time.  EX: prefix states, an observable or a
// re-projection are asked for (their code keeps registers alive that the plain chain needs
// for factors in flight).
template <int D, int PH, int EX, int SC>
__global__ __launch_bounds__(RC<D>::THREADS, D <= 32 ? 2 : 1) void chain_kernel(TView tv_in, SmallChainArgs a, int rep) {
    using C = RC<D>;
    TView tv = tv_in;
    tv.phased = kind_phased(PH);
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ double red[C::W];
    __shared__ int flag;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // rep lane groups hold one instance (d <= 16); the first of them reports and stores
    const int grp = lane / C::LPI, ipw = C::IPW / rep, inst = grp % ipw;
    const int b = blockIdx.x * ipw + inst;
    const bool valid = b < a.B, first = valid && grp < ipw;
    const int len = valid ? (a.n_steps ? a.n_steps[b] : a.N_max) : 0;
    int N = len;
    if constexpr (C::COL) {
#pragma unroll
        for (int off = 32; off >= C::LPI; off >>= 1) N = max(N, __shfl_xor(N, off, 64));
    }
    N = __builtin_amdgcn_readfirstlane(N);
    const bool needs_mat = EX && (a.obs_out || a.reproject_every > 0);
    const ChainLds<D, PH> lay(tv.K, rep, needs_mat, EX && a.obs_out ? a.obs_width : 0);
    float2* Xs = reinterpret_cast<float2*>(lds + lay.mat) + grp * D * C::LD;
    const int drift = (a.drift0 + (valid ? b : 0)) % tv.n_drift;
    constexpr int KK = kind_phased(PH) ? 2 : 1;
    Steps<D, PH> st(tv, lds + wave * Steps<D, PH>::lds_bytes(tv.K, rep),
                    a.u + (long long)(valid ? b : 0) * a.N_max * tv.K * KK, len, drift, lane, inst,
                    grp / ipw * C::LPI + lane % C::LPI, rep, wave == 0);
    float2 x[C::NR];
    if (valid && a.X0)
        load_state<D>(x, a.X0 + (long long)b * D * D, D, lane, wave);
    else
        identity_state<D>(x, lane, wave);
    float2 dph[C::NR];
    if constexpr (!kind_phased(PH)) drift_rows<D>(tv, drift, lane, dph);
    Observable<D> ob{};
    if constexpr (EX) {
        if (a.obs_out)
            ob.setup(a, reinterpret_cast<float2*>(lds + lay.obs_v), reinterpret_cast<int*>(lds + lay.obs_c),
                     reinterpret_cast<double*>(lds + lay.obs_f), &flag, lane, wave);
        if (a.X_prefix) ob.masks = false;   // prefix states leave as they are
        if constexpr (Observable<D>::XOR) {
            if (ob.masks) hadamard_lanes<D>(x, lane);
        }
    }
    const bool leader = st.lt == 0 && wave == 0;
    bool ragged = false;
    if constexpr (C::COL) ragged = a.n_steps != nullptr;
    if constexpr (EX) {
        // from one re-projection to the next
        int n0 = 0;
        while (n0 < N) {
            int n1 = N;
            bool rep_here = false;
            if (a.reproject_every > 0) {
                const int left = a.reproject_every - (a.step_offset % a.reproject_every + n0 % a.reproject_every) % a.reproject_every;
                if (left <= N - n0) {
                    n1 = n0 + left;
                    rep_here = true;
                }
            }
            const int n_last = n1 - 1;
            auto after = [&](int n) __attribute__((always_inline)) {
                const bool active = n < len;
                if (a.X_prefix && active && first)
                    store_state<D>(x, a.X_prefix + ((long long)b * a.N_max + n) * D * D, D, lane, wave);
                if (a.obs_out) {
                    const double m = ob.value(x, Xs, reinterpret_cast<const float2*>(lds + lay.obs_v),
                                              reinterpret_cast<const int*>(lds + lay.obs_c), lane, wave, red);
                    if (active && leader) a.obs_out[(long long)b * a.N_max + n] = m;
                }
            };
            walk<D, PH, 1, D <= 8 ? 2 : 1, SC <= (D <= 8 ? 2 : 1) ? SC : 0>(
                x, st, n0, n1, drift, ragged, dph, [](int) {}, [&](int n) __attribute__((always_inline)) {
                    if (!(rep_here && n == n_last)) after(n);
                });
            if (rep_here) {
                reproject<D>(x, Xs, ob.masks ? 1.f / D : 1.f, n_last < len, lane, wave, red, tv.flags, leader);
                after(n_last);
            }
            n0 = n1;
        }
    } else {
        walk<D, PH, 1, C::U, SC>(x, st, 0, N, drift, ragged, dph, [](int) {}, [](int) {});
    }
    if constexpr (EX && Observable<D>::XOR) {
        if (ob.masks) {
            hadamard_lanes<D>(x, lane);
#pragma unroll
            for (int r = 0; r < C::NR; ++r) x[r] = make_float2(x[r].x * (1.f / D), x[r].y * (1.f / D));
        }
    }
    if (first) store_state<D>(x, a.X_out + (long long)b * D * D, D, lane, wave);
}

// Every step propagator on its own (a wave takes the steps of one instance in groups of a
// header batch): the first factor is loaded as the state itself, scaled by columns, so K
// slots cost K - 1 products.
template <int D, int PH>
__global__ __launch_bounds__(RC<D>::THREADS) void compose_kernel(TView tv_in, SmallChainArgs a, int groups) {
    using C = RC<D>;
    TView tv = tv_in;
    tv.phased = kind_phased(PH);
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slot = lane / C::LPI;
    const long long unit = (long long)blockIdx.x * C::IPW + slot;      // (instance, group of steps)
    const bool valid = unit < (long long)a.B * groups;
    const int b = valid ? (int)(unit / groups) : 0, grp = valid ? (int)(unit % groups) : 0;
    const int whole = valid ? (a.n_steps ? a.n_steps[b] : a.N_max) : 0;
    const int drift = (a.drift0 + b) % tv.n_drift;
    constexpr int KK = kind_phased(PH) ? 2 : 1;
    Steps<D, PH> st(tv, lds + wave * Steps<D, PH>::lds_bytes(tv.K, 1), a.u + (long long)b * a.N_max * tv.K * KK, whole,
                    drift, lane, slot, lane % C::LPI, 1, wave == 0 && !a.quiet);
    const int T = st.T, S = st.S, col = reg_col<D>(lane, wave);
    st.fetch(grp);
    st.form(grp);
    st.phases(grp);
    Scales<D, PH> sc;
    if constexpr (!kind_phased(PH)) {
        drift_rows<D>(tv, drift, lane, sc.pre);
#pragma unroll
        for (int r = 0; r < C::NR; ++r) sc.post[r] = sc.pre[r];
    }
    // the scaling on the right of the first factor, at this lane's column
    float2 vcol = make_float2(1.f, 0.f);
    if constexpr (!kind_phased(PH)) {
        if (tv.diag) vcol = to_f2(expmi((tv.strang ? 0.5 * tv.dt : tv.dt) * tv.h[(long long)drift * D + col]));
    }
    for (int t = 0; t < T; ++t) {
        const int n = grp * T + t;
        const bool act = n < whole;
        if (!__any(act)) break;
        float2 x[C::NR];
        int s = 0;
        if constexpr (kind_phased(PH)) sc.load(st, t);
        if (tv.diag) {
            float2 sc = vcol;
            if constexpr (kind_phased(PH)) sc = st.pre[t * D + col];
            const Slot o = find_slot<D, PH, false>(st, st.place_code(grp, t * S), 0);
            if (o.on) {
#pragma unroll
                for (int r = 0; r < C::NR; ++r) {
                    const int row = reg_row<D>(r, lane);
                    const float2 f = o.sg < 0.f ? cconj(gld2(o.p + col * D + row)) : gld2(o.p + row * D + col);
                    x[r] = make_float2(fmaf(-f.y, sc.y, f.x * sc.x), fmaf(f.y, sc.x, f.x * sc.y));   // as a product rounds
                }
            } else {
#pragma unroll
                for (int r = 0; r < C::NR; ++r) x[r] = reg_row<D>(r, lane) == col ? sc : make_float2(0.f, 0.f);
            }
            s = 1;
        } else {
            load_state<D>(x, tv.V + (long long)drift * tv.ent, D, lane, wave);
            if constexpr (kind_phased(PH)) scale_rows<D>(x, sc.pre, false, true, act);
        }
        Ahead<D, 1> f;
        if (s < S) fetch_slot<D, 1>(f, 0, find_slot<D, PH, false>(st, st.place_code(grp, t * S + s), s), lane);
        for (; s + 1 < S; ++s)
            apply_slot<D, 1, false>(x, f, 0, find_slot<D, PH, false>(st, st.place_code(grp, t * S + s + 1), s + 1), lane);
        if (s < S) apply_last<D, 1>(x, f, 0);
        if (kind_phased(PH) || tv.strang) scale_rows<D>(x, sc.post, false, true, act);
        if (act) store_state<D>(x, a.X_out + ((long long)b * a.N_max + n) * D * D, D, lane, wave);
    }
}

// lane groups per instance (d <= 16): batches of at most a wave per SIMD spread over the chip,
// one instance per wave in the limit, where a wave's time per step does not depend on how many
// instances it holds and the header work of one instance is shared by its lane groups
template <int D>
int lane_groups(int B) {
    int rep = 1;
    while (2 * rep <= RC<D>::IPW && (long long)B * 2 * rep <= 1024LL * RC<D>::IPW) rep *= 2;
    return rep;
}

template <int D, int PH>
hipError_t launch_chain(const TView& tv, const SmallChainArgs& a, hipStream_t st) {
    using C = RC<D>;
    if (a.compose) {
        const int T = 1 << batch_shift<D>(tv.K, 1), groups = (a.N_max + T - 1) / T;
        const size_t bytes = C::W * Steps<D, PH>::lds_bytes(tv.K, 1);
        const void* k = (const void*)compose_kernel<D, PH>;
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
        const long long units = (long long)a.B * groups;
        hipLaunchKernelGGL((compose_kernel<D, PH>), dim3((unsigned)((units + C::IPW - 1) / C::IPW)), dim3(C::THREADS),
                           bytes, st, tv, a, groups);
        return hipGetLastError();
    }
    const bool ex = a.X_prefix || a.obs_out || a.reproject_every > 0;
    const int rep = lane_groups<D>(a.B), ipw = C::IPW / rep;
    const ChainLds<D, PH> lay(tv.K, rep, ex && (a.obs_out || a.reproject_every > 0), ex && a.obs_out ? a.obs_width : 0);
    const dim3 grid((a.B + ipw - 1) / ipw), block(C::THREADS);
    auto launch = [&](auto kernel) -> hipError_t {
        hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lay.total);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, grid, block, lay.total, st, tv, a, rep);
        return hipGetLastError();
    };
    const int sc = PH <= 1 && tv.cache ? known_slots<D>(tv.K) : 0;
    if constexpr (PH <= 1) {
        if constexpr (known_slots<D>(1) == 1) {
            if (sc == 1) return ex ? launch(chain_kernel<D, PH, 1, 1>) : launch(chain_kernel<D, PH, 0, 1>);
        }
        if constexpr (known_slots<D>(2) == 2) {
            if (sc == 2) return ex ? launch(chain_kernel<D, PH, 1, 2>) : launch(chain_kernel<D, PH, 0, 2>);
        }
    }
    return ex ? launch(chain_kernel<D, PH, 1, 0>) : launch(chain_kernel<D, PH, 0, 0>);
}

template <int D>
hipError_t launch_chain_ph(const TView& tv, const SmallChainArgs& a, hipStream_t st) {
    switch (step_kind(tv)) {
        case 0: return launch_chain<D, 0>(tv, a, st);
        case 1: return launch_chain<D, 1>(tv, a, st);
        case 2: return launch_chain<D, 2>(tv, a, st);
        default: return launch_chain<D, 3>(tv, a, st);
    }
}

}  // namespace

hipError_t small_chain(const redo_table_s* t, const SmallChainArgs& a, hipStream_t st) {
    const TView tv = view_of(t);
    switch (tv.d) {
        case 2: return launch_chain_ph<2>(tv, a, st);
        case 4: return launch_chain_ph<4>(tv, a, st);
        case 8: return launch_chain_ph<8>(tv, a, st);
        case 16: return launch_chain_ph<16>(tv, a, st);
        case 32: return launch_chain_ph<32>(tv, a, st);
        case 64: return launch_chain_ph<64>(tv, a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace redo
