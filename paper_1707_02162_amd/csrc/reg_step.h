// The register-resident form of a step at d = 2 .. 64 (device code shared by the fused
// chain and GRAPE kernels).
//
// X_n = U_n X_{n-1} acts on the columns of X one by one, so a lane keeps its part of a
// column in registers for the whole chain and only the factors move: the state never
// goes through LDS and no barrier separates two products.  The layouts are those in
// which the result registers of one matrix-core product are the right operand of the
// next:
//   d = 4, 8, 16  v_mfma_f32_4x4x1 (16 blocks): lane = column, all d rows in registers,
//               64 / d instances per wave.  The d / 4 neighbouring blocks of an instance hold
//               its columns and share the left operand (cbsz / abid).  One k at a time, so a
//               result element is the same chain of FMAs as a scalar complex product.
//   d = 32, 64  v_mfma_f32_16x16x4: a wave holds 16 columns; lane (q, j) = (lane / 16,
//               lane % 16) holds four rows of column j per 16-row tile.  d = 32: rows
//               16 t + 4 r + q, from a left operand whose rows are dealt out in that order, so
//               that the k-steps (t, r) run over k = 16 t + 4 r + q, in blocks of four
//               ascending k.  d = 64: rows 16 t + 4 q + r and k-steps in the same order, where a
//               lane's part of a row of the left operand is four neighbours (16-byte loads).
//   d = 2       vector FMAs, lane = column.
// The codes and phases of several steps at once are formed by all lanes of an instance
// (Steps), one batch ahead of their use, so that the factor loads of later products are
// in flight while the current one runs.
//
// Bound: the issue of the matrix instructions where the batch fills the card (d = 64, 256 chains
// of 1000 steps: 5.0 ms, 70 % of the FP32 matrix rate; 8.6 ms with the products staged in LDS), the
// latency of one dependent product per step where it does not (one d = 4 chain of 50 steps: 44 us
// against 141, three quarters of it the launch and 64 steps' headers).  d = 8, 16,384 chains of
// 2000 steps with the observable: 3.1 ms against 8.8.
#pragma once
#include "redo_internal.h"

namespace redo {

constexpr int KMAX = 16;

struct TView {
    const float2* T;
    const float2* cache;   // every level composed (process 3): [K][levels][d][d], or null
    const float2* V;
    const double* h;
    const double* g;
    const signed char* g2;   // 2 g as integers (every g a half-integer), or null
    const float2* S;
    const int* spc;          // sparsity pattern of the generators: columns [d][spw] ...
    const double2* spv;      // ... and values [K][d][spw], spw = 0: none
    DeviceFlags* flags;
    long long ent;   // d*d
    int d, K, P, base, phased, diag, n_drift;
    int levels;            // cache levels (q = 0 .. levels - 1)
    int strang;            // 1: U_n = V(dt/2) C_n V(dt/2) (diagonal drift)
    int sym;               // cached levels exactly symmetric (real generators): R^dag = conj(R)
    int spw;
    double eps, qmax, dt;
};

namespace {

inline TView view_of(const redo_table_s* t) {
    TView v;
    v.T = t->T32;
    // the fused kernels use the level cache only when it holds every level
    const bool all = t->cache && t->cache_lo == 0 && (double)t->cache_hi >= t->qmax;
    v.cache = all ? t->cache : nullptr;
    v.levels = all ? t->cache_hi + 1 : 0;
    v.V = t->V32;
    v.h = t->h64;
    v.g = t->g64;
    v.g2 = t->g2;
    v.S = t->S32;
    v.spc = t->spat_cols;
    v.spv = t->spat_vals;
    v.spw = t->spat_w;
    v.flags = t->flags;
    v.ent = t->entry_elems;
    v.d = t->desc.d;
    v.K = t->desc.K;
    v.P = t->desc.digits;
    v.base = t->desc.base;
    v.phased = t->desc.phased;
    v.diag = t->desc.drift_is_diag;
    v.n_drift = t->desc.n_drift;
    v.eps = t->desc.eps;
    v.qmax = t->qmax;
    v.dt = t->desc.dt;
    v.strang = t->desc.splitting;
    v.sym = all ? 1 : 0;
    for (int k = 0; k < t->desc.K; ++k) v.sym = v.sym && t->s_real[k];
    return v;
}

template <int D>
struct RC {
    static constexpr bool COL = D <= 16;              // lane = column
    static constexpr int LPI = COL ? D : 64;          // lanes of a wave per instance
    static constexpr int W = COL ? 1 : D / 16;        // waves per instance (16 columns each)
    static constexpr int IPW = 64 / LPI;              // instances per wave
    static constexpr int THREADS = 64 * W;            // a workgroup is one wave, or one instance
    static constexpr int NR = COL ? D : D / 4;        // complex state registers per lane
    static constexpr int NP = COL ? 1 : D / 16;       // row tiles of a factor, loaded piece by piece
    static constexpr int FE = D == 2 ? 4 : COL ? D : D / 4;   // complex per piece
    static constexpr int LD = COL ? D + 2 : D + 1;    // row length of a matrix parked in LDS
    // products whose factors are in flight ahead of the current one: enough to cover a load
    // from L2 (a product is 16 .. 256 matrix-core instructions, 128 .. 8192 cycles)
    static constexpr int U = D <= 4 ? 4 : D <= 16 ? 2 : D == 32 ? 2 : 1;
    static constexpr int EB = COL ? 8 : 64;           // (step, channel) pairs per batch of headers (times `rep`)
    static constexpr int EPL = COL ? 16 / D : 1;      // headers a lane forms per batch, at most (K <= 16)
};

// A wave of few instances (d <= 16, batches that leave the chip mostly idle) takes IPW / rep of
// them: `rep` lane groups then hold the same instance, and form its headers together, rep times
// as many steps per batch.  A power of two.
template <int D>
__host__ __device__ __forceinline__ int batch_shift(int K, int rep) {   // steps per batch: 1 << batch_shift
    const int t = RC<D>::EB * rep / K, most = RC<D>::COL ? 64 : 8;
    int s = 0;
    while ((2 << s) <= t && (2 << s) <= most) ++s;
    return s;
}
template <int D>
__host__ __device__ __forceinline__ int batch_entries(int K, int rep) {
    return (1 << batch_shift<D>(K, rep)) * K;
}

typedef float fx4 __attribute__((ext_vector_type(4)));

template <int D>
__device__ __forceinline__ int reg_row(int r, int lane) {
    if constexpr (RC<D>::COL)
        return r;
    else if constexpr (D == 32)
        return 16 * (r >> 2) + 4 * (r & 3) + (lane >> 4);
    else
        return 16 * (r >> 2) + 4 * (lane >> 4) + (r & 3);
}
template <int D>
__device__ __forceinline__ int reg_col(int lane, int wave) {
    if constexpr (RC<D>::COL)
        return lane % D;
    else
        return 16 * wave + (lane & 15);
}

// lanes of one wave exchanging data through LDS: program order is enough, the compiler must keep it
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// the threads of one instance
template <int D>
__device__ __forceinline__ void inst_sync() {
    if constexpr (RC<D>::W > 1)
        __syncthreads();
    else
        wave_sync();
}

// Complex products with the fused operations spelled out: the same bits in every copy that the
// compiler makes of a step (left to contract a b - c d itself, it fuses either product).
__device__ __forceinline__ float2 cmulx(float2 a, float2 b) {
    return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.y, b.x, a.x * b.y));
}
__device__ __forceinline__ double2 zmulx(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.y, b.x, a.x * b.y));
}
__device__ __forceinline__ double2 zpowx(double2 z, int m) {   // zpow
    if (m < 0) {
        z.y = -z.y;
        m = -m;
    }
    double2 r = make_double2(1.0, 0.0);
    for (int i = 0; i < m; ++i) r = zmulx(r, z);
    return r;
}

__device__ __forceinline__ float2 to_f2(double2 e) { return make_float2((float)e.x, (float)e.y); }

// ---------------------------------------------------------------- factors
// The factors come through computed pointers, which the compiler cannot place in an address
// space: marked as global memory, their loads wait on the vector-memory counter only.
typedef float gv4 __attribute__((ext_vector_type(4)));
typedef float gv2f __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const gv4 gcv4f;
typedef __attribute__((address_space(1))) const gv2f gcv2f;
__device__ __forceinline__ float4 gld4(const float2* p) {
    const gv4 v = *(gcv4f*)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float2 gld2(const float2* p) {
    const gv2f v = *(gcv2f*)p;
    return make_float2(v.x, v.y);
}

template <int D>
struct Frag {
    float2 v[RC<D>::FE];
};

// the row of a 16-row tile that a lane brings of the left operand: the matrix core puts result row m
// into register m % 4 of lane quarter m / 4
template <int D>
__device__ __forceinline__ int tile_row(int lane) {
    const int m = lane & 15;
    return D == 32 ? 4 * (m & 3) + (m >> 2) : m;
}

// piece p of the left operand from a row-major matrix of row length ld: rows of A, or (tr)
// columns of A, that is A^T; the conjugation of an adjoint is the product's sign sg
template <int D>
__device__ __forceinline__ void load_piece(Frag<D>& f, const float2* __restrict__ A, bool tr, int p, int lane) {
    if constexpr (D == 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 2; ++k) f.v[2 * i + k] = gld2(A + (tr ? 2 * k + i : 2 * i + k));
    } else if constexpr (RC<D>::COL) {
        const int i = lane % D;
        if (!tr) {
#pragma unroll
            for (int k = 0; k < D; k += 2) {
                const float4 w = gld4(A + i * D + k);
                f.v[k] = make_float2(w.x, w.y);
                f.v[k + 1] = make_float2(w.z, w.w);
            }
        } else {
#pragma unroll
            for (int k = 0; k < D; ++k) f.v[k] = gld2(A + k * D + i);
        }
    } else {
        const int i = 16 * p + tile_row<D>(lane);
#pragma unroll
        for (int t = 0; t < D / 16; ++t) {
            if (D == 64 && !tr) {
                const int k0 = 16 * t + 4 * (lane >> 4);
#pragma unroll
                for (int r = 0; r < 4; r += 2) {
                    const float4 w = gld4(A + i * D + k0 + r);
                    f.v[4 * t + r] = make_float2(w.x, w.y);
                    f.v[4 * t + r + 1] = make_float2(w.z, w.w);
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = reg_row<D>(4 * t + r, lane);
                    f.v[4 * t + r] = gld2(A + (tr ? k * D + i : i * D + k));
                }
            }
        }
    }
}

// rows of a matrix parked in LDS (row length LD) as the left operand
template <int D>
__device__ __forceinline__ void load_piece_lds(Frag<D>& f, const float2* A, int p, int lane) {
    using C = RC<D>;
    if constexpr (D == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f.v[e] = A[e / 2 * C::LD + e % 2];
    } else if constexpr (C::COL) {
#pragma unroll
        for (int k = 0; k < D; k += 2) {
            const float4 w = *reinterpret_cast<const float4*>(A + lane % D * C::LD + k);
            f.v[k] = make_float2(w.x, w.y);
            f.v[k + 1] = make_float2(w.z, w.w);
        }
    } else {
        const int i = 16 * p + tile_row<D>(lane);
#pragma unroll
        for (int r = 0; r < C::NR; ++r) f.v[r] = A[i * C::LD + reg_row<D>(r, lane)];
    }
}

// one k of every row block: c[rb] += a (of block rb) b
template <int NB, int CB>
__device__ __forceinline__ void mfma_blocks(float a, float b, fx4 (&c)[NB]) {
    c[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c[0], CB, 0, 0);
    if constexpr (NB > 1) c[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c[1], CB, 1, 0);
    if constexpr (NB > 2) {
        c[2] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c[2], CB, 2, 0);
        c[3] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c[3], CB, 3, 0);
    }
}

// row tile p of y = A x (sg = 1) or conj(A) x (sg = -1); b1 = -sg x.y, b2 = sg x.x.  ADJ: the order of
// the two products in the imaginary part that L <- L U has (y = (L U)^dag = U^dag L^dag)
template <int D, bool ADJ>
__device__ __forceinline__ void mul_piece(float2 (&y)[RC<D>::NR], const Frag<D>& f, const float2 (&x)[RC<D>::NR],
                                          const float (&b1)[RC<D>::NR], const float (&b2)[RC<D>::NR], int p) {
    if constexpr (D == 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            y[i] = make_float2(0.f, 0.f);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float2 a = f.v[2 * i + k];
                y[i].x = fmaf(a.x, x[k].x, y[i].x);
                y[i].x = fmaf(a.y, b1[k], y[i].x);
                y[i].y = ADJ ? fmaf(a.y, b2[k], y[i].y) : fmaf(a.x, x[k].y, y[i].y);
                y[i].y = ADJ ? fmaf(a.x, x[k].y, y[i].y) : fmaf(a.y, b2[k], y[i].y);
            }
        }
    } else if constexpr (RC<D>::COL) {
        // the left operand of row block rb is what block rb of the instance's group holds (abid)
        constexpr int NB = D / 4, CB = D == 4 ? 0 : D == 8 ? 1 : 2;
        fx4 cr[NB], ci[NB];
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) cr[rb] = ci[rb] = fx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const float i0 = ADJ ? f.v[k].y : f.v[k].x, v0 = ADJ ? b2[k] : x[k].y;
            const float i1 = ADJ ? f.v[k].x : f.v[k].y, v1 = ADJ ? x[k].y : b2[k];
            mfma_blocks<NB, CB>(f.v[k].x, x[k].x, cr);
            mfma_blocks<NB, CB>(i0, v0, ci);
            mfma_blocks<NB, CB>(f.v[k].y, b1[k], cr);
            mfma_blocks<NB, CB>(i1, v1, ci);
        }
#pragma unroll
        for (int r = 0; r < D; ++r) y[r] = make_float2(cr[r / 4][r % 4], ci[r / 4][r % 4]);
    } else {
        fx4 cr = {0.f, 0.f, 0.f, 0.f}, ci = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < RC<D>::NR; ++k) {
            const float i0 = ADJ ? f.v[k].y : f.v[k].x, v0 = ADJ ? b2[k] : x[k].y;
            const float i1 = ADJ ? f.v[k].x : f.v[k].y, v1 = ADJ ? x[k].y : b2[k];
            cr = __builtin_amdgcn_mfma_f32_16x16x4f32(f.v[k].x, x[k].x, cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f32_16x16x4f32(i0, v0, ci, 0, 0, 0);
            cr = __builtin_amdgcn_mfma_f32_16x16x4f32(f.v[k].y, b1[k], cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f32_16x16x4f32(i1, v1, ci, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) y[4 * p + r] = make_float2(cr[r], ci[r]);
    }
}

template <int D>
__device__ __forceinline__ void mul_operands(const float2 (&x)[RC<D>::NR], float sg, float (&b1)[RC<D>::NR],
                                    float (&b2)[RC<D>::NR]) {
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) {
        b1[r] = -sg * x[r].y;
        b2[r] = sg * x[r].x;
    }
}

// x <- A x (or conj) with every piece at hand
template <int D, bool ADJ = false>
__device__ __forceinline__ void mul_full(float2 (&x)[RC<D>::NR], const Frag<D> (&f)[RC<D>::NP], float sg) {
    float b1[RC<D>::NR], b2[RC<D>::NR];
    float2 y[RC<D>::NR];
    mul_operands<D>(x, sg, b1, b2);
#pragma unroll
    for (int p = 0; p < RC<D>::NP; ++p) mul_piece<D, ADJ>(y, f[p], x, b1, b2, p);
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) x[r] = y[r];
}

// ---------------------------------------------------------------- state <-> memory (row-major d x d)
template <int D>
__device__ __forceinline__ void load_state(float2 (&x)[RC<D>::NR], const float2* src, int ld, int lane, int wave) {
    const int c = reg_col<D>(lane, wave);
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) x[r] = src[reg_row<D>(r, lane) * ld + c];
}
template <int D>
__device__ __forceinline__ void store_state(const float2 (&x)[RC<D>::NR], float2* dst, int ld, int lane, int wave) {
    const int c = reg_col<D>(lane, wave);
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) dst[reg_row<D>(r, lane) * ld + c] = x[r];
}
template <int D>
__device__ __forceinline__ void identity_state(float2 (&x)[RC<D>::NR], int lane, int wave) {
    const int c = reg_col<D>(lane, wave);
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) x[r] = make_float2(reg_row<D>(r, lane) == c ? 1.f : 0.f, 0.f);
}

// ---------------------------------------------------------------- sums over an instance
// lane i of a double from the lane that the DPP control names (all lanes on)
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// over its lanes in the wave (every lane gets the sum); call with every lane of the wave on
template <int D>
__device__ __forceinline__ double lane_sum(double v) {
    v += dpp_double<0xB1>(v);                                  // lane ^ 1
    if constexpr (RC<D>::LPI >= 4) v += dpp_double<0x4E>(v);   // lane ^ 2
    if constexpr (RC<D>::LPI >= 8) v += dpp_double<0x141>(v);  // the other quad of each eight
    if constexpr (RC<D>::LPI >= 16) v += dpp_double<0x140>(v); // the other eight of each sixteen
    if constexpr (RC<D>::LPI == 64) {
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
    }
    return v;
}
// over the whole instance; scratch: W doubles of LDS, free before and after (W > 1: two barriers)
template <int D>
__device__ __forceinline__ double inst_sum(double v, double* scratch) {
    v = lane_sum<D>(v);
    if constexpr (RC<D>::W > 1) {
        __syncthreads();
        if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
        __syncthreads();
        v = scratch[0];
#pragma unroll
        for (int w = 1; w < RC<D>::W; ++w) v += scratch[w];
    }
    return v;
}

// ---------------------------------------------------------------- steps
// Kinds of step: signed channels (0) and phased channels with half-integer phase generators (1),
// both with a diagonal drift; phased (2) and signed (3) with anything else, a dense drift or
// other phase generators.
constexpr bool kind_phased(int ph) { return ph == 1 || ph == 2; }
constexpr bool kind_general(int ph) { return ph >= 2; }
inline int step_kind(const TView& tv) {
    if (!tv.phased) return tv.diag ? 0 : 3;
    return tv.diag && tv.g2 ? 1 : 2;
}

// Eq. cgrain of a control held in registers, and exp(i phi / 2) of a phased one: quantise_one
// and half_phase with the modulus shared between them
template <int PH>
__device__ __forceinline__ int quantise_reg(double ux, double uy, double eps, double qmax, double2& rot,
                                   DeviceFlags* flags) {
    const double om = kind_phased(PH) ? sqrt(ux * ux + uy * uy) : fabs(ux);
    rot = make_double2(PH == 1 ? 1.0 : 0.0, 0.0);
    if (!(om <= 1.7976931348623157e308)) {   // NaN or Inf
        if (flags) atomicOr(&flags->nonfinite, 1u);
        return 0;
    }
    double qf = floor(om / eps + 0.5);
    if (qf > qmax) {
        if (flags) atomicAdd(&flags->clamped, 1ull);
        qf = qmax;
    }
    if constexpr (PH == 2) rot.x = atan2(uy, ux);
    if constexpr (PH == 1) {
        if (om == 0.0) {
            rot = signbit(ux) ? make_double2(0.0, copysign(1.0, uy)) : make_double2(1.0, copysign(0.0, uy));
        } else {
            // the larger of |cos(phi/2)|, |sin(phi/2)| from a square root, the other from sin(phi)
            const double c = ux / om, s = uy / om;
            const double big = sqrt(0.5 * (1.0 + fabs(c))), small = fabs(s) / (2.0 * big);
            rot = c >= 0.0 ? make_double2(big, copysign(small, s)) : make_double2(small, copysign(big, uy));
        }
    }
    const int q = (int)qf;
    return !kind_phased(PH) && ux < 0.0 ? -q : q;
}

// One instance's steps as a lane sees them: for a batch of T consecutive steps, the codes
// (Sec. II, Eq. cgrain) and, for phased channels, the half-angle phases are formed by all
// lanes of the instance from controls loaded one batch earlier, and from them the row
// scalings pre = Z^dag V and post = Z of every step (Sec. III, Eqs. vn, vnd; Strang: the
// two half drifts), FP64 rounded once.  Codes are kept for two batches (the current one
// and the next in the direction of travel), so the factor pointers of later products are
// known early.  Everything here is private to a wave.
template <int D, int PH>
struct Steps {
    using C = RC<D>;
    static constexpr bool PHASED = kind_phased(PH);
    const TView& tv;
    const float* ub;       // controls of step 0
    int lane, lt, lpi, len, lo, hi, T, tsh, E, S, PE;
    bool report;
    int* hq;               // [2][E] codes
    double2* rot;          // [2][E] exp(i phi / 2) (half-integer generators) or (phi, 0)
    float2 *pre, *post;    // [T][D] (PH, or post of Strang)
    float ux[C::EPL], uy[C::EPL];
    int et[C::EPL], ek[C::EPL];        // step within the batch and channel of this lane's entries
    double2 vrow;                      // drift phase of row lt % D, the row whose scalings this lane forms
    unsigned long long g2lo, g2hi;     // 2 g of that row, a byte per channel

    static __host__ __device__ size_t inst_bytes(int K, int rep) {
        const size_t E = batch_entries<D>(K, rep), T = (size_t)1 << batch_shift<D>(K, rep);
        return ((2 * E * sizeof(int) + 15) & ~size_t(15)) + (PHASED ? 2 * E * sizeof(double2) + 2 * T * D * sizeof(float2) : 0);
    }
    static __host__ __device__ size_t lds_bytes(int K, int rep) {   // per wave
        return C::IPW / rep * inst_bytes(K, rep);
    }
    // inst: the instance's place in the wave; lt_: this lane's place among the lpi lanes that hold it
    __device__ __forceinline__ Steps(const TView& tv_, char* lds, const float* u0, int len_, int drift, int lane_, int inst, int lt_,
                     int rep, bool rep_flags)
        : tv(tv_), ub(u0), lane(lane_), lt(lt_), lpi(C::LPI * rep), len(len_), lo(0), hi(len_), report(rep_flags) {
        tsh = batch_shift<D>(tv.K, rep);
        T = 1 << tsh;
        E = T * tv.K;
        PE = tv.cache ? 1 : tv.P;
        S = tv.K * PE;
        char* p = lds + inst * inst_bytes(tv.K, rep);
        hq = reinterpret_cast<int*>(p);
        rot = reinterpret_cast<double2*>(p + ((2 * E * sizeof(int) + 15) & ~size_t(15)));
        pre = reinterpret_cast<float2*>(rot + 2 * E);
        post = pre + T * D;
        static_assert(C::LPI % D == 0, "a lane forms the scalings of one row");
        const int row = lt % D;
        vrow = make_double2(1.0, 0.0);
        g2lo = g2hi = 0;
        if constexpr (PHASED) {
            if (tv.diag) vrow = expmi((tv.strang ? 0.5 * tv.dt : tv.dt) * tv.h[(long long)drift * D + row]);
            if constexpr (PH == 1)
                for (int k = 0; k < tv.K; ++k) {
                    const unsigned long long m = (unsigned char)tv.g2[k * D + row];
                    if (k < 8)
                        g2lo |= m << (8 * k);
                    else
                        g2hi |= m << (8 * (k - 8));
                }
        }
#pragma unroll
        for (int i = 0; i < C::EPL; ++i) {
            const int e = lt + lpi * i;
            et[i] = e < E ? e / tv.K : -1;
            ek[i] = e % tv.K;
        }
    }
    // controls of a batch into registers
    __device__ __forceinline__ void fetch(int batch) {
#pragma unroll
        for (int i = 0; i < C::EPL; ++i) {
            const int n = batch * T + et[i], k = ek[i];
            ux[i] = uy[i] = 0.f;
            if (et[i] >= 0 && n >= lo && n < hi) {
                if constexpr (PHASED) {
                    const float2 w = *reinterpret_cast<const float2*>(ub + ((long long)n * tv.K + k) * 2);
                    ux[i] = w.x;
                    uy[i] = w.y;
                } else {
                    ux[i] = ub[(long long)n * tv.K + k];
                }
            }
        }
    }
    // their codes and phases into LDS
    __device__ __forceinline__ void form(int batch) {
#pragma unroll
        for (int i = 0; i < C::EPL; ++i) {
            if (lpi * i >= E) break;   // the same for every lane
            const int e = lt + lpi * i;
            const int n = batch * T + et[i];
            if (et[i] < 0) continue;
            int q = 0;
            double2 ro = make_double2(PH == 1 ? 1.0 : 0.0, 0.0);
            if (n >= lo && n < hi)
                q = quantise_reg<PH>((double)ux[i], (double)uy[i], tv.eps, tv.qmax, ro, report ? tv.flags : nullptr);
            hq[(batch & 1) * E + e] = q;
            if constexpr (PHASED) rot[(batch & 1) * E + e] = ro;
        }
        wave_sync();
    }
    // exp(+i theta_row), theta = sum_k phi_k g_k[row], of step t of the batch whose phases are in
    // rt, for the row of this lane
    __device__ __forceinline__ double2 rotation(int t, const double2* rt) const {
        if constexpr (PH == 1) {
            double2 P = make_double2(1.0, 0.0);
            for (int k = 0; k < tv.K; ++k) {
                const int m = (signed char)((k < 8 ? g2lo >> (8 * k) : g2hi >> (8 * (k - 8))) & 0xff);
                P = zmulx(P, zpowx(rt[t * tv.K + k], m));
            }
            return P;
        } else {
            double th = 0.0;
            for (int k = 0; k < tv.K; ++k) th = fma(rt[t * tv.K + k].x, tv.g[k * D + lt % D], th);
            return zconj(expmi(th));
        }
    }
    // the row scalings of a batch from the phases in rot (phased channels)
    __device__ __forceinline__ void phases(int batch) {
        if constexpr (PHASED) {
            for (int e = lt; e < T * D; e += lpi) {
                const int t = e / D;
                float2 a = make_float2(1.f, 0.f), b = a;
                if (batch * T + t < hi) {
                    const double2 P = rotation(t, rot + (batch & 1) * E);
                    a = to_f2(tv.diag ? zmulx(vrow, P) : P);
                    b = to_f2(tv.strang ? zmulx(zconj(P), vrow) : zconj(P));
                }
                pre[e] = a;
                post[e] = b;
            }
            wave_sync();
        }
    }
    // the steps that the coming walk takes (the codes of others are 0)
    __device__ __forceinline__ void range(int n0, int n1) {
        lo = n0;
        hi = min(len, n1);
    }
    // Before the first step: batch b0 formed, the next one's controls on the way.
    __device__ __forceinline__ void start(int b0, int dir) {
        fetch(b0);
        form(b0);
        fetch(b0 + dir);
    }
    // On entering a batch: its scalings, then the codes of the next one and the controls after it.
    __device__ __forceinline__ void enter(int batch, int dir) {
        phases(batch);
        form(batch + dir);
        fetch(batch + 2 * dir);
    }
    __device__ __forceinline__ double2 phase(int n, int k) const {
        return rot[((n >> tsh) & 1) * E + (n & (T - 1)) * tv.K + k];
    }
    __device__ __forceinline__ int code(int n, int k) const {
        return hq[((n >> tsh) & 1) * E + (n & (T - 1)) * tv.K + k];
    }
    // the code of place pos (slots in the order of a step, steps ascending) of a batch
    __device__ __forceinline__ int place_code(int batch, int pos) const {
        const int* h = hq + (batch & 1) * E;
        return tv.cache ? h[pos] : h[pos / tv.P];
    }
    // the factor of slot sl for code q; on: not the identity (the pointer is a valid one all the
    // same), adj: it enters as its adjoint
    __device__ __forceinline__ const float2* factor(int q, int sl, bool& on, bool& adj) const {
        const int aq = q < 0 ? -q : q;
        adj = q < 0;
        if (tv.cache) {
            on = aq != 0;
            return tv.cache + ((long long)sl * tv.levels + aq) * tv.ent;
        }
        const int c = digit_of(q, sl % tv.P, tv.base);
        on = c != 0;
        return tv.T + ((long long)sl * (tv.base - 1) + (on ? c - 1 : 0)) * tv.ent;
    }
};

// A stream of products x <- F x (or F^dag x) whose factors are fetched U products ahead.
template <int D, int U>
struct Ahead {
    Frag<D> f[U][RC<D>::NP];
    float sg[U];
    bool on[U];
};

template <int D>
__device__ __forceinline__ const float2* uniform_ptr(const float2* p) {
    if constexpr (!RC<D>::COL) {   // one instance per wave: the pointer is the same in every lane
        const unsigned long long v = (unsigned long long)p;
        const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
        const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
        return (const float2*)(((unsigned long long)hi << 32) | lo);
    } else {
        return p;
    }
}

// a factor's place and how it enters
struct Slot {
    const float2* p;   // always readable
    float sg;          // -1: conjugated
    bool on;           // false: the identity
    bool tr;           // read by columns (an adjoint that is not the conjugate)
};
// slot sl with code q; DAG: the whole step is applied as its adjoint.  Past an instance's length
// the codes are 0, the identity.
template <int D, int PH, bool DAG>
__device__ __forceinline__ Slot find_slot(const Steps<D, PH>& st, int q, int sl) {
    Slot o;
    bool adj = false;
    if constexpr (!RC<D>::COL) q = __builtin_amdgcn_readfirstlane(q);
    o.p = uniform_ptr<D>(st.factor(q, sl, o.on, adj));
    if constexpr (kind_phased(PH)) adj = false;   // their codes are not negative
    adj = adj != DAG;
    o.sg = adj ? -1.f : 1.f;
    o.tr = adj && !st.tv.sym;
    return o;
}
template <int D, int U>
__device__ __forceinline__ void fetch_slot(Ahead<D, U>& a, int i, const Slot& o, int lane) {
    a.on[i] = o.on;
    a.sg[i] = o.sg;
#pragma unroll
    for (int q = 0; q < RC<D>::NP; ++q) load_piece<D>(a.f[i][q], o.p, o.tr, q, lane);
}

// x <- y where the factor is not the identity
template <int D>
__device__ __forceinline__ void take_product(float2 (&x)[RC<D>::NR], const float2 (&y)[RC<D>::NR], bool on) {
    if (!RC<D>::COL || __all(on)) {
        if (on) {
#pragma unroll
            for (int r = 0; r < RC<D>::NR; ++r) x[r] = y[r];
        }
    } else {
        // the instances of a wave differ
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) {
            x[r].x = on ? y[r].x : x[r].x;
            x[r].y = on ? y[r].y : x[r].y;
        }
    }
}

// x <- the factor in ring place i times x (identity factors leave x as it is), and the next
// factor of that place on its way, piece by piece behind the products.  The product always runs
// and its result is taken or not: one straight piece of code, in which the factors in flight
// keep their registers.
template <int D, int U, bool ADJ>
__device__ __forceinline__ void apply_slot(float2 (&x)[RC<D>::NR], Ahead<D, U>& a, int i, const Slot& next, int lane) {
    constexpr int NR = RC<D>::NR, NP = RC<D>::NP;
    float b1[NR], b2[NR];
    float2 y[NR];
    mul_operands<D>(x, a.sg[i], b1, b2);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        mul_piece<D, ADJ>(y, a.f[i][p], x, b1, b2, p);
        load_piece<D>(a.f[i][p], next.p, next.tr, p, lane);
    }
    take_product<D>(x, y, a.on[i]);
    a.on[i] = next.on;
    a.sg[i] = next.sg;
}
template <int D, int U>
__device__ __forceinline__ void apply_last(float2 (&x)[RC<D>::NR], const Ahead<D, U>& a, int i) {
    float2 y[RC<D>::NR];
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) y[r] = x[r];
    mul_full<D>(y, a.f[i], a.sg[i]);
    take_product<D>(x, y, a.on[i]);
}

// the row scalings of a step on the rows a lane holds; ragged: some instance of the wave may be
// past its length
template <int D>
__device__ __forceinline__ void scale_rows(float2 (&x)[RC<D>::NR], const float2 (&s)[RC<D>::NR], bool conj, bool ragged,
                                  bool act) {
    if (!RC<D>::COL || !ragged) {
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) x[r] = conj ? cmulx(x[r], cconj(s[r])) : cmulx(s[r], x[r]);
    } else {
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) {
            const float2 y = conj ? cmulx(x[r], cconj(s[r])) : cmulx(s[r], x[r]);
            x[r].x = act ? y.x : x[r].x;
            x[r].y = act ? y.y : x[r].y;
        }
    }
}
template <int D, int PH>
struct Scales {
    float2 pre[RC<D>::NR], post[RC<D>::NR];
    __device__ __forceinline__ void load(const Steps<D, PH>& st, int t) {
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) {
            pre[r] = st.pre[t * D + reg_row<D>(r, st.lane)];
            post[r] = st.post[t * D + reg_row<D>(r, st.lane)];
        }
    }
};

// drift phases of the rows a lane holds (unphased channels: constant along the chain): lane i of an
// instance forms row i % D
template <int D>
__device__ __forceinline__ void drift_rows(const TView& tv, int drift, int lane, float2 (&dph)[RC<D>::NR]) {
    const int base = lane - lane % RC<D>::LPI;
    float2 v = make_float2(1.f, 0.f);
    if (tv.diag) v = to_f2(expmi((tv.strang ? 0.5 * tv.dt : tv.dt) * tv.h[(long long)drift * D + lane % RC<D>::LPI % D]));
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) {
        const int from = base + reg_row<D>(r, lane);
        dph[r] = make_float2(__shfl(v.x, from, 64), __shfl(v.y, from, 64));
    }
}

// a dense drift: x <- V x or V^dag x
template <int D>
__device__ __forceinline__ void dense_drift(float2 (&x)[RC<D>::NR], const float2* V, bool dag, bool act, int lane) {
    Frag<D> f[RC<D>::NP];
#pragma unroll
    for (int q = 0; q < RC<D>::NP; ++q) load_piece<D>(f[q], V, dag, q, lane);
    float2 y[RC<D>::NR];
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) y[r] = x[r];
    if (dag)
        mul_full<D, true>(y, f, -1.f);
    else
        mul_full<D, false>(y, f, 1.f);
#pragma unroll
    for (int r = 0; r < RC<D>::NR; ++r) {
        x[r].x = act ? y[r].x : x[r].x;
        x[r].y = act ? y[r].y : x[r].y;
    }
}

// Walks the steps n0 .. n1 - 1 in order: forward (DIR = 1, x <- U_n x) or adjoint (DIR = -1,
// x <- U_n^dag x, from n1 - 1 down).  begin(n) runs before step n, end(n) after it.  The range
// is uniform over the wave (over the workgroup at d >= 32).  U: products whose factors are in
// flight; the slots of a batch of steps are padded to whole rounds of the ring with empty ones,
// and the codes of a round are read a round before its factors are fetched.  SC: the slots per
// step when they are known (1 or 2 cached channels: the bookkeeping of a place folds into the
// unrolled round), else 0.  dph: drift_rows, unphased channels.
template <int D, int PH, int DIR, int U, int SC, class Begin, class End>
__device__ __forceinline__ void walk(float2 (&x)[RC<D>::NR], Steps<D, PH>& st, int n0, int n1, int drift, bool ragged,
                            const float2 (&dph)[RC<D>::NR], Begin begin, End end) {
    constexpr bool dag = DIR < 0, PHASED = kind_phased(PH), GEN = kind_general(PH);
    // the scalings of the next step are read ahead where the registers allow it
    constexpr bool AHEAD = D <= 32;
    static_assert(SC == 0 || U % SC == 0 || SC == 1, "whole steps per round");
    if (n0 >= n1) return;
    const TView& tv = st.tv;
    const int S = SC ? SC : st.S, T = st.T, TS = T * S, rounds = SC ? TS / U : (TS + U - 1) / U;
    const int first = dag ? n1 - 1 : n0, last = dag ? n0 : n1 - 1;
    Scales<D, PH> sc;
    if constexpr (!PHASED) {
#pragma unroll
        for (int r = 0; r < RC<D>::NR; ++r) sc.pre[r] = sc.post[r] = dph[r];
    }
    const bool dense = GEN && !tv.diag;
    const bool has_pre = PHASED || !dense, has_post = PHASED || tv.strang;
    const float2* V = tv.V + (long long)drift * tv.ent;
    Ahead<D, U> a;
    const int bfirst = first >> st.tsh, blast = last >> st.tsh;
    int cq[U];                       // codes of the round to be fetched next: round cr of batch cb
    int cb = bfirst, cr = 0;
    auto read_round = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int pos = cr * U + i;
            if constexpr (SC > 0)
                cq[i] = st.hq[(cb & 1) * st.E + (dag ? TS - 1 - pos : pos)];
            else
                cq[i] = pos < TS ? st.place_code(cb, dag ? TS - 1 - pos : pos) : 0;
        }
    };
    auto slot_at = [&](int i) __attribute__((always_inline)) {      // place i of that round
        const int pos = cr * U + i;
        int sl;
        if constexpr (SC > 0)
            sl = dag ? SC - 1 - i % SC : i % SC;
        else
            sl = pos < TS ? (dag ? TS - 1 - pos : pos) % S : 0;
        return find_slot<D, PH, dag>(st, cq[i], sl);
    };
    auto next_round = [&]() __attribute__((always_inline)) {
        if (++cr == rounds) {
            cr = 0;
            cb += DIR;
        }
    };
    st.range(n0, n1);
    st.start(bfirst, DIR);
    read_round();
#pragma unroll
    for (int i = 0; i < U; ++i) fetch_slot<D, U>(a, i, slot_at(i), st.lane);
    next_round();
    for (int bt = bfirst; dag ? bt >= blast : bt <= blast; bt += DIR) {
        st.enter(bt, DIR);
        if (bt == bfirst) read_round();
        int t = 0, s = 0;
        if constexpr (PHASED && AHEAD) {
            const int nf = dag ? min(bt * T + T - 1, n1 - 1) : max(bt * T, n0);
            sc.load(st, nf & (T - 1));
        }
#pragma unroll 1
        for (int rd = 0; rd < rounds; ++rd) {
            Slot nx[U];
#pragma unroll
            for (int i = 0; i < U; ++i) nx[i] = slot_at(i);
            next_round();
            read_round();
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int tt = SC ? rd * (U / (SC ? SC : 1)) + i / (SC ? SC : 1) : t, ss = SC ? i % (SC ? SC : 1) : s;
                const int n = bt * T + (dag ? T - 1 - tt : tt);
                const bool live = (SC || tt < T) && n >= n0 && n < n1;
                if (ss == 0 && live) {
                    begin(n);
                    const bool act = n < st.len;
                    if constexpr (PHASED && !AHEAD) sc.load(st, n & (T - 1));
                    if constexpr (!dag) {
                        if (dense) dense_drift<D>(x, V, false, act, st.lane);
                        if (has_pre) scale_rows<D>(x, sc.pre, false, ragged, act);
                    } else {
                        if (has_post) scale_rows<D>(x, sc.post, true, ragged, act);
                    }
                }
                apply_slot<D, U, dag>(x, a, i, nx[i], st.lane);
                if (ss == S - 1 && live) {
                    const bool act = n < st.len;
                    if constexpr (!dag) {
                        if (has_post) scale_rows<D>(x, sc.post, false, ragged, act);
                    } else {
                        if (has_pre) scale_rows<D>(x, sc.pre, true, ragged, act);
                        if (dense) dense_drift<D>(x, V, true, act, st.lane);
                    }
                    if constexpr (PHASED && AHEAD) {
                        if (tt + 1 < T) sc.load(st, dag ? T - 2 - tt : tt + 1);
                    }
                    end(n);
                }
                if constexpr (SC == 0) {
                    if (++s == S) {
                        s = 0;
                        ++t;
                    }
                }
            }
        }
    }
}

// the slots per step that the kernels of a dimension know at compile time, else 0
template <int D>
constexpr int known_slots(int s) {
    return (s == 1 && D >= 4) || (s == 2 && (D == 4 || D == 16)) ? s : 0;
}

}  // namespace
}  // namespace redo
