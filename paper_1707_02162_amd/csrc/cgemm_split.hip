// Split 16-bit batched complex GEMM on CDNA4 matrix cores (GemmDesc contract of cgemm.hip, opB = 0):
// the FP32 step products of the large-d chains in split FP16, for operands whose columns have
// norms near one, that is for unitary factors and states; and, for factors that are real in a
// diagonal gauge, also the split-BF16 ones from panels.
#include <type_traits>

#include "cgemm_common.h"

namespace redo {
namespace {

// ---------------------------------------------------------------------------
// An FP32 operand x is carried as hi = RNE_fp16(2^13 x) and lo = RNE_fp16(2^13 x - hi): 22 bits
// and the sign of lo, that is all of x's 24 or all but the last.  A real product is
// hi*hi + hi*lo + lo*hi on v_mfma_f32_32x32x16_f16 with FP32 accumulation (lo*lo, 2^-24 relative,
// is dropped), divided by 2^26 at the end (exact).  |x| <= 2 stays clear of overflow, and a lo
// below FP16's normal range is off by 2^-38 at most: the unit columns of a state or factor lose
// nothing that FP32 sums keep.  States outside (a start given by the caller) take cgemm_kernel:
// the entry's `active` is 2 instead of 1.
//
// 24 d^3 MFMA operations at 16 times the FP32 rate instead of 8 d^3 (4M) or 6 d^3 (3M).  512
// products at d = 1024 on 128 x 128 tiles: 13.5 ms (0.98 PFLOP/s executed, the rate of a large
// BF16 library product on this card; the clock drops under the load), on 128 x 64 tiles 14.8 ms,
// against 27.2 ms for cgemm_kernel's 3M form.  Three real products (Gauss) took 16.3 and 18.4 ms
// on these tiles: half as much again through LDS, and too few waves for 192 accumulators.
//
// Factors real in a gauge (collective and single-spin drives, REAL): 12 d^3, 9.5 ms.  No zero is
// multiplied any more, and the clock is 1.9 GHz; the matrix cores are busy a third of the time, the
// vector ALUs (splits, gauge, k-scaling) as long.  128 x 64 tiles 12.3 ms; lines touched ahead into
// L2 changed nothing.  Split BF16 from panels, 256 products at d = 512: 0.66 ms against 0.79.
//
// Error against FP64, relative, after chains of 16 .. 100 steps, FP32 4M / 3M / here: Ising drive
// d = 256 1.1 / 1.5 / 0.6e-6, d = 1024 2.0 / 2.6 / 1.1e-6; levels of a collective drive d = 256
// 2.9 / 3.4 / 1.6e-6; digit operators d = 256 3.6 / 4.3 / 3.2e-6, d = 1024 4.1 / 3.7 / 2.8e-6
// (and complex factors, dense generators: d = 192 5.9 / 5.2 / 3.0e-6, d = 320 3.7 / 3.9 / 1.9e-6).
// Digit operators at d = 128 (nearly the identity: the MFMA truncates the small products against
// the large one) 2.3 / 2.9 / 3.1e-6: below d = 192 the chains keep FP32 products.
// ---------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// the two element types: scale of the operands, 1 / scale^2, MFMA
struct Half {
    typedef f16x2 x2;
    typedef f16x8 x8;
    static constexpr float SCALE = 8192.f, UNSCALE = 1.f / (8192.f * 8192.f);
    static __device__ inline floatx16 mfma(x8 a, x8 b, floatx16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};
struct Bf16 {
    typedef bf16x2 x2;
    typedef bf16x8 x8;
    static constexpr float SCALE = 1.f, UNSCALE = 1.f;
    static __device__ inline floatx16 mfma(x8 a, x8 b, floatx16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};

// two values at once: hp = (hi(b) << 16) | hi(a), lp likewise for the remainders
template <class E>
__device__ inline void split_x2(float a, float b, unsigned& hp, unsigned& lp) {
    const typename E::x2 h = __builtin_convertvector(f32x2{a, b}, typename E::x2);
    const typename E::x2 l = __builtin_convertvector(f32x2{a - (float)h.x, b - (float)h.y}, typename E::x2);
    hp = __builtin_bit_cast(unsigned, h);
    lp = __builtin_bit_cast(unsigned, l);
}

template <class E>
__device__ inline unsigned tail_x2(float a, float b, unsigned hp, unsigned lp) {
    const typename E::x2 h = __builtin_bit_cast(typename E::x2, hp), l = __builtin_bit_cast(typename E::x2, lp);
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a - (float)h.x - (float)l.x, b - (float)h.y - (float)l.y},
                                                                typename E::x2));
}

// FORM 0: the three partial products of every real product share one accumulator.
// FORM 1: the small ones, hi*lo and lo*hi, have accumulators of their own, and the sum over k
// takes a third of the roundings.  FORM 2: as 1, and A with the one bit that hi and lo can leave
// out, in a third plane (times hi of B): a digit operator is applied again and again, and what its
// split leaves out adds up.
template <int BM, int BN, int FORM, bool REAL>
struct HCfg {
    // planes of A: re hi, re lo, im hi, im lo (re tail, im tail); REAL: hi, lo (tail)
    static constexpr int NPA = (FORM == 2 ? 6 : 4) / (REAL ? 2 : 1);
    static constexpr int WM = BM / 2, WN = BN / 2;      // wave tile, waves 2 x 2
    static constexpr int FM = WM / 32, FN = WN / 32;
    static constexpr int RA = BM * KT / 256, RB = BN * KT / 256;   // k-run of a thread
    // halves per plane: 32-byte rows (KT values); planes 32 bytes apart beyond their size for 128 rows
    static constexpr int APLANE = BM * KT + (BM == 128 ? 16 : 0), BPLANE = BN * KT + (BN == 128 ? 16 : 0);
    static constexpr int ASZ = NPA * APLANE, BSZ = 4 * BPLANE;
};

// LDS offset (halves) of element (row, k) of plane p: the two 16-byte halves of a row swap when
// bits 2 and 3 of the row differ (bank conflicts, as in the split-BF16 kernel)
template <int PLANE>
__device__ inline int hp_off(int row, int p, int k) {
    return p * PLANE + row * KT + ((((k >> 3) ^ (row >> 2) ^ (row >> 3)) & 1) << 3) + (k & 7);
}

// a thread's row (column of B) and first k: runs of 8 (128 rows) or 4 (64 rows)
template <int R>
__device__ inline void run_of(int& row, int& k) {
    const int t = threadIdx.x;
    if constexpr (R == 8) {
        row = (t & 15) + 16 * (t >> 5);
        k = 8 * ((t >> 4) & 1);
    } else {
        row = (t >> 1) & 63;
        k = 4 * ((t & 1) + 2 * (t >> 7));
    }
}

__device__ inline unsigned ldgu(const unsigned* p) { return *(__attribute__((address_space(1))) const unsigned*)p; }

// R consecutive k of one row: contiguous in memory, or a column of the stored matrix
// base: the stage's first element, uniform; off: the thread's part in bytes (run_offset), so that
// the addresses cost scalar instructions
template <int R, bool STRIDED>
__device__ inline unsigned run_offset(int d) {
    int row, k;
    run_of<R>(row, k);
    return STRIDED ? (unsigned)((k * d + row) * 8) : (unsigned)((row * d + k) * 8);
}
template <int R, bool STRIDED>
__device__ inline void load_run(const float2* base, int d, unsigned off, float2 (&v)[R]) {
    typedef __attribute__((address_space(1))) const char gchar;
    if constexpr (STRIDED) {
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const v2f w = *(gcv2*)((gchar*)(base + (long long)m * d) + off);
            v[m] = f2(w.x, w.y);
        }
    } else {
#pragma unroll
        for (int m = 0; m < R; m += 2) {
            const v4f w = *(gcv4*)((gchar*)(base + m) + off);
            v[m] = f2(w.x, w.y);
            v[m + 1] = f2(w.z, w.w);
        }
    }
}

template <int R, int PLANE, int NP>
__device__ inline void store_planes(const unsigned (&w)[NP][R / 2], unsigned short* S) {
    int row, k;
    run_of<R>(row, k);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        unsigned short* o = S + hp_off<PLANE>(row, p, k);
        if constexpr (R == 8)
            *reinterpret_cast<uint4*>(o) = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
        else
            *reinterpret_cast<uint2*>(o) = make_uint2(w[p][0], w[p][1]);
    }
}

// re, im: factors of the two parts (the operands' scale and the conjugation)
template <class E, int R, int PLANE, int NP>
__device__ inline void store_run(const float2 (&v)[R], float re, float im, unsigned short* S) {
    unsigned w[NP][R / 2];   // [plane][k pair]
#pragma unroll
    for (int q = 0; q < R / 2; ++q) {
        const float ar = v[2 * q].x * re, br = v[2 * q + 1].x * re, ai = v[2 * q].y * im, bi = v[2 * q + 1].y * im;
        split_x2<E>(ar, br, w[0][q], w[1][q]);
        split_x2<E>(ai, bi, w[2][q], w[3][q]);
        if constexpr (NP == 6) {
            w[4][q] = tail_x2<E>(ar, br, w[0][q], w[1][q]);
            w[5][q] = tail_x2<E>(ai, bi, w[2][q], w[3][q]);
        }
    }
    store_planes<R, PLANE, NP>(w, S);
}

// A real in its gauge: per element the real part where row and column have one colour, else the
// imaginary part (negative for rows of colour 0).  cm: all ones where k's colour is 1, rowm: the
// same for the row; flip: the sign bit where the imaginary part is taken negative
template <class E, int R, int PLANE, int NP>
__device__ inline void store_run_real(const float2 (&v)[R], const unsigned (&cm)[R], unsigned rowm, unsigned flip,
                                      unsigned short* S) {
    unsigned w[NP][R / 2];
#pragma unroll
    for (int q = 0; q < R / 2; ++q) {
        auto pick = [&](float2 x, unsigned m) {
            return __uint_as_float(((__float_as_uint(x.y) ^ flip) & m) | (__float_as_uint(x.x) & ~m));
        };
        const float a = pick(v[2 * q], cm[2 * q] ^ rowm) * E::SCALE, b = pick(v[2 * q + 1], cm[2 * q + 1] ^ rowm) * E::SCALE;
        split_x2<E>(a, b, w[0][q], w[1][q]);
        if constexpr (NP == 3) w[2][q] = tail_x2<E>(a, b, w[0][q], w[1][q]);
    }
    store_planes<R, PLANE, NP>(w, S);
}

template <class X8>
__device__ inline X8 neg8(X8 x) {
    uint4 u = __builtin_bit_cast(uint4, x);
    u.x ^= 0x80008000u;
    u.y ^= 0x80008000u;
    u.z ^= 0x80008000u;
    u.w ^= 0x80008000u;
    return __builtin_bit_cast(X8, u);
}

// REAL: the factors are real in a diagonal gauge (GemmDesc::colour), two real products instead of
// four.  PANEL: A from its pre-split panels (REAL, 128 rows)
// op(A) = A (AH false) or A^H is a property of the entry and chosen once per workgroup, so that the
// loads of a stage do not end in a merge of two branches: there the compiler waits for them, and
// the stage's latency is no longer hidden (as it did for a load that the last stage leaves out).
template <class E, int BM, int BN, int FORM, bool REAL, bool PANEL, bool AH, bool GRAM>
__device__ __forceinline__ void split_tile(const GemmDesc& g, int d, int i0, int j0,
                                           unsigned short (*As)[HCfg<BM, BN, FORM, REAL>::ASZ],
                                           unsigned short (*Bs)[HCfg<BM, BN, FORM, REAL>::BSZ], float2 (*Ks)[KT]) {
    using C = HCfg<BM, BN, FORM, REAL>;
    typedef typename E::x8 x8;
    static_assert(!PANEL || (REAL && BM == 128), "panels: real factors, 128-row tiles");
    constexpr int NPA = C::NPA;
    const int nk = d / KT;
    const bool scaled = g.kscale != nullptr;
    const float2* ksrc = (scaled ? g.kscale : g.B) + (threadIdx.x & (KT - 1));
    float2 kreg;   // k-scaling on its way to LDS (every thread one of the stage's KT factors)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi0 = (wave >> 1) * C::WM, wj0 = (wave & 1) * C::WN;
    constexpr int NACC = FORM == 0 ? 2 : 4;
    floatx16 acc[NACC][C::FM][C::FN];
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int ib = 0; ib < C::FM; ++ib)
#pragma unroll
            for (int jb = 0; jb < C::FN; ++jb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][ib][jb][r] = 0.f;
    float2 ra[C::RA], rb[C::RB];
    unsigned cm[REAL ? C::RA : 1], rowm = 0, flip = 0;   // colours of the run's k; of its row
    int arow, ak;
    run_of<C::RA>(arow, ak);
    const unsigned aoff = run_offset<C::RA, AH>(d), boff = run_offset<C::RB, true>(d);
    if constexpr (REAL) {
        rowm = ldgu(g.colour + i0 + arow);
        // op(A) = A^H, or the conjugate of the (symmetric) panel matrix: the imaginary part negated
        flip = ((rowm == 0) != (PANEL ? g.conjA != 0 : AH)) ? 0x80000000u : 0u;
    }
    auto load = [&](int kt) {
        if constexpr (REAL) {
            const unsigned* c = g.colour + kt * KT;
#pragma unroll
            for (int q = 0; q < C::RA; ++q) cm[q] = ldgu(c + ak + q);
        }
        if constexpr (PANEL) {
            typedef __attribute__((address_space(1))) const char gchar;
            const uint16_t* s = g.Abf + ((long long)kt * d + i0) * 64;
            const unsigned o = (unsigned)(arow * 128 + ak * 2);
#pragma unroll
            for (int p = 0; p < 4; ++p) {   // re hi, re lo, im hi, im lo
                const v4f w = *(gcv4*)((gchar*)(s + 16 * p) + o);
                ra[2 * p] = f2(w.x, w.y);
                ra[2 * p + 1] = f2(w.z, w.w);
            }
        } else {
            load_run<C::RA, AH>(AH ? g.A + (long long)kt * KT * d + i0 : g.A + (long long)i0 * d + kt * KT, d, aoff, ra);
        }
        load_run<C::RB, true>(g.B + (long long)kt * KT * d + j0, d, boff, rb);
    };
    auto store = [&](int kt, int buf) {
        if constexpr (PANEL) {
            const unsigned f = flip | flip >> 16;
            unsigned w[2][4];
            auto word = [&](int p, int q) {
                const float2 x = ra[2 * p + q / 2];
                return __float_as_uint(q & 1 ? x.y : x.x);
            };
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned m = ((cm[2 * q] & 0xffffu) | (cm[2 * q + 1] & 0xffff0000u)) ^ rowm;
                    w[h][q] = ((word(2 + h, q) ^ f) & m) | (word(h, q) & ~m);
                }
            store_planes<8, C::APLANE, 2>(w, As[buf]);
        } else if constexpr (REAL) {
            store_run_real<E, C::RA, C::APLANE, NPA>(ra, cm, rowm, flip, As[buf]);
        } else {
            store_run<E, C::RA, C::APLANE, NPA>(ra, E::SCALE, AH ? -E::SCALE : E::SCALE, As[buf]);
        }
        if (scaled) {   // Ks holds the scale already
            int row, k;
            run_of<C::RB>(row, k);
#pragma unroll
            for (int m = 0; m < C::RB; ++m) rb[m] = cmul(Ks[kt % 3][k + m], rb[m]);
            store_run<E, C::RB, C::BPLANE, 4>(rb, 1.f, 1.f, Bs[buf]);
        } else {
            store_run<E, C::RB, C::BPLANE, 4>(rb, E::SCALE, E::SCALE, Bs[buf]);
        }
    };
    auto load_k = [&](int kt) { kreg = ldg2(ksrc + kt * KT); };
    auto store_k = [&](int kt) { Ks[kt % 3][threadIdx.x & (KT - 1)] = f2(kreg.x * E::SCALE, kreg.y * E::SCALE); };
    load(0);
    load_k(0);
    store_k(0);
    load_k(1);
    store_k(1);
    load_k(min(2, nk - 1));
    __syncthreads();
    store(0, 0);
    load(1);
    __syncthreads();
    const int koff = 8 * (lane >> 5);
    auto products = [&](int buf, auto between) __attribute__((always_inline)) {
        x8 a[C::FM][NPA], b[C::FN][4];
#pragma unroll
        for (int ib = 0; ib < C::FM; ++ib)
#pragma unroll
            for (int p = 0; p < NPA; ++p)
                a[ib][p] = *reinterpret_cast<const x8*>(As[buf] + hp_off<C::APLANE>(wi0 + ib * 32 + (lane & 31), p, koff));
#pragma unroll
        for (int jb = 0; jb < C::FN; ++jb)
#pragma unroll
            for (int p = 0; p < 4; ++p)
                b[jb][p] = *reinterpret_cast<const x8*>(Bs[buf] + hp_off<C::BPLANE>(wj0 + jb * 32 + (lane & 31), p, koff));
        // the nth of hi*hi, hi*lo, lo*hi of planes pa, pb into accumulator x
        auto prod = [&](int x, int pa, int pb, bool neg) __attribute__((always_inline)) {
#pragma unroll
            for (int ib = 0; ib < C::FM; ++ib) {
                const x8 av = neg ? neg8(a[ib][pa]) : a[ib][pa];
#pragma unroll
                for (int jb = 0; jb < C::FN; ++jb) acc[x][ib][jb] = E::mfma(av, b[jb][pb], acc[x][ib][jb]);
            }
        };
        constexpr int c = FORM == 0 ? 0 : 2;
        if constexpr (REAL) {
            // Cr += A Br,  Ci += A Bi
            prod(0, 0, 0, false); prod(1, 0, 2, false);
            between();
            prod(c, 0, 1, false); prod(c + 1, 0, 3, false);
            prod(c, 1, 0, false); prod(c + 1, 1, 2, false);
            if constexpr (FORM == 2) {
                prod(c, 2, 0, false); prod(c + 1, 2, 2, false);
            }
        } else {
            // Cr += Ar Br - Ai Bi,  Ci += Ar Bi + Ai Br
            prod(0, 0, 0, false); prod(1, 0, 2, false);
            prod(c, 0, 1, false); prod(c + 1, 0, 3, false);
            prod(c, 1, 0, false); prod(c + 1, 1, 2, false);
            between();
            prod(0, 2, 2, true);  prod(1, 2, 0, false);
            prod(c, 2, 3, true);  prod(c + 1, 2, 1, false);
            prod(c, 3, 2, true);  prod(c + 1, 3, 0, false);
            if constexpr (FORM == 2) {
                prod(c, 4, 0, false); prod(c + 1, 4, 2, false);
                prod(c, 5, 2, true);  prod(c + 1, 5, 0, false);
            }
        }
    };
    // In the middle of a stage's products the new tiles have had longer to arrive, and the first
    // products need not wait for the LDS stores (split BF16, 256 products at d = 512: 31.3 -> 29.1 ms
    // for 32 steps; 64 x 64 tiles 2 %); the large FP16 tiles would spill (201 -> 217 ms, 512 x 16
    // products at d = 1024)
    constexpr bool MID = !(BN == 128 && std::is_same<E, Half>::value);
    // stage kt: the tiles of kt + 1, loaded during the last stage, go to LDS; those of kt + 2 are
    // loaded, to arrive behind the products of kt.  The k-scaling is one stage further ahead
    for (int kt = 0; kt + 2 < nk; ++kt) {
        auto advance = [&]() __attribute__((always_inline)) {
            store_k(kt + 2);
            store(kt + 1, (kt & 1) ^ 1);
            load(kt + 2);
            load_k(min(kt + 3, nk - 1));
        };
        if constexpr (MID) {
            products(kt & 1, advance);
        } else {
            advance();
            products(kt & 1, [] {});
        }
        __syncthreads();
    }
    store(nk - 1, (nk - 1) & 1);
    products((nk - 2) & 1, [] {});
    __syncthreads();
    products((nk - 1) & 1, [] {});
#pragma unroll
    for (int ib = 0; ib < C::FM; ++ib)
#pragma unroll
        for (int jb = 0; jb < C::FN; ++jb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = i0 + wi0 + ib * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                const int j = j0 + wj0 + jb * 32 + (lane & 31);
                float2 v = f2(acc[0][ib][jb][r], acc[1][ib][jb][r]);
                if constexpr (FORM != 0) v = cadd(v, f2(acc[2][ib][jb][r], acc[3][ib][jb][r]));
                v.x *= E::UNSCALE;
                v.y *= E::UNSCALE;
                if (g.rscale) v = cmul(ldg2(g.rscale + i), v);
                if (g.cscale) v = cmul(v, ldg2(g.cscale + j));
                v.x *= g.alpha;
                v.y *= g.alpha;
                if (g.addend) v = cadd(v, ldg2(g.addend + (long long)i * d + j));
                if (i == j) v.x += g.beta_identity;
                store_c<GRAM>(g, d, i, j, v);
            }
}

template <class E, int BM, int BN, int FORM, bool REAL, bool PANEL, int ROLE, int WPS>
__global__ __launch_bounds__(256, WPS) void cgemm_split_kernel(int d, const GemmDesc* __restrict__ descs) {
    using C = HCfg<BM, BN, FORM, REAL>;
    __shared__ __attribute__((aligned(16))) unsigned short As[2][C::ASZ];
    __shared__ __attribute__((aligned(16))) unsigned short Bs[2][C::BSZ];
    __shared__ float2 Ks[3][KT];   // k-scaling of stages kt, kt + 1, kt + 2 in turn
    constexpr bool GRAM = ROLE == GEMM_ROLE_GRAM;
    const int tiles_n = d / BN;
    int ntile;
    if constexpr (GRAM) ntile = (int)gram_tile_count<BM, BN>(d);
    else ntile = (d / BM) * tiles_n;
    int bid = blockIdx.x;
    const int nb = gridDim.x;
    if (nb % NXCD == 0) bid = (bid % NXCD) * (nb / NXCD) + bid / NXCD;
    const int be = bid / ntile, tile = bid % ntile;
    const GemmDesc g = descs[be];
    if (g.active != 1) return;
    int i0, j0;
    if constexpr (GRAM) {
        gram_tile<BM, BN>(d, tile, i0, j0);
    } else {
        i0 = (tile / tiles_n) * BM;
        j0 = (tile % tiles_n) * BN;
    }
    if (g.A == nullptr || g.B == nullptr) {
        copy_tile(g, d, i0, j0, BM, BN);
        return;
    }
    // opB == 0 in every entry of a chain or Gram product
    if constexpr (GRAM) {
        split_tile<E, BM, BN, FORM, REAL, PANEL, true, true>(g, d, i0, j0, As, Bs, Ks);
    } else if constexpr (PANEL) {
        split_tile<E, BM, BN, FORM, REAL, PANEL, false, false>(g, d, i0, j0, As, Bs, Ks);
    } else {
        if (g.opA)
            split_tile<E, BM, BN, FORM, REAL, PANEL, true, false>(g, d, i0, j0, As, Bs, Ks);
        else
            split_tile<E, BM, BN, FORM, REAL, PANEL, false, false>(g, d, i0, j0, As, Bs, Ks);
    }
}

template <class E, int BM, int BN, int FORM, bool REAL, bool PANEL, int WPS>
hipError_t launch_h(int d, int batch, const GemmDesc* descs, hipStream_t st, int role) {
    const long long tiles = role == GEMM_ROLE_GRAM ? gram_tile_count<BM, BN>(d) : (long long)(d / BM) * (d / BN);
    const long long blocks = tiles * batch;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if constexpr (!REAL) {
        if (role == GEMM_ROLE_GRAM) {
            hipLaunchKernelGGL((cgemm_split_kernel<E, BM, BN, FORM, REAL, PANEL, GEMM_ROLE_GRAM, WPS>), dim3((unsigned)blocks),
                               dim3(256), 0, st, d, descs);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((cgemm_split_kernel<E, BM, BN, FORM, REAL, PANEL, GEMM_ROLE_STEP, WPS>), dim3((unsigned)blocks),
                       dim3(256), 0, st, d, descs);
    return hipGetLastError();
}

template <bool REAL>
hipError_t launch_fp16(int d, int batch, const GemmDesc* descs, hipStream_t st, int role, bool big, bool exact_a) {
    // 128 x 128 tiles have no registers for separate accumulators; from d = 512 the sums' own
    // roundings exceed the splits', in either form
    if (big && d >= 512) return launch_h<Half, 128, 128, 0, REAL, false, 2>(d, batch, descs, st, role);
    if (exact_a && d < 512)
        return big ? launch_h<Half, 128, 64, 2, REAL, false, 2>(d, batch, descs, st, role)
                   : launch_h<Half, 64, 64, 2, REAL, false, 3>(d, batch, descs, st, role);
    return big ? launch_h<Half, 128, 64, 1, REAL, false, 2>(d, batch, descs, st, role)
               : launch_h<Half, 64, 64, 1, REAL, false, 3>(d, batch, descs, st, role);
}

}  // namespace

hipError_t cgemm_fp16_launch(int d, int batch, const GemmDesc* descs, hipStream_t st, int role, bool big, bool exact_a,
                             bool real) {
    return real && role != GEMM_ROLE_GRAM ? launch_fp16<true>(d, batch, descs, st, role, big, exact_a)
                                          : launch_fp16<false>(d, batch, descs, st, role, big, exact_a);
}

hipError_t cgemm_bf16_real_launch(int d, int batch, const GemmDesc* descs, hipStream_t st) {
    return launch_h<Bf16, 128, 128, 0, true, true, 2>(d, batch, descs, st, GEMM_ROLE_STEP);
}

}  // namespace redo
