// Split-FP16 batched complex GEMM on CDNA4 matrix cores: the FP32 step products of the
// large-d chains (GemmDesc contract of cgemm.hip) for operands whose columns have norms
// near one, that is for unitary factors and states.
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
// 12 d^3 MFMA operations at 16 times the FP32 rate instead of 8 d^3 (4M) or 6 d^3 (3M).  512
// products at d = 1024 on 128 x 128 tiles: 13.5 ms (0.98 PFLOP/s executed, the rate of a large
// BF16 library product on this card; the clock drops under the load), on 128 x 64 tiles 14.8 ms,
// against 27.2 ms for cgemm_kernel's 3M form.  Three real products (Gauss) took 16.3 and 18.4 ms
// on these tiles: half as much again through LDS, and too few waves for 192 accumulators.
//
// Error against FP64, relative, after chains of 16 .. 100 steps, FP32 4M / 3M / here: Ising drive
// d = 256 1.1 / 1.5 / 0.7e-6, d = 1024 2.0 / 2.6 / 1.3e-6; levels of a collective drive d = 256
// 2.9 / 3.4 / 1.9e-6; digit operators d = 256 3.6 / 4.3 / 3.4e-6, d = 1024 4.1 / 3.7 / 3.0e-6.
// Digit operators at d = 128 (nearly the identity: the MFMA truncates the small products against
// the large one) 2.3 / 2.9 / 3.1e-6: below d = 192 the chains keep FP32 products.
// ---------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr float FSCALE = 8192.f, FUNSCALE = 1.f / (8192.f * 8192.f);

// two values at once: hp = (hi(b) << 16) | hi(a), lp likewise for the remainders
__device__ inline void split_f16x2(float a, float b, unsigned& hp, unsigned& lp) {
    const f16x2 h = __builtin_convertvector(f32x2{a, b}, f16x2);
    const f16x2 l = __builtin_convertvector(f32x2{a - (float)h.x, b - (float)h.y}, f16x2);
    hp = __builtin_bit_cast(unsigned, h);
    lp = __builtin_bit_cast(unsigned, l);
}

__device__ inline unsigned tail_f16x2(float a, float b, unsigned hp, unsigned lp) {
    const f16x2 h = __builtin_bit_cast(f16x2, hp), l = __builtin_bit_cast(f16x2, lp);
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a - (float)h.x - (float)l.x, b - (float)h.y - (float)l.y}, f16x2));
}

// FORM 0: the three partial products of every real product share one accumulator.
// FORM 1: the small ones, hi*lo and lo*hi, have accumulators of their own, and the sum over k
// takes a third of the roundings.  FORM 2: as 1, and A with the one bit that hi and lo can leave
// out, in a third plane (times hi of B): a digit operator is applied again and again, and what its
// split leaves out adds up.
template <int BM, int BN, int FORM>
struct HCfg {
    static constexpr int NPA = FORM == 2 ? 6 : 4;   // planes re hi, re lo, im hi, im lo (re tail, im tail)
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

// R consecutive k of one row: contiguous in memory, or a column of the stored matrix
template <int R>
__device__ inline void load_run(const float2* p, int d, bool strided, int row0, int k0, float2 (&v)[R]) {
    int row, k;
    run_of<R>(row, k);
    if (strided) {
        const float2* s = p + (long long)(k0 + k) * d + row0 + row;
#pragma unroll
        for (int m = 0; m < R; ++m) v[m] = ldg2(s + (long long)m * d);
    } else {
        const float2* s = p + (long long)(row0 + row) * d + k0 + k;
#pragma unroll
        for (int m = 0; m < R; m += 2) {
            const float4 w = ldg4(s + m);
            v[m] = f2(w.x, w.y);
            v[m + 1] = f2(w.z, w.w);
        }
    }
}

template <int R, int PLANE, int NP>
__device__ inline void store_run(const float2 (&v)[R], float im, _Float16* S) {
    int row, k;
    run_of<R>(row, k);
    unsigned w[NP][R / 2];   // [plane][k pair]
#pragma unroll
    for (int q = 0; q < R / 2; ++q) {
        const float ar = v[2 * q].x * FSCALE, br = v[2 * q + 1].x * FSCALE, ai = v[2 * q].y * im, bi = v[2 * q + 1].y * im;
        split_f16x2(ar, br, w[0][q], w[1][q]);
        split_f16x2(ai, bi, w[2][q], w[3][q]);
        if constexpr (NP == 6) {
            w[4][q] = tail_f16x2(ar, br, w[0][q], w[1][q]);
            w[5][q] = tail_f16x2(ai, bi, w[2][q], w[3][q]);
        }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        _Float16* o = S + hp_off<PLANE>(row, p, k);
        if constexpr (R == 8)
            *reinterpret_cast<uint4*>(o) = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
        else
            *reinterpret_cast<uint2*>(o) = make_uint2(w[p][0], w[p][1]);
    }
}

__device__ inline f16x8 neg8(f16x8 x) {
    uint4 u = __builtin_bit_cast(uint4, x);
    u.x ^= 0x80008000u;
    u.y ^= 0x80008000u;
    u.z ^= 0x80008000u;
    u.w ^= 0x80008000u;
    return __builtin_bit_cast(f16x8, u);
}

#define MFH(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_f16((a), (b), (c), 0, 0, 0)

template <int BM, int BN, int FORM, int ROLE, int WPS>
__global__ __launch_bounds__(256, WPS) void cgemm_fp16_kernel(int d, const GemmDesc* __restrict__ descs) {
    using C = HCfg<BM, BN, FORM>;
    constexpr int NPA = C::NPA;
    __shared__ __attribute__((aligned(16))) _Float16 As[2][C::ASZ];
    __shared__ __attribute__((aligned(16))) _Float16 Bs[2][C::BSZ];
    __shared__ float2 Ks[3][KT];   // k-scaling of stages kt, kt + 1, kt + 2
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
    const int nk = d / KT;
    ks_fetch(g, 0, Ks);
    if (nk > 1) ks_fetch(g, 1, Ks);
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
    const bool sa = g.opA != 0, sb = g.opB == 0;
    const float ima = g.opA ? -FSCALE : FSCALE, imb = g.opB ? -FSCALE : FSCALE;
    float2 ra[C::RA], rb[C::RB];
    auto load = [&](int kt) {
        load_run<C::RA>(g.A, d, sa, i0, kt * KT, ra);
        load_run<C::RB>(g.B, d, sb, j0, kt * KT, rb);
    };
    auto store = [&](int kt, int buf) {
        store_run<C::RA, C::APLANE, NPA>(ra, ima, As[buf]);
        float im = imb;
        if (g.kscale != nullptr) {
            int row, k;
            run_of<C::RB>(row, k);
#pragma unroll
            for (int m = 0; m < C::RB; ++m) rb[m] = cmul(Ks[kt % 3][k + m], g.opB ? cconj(rb[m]) : rb[m]);
            im = FSCALE;
        }
        store_run<C::RB, C::BPLANE, 4>(rb, im, Bs[buf]);
    };
    load(0);
    if (g.kscale != nullptr) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // Ks[0], Ks[1] landed
        __syncthreads();
    }
    store(0, 0);
    __syncthreads();
    const int koff = 8 * (lane >> 5);
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load(kt + 1);
        // slot (kt + 2) % 3 was last read by the store of stage kt - 1, before the previous barrier
        if (kt + 2 < nk) ks_fetch(g, kt + 2, Ks);
        f16x8 a[C::FM][NPA], b[C::FN][4];
#pragma unroll
        for (int ib = 0; ib < C::FM; ++ib)
#pragma unroll
            for (int p = 0; p < NPA; ++p)
                a[ib][p] = *reinterpret_cast<const f16x8*>(As[buf] + hp_off<C::APLANE>(wi0 + ib * 32 + (lane & 31), p, koff));
#pragma unroll
        for (int jb = 0; jb < C::FN; ++jb)
#pragma unroll
            for (int p = 0; p < 4; ++p)
                b[jb][p] = *reinterpret_cast<const f16x8*>(Bs[buf] + hp_off<C::BPLANE>(wj0 + jb * 32 + (lane & 31), p, koff));
        // the nth of hi*hi, hi*lo, lo*hi of planes pa, pb into accumulator x
        auto prod = [&](int x, int pa, int pb, bool neg) __attribute__((always_inline)) {
#pragma unroll
            for (int ib = 0; ib < C::FM; ++ib) {
                const f16x8 av = neg ? neg8(a[ib][pa]) : a[ib][pa];
#pragma unroll
                for (int jb = 0; jb < C::FN; ++jb) acc[x][ib][jb] = MFH(av, b[jb][pb], acc[x][ib][jb]);
            }
        };
        // Cr += Ar Br - Ai Bi,  Ci += Ar Bi + Ai Br
        constexpr int c = FORM == 0 ? 0 : 2;
        prod(0, 0, 0, false);     prod(1, 0, 2, false);
        prod(c, 0, 1, false);     prod(c + 1, 0, 3, false);
        prod(c, 1, 0, false);     prod(c + 1, 1, 2, false);
        prod(0, 2, 2, true);      prod(1, 2, 0, false);
        prod(c, 2, 3, true);      prod(c + 1, 2, 1, false);
        prod(c, 3, 2, true);      prod(c + 1, 3, 0, false);
        if constexpr (FORM == 2) {
            prod(c, 4, 0, false); prod(c + 1, 4, 2, false);
            prod(c, 5, 2, true);  prod(c + 1, 5, 0, false);
        }
        if (kt + 1 < nk) store(kt + 1, buf ^ 1);
        if (g.kscale != nullptr) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this stage's ks_fetch landed
        __syncthreads();
    }
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
                v.x *= FUNSCALE;
                v.y *= FUNSCALE;
                if (g.rscale) v = cmul(ldg2(g.rscale + i), v);
                if (g.cscale) v = cmul(v, ldg2(g.cscale + j));
                v.x *= g.alpha;
                v.y *= g.alpha;
                if (g.addend) v = cadd(v, ldg2(g.addend + (long long)i * d + j));
                if (i == j) v.x += g.beta_identity;
                store_c<GRAM>(g, d, i, j, v);
            }
}

#undef MFH

template <int BM, int BN, int FORM, int WPS>
hipError_t launch_h(int d, int batch, const GemmDesc* descs, hipStream_t st, int role) {
    const long long tiles = role == GEMM_ROLE_GRAM ? gram_tile_count<BM, BN>(d) : (long long)(d / BM) * (d / BN);
    const long long blocks = tiles * batch;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (role == GEMM_ROLE_GRAM)
        hipLaunchKernelGGL((cgemm_fp16_kernel<BM, BN, FORM, GEMM_ROLE_GRAM, WPS>), dim3((unsigned)blocks), dim3(256), 0, st,
                           d, descs);
    else
        hipLaunchKernelGGL((cgemm_fp16_kernel<BM, BN, FORM, GEMM_ROLE_STEP, WPS>), dim3((unsigned)blocks), dim3(256), 0, st,
                           d, descs);
    return hipGetLastError();
}

}  // namespace

hipError_t cgemm_fp16_launch(int d, int batch, const GemmDesc* descs, hipStream_t st, int role, bool big, bool exact_a) {
    // 128 x 128 tiles have no registers for separate accumulators; from d = 512 the sums' own
    // roundings exceed the splits', in either form
    if (big && d >= 512) return launch_h<128, 128, 0, 2>(d, batch, descs, st, role);
    if (exact_a && d < 512)
        return big ? launch_h<128, 64, 2, 2>(d, batch, descs, st, role) : launch_h<64, 64, 2, 3>(d, batch, descs, st, role);
    return big ? launch_h<128, 64, 1, 2>(d, batch, descs, st, role) : launch_h<64, 64, 1, 3>(d, batch, descs, st, role);
}

}  // namespace redo
