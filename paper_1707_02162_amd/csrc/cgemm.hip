// Batched complex GEMM on CDNA4 matrix cores for the large-d REDO path.
//
// Every product the method performs at d >= 128 is a dense d x d complex
// contraction: a table factor applied to the chain state (Sec. II, process 2;
// Sec. III, chain of Eq. propUn), a Newton-Schulz re-projection, or a
// backward-scan product of the adjoint.  One launch runs a batch of
// independent products, each described by a GemmDesc:
//
//     C = alpha * diag(rs) op(A) diag(ks) op(B) diag(cs) + beta I
//
// with op in {N, H}; A = NULL means the identity, as does B = NULL: such an
// entry's tiles are scaled copies, done by the same launch.  FP32 complex
// products use v_mfma_f32_32x32x2_f32 either as four real products (4M) or three
// (Gauss, 3M); FP32 accumulation throughout (this file); split-BF16 products are
// in cgemm_bf16.hip, split-FP16 products in cgemm_split.hip.
// Tiles are staged through double-buffered LDS; tiles of one batch entry
// are mapped to one XCD so its operands are shared in that XCD's L2.
#include <cstdlib>
#include <string>
#include <type_traits>

#include "cgemm_common.h"

namespace redo {
namespace {

// global -> registers for one stage; AH, BH: op(A) = A^H, op(B) = B^H
template <int BM, int BN, bool AH, bool BH>
__device__ inline void load_tiles(const GemmDesc& g, int d, int i0, int j0, int k0, float4 (&ra)[GCfg<BM, BN>::AV],
                                  float4 (&rb)[GCfg<BM, BN>::BV]) {
    using C = GCfg<BM, BN>;
    const int t = threadIdx.x;
#pragma unroll
    for (int m = 0; m < C::AV; ++m) {
        const int e = t + C::THREADS * m;
        ra[m] = AH ? ldg4(g.A + (long long)(k0 + e / (BM / 2)) * d + i0 + 2 * (e % (BM / 2)))
                   : ldg4(g.A + (long long)(i0 + e / (KT / 2)) * d + k0 + 2 * (e % (KT / 2)));
    }
#pragma unroll
    for (int m = 0; m < C::BV; ++m) {
        const int e = t + C::THREADS * m;
        rb[m] = BH ? ldg4(g.B + (long long)(j0 + e / (KT / 2)) * d + k0 + 2 * (e % (KT / 2)))
                   : ldg4(g.B + (long long)(k0 + e / (BN / 2)) * d + j0 + 2 * (e % (BN / 2)));
    }
}

// registers -> LDS (k-major tiles As[k][i], Bs[k][j]); conjugation, transposition and the k-scaling
// (the stage's KT factors in ks, or null) here
template <int BM, int BN, bool AH, bool BH>
__device__ inline void store_stage(const float4 (&ra)[GCfg<BM, BN>::AV], const float4 (&rb)[GCfg<BM, BN>::BV],
                                   const float2* ks, float2* As, float2* Bs) {
    using C = GCfg<BM, BN>;
    const int t = threadIdx.x;
#pragma unroll
    for (int m = 0; m < C::AV; ++m) {
        const int e = t + C::THREADS * m;
        const float4 v = ra[m];
        if constexpr (!AH) {
            const int row = e / (KT / 2), kq = e % (KT / 2);
            As[(2 * kq) * C::LDA + row] = f2(v.x, v.y);
            As[(2 * kq + 1) * C::LDA + row] = f2(v.z, v.w);
        } else {
            const int kr = e / (BM / 2), iq = e % (BM / 2);
            *reinterpret_cast<float4*>(As + kr * C::LDA + 2 * iq) = make_float4(v.x, -v.y, v.z, -v.w);
        }
    }
#pragma unroll
    for (int m = 0; m < C::BV; ++m) {
        const int e = t + C::THREADS * m;
        const float4 v = rb[m];
        if constexpr (!BH) {
            const int kr = e / (BN / 2), jq = e % (BN / 2);
            float2 a = f2(v.x, v.y), b = f2(v.z, v.w);
            if (ks) {
                const float2 s = ks[kr];
                a = cmul(s, a);
                b = cmul(s, b);
            }
            *reinterpret_cast<float4*>(Bs + kr * C::LDB + 2 * jq) = make_float4(a.x, a.y, b.x, b.y);
        } else {
            const int row = e / (KT / 2), kq = e % (KT / 2);
            float2 a = f2(v.x, -v.y), b = f2(v.z, -v.w);
            if (ks) {
                a = cmul(ks[2 * kq], a);
                b = cmul(ks[2 * kq + 1], b);
            }
            Bs[(2 * kq) * C::LDB + row] = a;
            Bs[(2 * kq + 1) * C::LDB + row] = b;
        }
    }
}

// One output tile.  A stage's tiles are loaded two stages ahead of their products and go to LDS
// one ahead, in the middle of a stage's products: op(A), op(B) and the presence of a k-scaling are
// template parameters, since the compiler moves nothing across a branch.  The order of the sums
// over k is that of the index.  Two products at d = 1024 (64 x 64 tiles, two workgroups per CU, 3M):
// 134 us with loads one stage ahead and stores after the products, 121 with stores before them,
// 115 so (84 us at the rate of a large FP32 product); four at d = 512 (one workgroup per CU, 4M)
// 52.2, 52.2 and 51.8 us.
template <int BM, int BN, int MODE, bool GRAM, bool AH, bool BH, bool SCALED>
__device__ __forceinline__ void fp32_tile(const GemmDesc& g, int d, int i0, int j0, float2 (*As)[KT * GCfg<BM, BN>::LDA],
                                          float2 (*Bs)[KT * GCfg<BM, BN>::LDB], float2 (*Ks)[KT]) {
    using C = GCfg<BM, BN>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi0 = (wave >> 1) * C::WM, wj0 = (wave & 1) * C::WN;
    const int nk = d / KT;
    constexpr int NACC = MODE == 0 ? 2 : 3;
    floatx16 acc[NACC][C::FM][C::FN];
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int ib = 0; ib < C::FM; ++ib)
#pragma unroll
            for (int jb = 0; jb < C::FN; ++jb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][ib][jb][r] = 0.f;

    float4 ra[C::AV], rb[C::BV];
    float2 kreg = f2(0.f, 0.f);   // k-scaling on its way to LDS (every thread one of the stage's KT factors)
    auto load = [&](int kt) { load_tiles<BM, BN, AH, BH>(g, d, i0, j0, kt * KT, ra, rb); };
    auto store = [&](int kt, int buf) {
        store_stage<BM, BN, AH, BH>(ra, rb, SCALED ? Ks[kt % 3] : nullptr, As[buf], Bs[buf]);
    };
    auto load_k = [&](int kt) {
        if constexpr (SCALED) kreg = ldg2(g.kscale + kt * KT + (threadIdx.x & (KT - 1)));
    };
    auto store_k = [&](int kt) {
        if constexpr (SCALED) Ks[kt % 3][threadIdx.x & (KT - 1)] = kreg;
    };
    auto products = [&](int buf, auto k0, auto k1) __attribute__((always_inline)) {
        const float2* Ab = As[buf];
        const float2* Bb = Bs[buf];
#pragma unroll
        for (int kk = k0.value; kk < k1.value; kk += 2) {
            const int kr = kk + (lane >> 5);
            float2 a[C::FM], b[C::FN];
#pragma unroll
            for (int ib = 0; ib < C::FM; ++ib) a[ib] = Ab[kr * C::LDA + wi0 + ib * 32 + (lane & 31)];
#pragma unroll
            for (int jb = 0; jb < C::FN; ++jb) b[jb] = Bb[kr * C::LDB + wj0 + jb * 32 + (lane & 31)];
            auto mf = [&](int x, auto pa, auto pb) __attribute__((always_inline)) {
#pragma unroll
                for (int ib = 0; ib < C::FM; ++ib)
#pragma unroll
                    for (int jb = 0; jb < C::FN; ++jb)
                        acc[x][ib][jb] = __builtin_amdgcn_mfma_f32_32x32x2f32(pa(a[ib]), pb(b[jb]), acc[x][ib][jb], 0, 0, 0);
            };
            auto re = [](float2 v) { return v.x; };
            auto im = [](float2 v) { return v.y; };
            if constexpr (MODE == 0) {
                mf(0, re, re);
                mf(1, re, im);
                mf(0, [](float2 v) { return -v.y; }, im);
                mf(1, im, re);
            } else {
                auto sum = [](float2 v) { return v.x + v.y; };
                mf(0, re, re);
                mf(1, im, im);
                mf(2, sum, sum);
            }
        }
    };
    using K0 = std::integral_constant<int, 0>;
    using KH = std::integral_constant<int, KT / 2>;
    using K1 = std::integral_constant<int, KT>;
    // d >= 64 in multiples of 64: at least four stages
    load(0);
    load_k(0);
    store_k(0);
    load_k(1);
    store_k(1);
    load_k(2);
    if constexpr (SCALED) __syncthreads();
    store(0, 0);
    load(1);
    __syncthreads();
    for (int kt = 0; kt + 2 < nk; ++kt) {
        products(kt & 1, K0{}, KH{});
        store_k(kt + 2);
        store(kt + 1, (kt & 1) ^ 1);
        load(kt + 2);
        load_k(min(kt + 3, nk - 1));
        products(kt & 1, KH{}, K1{});
        __syncthreads();
    }
    store(nk - 1, (nk - 1) & 1);
    products((nk - 2) & 1, K0{}, K1{});
    __syncthreads();
    products((nk - 1) & 1, K0{}, K1{});
    // epilogue: element (i, j) of a 32x32 block lives in lane j + 32 * ((i / 4) % 2), register 4 * (i / 8) + i % 4
#pragma unroll
    for (int ib = 0; ib < C::FM; ++ib)
#pragma unroll
        for (int jb = 0; jb < C::FN; ++jb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = i0 + wi0 + ib * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                const int j = j0 + wj0 + jb * 32 + (lane & 31);
                float2 v;
                if constexpr (MODE == 0) {
                    v = f2(acc[0][ib][jb][r], acc[1][ib][jb][r]);
                } else {
                    const float t1 = acc[0][ib][jb][r], t2 = acc[1][ib][jb][r], t3 = acc[2][ib][jb][r];
                    v = f2(t1 - t2, t3 - t1 - t2);
                }
                if (g.rscale) v = cmul(ldg2(g.rscale + i), v);
                if (g.cscale) v = cmul(v, ldg2(g.cscale + j));
                v.x *= g.alpha;
                v.y *= g.alpha;
                if (g.addend) v = cadd(v, ldg2(g.addend + (long long)i * d + j));
                if (i == j) v.x += g.beta_identity;
                store_c<GRAM>(g, d, i, j, v);
            }
}

// MODE 0: 4M, MODE 1: 3M (Gauss).  ROLE separates the instantiations that the
// method's chain step products (0), the plain-exponential comparison point (1), the
// Newton-Schulz re-projections (2) and the composition of single step propagators (3)
// launch, so that profiles attribute their time apart; the code is the same.  The Gram
// role (4, a re-projection's A^H A) runs only the tiles that meet the upper triangle and
// mirrors them (gram_tile, store_c).
template <int BM, int BN, int MODE, int ROLE>
// at least three waves per SIMD: the 3M form then keeps its 96 accumulators in VGPRs
// (167 registers, no spills) instead of two waves with AGPRs, 240 -> 218 ms for 4096
// products at d = 1024; the LDS already bounds every form at three workgroups per CU
__global__ __launch_bounds__(256, 3) void cgemm_kernel(int d, int only, const GemmDesc* __restrict__ descs) {
    using C = GCfg<BM, BN>;
    __shared__ float2 As[2][KT * C::LDA];
    __shared__ float2 Bs[2][KT * C::LDB];
    __shared__ float2 Ks[3][KT];   // k-scaling of stages kt, kt + 1, kt + 2 in turn
    constexpr bool GRAM = ROLE == GEMM_ROLE_GRAM;
    const int tiles_n = d / BN;
    const int ntile = GRAM ? (int)gram_tile_count<BM, BN>(d) : (d / BM) * tiles_n;
    int bid = blockIdx.x;
    const int nb = gridDim.x;
    if (nb % NXCD == 0) bid = (bid % NXCD) * (nb / NXCD) + bid / NXCD;
    const int be = bid / ntile, tile = bid % ntile;
    const GemmDesc g = descs[be];
    if (only ? g.active != only : !g.active) return;
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
    if constexpr (GRAM) {
        fp32_tile<BM, BN, MODE, true, true, false, false>(g, d, i0, j0, As, Bs, Ks);
    } else if (g.kscale) {
        if (g.opB) {
            if (g.opA) fp32_tile<BM, BN, MODE, false, true, true, true>(g, d, i0, j0, As, Bs, Ks);
            else fp32_tile<BM, BN, MODE, false, false, true, true>(g, d, i0, j0, As, Bs, Ks);
        } else {
            if (g.opA) fp32_tile<BM, BN, MODE, false, true, false, true>(g, d, i0, j0, As, Bs, Ks);
            else fp32_tile<BM, BN, MODE, false, false, false, true>(g, d, i0, j0, As, Bs, Ks);
        }
    } else {
        if (g.opB) {
            if (g.opA) fp32_tile<BM, BN, MODE, false, true, true, false>(g, d, i0, j0, As, Bs, Ks);
            else fp32_tile<BM, BN, MODE, false, false, true, false>(g, d, i0, j0, As, Bs, Ks);
        } else {
            if (g.opA) fp32_tile<BM, BN, MODE, false, true, false, false>(g, d, i0, j0, As, Bs, Ks);
            else fp32_tile<BM, BN, MODE, false, false, false, false>(g, d, i0, j0, As, Bs, Ks);
        }
    }
}

template <int BM, int BN, int MODE>
hipError_t launch(int d, int batch, const GemmDesc* descs, hipStream_t st, int role, int only) {
    const long long tiles = role == GEMM_ROLE_GRAM ? gram_tile_count<BM, BN>(d) : (long long)(d / BM) * (d / BN);
    const long long blocks = tiles * batch;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (role == GEMM_ROLE_GRAM)
        hipLaunchKernelGGL((cgemm_kernel<BM, BN, MODE, GEMM_ROLE_GRAM>), dim3((unsigned)blocks), dim3(256), 0, st, d,
                           only, descs);
    else if (role == GEMM_ROLE_REPROJECT)
        hipLaunchKernelGGL((cgemm_kernel<BM, BN, MODE, 2>), dim3((unsigned)blocks), dim3(256), 0, st, d, only, descs);
    else if (role == GEMM_ROLE_COMPOSE)
        hipLaunchKernelGGL((cgemm_kernel<BM, BN, MODE, 3>), dim3((unsigned)blocks), dim3(256), 0, st, d, only, descs);
    else if (role == GEMM_ROLE_EXPM)
        hipLaunchKernelGGL((cgemm_kernel<BM, BN, MODE, 1>), dim3((unsigned)blocks), dim3(256), 0, st, d, only, descs);
    else
        hipLaunchKernelGGL((cgemm_kernel<BM, BN, MODE, 0>), dim3((unsigned)blocks), dim3(256), 0, st, d, only, descs);
    return hipGetLastError();
}

}  // namespace

// precision: 0 = 4M FP32, 1 = 3M FP32, 2 = split BF16 (hi*hi + hi*lo + lo*hi), GEMM_FP16*: split FP16
hipError_t cgemm_batched(int d, int batch, const GemmDesc* descs, int precision, hipStream_t st, int role, int only) {
    if (d % 64 != 0 || batch < 1) return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    const bool big = cgemm_big(d, batch);
    void* tok = nullptr;
    const bool prof = profiling_on() && !only;   // the launch for the entries left over is not one of products
    if (prof) profile_begin(st, &tok, role == GEMM_ROLE_REPROJECT || role == GEMM_ROLE_GRAM ? 2 : 0);
    // 128x64 tiles: three workgroups per CU for 4M (64 accumulator registers per lane); 3M (96)
    // is also faster there than on 128x128 tiles (240 vs 280 ms for 4096 products at d = 1024)
    const bool real = (precision & GEMM_REAL) != 0;
    precision &= ~GEMM_REAL;
    if (precision >= GEMM_FP16)
        e = cgemm_fp16_launch(d, batch, descs, st, role, big, precision == GEMM_FP16_EXACT_A, real);
    else if (precision == 2 && real && role == GEMM_ROLE_STEP)
        e = cgemm_bf16_real_launch(d, batch, descs, st);
    else if (precision == 2)
        e = cgemm_bf16_launch(d, batch, descs, st, role, big);
    else if (precision == 1)
        e = big ? launch<128, 64, 1>(d, batch, descs, st, role, only) : launch<64, 64, 1>(d, batch, descs, st, role, only);
    else
        e = big ? launch<128, 64, 0>(d, batch, descs, st, role, only) : launch<64, 64, 0>(d, batch, descs, st, role, only);
    if (prof) profile_end(st, tok);
    return e;
}

}  // namespace redo
