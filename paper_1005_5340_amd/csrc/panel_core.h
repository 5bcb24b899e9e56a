// Core of the panel GEMMs (kernels_panel.hip, kernels_crt.hip): dense products
// whose operands lie in 16-byte blocks of consecutive k.
//
// Panel layout.  An operand with R rows (columns of B) and K reduction
// entries is stored in 16-byte blocks (8 of BF16, 16 of INT8): block kb of
// row r is uint4 number kb * ld + r of its plane, ld >= R.  That is what one
// lane of a 32x32 MFMA supplies (lane l: row l % 32, k-block l / 32 of the
// instruction's two), so a tile is a set of contiguous runs in global memory,
// goes straight to LDS (16 bytes per lane, consecutive lanes to consecutive
// addresses) and is read back without bank conflicts and without padding.  A
// and B use the same k order inside a block, so the order itself does not
// matter.  D of a 32x32 MFMA: element r of lane l is row
// 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
#pragma once

#include "common.h"

#include <type_traits>

namespace chi0 {

#define CHI0_GLOBAL __attribute__((address_space(1)))
#define CHI0_LDS __attribute__((address_space(3)))

// Workgroup id -> work id, each of the 8 XCDs on one contiguous range.
__device__ __forceinline__ int panel_xcd(int wid, int n) {
    const int q = n / 8, r = n % 8;
    const int x = wid % 8, local = wid / 8;
    return x * q + (x < r ? x : r) + local;
}

// A BM x BN tile by WM x WN wavefronts of TM x TN 32x32 MFMA tiles; F gives
// the planes PL per operand, the accumulator type and the products of a step.
template <class F, int BM_, int BN_, int WM_, int WN_, int KB_>
struct PanelShape {
    typedef F Form;
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KB = KB_, PL = F::PL, NT = WM * WN * 64;
    static constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    static constexpr int SA = KB * BM, SB = KB * BN, KS = KB / 2;
    static constexpr int STAGE = PL * (SA + SB);   // uint4s of LDS per stage (two are needed)
    static_assert(SA % NT == 0 && SB % NT == 0 && KB % 2 == 0, "whole 16-byte chunks per thread");
    typedef typename F::acc Acc[TM][TN];
};

// B taken from its panels (the other source is in kernels_panel.hip)
struct PanelNoRaw {
    static constexpr bool on = false;
    __device__ __forceinline__ void load(int) {}
    __device__ __forceinline__ void store(uint4 *) {}
};

// acc = the tile's product over KT stages of KB k-blocks, A and B pointing at
// the tile's first k-block and row / column.  Two stages of LDS (s0, s1) are
// filled in turn by direct-to-LDS loads.  The fragments of a step are read
// while the MFMAs of the step before run, also across the stage boundary: the
// last step's fragments are in registers when the workgroup meets at the
// barrier, so the loads that refill the freed stage and the first fragment
// reads of the next one are issued ahead of the last step's MFMAs and a load
// has a whole stage of MFMAs to land.
template <class P, class Raw>
__device__ __forceinline__ void panel_product(typename P::Acc &acc, uint4 *s0, uint4 *s1, int KT,
                                              const uint4 *__restrict__ A, int lda, int64_t apl,
                                              const uint4 *__restrict__ B, int64_t ldb, int64_t bpl, Raw raw) {
    constexpr int BM = P::BM, BN = P::BN, PL = P::PL, NT = P::NT, TM = P::TM, TN = P::TN, SA = P::SA, SB = P::SB,
                  KB = P::KB, KS = P::KS;
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wv % P::WM, wn = wv / P::WM, lr = lane & 31, lk = lane >> 5;

    auto load = [&](uint4 *dst, int kt) {
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) {
#pragma unroll
            for (int c = 0; c < SA / NT; ++c) {
                const int ch = c * NT + t;
                const uint4 *g = A + pl * apl + (int64_t)(kt * KB + ch / BM) * lda + ch % BM;
                __builtin_amdgcn_global_load_lds((const CHI0_GLOBAL void *)g,
                                                 (CHI0_LDS void *)(dst + pl * SA + c * NT + wv * 64), 16, 0, 0);
            }
#pragma unroll
            for (int c = 0; c < (Raw::on ? 0 : SB / NT); ++c) {
                const int ch = c * NT + t;
                const uint4 *g = B + pl * bpl + (int64_t)(kt * KB + ch / BN) * ldb + ch % BN;
                __builtin_amdgcn_global_load_lds((const CHI0_GLOBAL void *)g,
                                                 (CHI0_LDS void *)(dst + PL * SA + pl * SB + c * NT + wv * 64), 16,
                                                 0, 0);
            }
        }
        raw.load(kt);
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    uint4 fa[2][PL][TM], fb[2][PL][TN];   // fragments of two steps
    auto read = [&](int w, const uint4 *src, int ks) {
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[w][pl][j] = src[PL * SA + pl * SB + (2 * ks + lk) * BN + wn * (BN / P::WN) + j * 32 + lr];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[w][pl][i] = src[pl * SA + (2 * ks + lk) * BM + wm * (BM / P::WM) + i * 32 + lr];
        }
    };
    auto mma = [&](int w) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                uint4 a[PL], b[PL];
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) {
                    a[pl] = fa[w][pl][i];
                    b[pl] = fb[w][pl][j];
                }
                acc[i][j] = P::Form::mma(a, b, acc[i][j]);
            }
    };
    // every wavefront's loads have landed and every fragment read is done
    auto meet = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        __syncthreads();
    };
    // Stage kt in `cur`, its first step's fragments already in set W0.  Past the
    // last stage the fragment read of `nxt` takes what LDS holds and is not used.
    auto stage = [&](auto W0, uint4 *cur, uint4 *nxt, int kt) {
        constexpr int w0 = decltype(W0)::value;
#pragma unroll
        for (int ks = 0; ks + 1 < KS; ++ks) {
            read((w0 + ks + 1) & 1, cur, ks + 1);
            __builtin_amdgcn_sched_barrier(0);
            mma((w0 + ks) & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (Raw::on && kt + 1 < KT) raw.store(nxt + PL * SA);
        meet();
        if (kt + 2 < KT) load(cur, kt + 2);
        read((w0 + KS) & 1, nxt, 0);
        __builtin_amdgcn_sched_barrier(0);
        mma((w0 + KS - 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
    };
    load(s0, 0);
    raw.store(s0 + PL * SA);
    meet();
    if (KT > 1) load(s1, 1);
    read(0, s0, 0);
    int kt = 0;
    for (; kt + 2 <= KT; kt += 2) {
        stage(std::integral_constant<int, 0>{}, s0, s1, kt);
        stage(std::integral_constant<int, KS & 1>{}, s1, s0, kt + 1);
    }
    if (kt < KT) stage(std::integral_constant<int, 0>{}, s0, s1, kt);
}

}  // namespace chi0
