// The virtual-orbital transforms (Sec. 4.2, Table t:flops steps 3 and 4) of the
// low-precision operator, on BF16 panels (panel_core.h).
#include "panel_core.h"

namespace chi0 {

// Tiles of 128x128 from which those are used.  With half as many as CUs they
// beat the 64x64 tiles, whose split-K then needs a reduction (chi0 in split
// BF16, 64x64 against 128x128: 60 atoms, 12 vectors, 135 tiles 196 / 180 us;
// 131 atoms, 5 vectors, 155 tiles 186 / 172 us; 200 atoms, 4 vectors 493 /
// 442 us); below, the split fills the chip better (60 atoms, 4 vectors, 45
// tiles 130 / 146 us; 100 atoms, 3 vectors, 68 tiles 139 / 154 us).
constexpr int PANEL_BIG = 128;

typedef float flt16 __attribute__((ext_vector_type(16)));
typedef float flt2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr float BF16_MAX = 0x1.FEp127f;

// One k-block of 8 values as PL planes: bf16(x), then one BF16 of what the
// planes before leave (all to nearest even); x is overwritten.  With three planes
// the first one stops at the largest finite BF16, so that FP32 values which would
// round past it (above 3.39e38) are held too.  An infinity gives NaN: its
// remainder has none.
template <int PL>
__device__ __forceinline__ void panel_cut(float (&x)[8], uint4 (&out)[PL]) {
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) {
        uint32_t w[4];
#pragma unroll
        for (int c = 0; c < 8; c += 2) {
            flt2 v{x[c], x[c + 1]};
            if (PL == 3 && pl == 0)
                v = flt2{__builtin_amdgcn_fmed3f(v.x, -BF16_MAX, BF16_MAX), __builtin_amdgcn_fmed3f(v.y, -BF16_MAX, BF16_MAX)};
            const bf16x2 h = __builtin_convertvector(v, bf16x2);
            w[c / 2] = __builtin_bit_cast(uint32_t, h);
            x[c] -= __uint_as_float(w[c / 2] << 16);
            x[c + 1] -= __uint_as_float(w[c / 2] & 0xFFFF0000u);
        }
        out[pl] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// C [M][ldc] (FP32) = A B, A and B as PL planes of BF16 (hi, then the
// rounded remainders).  PL = 2 (split BF16 x 3) sums lo hi + hi lo + hi hi,
// which drops parts of 2^-17 of a product.  PL = 3 holds an FP32 value whole
// (3 x 8 bits; one below 2^-110 to 2^-134, half of the least BF16 subnormal) and
// sums the six products of planes x + y <= 2, smallest first: the rest is below
// 2^-25 of a product, under the rounding of the FP32 accumulation.
//
// blockIdx.y selects a k range of nkb_split k-blocks (at least one stage),
// whose raw sums go to a C slice of their own.
//
// Bound by the matrix cores' sustained rate: 128x128 tiles execute 1.0-1.1
// PFLOP/s of BF16 (a library product of 8192^3 reaches 1.05 on this card).
// The 64x64-tile kernel with 16x16x32 MFMAs and operands staged through
// registers that this replaces was bound by its LDS reads (a 16-byte fragment
// per 1.5 MFMAs; here one per 1.5 MFMAs of twice the work) and ran at 0.54:
// 400-atom transforms of 32 vectors (3200 x 128000 x 5200) 23.6 and 22.3 ms
// before, 12.4 and 11.9 ms now; 200 atoms, 24 vectors 705 and 663 -> 480 and
// 390 us.  The frequency factor costs 64 outputs per lane some 20 FP64
// instructions each; with two divisions, LDS lane exchanges and loads between
// the stores it was 20-25 us per launch of one round of tiles, now 8-15.
//
// RAW takes B as it is, FP32 [K][ldb], and cuts it into planes on the way to
// LDS: each thread loads the 8 values of one k-block of one column a stage
// ahead and stores its planes before the workgroup meets.  Every row of tiles
// cuts B again, so it is for few rows of tiles, where it saves a launch
// (3-5 us of a 45-130 us chi0).
//
// PL = 3 replaces FP32 MFMA (157 TFLOP/s peak, 75-82 reached): chi0 in FP32
// 131 atoms, 24 vectors 611 -> 479 us, 200 atoms, 24 vectors 3.31 -> 2.57 ms,
// 400 atoms, 8 vectors 19.5 -> 14.0 ms; its error against 64 bits is a tenth
// smaller (4.3e-7 -> 3.8e-7 of chi0 z).
template <int PL_>
struct FormBF {
    static constexpr int PL = PL_;
    typedef flt16 acc;
    static __device__ __forceinline__ acc mma(const uint4 (&a)[PL], const uint4 (&b)[PL], acc c) {
        auto mm = [&](int x, int y) {
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[x]),
                                                        __builtin_bit_cast(bf16x8, b[y]), c, 0, 0, 0);
        };
        if constexpr (PL == 3) {
            mm(2, 0);
            mm(0, 2);
            mm(1, 1);
        }
        mm(1, 0);
        mm(0, 1);
        mm(0, 0);
        return c;
    }
};

// FP32 column of B cut on the way to LDS: thread t takes k-block t / BN of
// the stage in column t % BN.
template <class P>
struct PanelRaw {
    static constexpr bool on = true;
    static_assert(P::SB == P::NT, "one k-block of B per thread");
    const float *src;   // row 0 of the thread's column
    int64_t ldb;
    int k_first, K;     // first k of stage 0 for this thread
    bool ok;
    float x[8];
    __device__ __forceinline__ void load(int kt) {
        const int k0 = k_first + kt * P::KB * 8;
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = (ok && k0 + c < K) ? src[(int64_t)(k0 + c) * ldb] : 0.f;
    }
    __device__ __forceinline__ void store(uint4 *dst) {
        uint4 w[P::PL];
        panel_cut<P::PL>(x, w);
#pragma unroll
        for (int pl = 0; pl < P::PL; ++pl) dst[pl * P::SB + threadIdx.x] = w[pl];
    }
};

template <class P, bool LORENTZ, bool RAW>
__global__ __launch_bounds__(P::NT)
void k_panel_gemm(int M, int N, int K, int ntm, int ntn, int nkb, int nkb_split, const uint4 *__restrict__ A,
                  int lda, int64_t apl, const void *__restrict__ Bv, int64_t ldb, int64_t bpl, float *__restrict__ C,
                  int ldc, int col0, LorentzArgs la) {
    constexpr int BM = P::BM, BN = P::BN, WM = P::WM, WN = P::WN, TM = P::TM, TN = P::TN;
    __shared__ uint4 s0[P::STAGE], s1[P::STAGE];
    const int tile = panel_xcd(blockIdx.x, ntm * ntn);
    const int m0 = (tile % ntm) * BM, n0 = (tile / ntm) * BN;
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wv % WM, wn = wv / WM, lr = lane & 31, lk = lane >> 5;
    const int kb0 = blockIdx.y * nkb_split, KT = min(nkb_split, nkb - kb0) / P::KB;
    A += (int64_t)kb0 * lda + m0;
    C += (int64_t)blockIdx.y * M * ldc;
    typename P::Acc acc;
    if constexpr (RAW) {
        const int n = n0 + t % BN;
        PanelRaw<P> raw{static_cast<const float *>(Bv) + n, ldb, (kb0 + t / BN) * 8, K, n < N, {}};
        panel_product<P>(acc, s0, s1, KT, A, lda, apl, (const uint4 *)nullptr, 0, 0, raw);
    } else {
        panel_product<P>(acc, s0, s1, KT, A, lda, apl, static_cast<const uint4 *>(Bv) + (int64_t)kb0 * ldb + n0, ldb,
                         bpl, PanelNoRaw{});
    }

#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = n0 + wn * (BN / WN) + j * 32 + lr;
        const bool ok = col < N;
        const int cc = ok ? col0 + col : 0, E = LORENTZ ? cc / la.ncp : 0, jj = LORENTZ ? cc - E * la.ncp : 0;
        const Lorentz lz(LORENTZ ? la.omega[jj >> 1] : 0.0, la.eps, la.occ, jj & 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            // element 4 q + r: row row0 + 8 q + r, four consecutive rows (the frequency
            // factor's M is a multiple of 64)
            const int row0 = m0 + wm * (BM / WM) + i * 32 + 4 * lk;
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = acc[i][j][r];
            if (LORENTZ) {
                // the transition energies of the 16 rows first: loaded between the
                // stores each would wait for a memory latency of its own
                double2 D[8];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = row0 + 8 * q;
                    const double2 *d = reinterpret_cast<const double2 *>(la.Dlt + (int64_t)E * la.nv_pad +
                                                                         (row < M ? row : 0));
                    D[2 * q] = d[0];
                    D[2 * q + 1] = d[1];
                }
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    v[r] = (float)lz.apply(r & 1 ? D[r / 2].y : D[r / 2].x, v[r], lane_pair(v[r]));
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = row0 + 8 * (r / 4) + r % 4;
                if (ok && row < M) __builtin_nontemporal_store(v[r], &C[(int64_t)row * ldc + col]);
            }
        }
    }
}

// X [K][ldx] -> PL planes of BF16 panels, columns n < N (zero for k >= K and
// up to ld): plane 0 holds bf16(x), each further one bf16 of what the planes
// before leave.  Thread (kb, n) reads the 8 rows of its block in column n
// (coalesced over n) and writes 16 bytes per plane.
template <int PL, class T>
__global__ __launch_bounds__(256)
void k_panel_split(const T *__restrict__ X, int K, int N, int64_t ldx, int nkb, int ld, uint4 *__restrict__ out,
                   int64_t plane) {
    const int64_t total = (int64_t)nkb * ld;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
        const int kb = (int)(idx / ld), n = (int)(idx % ld);
        float x[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int k = kb * 8 + c;
            x[c] = (n < N && k < K) ? (float)X[(int64_t)k * ldx + n] : 0.f;
        }
        uint4 w[PL];
        panel_cut<PL>(x, w);
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) out[pl * plane + idx] = w[pl];
    }
}

__global__ __launch_bounds__(256) void k_to_f32(const double *__restrict__ x, float *__restrict__ y, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        y[i] = (float)x[i];
}

template <int PL, class T>
static void split_any(hipStream_t s, const T *X, int K, int N, int64_t ldx, int nkb, int ld, uint4 *out,
                      int64_t plane) {
    int64_t blocks = ((int64_t)nkb * ld + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL((k_panel_split<PL, T>), dim3((unsigned)blocks), dim3(256), 0, s, X, K, N, ldx, nkb, ld, out,
                       plane);
}

void launch_panel_bf16(hipStream_t s, const double *X, int K, int N, int64_t ldx, PanelDev *p) {
    split_any<PANEL_BF, double>(s, X, K, N, ldx, p->nkb, p->ld, reinterpret_cast<uint4 *>(p->data), p->plane);
}

template <int PL, int BM, int BN, bool LORENTZ, bool RAW>
static void panel_launch(hipStream_t s, int M, int N, int K, int S, int nkb_split, const PanelDev &A, const void *B,
                         int64_t ldb, float *C, int ldc, int col0, const LorentzArgs &la) {
    const int ntm = (M + BM - 1) / BM, ntn = (N + BN - 1) / BN;
    typedef PanelShape<FormBF<PL>, BM, BN, 2, 2, PL * BM <= 256 ? 4 : 2> P;
    hipLaunchKernelGGL((k_panel_gemm<P, LORENTZ, RAW>), dim3(ntm * ntn, S), dim3(P::NT), 0, s, M, N, K, ntm, ntn, A.nkb, nkb_split, reinterpret_cast<const uint4 *>(A.data),
                       A.ld, A.plane, B, ldb, (int64_t)A.nkb * ldb, C, ldc, col0, la);
}

template <int PL>
static void panel_gemm_any(Tracer *t, hipStream_t s, const char *name, int M, int N, int K, const PanelDev &A,
                           const float *B, int64_t ldb, void *work, size_t work_bytes, void *scratch,
                           size_t scratch_bytes, float *C, int ldc, double flops, double bytes,
                           const LorentzArgs *la) {
    const int nkb = A.nkb, KT = nkb / PANEL_KB;
    const LorentzArgs none{};
    if ((int64_t)((M + 127) / 128) * ((N + 127) / 128) < PANEL_BIG) {
        // 64x64 tiles, B cut in the kernel; k splits of at least 4 stages
        const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
        int S = 1;
        while (scratch && S < 16 && tiles * S < 1024 && KT / (2 * S) >= 4 &&
               (size_t)(2 * S) * M * (size_t)N * sizeof(float) <= scratch_bytes)
            S *= 2;
        const int kts = (KT + S - 1) / S;
        S = (KT + kts - 1) / kts;
        trace_begin(t, name, s);
        if (S > 1)
            panel_launch<PL, 64, 64, false, true>(s, M, N, K, S, kts * PANEL_KB, A, B, ldb,
                                                  static_cast<float *>(scratch), N, 0, none);
        else if (la)
            panel_launch<PL, 64, 64, true, true>(s, M, N, K, 1, nkb, A, B, ldb, C, ldc, 0, *la);
        else
            panel_launch<PL, 64, 64, false, true>(s, M, N, K, 1, nkb, A, B, ldb, C, ldc, 0, none);
        trace_end(t, s, flops, bytes);
        if (S > 1) launch_splitk_reduce_f32(t, s, M, N, S, static_cast<const float *>(scratch), C, ldc, la);
        return;
    }
    // columns whose B panels fit the workspace at once
    const int64_t fit = (int64_t)(work_bytes / ((size_t)PL * nkb * 16)) / PANEL_LD * PANEL_LD;
    const int nch = (int)((N + fit - 1) / fit), chunk = (int)round_up((N + nch - 1) / nch, PANEL_LD);   // equal chunks
    uint4 *bp = static_cast<uint4 *>(work);
    for (int c0 = 0; c0 < N; c0 += chunk) {
        const int n = std::min(chunk, N - c0), ld = (int)round_up(n, PANEL_LD);
        const double share = (double)n / N;
        trace_begin(t, "bf16_split", s);
        split_any<PL, float>(s, B + c0, K, n, ldb, nkb, ld, bp, (int64_t)nkb * ld);
        trace_end(t, s, 0.0, (4.0 + 2.0 * PL) * (double)K * n);
        trace_begin(t, name, s);
        if (la)
            panel_launch<PL, 128, 128, true, false>(s, M, n, K, 1, nkb, A, bp, ld, C + c0, ldc, c0, *la);
        else
            panel_launch<PL, 128, 128, false, false>(s, M, n, K, 1, nkb, A, bp, ld, C + c0, ldc, c0, none);
        trace_end(t, s, flops * share, bytes * share);
    }
}

void launch_panel_gemm(Tracer *t, hipStream_t s, const char *name, int planes, int M, int N, int K,
                       const PanelDev &A, const float *B, int64_t ldb, void *work, size_t work_bytes, void *scratch,
                       size_t scratch_bytes, float *C, int ldc, double flops, double bytes, const LorentzArgs *la) {
    if (planes == 2)
        panel_gemm_any<2>(t, s, name, M, N, K, A, B, ldb, work, work_bytes, scratch, scratch_bytes, C, ldc, flops,
                          bytes, la);
    else
        panel_gemm_any<3>(t, s, name, M, N, K, A, B, ldb, work, work_bytes, scratch, scratch_bytes, C, ldc, flops,
                          bytes, la);
}

void launch_to_f32(hipStream_t s, const double *x, float *y, int64_t n) {
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (n > 0) hipLaunchKernelGGL(k_to_f32, dim3((unsigned)blocks), dim3(256), 0, s, x, y, n);
}

}  // namespace chi0
