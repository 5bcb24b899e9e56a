// Matrix-core kernels of the orbital transforms (Sec. 4.2, Table t:flops steps
// 2-5) and the kernel matrix-vector product (Sec. 4.1): the FP64 dense GEMMs
// and the gathered occupied transforms in FP64 and FP32.
//
// A 16 x 16 output tile per K step of 4 on 64-lane wavefronts, lane l = 0..63:
//   B (4 x 16):  lane l holds B[l / 16][l % 16]
//   D (16 x 16): element r of lane l holds D[row(l, r)][l % 16]
// FP64 uses v_mfma_f64_4x4x4_4b_f64: four 4x4x4 products per instruction,
// lane l = 16 h + 4 q + p holding A[q-th block][p][h], B[block q][h][p] and
// D[block q][h][p].  Issuing one instruction per 4-row strip r of the tile,
// with block q = the 4-column group of B, makes B and D the same lanes as a
// 16x16x4 product:  A fragment r holds A[4r + l % 4][l / 16], and
// row(l, r) = 4r + l/16.  On gfx950 this form runs at ~72 TFLOP/s against
// ~50 for v_mfma_f64_16x16x4f64 (register-only throughput probes).
// FP32 uses v_mfma_f32_16x16x4f32: A[l % 16][l / 16], row(l, r) = 4(l/16) + r.
// (Lane layouts checked on gfx950 with one-hot lane probes.)
#include "common.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace chi0 {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef float flt4 __attribute__((ext_vector_type(4)));

// NA A fragments per 16 x 16 tile and K step; a_row(l, r) is the tile row
// that lane l supplies in fragment r.
struct Mma4 {
    typedef dbl4 acc;
    static constexpr int NA = 4;
    static __device__ __forceinline__ acc zero() { return acc{0.0, 0.0, 0.0, 0.0}; }
    static __device__ __forceinline__ int a_row(int lane, int r) { return 4 * r + (lane & 3); }
    static __device__ __forceinline__ acc op(const double (&a)[NA], double b, acc c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[r], b, c[r], 0, 0, 0);
        return c;
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }
};
// The kernels for few columns take the single 16x16x4 FP64 product per tile
// (A[l % 16][l / 16]): they wait on memory, not on the MFMA rate, and load one
// value of A per lane and k step instead of four.
struct Mma16d {
    typedef dbl4 acc;
    static constexpr int NA = 1;
    static __device__ __forceinline__ acc zero() { return acc{0.0, 0.0, 0.0, 0.0}; }
    static __device__ __forceinline__ int a_row(int lane, int) { return lane & 15; }
    static __device__ __forceinline__ acc op(const double (&a)[NA], double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }
    // row R of the tile is element elem(R) of the lanes 16 quarter(R) ... + 15
    static __device__ __forceinline__ int elem(int R) { return R >> 2; }
    static __device__ __forceinline__ int quarter(int R) { return R & 3; }
};
struct Mma16f {
    typedef flt4 acc;
    static constexpr int NA = 1;
    static __device__ __forceinline__ acc zero() { return acc{0.f, 0.f, 0.f, 0.f}; }
    static __device__ __forceinline__ int a_row(int lane, int) { return lane & 15; }
    static __device__ __forceinline__ acc op(const float (&a)[NA], float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
    static __device__ __forceinline__ int elem(int R) { return R & 3; }
    static __device__ __forceinline__ int quarter(int R) { return R >> 2; }
};

// four consecutive elements (16 B aligned for float, 2 x 16 B for double)
__device__ __forceinline__ void load4(const double *p, double *v) {
    const double2 a = reinterpret_cast<const double2 *>(p)[0], b = reinterpret_cast<const double2 *>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ __forceinline__ void load4(const float *p, float *v) {
    const float4 a = reinterpret_cast<const float4 *>(p)[0];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
}

// Workgroup id -> tile id such that each of the 8 XCDs (which receive
// consecutive workgroup ids round robin) works on one contiguous range of
// tiles; tiles that share an operand strip then share that XCD's L2.
__device__ __forceinline__ int xcd_remap(int wid, int n) {
    const int q = n / 8, r = n % 8;
    const int x = wid % 8, local = wid / 8;
    return x * q + (x < r ? x : r) + local;
}

// ------------------------------------------------------------------ dense GEMM
// C[M x N] = A[M x K] B[K x N], row-major, M % BM == 0, K % 16 == 0, N masked.
// Optional epilogue (b2)+(c): C column n <-> (E, j) with E = n / ncp,
// j = n % ncp; columns 2r and 2r+1 hold Re and Im of RHS r; row = virtual F.
// Split-K: blockIdx.y selects a K range of length K (the per-split length);
// A and B are advanced by it and each split writes raw partial sums to its
// own C slice (C + split * M * ldc), summed later by k_splitk_reduce.
// The tile shape (BM x BN, WM x WN wavefronts) changes only which workgroup
// computes an element, never the order of its k accumulation, so every tile
// variant gives bit-identical results and the autotuner may pick any of them.
template <int BM, int BN, int WM, int WN, bool LORENTZ, int BK>
__device__ __forceinline__ void dgemm_tile(int m0, int n0, int N, int K, const double *__restrict__ A, int lda,
                                           const double *__restrict__ B, int ldb, double *__restrict__ C, int ldc,
                                           int col0, const LorentzArgs &la) {
    constexpr int NT = WM * WN * 64;
    constexpr int TM = BM / WM / 16;
    constexpr int TN = BN / WN / 16;
    constexpr int CA = BM * (BK / 4) / NT;   // 4-element A chunks per thread per tile
    constexpr int CB = BK * (BN / 4) / NT;   // 4-element B chunks per thread per tile
    static_assert(CA >= 1 && CB >= 1 && CA * NT == BM * (BK / 4) && CB * NT == BK * (BN / 4),
                  "tile shape must split into whole 4-element chunks per thread");
    __shared__ double As[2][BK][BM + 1];
    __shared__ double Bs[2][BK][BN];

    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int wm = wv % WM, wn = wv / WM;

    // global -> register mapping: chunk q of a thread is chunk t + q NT of the tile
    int a_row[CA], a_k[CA], b_k[CB], b_n[CB];
#pragma unroll
    for (int q = 0; q < CA; ++q) {
        const int ch = t + q * NT;
        a_row[q] = ch / (BK / 4);
        a_k[q] = (ch % (BK / 4)) * 4;
    }
#pragma unroll
    for (int q = 0; q < CB; ++q) {
        const int ch = t + q * NT;
        b_k[q] = ch / (BN / 4);
        b_n[q] = (ch % (BN / 4)) * 4;
    }

    double ra[CA][4], rb[CB][4];
    auto load = [&](int kt) {
#pragma unroll
        for (int q = 0; q < CA; ++q) load4(A + (int64_t)(m0 + a_row[q]) * lda + kt * BK + a_k[q], ra[q]);
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            const double *bp = B + (int64_t)(kt * BK + b_k[q]) * ldb + n0 + b_n[q];
            if (n0 + b_n[q] + 3 < N) {
                load4(bp, rb[q]);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) rb[q][c] = (n0 + b_n[q] + c < N) ? bp[c] : 0.0;
            }
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int q = 0; q < CA; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) As[buf][a_k[q] + c][a_row[q]] = ra[q][c];
#pragma unroll
        for (int q = 0; q < CB; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) Bs[buf][b_k[q]][b_n[q] + c] = rb[q][c];
    };

    Mma4::acc acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = Mma4::zero();

    const int KT = K / BK;
    load(0);
    store(0);
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < KT) load(kt + 1);
#pragma unroll
        for (int ks = 0; ks < BK / 4; ++ks) {
            const int kk = ks * 4 + lane / 16;
            double af[TM][Mma4::NA], bf[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < Mma4::NA; ++r)
                    af[i][r] = As[cur][kk][wm * (BM / WM) + i * 16 + Mma4::a_row(lane, r)];
#pragma unroll
            for (int j = 0; j < TN; ++j) bf[j] = Bs[cur][kk][wn * (BN / WN) + j * 16 + (lane & 15)];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = Mma4::op(af[i], bf[j], acc[i][j]);
        }
        if (kt + 1 < KT) store(cur ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = n0 + wn * (BN / WN) + j * 16 + (lane & 15);
        const bool ok = col < N;
        const int cc = ok ? col0 + col : 0, E = LORENTZ ? cc / la.ncp : 0, jj = LORENTZ ? cc - E * la.ncp : 0;
        const Lorentz lz(LORENTZ ? la.omega[jj >> 1] : 0.0, la.eps, la.occ, jj & 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int rbase = m0 + wm * (BM / WM) + i * 16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = rbase + Mma4::row(lane, r);
                double v = acc[i][j][r];
                if (LORENTZ) v = lz.apply(la.Dlt[(int64_t)E * la.nv_pad + row], v, lane_pair(v));
                // the output is read by the next kernel only: a streaming store
                if (ok) __builtin_nontemporal_store(v, &C[(int64_t)row * ldc + col]);
            }
        }
    }
}

template <int BM, int BN, int WM, int WN, bool LORENTZ, int BK = 16>
__global__ __launch_bounds__(WM * WN * 64)
void k_dgemm(int M, int N, int K, const double *__restrict__ A, int lda,
             const double *__restrict__ B, int ldb, double *__restrict__ C, int ldc,
             int m_fastest, LorentzArgs la) {
    const int ntm = M / BM, ntn = (N + BN - 1) / BN;
    const int tile = xcd_remap(blockIdx.x, ntm * ntn);
    const int tm = m_fastest ? tile % ntm : tile / ntn;
    const int tn = m_fastest ? tile / ntm : tile % ntn;
    dgemm_tile<BM, BN, WM, WN, LORENTZ, BK>(tm * BM, tn * BN, N, K, A + (int64_t)blockIdx.y * K, lda,
                                            B + (int64_t)blockIdx.y * K * ldb, ldb,
                                            C + (int64_t)blockIdx.y * M * ldc, ldc, 0, la);
}

// The 64 x 64 tiles of a product that lie in a flagged tile; row tiles fastest.
template <bool LORENTZ>
__global__ __launch_bounds__(256)
void k_dgemm_flagged(int ntm, int N, int K, const double *__restrict__ A, int lda, const double *__restrict__ B,
                     int ldb, double *__restrict__ C, int ldc, int col0, LorentzArgs la,
                     const uint8_t *__restrict__ flag, int fn) {
    const int m0 = blockIdx.x % ntm * 64, n0 = blockIdx.x / ntm * 64;
    if (!flag[m0 / CRT_FM * fn + n0 / CRT_FN]) return;
    dgemm_tile<64, 64, 2, 2, LORENTZ, 16>(m0, n0, N, K, A, lda, B, ldb, C, ldc, col0, la);
}

// C = sum over splits of the partial products; optional Lorentzian epilogue.
template <class T>
__global__ __launch_bounds__(256)
void k_splitk_reduce(int M, int N, int S, const T *__restrict__ part, int64_t slice,
                     T *__restrict__ C, int ldc, int factor, LorentzArgs la) {
    const int64_t npair = (int64_t)M * ((N + 1) / 2);
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < npair;
         idx += (int64_t)gridDim.x * 256) {
        const int row = (int)(idx / ((N + 1) / 2));
        const int col = 2 * (int)(idx % ((N + 1) / 2));
        const int64_t o = (int64_t)row * ldc + col;
        const int64_t op = (int64_t)row * N + col;
        const bool two = col + 1 < N;
        double re = 0.0, im = 0.0;
        for (int s2 = 0; s2 < S; ++s2) {
            re += (double)part[s2 * slice + op];
            if (two) im += (double)part[s2 * slice + op + 1];
        }
        if (factor) {
            const int E = col / la.ncp, jj = col - E * la.ncp;
            const double D = la.Dlt[(int64_t)E * la.nv_pad + row], w = la.omega[jj >> 1], re0 = re;
            re = Lorentz(w, la.eps, la.occ, 0).apply(D, re0, im);
            im = Lorentz(w, la.eps, la.occ, 1).apply(D, im, re0);
        }
        C[o] = (T)re;
        if (two) C[o + 1] = (T)im;
    }
}

// C = A B (+ Lorentzian factor) for few columns.  One workgroup: 16 TM x 16 TN
// outputs; its NW waves take turns over k, 8 KU at a time straight into registers
// (a lane loads two adjacent k of A; they feed two products whose k slots are the
// lanes' even and odd k), and their sums are added in wave order through LDS,
// where the factor is applied.  K % 16 == 0, N even with the factor.
// The tiled kernel with split K needs a second launch and a pass over the
// partial products there and waits for a barrier per 16 k.
template <int TM, int TN, int NW, int KU, bool LORENTZ>
__global__ __launch_bounds__(NW * 64)
void k_dgemm_few(int N, int K, const double *__restrict__ A, int lda, const double *__restrict__ B, int ldb,
                 double *__restrict__ C, int ldc, LorentzArgs la) {
    __shared__ double red[NW][TM][TN][4][64];
    const int m0 = blockIdx.x * 16 * TM, n0 = blockIdx.y * 16 * TN;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lk = lane >> 4;
    dbl4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = dbl4{0.0, 0.0, 0.0, 0.0};
    for (int k0 = wv * 8 * KU; k0 < K; k0 += NW * 8 * KU) {
        double2 a[KU][TM];
        double b0[KU][TN], b1[KU][TN];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int k = k0 + 8 * u + 2 * lk;
            const bool ok = k < K;
#pragma unroll
            for (int i = 0; i < TM; ++i)
                a[u][i] = ok ? *reinterpret_cast<const double2 *>(A + (int64_t)(m0 + 16 * i + lr) * lda + k)
                             : make_double2(0.0, 0.0);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int n = n0 + 16 * j + lr;
                b0[u][j] = ok && n < N ? B[(int64_t)k * ldb + n] : 0.0;
                b1[u][j] = ok && n < N ? B[(int64_t)(k + 1) * ldb + n] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < KU; ++u)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][i].x, b0[u][j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][i].y, b1[u][j], acc[i][j], 0, 0, 0);
                }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wv][i][j][r][lane] = acc[i][j][r];
    __syncthreads();
    for (int q = t; q < 256 * TM * TN; q += NW * 64) {   // whole wavefronts
        const int row = q / (16 * TN), c = q % (16 * TN), n = n0 + c;
        const int R = row % 16, l = (R & 3) * 16 + c % 16;
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[w][row / 16][c / 16][R >> 2][l];
        if (LORENTZ) {
            const int E = n < N ? n / la.ncp : 0, jj = n < N ? n - E * la.ncp : c & 1;
            const Lorentz lz(la.omega[jj >> 1], la.eps, la.occ, jj & 1);
            v = lz.apply(la.Dlt[(int64_t)E * la.nv_pad + m0 + row], v, lane_pair(v));
        }
        if (n < N) C[(int64_t)(m0 + row) * ldc + n] = v;
    }
}

// Up to 8e8 multiply-adds the split-k form is faster; past that its operand
// reads (32 x 32 tiles) bound it.  16 x 16 tiles up to 2^17 outputs, where the
// larger ones would be fewer than 128 workgroups.  us at M x N x K, tiled kernel and
// its reduction / 16 x 16 / 32 x 32: 64x96x112 8.6 / 2.7 / 3.7; 64x1152x112 9.2 /
// 3.3 / 3.8; 320x480x544 15.3 / 11.0 / 9.4; 320x1440x544 21.7 / 24.7 / 16.4;
// 576x2880x304 (5e8) 37.3 / 45.1 / 29.6.  Against the tiled kernel without split K
// (choose_splits): 320x3840x544 (6.7e8) 45.4 / 35.5, 576x3840x304 36.7 / 36.9,
// 320x4800x544 (8.4e8) 44.4 / 42.3, 576x4800x304 36.7 / 44.4, 320x5760x544 (1e9)
// 46 / 53.9.
constexpr int64_t FEW_WORK = 800000000LL, FEW_SMALL = 131072;

template <int TM, int TN, int NW, int KU>
static void launch_few(Tracer *t, hipStream_t s, const char *name, int M, int N, int K, const double *A, int lda,
                       const double *B, int ldb, double *C, int ldc, double flops, double bytes, bool lorentz,
                       const LorentzArgs &la) {
    const dim3 grid(M / (16 * TM), (N + 16 * TN - 1) / (16 * TN));
    trace_begin(t, name, s);
    if (lorentz)
        hipLaunchKernelGGL((k_dgemm_few<TM, TN, NW, KU, true>), grid, dim3(NW * 64), 0, s, N, K, A, lda, B, ldb, C, ldc,
                           la);
    else
        hipLaunchKernelGGL((k_dgemm_few<TM, TN, NW, KU, false>), grid, dim3(NW * 64), 0, s, N, K, A, lda, B, ldb, C,
                           ldc, la);
    trace_end(t, s, flops, bytes);
}

// Number of K splits: enough workgroups to fill 256 CUs a few times over,
// each split keeping >= 4 K tiles of 16; limited by the scratch capacity.  The
// splits have equal lengths *ks of whole tiles; S *ks may exceed K (the last
// split then sums zero padding) but not kpad, the operands' K extent.  One tile
// per CU is enough to go without: the partial sums' way through memory costs more
// than idle matrix cores (us, split and summed / whole: 320x5760x544 59.8 / 46,
// 576x5760x304 60.0 / 46, 576x3000x576 53.4 / 48.9, 1280x1600x1008 90.7 / 82.2).
static int choose_splits(int M, int N, int K, int kpad, size_t scratch_elems, int *ks) {
    const int tiles = (M / 64) * ((N + 63) / 64);
    const int KT = K / 16;
    int S = 1;
    while (tiles < 256 && S < 16 && tiles * S < 1024) {
        const int S2 = 2 * S, kt2 = (KT + S2 - 1) / S2;
        if (kt2 < 4 || (int64_t)S2 * kt2 * 16 > kpad || (size_t)S2 * M * (size_t)N > scratch_elems) break;
        S = S2;
    }
    *ks = (KT + S - 1) / S * 16;
    return S;
}

template <class T>
static void reduce_splits(Tracer *t, hipStream_t s, int M, int N, int S, const T *scratch, T *C,
                          int ldc, bool lorentz, const LorentzArgs &la) {
    const int64_t npair = (int64_t)M * ((N + 1) / 2);
    int64_t blocks = (npair + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    trace_begin(t, "splitk_reduce", s);
    hipLaunchKernelGGL(k_splitk_reduce<T>, dim3((unsigned)blocks), dim3(256), 0, s, M, N, S, scratch,
                       (int64_t)M * N, C, ldc, lorentz ? 1 : 0, la);
    trace_end(t, s, (double)S * M * N, (double)sizeof(T) * ((double)S + 1.0) * M * N);
}

const char *const kGemmVariantNames[GEMM_VARIANTS] = {"64x64", "64x128", "128x64", "128x128",
                                                      "64x64/k32", "64x128/k32"};
static const int kVarBM[GEMM_VARIANTS] = {64, 64, 128, 128, 64, 64};
static const int kVarBK[GEMM_VARIANTS] = {16, 16, 16, 16, 32, 32};

GemmTuner::~GemmTuner() {
    for (hipEvent_t &e : ev)
        if (e) (void)hipEventDestroy(e);
}

template <bool LZ>
static void launch_variant(int v, hipStream_t s, dim3 grid_s, int M, int N, int K, const double *A, int lda,
                           const double *B, int ldb, double *C, int ldc, int m_fastest, const LorentzArgs &la) {
    const int S = grid_s.y;
    auto tiles = [&](int bm, int bn) { return (unsigned)((M / bm) * ((N + bn - 1) / bn)); };
    switch (v) {
    case 1:
        hipLaunchKernelGGL((k_dgemm<64, 128, 2, 2, LZ>), dim3(tiles(64, 128), S), dim3(256), 0, s,
                           M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        break;
    case 2:
        hipLaunchKernelGGL((k_dgemm<128, 64, 2, 2, LZ>), dim3(tiles(128, 64), S), dim3(256), 0, s,
                           M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        break;
    case 3:
        hipLaunchKernelGGL((k_dgemm<128, 128, 2, 2, LZ>), dim3(tiles(128, 128), S), dim3(256), 0, s,
                           M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        break;
    case 4:
        hipLaunchKernelGGL((k_dgemm<64, 64, 2, 2, LZ, 32>), dim3(tiles(64, 64), S), dim3(256), 0, s,
                           M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        break;
    case 5:
        hipLaunchKernelGGL((k_dgemm<64, 128, 2, 2, LZ, 32>), dim3(tiles(64, 128), S), dim3(256), 0, s,
                           M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        break;
    default:
        hipLaunchKernelGGL((k_dgemm<64, 64, 2, 2, LZ>), dim3(tiles(64, 64), S), dim3(256), 0, s,
                           M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        break;
    }
}

// Variant for this call: the tuned one for its key, tuning first if the key is new.
template <bool LZ>
static int pick_variant(GemmTuner *tu, hipStream_t s, const char *name, int S, int M, int N, int K,
                        const double *A, int lda, const double *B, int ldb, double *C, int ldc, int m_fastest,
                        const LorentzArgs &la) {
    if (!tu) return 0;
    if (tu->force >= 0 && tu->force < GEMM_VARIANTS)
        return (M % kVarBM[tu->force] == 0 && K % kVarBK[tu->force] == 0) ? tu->force : 0;
    if (!tu->enabled) return 0;
    const int nb = (int)std::floor(2.0 * std::log2((double)std::max(N, 1)));
    const std::string key = std::string(name) + " M=" + std::to_string(M) +
                            " K=" + std::to_string(K * S) + " S=" + std::to_string(S) + " N~2^" +
                            std::to_string(nb / 2) + (nb % 2 ? ".5" : "");
    auto it = tu->table.find(key);
    if (it != tu->table.end()) return it->second.variant;
    GemmTuner::Entry e;
    for (hipEvent_t &ev : tu->ev)
        if (!ev && hipEventCreate(&ev) != hipSuccess) return 0;
    float best = 0.f;
    for (int v = 0; v < GEMM_VARIANTS; ++v) {
        if (M % kVarBM[v] != 0 || K % kVarBK[v] != 0) continue;
        launch_variant<LZ>(v, s, dim3(1, S), M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        // best of three timed launches: one launch's time varies by several per cent
        float tmin = 0.f;
        for (int rep = 0; rep < 3; ++rep) {
            (void)hipEventRecord(tu->ev[0], s);
            launch_variant<LZ>(v, s, dim3(1, S), M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
            (void)hipEventRecord(tu->ev[1], s);
            float ms = 0.f;
            if (hipEventSynchronize(tu->ev[1]) != hipSuccess ||
                hipEventElapsedTime(&ms, tu->ev[0], tu->ev[1]) != hipSuccess)
                return 0;
            tmin = rep == 0 ? ms : std::min(tmin, ms);
        }
        e.us[v] = 1e3f * tmin;
        if (best == 0.f || e.us[v] < best) {
            best = e.us[v];
            e.variant = v;
        }
    }
    tu->table.emplace(key, e);
    return e.variant;
}

static void gemm_any(Tracer *t, hipStream_t s, const char *name, int M, int N, int K, int kpad,
                     const double *A, int lda, const double *B, int ldb, double *C, int ldc,
                     double flops, double bytes, bool lorentz, const LorentzArgs &la,
                     void *scratch, size_t scratch_bytes, GemmTuner *tu) {
    if ((int64_t)M * N * K <= FEW_WORK) {   // whatever the tuner's mode: results never depend on it
        if ((int64_t)M * N <= FEW_SMALL)
            launch_few<1, 1, 8, 4>(t, s, name, M, N, K, A, lda, B, ldb, C, ldc, flops, bytes, lorentz, la);
        else
            launch_few<2, 2, 8, 2>(t, s, name, M, N, K, A, lda, B, ldb, C, ldc, flops, bytes, lorentz, la);
        return;
    }
    int ks = K;
    const int S = scratch ? choose_splits(M, N, K, kpad, scratch_bytes / sizeof(double), &ks) : 1;
    const int m_fastest = (M / 64) <= ((N + 63) / 64);
    if (S == 1) {
        if (lorentz) {
            const int v = pick_variant<true>(tu, s, name, 1, M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
            trace_begin(t, name, s);
            launch_variant<true>(v, s, dim3(1, 1), M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        } else {
            const int v = pick_variant<false>(tu, s, name, 1, M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
            trace_begin(t, name, s);
            launch_variant<false>(v, s, dim3(1, 1), M, N, K, A, lda, B, ldb, C, ldc, m_fastest, la);
        }
        trace_end(t, s, flops, bytes);
        return;
    }
    // partial products with ldc = N into scratch, then the reduction (+ epilogue)
    double *part = static_cast<double *>(scratch);
    const int v = pick_variant<false>(tu, s, name, S, M, N, ks, A, lda, B, ldb, part, N, m_fastest, la);
    trace_begin(t, name, s);
    launch_variant<false>(v, s, dim3(1, S), M, N, ks, A, lda, B, ldb, part, N, m_fastest, la);
    trace_end(t, s, flops, bytes);
    reduce_splits<double>(t, s, M, N, S, part, C, ldc, lorentz, la);
}

void launch_dgemm(Tracer *t, hipStream_t s, const char *name, int M, int N, int K, int kpad,
                  const double *A, int lda, const double *B, int ldb, double *C, int ldc,
                  double flops, double bytes, double *scratch, size_t scratch_doubles, GemmTuner *tu) {
    LorentzArgs la{};
    gemm_any(t, s, name, M, N, K, kpad, A, lda, B, ldb, C, ldc, flops, bytes, false, la, scratch,
                     scratch_doubles * sizeof(double), tu);
}

void launch_dgemm_lorentz(Tracer *t, hipStream_t s, int M, int N, int K, int kpad,
                          const double *A, int lda, const double *B, int ldb, double *C, int ldc,
                          const double *Dlt, int nv_pad, const double *omega, double eps,
                          double occ, int ncp, double flops, double bytes, double *scratch,
                          size_t scratch_doubles, GemmTuner *tu) {
    LorentzArgs la{Dlt, omega, nv_pad, ncp, eps, occ};
    gemm_any(t, s, "virt_transform_lorentz", M, N, K, kpad, A, lda, B, ldb, C, ldc, flops, bytes,
                     true, la, scratch, scratch_doubles * sizeof(double), tu);
}

void launch_dgemm_flagged(hipStream_t s, int M, int N, int K, const double *A, int lda, const double *B, int ldb,
                          double *C, int ldc, int col0, const LorentzArgs *la, const uint8_t *flag, int fn) {
    const int ntm = M / 64;
    const dim3 grid((unsigned)((int64_t)ntm * ((N + 63) / 64)));
    LorentzArgs none{};
    hipLaunchKernelGGL(la ? k_dgemm_flagged<true> : k_dgemm_flagged<false>, grid, dim3(256), 0, s, ntm, N, K, A, lda, B,
                       ldb, C, ldc, col0, la ? *la : none, flag, fn);
}

void launch_splitk_reduce_f32(Tracer *t, hipStream_t s, int M, int N, int S, const float *part,
                              float *C, int ldc, const LorentzArgs *la) {
    LorentzArgs none{};
    reduce_splits<float>(t, s, M, N, S, part, C, ldc, la != nullptr, la ? *la : none);
}

template <class T> struct OccMma;      // tiles staged in LDS
template <class T> struct OccFewMma;   // operands straight from memory: one A value per lane
template <> struct OccFewMma<double> { typedef Mma16d type; };
template <> struct OccFewMma<float> { typedef Mma16f type; };
template <> struct OccMma<double> { typedef Mma4 type; };
template <> struct OccMma<float> { typedef Mma16f type; };

// ------------------------------------------------------- (b1) occupied transform
// The gathered transforms multiply by one atom's orbitals b at a time, for every
// column j; their output columns are the packed pairs n = b nc + j of the column
// atom (nB nc of them), cut into tiles.  A few right-hand sides therefore fill
// the tiles: one complex vector (nc = 2) on a 9-orbital atom is 18 pairs, two
// 16-column tiles, not nine of which 2 columns are used.
//
// Both large kernels: NW wavefronts of 16 rows (states) each times TN 16-column
// tiles of pairs.  The reduction comes in chunks of 16 through one LDS buffer,
// with the next chunk's loads issued before the current chunk's MFMAs; a second
// buffer was no faster, the workgroups it leaves no room for hide as much.  The
// order of the workgroups decides what is read at once.  Transform: the tiles of
// states of one atom's pairs side by side (they share dV).  Back: the tiles of
// pairs of one row tile, then the atoms, so that few workgroups read the same
// part of Ut at the same time (row tiles side by side: 195 -> 282 us at 60 atoms,
// 256 columns).
// us before (64 rows, 144 pairs, 16x16x4 products) and now, transform + back: 60
// atoms 9 orbitals, 48 columns 54 + 64 -> 45 + 48, 256 columns 203 + 205 -> 175 +
// 181 (43 TFLOP/s); 200 atoms, 24 columns 250 + 294 -> 229 + 287; 400 atoms 13
// orbitals, 32 columns 2677 + 2729 -> 2613 + 2800 (there by the operands' second
// reads); FP32 60 atoms, 120 columns 109 + 73 -> 65 + 64, 131 atoms, 48 columns 82
// + 71 -> 56 + 57; 400 atoms, 64 columns 4607 + 3143 -> 2807 + 2867.
constexpr int OCC_NT = 9;   // most 16-column tiles per workgroup
// wavefronts per workgroup: FP32 tiles are small enough for 128 rows (60 atoms, 48
// columns 64 rows 9 % slower), FP64 with 128 rows 5-17 % slower at few rows per atom
template <class T> constexpr int OCC_WAVES = sizeof(T) == 4 ? 8 : 4;

// pairs (n, n + 1) of one row, n even; PAIR: the row is 16-byte (8 in FP32) aligned
template <class T, bool PAIR, class S>
__device__ __forceinline__ void load_pair(const S *p, bool ok0, bool ok1, T &v0, T &v1) {
    if (PAIR) {
        typedef S vec2 __attribute__((ext_vector_type(2)));
        const vec2 v = ok0 ? *reinterpret_cast<const vec2 *>(p) : vec2{S(0), S(0)};
        v0 = (T)v.x;
        v1 = (T)v.y;
    } else {
        v0 = ok0 ? (T)p[0] : T(0);
        v1 = ok1 ? (T)p[1] : T(0);
    }
}

// Tt[b][E*nc + j] = sum_{A in nbr(B)} sum_{a in A} Xo[a][E] dV[(k(A,B), a, b)][j]
// One workgroup: column atom B, 16 NW occupied states, 16 TN packed pairs.  The
// row numbers of a chunk are loaded one chunk before its operands.  Row g of dV
// holds the pairs of B contiguously (dV[(k, a, b)][j] = dV[k_a nc + n]), so a
// chunk's pairs are one coalesced run per gathered row.  T is the arithmetic type
// (FP64, or FP32 for the low-precision operator); dV is always FP64 and rounded to
// T when staged.  A wavefront whose states lie past No16 skips its MFMAs (zeros).
// PAIR: nc is even.
template <class T, int NW, int TN, bool PAIR>
__global__ __launch_bounds__(NW * 64)
void k_occ_transform(BlockMapDev bm, int mtiles, int ntiles, const T *__restrict__ Xo, int no_pad, int no16,
                     const double *__restrict__ dV, T *__restrict__ Tt, int nc) {
    typedef typename OccMma<T>::type MM;
    constexpr int BM = 16 * NW, BN = 16 * TN, TR = 4 * NW, ND = (BN + 2 * TR - 1) / (2 * TR);
    const int B = blockIdx.x / (mtiles * ntiles), e0 = blockIdx.x % mtiles * BM, n0 = blockIdx.x / mtiles % ntiles * BN;
    const int g0 = bm.col_gstart[B], g1 = bm.col_gstart[B + 1];
    const int boff = bm.atom_off[B], nn = (bm.atom_off[B + 1] - boff) * nc;
    if (n0 >= nn) return;
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const bool live = e0 + 16 * wv < no16;
    __shared__ T Xs[16][BM];
    __shared__ T Ds[16][BN];

    typename MM::acc acc[TN];
#pragma unroll
    for (int i = 0; i < TN; ++i) acc[i] = MM::zero();

    // staging: row t / TR of the chunk, 4 states and ND pairs of columns per thread
    const int sr = t / TR, xc = (t % TR) * 4, dc = (t % TR) * 2;
    int32_t xrow = 0;
    int64_t ent = 0;
    auto rows = [&](int gc) {
        const int g = gc + sr;
        xrow = g < g1 ? bm.g_xrow[g] : -1;
        ent = g < g1 ? bm.g_ent[g] : 0;
    };
    T xv[4], dv[ND][2];
    auto fetch = [&]() {
        xv[0] = xv[1] = xv[2] = xv[3] = T(0);
        if (xrow >= 0 && e0 + xc < no_pad) load4(Xo + (int64_t)xrow * no_pad + e0 + xc, xv);
        const double *src = dV + ent * nc + n0 + dc;
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const int c = 2 * TR * i + dc;
            load_pair<T, PAIR>(src + 2 * TR * i, xrow >= 0 && c < BN && n0 + c < nn,
                               xrow >= 0 && c < BN && n0 + c + 1 < nn, dv[i][0], dv[i][1]);
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int c = 0; c < 4; ++c) Xs[sr][xc + c] = xv[c];
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const int c = 2 * TR * i + dc;
            if (c >= BN) continue;
            Ds[sr][c] = dv[i][0];
            Ds[sr][c + 1] = dv[i][1];
        }
    };
    rows(g0);
    fetch();
    rows(g0 + 16);
    for (int gc = g0; gc < g1; gc += 16) {
        store();
        __syncthreads();
        if (gc + 16 < g1) {
            fetch();
            rows(gc + 32);
        }
        if (live) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int kk = ks * 4 + (lane >> 4);
                T a[MM::NA], b[TN];
#pragma unroll
                for (int r = 0; r < MM::NA; ++r) a[r] = Xs[kk][16 * wv + MM::a_row(lane, r)];
#pragma unroll
                for (int i = 0; i < TN; ++i) b[i] = Ds[kk][16 * i + (lane & 15)];
#pragma unroll
                for (int i = 0; i < TN; ++i) acc[i] = MM::op(a, b[i], acc[i]);
            }
        }
        __syncthreads();
    }
    if (e0 + 16 * wv >= no_pad) return;
    const int64_t ldT = (int64_t)no_pad * nc;
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        const int n = n0 + 16 * i + (lane & 15);
        if (n >= nn) continue;
        const int b = n / nc, j = n - b * nc;
        T *dst = Tt + (int64_t)(boff + b) * ldT + (int64_t)(e0 + 16 * wv) * nc + j;
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[(int64_t)MM::row(lane, r) * nc] = acc[i][r];
    }
}

// Where the launch above leaves most of the chip waiting.  One workgroup: column
// atom B, 16 TE occupied states, NT tiles of pairs; its NW waves take turns over
// the gathered rows, 4 KU at a time straight into registers (the kernel above
// pays two barriers and a memory latency per 16 rows), and their sums are added
// in wave order through LDS.
template <class T, int TE, int NT, int NW, int KU>
__global__ __launch_bounds__(NW * 64)
void k_occ_transform_few(BlockMapDev bm, const T *__restrict__ Xo, int no_pad,
                         const double *__restrict__ dV, T *__restrict__ Tt, int nc) {
    typedef typename OccFewMma<T>::type MM;
    const int B = blockIdx.x, e0 = blockIdx.y * 16 * TE, n0 = blockIdx.z * 16 * NT;
    const int g0 = bm.col_gstart[B], g1 = bm.col_gstart[B + 1];
    const int boff = bm.atom_off[B], nB = bm.atom_off[B + 1] - boff;
    const int n1 = min(nB * nc, n0 + 16 * NT);   // this workgroup's pairs: n0 <= n < n1
    if (n0 >= n1) return;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lk = lane >> 4;
    __shared__ T red[NW][TE][NT][4][64];

    typename MM::acc acc[TE][NT];
#pragma unroll
    for (int e = 0; e < TE; ++e)
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[e][i] = MM::zero();
    for (int gc = g0 + wv * 4 * KU; gc < g1; gc += NW * 4 * KU) {
        T a[KU][TE][1], b[KU][NT];
        int32_t xr[KU];
        int64_t ge[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int g = gc + 4 * u + lk;
            xr[u] = g < g1 ? bm.g_xrow[g] : 0;
            ge[u] = g < g1 ? bm.g_ent[g] : 0;
        }
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const bool ok = gc + 4 * u + lk < g1;
#pragma unroll
            for (int e = 0; e < TE; ++e) a[u][e][0] = ok ? Xo[(int64_t)xr[u] * no_pad + e0 + 16 * e + lr] : T(0);
#pragma unroll
            for (int i = 0; i < NT; ++i)
                b[u][i] = (ok && n0 + 16 * i + lr < n1) ? (T)dV[ge[u] * nc + n0 + 16 * i + lr] : T(0);
        }
#pragma unroll
        for (int u = 0; u < KU; ++u)
#pragma unroll
            for (int e = 0; e < TE; ++e)
#pragma unroll
                for (int i = 0; i < NT; ++i) acc[e][i] = MM::op(a[u][e], b[u][i], acc[e][i]);
    }
#pragma unroll
    for (int e = 0; e < TE; ++e)
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wv][e][i][r][lane] = acc[e][i][r];
    __syncthreads();
    // (b, E, j) in the order of memory; a group may begin and end inside one b
    const int b0 = n0 / nc, nb = (n1 - 1) / nc - b0 + 1, run = 16 * TE * nc;
    for (int q = t; q < nb * run; q += NW * 64) {
        const int j = q % nc, E = q / nc % (16 * TE), b = b0 + q / run, n = b * nc + j;
        if (n < n0 || n >= n1) continue;
        const int R = E % 16, l = MM::quarter(R) * 16 + (n - n0) % 16;
        T v = T(0);
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[w][E / 16][(n - n0) / 16][MM::elem(R)][l];
        Tt[((int64_t)(boff + b) * no_pad + e0 + E) * nc + j] = v;
    }
}

// The same split for the way back: column atom B, 16 of its gathered rows, NT
// tiles of pairs; the waves take turns over the occupied states, 8 KU at a time.
// A lane loads two adjacent states of X; they feed two products whose k slots are
// the lanes' even and odd states.
template <class T, int NT, int NW, int KU>
__global__ __launch_bounds__(NW * 64)
void k_occ_back_few(BlockMapDev bm, const T *__restrict__ Xo, int no_pad, int no_sum,
                    const T *__restrict__ Ut, double *__restrict__ W, int nc) {
    typedef typename OccFewMma<T>::type MM;
    const int B = blockIdx.x, n0 = blockIdx.z * 16 * NT;
    const int g1 = bm.col_gstart[B + 1], g0 = bm.col_gstart[B] + blockIdx.y * 16;
    if (g0 >= g1) return;
    const int boff = bm.atom_off[B], nB = bm.atom_off[B + 1] - boff;
    const int n1 = min(nB * nc, n0 + 16 * NT);
    if (n0 >= n1) return;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lk = lane >> 4;
    const int64_t ldT = (int64_t)no_pad * nc;
    __shared__ T red[NW][NT][4][64];

    typename MM::acc acc[NT];
    const T *up[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        acc[i] = MM::zero();
        const int n = n0 + 16 * i + lr, b = n / nc;
        up[i] = n < n1 ? Ut + (boff + b) * ldT + n - b * nc : nullptr;
    }
    const T *xp = g0 + lr < g1 ? Xo + (int64_t)bm.g_xrow[g0 + lr] * no_pad : nullptr;
    for (int E0 = wv * 8 * KU; E0 < no_sum; E0 += NW * 8 * KU) {
        T a0[KU][1], a1[KU][1], u0[KU][NT], u1[KU][NT];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int E = E0 + 8 * u + 2 * lk;   // even, as no_sum is
            const bool ok = E < no_sum;
            a0[u][0] = ok && xp ? xp[E] : T(0);
            a1[u][0] = ok && xp ? xp[E + 1] : T(0);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                u0[u][i] = ok && up[i] ? up[i][(int64_t)E * nc] : T(0);
                u1[u][i] = ok && up[i] ? up[i][(int64_t)(E + 1) * nc] : T(0);
            }
        }
#pragma unroll
        for (int u = 0; u < KU; ++u)
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                acc[i] = MM::op(a0[u], u0[u][i], acc[i]);
                acc[i] = MM::op(a1[u], u1[u][i], acc[i]);
            }
    }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wv][i][r][lane] = acc[i][r];
    __syncthreads();
    for (int q = t; q < 16 * (n1 - n0); q += NW * 64) {
        const int row = q / (n1 - n0), p = q - row * (n1 - n0);
        if (g0 + row >= g1) break;
        const int r = MM::elem(row), l = MM::quarter(row) * 16 + p % 16;
        T v = T(0);
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[w][p / 16][r][l];
        W[bm.g_ent[g0 + row] * nc + n0 + p] = (double)v;
    }
}

// The split kernels' shapes: 2 x 1 tiles of (states, pairs) for the transform,
// 1 x 2 tiles of (rows, pairs) on the way back, eight wavefronts (four, or twice
// the tiles or the loads per round, were 5-30 % slower at 60 atoms).
constexpr int OCCF_TE = 2, OCCF_TT = 1, OCCF_TB = 2, OCCF_NW = 8;

// Their lines.  The transform: up to 1024 workgroups, past that the operands read
// again by each workgroup cost more than the waits.  us, split / staged kernel
// (with the tracer's ~5 us): 12 atoms 9 orbitals, 24 columns 8.2 / 9.5 (336), 80
// columns 14.6 / 11.2 (1080); 24 atoms 13 orbitals, 8 columns 11.5 / 14.6 (672), 16
// columns 17.7 / 17.2 (1248); 60 atoms 9 orbitals, 2 columns 12.0 / 13.0 (960), 8
// columns 21.4 / 18.4 (2400); 131 atoms 7 orbitals, 2 columns 16.8 / 14.8 (1834).
// Back: up to 128 pairs per atom and 4e8 operations.  60 atoms, 2 columns 12.6 /
// 14.0, 12 columns 21.7 / 23.4 (108 pairs, 3.5e8), 24 columns 33.2 / 30.1 (7e8);
// 131 atoms, 6 columns 27.7 / 30.1 (3.1e8), 14 columns 58.4 / 39.6 (7.2e8); 24
// atoms, 8 columns 12.3 / 12.6 (104 pairs), 16 columns 16.5 / 14.5 (208); 400 atoms
// 4 orbitals, 2 columns 41.7 / 53.2 (2.8e8), 8 columns 65.9 / 54.1 (1.1e9).
constexpr int64_t OCCF_GROUPS = 1024;
constexpr double OCCF_WORK = 4e8;
constexpr int OCCF_PAIRS = 128;

static inline int occ_few_groups(const BlockMapDev &bm, int nc, int nt) {
    return (bm.nb_max * nc + 16 * nt - 1) / (16 * nt);
}

// Pair tiles per workgroup, with `rest` workgroups per tile of pairs: the least
// time at tn + 3 per workgroup (its own rows or states cost about three tiles of
// pairs) and 1536 workgroups at once.  (Nine tiles always: 61 -> 48 us for the way
// back of 60 atoms, 48 columns; the least padding always: 2613 -> 3042 us for the
// transform of 400 atoms, 32 columns.  Both transforms over 30 sizes, 24 to 200
// atoms and 8 to 256 columns in FP64 and FP32, against these constants: tn + 1 0.2 %
// slower on average (one size by 5 %), tn + 6 1.6 % (10 %), 768 workgroups 1.8 % (18
// %), 3072 0.9 % (10 %; 8 % faster at best).)
static inline int occ_pair_tiles(const BlockMapDev &bm, int nc, int64_t rest) {
    const int n16 = (bm.nb_max * nc + 15) / 16;
    int best = OCC_NT;
    double least = 0.0;
    for (int tn = OCC_NT; tn >= 2; --tn) {
        const double cost = (tn + 3) * std::max(1.0, (double)(rest * ((n16 + tn - 1) / tn)) / 1536.0);
        if (tn == OCC_NT || cost < least) {
            least = cost;
            best = tn;
        }
    }
    return best;
}

// Calls f(std::integral_constant<int, tn>) for 2 <= tn <= OCC_NT.
template <int TN = OCC_NT, class F> static void with_tiles(int tn, const F &f) {
    if constexpr (TN > 2) {
        if (tn < TN) return with_tiles<TN - 1>(tn, f);
    }
    f(std::integral_constant<int, TN>{});
}

template <class T>
static void occ_transform_any(Tracer *t, hipStream_t s, const char *name, const BlockMapDev &bm,
                              int n_atoms, const T *Xo, int no_pad, int no16, const double *dV, T *Tt, int nc,
                              const WorkSizes &ws) {
    trace_begin(t, name, s);
    if ((int64_t)n_atoms * (no_pad / (16 * OCCF_TE)) * occ_few_groups(bm, nc, OCCF_TT) <= OCCF_GROUPS)
        hipLaunchKernelGGL((k_occ_transform_few<T, OCCF_TE, OCCF_TT, OCCF_NW, 2>),
                           dim3(n_atoms, no_pad / (16 * OCCF_TE), occ_few_groups(bm, nc, OCCF_TT)),
                           dim3(OCCF_NW * 64), 0, s, bm, Xo, no_pad, dV, Tt, nc);
    else {
        constexpr int NW = OCC_WAVES<T>;
        const int mt = (no_pad + 16 * NW - 1) / (16 * NW), tn = occ_pair_tiles(bm, nc, (int64_t)n_atoms * mt);
        const int nt = (bm.nb_max * nc + 16 * tn - 1) / (16 * tn);
        const dim3 grid((unsigned)(n_atoms * mt * nt));
        with_tiles(tn, [&](auto c) {
            constexpr int TN = decltype(c)::value;
            if (nc % 2 == 0)
                hipLaunchKernelGGL((k_occ_transform<T, NW, TN, true>), grid, dim3(NW * 64), 0, s, bm, mt, nt, Xo,
                                   no_pad, no16, dV, Tt, nc);
            else
                hipLaunchKernelGGL((k_occ_transform<T, NW, TN, false>), grid, dim3(NW * 64), 0, s, bm, mt, nt, Xo,
                                   no_pad, no16, dV, Tt, nc);
        });
    }
    trace_end(t, s, 2.0 * ws.No * ws.nnzB * nc,
              8.0 * ws.nnzB * nc + sizeof(T) * (ws.N * ws.No + ws.N * ws.No * nc));
}

void launch_occ_transform(Tracer *t, hipStream_t s, const BlockMapDev &bm, int n_atoms,
                          const double *Xo, int no_pad, int no16, const double *dV, double *Tt,
                          int nc, const WorkSizes &ws) {
    occ_transform_any<double>(t, s, "occ_transform", bm, n_atoms, Xo, no_pad, no16, dV, Tt, nc, ws);
}

void launch_occ_transform_f32(Tracer *t, hipStream_t s, const BlockMapDev &bm, int n_atoms,
                              const float *Xo, int no_pad, int no16, const double *dV, float *Tt,
                              int nc, const WorkSizes &ws) {
    occ_transform_any<float>(t, s, "occ_transform_f32", bm, n_atoms, Xo, no_pad, no16, dV, Tt, nc, ws);
}

// ------------------------------------------------------ (b4) back to the pattern
// W[(k(A,B), a, b)][j] = sum_E Xo[a][E] Ut[b][E*nc + j] for (A, B) in the pattern.
// One workgroup: column atom B, 16 NW of its gathered rows (A, a), 16 TN packed
// pairs n = b nc + j; wave w owns rows 16w..16w+15.  The occupied states E < no_sum
// come in chunks of 16.  A wave whose rows lie past the atom's last gathered row
// stages its share of the operands and skips the MFMAs.  Accumulation in T; W is
// FP64.  PAIR: nc is even.
template <class T, int NW, int TN, bool PAIR>
__global__ __launch_bounds__(NW * 64)
void k_occ_back(BlockMapDev bm, int n_atoms, int ntiles, const T *__restrict__ Xo, int no_pad, int no_sum,
                const T *__restrict__ Ut, double *__restrict__ W, int nc) {
    typedef typename OccMma<T>::type MM;
    constexpr int BM = 16 * NW, BN = 16 * TN, TR = 4 * NW, NP = (BN + 2 * TR - 1) / (2 * TR);
    const int B = blockIdx.x / ntiles % n_atoms, n0 = blockIdx.x % ntiles * BN, mt = blockIdx.x / (ntiles * n_atoms);
    const int g1 = bm.col_gstart[B + 1];
    const int g0 = bm.col_gstart[B] + mt * BM;
    if (g0 >= g1) return;
    const int boff = bm.atom_off[B], nn = (bm.atom_off[B + 1] - boff) * nc;
    if (n0 >= nn) return;
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const bool live = g0 + wv * 16 < g1;
    const int64_t ldT = (int64_t)no_pad * nc;
    __shared__ T Xs[16][BM + 1];
    __shared__ T Us[16][BN];

    typename MM::acc acc[TN];
#pragma unroll
    for (int i = 0; i < TN; ++i) acc[i] = MM::zero();

    const int xr = t / 4, xc = (t % 4) * 4, xg = g0 + xr;
    const T *xsrc = (xg < g1) ? Xo + (int64_t)bm.g_xrow[xg] * no_pad + xc : nullptr;
    // pairs (n, n + 1) of this thread, n = n0 + 2 TR i + un, at Ut[(boff + b) ldT + E nc + j]
    const int ue = t / TR, un = (t % TR) * 2;
    const T *up[NP][PAIR ? 1 : 2];
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int h = 0; h < (PAIR ? 1 : 2); ++h) {
            const int n = n0 + 2 * TR * i + un + h, b = n / nc, j = n - b * nc;
            up[i][h] = n < nn && 2 * TR * i + un < BN ? Ut + (int64_t)(boff + b) * ldT + (int64_t)ue * nc + j : nullptr;
        }
    T xv[4], uv[NP][2];
    auto fetch = [&](int E0) {
        xv[0] = xv[1] = xv[2] = xv[3] = T(0);
        if (xsrc) load4(xsrc + E0, xv);
        const int64_t o = (int64_t)E0 * nc;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if (PAIR) {
                load_pair<T, true>(up[i][0] + o, up[i][0] != nullptr, false, uv[i][0], uv[i][1]);
            } else {
                uv[i][0] = up[i][0] ? up[i][0][o] : T(0);
                uv[i][1] = up[i][PAIR ? 0 : 1] ? up[i][PAIR ? 0 : 1][o] : T(0);
            }
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int c = 0; c < 4; ++c) Xs[xc + c][xr] = xv[c];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if (2 * TR * i + un >= BN) continue;
            Us[ue][2 * TR * i + un] = uv[i][0];
            Us[ue][2 * TR * i + un + 1] = uv[i][1];
        }
    };
    fetch(0);
    for (int E0 = 0; E0 < no_sum; E0 += 16) {
        store();
        __syncthreads();
        if (E0 + 16 < no_sum) fetch(E0 + 16);
        if (live) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int kk = ks * 4 + (lane >> 4);
                T a[MM::NA], b[TN];
#pragma unroll
                for (int r = 0; r < MM::NA; ++r) a[r] = Xs[kk][wv * 16 + MM::a_row(lane, r)];
#pragma unroll
                for (int i = 0; i < TN; ++i) b[i] = Us[kk][16 * i + (lane & 15)];
#pragma unroll
                for (int i = 0; i < TN; ++i) acc[i] = MM::op(a, b[i], acc[i]);
            }
        }
        __syncthreads();
    }
    if (!live) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int g = g0 + wv * 16 + MM::row(lane, r);
        if (g < g1) {
            double *dst = W + (int64_t)bm.g_ent[g] * nc;   // row (k, a, b) = g_ent[g] + b: column b nc + j
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                const int n = n0 + 16 * i + (lane & 15);
                if (n < nn) dst[n] = (double)acc[i][r];
            }
        }
    }
}

template <class T>
static void occ_back_any(Tracer *t, hipStream_t s, const char *name, const BlockMapDev &bm,
                         int n_atoms, int max_rows, const T *Xo, int no_pad, int no_sum, const T *Ut,
                         double *W, int nc, const WorkSizes &ws) {
    trace_begin(t, name, s);
    if (bm.nb_max * nc <= OCCF_PAIRS && 2.0 * ws.No * ws.nnzB * nc <= OCCF_WORK)
        hipLaunchKernelGGL((k_occ_back_few<T, OCCF_TB, OCCF_NW, 1>),
                           dim3(n_atoms, (max_rows + 15) / 16, occ_few_groups(bm, nc, OCCF_TB)), dim3(OCCF_NW * 64), 0,
                           s, bm, Xo, no_pad, no_sum, Ut, W, nc);
    else {
        constexpr int NW = OCC_WAVES<T>;
        const int mt = (max_rows + 16 * NW - 1) / (16 * NW), tn = occ_pair_tiles(bm, nc, (int64_t)n_atoms * mt);
        const int nt = (bm.nb_max * nc + 16 * tn - 1) / (16 * tn);
        const dim3 grid((unsigned)(n_atoms * mt * nt));
        with_tiles(tn, [&](auto c) {
            constexpr int TN = decltype(c)::value;
            if (nc % 2 == 0)
                hipLaunchKernelGGL((k_occ_back<T, NW, TN, true>), grid, dim3(NW * 64), 0, s, bm, n_atoms, nt, Xo,
                                   no_pad, no_sum, Ut, W, nc);
            else
                hipLaunchKernelGGL((k_occ_back<T, NW, TN, false>), grid, dim3(NW * 64), 0, s, bm, n_atoms, nt, Xo,
                                   no_pad, no_sum, Ut, W, nc);
        });
    }
    trace_end(t, s, 2.0 * ws.No * ws.nnzB * nc,
              sizeof(T) * (ws.N * ws.No * nc + ws.N * ws.No) + 8.0 * ws.nnzB * nc);
}

void launch_occ_back(Tracer *t, hipStream_t s, const BlockMapDev &bm, int n_atoms, int max_rows,
                     const double *Xo, int no_pad, int no_sum, const double *Ut, double *W, int nc,
                     const WorkSizes &ws) {
    occ_back_any<double>(t, s, "occ_back", bm, n_atoms, max_rows, Xo, no_pad, no_sum, Ut, W, nc, ws);
}

void launch_occ_back_f32(Tracer *t, hipStream_t s, const BlockMapDev &bm, int n_atoms, int max_rows,
                         const float *Xo, int no_pad, int no_sum, const float *Ut, double *W, int nc,
                         const WorkSizes &ws) {
    occ_back_any<float>(t, s, "occ_back_f32", bm, n_atoms, max_rows, Xo, no_pad, no_sum, Ut, W, nc, ws);
}

// ---------------------------------------------------------- (e) skinny K z
// Zout[mu][j] = sum_nu K[mu][nu] Zin[nu][j] for a few columns j < nc: K
// streams from HBM once per product.
// Up to two right-hand sides (nc = 1..4 real columns): a wavefront owns RW
// rows and every lane reads 16-byte pairs of K columns, U pairs of chunks in
// flight per row; the two Zin rows a lane needs (2 nc doubles, contiguous) are
// read through the cache.  Four times the wavefronts of the LDS-staged form,
// with no barrier in the loop.
template <int NC, int RW>
__global__ __launch_bounds__(256)
void k_kmatvec_lanes(int P_pad, const double *__restrict__ K, const double *__restrict__ Zin,
                     double *__restrict__ Zout) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int row0 = (blockIdx.x * 4 + wv) * RW;
    double acc[RW][NC];
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int j = 0; j < NC; ++j) acc[r][j] = 0.0;
    for (int c0 = 2 * lane; c0 < P_pad; c0 += 128 * U) {
        double2 kv[U][RW];
        double2 zv[U][NC];   // Zin rows nu and nu + 1: 2 NC doubles
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int nu = c0 + 128 * u;
            const bool ok = nu < P_pad;
#pragma unroll
            for (int r = 0; r < RW; ++r)
                kv[u][r] = ok ? *reinterpret_cast<const double2 *>(K + (int64_t)(row0 + r) * P_pad + nu)
                              : make_double2(0.0, 0.0);
#pragma unroll
            for (int h = 0; h < NC; ++h)
                zv[u][h] = ok ? reinterpret_cast<const double2 *>(Zin + (int64_t)nu * NC)[h]
                              : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double *z = reinterpret_cast<const double *>(zv[u]);   // z[0..NC): row nu, z[NC..2NC): nu + 1
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int j = 0; j < NC; ++j) acc[r][j] += kv[u][r].x * z[j] + kv[u][r].y * z[NC + j];
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            double v = acc[r][j];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if (lane == 0) Zout[(int64_t)(row0 + r) * NC + j] = v;
        }
}

// 5..32 real columns on the FP64 matrix cores (CT 16-column tiles).  A
// workgroup owns 16 RT rows; its NW waves split the reduction over nu in
// interleaved chunks of 8 U columns and add their 16x16 accumulators in a
// fixed order through LDS at the end.  Each lane streams K as 16-byte loads of
// two adjacent columns; the two columns feed two 16x16x4 MFMAs whose k slots
// are the lanes' even and odd columns, with Zin rows taken in the same order.
// Zin (P_pad x nc, a few MB) is read through the cache; no barrier in the
// loop.  With PF the loads of the wave's next chunk are issued before the
// MFMAs of the current one.
// Bound by the loads in flight: by too few workgroups where P_pad / 32 is
// below the CU count (16 rows per workgroup and 8 waves then), by the reads of
// Zin, which every workgroup repeats, where P_pad is large (32 rows).
// (LDS-staged form: 0.25-3.4 TB/s; non-temporal loads of K were 10 % slower.)
template <int RT, int CT, int U, bool PF, int NW>
__global__ __launch_bounds__(NW * 64)
void k_kmatvec_mfma(int P_pad, const double *__restrict__ K, const double *__restrict__ Zin,
                    double *__restrict__ Zout, int nc) {
    __shared__ dbl4 red[NW - 1][RT][CT][64];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int row0 = blockIdx.x * 16 * RT;
    const int lr = lane & 15, lk = lane >> 4;
    dbl4 acc[RT][CT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[r][c] = dbl4{0.0, 0.0, 0.0, 0.0};
    constexpr int KW = 8 * U;
    double2 a[U][RT];
    double b0[U][CT], b1[U][CT];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kk = k0 + 8 * u + 2 * lk;   // even; P_pad is a multiple of 64
            const bool ok = kk < P_pad;
#pragma unroll
            for (int r = 0; r < RT; ++r)
                a[u][r] = ok ? *reinterpret_cast<const double2 *>(K + (int64_t)(row0 + 16 * r + lr) * P_pad + kk)
                              : make_double2(0.0, 0.0);
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int col = 16 * c + lr;
                b0[u][c] = (ok && col < nc) ? Zin[(int64_t)kk * nc + col] : 0.0;
                b1[u][c] = (ok && col < nc) ? Zin[(int64_t)(kk + 1) * nc + col] : 0.0;
            }
        }
    };
    auto mma = [&](const double2 (&ca)[U][RT], const double (&c0)[U][CT], const double (&c1)[U][CT]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(ca[u][r].x, c0[u][c], acc[r][c], 0, 0, 0);
                    acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(ca[u][r].y, c1[u][c], acc[r][c], 0, 0, 0);
                }
    };
    if constexpr (PF) {
        int k0 = wv * KW;
        if (k0 < P_pad) fetch(k0);
        for (; k0 < P_pad; k0 += NW * KW) {
            double2 ca[U][RT];
            double c0[U][CT], c1[U][CT];
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int r = 0; r < RT; ++r) ca[u][r] = a[u][r];
#pragma unroll
                for (int c = 0; c < CT; ++c) { c0[u][c] = b0[u][c]; c1[u][c] = b1[u][c]; }
            }
            if (k0 + NW * KW < P_pad) fetch(k0 + NW * KW);
            mma(ca, c0, c1);
        }
    } else {
        for (int k0 = wv * KW; k0 < P_pad; k0 += NW * KW) {
            fetch(k0);
            mma(a, b0, b1);
        }
    }
    if (wv > 0)
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) red[wv - 1][r][c][lane] = acc[r][c];
    __syncthreads();
    if (wv != 0) return;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            dbl4 v = acc[r][c];
#pragma unroll
            for (int w = 0; w < NW - 1; ++w) v += red[w][r][c][lane];
            const int col = 16 * c + lr;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col < nc) Zout[(int64_t)(row0 + 16 * r + 4 * e + lk) * nc + col] = v[e];
        }
}

// Products below which a workgroup takes 16 rows instead of 32 (us at 8 and 24
// columns, 32 / 16 rows: P = 448: 8.2 / 5.0, 10.9 / 6.5; 1024: 15.5 / 7.7, 20.9 /
// 11.2; 3328: 42.5 / 21.0, 67.5 / 30.7; 6400: 84 / 87, 95 / 124; 12416: 288 / 326,
// 386 / 463).  Eight waves of two k-steps at 32 rows and two column tiles
// replace four of four (6400: 153 -> 95, 12416: 390 -> 386).
constexpr int KMV_SMALL = 5120;

void launch_kmatvec_skinny(Tracer *t, hipStream_t s, int P_pad, const double *K,
                           const double *Zin, double *Zout, int nc, double P) {
    trace_begin(t, "kernel_matvec", s);
    if (nc == 1)
        hipLaunchKernelGGL((k_kmatvec_lanes<1, 1>), dim3(P_pad / 4), dim3(256), 0, s, P_pad, K, Zin, Zout);
    else if (nc == 2)
        hipLaunchKernelGGL((k_kmatvec_lanes<2, 1>), dim3(P_pad / 4), dim3(256), 0, s, P_pad, K, Zin, Zout);
    else if (nc == 3)
        hipLaunchKernelGGL((k_kmatvec_lanes<3, 1>), dim3(P_pad / 4), dim3(256), 0, s, P_pad, K, Zin, Zout);
    else if (nc == 4)
        hipLaunchKernelGGL((k_kmatvec_lanes<4, 2>), dim3(P_pad / 8), dim3(256), 0, s, P_pad, K, Zin, Zout);
    else if (nc <= 16 && P_pad < KMV_SMALL)
        hipLaunchKernelGGL((k_kmatvec_mfma<1, 1, 4, true, 8>), dim3(P_pad / 16), dim3(512), 0, s, P_pad, K, Zin,
                           Zout, nc);
    else if (nc <= 16)
        hipLaunchKernelGGL((k_kmatvec_mfma<2, 1, 8, true, 4>), dim3(P_pad / 32), dim3(256), 0, s, P_pad, K, Zin,
                           Zout, nc);
    else if (P_pad < KMV_SMALL)
        hipLaunchKernelGGL((k_kmatvec_mfma<1, 2, 4, false, 8>), dim3(P_pad / 16), dim3(512), 0, s, P_pad, K, Zin,
                           Zout, nc);
    else
        hipLaunchKernelGGL((k_kmatvec_mfma<2, 2, 2, true, 8>), dim3(P_pad / 32), dim3(512), 0, s, P_pad, K, Zin,
                           Zout, nc);
    trace_end(t, s, 2.0 * P * P * nc, 8.0 * (P * P + 2.0 * P * nc));
}

}  // namespace chi0
