// FP64 dense products on the INT8 matrix cores (Sec. 4.2, Table t:flops steps 3
// and 4 at large sizes): residue arithmetic in the sense of the Chinese
// remainder theorem, as proposed for matrix products by Ozaki, Uchino and
// Imamura ("Ozaki scheme II", 2025).
//
//   1. Row i of A and column j of B are scaled and rounded to integers
//      A' = rint(2^e m A), B' likewise (a scale per row / column, below).
//   2. For each of CRT_S pairwise coprime moduli p <= 256 the residues of A'
//      and B' (one signed byte each) are multiplied on the INT8 matrix cores,
//      which accumulate exactly in 32 bits for K < 2^17, and reduced mod p.
//   3. C' = A' B' is the one integer in (-P/2, P/2), P the product of the
//      moduli, with these residues; it is put together in FP64 and scaled back.
// Steps 2 and 3 are exact up to 2^-80 P, so the error is that of the rounding
// in 1, below.  INT8 runs at 64 times the FP64 matrix rate on this card, so
// CRT_S = 14 products, with the passes over memory that 1-3 add, are faster
// than one in FP64 where both M and K are large.
//
// Scales.  |C'_ij| <= |A'_i| |B'_j| (2-norms) has to stay below P/2 =
// 2^109.36: rows of A' get the norm 2^54.6 and columns of B' 2^54.75, and no
// entry may exceed 2^53.  An entry is then rounded to 2^-54.7 of the norm of
// its row or column, however small it is, so the error of C_ij is bounded by
// the norms of row i and column j, not by S_ij = sum_k |A_ik| |B_kj| as that of
// an FP64 sum of K products is: K 2^-53 S_ij.  Where S_ij is far below
// |A_i| |B_j| (large entries of one operand meet zeros or small ones of the
// other: symmetry, separate fragments, one transition close to resonance) the
// rounded operands are not good enough.  So every product is checked first:
//
//   0. k_crt_check bounds S_ij from below by a product of the operands'
//      magnitudes, one byte (e5m2) each, rounded down: one INT8-sized product
//      more.  The 64 x 128 tiles in which any element's rounding error may
//      exceed the K 2^-53 S_ij of an FP64 sum are left out of steps 2 and 3
//      and computed by the FP64 GEMM (launch_dgemm_flagged).
//
// Every element therefore keeps the bound of an FP64 sum.  The check and the empty
// launches for the FP64 tiles take 2.5 + 0.1 ms of 43 (400 atoms, 16 vectors), 0.11 +
// 0.02 of 2.45 (200 atoms, 12 vectors).  How many tiles leave depends on the
// vectors and the broadening, chi0 z in us (FP64 kernels alone / this way):
//                              200 atoms, 12   150 atoms, 5   400 atoms, 4
//   random or graded vectors     3016 / 2470     822 /  674   19100 / 11060
//   unit vectors                 3018 / 2647     821 /  736   19080 / 10680
//   eps 1e-4 (else 1e-2)         3013 / 3112     822 /  880   19110 / 12510
//   eps 1e-8                     3003 / 3055     826 /  864   19230 / 17160
//
// Relative error of the transforms of dense orbitals (sampled against extended
// precision, two seeds), this way and by the FP64 GEMM, in 1e-16:
//   K   470   528   550   810   900  1000  1690  1800  3200  5200
//       4.5   4.8   4.9   5.1   4.7   6.0   6.3   7.2   8.4  10.6
//       5.4   6.4   6.4   5.9   5.0   8.7   9.6  13.2  22.8  25.9
//
// A column with an infinity or NaN goes to the FP64 GEMM too (without the
// check, in the test hook alone, it gives NaN).
#include "panel_core.h"

namespace chi0 {

typedef int int4v __attribute__((ext_vector_type(4)));
typedef int int8v __attribute__((ext_vector_type(8)));
typedef int int16v __attribute__((ext_vector_type(16)));
typedef float flt16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int kMod[CRT_S] = {256, 253, 251, 249, 247, 241, 239, 235, 233, 229, 227, 223, 217, 211};
constexpr double kNormA = 54.6, kNormB = 54.75;   // log2 of the integer rows' and columns' norms
constexpr double kRint = 6755399441055744.0;      // 1.5 2^52: x + kRint holds rint(x) in its low word

constexpr double mod_product() {
    double p = 1.0;
    for (int i = 0; i < CRT_S; ++i) p *= kMod[i];
    return p;
}
// w_i = (P / p_i)^-1 mod p_i, over p_i: C' / P = sum_i c_i w_i mod 1.  Its
// numerator is the weight of modulus i.
constexpr int64_t mod_weight(int i) {
    int64_t r = 1;
    for (int j = 0; j < CRT_S; ++j)
        if (j != i) r = r * kMod[j] % kMod[i];
    int64_t q = 1;
    while (r * q % kMod[i] != 1) ++q;
    return q;
}
// w_i = hi + lo: hi a multiple of 2^-42, so that the sum of c_i hi is exact
constexpr int64_t kHiScale = 1ll << 42;
constexpr int64_t weight_hi_int(int i) { return (mod_weight(i) * kHiScale + kMod[i] / 2) / kMod[i]; }
constexpr double weight_hi(int i) { return (double)weight_hi_int(i) / (double)kHiScale; }
constexpr double weight_lo(int i) {
    return (double)(mod_weight(i) * kHiScale - weight_hi_int(i) * kMod[i]) / (double)kMod[i] / (double)kHiScale;
}
struct Weights {
    double hi[CRT_S], lo[CRT_S];
};
constexpr Weights make_weights() {
    Weights w{};
    for (int i = 0; i < CRT_S; ++i) {
        w.hi[i] = weight_hi(i);
        w.lo[i] = weight_lo(i);
    }
    return w;
}
constexpr Weights kW = make_weights();

struct ModTable {
    double inv[CRT_S];
    int p[CRT_S];
};
constexpr ModTable make_mods() {
    ModTable t{};
    for (int i = 0; i < CRT_S; ++i) {
        t.inv[i] = 1.0 / kMod[i];
        t.p[i] = kMod[i];
    }
    return t;
}
__constant__ ModTable kModDev = make_mods();

__device__ __forceinline__ uint32_t low_word(double x) { return (uint32_t)__double_as_longlong(x); }
// four low bytes -> one word
__device__ __forceinline__ uint32_t pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x0c0c0400), hi = __builtin_amdgcn_perm(d, c, 0x0c0c0400);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100);
}

struct FormI8 {
    static constexpr int PL = 1;
    typedef int16v acc;
    static __device__ __forceinline__ acc mma(const uint4 (&a)[1], const uint4 (&b)[1], acc c) {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(int4v, a[0]), __builtin_bit_cast(int4v, b[0]),
                                                     c, 0, 0, 0);
    }
};

// Products of magnitudes, e5m2 bytes.  The 32x32x64 product (twice the rate of the
// 32x32x16 one) takes 32 bytes of a lane: 16 of each half of the k-blocks, which
// are the two planes here.
struct FormMag {
    static constexpr int PL = 2;
    typedef flt16 acc;
    static __device__ __forceinline__ int8v both(const uint4 (&x)[2]) {
        return int8v{(int)x[0].x, (int)x[0].y, (int)x[0].z, (int)x[0].w, (int)x[1].x, (int)x[1].y, (int)x[1].z, (int)x[1].w};
    }
    static __device__ __forceinline__ acc mma(const uint4 (&a)[2], const uint4 (&b)[2], acc c) {
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(both(a), both(b), c, 1, 1, 0, 0, 0, 0);   // no scales
    }
};

// Magnitude bytes hold |a'| 2^-MAG_SHIFT, at most 2^15, rounded towards zero; a
// value below the least normal one, 2^-14, is that (0 stays 0), so that a product
// of magnitudes is zero only where every product of the operands is.
constexpr int MAG_SHIFT = 38;
constexpr double MAG_SCALE = 1.0 / (double)(1ll << MAG_SHIFT);
constexpr float MAG_LEAST = 0x1p-14f;
__device__ __forceinline__ float mag_of(double a, bool nonzero) {
    return fmaxf((float)(fabs(a) * MAG_SCALE), nonzero ? MAG_LEAST : 0.f);
}
// e5m2 is the upper byte of an FP16 value
__device__ __forceinline__ uint32_t mag_pack4(const float (&f)[4]) {
    return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[2], f[3])),
                                 __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[0], f[1])), 0x07050301);
}

}  // namespace

// Scale 2^e m of a column from its sum of squares and largest entry: its norm
// is brought to 2^lnorm and its largest entry to at most 2^53.  bad != 0 (a
// NaN): the column holds an infinity or NaN, m becomes NaN.  A norm out of
// range for its sum of squares is replaced by its bound sqrt(K) max.  nrm: the
// scaled column's norm (or the bound; NaN if m is).
__device__ __forceinline__ void crt_scale(double ss, double mx, double bad, int K, double lnorm, double &m, int &e,
                                          float &nrm) {
    m = 1.0;
    e = 0;
    nrm = 0.f;
    if (bad != 0.0) {
        m = bad;
        nrm = (float)bad;
    } else if (mx > 0.0) {
        int em;
        const double fm = frexp(mx, &em);   // mx = fm 2^em
        const double lmax = log2(fm) + em;
        const double ln = ss > 1e-280 && ss < 1e300 ? 0.5 * log2(ss) : 0.5 * log2((double)K) + lmax;
        const double l = fmin(lnorm - ln, 52.9999 - lmax);
        e = (int)floor(l);
        m = exp2(l - e);
        nrm = (float)exp2(l + ln);
    }
}

// Residues of 16 entries a 2^e m, rounded to whole numbers of at most 53 bits,
// for every modulus, and their magnitudes: 16 bytes per plane.  a mod p is the
// low byte of lo(a) - lo(rint(a / p)) p, whatever the higher bits are.
__device__ __forceinline__ void crt_residues(double (&a)[16], int e, double m, uint4 *__restrict__ out,
                                             int64_t plane) {
    uint32_t lo[16], mag[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float f[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double x = ldexp(a[4 * q + c], e) * m;
            f[c] = mag_of(x, a[4 * q + c] != 0.0);
            a[4 * q + c] = rint(x);
        }
        mag[q] = mag_pack4(f);
    }
    out[CRT_S * plane] = make_uint4(mag[0], mag[1], mag[2], mag[3]);
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        lo[c] = low_word(__builtin_fma(rint(a[c] * 0x1p-32), -0x1p32, a[c]) + kRint);
    }
#pragma unroll
    for (int i = 0; i < CRT_S; ++i) {
        uint32_t w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t r[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double t = __builtin_fma(a[4 * q + c], 1.0 / kMod[i], kRint);
                r[c] = lo[4 * q + c] - __umul24(low_word(t), (uint32_t)kMod[i]);
            }
            w[q] = pack4(r[0], r[1], r[2], r[3]);
        }
        out[i * plane] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Scales and residues of the columns n < N of X [K][ldx] (zero for k >= K and
// up to ld) in one pass: a workgroup holds COLS whole columns in registers,
// ITEMS k-blocks of 16 rows per thread, forms their scales and writes 16
// bytes per plane and k-block.  Bound by memory: 8 bytes read and CRT_P
// written per entry, at 3.7-4.5 TB/s.  (As two kernels, which read X twice, 200
// atoms, 12 vectors: 459 us for both transforms, now 270-315; 400 atoms, 16
// vectors 6.4 -> 3.4 ms.)
template <int COLS, int ITEMS>
__global__ __launch_bounds__(1024)
void k_crt_cut(const double *__restrict__ X, int K, int N, int64_t ldx, double lnorm, CrtScales sc, int nkb, int ld,
               uint4 *__restrict__ out, int64_t plane) {
    __shared__ double sh[4][16][COLS];
    __shared__ double shm[COLS];
    __shared__ int she[COLS];
    const int t = threadIdx.x, lane = t & 63, col = t % COLS;
    const int n = panel_xcd(blockIdx.x, gridDim.x) * COLS + col;
    double a[ITEMS][16], ss = 0.0, mx = 0.0, bad = 0.0, nz = 0.0;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q)
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const int k = (t / COLS + q * (1024 / COLS)) * 16 + c;
            a[q][c] = (n < N && k < K) ? X[(int64_t)k * ldx + n] : 0.0;
        }
#pragma unroll
    for (int q = 0; q < ITEMS; ++q)
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            ss += a[q][c] * a[q][c];
            mx = fmax(mx, fabs(a[q][c]));
            bad += a[q][c] * 0.0;   // NaN after an infinity or NaN
            nz += a[q][c] != 0.0 ? 1.0 : 0.0;
        }
#pragma unroll
    for (int o = 32; o >= COLS; o >>= 1) {
        ss += __shfl_xor(ss, o);
        mx = fmax(mx, __shfl_xor(mx, o));
        bad += __shfl_xor(bad, o);
        nz += __shfl_xor(nz, o);
    }
    if (lane < COLS) {
        sh[0][t >> 6][lane] = ss;
        sh[1][t >> 6][lane] = mx;
        sh[2][t >> 6][lane] = bad;
        sh[3][t >> 6][lane] = nz;
    }
    __syncthreads();
    if (t < COLS) {
        ss = mx = bad = nz = 0.0;
        for (int g = 0; g < 16; ++g) {
            ss += sh[0][g][t];
            mx = fmax(mx, sh[1][g][t]);
            bad += sh[2][g][t];
            nz += sh[3][g][t];
        }
        double m;
        int e;
        float nrm;
        crt_scale(ss, mx, bad, K, lnorm, m, e, nrm);
        shm[t] = m;
        she[t] = e;
        if (n < N) sc.put(n, m, e, nrm, nz);
    }
    __syncthreads();
    const double m = shm[col];
    const int e = she[col];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const int kb = t / COLS + q * (1024 / COLS);
        if (kb < nkb) crt_residues(a[q], e, m, out + (int64_t)kb * ld + n, plane);
    }
}

// The same as two kernels, for columns too long for a workgroup's registers.
// Scales: 64 columns x 16 row groups per workgroup; sums in a fixed order.
__global__ __launch_bounds__(1024)
void k_crt_scale_long(const double *__restrict__ X, int K, int N, int64_t ldx, double lnorm, CrtScales sc) {
    __shared__ double sh[4][16][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6, n = blockIdx.x * 64 + lane;
    double ss = 0.0, mx = 0.0, bad = 0.0, nz = 0.0;
    if (n < N) {
        const double *x = X + n;
#pragma unroll 8
        for (int k = g; k < K; k += 16) {
            const double v = x[(int64_t)k * ldx];
            ss += v * v;
            mx = fmax(mx, fabs(v));
            bad += v * 0.0;
            nz += v != 0.0 ? 1.0 : 0.0;
        }
    }
    sh[0][g][lane] = ss;
    sh[1][g][lane] = mx;
    sh[2][g][lane] = bad;
    sh[3][g][lane] = nz;
    __syncthreads();
    if (g != 0 || n >= N) return;
#pragma unroll
    for (int i = 1; i < 16; ++i) {
        ss += sh[0][i][lane];
        mx = fmax(mx, sh[1][i][lane]);
        bad += sh[2][i][lane];
        nz += sh[3][i][lane];
    }
    double m;
    int e;
    float nrm;
    crt_scale(ss, mx, bad, K, lnorm, m, e, nrm);
    sc.put(n, m, e, nrm, nz);
}

// Residues by the scales: thread (kb, n), 16 rows of one column.
__global__ __launch_bounds__(256)
void k_crt_cut_long(const double *__restrict__ X, int K, int N, int64_t ldx, const double *__restrict__ sm,
                    const int *__restrict__ se, int nkb, int ld, uint4 *__restrict__ out, int64_t plane) {
    const int64_t total = (int64_t)nkb * ld;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
        const int kb = (int)(idx / ld), n = (int)(idx % ld);
        const double m = n < N ? sm[n] : 0.0;
        const int e = n < N ? se[n] : 0;
        double a[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const int k = kb * 16 + c;
            a[c] = (n < N && k < K) ? X[(int64_t)k * ldx + n] : 0.0;
        }
        crt_residues(a, e, m, out + idx, plane);
    }
}

// flag[row / 64][column / 128] = 1 where the rounding of the operands may be
// worse than that of an FP64 sum.  In units of the integer operands: rounding a
// to A' changes a non-zero entry by at most 1/2 and leaves a zero alone, so C'_ij
// is off by at most err = (|a_i| qb_j + qa_i |B'_j|) / 2 with q the root of the
// number of non-zero entries.  The product m_ij of the magnitudes is at most
// 2^(-2 MAG_SHIFT) S_ij + 4 K (an entry raised to the least magnitude adds at most
// 2^-14 2^15, K of them in either operand); its FP32 sum may be too large by K / 64
// roundings (K 2^-22 covers them) and leaves out small terms beside large ones (up to
// 4e-4 of the 64 products of an instruction).  Scaling and joining round another 8 times.  So
//   m_ij >= (4 K + err 2^(53 - 2 MAG_SHIFT) / (K - 8)) (1 + K 2^-22)
// is enough for err <= (K - 8) 2^-53 S_ij.  m_ij = 0: every product is exactly zero.
// A NaN (a column with an infinity or NaN has a NaN norm) fails the test.
// Bound by the wait of a tile of few stages: 1.1 PFLOP/s and matrix cores busy 23 %
// of the cycles at K = 1000-1800, 1.7 and 33 % at 3200-5200.
template <class P>
__global__ __launch_bounds__(P::NT, 3)
void k_crt_check(int ntm, int ntn, int nkb, int K, int N, const uint4 *__restrict__ A, int lda,
                 const float *__restrict__ an, const float *__restrict__ aq, const uint4 *__restrict__ B, int ldb,
                 const float *__restrict__ bn, const float *__restrict__ bq, uint8_t *__restrict__ flag, int fm, int fn) {
    __shared__ uint4 s0[P::STAGE], s1[P::STAGE];
    __shared__ int found[P::BM / CRT_FM];
    if (threadIdx.x < P::BM / CRT_FM) found[threadIdx.x] = 0;
    const int tile = panel_xcd(blockIdx.x, ntm * ntn);
    const int m0 = (tile % ntm) * P::BM, n0 = (tile / ntm) * P::BN;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv % P::WM, wn = wv / P::WM, lr = lane & 31, lk = lane >> 5;
    typename P::Acc acc;
    const int half = nkb / 2;
    panel_product<P>(acc, s0, s1, half / P::KB, A + m0, lda, (int64_t)half * lda, B + n0, ldb, (int64_t)half * ldb,
                     PanelNoRaw{});
    const float margin = 1.f + 0x1p-22f * (float)K;
    const float ce = margin * 0.5f * (1.f / (float)(1 << (2 * MAG_SHIFT - 53))) / (float)(K > 9 ? K - 8 : 1);
    const float ck = margin * 4.f * (float)K;
    int bad = 0;
#pragma unroll
    for (int j = 0; j < P::TN; ++j) {
        const int col = n0 + wn * (P::BN / P::WN) + j * 32 + lr;
        const float nb = col < N ? bn[col] * ce : 0.f, qb = col < N ? bq[col] * ce : 0.f;
#pragma unroll
        for (int i = 0; i < P::TM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = m0 + wm * (P::BM / P::WM) + i * 32 + 8 * q + 4 * lk;
                const float4 na = *reinterpret_cast<const float4 *>(an + row);
                const float4 qa = *reinterpret_cast<const float4 *>(aq + row);
                const float need[4] = {ck + na.x * qb + qa.x * nb, ck + na.y * qb + qa.y * nb,
                                       ck + na.z * qb + qa.z * nb, ck + na.w * qb + qa.w * nb};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float m = acc[i][j][4 * q + c];
                    bad |= !(m >= need[c]) && !(m == 0.f && need[c] >= 0.f);
                }
            }
    }
    static_assert(P::BN == CRT_FN && P::BM / P::WM <= CRT_FM, "a wavefront's rows share a flag");
    if (__any(bad) && lane == 0) atomicOr(&found[wm * (P::BM / P::WM) / CRT_FM], 1);
    __syncthreads();
    const int r = m0 / CRT_FM + threadIdx.x;
    if (threadIdx.x < P::BM / CRT_FM && r < fm) flag[r * fn + n0 / CRT_FN] = (uint8_t)found[threadIdx.x];
}

// Residues of the products: work id = (modulus, column tile, row tile), row
// tiles fastest.  Bound by the INT8 matrix cores' sustained rate: 1.6-2.15
// POP/s at K >= 1000 (a library product of 8192^3 reaches 2.11 on this card);
// they are busy 55 % of the cycles at K = 3200 and 5200, 40-43 % at 1800 and 1000,
// where a tile's start and end weigh more.  out[modulus][row / 4][ld] holds four
// consecutive rows of a column per word.
template <class P>
__global__ __launch_bounds__(P::NT)
void k_crt_gemm(int ntm, int ntn, int nkb, const uint4 *__restrict__ A, int lda, int64_t apl,
                const uint4 *__restrict__ B, int ldb, int64_t bpl, uint32_t *__restrict__ out,
                const uint8_t *__restrict__ flag, int fm, int fn) {
    __shared__ uint4 s0[P::STAGE], s1[P::STAGE];
    const int ntile = ntm * ntn;
    const int id = panel_xcd(blockIdx.x, ntile * CRT_S);
    const int pm = id / ntile, tile = id % ntile;
    const int m0 = (tile % ntm) * P::BM, n0 = (tile / ntm) * P::BN;
    if (flag) {   // nothing of this tile is wanted
        bool none = true;
#pragma unroll
        for (int a = 0; a < P::BM / CRT_FM; ++a)
#pragma unroll
            for (int b = 0; b < P::BN / CRT_FN; ++b) {
                const int r = m0 / CRT_FM + a;
                none = none && (r >= fm || flag[r * fn + n0 / CRT_FN + b]);
            }
        if (none) return;
    }
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv % P::WM, wn = wv / P::WM, lr = lane & 31, lk = lane >> 5;
    typename P::Acc acc;
    panel_product<P>(acc, s0, s1, nkb / P::KB, A + pm * apl + m0, lda, apl, B + pm * bpl + n0, ldb, bpl,
                     PanelNoRaw{});
    const double inv = kModDev.inv[pm];
    const uint32_t p = (uint32_t)kModDev.p[pm];
    out += (int64_t)pm * (ntm * P::BM / 4) * ldb;
#pragma unroll
    for (int j = 0; j < P::TN; ++j) {
        const int col = n0 + wn * (P::BN / P::WN) + j * 32 + lr;
#pragma unroll
        for (int i = 0; i < P::TM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int quad = (m0 + wm * (P::BM / P::WM) + i * 32 + 8 * q + 4 * lk) / 4;
                uint32_t r[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int g = acc[i][j][4 * q + c];
                    r[c] = (uint32_t)g - __umul24(low_word(__builtin_fma((double)g, inv, kRint)), p);
                }
                out[(int64_t)quad * ldb + col] = pack4(r[0], r[1], r[2], r[3]);
            }
    }
}

// *n += number of flags set (test hook)
__global__ __launch_bounds__(256)
void k_crt_count(const uint8_t *__restrict__ flag, int nf, int *__restrict__ n) {
    int c = 0;
    for (int i = threadIdx.x; i < nf; i += 256) c += flag[i];
    if (c) atomicAdd(n, c);
}

// C [M][ldc] from the residues (quads of rows, `quads` of them per modulus);
// M % 4 == 0, rows' and columns' scales undone; optionally the frequency
// factor of column col0 + n (LORENTZ).  Thread (quad, n).  Bound by memory:
// CRT_S bytes read and 8 written per entry.
template <bool LORENTZ>
__global__ __launch_bounds__(256)
void k_crt_join(int M, int N, const uint32_t *__restrict__ res, int quads, int ld, const double *__restrict__ ai,
                const int *__restrict__ ae, const double *__restrict__ bi, const int *__restrict__ be,
                double *__restrict__ C, int ldc, int col0, LorentzArgs la, const uint8_t *__restrict__ flag,
                int fn) {
    const int n = blockIdx.x * 256 + threadIdx.x, quad = blockIdx.y;
    if (flag && flag[quad / (CRT_FM / 4) * fn + n / CRT_FN]) return;   // whole wavefronts
    const uint32_t *r = res + (int64_t)quad * ld + n;   // n < ld: the grid covers whole tiles of columns
    uint32_t w[CRT_S];
#pragma unroll
    for (int i = 0; i < CRT_S; ++i) w[i] = r[(int64_t)i * quads * ld];
    const bool ok = n < N;
    const double sb = ok ? mod_product() * bi[n] : 0.0;
    const int eb = ok ? be[n] : 0;
    const int cc = ok ? col0 + n : 0, E = LORENTZ ? cc / la.ncp : 0, jj = LORENTZ ? cc - E * la.ncp : 0;
    const Lorentz lz(LORENTZ ? la.omega[jj >> 1] : 0.0, la.eps, la.occ, jj & 1);
    double v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        double h = 0.0, l = 0.0;
#pragma unroll
        for (int i = 0; i < CRT_S; ++i) {
            const double x = (double)((int32_t)(w[i] << (24 - 8 * c)) >> 24);
            h = __builtin_fma(x, kW.hi[i], h);
            l = __builtin_fma(x, kW.lo[i], l);
        }
        const double f = (h - rint(h)) + l;   // C' / P
        const int row = 4 * quad + c;
        v[c] = ldexp(f * (sb * ai[row]), -(ae[row] + eb));
    }
    if (LORENTZ) {
        const double2 *D = reinterpret_cast<const double2 *>(la.Dlt + (int64_t)E * la.nv_pad + 4 * quad);
        const double2 D0 = D[0], D1 = D[1];
        v[0] = lz.apply(D0.x, v[0], lane_pair(v[0]));
        v[1] = lz.apply(D0.y, v[1], lane_pair(v[1]));
        v[2] = lz.apply(D1.x, v[2], lane_pair(v[2]));
        v[3] = lz.apply(D1.y, v[3], lane_pair(v[3]));
    }
    if (!ok) return;
#pragma unroll
    for (int c = 0; c < 4; ++c) __builtin_nontemporal_store(v[c], &C[(int64_t)(4 * quad + c) * ldc + n]);
}

template <int COLS, int ITEMS>
static void crt_cut_launch(hipStream_t s, const double *X, int K, int N, int64_t ldx, double lnorm, CrtDev &p) {
    hipLaunchKernelGGL((k_crt_cut<COLS, ITEMS>), dim3(p.p.ld / COLS), dim3(1024), 0, s, X, K, N, ldx, lnorm, p.sc,
                       p.p.nkb, p.p.ld, reinterpret_cast<uint4 *>(p.p.data), p.p.plane);
}

static void crt_cut(hipStream_t s, const double *X, int K, int N, int64_t ldx, double lnorm, CrtDev &p) {
    const int nkb = p.p.nkb;
    if (nkb <= 64) {
        crt_cut_launch<16, 1>(s, X, K, N, ldx, lnorm, p);
    } else if (nkb <= 128) {
        crt_cut_launch<16, 2>(s, X, K, N, ldx, lnorm, p);
    } else if (nkb <= 256) {
        crt_cut_launch<8, 2>(s, X, K, N, ldx, lnorm, p);
    } else if (nkb <= 384) {
        crt_cut_launch<8, 3>(s, X, K, N, ldx, lnorm, p);
    } else {
        hipLaunchKernelGGL(k_crt_scale_long, dim3((N + 63) / 64), dim3(1024), 0, s, X, K, N, ldx, lnorm, p.sc);
        int64_t blocks = ((int64_t)nkb * p.p.ld + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(k_crt_cut_long, dim3((unsigned)blocks), dim3(256), 0, s, X, K, N, ldx,
                           (const double *)p.sc.sm, (const int *)p.sc.se, nkb, p.p.ld, reinterpret_cast<uint4 *>(p.p.data),
                           p.p.plane);
    }
}

void launch_crt_operand(hipStream_t s, const double *X, int K, int N, int64_t ldx, CrtDev &p) {
    crt_cut(s, X, K, N, ldx, kNormA, p);
}

// The INT8 products replace 2 M K N operations at 40-55 TFLOP/s by 30 M K N (with
// the check) at 1.1-2.1 POP/s and 24 (M + K) N bytes, so what counts is
// h = M K / (M + K).  chi0 z in FP64 and this way, us, by vectors:
//   h (N, Nv)             1           3           8            16            64
//   650 (1800, 1000)   391 / 353   850 / 722  1989 / 1636  3819 / 3201
//   555 (1500, 860)    271 / 235   517 / 424  1183 /  978  2226 / 1930  8378 / 7327
//   480 (1300, 740)    200 / 194   383 / 339   813 /  746  1562 / 1448  5845 / 5346
//   444 (1200, 700)    187 / 191   345 / 302   694 /  652  1297 / 1272  4779 / 4731
//   406 (1100, 630)    156 / 172   274 / 265   585 /  541  1056 / 1031  3859 / 3881
//   350 (917, 528)     105 / 144   207 / 201   343 /  363   635 /  679  2278 / 2567
// Up to CRT_FEW columns it also wins between 400 and 460, where the FP64 tiles are few
// (12 vectors at 406: 820 / 780; 372, 5 and 7 vectors: 328 / 323, 387 / 392); below
// 1024 columns the fixed cost of its five kernels shows.  K < 2^17: exact 32-bit sums.
bool crt_pays(int M, int K, int64_t N) {
    const double h = (double)M * K / ((double)M + K);
    return K < (1 << 17) && M < (1 << 17) && N >= 1024 && (h >= 460.0 || (h >= 400.0 && N <= CRT_FEW));
}

// bytes of workspace per column of B: scale (28) and flags (one byte per 64 x 128
// tile: 16 a column are enough for M <= 2^17), planes of B, residues of C
constexpr int CRT_COL_HEAD = 28 + 16;
static int64_t crt_column_bytes(int rows, int nkb) {
    return CRT_COL_HEAD + (int64_t)CRT_P * nkb * 16 + (int64_t)CRT_S * rows;
}

int64_t crt_work_bytes(int M, int K, int64_t N) {
    return crt_column_bytes((int)round_up(M, CRT_LD), (int)round_up((K + 15) / 16, CRT_KB)) * round_up(N, CRT_LD);
}

template <class P>
static void crt_gemm_launch(hipStream_t s, int rows, const CrtDev &A, const CrtDev &B, uint32_t *res,
                            const uint8_t *flag, int fm) {
    const int ntm = rows / P::BM, ntn = B.p.ld / P::BN;
    hipLaunchKernelGGL((k_crt_gemm<P>), dim3(ntm * ntn * CRT_S), dim3(P::NT), 0, s, ntm, ntn, A.p.nkb,
                       reinterpret_cast<const uint4 *>(A.p.data), A.p.ld, A.p.plane,
                       reinterpret_cast<const uint4 *>(B.p.data), B.p.ld, B.p.plane, res, flag, fm, B.p.ld / CRT_FN);
}

// Stages of two k-blocks of either half, which any operand has whole ones of.  us for
// both transforms, 200 atoms, 12 vectors / 400 atoms, 4: 120 / 677; stages of four
// where the blocks are a multiple of 8, 125 / 652; two workgroups per CU instead of
// three 154 / 655; 64 x 128 tiles 157 / 814, 256 x 128 209 / 855, 256 x 256 154 / 685.
static void crt_check(hipStream_t s, int K, int N, const CrtDev &A, const CrtDev &B, uint8_t *flag, int fm) {
    typedef PanelShape<FormMag, 128, CRT_FN, 2, 2, 2> P;
    static_assert(CRT_KB % (2 * P::KB) == 0, "whole stages in either half");
    const int ntm = (fm * CRT_FM + P::BM - 1) / P::BM, fn = B.p.ld / CRT_FN;
    hipLaunchKernelGGL((k_crt_check<P>), dim3(ntm * fn), dim3(P::NT), 0, s, ntm, fn, A.p.nkb, K, N,
                       reinterpret_cast<const uint4 *>(A.p.data) + CRT_S * A.p.plane, A.p.ld, (const float *)A.sc.nrm,
                       (const float *)A.sc.rnz, reinterpret_cast<const uint4 *>(B.p.data) + CRT_S * B.p.plane, B.p.ld,
                       (const float *)B.sc.nrm, (const float *)B.sc.rnz, flag, fm, fn);
}

void launch_crt_gemm(Tracer *t, hipStream_t s, const char *name, int M, int N, int K, const CrtDev &A,
                     const double *B, int64_t ldb, void *work, size_t work_bytes, double *C, int ldc, double flops,
                     double bytes, const LorentzArgs *la, const CrtExact *exact, int *flagged) {
    const int nkb = A.p.nkb;
    const int64_t fit = (int64_t)work_bytes / crt_column_bytes((int)round_up(M, CRT_LD), nkb) / CRT_LD * CRT_LD;
    // as few chunks as fit, of equal size
    const int nch = (int)((N + fit - 1) / fit), chunk = (int)round_up((N + nch - 1) / nch, CRT_LD);
    // rows of tiles: 256 rows have fewer LDS reads per MFMA (M = 3200, K = 5200: 2.15 against 1.95
    // POP/s); 128 waste fewer rows, and two such workgroups per CU hide each other's start and
    // end where K is short (M = 528, K = 917: 60 against 68 us for 5600 columns)
    const int m256 = (M + 255) / 256 * 256, m128 = (M + 127) / 128 * 128;
    const bool big = K >= 1024 && m256 <= 1.07 * m128;
    const int rows = big ? m256 : m128, quads = rows / 4, fm = (M + CRT_FM - 1) / CRT_FM;
    const LorentzArgs none{};
    for (int c0 = 0; c0 < N; c0 += chunk) {
        const int n = std::min(chunk, N - c0), ld = (int)round_up(n, CRT_LD), fn = ld / CRT_FN;
        const double share = (double)n / N;
        CrtDev b;
        b.p.ld = ld;
        b.p.nkb = nkb;
        b.p.plane = (int64_t)nkb * ld;
        b.sc.sm = static_cast<double *>(work);
        b.sc.si = b.sc.sm + ld;
        b.sc.se = reinterpret_cast<int *>(b.sc.si + ld);
        b.sc.nrm = reinterpret_cast<float *>(b.sc.se + ld);
        b.sc.rnz = b.sc.nrm + ld;
        uint8_t *flag = exact ? reinterpret_cast<uint8_t *>(b.sc.rnz + ld) : nullptr;
        b.p.data = static_cast<char *>(work) + (int64_t)CRT_COL_HEAD * ld;
        uint32_t *res = reinterpret_cast<uint32_t *>(static_cast<uint4 *>(b.p.data) + CRT_P * b.p.plane);
        trace_begin(t, "crt_cut", s);
        crt_cut(s, B + c0, K, n, ldb, kNormB, b);
        trace_end(t, s, 0.0, (16.0 + CRT_P) * (double)K * n);
        if (flag) {
            trace_begin(t, "crt_check", s);
            crt_check(s, K, n, A, b, flag, fm);
            trace_end(t, s, 2.0 * M * (double)K * n, (double)K * (M + n));
            if (flagged)
                hipLaunchKernelGGL(k_crt_count, dim3(1), dim3(256), 0, s, (const uint8_t *)flag, fm * fn, flagged);
        }
        trace_begin(t, name, s);
        if (big && nkb % 8 == 0)
            crt_gemm_launch<PanelShape<FormI8, 256, 256, 2, 4, 8>>(s, rows, A, b, res, flag, fm);
        else if (big)
            crt_gemm_launch<PanelShape<FormI8, 256, 256, 2, 4, 4>>(s, rows, A, b, res, flag, fm);
        else
            crt_gemm_launch<PanelShape<FormI8, 128, 256, 2, 4, 4>>(s, rows, A, b, res, flag, fm);
        trace_end(t, s, flops * share, bytes * share);
        trace_begin(t, "crt_join", s);
        hipLaunchKernelGGL(la ? k_crt_join<true> : k_crt_join<false>, dim3(ld / 256, M / 4), dim3(256), 0, s, M, n,
                           (const uint32_t *)res, quads, ld, (const double *)A.sc.si, (const int *)A.sc.se,
                           (const double *)b.sc.si, (const int *)b.sc.se, C + c0, ldc, c0, la ? *la : none,
                           (const uint8_t *)flag, fn);
        trace_end(t, s, 0.0, (CRT_S + 8.0) * (double)M * n);
        if (flag) {
            trace_begin(t, "crt_fp64_tiles", s);
            launch_dgemm_flagged(s, M, n, exact->K, exact->A, exact->lda, B + c0, (int)ldb, C + c0, ldc, c0, la, flag, fn);
            trace_end(t, s);
        }
    }
}

}  // namespace chi0
