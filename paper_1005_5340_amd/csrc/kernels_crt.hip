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
// its row or column, and the error of C_ij is about |A_i| |B_j| 2^-55.  An
// FP64 sum of K products rounds K times.  Relative error of the transforms
// (sampled against extended precision, two seeds), this way and by the FP64
// GEMM, in 1e-16:
//   K   470   528   550   810   900  1000  1690  1800  3200  5200
//       4.5   4.8   4.9   5.1   4.7   6.0   6.3   7.2   8.4  10.6
//       5.4   6.4   6.4   5.9   5.0   8.7   9.6  13.2  22.8  25.9
//
// A column with an infinity or NaN gives NaN.
#include "panel_core.h"

namespace chi0 {

typedef int int4v __attribute__((ext_vector_type(4)));
typedef int int16v __attribute__((ext_vector_type(16)));

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

}  // namespace

// Scale 2^e m of a column from its sum of squares and largest entry: its norm
// is brought to 2^lnorm and its largest entry to at most 2^53.  bad != 0 (a
// NaN): the column holds an infinity or NaN, m becomes NaN.  A norm out of
// range for its sum of squares is replaced by its bound sqrt(K) max.
__device__ __forceinline__ void crt_scale(double ss, double mx, double bad, int K, double lnorm, double &m, int &e) {
    m = 1.0;
    e = 0;
    if (bad != 0.0) {
        m = bad;
    } else if (mx > 0.0) {
        int em;
        const double fm = frexp(mx, &em);   // mx = fm 2^em
        const double lmax = log2(fm) + em;
        const double ln = ss > 1e-280 && ss < 1e300 ? 0.5 * log2(ss) : 0.5 * log2((double)K) + lmax;
        const double l = fmin(lnorm - ln, 52.9999 - lmax);
        e = (int)floor(l);
        m = exp2(l - e);
    }
}

// Residues of 16 entries a 2^e m, rounded to whole numbers of at most 53 bits,
// for every modulus: 16 bytes per plane.  a mod p is the low byte of
// lo(a) - lo(rint(a / p)) p, whatever the higher bits are.
__device__ __forceinline__ void crt_residues(double (&a)[16], int e, double m, uint4 *__restrict__ out,
                                             int64_t plane) {
    uint32_t lo[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        a[c] = rint(ldexp(a[c], e) * m);
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
// bytes per plane and k-block.  Bound by memory: 8 bytes read and CRT_S
// written per entry, at 3.7-4.5 TB/s.  (As two kernels, which read X twice, 200
// atoms, 12 vectors: 459 us for both transforms, now 270-315; 400 atoms, 16
// vectors 6.4 -> 3.4 ms.)
template <int COLS, int ITEMS>
__global__ __launch_bounds__(1024)
void k_crt_cut(const double *__restrict__ X, int K, int N, int64_t ldx, double lnorm, double *__restrict__ sm,
               double *__restrict__ si, int *__restrict__ se, int nkb, int ld, uint4 *__restrict__ out,
               int64_t plane) {
    __shared__ double sh[3][16][COLS];
    __shared__ double shm[COLS];
    __shared__ int she[COLS];
    const int t = threadIdx.x, lane = t & 63, col = t % COLS;
    const int n = panel_xcd(blockIdx.x, gridDim.x) * COLS + col;
    double a[ITEMS][16], ss = 0.0, mx = 0.0, bad = 0.0;
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
        }
#pragma unroll
    for (int o = 32; o >= COLS; o >>= 1) {
        ss += __shfl_xor(ss, o);
        mx = fmax(mx, __shfl_xor(mx, o));
        bad += __shfl_xor(bad, o);
    }
    if (lane < COLS) {
        sh[0][t >> 6][lane] = ss;
        sh[1][t >> 6][lane] = mx;
        sh[2][t >> 6][lane] = bad;
    }
    __syncthreads();
    if (t < COLS) {
        ss = mx = bad = 0.0;
        for (int g = 0; g < 16; ++g) {
            ss += sh[0][g][t];
            mx = fmax(mx, sh[1][g][t]);
            bad += sh[2][g][t];
        }
        double m;
        int e;
        crt_scale(ss, mx, bad, K, lnorm, m, e);
        shm[t] = m;
        she[t] = e;
        if (n < N) {
            sm[n] = m;
            si[n] = 1.0 / m;
            se[n] = e;
        }
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
void k_crt_scale_long(const double *__restrict__ X, int K, int N, int64_t ldx, double lnorm, double *__restrict__ sm,
                      double *__restrict__ si, int *__restrict__ se) {
    __shared__ double sh[3][16][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6, n = blockIdx.x * 64 + lane;
    double ss = 0.0, mx = 0.0, bad = 0.0;
    if (n < N) {
        const double *x = X + n;
#pragma unroll 8
        for (int k = g; k < K; k += 16) {
            const double v = x[(int64_t)k * ldx];
            ss += v * v;
            mx = fmax(mx, fabs(v));
            bad += v * 0.0;
        }
    }
    sh[0][g][lane] = ss;
    sh[1][g][lane] = mx;
    sh[2][g][lane] = bad;
    __syncthreads();
    if (g != 0 || n >= N) return;
#pragma unroll
    for (int i = 1; i < 16; ++i) {
        ss += sh[0][i][lane];
        mx = fmax(mx, sh[1][i][lane]);
        bad += sh[2][i][lane];
    }
    double m;
    int e;
    crt_scale(ss, mx, bad, K, lnorm, m, e);
    sm[n] = m;
    si[n] = 1.0 / m;
    se[n] = e;
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

// Residues of the products: work id = (modulus, column tile, row tile), row
// tiles fastest.  Bound by the INT8 matrix cores' sustained rate: 1.7-2.15
// POP/s at K >= 1000 (a library product of 8192^3 reaches 2.11 on this card).  out[modulus][row / 4][ld] holds four consecutive rows of a
// column per word.
template <class P>
__global__ __launch_bounds__(P::NT)
void k_crt_gemm(int ntm, int ntn, int nkb, const uint4 *__restrict__ A, int lda, int64_t apl,
                const uint4 *__restrict__ B, int ldb, int64_t bpl, uint32_t *__restrict__ out) {
    __shared__ uint4 s0[P::STAGE], s1[P::STAGE];
    const int ntile = ntm * ntn;
    const int id = panel_xcd(blockIdx.x, ntile * CRT_S);
    const int pm = id / ntile, tile = id % ntile;
    const int m0 = (tile % ntm) * P::BM, n0 = (tile / ntm) * P::BN;
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

// C [M][ldc] from the residues (quads of rows, `quads` of them per modulus);
// M % 4 == 0, rows' and columns' scales undone; optionally the frequency
// factor of column col0 + n (LORENTZ).  Thread (quad, n).  Bound by memory:
// CRT_S bytes read and 8 written per entry.
template <bool LORENTZ>
__global__ __launch_bounds__(256)
void k_crt_join(int M, int N, const uint32_t *__restrict__ res, int quads, int ld, const double *__restrict__ ai,
                const int *__restrict__ ae, const double *__restrict__ bi, const int *__restrict__ be,
                double *__restrict__ C, int ldc, int col0, LorentzArgs la) {
    const int n = blockIdx.x * 256 + threadIdx.x, quad = blockIdx.y;
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
    hipLaunchKernelGGL((k_crt_cut<COLS, ITEMS>), dim3(p.p.ld / COLS), dim3(1024), 0, s, X, K, N, ldx, lnorm, p.sm,
                       p.si, p.se, p.p.nkb, p.p.ld, reinterpret_cast<uint4 *>(p.p.data), p.p.plane);
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
        hipLaunchKernelGGL(k_crt_scale_long, dim3((N + 63) / 64), dim3(1024), 0, s, X, K, N, ldx, lnorm, p.sm, p.si,
                           p.se);
        int64_t blocks = ((int64_t)nkb * p.p.ld + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(k_crt_cut_long, dim3((unsigned)blocks), dim3(256), 0, s, X, K, N, ldx,
                           (const double *)p.sm, (const int *)p.se, nkb, p.p.ld, reinterpret_cast<uint4 *>(p.p.data),
                           p.p.plane);
    }
}

void launch_crt_operand(hipStream_t s, const double *X, int K, int N, int64_t ldx, CrtDev &p) {
    crt_cut(s, X, K, N, ldx, kNormA, p);
}

// The INT8 products replace 2 M K N operations at 40-55 TFLOP/s by 28 M K N at
// 1.1-1.9 POP/s and 22 (M + K) N bytes, so what counts is M K / (M + K).
// chi0 z in FP64 and this way, us (200 atoms: M K / (M + K) = 643):
//   vectors      3            8            16           32
//   643      949 /  748  2067 / 1573  3913 / 2974  7486 / 5656
//   355      294 /  246   567 /  490   950 /  907  1664 / 1659
//   335      242 /  201   424 /  382   717 /  706  1220 / 1250
//   297      200 /  172   329 /  304   536 /  542   937 / 1016
//   193      121 /  132   188 /  180   265 /  274   413 /  481
// Up to 8192 columns it also wins below 345, where the FP64 tiles are few and
// need split-K; below 1024 columns the fixed cost of its three kernels shows
// (335, 1 vector, 778 columns: 144 / 146).  K < 2^17: exact 32-bit sums.
bool crt_pays(int M, int K, int64_t N) {
    const double h = (double)M * K / ((double)M + K);
    return K < (1 << 17) && N >= 1024 && (h >= 345.0 || (h >= 290.0 && N <= 8192));
}

// bytes of workspace per column of B: residues of B and of C, scale
static int64_t crt_column_bytes(int rows, int nkb) { return (int64_t)CRT_S * nkb * 16 + (int64_t)CRT_S * rows + 32; }

int64_t crt_work_bytes(int M, int K, int64_t N) {
    return crt_column_bytes((int)round_up(M, CRT_LD), (int)round_up((K + 15) / 16, CRT_KB)) * round_up(N, CRT_LD);
}

template <class P>
static void crt_gemm_launch(hipStream_t s, int rows, const CrtDev &A, const CrtDev &B, uint32_t *res) {
    const int ntm = rows / P::BM, ntn = B.p.ld / P::BN;
    hipLaunchKernelGGL((k_crt_gemm<P>), dim3(ntm * ntn * CRT_S), dim3(P::NT), 0, s, ntm, ntn, A.p.nkb,
                       reinterpret_cast<const uint4 *>(A.p.data), A.p.ld, A.p.plane,
                       reinterpret_cast<const uint4 *>(B.p.data), B.p.ld, B.p.plane, res);
}

void launch_crt_gemm(Tracer *t, hipStream_t s, const char *name, int M, int N, int K, const CrtDev &A,
                     const double *B, int64_t ldb, void *work, size_t work_bytes, double *C, int ldc, double flops,
                     double bytes, const LorentzArgs *la) {
    const int nkb = A.p.nkb;
    const int64_t fit = (int64_t)work_bytes / crt_column_bytes((int)round_up(M, CRT_LD), nkb) / CRT_LD * CRT_LD;
    // as few chunks as fit, of equal size
    const int nch = (int)((N + fit - 1) / fit), chunk = (int)round_up((N + nch - 1) / nch, CRT_LD);
    // rows of tiles: 256 rows have fewer LDS reads per MFMA (M = 3200, K = 5200: 2.15 against 1.95
    // POP/s); 128 waste fewer rows, and two such workgroups per CU hide each other's start and
    // end where K is short (M = 528, K = 917: 60 against 68 us for 5600 columns)
    const int m256 = (M + 255) / 256 * 256, m128 = (M + 127) / 128 * 128;
    const bool big = K >= 1024 && m256 <= 1.07 * m128;
    const int rows = big ? m256 : m128, quads = rows / 4;
    const LorentzArgs none{};
    for (int c0 = 0; c0 < N; c0 += chunk) {
        const int n = std::min(chunk, N - c0), ld = (int)round_up(n, CRT_LD);
        const double share = (double)n / N;
        CrtDev b;
        b.p.ld = ld;
        b.p.nkb = nkb;
        b.p.plane = (int64_t)nkb * ld;
        b.sm = static_cast<double *>(work);
        b.si = b.sm + ld;
        b.se = reinterpret_cast<int *>(b.si + ld);
        b.p.data = b.sm + 4 * ld;
        uint32_t *res = reinterpret_cast<uint32_t *>(static_cast<uint4 *>(b.p.data) + CRT_S * b.p.plane);
        trace_begin(t, "crt_cut", s);
        crt_cut(s, B + c0, K, n, ldb, kNormB, b);
        trace_end(t, s, 0.0, (16.0 + CRT_S) * (double)K * n);
        trace_begin(t, name, s);
        if (big && nkb % 8 == 0)
            crt_gemm_launch<PanelShape<FormI8, 256, 256, 2, 4, 8>>(s, rows, A, b, res);
        else if (big)
            crt_gemm_launch<PanelShape<FormI8, 256, 256, 2, 4, 4>>(s, rows, A, b, res);
        else
            crt_gemm_launch<PanelShape<FormI8, 128, 256, 2, 4, 4>>(s, rows, A, b, res);
        trace_end(t, s, flops * share, bytes * share);
        trace_begin(t, "crt_join", s);
        if (la)
            hipLaunchKernelGGL(k_crt_join<true>, dim3(ld / 256, M / 4), dim3(256), 0, s, M, n, (const uint32_t *)res,
                               quads, ld, (const double *)A.si, (const int *)A.se, (const double *)b.si,
                               (const int *)b.se, C + c0, ldc, c0, *la);
        else
            hipLaunchKernelGGL(k_crt_join<false>, dim3(ld / 256, M / 4), dim3(256), 0, s, M, n, (const uint32_t *)res,
                               quads, ld, (const double *)A.si, (const int *)A.se, (const double *)b.si,
                               (const int *)b.se, C + c0, ldc, c0, none);
        trace_end(t, s, 0.0, (CRT_S + 8.0) * (double)M * n);
    }
}

}  // namespace chi0
