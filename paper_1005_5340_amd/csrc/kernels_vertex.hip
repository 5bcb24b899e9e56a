// Vertex kernels of the matrix-free chi0 product (Sec. 4.2, Table t:flops
// steps 2 and 5): the contraction of the product-space vector with the
// sparse vertex, dV_ab = sum_mu z_mu V_mu^{ab}, and its transpose, the
// projection n_mu = sum_ab V_mu^{ab} W_ab.
//
// The vertex is stored per atom-pair block (A, B) as a panel holding, for
// every product whose support covers (A, B), its n_A x n_B sub-block.  Both
// kernels walk one block per workgroup, so every vertex element is read
// once per call and no atomics are needed: the projection writes one
// partial sum per (block, product) and a second pass adds the (at most 4)
// partials of each product in a fixed order.
#include "common.h"

namespace chi0 {

typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ dbl4 mfma16(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Both vertex kernels are small GEMMs per atom-pair block on the FP64 matrix
// cores (16x16x4; lane l holds A[l%16][l/16], B[l/16][l%16] and returns
// D[4r + l/16][l%16]).  A workgroup owns one block and VC 16-column MFMA
// blocks; wave w of four owns the 16-row blocks w, w+4, w+8, w+12 of the
// block's output.  Each round issues the operand loads of KU k-steps before
// their MFMAs, so a round costs about one memory latency, and the time is set
// by the rounds of the longest block: a diagonal block (A, A) carries every
// product that involves atom A (175 at 60 atoms, where others carry 8).
//
// The split kernels take 16 columns of a block per workgroup of eight
// wavefronts: groups of row blocks times slices of the reduction, which cut the
// longest block's rounds; the slices' sums are added in a fixed order through
// LDS.  How a workgroup splits depends on its block alone.  One vector, 60
// atoms: gather 18.6 -> 13.9 us, projection 14.7 -> 8.9 us; projection at 12
// atoms, 48 columns 15.5 -> 7.9 (with the tracer's ~5 us).
constexpr int VRB = 4;     // 16-row MFMA blocks per wave (rows <= 256 = NB_MAX^2)
constexpr int PCH = 256;   // product ids staged in LDS per chunk

// (a) dV[(ent_k + ab)][j] = sum_i Vp[k][i][ab] * Z[pidx[k][i]][j]
//     rows = ab (n_A n_B), K = the block's products, columns = j.
template <int VC, int KU>
__global__ __launch_bounds__(256)
void k_vertex_gather(BlockMapDev bm, const double *__restrict__ Z, double *__restrict__ dV, int nc) {
    __shared__ int32_t ps[PCH];
    const int k = blockIdx.x, j0 = blockIdx.y * 16 * VC;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int nAB = bm.blk_na[k] * bm.blk_nb[k];
    const int np = bm.blk_nprod[k];
    const double *Vk = bm.Vp + bm.blk_vstart[k];
    const int32_t *pk = bm.pidx + bm.blk_pstart[k];
    const int64_t ent = bm.blk_ent[k];
    const int nrb = (nAB + 15) / 16, ncb = min(VC, (nc - j0 + 15) / 16);
    const int lr = lane & 15, lk = lane >> 4;

    dbl4 acc[VRB][VC];
#pragma unroll
    for (int r = 0; r < VRB; ++r)
#pragma unroll
        for (int c = 0; c < VC; ++c) acc[r][c] = dbl4{0.0, 0.0, 0.0, 0.0};

    for (int c0 = 0; c0 < np; c0 += PCH) {
        const int cn = min(PCH, np - c0);
        __syncthreads();
        if (t < cn) ps[t] = pk[c0 + t];
        __syncthreads();
        // KU k-steps of 4 products per round: all their loads are issued
        // before their MFMAs; k-steps past the chunk's end are skipped
        for (int i0 = 0; i0 < cn; i0 += 4 * KU) {
            double a[KU][VRB], b[KU][VC];
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const int kk = i0 + 4 * u + lk;
                const bool kv = kk < cn;
                const int64_t zrow = kv ? (int64_t)ps[kk] * nc : 0;
#pragma unroll
                for (int r = 0; r < VRB; ++r) {
                    const int row = (wv + 4 * r) * 16 + lr;
                    a[u][r] = (kv && row < nAB) ? Vk[(int64_t)(c0 + kk) * nAB + row] : 0.0;
                }
#pragma unroll
                for (int c = 0; c < VC; ++c) {
                    const int j = j0 + c * 16 + lr;
                    b[u][c] = (kv && j < nc) ? Z[zrow + j] : 0.0;
                }
            }
#pragma unroll
            for (int r = 0; r < VRB; ++r) {
                if (wv + 4 * r >= nrb) continue;
#pragma unroll
                for (int u = 0; u < KU; ++u) {
                    if (i0 + 4 * u >= cn) continue;
#pragma unroll
                    for (int c = 0; c < VC; ++c)
                        if (c < ncb) acc[r][c] = mfma16(a[u][r], b[u][c], acc[r][c]);
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < VRB; ++r) {
        if (wv + 4 * r >= nrb) continue;
#pragma unroll
        for (int c = 0; c < VC; ++c) {
            const int j = j0 + c * 16 + lr;
            if (c >= ncb || j >= nc) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = (wv + 4 * r) * 16 + 4 * e + lk;
                if (row < nAB) dV[(ent + row) * nc + j] = acc[r][c][e];
            }
        }
    }
}

// Sum over the KS slices of a workgroup of 8 wavefronts (wave = slice RG +
// group) in a fixed order; slice 0 holds the result.  red: 4 wavefronts' sums.
template <int NR>
__device__ __forceinline__ void vertex_sum_slices(dbl4 (&acc)[NR], int KS, int RG, int wv, int lane,
                                                  dbl4 (*red)[NR][64]) {
    for (int h = KS / 2; h >= 1; h /= 2) {   // uniform over the workgroup
        const int hi = wv - h * RG;          // place of the slice h above
        if (hi >= 0 && wv < 2 * h * RG)
#pragma unroll
            for (int r = 0; r < NR; ++r) red[hi][r][lane] = acc[r];
        __syncthreads();
        if (wv < h * RG)
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] += red[wv][r][lane];
        __syncthreads();
    }
}

// The gather for up to 16 columns and few blocks.
template <int KU>
__global__ __launch_bounds__(512)
void k_vertex_gather_split(BlockMapDev bm, const double *__restrict__ Z, double *__restrict__ dV, int nc) {
    __shared__ dbl4 red[4][VRB][64];
    const int k = blockIdx.x, j = threadIdx.x & 15;   // block, this lane's column
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nAB = bm.blk_na[k] * bm.blk_nb[k];
    const int np = bm.blk_nprod[k];
    const double *Vk = bm.Vp + bm.blk_vstart[k];
    const int32_t *pk = bm.pidx + bm.blk_pstart[k];
    const int64_t ent = bm.blk_ent[k];
    const int nrb = (nAB + 15) / 16;
    const int lr = lane & 15, lk = lane >> 4;
    // one round of products: every wave its own rows.  More: two or four row
    // groups (of VRB row blocks each: 128 or 256 rows) and the slices.
    const int RG = np <= 4 * KU ? 8 : nrb <= 2 * VRB ? 2 : 4, KS = 8 / RG;
    const int rg = wv % RG, ks = wv / RG;

    dbl4 acc[VRB];
#pragma unroll
    for (int r = 0; r < VRB; ++r) acc[r] = dbl4{0.0, 0.0, 0.0, 0.0};

    for (int i0 = ks * 4 * KU; i0 < np; i0 += KS * 4 * KU) {
        double a[KU][VRB], b[KU];
        int32_t pz[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int kk = i0 + 4 * u + lk;
            pz[u] = kk < np ? pk[kk] : 0;
        }
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int kk = i0 + 4 * u + lk;
            const bool kv = kk < np;
#pragma unroll
            for (int r = 0; r < VRB; ++r) {
                const int row = (rg + RG * r) * 16 + lr;
                a[u][r] = (kv && row < nAB) ? Vk[(int64_t)kk * nAB + row] : 0.0;
            }
            b[u] = (kv && j < nc) ? Z[(int64_t)pz[u] * nc + j] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < VRB; ++r) {
            if (rg + RG * r >= nrb) continue;
#pragma unroll
            for (int u = 0; u < KU; ++u)
                if (i0 + 4 * u < np) acc[r] = mfma16(a[u][r], b[u], acc[r]);
        }
    }
    vertex_sum_slices<VRB>(acc, KS, RG, wv, lane, red);
    if (ks != 0 || j >= nc) return;
#pragma unroll
    for (int r = 0; r < VRB; ++r) {
        if (rg + RG * r >= nrb) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = (rg + RG * r) * 16 + 4 * e + lk;
            if (row < nAB) dV[(ent + row) * nc + j] = acc[r][e];
        }
    }
}

// Blocks (times 16-column groups, the projection) up to which the kernels split,
// the gather for up to 16 columns; the projection of up to 16 columns splits for
// any number of blocks.  The gather's limit of 16 columns is not one of speed (12
// atoms, 48 columns: 16.1 us with four waves, 12.1 with eight): the two-sided
// Lanczos recursion stops at a step that follows the rounding (4950-6130 steps over
// summation orders at 12 atoms), and the order of the split sums takes it out of
// the band around the oracle's count that its test allows.  Past four workgroups per CU the launch runs in several
// waves and the idle wavefronts of the short blocks cost more than the long ones
// gain (gather, us, four waves / eight: 758 blocks 20.3 / 14.8, 780 17.2 / 14.9;
// 1246 12.7 / 17.0, 1349 12.8 / 18.9, 1954 23.5 / 28.2).
constexpr int VSPLIT_BLK = 1024;

// 16-column MFMA blocks per workgroup for nc columns: 1 up to 16 columns,
// 2 up to 32, else 4
static int vertex_vc(int nc) { return nc <= 16 ? 1 : nc <= 32 ? 2 : 4; }

void launch_vertex_gather(Tracer *t, hipStream_t s, const BlockMapDev &bm, int n_blk,
                          const double *Z, double *dV, int nc, const WorkSizes &ws) {
    const int vc = vertex_vc(nc);
    dim3 grid(n_blk, (nc + 16 * vc - 1) / (16 * vc));
    trace_begin(t, "vertex_gather", s);
    if (vc == 1 && n_blk <= VSPLIT_BLK)
        hipLaunchKernelGGL((k_vertex_gather_split<8>), dim3(n_blk), dim3(512), 0, s, bm, Z, dV, nc);
    else if (vc == 1)
        hipLaunchKernelGGL((k_vertex_gather<1, 8>), grid, dim3(256), 0, s, bm, Z, dV, nc);
    else if (vc == 2)
        hipLaunchKernelGGL((k_vertex_gather<2, 8>), grid, dim3(256), 0, s, bm, Z, dV, nc);
    else
        hipLaunchKernelGGL((k_vertex_gather<4, 4>), grid, dim3(256), 0, s, bm, Z, dV, nc);
    trace_end(t, s, 2.0 * ws.sum_s2 * nc, 8.0 * (ws.sum_s2 + ws.P * nc + ws.nnzB * nc));
}

// (d), first pass: part[pstart_k + i][j] = sum_ab Vp[k][i][ab] * W[(ent_k + ab)][j]
//     rows = the block's products, K = ab, columns = j.
// A workgroup whose products fit one 16-row MFMA block (every off-diagonal
// block: it carries only its pair's bilocal products) would leave three of
// its four waves idle through the whole ab range; there the waves take
// turns over the rounds of k-steps instead (wave w the rounds w, w+4, ...)
// and their partial sums are added in wave order through LDS.
template <int VC, int KU>
__global__ __launch_bounds__(256)
void k_vertex_contract(BlockMapDev bm, const double *__restrict__ W, double *__restrict__ part,
                       int nc) {
    __shared__ dbl4 red[3][VC][64];   // partial sums of waves 1-3 when the k range is split
    const int k = blockIdx.x, j0 = blockIdx.y * 16 * VC, rb0 = blockIdx.z * 4 * VRB;
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nAB = bm.blk_na[k] * bm.blk_nb[k];
    const int np = bm.blk_nprod[k];
    const double *Vk = bm.Vp + bm.blk_vstart[k];
    const int64_t ent = bm.blk_ent[k];
    const int64_t p0 = bm.blk_pstart[k];
    const int nrb = (np + 15) / 16, ncb = min(VC, (nc - j0 + 15) / 16);
    if (rb0 >= nrb) return;
    const int lr = lane & 15, lk = lane >> 4;
    const bool split = nrb - rb0 == 1;          // uniform over the workgroup
    const int rw = split ? 0 : wv;              // this wave's first row block (past rb0)
    const int kstep = (split ? 4 : 1) * 4 * KU; // ab advanced per round of this wave

    dbl4 acc[VRB][VC];
#pragma unroll
    for (int r = 0; r < VRB; ++r)
#pragma unroll
        for (int c = 0; c < VC; ++c) acc[r][c] = dbl4{0.0, 0.0, 0.0, 0.0};

    for (int a0 = (split ? wv : 0) * 4 * KU; a0 < nAB; a0 += kstep) {
        double a[KU][VRB], b[KU][VC];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int kk = a0 + 4 * u + lk;
            const bool kv = kk < nAB;
#pragma unroll
            for (int r = 0; r < VRB; ++r) {
                const int i = (rb0 + rw + 4 * r) * 16 + lr;
                a[u][r] = (kv && i < np) ? Vk[(int64_t)i * nAB + kk] : 0.0;
            }
#pragma unroll
            for (int c = 0; c < VC; ++c) {
                const int j = j0 + c * 16 + lr;
                b[u][c] = (kv && j < nc) ? W[(ent + kk) * nc + j] : 0.0;
            }
        }
#pragma unroll
        for (int r = 0; r < VRB; ++r) {
            if (rb0 + rw + 4 * r >= nrb) continue;
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                if (a0 + 4 * u >= nAB) continue;
#pragma unroll
                for (int c = 0; c < VC; ++c)
                    if (c < ncb) acc[r][c] = mfma16(a[u][r], b[u][c], acc[r][c]);
            }
        }
    }
    if (split) {
        if (wv > 0)
#pragma unroll
            for (int c = 0; c < VC; ++c) red[wv - 1][c][lane] = acc[0][c];
        __syncthreads();
        if (wv > 0) return;
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
            for (int c = 0; c < VC; ++c) acc[0][c] += red[w][c][lane];
    }
#pragma unroll
    for (int r = 0; r < VRB; ++r) {
        if (rb0 + rw + 4 * r >= nrb) continue;
#pragma unroll
        for (int c = 0; c < VC; ++c) {
            const int j = j0 + c * 16 + lr;
            if (c >= ncb || j >= nc) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = (rb0 + rw + 4 * r) * 16 + 4 * e + lk;
                if (i < np) part[(p0 + i) * nc + j] = acc[r][c][e];
            }
        }
    }
}

// The projection, 16 columns per workgroup: 8 wavefronts, four 16-row blocks of
// products per workgroup (blockIdx.z) in two slices of ab, or one row block in
// eight.  Also for many blocks (us, 2 columns: 758 blocks 17.4 -> 12.4, 2908
// 20.3 -> 18.1, 5476 54.4 -> 41.5).
template <int KU>
__global__ __launch_bounds__(512)
void k_vertex_contract_split(BlockMapDev bm, const double *__restrict__ W, double *__restrict__ part, int nc) {
    __shared__ dbl4 red[4][1][64];
    const int k = blockIdx.x, rb0 = blockIdx.z * 4, j = blockIdx.y * 16 + (threadIdx.x & 15);
    const int np = bm.blk_nprod[k], nrb = (np + 15) / 16;
    if (rb0 >= nrb) return;   // uniform over the workgroup
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nAB = bm.blk_na[k] * bm.blk_nb[k];
    const double *Vk = bm.Vp + bm.blk_vstart[k];
    const int64_t ent = bm.blk_ent[k];
    const int64_t p0 = bm.blk_pstart[k];
    const int lr = lane & 15, lk = lane >> 4;
    const int RG = nrb - rb0 == 1 ? 1 : 4, KS = 8 / RG;
    const int rg = wv % RG, ks = wv / RG;
    const int i = (rb0 + rg) * 16 + lr;   // this lane's product row

    dbl4 acc[1] = {dbl4{0.0, 0.0, 0.0, 0.0}};
    // slice ks takes the k-steps ks, ks + KS, ...
    for (int a0 = ks * 4; a0 < nAB; a0 += KU * KS * 4) {
        double a[KU], b[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int kk = a0 + 4 * KS * u + lk;
            const bool kv = kk < nAB;
            a[u] = (kv && i < np) ? Vk[(int64_t)i * nAB + kk] : 0.0;
            b[u] = (kv && j < nc) ? W[(ent + kk) * nc + j] : 0.0;
        }
        if (rb0 + rg >= nrb) continue;
#pragma unroll
        for (int u = 0; u < KU; ++u)
            if (a0 + 4 * KS * u < nAB) acc[0] = mfma16(a[u], b[u], acc[0]);
    }
    vertex_sum_slices<1>(acc, KS, RG, wv, lane, red);
    if (ks != 0 || rb0 + rg >= nrb || j >= nc) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = (rb0 + rg) * 16 + 4 * e + lk;
        if (row < np) part[(p0 + row) * nc + j] = acc[0][e];
    }
}

// (d), second pass: Y[mu][j] = sum over the (block, slot) entries of mu, in order.
__global__ __launch_bounds__(256)
void k_vertex_reduce(BlockMapDev bm, int P, const double *__restrict__ part,
                     double *__restrict__ Y, int nc) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)P * nc) return;
    const int mu = (int)(idx / nc), j = (int)(idx % nc);
    double acc = 0.0;
    for (int64_t s = bm.prod_pstart[mu]; s < bm.prod_pstart[mu + 1]; ++s)
        acc += part[bm.prod_plist[s] * nc + j];
    Y[idx] = acc;
}

// The same sums written to Y and to the caller's vectors out [nc / 2][P]
// complex: 32 products by 8 vectors per workgroup, turned through LDS so that
// the partial sums and Y move in 128-byte runs and out in 512-byte ones.  One
// launch and one pass over Y less than the sums and a transpose apart.
__global__ __launch_bounds__(256)
void k_vertex_reduce_rows(BlockMapDev bm, int P, const double *__restrict__ part, double *__restrict__ Y, int nc,
                          double *__restrict__ out) {
    __shared__ double2 tile[8][33];
    const int t = threadIdx.x, mu0 = blockIdx.x * 32, r0 = blockIdx.y * 8, nb = nc / 2;
    const int mu = mu0 + t / 8, r = r0 + t % 8;
    if (mu < P && r < nb) {
        double2 acc = make_double2(0.0, 0.0);
        for (int64_t s = bm.prod_pstart[mu]; s < bm.prod_pstart[mu + 1]; ++s) {
            const double2 v = reinterpret_cast<const double2 *>(part)[bm.prod_plist[s] * nb + r];
            acc.x += v.x;
            acc.y += v.y;
        }
        reinterpret_cast<double2 *>(Y)[(int64_t)mu * nb + r] = acc;
        tile[t % 8][t / 8] = acc;
    }
    __syncthreads();
    const int mo = mu0 + t % 32, ro = r0 + t / 32;
    if (mo < P && ro < nb) reinterpret_cast<double2 *>(out)[(int64_t)ro * P + mo] = tile[t / 32][t % 32];
}

// The same sums where a solver step wants them (StepOut), turned through LDS too:
// one launch and one pass over Y less, and all of the chip instead of one
// workgroup per job (60 atoms, 12 jobs: 4.3 + 8.3 us before).
__global__ __launch_bounds__(256)
void k_vertex_reduce_step(BlockMapDev bm, int P, const double *__restrict__ part, double *__restrict__ Y, int nc,
                          StepOut so) {
    __shared__ double2 tile[8][33];
    const int t = threadIdx.x, mu0 = blockIdx.x * 32, q0 = blockIdx.y * 8, nb = nc / 2;
    const int mu = mu0 + t / 8, q = q0 + t % 8;
    if (mu < P && q < nb) {
        double2 acc = make_double2(0.0, 0.0);
        for (int64_t s = bm.prod_pstart[mu]; s < bm.prod_pstart[mu + 1]; ++s) {
            const double2 v = reinterpret_cast<const double2 *>(part)[bm.prod_plist[s] * nb + q];
            acc.x += v.x;
            acc.y += v.y;
        }
        if (so.jobs[q].type != JOB_ARNOLDI) reinterpret_cast<double2 *>(Y)[(int64_t)mu * nb + q] = acc;
        tile[t % 8][t / 8] = acc;
    }
    __syncthreads();
    const int mo = mu0 + t % 32, qo = q0 + t / 32;
    if (mo >= P || qo >= nb) return;
    const Job jb = so.jobs[qo];
    if (jb.type != JOB_ARNOLDI) return;
    const int64_t vlen = (int64_t)so.sl.P_pad * 2;
    double *V = so.sl.V + jb.slot * so.sl.vstride + (int64_t)jb.j * vlen;
    const double2 v = reinterpret_cast<const double2 *>(V)[mo], y = tile[t / 32][t % 32];
    reinterpret_cast<double2 *>(V + vlen)[mo] = make_double2(v.x - y.x, v.y - y.y);
}

void launch_vertex_contract(Tracer *t, hipStream_t s, const BlockMapDev &bm, int n_blk, int P,
                            const double *W, double *part, double *Y, int nc, const WorkSizes &ws,
                            int max_nprod, double *out, const StepOut *step) {
    const int vc = vertex_vc(nc), nrb = (max_nprod + 15) / 16;
    dim3 grid(n_blk, (nc + 16 * vc - 1) / (16 * vc), (nrb + 4 * VRB - 1) / (4 * VRB));
    trace_begin(t, "vertex_contract", s);
    const int c16 = (nc + 15) / 16;
    if (vc == 1 || n_blk * c16 <= VSPLIT_BLK)
        hipLaunchKernelGGL((k_vertex_contract_split<12>), dim3(n_blk, c16, (nrb + 3) / 4), dim3(512), 0, s, bm, W,
                           part, nc);
    else if (vc == 2)
        hipLaunchKernelGGL((k_vertex_contract<2, 8>), grid, dim3(256), 0, s, bm, W, part, nc);
    else
        hipLaunchKernelGGL((k_vertex_contract<4, 4>), grid, dim3(256), 0, s, bm, W, part, nc);
    trace_end(t, s, 2.0 * ws.sum_s2 * nc, 8.0 * (ws.sum_s2 + ws.nnzB * nc + ws.npart * nc));
    const int64_t n = (int64_t)P * nc;
    trace_begin(t, "vertex_reduce", s);
    const dim3 turned((P + 31) / 32, (nc / 2 + 7) / 8);
    if (out)
        hipLaunchKernelGGL(k_vertex_reduce_rows, turned, dim3(256), 0, s, bm, P, part, Y, nc, out);
    else if (step)
        hipLaunchKernelGGL(k_vertex_reduce_step, turned, dim3(256), 0, s, bm, P, part, Y, nc, *step);
    else
        hipLaunchKernelGGL(k_vertex_reduce, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, bm, P, part, Y,
                           nc);
    trace_end(t, s, ws.npart * nc, 8.0 * (ws.npart * nc + ws.P * nc));
}

}  // namespace chi0
