// Small dense linear algebra of the projector refresh (paper Sec. 1: P = leading
// left singular vectors of the gradient, recomputed every ~200 steps).  The
// large products run on the grouped fp32 GEMM (those with a bf16 gradient on
// k_sketch_product); this file holds what sits between them, one launch for all matrices of the layer set:
//
//   k_fill_gaussian     random sketch Omega (counter-based generator, Box-Muller)
//   k_inverse_factor    Linv = L^{-1} as float, where S = L L^T is a symmetric product (the GEMM then
//                       applies X <- X Linv^T): one workgroup per matrix, fp64 in registers, orders
//                       up to kFactorMax
//   k_sum_planes, k_chol_*, k_tri_*   the same for larger orders: T = S, T = L L^T in place (fp64,
//                       right-looking, panels of 32 columns), Linv by 32 x 32 blocks
//   k_jacobi_*          blocked one-sided Jacobi on the rows of L^T (floats, in the Linv buffer), where
//                       L L^T is the l x l Rayleigh-Ritz matrix T = (Q^T G)(Q^T G)^T: at convergence
//                       row i = ritz_i * u_i^T
//   k_ritz_sort / k_build_rotation   order by descending Ritz value, stage U[:, top r]
//   k_sign_fix          copy the orthonormalised basis into P, largest-magnitude entry of each
//                       column made positive
#include "eliminate16.h"
#include "ng_internal.h"
#include "split_bf16.h"
#include "state_math.h"

namespace ng {

// ------------------------------------------------------------------ random sketch
__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

__device__ __forceinline__ float gaussian(unsigned long long key, long long i) {
    const unsigned long long z = mix64(key + (unsigned long long)(i + 1) * 0x9E3779B97F4A7C15ULL);
    const float u1 = ((float)(unsigned int)(z >> 40) + 1.0f) * (1.0f / 16777216.0f);      // (0, 1]
    const float u2 = (float)(unsigned int)((z >> 8) & 0xFFFFFFu) * (1.0f / 16777216.0f);   // [0, 1)
    return sqrtf(-2.0f * logf(u1)) * cosf(6.28318530717958647692f * u2);
}

// Matrices with sketch planes: eight rows of one column per thread, rounded to bf16, as the octets that a gradient
// product reads.  PLANES: the set has such matrices.
template <bool PLANES>
__global__ __launch_bounds__(256) void k_fill_gaussian(const MatDev* __restrict__ mats, unsigned long long seed,
                                                       unsigned long long call_id) {
    const MatDev& md = mats[blockIdx.y];
    const unsigned long long key =
        mix64(seed ^ (call_id * 0x9E3779B97F4A7C15ULL) ^ ((unsigned long long)(blockIdx.y + 1) * 0xD1B54A32D192ED03ULL));
    const int n = md.n, l = md.l;
    const bool plane = PLANES && md.Yp != nullptr;
    const long long total = plane ? (long long)((n + 7) / 8) * l : (long long)n * l;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
        if (!plane) {
            md.Yb[i] = gaussian(key, i);
            continue;
        }
        const int oct = (int)(i / l), col = (int)(i - (long long)oct * l);
        typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
        bf16x8_t v;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = (__bf16)(8 * oct + e < n ? gaussian(key, (long long)(8 * oct + e) * l + col) : 0.f);
        *reinterpret_cast<bf16x8_t*>(sketch_plane(md, false, 0) + 8 * i) = v;
    }
}

hipError_t launch_fill_gaussian(const MatDev* mats, int n_mats, int max_rows, bool planes, unsigned long long seed,
                                unsigned long long call_id, hipStream_t stream) {
    int gx = (max_rows + 3) / 4;   // grid-stride loop covers the rest
    if (gx < 1) gx = 1;
    if (gx > 4096) gx = 4096;
    if (planes) hipLaunchKernelGGL(k_fill_gaussian<true>, dim3((gx + 7) / 8, n_mats), dim3(256), 0, stream, mats, seed, call_id);
    else hipLaunchKernelGGL(k_fill_gaussian<false>, dim3(gx, n_mats), dim3(256), 0, stream, mats, seed, call_id);
    return hipGetLastError();
}

// ------------------------------------------------------------------ Cholesky (fp64, in place, lower)
__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Right-looking blocked factorisation, panels of kCholNB columns, three launches per panel:
//   k_chol_diag    factor the kCholNB x kCholNB diagonal block in LDS (one workgroup per matrix)
//   k_chol_panel   rows below it: X L11^T = A21, one thread per row
//   k_chol_update  trailing lower triangle -= L21 L21^T, 64 x 64 tiles
// which: 0 -> order l, 1 -> order r.  T has leading dimension lp.  k_chol_shift first adds
// shift_rel * trace(T) to the diagonal.  A non-positive pivot sets bit 2 of *status (the pivot is
// replaced by 1).  Only the lower triangle is read and written.
constexpr int kCholNB = 32;
constexpr int kJacobiFlags = 64;     // entries of MatDev::jflag: the largest refresh_sweeps

// (the shift itself is left in md.ritz[0], free while a factor is computed: the pivots' lower bound where one is asked for)
__global__ __launch_bounds__(256) void k_chol_shift(const MatDev* __restrict__ mats, int which, double shift_rel) {
    __shared__ double red[4];
    const MatDev& md = mats[blockIdx.x];
    const int nn = which == 0 ? md.l : md.r;
    const long long ld = md.lp;
    double* __restrict__ A = md.T;
    const int tid = threadIdx.x;
    double tr = 0.0;
    for (int i = tid; i < nn; i += 256) tr += A[i * ld + i];
    tr = wave_sum_d(tr);
    if ((tid & 63) == 0) red[tid >> 6] = tr;
    __syncthreads();
    const double shift = shift_rel * (((red[0] + red[1]) + red[2]) + red[3]);
    for (int i = tid; i < nn; i += 256) A[i * ld + i] += shift;
    if (tid == 0) md.ritz[0] = shift;
}

__global__ __launch_bounds__(256) void k_chol_diag(const MatDev* __restrict__ mats, int which, int k0, int bounded, int* status) {
    __shared__ double D[kCholNB][kCholNB + 1];
    const MatDev& md = mats[blockIdx.x];
    const int nn = which == 0 ? md.l : md.r;
    if (k0 >= nn) return;
    const long long ld = md.lp;
    double* __restrict__ A = md.T;
    const int tid = threadIdx.x;
    for (int q = tid; q < kCholNB * kCholNB; q += 256) {
        const int i = q / kCholNB, j = q % kCholNB;
        double v = i == j ? 1.0 : 0.0;            // identity padding past the matrix order
        if (k0 + i < nn && j <= i) v = A[(long long)(k0 + i) * ld + k0 + j];
        D[i][j] = v;
    }
    __syncthreads();
    bool bad = false;
    const double least = bounded ? 0.25 * md.ritz[0] : 0.0;
    for (int k = 0; k < kCholNB; ++k) {
        double d = D[k][k];
        d = d < least ? least : d;
        if (!(d > 0.0) || !(d < 1.0e300)) {
            bad = true;
            d = 1.0;
        }
        const double rd = 1.0 / d;
        // rank-one update of the columns right of k with the still unscaled column k
        for (int q = tid; q < kCholNB * kCholNB; q += 256) {
            const int i = q / kCholNB, j = q % kCholNB;
            if (j > k && i >= j) D[i][j] -= D[i][k] * D[j][k] * rd;
        }
        __syncthreads();
        // column k is final now and not read again: scale it
        if (tid < kCholNB) {
            const double sd = sqrt(d);
            if (tid == k) D[k][k] = sd;
            else if (tid > k) D[tid][k] *= 1.0 / sd;
        }
    }
    __syncthreads();
    for (int q = tid; q < kCholNB * kCholNB; q += 256) {
        const int i = q / kCholNB, j = q % kCholNB;
        if (k0 + i < nn && j <= i) A[(long long)(k0 + i) * ld + k0 + j] = D[i][j];
    }
    if (bad && tid == 0) atomicOr(status, 4);
}

__global__ __launch_bounds__(256) void k_chol_panel(const MatDev* __restrict__ mats, int which, int k0) {
    __shared__ double Ls[kCholNB][kCholNB + 1];
    __shared__ double invd[kCholNB];
    const MatDev& md = mats[blockIdx.y];
    const int nn = which == 0 ? md.l : md.r;
    const int row0 = k0 + kCholNB + blockIdx.x * 256;
    if (row0 >= nn) return;               // (then k0 + kCholNB < nn: all panel columns exist)
    const long long ld = md.lp;
    double* __restrict__ A = md.T;
    const int tid = threadIdx.x;
    for (int q = tid; q < kCholNB * kCholNB; q += 256) {
        const int i = q / kCholNB, j = q % kCholNB;
        Ls[i][j] = j <= i ? A[(long long)(k0 + i) * ld + k0 + j] : 0.0;
    }
    __syncthreads();
    if (tid < kCholNB) invd[tid] = 1.0 / Ls[tid][tid];
    __syncthreads();
    const int i = row0 + tid;
    if (i >= nn) return;
    double* __restrict__ row = A + (long long)i * ld + k0;
    double x[kCholNB];
#pragma unroll
    for (int j = 0; j < kCholNB; ++j) x[j] = row[j];
#pragma unroll
    for (int j = 0; j < kCholNB; ++j) {
        double acc = x[j];
#pragma unroll
        for (int t = 0; t < j; ++t) acc -= x[t] * Ls[j][t];
        x[j] = acc * invd[j];
    }
#pragma unroll
    for (int j = 0; j < kCholNB; ++j) row[j] = x[j];
}

__global__ __launch_bounds__(256) void k_chol_update(const MatDev* __restrict__ mats, int which, int k0) {
    __shared__ double As[64][kCholNB + 1];
    __shared__ double Bs[64][kCholNB + 1];
    if (blockIdx.y > blockIdx.x) return;  // lower triangle of tiles only
    const MatDev& md = mats[blockIdx.z];
    const int nn = which == 0 ? md.l : md.r;
    const int base = k0 + kCholNB;
    const int r0 = base + 64 * blockIdx.x, c0 = base + 64 * blockIdx.y;
    if (r0 >= nn) return;
    const long long ld = md.lp;
    double* __restrict__ A = md.T;
    const int tid = threadIdx.x;
    for (int q = tid; q < 64 * kCholNB; q += 256) {
        const int rr = q / kCholNB, t = q % kCholNB;
        As[rr][t] = r0 + rr < nn ? A[(long long)(r0 + rr) * ld + k0 + t] : 0.0;
        Bs[rr][t] = c0 + rr < nn ? A[(long long)(c0 + rr) * ld + k0 + t] : 0.0;
    }
    __syncthreads();
    const int tx = tid & 15, ty = tid >> 4;   // outputs (ty + 16 e, tx + 16 f)
    double acc[4][4] = {};
#pragma unroll 4
    for (int t = 0; t < kCholNB; ++t) {
        double av[4], bv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            av[e] = As[ty + 16 * e][t];
            bv[e] = Bs[tx + 16 * e][t];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int f = 0; f < 4; ++f) acc[e][f] += av[e] * bv[f];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int i = r0 + ty + 16 * e, j = c0 + tx + 16 * f;
            if (i < nn && j <= i) A[(long long)i * ld + j] -= acc[e][f];
        }
}

// T (lower triangle) = the sum of a symmetric product's planes
__global__ __launch_bounds__(256) void k_sum_planes(const MatDev* __restrict__ mats, const SymPlanes* __restrict__ sym) {
    const MatDev& md = mats[blockIdx.y];
    const SymPlanes sp = sym[blockIdx.y];
    const long long nn = sp.order, pitch = sp.pitch;
    double* __restrict__ T = md.T;
    for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < nn * nn; q += (long long)gridDim.x * 256) {
        const long long i = q / nn, j = q - i * nn;
        if (j > i) continue;
        double v = 0.0;
        for (int c = 0; c < sp.count; ++c) v += (double)sp.p[c * pitch + q];
        T[i * md.lp + j] = v;
    }
}

// bounded: pivots below a quarter of the shift count as that
static hipError_t launch_cholesky(const MatDev* mats, int n_mats, int which, int max_order, double shift_rel,
                                  bool bounded, int* status, hipStream_t stream) {
    if (shift_rel > 0.0)
        hipLaunchKernelGGL(k_chol_shift, dim3(n_mats), dim3(256), 0, stream, mats, which, shift_rel);
    for (int k0 = 0; k0 < max_order; k0 += kCholNB) {
        hipLaunchKernelGGL(k_chol_diag, dim3(n_mats), dim3(256), 0, stream, mats, which, k0, (int)bounded, status);
        const int below = max_order - k0 - kCholNB;
        if (below <= 0) break;
        hipLaunchKernelGGL(k_chol_panel, dim3((below + 255) / 256, n_mats), dim3(256), 0, stream, mats, which, k0);
        const int nt = (below + 63) / 64;
        hipLaunchKernelGGL(k_chol_update, dim3(nt, nt, n_mats), dim3(256), 0, stream, mats, which, k0);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ inverse of the Cholesky factor
// Linv = L^{-1} (lower triangular, float), by 32 x 32 blocks: X_ii = L_ii^{-1}, and below the diagonal
//   X_ij = -L_ii^{-1} (sum_{k=j..i-1} L_ik X_kj),
// so a block column of the inverse depends only on itself.  k_tri_diag_inverse inverts the diagonal
// blocks by forward substitution (one lane per column); k_tri_inverse_blocks gives a workgroup one block
// column and walks down its block rows: both products of a block run on fp64 MFMA (16x16x4; lane L
// supplies A[L%16][L/16] and B[L/16][L%16], element e of its result is D[4e + L/16][L%16]), the sum
// over k from L in global memory and the solved blocks above (LDS, floats), the multiplication by
// the inverted diagonal block from that block (global, floats) and the sum (LDS, doubles).  16
// dependent block steps at order 512 instead of the 128 four-row steps of a substitution over the
// whole column.  A solved entry is rounded to float before anything reads it back, so the stored
// inverse is what the rows below were computed from.  Rows and columns >= the order read as
// those of an identity and are not written.
typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
constexpr int kTriNB = 32;

__global__ __launch_bounds__(64) void k_tri_diag_inverse(const MatDev* __restrict__ mats, int which) {
    __shared__ double Ls[2][kTriNB][kTriNB + 1], Xl[2][kTriNB][kTriNB + 1];
    const MatDev& md = mats[blockIdx.y];
    const int nn = which == 0 ? md.l : md.r;
    const long long ld = md.lp;
    const int half = threadIdx.x >> 5, c = threadIdx.x & 31;
    const int r0 = (2 * (int)blockIdx.x + half) * kTriNB;
    const double* __restrict__ L = md.T;
    // (no early return: both halves meet at the barrier; a half past the order works on an identity)
    for (int i = 0; i < kTriNB; ++i) {
        const int gi = r0 + i, gc = r0 + c;
        double v = (i == c) ? 1.0 : 0.0;
        if (gi < nn && gc < nn && c <= i) v = L[(long long)gi * ld + gc];
        Ls[half][i][c] = v;
    }
    __syncthreads();
    // column c of the inverse: x_i = (e_i - sum_{k=c..i-1} L_ik x_k) / L_ii, x_i = 0 above the diagonal
    float* __restrict__ Xg = md.Linv;
    for (int i = 0; i < kTriNB; ++i) {
        double xi = 0.0;
        if (i >= c) {
            double tot = 0.0;
            for (int k = c; k < i; ++k) tot += Ls[half][i][k] * Xl[half][k][c];
            xi = (double)(float)(((i == c ? 1.0 : 0.0) - tot) / Ls[half][i][i]);
        }
        Xl[half][i][c] = xi;       // read back by this lane only
        if (r0 + i < nn && r0 + c < nn) Xg[(long long)(r0 + i) * ld + r0 + c] = (float)xi;
    }
}

// XLDS: the solved blocks of the column are kept in LDS (as two 16-column halves, [half][row][16]:
// the four rows of an MFMA operand are 64 consecutive floats); otherwise they are read back from Linv
// in global memory, which the barrier of each block step makes visible inside the workgroup.
template <bool XLDS>
__global__ __launch_bounds__(256) void k_tri_inverse_blocks(const MatDev* __restrict__ mats, int which) {
    extern __shared__ __attribute__((aligned(16))) unsigned char tri_smem[];
    const MatDev& md = mats[blockIdx.y];
    const int nn = which == 0 ? md.l : md.r;
    const int nb = (nn + kTriNB - 1) / kTriNB;
    // Block column b costs (nb - b)^2.  Workgroup ids go round-robin over the 8 XCDs, so with a block
    // count that is a multiple of 8 a plain b = blockIdx.x would give one XCD the two most expensive
    // columns of every matrix; rotating by the matrix index spreads them.
    const int jb = (int)((blockIdx.x + blockIdx.y) % gridDim.x);
    if (jb >= nb) return;
    const long long ld = md.lp;
    const double* __restrict__ L = md.T;
    float* __restrict__ Xg = md.Linv;
    const int c0 = jb * kTriNB;
    const int rows = (nb - jb) * kTriNB;                     // rows c0 .. of the block column, padded
    double* Ssm = reinterpret_cast<double*>(tri_smem);       // [2][32][16]
    float* Xs = reinterpret_cast<float*>(Ssm + 2 * kTriNB * 16);   // [2][rows][16] (XLDS)
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int l16 = lane & 15, lq = lane >> 4, tr = wv >> 1, tc = wv & 1;
    const int col = c0 + 16 * tc + l16;                      // this lane's column of the result tiles
    const bool col_ok = col < nn;

    // rows above the block column: exact zeros
    for (int q = tid; q < c0 * kTriNB; q += 256) {
        const int i = q / kTriNB, cc = q % kTriNB;
        if (c0 + cc < nn) Xg[(long long)i * ld + c0 + cc] = 0.f;
    }
    if (XLDS) {
        // the diagonal block, as the first kernel left it
        for (int q = tid; q < kTriNB * kTriNB; q += 256) {
            const int i = q / kTriNB, cc = q % kTriNB;
            const bool in = c0 + i < nn && c0 + cc < nn;
            Xs[((cc >> 4) * rows + i) * 16 + (cc & 15)] = in ? Xg[(long long)(c0 + i) * ld + c0 + cc] : 0.f;
        }
    }
    __syncthreads();

    for (int ib = jb + 1; ib < nb; ++ib) {
        const int r0 = ib * kTriNB;
        // the inverted diagonal block of this block row (does not depend on the sum: fetched first)
        float dinv[8];
        {
            const int gi = r0 + 16 * tr + l16;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int gk = r0 + 4 * u + lq;
                dinv[u] = (gi < nn && gk < nn) ? Xg[(long long)gi * ld + gk] : 0.f;
            }
        }
        // S = sum_k L[ib][k] X[k][jb] over the columns c0 .. r0-1 (all below the order): tile (tr, tc)
        double4_t acc = {0.0, 0.0, 0.0, 0.0};
        {
            const int gi = r0 + 16 * tr + l16;
            const bool rok = gi < nn;
            const double* __restrict__ lrow = L + (long long)(rok ? gi : 0) * ld + c0 + lq;
            const int nk = r0 - c0;
            for (int k = 0; k < nk; k += 16) {              // nk % 32 == 0: four k-steps per pass
                double a[4];
                float b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = rok ? lrow[k + 4 * u] : 0.0;
                    const int kr = k + 4 * u + lq;           // row of the block column, from c0
                    b[u] = XLDS ? Xs[(tc * rows + kr) * 16 + l16]
                                : (col_ok ? Xg[(long long)(c0 + kr) * ld + col] : 0.f);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], (double)b[u], acc, 0, 0, 0);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) Ssm[(tc * kTriNB + 16 * tr + 4 * e + lq) * 16 + l16] = acc[e];
        __syncthreads();
        // X[ib][jb] = -Dinv S
        double4_t o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 8; ++u)
            o = __builtin_amdgcn_mfma_f64_16x16x4f64((double)dinv[u], Ssm[(tc * kTriNB + 4 * u + lq) * 16 + l16], o, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * tr + 4 * e + lq;              // row inside the block
            const float xf = (float)(-o[e]);
            if (XLDS) Xs[(tc * rows + (r0 - c0) + i) * 16 + l16] = xf;
            if (r0 + i < nn && col_ok) Xg[(long long)(r0 + i) * ld + col] = xf;
        }
        __syncthreads();
    }
}

static hipError_t launch_tri_inverse(const MatDev* mats, int n_mats, int which, int max_order, hipStream_t stream) {
    const int nb = (max_order + kTriNB - 1) / kTriNB;
    if (nb <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tri_diag_inverse, dim3((nb + 1) / 2, n_mats), dim3(64), 0, stream, mats, which);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    static bool attr_done = false;
    constexpr size_t kBudget = 150 * 1024;
    if (!attr_done) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_tri_inverse_blocks<true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBudget);
        attr_done = true;
    }
    const size_t s_bytes = (size_t)2 * kTriNB * 16 * sizeof(double);
    const size_t x_bytes = (size_t)2 * nb * kTriNB * 16 * sizeof(float);
    if (s_bytes + x_bytes <= kBudget)
        hipLaunchKernelGGL(k_tri_inverse_blocks<true>, dim3(nb, n_mats), dim3(256), s_bytes + x_bytes, stream, mats, which);
    else
        hipLaunchKernelGGL(k_tri_inverse_blocks<false>, dim3(nb, n_mats), dim3(256), s_bytes, stream, mats, which);
    return hipGetLastError();
}

// ------------------------------------------------------------------ inverse factor in one workgroup
// Linv = L^{-1} for S = L L^T (+ shift_rel * trace(S) on the diagonal), order nn <= kFactorMax, S the sum
// of float planes.  The lower triangle lives in the registers of eight wavefronts as 32 x 32 blocks in
// the layout of fp64 MFMA results (block t = i (i+1)/2 + j belongs to wavefront t % 8), and it is
// inverted in place, right-looking, one panel k of 32 columns at a time:
//   D    = L_kk^{-1}, by one wavefront (factor_diag)
//   L_ik = A_ik D^T  (i > k)          from then on slot (i, k) holds the running sum of X_ik instead
//   X_kj = D R_kj    (j < k), X_kk = D     a finished block row of the inverse
//   A_ij -= L_ik L_jk^T (j > k),  R_ij -= L_ik X_kj (j <= k)     every slot with i > k
// Every slot below the panel takes one product per panel, so the wavefronts stay evenly loaded, and
// nothing but the planes and the result touches memory: the three launches per panel of the path for
// larger orders cost 410 us at order 256 (168 matrices), most of it launches and the diagonal blocks.
constexpr int kFacPitch = 34;                      // doubles per LDS row: the 16 rows of an operand on distinct banks
constexpr int kFacBlock = 32 * kFacPitch;          // doubles per 32 x 32 block
constexpr int kFacNB = kFactorMax / 32;            // block rows

// A wavefront's LDS operations complete in order; this keeps the compiler to the order as well where its
// lanes hand each other values.
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// X = L^{-1} of a 32 x 32 block A = L L^T (lower triangle in LDS; overwritten) by one wavefront, as two 16 x 16
// eliminations: the first carries the identity (lanes 0..15: X11) and A21^T (lanes 16..31: L21), the
// second the identity.  The multipliers of a step reach the lanes by a broadcast inside each row of
// 16, so a step is a pivot's reciprocal root and at most 15 x 2 multiply-adds, and the code is one small
// loop body (unrolled over 32 x 32 with lane reads through scalar registers it was 13 us, mostly
// instruction fetch).  Lt (LT): L^T as well.  Returns true if a pivot was not positive and finite (it is
// replaced by 1).
template <bool LT>
__device__ __forceinline__ bool factor_diag(double* __restrict__ A, double* __restrict__ X, double* __restrict__ Lt,
                                            double least, int lane) {
    const int c = lane & 15, g = lane >> 4;
    bool bad = false;
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        const int o = 16 * half;
        double* blk = A + o * kFacPitch + o;
        double a[16], v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            a[i] = blk[(i > c ? i : c) * kFacPitch + (i > c ? c : i)];
            v[i] = g == 1 ? A[(16 + c) * kFacPitch + i] : (i == c ? 1.0 : 0.0);
        }
        eliminate16<0>(a, v, least, bad);
        if (g == 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) X[(o + i) * kFacPitch + o + c] = v[i];
            if (LT) {
#pragma unroll
                for (int i = 0; i < 16; ++i) Lt[(o + i) * kFacPitch + o + c] = c >= i ? a[i] : 0.0;
            }
        }
        if (LT && half == 0 && g == 1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                Lt[i * kFacPitch + 16 + c] = v[i];
                Lt[(16 + i) * kFacPitch + c] = 0.0;
            }
        }
        if (half == 0) {
            if (g == 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i) A[(16 + c) * kFacPitch + i] = v[i];      // L21
            }
            lds_order();
            // A22 -= L21 L21^T
            double4_t t;
            double* a22 = A + 16 * kFacPitch + 16;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = a22[(4 * e + g) * kFacPitch + c];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double x = A[(16 + c) * kFacPitch + 4 * u + g];
                t = __builtin_amdgcn_mfma_f64_16x16x4f64(-x, x, t, 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) a22[(4 * e + g) * kFacPitch + c] = t[e];
        }
        lds_order();
    }
    // X21 = -X22 (L21 X11), X12 = 0; the product in the middle takes the place of A11
    double4_t t = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u)
        t = __builtin_amdgcn_mfma_f64_16x16x4f64(A[(16 + c) * kFacPitch + 4 * u + g], X[(4 * u + g) * kFacPitch + c], t, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) A[(4 * e + g) * kFacPitch + c] = t[e];
    lds_order();
    t = (double4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u)
        t = __builtin_amdgcn_mfma_f64_16x16x4f64(-X[(16 + c) * kFacPitch + 16 + 4 * u + g], A[(4 * u + g) * kFacPitch + c], t, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        X[(16 + 4 * e + g) * kFacPitch + c] = t[e];
        X[(4 * e + g) * kFacPitch + 16 + c] = 0.0;
    }
    return bad;
}

// A workgroup's part of a ClearShare.  A CU stores 18 to 28 GB/s of zeros however many wavefronts it has at it, so a launch of
// its own takes the whole chip to clear at 4.7 to 5.9 TB/s (350M set, 5.2 GB with the padding of its panels: 0.89 ms).  The
// Jacobi's rounds use next to no memory bandwidth: beside 60 of them the refresh of that set takes 12.83 -> 11.95 ms.  Where the
// visits leave CUs to spare, a round is the latency of one visit and the clearing is better beside the factors, which have one
// workgroup per matrix (60M set 1663 -> 1658 us beside the rounds, 1672 -> 1642 beside seven factors; the
// 350M set 12.55 ms beside the factors, whose 88 idle CUs and 195 us are not enough for it).
// Every workgroup has as many bytes as any other, a run of them across the matrices.  (With eight pieces per matrix one matrix had
// eight workgroups: refresh of a 1024 x 128256 at rank 128, 1.06 GB of history, 10.90 ms, against 9.60 with a launch of its own and
// 9.48 now; 40 of 1024 x 16384 at rank 64 4.27, 4.21, 4.00.)
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void clear_share(const MatDev* __restrict__ mats, int n_mats, const ClearShare& cs, int block) {
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    unsigned long long at, end;
    clear_range(cs, block, &at, &end);
    if (at < end) {
        // the last matrix that starts at or before the first unit
        const int lane = threadIdx.x & 63;
        int i = -1;
        for (int b = 0; b < n_mats; b += 64) i += __popcll(__ballot(b + lane < n_mats && mats[b + lane < n_mats ? b + lane : 0].clear_off <= at));
        for (; at < end; ++i) {
            const MatDev& md = mats[i];
            const unsigned long long behind = i + 1 < n_mats ? mats[i + 1].clear_off : cs.units, last = behind < end ? behind : end;
            u32x4_t* __restrict__ h = reinterpret_cast<u32x4_t*>(md.H);
            for (unsigned long long q = at - md.clear_off + threadIdx.x; q < last - md.clear_off; q += blockDim.x)
                __builtin_nontemporal_store(zero, h + q);
            at = last;
        }
    }
    if (cs.part == 0)
        for (int i = block; i < n_mats; i += cs.blocks) {
            u32x4_t* __restrict__ k = reinterpret_cast<u32x4_t*>(mats[i].K);
            for (unsigned long long q = threadIdx.x; q < cs.k_bytes / 16; q += blockDim.x) k[q] = zero;
        }
}

//
// FACTOR: the rows of L^T instead (zero below the diagonal and in the padding), where the Jacobi works on
// them: the same elimination without its right-hand side.  Pivots are kept above a quarter of the shift.
//
// WAVES wavefronts hold up to SLOTS blocks each (one more takes the diagonal blocks): 7 x 6 covers order 256 within
// 256 registers; orders up to 128 take 10 x 1, every block of a panel at work at once and a fraction of the code.
template <bool FACTOR, int WAVES, int SLOTS>
__global__ __launch_bounds__(64 * (WAVES + 1)) void k_inverse_factor(const MatDev* __restrict__ mats,
                                                           const SymPlanes* __restrict__ sym, double shift_rel, int max_nb,
                                                           int n_mats, ClearShare share, int* status) {
    if (!FACTOR && (int)blockIdx.x >= n_mats) {      // (nothing is cleared beside FACTOR: its launches come after the last share)
        clear_share(mats, n_mats, share, (int)blockIdx.x - n_mats);
        return;
    }
    extern __shared__ __attribute__((aligned(16))) double fac_smem[];
    __shared__ double red[WAVES];
    const MatDev& md = mats[blockIdx.x];
    const SymPlanes sp = sym[blockIdx.x];
    const int nn = sp.order, nb = (nn + 31) / 32;
    const long long pitch = sp.pitch;
    double* Am = fac_smem;                              // the diagonal block
    double* Dm = Am + kFacBlock;                        // its inverse factor
    double* Lp = Dm + kFacBlock;                        // block rows 1 .. of the panel (block i at i - 1)
    double* Xp = Lp + (max_nb - 1) * kFacBlock;         // block columns 0 .. of the inverse's row (block j at j)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int l16 = lane & 15, lq = lane >> 4;
    const float* __restrict__ S = sp.p;

    if (FACTOR && tid < kJacobiFlags) md.jflag[tid] = 0;
    if (wv == WAVES) {            // the wavefront of the diagonal blocks
        double least = 0.0;
        if (shift_rel > 0.0) {
            __syncthreads();
            if (FACTOR) {
#pragma unroll
                for (int w = 0; w < WAVES; ++w) least += red[w];
                least *= 0.25 * shift_rel;
            }
        }
        for (int k = 0; k < nb; ++k) {
            __syncthreads();
            if (factor_diag<FACTOR>(Am, Dm, Xp, least, lane) && lane == 0) atomicOr(status, 4);
            __syncthreads();
            __syncthreads();
            if (k + 1 < nb) __syncthreads();
        }
        return;
    }

    // this wavefront's blocks
    int bi[SLOTS], bj[SLOTS];
    double4_t acc[SLOTS][2][2];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int t = wv + WAVES * s;
        int i = 0;
        while ((i + 1) * (i + 2) / 2 <= t) ++i;
        bi[s] = i < nb ? i : -1;
        bj[s] = t - i * (i + 1) / 2;
        const int row0 = 32 * i + lq, col0 = 32 * bj[s] + l16;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            const int row = row0 + 16 * (x >> 3) + 4 * (x & 3), col = col0 + 16 * ((x >> 2) & 1);
            acc[s][x >> 3][(x >> 2) & 1][x & 3] = row == col && row >= nn ? 1.0 : 0.0;   // identity past the order
        }
        if (bi[s] < 0) continue;
        __builtin_amdgcn_sched_barrier(0);
        for (int c = 0; c < sp.count; c += 2) {        // two planes' loads in flight
            float f[2][16];
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const float* __restrict__ p = S + (c + y < sp.count ? c + y : c) * pitch;
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int row = row0 + 16 * (x >> 3) + 4 * (x & 3), col = col0 + 16 * ((x >> 2) & 1);
                    f[y][x] = p[row < nn && col <= row ? (unsigned)(row * nn + col) : 0u];
                }
            }
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int row = row0 + 16 * (x >> 3) + 4 * (x & 3), col = col0 + 16 * ((x >> 2) & 1);
                    const bool in = row < nn && col <= row && c + y < sp.count;
                    acc[s][x >> 3][(x >> 2) & 1][x & 3] += in ? (double)f[y][x] : 0.0;
                }
        }
    }
    if (shift_rel > 0.0) {
        double tr = 0.0;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const int row = 32 * bi[s] + lq + 16 * (x >> 3) + 4 * (x & 3), col = 32 * bj[s] + l16 + 16 * ((x >> 2) & 1);
                if (bi[s] >= 0 && row == col && row < nn) tr += acc[s][x >> 3][(x >> 2) & 1][x & 3];
            }
        tr = wave_sum_d(tr);
        if (lane == 0) red[wv] = tr;
        __syncthreads();
        double shift = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) shift += red[w];
        shift *= shift_rel;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const int row = 32 * bi[s] + lq + 16 * (x >> 3) + 4 * (x & 3), col = 32 * bj[s] + l16 + 16 * ((x >> 2) & 1);
                if (bi[s] >= 0 && row == col && row < nn) acc[s][x >> 3][(x >> 2) & 1][x & 3] += shift;
            }
    }
    float* __restrict__ Xg = md.Linv;
    const int ld = md.lp;
    // blocks above the diagonal (FACTOR: below it): zeros
    for (int q = tid; q < nb * nb * 1024; q += 64 * WAVES) {
        const int i = (q >> 10) / nb, j = (q >> 10) % nb;
        const int row = 32 * i + ((q >> 5) & 31), col = 32 * j + (q & 31);
        if (FACTOR ? j < i : (j > i && row < nn && col < nn)) Xg[row * ld + col] = 0.f;
    }
    // FACTOR: a block of L^T, from LDS (B(r, c) = src[r * sr + c * scol]) to rows 32 i .., columns 32 j ..
    auto store_rows = [&](const double* src, int sr, int scol, int i, int j) {
        const int c = lane & 31;
#pragma unroll 4
        for (int r = lane >> 5; r < 32; r += 2) {
            const int row = 32 * i + r, col = 32 * j + c;
            Xg[row * ld + col] = row < nn && col < nn ? (float)src[r * sr + c * scol] : 0.f;
        }
    };

    auto put = [&](double* dst, const double4_t (&t)[2][2]) {      // a result block -> LDS
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[(16 * a + 4 * e + lq) * kFacPitch + 16 * b + l16] = t[a][b][e];
    };
    // t += sign * A B, B(k, c) = B[k * bk + c * bc]
    auto mul = [&](double4_t (&t)[2][2], const double* A, const double* B, int bk, int bc, double sign) {
        const double* pa = A + l16 * kFacPitch + lq;
        const double* pb = B + lq * bk + l16 * bc;
        const int b16 = 16 * bc, bk4 = 4 * bk;
#pragma unroll 2
        for (int u = 0; u < 8; ++u) {
            const double a0 = sign * pa[4 * u], a1 = sign * pa[16 * kFacPitch + 4 * u];
            const double b0 = pb[0], b1 = pb[b16];
            pb += bk4;
            t[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, t[0][0], 0, 0, 0);
            t[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, t[0][1], 0, 0, 0);
            t[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, t[1][0], 0, 0, 0);
            t[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, t[1][1], 0, 0, 0);
        }
    };
    auto clear = [&](double4_t (&t)[2][2]) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) t[a][b] = (double4_t){0.0, 0.0, 0.0, 0.0};
    };

    for (int k = 0; k < nb; ++k) {
        // opaque to the compiler, so that it forms addresses where they are used: hoisted out of the loop
        // they take more registers than the blocks leave
        asm volatile("" : "+v"(l16), "+v"(lq));
        // the panel's blocks and the inverse's unfinished row go to LDS
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (bi[s] < k) continue;
            if (bi[s] == k && bj[s] == k) put(Am, acc[s]);
            else if (bj[s] == k) put(Lp + (bi[s] - 1) * kFacBlock, acc[s]);
            else if (!FACTOR && bi[s] == k) put(Xp + bj[s] * kFacBlock, acc[s]);
        }
        __syncthreads();
        __syncthreads();     // (D is ready)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (bi[s] < k) continue;
            if (bi[s] > k) {
                if (bj[s] != k) continue;
                double* blk = Lp + (bi[s] - 1) * kFacBlock;     // L_ik = A_ik D^T
                clear(acc[s]);
                mul(acc[s], blk, Dm, 1, kFacPitch, 1.0);
                put(blk, acc[s]);                               // (this wavefront has read the block to its end)
                if (FACTOR) {
                    lds_order();
                    store_rows(blk, 1, kFacPitch, k, bi[s]);
                }
                clear(acc[s]);                                  // X_ik starts from zero
            } else if (FACTOR) {
                if (bj[s] == k) store_rows(Xp, kFacPitch, 1, k, k);
            } else {
                if (bj[s] == k) {                               // X_kk = D
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int b = 0; b < 2; ++b)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                acc[s][a][b][e] = Dm[(16 * a + 4 * e + lq) * kFacPitch + 16 * b + l16];
                } else {                                        // X_kj = D R_kj
                    clear(acc[s]);
                    mul(acc[s], Dm, Xp + bj[s] * kFacBlock, kFacPitch, 1, 1.0);
                    put(Xp + bj[s] * kFacBlock, acc[s]);
                }
                const int row0 = 32 * k + lq, col0 = 32 * bj[s] + l16;
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int row = row0 + 16 * a + 4 * e, col = col0 + 16 * b;
                            if (row < nn && col < nn) Xg[(unsigned)(row * ld + col)] = (float)acc[s][a][b][e];
                        }
            }
        }
        __syncthreads();
        if (k + 1 == nb) break;
        asm volatile("" : "+v"(l16), "+v"(lq));
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (bi[s] <= k || (FACTOR && bj[s] <= k)) continue;
            // A_ij -= L_ik L_jk^T right of the panel, R_ij -= L_ik X_kj up to it
            const bool right = bj[s] > k;
            const double* B = right ? Lp + (bj[s] - 1) * kFacBlock : bj[s] == k ? Dm : Xp + bj[s] * kFacBlock;
            mul(acc[s], Lp + (bi[s] - 1) * kFacBlock, B, right ? 1 : kFacPitch, right ? kFacPitch : 1, -1.0);
        }
        __syncthreads();     // the panel's buffers are written again
    }
}

// The same for orders up to 32: one block, one wavefront per matrix.  Most of the large kernel's time there was
// fetching its code (14 us for one 32 x 32 block).
template <bool FACTOR>
__global__ __launch_bounds__(64) void k_inverse_factor_small(const MatDev* __restrict__ mats,
                                                             const SymPlanes* __restrict__ sym,
                                                             double shift_rel, int n_mats, ClearShare share, int* status) {
    if (!FACTOR && (int)blockIdx.x >= n_mats) {      // (nothing is cleared beside FACTOR: its launches come after the last share)
        clear_share(mats, n_mats, share, (int)blockIdx.x - n_mats);
        return;
    }
    __shared__ __attribute__((aligned(16))) double Am[kFacBlock], Dm[kFacBlock], Lt[FACTOR ? kFacBlock : 1];
    const MatDev& md = mats[blockIdx.x];
    const SymPlanes sp = sym[blockIdx.x];
    const int nn = sp.order, lane = threadIdx.x, c = lane & 31, h = lane >> 5;
    // lane (c, h): column c, rows h, h + 2, ...; the lower triangle of the sum of the planes
    double v[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) v[x] = c == 2 * x + h && c >= nn ? 1.0 : 0.0;      // identity past the order
    for (int y = 0; y < sp.count; y += 2) {
        const float* __restrict__ p0 = sp.p + y * sp.pitch;
        const float* __restrict__ p1 = y + 1 < sp.count ? p0 + sp.pitch : p0;
        float f[2][16];
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            const int row = 2 * x + h;
            const int at = row < nn && c <= row ? row * nn + c : 0;
            f[0][x] = p0[at];
            f[1][x] = p1[at];
        }
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            const int row = 2 * x + h;
            if (row < nn && c <= row) {
                v[x] += (double)f[0][x];
                if (y + 1 < sp.count) v[x] += (double)f[1][x];
            }
        }
    }
    double shift = 0.0;
    if (shift_rel > 0.0) {
        double tr = 0.0;
#pragma unroll
        for (int x = 0; x < 16; ++x) tr += c == 2 * x + h && c < nn ? v[x] : 0.0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off, 64);
        shift = shift_rel * tr;
    }
#pragma unroll
    for (int x = 0; x < 16; ++x) Am[(2 * x + h) * kFacPitch + c] = v[x] + (c == 2 * x + h && c < nn ? shift : 0.0);
    if (FACTOR && lane < kJacobiFlags) md.jflag[lane] = 0;
    lds_order();
    if (factor_diag<FACTOR>(Am, Dm, Lt, FACTOR ? 0.25 * shift : 0.0, lane) && lane == 0) atomicOr(status, 4);
    lds_order();
    float* __restrict__ X = md.Linv;
    const int lp = md.lp;
#pragma unroll
    for (int x = 0; x < 16; ++x) {
        const int row = 2 * x + h;
        if (FACTOR) X[row * lp + c] = row < nn && c < nn ? (float)Lt[row * kFacPitch + c] : 0.f;
        else if (row < nn && c < nn) X[row * lp + c] = c <= row ? (float)Dm[row * kFacPitch + c] : 0.f;
    }
}

// CholeskyQR of a sketch of up to 32 columns in one launch, a workgroup per matrix: X (rows x nn) becomes X L^{-T}, where
// X^T X (+ shift on the diagonal) = L L^T, once or twice over.  Each pass reads the sketch twice, once as the rows that a
// lane group contracts over and once as the rows of a result; kOrthoWaves wavefronts take 32 rows at a time for both
// products, another one the factor in between, during which the first rows for the second product are on their way.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kOrthoWaves = 8;

// The arithmetic of both products: fp64 for the last basis and the new projector, fp32 for the bases inside the subspace
// iteration, which have to stay apart and no more.  (With fp32 throughout the projector of a 256 x 512 gradient was 4.66e-7
// from the exact one, a root mean square over eight draws; with products of three bf16 planes, which round once per 16
// products and not once per product, 4.58e-7.  A 16 x 16 x 4 product is 64 cycles in fp64, 32 in fp32.)
// row_of: the row of a result's 16 that element e of lane group g holds.
template <bool EXACT>
struct OrthoMath {
    using T = double;
    using T4 = double4_t;
    static __device__ __forceinline__ T4 mul(double a, double b, T4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row_of(int e, int g) { return 4 * e + g; }
};
template <>
struct OrthoMath<false> {
    using T = float;
    using T4 = f32x4_t;
    static __device__ __forceinline__ T4 mul(float a, float b, T4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row_of(int e, int g) { return 4 * g + e; }
};

// A chunk's 32 rows as the two products take them, zero past the last row and column.  (Its start and the steps to its
// rows are the same for every lane: one address in scalar registers per load and one offset per lane.)
// rows 16 x + 4 g + e, columns c + 16 t: what the Gram matrix is contracted over
__device__ __forceinline__ void ortho_gram_rows(const float* src, int row0, int rows, int nn, int c, int g, float (&y)[2][4][2]) {
    const unsigned at[2] = {(unsigned)(4 * g * nn + (c < nn ? c : 0)), (unsigned)(4 * g * nn + (c + 16 < nn ? c + 16 : 0))};
    if (row0 + 32 <= rows) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < 2; ++t) y[x][e][t] = (src + (row0 + 16 * x + e) * nn)[at[t]];
    } else {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const bool in = row0 + 16 * x + 4 * g + e < rows;
                    const float q = in ? (src + (row0 + 16 * x + e) * nn)[at[t]] : 0.f;
                    y[x][e][t] = q;
                }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < 2; ++t) y[x][e][t] = c + 16 * t < nn ? y[x][e][t] : 0.f;
}

// rows 16 x + c, columns 16 h + 4 g + u: what the second product multiplies; in fp64 row 4 (c % 4) + c / 4 in place of c, which
// makes the four results of a lane consecutive rows there as well
template <bool EXACT>
__device__ __forceinline__ void ortho_rows(const float* src, int row0, int rows, int nn, int lane_c, int g, f32x4_t (&y)[2][2]) {
    const int c = EXACT ? 4 * (lane_c & 3) + (lane_c >> 2) : lane_c;
    if ((nn & 3) == 0) {                     // (uniform)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool in = row0 + 16 * x + c < rows && 16 * h + 4 * g < nn;
                const unsigned at = (unsigned)(in ? (16 * x + c) * nn + 16 * h + 4 * g : 0);
                const f32x4_t q = *reinterpret_cast<const f32x4_t*>(src + row0 * nn + at);
#pragma unroll
                for (int u = 0; u < 4; ++u) y[x][h][u] = in ? q[u] : 0.f;
            }
    } else {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool in = row0 + 16 * x + c < rows && 16 * h + 4 * g + u < nn;
                    const unsigned at = (unsigned)(in ? (16 * x + c) * nn + 16 * h + 4 * g + u : 0);
                    const float q = (src + row0 * nn)[at];
                    y[x][h][u] = in ? q : 0.f;
                }
    }
}

// Rows row0, row0 + 32 kOrthoWaves, ... of src times L^{-T} (Dm: L^{-1}); y: the first 32 of them.
template <bool EXACT>
__device__ __forceinline__ void ortho_apply(const MatDev& md, const double* Dm, const float* src, float* dst, int row0, int rows, int nn,
                                            int c, int g, int np, bool twice, f32x4_t (&y)[2][2]) {
    using M = OrthoMath<EXACT>;
    using T = typename M::T;
    // element (k, j) of L^{-T}, k = 16 h + 4 g + u, j = c (+ 16): zero below the diagonal
    T b0[4], b1[2][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        b0[u] = 4 * g + u <= c ? (T)Dm[c * kFacPitch + 4 * g + u] : (T)0;
        b1[0][u] = (T)Dm[(16 + c) * kFacPitch + 4 * g + u];
        b1[1][u] = 4 * g + u <= c ? (T)Dm[(16 + c) * kFacPitch + 16 + 4 * g + u] : (T)0;
    }
    for (; row0 < rows; row0 += 32 * kOrthoWaves) {
        f32x4_t next[2][2];
        if (row0 + 32 * kOrthoWaves < rows) ortho_rows<EXACT>(src, row0 + 32 * kOrthoWaves, rows, nn, c, g, next);
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            typename M::T4 q[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                q[0] = M::mul(y[x][0][u], b0[u], q[0]);
                q[1] = M::mul(y[x][0][u], b1[0][u], q[1]);
                q[1] = M::mul(y[x][1][u], b1[1][u], q[1]);
            }
            const int r0 = row0 + 16 * x + 4 * g;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int col = c + 16 * t;
                float z[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) z[e] = (float)q[t][e];
                if (np > 0 && col < nn && (r0 & ~7) < rows) {
                    // half an octet of a sketch plane, rows past the last zero
                    unsigned lo[3], hi[3];
                    split2<3>(r0 < rows ? z[0] : 0.f, r0 + 1 < rows ? z[1] : 0.f, lo);
                    split2<3>(r0 + 2 < rows ? z[2] : 0.f, r0 + 3 < rows ? z[3] : 0.f, hi);
                    const long long at = ((long long)(r0 >> 3) * nn + col) * 8 + (r0 & 4);
#pragma unroll
                    for (int p = 0; p < 3; ++p)
                        if (p < np) *reinterpret_cast<u32x2_t*>(sketch_plane(md, twice, p) + at) = (u32x2_t){lo[p], hi[p]};
                }
                if (np == 0 || twice) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (r0 + e < rows && col < nn) (dst + (row0 + 16 * x + e) * nn)[(unsigned)(4 * g * nn + col)] = z[e];
                }
            }
            y[x][0] = next[x][0];
            y[x][1] = next[x][1];
        }
    }
}

template <bool EXACT>
__global__ __launch_bounds__(64 * (kOrthoWaves + 1)) void k_orthonormalise_small(const MatDev* __restrict__ mats, int which, int passes,
                                                                                 double shift_rel, int planes, int n_mats,
                                                                                 ClearShare share, int* status) {
    if ((int)blockIdx.x >= n_mats) {
        clear_share(mats, n_mats, share, (int)blockIdx.x - n_mats);
        return;
    }
    __shared__ __attribute__((aligned(16))) double Am[kFacBlock], sums[kOrthoWaves * 3 * 256 * sizeof(typename OrthoMath<EXACT>::T) / sizeof(double)];
    using M = OrthoMath<EXACT>;
    using T = typename M::T;
    T* const part = reinterpret_cast<T*>(sums);      // [kOrthoWaves][3][256]
    double* const Dm = sums;                 // (the partial sums are in Am by the time the factor is written)
    static_assert(sizeof(sums) >= kFacBlock * sizeof(double), "");
    const MatDev& md = mats[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int nn = which == kOrthoP ? md.r : md.l, rows = which == kOrthoB ? md.n : md.m;
    float* const first = which == kOrthoP ? md.P : which == kOrthoB ? md.Yb : md.Ya;
    float* const other = which == kOrthoP ? md.Ya : md.Yc;
    if (w == kOrthoWaves) {
        for (int pass = 0; pass < passes; ++pass) {
            __syncthreads();
            __syncthreads();
            if (pass == 0 && shift_rel > 0.0) {
                const double d = lane < nn ? Am[lane * (kFacPitch + 1)] : 0.0;
                double tr = d;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off, 64);
                if (lane < nn) Am[lane * (kFacPitch + 1)] = d + shift_rel * tr;
                lds_order();
            }
            if (factor_diag<false>(Am, Dm, nullptr, 0.0, lane) && lane == 0) atomicOr(status, 4);
            __syncthreads();
            __syncthreads();
        }
        return;
    }
    for (int pass = 0; pass < passes; ++pass) {
        const float* src = pass ? other : first;
        float* dst = pass ? first : other;
        typename M::T4 g00 = {0, 0, 0, 0}, g10 = g00, g11 = g00;
        for (int row0 = 32 * w; row0 < rows; row0 += 32 * kOrthoWaves) {
            float y[2][4][2];
            ortho_gram_rows(src, row0, rows, nn, c, g, y);
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    g00 = M::mul(y[x][e][0], y[x][e][0], g00);
                    g10 = M::mul(y[x][e][1], y[x][e][0], g10);
                    g11 = M::mul(y[x][e][1], y[x][e][1], g11);
                }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            part[768 * w + 64 * e + lane] = g00[e];
            part[768 * w + 256 + 64 * e + lane] = g10[e];
            part[768 * w + 512 + 64 * e + lane] = g11[e];
        }
        __syncthreads();
        for (int i = tid; i < 3 * 256; i += 64 * kOrthoWaves) {
            double sum = 0.0;
#pragma unroll
            for (int q = 0; q < kOrthoWaves; ++q) sum += (double)part[768 * q + i];
            const int row = (i >= 256 ? 16 : 0) + M::row_of((i & 255) >> 6, (i & 63) >> 4), col = (i >= 512 ? 16 : 0) + (i & 15);
            Am[row * kFacPitch + col] = row < nn && col < nn ? sum : row == col ? 1.0 : 0.0;      // identity past the order
        }
        __syncthreads();
        f32x4_t y[2][2];
        if (32 * w < rows) ortho_rows<EXACT>(src, 32 * w, rows, nn, c, g, y);
        __syncthreads();
        const int np = pass + 1 == passes && md.Yp != nullptr ? planes : 0;
        ortho_apply<EXACT>(md, Dm, src, dst, 32 * w, rows, nn, c, g, np, passes == 2, y);
        __syncthreads();
    }
}

hipError_t launch_orthonormalise_small(int which, int passes, double shift_rel, int planes, const MatDev* mats, int n_mats,
                                       ClearShare clear, int* status, hipStream_t stream) {
    const dim3 grid(n_mats + clear.blocks), block(64 * (kOrthoWaves + 1));
    if (passes == 2 || which == kOrthoP)
        hipLaunchKernelGGL(k_orthonormalise_small<true>, grid, block, 0, stream, mats, which, passes, shift_rel, planes, n_mats, clear, status);
    else
        hipLaunchKernelGGL(k_orthonormalise_small<false>, grid, block, 0, stream, mats, which, passes, shift_rel, planes, n_mats, clear, status);
    return hipGetLastError();
}

template <bool FACTOR, int WAVES, int SLOTS>
static hipError_t run_factor_blocks(const MatDev* mats, const SymPlanes* sym, int n_mats, int nb, double shift_rel,
                                    const ClearShare& clear, int* status, hipStream_t stream) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(k_inverse_factor<FACTOR, WAVES, SLOTS>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       2 * kFacNB * kFacBlock * (int)sizeof(double));
    (void)attr;
    const size_t lds = (size_t)2 * nb * kFacBlock * sizeof(double);
    hipLaunchKernelGGL((k_inverse_factor<FACTOR, WAVES, SLOTS>), dim3(n_mats + clear.blocks), dim3(64 * (WAVES + 1)), lds,
                       stream, mats, sym, shift_rel, nb, n_mats, clear, status);
    return hipGetLastError();
}

template <bool FACTOR>
static hipError_t run_factor(const MatDev* mats, const SymPlanes* sym, int n_mats, int max_order, double shift_rel,
                             const ClearShare& clear, int* status, hipStream_t stream) {
    if (max_order <= 32) {
        hipLaunchKernelGGL(k_inverse_factor_small<FACTOR>, dim3(n_mats + clear.blocks), dim3(64), 0, stream, mats, sym, shift_rel,
                           n_mats, clear, status);
        return hipGetLastError();
    }
    const int nb = (max_order + 31) / 32;
    if (nb <= 4) return run_factor_blocks<FACTOR, 10, 1>(mats, sym, n_mats, nb, shift_rel, clear, status, stream);
    return run_factor_blocks<FACTOR, 7, 6>(mats, sym, n_mats, nb, shift_rel, clear, status, stream);
}

// Workgroups that clear `bytes` beside a launch: as many as there are places, or fewer, so that each has about as much as it
// stores while the launch lasts; spread wider, the stores hold up what the launch is there for.  Refresh (us) at 64 KB / 128 KB /
// 256 KB / 512 KB / 1 MB / 2 MB / 4 MB each:
//   orders up to 32: six 2048-wide blocks at rank 24 1706 / 1705 / 1723 / 1739 / 1844 / 2055 / 2430, one 1024 x 32000 1447 / 1445 / 1444 / 1456 /
//     1488 / 1580 / 1783
//   other factors: 60M set 1597 / 1596 / 1594 / 1590 / 1589 / 1590 / 1674, eight 1024 x 16384 at rank 128 2682 / 2681 / 2682 / 2680 / 2646 / 2620 / 2677,
//     one 768 x 50257 4270 / 4286 / 4284 / 4257 / 4255 / 4256 / 4335
//   rounds, at 256 KB / 512 KB / 768 KB / 1 MB / 2 MB: 350M set 11642 / 11593 / 11550 / 11576 / 12336, 130M set 6940 / 6921 / 6917 / 6916 / 7361
constexpr unsigned long long kClearSmall = 128 << 10, kClearFactor = 1 << 20, kClearRound = 768 << 10;
static int clear_blocks(unsigned long long bytes, unsigned long long each, int places) {
    const unsigned long long wanted = (bytes + each - 1) / each;
    return wanted < (unsigned)places ? (int)wanted : places;
}

int clear_share_blocks(int n_mats, int max_order, int max_pairs, unsigned long long bytes) {
    if (max_order <= 32) return clear_blocks(bytes, kClearSmall, 512);
    if (max_order > kFactorMax || (long long)n_mats * max_pairs > 512 || n_mats > 192) return 0;
    return clear_blocks(bytes, kClearFactor, 256 - n_mats);
}

hipError_t launch_inverse_factor(GemmOp op, const MatDev* mats, const SymPlanes* sym, int n_mats, int max_order,
                                 double shift_rel, ClearShare clear, int* status, hipStream_t stream) {
    if (max_order <= kFactorMax) return run_factor<false>(mats, sym, n_mats, max_order, shift_rel, clear, status, stream);
    const int which = op == OP_GRAM_P ? 1 : 0;
    hipLaunchKernelGGL(k_sum_planes, dim3(64, n_mats), dim3(256), 0, stream, mats, sym);
    hipError_t e = launch_cholesky(mats, n_mats, which, max_order, shift_rel, false, status, stream);
    if (e != hipSuccess) return e;
    return launch_tri_inverse(mats, n_mats, which, max_order, stream);
}

// ------------------------------------------------------------------ blocked one-sided Jacobi
// X (lp x lp, row-major) starts as L^T, where T + shift = L L^T (rows/columns >= l zero).  With
// T = U Lambda^2 U^T the singular vectors of L are U, so rotating ROWS of L^T until they are mutually
// orthogonal gives X = Lambda U^T: row i is ritz_i * u_i^T, ritz the singular value of the gradient (up to
// the shift, which moves every eigenvalue of T alike).  Started from T itself the rows carry the squares of
// those values: what lies below 2.4e-4 of the largest drowns in the rounding of the rows as floats, and a signal
// over a floor takes many sweeps more (rank 128 over a floor of 1e-4 at order 256: 12 to 15, from L^T 7 or 8).
// The shift of 1e-6 trace(T) keeps every row at least 1e-3 of the gradient's norm long; directions whose squared
// values differ by less than 3e-4 of the shift may end as a mixture among themselves.
// Rows are grouped in blocks of 16; one workgroup takes a pair of blocks (a "visit"): it forms the 32 x 32
// Gram matrix of the 32 rows, runs one cyclic Jacobi sweep on that small matrix with the rotations
// accumulated in V, and applies X <- V X to the rows.  Block pairs follow a round-robin tournament so the
// lp/16 - 1 rounds of one sweep meet every block pair once.
__device__ __forceinline__ void tournament_pair(int players, int round, int k, int* a, int* b) {
    const int N = players - 1;
    if (k == 0) {
        *a = N;
        *b = round % N;
    } else {
        *a = (round + k) % N;
        *b = (round - k + N) % N;
    }
}

// The rows that the Jacobi rotates are kept as floats (the result, a rotation stored as floats, needs
// no more; every product and sum on them is still formed in fp64), in the buffer of the inverse Cholesky
// factor, which is free between the last orthonormalisation and the one of the new projector.
__device__ __forceinline__ float* jacobi_rows(const MatDev& md) { return md.Linv; }

// L^T of T = L L^T (orders above kFactorMax: T holds L), zero below the diagonal and in the padding
__global__ __launch_bounds__(256) void k_jacobi_prepare(const MatDev* __restrict__ mats) {
    __shared__ float tile[32][33];
    const MatDev& md = mats[blockIdx.z];
    const int lp = md.lp, l = md.l;
    const int i0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
    if (i0 >= lp || j0 >= lp) return;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kJacobiFlags) md.jflag[threadIdx.x] = 0;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int y = ty; y < 32; y += 8) {      // rows j0 + y of L, columns i0 + tx
        const int j = j0 + y, i = i0 + tx;
        tile[y][tx] = (i <= j && j < l) ? (float)md.T[(long long)j * lp + i] : 0.f;
    }
    __syncthreads();
    float* __restrict__ X = jacobi_rows(md);
    for (int y = ty; y < 32; y += 8) X[(long long)(i0 + y) * lp + j0 + tx] = tile[tx][y];
}

hipError_t launch_jacobi_prepare(const MatDev* mats, const SymPlanes* sym, int n_mats, int max_l, int max_lp, int* status,
                                 hipStream_t stream) {
    // the shift leaves the eigenvectors alone and covers the rounding of T; what it hides: see the comment on the rows
    constexpr double kShift = 1e-6;
    if (max_l <= kFactorMax) return run_factor<true>(mats, sym, n_mats, max_l, kShift, ClearShare(), status, stream);
    hipLaunchKernelGGL(k_sum_planes, dim3(64, n_mats), dim3(256), 0, stream, mats, sym);
    const hipError_t e = launch_cholesky(mats, n_mats, 0, max_l, kShift, true, status, stream);
    if (e != hipSuccess) return e;
    const unsigned nt = (unsigned)(max_lp + 31) / 32;
    hipLaunchKernelGGL(k_jacobi_prepare, dim3(nt, nt, n_mats), dim3(256), 0, stream, mats);
    return hipGetLastError();
}

// ------------------------------------------------------------------ block rotation through the Gram matrix
// One visit of a pair of 16-row blocks (32 rows of length lp, floats in global memory):
//   S = X X^T          32 x 32 Gram of the rows, fp64 MFMA (16x16x4), the columns split over the wavefronts
//   small sweep        rounds of 16 disjoint rotations each, applied two-sidedly to S (S <- J S J^T) and
//                      accumulated in V (V <- J V): the rotations that a row-by-row Jacobi would apply,
//                      decided from S instead of fresh dot products.  Round 0 of a sweep takes all 496
//                      row pairs of the visit (31 rounds), every other round the 256 pairs with a row
//                      in each block (16 rounds)
//   X <- V X           fp64 MFMA, each wavefront owns 16-column tiles, written straight back to memory
// so the 32 rows are read twice per visit instead of 2 x 31 times.
//
// The small sweep is a chain of dependent rounds, and one wavefront (two where there are four: SweepHalf) runs it in registers; another one follows
// it round by round and accumulates V.  (With S and V in LDS and eight wavefronts a round was two barriers
// and 14 LDS accesses per thread, 0.7 us.)  The rounds go through the pairs (i, i xor x).  A phase is the
// x with highest bit f: the 16 indexes with bit f clear are "lower", the others "upper", both numbered by
// their other bits, and round x = 2^f + g pairs lower k with upper k xor g.  Lane (k, z), k = lane % 16, holds the
// columns lower k and upper k xor g, of the rows lower 4z + i and upper (4z + i) xor g, i = 0..3: four 2 x 2
// blocks that a round transforms where they are.  Going on to the next g moves the upper columns between
// the lanes of a row of 16, by one DPP pattern (g runs 0 1 3 2, 5 4 6 7, 15 14 12 13, 10 11 9 8: steps xor
// 1, 2, 7 and 8), and the upper rows between registers, at compile time inside a group of four, with an
// exchange between the rows of 16 lanes after each group.  Between phases bits f and f + 1 change places.
// The lane on the diagonal (z = k / 4) computes the rotation of pair k and publishes it through LDS.
// Rotations are kept in scaled form: a row or column is its scale times what is stored, and a rotation by the
// tangent t multiplies both scales by its cosine and adds p = t e_b / e_a times one stored row to the
// other: half the multiply-adds, and the cosine is off the chain.
// (operand and result layout of v_mfma_f64_16x16x4_f64 as stated at the triangular inverse; checked on
// the device)
constexpr int kJgRounds = 31;                     // most rounds of a small sweep
constexpr int kJgCoef = kJgRounds * 48 + 32;      // doubles of their coefficients and the scales
constexpr int kJgLd = 34;      // row length of S and V in LDS: the 16 rows of an operand on distinct banks

// tangent of the rotation that orthogonalises two rows with squared norms al, be and inner product ga (the
// same angle as a row-by-row kernel's).  Reciprocal and reciprocal square root start from the hardware
// approximations and take Newton steps.
__device__ __forceinline__ double rsq_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = y * (1.5 - 0.5 * x * y * y);
    return y * (1.5 - 0.5 * x * y * y);
}
__device__ __forceinline__ double rotation_tan(double al, double be, double ga) {
    const double d = be - al, g2 = 2.0 * ga;
    const double q = d * d + g2 * g2;
    // (the angle only has to be good enough to shrink the coupling quadratically: one Newton step)
    double y = __builtin_amdgcn_rsq(q);
    y = y * (1.5 - 0.5 * q * y * y);
    const double den = fabs(d) + q * y;                              // |d| + sqrt(d^2 + 4 ga^2)
    double rd = __builtin_amdgcn_rcp(den);
    rd = rd * (2.0 - den * rd);
    return (d >= 0.0 ? g2 : -g2) * rd;
}

// (on the halves: written as one conditional on doubles the compiler turns a tree of them into an array in scratch memory)
__device__ __forceinline__ double select_d(bool c, double a, double b) {
    const int lo = c ? __double2loint(a) : __double2loint(b), hi = c ? __double2hiint(a) : __double2hiint(b);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ void swap_d(double& a, double& b) {
    const double t = a;
    a = b;
    b = t;
}
// the value of the partner lane inside the row of 16 lanes
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor3 = 0x1B, kDppXor7 = 0x141, kDppXor8 = 0x128;
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
// BIT 0: rows of 16 lanes 1 and 3 of a change places with rows 0 and 2 of b; BIT 1: rows 2, 3 of a with 0, 1 of b
template <int BIT>
__device__ __forceinline__ void row_swap(double& a, double& b) {
    u32x2_t lo, hi;
    if (BIT == 0) {
        lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
        hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    } else {
        lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
        hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    }
    a = __hiloint2double((int)hi.x, (int)lo.x);
    b = __hiloint2double((int)hi.y, (int)lo.y);
}
// the value of the lane whose z differs in bit BIT
template <int BIT>
__device__ __forceinline__ double row_flip(double v, int z) {
    double a = v, b = v;
    row_swap<BIT>(a, b);
    return (z & (1 << BIT)) ? a : b;
}

// Two columns (c = 0, 1) of the rows a lane holds.
struct JacobiRows {
    double lo[4][2], up[4][2];
    // the upper rows go from one group of four rounds to the next: register bit LOW, bit 2 + BIT of the numbering
    template <int LOW, int BIT>
    __device__ __forceinline__ void next_group(int z) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (!(i & (1 << LOW))) swap_d(up[i][c], up[i | (1 << LOW)][c]);
            }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) up[i][c] = row_flip<BIT>(up[i][c], z);
    }
    // the bit that separates lower from upper changes places with bit p (uniform) of the numbering
    __device__ __forceinline__ void exchange_rows(int p) {
        if (p == 0) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                swap_d(lo[1][c], up[0][c]);
                swap_d(lo[3][c], up[2][c]);
            }
        } else if (p == 1) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                swap_d(lo[2][c], up[0][c]);
                swap_d(lo[3][c], up[1][c]);
            }
        } else if (p == 2) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) row_swap<0>(lo[i][c], up[i][c]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) row_swap<1>(lo[i][c], up[i][c]);
        }
    }
    // round r of a group: stored lower row -= p * upper, stored upper row += q * lower
    template <int R>
    __device__ __forceinline__ void rotate_rows(const double (&p)[4], const double (&q)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double l = fma(-p[i], up[i ^ R][c], lo[i][c]);
                up[i ^ R][c] = fma(q[i], lo[i][c], up[i ^ R][c]);
                lo[i][c] = l;
            }
    }
};

// index with number k among the lower (upper = 0) or upper ones of phase f
__device__ __forceinline__ int jacobi_index(int f, int k, int upper) {
    return ((k >> f) << (f + 1)) | (upper << f) | (k & ((1 << f) - 1));
}

// The rounds of a small sweep in order.  A: a wavefront's side of them -- round<R>(), step<DPP>() (upper
// columns move), next_group<LOW, BIT>(), exchange(f).
template <class A>
__device__ __forceinline__ void jacobi_rounds(A& s, bool cross) {
    for (int f = cross ? 4 : 0;; ++f) {
        const int groups = f > 2 ? 1 << (f - 2) : 1;
        for (int n = 0;; ++n) {
            s.template round<0>();
            if (f > 0) {
                s.template step<kDppXor1>();
                s.template round<1>();
            }
            if (f > 1) {
                s.template step<kDppXor2>();
                s.template round<3>();
                s.template step<kDppXor1>();
                s.template round<2>();
            }
            if (n + 1 == groups) break;
            if (n == 1) {
                s.template step<kDppXor8>();
                s.template next_group<1, 1>();
            } else {
                s.template step<kDppXor7>();
                s.template next_group<0, 0>();
            }
        }
        if (f == 4) break;
        // back to g = 0 (from 1, 2, 7), then the next phase
        if (f == 1) s.template step<kDppXor1>();
        if (f == 2) s.template step<kDppXor2>();
        if (f == 3) {
            s.template step<kDppXor7>();
            s.template next_group<0, 0>();
        }
        s.exchange(f);
    }
}

// One bare barrier per round: what the sweeping wavefront wrote before it has landed.
__device__ __forceinline__ void sweep_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Coefficients of a round in LDS: p, q of the 16 pairs, then their tangents.
constexpr int kJgRoundCoef = 48;

// lanes with the bit set give their lower column to, and take the upper column of, the lane without it
template <int A, int B>
__device__ __forceinline__ void exchange_pair(double& lo, double& up, bool set) {
    double pl = dpp_d<A>(lo), pu = dpp_d<A>(up);
    if (B != 0) {
        pl = dpp_d<B ? B : A>(pl);
        pu = dpp_d<B ? B : A>(pu);
    }
    lo = set ? pu : lo;
    up = set ? up : pl;
}

// The wavefront that runs the sweep on S.
struct SweepMain {
    JacobiRows S;
    double scl, scu, iscl, iscu;      // scales of this lane's two columns and their reciprocals
    double smax;                      // largest diagonal entry (scale of the rounding noise inside the visit)
    double* rc;                       // this round's coefficients
    int k, z, nrot;

    __device__ __forceinline__ void init(const double* S0, double* coef, bool cross, int lane) {
        k = lane & 15;
        z = lane >> 4;
        rc = coef;
        nrot = 0;
        scl = scu = iscl = iscu = 1.0;
        const int f = cross ? 4 : 0;
        const int cl = jacobi_index(f, k, 0), cu = jacobi_index(f, k, 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double* rl = S0 + jacobi_index(f, 4 * z + i, 0) * kJgLd;
            const double* ru = S0 + jacobi_index(f, 4 * z + i, 1) * kJgLd;
            S.lo[i][0] = rl[cl];
            S.lo[i][1] = rl[cu];
            S.up[i][0] = ru[cl];
            S.up[i][1] = ru[cu];
        }
        smax = S0[(lane & 31) * kJgLd + (lane & 31)];
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) smax = fmax(smax, __shfl_xor(smax, off, 64));
    }
    template <int R>
    __device__ __forceinline__ void round() {
        // the 2 x 2 block on the diagonal, valid in the lanes with z = k / 4
        const bool k0 = k & 1, k1 = k & 2;
        const double ee = scl * scu;
        const double ga = ee * select_d(k1, select_d(k0, S.up[3 ^ R][0], S.up[2 ^ R][0]), select_d(k0, S.up[1 ^ R][0], S.up[0 ^ R][0]));
        const double al = scl * scl * select_d(k1, select_d(k0, S.lo[3][0], S.lo[2][0]), select_d(k0, S.lo[1][0], S.lo[0][0]));
        const double be = scu * scu * select_d(k1, select_d(k0, S.up[3 ^ R][1], S.up[2 ^ R][1]), select_d(k0, S.up[1 ^ R][1], S.up[0 ^ R][1]));
        const bool rotate = (al > 0.0) && (be > 0.0) && (ga * ga > 1.0e-15 * al * be);
        double tn = rotation_tan(al, be, ga);
        tn = rotate ? tn : 0.0;
        const bool owner = z == (k >> 2);
        if (owner) {
            rc[2 * k] = tn * (scu * iscl);
            rc[2 * k + 1] = tn * (scl * iscu);
            rc[32 + k] = tn;
        }
        sweep_barrier();
        // A coupling below the visit's own rounding noise (entries that went through rotations with much
        // larger rows), or one below ~3e-4 of the two rows' norms (what is left after a sweep of such
        // rotations is quadratically smaller, ~1e-7: the rounding of the float the result is stored in),
        // is applied but does not keep the sweep loop alive
        if (owner && rotate && fabs(ga) > 8.0e-15 * smax && ga * ga > 1.0e-7 * al * be) ++nrot;
        double p[4], q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = rc[2 * (4 * z + i)];
            q[i] = rc[2 * (4 * z + i) + 1];
        }
        const double pc = rc[2 * k], qc = rc[2 * k + 1], t = rc[32 + k];
        S.template rotate_rows<R>(p, q);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double l = fma(-pc, S.lo[i][1], S.lo[i][0]), u = fma(-pc, S.up[i][1], S.up[i][0]);
            S.lo[i][1] = fma(qc, S.lo[i][0], S.lo[i][1]);
            S.up[i][1] = fma(qc, S.up[i][0], S.up[i][1]);
            S.lo[i][0] = l;
            S.up[i][0] = u;
        }
        const double c2 = fma(t, t, 1.0), c = rsq_nr(c2), ic = c2 * c;
        scl *= c;
        scu *= c;
        iscl *= ic;
        iscu *= ic;
        rc += kJgRoundCoef;
    }
    template <int CTRL>
    __device__ __forceinline__ void step() {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            S.lo[i][1] = dpp_d<CTRL>(S.lo[i][1]);
            S.up[i][1] = dpp_d<CTRL>(S.up[i][1]);
        }
        scu = dpp_d<CTRL>(scu);
        iscu = dpp_d<CTRL>(iscu);
    }
    template <int LOW, int BIT>
    __device__ __forceinline__ void next_group() { S.template next_group<LOW, BIT>(z); }
    template <int A, int B>
    __device__ __forceinline__ void exchange_columns(bool set) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            exchange_pair<A, B>(S.lo[i][0], S.lo[i][1], set);
            exchange_pair<A, B>(S.up[i][0], S.up[i][1], set);
        }
        exchange_pair<A, B>(scl, scu, set);
        exchange_pair<A, B>(iscl, iscu, set);
    }
    __device__ __forceinline__ void exchange(int f) {
        S.exchange_rows(f);
        const bool set = (k >> f) & 1;
        if (f == 0) exchange_columns<kDppXor1, 0>(set);
        else if (f == 1) exchange_columns<kDppXor2, 0>(set);
        else if (f == 2) exchange_columns<kDppXor7, kDppXor3>(set);
        else exchange_columns<kDppXor8, 0>(set);
    }
    __device__ __forceinline__ void finish(double* scales) const {      // phase 4 ended at g = 8
        if (z == 0) {
            scales[k] = scl;
            scales[16 + (k ^ 8)] = scu;
        }
    }
};

// Where a visit has wavefronts to spare (NW = 4), two run the sweep, eight of the sixteen row pairs each: a round is the latency
// of one wavefront's chain and issue, and half of its rows is half of its multiply-adds, moves and selections.
// Wavefront h holds the rows 8 h + 2 z + i, lower and upper, i = 0, 1: bit 0 of a row's number is the register, bits 1 and 2
// are the row of 16 lanes and bit 3 the wavefront.  So what SweepMain does with register bit 1 is an exchange between rows of
// 16 lanes here, what it does with z bit 1 one between the wavefronts, through LDS; both wavefronts hold all
// columns and keep the scales.  The rotations are the same, bit for bit.  (Refresh of
// the 60M set 1658 -> 1615 us, of one 32-row matrix 344 -> 340.  What is left of a round, some 1000 cycles, is the way of
// the coefficients: 110 to write them to LDS, 75 at the barrier, 290 to read them, against 100 for the multiply-adds; without
// the tangent's divisions, or without the accumulation of V, it takes as long.)
struct SweepHalf {
    double lo[2][2], up[2][2];
    double scl, scu, iscl, iscu;
    double smax;
    double* rc;
    double* xbuf;                     // [2 wavefronts][4][64]
    int k, z, h, nrot;

    __device__ __forceinline__ void init(const double* S0, double* coef, double* exchange_buffer, bool cross, int lane, int half) {
        k = lane & 15;
        z = lane >> 4;
        h = half;
        rc = coef;
        xbuf = exchange_buffer;
        nrot = 0;
        scl = scu = iscl = iscu = 1.0;
        const int f = cross ? 4 : 0;
        const int cl = jacobi_index(f, k, 0), cu = jacobi_index(f, k, 1);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const double* rl = S0 + jacobi_index(f, 8 * h + 2 * z + i, 0) * kJgLd;
            const double* ru = S0 + jacobi_index(f, 8 * h + 2 * z + i, 1) * kJgLd;
            lo[i][0] = rl[cl];
            lo[i][1] = rl[cu];
            up[i][0] = ru[cl];
            up[i][1] = ru[cu];
        }
        smax = S0[(lane & 31) * kJgLd + (lane & 31)];
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) smax = fmax(smax, __shfl_xor(smax, off, 64));
    }
    template <int BIT>
    __device__ __forceinline__ void flip() {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) up[i][c] = row_flip<BIT>(up[i][c], z);
    }
    // these four values of a lane change places with the other wavefront's
    __device__ __forceinline__ void trade(double (&mine)[2][2]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) xbuf[256 * h + 64 * v + 16 * z + k] = mine[v >> 1][v & 1];
        sweep_barrier();
#pragma unroll
        for (int v = 0; v < 4; ++v) mine[v >> 1][v & 1] = xbuf[256 * (1 - h) + 64 * v + 16 * z + k];
    }
    template <int R>
    __device__ __forceinline__ void round() {
        constexpr int X = R & 1;
        if (R == 3) flip<0>();                       // rounds 0 1 3 2: bit 1 is set from here on
        const bool k0 = k & 1;
        const double ee = scl * scu;
        const double ga = ee * select_d(k0, up[1 ^ X][0], up[0 ^ X][0]);
        const double al = scl * scl * select_d(k0, lo[1][0], lo[0][0]);
        const double be = scu * scu * select_d(k0, up[1 ^ X][1], up[0 ^ X][1]);
        const bool rotate = (al > 0.0) && (be > 0.0) && (ga * ga > 1.0e-15 * al * be);
        double tn = rotation_tan(al, be, ga);
        tn = rotate ? tn : 0.0;
        const bool owner = z == ((k >> 1) & 3) && h == (k >> 3);
        if (owner) {
            rc[2 * k] = tn * (scu * iscl);
            rc[2 * k + 1] = tn * (scl * iscu);
            rc[32 + k] = tn;
        }
        sweep_barrier();
        if (owner && rotate && fabs(ga) > 8.0e-15 * smax && ga * ga > 1.0e-7 * al * be) ++nrot;   // (as SweepMain)
        double p[2], q[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            p[i] = rc[2 * (8 * h + 2 * z + i)];
            q[i] = rc[2 * (8 * h + 2 * z + i) + 1];
        }
        const double pc = rc[2 * k], qc = rc[2 * k + 1], t = rc[32 + k];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double l = fma(-p[i], up[i ^ X][c], lo[i][c]);
                up[i ^ X][c] = fma(q[i], lo[i][c], up[i ^ X][c]);
                lo[i][c] = l;
            }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const double l = fma(-pc, lo[i][1], lo[i][0]), u = fma(-pc, up[i][1], up[i][0]);
            lo[i][1] = fma(qc, lo[i][0], lo[i][1]);
            up[i][1] = fma(qc, up[i][0], up[i][1]);
            lo[i][0] = l;
            up[i][0] = u;
        }
        const double c2 = fma(t, t, 1.0), c = rsq_nr(c2), ic = c2 * c;
        scl *= c;
        scu *= c;
        iscl *= ic;
        iscu *= ic;
        rc += kJgRoundCoef;
    }
    template <int CTRL>
    __device__ __forceinline__ void step() {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            lo[i][1] = dpp_d<CTRL>(lo[i][1]);
            up[i][1] = dpp_d<CTRL>(up[i][1]);
        }
        scu = dpp_d<CTRL>(scu);
        iscu = dpp_d<CTRL>(iscu);
    }
    template <int LOW, int BIT>
    __device__ __forceinline__ void next_group() {
        if (LOW == 0) {                              // bits 0 and 2; bit 1 back from rounds 3 and 2
#pragma unroll
            for (int c = 0; c < 2; ++c) swap_d(up[0][c], up[1][c]);
            flip<0>();
            flip<1>();
        } else {                                     // bits 1, which rounds 3 and 2 have set, and 3
            trade(up);
        }
    }
    template <int A, int B>
    __device__ __forceinline__ void exchange_columns(bool set) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            exchange_pair<A, B>(lo[i][0], lo[i][1], set);
            exchange_pair<A, B>(up[i][0], up[i][1], set);
        }
        exchange_pair<A, B>(scl, scu, set);
        exchange_pair<A, B>(iscl, iscu, set);
    }
    __device__ __forceinline__ void exchange(int f) {
        const bool set = (k >> f) & 1;
        if (f == 0) {
#pragma unroll
            for (int c = 0; c < 2; ++c) swap_d(lo[1][c], up[0][c]);
            exchange_columns<kDppXor1, 0>(set);
        } else if (f == 1) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) row_swap<0>(lo[i][c], up[i][c]);
            exchange_columns<kDppXor2, 0>(set);
        } else if (f == 2) {
            flip<0>();                               // bit 1 back from rounds 3 and 2
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) row_swap<1>(lo[i][c], up[i][c]);
            exchange_columns<kDppXor7, kDppXor3>(set);
        } else {
            double mine[2][2];
#pragma unroll
            for (int v = 0; v < 4; ++v) mine[v >> 1][v & 1] = select_d(h == 0, up[v >> 1][v & 1], lo[v >> 1][v & 1]);
            trade(mine);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                up[v >> 1][v & 1] = select_d(h == 0, mine[v >> 1][v & 1], up[v >> 1][v & 1]);
                lo[v >> 1][v & 1] = select_d(h == 0, lo[v >> 1][v & 1], mine[v >> 1][v & 1]);
            }
            exchange_columns<kDppXor8, 0>(set);
        }
    }
    __device__ __forceinline__ void finish(double* scales) const {      // phase 4 ended at g = 8
        if (h == 0 && z == 0) {
            scales[k] = scl;
            scales[16 + (k ^ 8)] = scu;
        }
    }
};

// The wavefront that accumulates V: lane (k, z) holds columns k and 16 + k.  SPLIT: beside two SweepHalf, whose barriers it joins.
template <bool SPLIT>
struct SweepVectors {
    JacobiRows V;
    const double* rc;
    int k, z;
    __device__ __forceinline__ void init(const double* coef, bool cross, int lane) {
        k = lane & 15;
        z = lane >> 4;
        rc = coef;
        const int f = cross ? 4 : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                V.lo[i][c] = jacobi_index(f, 4 * z + i, 0) == k + 16 * c ? 1.0 : 0.0;
                V.up[i][c] = jacobi_index(f, 4 * z + i, 1) == k + 16 * c ? 1.0 : 0.0;
            }
    }
    template <int R>
    __device__ __forceinline__ void round() {
        sweep_barrier();
        double p[4], q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = rc[2 * (4 * z + i)];
            q[i] = rc[2 * (4 * z + i) + 1];
        }
        V.template rotate_rows<R>(p, q);
        rc += kJgRoundCoef;
    }
    template <int CTRL>
    __device__ __forceinline__ void step() {}
    template <int LOW, int BIT>
    __device__ __forceinline__ void next_group() {
        if (SPLIT && LOW == 1) sweep_barrier();
        V.template next_group<LOW, BIT>(z);
    }
    __device__ __forceinline__ void exchange(int f) {
        if (SPLIT && f == 3) sweep_barrier();
        V.exchange_rows(f);
    }
    __device__ __forceinline__ void store(double* Vout, const double* scales) const {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rl = 4 * z + i, ru = 16 + (rl ^ 10);      // phase 4 ended with the registers at g = 8 + 2
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                Vout[rl * kJgLd + k + 16 * c] = V.lo[i][c] * scales[rl];
                Vout[ru * kJgLd + k + 16 * c] = V.up[i][c] * scales[ru];
            }
        }
    }
};

// LDS of a visit by NW wavefronts, in doubles: the partial Gram tiles, whose place S and then V take, and the
// coefficients
template <int NW>
__host__ __device__ constexpr int jacobi_visit_lds() {
    return (NW * 768 > 32 * kJgLd ? NW * 768 : 32 * kJgLd) + kJgCoef;
}

// One visit of blocks bp, bq by NW wavefronts; `sweeper` (0 .. NW - 1) runs the small sweep.  Ends on a barrier.
template <int NW>
__device__ __forceinline__ int jacobi_visit(float* __restrict__ X, int lp, int bp, int bq, bool cross, int sweeper,
                                            double* __restrict__ smem) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    double* coef = smem + (jacobi_visit_lds<NW>() - kJgCoef);
    float* Xp = X + (long long)bp * 16 * lp;   // rows 0..15 of the pair
    float* Xq = X + (long long)bq * 16 * lp;   // rows 16..31
    // ---- Gram: each wavefront takes its share of the columns and computes the tiles (0,0), (1,0), (1,1)
    // from the same two operands per k-step; (0,1) is the transpose of (1,0).  The partials are added in
    // a fixed order.
    {
        double4_t g00 = {0.0, 0.0, 0.0, 0.0}, g10 = {0.0, 0.0, 0.0, 0.0}, g11 = {0.0, 0.0, 0.0, 0.0};
        const int cols = lp / NW;                  // lp % 32 == 0: cols % 4 == 0
        // A lane reads four consecutive columns of its row, 16 columns per 16 lanes and chunk; k-step
        // u of a chunk contracts over element u of every lane, i.e. over the columns 4 (L/16) + u:
        // both operands are the same rows, so any order of the contraction serves.
        const float* p0 = Xp + (long long)l16 * lp + wv * cols + 4 * lq;
        const float* p1 = Xq + (long long)l16 * lp + wv * cols + 4 * lq;
        const f32x4_t zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int k = 0; k < cols; k += 16) {
            const bool in = k + 4 * lq < cols;
            const f32x4_t x0 = in ? *reinterpret_cast<const f32x4_t*>(p0 + k) : zero4;
            const f32x4_t x1 = in ? *reinterpret_cast<const f32x4_t*>(p1 + k) : zero4;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double a0 = (double)x0[u], a1 = (double)x1[u];
                g00 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, a0, g00, 0, 0, 0);
                g10 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, a0, g10, 0, 0, 0);
                g11 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, a1, g11, 0, 0, 0);
            }
        }
        double* dst = smem + wv * 768;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dst[e * 64 + lane] = g00[e];
            dst[256 + e * 64 + lane] = g10[e];
            dst[512 + e * 64 + lane] = g11[e];
        }
    }
    __syncthreads();
    {
        // the sums wait in registers until every partial has been read, because S overwrites them
        constexpr int PER = 12 / NW;
        double v[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            v[q] = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) v[q] += smem[w * 768 + tid + 64 * NW * q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int idx = tid + 64 * NW * q;
            // element e of lane L is entry (4e + L/16, L%16) of its tile
            const int tile = idx >> 8, e = (idx >> 6) & 3, ln = idx & 63;
            const int ii = 4 * e + (ln >> 4), jj = ln & 15;
            if (tile == 0) {
                smem[ii * kJgLd + jj] = v[q];
            } else if (tile == 1) {
                smem[(16 + ii) * kJgLd + jj] = v[q];
                smem[jj * kJgLd + 16 + ii] = v[q];
            } else {
                smem[(16 + ii) * kJgLd + 16 + jj] = v[q];
            }
        }
    }
    __syncthreads();
    int nrot = 0;
    double* scales = coef + kJgRounds * kJgRoundCoef;
    constexpr bool kSplit = NW == 4;
    if (wv == (sweeper + 1) % NW) {
        SweepVectors<kSplit> v;
        v.init(coef, cross, lane);
        jacobi_rounds(v, cross);
        __syncthreads();
        v.store(smem, scales);
    } else if (kSplit && (wv == sweeper || wv == (sweeper + 2) % NW)) {
        SweepHalf m;
        m.init(smem, coef, smem + 32 * kJgLd, cross, lane, wv == sweeper ? 0 : 1);
        jacobi_rounds(m, cross);
        m.finish(scales);
        nrot = m.nrot;
        __syncthreads();
    } else if (!kSplit) {
        SweepMain m;
        m.init(smem, coef, cross, lane);
        jacobi_rounds(m, cross);
        m.finish(scales);
        nrot = m.nrot;
        __syncthreads();
    } else {
        for (int n = cross ? 17 : kJgRounds + 2; n > 0; --n) sweep_barrier();
        __syncthreads();
    }
    __syncthreads();
    // ---- X <- V X: wavefront wv takes the 16-column tiles wv, wv + NW, ...; both 16-row halves
    double va[2][8];                             // A[L%16][k + L/16] = V[L%16][k + L/16], k = 4u
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        va[0][u] = smem[l16 * kJgLd + 4 * u + lq];
        va[1][u] = smem[(16 + l16) * kJgLd + 4 * u + lq];
    }
    const int nct = lp / 16;
    const unsigned rowoff = (unsigned)lq * (unsigned)lp + (unsigned)l16, lp4 = 4u * (unsigned)lp;
    for (int ct = wv; ct < nct; ct += NW) {
        // B[k + L/16][L%16] = X[k + L/16][c0 + L%16], k = 4u: rows 0..15 from Xp, 16..31 from Xq; element e
        // of a result tile is row 4e + L/16 of its half: the same offsets
        const unsigned base = rowoff + 16u * (unsigned)ct;
        float bx[8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bx[u] = Xp[base + u * lp4];
            bx[4 + u] = Xq[base + u * lp4];
        }
        double4_t o0 = {0.0, 0.0, 0.0, 0.0}, o1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            o0 = __builtin_amdgcn_mfma_f64_16x16x4f64(va[0][u], (double)bx[u], o0, 0, 0, 0);
            o1 = __builtin_amdgcn_mfma_f64_16x16x4f64(va[1][u], (double)bx[u], o1, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            Xp[base + e * lp4] = (float)o0[e];
            Xq[base + e * lp4] = (float)o1[e];
        }
    }
    __syncthreads();
    return nrot;
}

// MatDev::jflag[sweep]: rotations of a sweep that keep the loop alive.  A sweep runs unless the one before it
// had none (a skipped sweep leaves its own count at zero).

// Round `round` of sweep `sweep`: one workgroup per pair of blocks.  Round 0 of a sweep (every block is in
// exactly one pair) rotates all 496 row pairs of a visit; the other rounds only the 256 pairs with one row
// in each block: the pairs inside a block would otherwise be rotated again in each of its nb - 1 visits
// of the sweep.
template <int NW>
__global__ __launch_bounds__(64 * NW, 3) void k_jacobi_round(const MatDev* __restrict__ mats, int n_mats, int pairs, bool local,
                                                             int sweep, int round, int visits, ClearShare share) {
    __shared__ __attribute__((aligned(16))) double smem[jacobi_visit_lds<NW>()];
    if ((int)blockIdx.x >= visits) {
        clear_share(mats, n_mats, share, (int)blockIdx.x - visits);
        return;
    }
    const int seq = (int)(local ? blockIdx.x >> 3 : blockIdx.x);
    const int mat = local ? seq / pairs * 8 + (int)(blockIdx.x & 7) : seq / pairs, pair = seq % pairs;
    if (mat >= n_mats) return;
    const MatDev& md = mats[mat];
    const int lp = md.lp;
    const int nb = lp / 16;
    if (pair >= nb / 2 || round >= nb - 1) return;
    if (sweep > 0 && md.jflag[sweep - 1] == 0) return;
    int bp, bq;
    tournament_pair(nb, round, pair, &bp, &bq);
    const bool cross = round != 0;
    // a block of padding rows only has nothing to rotate (in round 0 its partner still has its own pairs)
    if (cross ? (bp * 16 >= md.l || bq * 16 >= md.l) : (bp * 16 >= md.l && bq * 16 >= md.l)) return;
    // Which wavefront runs the small sweep: those of the workgroups that share a CU (ids 256 apart) are to be on
    // different SIMDs, because one alone fills its SIMD's issue (two on one take twice as long).  For two wavefronts per
    // visit the choice was measured, by visits per CU: the first always with four, else the second in the third of six
    // turns only.  Refresh in us with the first always / the second in the third turn / the second in every other pair of turns:
    //   3 per CU, 84 matrices of order 256 5260 / 5220 / 5222, 160 of 128 1774 / 1762 / 1762
    //   4         112 of 256 5545 / 5734 / 5681, 128 of 256 5744 / 5978 / 5925, 256 of 128 1937 / 2024 / 2012
    //   5         144 of 256 6769 / 6756 / 7043, 96 of 384 18657 / 18534 / 19017
    //   6         168 of 256 6979 / 7004 / 7231, 84 of 512 30669 / 30689 / 30932
    //   8         256 of 256 9962 / 9787 / 9873
    const int turn = (int)(blockIdx.x / 256), per_cu = (visits + 255) / 256;
    const int sweeper = NW == 2 ? per_cu != 4 && turn % 6 == 2 : turn % NW;
    const int nrot = jacobi_visit<NW>(jacobi_rows(md), lp, bp, bq, cross, sweeper, smem);
    if (nrot) atomicAdd(&md.jflag[sweep], nrot);
}

// Sweeps first .. last - 1 of a whole matrix by one workgroup, visit after visit: all of them where a matrix is a
// single pair of blocks, and otherwise what is left after the sweeps that nearly every matrix needs (a
// launch per round costs 2 us also where every matrix has converged).
__global__ __launch_bounds__(256, 2) void k_jacobi_sweeps(const MatDev* __restrict__ mats, int first, int last) {
    __shared__ __attribute__((aligned(16))) double smem[jacobi_visit_lds<4>()];
    __shared__ int total;
    const MatDev& md = mats[blockIdx.x];
    const int lp = md.lp, l = md.l, nb = lp / 16;
    float* X = jacobi_rows(md);
    if (first > 0 && md.jflag[first - 1] == 0) return;
    for (int sweep = first; sweep < last; ++sweep) {
        if (threadIdx.x == 0) total = 0;
        __syncthreads();
        for (int round = 0; round < nb - 1; ++round)
            for (int pair = 0; pair < nb / 2; ++pair) {
                int bp, bq;
                tournament_pair(nb, round, pair, &bp, &bq);
                const bool cross = round != 0;
                if (cross ? (bp * 16 >= l || bq * 16 >= l) : (bp * 16 >= l && bq * 16 >= l)) continue;
                const int nrot = jacobi_visit<4>(X, lp, bp, bq, cross, 0, smem);
                if (nrot) atomicAdd(&total, nrot);
            }
        __syncthreads();
        const int n = total;
        __syncthreads();
        if (threadIdx.x == 0) md.jflag[sweep] = n;
        if (n == 0) break;
    }
}

hipError_t launch_jacobi(const MatDev* mats, int n_mats, int max_pairs, int sweeps, ClearShare clear, bool* cleared, hipStream_t stream) {
    if (max_pairs < 1) max_pairs = 1;
    int done = 0;
    *cleared = false;
    if (max_pairs > 1) {
        // Sweeps needed, the last one without a rotation included, with 0 to 2 power passes on noise, signals of half and
        // of the full rank over floors of 1e-2 and 1e-4, graded and clustered columns, a single spike: at most 8 up
        // to order 128, 9 from 192 to 320.  A serial sweep is 120 visits of 14 us at order 256, 1.7 ms, and grows
        // with the square of the order: one refresh in a few pays one there (noise 3.2 -> 4.9 ms), where one more
        // launched sweep would cost every refresh 15 empty launches of 2 us.
        done = max_pairs > 32 ? sweeps : max_pairs > 8 ? 14 : 8;
        if (done > sweeps) done = sweeps;
        // Workgroup ids go round-robin over the 8 XCDs.  All visits of a matrix on one XCD find its rows in that L2 (rows
        // change blocks every round); where that would load the XCDs unevenly beyond one visit per CU, they are spread.
        const int turns = (n_mats + 7) / 8;
        const bool local = turns * max_pairs <= 32 || turns * 8 <= n_mats + n_mats / 4;
        const int visits = max_pairs * (local ? 8 * turns : n_mats);
        // Four wavefronts per visit where the visits leave CUs to spare (the products of a visit in half the
        // time), two otherwise (twice the visits per CU).
        const bool few = (long long)max_pairs * n_mats <= 512;
        // The clearing, if there is some to do, goes beside the rounds of the first four sweeps, which nearly every matrix
        // needs, in the places that the visits leave on the chip.
        const int places = few ? 3 * 256 : 6 * 256, idle = (places - visits % places) % places;
        const bool wanted = clear.parts > 0 && idle >= 64;
        clear.parts = (done < 4 ? done : 4) * (2 * max_pairs - 1);
        clear.blocks = wanted ? clear_blocks(clear.units * 16 / (unsigned)clear.parts, kClearRound, idle < 256 ? idle : 256) : 0;
        *cleared = clear.blocks > 0;
        for (int sw = 0; sw < done; ++sw)
            for (int round = 0; round < 2 * max_pairs - 1; ++round) {
                clear.part = sw * (2 * max_pairs - 1) + round;
                const dim3 g(visits + (clear.part < clear.parts ? clear.blocks : 0));
                if (few) hipLaunchKernelGGL(k_jacobi_round<4>, g, dim3(256), 0, stream, mats, n_mats, max_pairs, local, sw, round, visits, clear);
                else hipLaunchKernelGGL(k_jacobi_round<2>, g, dim3(128), 0, stream, mats, n_mats, max_pairs, local, sw, round, visits, clear);
            }
    }
    if (done < sweeps) hipLaunchKernelGGL(k_jacobi_sweeps, dim3(n_mats), dim3(256), 0, stream, mats, done, sweeps);
    return hipGetLastError();
}

// Ritz values (row norms), descending order, then the l x r rotation U[:, top r] as floats in Bm.
// (sixteen wavefronts, four rows each in flight: with four wavefronts a row at a time 112 us for 168 matrices of
// order 256, with sixteen 38; a chain of memory latencies, so a row's loads go out together and the values are compared in LDS)
constexpr int kSortThreads = 1024;
__global__ __launch_bounds__(kSortThreads) void k_ritz_sort(const MatDev* __restrict__ mats, int sweeps, int* status) {
    __shared__ double vals[kSortThreads];
    const MatDev& md = mats[blockIdx.x];
    const int lp = md.lp;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int i = 4 * wv; i < lp; i += 4 * (kSortThreads / 64)) {      // lp % 32 == 0
        const float* __restrict__ row = jacobi_rows(md) + (long long)i * lp;
        double a[4] = {0.0, 0.0, 0.0, 0.0};
        for (int c = lane; c < lp; c += 256) {
            float x[4][4];
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int u = 0; u < 4; ++u) x[h][u] = row[(long long)u * lp + (c + 64 * h < lp ? c + 64 * h : lane)];
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double y = c + 64 * h < lp ? (double)x[h][u] : 0.0;
                    a[u] += y * y;
                }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double v = ritz_value(wave_sum_d(a[u]));
            if (lane == 0) {
                md.ritz[i + u] = v;
                if (lp <= kSortThreads) vals[i + u] = v;
            }
        }
    }
    __syncthreads();
    __threadfence_block();
    bool bad = false;
    if (lp <= kSortThreads) {
        // as many lanes per value as the workgroup has (a power of two), each compares it with its share of the others
        int per = 1;
        while (2 * per * lp <= kSortThreads && per < 64) per *= 2;
        const int i = threadIdx.x / per, sub = threadIdx.x & (per - 1);
        if (i < lp) {
            int place = ritz_place(vals, lp, i, sub, per);
            for (int off = 1; off < per; off *= 2) place += __shfl_xor(place, off, 64);
            if (sub == 0) {
                md.order[place] = i;
                if (place < md.r && !(vals[i] > 0.0)) bad = true;
            }
        }
    } else {
        for (int i = threadIdx.x; i < lp; i += kSortThreads) {
            const int place = ritz_place(md.ritz, lp, i);
            md.order[place] = i;
            if (place < md.r && !(md.ritz[i] > 0.0)) bad = true;
        }
    }
    if (bad) atomicOr(status, 8);
    // no sweep without a rotation was seen before the sweep limit
    if (threadIdx.x == 0 && md.jflag[sweeps - 1] != 0) atomicOr(status, kStatusNotConverged);
}

__global__ __launch_bounds__(256) void k_build_rotation(const MatDev* __restrict__ mats) {
    const MatDev& md = mats[blockIdx.y];
    const int l = md.l, r = md.r, lp = md.lp;
    const long long total = (long long)l * r;
    for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < total; q += (long long)gridDim.x * 256) {
        const int k = (int)(q / r), j = (int)(q % r);
        const int src = md.order[j];
        const double nrm = md.ritz[src];
        md.Bm[q] = nrm > 0.0 ? (float)((double)jacobi_rows(md)[(long long)src * lp + k] / nrm) : 0.f;
    }
}

hipError_t launch_jacobi_finish(const MatDev* mats, int n_mats, int sweeps, int* status, hipStream_t stream) {
    hipLaunchKernelGGL(k_ritz_sort, dim3(n_mats), dim3(kSortThreads), 0, stream, mats, sweeps, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_build_rotation, dim3(128, n_mats), dim3(256), 0, stream, mats);
    return hipGetLastError();
}

// ------------------------------------------------------------------ sign convention, copy into P
// Source: Ya viewed as [m][r].  Each column is multiplied by the sign of its entry of largest
// magnitude (first one on ties) and written to P.
// A workgroup takes 32 columns; 32 threads share a column, each with eight rows in flight.  (Four threads per
// column and one row at a time: 540 us for 168 projectors of 1024 x 256, 23 us for one of 256 x 32.)
//
// COPIES: the bf16 copies of P as well (layouts: k_make_bf16_copies), whose blocks of 32 are this workgroup's columns: P is not read
// again, and the copies go out 16 bytes per thread.
constexpr int kSignRows = 32;
template <bool COPIES>
__global__ __launch_bounds__(32 * kSignRows) void k_sign_fix(const MatDev* __restrict__ mats) {
    __shared__ float best[kSignRows][33];
    __shared__ int besti[kSignRows][33];
    __shared__ float tile[8][32][33];        // (COPIES)
    const MatDev& md = mats[blockIdx.y];
    const int r = md.r, m = md.m;
    const int tc = threadIdx.x & 31, rg = threadIdx.x >> 5;
    const int c = blockIdx.x * 32 + tc;
    if (blockIdx.x * 32 >= r) return;
    const float* __restrict__ src = md.Ya;
    float bv = -1.f;
    int bi = 0;
    if (c < r)
        for (int i = rg; i < m; i += 8 * kSignRows) {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = src[(long long)(i + u * kSignRows < m ? i + u * kSignRows : i) * r + c];
#pragma unroll
            for (int u = 0; u < 8; ++u) {       // (ascending rows: the first one on ties)
                const float x = fabsf(a[u]);
                if (i + u * kSignRows < m && x > bv) {
                    bv = x;
                    bi = i + u * kSignRows;
                }
            }
        }
    best[rg][tc] = bv;
    besti[rg][tc] = bi;
    __syncthreads();
    if (!COPIES && c >= r) return;
    const int cs = c < r ? c : r - 1;
    float v = best[0][tc];
    int idx = besti[0][tc];
    for (int g = 1; g < kSignRows; ++g) {
        const float v2 = best[g][tc];
        const int i2 = besti[g][tc];
        if (v2 > v || (v2 == v && i2 < idx)) { v = v2; idx = i2; }
    }
    const float sgn = src[(long long)idx * r + cs] < 0.f ? -1.f : 1.f;
    if constexpr (!COPIES) {
        for (int i = rg; i < m; i += 8 * kSignRows) {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = src[(long long)(i + u * kSignRows < m ? i + u * kSignRows : i) * r + c];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i + u * kSignRows < m) md.P[(long long)(i + u * kSignRows) * r + c] = sgn * a[u];
        }
    } else {
        for (int i0 = 0; i0 < m; i0 += 8 * kSignRows) {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + rg + u * kSignRows;
                a[u] = src[(long long)(i < m ? i : m - 1) * r + cs];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + rg + u * kSignRows;
                const bool in = i < m && c < r;
                const float x = sgn * a[u];
                if (in) md.P[(long long)i * r + c] = x;
                tile[u][rg][tc] = in ? x : 0.f;
            }
            __syncthreads();
            const int q = threadIdx.x >> 7, x = (threadIdx.x & 127) >> 2, o = 8 * (threadIdx.x & 3);
            const int ib = i0 + 32 * q, rho = blockIdx.x * 32 + x;
            if (ib + x < m) {
                u32x4_t w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(tile[q][x][o + 2 * e], tile[q][x][o + 2 * e + 1]);
                *reinterpret_cast<u32x4_t*>(md.Pb + ((long long)blockIdx.x * m + ib + x) * 32 + o) = w;
            }
            if (ib < m && rho < r) {
                u32x4_t w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(tile[q][o + 2 * e][x], tile[q][o + 2 * e + 1][x]);
                *reinterpret_cast<u32x4_t*>(md.PbT + ((long long)(ib >> 5) * r + rho) * 32 + o) = w;
            }
            __syncthreads();
        }
    }
}

// The copies beside the signs save a launch and a pass over P, but a workgroup goes down all rows of its columns, 256 at a time,
// where a launch of their own has a workgroup per 32.  Refreshes with the copies apart and beside, all else equal (us; runs of one
// side differ by 1 or 2 in a thousand):
//   few workgroups: 256 x 512 at rank 32 (1) 263.8 -> 261.2, 512 x 512 304.2 -> 303.3, 768 x 512 342.0 -> 342.2, 1024 x 512 378.9 -> 381.0,
//     2048 x 1024 at rank 64 (2) 720.4 -> 725.8, 16000 x 512 1778 -> 1853
//   32 of 1024 x 512 at rank 64 (64) 699.8 -> 700.5, 32 of 2048 x 512 (64) 840.2 -> 838.6, 72 of up to 3072 rows at rank 8 (72) 855.1 -> 861.7
//   32 of 2048 x 512 at rank 128 (128) 1602 -> 1598, 4096 x 512 2062 -> 2048, 8192 x 512 2990 -> 2957, 16 of 16000 x 512 at rank 256 (128)
//     7682 -> 7597, 60M set (224) 1615 -> 1610, 350M set (1344) 12.21 -> 12.16 ms
bool sign_fix_copies(int n_mats, int max_m, int max_r) {
    return max_m <= 512 || (long long)((max_r + 31) / 32) * n_mats >= 128;
}

hipError_t launch_sign_fix(const MatDev* mats, int n_mats, int max_r, bool copies, hipStream_t stream) {
    const dim3 grid((max_r + 31) / 32, n_mats), block(32 * kSignRows);
    if (copies) hipLaunchKernelGGL(k_sign_fix<true>, grid, block, 0, stream, mats);
    else hipLaunchKernelGGL(k_sign_fix<false>, grid, block, 0, stream, mats);
    return hipGetLastError();
}

}  // namespace ng
