// Grouped fp32 GEMM on the fp32 MFMA (v_mfma_f32_32x32x2_f32), one launch for
// all matrices of the layer set.  It serves the NG_F32 step (projection
// R = P^T G, paper Sec. 1; update W -= lr (scale P N + wd W), paper Sec. 2.2)
// and every dense product of the projector refresh.  Operands are described as
// strided views A(i,k), B(k,j) so one kernel covers all transpositions; an
// operand may be stored as float or bf16 (gradients).
//
// Tile 128 x 128 per workgroup (4 wavefronts of 64 x 64), BK = 16, two LDS tile buffers (one barrier
// per k-step) and two register sets (a tile's loads are issued two k-steps ahead).
// MFMA 32x32x2 f32 operand layout: lane L supplies A[i = L%32][k = L/32] and
// B[k = L/32][j = L%32]; the 16 accumulators of lane L are
// D[8*g + 4*(L/32) + e][L%32], index 4*g + e.
#include "ng_internal.h"

namespace ng {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

enum { EPI_F32 = 0, EPI_W_F32 = 1 };

struct GemmView {
    const void* A;
    const void* B;
    void* C;
    long long sAi, sAk, sBk, sBj, ldc;     // C is always row-major with leading dimension ldc
    int M, N, K;      // C is M x N, contraction length K
    int Nvalid;       // columns j >= Nvalid of B read as zero (padding columns of the r x ldn space)
    int a_bf16, b_bf16;
    int epi;
    int b_tri;        // B(k, j) = 0 for k > j (the transposed inverse Cholesky factor): a tile stops at its last column
    int sym;          // C = X^T X: only tiles on or below the diagonal are computed, as partial planes (see sym_planes)
};

__host__ __device__ inline GemmView gemm_view(int op, const MatDev& md, const MatDyn* dy, int grad_dtype,
                                              int slot = 0, int hist_bf16 = 0) {
    GemmView v;
    v.a_bf16 = 0;
    v.b_bf16 = 0;
    v.epi = EPI_F32;
    v.b_tri = 0;
    v.sym = 0;
    const int gb = (grad_dtype == NG_BF16) ? 1 : 0;
    const void* G = dy ? dy->g : nullptr;
    // Strides of the m x n matrix the kernels see inside the caller's row-major gradient: for the
    // right side that matrix is the transpose of the caller's.
    const bool right = md.side == NG_SIDE_RIGHT;
    const long long g_row = right ? 1 : md.ld_g, g_col = right ? md.ld_g : 1;
    switch (op) {
        case OP_PROJECT_F32:
            v.A = md.P; v.sAi = 1; v.sAk = md.r;
            v.B = G; v.sBk = g_row; v.sBj = g_col; v.b_bf16 = gb;
            v.M = md.r; v.N = md.ldn; v.Nvalid = md.n; v.K = md.m;
            v.C = md.H + (long long)(dy ? dy->head : 0) * md.slot_elems; v.ldc = md.ldn;
            break;
        case OP_UPDATE_F32:
            if (!right) {       // W (m x n) -= P N
                v.A = md.P; v.sAi = md.r; v.sAk = 1;
                v.B = md.N; v.sBk = md.ldn; v.sBj = 1;
                v.M = md.m; v.N = md.n; v.Nvalid = md.n;
            } else {            // the caller's W is n x m here: W -= N^T P^T, in W's own orientation
                v.A = md.N; v.sAi = 1; v.sAk = md.ldn;
                v.B = md.P; v.sBk = 1; v.sBj = md.r;
                v.M = md.n; v.N = md.m; v.Nvalid = md.m;
            }
            v.K = md.r;
            v.C = dy ? dy->w : nullptr; v.ldc = md.ld_w; v.epi = EPI_W_F32;
            break;
        case OP_G_B2A:
        case OP_G_C2A:
            v.A = G; v.sAi = g_row; v.sAk = g_col; v.a_bf16 = gb;
            v.B = (op == OP_G_B2A) ? md.Yb : md.Yc; v.sBk = md.l; v.sBj = 1;
            v.M = md.m; v.N = md.l; v.Nvalid = md.l; v.K = md.n;
            v.C = md.Ya; v.ldc = md.l;
            break;
        case OP_GT_C2B:
            v.A = G; v.sAi = g_col; v.sAk = g_row; v.a_bf16 = gb;
            v.B = md.Yc; v.sBk = md.l; v.sBj = 1;
            v.M = md.n; v.N = md.l; v.Nvalid = md.l; v.K = md.m;
            v.C = md.Yb; v.ldc = md.l;
            break;
        case OP_GRAM_A:
        case OP_GRAM_B:
        case OP_GRAM_CA:
        case OP_GRAM_CB: {
            const float* Y = (op == OP_GRAM_A) ? md.Ya : (op == OP_GRAM_B) ? md.Yb : md.Yc;
            v.A = Y; v.sAi = 1; v.sAk = md.l;
            v.B = Y; v.sBk = md.l; v.sBj = 1;
            v.M = md.l; v.N = md.l; v.Nvalid = md.l;
            v.K = (op == OP_GRAM_A || op == OP_GRAM_CA) ? md.m : md.n;
            v.C = nullptr; v.ldc = md.l; v.sym = 1;   // C: the planes
            break;
        }
        case OP_APPLY_A2C:
        case OP_APPLY_B2C:
        case OP_APPLY_C2A:
        case OP_APPLY_C2B: {
            const bool rows_m = (op == OP_APPLY_A2C || op == OP_APPLY_C2A);
            v.A = (op == OP_APPLY_A2C) ? md.Ya : (op == OP_APPLY_B2C) ? md.Yb : md.Yc;
            v.sAi = md.l; v.sAk = 1;
            v.B = md.Linv; v.sBk = 1; v.sBj = md.lp;          // B(k, j) = Linv[j][k]
            v.M = rows_m ? md.m : md.n; v.N = md.l; v.Nvalid = md.l; v.K = md.l;
            v.C = (op == OP_APPLY_C2A) ? md.Ya : (op == OP_APPLY_C2B) ? md.Yb : md.Yc;
            v.ldc = md.l; v.b_tri = 1;
            break;
        }
        case OP_QT_G:
            v.A = md.Ya; v.sAi = 1; v.sAk = md.l;
            v.B = G; v.sBk = g_row; v.sBj = g_col; v.b_bf16 = gb;
            v.M = md.l; v.N = md.ldn; v.Nvalid = md.n; v.K = md.m;
            v.C = md.Bm; v.ldc = md.ldn;
            break;
        case OP_B_BT:
            v.A = md.Bm; v.sAi = md.ldn; v.sAk = 1;
            v.B = md.Bm; v.sBk = 1; v.sBj = md.ldn;
            v.M = md.l; v.N = md.l; v.Nvalid = md.l; v.K = md.n;
            v.C = nullptr; v.ldc = md.l; v.sym = 1;
            break;
        case OP_ROTATE:   // P = Ya * Urot, Urot (l x r, float) staged in Bm
            v.A = md.Ya; v.sAi = md.l; v.sAk = 1;
            v.B = md.Bm; v.sBk = md.r; v.sBj = 1;
            v.M = md.m; v.N = md.r; v.Nvalid = md.r; v.K = md.l;
            v.C = md.P; v.ldc = md.r;
            break;
        case OP_GRAM_P:
            v.A = md.P; v.sAi = 1; v.sAk = md.r;
            v.B = md.P; v.sBk = md.r; v.sBj = 1;
            v.M = md.r; v.N = md.r; v.Nvalid = md.r; v.K = md.m;
            v.C = nullptr; v.ldc = md.r; v.sym = 1;
            break;
        case OP_T_CARRY:   // change of basis T = P_new^T P_old, P_old saved in Yc
            v.A = md.P; v.sAi = 1; v.sAk = md.r;
            v.B = md.Yc; v.sBk = md.r; v.sBj = 1;
            v.M = md.r; v.N = md.r; v.Nvalid = md.r; v.K = md.m;
            v.C = md.Linv; v.ldc = md.lp;
            break;
        case OP_CARRY_SLOT:   // carry = T H[slot]
            v.A = md.Linv; v.sAi = md.lp; v.sAk = 1;
            if (hist_bf16) v.B = reinterpret_cast<const unsigned short*>(md.H) + (long long)slot * md.slot_elems;
            else v.B = md.H + (long long)slot * md.slot_elems;
            v.b_bf16 = hist_bf16;
            v.sBk = md.ldn; v.sBj = 1;
            v.M = md.r; v.N = md.ldn; v.Nvalid = md.ldn; v.K = md.r;
            v.C = md.carry; v.ldc = md.ldn;
            break;
        case OP_APPLY_P2A:
        default:
            v.A = md.P; v.sAi = md.r; v.sAk = 1;
            v.B = md.Linv; v.sBk = 1; v.sBj = md.lp;
            v.M = md.m; v.N = md.r; v.Nvalid = md.r; v.K = md.r;
            v.C = md.Ya; v.ldc = md.r; v.b_tri = 1;
            break;
    }
    return v;
}

void gemm_f32_dims(int op, const MatDev& md, int* M, int* N, int* K) {
    GemmView v = gemm_view(op, md, nullptr, NG_F32);
    *M = v.M;
    *N = v.N;
    *K = v.K;
}

#define NG_AS1 __attribute__((address_space(1)))
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef f32x4_t __attribute__((aligned(4))) f32x4_a4;          // 16-byte access at 4-byte alignment
typedef unsigned short u16x4_t __attribute__((ext_vector_type(4)));
typedef u16x4_t __attribute__((aligned(2))) u16x4_a2;          // 8-byte access at 2-byte alignment

// Element idx of an operand (float or bf16), as a float.
template <bool BF>
__device__ __forceinline__ float load1(const NG_AS1 unsigned char* p, long long idx) {
    if (BF) return __uint_as_float((unsigned int)reinterpret_cast<const NG_AS1 unsigned short*>(p)[idx] << 16);
    return reinterpret_cast<const NG_AS1 float*>(p)[idx];
}

// Four consecutive operand elements from a byte address, as floats.
template <bool BF>
__device__ __forceinline__ f32x4_t load4(const NG_AS1 unsigned char* p) {
    if (BF) {
        const u16x4_t u = *reinterpret_cast<const NG_AS1 u16x4_a2*>(p);
        f32x4_t o;
        o.x = __uint_as_float((unsigned int)u.x << 16);
        o.y = __uint_as_float((unsigned int)u.y << 16);
        o.z = __uint_as_float((unsigned int)u.z << 16);
        o.w = __uint_as_float((unsigned int)u.w << 16);
        return o;
    }
    return *reinterpret_cast<const NG_AS1 f32x4_a4*>(p);
}

// One operand of a tile: T (tile index) x K (contraction), TS x BK per k-step, moved as vectors of four
// elements along the stride-1 dimension -- the tile index (TF) or the contraction.  tile-fast: positions
// 4 (t % (TS/4)) of the tile index at k = t / (TS/4) + (1024/TS) q; k-fast: k = 4 (t % (BK/4)) at tile
// index t / (BK/4) + (1024/BK) q.
template <int TS, int BK, bool TF, bool BF>
struct F32Src {
    static constexpr int NV = TS * BK / 1024, LDT = TS + 4, ES = BF ? 2 : 4, KT = BK / 4, TQ = 1024 / BK;
    const NG_AS1 unsigned char* base;   // element (0, 0)
    const NG_AS1 unsigned char* safe;   // 16 readable bytes
    const NG_AS1 unsigned char* ptr[NV];
    long long st, sk;                   // element strides along T and K
    int t0, k0, lim, K;                 // this thread's first position, valid tile indexes, contraction length
    __device__ __forceinline__ void init(const void* p, const void* safe_, long long st_, long long sk_, int tile0,
                                         int lim_, int K_, int t) {
        base = (const NG_AS1 unsigned char*)p;
        safe = (const NG_AS1 unsigned char*)safe_;
        st = st_;
        sk = sk_;
        lim = lim_;
        K = K_;
        t0 = tile0 + (TF ? 4 * (t % (TS / 4)) : t / KT);
        k0 = TF ? t / (TS / 4) : 4 * (t % KT);
#pragma unroll
        for (int q = 0; q < NV; ++q)
            ptr[q] = base + (TF ? (long long)t0 + (long long)(k0 + (1024 / TS) * q) * sk
                                : (long long)(t0 + TQ * q) * st + k0) * ES;
    }
    // k-step kt, wholly inside the operand
    __device__ __forceinline__ void fetch(int kt, f32x4_t (&r)[NV]) const {
        const long long off = (TF ? (long long)BK * sk : (long long)BK) * ES * kt;
#pragma unroll
        for (int q = 0; q < NV; ++q) r[q] = load4<BF>(ptr[q] + off);
    }
    // k-step kt at the operand's edge, zero outside: whole vectors from clamped addresses; the lanes whose vector
    // straddles the edge (only where the edge is not a multiple of four) read theirs element by element
    __device__ __forceinline__ void fetch_edge(int kt, f32x4_t (&r)[NV]) const {
        const bool straddles = ((TF ? lim : K) & 3) != 0;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int i = TF ? t0 : t0 + TQ * q;
            const int k = kt * BK + (TF ? k0 + (1024 / TS) * q : k0);
            const bool in = i < lim && k < K;
            const bool all = in && (TF ? i + 4 <= lim : k + 4 <= K);
            const f32x4_t v = load4<BF>(all ? base + ((long long)i * st + (long long)k * sk) * ES : safe);
#pragma unroll
            for (int x = 0; x < 4; ++x) r[q][x] = all ? v[x] : 0.f;
            if (straddles && in && !all) {
#pragma unroll
                for (int x = 0; x < 3; ++x)
                    if ((TF ? i : k) + x < (TF ? lim : K)) r[q][x] = load1<BF>(base, (long long)i * st + (long long)k * sk + x);
            }
        }
    }
    __device__ __forceinline__ void stage(const f32x4_t (&r)[NV], float (*S)[LDT], int t) const {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            if (TF) {
                *reinterpret_cast<f32x4_t*>(&S[t / (TS / 4) + (1024 / TS) * q][4 * (t % (TS / 4))]) = r[q];
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x) S[4 * (t % KT) + x][t / KT + TQ * q] = r[q][x];
            }
        }
    }
};

// Tile TS x TS per workgroup (128: four wavefronts of 64 x 64 = 2 x 2 MFMA blocks of 32 x 32; 64: one
// block per wavefront, for products with a short side, a short contraction or few tiles).  BK = 16 (32 with the
// small tile: half the barriers, but three mid-size matrices' step 73.8 -> 78.4 us).
// AI / BJ: the tile index is operand A's / B's stride-1 dimension (else the contraction is); ABF / BBF:
// operand A / B is stored as bf16; SYM: a symmetric product (partial planes).  side >= 0: only matrices
// of that side.  A tile whose rows and columns all exist takes whole vectors without a test (only a
// last partial k-step is read element by element); with the tests of every vector, and of every MFMA
// block against the product's edge, in the loop the products ran at a quarter of the fp32 MFMA rate.
template <int TS>
struct F32Tiles {
    static constexpr int BK = kSymStep, LDT = TS + 4;
    float a[2][BK][LDT], b[2][BK][LDT];   // two tile buffers: one barrier per k-step
};

template <int TS, bool AI, bool BJ, bool ABF, bool BBF, bool SYM>
__device__ __forceinline__ void gemm_f32_tile(int op, const MatDev* __restrict__ mats, const MatDyn* __restrict__ dyn,
                                              int grad_dtype, const StepScalars& sc, const SymPlanes* __restrict__ sym,
                                              F32Tiles<TS>& lds) {
    constexpr int BK = F32Tiles<TS>::BK, LDT = F32Tiles<TS>::LDT;
    constexpr int NB = TS / 64;          // 32 x 32 blocks per wavefront and dimension
    typedef F32Src<TS, BK, AI, ABF> SA;
    typedef F32Src<TS, BK, BJ, BBF> SB;
    constexpr int NV = SA::NV;
    const MatDev& md = mats[blockIdx.z];
    GemmView v = gemm_view(op, md, &dyn[blockIdx.z], grad_dtype, sc.slot, sc.hist_bf16);
    // The grid is 1-D over the tiles of the largest matrix, padded to a multiple of 8: hardware workgroup
    // id w runs on XCD w % 8, and the eight XCDs each work through a contiguous run of this matrix's
    // tiles (the column tiles of one row tile share the rows of A through that XCD's L2).  Which XCD takes
    // the first run turns with the matrix: a matrix of few tiles fills the first runs only, and with the
    // first always on XCD 0 most of the chip idled (56 products of one 128 x 128 tile in two halves: all
    // on two XCDs, 106 us).
    const int nxm = (v.N + TS - 1) / TS, nym = (v.M + TS - 1) / TS;   // this matrix's own tiles
    // symmetric results: nym (nym + 1) / 2 tiles, one work item each per plane
    SymPlanes sp{nullptr, 0, 1, 0};
    if (SYM) sp = sym[blockIdx.z];
    // the projection of a small layer set is cut along the contraction as well
    const bool split = !SYM && op == OP_PROJECT_F32 && md.proj_chunks > 0;
    if (split)
        sp = SymPlanes{step_scratch<float>(dyn, md.proj_parts_off), 0, md.proj_chunks, (long long)md.proj_rows * md.ldn};
    const int items = (SYM ? nym * (nym + 1) / 2 : nxm * nym) * sp.count;
    const int per = (items + 7) / 8;
    const int slot = (int)(blockIdx.x / 8);
    const int runs = (items + per - 1) / per;    // runs that hold any tile
    const int run = (int)((blockIdx.x + blockIdx.z * (unsigned)runs) % 8);
    int tile = run * per + slot;
    if (slot >= per || tile >= items) return;
    int i0, j0;
    if (SYM || split) {
        const int plane = tile % sp.count;
        tile /= sp.count;
        // this plane's run of the contraction (an empty one leaves zeros)
        const int kc = ((v.K + sp.count - 1) / sp.count + BK - 1) / BK * BK;
        const int k0 = plane * kc < v.K ? plane * kc : v.K;
        v.A = (const unsigned char*)v.A + (long long)k0 * v.sAk * (ABF ? 2 : 4);
        v.B = (const unsigned char*)v.B + (long long)k0 * v.sBk * (BBF ? 2 : 4);
        v.K = v.K - k0 < kc ? v.K - k0 : kc;
        v.C = sp.p + plane * sp.pitch;
    }
    if (SYM) {
        int ti = 0;
        while (tile >= ti + 1) {      // row ti of the triangle holds ti + 1 tiles
            tile -= ti + 1;
            ++ti;
        }
        i0 = ti * TS;
        j0 = tile * TS;
    } else {
        i0 = (tile / nxm) * TS;
        j0 = (tile % nxm) * TS;
    }
    if (v.b_tri && j0 + TS < v.K) v.K = j0 + TS;   // rows k > j of B are zero

    const int t = threadIdx.x;
    const int lane = t & 63, wv = t >> 6;
    const int wm = wv >> 1, wn = wv & 1;
    const int li = lane & 31, h = lane >> 5;

    floatx16 acc[NB][NB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[a][b][x] = 0.f;

    SA sa;
    SB sb;
    sa.init(v.A, mats, v.sAi, v.sAk, i0, v.M, v.K, t);
    sb.init(v.B, mats, v.sBj, v.sBk, j0, v.Nvalid, v.K, t);

    auto multiply = [&](int buf) {
        const float (*As)[LDT] = lds.a[buf];
        const float (*Bs)[LDT] = lds.b[buf];
#pragma unroll
        for (int kk = 0; kk < BK; kk += 2) {
            float a[NB], b[NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                a[x] = As[kk + h][wm * (TS / 2) + 32 * x + li];
                b[x] = Bs[kk + h][wn * (TS / 2) + 32 * x + li];
            }
#pragma unroll
            for (int x = 0; x < NB; ++x)
#pragma unroll
                for (int y = 0; y < NB; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[x], b[y], acc[x][y], 0, 0, 0);
        }
    };

    // Two register sets: a tile's loads are issued two k-steps before it is written to LDS (one step
    // ahead is not enough for operands that stream from HBM).  Iteration kt: tile kt + 1 goes from its
    // register set into the LDS buffer that tile kt - 1 was read from (everyone has passed the barrier that
    // ended that step), the set is refilled with the loads of tile kt + 3, tile kt is multiplied, one barrier.
    // (an odd number of k-steps gets one of zeros: leaving the loop in its middle would cost a second set of accumulators)
    const int nk = (v.K + 2 * BK - 1) / (2 * BK) * 2;
    // k-steps that each operand reads as whole vectors: an edge of one does not put the other on the clamped path
    // (fp32 steps, two 1168-wide blocks at rank 292: 1055 -> 963 us; four 1000-wide ones at rank 500: 1731 -> 1604)
    const int wholea = i0 + TS <= v.M ? v.K / BK : 0, wholeb = j0 + TS <= v.Nvalid ? v.K / BK : 0;
    f32x4_t ra0[NV], rb0[NV], ra1[NV], rb1[NV];
    auto fetch = [&](int kt, f32x4_t (&ra)[NV], f32x4_t (&rb)[NV]) {
        if (kt >= nk) return;
        if (kt < wholea) sa.fetch(kt, ra);
        else sa.fetch_edge(kt, ra);
        if (kt < wholeb) sb.fetch(kt, rb);
        else sb.fetch_edge(kt, rb);
    };
    auto stage = [&](const f32x4_t (&ra)[NV], const f32x4_t (&rb)[NV], int buf) {
        sa.stage(ra, lds.a[buf], t);
        sb.stage(rb, lds.b[buf], t);
    };
    if (nk > 0) {
        fetch(0, ra0, rb0);
        fetch(1, ra1, rb1);
        stage(ra0, rb0, 0);
        fetch(2, ra0, rb0);
        __syncthreads();
        for (int kt = 0; kt < nk; kt += 2) {
            stage(ra1, rb1, 1);
            fetch(kt + 3, ra1, rb1);
            multiply(0);
            __syncthreads();
            if (kt + 2 < nk) stage(ra0, rb0, 0);
            fetch(kt + 4, ra0, rb0);
            multiply(1);
            __syncthreads();
        }
    }

    const bool whole = i0 + TS <= v.M && j0 + TS <= v.N;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj) {
            const int col = j0 + wn * (TS / 2) + bj * 32 + li;
            const int row0 = i0 + wm * (TS / 2) + bi * 32 + 4 * h;
            NG_AS1 float* C = (NG_AS1 float*)v.C + (long long)row0 * v.ldc + col;
            if (v.epi == EPI_W_F32) {
                float w[16];
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int dr = 8 * (x >> 2) + (x & 3);
                    const bool in = whole || (row0 + dr < v.M && col < v.N);
                    w[x] = in ? C[dr * v.ldc] : 0.f;
                }
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int dr = 8 * (x >> 2) + (x & 3);
                    if (whole || (row0 + dr < v.M && col < v.N))
                        C[dr * v.ldc] = w[x] - (sc.lr_scale * acc[bi][bj][x] + sc.lr_wd * w[x]);
                }
            } else if (whole) {
#pragma unroll
                for (int x = 0; x < 16; ++x) C[(8 * (x >> 2) + (x & 3)) * v.ldc] = acc[bi][bj][x];
            } else {
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int dr = 8 * (x >> 2) + (x & 3);
                    if (row0 + dr < v.M && col < v.N) C[dr * v.ldc] = acc[bi][bj][x];
                }
            }
        }
}

template <int TS, bool AI, bool BJ, bool ABF, bool BBF, bool SYM>
__global__ __launch_bounds__(256, TS == 128 ? 3 : 6) void k_gemm_f32(int op, const MatDev* __restrict__ mats,
                                                  const MatDyn* __restrict__ dyn, int grad_dtype,
                                                  StepScalars sc, const SymPlanes* __restrict__ sym, int side) {
    __shared__ __attribute__((aligned(16))) F32Tiles<TS> lds;
    if (side >= 0 && mats[blockIdx.z].side != side) return;
    gemm_f32_tile<TS, AI, BJ, ABF, BBF, SYM>(op, mats, dyn, grad_dtype, sc, sym, lds);
}

// fp32 layer sets with both sides: AL / BL are a left-side matrix's layouts, AR / BR a right-side one's.  A launch
// per side has two ends at which the chip runs empty, the second for the few matrices of one side (four blocks
// of width 450 at rank 56, 24 left and 4 right: step 138.8 -> 114.9 us).
template <int TS, bool AL, bool BL, bool AR, bool BR>
__global__ __launch_bounds__(256, TS == 128 ? 3 : 6) void k_gemm_f32_sides(int op, const MatDev* __restrict__ mats,
                                                  const MatDyn* __restrict__ dyn, StepScalars sc) {
    __shared__ __attribute__((aligned(16))) F32Tiles<TS> lds;
    if (mats[blockIdx.z].side == NG_SIDE_RIGHT)
        gemm_f32_tile<TS, AR, BR, false, false, false>(op, mats, dyn, NG_F32, sc, nullptr, lds);
    else
        gemm_f32_tile<TS, AL, BL, false, false, false>(op, mats, dyn, NG_F32, sc, nullptr, lds);
}

// max_m, max_n, max_k: the largest dimensions of this product over the layer set.  The 128 tile is used
// when neither side nor the contraction is short (a short side wastes most of a big tile, a short
// contraction leaves only the read-modify-write of the output, which wants many small workgroups) and
// its tiles, counted as if every matrix were as large as the largest, are 512 or more.  (Sets of unequal matrices have
// fewer: the 60M set's products Y L^-T are counted as 616 and are 280 or 336, one to two per CU.)
template <int TS>
static void run_gemm_f32(dim3 g, int op, const MatDev* mats, const MatDyn* dyn, int grad_dtype, StepScalars sc,
                         bool ai, bool bj, bool abf, bool bbf, bool sym,
                         const SymPlanes* planes, int side, hipStream_t stream) {
#define NG_GEMM_CASE(AI, BJ, ABF, BBF, SYM)                                                                      \
    if (ai == AI && bj == BJ && abf == ABF && bbf == BBF && sym == SYM) {                                        \
        k_gemm_f32<TS, AI, BJ, ABF, BBF, SYM><<<g, dim3(256), 0, stream>>>(op, mats, dyn, grad_dtype, sc, planes, side); \
        return;                                                                                                  \
    }
    NG_GEMM_CASE(true, true, false, false, true)      // the Gram matrices of the sketch and of P
    NG_GEMM_CASE(false, false, false, false, true)    // B B^T
    NG_GEMM_CASE(true, true, false, false, false)
    NG_GEMM_CASE(true, false, false, false, false)
    NG_GEMM_CASE(false, true, false, false, false)
    NG_GEMM_CASE(false, false, false, false, false)
    NG_GEMM_CASE(true, true, true, false, false)      // bf16 gradient as A
    NG_GEMM_CASE(false, true, true, false, false)
    NG_GEMM_CASE(true, true, false, true, false)      // as B
    NG_GEMM_CASE(true, false, false, true, false)
    NG_GEMM_CASE(false, true, false, true, false)     // bf16 history slot
#undef NG_GEMM_CASE
}

template <int TS>
static bool run_gemm_f32_sides(dim3 g, int op, const MatDev* mats, const MatDyn* dyn, StepScalars sc, const GemmView& l,
                               const GemmView& r, hipStream_t stream) {
    if (l.a_bf16 || l.b_bf16 || r.a_bf16 || r.b_bf16 || l.sym) return false;
#define NG_SIDES_CASE(AL, BL, AR, BR)                                                                            \
    if ((l.sAi == 1) == AL && (l.sBj == 1) == BL && (r.sAi == 1) == AR && (r.sBj == 1) == BR) {                  \
        k_gemm_f32_sides<TS, AL, BL, AR, BR><<<g, dim3(256), 0, stream>>>(op, mats, dyn, sc);                    \
        return true;                                                                                             \
    }
    NG_SIDES_CASE(true, true, true, false)     // P^T G, Y^T G
    NG_SIDES_CASE(false, true, true, false)    // P N and N^T P^T
    NG_SIDES_CASE(false, true, true, true)     // G Y
    NG_SIDES_CASE(true, true, false, true)     // G^T Y
#undef NG_SIDES_CASE
    return false;
}

// sides: bit 0 = left-side matrices present, bit 1 = right-side ones.  The products with the gradient or the
// weight read their operands along other dimensions on the right side: one kernel with both forms for fp32 sets that
// have both sides, else one launch per side that is present.
hipError_t launch_gemm_f32(GemmOp op, const MatDev* mats, const MatDyn* dyn, int n_mats, int max_m, int max_n,
                           int max_k, int grad_dtype, StepScalars sc, int max_split, const SymPlanes* sym,
                           int sides, hipStream_t stream) {
    // layouts and types of the operands are properties of the product and the side
    auto view = [&](int side) {
        MatDev probe{};
        probe.side = side;
        probe.ld_g = probe.ldn = probe.l = probe.lp = probe.r = 2;   // (any stride but 1)
        return gemm_view((int)op, probe, nullptr, grad_dtype, sc.slot, sc.hist_bf16);
    };
    const GemmView left = view(NG_SIDE_LEFT), right = view(NG_SIDE_RIGHT);
    const bool by_side = (left.sAi == 1) != (right.sAi == 1) || (left.sBj == 1) != (right.sBj == 1);
    auto count = [&](int ts) {
        const long long nx = (max_n + ts - 1) / ts, ny = (max_m + ts - 1) / ts;
        return (left.sym ? ny * (ny + 1) / 2 : nx * ny) * (max_split > 1 ? max_split : 1);
    };
    // (a split projection is a small one: its chunks were counted in 64 x 64 tiles)
    const bool big = max_m >= 128 && max_n >= 128 && max_k >= 64 && count(128) * n_mats >= 512 &&
                     !(op == OP_PROJECT_F32 && max_split > 0);
    const dim3 g((unsigned)((count(big ? 128 : 64) + 7) / 8 * 8), 1, n_mats);
    if (by_side && sides == 3 && grad_dtype == NG_F32 &&
        (big ? run_gemm_f32_sides<128>(g, (int)op, mats, dyn, sc, left, right, stream)
             : run_gemm_f32_sides<64>(g, (int)op, mats, dyn, sc, left, right, stream)))
        return hipGetLastError();
    for (int side = 0; side < 2; ++side) {
        if (by_side ? !(sides & (1 << side)) : side == 1) continue;
        const GemmView& v = side == NG_SIDE_RIGHT && by_side ? right : left;
        const int filter = by_side && sides == 3 ? side : -1;
        if (big) run_gemm_f32<128>(g, (int)op, mats, dyn, grad_dtype, sc, v.sAi == 1, v.sBj == 1, v.a_bf16, v.b_bf16, v.sym != 0, sym, filter, stream);
        else run_gemm_f32<64>(g, (int)op, mats, dyn, grad_dtype, sc, v.sAi == 1, v.sBj == 1, v.a_bf16, v.b_bf16, v.sym != 0, sym, filter, stream);
    }
    return hipGetLastError();
}

}  // namespace ng
