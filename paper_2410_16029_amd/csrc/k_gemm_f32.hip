// Grouped fp32 GEMM, one launch for all matrices of the layer set.  It serves the NG_F32 step (projection
// R = P^T G, paper Sec. 1; update W -= lr (scale P N + wd W), paper Sec. 2.2)
// and every dense product of the projector refresh.  Operands are described as
// strided views A(i,k), B(k,j) so one kernel covers all transpositions; an
// operand may be stored as float or bf16 (gradients).
//
// The products run on the bf16 MFMA, each operand split into three bf16 planes on its way into LDS (F32Src).
// On the fp32 MFMA (v_mfma_f32_32x32x2_f32) they reached half of its rate.  Before / now, and the rms error of a sum of 600
// terms relative to the root of the sum of its squared terms, 4.4e-7 / 1.4e-7: 168 Gram matrices of 1024..2736 x 256
// 266 / 182 us, 168 products with a 256 x 256 factor 293 / 188 us, fp32 step of eight mid-size blocks 974 / 658 us.
// What bounds them now: 128 x 128 tiles of 6 to 10 k-steps, each with its split, two barriers and the latency of the
// first loads: in the refresh of 168 matrices of 1024..2736 at rank 256 the matrix cores are busy 25-40 % of the cycles, the
// wavefronts wait a third to two fifths of theirs, with 1.3-1.6 of the two per SIMD there on average.
//
// Tile 128 x 128 per workgroup (4 wavefronts of 64 x 64, two workgroups per CU), BK = 32.  Tried: eight wavefronts of 64 x
// 32, two LDS buffers and three register sets (one workgroup per CU): 290 us.
// MFMA 32x32x16 bf16 operand layout: lane L supplies eight consecutive k, 8 (L/32) .. of A row L%32 and of B column L%32;
// the 16 accumulators of lane L are D[8*g + 4*(L/32) + e][L%32], index 4*g + e.
#include <type_traits>

#include "ng_internal.h"
#include "split_bf16.h"

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

// Every operand value x goes into LDS as three bf16 planes, 2^16 x = x0 + x1 + x2 (each the rounding of what the ones before
// leave: 24 bits, the float itself; every float is a multiple of 2^-149, bf16's subnormals of 2^-133, hence the factor: without
// it operands below 2^-110 lost bits, 2.7e-6 of a product at 1e-35), and a product of two operands is six bf16 MFMA products,
//   a b = a0 b0 + (a0 b1 + a1 b0 + a1 b1 + a0 b2 + a2 b0),
// which drops a1 b2 + a2 b1 + a2 b2, together at most 2^-24 (1 + 2^-10) |a b|.
// a0 b0 has an accumulator of its own, which is rounded once per 16 contraction steps (the fp32 MFMA rounds every
// two), and the other five share one that is some 2^-8 as large: the sums are closer to 64 bits than the fp32
// MFMA's, at three eighths of its matrix-core time.
// A gradient (or history slot) stored as bf16 has one plane.
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

constexpr float kSplitUp = 65536.f;

// One operand of a tile: T (tile index) x K (contraction), TS x BK per k-step, moved as vectors of four
// elements along the stride-1 dimension -- the tile index (TF) or the contraction -- and kept in LDS as NP planes
// [T][K], K contiguous (what the MFMA reads).  tile-fast: a thread has 4 tile indexes of BK / KG consecutive k, the
// k-groups fastest over the lanes (LDS writes of one instruction on distinct banks, 128 consecutive bytes in memory);
// k-fast: 4 consecutive k at tile index t / (BK/4) + (1024/BK) q.
template <int TS, int BK, bool TF, bool BF>
struct F32Src {
    static constexpr int NV = TS * BK / 1024, LDK = BK + 8, ES = BF ? 2 : 4, KT = BK / 4, TQ = 1024 / BK;
    static constexpr int KG = 1024 / TS, NP = BF ? 1 : 3, PLANE = TS * LDK;      // PLANE: bf16 elements per plane
    static_assert(BK / KG == NV, "vectors of a tile-fast thread");
    const NG_AS1 unsigned char* base;   // element (0, 0)
    const NG_AS1 unsigned char* safe;   // 16 readable bytes
    long long st, sk;                   // element strides along T and K
    unsigned off[NV];                   // byte offsets of this thread's vectors of k-step 0 (an operand is below 2 GiB)
    int t0, k0, lim, K;                 // this thread's first position, valid tile indexes, contraction length
    int shift;                          // tile-fast: elements by which a vector that straddles the edge was moved back
    __device__ __forceinline__ void init(const void* p, const void* safe_, long long st_, long long sk_, int tile0,
                                         int lim_, int K_, int t) {
        base = (const NG_AS1 unsigned char*)p;
        safe = (const NG_AS1 unsigned char*)safe_;
        st = st_;
        sk = sk_;
        lim = lim_;
        K = K_;
        t0 = tile0 + (TF ? 4 * (t / KG) : t / KT);
        k0 = TF ? NV * (t % KG) : 4 * (t % KT);
        // what lies past the operand's last tile index is read from inside it: it only reaches results that are not stored
        const int ti = TF ? (t0 + 4 <= lim ? t0 : lim >= 4 ? lim - 4 : 0) : t0;
        shift = TF && t0 < lim ? t0 - ti : 0;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int i = TF ? ti : t0 + TQ * q < lim ? t0 + TQ * q : lim - 1;
            off[q] = (unsigned)((TF ? (long long)i + (long long)(k0 + q) * sk : (long long)i * st + k0) * ES);
        }
    }
    // (a tile-fast operand of fewer than four tile indexes has no whole vectors)
    __device__ __forceinline__ int whole_steps() const { return TF && lim < 4 ? 0 : K / BK; }
    // k-step kt < whole_steps(): whole vectors, no tests
    __device__ __forceinline__ void fetch(int kt, f32x4_t (&r)[NV]) const {
        const NG_AS1 unsigned char* p = base + (TF ? (long long)BK * sk : (long long)BK) * ES * kt;      // uniform
#pragma unroll
        for (int q = 0; q < NV; ++q) r[q] = load4<BF>(p + off[q]);
    }
    // the straddling vectors' elements back to their places (tiles at such an edge only)
    __device__ __forceinline__ void realign(f32x4_t (&r)[NV]) const {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            if (shift & 1) r[q] = (f32x4_t){r[q].y, r[q].z, r[q].w, 0.f};
            if (shift & 2) r[q] = (f32x4_t){r[q].z, r[q].w, 0.f, 0.f};
        }
    }
    // any k-step, zero outside the operand: whole vectors from clamped addresses; the lanes whose vector straddles the
    // edge (only where the edge is not a multiple of four) read theirs element by element
    __device__ __forceinline__ void fetch_edge(int kt, f32x4_t (&r)[NV]) const {
        const bool straddles = ((TF ? lim : K) & 3) != 0;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int i = TF ? t0 : t0 + TQ * q;
            const int k = kt * BK + (TF ? k0 + q : k0);
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
    // the planes -> S (PLANE elements each)
    __device__ __forceinline__ void stage(const f32x4_t (&r)[NV], bf16_t* S, int t) const {
#pragma unroll
        for (int y = 0; y < (TF ? 4 : NV); ++y) {
            bf16_t* dst = S + (TF ? 4 * (t / KG) + y : t / KT + TQ * y) * LDK + k0;
            constexpr int PAIRS = TF ? NV / 2 : 2;
            unsigned p[PAIRS][NP];
            constexpr float up = BF ? 1.f : kSplitUp;
#pragma unroll
            for (int c = 0; c < PAIRS; ++c)
                split2<NP>(up * (TF ? r[2 * c][y] : r[y % NV][2 * c]), up * (TF ? r[2 * c + 1][y] : r[y % NV][2 * c + 1]), p[c]);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if (PAIRS == 2) *reinterpret_cast<uint2*>(dst + i * PLANE) = make_uint2(p[0][i], p[PAIRS - 1][i]);
                else *reinterpret_cast<unsigned*>(dst + i * PLANE) = p[0][i];
            }
        }
    }
};

// Tile TS x TS per workgroup (128: four wavefronts of 64 x 64 = 2 x 2 MFMA blocks of 32 x 32; 64: one
// block per wavefront, for products with a short side, a short contraction or few tiles).
// AI / BJ: the tile index is operand A's / B's stride-1 dimension (else the contraction is); ABF / BBF:
// operand A / B is stored as bf16; SYM: a symmetric product (partial planes).  only >= 0: matrices of that side,
// or those without sketch planes.  A tile whose rows and columns all exist takes whole vectors without a test (only a
// last partial k-step is read element by element); with the tests of every vector, and of every MFMA
// block against the product's edge, in the loop the products ran at a quarter of the fp32 MFMA rate.
constexpr int kF32BK = 32;             // contraction steps per LDS tile
constexpr int kOnlyPlaneless = 2;
template <int TS>
struct F32Tiles {
    bf16_t a[3 * TS * (kF32BK + 8)], b[3 * TS * (kF32BK + 8)];   // three planes each, rows padded by 16 bytes
};

// A barrier that waits for this wave's LDS accesses only: __syncthreads() would also wait for the operand loads in
// flight, i.e. expose a memory latency in every k-step.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A wavefront's blocks once more, on the fp32 MFMA and straight from memory: the planes cannot stand for an infinity, whose
// lower planes are NaN and whose products with the other operand's lower planes are infinities of either sign, nor for
// values from 2^112 on, nor for sums from 2^96 on (both carry the planes' factor).  Each shows as a result that is not
// finite, so such results are formed again; i, j: this lane's first row and column.  Step of 56 matrices (60M set, rank 128)
// with finite gradients / an infinity in each / nothing but NaN: 270 / 462 / 518 us, of 28 of the 350M set 692 / 1336 / 1529
// (all products on the fp32 MFMA, from LDS tiles: 491 / 543 / 521 and 896 / 948 / 910).
template <int NB, bool AI, bool BJ, bool ABF, bool BBF>
__device__ __forceinline__ void fp32_again(floatx16 (&acc)[NB][NB], const GemmView& v, int i, int j, int h) {
    const NG_AS1 unsigned char *pa[NB], *pb[NB];
#pragma unroll
    for (int x = 0; x < NB; ++x) {
        // (rows and columns past the product's edge re-read its last ones: their results are not stored, or zeroed)
        const int row = i + 32 * x < v.M ? i + 32 * x : v.M - 1, col = j + 32 * x < v.Nvalid ? j + 32 * x : v.Nvalid - 1;
        pa[x] = (const NG_AS1 unsigned char*)v.A + row * v.sAi * (ABF ? 2 : 4);
        pb[x] = (const NG_AS1 unsigned char*)v.B + col * v.sBj * (BBF ? 2 : 4);
#pragma unroll
        for (int y = 0; y < NB; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.f;
    }
    auto multiply = [&](const float (&a)[NB], const float (&b)[NB]) {
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
            for (int y = 0; y < NB; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[x], b[y], acc[x][y], 0, 0, 0);
    };
    // four consecutive k per half of the wavefront: one vector of an operand that has them side by side
    auto four = [](auto bf, bool fast, const NG_AS1 unsigned char* p, int k, long long sk) {
        constexpr bool BF = decltype(bf)::value;
        if (fast) return load4<BF>(p + (long long)k * (BF ? 2 : 4));
        return (f32x4_t){load1<BF>(p, k * sk), load1<BF>(p, (k + 1) * sk), load1<BF>(p, (k + 2) * sk), load1<BF>(p, (k + 3) * sk)};
    };
    const int whole = v.K / 8 * 8;
#pragma unroll 2
    for (int k0 = 0; k0 < whole; k0 += 8) {
        f32x4_t a4[NB], b4[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            a4[x] = four(std::bool_constant<ABF>(), !AI, pa[x], k0 + 4 * h, v.sAk);
            b4[x] = four(std::bool_constant<BBF>(), !BJ, pb[x], k0 + 4 * h, v.sBk);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float a[NB], b[NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                a[x] = a4[x][e];
                b[x] = b4[x][e];
            }
            multiply(a, b);
        }
    }
    for (int k0 = whole; k0 < v.K; k0 += 2) {
        const bool in = k0 + h < v.K;
        const int k = in ? k0 + h : v.K - 1;
        float a[NB], b[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            a[x] = in ? load1<ABF>(pa[x], k * v.sAk) : 0.f;
            b[x] = in ? load1<BBF>(pb[x], k * v.sBk) : 0.f;
        }
        multiply(a, b);
    }
}

template <int TS, bool AI, bool BJ, bool ABF, bool BBF, bool SYM>
__device__ __forceinline__ void gemm_f32_tile(int op, const MatDev* __restrict__ mats, const MatDyn* __restrict__ dyn,
                                              int grad_dtype, const StepScalars& sc, const SymPlanes* __restrict__ sym,
                                              F32Tiles<TS>& lds) {
    constexpr int BK = kF32BK;
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
        const int kc = ((v.K + sp.count - 1) / sp.count + kSymStep - 1) / kSymStep * kSymStep;
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

    floatx16 acc[NB][NB], low[NB][NB];      // a0 b0, and the five smaller products
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[a][b][x] = low[a][b][x] = 0.f;

    SA sa;
    SB sb;
    sa.init(v.A, mats, v.sAi, v.sAk, i0, v.M, v.K, t);
    sb.init(v.B, mats, v.sBj, v.sBk, j0, v.Nvalid, v.K, t);

    auto multiply = [&]() {
        const bf16_t* pa = lds.a + (wm * (TS / 2) + li) * SA::LDK + 8 * h;
        const bf16_t* pb = lds.b + (wn * (TS / 2) + li) * SB::LDK + 8 * h;
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            bf16x8_t a[SA::NP][NB], b[SB::NP][NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
#pragma unroll
                for (int i = 0; i < SA::NP; ++i)
                    a[i][x] = *reinterpret_cast<const bf16x8_t*>(pa + i * SA::PLANE + 32 * x * SA::LDK + kk);
#pragma unroll
                for (int i = 0; i < SB::NP; ++i)
                    b[i][x] = *reinterpret_cast<const bf16x8_t*>(pb + i * SB::PLANE + 32 * x * SB::LDK + kk);
            }
#pragma unroll
            for (int ia = 0; ia < SA::NP; ++ia)
#pragma unroll
                for (int ib = 0; ib < SB::NP && ia + ib < 3; ++ib)
#pragma unroll
                    for (int x = 0; x < NB; ++x)
#pragma unroll
                        for (int y = 0; y < NB; ++y) {
                            floatx16& c = ia + ib == 0 ? acc[x][y] : low[x][y];
                            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ia][x], b[ib][y], c, 0, 0, 0);
                        }
        }
    };

    // The loads of tile kt + 1 are in flight while tile kt is multiplied; one LDS tile (a second would leave room for
    // one workgroup per CU instead of two, whose staging and products overlap).  The loop has no branch around a load
    // (the compiler waits for the load where such paths meet): whole k-steps of both operands first, what is left after.
    const int nk = (v.K + BK - 1) / BK;
    const int whole_a = sa.whole_steps(), whole_b = sb.whole_steps();
    const int nw = whole_a < whole_b ? whole_a : whole_b;
    // (uniform) tiles with vectors that straddle the last tile index
    const bool back_a = AI && (v.M & 3) != 0 && i0 + TS > v.M, back_b = BJ && (v.Nvalid & 3) != 0 && j0 + TS > v.Nvalid;
    f32x4_t ra[NV], rb[NV];
    auto stage = [&]() {
        sa.stage(ra, lds.a, t);
        sb.stage(rb, lds.b, t);
    };
    if (nw > 0) {
        sa.fetch(0, ra);
        sb.fetch(0, rb);
        for (int kt = 0; kt < nw; ++kt) {
            if (back_a) sa.realign(ra);
            if (back_b) sb.realign(rb);
            stage();
            const int next = kt + 1 < nw ? kt + 1 : kt;
            sa.fetch(next, ra);
            sb.fetch(next, rb);
            lds_barrier();
            multiply();
            lds_barrier();
        }
    }
    for (int kt = nw; kt < nk; ++kt) {
        sa.fetch_edge(kt, ra);
        sb.fetch_edge(kt, rb);
        stage();
        lds_barrier();
        multiply();
        lds_barrier();
    }
    constexpr float down = 1.f / ((ABF ? 1.f : kSplitUp) * (BBF ? 1.f : kSplitUp));
    bool finite = true;
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc[x][y][e] = down * (acc[x][y][e] + low[x][y][e]);
                finite = finite && fabsf(acc[x][y][e]) <= 3.402823466e38f;
            }
    if (__any(!finite)) fp32_again<NB, AI, BJ, ABF, BBF>(acc, v, i0 + wm * (TS / 2) + li, j0 + wn * (TS / 2) + li, h);

    // columns from Nvalid on (the padding of a state's rows) are zero
    if (j0 + TS > v.Nvalid) {
#pragma unroll
        for (int y = 0; y < NB; ++y) {
            const bool in = j0 + wn * (TS / 2) + 32 * y + li < v.Nvalid;
#pragma unroll
            for (int x = 0; x < NB; ++x)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[x][y][e] = in ? acc[x][y][e] : 0.f;
        }
    }

    // the sketch planes that a gradient product reads next: octets of rows (a lane's four rows are half an octet), rows past
    // the last zero
    if (v.b_tri && sc.planes > 0 && md.Yp != nullptr) {
        bf16_t* planes[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) planes[p] = sketch_plane(md, op == OP_APPLY_C2A, p);
#pragma unroll
        for (int bi = 0; bi < NB; ++bi)
#pragma unroll
            for (int bj = 0; bj < NB; ++bj) {
                const int col = j0 + wn * (TS / 2) + bj * 32 + li;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int oct = i0 + wm * (TS / 2) + bi * 32 + 8 * g;       // its first row
                    float x[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = oct + 4 * h + e < v.M ? acc[bi][bj][4 * g + e] : 0.f;
                    unsigned lo[3], hi[3];
                    split2<3>(x[0], x[1], lo);
                    split2<3>(x[2], x[3], hi);
                    if (oct < v.M && col < v.N) {
                        const long long at = ((long long)(oct >> 3) * md.l + col) * 8 + 4 * h;
#pragma unroll
                        for (int p = 0; p < 3; ++p)
                            if (p < sc.planes) *(NG_AS1 u32x2_t*)((NG_AS1 bf16_t*)planes[p] + at) = (u32x2_t){lo[p], hi[p]};
                    }
                }
            }
        if (sc.planes_only) return;
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
__global__ __launch_bounds__(256, TS == 128 ? 2 : 4) void k_gemm_f32(int op, const MatDev* __restrict__ mats,
                                                  const MatDyn* __restrict__ dyn, int grad_dtype,
                                                  StepScalars sc, const SymPlanes* __restrict__ sym, int only) {
    __shared__ __attribute__((aligned(16))) F32Tiles<TS> lds;
    if (only >= 0 && (only == kOnlyPlaneless ? mats[blockIdx.z].Yp != nullptr : mats[blockIdx.z].side != only)) return;
    gemm_f32_tile<TS, AI, BJ, ABF, BBF, SYM>(op, mats, dyn, grad_dtype, sc, sym, lds);
}

// fp32 layer sets with both sides: AL / BL are a left-side matrix's layouts, AR / BR a right-side one's.  A launch
// per side has two ends at which the chip runs empty, the second for the few matrices of one side (four blocks
// of width 450 at rank 56, 24 left and 4 right: step 138.8 -> 114.9 us).
template <int TS, bool AL, bool BL, bool AR, bool BR>
__global__ __launch_bounds__(256, TS == 128 ? 2 : 4) void k_gemm_f32_sides(int op, const MatDev* __restrict__ mats,
                                                  const MatDyn* __restrict__ dyn, StepScalars sc) {
    __shared__ __attribute__((aligned(16))) F32Tiles<TS> lds;
    if (mats[blockIdx.z].side == NG_SIDE_RIGHT)
        gemm_f32_tile<TS, AR, BR, false, false, false>(op, mats, dyn, NG_F32, sc, nullptr, lds);
    else
        gemm_f32_tile<TS, AL, BL, false, false, false>(op, mats, dyn, NG_F32, sc, nullptr, lds);
}

// The refresh's products with one side of up to 32 (the gradient with a narrow sketch, the rotation of a narrow basis) of
// sets so small that a 64 x 64 tile per workgroup leaves most of the chip idle and each tile's k-steps follow one another:
// a workgroup takes 16 indexes of the long side and all of the short one, its wavefronts 32 indexes of the contraction at
// a time, in fp64 (16 x 16 x 4 MFMA), and their sums are added up through LDS.  Such a product of one 256 x 512 matrix at
// l = 32, a chain of 16 k-steps in the large kernel, was 12 us; its refresh 280 -> 234 us, one of 1024 x 1024 463 -> 348, one of
// 4096 x 4096 at l = 32 1040 -> 612.  The limit: sets of 256 x 512 with 640 workgroups 334 -> 318, 768 x 768 with 768 405 -> 383,
// 1024 x 1024 with 768 496 -> 461 and 1024 500 -> 505, 768 x 768 with 1152 434 -> 451: fp64 runs at an eighth of the bf16 planes' rate.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
constexpr int kFewRows = 16, kFewSide = 32, kFewWaves = 8, kFewBlocks = 768;

__global__ __launch_bounds__(64 * kFewWaves) void k_gemm_f32_few(int op, const MatDev* __restrict__ mats, const MatDyn* __restrict__ dyn) {
    __shared__ double sums[kFewWaves][2][256];
    const GemmView v = gemm_view(op, mats[blockIdx.y], dyn ? dyn + blockIdx.y : nullptr, NG_F32);
    // L (long side x contraction) times S (contraction x short side)
    const bool b_long = op == OP_QT_G;
    const float* __restrict__ L = (const float*)(b_long ? v.B : v.A);
    const float* __restrict__ S = (const float*)(b_long ? v.A : v.B);
    const long long li = b_long ? v.sBj : v.sAi, lk = b_long ? v.sBk : v.sAk;
    const unsigned sk = (unsigned)(b_long ? v.sAk : v.sBk);          // (the short side's indexes are adjacent)
    const int rows = b_long ? v.Nvalid : v.M, cols = b_long ? v.M : v.N;
    const int i0 = kFewRows * blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (i0 >= (b_long ? v.N : v.M)) return;
    const int c = lane & 15, g = lane >> 4;
    const NG_AS1 float* row = (const NG_AS1 float*)L + (i0 + c < rows ? i0 + c : 0) * li;
    const unsigned at[2] = {(unsigned)(c < cols ? c : 0), (unsigned)(c + 16 < cols ? c + 16 : 0)};
    f64x4_t acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
    for (int k0 = 32 * w; k0 < v.K; k0 += 32 * kFewWaves) {
        float a[2][4], b[2][4][2];
        // indexes k0 + 16 h + 4 g + u of the contraction
        if (lk == 1 && k0 + 32 <= v.K) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4_t q = *(const NG_AS1 f32x4_a4*)(row + k0 + 16 * h + 4 * g);
#pragma unroll
                for (int u = 0; u < 4; ++u) a[h][u] = q[u];
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = k0 + 16 * h + 4 * g + u;
                    a[h][u] = row[(k < v.K ? k : 0) * lk];
                }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + 16 * h + 4 * g + u;
                const NG_AS1 float* s = (const NG_AS1 float*)S + (unsigned)(k < v.K ? k : 0) * sk;
#pragma unroll
                for (int t = 0; t < 2; ++t) b[h][u][t] = s[at[t]];
            }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = k0 + 16 * h + 4 * g + u < v.K;
                const double x = in && i0 + c < rows ? a[h][u] : 0.f;
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, (double)(in && c + 16 * t < cols ? b[h][u][t] : 0.f), acc[t], 0, 0, 0);
            }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) sums[w][t][64 * e + lane] = acc[t][e];
    __syncthreads();
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < kFewWaves; ++q) sum += sums[q][tid >> 8][tid & 255];
    const int i = i0 + 4 * ((tid & 255) >> 6) + ((tid & 63) >> 4), j = 16 * (tid >> 8) + (tid & 15);
    if (j >= cols || i >= (b_long ? v.N : v.M)) return;
    NG_AS1 float* C = (NG_AS1 float*)v.C;
    if (b_long) C[(long long)j * v.ldc + i] = (float)sum;
    else C[(long long)i * v.ldc + j] = (float)sum;
}

// max_m, max_n, max_k: the largest dimensions of this product over the layer set; tiles: its 128 x 128 tiles.  The large
// tile, half of the operand bytes per product, is used from 1536 tiles (three per workgroup slot) on for runs of the
// contraction of 256, from 512 on for runs of 768: the small one, a quarter of the work per workgroup, hides more of each
// one's first loads and of its epilogue.  Small against large tiles: fp32 step of 56 matrices of the 60M set at rank 128 (1568 tiles) 353 -> 297 us, 14
// of them 122 -> 103; refresh of that set 1790 -> 1700; of 84 768-wide matrices (1248 tiles, runs of 256) 7259 -> 7149; but
// 14 and 28 matrices of the 350M set in fp32 (1568 and 3136 tiles, runs of 256) 404 -> 406 and 700 -> 714, refresh of
// that set in bf16 12.49 -> 12.75 ms, projection of the 28 in fp32 (672 tiles, runs of 1024 and more): step 689 -> 712.
bool f32_tile_large(GemmOp op, int max_m, int max_n, int max_k, long long tiles, int max_split) {
    // (a split projection is a small one: its chunks were counted in 64 x 64 tiles)
    if (op == OP_PROJECT_F32 && max_split > 0) return false;
    const int run = max_k / (max_split > 1 ? max_split : 1);
    return max_m >= 128 && max_n >= 128 && run >= 256 && tiles >= 512 && tiles * run >= 1536 * 256;
}

template <int TS>
static void run_gemm_f32(dim3 g, int op, const MatDev* mats, const MatDyn* dyn, int grad_dtype, StepScalars sc,
                         bool ai, bool bj, bool abf, bool bbf, bool sym,
                         const SymPlanes* planes, int only, hipStream_t stream) {
#define NG_GEMM_CASE(AI, BJ, ABF, BBF, SYM)                                                                      \
    if (ai == AI && bj == BJ && abf == ABF && bbf == BBF && sym == SYM) {                                        \
        k_gemm_f32<TS, AI, BJ, ABF, BBF, SYM><<<g, dim3(256), 0, stream>>>(op, mats, dyn, grad_dtype, sc, planes, only); \
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
// have both sides, else one launch per side that is present.  (Sets with sketch planes have left-side matrices only.)
hipError_t launch_gemm_f32(GemmOp op, const MatDev* mats, const MatDyn* dyn, int n_mats, int max_m, int max_n,
                           int max_k, long long tiles, int grad_dtype, StepScalars sc, int max_split,
                           const SymPlanes* sym, int sides, bool planeless, hipStream_t stream) {
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
    const int few = op == OP_QT_G ? max_m : max_n, many = op == OP_QT_G ? max_n : max_m;
    if ((op == OP_ROTATE || (grad_dtype == NG_F32 && (op == OP_G_B2A || op == OP_G_C2A || op == OP_GT_C2B || op == OP_QT_G))) &&
        !planeless && few <= kFewSide && (long long)((many + kFewRows - 1) / kFewRows) * n_mats <= kFewBlocks) {
        k_gemm_f32_few<<<dim3((many + kFewRows - 1) / kFewRows, n_mats), dim3(64 * kFewWaves), 0, stream>>>((int)op, mats, dyn);
        return hipGetLastError();
    }
    const bool big = f32_tile_large(op, max_m, max_n, max_k, tiles, max_split);
    const dim3 g((unsigned)((count(big ? 128 : 64) + 7) / 8 * 8), 1, n_mats);
    if (by_side && sides == 3 && grad_dtype == NG_F32 &&
        (big ? run_gemm_f32_sides<128>(g, (int)op, mats, dyn, sc, left, right, stream)
             : run_gemm_f32_sides<64>(g, (int)op, mats, dyn, sc, left, right, stream)))
        return hipGetLastError();
    for (int side = 0; side < 2; ++side) {
        if (by_side ? !(sides & (1 << side)) : side == 1) continue;
        const GemmView& v = side == NG_SIDE_RIGHT && by_side ? right : left;
        const int filter = planeless ? kOnlyPlaneless : by_side && sides == 3 ? side : -1;
        if (big) run_gemm_f32<128>(g, (int)op, mats, dyn, grad_dtype, sc, v.sAi == 1, v.sBj == 1, v.a_bf16, v.b_bf16, v.sym != 0, sym, filter, stream);
        else run_gemm_f32<64>(g, (int)op, mats, dyn, grad_dtype, sc, v.sAi == 1, v.sBj == 1, v.a_bf16, v.b_bf16, v.sym != 0, sym, filter, stream);
    }
    return hipGetLastError();
}

}  // namespace ng
