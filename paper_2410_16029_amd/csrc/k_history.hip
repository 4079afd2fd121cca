// The two passes of a step over the history in one launch (paper Sec. 2.4 and the Adam equations of Sec. 2.2):
//
//   y_j = <R, H_j>_F,  (lambda I + K/s) w = e_head,  g~ = sum_j w_j H_j,  M, V, N
//
// w needs every y_j of its matrix before the first element can be transformed, so the history is needed twice.  A workgroup
// keeps its tile of all s slots in registers (and LDS) between the two: history, M and V are read from memory once.  No cache
// would do that: a second read from the 256 MB memory-side cache goes at the 6.9 TB/s of one from HBM.
//
// What bounds it: while a matrix's tiles wait for w their places are taken, and 128 MB of history fit the chip.  At
// 7 TB/s that is 19 us from a tile's first load to its last, so what counts is the way from the last tile's sums to w:
//   - a workgroup per matrix only solves; it factors the known part of the system while the sums form (350M set 1787 ->
//     1533 us a step, against the last tile's workgroup solving);
//   - tiles count themselves in and look for w on eight lines per matrix (on one, history phase of the 350M set
//     1543 us, on eight 1099);
//   - the slots that fit LDS go there, which makes room for a fourth workgroup per CU.
// Kernel times (us, medians of 40 launches; without any waiting, results wrong / as it is / gram row, solve and transform in
// separate launches): 60M set 52 / 54 / 84, 130M 196 / 213 / 311, 350M 922 / 1010 / 1471, the 2048-wide matrices of the 1.1B
// set, of 512 tiles each, 1866 / 2485 / 2790.  Their bytes once at the 6.95 TB/s of a plain read: 39, 175, 768, 1485.
// Tried: the last tiles of a matrix too large for the chip kept and the others read
// twice in the same launch (1.1B set 6.0 ms against 5.8 in separate launches); fewer loads in flight per workgroup
// (the same).
//
// No progress depends on workgroups being on the chip together (wait_for_weights).  The split counts on a whole chip, 256 CUs,
// all the same: where others hold part of it, or the device is a partition, matrices of many tiles have workgroups that
// have not started after 100 us, and lose that time and a second read of the tiles that give way.
#include "state_math.h"

namespace ng {

namespace {

// One row of a lane's slot data: four columns, as floats or bf16
template <bool HB>
struct HistVec {
    typedef u32x4_t type;
};
template <>
struct HistVec<true> {
    typedef u32x2_t type;
};
template <bool HB>
__device__ __forceinline__ typename HistVec<HB>::type load_raw(const NG_AS1 unsigned char* slot, unsigned off) {
    return __builtin_nontemporal_load((const NG_AS1 typename HistVec<HB>::type*)(slot + off));
}
__device__ __forceinline__ f32x4_t widen(const u32x4_t v) {
    return (f32x4_t){__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
}
__device__ __forceinline__ f32x4_t widen(const u32x2_t v) {
    return (f32x4_t){__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                     __uint_as_float(v.y & 0xffff0000u)};
}

// A workgroup's tile: nb bands of eight rows, 4 / nb wavefronts side by side.  A lane has RT rows of four columns; LPO lanes
// share the rows of a band.  Rows and columns past the edge re-read the last ones; what they give is dropped.
template <int RT>
struct HistTile {
    static constexpr int LPO = 8 / RT, WC = 64 / LPO * 4;
    int band0, col0, nrow;
    unsigned eoff[RT];
    __device__ __forceinline__ HistTile(const MatDev& md, const TileRef& it, int wv, int lane) {
        const int nbs = (it.pad >> 2) & 3;
        band0 = it.ti + 8 * (wv & ((1 << nbs) - 1));
        col0 = it.tj + WC * (wv >> nbs) + (lane / LPO) * 4;
        const int row0 = band0 + RT * (lane & (LPO - 1));
        const int left = md.r - row0;
        nrow = col0 >= md.ldn || left < 0 ? 0 : (left < RT ? left : RT);
        const StatePanel sp = state_panel(md.r, md.pw, it.tj);
#pragma unroll
        for (int e = 0; e < RT; ++e) eoff[e] = sp.at(row0 + e < md.r ? row0 + e : md.r - 1, col0 < md.ldn ? col0 : it.tj);
    }
};

// M and V of two rows and four columns of a lane
struct Moments {
    f32x4_t m[2], v[2];
    template <int RT>
    __device__ __forceinline__ void load(const MatDev& md, const unsigned (&eoff)[RT], int e0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const unsigned off = eoff[e0 + u] * 4u;
            m[u] = __builtin_nontemporal_load((const NG_AS1 f32x4_t*)((const NG_AS1 unsigned char*)md.M + off));
            v[u] = __builtin_nontemporal_load((const NG_AS1 f32x4_t*)((const NG_AS1 unsigned char*)md.V + off));
        }
    }
};

// M, V and N of a tile from its transformed gradient; the moments of the first PF pairs of rows are in `ahead`
template <int RT, bool BF16_N, int PF>
__device__ __forceinline__ void finish_tile(const MatDev& md, const HistTile<RT>& tl, const f32x4_t (&g)[RT],
                                            const Moments* ahead, const StepScalars& sc, float bc1, float bc2, int lane, int* status) {
    constexpr int LPO = 8 / RT;
    NG_AS1 unsigned char* Mb = (NG_AS1 unsigned char*)md.M;
    NG_AS1 unsigned char* Vb = (NG_AS1 unsigned char*)md.V;
    u32x4_t pk[RT / 2];                  // bf16 N: element c is column c of rows (2 u, 2 u + 1)
    bool bad = false;
#pragma unroll
    for (int u2 = 0; u2 < RT / 2; ++u2) {
        Moments mo;
        if (u2 < PF) mo = ahead[u2];
        else mo.template load<RT>(md, tl.eoff, 2 * u2);
        f32x4_t nv[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = 2 * u2 + u;
            const unsigned off = tl.eoff[e] * 4u;
            const f32x4_t o = adam4(mo.m[u], mo.v[u], g[e], sc, bc1, bc2);
            const bool live = e < tl.nrow;
            if (live) {
                __builtin_nontemporal_store(mo.m[u], (NG_AS1 f32x4_t*)(Mb + off));
                __builtin_nontemporal_store(mo.v[u], (NG_AS1 f32x4_t*)(Vb + off));
            }
            bad |= live && any_not_finite(o);
#pragma unroll
            for (int x = 0; x < 4; ++x) nv[u][x] = live ? o[x] : 0.f;
            if (!BF16_N && live) *(NG_AS1 f32x4_t*)((NG_AS1 unsigned char*)md.N + off) = nv[u];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) pk[u2][c] = pack_bf16x2(nv[0][c], nv[1][c]);
    }
    if (BF16_N) {
        // [octet][col][8]: the lanes of a band hold its rows, RT each, for the same columns; they exchange until each has
        // all eight rows of RT / 2 columns, which are whole 16-byte octets next to each other
        const int q = lane & (LPO - 1);
        const bool store = tl.col0 < md.ldn && tl.band0 < md.r;
        NG_AS1 u32x4_t* Np = (NG_AS1 u32x4_t*)((NG_AS1 bf16_t*)md.N + ((long long)(tl.band0 >> 3) * md.ldn + tl.col0 + RT / 2 * q) * 8);
        auto give = [](unsigned v) { return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xf, 0xf, false); };   // lane ^ 1
        if constexpr (RT == 4) {
            // the even lane keeps columns 0 and 1, the odd one 2 and 3
            const u32x4_t a = pk[0], b = pk[RT / 2 - 1];
            const unsigned a0 = give(q ? a.x : a.z), b0 = give(q ? b.x : b.z), a1 = give(q ? a.y : a.w), b1 = give(q ? b.y : b.w);
            const u32x4_t oa = {q ? a0 : a.x, q ? b0 : b.x, q ? a.z : a0, q ? b.z : b0};
            const u32x4_t ob = {q ? a1 : a.y, q ? b1 : b.y, q ? a.w : a1, q ? b.w : b1};
            if (store) {
                Np[0] = oa;
                Np[1] = ob;
            }
        } else {
            // four lanes: a 4 x 4 transposition, lane q ends with column q
            auto give2 = [](unsigned v) { return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xf, 0xf, false); };   // lane ^ 2
            const bool o1 = q & 1, o2 = q & 2;
            const u32x4_t a = pk[0];
            const unsigned g0 = give(o1 ? a.x : a.y), g1 = give(o1 ? a.z : a.w);
            const u32x4_t t = {o1 ? g0 : a.x, o1 ? a.y : g0, o1 ? g1 : a.z, o1 ? a.w : g1};
            const unsigned h0 = give2(o2 ? t.x : t.z), h1 = give2(o2 ? t.y : t.w);
            const u32x4_t o = {o2 ? h0 : t.x, o2 ? h1 : t.y, o2 ? t.z : h0, o2 ? t.w : h1};
            if (store) Np[0] = o;
        }
    }
    if (bad) atomicOr(status, 2);
}

// R of a lane from the row chunks that a split fp32 projection left, added in chunk order
template <int RT>
__device__ __forceinline__ void sum_chunks(const MatDev& md, const MatDyn* dyn, int nparts, const unsigned (&eoff)[RT], f32x4_t (&sum)[RT]) {
    constexpr int NC = 16 / RT;
    const NG_AS1 unsigned char* pp = (const NG_AS1 unsigned char*)step_scratch<float>(dyn, md.proj_parts_off);
    const unsigned long long cstride = (unsigned long long)md.proj_rows * md.ldn * 4u;
#pragma unroll
    for (int e = 0; e < RT; ++e) sum[e] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    for (int c = 0; c < nparts; c += NC) {
        f32x4_t v[NC][RT];
#pragma unroll
        for (int u = 0; u < NC; ++u)
#pragma unroll
            for (int e = 0; e < RT; ++e) v[u][e] = *(const NG_AS1 f32x4_t*)(pp + (c + u < nparts ? c + u : c) * cstride + eoff[e] * 4u);
#pragma unroll
        for (int u = 0; u < NC; ++u)
#pragma unroll
            for (int e = 0; e < RT; ++e)
#pragma unroll
                for (int x = 0; x < 4; ++x) sum[e][x] += c + u < nparts ? v[u][e][x] : 0.f;
    }
}

}  // namespace

#define NG_AS3 __attribute__((address_space(3)))

namespace {

// What the wavefronts of a workgroup hand to each other
struct HistShared {
    double red[4][16], A[16][17], bc[256];
    float w[16];                         // weights in the order of a tile's slots, R's first
    // One word per decision of the first wavefront, written in one place and read behind a barrier: a wavefront that has not
    // read a decision yet must not find the next one there (the first runs ahead of it until their next barrier).
    int tile_cmd, solver_cmd, taken;
};
enum { kGo, kExit, kSolve };
__device__ __forceinline__ int wave_lane() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// Workgroups of the matrix, the solver's among them, that have not started.  (First wavefront; a look at eight lines, for those
// that have waited for long.)
__device__ __forceinline__ unsigned not_started(const HistoryLine* lines, int T, int lane) {
    unsigned n = 0;
    if (lane < kHistoryLines) n = __hip_atomic_load(&lines[lane].started, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int sum = 0;
#pragma unroll
    for (int l = 0; l < kHistoryLines; ++l) sum += __builtin_amdgcn_readlane((int)n, l);
    return (unsigned)(T + 1 - sum);
}

// First wavefront of a tile whose share is counted in: w from its line, every component with its mark.  After every wait_ticks
// of waiting it looks how many workgroups of its matrix have not started, which may need the places of those that have: the
// first that many tiles are left to whoever takes their bits, then twice as many, and so on.  Those that have started all arrive,
// so nobody leaves when all have; kHistoryPatience looks end any wait.  (When every tile left at the first look, a matrix whose
// last two tiles stood behind a neighbour's, on a first step with its page tables still to be walked, went through the few that
// were still there one tile after the other: first step of the 1.1B set 32 to 39 ms.)  The bit is set before w is looked at for the last time, and the solver goes
// through the bits after w is there: either this workgroup sees w and takes the bit back, or the solver sees the bit.
// `help`: others of the matrix had been left when the solver was done.
__device__ __forceinline__ int wait_for_weights(HistShared& sh, HistoryLine* lines, int part, int T, int s, int head, int lane,
                                                unsigned wait_ticks, bool& help) {
    HistoryLine* line = lines + (part & (kHistoryLines - 1));
    unsigned* leftover = reinterpret_cast<unsigned*>(lines + kHistoryLines) + (part >> 5);
    const unsigned bit = 1u << (part & 31);
    const int j = head + lane < s ? head + lane : head + lane - s;
    unsigned start = (unsigned)__builtin_amdgcn_s_memrealtime();
    unsigned looks = 0;
    bool late = false;
    for (;;) {
        unsigned long long v = 1ull << 32;
        if (lane < s) v = __hip_atomic_load(line->w + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__all((int)((v >> 32) != 0ull))) {
            if (lane < 16) sh.w[lane] = lane < s ? __uint_as_float((unsigned)v) : 0.f;
            help = __builtin_amdgcn_readfirstlane((int)(v >> 32)) != 1;
            if (!late) return kGo;
            unsigned old = 0;
            if (lane == 0) old = __hip_atomic_fetch_and(leftover, ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return (__builtin_amdgcn_readfirstlane(old) & bit) ? kGo : kExit;
        }
        if (late) return kExit;
        bool leave = false;
        const unsigned now = (unsigned)__builtin_amdgcn_s_memrealtime();
        if (now - start > wait_ticks) {
            leave = history_leaves(part, not_started(lines, T, lane), looks++) || wait_ticks == 0;
            start = now;
        }
        if (leave) {
            late = true;
            if (lane == 0) __hip_atomic_store((unsigned*)&line->arrived_late + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) __hip_atomic_fetch_or(leftover, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else {
            __builtin_amdgcn_s_sleep(8);
        }
    }
}

// The s x s system of a matrix.  `tile`: -1 for the workgroup whose item this is; the tile of the one that had the last
// share to add after that one had waited too long.  Returns false where the system is left to the other.
// The solve in two parts, so that little is left when the last sums arrive (it was 3 to 6 us of every tile's wait): X = L^{-1}
// of the system without row and column `head`, which needs nothing of this step, and then with `head` ordered last
// u = X b, the last pivot d = lambda + y_head / s - u.u, w = (-X^T u, 1) / d.
__device__ __forceinline__ bool solve_matrix(HistShared& sh, const MatDev& md, const MatDyn* dyn, const MatDyn& dy, HistoryLine* lines,
                                             int tile, const StepScalars& sc, unsigned wait_ticks, int* status, int tid, int wv) {
    const int lane = tid & 63;
    const int s = sc.s, head = dy.head, T = md.hist_tiles;
    // normaliser of the empirical Fisher: 1/s, or 1/(valid slots after this push) while the ring fills
    const double lam = (double)sc.lambda, inv_s = 1.0 / (double)(sc.norm_count ? dy.count : s);
    bool late = false;
    if (wv == 0) {
        if (tile < 0 && lane == 0) __hip_atomic_fetch_add(&lines->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int q = lane; q < s * s; q += 64) {
            const int i = q / s, j = q - i * s;
            sh.A[i][j] = md.K[q];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        bool bad = false;
        double v[16];
        factor16<17>(&sh.A[0][0], s, head, lane, lam, inv_s, v, bad);
        if (bad) atomicOr(status, 1);
        if (lane < 16) {
#pragma unroll
            for (int k = 0; k < 16; ++k) sh.A[k][lane] = v[k];
        }
        // Until all tiles are counted in.  Nothing says that they start while this workgroup holds its place: if some have not
        // after a while, it gives way, and the last of them solves.
        unsigned start = (unsigned)__builtin_amdgcn_s_memrealtime();
        unsigned looks = 0;
        int c = kGo;
        for (;;) {
            // (the count and whether tiles were left, one line of the matrix per lane)
            unsigned long long v = 0;
            if (lane < kHistoryLines) v = __hip_atomic_load(&lines[lane].arrived_late, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            late = __any((int)((v >> 32) != 0ull));
            if (tile >= 0) break;
            unsigned n = (unsigned)v;
            for (int d = 1; d < kHistoryLines; d *= 2) n += __shfl_xor(n, d);
            if (__builtin_amdgcn_readfirstlane(n) == (unsigned)T) break;
            const unsigned now = (unsigned)__builtin_amdgcn_s_memrealtime();
            const bool look = now - start > wait_ticks;
            if (look) start = now;
            if (look && (not_started(lines, T, lane) > 0 || ++looks == kHistoryPatience || wait_ticks == 0)) {
                unsigned there = 0;
                if (lane == 0) there = __hip_atomic_exchange(&lines->state, kSolverGone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kAllThere;
                if (!__builtin_amdgcn_readfirstlane(there)) c = kExit;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        if (lane == 0) sh.solver_cmd = c;
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(sh.solver_cmd) == kExit) return false;
    const double* parts = step_scratch<double>(dyn, md.dot_parts_off);
    const int nsub = T > 256 ? sum_dot_parts<true, 32>(parts, T, s, tid, sh.bc) : sum_dot_parts<true>(parts, T, s, tid, sh.bc);
    __syncthreads();
    if (tid < 16) {
        double v = 0.0;
        if (tid < s) {
            for (int q = 0; q < nsub; ++q) v += sh.bc[q * s + tid];
            md.K[(long long)head * s + tid] = v;
            md.K[(long long)tid * s + head] = v;
        }
        sh.red[0][tid] = v;
    }
    __syncthreads();
    if (wv == 0) {
        bool bad = false;
        const int k = lane & 15;
        double u = 0.0, w = 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) u = fma(sh.A[k][q], q == head ? 0.0 : sh.red[0][q] * inv_s, u);
        if (lane < 16) sh.red[1][k] = u;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        double d = fma(sh.red[0][head], inv_s, lam);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const double uq = sh.red[1][q];
            d = fma(-uq, uq, d);
            w = fma(sh.A[q][k], uq, w);
        }
        if (!(d > 0.0) || !(d < 1.0e300)) {
            bad = true;
            d = 1.0;
        }
        w = (k == head ? 1.0 : -w) / d;
        if (lane < 16) sh.w[lane] = 0.f;
        if (lane < s) {
            if (!(fabs(w) < 1.0e300)) bad = true;
            for (int q = 0; q < kHistoryLines; ++q)
                __hip_atomic_store(lines[q].w + lane, (late ? 3ull << 32 : 1ull << 32) | __float_as_uint((float)w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sh.w[lane >= head ? lane - head : lane - head + s] = (float)w;
            md.w64[lane] = w;
            md.w32[lane] = (float)w;
        }
        if (bad) atomicOr(status, 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // w is there before the bits are looked at
    }
    __syncthreads();
    return true;
}

// A tile whose slots are read again
template <int RT, bool HB, bool BF16_N>
__device__ __forceinline__ void transform_tile(const HistShared& sh, const MatDev& md, const MatDyn* dyn, const MatDyn& dy, const TileRef& at,
                                               const StepScalars& sc, int wv, int lane, int* status) {
    constexpr unsigned HS = HB ? 2u : 4u;
    const unsigned long long slot_bytes = (unsigned long long)md.slot_elems * HS;
    const int s = sc.s, head = dy.head;
    const HistTile<RT> tl(md, at, wv, lane);
    f32x4_t g[RT];
#pragma unroll
    for (int e = 0; e < RT; ++e) g[e] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    int j = 0;
    if constexpr (!BF16_N) {
        if (md.proj_chunks > 0) {            // (the slot was written in this launch, not necessarily on this XCD)
            sum_chunks<RT>(md, dyn, md.proj_chunks, tl.eoff, g);
            const float wj = sh.w[0];
#pragma unroll
            for (int e = 0; e < RT; ++e) g[e] *= wj;
            j = 1;
        }
    }
    int p = head + j < s ? head + j : 0;
#pragma unroll 4
    for (; j < s; ++j) {
        const NG_AS1 unsigned char* slot = (const NG_AS1 unsigned char*)md.H + (unsigned long long)p * slot_bytes;
        const float wj = sh.w[j];
#pragma unroll
        for (int e = 0; e < RT; ++e) {
            const f32x4_t a = widen(load_raw<HB>(slot, tl.eoff[e] * HS));
#pragma unroll
            for (int x = 0; x < 4; ++x) g[e][x] = fmaf(wj, a[x], g[e][x]);
        }
        p = p + 1 < s ? p + 1 : 0;
    }
    finish_tile<RT, BF16_N, 0>(md, tl, g, nullptr, sc, dy.bc1, dy.bc2, lane, status);
}

}  // namespace

// S: slots that the registers and LDS have room for, the last NL of them in LDS; PF pairs of rows have their moments
// requested before the weights are there.
template <int S, int RT, int NL, int PF, bool HB, bool BF16_N, int OCC>
__global__ __launch_bounds__(256, OCC) void k_history(const MatDev* __restrict__ mats, const MatDyn* __restrict__ dyn,
                                                      const TileRef* __restrict__ items, StepScalars sc,
                                                      unsigned wait_ticks, int* status) {
    typedef typename HistVec<HB>::type hist_t;
    static_assert(NL == 0 || !HB, "rows of 16 bytes go straight into LDS");
    static_assert(NL == 0 || BF16_N, "where R may be summed here, every slot beyond s is in registers");
    constexpr int NR = S - NL;
    constexpr unsigned HS = HB ? 2u : 4u;
    __shared__ __align__(16) unsigned char kept[NL > 0 ? NL * RT * 4096 : 16];   // [slot][row][thread] x 16 bytes
    __shared__ HistShared sh;

    // copies: what is read before the first store comes by scalar loads, all of it once
    const TileRef it = items[blockIdx.x];
    const MatDev md = mats[it.mat];
    const MatDyn dy = dyn[it.mat];
    // (the lane is counted anew where it is needed: kept from the start, the thread's index cost a trip through memory)
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s = sc.s, T = md.hist_tiles;
    HistoryLine* lines = step_scratch<HistoryLine>(dyn, md.hist_sync_off);
    bool solving = (it.pad & 1) == kHistorySolve, solved = false;
    int tile = -1;                       // of a workgroup that solves though it had a tile

    // (A loop that comes back for the rare case, so that the code below is there once: with the solver's code behind the tile's
    // the compiler kept the tile's registers for it as well and stored them to memory.)
    for (;;) {
        if (solving) {
            // (copies that the compiler cannot tell from others: it does nothing of this part ahead of a tile, where it would
            // cost registers)
            int lane = wave_lane(), pad = it.pad;
            asm volatile("" : "+v"(lane), "+s"(pad));
            if (!solved && !solve_matrix(sh, md, dyn, dy, lines, tile, sc, wait_ticks, status, 64 * wv + lane, wv)) return;
            // the tiles that were left, as a rule none, whoever takes their bits: the solver, and workgroups that see them left
            const int nbs = (pad >> 2) & 3, rows = 8 << nbs, cols = HistTile<RT>::WC * (4 >> nbs), across = (md.ldn + cols - 1) / cols;
            unsigned* leftover = reinterpret_cast<unsigned*>(lines + kHistoryLines);
            int word = 0, t = tile;
            for (;; t = -1) {
                __syncthreads();
                if (wv == 0 && t < 0) {
                    int taken = -1;
                    while (word < (T + 31) / 32 && taken < 0) {
                        unsigned m = 0;
                        if (lane == 0) m = __hip_atomic_load(leftover + word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        m = __builtin_amdgcn_readfirstlane(m);
                        if (m == 0) {
                            ++word;
                            continue;
                        }
                        const int b = __builtin_ctz(m);
                        if (lane == 0) m = __hip_atomic_fetch_and(leftover + word, ~(1u << b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if ((__builtin_amdgcn_readfirstlane(m) >> b) & 1u) taken = 32 * word + b;
                    }
                    if (lane == 0) sh.taken = taken;
                }
                __syncthreads();
                if (t < 0) t = __builtin_amdgcn_readfirstlane(sh.taken);
                if (t < 0) return;
                const TileRef at = {it.mat, t / across * rows, t % across * cols, nbs << 2};
                transform_tile<RT, HB, BF16_N>(sh, md, dyn, dy, at, sc, wv, lane, status);
            }
        }
        int lane = wave_lane(), head = dy.head;
        asm volatile("" : "+v"(lane), "+s"(head));     // (nor this part ahead of the loop)
        const int tid = 64 * wv + lane;
        const HistTile<RT> tl(md, it, wv, lane);
        const int part = it.pad >> 4;
        const unsigned long long slot_bytes = (unsigned long long)md.slot_elems * HS;
        // slot (head + j) mod s; a slot beyond s re-reads R, with weight 0, or where R is still to be summed is taken as zero
        // below (what the slot held before may be anything)
        const NG_AS1 unsigned char* const first = (const NG_AS1 unsigned char*)md.H;
        const NG_AS1 unsigned char* const mine = first + (unsigned long long)head * slot_bytes;
        const NG_AS1 unsigned char* slot = mine;
        hist_t h[NR][RT];                    // h[0]: R
        const int nparts = BF16_N ? 0 : md.proj_chunks;
#pragma unroll
        for (int j = 0; j < S; ++j) {
            if (j < NR) {
                if (BF16_N || j > 0 || nparts == 0) {
#pragma unroll
                    for (int e = 0; e < RT; ++e) h[j < NR ? j : 0][e] = load_raw<HB>(slot, tl.eoff[e] * HS);
                }
            } else {
#pragma unroll
                for (int e = 0; e < RT; ++e)     // (2: streamed, as the loads into registers)
                    __builtin_amdgcn_global_load_lds((const NG_AS1 void*)(slot + tl.eoff[e] * HS),
                                                     (NG_AS3 void*)(kept + ((j - NR) * RT + e) * 4096 + wv * 1024), 16, 0, 2);
            }
            slot = j + 1 >= s ? mine : head + j + 1 == s ? first : slot + slot_bytes;
        }
        if (wv == 0 && lane == 0)
            __hip_atomic_fetch_add(&lines[part & (kHistoryLines - 1)].started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if constexpr (!BF16_N) {
            if (nparts > 0) {
                f32x4_t sum[RT];
                sum_chunks<RT>(md, dyn, nparts, tl.eoff, sum);
                NG_AS1 unsigned char* r_slot = (NG_AS1 unsigned char*)mine;
#pragma unroll
                for (int e = 0; e < RT; ++e) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) h[0][e][x] = __float_as_uint(sum[e][x]);
                    if (e < tl.nrow) *(NG_AS1 f32x4_t*)(r_slot + tl.eoff[e] * 4u) = sum[e];
                }
#pragma unroll
                for (int j = 1; j < NR; ++j)
#pragma unroll
                    for (int e = 0; e < RT; ++e)
#pragma unroll
                        for (int x = 0; x < 4; ++x) h[j][e][x] = j < s ? h[j][e][x] : 0u;
            }
        }
        auto kept_at = [&](int j, int e) -> hist_t { return *(const hist_t*)(kept + ((j - NR) * RT + e) * 4096 + tid * 16); };
        // the tile's share of the Gram row: fp32 products and 4-term sums, everything beyond in fp64 and in a fixed order
        constexpr int NS = 4;
        static_assert(S % NS == 0, "sums go over the lanes four at a time");
#pragma unroll
        for (int j0 = 0; j0 < S; j0 += NS) {
            double acc[NS];
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                acc[j] = 0.0;
#pragma unroll
                for (int e = 0; e < RT; ++e) {
                    hist_t raw;
                    if (j0 + j < NR) raw = h[j0 + j < NR ? j0 + j : 0][e];
                    else raw = kept_at(j0 + j, e);
                    const f32x4_t a = widen(raw), b = widen(h[0][e]);
                    float p = a.x * b.x;
                    p = fmaf(a.y, b.y, p);
                    p = fmaf(a.z, b.z, p);
                    p = fmaf(a.w, b.w, p);
                    acc[j] += (double)(e < tl.nrow ? p : 0.f);
                }
                if (HB) __builtin_amdgcn_sched_barrier(0);
            }
            wave_sums<NS, 0>(acc, lane);
            if ((lane & (64 / NS - 1)) == 0) sh.red[wv][j0 + wave_sums_slot<NS>(lane)] = acc[0];
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        int c = kGo;
        if (wv == 0) {
            if (lane < s) {
                const double v = ((sh.red[0][lane] + sh.red[1][lane]) + sh.red[2][lane]) + sh.red[3][lane];
                const int j = head + lane < s ? head + lane : head + lane - s;
                __hip_atomic_store(step_scratch<double>(dyn, md.dot_parts_off) + (long long)part * s + j, v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            // the sums are where every XCD sees them before the tile counts as there
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            unsigned gone = 0;
            if (lane == 0) {
                const int l = part & (kHistoryLines - 1);
                const unsigned all = (unsigned)(T - l + kHistoryLines - 1) / kHistoryLines, used = T < kHistoryLines ? T : kHistoryLines;
                if (__hip_atomic_fetch_add((unsigned*)&lines[l].arrived_late, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == all &&
                    __hip_atomic_fetch_add(&lines->full, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == used)
                    gone = __hip_atomic_exchange(&lines->state, kAllThere, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kSolverGone;
            }
            if (__builtin_amdgcn_readfirstlane(gone)) c = kSolve;
        }
        Moments ahead[PF > 0 ? PF : 1];
#pragma unroll
        for (int k = 0; k < PF; ++k) ahead[k].template load<RT>(md, tl.eoff, 2 * k);
        if (wv == 0) {
            bool help = false;
            if (c == kGo) c = wait_for_weights(sh, lines, part, T, s, head, lane, wait_ticks, help);
            if (lane == 0) sh.tile_cmd = c | (help ? 16 : 0);
        }
        __syncthreads();
        const int cmd = __builtin_amdgcn_readfirstlane(sh.tile_cmd);
        if ((cmd & 15) == kGo) {
            f32x4_t g[RT];
#pragma unroll
            for (int e = 0; e < RT; ++e) g[e] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const float wj = sh.w[j];
#pragma unroll
                for (int e = 0; e < RT; ++e) {
                    hist_t raw;
                    if (j < NR) raw = h[j < NR ? j : 0][e];
                    else raw = kept_at(j, e);
                    if (HB) asm volatile("" : "+v"(raw));      // (widened again, not kept widened from above)
                    const f32x4_t a = widen(raw);
#pragma unroll
                    for (int x = 0; x < 4; ++x) g[e][x] = fmaf(wj, a[x], g[e][x]);
                }
                if (HB) __builtin_amdgcn_sched_barrier(0);
            }
            finish_tile<RT, BF16_N, PF>(md, tl, g, ahead, sc, dy.bc1, dy.bc2, lane, status);
        }
        if (cmd == kExit || cmd == kGo) return;
        solving = true;
        if ((cmd & 15) == kSolve) tile = part;
        else solved = true;
    }
}

// The kernels by slots and types: S, RT, NL, PF, types, workgroups per CU, and the most tiles of a matrix that takes this route.
// Beyond about half of the tiles that the chip holds, a matrix waits for itself: its first tiles hold their places until the
// last ones have found one.  Whole steps of sets of one shape, separate launches against this (us): rank 512 at 16
// float slots 353 -> 249 (128 tiles ... wide 1024), 338 -> 317 (2048 wide, 512 tiles), 371 -> 365 (3072, 768), and at 4096 (1024
// tiles) 20 times slower for want of places; at 8 float slots 344 -> 297 (384 tiles), 334 -> 303 (512); bf16 slots,
// 16 of them 225 -> 193 (256), 244 -> 226 (384), 234 -> 233 (512); 8 of them 244 -> 224 (384), 238 -> 248 (512); 4 float slots
// 237 -> 226 (384), 235 -> 248 (512).  fp32 sets at 4 slots 90 -> 88 (64), 139 -> 142 (256).
// Every instance at its limit, sets of one and of six matrices of rank 512, then of rank 128 and four times the width:
//   bf16 slots   4: 57 -> 53, 91 -> 84, 44 -> 41, 103 -> 98      8: 67 -> 62, 165 -> 148, 60 -> 55, 196 -> 182
//               16: 78 -> 69, 223 -> 206, 69 -> 62, 246 -> 240
//   float slots  4: 70 -> 63, 164 -> 146, 60 -> 55, 198 -> 183   8: 87 -> 68, 210 -> 186, 76 -> 59, 245 -> 223
//               16: 92 -> 70, 206 -> 182, 77 -> 56, 229 -> 206
//   fp32 sets    4: 52 -> 47, 104 -> 97, 45 -> 41, 116 -> 112    8: 64 -> 54, 173 -> 161, 61 -> 51, 204 -> 194
//               16: 75 -> 58, 205 -> 199, 72 -> 55, 232 -> 232
#define NG_HISTORY_CASES(X)                                     \
    if (hist_bf16) {                                            \
        if (s <= 4) X(4, 4, 0, 1, true, true, 4, 192);          \
        else if (s <= 8) X(8, 4, 0, 1, true, true, 4, 384);     \
        else X(16, 4, 0, 0, true, true, 3, 384);                \
    } else if (bf16_n) {                                        \
        if (s <= 4) X(4, 4, 0, 1, false, true, 4, 384);         \
        else if (s <= 8) X(8, 4, 0, 0, false, true, 3, 384);    \
        else X(16, 2, 4, 0, false, true, 4, 512);               \
    } else {                                                    \
        if (s <= 4) X(4, 2, 0, 1, false, false, 4, 128);        \
        else if (s <= 8) X(8, 2, 0, 1, false, false, 3, 256);   \
        else X(16, 2, 0, 1, false, false, 2, 256);              \
    }

void history_shape(int s, int hist_bf16, int bf16_n, int* lane_rows, int* wave_cols, int* most_tiles) {
#define NG_HISTORY_SHAPE(S, RT, NL, PF, HB, BN, OCC, MOST)      \
    do {                                                        \
        *lane_rows = RT;                                        \
        *wave_cols = HistTile<RT>::WC;                          \
        *most_tiles = MOST;                                     \
        static_assert(MOST <= 256 * OCC / 2, "a matrix, its solver and nearly all of the next one on the chip"); \
    } while (0)
    NG_HISTORY_CASES(NG_HISTORY_SHAPE)
#undef NG_HISTORY_SHAPE
}

hipError_t launch_history(const MatDev* mats, const MatDyn* dyn, const TileRef* items, int n_items, StepScalars sc,
                          int grad_dtype, unsigned wait_ticks, int* status, hipStream_t stream) {
    if (n_items == 0) return hipSuccess;
    const int s = sc.s;
    const bool hist_bf16 = sc.hist_bf16, bf16_n = grad_dtype == NG_BF16;
#define NG_HISTORY_LAUNCH(S, RT, NL, PF, HB, BN, OCC, MOST)                                                                   \
    hipLaunchKernelGGL((k_history<S, RT, NL, PF, HB, BN, OCC>), dim3(n_items), dim3(256), 0, stream, mats, dyn, items, sc, \
                       wait_ticks, status)
    NG_HISTORY_CASES(NG_HISTORY_LAUNCH)
#undef NG_HISTORY_LAUNCH
    return hipGetLastError();
}

}  // namespace ng
