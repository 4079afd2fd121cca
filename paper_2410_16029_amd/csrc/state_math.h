// Device helpers shared by the kernels that stream M, V and the history (k_elementwise.hip, k_history.hip).
#pragma once

#include "eliminate16.h"
#include "ng_internal.h"

namespace ng {

// Pointers read out of the per-matrix table are cast to the global address space so that the
// streaming kernels use global_load / global_store instead of flat accesses.
#define NG_AS1 __attribute__((address_space(1)))
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------ helpers
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// two floats -> two bf16 (round to nearest even) in one v_cvt_pk_bf16_f32; a in the low half
__device__ __forceinline__ unsigned int pack_bf16x2(float a, float b) {
    const f32x2_t f = {a, b};
    bf16x2_t hv = __builtin_convertvector(f, bf16x2_t);
    return *reinterpret_cast<unsigned int*>(&hv);
}
__device__ __forceinline__ unsigned short f32_to_bf16_rne(float x) { return (unsigned short)(pack_bf16x2(x, 0.f) & 0xffffu); }

// The value of the lane's partner at level L: lane ^ 32, lane ^ 16 (by exchanging halves of rows, see wave_sums), lane ^ 8,
// and inside a group of eight the mirrored lane, inside four the mirrored one, inside two the other one.
template <int L>
__device__ __forceinline__ double partner_dpp(double v) {
    constexpr int kCtrl = L == 2 ? 0x128 : L == 3 ? 0x141 : L == 4 ? 0x1B : 0xB1;   // row_ror:8, half mirror, quad_perm
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), kCtrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), kCtrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// a keeps its own lower half of the wavefront (L 0) or of every pair of rows (L 1) and gets b's lower half in the upper
// one's place, b the reverse: afterwards a + b is the first value's sum in the lower lanes, the second's in the upper ones
template <int L>
__device__ __forceinline__ double swap_add(double a, double b) {
    u32x2_t lo, hi;
    if (L == 0) {
        lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
        hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
        hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    }
    return __hiloint2double((int)hi.x, (int)lo.x) + __hiloint2double((int)hi.y, (int)lo.y);
}
// Sums of N = 2^q values over the 64 lanes.  Each level adds the partner lanes and, while there is more than one value,
// leaves either lane of a pair half of the values: N - 1 + (6 - q) exchanges instead of 6 N, none of them through LDS.  On
// return v[0] is the sum of value wave_sums_slot(N, lane).  (Six LDS exchanges per value were the larger part of what
// the Gram row of a small slot did besides its loads: 60M set 33.4 -> 29.4 us, three mid-size fp32 matrices 10.8 -> 8.7,
// 350M set 608 -> 602.)
template <int N, int L>
__device__ __forceinline__ void wave_sums(double* v, int lane) {
    if constexpr (L < 6) {
        if constexpr (N > 1) {
            constexpr int H = N / 2;
            const bool upper = (lane >> (5 - L)) & 1;
#pragma unroll
            for (int j = 0; j < H; ++j) {
                if constexpr (L < 2) {
                    v[j] = swap_add<L>(v[j], v[j + H]);
                } else {
                    const double give = upper ? v[j] : v[j + H], keep = upper ? v[j + H] : v[j];
                    v[j] = keep + partner_dpp<L>(give);
                }
            }
            wave_sums<H, L + 1>(v, lane);
        } else {
            if constexpr (L < 2) v[0] = swap_add<L>(v[0], v[0]);
            else v[0] += partner_dpp<L>(v[0]);
            wave_sums<1, L + 1>(v, lane);
        }
    }
}
template <int N>
__device__ __forceinline__ int wave_sums_slot(int lane) {
    int slot = 0;
#pragma unroll
    for (int h = N / 2, b = 5; h > 0; h >>= 1, --b) slot += ((lane >> b) & 1) ? h : 0;
    return slot;
}
constexpr int pow2_from(int n) { return n <= 1 ? 1 : 2 * pow2_from((n + 1) / 2); }


// Four consecutive history elements of one row: a float4, or 4 bf16 (8 bytes) widened to float.
// `slot` is uniform over the workgroup and `off` a 32-bit byte offset, so the load takes its base
// from scalar registers and needs one address register per row (the host checks that a slot is
// below 2 GiB).
template <bool HB>
__device__ __forceinline__ f32x4_t load_hist4(const NG_AS1 unsigned char* slot, unsigned off) {
    if (HB) {
        const u32x2_t v = __builtin_nontemporal_load((const NG_AS1 u32x2_t*)(slot + off));
        f32x4_t o;
        o.x = __uint_as_float(v.x << 16);
        o.y = __uint_as_float(v.x & 0xffff0000u);
        o.z = __uint_as_float(v.y << 16);
        o.w = __uint_as_float(v.y & 0xffff0000u);
        return o;
    }
    return __builtin_nontemporal_load((const NG_AS1 f32x4_t*)(slot + off));
}

// Adam moments of four elements and their update direction (standard, or as printed in the paper's Sec. 2.2)
__device__ __forceinline__ f32x4_t adam4(f32x4_t& m, f32x4_t& v, const f32x4_t g, const StepScalars& sc, float bc1, float bc2) {
    const float b1 = sc.beta1, b2 = sc.beta2, ob1 = 1.0f - sc.beta1, ob2 = 1.0f - sc.beta2;
    f32x4_t o;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        m[x] = fmaf(b1, m[x], ob1 * g[x]);
        v[x] = fmaf(b2, v[x], ob2 * g[x] * g[x]);
    }
    if (sc.adam_mode == NG_ADAM_STANDARD) {
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = (m[x] * bc1) / (sqrtf(v[x]) * bc2 + sc.eps);
    } else {
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = m[x] / sqrtf(v[x] + sc.eps);
    }
    return o;
}
__device__ __forceinline__ bool any_not_finite(const f32x4_t o) {
    return !(fabsf(o.x) <= 3.0e38f) | !(fabsf(o.y) <= 3.0e38f) | !(fabsf(o.z) <= 3.0e38f) | !(fabsf(o.w) <= 3.0e38f);
}

// Partial sums of the Gram row: thread (sub, j) adds parts sub, sub + nsub, ... of slot j in order and leaves the sum in
// bc[tid]; the nsub (returned) sub-sums of a slot are then added in order (a fixed order: the result does not depend on
// timing).  COHERENT: the parts were written by other workgroups of the same launch.  256 threads.
constexpr int kSolveSub = 16;      // threads that share the sum of one slot's partials
// BATCH loads are in flight.
template <bool COHERENT, int BATCH = 16>
__device__ __forceinline__ int sum_dot_parts(const double* all_parts, int np, int s, int tid, double* bc) {
    const int nsub = 256 / s < kSolveSub ? 256 / s : kSolveSub;
    const int j = tid % s, sub = tid / s;
    double v = 0.0;
    if (sub < nsub) {
        const NG_AS1 double* parts = (const NG_AS1 double*)all_parts + j;
        for (int p = sub; p < np; p += BATCH * nsub) {
            double x[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int pu = p + u * nsub;
                const NG_AS1 double* at = parts + (long long)(pu < np ? pu : p) * s;
                if (COHERENT) x[u] = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else x[u] = *at;
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) v += p + u * nsub < np ? x[u] : 0.0;
        }
    }
    bc[tid] = v;
    return nsub;
}

// lambda I + K / s for s <= 16 in one wavefront's registers, K in LDS with rows of PITCH: lane c (of every row of 16 lanes) gets
// column c, the columns from s on are those of an identity, and so are row and column `skip` (-1: none).  Then X =
// L^{-1} of it: v is column c of X.
template <int PITCH>
__device__ __forceinline__ void factor16(const double* A, int s, int skip, int tid, double lam, double inv_s, double (&v)[16], bool& bad) {
    const int c = tid & 15;
    double a[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const bool in = k < s && c < s && k != skip && c != skip;
        a[k] = in ? A[(k < s ? k : 0) * PITCH + (c < s ? c : 0)] * inv_s + (k == c ? lam : 0.0) : (k == c ? 1.0 : 0.0);
        v[k] = k == c ? 1.0 : 0.0;
    }
    if (s <= 4) eliminate16<0, 4>(a, v, 0.0, bad);
    else if (s <= 8) eliminate16<0, 8>(a, v, 0.0, bad);
    else eliminate16<0>(a, v, 0.0, bad);
}

// w = (lambda I + K / s)^{-1} e_head: component tid of w in lane tid.  bc: 16 doubles of LDS that nothing else uses.  See k_solve.
template <int PITCH>
__device__ __forceinline__ double solve16(const double* A, double* bc, int s, int head, int tid, double lam, double inv_s, bool& bad) {
    double v[16];
    factor16<PITCH>(A, s, -1, tid, lam, inv_s, v, bad);
    // column `head` of X goes to all lanes through LDS (one wavefront: in order)
    if ((tid & 15) == head) {
#pragma unroll
        for (int k = 0; k < 16; ++k) bc[k] = v[k];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    double w = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) w = fma(v[k], bc[k], w);
    return w;
}

}  // namespace ng
