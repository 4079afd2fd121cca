// Cholesky elimination of a 16 x 16 block (fp64) inside a wavefront's registers, shared by the refresh's inverse
// factor and the step's s x s solve.
#pragma once

#include <hip/hip_runtime.h>

namespace ng {

// lane K of the lane's own row of 16, in every lane of that row.  (Every lane has a source, so the old value does not
// matter; naming v as it cost a copy and two wait states per broadcast.)
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 | K, 0xf, 0xf, true);
}

// Step K of the elimination of a 16 x 16 block: a holds column lane % 16 of it (in every row of 16 lanes), v
// the columns of a right-hand side.  Row K becomes the row of the factor, scaled by 1 / sqrt(pivot).  A pivot
// below `least` counts as that.  Rows and columns from END on are those of an identity and stay as they are.
template <int K, int END = 16>
__device__ __forceinline__ void eliminate16(double (&a)[16], double (&v)[16], double least, bool& bad) {
    if constexpr (K < END) {
        double d = row_bcast<K>(a[K]);
        d = d < least ? least : d;
        const bool ok = (d > 0.0) && (d < 1.0e300);
        bad |= !ok;
        d = ok ? d : 1.0;
        double rs = __builtin_amdgcn_rsq(d);
        rs = rs * (1.5 - 0.5 * d * rs * rs);
        rs = rs * (1.5 - 0.5 * d * rs * rs);
        v[K] *= rs;
        a[K] *= rs;
        const double wv = -rs * v[K], wa = -rs * a[K];
#pragma unroll
        for (int i = K + 1; i < END; ++i) {
            const double m = row_bcast<K>(a[i]);
            v[i] = fma(m, wv, v[i]);
            a[i] = fma(m, wa, a[i]);
        }
        eliminate16<K + 1, END>(a, v, least, bad);
    }
}

}  // namespace ng
