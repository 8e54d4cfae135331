// The end of a pass over T that sums dbar and the scalars: shared by the kernel
// that does only that and the one that splits T into bfloat16 terms.
#pragma once

#include "common.h"

namespace eor {

// A workgroup of 256 threads, 64 columns (thread % 64) by four shares of the rows
// s_lo .. s_hi - 1 of slice blockIdx.y: the shares' sums v of column j go to
// partial; the first column block also writes 1 / sigma_s^2 and the slice's
// share of c and of -sum ln sigma_s^2.
__device__ inline void vectors_finish(double2 sum, int64_t s_lo, int64_t s_hi, int64_t j, int64_t n,
                                      const double *noise_var, const double2 *d, double *invvar, double2 *partial,
                                      double2 *scal_part) {
    __shared__ double2 red[4][64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t split = blockIdx.y;
    red[w][lane] = sum;
    __syncthreads();
    if (w == 0 && j < n) {
        double2 v = red[0][lane];
#pragma unroll
        for (int u = 1; u < 4; ++u) {
            v.x += red[u][lane].x;
            v.y += red[u][lane].y;
        }
        partial[split * n + j] = v;
    }
    if (blockIdx.x != 0) return;
    double c = 0.0, l = 0.0;
    for (int64_t s = s_lo + tid; s < s_hi; s += 256) {
        const double nv = noise_var[s];
        const double2 ds = d[s];
        invvar[s] = 1.0 / nv;
        c += (ds.x * ds.x + ds.y * ds.y) / nv;
        l += log(nv);
    }
    // fixed tree, so that the result does not depend on timing
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        c += __shfl_xor(c, o);
        l += __shfl_xor(l, o);
    }
    __syncthreads();
    if (lane == 0) red[w][0] = make_double2(c, l);
    __syncthreads();
    if (tid == 0) {
        const double2 a = red[0][0], b = red[1][0], e = red[2][0], f = red[3][0];
        scal_part[split] = make_double2((a.x + b.x) + (e.x + f.x), (a.y + b.y) + (e.y + f.y));
    }
}

}  // namespace eor
