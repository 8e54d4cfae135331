// Cholesky factorisation and inverse of one S x S Hermitian tile (S = 64 or
// 32) in LDS, by one workgroup.
#pragma once

#include <utility>

#include "common.h"

namespace eor {

__device__ inline d4 mfma64(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Every value that steers a loop or branch containing a barrier is passed
// through readfirstlane, so the compiler sees it as wave-uniform and emits
// scalar branches. Left as per-lane values (they come from LDS or global
// memory), the structurizer may place a barrier inside a per-lane loop and
// different waves then execute different numbers of barriers.
__device__ inline int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Hides a lane-dependent value from loop-invariant code motion: addresses
// derived from it are formed where they are used instead of being hoisted
// out of the column loop, where they would stay live (and spill) across
// every tile update.
__device__ inline int opaque(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Lane C of each row of 16 lanes, to all lanes of the row.
template <int C>
__device__ __forceinline__ double row_bcast(double x) {
    constexpr int ROW_NEWBCAST = 0x150;
    const long long v = __builtin_amdgcn_update_dpp((long long)0, __double_as_longlong(x), ROW_NEWBCAST + C, 0xf, 0xf, true);
    return __longlong_as_double(v);
}

__device__ __forceinline__ double read_lane(double x, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
    return __hiloint2double(hi, lo);
}

// Orders one wave's LDS accesses across its lanes. The hardware performs a
// wave's LDS instructions in program order; the wave-scope release, wave
// barrier and acquire keep the compiler from moving a lane's load of a value
// that another lane stores (or a store that another lane's load must precede)
// across this point. No instruction is emitted for it.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave's 16 x 16 block in registers: lane (l16, q) holds row l16, columns
// q + 4 u, of the block (a) and of what the row operations make of the
// identity (v).
struct Block16 {
    double ar[4], ai[4];
    double vr[4], vi[4];
    double piv;  // pivot of row l16
};

// Elimination step C on [block | identity]: rows r > C lose m_r = a_rC / d_C
// times row C. Columns already eliminated are not kept. The pivot is taken
// here: a NaN further right reaches the rows above in a later step.
template <int C>
__device__ __forceinline__ void eliminate(Block16 &b, int l16) {
    constexpr int U = C / 4, Q = C % 4;
    const double d = read_lane(b.ar[U], 16 * Q + C);
    b.piv = l16 == C ? d : b.piv;
    if constexpr (C == 15) return;
    const double cr = __shfl(b.ar[U], 16 * Q + l16), ci = __shfl(b.ai[U], 16 * Q + l16);
    const double inv = l16 > C ? 1.0 / d : 0.0;
    const double mr = cr * inv, mi = ci * inv;
#pragma unroll
    for (int u = (C + 1) / 4; u < 4; ++u) {
        const double xr = b.ar[u], xi = b.ai[u];
        b.ar[u] = fma(row_bcast<C>(xi), mi, fma(row_bcast<C>(xr), -mr, xr));
        b.ai[u] = fma(row_bcast<C>(xr), -mi, fma(row_bcast<C>(xi), -mr, xi));
    }
#pragma unroll
    for (int u = 0; u <= U; ++u) {
        const double xr = b.vr[u], xi = b.vi[u];
        b.vr[u] = fma(row_bcast<C>(xi), mi, fma(row_bcast<C>(xr), -mr, xr));
        b.vi[u] = fma(row_bcast<C>(xr), -mi, fma(row_bcast<C>(xi), -mr, xi));
    }
}

template <int... C>
__device__ __forceinline__ void eliminate_all(Block16 &b, int l16, std::integer_sequence<int, C...>) {
    (eliminate<C>(b, l16), ...);
}

// Blocks of 16 columns of tile j of side S that hold any of n columns.
template <int S>
__device__ inline int real_blocks(int64_t n, int j) {
    const int64_t left = n - (int64_t)S * j;
    return left >= S ? S / 16 : left <= 0 ? 0 : (int)((left + 15) / 16);
}

// D (S x S, column-major with leading dimension S + 1; read are the 16 x 16 blocks
// of the lower triangle, those on the diagonal in both of theirs) becomes L^{-1} of its Cholesky factor L in its lower 16 x 16 blocks (the
// blocks on the diagonal with exact zeros above theirs; the blocks above the
// diagonal hold no result); dg receives the pivots L_cc^2. Called by all NW
// waves (NW >= S / 16), after a barrier that follows the last write of D.
// Returns 0, or the 1-based column of the first pivot that is not positive
// and finite (the same value in every wave); ends with a barrier. Only the
// first nb <= S / 16 block columns are eliminated: what lies beyond has to be
// the identity (the padding of a last tile), which is its own inverse: of the
// 12.7 us below, 3.2 us per block left out.
//
// Bound by a serial chain: the S pivots in turn. Blocked on 16 x 16 blocks so
// that the chain runs in one wave's registers: wave 0 eliminates the block on
// the diagonal and carries the identity along, which gives that block's
// inverse V_kk (the four lane rows share the 32 columns; row C is broadcast
// inside a lane row by DPP, the multipliers across lane rows by a shuffle).
// Beside it, waves 1 .. kb sum the products L_kb,t V_t,j of row kb of the
// inverse. Then, on FP64 MFMA, one wave per block: the panel L_i,kb = D_i,kb
// V_kk^H, the row V_kb,j = -V_kk sum (column j of the inverse is always wave
// j + 1's), and after a barrier the update of the blocks right of kb. Two
// barriers per block column instead of one per column; the leading dimension
// S + 1 keeps every operand read free of bank conflicts. Which wave forms a
// block does not change its bits. At S = 64 with eight waves 12.7 us (30460
// cycles, of which 4 x 4040 are the eliminations, about 60 instructions a step at
// four cycles); with one barrier per column and a separate blocked inverse about
// 60 us more.
template <int S, int NW>
__device__ __forceinline__ int tile_factor(double2 *D, double *dg, int *fail_sh, int nb) {
    constexpr int LD = S + 1;
    const int tid = opaque(threadIdx.x);
    const int wv = uniform(tid >> 6), l16 = tid & 15, q = (tid >> 4) & 3;
    if (tid >= 16 * nb && tid < S) dg[tid] = 1.0;
#pragma unroll 1
    for (int kb = 0; kb < nb; ++kb) {
        const int k0 = 16 * kb;
        // the row of the inverse that this wave forms: block (kb, jb)
        const int jb = wv - 1;
        const bool inv = wv >= 1 && wv <= kb;
        d4 yr = d4{0, 0, 0, 0}, yi = d4{0, 0, 0, 0};
        if (wv == 0) {
            Block16 b;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double2 x = D[(k0 + q + 4 * u) * LD + k0 + l16];
                b.ar[u] = x.x;
                b.ai[u] = x.y;
                b.vr[u] = l16 == q + 4 * u ? 1.0 : 0.0;
                b.vi[u] = 0.0;
            }
            b.piv = 1.0;
            eliminate_all(b, l16, std::make_integer_sequence<int, 16>());
            const double piv = b.piv;
            const unsigned bad = (unsigned)__ballot(!(piv > 0.0) || !isfinite(piv)) & 0xffffu;
            const double is = 1.0 / sqrt(piv);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                D[(k0 + q + 4 * u) * LD + k0 + l16] = make_double2(b.vr[u] * is, b.vi[u] * is);
            if (q == 0) dg[k0 + l16] = piv;
            if (tid == 0) *fail_sh = bad ? k0 + __ffs(bad) : 0;
        } else if (inv) {
            // sum_t L_kb,t V_t,jb: lane holds [q + 4 r][l16], the second
            // operand of the product with V_kk below
            d4 t1 = d4{0, 0, 0, 0}, t2 = d4{0, 0, 0, 0}, t3 = d4{0, 0, 0, 0};
#pragma unroll 1
            for (int t = jb; t < kb; ++t) {
#pragma unroll
                for (int s = 0; s < 16; s += 4) {
                    const double2 l = D[(16 * t + s + q) * LD + k0 + l16];       // L[k0 + l16][16 t + s + q]
                    const double2 v = D[(16 * jb + l16) * LD + 16 * t + s + q];  // V[16 t + s + q][16 jb + l16]
                    t1 = mfma64(l.x, v.x, t1);
                    t2 = mfma64(l.y, v.y, t2);
                    t3 = mfma64(l.x + l.y, v.x + v.y, t3);
                }
            }
            yr = t1 - t2;
            yi = t3 - t1 - t2;
        }
        __syncthreads();
        const int f = uniform(*fail_sh);
        if (f) {
            __syncthreads();  // fail_sh is read by every wave before anything else is written
            return f;
        }
        if (wv > kb && wv < nb) {
            // L_i,kb = D_i,kb V_kk^H, i = wv: lane holds [q + 4 r][l16]
            d4 t1 = d4{0, 0, 0, 0}, t2 = d4{0, 0, 0, 0}, t3 = d4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 16; s += 4) {
                const double2 x = D[(k0 + s + q) * LD + 16 * wv + l16];
                const double2 v = D[(k0 + s + q) * LD + k0 + l16];
                t1 = mfma64(x.x, v.x, t1);
                t2 = mfma64(x.y, v.y, t2);
                t3 = mfma64(x.x + x.y, v.x - v.y, t3);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                D[(k0 + l16) * LD + 16 * wv + q + 4 * r] = make_double2(t1[r] + t2[r], t3[r] - t1[r] + t2[r]);
        } else if (inv) {
            d4 t1 = d4{0, 0, 0, 0}, t2 = d4{0, 0, 0, 0}, t3 = d4{0, 0, 0, 0};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double2 v = D[(k0 + 4 * r + q) * LD + k0 + l16];  // V_kk[l16][4 r + q]
                t1 = mfma64(v.x, yr[r], t1);
                t2 = mfma64(v.y, yi[r], t2);
                t3 = mfma64(v.x + v.y, yr[r] + yi[r], t3);
            }
            yr = -(t1 - t2);
            yi = -(t3 - t1 - t2);
        }
        __syncthreads();
        if (inv) {  // replaces L_kb,jb, which no wave reads any more
#pragma unroll
            for (int r = 0; r < 4; ++r) D[(16 * jb + l16) * LD + k0 + q + 4 * r] = make_double2(yr[r], yi[r]);
        }
        // D_i,j -= L_i,kb L_j,kb^H for kb < j <= i, block idx of the row order.
        // Wave 0 takes only the next block on the diagonal and goes on to
        // eliminate it; the others' blocks and rows of the inverse are read
        // after the next barrier, or by the wave that stored them.
        const int nblk = (nb - 1 - kb) * (nb - kb) / 2;
#pragma unroll 1
        for (int idx = wv; idx < nblk; idx += wv == 0 ? nblk : NW - 1) {
            int i = 0;
            while ((i + 1) * (i + 2) / 2 <= idx) ++i;
            const int j = idx - i * (i + 1) / 2;
            const int ri = k0 + 16 + 16 * i, rj = k0 + 16 + 16 * j;
            d4 t1 = d4{0, 0, 0, 0}, t2 = d4{0, 0, 0, 0}, t3 = d4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 16; s += 4) {
                const double2 x = D[(k0 + s + q) * LD + ri + l16];
                const double2 v = D[(k0 + s + q) * LD + rj + l16];
                t1 = mfma64(x.x, v.x, t1);
                t2 = mfma64(x.y, v.y, t2);
                t3 = mfma64(x.x + x.y, v.x - v.y, t3);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double2 &e = D[(rj + l16) * LD + ri + q + 4 * r];
                e = make_double2(e.x - (t1[r] + t2[r]), e.y - (t3[r] - t1[r] + t2[r]));
            }
        }
        wave_sync();
    }
    __syncthreads();
    return 0;
}

// y = V w for the rows 16 wv + l16 of one wave: the four lanes of a row take
// every fourth column each, up to the end of the row's block on the
// diagonal; every lane of the row returns the sum.
template <int S>
__device__ __forceinline__ double2 tile_solve(const double2 *V, const double2 *w, int wv, int l16, int q) {
    constexpr int LD = S + 1;
    double sr = 0.0, si = 0.0;
#pragma unroll 4
    for (int c = q; c < 16 * (wv + 1); c += 4) {
        const double2 x = V[c * LD + 16 * wv + l16], u = w[c];
        sr += x.x * u.x - x.y * u.y;
        si += x.x * u.y + x.y * u.x;
    }
#pragma unroll
    for (int m = 16; m <= 32; m <<= 1) {
        sr += __shfl_xor(sr, m);
        si += __shfl_xor(si, m);
    }
    return make_double2(sr, si);
}

}  // namespace eor
