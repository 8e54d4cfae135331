// Device code of the likelihood's tile steps: panel update, tile below the
// diagonal, theta terms and result.
#pragma once

#include "common.h"
#include "tile_factor.h"

namespace eor {

constexpr int A_COL_BYTES = TS * 16;  // one column of a storage tile of A
constexpr int ALIGN_COLS = 64;        // panel columns between re-alignments of the workgroup's waves

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

template <class T>
__device__ inline T *uniform_ptr(T *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T *)(((uint64_t)hi << 32) | lo);
}

// A load from global memory. The pointers of the descriptors come out of
// memory, so the compiler would use flat loads for them, and with one of those
// in flight it can only wait for all loads at once (vmcnt(0)): inside the
// panel update that drains the prefetch at every step.
template <class T>
__device__ inline T ldg(const T *p) {
    return *(const T __attribute__((address_space(1))) *)p;
}

// Raw buffer over nbytes at p (a wave-uniform address). A load whose vector
// offset (plus instruction offset) is not below nbytes returns zero and
// touches no memory; the scalar offset is not part of that range check, so
// every load keeps its scalar offset inside the buffer whenever nbytes > 0.
__device__ inline rsrc_t make_rsrc(const void *p, int64_t nbytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)nbytes, 0x00020000);
}

__device__ inline double2 ld2(rsrc_t r, int voff, int soff) {
    const u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    double2 x;
    __builtin_memcpy(&x, &v, sizeof(x));
    return x;
}

__device__ inline double ld1(rsrc_t r, int voff, int soff) {
    const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    double x;
    __builtin_memcpy(&x, &v, sizeof(x));
    return x;
}

typedef double dv2 __attribute__((ext_vector_type(2)));

__device__ inline double2 ldd2(const double2 *p) {
    const dv2 v = ldg((const dv2 *)p);
    return make_double2(v.x, v.y);
}

__device__ inline void std2(double2 *p, double x, double y) {
    *(dv2 __attribute__((address_space(1))) *)p = dv2{x, y};
}

// |y|^2, with the rounding of one fixed sequence of operations.
__device__ __forceinline__ double abs2(double2 y) { return fma(y.x, y.x, y.y * y.y); }

// Operands of one k-step (4 consecutive columns k0..k0+3 of the panels) for
// a factorisation tile of side S = 16 NCB.
template <int NCB>
struct Step {
    double2 p;       // P[16w + l16][k0 + q]
    double2 qv[NCB]; // Q[16cb + l16][k0 + q]
};

// P's descriptor starts at row 16w, Q's at row 0; voff = (S q + l16) * 16.
template <int NCB>
__device__ inline void load_step(Step<NCB> &s, rsrc_t P, rsrc_t Q, int voff, int soff) {
    s.p = ld2(P, voff, soff);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) s.qv[cb] = ld2(Q, voff + 16 * 16 * cb, soff);
}

// t += P Q^H for one k-step with three real products per complex product
// (Gauss): with p = P, q = Q,
//   T1 = qr pr,  T2 = qi pi,  T3 = (qr - qi)(pr + pi)
//   re = T1 + T2,  im = T3 - T1 + T2  (= qr pi - qi pr)
template <int NCB>
__device__ inline void mma_step(const Step<NCB> &s, d4 t1[NCB], d4 t2[NCB], d4 t3[NCB]) {
    const double ps = s.p.x + s.p.y;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        t1[cb] = mfma64(s.qv[cb].x, s.p.x, t1[cb]);
        t2[cb] = mfma64(s.qv[cb].y, s.p.y, t2[cb]);
        t3[cb] = mfma64(s.qv[cb].x - s.qv[cb].y, ps, t3[cb]);
    }
}

// X = A - P Q^H over K columns (K a multiple of S), returned as (xr, xi) in
// the accumulator layout. The A tile goes straight into the accumulators
// (T1 = 0, T2 = -Re A, T3 = Re A - Im A, so that the final combine gives
// -(S - A)), issued before the panel prefetch so that its latency overlaps
// it. A is read from its 64 x 64 storage tiles (column stride 64 whatever S),
// the panels from L's S x S tiles (column stride S). All waves of the
// workgroup re-align once per 64 columns so that the column panel Q, which
// all of them read, is fetched from HBM once.
template <int S, int STAGES>
__device__ __forceinline__ void tile_update(rsrc_t A, rsrc_t P, rsrc_t Q, int K, int voff, int voffA, d4 xr[S / 16],
                                   d4 xi[S / 16]) {
    constexpr int NCB = S / 16;
    constexpr int COLB = S * 16;  // one column of an L tile (or panel), bytes
    d4 t1[NCB], t3[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // A[16w + l16][16cb + 4r + q]: column (16cb + 4r + q), row 16w + l16
            const int so = (16 * cb + 4 * r) * A_COL_BYTES;
            xr[cb][r] = ld1(A, voffA, so);
            t3[cb][r] = ld1(A, voffA + 8, so);
        }
    }
    // The last STAGES - 1 prefetch slots of the loop have no step left to
    // load: they reload step K - 4 (a clamp on the scalar offset) and are
    // never used. The loads stay unconditional, since a guarded load would
    // make the compiler's wait counts conservative at the merge and drain the
    // whole prefetch once per loop iteration; and they stay inside the panel,
    // since past it lies tile (i, j), which this unit stores afterwards (no
    // line of it may be cached on the CU before that store).
    // The prologue keeps its program order (sched_barrier): with step 0's
    // loads issued first, the loop's first wait is the same partial count
    // as in every later iteration instead of a full drain.
    Step<NCB> buf[STAGES];
#pragma unroll
    for (int s0 = 0; s0 < STAGES - 1; ++s0) {
        load_step(buf[s0], P, Q, voff, 4 * s0 * COLB);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        t1[cb] = d4{0, 0, 0, 0};
        t3[cb] = xr[cb] - t3[cb];
        xr[cb] = -xr[cb];  // T2
    }
    d4 *t2 = xr;
    for (int k0 = 0; k0 < K; k0 += 4 * STAGES) {
        if ((k0 & (ALIGN_COLS - 1)) == 0) __syncthreads();
#pragma unroll
        for (int u = 0; u < STAGES; ++u) {
            const int kl = min(k0 + 4 * (u + STAGES - 1), K - 4);
            load_step(buf[(u + STAGES - 1) % STAGES], P, Q, voff, kl * COLB);
            __builtin_amdgcn_sched_barrier(0);
            mma_step(buf[u], t1, t2, t3);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        const d4 a = t1[cb], b = t2[cb];
        xr[cb] = -(a + b);
        xi[cb] = a - b - t3[cb];
    }
}

// The 16 x 16 blocks of a diagonal tile that wave w forms: of the ten in the
// lower triangle (the factorisation reads no others) three each, one the last
// wave, in place of four each with six above the diagonal: 9 instead of 12
// products a step. Block b lies in rows 16 r(b), columns 16 c(b): (x1, x0), (x1,
// x1), (p2, q2); the last wave's second and third are not used. 512 theta at n =
// 4096 599 -> 595 ms, 256 at n = 2048 39.5 -> 38.9 ms; where the update of a
// diagonal tile is part of the chain, one theta at n = 4096 1.87 -> 1.72 ms.
struct DiagBlocks {
    int x0, x1, p2, q2;
    __device__ DiagBlocks(int w) : x0(w == 3 ? 2 : 0), x1(w == 0 ? 1 : w == 1 ? 2 : 3), p2(w == 0 ? 0 : x1), q2(w == 0 ? 0 : 1) {}
    __device__ int r(int b) const { return b < 2 ? x1 : p2; }
    __device__ int c(int b) const { return b == 0 ? x0 : b == 1 ? x1 : q2; }
};

// Rows 16 x + l16 of one step of the panel, for the four slabs of DiagBlocks.
struct DiagStep {
    double2 x0, x1, p2, q2;
};

__device__ __forceinline__ void mma_diag(const DiagStep &s, d4 t1[3], d4 t2[3], d4 t3[3]) {
    auto block = [&](int b, double2 p, double2 q) {
        t1[b] = mfma64(q.x, p.x, t1[b]);
        t2[b] = mfma64(q.y, p.y, t2[b]);
        t3[b] = mfma64(q.x - q.y, p.x + p.y, t3[b]);
    };
    block(0, s.x1, s.x0);
    block(1, s.x1, s.x1);
    block(2, s.p2, s.q2);
}

// tile_update for a diagonal tile of side 64 (A its storage tile, Q the row panel),
// in the blocks of DiagBlocks.
template <int STAGES>
__device__ __forceinline__ void diag_update(rsrc_t A, rsrc_t Q, int K, int voff, const DiagBlocks &B, d4 xr[3],
                                            d4 xi[3]) {
    constexpr int COLB = TS * 16;
    auto load = [&](DiagStep &s, int soff) {
        s.x0 = ld2(Q, voff, soff + 256 * B.x0);
        s.x1 = ld2(Q, voff, soff + 256 * B.x1);
        s.p2 = ld2(Q, voff, soff + 256 * B.p2);
        s.q2 = ld2(Q, voff, soff + 256 * B.q2);
    };
    d4 t1[3], t3[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int so = (16 * B.c(b) + 4 * r) * A_COL_BYTES + 256 * B.r(b);
            xr[b][r] = ld1(A, voff, so);
            t3[b][r] = ld1(A, voff + 8, so);
        }
    }
    DiagStep buf[STAGES];
#pragma unroll
    for (int s0 = 0; s0 < STAGES - 1; ++s0) {
        load(buf[s0], 4 * s0 * COLB);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        t1[b] = d4{0, 0, 0, 0};
        t3[b] = xr[b] - t3[b];
        xr[b] = -xr[b];  // T2
    }
    d4 *t2 = xr;
    for (int k0 = 0; k0 < K; k0 += 4 * STAGES) {
        if ((k0 & (ALIGN_COLS - 1)) == 0) __syncthreads();
#pragma unroll
        for (int u = 0; u < STAGES; ++u) {
            const int kl = min(k0 + 4 * (u + STAGES - 1), K - 4);
            load(buf[(u + STAGES - 1) % STAGES], kl * COLB);
            __builtin_amdgcn_sched_barrier(0);
            mma_diag(buf[u], t1, t2, t3);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const d4 a = t1[b], c = t2[b];
        xr[b] = -(a + c);
        xi[b] = a - c - t3[b];
    }
}

// Column boundary. Tiles of L and entries of w written in one column are read
// in later columns by other waves of the workgroup. The workgroup-scope
// release and acquire of __syncthreads make that safe only through the CU's
// vector L1, which all waves of the workgroup share: the compiler emits no
// wait for stores and no L1 invalidation for them. Both are made explicit
// here: every wave waits until its own stores have completed (vmcnt(0)), and
// after the barrier an agent-scope acquire drops the CU's L1 (buffer_inv), so
// every later load of L or w misses it and is served from L2, where the
// completed stores are. A line cached before a store to it, whether by this
// task or by the previous task in the same slot, can then never be read.
__device__ inline void column_barrier() {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); expcnt and lgkmcnt left at their maximum
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// The barriers of tile_update over K columns, for a group without a tile in
// the current round: every wave of the workgroup must pass the same number.
__device__ inline void panel_barriers(int K) {
    for (int k0 = 0; k0 < K; k0 += ALIGN_COLS) __syncthreads();
}

// Bins whose 1 / phi_b a workgroup keeps in LDS; with more bins the rest are
// formed where they are used.
constexpr int BIN_TABLE = 256;

// ln det Phi over the binned coefficients (NaN where theta or a prior
// variance is invalid), one thread per bin (a thread that did all bins in
// turn spent microseconds in exp10 and log before the first load of A),
// summed in bin order; invphi receives 1 / phi_b of the first BIN_TABLE bins.
// Called by all of at least BIN_TABLE threads.
__device__ __forceinline__ double theta_terms(const InstDesc &I, const double *th, double *lnphi, double *invphi,
                                              int tid) {
    double ldp = 0.0;
    for (int b0 = 0; b0 < I.n_k; b0 += BIN_TABLE) {
        if (b0) __syncthreads();
        const int b = b0 + tid;
        if (tid < BIN_TABLE && b < I.n_k) {
            const double tb = th[b], phi = I.bin_scale[b] * exp10(tb);
            const int cnt = I.bin_count[b];
            const bool bad = !isfinite(tb) || (cnt > 0 && (!(phi > 0.0) || !isfinite(phi)));
            lnphi[tid] = bad ? NAN : cnt > 0 ? (double)cnt * log(phi) : 0.0;
            if (b0 == 0) invphi[tid] = 1.0 / phi;
        }
        __syncthreads();
        for (int e = 0; e < min(BIN_TABLE, I.n_k - b0); ++e) ldp += lnphi[e];
    }
    return ldp;
}

// A tile below the diagonal, from X in the accumulator layout: L_ij = X
// Linv^H, stored at Lt (column-major, leading dimension S), and w_i - L_ij
// y_j from w_old to w_new (which may be the same). Linv and y_j in LDS; wave
// w holds rows 16w .. 16w + 15.
template <int S>
__device__ __forceinline__ void tile_below(const double2 *Linv, const double2 *yj, const d4 xr[S / 16],
                                           const d4 xi[S / 16], double2 *Lt, const double2 *w_old, double2 *w_new,
                                           int w) {
    constexpr int NCB = S / 16;
    const int lane = opaque(threadIdx.x & 63), l16 = lane & 15, q = lane >> 4;
    // Y[i][c'] = sum_c X[i][c] conj(Linv[c'][c]); Linv is lower
    // triangular, so output block cb2 needs column blocks cb <= cb2.
    double2 *Lij = Lt + l16 * S + 16 * w + q;  // Y[16w + q][l16]
    // w_i of row 16w + q + 4 l16, in the lanes l16 < 4; in flight during the products
    const int wrow = 16 * w + q + 4 * (l16 & 3);
    const double2 wold = ldd2(w_old + wrow);
    const int lt = q * (S + 1) + l16;  // Linv[l16][q] in LDS
    double wr[4] = {0, 0, 0, 0}, wi[4] = {0, 0, 0, 0};
#pragma unroll
    for (int cb2 = 0; cb2 < NCB; ++cb2) {
        // x conj(l) with three real products (Gauss):
        //   T1 = xr lr, T2 = xi li, T3 = (xr + xi)(lr - li)
        //   re = T1 + T2, im = xi lr - xr li = T3 - T1 + T2
        d4 t1 = d4{0, 0, 0, 0}, t2 = d4{0, 0, 0, 0}, t3 = d4{0, 0, 0, 0};
#pragma unroll
        for (int cb = 0; cb <= cb2; ++cb) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // Linv[16cb2 + l16][16cb + 4r + q]
                const double2 lv = Linv[lt + (16 * cb + 4 * r) * (S + 1) + 16 * cb2];
                const double ar = xr[cb][r], ai = xi[cb][r];
                t1 = mfma64(ar, lv.x, t1);
                t2 = mfma64(ai, lv.y, t2);
                t3 = mfma64(ar + ai, lv.x - lv.y, t3);
            }
        }
        const d4 yR = t1 + t2, yI = t3 - t1 + t2;
        // lane holds Y[16w + q + 4r][16cb2 + l16]
        const double2 yc = yj[16 * cb2 + l16];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            std2(Lij + 16 * cb2 * S + 4 * r, yR[r], yI[r]);
            wr[r] += yR[r] * yc.x - yI[r] * yc.y;
            wi[r] += yR[r] * yc.y + yI[r] * yc.x;
        }
    }
    // sum over the 16 lanes that share q (the columns), fixed tree
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int m = 8; m >= 1; m >>= 1) {
            wr[r] += __shfl_xor(wr[r], m);
            wi[r] += __shfl_xor(wi[r], m);
        }
    }
    // lane l16 < 4 takes the sums of r = l16
    if (l16 < 4) {
        const double sr = l16 == 0 ? wr[0] : l16 == 1 ? wr[1] : l16 == 2 ? wr[2] : wr[3];
        const double si = l16 == 0 ? wi[0] : l16 == 1 ? wi[1] : l16 == 2 ? wi[2] : wi[3];
        std2(w_new + wrow, wold.x - sr, wold.y - si);
    }
}

// Sums over the rows of a tile, one per lane of a wave, by a fixed tree.
__device__ __forceinline__ void row_sums(double q0, double l0, double &quad, double &logdet) {
    quad = q0;
    logdet = l0;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        quad += __shfl_xor(quad, m);
        logdet += __shfl_xor(logdet, m);
    }
}

// One theta's outputs; info != 0 is a failure.
__device__ __forceinline__ void write_result(const InstDesc &I, const CallDesc &C, int64_t bt, int info, double ldp,
                                             double logdet, double quad) {
    if (C.info) C.info[bt] = info;
    if (info) {
        C.logL[bt] = -INFINITY;
        if (C.terms) {
            for (int e = 0; e < 4; ++e) C.terms[4 * bt + e] = NAN;
        }
        return;
    }
    const double c = I.scal[0], ldphi = ldp + I.fixed_logv;
    C.logL[bt] = (I.khost + I.scal[1]) - ldphi - logdet - (c - quad);
    if (C.terms) {
        C.terms[4 * bt + 0] = logdet;
        C.terms[4 * bt + 1] = quad;
        C.terms[4 * bt + 2] = ldphi;
        C.terms[4 * bt + 3] = c;
    }
}

}  // namespace eor
