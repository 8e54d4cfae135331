// The likelihood of few theta: the tiles of each theta's factor dealt to all
// workgroups of the GPU.
//
// likelihood.hip gives a theta to one workgroup, which fills the GPU with 256
// of them and leaves it idle with few: one theta at n = 4096 took 255 ms on
// one of 256 CUs. Here a unit of work is one 64 x 64 tile of one theta's L,
// computed left-looking by a workgroup of four waves:
//
//   tile (i, j), i > j:  X = A_ij - sum_{k<j} L_ik L_jk^H   as k's tiles finish
//                        L_ij = X Linv_jj^H,  w_i -= L_ij y_j
//   tile (j, j):         D = A_jj + diag(Phi^{-1}) - sum_{k<j} L_jk L_jk^H,
//                        Linv_jj and the pivots, y_j = Linv_jj w_j
//
// with the same sums in the same order as in likelihood.hip, so that a
// theta's result does not depend on which of the two computed it.
//
// Order and progress. Units are numbered by tile columns counted from the
// last one (so that theta of different sizes end together), within a column
// diagonal tiles first, and taken from one counter. A unit needs only tiles
// of earlier columns and of the diagonal of its own column, all of them
// units with smaller numbers, and a unit is taken by a workgroup that is
// already running: every wait is for a running workgroup, whose own waits go
// to smaller numbers yet, so the smallest unfinished unit never waits and
// all waits end, however few workgroups are resident. Row i's tiles finish in
// order (tile (i, j) itself reads tile (i, j - 1)), so one counter per row
// holds its progress. A workgroup publishes a tile by waiting for its stores
// in every wave, a barrier, an agent-scope release and the row's counter
// (the XCDs' L2 caches are not coherent by themselves); a reader polls the
// counter and follows with an agent-scope acquire. A theta that fails sets a
// stop word, its other units return at their next wait, and the last unit
// of a theta clears its progress words for the next launch.
//
// What bounds it: with few theta the chain from one diagonal tile to the next.
// Tile (j+1, j) would be formed, announced and read back between the two;
// instead its unit hands over X (what Linv_jj is still to be applied to) while
// tile (j, j) is being factored, and the unit of tile (j+1, j+1) forms L_(j+1)j
// itself and updates from LDS (last_update); Linv_jj is announced by itself,
// before y_j; and a diagonal tile is formed only in its lower triangle
// (DiagBlocks). A column takes 27 us, 37 without the three (factor 14.4, stored and
// announced 2, seen and loaded 2.3, tile below 4.3, update and move to LDS 4). With
// one workgroup per CU (spread_per_cu) one theta at n = 4096 takes 1.72 ms (253 by
// one workgroup of likelihood.hip), at n = 2048 0.85 (33.5), at n = 200 95 us (168).
// With many theta the FP64 matrix cores and the panels' traffic (each unit streams
// both of its panels alone) bound: 64 theta at n = 4096 78.5 ms = 74.7 TFLOP/s,
// against 79 with 256 theta of one workgroup each, where two tiles share a panel;
// so full rounds stay there (route.h). Nothing is handed over then: with it 64 theta
// at n = 1003 took 1.89 ms, 1.75 without.
#include <algorithm>

#include "like_device.h"
#include "spread.h"

namespace eor {

namespace {

struct SpreadShared {
    double2 Dt[TS * (TS + 1)];  // diagonal tile: D, then Linv; other tiles: Linv of their column
    double2 wv[TS];             // w_j
    double2 ys[TS];             // y_j
    double dg[TS];              // pivots
    double red[2][TS];
    double lnphi[BIN_TABLE];
    double invphi[BIN_TABLE];
    unsigned unit;
    int seen;
    int fail;
};

typedef int32_t __attribute__((address_space(1))) gword;  // a word in global memory

__device__ inline int load_word(const int32_t *p) {
    return __hip_atomic_load((const gword *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void store_word(int32_t *p, int v) {
    __hip_atomic_store((gword *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void wait_vmem() {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
}

// Everything the workgroup's waves have stored and waited for becomes visible
// to the other XCDs. The fence starts a write-back of the XCD's L2
// (buffer_wbl2), which the compiler does not count among the operations that a
// following store waits for once no store of the wave itself is pending: left
// to it, the word that announces a tile could be seen before the tile (1 theta
// in 4000 at n = 1030 came out with a stale line). Waited for explicitly.
__device__ inline void release() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    wait_vmem();
}

// The same for the invalidation that an acquire starts (buffer_inv): complete
// before the barrier that lets the workgroup's other waves load.
__device__ inline void acquire() {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    wait_vmem();
}

// Until rows i and j both have more than k finished tiles: the smaller of the
// two counts, or -1 if the theta has failed. Called by the whole workgroup;
// what the finished tiles' units wrote is visible afterwards.
__device__ inline int wait_tiles(const int32_t *prog, int stop, int i, int j, int k, int slack, int *seen) {
    if (threadIdx.x == 0) {
        int v;
        for (;;) {
            const int a = load_word(prog + i), b = load_word(prog + j), s = load_word(prog + stop);
            v = s ? -1 : min(a, b);
            if (s || v > k) break;
            if (slack <= 0)
                __builtin_amdgcn_s_sleep(1);
            else if (slack == 1)
                __builtin_amdgcn_s_sleep(16);
            else
                __builtin_amdgcn_s_sleep(127);
        }
        acquire();
        *seen = v;
    }
    __syncthreads();
    const int v = uniform(*seen);
    __syncthreads();  // before the next wait's store
    return v;
}

// Every wave's stores so far become visible, then word = v.
__device__ inline void publish(int32_t *word, int v) {
    wait_vmem();
    __syncthreads();
    if (threadIdx.x == 0) {
        release();
        store_word(word, v);
    }
}

constexpr int STAGES = 4;
constexpr int COLB = TS * 16;  // one column of a tile, bytes

// Accumulators of X = A - P Q^H (see tile_update): t1 += .., over the tiles
// k0 .. k1 - 1 of both panels. The prefetch stays inside them.
__device__ __forceinline__ void accumulate(rsrc_t P, rsrc_t Q, int k0, int k1, int voff, d4 t1[4], d4 t2[4], d4 t3[4]) {
    const int beg = k0 * TS, end = k1 * TS;
    Step<4> buf[STAGES];
#pragma unroll
    for (int s0 = 0; s0 < STAGES - 1; ++s0) {
        load_step(buf[s0], P, Q, voff, (beg + 4 * s0) * COLB);
        __builtin_amdgcn_sched_barrier(0);
    }
    int c = beg;  // end > beg
#pragma unroll 1
    do {
        if ((c & (ALIGN_COLS - 1)) == 0) __syncthreads();
#pragma unroll
        for (int u = 0; u < STAGES; ++u) {
            const int cl = min(c + 4 * (u + STAGES - 1), end - 4);
            load_step(buf[(u + STAGES - 1) % STAGES], P, Q, voff, cl * COLB);
            __builtin_amdgcn_sched_barrier(0);
            mma_step(buf[u], t1, t2, t3);
            __builtin_amdgcn_sched_barrier(0);
        }
        c += 4 * STAGES;
    } while (c < end);
}

// sum(k, e) over the tiles k .. e - 1 of rows i and j that have finished, until
// kend; false if the theta has failed.
template <class F>
__device__ __forceinline__ bool as_they_finish(SpreadShared &sh, const int32_t *prog, int stop, int i, int j, int kend,
                                               F &&sum) {
    int k = 0;
#pragma unroll 1
    while (k < kend) {
        const int v = wait_tiles(prog, stop, i, j, k, i <= j + 1 ? j - k - 1 : j - k, &sh.seen);
        if (v < 0) return false;
        const int e = min(v, kend);
        sum(k, e);
        k = e;
    }
    return true;
}

// Accumulators of X = A_ij - sum_{k < kend} L_ik L_jk^H as the tiles finish
// (kend <= j), in tile_update's form: t1, xr = T2, t3; false if the theta has
// failed.
__device__ __forceinline__ bool spread_sum(SpreadShared &sh, const double2 *A, const double2 *L, const int32_t *prog,
                                           int stop, int i, int j, int kend, int w, d4 t1[4], d4 xr[4], d4 t3[4]) {
    const int lane = opaque(threadIdx.x & 63), l16 = lane & 15, q = lane >> 4;
    const int64_t aoff = tile_index(i, j) * TS2 + 16 * w;
    const rsrc_t Ar = make_rsrc(A + aoff, (int64_t)(TS2 - 16 * w) * 16);
    const int voff = (q * TS + l16) * 16;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int so = (16 * cb + 4 * r) * A_COL_BYTES;
            xr[cb][r] = ld1(Ar, voff, so);
            t3[cb][r] = ld1(Ar, voff + 8, so);
        }
    }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
        t1[cb] = d4{0, 0, 0, 0};
        t3[cb] = xr[cb] - t3[cb];
        xr[cb] = -xr[cb];
    }
    const rsrc_t Pr = make_rsrc(L + tile_index(i, 0) * TS2 + 16 * w, (int64_t)kend * TS * COLB);
    const rsrc_t Qr = make_rsrc(L + tile_index(j, 0) * TS2, (int64_t)kend * TS * COLB);
    return as_they_finish(sh, prog, stop, i, j, kend,
                          [&](int k, int e) { accumulate(Pr, Qr, k, e, voff, t1, xr, t3); });
}

// accumulate for a diagonal tile: P = Q, the blocks of DiagBlocks.
__device__ __forceinline__ void accumulate_diag(rsrc_t Q, int k0, int k1, int voff, const DiagBlocks &B, d4 t1[3],
                                                d4 t2[3], d4 t3[3]) {
    const int beg = k0 * TS, end = k1 * TS;
    auto load = [&](DiagStep &s, int col) {
        s.x0 = ld2(Q, voff, col * COLB + 256 * B.x0);
        s.x1 = ld2(Q, voff, col * COLB + 256 * B.x1);
        s.p2 = ld2(Q, voff, col * COLB + 256 * B.p2);
        s.q2 = ld2(Q, voff, col * COLB + 256 * B.q2);
    };
    DiagStep buf[STAGES];
#pragma unroll
    for (int s0 = 0; s0 < STAGES - 1; ++s0) {
        load(buf[s0], beg + 4 * s0);
        __builtin_amdgcn_sched_barrier(0);
    }
    int c = beg;  // end > beg
#pragma unroll 1
    do {
        if ((c & (ALIGN_COLS - 1)) == 0) __syncthreads();
#pragma unroll
        for (int u = 0; u < STAGES; ++u) {
            load(buf[(u + STAGES - 1) % STAGES], min(c + 4 * (u + STAGES - 1), end - 4));
            __builtin_amdgcn_sched_barrier(0);
            mma_diag(buf[u], t1, t2, t3);
            __builtin_amdgcn_sched_barrier(0);
        }
        c += 4 * STAGES;
    } while (c < end);
}

// spread_sum for diagonal tile j.
__device__ __forceinline__ bool spread_sum_diag(SpreadShared &sh, const double2 *A, const double2 *L,
                                                const int32_t *prog, int stop, int j, int kend, const DiagBlocks &B,
                                                d4 t1[3], d4 xr[3], d4 t3[3]) {
    const int lane = opaque(threadIdx.x & 63), l16 = lane & 15, q = lane >> 4;
    const rsrc_t Ar = make_rsrc(A + tile_index(j, j) * TS2, (int64_t)TS2 * 16);
    const int voff = (q * TS + l16) * 16;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int so = (16 * B.c(b) + 4 * r) * A_COL_BYTES + 256 * B.r(b);
            xr[b][r] = ld1(Ar, voff, so);
            t3[b][r] = ld1(Ar, voff + 8, so);
        }
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        t1[b] = d4{0, 0, 0, 0};
        t3[b] = xr[b] - t3[b];
        xr[b] = -xr[b];
    }
    const rsrc_t Qr = make_rsrc(L + tile_index(j, 0) * TS2, (int64_t)kend * TS * COLB);
    return as_they_finish(sh, prog, stop, j, j, kend,
                          [&](int k, int e) { accumulate_diag(Qr, k, e, voff, B, t1, xr, t3); });
}

// X from its accumulators: real part into xr = T2, imaginary part into t3.
template <int NB>
__device__ __forceinline__ void spread_x(const d4 *t1, d4 *xr, d4 *t3) {
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
        const d4 a = t1[cb], b = xr[cb];
        xr[cb] = -(a + b);
        t3[cb] = a - b - t3[cb];
    }
}

// Where the unit of diagonal tile j leaves ln d of a row: in the tile's slot of
// L, above the blocks of Linv (columns 48 and 49, rows 0 .. 15).
__device__ inline double *lnd_of(double2 *L, int j, int row) {
    return (double *)(L + tile_index(j, j) * TS2 + (48 + (row >> 5)) * TS) + (row & 31);
}

// Rows and columns of the element that thread tid moves of lower block b
// (0 .. 9, row order) of a tile of 4 x 4 blocks of 16 x 16.
__device__ inline void lower_block(int b, int tid, int &row, int &col) {
    const int bi = b < 1 ? 0 : b < 3 ? 1 : b < 6 ? 2 : 3, bj = b - bi * (bi + 1) / 2;
    row = 16 * bi + (tid & 15);
    col = 16 * bj + (tid >> 4);
}

// Linv_jj, once published, into Dt.
__device__ __forceinline__ void load_linv(SpreadShared &sh, const double2 *L, int j, int tid) {
    const double2 *V = L + tile_index(j, j) * TS2;
    double2 v[10];
#pragma unroll
    for (int b = 0; b < 10; ++b) {
        int row, col;
        lower_block(b, tid, row, col);
        v[b] = ldd2(V + col * TS + row);
    }
#pragma unroll
    for (int b = 0; b < 10; ++b) {
        int row, col;
        lower_block(b, tid, row, col);
        sh.Dt[col * (TS + 1) + row] = v[b];
    }
}

// The last update of diagonal tile j, k = j - 1, with the tile L_jk formed
// here as well: its unit hands over X = L_jk Linv_kk^-H in tile (j, j)'s slot of
// L while Linv_kk is still being computed, so that from Linv_kk to this
// update nothing passes between workgroups. t1, t2, t3 += L_jk L_jk^H. False if
// the theta has failed.
__device__ __forceinline__ bool last_update(SpreadShared &sh, const double2 *L, const int32_t *prog, int stop, int j,
                                            const DiagBlocks &B, int w, d4 t1[3], d4 t2[3], d4 t3[3]) {
    constexpr int LD = TS + 1;
    if (wait_tiles(prog, stop, stop + 3, stop + 3, j - 1, 1, &sh.seen) < 0) return false;
    const int tid = opaque(threadIdx.x), l16 = tid & 15, q = (tid >> 4) & 3;
    d4 xr[4], xi[4];
    const double2 *X = L + tile_index(j, j) * TS2 + tid;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double2 v = ldd2(X + (4 * cb + r) * 256);
            xr[cb][r] = v.x;
            xi[cb][r] = v.y;
        }
    if (wait_tiles(prog, stop, stop + 4, stop + 4, j - 1, 0, &sh.seen) < 0) return false;
    load_linv(sh, L, j - 1, tid);
    __syncthreads();
    // Y = X Linv^H as in tile_below, last column block first: it alone needs all of X
    d4 yr[4], yi[4];
    const int lt = q * LD + l16;
#pragma unroll
    for (int cb2 = 3; cb2 >= 0; --cb2) {
        d4 s1 = d4{0, 0, 0, 0}, s2 = d4{0, 0, 0, 0}, s3 = d4{0, 0, 0, 0};
#pragma unroll
        for (int cb = 0; cb <= cb2; ++cb) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double2 lv = sh.Dt[lt + (16 * cb + 4 * r) * LD + 16 * cb2];
                const double ar = xr[cb][r], ai = xi[cb][r];
                s1 = mfma64(ar, lv.x, s1);
                s2 = mfma64(ai, lv.y, s2);
                s3 = mfma64(ar + ai, lv.x - lv.y, s3);
            }
        }
        yr[cb2] = s1 + s2;
        yi[cb2] = s3 - s1 + s2;
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // lane holds Y[16w + q + 4r][16 cb + l16]
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            sh.Dt[(16 * cb + l16) * LD + 16 * w + q + 4 * r] = make_double2(yr[cb][r], yi[cb][r]);
    __syncthreads();
#pragma unroll 2
    for (int c = 0; c < TS; c += 4) {
        const double2 *col = sh.Dt + (c + q) * LD + l16;
        mma_diag(DiagStep{col[16 * B.x0], col[16 * B.x1], col[16 * B.p2], col[16 * B.q2]}, t1, t2, t3);
    }
    __syncthreads();
    return true;
}

// PER_CU workgroups of four waves per CU (spread_per_cu). Two: 256 registers a
// wave, and while one waits for a tile the other computes. One, with
// last_update: 256 registers as well (with 512 the accumulators move between the
// two register files, 36 us a column against 31). Neither form spills vector
// registers. GROUP: task, count and off are there; otherwise one instance, slots of
// one size and theta in order (as run-time choices they cost one theta at n = 200
// 95.9 us in place of 95.1).
template <int PER_CU, bool GROUP>
__global__ __launch_bounds__(256, 2) void spread_kernel(SpreadParams a) {
    constexpr bool hand = PER_CU == 1;
    __shared__ SpreadShared sh;
    const int w = uniform(threadIdx.x >> 6);
    // units before the current column, and its tile rows left
    int64_t base = 0;
    int rem = a.n_max;
    for (;;) {
        if (threadIdx.x == 0) {
            const unsigned t = atomicAdd(a.counter, 1u);
            if (t == (unsigned)a.units + gridDim.x - 1) atomicExch(a.counter, 0u);
            sh.unit = t;
        }
        __syncthreads();
        const int64_t t = (unsigned)uniform((int)sh.unit);
        __syncthreads();
        if (t >= a.units) break;
        int count;
        for (;;) {
            count = GROUP ? uniform(a.count[rem]) : a.ntask;
            if (t < base + (int64_t)count * rem) break;
            base += (int64_t)count * rem;
            --rem;
        }
        const int u = (int)((t - base) / count), slot = (int)(t - base - (int64_t)u * count);
        int inst = 0;
        int64_t bt = slot;
        if constexpr (GROUP) {
            const int2 td = a.task[slot];
            inst = uniform(td.x);
            bt = uniform(td.y);
        }
        const InstDesc &I = a.inst[inst];
        const CallDesc C = a.call[inst];
        const int N = uniform(I.N), j = N - rem, i = j + u, stop = a.n_max;
        const double2 *A = uniform_ptr(I.A);
        double2 *L, *yv;
        if constexpr (GROUP) {
            const longlong2 off = a.off[slot];
            L = uniform_ptr(a.Lw + off.x);
            yv = uniform_ptr(a.yw + off.y);
        } else {
            L = uniform_ptr(a.Lw + slot * a.slot_elems);
            yv = uniform_ptr(a.yw + slot * a.slot_y);
        }
        int32_t *prog = uniform_ptr(a.prog + (int64_t)slot * (a.n_max + SPREAD_EXTRA));
        d4 xr[4], xi[4];
        if (u <= 1) __builtin_amdgcn_s_setprio(2);
        if (u > 0) {
            bool ok;
            {
                d4 t1[4];
                ok = spread_sum(sh, A, L, prog, stop, i, j, j, w, t1, xr, xi);
                spread_x<4>(t1, xr, xi);
            }
            if (hand && ok && u == 1) {  // to the unit of diagonal tile i (last_update)
                const int tid = opaque(threadIdx.x);
                double2 *X = L + tile_index(i, i) * TS2 + tid;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) std2(X + (4 * cb + r) * 256, xr[cb][r], xi[cb][r]);
                publish(prog + stop + 3, i);
            }
            if (ok) ok = wait_tiles(prog, stop, j, j, j, 0, &sh.seen) >= 0;  // Linv_jj and y_j
            if (ok) {
                const int tid = opaque(threadIdx.x);
                if (tid < TS) sh.ys[tid] = ldd2(yv + j * TS + tid);
                load_linv(sh, L, j, tid);
                __syncthreads();
                double2 *wi = yv + i * TS;
                tile_below<TS>(sh.Dt, sh.ys, xr, xi, L + tile_index(i, j) * TS2, j == 0 ? I.dbar + i * TS : wi, wi, w);
                publish(prog + i, j + 1);
            }
        } else {
            const int tid = opaque(threadIdx.x), l16 = tid & 15;
            const int nb = real_blocks<TS>(uniform(I.n), j);
            const double *th = C.theta + bt * I.n_k;
            double iv[3];  // 1 / phi of the rows of blocks on the diagonal
#pragma unroll
            for (int b = 1; b < 3; ++b) {
                const int row = j * TS + 16 * (b == 1 ? DiagBlocks(w).x1 : 0) + l16;
                const int32_t bj = I.coef_bin[row];
                iv[b] = bj >= 0 ? 1.0 / (I.bin_scale[bj] * exp10(th[bj])) : I.coef_inv[row];
            }
            iv[0] = 0.0;
            // the theta's check comes with its first unit, ln det Phi with its last
            double ldp = 0.0;
            bool ok = true;
            if (j == 0 || j == N - 1) ldp = theta_terms(I, th, sh.lnphi, sh.invphi, tid);
            if (j == 0 && uniform(ldp == ldp ? 1 : 0) == 0) {
                ok = false;
                if (tid == 0) {
                    write_result(I, C, bt, -1, 0.0, 0.0, 0.0);
                    store_word(prog + stop, 1);
                }
            }
            const DiagBlocks B(w);
            if (ok) {
                d4 t1[3];
                ok = spread_sum_diag(sh, A, L, prog, stop, j, hand && j > 0 ? j - 1 : j, B, t1, xr, xi);
                if (hand && ok && j > 0) ok = last_update(sh, L, prog, stop, j, B, w, t1, xr, xi);
                spread_x<3>(t1, xr, xi);
            }
            if (ok) {
                const int tid = opaque(threadIdx.x), l16 = tid & 15, q = (tid >> 4) & 3;
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    if (w == 3 && b > 0) break;
                    const int lo = (16 * B.c(b) + q) * (TS + 1) + 16 * B.r(b) + l16;  // [16 r + l16][16 c + q]
                    const bool on = B.r(b) == B.c(b);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool diag = on && l16 == q + 4 * r;
                        sh.Dt[lo + 4 * r * (TS + 1)] = make_double2(diag ? xr[b][r] + iv[b] : xr[b][r], xi[b][r]);
                    }
                }
                __syncthreads();
                const int f = tile_factor<TS, 4>(sh.Dt, sh.dg, &sh.fail, nb);
                if (f) {
                    ok = false;
                    if (tid == 0) {
                        write_result(I, C, bt, j * TS + f, 0.0, 0.0, 0.0);
                        store_word(prog + stop, 1);
                    }
                }
            }
            auto store_linv = [&](int tid) {
                double2 *V = L + tile_index(j, j) * TS2;
#pragma unroll
                for (int b = 0; b < 10; ++b) {
                    int r, c;
                    lower_block(b, tid, r, c);
                    const double2 v = sh.Dt[c * (TS + 1) + r];
                    std2(V + c * TS + r, v.x, v.y);
                }
            };
            // to the next diagonal tile, which needs no y_j: 1.4 us earlier
            if (hand && ok && j < N - 1) {
                store_linv(opaque(threadIdx.x));
                publish(prog + stop + 4, j + 1);
            }
            // w_j, which tile (j, j - 1) completes beside the factorisation
            if (ok && j > 0) ok = wait_tiles(prog, stop, j, j, j - 1, 0, &sh.seen) >= 0;
            if (ok) {
                const int tid = opaque(threadIdx.x), l16 = tid & 15, q = (tid >> 4) & 3;
                const int row = 16 * w + l16;
                if (tid < TS) sh.wv[tid] = ldd2(j == 0 ? I.dbar + tid : yv + j * TS + tid);
                __syncthreads();
                const double2 y = tile_solve<TS>(sh.Dt, sh.wv, w, l16, q);
                if (q == 0) std2(yv + j * TS + row, y.x, y.y);
                if (j < N - 1) {
                    if (!hand) store_linv(tid);
                    publish(prog + j, j + 1);
                    // beside the chain of diagonal tiles: the column's ln d
                    if (q == 1) *lnd_of(L, j, row) = log(sh.dg[row]);
                    wait_vmem();
                    __syncthreads();
                    if (tid == 0) {
                        release();
                        atomicAdd(prog + a.n_max + 1, 1);
                    }
                } else {
                    wait_tiles(prog, stop, a.n_max + 1, a.n_max + 1, N - 2, 0, &sh.seen);  // every ln d
                    double acc = 0.0;
                    if (q == 0) {
#pragma unroll 8
                        for (int c = 0; c < N - 1; ++c) acc += abs2(ldd2(yv + c * TS + row));
                        acc += abs2(y);
                    } else if (q == 1) {
#pragma unroll 8
                        for (int c = 0; c < N - 1; ++c) acc += ldg(lnd_of(L, c, row));
                        acc += log(sh.dg[row]);
                    }
                    if (q < 2) sh.red[q][row] = acc;
                    __syncthreads();
                    if (tid < 64) {
                        double quad, logdet;
                        row_sums(sh.red[0][tid], sh.red[1][tid], quad, logdet);
                        if (tid == 0) write_result(I, C, bt, 0, ldp, logdet, quad);
                    }
                }
            }
        }
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();  // the next unit reuses the workgroup's LDS
        if (threadIdx.x == 0) {
            // released, so that no store of this unit to the words can land after they are cleared
            int32_t *done = prog + a.n_max + 2;
            wait_vmem();
            const int before = __hip_atomic_fetch_add((gword *)done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            if (before == N * (N + 1) / 2 - 1) {
                for (int e = 0; e < a.n_max + SPREAD_EXTRA; ++e) store_word(prog + e, 0);
            }
        }
    }
}

}  // namespace

hipError_t launch_spread(const SpreadParams &p, int num_cu, hipStream_t s) {
    const int64_t grid = std::min<int64_t>(p.units, (int64_t)p.per_cu * num_cu);
    if (grid < 1) return hipSuccess;
    const auto kernel = p.off ? (p.per_cu == 1 ? spread_kernel<1, true> : spread_kernel<2, true>)
                              : (p.per_cu == 1 ? spread_kernel<1, false> : spread_kernel<2, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace eor
