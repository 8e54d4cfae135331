// Per-theta marginal likelihood: assemble Sigma = A + Phi^{-1}(theta), factor
// Sigma = L L^H (blocked complex Cholesky, 64 x 64 tiles), forward-solve
// y = L^{-1} dbar, reduce ln det Sigma = 2 sum ln L_jj and ||y||^2 = dbar^H
// Sigma^{-1} dbar, and combine into logL.
//
// One workgroup owns one theta at a time and walks the tiles of L
// left-looking, column by column, with the forward substitution carried
// right-looking alongside (w starts as dbar):
//
//   for each tile column j:
//     diagonal:  D = A_jj + diag(Phi^{-1}) - sum_{k<j} L_jk L_jk^H (MFMA) -> LDS;
//                Linv = L_jj^{-1} of its Cholesky factor and the pivots
//                (tile_factor); y_j = Linv w_j
//     below:     for i > j: X = A_ij - sum_{k<j} L_ik L_jk^H (MFMA)
//                           L_ij = X Linv^H (MFMA, operand from LDS)
//                           w_i -= L_ij y_j
//
// The workgroup is G groups of four waves (G = 1 or 2, the tiles per pass).
// The units of column j are the diagonal tile (unit 0) and the tiles below
// it (unit u = tile j + u); they are dealt to the groups in rounds of G, so
// with G = 2 two tiles are updated at once against one stream of the column
// panel L_j,0..j-1, which the eight waves share through the CU's L1: a
// quarter less HBM traffic than two workgroups on separate thetas. In the
// first round group 1 updates tile j + 1 while group 0 forms the diagonal,
// and holds its accumulators until L_jj^{-1} is ready.
//
// The panel updates and the TRSM form each complex product from three real
// FP64 MFMAs (Gauss's trick) instead of four. A tile's
// accumulators start from A_ij (loaded while the panel prefetch is in
// flight), so the update ends with X itself.
//
// Every entry of L is written once and read back only as an MFMA operand,
// so Sigma is never materialised: A is read once per theta, tile by tile,
// where the factorisation first needs it. Tile-row i of the packed storage
// is a column-major 64 x 64j panel (leading dimension 64), so both operands
// of the update stream with unit stride. Panels and tiles are read through
// raw buffer descriptors built from wave-uniform bases: the k-step offset is
// a scalar register and each lane keeps one 32-bit offset, which leaves the
// vector registers to the accumulators and the prefetch.
//
// The FP64 16x16x4 MFMA takes its A operand as lane l -> A[l%16][l/16], its
// B operand as lane l -> B[l/16][l%16], and returns D[l/16 + 4r][l%16] in
// register r. Accumulator layout (wave w owns tile rows 16w..16w+15): for
// column block cb and register r, lane (q = lane/16, l16 = lane%16) holds
// element [16w + l16][16cb + q + 4r]. Register r of block cb is then
// directly the A operand of a 16x16x4 MFMA over columns 16cb + 4r .. +3,
// which is what the TRSM step consumes without any data movement.
#include "like_device.h"

namespace eor {

namespace {

// LDS of one workgroup, sized for the largest factorisation tile (64).
struct Shared {
    double2 Dt[TS * (TS + 1)];      // diagonal tile: D, then L_jj^{-1} (S x S, leading dimension S + 1)
    double2 wv[TS];                 // w_j = dbar_j - sum_{k<j} L_jk y_k
    double2 ys[TS];                 // y_j
    double dg[TS];                  // pivots of the current diagonal tile
    double red[2][TS];              // per row: sum over j of ln dg, of |y_j|^2
    double lnphi[BIN_TABLE];        // per bin: count ln phi_b (NaN where theta or phi is invalid)
    double invphi[BIN_TABLE];       // per bin: 1 / phi_b
    int task_sh;
    int fail_sh;
};

// One theta of one instance, factored in tiles of side S by a workgroup of NW
// waves: groups of S / 16 waves (each wave owning 16 rows of a tile), so
// NW / (S / 16) tiles of a column are updated per pass of its panel.
template <int S, int STAGES, int NW>
__device__ __forceinline__ void run_task(Shared &sh, double2 *L, double2 *yv, const InstDesc &I, const CallDesc &C,
                                int64_t bt) {
    constexpr int NT = 64 * NW;          // threads of the workgroup
    constexpr int GW = S / 16;           // waves per group
    constexpr int G = NW / GW;           // tiles per pass
    constexpr int NCB = S / 16;          // 16-column blocks of a tile
    constexpr int S2 = S * S;
    constexpr int COLB = S * 16;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int w = uniform((tid >> 6) % GW);    // row slab 16w..16w+15 of the group's tile
    const int grp = uniform((tid >> 6) / GW);  // group within the workgroup
    const int voff = (q * S + l16) * 16;       // lane offset of L panel loads (bytes)
    const int voffA = (q * TS + l16) * 16;     // lane offset of A tile loads (bytes)
    // tiles per side: the instance's N counts 64-wide tiles
    const int N = uniform(I.N) * (TS / S);
    const double2 *Ab = uniform_ptr(I.A);
    const double *th = C.theta + bt * I.n_k;
    const double ldp = theta_terms(I, th, sh.lnphi, sh.invphi, tid);
    const bool ok = ldp == ldp;
    // An invalid theta still falls through to the barrier that closes
    // the task: every lane must reconverge there before tid 0 fetches the
    // next task, or the lanes that skip tid 0's stores can be scheduled
    // around the loop on their own and spin on the old task index.
    const bool valid = uniform(ok ? 1 : 0) != 0;
    if (!valid && tid == 0) write_result(I, C, bt, -1, 0.0, 0.0, 0.0);
    // w = dbar; read back only after the barrier that opens column 0
    if (valid) {
        for (int e = tid; e < N * S; e += NT) {
            const double2 v = ldd2(I.dbar + e);
            std2(yv + e, v.x, v.y);
        }
    }

    // A diagonal tile of side 64 is formed in its lower triangle only
    constexpr bool lower = S == 64;
    const DiagBlocks B(w);

    // Row 16 w + l16 of every diagonal tile, in the waves of group 0: the lane
    // with q = 0 sums |y|^2 over the columns, the one with q = 1 ln dg.
    double acc = 0.0;
    int failed = 0;

    for (int j = 0; valid && j < N && !failed; ++j) {
        column_barrier();  // previous column's readers of Dt and writers of L and w are done
        const int K = j * S;
        const rsrc_t Qr = make_rsrc(L + tile_index(j, 0) * S2, (int64_t)K * COLB);
        const int units = N - j;  // unit 0: diagonal tile; unit u > 0: tile (j + u, j)

        for (int u0 = 0; u0 < units; u0 += G) {
            const int u = u0 + grp;
            const int i = j + u;
            d4 xr[NCB], xi[NCB];
            // Operands of the diagonal phase, in flight during the tile update:
            // w_j, and the bin or inverse variance of this lane's row.
            double2 wj = make_double2(0.0, 0.0);
            int32_t bj[2] = {0, 0};  // row of w, or (lower) rows of x1 and p2
            double ivj[2] = {0.0, 0.0};
            if (u == 0) {
                const int64_t g0 = (int64_t)j * S;
                if (tid < S) wj = ldd2(yv + g0 + tid);
#pragma unroll
                for (int e = 0; e < (lower ? 2 : 1); ++e) {
                    const int64_t row = g0 + 16 * (!lower ? w : e == 0 ? B.x1 : B.p2) + l16;
                    bj[e] = ldg(I.coef_bin + row);
                    ivj[e] = ldg(I.coef_inv + row);
                }
            }
            if (u < units) {
                // ---- X = A_ij - sum_k L_ik L_jk^H, in the accumulator layout.
                // Tile (i, j) of side S is the block at rows S (i mod m), columns
                // S (j mod m) of A's storage tile (i / m, j / m), m = 64 / S.
                constexpr int M = TS / S;
                const int64_t aoff = tile_index(i / M, j / M) * TS2 + (int64_t)(S * (j % M)) * TS + S * (i % M) + 16 * w;
                const rsrc_t Ar = make_rsrc(Ab + aoff, (int64_t)(tile_index(i / M, j / M) + 1) * TS2 * 16 - aoff * 16);
                if (lower && u == 0) {
                    diag_update<STAGES>(make_rsrc(Ab + tile_index(j, j) * TS2, (int64_t)TS2 * 16), Qr, K, voff, B, xr,
                                        xi);
                } else {
                    const rsrc_t Pr = make_rsrc(L + tile_index(i, 0) * S2 + 16 * w, (int64_t)K * COLB);
                    tile_update<S, STAGES>(Ar, Pr, Qr, K, voff, voffA, xr, xi);
                }
            } else {
                panel_barriers(K);  // no tile for this group in the last round
                // Defined on this path too: otherwise the compiler carries the
                // previous round's values across the loop (64 live registers).
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) xr[cb] = xi[cb] = d4{0, 0, 0, 0};
            }
            if (u == 0) {
                // D = X + diag(Phi^{-1}) -> LDS (column-major, leading dimension S + 1)
                const int lane = opaque(threadIdx.x & 63), l16 = lane & 15, q = lane >> 4;
#pragma unroll
                for (int e = 0; e < (lower ? 2 : 1); ++e)
                    if (bj[e] >= 0) ivj[e] = bj[e] < BIN_TABLE ? sh.invphi[bj[e]] : 1.0 / (I.bin_scale[bj[e]] * exp10(th[bj[e]]));
#pragma unroll
                for (int cb = 0; cb < (lower ? 3 : NCB); ++cb) {
                    if (lower && w == 3 && cb > 0) break;
                    const int rb = lower ? B.r(cb) : w, cc = lower ? B.c(cb) : cb;
                    const double iv = ivj[lower && cb == 2 ? 1 : 0];
                    const int lo = (16 * cc + q) * (S + 1) + 16 * rb + l16;  // [16 rb + l16][16 cc + q]
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool diag = cc == rb && l16 == q + 4 * r;
                        sh.Dt[lo + 4 * r * (S + 1)] = make_double2(diag ? xr[cb][r] + iv : xr[cb][r], xi[cb][r]);
                    }
                }
                if (tid < S) sh.wv[tid] = wj;
            }

            if (u0 == 0) {
                __syncthreads();
                const int f = tile_factor<S, NW>(sh.Dt, sh.dg, &sh.fail_sh, real_blocks<S>(uniform(I.n), j));
                if (f) {
                    failed = j * S + f;
                    break;
                }
                // ---- y_j = Linv w_j ---------------------------------------
                if (grp == 0) {
                    const int lane = opaque(threadIdx.x & 63), l16 = lane & 15, q = lane >> 4;
                    const int row = 16 * w + l16;
                    const double2 y = tile_solve<S>(sh.Dt, sh.wv, w, l16, q);
                    if (q == 0) {
                        std2(yv + (int64_t)j * S + row, y.x, y.y);
                        sh.ys[row] = y;
                        acc += abs2(y);
                    } else if (q == 1) {
                        acc += log(sh.dg[row]);
                    }
                }
                __syncthreads();
            }

            if (u > 0 && u < units) {
                // read in later columns only, after column_barrier
                double2 *wi = yv + (int64_t)i * S;
                tile_below<S>(sh.Dt, sh.ys, xr, xi, L + tile_index(i, j) * S2, wi, wi, w);
            }
        }
    }

    // ln det Sigma and |y|^2 over the rows of a tile
    double logdet = 0.0, quad = 0.0;
    if (valid && !failed) {
        if (grp == 0 && q < 2) sh.red[q][16 * w + l16] = acc;
        __syncthreads();
        if (tid < 64) row_sums(tid < S ? sh.red[0][tid] : 0.0, tid < S ? sh.red[1][tid] : 0.0, quad, logdet);
    }
    if (valid && tid == 0) write_result(I, C, bt, failed, ldp, logdet, quad);
}

// Persistent workgroups of NW waves: take (instance, theta) tasks in list
// order (the host sorts them longest first) until the list is exhausted, and
// factor each in the tile side its instance was given (64, or 32).
template <int STAGES, int NW>
__global__ __launch_bounds__(64 * NW, 8 / NW) void likelihood_kernel(LikeParams a) {
    __shared__ Shared sh;
    const int tid = threadIdx.x;
    double2 *L = uniform_ptr(a.Lw + (int64_t)blockIdx.x * a.slot_elems);
    double2 *yv = uniform_ptr(a.yw + (int64_t)blockIdx.x * a.slot_y);
    for (;;) {
        if (tid == 0) {
            // The counter starts at zero and is left at zero: every workgroup
            // takes one number past the list, and the last one taken resets
            // it (a separate launch to clear it took 4 us of a 180 us call).
            const unsigned t = atomicAdd(a.counter, 1u);
            if (t == (unsigned)a.ntask + gridDim.x - 1) atomicExch(a.counter, 0u);
            sh.task_sh = (int)t;
        }
        __syncthreads();
        const int t = uniform(sh.task_sh);
        __syncthreads();
        if (t >= a.ntask) break;
        int inst = 0;
        int64_t bt = t;
        if (a.task) {
            const int2 td = a.task[t];
            inst = uniform(td.x);
            bt = uniform(td.y);
        }
        const InstDesc I = a.inst[inst];
        const CallDesc C = a.call[inst];
        if (uniform(I.ts) == 32)
            run_task<32, STAGES, NW>(sh, L, yv, I, C, bt);
        else
            run_task<64, STAGES, NW>(sh, L, yv, I, C, bt);
        __syncthreads();  // slot workspace is reused by the next task
    }
}

}  // namespace

int like_max_resident_per_cu(int tiles) {
    int nb = 0;
    const hipError_t e =
        tiles == 2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, likelihood_kernel<4, 8>, 512, 0)
                   : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, likelihood_kernel<4, 4>, 256, 0);
    if (e != hipSuccess) return 1;
    return nb > 0 ? nb : 1;
}

hipError_t launch_likelihood(const LikeParams &p, const Tuning &t, int64_t grid, hipStream_t s) {
    if (grid < 1) return hipSuccess;
    const dim3 g((unsigned)grid);
    if (t.tiles == 2) {
        if (t.stages == 2)
            hipLaunchKernelGGL((likelihood_kernel<2, 8>), g, dim3(512), 0, s, p);
        else
            hipLaunchKernelGGL((likelihood_kernel<4, 8>), g, dim3(512), 0, s, p);
    } else {
        if (t.stages == 2)
            hipLaunchKernelGGL((likelihood_kernel<2, 4>), g, dim3(256), 0, s, p);
        else
            hipLaunchKernelGGL((likelihood_kernel<4, 4>), g, dim3(256), 0, s, p);
    }
    return hipGetLastError();
}

}  // namespace eor
