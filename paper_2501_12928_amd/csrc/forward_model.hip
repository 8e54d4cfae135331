// Instrument forward model: the dense matrix T that takes the model's
// coefficients (a Fourier-domain sky cube) to visibilities, from the uv
// sampling, the primary beam and the model's basis (the instrument model of
// the paper's "Running BayesEoR" section; the paper gives no formula, the
// visibility equation used is stated with eor_forward_model).
//
// For channel f, G_f[b][k] = sum_p E_f[b][p] S[p][k] with
//   E_f[b][p] = A[f][p] exp(-2 pi i nu_f / c (x_b l_p + y_b m_p)),
//   S[p][k]   = exp(2 pi i (u_k l_p + v_k m_p))
// (S does not depend on the channel: a small kernel writes it once). Then
// T[f n_bl + b][e n_uv + k] = norm Z[f][e] G_f[b][k] for every spectral
// mode e. Two kernels:
//  - fm_partial_kernel: one workgroup per 32 x 128 tile of G_f (32
//    baselines, so that each phase factor is made once for up to 128 uv
//    cells) and chunk of the pixels, on FP64 MFMA with three real 16x16x4
//    products per complex step (Gauss). The pixel sum is cut into chunks so
//    that there are several workgroups per resident slot (the chip then
//    stays evenly loaded to the end); each chunk's sum goes to its own
//    partial of G. Two workgroups share a CU (the register budget is bounded
//    for it).
//  - fm_expand_kernel: adds the partials in chunk order and writes T, one
//    thread per (row, uv cell) and all the spectral modes, so that T is
//    written once, in full rows (non-temporal stores: it is not read here).
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "common.h"

namespace eor {

namespace {

constexpr double C_LIGHT = 299792458.0;  // m / s
constexpr int FB = 32;                   // tile: 32 baselines ...
constexpr int FU = 128;                  // ... x 128 uv cells
constexpr int FK = 32;                   // pixels per stage of phase factors
constexpr int FC = 16;                   // pixels: granularity of the chunks

__device__ inline d4 mfma64(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// S[p][k] = exp(2 pi i (u_k l_p + v_k m_p)), [n_pix][n_uv].
__global__ void sky_modes_kernel(const double *__restrict__ lm, const double *__restrict__ uv, int64_t n_pix,
                                 int n_uv, double2 *__restrict__ S) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_pix * n_uv) return;
    const int64_t p = e / n_uv;
    const int k = (int)(e - p * n_uv);
    double s, c;
    sincospi(2.0 * (uv[2 * k] * lm[2 * p] + uv[2 * k + 1] * lm[2 * p + 1]), &s, &c);
    S[e] = make_double2(c, s);
}

struct FmArgs {
    const double *freq, *bl, *lm, *beam;
    const double2 *S;  // [n_pix][n_uv]
    int64_t n_pix, chunk;  // pixels; pixels per chunk (a multiple of FC)
    int n_freq, n_bl, n_uv, nbt, n_chunk;
    double2 *G;  // partials [n_chunk][n_freq n_bl][n_uv]
};

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// S at four pixels from p (uniform) and the lane's four columns: lane group q
// takes pixel p + q; zero past the last pixel. The descriptor covers the rows
// of S that exist, so the prefetch past a chunk's end needs no guard.
struct SStep {
    double2 v[4];
};

__device__ __forceinline__ void load_s(const FmArgs &a, SStep &x, int64_t p, const int voff[4]) {
    const int64_t left = a.n_pix - p;
    const rsrc_t R = __builtin_amdgcn_make_buffer_rsrc(const_cast<double2 *>(a.S + (left <= 0 ? 0 : p * a.n_uv)), (short)0,
                                                       (int)((left <= 0 ? 0 : left < 4 ? left : 4) * a.n_uv * 16), 0x00020000);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const u4 t = __builtin_amdgcn_raw_buffer_load_b128(R, voff[c], 0, 0);
        __builtin_memcpy(&x.v[c], &t, 16);
    }
}

// Direction and beam value of a pixel, from which a phase factor is made.
struct Pix {
    double2 lm;
    double beam;
};

// Pixel p, clamped to the last one.
__device__ __forceinline__ Pix load_pix(const FmArgs &a, int64_t p, const double2 *lm2, const double *beam) {
    const int64_t pc = min(p, a.n_pix - 1);
    return Pix{lm2[pc], beam[pc]};
}

// exp(2 pi i v) from the table of exp(2 pi i k / TURN): with k the nearest of
// the TURN directions, cos and sin of what is left (at most pi / TURN = 0.0123)
// by their Taylor polynomials, whose first terms left out are below 1e-17. The
// product is added to the table's value last, so that its error is one rounding
// beside the table's own. The reduction to |f| <= 1/2 is exact for every v.
// About 25 instructions against sincospi's 75, which cost SIMD time of the matrix
// cores (vector instructions do not run beside another wave's FP64 MFMA): 1.11
// against 1.15 ms for 20000 x 4096. T against 80-bit arithmetic: rms 4.8e-16 to
// 6.6e-16 over four instruments, with sincospi 5.0e-16 to 8.0e-16.
constexpr int TURN = 256;

__device__ __forceinline__ double2 cis_turns(double v, const double2 *turn) {
    const double f = v - rint(v), t = f * TURN, kd = rint(t);
    const double2 e = turn[(int)kd & (TURN - 1)];
    const double r = (t - kd) * (6.283185307179586476925 / TURN), r2 = r * r;
    const double sr = fma(r * r2, fma(r2, 1.0 / 120.0, -1.0 / 6.0), r);
    const double cm = r2 * fma(r2, fma(r2, -1.0 / 720.0, 1.0 / 24.0), -0.5);  // cos r - 1
    return make_double2(e.x + fma(-e.y, sr, e.x * cm), e.y + fma(e.x, sr, e.y * cm));
}

// E for one baseline at the pixel: A exp(-2 pi i nu / c (x l + y m)), with A =
// 0 past the chunk's end.
__device__ __forceinline__ double2 phase(const Pix &x, bool in, double fc, double bx, double by, const double2 *turn) {
    const double2 u = cis_turns(-fc * (bx * x.lm.x + by * x.lm.y), turn);
    const double beam = in ? x.beam : 0.0;
    return make_double2(beam * u.x, beam * u.y);
}

// One workgroup per (uv tile, chunk, channel, baseline tile), baseline tile
// fastest. Wave w owns tile rows (baselines) 16 (w % 2) .. + 15 and uv
// columns 64 (w / 2) .. + 63, as four 16-column blocks. Indices past the last
// baseline or uv cell are clamped to the last one (those rows and columns are
// never written); pixels past the chunk get a beam value of zero and pixels past
// the last a row of zeros of S, so they add nothing.
// S goes from L2 straight to the operand registers, three steps ahead; only the
// phase factors, which are made once for all waves, pass through LDS, in stages
// of 32 pixels with one barrier each; chunks are cut in units of 16 pixels, and
// one that ends with half a stage stops there (all 32 pixels of a last stage
// multiplied took 49 us in place of 33 for 3200 x 144 cells from 144 pixels in
// chunks of 16). (With both staged through LDS, 16 pixels
// and two barriers a stage, the waves of a workgroup held each other up: matrix
// cores busy 71% of a counter run, 1.19 ms for 20000 x 4096. Now 77%, 1.11 ms; at
// the clock it runs at, 2.1 GHz, the products alone take 0.94 ms. Two LDS buffers of
// 8 pixels instead gave 1.18.) At most 256 registers per lane (two workgroups
// per CU): the accumulators then live in ordinary vector registers, with no
// copies to and from the accumulation registers.
__global__ __launch_bounds__(256, 2) void fm_partial_kernel(FmArgs a) {
    __shared__ double2 Es[2][FB][FK + 1];  // [baseline][pixel]
    __shared__ double2 turn[TURN];         // exp(2 pi i k / TURN)
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, q = lane >> 4;
    const int wr = 16 * (w & 1), wc = 64 * (w >> 1);
    int64_t u = blockIdx.x;
    const int bt = (int)(u % a.nbt);
    u /= a.nbt;
    const int f = (int)(u % a.n_freq);
    u /= a.n_freq;
    const int ch = (int)(u % a.n_chunk);
    const int ut = (int)(u / a.n_chunk);
    const int b0 = bt * FB, k0 = ut * FU;
    const int64_t pbeg = ch * a.chunk, pend = min(a.n_pix, pbeg + a.chunk);
    const double fc = a.freq[f] / C_LIGHT;
    const double *beam = a.beam + (int64_t)f * a.n_pix;
    const double2 *lm2 = reinterpret_cast<const double2 *>(a.lm);
    // this thread's phase factors: baseline eb, pixels ep + 8 i of a stage
    const int eb = tid >> 3, ep = tid & 7;
    const int be = min(b0 + eb, a.n_bl - 1);
    const double bx = a.bl[2 * be], by = a.bl[2 * be + 1];
    int voff[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) voff[c] = (q * a.n_uv + min(k0 + wc + 16 * c + l16, a.n_uv - 1)) * 16;

    // Pipeline: S three steps of four pixels ahead; while the products of stage
    // s run, the phase factors of stage s + 1 are made, one between every two
    // steps, from pixel values loaded during stage s - 1, and go to the other LDS
    // buffer, and the pixel values of stage s + 2 are loaded.
    constexpr int NP = FK / 8, AHEAD = 3;
    SStep sb[AHEAD + 1];
    Pix x[NP];
    d4 t1[4], t2[4], t3[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) t1[c] = t2[c] = t3[c] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < NP; ++i) x[i] = load_pix(a, pbeg + ep + 8 * i, lm2, beam);
    {
        static_assert(TURN == 256, "one entry per thread");
        double sn, cs;
        sincospi(tid * (2.0 / TURN), &sn, &cs);
        turn[tid] = make_double2(cs, sn);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        if (8 * i == FC && pbeg + FC >= pend) break;
        Es[0][eb][ep + 8 * i] = phase(x[i], pbeg + ep + 8 * i < pend, fc, bx, by, turn);
        x[i] = load_pix(a, pbeg + FK + ep + 8 * i, lm2, beam);
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
        load_s(a, sb[u], pbeg + 4 * u, voff);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    int buf = 0;
    // Step u of the stage from p0; in a full stage, the phase factors of the next.
    auto step = [&](int64_t p0, int u, bool full) __attribute__((always_inline)) {
        if (full || u < FC / 4 - AHEAD) {
            load_s(a, sb[(u + AHEAD) % (AHEAD + 1)], p0 + 4 * (u + AHEAD), voff);
            __builtin_amdgcn_sched_barrier(0);
        }
        const double2 av = Es[buf][wr + l16][4 * u + q];
        const double as = av.x + av.y;
        const SStep &s = sb[u % (AHEAD + 1)];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            t1[c] = mfma64(av.x, s.v[c].x, t1[c]);
            t2[c] = mfma64(av.y, s.v[c].y, t2[c]);
            t3[c] = mfma64(as, s.v[c].x + s.v[c].y, t3[c]);
        }
        if (full && u % 2 == 1) {
            const int64_t p = p0 + FK + ep + 4 * (u - 1);
            Es[buf ^ 1][eb][ep + 4 * (u - 1)] = phase(x[u / 2], p < pend, fc, bx, by, turn);
            x[u / 2] = load_pix(a, p + FK, lm2, beam);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int64_t p0 = pbeg;
#pragma unroll 1
    for (; p0 + FC < pend; p0 += FK, buf ^= 1) {
#pragma unroll
        for (int u = 0; u < FK / 4; ++u) step(p0, u, true);
        __syncthreads();
    }
    if (p0 < pend) {  // a chunk may end with half a stage
#pragma unroll
        for (int u = 0; u < FC / 4; ++u) step(p0, u, false);
    }
    // lane holds G[b0 + wr + q + 4 r][k0 + wc + 16 c + l16]:
    // re = T1 - T2, im = T3 - T1 - T2
    double2 *G = a.G + ((int64_t)ch * a.n_freq + f) * a.n_bl * a.n_uv;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int b = b0 + wr + q + 4 * r;
        if (b >= a.n_bl) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int k = k0 + wc + 16 * c + l16;
            if (k >= a.n_uv) continue;
            G[(int64_t)b * a.n_uv + k] = make_double2(t1[c][r] - t2[c][r], t3[c][r] - t1[c][r] - t2[c][r]);
        }
    }
}

typedef double dv2 __attribute__((ext_vector_type(2)));

struct ExpArgs {
    const double2 *G;  // partials [n_chunk][rows][n_uv]
    const double2 *Z;  // [n_freq][n_eta]
    int64_t rows;      // n_freq n_bl
    int n_bl, n_uv, n_eta, n_chunk;
    double norm;
    double2 *T;
    int64_t ldT;
};

// T[row][e n_uv + k] = norm Z[f][e] sum_chunks G[chunk][row][k], row = f n_bl + b.
__global__ __launch_bounds__(256) void fm_expand_kernel(ExpArgs a) {
    const int64_t total = a.rows * a.n_uv;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = e / a.n_uv;
        const int k = (int)(e - row * a.n_uv);
        const int f = (int)(row / a.n_bl);
        double2 g = a.G[e];
        for (int c = 1; c < a.n_chunk; ++c) {
            const double2 h = a.G[(int64_t)c * total + e];
            g.x += h.x;
            g.y += h.y;
        }
        // T is written once and not read here: non-temporal stores
        dv2 *Trow = reinterpret_cast<dv2 *>(a.T + row * a.ldT + k);
        const double2 *Zf = a.Z + (int64_t)f * a.n_eta;
        for (int m = 0; m < a.n_eta; ++m) {
            const double2 z = Zf[m];
            const double zr = a.norm * z.x, zi = a.norm * z.y;
            const dv2 t = {zr * g.x - zi * g.y, zr * g.y + zi * g.x};
            __builtin_nontemporal_store(t, Trow + (int64_t)m * a.n_uv);
        }
    }
}

}  // namespace

}  // namespace eor

extern "C" eor_status eor_forward_model(int64_t n_freq, int64_t n_bl, int64_t n_pix, int64_t n_uv, int64_t n_eta,
                                        const double *freq, const double *bl, const double *lm, const double *beam,
                                        const double *uv, const double *Z, double norm, double *T, int64_t ldT,
                                        void *stream) {
    if (n_freq < 1 || n_bl < 1 || n_pix < 1 || n_uv < 1 || n_eta < 1 || n_freq > 65535 ||
        n_bl > (int64_t)65535 * 32 || n_uv > (int64_t)65535 * 64 || n_eta > (1 << 20) || n_pix > ((int64_t)1 << 31) ||
        n_pix * n_uv > ((int64_t)1 << 34))
        return eor::fail_status(EOR_ERR_ARG, "eor_forward_model: sizes out of range");
    if (!freq || !bl || !lm || !beam || !uv || !Z || !T)
        return eor::fail_status(EOR_ERR_ARG, "eor_forward_model: NULL array");
    if (ldT < n_eta * n_uv) return eor::fail_status(EOR_ERR_ARG, "eor_forward_model: ldT < n_eta n_uv");
    if (!std::isfinite(norm)) return eor::fail_status(EOR_ERR_ARG, "eor_forward_model: norm is not finite");
    // Pixel chunks: enough workgroups for several per resident slot (about
    // 2048 in all), at most 16 chunks and at least 16 pixels per chunk.
    const int64_t nbt = (n_bl + eor::FB - 1) / eor::FB, nut = (n_uv + eor::FU - 1) / eor::FU;
    const int64_t base = n_freq * nbt * nut, stages = (n_pix + eor::FC - 1) / eor::FC;
    int64_t want = (2048 + base - 1) / base;
    want = std::max<int64_t>(1, std::min<int64_t>({want, 16, stages}));
    int64_t chunk = ((stages + want - 1) / want) * eor::FC;
    // A workgroup's table and first phase factors cost as much as 16 pixels, so
    // where the chip (two workgroups per CU) stays full, two units a chunk: 3200 x 144
    // cells from 144 pixels 32.0 us against 35.5 (and 3.7 less for the writes of fewer
    // partials), 2400 x 128 from 169 pixels 21.8 against 24.8.
    if (chunk == eor::FC && base * want > 512) chunk = 2 * eor::FC;
    const int64_t n_chunk = (n_pix + chunk - 1) / chunk;
    const int64_t units = base * n_chunk, rows = n_freq * n_bl;
    if (units > (int64_t)INT32_MAX)
        return eor::fail_status(EOR_ERR_ARG, "eor_forward_model: more than 2^31 - 1 tiles");
    if (rows * n_uv > ((int64_t)1 << 40))  // keeps the partials' byte count far from overflow
        return eor::fail_status(EOR_ERR_ARG, "eor_forward_model: n_freq n_bl n_uv > 2^40");
    hipStream_t hs = (hipStream_t)stream;
    double2 *S = nullptr, *G = nullptr;
    hipError_t e = hipMallocAsync((void **)&S, (size_t)n_pix * n_uv * sizeof(double2), hs);
    if (e != hipSuccess) return eor::hip_status(e, "eor_forward_model scratch");
    e = hipMallocAsync((void **)&G, (size_t)n_chunk * rows * n_uv * sizeof(double2), hs);
    if (e != hipSuccess) {
        (void)hipFreeAsync(S, hs);
        return eor::hip_status(e, "eor_forward_model scratch");
    }
    const int64_t ns = n_pix * n_uv;
    hipLaunchKernelGGL(eor::sky_modes_kernel, dim3((unsigned)((ns + 255) / 256)), dim3(256), 0, hs, lm, uv, n_pix,
                       (int)n_uv, S);
    eor::FmArgs a;
    a.freq = freq;
    a.bl = bl;
    a.lm = lm;
    a.beam = beam;
    a.S = S;
    a.n_pix = n_pix;
    a.chunk = chunk;
    a.n_freq = (int)n_freq;
    a.n_bl = (int)n_bl;
    a.n_uv = (int)n_uv;
    a.nbt = (int)nbt;
    a.n_chunk = (int)n_chunk;
    a.G = G;
    hipLaunchKernelGGL(eor::fm_partial_kernel, dim3((unsigned)units), dim3(256), 0, hs, a);
    eor::ExpArgs x;
    x.G = G;
    x.Z = reinterpret_cast<const double2 *>(Z);
    x.rows = rows;
    x.n_bl = (int)n_bl;
    x.n_uv = (int)n_uv;
    x.n_eta = (int)n_eta;
    x.n_chunk = (int)n_chunk;
    x.norm = norm;
    x.T = reinterpret_cast<double2 *>(T);
    x.ldT = ldT;
    const int64_t eblocks = std::min<int64_t>((rows * n_uv + 255) / 256, 4096);
    hipLaunchKernelGGL(eor::fm_expand_kernel, dim3((unsigned)eblocks), dim3(256), 0, hs, x);
    e = hipGetLastError();
    (void)hipFreeAsync(G, hs);
    (void)hipFreeAsync(S, hs);
    return e == hipSuccess ? EOR_OK : eor::hip_status(e, "eor_forward_model");
}
