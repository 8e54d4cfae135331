// Reduced-precision forms of A = W^H W, W = N^{-1/2} T (rows scaled by
// 1/sigma_s), stored in FP64 in the same packed lower tiles as the FP64 path.
//
// FP32: W is formed in FP64 and rounded to complex64; each 64 x 64 tile is a
//   sum of FP32 MFMA (16x16x4) products accumulated in FP32 over chunks of
//   64 rows of W; the chunk partials are added into FP64 accumulators.
// BF16x3: W is formed in FP64, rounded to FP32, and every real and imaginary
//   part x is split into three bfloat16 terms x = h + m + l (+ a remainder
//   below 2^-24 |x|); a real product x y keeps the six leading cross products
//   hh' + hm' + mh' + hl' + mm' + lh' on BF16 MFMA (16x16x32) with FP32
//   accumulation, and again the 64-row chunk partials go to FP64.
// BF16x2: the cheaper split into two terms x = h + l (a remainder below
//   2^-16 |x|) and the three leading products hh' + hl' + lh'.
//
// Both MFMAs return D[4(l/16) + r][l%16] in register r (FP32 16x16x4 and
// BF16 16x16x32), with the A operand lane l = A[l%16][k-group l/16] and the B
// operand lane l = B[k-group l/16][l%16].
#include <algorithm>

#include "common.h"
#include "vectors.h"

namespace eor {

namespace {

// Rows of W accumulated in FP32 before the partial goes to FP64. The FP32
// error of a chunk grows with its length (positive diagonal terms make it
// systematic); 64 rows keep logL about ten times closer to FP64 than 256 at
// a negligible cost, and a multiple of 64 is what the split transpose needs.
constexpr int CHUNK_ROWS = 64;

__device__ inline f4 mfma32(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef short s8v __attribute__((ext_vector_type(8)));

__device__ inline f4 mfma_bf16(bf8 a, bf8 b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ inline void tile_of(int64_t t, int64_t &i, int64_t &j) {
    int64_t r = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (r * (r + 1) / 2 > t) --r;
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    i = r;
    j = t - r * (r + 1) / 2;
}

// Store a tile held as FP64 accumulators: lane holds
// A[64 ti + 16 w + l16][64 tj + 16 cb + 4 q + r].
__device__ inline void store_tile(double2 *__restrict__ Ap, int64_t ti, int64_t tj, int64_t n,
                                  const double (&sR)[4][4], const double (&sI)[4][4], int w, int l16,
                                  int q) {
    double2 *tile = Ap + tile_index(ti, tj) * TS2;
    const int row = 16 * w + l16;
    const int64_t grow = TS * ti + row;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int col = 16 * cb + 4 * q + r;
            const int64_t gcol = TS * tj + col;
            double2 v = make_double2(sR[cb][r], sI[cb][r]);
            if (grow == gcol) v.y = 0.0;
            if (grow >= n || gcol >= n) v = make_double2(grow == gcol ? 1.0 : 0.0, 0.0);
            tile[col * TS + row] = v;
        }
    }
}

// ---------------------------------------------------------------- FP32 ----

// W32[s][j] = complex64(T[s][j] / sigma_s), zero in the padding, and from the same
// pass over T the vectors (vectors_finish): a workgroup takes 64 columns and the
// row tiles of a slice. Reading T once instead of twice: the whole precompute
// 20000 x 4096 10.95 -> 10.76 ms, 8000 x 2048 1.369 -> 1.345 ms, 3000 x 1003 233 ->
// 228 us.
__global__ __launch_bounds__(256) void w32_kernel(const double2 *__restrict__ T, int64_t ldT, int64_t m, int64_t n,
                                                  const double *__restrict__ noise_var,
                                                  const double2 *__restrict__ d, int64_t m_pad, int64_t n_pad,
                                                  int64_t rows_per, float2 *__restrict__ W,
                                                  double *__restrict__ invvar, double2 *__restrict__ partial,
                                                  double2 *__restrict__ scal_part) {
    const int64_t j = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63), s_lo = (int64_t)blockIdx.y * rows_per;
    const int64_t s_end = s_lo + rows_per < m_pad ? s_lo + rows_per : m_pad;  // multiples of 64
    double sr = 0.0, si = 0.0;
#pragma unroll 4
    for (int64_t s = s_lo + (threadIdx.x >> 6); s < s_end; s += 4) {
        float2 v = make_float2(0.f, 0.f);
        if (s < m && j < n) {
            const double2 t = T[s * ldT + j], ds = d[s];
            const double wv = 1.0 / noise_var[s], sc = sqrt(wv);
            v = make_float2((float)(t.x * sc), (float)(t.y * sc));
            sr += (t.x * ds.x + t.y * ds.y) * wv;
            si += (t.x * ds.y - t.y * ds.x) * wv;
        }
        W[s * n_pad + j] = v;
    }
    vectors_finish(make_double2(sr, si), s_lo, s_end < m ? s_end : m, j, n, noise_var, d, invvar, partial, scal_part);
}

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

__device__ inline rsrc_t make_rsrc(const void *p, int64_t nbytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)nbytes, 0x00020000);
}

__device__ inline float2 ldf2(rsrc_t r, int voff) {
    const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, 0);
    float2 x;
    __builtin_memcpy(&x, &v, sizeof(x));
    return x;
}

// Operands of one 4-row step of W (row s0 + q in lane group q): the tile-row
// block W[s][64 ti + 16 w + l16] and the four tile-column blocks
// W[s][64 tj + 16 cb + l16].
struct F32Step {
    float2 a;
    float2 b[4];
};

constexpr int F32_STAGES = 4;  // steps in flight; divides the 16 steps of a chunk

// One work unit: tile u % tiles over rows [split * rows_per, ...), split =
// u / tiles, rows_per a multiple of CHUNK_ROWS; W is zero-padded to m_pad
// rows and n_pad columns, so every operand load is unguarded (the prefetch
// past the end of W reads zero through the descriptor). With one split the
// tile goes to A directly; otherwise to its slot of `out` (FP64), and the
// splits are added in a fixed order afterwards.
__global__ __launch_bounds__(256, 2) void herk_fp32_kernel(const float2 *__restrict__ W, int64_t m_pad,
                                                           int64_t n_pad, int64_t n, int64_t tiles,
                                                           int64_t rows_per, int splits,
                                                           double2 *__restrict__ out) {
    const int64_t unit = blockIdx.x;
    const int64_t tile = unit % tiles, split = unit / tiles;
    int64_t ti, tj;
    tile_of(tile, ti, tj);
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r0 = split * rows_per;
    const int64_t r1 = r0 + rows_per < m_pad ? r0 + rows_per : m_pad;
    // D[c][r] = sum_s b[s][c] conj(a[s][r]):  b = W[s][64 tj + c], a = W[s][64 ti + r]
    const int va = (int)((q * n_pad + TS * ti + 16 * w + l16) * 8);
    int vb[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) vb[cb] = (int)((q * n_pad + TS * tj + 16 * cb + l16) * 8);
    auto rows_at = [&](int64_t s) {
        const int64_t left = m_pad - s;
        return make_rsrc(W + (left <= 0 ? 0 : s * n_pad), left <= 0 ? 0 : (left < 4 ? left : 4) * n_pad * 8);
    };
    auto load = [&](F32Step &st, int64_t s) {
        const rsrc_t R = rows_at(s);
        st.a = ldf2(R, va);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) st.b[cb] = ldf2(R, vb[cb]);
    };

    double sR[4][4], sI[4][4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) sR[cb][r] = sI[cb][r] = 0.0;

    F32Step buf[F32_STAGES];
#pragma unroll
    for (int s0 = 0; s0 < F32_STAGES - 1; ++s0) {
        load(buf[s0], r0 + 4 * s0);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int64_t c0 = r0; c0 < r1; c0 += CHUNK_ROWS) {
        __syncthreads();  // keep the four waves together on the shared column block
        f4 aR[4], aI[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) aR[cb] = aI[cb] = f4{0, 0, 0, 0};
        for (int64_t s0 = c0; s0 < c0 + CHUNK_ROWS; s0 += 4 * F32_STAGES) {
#pragma unroll
            for (int u = 0; u < F32_STAGES; ++u) {
                load(buf[(u + F32_STAGES - 1) % F32_STAGES], s0 + 4 * (u + F32_STAGES - 1));
                const F32Step &st = buf[u];
                const float nai = -st.a.y;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) {
                    aR[cb] = mfma32(st.b[cb].x, st.a.x, aR[cb]);
                    aR[cb] = mfma32(st.b[cb].y, st.a.y, aR[cb]);
                    aI[cb] = mfma32(st.b[cb].y, st.a.x, aI[cb]);
                    aI[cb] = mfma32(st.b[cb].x, nai, aI[cb]);
                }
            }
        }
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sR[cb][r] += (double)aR[cb][r];
                sI[cb][r] += (double)aI[cb][r];
            }
    }
    if (splits == 1) {
        store_tile(out, ti, tj, n, sR, sI, w, l16, q);
        return;
    }
    // partial tile, column-major: lane holds [16 w + l16][16 cb + 4 q + r]
    double2 *dst = out + (split * tiles + tile) * TS2;
    const int row = 16 * w + l16;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[(16 * cb + 4 * q + r) * TS + row] = make_double2(sR[cb][r], sI[cb][r]);
}

// -------------------------------------------------------------- BF16x3 ----

__device__ inline unsigned short bf16_bits(float x) {
    // round to nearest even
    unsigned int u = __float_as_uint(x);
    const unsigned int lsb = (u >> 16) & 1u;
    u += 0x7fffu + lsb;
    return (unsigned short)(u >> 16);
}

__device__ inline float bf16_to_float(unsigned short h) { return __uint_as_float(((unsigned int)h) << 16); }

// Split planes, transposed and cut into steps of 32 rows: plane p (0..5 = re h,
// m, l, im h, m, l) of step t holds P[t][p][j][r] for the rows s = 32 t + r <
// m_pad (zero in the padding), so that a step of 64 columns of one plane, which
// the product copies to LDS, is 4 KiB in one piece. One block transposes a
// 64 x 64 tile of W through LDS.
constexpr int BF_STEP = 32;

//
// The same pass over T gives the vectors, as vectors_kernel does for the other
// precisions: a workgroup takes 64 columns and the row tiles of a slice, with
// the slice's partial sums of dbar and, in the first column block, 1 / sigma^2 and
// the share of the scalars. Reading T once instead of twice, and a launch less:
// the whole precompute 8000 x 2048 1.112 -> 1.089 ms (three terms), 797 -> 736 us
// (two), 1500 x 500 110 -> 99 us, 480 x 200 93 -> 80 us.
template <int NTERM>
__global__ __launch_bounds__(256) void split_kernel(const double2 *__restrict__ T, int64_t ldT,
                                                    int64_t m, int64_t n, const double *__restrict__ noise_var,
                                                    const double2 *__restrict__ d, int64_t n_pad, int64_t row_tiles,
                                                    int64_t tiles_per, unsigned short *__restrict__ P,
                                                    double *__restrict__ invvar, double2 *__restrict__ partial,
                                                    double2 *__restrict__ scal_part) {
    __shared__ __align__(4) unsigned short sh[2 * NTERM][64][66];
    const int64_t j0 = (int64_t)blockIdx.x * 64, t_lo = (int64_t)blockIdx.y * tiles_per;
    const int64_t t_hi = t_lo + tiles_per < row_tiles ? t_lo + tiles_per : row_tiles;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int col = threadIdx.x >> 2, ch = threadIdx.x & 3;  // 8 rows of a column per thread
    const int64_t j = j0 + tx;
    double sr = 0.0, si = 0.0;
    for (int64_t tile = t_lo; tile < t_hi; ++tile) {
        const int64_t s0 = 64 * tile;
#pragma unroll 4
        for (int rr = ty; rr < 64; rr += 4) {
            const int64_t s = s0 + rr;
            float xs[2] = {0.f, 0.f};
            if (s < m && j < n) {
                const double2 t = T[s * ldT + j], ds = d[s];
                const double wv = 1.0 / noise_var[s], sc = sqrt(wv);
                xs[0] = (float)(t.x * sc);
                xs[1] = (float)(t.y * sc);
                sr += (t.x * ds.x + t.y * ds.y) * wv;
                si += (t.x * ds.y - t.y * ds.x) * wv;
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                // each term is the bfloat16 nearest what the earlier ones leave
                float x = xs[c];
#pragma unroll
                for (int k = 0; k < NTERM; ++k) {
                    const unsigned short b = bf16_bits(x);
                    sh[NTERM * c + k][tx][rr] = b;
                    x = x - bf16_to_float(b);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int p = 0; p < 2 * NTERM; ++p) {
                const unsigned *src = reinterpret_cast<const unsigned *>(&sh[p][col][BF_STEP * t + 8 * ch]);
                const uint4 v = make_uint4(src[0], src[1], src[2], src[3]);
                *reinterpret_cast<uint4 *>(P + (((2 * tile + t) * 2 * NTERM + p) * n_pad + j0 + col) * BF_STEP + 8 * ch) = v;
            }
        }
        __syncthreads();
    }
    const int64_t s_hi = 64 * t_hi < m ? 64 * t_hi : m;
    vectors_finish(make_double2(sr, si), 64 * t_lo, s_hi, j, n, noise_var, d, invvar, partial, scal_part);
}

__device__ inline bf8 neg_bf8(bf8 x) {
    s8v v = __builtin_bit_cast(s8v, x);
    v ^= (short)0x8000;
    return __builtin_bit_cast(bf8, v);
}

// The leading products of x y with x and y split into NTERM bfloat16 terms,
// smallest first, term e being x[X[e]] y[Y[e]]: with three terms
// (h, m, l) the six of order at most 2^-16, with two (h, l) the three of
// order at most 2^-8.
template <int NTERM>
struct Prods;
template <>
struct Prods<3> {
    static constexpr int N = 6;
    static constexpr int X[6] = {2, 1, 0, 1, 0, 0};
    static constexpr int Y[6] = {0, 1, 2, 0, 1, 0};
};
template <>
struct Prods<2> {
    static constexpr int N = 3;
    static constexpr int X[3] = {1, 0, 0};
    static constexpr int Y[3] = {0, 1, 0};
};

// One workgroup of four waves per 128 x 64 block of A: tiles (2 I, j) and
// (2 I + 1, j). Per step of 32 rows it copies the panels of its 192 columns (2
// NTERM planes each: 72 KiB for three terms) into one of two LDS buffers; the
// next step's are read into registers while this step's are multiplied. Wave
// (wr, wc) owns the 64 rows of tile 2 I + wr and columns 32 wc .. + 31: eight 16
// x 16 blocks, so that one set of column operands serves four row blocks and
// one set of row operands two column blocks: 36 KiB of LDS reads per 192 MFMAs
// of a wave. (With 16 rows and 64 columns per wave, 30 KiB per 96, the LDS time of
// a step was nearly that of its MFMAs and, with one wave per SIMD, the two added
// up.) The FP64 sums of eight blocks and the operands in flight take 400
// registers, which one wave per SIMD has. The 16-byte pieces of a column are
// stored at piece ^ (column / 2) % 4, which makes the operand reads free of bank
// conflicts without padding. Each accumulator takes its products in a fixed
// order. 8000 x 2048, three terms: 953 us against 1042, 900 TFLOP/s where a large
// library product of the same type reaches 1075 on this card; the whole
// precompute 1.12 ms against 1.22, 20000 x 4096 8.4 ms against 10.0. Bound by the
// matrix cores and the clock they leave: reading a row block's operands beside the
// products of the one before, LDS stores spread likewise, changed nothing (965 us).
constexpr int BF_COLS = 192;  // columns of a step in LDS: 128 of the rows, 64 of the columns

// Work unit u: block u % units over the 32-row steps of rows [split rows_per,
// ...), split = u / units (rows_per a multiple of CHUNK_ROWS). With one split
// the tiles go to A; otherwise to their slots of `out` (FP64), and the splits
// are added in a fixed order afterwards.
template <int NTERM>
__global__ __launch_bounds__(256, 1) void herk_bf16_kernel(const unsigned short *__restrict__ P,
                                                           int64_t m_pad, int64_t n_pad, int64_t n, int64_t units,
                                                           int64_t rows_per, int splits,
                                                           double2 *__restrict__ out) {
    constexpr int NP = 2 * NTERM;   // planes: NTERM real, NTERM imaginary
    constexpr int NL = 3 * NP;      // 16-byte reads per thread per step: three tiles of columns, NP planes
    using PR = Prods<NTERM>;
    __shared__ __align__(16) unsigned short lds[2][NP * BF_COLS * BF_STEP];
    const int64_t unit = blockIdx.x % units, split = blockIdx.x / units;
    const int64_t r0 = split * rows_per;
    const int64_t r1 = r0 + rows_per < m_pad ? r0 + rows_per : m_pad;
    // unit = I (I + 1) + j, j <= 2 I + 1
    int64_t I = (int64_t)((sqrt(4.0 * (double)unit + 1.0) - 1.0) * 0.5);
    while (I * (I + 1) > unit) --I;
    while ((I + 1) * (I + 2) <= unit) ++I;
    const int64_t tj = unit - I * (I + 1), N = n_pad / TS;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wr = w & 1, wc = w >> 1;
    // the thread's piece of a 64-column group: column tid / 4, rows 8 (tid % 4) ..
    const int col = tid >> 2, ch = tid & 3;
    const int64_t tiles[3] = {2 * I, 2 * I + 1 < N ? 2 * I + 1 : 2 * I, tj};  // a missing tile reads another and is not stored
    int voff[3];
#pragma unroll
    for (int g = 0; g < 3; ++g) voff[g] = (int)((TS * tiles[g] + col) * (BF_STEP * 2)) + 16 * ch;
    const int dst = col * BF_STEP + 8 * (ch ^ ((col >> 1) & 3));
    s8v pre[NL];
    auto fetch = [&](int64_t s0) {
        const rsrc_t R = make_rsrc(P + (s0 / BF_STEP) * NP * n_pad * BF_STEP, NP * n_pad * BF_STEP * 2);
#pragma unroll
        for (int u = 0; u < NL; ++u)
            pre[u] = __builtin_bit_cast(s8v, __builtin_amdgcn_raw_buffer_load_b128(
                                                 R, voff[u % 3], (int)((u / 3) * n_pad * (BF_STEP * 2)), 0));
    };
    auto stash = [&](int b) {
#pragma unroll
        for (int u = 0; u < NL; ++u)
            *reinterpret_cast<s8v *>(&lds[b][((u / 3) * BF_COLS + TS * (u % 3)) * BF_STEP + dst]) = pre[u];
    };
    // operand of plane p: column c0 + l16 of the step (c0 a multiple of 16), rows 8 q ..
    const int opn = l16 * BF_STEP + 8 * (q ^ ((l16 >> 1) & 3));
    auto opnd = [&](int b, int p, int c0) {
        return __builtin_bit_cast(bf8, *reinterpret_cast<const s8v *>(&lds[b][(p * BF_COLS + c0) * BF_STEP + opn]));
    };
    double sR[4][2][4], sI[4][2][4];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) sR[rb][cb][r] = sI[rb][cb][r] = 0.0;

    fetch(r0);
    stash(0);
    __syncthreads();
    for (int64_t c0 = r0; c0 < r1; c0 += CHUNK_ROWS) {
        f4 aR[4][2], aI[4][2];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                aR[rb][cb] = f4{0, 0, 0, 0};
                aI[rb][cb] = f4{0, 0, 0, 0};
            }
#pragma unroll
        for (int b = 0; b < CHUNK_ROWS / BF_STEP; ++b) {  // two steps: LDS buffers 0 and 1
            const int64_t next = c0 + BF_STEP * (b + 1);
            if (next < r1) fetch(next);
            bf8 br[2][NTERM], bi[2][NTERM];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int t = 0; t < NTERM; ++t) {
                    br[cb][t] = opnd(b, t, 2 * TS + 32 * wc + 16 * cb);
                    bi[cb][t] = opnd(b, NTERM + t, 2 * TS + 32 * wc + 16 * cb);
                }
            // re: br ar + bi ai;  im: bi ar - br ai
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                bf8 ar[NTERM], ai[NTERM], nai[NTERM];
#pragma unroll
                for (int t = 0; t < NTERM; ++t) {
                    ar[t] = opnd(b, t, TS * wr + 16 * rb);
                    ai[t] = opnd(b, NTERM + t, TS * wr + 16 * rb);
                    nai[t] = neg_bf8(ai[t]);
                }
#pragma unroll
                for (int e = 0; e < PR::N; ++e)
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        aR[rb][cb] = mfma_bf16(br[cb][PR::X[e]], ar[PR::Y[e]], aR[rb][cb]);
                        aI[rb][cb] = mfma_bf16(bi[cb][PR::X[e]], ar[PR::Y[e]], aI[rb][cb]);
                    }
#pragma unroll
                for (int e = 0; e < PR::N; ++e)
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        aR[rb][cb] = mfma_bf16(bi[cb][PR::X[e]], ai[PR::Y[e]], aR[rb][cb]);
                        aI[rb][cb] = mfma_bf16(br[cb][PR::X[e]], nai[PR::Y[e]], aI[rb][cb]);
                    }
            }
            if (next < r1) stash(b ^ 1);
            __syncthreads();
        }
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sR[rb][cb][r] += (double)aR[rb][cb][r];
                    sI[rb][cb][r] += (double)aI[rb][cb][r];
                }
    }
    // lane holds [16 rb + l16][32 wc + 16 cb + 4 q + r] of tile (2 I + wr, j)
    const int64_t ti = 2 * I + wr;
    if (ti >= N || tj > ti) return;
    double2 *pt = splits == 1 ? out + tile_index(ti, tj) * TS2 : out + (split * n_tiles(N) + tile_index(ti, tj)) * TS2;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * rb + l16, c = 32 * wc + 16 * cb + 4 * q + r;
                const int64_t grow = TS * ti + row, gcol = TS * tj + c;
                double2 v = make_double2(sR[rb][cb][r], sI[rb][cb][r]);
                if (splits == 1) {
                    if (grow == gcol) v.y = 0.0;
                    if (grow >= n || gcol >= n) v = make_double2(grow == gcol ? 1.0 : 0.0, 0.0);
                }
                pt[c * TS + row] = v;
            }
}

}  // namespace

// Row slices of the FP32 product: herk_split's choice, in whole chunks.
void fp32_split(int64_t m_pad, int64_t N, int num_cu, int &splits, int64_t &rows_per) {
    herk_split(m_pad, N, num_cu, splits, rows_per);
    rows_per = (rows_per + CHUNK_ROWS - 1) / CHUNK_ROWS * CHUNK_ROWS;
}

// Blocks of 128 x 64 of the lower triangle: pairs of tile rows 2 I, 2 I + 1
// against tile columns j <= 2 I + 1 (a missing last tile row drops its own column).
int64_t bf16_units(int64_t N) { return (N / 2) * (N / 2 + 1) + (N % 2 ? N : 0); }

// Row slices of the split-BF16 product. Its workgroups fill a CU each, so a
// round is num_cu units; the slices (whole chunks) are chosen to minimise the
// chunks of the busiest CU, rounds x chunks per slice, at BF_CHUNK_US each, and
// 0.03 us per tile and slice for writing and adding its partial tiles. Measured:
// a chunk is 192 x 2 MFMAs of a wave, 2.6 us, plus its copies and FP64 sums; at
// 8000 x 2048 (272 blocks on 256 CUs) one slice would leave the second round
// nearly empty and cost 2 x 125 chunks, eight cost 9 x 16.
constexpr double BF_CHUNK_US = 3.3;

void bf16_split(int64_t m_pad, int64_t N, int num_cu, int &splits, int64_t &rows_per) {
    const int64_t units = bf16_units(N), slots = num_cu > 0 ? num_cu : 1, chunks = m_pad / CHUNK_ROWS;
    splits = 1;
    double best = 1e300;
    // up to eight slices, or as many as give every CU one
    const int64_t most = std::min(chunks, std::max<int64_t>(8, slots / units));
    for (int sp = 1; sp <= most; ++sp) {
        const int64_t per = (chunks + sp - 1) / sp;
        if ((sp - 1) * per >= chunks) continue;  // no empty slice
        const int64_t rounds = (units * sp + slots - 1) / slots;
        const double cost = (double)rounds * (double)per * BF_CHUNK_US + (sp > 1 ? 4.0 + 0.03 * (double)(sp * n_tiles(N)) : 0.0);
        if (cost < best - 1e-9) {
            best = cost;
            splits = sp;
        }
    }
    rows_per = (chunks + splits - 1) / splits * CHUNK_ROWS;
}

size_t lowp_scratch_bytes(eor_precision prec, int64_t m, int64_t n_pad, int num_cu) {
    const int64_t m_pad = (m + CHUNK_ROWS - 1) / CHUNK_ROWS * CHUNK_ROWS;
    if (prec == EOR_PREC_FP32) {
        int splits;
        int64_t rows_per;
        fp32_split(m_pad, n_pad / TS, num_cu, splits, rows_per);
        const size_t part = splits > 1 ? (size_t)splits * n_tiles(n_pad / TS) * TS2 * sizeof(double2) : 0;
        return (size_t)m_pad * n_pad * sizeof(float2) + part;
    }
    if (prec == EOR_PREC_BF16X3 || prec == EOR_PREC_BF16X2) {
        int splits;
        int64_t rows_per;
        bf16_split(m_pad, n_pad / TS, num_cu, splits, rows_per);
        const size_t part = splits > 1 ? (size_t)splits * n_tiles(n_pad / TS) * TS2 * sizeof(double2) : 0;
        return (size_t)(prec == EOR_PREC_BF16X3 ? 6 : 4) * m_pad * n_pad * sizeof(unsigned short) + part;
    }
    return 0;
}

// Row slices of the pass over T: whole tiles of rows, at most c.splits of them
// (the capacity of c.partial).
struct VecSlices {
    int64_t tiles, per;  // tiles of 64 rows in all, and of a slice
    int count;
    double2 *scal_part;
    VecSlices(const Context &c, int64_t m_pad)
        : tiles(m_pad / 64), per((tiles + c.splits - 1) / c.splits), count((int)((tiles + per - 1) / per)),
          scal_part(c.partial + (int64_t)count * c.n) {}
};

hipError_t launch_precompute_fp32(const Context &c, const double2 *T, int64_t ldT, const double *noise_var,
                                  const double2 *d, void *scratch, hipStream_t s) {
    const int64_t m_pad = (c.m + CHUNK_ROWS - 1) / CHUNK_ROWS * CHUNK_ROWS;
    float2 *W = (float2 *)scratch;
    const VecSlices v(c, m_pad);
    hipLaunchKernelGGL(w32_kernel, dim3((unsigned)(c.n_pad / 64), (unsigned)v.count), dim3(256), 0, s, T, ldT, c.m, c.n,
                       noise_var, d, m_pad, c.n_pad, 64 * v.per, W, c.invvar, c.partial, v.scal_part);
    const hipError_t e = launch_vectors_reduce(c, c.partial, v.scal_part, v.count, s);
    if (e != hipSuccess) return e;
    int splits;
    int64_t rows_per;
    fp32_split(m_pad, c.N, c.num_cu, splits, rows_per);
    const int64_t tiles = n_tiles(c.N);
    double2 *part = splits > 1 ? (double2 *)((char *)scratch + (size_t)m_pad * c.n_pad * sizeof(float2)) : c.A;
    hipLaunchKernelGGL(herk_fp32_kernel, dim3((unsigned)(tiles * splits)), dim3(256), 0, s, W, m_pad, c.n_pad,
                       c.n, tiles, rows_per, splits, part);
    if (splits > 1) return launch_herk_reduce(part, tiles, splits, c.n, c.A, s);
    return hipGetLastError();
}

hipError_t launch_precompute_bf16(const Context &c, const double2 *T, int64_t ldT, const double *noise_var,
                                  const double2 *d, void *scratch, int nterm, hipStream_t s) {
    const int64_t m_pad = (c.m + CHUNK_ROWS - 1) / CHUNK_ROWS * CHUNK_ROWS;
    unsigned short *P = (unsigned short *)scratch;
    const VecSlices v(c, m_pad);
    const dim3 sgrid((unsigned)(c.n_pad / 64), (unsigned)v.count);
    const int64_t tiles = n_tiles(c.N);
    int splits;
    int64_t rows_per;
    bf16_split(m_pad, c.N, c.num_cu, splits, rows_per);
    double2 *part = splits > 1 ? (double2 *)((char *)scratch + (size_t)(2 * nterm) * m_pad * c.n_pad *
                                                                 sizeof(unsigned short))
                               : c.A;
    const int64_t units = bf16_units(c.N);
    const dim3 hgrid((unsigned)(units * splits));
    if (nterm == 3) {
        hipLaunchKernelGGL(split_kernel<3>, sgrid, dim3(256), 0, s, T, ldT, c.m, c.n, noise_var, d, c.n_pad, v.tiles,
                           v.per, P, c.invvar, c.partial, v.scal_part);
        hipLaunchKernelGGL(herk_bf16_kernel<3>, hgrid, dim3(256), 0, s, P, m_pad, c.n_pad, c.n, units, rows_per,
                           splits, part);
    } else {
        hipLaunchKernelGGL(split_kernel<2>, sgrid, dim3(256), 0, s, T, ldT, c.m, c.n, noise_var, d, c.n_pad, v.tiles,
                           v.per, P, c.invvar, c.partial, v.scal_part);
        hipLaunchKernelGGL(herk_bf16_kernel<2>, hgrid, dim3(256), 0, s, P, m_pad, c.n_pad, c.n, units, rows_per,
                           splits, part);
    }
    const hipError_t e = launch_vectors_reduce(c, c.partial, v.scal_part, v.count, s);
    if (e != hipSuccess) return e;
    if (splits > 1) return launch_herk_reduce(part, tiles, splits, c.n, c.A, s);
    return hipGetLastError();
}

}  // namespace eor
