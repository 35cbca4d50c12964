// Any-shape batched plane product on the matrix cores in fp32 (v_mfma_f32_32x32x2_f32: fp32 operands, fp32
// accumulation).  This is the path for fp32 storage and for bf16 planes with a dimension below 8 (their values are widened
// to fp32 on the way into LDS, which is exact).  256 threads = four wavefronts; edges are zero-filled on load and masked on store.
//
// Large planes are bound by the fp32 matrix cores (157 TFLOP/s): 128 x 128 blocks, operands in 16-byte pieces, the next stage in registers
// while the current one is multiplied out of the other LDS buffer (one barrier per stage).  Small ones are bound by the latency
// of a chain of stages and by idle CUs: 32 x 32 blocks with the contraction shared (gemm_small_kernel).  In between, at contractions
// of one stage, 64 x 64 blocks of the former kind.
#include "stl_kernels.h"
#include "stl_device.h"
#include <algorithm>
#include <cmath>

namespace stl {

// MFMA accumulator layout of v_mfma_f32_32x32x2_f32: lane (j = lane % 32, h = lane / 32) supplies A[row j][k = h] and
// B[k = h][column j]; accumulator e of the lane is C[row 8 (e / 4) + 4 h + e % 4][column j].
// Three wavefronts per SIMD (for the 128 x 128 blocks at the price of eleven spilled registers; left alone the compiler takes registers for two): 1024-cube,
// r = 32, 770 -> 695 us, bf16 dWhat of 1024 x 1024 from four tile rows 57 -> 53.  With a sum into the output it helps some sizes and
// costs others (r = 32 of the latter 123 -> 100, r = 8 31 -> 36) and stays at two.
template <typename T, typename TO, bool ACC, int BT>
__global__ __launch_bounds__(256, BT == 128 && ACC ? 1 : 3) void gemm_generic_kernel(const T *__restrict__ A, const T *__restrict__ B,
                                                           TO *__restrict__ Out, int Mi, int Nj, int Kl, int a_km,
                                                           int b_km, int a_pg, int b_pg, int o_pg, int batch, int nb)
{
    constexpr int KC = BT == 64 ? 32 : 16, PAD = 4;    // contraction elements per stage
    constexpr int F = BT / 64;                         // 32 x 32 products per wavefront and dimension
    constexpr int CH = BT == 64 ? 2 : 1;               // sums of 16 contraction elements of a stage each, added up at the end
    constexpr int UNITS = BT * KC / 1024;              // 16-byte pieces per thread, operand and stage
    __shared__ __align__(16) float sA[2][KC][BT + PAD];    // [l][i]: a fragment read takes 32 consecutive i of one l
    __shared__ __align__(16) float sB[2][KC][BT + PAD];    // [l][j]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi = (wave >> 1) * (BT / 2), wj = (wave & 1) * (BT / 2);
    const int fj = lane & 31, fh = lane >> 5;
    const int nst = (Kl + KC - 1) / KC;
  for (int by = blockIdx.y; by * BT < Mi; by += gridDim.y)        // block rows beyond the grid's second extent
  for (int z = blockIdx.z; z < batch * nb; z += gridDim.z) {      // (stacked problem, plane) pairs
    const int p = z % batch, pb = z / batch;
    const int a_r0 = pb * (a_km ? Kl : Mi), b_r0 = pb * (b_km ? Kl : Nj), o_r0 = pb * Mi;
    // element (row, col) of plane p of an operand stored [row][col] with `ld` columns, rows in groups of pg
    auto at = [&](int row, int col, int pg, int ld) { return plane_row_base(row, pg, batch, ld) + (size_t)p * pg * ld + col; };
    const int i0 = by * BT, j0 = blockIdx.x * BT;
    f32x16_t acc[CH][F][F];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int a = 0; a < F; ++a)
#pragma unroll
            for (int b = 0; b < F; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[c][a][b][e] = 0.f;

    // stage -> registers -> LDS, four elements at a time along the dimension that is contiguous in memory
    f32x4_t ra[UNITS], rb[UNITS];
    auto fetch_one = [&](const T *X, int u, int l0, int c0, int total, int km, int r0, int pg) {
        if (!km) {
            const int l = l0 + 4 * (u % (KC / 4)), c = c0 + u / (KC / 4);
            return c < total ? load4<T>(X + at(r0 + c, l, pg, Kl), Kl - l) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
        const int c = c0 + 4 * (u % (BT / 4)), l = l0 + u / (BT / 4);
        return l < Kl ? load4<T>(X + at(r0 + l, c, pg, total), total - c) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto fetch = [&](int st) {
#pragma unroll
        for (int k = 0; k < UNITS; ++k) {
            const int u = threadIdx.x + 256 * k;
            ra[k] = fetch_one(A, u, st * KC, i0, Mi, a_km, a_r0, a_pg);
            rb[k] = fetch_one(B, u, st * KC, j0, Nj, b_km, b_r0, b_pg);
        }
    };
    auto put = [&](float (*s)[BT + PAD], int u, int km, f32x4_t v) {
        if (!km) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[4 * (u % (KC / 4)) + e][u / (KC / 4)] = v[e];
        } else {
            *reinterpret_cast<f32x4_t *>(&s[u / (BT / 4)][4 * (u % (BT / 4))]) = v;
        }
    };
    auto stage_in = [&](int buf) {
#pragma unroll
        for (int k = 0; k < UNITS; ++k) {
            const int u = threadIdx.x + 256 * k;
            put(sA[buf], u, a_km, ra[k]);
            put(sB[buf], u, b_km, rb[k]);
        }
    };

    fetch(0);
    __syncthreads();                                   // the previous block's last stage has been read
    stage_in(0);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        const int buf = st & 1;
        if (st + 1 < nst) fetch(st + 1);
        // a product takes l and l + 8, which lie half the banks apart (8 (BT + 4) = 32 mod 64 words)
#pragma unroll
        for (int s = 0; s < KC / 2; ++s) {
            const int l = 16 * (s >> 3) + (s & 7) + 8 * fh;
            float fa[F], fb[F];
#pragma unroll
            for (int u = 0; u < F; ++u) {
                fa[u] = sA[buf][l][wi + 32 * u + fj];
                fb[u] = sB[buf][l][wj + 32 * u + fj];
            }
#pragma unroll
            for (int u = 0; u < F; ++u)
#pragma unroll
                for (int v = 0; v < F; ++v) acc[CH == 2 ? s >> 3 : 0][u][v] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u], fb[v], acc[CH == 2 ? s >> 3 : 0][u][v], 0, 0, 0);
        }
        if (st + 1 < nst) {
            stage_in(buf ^ 1);                         // its readers passed the barrier below one stage ago
            __syncthreads();
        }
    }
    if constexpr (CH == 2) acc[0][0][0] += acc[1][0][0];
#pragma unroll
    for (int u = 0; u < F; ++u)
#pragma unroll
        for (int v = 0; v < F; ++v)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int gi = i0 + wi + 32 * u + 8 * (e >> 2) + 4 * fh + (e & 3), gj = j0 + wj + 32 * v + fj;
                if (gi < Mi && gj < Nj) {
                    TO *o = Out + at(o_r0 + gi, gj, o_pg, Nj);
                    if (ACC) Elem<TO>::st(o, Elem<TO>::ld(o) + acc[0][u][v][e]);
                    else Elem<TO>::st(o, acc[0][u][v][e]);
                }
            }
  }
}

// A 32 x 32 block of one plane per workgroup, whose four wavefronts share the contraction, 16 of a stage's 64 elements each, and add
// their sums up in LDS.  64 x 64 blocks give 49 planes of 64 x 64 49 workgroups and a chain of two stages, these four times as many
// and one stage of 16 KB in flight: 7.5 / 4.0 us.  64 planes of 60 x 2000 x 60: 101 / 40.
constexpr int kSmallBlock = 32, kSmallStage = 64, kSmallPitch = kSmallBlock + 4;
struct SmallLds {
    __align__(16) float a[kSmallStage][kSmallPitch];                         // [l][i]
    __align__(16) float b[kSmallStage][kSmallPitch];                         // [l][j]
    __align__(16) float red[4][kSmallBlock][kSmallPitch];
};
struct SmallProduct {
    const void *A, *B;
    void *Out;
    int Mi, Nj, Kl, a_km, b_km, tiles_m, tiles_n, total, batch;
    Div by_plane, by_row, by_batch;
    Lay la, lb, lo;
};
template <typename T, typename TO, bool ACC>
__device__ __forceinline__ void small_product(const SmallProduct &g, int v, SmallLds &m)
{
    constexpr int BT = kSmallBlock, KC = kSmallStage, PITCH = kSmallPitch;
    const T *A = (const T *)g.A, *B = (const T *)g.B;
    TO *Out = (TO *)g.Out;
    const int Mi = g.Mi, Nj = g.Nj, Kl = g.Kl, a_km = g.a_km, b_km = g.b_km, tiles_m = g.tiles_m, tiles_n = g.tiles_n, batch = g.batch;
    const Div &by_plane = g.by_plane, &by_row = g.by_row, &by_batch = g.by_batch;
    const Lay &la = g.la, &lb = g.lb, &lo = g.lo;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), fj = lane & 31, fh = lane >> 5;
    const int q = by_plane.of(v), rem = v - q * (tiles_m * tiles_n), bi = by_row.of(rem);
    const int i0 = bi * BT, j0 = (rem - bi * tiles_n) * BT, pb = by_batch.of(q), p = q - pb * batch;
    const T *Ap = A + (size_t)p * la.plane, *Bp = B + (size_t)p * lb.plane;

    // four elements along the dimension that is contiguous in memory: unit u of 512 per operand and stage
    auto fetch_one = [&](const T *X, const Lay &lay, int u, int l0, int c0, int total_c, int km, int r0) {
        const int c = c0 + (km ? 4 * (u & 7) : u >> 4), l = l0 + (km ? u >> 3 : 4 * (u & 15));
        const bool in = km ? l < Kl : c < total_c;
        return load4<T>(X + (in ? lay.row(r0 + (km ? l : c)) + (km ? c : l) : 0), in ? (km ? total_c - c : Kl - l) : 0);
    };
    auto put = [&](float (*s)[PITCH], int u, int km, f32x4_t w) {
        if (km) {
            *reinterpret_cast<f32x4_t *>(&s[u >> 3][4 * (u & 7)]) = w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[4 * (u & 15) + e][u >> 4] = w[e];
        }
    };
    f32x4_t ra[2], rb[2];
    auto fetch = [&](int l0) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            ra[k] = fetch_one(Ap, la, threadIdx.x + 256 * k, l0, i0, Mi, a_km, pb * (a_km ? Kl : Mi));
            rb[k] = fetch_one(Bp, lb, threadIdx.x + 256 * k, l0, j0, Nj, b_km, pb * (b_km ? Kl : Nj));
        }
    };
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    fetch(0);
    for (int l0 = 0; l0 < Kl; l0 += KC) {
        __syncthreads();                               // the previous stage has been read
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            put(m.a, threadIdx.x + 256 * k, a_km, ra[k]);
            put(m.b, threadIdx.x + 256 * k, b_km, rb[k]);
        }
        __syncthreads();
        if (l0 + KC < Kl) fetch(l0 + KC);
        // a product takes l and l + 8 (half the banks apart: 8 (BT + 4) = 32 mod 64 words)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int l = 16 * wave + s + 8 * fh;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(m.a[l][fj], m.b[l][fj], acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) m.red[wave][8 * (e >> 2) + 4 * fh + (e & 3)][fj] = acc[e];
    __syncthreads();
    // thread: row i, columns j .. j + 3
    const int i = threadIdx.x >> 3, j = 4 * (threadIdx.x & 7), gi = i0 + i, gj = j0 + j;
    if (gi >= Mi) return;
    f32x4_t w = *reinterpret_cast<const f32x4_t *>(&m.red[0][i][j]);
#pragma unroll
    for (int k = 1; k < 4; ++k) w += *reinterpret_cast<const f32x4_t *>(&m.red[k][i][j]);
    TO *o = Out + (size_t)p * lo.plane + lo.row(pb * Mi + gi) + gj;
    if constexpr (sizeof(TO) == 4) {
        if (gj + 4 <= Nj) {
            if (ACC) w += *reinterpret_cast<const f32x4_any_t *>(o);
            *reinterpret_cast<f32x4_any_t *>(o) = w;
            return;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (gj + e < Nj) Elem<TO>::st(o + e, ACC ? Elem<TO>::ld(o + e) + w[e] : w[e]);
}

template <typename T, typename TO, bool ACC>
__global__ __launch_bounds__(256) void gemm_small_kernel(const SmallProduct g)
{
    __shared__ SmallLds m;
    for (int v = blockIdx.x; v < g.total; v += gridDim.x) small_product<T, TO, ACC>(g, v, m);          // blocks beyond the grid
}

// Two products of a layer's gradients that do not depend on each other in one launch, fp32: the weight's, which ACC may add to what is there, and
// the input's.  The blocks with more stages come first (LAST_FIRST: the input's).
template <bool ACC, bool LAST_FIRST>
__global__ __launch_bounds__(256) void gemm_small_pair_kernel(const SmallProduct x, const SmallProduct y)
{
    __shared__ SmallLds m;
    const int v = blockIdx.x;
    if constexpr (LAST_FIRST) {
        if (v < y.total) small_product<float, float, false>(y, v, m);
        else small_product<float, float, ACC>(x, v - y.total, m);
    } else {
        if (v < x.total) small_product<float, float, ACC>(x, v, m);
        else small_product<float, float, false>(y, v - x.total, m);
    }
}

static bool small_args(const GemmDesc &g, const void *A, const void *B, void *Out, SmallProduct *x)
{
    GemmLays l;
    if (!l.set(g)) return false;
    // with at most 2^22 stacked tile rows and columns and 64 planes, what is not left to the large blocks stays far below 2^31 blocks
    const int tm = (g.Mi + kSmallBlock - 1) / kSmallBlock, tn = (g.Nj + kSmallBlock - 1) / kSmallBlock;
    *x = {A, B, Out, g.Mi, g.Nj, g.Kl, (int)g.a_kmajor, (int)g.b_kmajor, tm, tn, tm * tn * g.batch * g.nb, g.batch, Div::by(tm * tn), Div::by(tn),
          Div::by(g.batch), l.a, l.b, l.o};
    return true;
}

template <typename T, typename TO, bool ACC>
static hipError_t launch_small(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    SmallProduct x;
    if (!small_args(g, A, B, Out, &x)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_small_kernel<T, TO, ACC>), dim3(x.total > (1 << 22) ? 1 << 22 : x.total), dim3(256), 0, s, x);
    return hipGetLastError();
}

template <typename T, typename TO, bool ACC, int BT>
static hipError_t launch_large(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    const long zs = (long)g.batch * g.nb;
    const int rows = (g.Mi + BT - 1) / BT;
    dim3 grid((g.Nj + BT - 1) / BT, (unsigned)(rows > 65535 ? 65535 : rows), (unsigned)(zs > 65535 ? 65535 : zs));   // the kernel strides over both
    hipLaunchKernelGGL((gemm_generic_kernel<T, TO, ACC, BT>), grid, dim3(256), 0, s, (const T *)A, (const T *)B, (TO *)Out,
                       g.Mi, g.Nj, g.Kl, (int)g.a_kmajor, (int)g.b_kmajor, g.a_rows_per_group(), g.b_rows_per_group(),
                       g.o_rows_per_group(), g.batch, g.nb);
    return hipGetLastError();
}

// Edge of the block.  128 x 128 (a quarter of the operand traffic) once every CU has two, at contractions of one of its stages, which
// store most of the time, one: bf16 dWhat (and the encode before it) of 512 x 512 from 4 tile rows, r = 16 (256 blocks), 16.8 us against 18.9 at 32;
// the fp32 forward of 64 stacked problems of 82 x 32 x 82 tiles, r = 24 (1536 blocks), 80 against 87.
// Below that 32 x 32; but at contractions of up to 32, where its four wavefronts have a stage of 64 for half of it or less, 64 x 64 where a
// prediction of both times, us, from the blocks per CU says so (fitted to 264 products of 64 to 1500 tiles and 8 to 64 planes); the
// sums are the same bit for bit.  Operands that both lie along the contraction turn on their way to LDS, which costs the 32 x 32
// blocks more.  us at 128 / 64 / 32: fp32 Yhat
// 32 x (256 x 16 x 256) 13.4 / 8.5 / 9.3, 64 x (256 x 32 x 256) 16.0 / 13.9 / 15.3, 8 x (96 x 16 x 96) 11.4 / 5.9 / 4.0; bf16 dX of 256 x 256 from
// 7 tile columns, r = 40, 24.4 / 21.6 / 28.4, of 1000 x 64 from 6, r = 32, 21.4 / 18.2 / 21.8.
// Longer contractions stay with the 32 x 32 blocks also where one of the others is ahead (56 x (384 x 384 x 384) 82 / 96 / 98, 64 x (128 x 300 x
// 300) 48 / 34.5 / 42.7): those add a contraction up in one chain, these in four, with half the error against 64 bits (384 x 384 x 384 3.5e-7 / 1.8e-7).
int generic_block(const GemmDesc &g)
{
    auto blocks = [&](int bt) { return (double)((g.Mi + bt - 1) / bt) * ((g.Nj + bt - 1) / bt) * g.batch * g.nb / 256; };    // per CU
    if (g.Mi > 64 && g.Nj > 64 && blocks(128) >= (g.Kl <= 16 ? 1 : 2)) return 128;
    if (g.Kl > 32) return 32;
    const bool turns = !g.a_kmajor && !g.b_kmajor;
    const double t32 = 2.9 + blocks(32) * (turns ? 0.68 : 0.51), t64 = 1.4 + std::max(2.0, std::ceil(blocks(64))) * 2.13;
    return t32 <= t64 ? 32 : 64;
}

template <typename T, typename TO, bool ACC>
static hipError_t launch_t(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    switch (generic_block(g)) {
        case 128: return launch_large<T, TO, ACC, 128>(g, A, B, Out, s);
        case 64: return launch_large<T, TO, ACC, 64>(g, A, B, Out, s);
    }
    return launch_small<T, TO, ACC>(g, A, B, Out, s);
}

hipError_t launch_plane_gemm_generic(int dtype, const GemmDesc &g, const void *A, const void *B, void *Out,
                                     hipStream_t s)
{
    if (dtype == 0) {
        return g.accumulate ? launch_t<float, float, true>(g, A, B, Out, s) : launch_t<float, float, false>(g, A, B, Out, s);
    }
    if (g.out_f32)
        return g.accumulate ? launch_t<bf16_t, float, true>(g, A, B, Out, s)
                            : launch_t<bf16_t, float, false>(g, A, B, Out, s);
    return launch_t<bf16_t, bf16_t, false>(g, A, B, Out, s);
}

GemmPath plane_gemm_path(int dtype, const GemmDesc &g)
{
    if (dtype != 1) return GemmPath::generic;
    if (plane_gemm_rows_eligible(g)) return GemmPath::rows;
    if (plane_gemm_wide_eligible(g)) return GemmPath::wide;
    if (plane_gemm_pipe_eligible(g)) return GemmPath::pipe;
    return plane_gemm_mfma_eligible(g) ? GemmPath::staged : GemmPath::generic;
}

hipError_t launch_plane_gemm(int dtype, const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    switch (plane_gemm_path(dtype, g)) {
        case GemmPath::rows: return launch_plane_gemm_rows(g, A, B, Out, s);
        case GemmPath::wide: return launch_plane_gemm_wide(g, A, B, Out, s);
        case GemmPath::pipe: return launch_plane_gemm_pipe(g, A, B, Out, s);
        case GemmPath::staged: return launch_plane_gemm_mfma(g, A, B, Out, s);
        case GemmPath::generic: break;
    }
    return launch_plane_gemm_generic(dtype, g, A, B, Out, s);
}

// Whether launch_plane_gemm_pair runs the two as one launch.
bool plane_gemm_paired(int dtype, const GemmDesc &g1, const GemmDesc &g2)
{
    if (dtype != 0) return staged_pair_eligible(g1, g2) || pipe_pair_eligible(g1, g2);
    auto blocks = [](const GemmDesc &g) { return (double)((g.Mi + 31) / 32) * ((g.Nj + 31) / 32) * g.batch * g.nb; };
    return g1.Mi >= 1 && g1.out_f32 && !g2.out_f32 && !g2.accumulate && generic_block(g1) == 32 && generic_block(g2) == 32 && blocks(g1) + blocks(g2) < (1 << 22);
}

hipError_t launch_plane_gemm_pair(int dtype, const GemmDesc &g1, const void *A1, const void *B1, void *Out1, const GemmDesc &g2, const void *A2,
                                  const void *B2, void *Out2, hipStream_t s)
{
    if (plane_gemm_paired(dtype, g1, g2)) {
        if (dtype != 0)
            return staged_pair_eligible(g1, g2) ? launch_staged_pair(g1, A1, B1, Out1, g2, A2, B2, Out2, s)
                                                : launch_pipe_pair(g1, A1, B1, Out1, g2, A2, B2, Out2, s);
        SmallProduct x, y;
        if (!small_args(g1, A1, B1, Out1, &x) || !small_args(g2, A2, B2, Out2, &y)) return hipErrorInvalidValue;
        // Long chains of stages that begin last are what the launch waits for.  Whole backward passes, us, two launches / the weight's gradient first /
        // the longer contraction first: 128 x 37 x 957, r = 20 49.6 / 55.3 / 41.0, 53 x 134 x 670, r = 32 47.2 / 51.1 / 37.0, 43 x 3 x 1199, r = 49 56.2 /
        // 58.9 / 50.6; over 900 layers of up to 8192 x 1500 x 1500 at worst 0.90 times as fast as two launches and 0.98, in the mean 1.145 and 1.156.
        auto stages = [](const GemmDesc &g) { return (g.Kl + kSmallStage - 1) / kSmallStage; };
        const bool y_first = stages(g2) > stages(g1);
        auto kern = g1.accumulate ? (y_first ? gemm_small_pair_kernel<true, true> : gemm_small_pair_kernel<true, false>)
                                  : (y_first ? gemm_small_pair_kernel<false, true> : gemm_small_pair_kernel<false, false>);
        hipLaunchKernelGGL(kern, dim3(x.total + y.total), dim3(256), 0, s, x, y);
        return hipGetLastError();
    }
    const hipError_t e = launch_plane_gemm(dtype, g1, A1, B1, Out1, s);
    return e != hipSuccess ? e : launch_plane_gemm(dtype, g2, A2, B2, Out2, s);
}

}  // namespace stl
