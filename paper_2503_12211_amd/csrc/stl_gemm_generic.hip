// Any-shape batched plane product on the matrix cores in fp32 (v_mfma_f32_32x32x2_f32: fp32 operands, fp32
// accumulation).  This is the path for fp32 storage and for bf16 planes with a dimension below 8 (their values are widened
// to fp32 on the way into LDS, which is exact).  256 threads = four wavefronts, a BT x BT block of one plane; edges are
// zero-filled on load and masked on store.
//
// Large planes are bound by the fp32 matrix cores (157 TFLOP/s), small ones by the latency of a chain of stages, so the
// operands come in 16-byte pieces, the next stage is in registers while the current one is multiplied out of the other
// LDS buffer (one barrier per stage), and small problems take 64 x 64 blocks with 32 contraction elements per stage: fewer,
// longer stages over more workgroups.  49 planes of 64 x 64 x 64: 28 us with element-wise staging of 128 x 128 blocks, now 8.
#include "stl_kernels.h"
#include "stl_device.h"


namespace stl {

// MFMA accumulator layout of v_mfma_f32_32x32x2_f32: lane (j = lane % 32, h = lane / 32) supplies A[row j][k = h] and
// B[k = h][column j]; accumulator e of the lane is C[row 8 (e / 4) + 4 h + e % 4][column j].
// Three wavefronts per SIMD for the 128 x 128 blocks (at the price of eleven spilled registers; left alone the compiler takes
// registers for two): 1024-cube, r = 32, 770 -> 695 us, bf16 dWhat of 1024 x 1024 from four tile rows 57 -> 53.  With a sum into the
// output it helps some sizes and costs others (r = 32 of the latter 123 -> 100, r = 8 31 -> 36) and stays at two.
template <typename T, typename TO, bool ACC, int BT>
__global__ __launch_bounds__(256, BT == 128 && !ACC ? 3 : 1) void gemm_generic_kernel(const T *__restrict__ A, const T *__restrict__ B,
                                                           TO *__restrict__ Out, int Mi, int Nj, int Kl, int a_km,
                                                           int b_km, int a_pg, int b_pg, int o_pg, int batch, int nb)
{
    constexpr int KC = BT == 64 ? 32 : 16, PAD = 4;    // contraction elements per stage
    constexpr int F = BT / 64;                         // 32 x 32 products per wavefront and dimension
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
    f32x16_t acc[F][F];
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
        for (int b = 0; b < F; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;

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
                for (int v = 0; v < F; ++v) acc[u][v] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u], fb[v], acc[u][v], 0, 0, 0);
        }
        if (st + 1 < nst) {
            stage_in(buf ^ 1);                         // its readers passed the barrier below one stage ago
            __syncthreads();
        }
    }
#pragma unroll
    for (int u = 0; u < F; ++u)
#pragma unroll
        for (int v = 0; v < F; ++v)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int gi = i0 + wi + 32 * u + 8 * (e >> 2) + 4 * fh + (e & 3), gj = j0 + wj + 32 * v + fj;
                if (gi < Mi && gj < Nj) {
                    TO *o = Out + at(o_r0 + gi, gj, o_pg, Nj);
                    if (ACC) Elem<TO>::st(o, Elem<TO>::ld(o) + acc[u][v][e]);
                    else Elem<TO>::st(o, acc[u][v][e]);
                }
            }
  }
}

template <typename T, typename TO, bool ACC, int BT>
static hipError_t launch_bt(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    const long zs = (long)g.batch * g.nb;
    const int rows = (g.Mi + BT - 1) / BT;
    dim3 grid((g.Nj + BT - 1) / BT, (unsigned)(rows > 65535 ? 65535 : rows), (unsigned)(zs > 65535 ? 65535 : zs));   // the kernel strides over both
    hipLaunchKernelGGL((gemm_generic_kernel<T, TO, ACC, BT>), grid, dim3(256), 0, s, (const T *)A, (const T *)B, (TO *)Out,
                       g.Mi, g.Nj, g.Kl, (int)g.a_kmajor, (int)g.b_kmajor, g.a_rows_per_group(), g.b_rows_per_group(),
                       g.o_rows_per_group(), g.batch, g.nb);
    return hipGetLastError();
}

template <typename T, typename TO, bool ACC>
static hipError_t launch_t(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    // 128 x 128 blocks (half the operand traffic) once they give every CU one
    const double blocks = (double)((g.Mi + 127) / 128) * ((g.Nj + 127) / 128) * g.batch * g.nb;
    if (g.Mi > 64 && g.Nj > 64 && blocks >= 256) return launch_bt<T, TO, ACC, 128>(g, A, B, Out, s);
    return launch_bt<T, TO, ACC, 64>(g, A, B, Out, s);
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
    if (plane_gemm_wide_eligible(g)) return GemmPath::wide;
    if (plane_gemm_pipe_eligible(g)) return GemmPath::pipe;
    return plane_gemm_mfma_eligible(g) ? GemmPath::staged : GemmPath::generic;
}

hipError_t launch_plane_gemm(int dtype, const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    switch (plane_gemm_path(dtype, g)) {
        case GemmPath::wide: return launch_plane_gemm_wide(g, A, B, Out, s);
        case GemmPath::pipe: return launch_plane_gemm_pipe(g, A, B, Out, s);
        case GemmPath::staged: return launch_plane_gemm_mfma(g, A, B, Out, s);
        case GemmPath::generic: break;
    }
    return launch_plane_gemm_generic(dtype, g, A, B, Out, s);
}

}  // namespace stl
