// Plane products of few rows (a handful of tokens through a layer):
//     Out[p][i][j] = sum_l A[p](i,l) * B[p](l,j)       bf16 x bf16 -> fp32 -> bf16, Mi <= 32, p < r planes, B stored [l][j].
//
// Bound by reading the second operand once (67 MB of weight planes for 16 x 1024 x 1024 tiles at r = 32) or, where that is small,
// by the latency of the chain of stages.  The blocks of the LDS-DMA kernels bring up to eight times the rows there are through
// the same loads and wait at a barrier per 32 contraction elements.  Here nothing goes through LDS on the way in and no
// wavefront waits for another before the end: one workgroup owns 16 CW columns of a plane, its eight wavefronts take
// every eighth chunk of 32 contraction elements, with DEPTH chunks of both operands on their way in registers, and their sums are
// added up in LDS in a fixed order.  A lane loads CW neighbouring columns (lane % 16) of eight stored rows (lane / 16) and turns
// them in its registers, so that fragment c holds columns CW j + c of the block.  An operand stored [j][l] stays with the
// LDS-DMA kernels: its fragments are rows far apart, 64 bytes of each (16 x 1024 x 1024, r = 8: 7.1 there, 7.3 this way).
// Measured, us, 64 x 64 blocks of the LDS-DMA kernel -> here, 16 rows, r = 32, weights in the last-level cache (and, in brackets,
// from memory: a GB of them in turn): 1024 x 1024 15.3 -> 12.4, 5.4 TB/s (18.6 -> 15.6, 4.3 TB/s); 1024 x 256 8.5 -> 5.5 (9.1 -> 7.4);
// 512 x 512 6.6 -> 4.4 (7.6 -> 6.5); 4096 x 1024 (57 -> 52, 5.2 TB/s); 128 x 128 4.3 -> 3.5.  32 rows: 1024 x 1024 15.5 -> 13.4 (18.7 -> 16.4).
// Of fewer than 8 rows, which the fp32 matrix instructions took before, 4 rows: 1024 x 1024, r = 32 80 -> 12.0 (92 -> 15.1), 1024 x 256, r = 49
// 58 -> 6.4, 128 x 128, r = 32 9.0 -> 3.3.
#include "stl_gemm_pipe.h"

namespace stl {
namespace rows {

constexpr int NW = 8, BK = 32;

template <int CW> struct Seg;                                // CW bf16
template <> struct Seg<8> { typedef u32x4_t type; };
template <> struct Seg<4> { typedef u32x2_t type; };

// KTAIL: the contraction ends inside a chunk.
template <int FM, int CW, int DEPTH, bool KTAIL>
__global__ __launch_bounds__(NW * 64, FM * DEPTH * CW <= 16 ? 4 : 2) void gemm_rows_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B,
                                                                                  bf16_t *__restrict__ Out, int Mi, int Nj, int Kl, int tiles_n,
                                                                                  int total, Div by_row, Lay la, Lay lb, Lay lo)
{
    using pipe::static_for;
    typedef typename Seg<CW>::type seg_t;
    constexpr int COLS = 16 * CW, SLOT = 16 * FM * COLS;     // floats of one wavefront's sums
    __shared__ __align__(16) float red[NW / 2 * SLOT];
    const int bid = pipe::first_block(total);                // one block per workgroup; each XCD takes a contiguous eighth
    if (bid >= pipe::end_block(total)) return;
    const int p = by_row.of(bid), j0 = (bid - p * tiles_n) * COLS;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), n16 = lane & 15, kq = lane >> 4;
    const int nch = (Kl + BK - 1) / BK;

    // columns and rows past the edge feed only discarded outputs
    const int col = j0 + CW * n16 < Nj ? CW * n16 : Nj - CW - j0;
    const char *pb = reinterpret_cast<const char *>(B + (size_t)p * lb.plane + j0);
    const uint32_t ldb = (uint32_t)Nj * 2;      // bytes of a stored row
    const uint32_t off_b = 8 * kq * ldb + col * 2;
    const char *pa[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f) {
        const int i = 16 * f + n16;
        pa[f] = reinterpret_cast<const char *>(A + (size_t)p * la.plane + la.row(i < Mi ? i : Mi - 1) + 8 * kq);
    }

    u32x4_t ra[DEPTH][FM];
    seg_t rb[DEPTH][8];
    // chunk s; one beyond the last reads the last once more.  Pieces beyond the contraction's end come from its last eight elements
    // and are cleared before they are multiplied.
    auto fetch = [&](auto d_c, int s) {
        constexpr int d = decltype(d_c)::value;
        const int t = s < nch ? s : nch - 1;
        const char *b = pb + (size_t)t * BK * ldb;
        long off_a = (long)t * BK * 2;
        uint32_t off = off_b;
        if constexpr (KTAIL) {
            const int beyond = t * BK + 8 * kq - (Kl - 8), back = beyond > 0 ? beyond : 0;
            off_a -= back * 2;
            off -= back * ldb;
        }
#pragma unroll
        for (int f = 0; f < FM; ++f) ra[d][f] = *reinterpret_cast<const u32x4_t *>(pa[f] + off_a);
#pragma unroll
        for (int i = 0; i < 8; ++i) rb[d][i] = *reinterpret_cast<const seg_t *>(b + (off + i * ldb));
        __builtin_amdgcn_sched_barrier(0);
    };

    f32x4_t acc[FM][CW];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int c = 0; c < CW; ++c) acc[f][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](auto d_c, int s) {
        constexpr int d = decltype(d_c)::value;
        if (s >= nch) return;
        const uint32_t keep = !KTAIL || s * BK + 8 * kq < Kl ? 0xffffffffu : 0u;     // zeros in both: what lies there may be infinite
        if constexpr (KTAIL)
#pragma unroll
            for (int f = 0; f < FM; ++f) ra[d][f] &= keep;
        static_for<0, CW>([&](auto c_c) {
            constexpr int c = decltype(c_c)::value;
            u32x4_t v;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t x = rb[d][2 * i][c / 2], y = rb[d][2 * i + 1][c / 2];
                v[i] = c % 2 ? (x >> 16) | (y & 0xffff0000u) : (x & 0xffffu) | (y << 16);
            }
            if constexpr (KTAIL) v &= keep;
#pragma unroll
            for (int f = 0; f < FM; ++f)
                acc[f][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ra[d][f]), __builtin_bit_cast(bf16x8_t, v),
                                                                    acc[f][c], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    const int rounds = (nch + NW * DEPTH - 1) / (NW * DEPTH);
    static_for<0, DEPTH>([&](auto d_c) { fetch(d_c, wave + decltype(d_c)::value * NW); });
    int s = wave;
    for (int u = 1; u < rounds; ++u, s += NW * DEPTH)
        static_for<0, DEPTH>([&](auto d_c) {
            constexpr int d = decltype(d_c)::value;
            multiply(d_c, s + d * NW);
            fetch(d_c, s + (d + DEPTH) * NW);
        });
    static_for<0, DEPTH>([&](auto d_c) { multiply(d_c, s + decltype(d_c)::value * NW); });

    // accumulator e of fragment (f, c): row 16 f + 4 kq + e, column CW n16 + c
    auto at = [&](int slot, int f, int e) { return red + slot * SLOT + (16 * f + 4 * kq + e) * COLS + CW * n16; };
    auto each = [&](auto &&body) {
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c4 = 0; c4 < CW; c4 += 4) body(f, e, c4);
    };
    if (wave >= NW / 2)
        each([&](int f, int e, int c4) {
            *reinterpret_cast<f32x4_t *>(at(wave - NW / 2, f, e) + c4) =
                f32x4_t{acc[f][c4][e], acc[f][c4 + 1][e], acc[f][c4 + 2][e], acc[f][c4 + 3][e]};
        });
    __syncthreads();
    if (wave < NW / 2)
        each([&](int f, int e, int c4) {
            f32x4_t *o = reinterpret_cast<f32x4_t *>(at(wave, f, e) + c4);
            *o += f32x4_t{acc[f][c4][e], acc[f][c4 + 1][e], acc[f][c4 + 2][e], acc[f][c4 + 3][e]};
        });
    __syncthreads();
    // eight columns of one row per thread
    constexpr int PER_ROW = COLS / 8, PIECES = 16 * FM * PER_ROW;
#pragma unroll
    for (int q = threadIdx.x; q < PIECES; q += NW * 64) {
        const int i = q / PER_ROW, c = 8 * (q % PER_ROW);
        if (i >= Mi || j0 + c >= Nj) continue;
        const float *x = red + i * COLS + c;
        f32x4_t lo4 = *reinterpret_cast<const f32x4_t *>(x), hi4 = *reinterpret_cast<const f32x4_t *>(x + 4);
#pragma unroll
        for (int w = 1; w < NW / 2; ++w) {
            lo4 += *reinterpret_cast<const f32x4_t *>(x + w * SLOT);
            hi4 += *reinterpret_cast<const f32x4_t *>(x + w * SLOT + 4);
        }
        *reinterpret_cast<u32x4_t *>(Out + (size_t)p * lo.plane + lo.row(i) + j0 + c) =
            u32x4_t{pack_bf16x2(lo4[0], lo4[1]), pack_bf16x2(lo4[2], lo4[3]), pack_bf16x2(hi4[0], hi4[1]), pack_bf16x2(hi4[2], hi4[3])};
    }
}

}  // namespace rows

// Columns per lane: four where that many blocks leave no CU with two (more blocks, more loads per byte), else eight, the same
// bytes in lines twice as long.  us at four / eight, 16 rows: 1024 x 1024, r = 16 (256 blocks of 64 columns) 8.8 / 9.5, 2048 x 512, r = 32
// (256) 16.3 / 20.3; 192 x 768, r = 32 (384) 5.8 / 4.7, 1024 x 768, r = 32 (384) 13.7 / 12.2, 256 x 1024, r = 64 (1024) 10.5 / 8.7.
static long blocks_of(const GemmDesc &g, int cw) { return (long)((g.Nj + 16 * cw - 1) / (16 * cw)) * g.batch; }
static bool four_columns(const GemmDesc &g) { return blocks_of(g, 4) <= 256; }
int rows_columns(const GemmDesc &g) { return four_columns(g) ? 64 : 128; }

// Up to 16 rows it was nowhere slower than the LDS-DMA kernels over K = 8 ... 4096, N = 8 ... 4096, r = 1 ... 64 (64 x 64, r = 8
// 3.75 -> 3.6; 512 x 2048, r = 32 17.3 both).  17 to 32 rows take two fragments per column and one workgroup per CU: us there / here
// of 32 rows: 512 x 512, r = 32 7.1 / 5.8, 1024 x 1024, r = 32 (512 blocks of 64 columns) 19.9 / 17.1, 128 x 128, r = 32 4.4 / 4.2, but
// 64 x 64, r = 32 3.9 / 4.2 and, beyond one round of blocks of 128 columns, 512 x 1024, r = 49 15.2 / 17.2.
bool plane_gemm_rows_eligible(const GemmDesc &g)
{
    if (g.a_kmajor || !g.b_kmajor || g.out_f32 || g.accumulate || g.nb != 1 || g.Mi > 32 || g.Nj % 8 || g.Kl % 8) return false;
    if (g.Mi < 1 || g.Nj < 8 || g.Kl < 8 || g.batch < 1) return false;
    if (g.Mi > 16 && (g.Kl < 128 || blocks_of(g, 4) > 512)) return false;
    GemmLays l;
    return l.set(g) && l.b.shift == 31 && blocks_of(g, 4) <= 1 << 22;      // the weight's stored rows side by side; a launch's threads fit 32 bits
}

template <int FM, int CW, int DEPTH, bool KTAIL>
static hipError_t launch_rows_cfg(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    GemmLays l;
    if (!l.set(g)) return hipErrorInvalidValue;
    const int tiles_n = (g.Nj + 16 * CW - 1) / (16 * CW), total = (int)blocks_of(g, CW);
    hipLaunchKernelGGL((rows::gemm_rows_kernel<FM, CW, DEPTH, KTAIL>), dim3((unsigned)((total + 7) / 8 * 8)), dim3(rows::NW * 64), 0, s,
                       (const bf16_t *)A, (const bf16_t *)B, (bf16_t *)Out, g.Mi, g.Nj, g.Kl, tiles_n, total, Div::by(tiles_n), l.a, l.b, l.o);
    return hipGetLastError();
}

// One chunk in flight per wavefront where two or more workgroups share a CU, two elsewhere.
template <bool KTAIL>
static hipError_t launch_rows_form(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    if (g.Mi > 16) return four_columns(g) ? launch_rows_cfg<2, 4, 2, KTAIL>(g, A, B, Out, s) : launch_rows_cfg<2, 8, 2, KTAIL>(g, A, B, Out, s);
    return four_columns(g) ? launch_rows_cfg<1, 4, 2, KTAIL>(g, A, B, Out, s) : launch_rows_cfg<1, 8, 1, KTAIL>(g, A, B, Out, s);
}

hipError_t launch_plane_gemm_rows(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    if (!plane_gemm_rows_eligible(g)) return hipErrorInvalidValue;
    return g.Kl % rows::BK ? launch_rows_form<true>(g, A, B, Out, s) : launch_rows_form<false>(g, A, B, Out, s);
}

}  // namespace stl
