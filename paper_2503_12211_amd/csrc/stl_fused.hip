// Forward variants that keep the r encoded output planes on chip (Definition 3.1 / Eq. (2) evaluated per
// output block: encode -> per-plane MFMA accumulation over L -> one decode per output tile):
//
//   EPILOGUE: Xhat comes from HBM (written by the encode kernel); the plane products and the decode run here.
//   FUSED:    X itself is read; the encode of every X sub-block runs here on MFMA, so no plane tensor ever
//             touches HBM (optionally Yhat is written for the backward pass).
//
// One workgroup (8 wavefronts) owns a block of 32 x 32 output tiles (128 x 128 entries of C) and ALL r <= 32
// planes of it: wavefront w accumulates r / 8 neighbouring planes (one 32x32x16 MFMA tile per plane, K = 16 tile
// columns L per step).  Operand sub-blocks arrive by LDS-DMA in a ring of stages.  After the L loop the r x 1024
// fp32 accumulators are exchanged through LDS and every thread decodes 2 tiles with D in fp32.
// FUSED: wavefront w encodes the four tile rows whose X rows it fetched itself (16x16x32 MFMA, rows = the 16 tile columns of one
// tile row, columns = planes: a lane ends with four neighbouring L of a plane) one step ahead of the products, into the other of
// two buffers, so that a step has one barrier.
// A small problem is a chain of steps, and a step was the instructions on its way: with four wavefronts, conditions around the
// products that copied every accumulator twice per step, and an encode and a product in turn between two barriers it took 0.72 us,
// now 0.65 at r <= 16, where
// it waits for the stages to arrive (128 x 512 -> 512, r = 8: 10.4 -> 8.8 us; 32 x 512 -> 512, r = 32: 22.7 -> 15.7).
//
// Decode needs all planes of a tile in one workgroup, and r accumulator planes leave room for only ~1K output
// tiles per workgroup, so each operand element fetched from L2 feeds few MACs (16 flop per byte against 128 for a
// one-plane 256 x 256 block): this kernel is bound by the L2 -> LDS path, not by MFMA, and at every shape where the
// plane products take a measurable time the three-launch path is faster (6 x at the benchmark shape, where this
// kernel moves 26 GB through L2 at 21 TB/s, the rate the L2 -> LDS path gives).  It wins only where the whole
// operator is bound by launch latency: one launch instead of three for problems of a few microseconds, which is
// where the automatic variant choice uses it.
#include "stl_gemm_pipe.h"

namespace stl {
namespace fused {

using pipe::block_barrier;
using pipe::dma16;
using pipe::v4i16_t;

constexpr int BI = 32, BJ = 32, KC = 16, NW = 8;  // block: 32 x 32 tiles, 16 tile columns of X per step; wavefronts
constexpr int SX_BYTES = 4 * BI * KC * 4 * 2;     // X sub-block: 128 rows x 64 entries  = 16 KB
constexpr int SD_BYTES = 32 * 16 * 4;             // decoder in fp32
// per plane: Xhat stage 32 x 16 bf16 = 1 KB (encoded here: 32 bytes further apart, which spreads the planes of one write over the
// banks), What stage 16 x 32 bf16 = 1 KB, exchanged accumulators 32 x 32 fp32 = 4 KB
template <int RP, bool ENCODE, int NS>                                // NS: ring of stages (see block_forward_ring)
struct Map {
    static constexpr bool TWICE = ENCODE && RP <= 16 && NS > 2;       // two encoded stages (at 32 planes LDS holds one)
    static constexpr int PITCH = ENCODE ? 1024 + 32 : 1024;           // of a plane of Xhat
    static constexpr int A_STAGE = ENCODE ? SX_BYTES : RP * 1024, W_STAGE = RP * 1024;
    static constexpr int XH = NS * A_STAGE, XH_STAGE = ENCODE ? RP * PITCH : 0;
    static constexpr int W = XH + (TWICE ? 2 : 1) * XH_STAGE, LOOP = W + NS * W_STAGE;
    static constexpr int D = LOOP > RP * 4096 ? LOOP : RP * 4096, BYTES = D + SD_BYTES;
};

__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// ENCODE: true = FUSED (reads X), false = EPILOGUE (reads Xhat).  RP: planes padded to 8, 16 or 32 (sizes the LDS
// stages and the accumulators; planes beyond r are zeros and cost less than leaving them out).
template <int RP, bool ENCODE, bool GELU, int NS>
__global__ __launch_bounds__(NW * 64) void stl_block_kernel(const bf16_t *__restrict__ Xin,   // X (m x k) or Xhat (r x M x K)
                                                        const bf16_t *__restrict__ What, const bf16_t *__restrict__ E,
                                                        const bf16_t *__restrict__ Dm, bf16_t *__restrict__ C,
                                                        bf16_t *__restrict__ Ysave, int M, int K, int N, int r,
                                                        int blocks_j, int pg)
{
    typedef Map<RP, ENCODE, NS> L;
    constexpr int PW = RP / NW, AW = ENCODE ? 2 : PW;      // planes, and DMA instructions of the A side, per wavefront
    constexpr int LOADS = AW + PW;                                     // per wavefront and stage
    extern __shared__ __align__(16) char smem[];
    const char *sA = smem, *sW = smem + L::W;
    char *sXh = smem + L::XH;                         // FUSED only
    float *sD = reinterpret_cast<float *>(smem + L::D);
    const uint32_t lds0 = (uint32_t)(uintptr_t)STL_LDS(smem);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int I0 = (blockIdx.x / blocks_j) * BI, J0 = (blockIdx.x % blocks_j) * BJ;
    const size_t k_elems = (size_t)K * 4, n_elems = (size_t)N * 4;

    // the decoder waits in a register until the loop is under way, so that the first stages do not wait for it
    const bf16_t dreg = tid < r * 16 ? Dm[tid] : (bf16_t)0;
    // encoder fragments (FUSED): lane (plane 16g + j, kq) holds E[plane][4kq + e] in K slots 8kq + e, e < 4; zeros above
    const int j = lane & 15, kq = lane >> 4;
    bf16x8_t eb[ENCODE ? (RP + 15) / 16 : 1];
    if constexpr (ENCODE)
#pragma unroll
        for (int g = 0; g < (RP + 15) / 16; ++g) {
            u32x2_t ev = {0u, 0u};
            if (16 * g + j < r) ev = *reinterpret_cast<const u32x2_t *>(E + (16 * g + j) * 16 + 4 * kq);
            eb[g] = __builtin_bit_cast(bf16x8_t, u32x4_t{ev[0], ev[1], 0u, 0u});
        }

    // ---- DMA sources ------------------------------------------------------------------------------------
    // What: one instruction per plane (16 L rows x 64 bytes); lane -> (L = lane/4, 16-byte chunk = lane%4)
    const bf16_t *srcW[PW];
    {
        int jc = J0 + 8 * (lane & 3);
        jc = jc < N ? jc : N - 8;                     // columns past the edge feed only discarded outputs
#pragma unroll
        for (int t = 0; t < PW; ++t) {
            const int p = wave * PW + t;
            srcW[t] = What + ((size_t)(p < r ? p : 0) * K + (lane >> 2)) * N + jc;
        }
    }
    // A side
    const bf16_t *srcA[AW];
    if (ENCODE) {
        // X sub-block: 128 rows x 128 bytes as they lie; instruction q covers rows 8q..8q+7; wavefront w fetches tile rows 4w .. 4w + 3
#pragma unroll
        for (int t = 0; t < AW; ++t) {
            long gr = (long)I0 * 4 + 8 * (wave * AW + t) + (lane >> 3);
            gr = gr < (long)M * 4 ? gr : (long)M * 4 - 1;
            srcA[t] = Xin + (size_t)gr * k_elems + 8 * (lane & 7);
        }
    } else {
        // Xhat: one instruction per plane (32 I rows x 32 bytes); lane -> (I = lane/2, half = lane%2)
        int gi = I0 + (lane >> 1);
        gi = gi < M ? gi : M - 1;
#pragma unroll
        for (int t = 0; t < AW; ++t) {
            const int p = wave * PW + t;
            srcA[t] = Xin + plane_row_base(gi, pg, r, K) + (size_t)(p < r ? p : 0) * pg * K + 8 * (lane & 1);
        }
    }
    auto issue = [&](int c) {
        const int slot = c % NS;
#pragma unroll
        for (int t = 0; t < AW; ++t) {
            dma16(srcA[t], lds0 + slot * L::A_STAGE + (wave * AW + t) * 1024);
            srcA[t] += ENCODE ? KC * 4 : KC;          // 16 tile columns further
        }
#pragma unroll
        for (int t = 0; t < PW; ++t) {
            dma16(srcW[t], lds0 + L::W + slot * L::W_STAGE + (wave * PW + t) * 1024);
            srcW[t] += (size_t)KC * N;
        }
    };

    // ---- fragment offsets --------------------------------------------------------------------------------
    const int frow = lane & 31, fh = lane >> 5;
    const int offA = frow * 32 + fh * 16;             // Xhat stage of one plane: [I][16 L], 32-byte rows
    int offB[2];                                      // What stage of one plane: [16 L][32 J], 64-byte rows
    {
        const int i = lane & 15, blk = (lane >> 4) & 1;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) offB[kk] = (8 * fh + 4 * kk + (i >> 2)) * 64 + (16 * blk + 4 * (i & 3)) * 2;
    }

    f32x16_t acc[PW];
#pragma unroll
    for (int t = 0; t < PW; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;

    // this wavefront's four tile rows of stage c, from the X rows it fetched, into encoded stage buf
    auto encode = [&](int c, int buf) {
        const char *st = sA + (c % NS) * L::A_STAGE;
        char *out = sXh + buf * L::XH_STAGE;
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) {
            const int I = 4 * wave + ii;
            const u32x2_t x = *reinterpret_cast<const u32x2_t *>(st + (4 * I + kq) * 128 + j * 8);       // tile column j, matrix row kq
            const bf16x8_t hf = __builtin_bit_cast(bf16x8_t, u32x4_t{x[0], x[1], 0u, 0u});
#pragma unroll
            for (int g = 0; g < (RP + 15) / 16; ++g) {
                const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
                const f32x4_t o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hf, eb[g], zero, 0, 0, 0);
                if (16 * g + j < RP)                  // tile columns 4 kq .. 4 kq + 3 of plane 16 g + j
                    *reinterpret_cast<u32x2_t *>(out + (16 * g + j) * L::PITCH + I * 32 + kq * 8) =
                        u32x2_t{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
            }
        }
    };
    auto multiply = [&](const char *xh, int c) {
        const char *st = sW + (c % NS) * L::W_STAGE;
#pragma unroll
        for (int t = 0; t < PW; ++t) {
            const int p = wave * PW + t;
            const bf16x8_t a = *reinterpret_cast<const bf16x8_t *>(xh + p * L::PITCH + offA);
            const v4i16_t b0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16_t *)STL_LDS(st + p * 1024 + offB[0]));
            const v4i16_t b1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16_t *)STL_LDS(st + p * 1024 + offB[1]));
            struct { v4i16_t lo, hi; } both = {b0, b1};
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8_t, both), acc[t], 0, 0, 0);
        }
    };

    const int nch = K / KC;
#pragma unroll
    for (int c = 0; c < NS - 1; ++c)
        if (c < nch) issue(c);
    // Loads complete in the order they were issued; the waits leave the stages behind the one that is needed in flight.
    if constexpr (L::TWICE) {
        pipe::wait_stages<LOADS, NS - 2>(nch - 1);
        encode(0, 0);
        sD[tid] = bf16_to_f32(dreg);
        for (int c = 0; c < nch; ++c) {
            pipe::wait_stages<LOADS, NS - 3>(nch - 2 - c < 0 ? 0 : nch - 2 - c);       // stage c + 1 has landed
            wait_lds();
            block_barrier();                          // encoded stage c and What stage c visible to all; stage c - 1 is free
            if (c + NS - 1 < nch) issue(c + NS - 1);
            if (c + 1 < nch) encode(c + 1, (c + 1) & 1);
            multiply(sXh + (c & 1) * L::XH_STAGE, c);
        }
    } else {
        sD[tid] = bf16_to_f32(dreg);
        for (int c = 0; c < nch; ++c) {
            pipe::wait_stages<LOADS, NS - 2>(nch - 1 - c);                             // stage c has landed
            block_barrier();                          // for all; stage c - 1 is free
            if (c + NS - 1 < nch) issue(c + NS - 1);
            if (ENCODE) {
                encode(c, 0);
                wait_lds();
                block_barrier();                      // encoded stage visible to all wavefronts
            }
            multiply(ENCODE ? sXh : sA + (c % NS) * L::A_STAGE, c);
        }
    }

    // ---- exchange: accumulator e of plane p is Yhat[p][I = 8*(e/4) + 4h + e%4][J = lane%32] ---------------------
    block_barrier();
    float *sY = reinterpret_cast<float *>(smem);      // [p][I][J]
#pragma unroll
    for (int t = 0; t < PW; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) sY[((wave * PW + t) * BI + 8 * (e >> 2) + 4 * fh + (e & 3)) * BJ + frow] = acc[t][e];
    __syncthreads();

    // ---- decode: 2 tiles per thread, both per plane so that the decoder's row is read from LDS once ---------------------------
    float cq[2][16];
#pragma unroll
    for (int it = 0; it < 2; ++it)
#pragma unroll
        for (int q = 0; q < 16; ++q) cq[it][q] = 0.f;
    const int I = tid >> 5, J = tid & 31, gj = J0 + J;        // tile rows I, I + 16
#pragma unroll 4
    for (int p = 0; p < r; ++p) {
        float y[2];
#pragma unroll
        for (int it = 0; it < 2; ++it) y[it] = sY[(p * BI + I + 16 * it) * BJ + J];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const f32x4_t d = *reinterpret_cast<const f32x4_t *>(sD + p * 16 + 4 * q4);
#pragma unroll
            for (int it = 0; it < 2; ++it)
#pragma unroll
                for (int e = 0; e < 4; ++e) cq[it][4 * q4 + e] = fmaf(d[e], y[it], cq[it][4 * q4 + e]);
        }
    }
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int gi = I0 + I + 16 * it;
        if (gi >= M || gj >= N) continue;
        if (Ysave != nullptr)
            for (int p = 0; p < r; ++p)
                Ysave[plane_row_base(gi, pg, r, N) + (size_t)p * pg * N + gj] = f32_to_bf16(sY[(p * BI + I + 16 * it) * BJ + J]);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            float c0 = cq[it][4 * a], c1 = cq[it][4 * a + 1], c2 = cq[it][4 * a + 2], c3 = cq[it][4 * a + 3];
            if (GELU) { c0 = gelu_erf(c0); c1 = gelu_erf(c1); c2 = gelu_erf(c2); c3 = gelu_erf(c3); }
            const u32x2_t w = {pack_bf16x2(c0, c1), pack_bf16x2(c2, c3)};
            *reinterpret_cast<u32x2_t *>(C + ((size_t)gi * 4 + a) * n_elems + (size_t)gj * 4) = w;
        }
    }
}

}  // namespace fused

bool block_forward_eligible(int dtype, int M, int K, int N, int r)
{
    return dtype == 1 && r >= 1 && r <= 32 && (K % fused::KC) == 0 && (N % 8) == 0 && N >= 8 && M >= 1;
}

// Stages of the ring, at RP = 8, 16 or 32 padded planes.  While every CU has at most one block, LDS holds as many as fit; beyond, two
// where that gives a CU two blocks or more (all of it, at 9 to 16 planes with the encode and above 16, is one block's either
// way).  us, deep ring / two stages: encode in the kernel, r = 8, 8192 x 64 -> 4096 (2048 blocks) 31.6 / 20.8, 4096 x 2048 -> 2048 (512)
// 52.6 / 39.2, 4096 x 512 -> 1024 (256) 11.5 / 11.6; planes read, r = 8, 8192 x 64 -> 4096 34.3 / 18.7, r = 16 49.0 / 30.1;
// encode in the kernel, r = 16, 4096 x 1024 -> 1152 (288) 36.4 / 44.0.
constexpr int ring_stages(int RP, bool encode, bool shared)
{
    if (shared && (RP == 8 || (RP == 16 && !encode))) return 2;
    return RP == 8 ? 5 : RP == 32 ? 2 : encode ? 3 : 4;
}

static long block_count(int M, int N) { return (long)((M + fused::BI - 1) / fused::BI) * ((N + fused::BJ - 1) / fused::BJ); }

int block_forward_ring(bool encode, int M, int N, int r)
{
    return ring_stages(r <= 8 ? 8 : r <= 16 ? 16 : 32, encode, block_count(M, N) > pipe::cu_count());
}

template <int RP, bool ENCODE, bool GELU, int NS>
static hipError_t launch_block_ring(const void *Xin, const void *What, const void *E, const void *Dm, void *C, void *Ysave,
                                 int M, int K, int N, int r, int pg, hipStream_t s)
{
    auto kern = fused::stl_block_kernel<RP, ENCODE, GELU, NS>;
    constexpr int smem = fused::Map<RP, ENCODE, NS>::BYTES;
    static_assert(smem <= 160 * 1024, "LDS budget");
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, smem, granted); e != hipSuccess) return e;
    const int bj = (N + fused::BJ - 1) / fused::BJ;
    const long total = block_count(M, N);
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(fused::NW * 64), smem, s, (const bf16_t *)Xin, (const bf16_t *)What,
                       (const bf16_t *)E, (const bf16_t *)Dm, (bf16_t *)C, (bf16_t *)Ysave, M, K, N, r, bj, pg);
    return hipGetLastError();
}

template <int RP, bool ENCODE, bool GELU>
static hipError_t launch_block_t(const void *Xin, const void *What, const void *E, const void *Dm, void *C, void *Ysave,
                                 int M, int K, int N, int r, int pg, hipStream_t s)
{
    constexpr int ALONE = ring_stages(RP, ENCODE, false), SHARED = ring_stages(RP, ENCODE, true);
    return block_forward_ring(ENCODE, M, N, r) == ALONE
               ? launch_block_ring<RP, ENCODE, GELU, ALONE>(Xin, What, E, Dm, C, Ysave, M, K, N, r, pg, s)
               : launch_block_ring<RP, ENCODE, GELU, SHARED>(Xin, What, E, Dm, C, Ysave, M, K, N, r, pg, s);
}

template <int RP>
static hipError_t launch_block_rp(bool encode_in_kernel, const void *Xin, const void *What, const void *E,
                                  const void *Dm, void *C, void *Ysave, int M, int K, int N, int r, bool gelu, int pg,
                                  hipStream_t s)
{
    if (encode_in_kernel)
        return gelu ? launch_block_t<RP, true, true>(Xin, What, E, Dm, C, Ysave, M, K, N, r, pg, s)
                    : launch_block_t<RP, true, false>(Xin, What, E, Dm, C, Ysave, M, K, N, r, pg, s);
    return gelu ? launch_block_t<RP, false, true>(Xin, What, E, Dm, C, Ysave, M, K, N, r, pg, s)
                : launch_block_t<RP, false, false>(Xin, What, E, Dm, C, Ysave, M, K, N, r, pg, s);
}

hipError_t launch_block_forward(bool encode_in_kernel, const void *Xin, const void *What, const void *E, const void *Dm,
                                void *C, void *Ysave, int M, int K, int N, int r, bool gelu, int pg, hipStream_t s)
{
    if (pg <= 0) pg = M;
    if (encode_in_kernel && small_forward(M, N, r)) return launch_small_forward(Xin, What, E, Dm, C, Ysave, M, K, N, r, gelu, false, pg, s);
    if (r <= 8) return launch_block_rp<8>(encode_in_kernel, Xin, What, E, Dm, C, Ysave, M, K, N, r, gelu, pg, s);
    if (r <= 16) return launch_block_rp<16>(encode_in_kernel, Xin, What, E, Dm, C, Ysave, M, K, N, r, gelu, pg, s);
    return launch_block_rp<32>(encode_in_kernel, Xin, What, E, Dm, C, Ysave, M, K, N, r, gelu, pg, s);
}

}  // namespace stl
