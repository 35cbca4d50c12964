// The single-launch forward (see stl_fused.hip) of few blocks: a workgroup owns 16 x 16 output tiles and all r <= 32 planes of them.
//
// A problem of a few blocks is a chain of contraction steps on a few CUs: what it takes is the bytes that one CU brings in (of every 16 tile
// columns a block of BI x BJ tiles reads 512 BI bytes of X and 32 r BJ of What) and the instructions and waits of a step.  A
// quarter of the 32 x 32 tiles on four times as many CUs needs half the bytes on each.
//
// Eight wavefronts, 32 tile columns per step.  Both operands come through registers, DEPTH steps ahead: two (with three a step takes 5 to 9 %
// longer, with four 8 to 15: What's lines of 128 bytes, of which a block uses 32, push each other out of the L1; so it is they that bound a
// step of many planes).  Wavefront w encodes two tile
// rows (a lane holds a row of two neighbouring tiles, so that two products leave it with eight neighbouring columns of a plane: one
// 16-byte write), one step ahead of the products and into the other of two buffers: one barrier per step.  It accumulates planes w RP / 8 ..,
// whose part of What no other wavefront reads: it passes through LDS for the transposing reads alone, without a barrier.  The
// sums are exchanged through LDS in fp32 and decoded by MFMA, rows = the 16 entries of a tile, columns = tiles, so that a lane ends with a
// row of a tile: from fp32 (16x16x4, as the other single-launch form bit for bit), or rounded to bf16 first, which is what three
// launches do, bit for bit.
//
// us a call among others, 32 x 32 blocks / this / three launches: 128 x 512 -> 512, r = 8 8.8 / 5.2 / 11.4 (replayed from a graph, without what a host
// takes to enqueue a launch, 9.1 / 4.5 / 10.5); 1024 x 512 -> 1024, r = 8 9.1 / 5.3 / 11.5, r = 32 16.4 / 9.1 / 15.1; 256 x 2048 -> 512, r = 8 24.8 / 8.4 /
// 12.9; 1024 x 1024 -> 1024, r = 16 17.2 / 8.7 / 13.7, r = 32 25.4 / 13.8 / 17.1 (13.1 rounded: one product decodes what takes eight of fp32).
#include "stl_gemm_pipe.h"

namespace stl {
namespace fused_small {

using pipe::block_barrier;
using pipe::static_for;
using pipe::v4i16_t;

constexpr int BI = 16, BJ = 16, KC = 32, NW = 8, DEPTH = 2;

template <int RP>
struct Map {
    static constexpr int PW = RP / NW;
    static constexpr int PITCH = 1024 + 16, XH_STAGE = RP * PITCH;             // of a plane of Xhat, 16 I x 32 L: planes on different banks
    static constexpr int W = 2 * XH_STAGE, LOOP = W + RP * 1024;               // What: 32 L x 16 J per plane
    static constexpr int Y_PITCH = 256 + 16, Y = RP * Y_PITCH * 4;             // floats, of a plane of sums
    static constexpr int BYTES = LOOP > Y ? LOOP : Y;
};

// GELU on the output; RP: planes padded to 8, 16 or 32 (those beyond r are computed and dropped); ROUND: the sums are rounded to bf16
// before they are decoded
template <int RP, bool GELU, bool ROUND>
__global__ __launch_bounds__(NW * 64) void stl_small_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ What, const bf16_t *__restrict__ E,
                                                            const bf16_t *__restrict__ Dm, bf16_t *__restrict__ C, bf16_t *__restrict__ Ysave, int M,
                                                            int K, int N, int r, int blocks_i, int total, int pg)
{
    typedef Map<RP> L;
    constexpr int PW = L::PW, G = (RP + 15) / 16;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 15, kq = lane >> 4;

    // each XCD takes neighbouring block columns: the same part of What for all its workgroups
    const int v = pipe::first_block(total);
    if (v >= pipe::end_block(total)) return;
    const int J0 = v / blocks_i * BJ, I0 = v % blocks_i * BI;
    const size_t k_elems = (size_t)K * 4, n_elems = (size_t)N * 4;

    // encoder fragments: lane (plane 16 g + j, kq) holds E[plane][4 kq + e] in K slots 8 kq + e, e < 4; zeros above.  Decoder fragments:
    // lane (entry q = j, kq) holds D[d_plane(s)][q].  Planes beyond r are read as the last one and cleared where they are used, so that
    // no load hangs on a condition.
    u32x2_t er[G];
    constexpr int ND = ROUND ? 8 : RP / 4;            // planes of a lane: 8 kq + s, or 4 s + kq
    bf16_t dr[ND];
    auto d_plane = [&](int s) { return ROUND ? 8 * kq + s : 4 * s + kq; };
#pragma unroll
    for (int g = 0; g < G; ++g) er[g] = *reinterpret_cast<const u32x2_t *>(E + (16 * g + j < r ? 16 * g + j : r - 1) * 16 + 4 * kq);
#pragma unroll
    for (int s = 0; s < ND; ++s) dr[s] = Dm[(d_plane(s) < r ? d_plane(s) : r - 1) * 16 + j];

    // sources: X, matrix row kq of tile rows 2 w, 2 w + 1, tile columns 2 j, 2 j + 1; What, row lane / 2 of a plane, columns 8 (lane % 2) ..
    const bf16_t *srcX[2], *srcW[PW];
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) {
        long gr = ((long)I0 + 2 * wave + ii) * 4 + kq;
        gr = gr < (long)M * 4 ? gr : (long)M * 4 - 1;                          // rows past the edge feed only discarded outputs
        srcX[ii] = X + (size_t)gr * k_elems + 8 * j;
    }
    {
        int jc = J0 + 8 * (lane & 1);
        jc = jc < N ? jc : N - 8;                                              // so do columns
#pragma unroll
        for (int t = 0; t < PW; ++t) {
            const int p = wave * PW + t;
            srcW[t] = What + ((size_t)(p < r ? p : 0) * K + (lane >> 1)) * N + jc;
        }
    }
    const int nst = (K + KC - 1) / KC;
    u32x4_t xr[DEPTH][2], wr[DEPTH][PW];
    // step c; one beyond the last reads the last once more (a load that may or may not be issued would make the waits of those
    // around it wait for all)
    auto fetch = [&](auto d_c, int c) {
        constexpr int d = decltype(d_c)::value;
        c = c < nst ? c : nst - 1;
        // half of a last step (K is a multiple of 16): the other half is fetched from the first one's place and dropped
        const bool half = KC * c + 16 >= K;
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) xr[d][ii] = *reinterpret_cast<const u32x4_t *>(srcX[ii] + (size_t)c * (KC * 4) - (half && j >= 8 ? 64 : 0));
#pragma unroll
        for (int t = 0; t < PW; ++t) wr[d][t] = *reinterpret_cast<const u32x4_t *>(srcW[t] + ((size_t)c * KC - (half && lane >= 32 ? 16 : 0)) * N);
        __builtin_amdgcn_sched_barrier(0);
    };
    static_for<0, DEPTH>([&](auto d_c) { fetch(d_c, decltype(d_c)::value); });

#pragma unroll
    for (int g = 0; g < G; ++g)
        if (16 * g + j >= r) er[g] = u32x2_t{0u, 0u};
    f32x4_t acc[PW];
#pragma unroll
    for (int t = 0; t < PW; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    char *slab = smem + L::W + wave * (PW * 1024);
    bf16x8_t va[PW], vb[PW];
    // step c's operands into LDS: this wavefront's part of What, and of Xhat for all
    auto put = [&](auto d_c, int c) {
        constexpr int d = decltype(d_c)::value;
        const bool half = KC * c + 16 >= K;
#pragma unroll
        for (int t = 0; t < PW; ++t) *reinterpret_cast<u32x4_t *>(slab + t * 1024 + lane * 16) = half && lane >= 32 ? u32x4_t{0u, 0u, 0u, 0u} : wr[d][t];
        char *out = smem + (c & 1) * L::XH_STAGE;
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
            const int I = 2 * wave + ii;
            const u32x4_t x = xr[d][ii];
            const bf16x8_t h0 = __builtin_bit_cast(bf16x8_t, u32x4_t{x[0], x[1], 0u, 0u}), h1 = __builtin_bit_cast(bf16x8_t, u32x4_t{x[2], x[3], 0u, 0u});
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const bf16x8_t eb = __builtin_bit_cast(bf16x8_t, u32x4_t{er[g][0], er[g][1], 0u, 0u});
                const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
                const f32x4_t o0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, eb, zero, 0, 0, 0);
                const f32x4_t o1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1, eb, zero, 0, 0, 0);
                // tile columns 8 kq .. 8 kq + 7 of plane 16 g + j
                u32x4_t w = {pack_bf16x2(o0[0], o1[0]), pack_bf16x2(o0[1], o1[1]), pack_bf16x2(o0[2], o1[2]), pack_bf16x2(o0[3], o1[3])};
                if (half && kq >= 2) w = u32x4_t{0u, 0u, 0u, 0u};
                if (16 * g + j < RP) *reinterpret_cast<u32x4_t *>(out + (16 * g + j) * L::PITCH + I * 64 + ((kq ^ pipe::fswz(I)) << 4)) = w;
            }
        }
    };
    // fragments of step c
    auto read = [&](int c) {
        const char *xh = smem + (c & 1) * L::XH_STAGE;
#pragma unroll
        for (int t = 0; t < PW; ++t) {
            va[t] = *reinterpret_cast<const bf16x8_t *>(xh + (wave * PW + t) * L::PITCH + j * 64 + ((kq ^ pipe::fswz(j)) << 4));
            const char *w = slab + t * 1024 + (8 * kq + (j >> 2)) * 32 + (j & 3) * 8;
            const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16_t *)STL_LDS(w));
            const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16_t *)STL_LDS(w + 128));
            struct { v4i16_t a, b; } both = {lo, hi};
            vb[t] = __builtin_bit_cast(bf16x8_t, both);
        }
    };

    put(std::integral_constant<int, 0>{}, 0);
    auto step = [&](auto d_c, int c, auto last_c) {
        constexpr int d = decltype(d_c)::value;
        constexpr bool LAST = decltype(last_c)::value;      // of the last DEPTH steps: nothing to fetch, and there may be fewer
        if (LAST && c >= nst) return;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        block_barrier();                              // Xhat of step c visible to all; nobody reads step c - 1 any more
        read(c);
        if constexpr (!LAST) fetch(d_c, c + DEPTH);   // step c's registers are free
        if (!LAST || c + 1 < nst) put(std::integral_constant<int, (d + 1) % DEPTH>{}, c + 1);
#pragma unroll
        for (int t = 0; t < PW; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb[t], va[t], acc[t], 0, 0, 0);
    };
    int c = 0;
    for (; c + DEPTH < nst; c += DEPTH) static_for<0, DEPTH>([&](auto d_c) { step(d_c, c + decltype(d_c)::value, std::false_type{}); });
    static_for<0, DEPTH>([&](auto d_c) { step(d_c, c + decltype(d_c)::value, std::true_type{}); });

    // ---- exchange: element e of plane p's sums is Yhat[p][I = j][J = 4 kq + e] -------------------------------------------
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    block_barrier();
    float *sY = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int t = 0; t < PW; ++t) {
        const int p = wave * PW + t;
        if (p >= r) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f32x4_t *>(sY + p * L::Y_PITCH + j * 16 + 4 * kq) = acc[t];
    }
    __syncthreads();

    // ---- decode: tile rows 2 w, 2 w + 1; lane (tile column j, kq) ends with matrix row kq of its tile ----------------------
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) {
        const int I = 2 * wave + ii;
        f32x4_t c = {0.f, 0.f, 0.f, 0.f};
        if constexpr (ROUND) {
            u32x4_t dw, yw;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = 8 * kq + 2 * i;
                const float *y = sY + (p < RP ? p : 0) * L::Y_PITCH + I * 16 + j;
                dw[i] = (p < r ? dr[2 * i] : 0u) | (p + 1 < r ? (uint32_t)dr[2 * i + 1] << 16 : 0u);
                yw[i] = p < RP ? pack_bf16x2(y[0], y[L::Y_PITCH]) : 0u;
            }
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, dw), __builtin_bit_cast(bf16x8_t, yw), c, 0, 0, 0);
        } else {
#pragma unroll
            for (int s = 0; s < ND; ++s)
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(4 * s + kq < r ? bf16_to_f32(dr[s]) : 0.f, sY[(4 * s + kq) * L::Y_PITCH + I * 16 + j], c, 0, 0, 0);
        }
        if (GELU)
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = gelu_erf(c[e]);
        if (I0 + I < M && J0 + j < N) store4(C + ((size_t)(I0 + I) * 4 + kq) * n_elems + (size_t)(J0 + j) * 4, c);
    }
    if (Ysave != nullptr)                             // eight columns of a plane's row at a time
        for (int i = tid; i < r * 32; i += NW * 64) {
            const int p = i >> 5, I = (i >> 1) & 15, J = 8 * (i & 1);
            if (I0 + I >= M || J0 + J >= N) continue;
            const float *y = sY + p * L::Y_PITCH + I * 16 + J;
            const f32x4_t a = *reinterpret_cast<const f32x4_t *>(y), b = *reinterpret_cast<const f32x4_t *>(y + 4);
            *reinterpret_cast<u32x4_t *>(Ysave + plane_row_base(I0 + I, pg, r, N) + (size_t)p * pg * N + J0 + J) =
                u32x4_t{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3])};
        }
}

}  // namespace fused_small

static long small_blocks(int M, int N) { return (long)((M + fused_small::BI - 1) / fused_small::BI) * ((N + fused_small::BJ - 1) / fused_small::BJ); }

// A CU has a block, or at up to 16 planes two.  us, 32 x 32 blocks / this, with 384 and 512 blocks: r = 8 6.7 / 6.1 and 7.0 / 6.0 at K = 64, 12.8 / 9.3 and
// 13.2 / 10.4 at 192; r = 16, K = 128 11.2 / 8.7 and 12.2 / 10.6; r = 32 9.7 / 9.9 and 9.8 / 10.8 at K = 32, 11.9 / 11.1 and 12.3 / 12.3 at 64; with 1024
// blocks r = 8, K = 128 11.1 / 12.2.
bool small_forward(int M, int N, int r) { return small_blocks(M, N) <= (r <= 16 ? 2 : 1) * pipe::cu_count(); }

template <int RP, bool GELU, bool ROUND>
static hipError_t launch_small_cfg(const void *X, const void *What, const void *E, const void *Dm, void *C, void *Ysave, int M, int K, int N, int r,
                                   int pg, hipStream_t s)
{
    auto kern = fused_small::stl_small_kernel<RP, GELU, ROUND>;
    constexpr int smem = fused_small::Map<RP>::BYTES;
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, smem, granted); e != hipSuccess) return e;
    const int total = (int)small_blocks(M, N);
    hipLaunchKernelGGL(kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(fused_small::NW * 64), smem, s, (const bf16_t *)X, (const bf16_t *)What,
                       (const bf16_t *)E, (const bf16_t *)Dm, (bf16_t *)C, (bf16_t *)Ysave, M, K, N, r, (M + fused_small::BI - 1) / fused_small::BI, total, pg);
    return hipGetLastError();
}

hipError_t launch_small_forward(const void *X, const void *What, const void *E, const void *Dm, void *C, void *Ysave, int M, int K, int N, int r,
                                bool gelu, bool round, int pg, hipStream_t s)
{
    if (!block_forward_eligible(1, M, K, N, r) || !small_forward(M, N, r)) return hipErrorInvalidValue;
    if (pg <= 0) pg = M;
    auto launch = [&](auto rp_c) {
        constexpr int RP = decltype(rp_c)::value;
        if (round)
            return gelu ? launch_small_cfg<RP, true, true>(X, What, E, Dm, C, Ysave, M, K, N, r, pg, s)
                        : launch_small_cfg<RP, false, true>(X, What, E, Dm, C, Ysave, M, K, N, r, pg, s);
        return gelu ? launch_small_cfg<RP, true, false>(X, What, E, Dm, C, Ysave, M, K, N, r, pg, s)
                    : launch_small_cfg<RP, false, false>(X, What, E, Dm, C, Ysave, M, K, N, r, pg, s);
    };
    if (r <= 8) return launch(std::integral_constant<int, 8>{});
    if (r <= 16) return launch(std::integral_constant<int, 16>{});
    return launch(std::integral_constant<int, 32>{});
}

}  // namespace stl
