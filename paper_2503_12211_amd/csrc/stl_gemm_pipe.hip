// Pipelined batched plane products on the CDNA4 matrix cores (step (ii) of Algorithm 1, Claim 3.4):
//     Out[p][i][j] (+)= sum_l A[p](i,l) * B[p](l,j)       bf16 x bf16 -> fp32, p < r planes.
//
// One block of one plane per workgroup, 16x16x32 MFMA; HBM -> LDS goes through the LDS-DMA path
// (global_load_lds, 16 bytes per lane, no VGPR staging) into a ring of NS stages of 32 contraction
// elements each, issued NS-1 stages ahead of their use, so that an L2 / HBM miss has several
// MFMA stages of time to land.  Operands keep their memory orientation in LDS:
//   * contraction-contiguous operand ([row][l]): 64-byte LDS rows, fragments by ds_read_b128;
//   * contraction-major operand ([l][row]):      512-byte LDS rows, fragments by the transposing
//     ds_read_b64_tr_b16 (a 16-lane group turns 4 l-rows x 16 columns into 4 consecutive l per lane).
// An LDS-DMA instruction writes 64 lanes x 16 bytes contiguously, so bank swizzles are applied by
// permuting which global 16-byte chunk each lane fetches.
#include "stl_gemm_pipe.h"
#include <cmath>

namespace stl {

// A_T: A stored [l][i];  B_T: B stored [l][j].  Nj % 8 == 0 and Mi % 8 == 0 for A_T; a [row][l] operand needs Kl % 8 == 0.
// KTAIL: Kl is no multiple of 32.
//
// Blocks (see pipe_block for the choice): 256 x 256 for large planes (eight wavefronts of 128 x 64, four stages, one workgroup per CU: most flop per byte
// brought into LDS); 128 x 256 (the same with 64 x 64 each, five stages), 128 x 128 (four wavefronts of 64 x 64, four stages) and 64 x 64 (four of 32 x 32, eight stages of 8 KB) for
// planes that would leave CUs idle or whose time is the latency of the chain of stages.
//
// Persistent: the grid is one workgroup per CU (two of the smallest two blocks) and every workgroup walks over its share of the
// (plane, block) list.  When a block's MFMA loop ends, the first ring stages of the NEXT block are put in
// flight before the epilogue starts, so the HBM/L2 latency of the refill and the store traffic of the
// epilogue overlap instead of adding up.
template <int BM, int BN, int WAVES_M, int WAVES_N, int NS, bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL>
__global__ __launch_bounds__(WAVES_M *WAVES_N * 64) void gemm_pipe_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B,
                                                        TO *__restrict__ Out, int Mi, int Nj, int Kl, int tiles_m,
                                                        int tiles_n, int total, int a_pg, int b_pg, int o_pg, int batch)
{
    using namespace pipe;
    constexpr int NW = WAVES_M * WAVES_N, WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int FM = WM / 16, FN = WN / 16;
    constexpr int OPER_BYTES = BM * BKS * 2, STAGE_BYTES = (BM + BN) * BKS * 2;
    constexpr int D = (BM + BN) / 16 / NW;                 // DMA instructions per wavefront and stage
    constexpr int SLAB = slab_bytes<FM, FN, TO>();
    static_assert(NS >= 3, "ring depth");
    extern __shared__ __align__(16) char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: LDS-DMA destinations stay in SGPRs
    char *slab = smem + NS * STAGE_BYTES + wave * SLAB;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int per_plane = tiles_m * tiles_n;
    const int nks = (Kl + BKS - 1) / BKS;
    const uint32_t smem_lds = (uint32_t)(uintptr_t)STL_LDS(smem);

    Frag<A_T, BM> fa;
    Frag<B_T, BN> fb;
    fa.init(wm * WM, lane);
    fb.init(wn * WN, lane);

    // block list, block v -> (stacked problem, plane, block row, block column); the blocks of a workgroup are first_block(),
    // + block_step() ... below end_block()
    auto locate = [&](int v, int &pb, int &p, int &i0, int &j0) {
        const int q = v / per_plane;                 // (stacked problem, plane)
        const int rem = v - q * per_plane;
        pb = q / batch;
        p = q - pb * batch;
        i0 = (rem / tiles_n) * BM;
        j0 = (rem % tiles_n) * BN;
    };

    Src<A_T, BM, NW, KTAIL> sa;
    Src<B_T, BN, NW, KTAIL> sb;
    auto start_block = [&](int v) {      // point the DMA sources at block v and put its first NS-1 stages in flight
        // the lane id as an opaque value: what the sources derive from it is computed per block and occupies no registers while
        // the products run (spilled values would be reloaded between the loads issued here, and waited for with them)
        int sl = lane;
        asm volatile("" : "+v"(sl));
        int pb, p, i0, j0;
        locate(v, pb, p, i0, j0);
        sa.init(A, A_T ? Mi : Kl, i0, Mi, wave, sl, p, batch, a_pg, pb * (A_T ? Kl : Mi), Kl);
        sb.init(B, B_T ? Nj : Kl, j0, Nj, wave, sl, p, batch, b_pg, pb * (B_T ? Kl : Nj), Kl);
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) {
            if (s < nks) {
                sa.issue(smem_lds + s * STAGE_BYTES, wave, sl);
                sb.issue(smem_lds + s * STAGE_BYTES + OPER_BYTES, wave, sl);
            }
        }
    };

    const int step = block_step(), end = end_block(total);
    int v = first_block(total);
    if (v < end) start_block(v);

    WaveTile<FM, FN> w;
    for (; v < end; v += step) {
        int pb, p, i0, j0;
        locate(v, pb, p, i0, j0);
        w.clear();

        // Stage s+NS-1 is issued in iteration s; stage s+1 must have landed at the top of iteration s (its fragments are
        // fetched during stage s).  Stores of the previous epilogue may still be in flight: "at most N operations
        // outstanding" then over-waits but never under-waits.
        wait_stages<D, NS - 2>(nks - 1);
        block_barrier();
#pragma unroll
        for (int a = 0; a < FM; ++a) w.va[a] = fa.read(smem, a);
#pragma unroll
        for (int b = 0; b < FN; ++b) w.vb[0][b] = fb.read(smem + OPER_BYTES, b);

        // One stage.  STEADY: there is a stage to refill -- known at compile time, so that the loop over these stages
        // carries no test around the DMA instructions.  After the last stage the fragments of a stale ring slot are
        // fetched and never used.
        auto stage = [&](int s, auto par_c, auto steady_c) {
            constexpr int PAR = decltype(par_c)::value;
            constexpr bool STEADY = decltype(steady_c)::value;
            const bool refill = STEADY || s + NS - 1 < nks;
            if (STEADY) wait_vmcnt<D * (NS - 3)>();
            else wait_stages<D, NS - 3>(nks - 2 - s < 0 ? 0 : nks - 2 - s);
            block_barrier();   // stage s+1 visible to all; nobody reads stage s-1 any more
            const uint32_t dst = smem_lds + ((s + NS - 1) % NS) * STAGE_BYTES;
            const char *nxt = smem + ((s + 1) % NS) * STAGE_BYTES;
            if (KTAIL && !STEADY && s == nks - 1) w.mask(PAR, Kl - s * BKS, lane);
            w.template stage<PAR>([&](int f) { return fa.read(nxt, f); }, [&](int f) { return fb.read(nxt + OPER_BYTES, f); },
                                  [&](auto a_c) {
                                      // this wavefront's share of the refill, spread over the stage's products
                                      constexpr int a = decltype(a_c)::value, NA = decltype(sa)::NI, NB = decltype(sb)::NI;
                                      static_for<0, NA + NB>([&](auto j_c) {
                                          constexpr int j = decltype(j_c)::value;
                                          if constexpr (j * FM / (NA + NB) == a) {
                                              if (refill) {
                                                  if constexpr (j < NA) sa.issue_one(dst, wave, j);
                                                  else sb.issue_one(dst + OPER_BYTES, wave, j - NA);
                                              }
                                          }
                                      });
                                  });
            if (refill) {
                sa.next_stage(wave, lane);
                sb.next_stage(wave, lane);
            }
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        const int n_refill = nks > NS - 1 ? nks - (NS - 1) : 0;
        int s = 0;
        for (; s + 1 < n_refill; s += 2) {
            stage(s, I0{}, std::true_type{});
            stage(s + 1, I1{}, std::true_type{});
        }
        for (; s < nks; s += 2) {
            stage(s, I0{}, std::false_type{});
            if (s + 1 < nks) stage(s + 1, I1{}, std::false_type{});
        }

        // every wavefront is done with the ring: refill it for the next block before storing this one
        block_barrier();
        if (v + step < end) start_block(v + step);
        int el = lane;                                   // opaque, as above
        asm volatile("" : "+v"(el));
        w.template store<TO, ACC, false>(slab, Out + (size_t)p * o_pg * Nj, i0 + wm * WM, j0 + wn * WN, Mi, Nj, pb * Mi, o_pg, batch,
                                             el);
    }
}

bool plane_gemm_pipe_eligible(const GemmDesc &g)
{
    if (!plane_gemm_mfma_eligible(g)) return false;
    // 16-byte loads and stores at multiples of 16 bytes
    if (g.Nj % 8 || (g.a_kmajor && g.Mi % 8) || ((!g.a_kmajor || !g.b_kmajor) && g.Kl % 8)) return false;
    // a stage's 32 stored rows of an [l][row] operand stay inside one group (or there is one group only)
    auto stage_in_group = [&](int rows_per_group, bool grouped) { return rows_per_group % pipe::BKS == 0 || (!grouped && g.nb == 1); };
    if (g.a_kmajor && !stage_in_group(g.a_rows_per_group(), g.a_pg > 0)) return false;
    if (g.b_kmajor && !stage_in_group(g.b_rows_per_group(), g.b_pg > 0)) return false;
    // so do the rows of an epilogue pass
    if (g.o_pg > 0 && g.o_pg % 16) return false;
    // stacked problems: every problem's first stored row keeps those alignments; only the single-stage contraction
    // (attention-shaped products) is taken here, deeper stacked contractions go to the register-staged kernel
    if (g.nb > 1 && (g.Kl != pipe::BKS || (g.o_pg > 0 && g.Mi % 16))) return false;
    return pipe::offsets_fit(g);
}

// The block that takes the least time, from what each was seen to take (us, forward form, K = 32 .. 1024): a single round of
// blocks on the chip lasts a latency plus a time per stage, more where all CUs fetch and store at once; many rounds of the
// large blocks last a time per round, many small blocks a time per block.  M x K x N, r: us at 256 x 256 / 128 x 128 / 64 x 64:
//     16 x 1024 x 1024, 32: 24 / 17 / 16      256 x 256 x 256, 32: 11 / 7.8 / 7.6      512 x 512 x 512, 32: 18 / 16 / 27
//    512 x 192 x 768,  32: 13 / 13 / 28      512 x 768 x 192, 24: 21 / 14 / 14       1024 x 512 x 512, 32: 22 / 27 / 49
//   1024 x 1024 x 1024, 8: 26 / 25 / 37     2048 x 256 x 1024, 8: 16 / 18 / 38       4096 x 256 x 1024, 24: 69 / 89 / 209
// (before, every plane above 128 x 128 took 256 x 256 blocks, smaller ones register-staged 128 x 128 blocks: 24 us for
// the first of these and 10.7 for the second).
PipeBlock pipe_block(const GemmDesc &g)
{
    const double st = (g.Kl + pipe::BKS - 1) / pipe::BKS;
    auto blocks = [&](int bm, int bn) { return (double)((g.Mi + bm - 1) / bm) * ((g.Nj + bn - 1) / bn) * g.batch * g.nb; };
    // one workgroup per CU: full rounds, then a last round whose length grows with how many CUs it occupies
    auto rounds = [&](double b, double full, double lat, double load) {
        const double n = std::floor(b / 256), rem = b / 256 - n;
        return n > 0 ? n * full + (rem > 0 ? lat + rem * load : 0) : lat + rem * load;
    };
    // several workgroups per CU: latency of one block against the time all of them take
    auto many = [&](double lat, double work) { return std::sqrt(lat * lat + work * work); };
    const double t256 = rounds(blocks(256, 256), 5.3 + 0.83 * st, 6 + 0.56 * st, 2.5 + 0.2 * st);
    const double t128x256 = rounds(blocks(128, 256), 3.7 + 0.55 * st, 5 + 0.37 * st, 1.5 + 0.13 * st);
    const double t128 = many(4.1 + 0.375 * st, blocks(128, 128) * (0.005 + 0.00122 * st));
    const double t64 = many(4.6 + 0.13 * st, blocks(64, 64) * (0.006 + 0.00047 * st));
    if (t256 <= t128x256 && t256 <= t128 && t256 <= t64) return PipeBlock::b256;
    if (t128x256 <= t128 && t128x256 <= t64) return PipeBlock::b128x256;
    return t128 <= t64 ? PipeBlock::b128 : PipeBlock::b64;
}

static int cu_count()
{
    static const int n = []() {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
        return cus;
    }();
    return n;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int NS, bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL>
static hipError_t launch_pipe_cfg(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    constexpr int NW = WAVES_M * WAVES_N;
    auto kern = gemm_pipe_kernel<BM, BN, WAVES_M, WAVES_N, NS, A_T, B_T, TO, ACC, KTAIL>;
    constexpr int smem = NS * (BM + BN) * pipe::BKS * 2 + NW * pipe::slab_bytes<BM / WAVES_M / 16, BN / WAVES_N / 16, TO>();
    static_assert(smem <= 160 * 1024, "LDS budget");
    constexpr int per_cu = 160 * 1024 / smem > 2 ? 2 : 160 * 1024 / smem;
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, granted); e != hipSuccess) return e;
    const int tiles_m = (g.Mi + BM - 1) / BM, tiles_n = (g.Nj + BN - 1) / BN;
    const long total = (long)tiles_m * tiles_n * g.batch * g.nb;
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    const int wgs = cu_count() * per_cu;                   // they walk the block list
    const unsigned grid = pipe::list_grid(total, wgs);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NW * 64), smem, s, (const bf16_t *)A, (const bf16_t *)B, (TO *)Out, g.Mi, g.Nj,
                       g.Kl, tiles_m, tiles_n, (int)total, g.a_rows_per_group(), g.b_rows_per_group(), g.o_rows_per_group(), g.batch);
    return hipGetLastError();
}

template <bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL>
static hipError_t launch_pipe_block(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    switch (pipe_block(g)) {
        case PipeBlock::b256: return launch_pipe_cfg<256, 256, 2, 4, 4, A_T, B_T, TO, ACC, KTAIL>(g, A, B, Out, s);
        case PipeBlock::b128x256: return launch_pipe_cfg<128, 256, 2, 4, 5, A_T, B_T, TO, ACC, KTAIL>(g, A, B, Out, s);
        case PipeBlock::b128: return launch_pipe_cfg<128, 128, 2, 2, 4, A_T, B_T, TO, ACC, KTAIL>(g, A, B, Out, s);
        case PipeBlock::b64: return launch_pipe_cfg<64, 64, 2, 2, 8, A_T, B_T, TO, ACC, KTAIL>(g, A, B, Out, s);
    }
    return hipErrorInvalidValue;
}

template <bool A_T, bool B_T, typename TO, bool ACC>
static hipError_t launch_pipe_tail(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    return g.Kl % pipe::BKS ? launch_pipe_block<A_T, B_T, TO, ACC, true>(g, A, B, Out, s)
                            : launch_pipe_block<A_T, B_T, TO, ACC, false>(g, A, B, Out, s);
}

// The [l][row] form of an operand is chosen per operand; the fp32 (weight-gradient) output exists for the
// doubly contraction-major form only, which is the only one the library asks for.
static hipError_t launch_pipe_form(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    if (g.out_f32) {
        if (!(g.a_kmajor && g.b_kmajor)) return hipErrorInvalidValue;
        return g.accumulate ? launch_pipe_tail<true, true, float, true>(g, A, B, Out, s)
                            : launch_pipe_tail<true, true, float, false>(g, A, B, Out, s);
    }
    if (g.accumulate) return hipErrorInvalidValue;
    if (g.a_kmajor) {
        if (!g.b_kmajor) return hipErrorInvalidValue;
        return launch_pipe_tail<true, true, bf16_t, false>(g, A, B, Out, s);
    }
    if (g.b_kmajor) return launch_pipe_tail<false, true, bf16_t, false>(g, A, B, Out, s);
    return launch_pipe_tail<false, false, bf16_t, false>(g, A, B, Out, s);
}

hipError_t launch_plane_gemm_pipe(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    // refuse here as well what plane_gemm_pipe_eligible excludes, so that a change of the dispatch rule cannot reach a
    // form of the kernel that no test covers (stacked problems with more than one contraction stage among them)
    if (!plane_gemm_pipe_eligible(g)) return hipErrorInvalidValue;
    return launch_pipe_form(g, A, B, Out, s);
}

}  // namespace stl
