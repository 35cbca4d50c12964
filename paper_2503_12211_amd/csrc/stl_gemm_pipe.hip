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
//
// SPLIT (256 x 256 only): the blocks of a last round that is not full are dealt to all workgroups in parts (see pipe_split).
template <int BM, int BN, int WAVES_M, int WAVES_N, int NS, bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL, pipe::Split SPLIT>
__global__ __launch_bounds__(WAVES_M *WAVES_N * 64) void gemm_pipe_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B, TO *__restrict__ Out,
                                                                      int Mi, int Nj, int Kl, int tiles_m, int tiles_n, int total, int a_pg, int b_pg,
                                                                      int o_pg, int batch)
{
    using namespace pipe;
    const Products<TO> g{A, B, Out, Mi, Nj, Kl, a_pg, b_pg, o_pg, batch};
    extern __shared__ __align__(16) char smem[];
    typedef BlockRing<BM, BN, WAVES_M, WAVES_N, NS, A_T, B_T, TO, ACC, KTAIL> Ring;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: LDS-DMA destinations stay in SGPRs
    char *slab = smem + NS * Ring::STAGE_BYTES + wave * Ring::SLAB;
    const int per_plane = tiles_m * tiles_n, nks = (g.Kl + BKS - 1) / BKS;
    const uint32_t smem_lds = (uint32_t)(uintptr_t)STL_LDS(smem);

    // block list, block v -> (stacked problem, plane, block row, block column); the blocks of a workgroup are first_block(),
    // + block_step() ... below end_block()
    auto locate = [&](int v, int &pb, int &p, int &i0, int &j0) {
        const int q = v / per_plane;                 // (stacked problem, plane)
        const int rem = v - q * per_plane;
        pb = q / g.batch;
        p = q - pb * g.batch;
        i0 = (rem / tiles_n) * BM;
        j0 = (rem % tiles_n) * BN;
    };
    Ring ring;
    ring.init(wave, lane);
    auto start_block = [&](int v) {
        int pb, p, i0, j0;
        locate(v, pb, p, i0, j0);
        ring.start(g, nks, pb, p, i0, j0, smem_lds, wave, lane);
    };

    const int step = block_step(), end = SPLIT == Split::none ? end_block(total) : whole_end(total);
    int v = first_block(total);
    if constexpr (SPLIT == Split::none) {
        if (v < end) start_block(v);
        for (; v < end; v += step) {
            int pb, p, i0, j0;
            locate(v, pb, p, i0, j0);
            ring.block(g, nks, smem, smem_lds, slab, pb, p, i0, j0, wave, lane, [&]() {
                if (v + step < end) start_block(v + step);
            });
        }
    } else {
        PartWalk<SPLIT, SPLIT == Split::b128 ? 8 : 5, A_T, B_T, TO, ACC, KTAIL> parts;
        start_block(v);                                          // every workgroup has a whole block: total >= the grid
        for (; v < end; v += step) {
            int pb, p, i0, j0;
            locate(v, pb, p, i0, j0);
            ring.block(g, nks, smem, smem_lds, slab, pb, p, i0, j0, wave, lane, [&]() {
                if (v + step < end) start_block(v + step);
                else parts.begin(g, nks, end, total, tiles_m, tiles_n, smem_lds, wave, lane);
            });
        }
        parts.run(g, nks, smem, smem_lds, slab, wave, lane);
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

// The block that takes the least time, predicted from rounds of blocks over the workgroups that the chip holds (one per CU, two of
// the smaller blocks): a full round costs a time per stage and per byte stored, the last one a latency, a time per stage and
// more of both the more CUs it occupies.  Coefficients are least squares over 187 shapes (M from 16 to 4096 tiles, K and N from 32 to
// 1280, 8 to 64 planes, all product forms, 749 points); over shapes left out of the fit the block taken was 0.9 % slower than the
// fastest on average and at most 25 % (2.3 and 29 % with a rule of fewer terms that knew no rounds of the smaller blocks and
// no output type, which had 62 of 503 large planes more than 3 % slower than 256 x 256).  Some of them, us at
// 256 x 256 / 128 x 256 / 128 x 128 / 64 x 64:
//   Yhat   16 x 1024 x 1024, 32: 25 / 18 / 18 / 16    256 x 256 x 256, 32: 11 / 9.4 / 8.1 / 8.1    512 x 512 x 512, 32: 18 / 16 / 16 / 27
//        1024 x 256 x 256,  49: 15 / 18 / 19 / 31   1024 x 1024 x 1024, 8: 26 / 22 / 24 / 38     4096 x 256 x 1024, 24: 81 / 96 / 103 / 211
//   dXhat  208 x 128 x 624,  24: 17 / 13 / 12 / 7.8  3064 x 352 x 688, 12: 42 / 45 / 37 / 55
//   dWhat 1024 x 1024 x 1024, 8: 30 / 26 / 26 / 45   1024 x 1024 x 1024, 32: 77 / 101 / 116 / 189  2048 x 256 x 256, 49: 49 / 38 / 35 / 40
//   added to what is there  256 x 512 x 512, 49: 26 / 30 / 29 / 41   1024 x 1024 x 1024, 8: 39 / 31 / 31 / 50
//
// Split: what is left of the 256 x 256 blocks behind their last whole round (pipe_split) takes a time of the same form, in parts of 128 x 256 or
// 128 x 128; so does whole + parts compare with the other blocks.  Coefficients: least squares over 320 shapes of 1 to 8 rounds that end in one
// that is not full, 1.1 % slower than the fastest on average where taken at face value, but up to 19 % slower than without parts; taken where
// 5 % ahead, on 1 of the 320 more than 2 % slower (3), and all of them 2.1 % faster in the mean.  us whole / 128 x 256 / 128 x 128:
//   Yhat  1024 x 1024 x 1024, 49 (3.06 rounds): 111 / 104 / 103    4096 x 1024 x 256, 24 (1.5): 57 / 53 / 59    1500 x 1024 x 768, 16 (1.13): 51 / 42 / 40
//   dXhat 1024 x 1024 x 1024, 20 (1.25): 50 / 43 / 41              3200 x 192 x 768, 32 (1.63): 43 / 49 / 50
//   dWhat 3200 x 768 x 768, 32 (1.13): 161 / 139 / 129             added to what is there, 3072 x 768 x 1024, 32 (1.5): 195 / 171 / 190
namespace {
struct BlockCost {
    int m, n, workgroups;
    double round, round_stage, round_out;              // a full round: base, per stage of 32, per output size (2 bytes)
    double last, last_stage, last_out;                 // a last one that is not full
    double load_stage, load_out;                       // times the share of workgroups that it occupies
    double time(double full, double rem, const GemmDesc &g) const
    {
        const double st = (g.Kl + pipe::BKS - 1) / pipe::BKS, out = g.out_f32 ? (g.accumulate ? 4 : 2) : 1;
        return full * (round + round_stage * st + round_out * out) +
               (rem > 0 ? last + last_stage * st + last_out * out + rem * (load_stage * st + load_out * out) : 0);
    }
    double blocks(const GemmDesc &g) const { return (double)((g.Mi + m - 1) / m) * ((g.Nj + n - 1) / n) * g.batch * g.nb; }
    double time(const GemmDesc &g) const
    {
        const double x = blocks(g) / workgroups, full = std::floor(x);
        return time(full, x - full, g);
    }
};
constexpr BlockCost kCost[] = {{256, 256, 256, 0.94, 0.80, 4.58, 4.18, 0.60, 1.44, 0.19, 2.10},        // in the order of PipeBlock
                               {128, 256, 256, 1.34, 0.52, 2.40, 3.94, 0.42, 1.11, 0.12, 1.02},
                               {128, 128, 512, 1.08, 0.60, 2.13, 3.32, 0.36, 0.57, 0.32, 1.84},
                               {64, 64, 512, 1.86, 0.26, 0.59, 3.19, 0.14, 0.18, 0.19, 1.23}};
constexpr BlockCost kParts[] = {{128, 256, 256, 0.10, 0.37, 2.72, 4.15, 0.20, 1.58, 0.08, 1.00},       // behind whole rounds of 256 x 256
                                {128, 128, 256, 1.56, 0.27, 1.31, 5.24, 0.08, 0.70, 0.16, 0.18}};

// the choice of pipe_block and pipe_split
void pipe_choice(const GemmDesc &g, PipeBlock *block, PlaneSplit *split)
{
    int best = 0;
    double t = kCost[0].time(g);
    for (int i = 1; i < 4; ++i) {
        const double ti = kCost[i].time(g);
        if (ti < t) t = ti, best = i;
    }
    *block = (PipeBlock)best;
    *split = PlaneSplit::none;
    // in parts: the whole-line form and the fp32 outputs
    if (g.nb > 1 || !(g.out_f32 || (!g.a_kmajor && g.Kl % 64 == 0))) return;
    const double blocks = kCost[0].blocks(g), x = blocks / kCost[0].workgroups, full = std::floor(x);
    if (full < 1 || x == full || blocks < pipe::cu_count()) return;      // every workgroup begins with a whole block
    t *= 0.95;
    for (int i = 0; i < 2; ++i) {
        const double parts = (x - full) * kParts[i].blocks(g) / blocks, whole = std::floor(parts);
        const double ti = kCost[0].time(full, 0, g) + kParts[i].time(whole, parts - whole, g);
        if (ti < t) {
            t = ti;
            *block = PipeBlock::b256;
            *split = i ? PlaneSplit::b128 : PlaneSplit::b128x256;
        }
    }
}
}  // namespace

PipeBlock pipe_block(const GemmDesc &g)
{
    PipeBlock b;
    PlaneSplit s;
    pipe_choice(g, &b, &s);
    return b;
}

PlaneSplit pipe_split(const GemmDesc &g)
{
    PipeBlock b;
    PlaneSplit s;
    pipe_choice(g, &b, &s);
    return s;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int NS, bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL, pipe::Split SPLIT>
static hipError_t launch_pipe_cfg(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    auto kern = gemm_pipe_kernel<BM, BN, WAVES_M, WAVES_N, NS, A_T, B_T, TO, ACC, KTAIL, SPLIT>;
    typedef pipe::BlockRing<BM, BN, WAVES_M, WAVES_N, NS, A_T, B_T, TO, ACC, KTAIL> Ring;
    constexpr int smem = NS * Ring::STAGE_BYTES + Ring::NW * Ring::SLAB;
    static_assert(smem <= 160 * 1024, "LDS budget");
    constexpr int per_cu = 160 * 1024 / smem > 2 ? 2 : 160 * 1024 / smem;
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, smem, granted); e != hipSuccess) return e;
    const int tiles_m = (g.Mi + BM - 1) / BM, tiles_n = (g.Nj + BN - 1) / BN;
    const long total = (long)tiles_m * tiles_n * g.batch * g.nb;
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    const int wgs = pipe::cu_count() * per_cu;                   // they walk the block list
    const unsigned grid = pipe::list_grid(total, wgs);
    if (SPLIT != pipe::Split::none && total < (long)grid) return hipErrorInvalidValue;      // every workgroup begins with a whole block
    hipLaunchKernelGGL(kern, dim3(grid), dim3(Ring::NW * 64), smem, s, (const bf16_t *)A, (const bf16_t *)B, (TO *)Out, g.Mi, g.Nj,
                       g.Kl, tiles_m, tiles_n, (int)total, g.a_rows_per_group(), g.b_rows_per_group(), g.o_rows_per_group(), g.batch);
    return hipGetLastError();
}

template <bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL>
static hipError_t launch_pipe_block(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    using pipe::Split;
    switch (pipe_block(g)) {
        case PipeBlock::b256:
            if constexpr (sizeof(TO) == 4) {
                switch (pipe_split(g)) {
                    case Split::b128x256: return launch_pipe_cfg<256, 256, 2, 4, 4, A_T, B_T, TO, ACC, KTAIL, Split::b128x256>(g, A, B, Out, s);
                    case Split::b128: return launch_pipe_cfg<256, 256, 2, 4, 4, A_T, B_T, TO, ACC, KTAIL, Split::b128>(g, A, B, Out, s);
                    case Split::none: break;
                }
            }
            return launch_pipe_cfg<256, 256, 2, 4, 4, A_T, B_T, TO, ACC, KTAIL, Split::none>(g, A, B, Out, s);
        case PipeBlock::b128x256: return launch_pipe_cfg<128, 256, 2, 4, 5, A_T, B_T, TO, ACC, KTAIL, Split::none>(g, A, B, Out, s);
        case PipeBlock::b128: return launch_pipe_cfg<128, 128, 2, 2, 4, A_T, B_T, TO, ACC, KTAIL, Split::none>(g, A, B, Out, s);
        case PipeBlock::b64: return launch_pipe_cfg<64, 64, 2, 2, 8, A_T, B_T, TO, ACC, KTAIL, Split::none>(g, A, B, Out, s);
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
