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
#include <algorithm>
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

// The same for 256 x 256 blocks, of which those of a last round that is not full are dealt to all workgroups in parts (see pipe_split).  A
// kernel of its own: with its blocks in BlockRing the one above has a few scalar instructions more per stage, 1 % of a small layer.  So the
// stages of a block, their waits and their order, are written down there, in BlockRing::block and (whole lines) in gemm_pipe_wide_kernel: what is
// changed in one belongs in all three.
template <bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL, pipe::Split SPLIT>
__global__ __launch_bounds__(512) void gemm_pipe_split_kernel(const pipe::Products<TO> g, int tiles_m, int tiles_n, int total)
{
    using namespace pipe;
    extern __shared__ __align__(16) char smem[];
    typedef BlockRing<256, 256, 2, 4, 4, A_T, B_T, TO, ACC, KTAIL> Ring;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: LDS-DMA destinations stay in SGPRs
    char *slab = smem + 4 * Ring::STAGE_BYTES + wave * Ring::SLAB;
    const int per_plane = tiles_m * tiles_n, nks = (g.Kl + BKS - 1) / BKS;
    const uint32_t smem_lds = (uint32_t)(uintptr_t)STL_LDS(smem);
    auto locate = [&](int v, int &p, int &i0, int &j0) {
        p = v / per_plane;
        const int rem = v - p * per_plane;
        i0 = (rem / tiles_n) * 256;
        j0 = (rem % tiles_n) * 256;
    };
    Ring ring;
    ring.init(wave, lane);
    auto start_block = [&](int v) {
        int p, i0, j0;
        locate(v, p, i0, j0);
        ring.start(g, nks, 0, p, i0, j0, smem_lds, wave, lane);
    };
    PartWalk<SPLIT, SPLIT == Split::b128 ? 8 : 5, A_T, B_T, TO, ACC, KTAIL> parts;
    const int step = block_step(), end = whole_end(total);
    int v = first_block(total);
    start_block(v);                                                  // every workgroup has a whole block: total >= the grid
    for (; v < end; v += step) {
        int p, i0, j0;
        locate(v, p, i0, j0);
        ring.block(g, nks, smem, smem_lds, slab, 0, p, i0, j0, wave, lane, [&]() {
            if (v + step < end) start_block(v + step);
            else parts.begin(g, nks, end, total, tiles_m, tiles_n, smem_lds, wave, lane);
        });
    }
    parts.run(g, nks, smem, smem_lds, slab, wave, lane);
}

// The weight gradient (A and B [l][.], fp32 output, ACC: added to what is there) and the input gradient (A [row][l], B [j][l]) of a small layer in one
// launch, which do not depend on each other: one block per workgroup, those of the first product and then those of the second.
struct PairGeometry {
    int tiles_n, per_plane, total;
};
template <int B1, int B2, bool ACC>
__global__ __launch_bounds__(256) void gemm_pipe_pair_kernel(const pipe::Products<float> x, const PairGeometry gx, const pipe::Products<bf16_t> y,
                                                             const PairGeometry gy)
{
    using namespace pipe;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: LDS-DMA destinations stay in SGPRs
    const uint32_t smem_lds = (uint32_t)(uintptr_t)STL_LDS(smem);
    const int grid1 = (gx.total + 7) / 8 * 8;
    auto run = [&](auto &&ring, const auto &g, const PairGeometry &geo, int b, auto edge_c) {
        typedef std::remove_reference_t<decltype(ring)> Ring;
        constexpr int EDGE = decltype(edge_c)::value;
        const int v = (int)((long)(b & 7) * geo.total / 8) + (b >> 3);     // each XCD takes a contiguous eighth of both lists
        if (v >= (int)((long)((b & 7) + 1) * geo.total / 8)) return;
        const int p = v / geo.per_plane, rem = v - p * geo.per_plane, i0 = rem / geo.tiles_n * EDGE, j0 = rem % geo.tiles_n * EDGE;
        const int nks = (g.Kl + BKS - 1) / BKS;
        ring.init(wave, lane);
        ring.start(g, nks, 0, p, i0, j0, smem_lds, wave, lane);
        ring.block(g, nks, smem, smem_lds, smem + Ring::STAGES * Ring::STAGE_BYTES + wave * Ring::SLAB, 0, p, i0, j0, wave, lane, [] {});
    };
    if ((int)blockIdx.x < grid1)
        run(BlockRing<B1, B1, 2, 2, B1 == 64 ? 8 : 4, true, true, float, ACC, true>(), x, gx, (int)blockIdx.x, std::integral_constant<int, B1>{});
    else
        run(BlockRing<B2, B2, 2, 2, B2 == 64 ? 8 : 4, false, false, bf16_t, false, true>(), y, gy, (int)blockIdx.x - grid1, std::integral_constant<int, B2>{});
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

// the choice of pipe_block and pipe_split, and its predicted time in us
struct PipeChoice {
    PipeBlock block;
    PlaneSplit split;
    double us;
};
PipeChoice pipe_choice(const GemmDesc &g)
{
    PipeChoice c{PipeBlock::b256, PlaneSplit::none, kCost[0].time(g)};
    for (int i = 1; i < 4; ++i) {
        const double ti = kCost[i].time(g);
        if (ti < c.us) c.us = ti, c.block = (PipeBlock)i;
    }
    // in parts: the whole-line form and the fp32 outputs
    if (g.nb > 1 || !(g.out_f32 || (!g.a_kmajor && g.Kl % 64 == 0))) return c;
    const double blocks = kCost[0].blocks(g), x = blocks / kCost[0].workgroups, full = std::floor(x);
    if (full < 1 || x == full || blocks < pipe::cu_count()) return c;      // every workgroup begins with a whole block
    double limit = 0.95 * c.us;
    for (int i = 0; i < 2; ++i) {
        const double parts = (x - full) * kParts[i].blocks(g) / blocks, whole = std::floor(parts);
        const double ti = kCost[0].time(full, 0, g) + kParts[i].time(whole, parts - whole, g);
        if (ti < limit) {
            limit = ti;
            c = {PipeBlock::b256, i ? PlaneSplit::b128 : PlaneSplit::b128x256, ti};
        }
    }
    return c;
}
}  // namespace

PipeBlock pipe_block(const GemmDesc &g) { return pipe_choice(g).block; }

PlaneSplit pipe_split(const GemmDesc &g) { return pipe_choice(g).split; }

template <int BM, int BN, int WAVES_M, int WAVES_N, int NS, bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL>
static hipError_t launch_pipe_cfg(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    constexpr int NW = WAVES_M * WAVES_N;
    auto kern = gemm_pipe_kernel<BM, BN, WAVES_M, WAVES_N, NS, A_T, B_T, TO, ACC, KTAIL>;
    constexpr int smem = NS * (BM + BN) * pipe::BKS * 2 + NW * pipe::slab_bytes<BM / WAVES_M / 16, BN / WAVES_N / 16, TO>();
    static_assert(smem <= 160 * 1024, "LDS budget");
    constexpr int per_cu = 160 * 1024 / smem > 2 ? 2 : 160 * 1024 / smem;
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, smem, granted); e != hipSuccess) return e;
    const int tiles_m = (g.Mi + BM - 1) / BM, tiles_n = (g.Nj + BN - 1) / BN;
    const long total = (long)tiles_m * tiles_n * g.batch * g.nb;
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    const int wgs = pipe::cu_count() * per_cu;                   // they walk the block list
    const unsigned grid = pipe::list_grid(total, wgs);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NW * 64), smem, s, (const bf16_t *)A, (const bf16_t *)B, (TO *)Out, g.Mi, g.Nj,
                       g.Kl, tiles_m, tiles_n, (int)total, g.a_rows_per_group(), g.b_rows_per_group(), g.o_rows_per_group(), g.batch);
    return hipGetLastError();
}

template <bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL, pipe::Split SPLIT>
static hipError_t launch_pipe_split(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    auto kern = gemm_pipe_split_kernel<A_T, B_T, TO, ACC, KTAIL, SPLIT>;
    typedef pipe::BlockRing<256, 256, 2, 4, 4, A_T, B_T, TO, ACC, KTAIL> Ring;
    constexpr int smem = 4 * Ring::STAGE_BYTES + Ring::NW * Ring::SLAB;
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, smem, granted); e != hipSuccess) return e;
    const int tiles_m = (g.Mi + 255) / 256, tiles_n = (g.Nj + 255) / 256;
    const long total = (long)tiles_m * tiles_n * g.batch;
    const unsigned grid = pipe::list_grid(total, pipe::cu_count());
    if (total > 0x7fffffffL || total < (long)grid || g.nb != 1) return hipErrorInvalidValue;      // every workgroup begins with a whole block
    const pipe::Products<TO> pr{(const bf16_t *)A, (const bf16_t *)B, (TO *)Out, g.Mi, g.Nj, g.Kl, g.a_rows_per_group(), g.b_rows_per_group(),
                                g.o_rows_per_group(), g.batch};
    hipLaunchKernelGGL(kern, dim3(grid), dim3(512), smem, s, pr, tiles_m, tiles_n, (int)total);
    return hipGetLastError();
}

template <bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL>
static hipError_t launch_pipe_block(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    using pipe::Split;
    if constexpr (sizeof(TO) == 4) {
        switch (pipe_split(g)) {
            case Split::b128x256: return launch_pipe_split<A_T, B_T, TO, ACC, KTAIL, Split::b128x256>(g, A, B, Out, s);
            case Split::b128: return launch_pipe_split<A_T, B_T, TO, ACC, KTAIL, Split::b128>(g, A, B, Out, s);
            case Split::none: break;
        }
    }
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

// Edges of the two products' blocks in one launch: 64 x 64 where that is a product's own choice, else 128 x 128.
static int pair_edge(const GemmDesc &g) { return pipe_block(g) == PipeBlock::b64 ? 64 : 128; }

// One launch where its predicted time is less than that of two.  The form of the prediction: a latency, the stages of the longer
// contraction, and per product its rounds of blocks, two to a CU, a time per stage and per byte stored each; least squares over 330 layers of
// 4 to 2500 x 32 to 1200 x 32 to 1200 tiles, 8 to 64 planes, 8.5 % off in the root mean square.  Of those layers it takes 321, which are 1.5 times as fast
// as in two launches in the mean, two of them slower by more than 2 % (7 %).  us, two launches / one: 45 x 64 x 112, r = 48 9.3 / 5.2; 256 x 256 x 256,
// r = 32 14.9 / 12.8; 1137 x 88 x 800, r = 32 41.6 / 23.6; 268 x 896 x 784, r = 49 112 / 101; and where two launches keep the large blocks, 3200 x 192 x 768,
// r = 32 103.6 / 109.5; 2048 x 1024 x 1024, r = 32 270 / 372.
bool pipe_pair_eligible(const GemmDesc &g1, const GemmDesc &g2)
{
    if (g1.nb != 1 || g2.nb != 1 || !g1.out_f32 || !(g1.a_kmajor && g1.b_kmajor) || g2.out_f32 || g2.accumulate || g2.a_kmajor || g2.b_kmajor) return false;
    if (!plane_gemm_pipe_eligible(g1) || !plane_gemm_pipe_eligible(g2)) return false;
    auto rounds = [](const GemmDesc &g, int e) { return (double)((g.Mi + e - 1) / e) * ((g.Nj + e - 1) / e) * g.batch / 512; };
    const int e1 = pair_edge(g1), e2 = pair_edge(g2);
    const double st1 = (g1.Kl + pipe::BKS - 1) / pipe::BKS, st2 = (g2.Kl + pipe::BKS - 1) / pipe::BKS, out1 = g1.accumulate ? 4 : 2;
    const double us = 4.10 + 0.117 * std::max(st1, st2) + rounds(g1, e1) * (e1 == 64 ? 0.44 + 0.179 * st1 + 0.58 * out1 : 1.52 + 0.538 * st1 + 1.26 * out1) +
                      rounds(g2, e2) * (e2 == 64 ? 1.26 + 0.221 * st2 : 2.37 + 0.664 * st2);
    return us < 0.97 * (pipe_choice(g1).us + pipe_choice(g2).us);
}

template <int B1, int B2, bool ACC>
static hipError_t launch_pipe_pair_cfg(const GemmDesc &g1, const void *A1, const void *W1, void *Out1, const GemmDesc &g2, const void *A2, const void *W2,
                                       void *Out2, hipStream_t s)
{
    auto kern = gemm_pipe_pair_kernel<B1, B2, ACC>;
    typedef pipe::BlockRing<B1, B1, 2, 2, B1 == 64 ? 8 : 4, true, true, float, ACC, true> R1;
    typedef pipe::BlockRing<B2, B2, 2, 2, B2 == 64 ? 8 : 4, false, false, bf16_t, false, true> R2;
    constexpr int lds1 = R1::STAGES * R1::STAGE_BYTES + R1::NW * R1::SLAB, lds2 = R2::STAGES * R2::STAGE_BYTES + R2::NW * R2::SLAB;
    constexpr int smem = lds1 > lds2 ? lds1 : lds2;
    static_assert(2 * smem <= 160 * 1024, "two workgroups per CU");
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, smem, granted); e != hipSuccess) return e;
    auto geometry = [](const GemmDesc &g, int edge) {
        const int tm = (g.Mi + edge - 1) / edge, tn = (g.Nj + edge - 1) / edge;
        return PairGeometry{tn, tm * tn, tm * tn * g.batch};
    };
    const PairGeometry gx = geometry(g1, B1), gy = geometry(g2, B2);
    const pipe::Products<float> x{(const bf16_t *)A1, (const bf16_t *)W1, (float *)Out1, g1.Mi, g1.Nj, g1.Kl, g1.a_rows_per_group(), g1.b_rows_per_group(),
                                  g1.o_rows_per_group(), g1.batch};
    const pipe::Products<bf16_t> y{(const bf16_t *)A2, (const bf16_t *)W2, (bf16_t *)Out2, g2.Mi, g2.Nj, g2.Kl, g2.a_rows_per_group(), g2.b_rows_per_group(),
                                   g2.o_rows_per_group(), g2.batch};
    hipLaunchKernelGGL(kern, dim3((unsigned)((gx.total + 7) / 8 * 8 + (gy.total + 7) / 8 * 8)), dim3(256), smem, s, x, gx, y, gy);
    return hipGetLastError();
}

hipError_t launch_pipe_pair(const GemmDesc &g1, const void *A1, const void *B1, void *Out1, const GemmDesc &g2, const void *A2, const void *B2, void *Out2,
                            hipStream_t s)
{
    if (!pipe_pair_eligible(g1, g2)) return hipErrorInvalidValue;
    const bool small1 = pair_edge(g1) == 64, small2 = pair_edge(g2) == 64;
    auto launch = [&](auto acc_c) -> hipError_t {
        constexpr bool ACC = decltype(acc_c)::value;
        if (small1)
            return small2 ? launch_pipe_pair_cfg<64, 64, ACC>(g1, A1, B1, Out1, g2, A2, B2, Out2, s)
                          : launch_pipe_pair_cfg<64, 128, ACC>(g1, A1, B1, Out1, g2, A2, B2, Out2, s);
        return small2 ? launch_pipe_pair_cfg<128, 64, ACC>(g1, A1, B1, Out1, g2, A2, B2, Out2, s)
                      : launch_pipe_pair_cfg<128, 128, ACC>(g1, A1, B1, Out1, g2, A2, B2, Out2, s);
    };
    return g1.accumulate ? launch(std::true_type{}) : launch(std::false_type{});
}

}  // namespace stl
