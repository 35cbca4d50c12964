// Pipelined plane products whose first operand is stored [row][l] (the forward products Yhat[p] = Xhat[p] What[p] and
// the input-gradient products dXhat[p] = dYhat[p] What[p]^T), with that operand fetched as whole 128-byte lines.
//
// Same kernel as gemm_pipe_kernel in every other respect (256 x 256 block, eight wavefronts of 128 x 64, 16x16x32
// MFMA, persistent block list, next block's first loads in flight during the epilogue, wavefront-private epilogue
// slab), and the same products in the same order: results are bit-identical.  What differs is the path of the first
// operand into LDS (SrcWide / FragWide in stl_gemm_pipe.h): slots of 64 contraction elements that serve two stages
// each, filled half a slot per stage, three slots deep; the second operand keeps its ring of four 32-element stages.
// LDS: 3 x 32 KB + 4 x 16 KB = the whole 160 KB; the epilogue slabs lie in the third slot of the first operand,
// which is idle from the last stage of a block until the first stage of the next one has passed its barrier.
#include "stl_gemm_pipe.h"

namespace stl {

// B_T: second operand stored [l][j]; otherwise [j][l] (32-element stages, half lines, as in gemm_pipe_kernel).
// Requires Kl % 64 == 0.  One problem per launch (no stacking).
// SPLIT: the blocks of a last round that is not full are dealt to all workgroups in parts (see pipe_split), whose rings lie
// on both sides of the epilogue slabs.
template <bool B_T, pipe::Split SPLIT>
__global__ __launch_bounds__(512) void gemm_pipe_wide_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B,
                                                             bf16_t *__restrict__ Out, int Mi, int Nj, int Kl, int tiles_m,
                                                             int tiles_n, int total, int a_pg, int b_pg, int o_pg, int batch)
{
    using namespace pipe;
    constexpr int BM = 256, BN = 256, NW = 8, WAVES_N = 4, WM = 128, WN = 64, FM = WM / 16, FN = WN / 16, NSB = 4;
    constexpr int A_SLOT = BM * 128, B_STAGE = BN * BKS * 2, B_BASE = 3 * A_SLOT;
    constexpr int SLAB = slab_bytes<FM, FN, bf16_t>();
    static_assert(B_BASE + NSB * B_STAGE == 160 * 1024 && NW * SLAB <= A_SLOT, "LDS map");
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: LDS-DMA destinations stay in SGPRs
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    char *slab = smem + 2 * A_SLOT + wave * SLAB;
    const int per_plane = tiles_m * tiles_n;
    const int nks = Kl / BKS;                          // even
    const uint32_t smem_lds = (uint32_t)(uintptr_t)STL_LDS(smem);

    FragWide<BM> fa;
    Frag<B_T, BN> fb;
    fa.init(wm * WM, lane);
    fb.init(wn * WN, lane);

    auto locate = [&](int v, int &p, int &i0, int &j0) {
        p = v / per_plane;
        const int rem = v - p * per_plane;
        i0 = (rem / tiles_n) * BM;
        j0 = (rem % tiles_n) * BN;
    };

    SrcWide<BM, NW> sa;
    Src<B_T, BN, NW, false> sb;
    // LDS addresses: first-operand slot of pair j, second-operand stage s
    auto a_slot = [&](int pair) { return (pair % 3) * A_SLOT; };
    auto b_slot = [&](int s) { return B_BASE + (s % NSB) * B_STAGE; };
    // Issue order of a block, per wavefront (H = half slot of the first operand, numbered 2 * pair + half; B = stage of
    // the second): H0 B0 H1 B1 H2 B2 H3 before the loop, then H(s+4) B(s+3) in iteration s -- four instructions per
    // iteration as long as both exist.
    auto start_block = [&](int v) {
        // the lane id as an opaque value: what the sources derive from it is computed per block and occupies no registers while
        // the products run (spilled values would be reloaded between the loads issued here, and waited for with them)
        int sl = lane;
        asm volatile("" : "+v"(sl));
        int p, i0, j0;
        locate(v, p, i0, j0);
        sa.init(A, Kl, i0, Mi, wave, sl, p, batch, a_pg, 0);
        sb.init(B, B_T ? Nj : Kl, j0, Nj, wave, sl, p, batch, b_pg, 0, Kl);
        sa.template issue_half<0>(smem_lds + a_slot(0), wave);
        sb.issue(smem_lds + b_slot(0), wave, sl);
        sa.template issue_half<1>(smem_lds + a_slot(0), wave);
        sb.issue(smem_lds + b_slot(1), wave, sl);
        if (nks > 2) {
            sa.template issue_half<0>(smem_lds + a_slot(1), wave);
            sb.issue(smem_lds + b_slot(2), wave, sl);
            sa.template issue_half<1>(smem_lds + a_slot(1), wave);
        }
    };

    // block v, whose first loads are in flight: its stages, next() (the loads of what follows) and its stores
    auto block = [&](int v, auto &&next) {
        int p, i0, j0;
        locate(v, p, i0, j0);
        WaveTile<FM, FN> w;
        w.clear();
        // Loads complete in the order they were issued.  Before the first fragments are read H0, B0, H1 must have
        // landed: everything but the last eight instructions (B1 H2 B2 H3) when the contraction has more than one
        // pair, everything but B1 otherwise.  (Stores of the previous epilogue may still be in flight: "at most N
        // outstanding" then over-waits, never under-waits.)
        if (nks > 2) wait_vmcnt<8>();
        else wait_vmcnt<2>();
        block_barrier();
#pragma unroll
        for (int a = 0; a < FM; ++a) w.va[a] = fa.read(smem + a_slot(0), a, 0);
#pragma unroll
        for (int b = 0; b < FN; ++b) w.vb[0][b] = fb.read(smem + b_slot(0), b);

        // One stage s = 2 * pair + SP.  RA: half slot s + 4 of the first operand is fetched; RB: stage s + 3 of the second.
        // At the top of iteration s everything issued up to iteration s - 2 must have landed (stage s + 1 of both
        // operands, whose fragments are fetched meanwhile; it lies in the same slot of the first operand when s is even); what
        // iteration s - 1 issued may still be in flight: WAIT instructions.
        auto stage = [&](int s, auto sp_c, auto ra_c, auto rb_c, auto wait_c) {
            constexpr int SP = decltype(sp_c)::value, WAIT = decltype(wait_c)::value;
            constexpr bool RA = decltype(ra_c)::value, RB = decltype(rb_c)::value;
            if constexpr (WAIT >= 0) wait_vmcnt<WAIT>();
            block_barrier();   // stage s+1 visible to all; nobody reads stage s-1 any more
            const int pair = s >> 1;
            const uint32_t dst_a = smem_lds + a_slot(pair + 2), dst_b = smem_lds + b_slot(s + NSB - 1);
            const char *nxt_a = smem + a_slot(pair + SP), *nxt_b = smem + b_slot(s + 1);
            w.template stage<SP>([&](int f) { return fa.read(nxt_a, f, SP ^ 1); }, [&](int f) { return fb.read(nxt_b, f); },
                                 [&](auto a_c) {
                                     constexpr int a = decltype(a_c)::value, NA = decltype(sa)::NI, NB = decltype(sb)::NI;
                                     static_for<0, NA + NB>([&](auto j_c) {
                                         constexpr int j = decltype(j_c)::value;
                                         if constexpr (j * FM / (NA + NB) == a) {
                                             if constexpr (RA && j < NA) sa.template issue_one<SP>(dst_a, wave, j);
                                             if constexpr (RB && j >= NA) sb.issue_one(dst_b, wave, j - NA);
                                         }
                                     });
                                 });
            if constexpr (RA) sa.template next_pair<SP>();
            if constexpr (RB) sb.next_stage(wave, lane);
        };
        using T_ = std::true_type;
        using F_ = std::false_type;
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using W4 = std::integral_constant<int, 4>;
        using W2 = std::integral_constant<int, 2>;
        using W0 = std::integral_constant<int, 0>;
        using WN_ = std::integral_constant<int, -1>;
        // stages s <= nks - 5 fetch both operands; s = nks - 4 (even) only the second; the last three nothing
        int s = 0;
        for (; s + 5 < nks; s += 2) {            // both stages of the pair at most nks - 5
            stage(s, I0{}, T_{}, T_{}, W4{});
            stage(s + 1, I1{}, T_{}, T_{}, W4{});
        }
        if (nks >= 4) {                          // s = nks - 4, nks - 3
            stage(s, I0{}, F_{}, T_{}, W4{});
            stage(s + 1, I1{}, F_{}, F_{}, W2{});
            s += 2;
        }
        stage(s, I0{}, F_{}, F_{}, W0{});        // s = nks - 2, nks - 1
        stage(s + 1, I1{}, F_{}, F_{}, WN_{});

        // every wavefront is done with the ring: refill it for the next block before storing this one
        block_barrier();
        next();
        int el = lane;                                   // opaque, as above
        asm volatile("" : "+v"(el));
        w.template store<bf16_t, false, false>(slab, Out + (size_t)p * o_pg * Nj, i0 + wm * WM, j0 + wn * WN, Mi, Nj, 0, o_pg, batch, el);
    };

    const int step = block_step(), end = SPLIT == Split::none ? end_block(total) : whole_end(total);
    int v = first_block(total);
    if constexpr (SPLIT == Split::none) {
        if (v < end) start_block(v);
        for (; v < end; v += step)
            block(v, [&]() {
                if (v + step < end) start_block(v + step);
            });
    } else {
        const Products<bf16_t> g{A, B, Out, Mi, Nj, Kl, a_pg, b_pg, o_pg, batch};
        constexpr int STAGE = (128 + Part<SPLIT>::N) * BKS * 2, LOW = 2 * A_SLOT / STAGE, HIGH = 3 * A_SLOT, N_UP = (160 * 1024 - HIGH) / STAGE;
        PartWalk<SPLIT, LOW + N_UP, false, B_T, bf16_t, false, false, LOW, HIGH> parts;
        start_block(v);                                          // every workgroup has a whole block: total >= the grid
        for (; v < end; v += step)
            block(v, [&]() {
                if (v + step < end) start_block(v + step);
                else parts.begin(g, nks, end, total, tiles_m, tiles_n, smem_lds, wave, lane);
            });
        parts.run(g, nks, smem, smem_lds, slab, wave, lane);
    }
}

bool plane_gemm_wide_eligible(const GemmDesc &g)
{
    return plane_gemm_pipe_eligible(g) && !g.a_kmajor && !g.out_f32 && !g.accumulate && g.nb == 1 && g.Kl % 64 == 0 && pipe_block(g) == PipeBlock::b256;
}

template <bool B_T, pipe::Split SPLIT>
static hipError_t launch_wide_cfg(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    auto kern = gemm_pipe_wide_kernel<B_T, SPLIT>;
    constexpr int smem = 160 * 1024;
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, smem, granted); e != hipSuccess) return e;
    const int tiles_m = (g.Mi + 255) / 256, tiles_n = (g.Nj + 255) / 256;
    const long total = (long)tiles_m * tiles_n * g.batch;
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    const unsigned grid = pipe::list_grid(total, pipe::cu_count());
    if (SPLIT != pipe::Split::none && total < (long)grid) return hipErrorInvalidValue;      // every workgroup begins with a whole block
    hipLaunchKernelGGL(kern, dim3(grid), dim3(512), smem, s, (const bf16_t *)A, (const bf16_t *)B, (bf16_t *)Out, g.Mi, g.Nj, g.Kl,
                       tiles_m, tiles_n, (int)total, g.a_rows_per_group(), g.b_rows_per_group(), g.o_rows_per_group(), g.batch);
    return hipGetLastError();
}

template <bool B_T>
static hipError_t launch_wide(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    using pipe::Split;
    switch (pipe_split(g)) {
        case Split::b128x256: return launch_wide_cfg<B_T, Split::b128x256>(g, A, B, Out, s);
        case Split::b128: return launch_wide_cfg<B_T, Split::b128>(g, A, B, Out, s);
        case Split::none: return launch_wide_cfg<B_T, Split::none>(g, A, B, Out, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_plane_gemm_wide(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    if (!plane_gemm_wide_eligible(g)) return hipErrorInvalidValue;
    return g.b_kmajor ? launch_wide<true>(g, A, B, Out, s) : launch_wide<false>(g, A, B, Out, s);
}

}  // namespace stl
