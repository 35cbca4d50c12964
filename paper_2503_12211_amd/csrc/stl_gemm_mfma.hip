// Batched plane products on the CDNA4 matrix cores (step (ii) of Algorithm 1, Claim 3.4):
//     Out[p][i][j] (+)= sum_l A[p](i,l) * B[p](l,j)       bf16 x bf16 -> fp32, p < r planes,
// for what the LDS-DMA kernels do not take: contiguous dimensions that are no multiple of 8 (250 tile columns of a 1000-class head,
// 50 tile rows of 200 tokens), whose rows begin at any even address, and stacked problems with more than one stage.
//
// One workgroup owns a BM x BN block of one plane, 16x16x32 MFMA.  Operands go from HBM to LDS through registers, 16 bytes at a time
// from any even address, into the LDS layouts of the LDS-DMA kernels (fragment addressing and swizzles of stl_gemm_pipe.h): an
// operand whose contiguous dimension is not the contraction keeps its orientation and is read by the transposing
// ds_read_b64_tr_b16.  A stage is 64 contraction elements, two pieces of 32; LDS is double buffered and the next PF stages are in
// registers.
// What bounds it: the latency of a chain of short stages, and before that the instructions around each load, since the products
// themselves are a few MFMAs.  Hence row addresses are computed once per workgroup (or by two multiply-adds per load where the rows
// are the contraction; groups of rows by a shift, not a division), the incomplete last chunk of a row costs nothing where a
// block has none, and accumulators leave as 8-byte pieces through a slab of the wavefront's own.
// Measured, us, with the operands transposed in registers, addresses and chunk ends computed at every load and one stage in flight ->
// now: 512 x 192 x 250 tiles, r = 32 (Yhat / dXhat / dWhat) 14.4 / 13.3 / 28 -> 8.6 / 8.9 / 11; 512 x 1023 x 1024, r = 32 (Yhat) 52 -> 40;
// 96 x (50 x 16 x 50), r = 32 (the three products) 19 / 17.5 / 16 -> 8.5 / 8.4 / 8.3 for 15 MB of output or input planes each.
#include "stl_gemm_pipe.h"
#include <cmath>

namespace stl {
namespace staged {

constexpr int BK = 64;      // contraction elements per LDS stage, in two pieces of pipe::BKS

// eight elements moved h places towards the first, zeros behind them, any h >= 0
__device__ __forceinline__ u32x4_t settle(u32x4_t v, int h) { return h <= 0 ? v : h >= 8 ? u32x4_t{0u, 0u, 0u, 0u} : shift_down(v, h); }

// One operand's share of a thread: NC 16-byte chunks per piece of 32 contraction elements.
//   [row][l]: chunk id = tid + j NT is (row id / 4, elements 8 (id % 4) ..);   [l][row]: (l = id / (ROWS / 8), rows 8 (id % (ROWS / 8)) ..)
// The swizzles repeat over the rows that j steps by, so that a thread's chunks are a fixed distance apart in LDS.  A chunk that
// reaches beyond its row is read as the eight elements that end with the row and moved into place on its way to LDS, so
// that no load waits for another; elements beyond the contraction become zeros there.
template <bool KMAJOR, int ROWS, int NT>
struct Piece {
    static constexpr int NC = ROWS * 4 / NT, CPR = ROWS / 8;
    static constexpr int BYTES = ROWS * 64;                    // of a piece in LDS
    static constexpr int STEP = KMAJOR ? NT / CPR : NT / 4;    // rows that j steps by
    static_assert(NC >= 1 && STEP % 16 == 0, "every thread takes chunks whose swizzle does not depend on j");
    const bf16_t *src[KMAJOR ? 1 : NC];     // [row][l]: the rows; [l][row]: this thread's column of row 0
    int lds, k, over;                       // LDS offset of chunk 0; contraction offset in a piece; elements beyond the row's end ([l][row])
    bool edge;                              // the block has rows beyond the operand's ([l][row])
    __device__ __forceinline__ void init(const bf16_t *base, const Lay &lay, int row0, int total, int roff, int tid)
    {
        if constexpr (!KMAJOR) {
            const int row = tid >> 2, c = tid & 3;
            lds = row * 64 + ((c ^ pipe::fswz(row)) << 4);
            k = 8 * c;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                int g = row0 + row + j * STEP;
                g = g < total ? g : total - 1;                 // rows past the edge feed only discarded outputs
                src[j] = base + lay.row(roff + g);
            }
        } else {
            const int c = tid % CPR, col = row0 + 8 * c;
            k = tid / CPR;
            lds = k * (ROWS * 2) + ((c ^ pipe::gswz<ROWS>(k)) << 4);
            edge = row0 + ROWS > total;
            over = col - (total - 8);
            src[0] = base + (over > 0 ? total - 8 : col);
        }
    }
    // the piece of the contraction elements l0 .. l0 + 31, as it lies in memory
    __device__ __forceinline__ void load(u32x4_t (&v)[NC], const Lay &lay, int roff, int l0, int Kl) const
    {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            if constexpr (!KMAJOR) {
                const int l = l0 + k;
                v[j] = *reinterpret_cast<const u32x4_any_t *>(src[j] + (l < Kl - 8 ? l : Kl - 8));
            } else {
                const int l = l0 + k + j * STEP;
                v[j] = *reinterpret_cast<const u32x4_any_t *>(src[0] + lay.row(roff + (l < Kl ? l : Kl - 1)));
            }
        }
    }
    __device__ __forceinline__ void put(char *piece, u32x4_t (&v)[NC], int l0, int Kl) const
    {
        const bool tail = l0 + pipe::BKS > Kl;
        if (tail || (KMAJOR && edge)) {
#pragma unroll
            for (int j = 0; j < NC; ++j) v[j] = settle(v[j], KMAJOR ? (l0 + k + j * STEP < Kl ? over : 8) : l0 + k - (Kl - 8));
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) *reinterpret_cast<u32x4_t *>(piece + lds + j * STEP * (KMAJOR ? ROWS * 2 : 64)) = v[j];
    }
};

// A_T: A stored [l][i];  B_T: B stored [l][j].  (false: stored [i][l] resp. [j][l].)
// PF: stages on their way in registers (1 or 2); 0: the contraction is a single stage.  KS: groups of WAVES_M x WAVES_N wavefronts
// that take every KS-th stage each, their sums added up in LDS at the end.
// The block `bid` of the list of (stacked problem, plane, block row, block column).
template <int BM, int BN, int WAVES_M, int WAVES_N, int PF, int KS, bool A_T, bool B_T, typename TO, bool ACC>
__device__ __forceinline__ void staged_product(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B, TO *__restrict__ Out, int Mi, int Nj, int Kl,
                                               int tiles_m, int tiles_n, int bid, int batch, Div by_plane, Div by_row, Div by_batch, const Lay &la,
                                               const Lay &lb, const Lay &lo, char *smem)
{
    using pipe::static_for;
    constexpr int NT = WAVES_M * WAVES_N * 64, WM = BM / WAVES_M, WN = BN / WAVES_N, FM = WM / 16, FN = WN / 16;
    typedef Piece<A_T, BM, NT> PA;
    typedef Piece<B_T, BN, NT> PB;
    constexpr int STAGE = 2 * (PA::BYTES + PB::BYTES);
    // blocks of narrow outputs: fragments that lie beyond the output take no part
    constexpr bool NARROW = BM == 64;
    const int q = by_plane.of(bid), rem = bid - q * (tiles_m * tiles_n);   // (stacked problem, plane)
    const int bi = by_row.of(rem), i0 = bi * BM, j0 = (rem - bi * tiles_n) * BN;
    const int pb = by_batch.of(q), p = q - pb * batch;

    const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    const int tid = KS == 1 ? threadIdx.x : threadIdx.x % NT, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    char *own = smem + group * (2 * STAGE);                     // this group's two buffers
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int a_roff = pb * (A_T ? Kl : Mi), b_roff = pb * (B_T ? Kl : Nj);
    PA pa;
    PB pbt;
    pa.init(A + (size_t)p * la.plane, la, i0, Mi, a_roff, tid);
    pbt.init(B + (size_t)p * lb.plane, lb, j0, Nj, b_roff, tid);
    pipe::Frag<A_T, BM> fa;
    pipe::Frag<B_T, BN> fb;
    fa.init(wm * WM, lane);
    fb.init(wn * WN, lane);

    constexpr int SETS = PF ? PF : 1;
    u32x4_t ra[SETS][2][PA::NC], rb[SETS][2][PB::NC];
    auto fetch = [&](auto set_c, int st) {
        constexpr int S = decltype(set_c)::value;
        static_for<0, 2>([&](auto h_c) {
            constexpr int h = decltype(h_c)::value;
            const int l0 = st * BK + h * pipe::BKS;
            if (h == 0 || l0 < Kl) {
                pa.load(ra[S][h], la, a_roff, l0, Kl);
                pbt.load(rb[S][h], lb, b_roff, l0, Kl);
            }
        });
    };
    auto put = [&](auto set_c, int st, int buf) {
        constexpr int S = decltype(set_c)::value;
        char *stage = own + buf * STAGE;
        static_for<0, 2>([&](auto h_c) {
            constexpr int h = decltype(h_c)::value;
            if (h == 0 || st * BK + h * pipe::BKS < Kl) {
                pa.put(stage + h * PA::BYTES, ra[S][h], st * BK + h * pipe::BKS, Kl);
                pbt.put(stage + 2 * PA::BYTES + h * PB::BYTES, rb[S][h], st * BK + h * pipe::BKS, Kl);
            }
        });
    };

    pipe::acc4_t acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = pipe::acc4_t{0.f, 0.f, 0.f, 0.f};
    const int row0 = i0 + wm * WM, col0 = j0 + wn * WN;         // the wavefront's corner of the output
    const bool idle = NARROW && row0 >= Mi;
    auto multiply = [&](int st, int buf) {
        const char *stage = own + buf * STAGE;
        static_for<0, 2>([&](auto h_c) {
            constexpr int h = decltype(h_c)::value;
            if (idle || (h && st * BK + h * pipe::BKS >= Kl)) return;
            const char *sa = stage + h * PA::BYTES, *sb = stage + 2 * PA::BYTES + h * PB::BYTES;
            bf16x8_t va[FM];
#pragma unroll
            for (int a = 0; a < FM; ++a) va[a] = fa.read(sa, a);
            static_for<0, FN>([&](auto b_c) {
                constexpr int b = decltype(b_c)::value;
                if (NARROW && b && col0 + 16 * b >= Nj) return;
                const bf16x8_t vb = fb.read(sb, b);
                // operands as (second, first): a lane ends with four consecutive output columns
#pragma unroll
                for (int a = 0; a < FM; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb, va[a], acc[a][b], 0, 0, 0);
            });
        });
    };

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, SETS - 1>;
    const int nst = (Kl + BK - 1) / BK;
    if constexpr (PF == 0) {
        fetch(I0{}, 0);
        put(I0{}, 0, 0);
        __syncthreads();
        multiply(0, 0);
        __syncthreads();
    } else {
        // round u: the group's stage st = KS u + group is multiplied, its next one goes from registers to the other buffer (whose
        // readers passed the barrier one round ago), the one PF rounds on is asked for; cur: register set of stage st
        const int rounds = (nst + KS - 1) / KS;
        if (group < nst) fetch(I0{}, group);
        if (PF == 2 && group + KS < nst) fetch(I1{}, group + KS);
        if (group < nst) put(I0{}, group, 0);
        __syncthreads();
        auto round = [&](int u, auto cur, auto nxt) {
            const int st = KS * u + group;
            if (st + PF * KS < nst) fetch(cur, st + PF * KS);
            if (st < nst) multiply(st, u & 1);
            if (st + KS < nst) put(nxt, st + KS, (u & 1) ^ 1);
            __syncthreads();
        };
        for (int u = 0; u < rounds; u += 2) {
            round(u, I0{}, I1{});
            if (u + 1 < rounds) round(u + 1, I1{}, I0{});
        }
    }
    if constexpr (KS > 1) {
        constexpr int PER = FM * FN * 16;                       // bytes of a thread's sums
        static_assert(PER * NT <= 2 * STAGE, "a group's sums fit its buffers");
        auto at = [&](int g, int i) { return reinterpret_cast<pipe::acc4_t *>(smem + g * (2 * STAGE) + (i * NT + tid) * 16); };
        if (group > 0)
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b) *at(group, a * FN + b) = acc[a][b];
        __syncthreads();
        if (group > 0) return;
#pragma unroll
        for (int g = 1; g < KS; ++g)
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b) acc[a][b] += *at(g, a * FN + b);
    }

    // Epilogue: 16 rows at a time through a slab that belongs to the wavefront alone (its LDS operations execute in order: no
    // barrier), leaving as row-contiguous 16-byte pieces; rows begin at any element.
    if (idle) return;
    constexpr int ES = sizeof(TO), RB = WN * ES, CH = RB / 16, LD = 16 * CH / 64;
    static_assert(16 * RB * WAVES_M * WAVES_N <= STAGE, "epilogue slabs lie in the first stage");
    auto swz = [](int row) { return CH == 16 ? row & 15 : (row >> 1) & 7; };
    char *slab = smem + wave * (16 * RB);
    const int wr = lane & 15, rr = lane / CH, rc = lane % CH, gj = col0 + rc * (16 / ES);
    TO *outp = Out + (size_t)p * lo.plane + gj;
    static_for<0, FM>([&](auto a_c) {
        constexpr int a = decltype(a_c)::value;
        char *rowp = slab + wr * RB;
        asm volatile("" ::: "memory");
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            const pipe::acc4_t v = acc[a][b];
            if constexpr (ES == 2)
                *reinterpret_cast<u32x2_t *>(rowp + (((2 * b + (lane >> 5)) ^ swz(wr)) << 4) + ((lane >> 4) & 1) * 8) =
                    u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            else
                *reinterpret_cast<f32x4_t *>(rowp + (((4 * b + (lane >> 4)) ^ swz(wr)) << 4)) = v;
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int row = i * (64 / CH) + rr, gi = row0 + 16 * a + row;
            const u32x4_t w = *reinterpret_cast<const u32x4_t *>(slab + row * RB + ((rc ^ swz(row)) << 4));
            if (gi >= Mi || gj >= Nj) continue;
            TO *o = outp + lo.row(pb * Mi + gi);
            if constexpr (ES == 2) {
                store8<true>(reinterpret_cast<bf16_t *>(o), Nj - gj, w);
            } else {
                f32x4_t nw = __builtin_bit_cast(f32x4_t, w);
                if (gj + 4 <= Nj) {
                    if constexpr (ACC) nw += *reinterpret_cast<const f32x4_any_t *>(o);
                    *reinterpret_cast<f32x4_any_t *>(o) = nw;
                } else {
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (gj + e < Nj) o[e] = ACC ? o[e] + nw[e] : nw[e];
                }
            }
        }
    });
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int PF, int KS, bool A_T, bool B_T, typename TO, bool ACC>
__global__ __launch_bounds__(WAVES_M *WAVES_N *KS * 64, BM == 64 ? (PF == 0 ? 8 : KS == 1 ? 5 : 4) : 2) void gemm_mfma_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B,
                                                                          TO *__restrict__ Out, int Mi, int Nj, int Kl, int tiles_m, int tiles_n,
                                                                          int base, int total, int batch, Div by_plane, Div by_row, Div by_batch, Lay la,
                                                                          Lay lb, Lay lo)
{
    extern __shared__ __align__(16) char smem[];
    const int bid = pipe::first_block(total);                   // one block per workgroup; each XCD takes a contiguous eighth
    if (bid >= pipe::end_block(total)) return;
    staged_product<BM, BN, WAVES_M, WAVES_N, PF, KS, A_T, B_T, TO, ACC>(A, B, Out, Mi, Nj, Kl, tiles_m, tiles_n, base + bid, batch, by_plane, by_row, by_batch,
                                                                        la, lb, lo, smem);
}

// Two products of 64 x 64 blocks in one launch: the blocks of the first, then those of the second.
struct Product {
    const bf16_t *A, *B;
    void *Out;
    int Mi, Nj, Kl, tiles_m, tiles_n, total, batch;
    Div by_plane, by_row, by_batch;
    Lay la, lb, lo;
};
template <int PF, bool A1, bool B1, typename T1, bool ACC1, bool A2, bool B2, typename T2>
__global__ __launch_bounds__(256, PF == 0 ? 8 : 5) void gemm_pair_kernel(const Product x, const Product y)
{
    extern __shared__ __align__(16) char smem[];
    const int grid1 = (x.total + 7) / 8 * 8, bx = (int)blockIdx.x;
    // each XCD takes a contiguous eighth of both lists
    auto place = [](int b, int total) { return (b >> 3) < (int)((long)((b & 7) + 1) * total / 8 - (long)(b & 7) * total / 8) ? (int)((long)(b & 7) * total / 8) + (b >> 3) : -1; };
    if (bx < grid1) {
        const int bid = place(bx, x.total);
        if (bid >= 0)
            staged_product<64, 64, 4, 1, PF, 1, A1, B1, T1, ACC1>(x.A, x.B, (T1 *)x.Out, x.Mi, x.Nj, x.Kl, x.tiles_m, x.tiles_n, bid, x.batch, x.by_plane,
                                                                  x.by_row, x.by_batch, x.la, x.lb, x.lo, smem);
    } else {
        const int bid = place(bx - grid1, y.total);
        if (bid >= 0)
            staged_product<64, 64, 4, 1, PF, 1, A2, B2, T2, false>(y.A, y.B, (T2 *)y.Out, y.Mi, y.Nj, y.Kl, y.tiles_m, y.tiles_n, bid, y.batch, y.by_plane,
                                                                   y.by_row, y.by_batch, y.la, y.lb, y.lo, smem);
    }
}

}  // namespace staged

// ---- host side ---------------------------------------------------------------------------
bool plane_gemm_mfma_eligible(const GemmDesc &g)
{
    if (g.Mi < 1 || g.Nj < 1 || g.Kl < 1 || g.batch < 1) return false;
    if (g.accumulate && !g.out_f32) return false;
    // instantiated operand forms: forward [i][l]x[l][j], input gradient [i][l]x[j][l] (storage out),
    // weight gradient [l][i]x[l][j] (fp32 out, or storage out for a run-time encoded second operand)
    if (g.a_kmajor ? !g.b_kmajor : g.out_f32) return false;
    // 16-byte global loads along each operand's contiguous dimension, at any even address
    return g.Mi >= 8 && g.Nj >= 8 && g.Kl >= 8;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int PF, int KS, bool A_T, bool B_T, typename TO, bool ACC>
static hipError_t launch_cfg(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    auto kern = staged::gemm_mfma_kernel<BM, BN, WAVES_M, WAVES_N, PF, KS, A_T, B_T, TO, ACC>;
    constexpr int stage = (BM + BN) * staged::BK * 2, most = 2 * stage * KS;
    // a contraction of one stage needs one: more workgroups per CU to hide its loads
    const int smem = g.Kl > staged::BK ? most : stage;
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, most, granted); e != hipSuccess) return e;
    GemmLays l;
    if (!l.set(g)) return hipErrorInvalidValue;
    const int tiles_m = (g.Mi + BM - 1) / BM, tiles_n = (g.Nj + BN - 1) / BN;
    const long total = (long)tiles_m * tiles_n * g.batch * g.nb;
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    constexpr long kMost = 1 << 22;                        // blocks of a launch: its threads have to fit 32 bits
    for (long base = 0; base < total; base += kMost) {
        const long n = total - base < kMost ? total - base : kMost;
        hipLaunchKernelGGL(kern, dim3((unsigned)((n + 7) / 8 * 8)), dim3(WAVES_M * WAVES_N * KS * 64), smem, s, (const bf16_t *)A,
                           (const bf16_t *)B, (TO *)Out, g.Mi, g.Nj, g.Kl, tiles_m, tiles_n, (int)base, (int)n, g.batch,
                           Div::by(tiles_m * tiles_n), Div::by(tiles_n), Div::by(g.batch), l.a, l.b, l.o);
    }
    return hipGetLastError();
}

static bool any_width(const GemmDesc &g) { return g.Mi % 8 || g.Nj % 8 || g.Kl % 8; }

// Edge of the (square) block.  A product with a single stage, or an output that a 64 x 64 block covers in one dimension, takes 64 x 64
// blocks however many there are (us at 64 / 128 / 256: Yhat 2048 x 50 x 513, r = 32 20 / 23 / 22; forward and backward of 96 x (64 x 64 x 20),
// r = 32 96 / 136 / 242, of 96 x (128 x 16 x 128) 212 / 235 / 370).
int staged_block(const GemmDesc &g)
{
    if (g.Mi <= 64 || g.Nj <= 64 || g.Kl <= staged::BK) return 64;
    // multiples of 8, stacked problems: 256 x 256 blocks, 8 wavefronts of 128 x 64, for large planes, 128 x 128, 4 of 64 x 64, for others
    if (!any_width(g)) return g.Mi > 128 && g.Nj > 128 ? 256 : 128;
    auto blocks = [&](int b) { return (double)((g.Mi + b - 1) / b) * ((g.Nj + b - 1) / b) * g.batch * g.nb; };
    // A bigger block moves fewer bytes per product, idle CUs and the latency of its longer stages cost more; sparse second rounds
    // of the big ones most of all.  us at 256 / 128 / 64:
    //   Yhat  512 x 1023 x 1024, 32: 41 / 51 / 79 (256 blocks of 256)    256 x 1023 x 1024, 32: 38 / 28 / 44    128 x 1023 x 1024, 32: 37 / 22 / 27
    //         2048 x 513 x 513, 32: 74 / 87 / 108                        1000 x 513 x 513, 8: 26 / 21 / 20 (320 blocks of 128)
    //         1024 x 192 x 250, 32: 14 / 11 / 13                         512 x 192 x 250, 32: 12.1 / 8.5 / 8.3 (256 of 128)
    //   dWhat and the encode before it: 2048 x 513 x 513, 32: 189 / 136 / 141 (288 of 256)    1023 x 257 x 513, 16: 59 / 42 / 32
    const double b256 = blocks(256);
    if (g.Mi > 128 && g.Nj > 128 && b256 >= 192 * std::ceil(b256 / 256)) return 256;
    return g.Mi > 64 && g.Nj > 64 && blocks(128) >= (g.Kl > 640 ? 256 : 384) ? 128 : 64;
}

// Groups of wavefronts that share the contraction of a 64 x 64 block: where the blocks leave CUs idle and the chain of stages is
// long, each group has loads of its own in flight.  us with 1 / 2 / 4 groups: Yhat 64 x 500 x 500, 32 (256 blocks, 8 stages) 10.0 / 7.5 / 8.0,
// 512 x 192 x 250, 32 (1024 blocks, 3 stages) 8.5 / 10.4 / 14.8; dWhat and the encode before it 512 x 192 x 250, 32 (384, 8) 18.5 / 16.8 / 20.2,
// 3000 x 100 x 100, 8 (32, 47) 56 / 35 / 27, 1023 x 257 x 513, 16 (720, 16) 32 / 32 / 38.  0: one stage, one group.
int staged_groups(const GemmDesc &g)
{
    if (g.Kl <= staged::BK) return 0;
    const double blocks = (double)((g.Mi + 63) / 64) * ((g.Nj + 63) / 64) * g.batch * g.nb;
    const int stages = (g.Kl + staged::BK - 1) / staged::BK;
    return blocks <= 256 && stages >= 12 ? 4 : blocks <= 512 && stages >= 4 ? 2 : 1;
}

template <bool A_T, bool B_T, typename TO, bool ACC>
static hipError_t launch_block(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    switch (staged_block(g)) {
        case 256: return launch_cfg<256, 256, 2, 4, 1, 1, A_T, B_T, TO, ACC>(g, A, B, Out, s);
        case 128: return launch_cfg<128, 128, 2, 2, 2, 1, A_T, B_T, TO, ACC>(g, A, B, Out, s);
    }
    switch (staged_groups(g)) {
        case 0: return launch_cfg<64, 64, 4, 1, 0, 1, A_T, B_T, TO, ACC>(g, A, B, Out, s);
        case 4: return launch_cfg<64, 64, 4, 1, 2, 4, A_T, B_T, TO, ACC>(g, A, B, Out, s);
        case 2: return launch_cfg<64, 64, 4, 1, 2, 2, A_T, B_T, TO, ACC>(g, A, B, Out, s);
    }
    return launch_cfg<64, 64, 4, 1, 2, 1, A_T, B_T, TO, ACC>(g, A, B, Out, s);
}

hipError_t launch_plane_gemm_mfma(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s)
{
    if (!plane_gemm_mfma_eligible(g)) return hipErrorInvalidValue;
    if (g.out_f32)                                       // only the weight-gradient product stores fp32
        return g.accumulate ? launch_block<true, true, float, true>(g, A, B, Out, s)
                            : launch_block<true, true, float, false>(g, A, B, Out, s);
    if (g.a_kmajor) return launch_block<true, true, bf16_t, false>(g, A, B, Out, s);
    return g.b_kmajor ? launch_block<false, true, bf16_t, false>(g, A, B, Out, s) : launch_block<false, false, bf16_t, false>(g, A, B, Out, s);
}

// Pairs: a gradient of few blocks is the latency of its chain of stages, and two that read the same planes and write different ones
// need not wait for each other.  us, two launches / one, r = 32: dWhat and dXhat of 512 x 192 x 250 18.0 / 14.0, of 64 x 128 x 96 8.6 / 5.7, dAhat
// and dBhat of 96 x (50 x 16 x 50) 14.1 / 11.5; whole backward passes over 228 layers of odd widths 1.16 times as fast in the mean, over
// 259 pairs of activations 1.15.  A block has one group of wavefronts.  Where two groups would share a contraction that is
// little lost (of up to 7 stages 0.99 to 1.33, of 8 to 11 0.93 to 1.30, 1.07 in the mean of 174); one that four would share is a chain longer than all the rest: whole
// backward passes of 5886 x 15 x 82, r = 3 59.7 / 104, 7037 x 9 x 69, r = 32 85 / 121, 750 x 12 x 159, r = 3 19.9 / 21.6, 837 x 52 x 126, r = 64
// 34.8 / 36.6, in the mean of 45 1.2 times as long (at best 1.06 times as fast): such products stay apart.  Where the contraction of
// one product alone is a single stage, a block has the registers and LDS of two: many blocks of that kind stay apart too (96 x (256 x 256 x 8), 61440
// blocks, 206 / 244; 48 x (145 x 145 x 32), 9216, 23.9 / 26.1; 2640 blocks 20.2 / 17.4, 3500 19.5 / 18.5).
bool staged_pair_eligible(const GemmDesc &g1, const GemmDesc &g2)
{
    if (plane_gemm_path(1, g1) != GemmPath::staged || plane_gemm_path(1, g2) != GemmPath::staged) return false;
    if (staged_block(g1) != 64 || staged_block(g2) != 64 || staged_groups(g1) == 4 || staged_groups(g2) == 4) return false;
    auto blocks = [](const GemmDesc &g) { return (double)((g.Mi + 63) / 64) * ((g.Nj + 63) / 64) * g.batch * g.nb; };
    return blocks(g1) + blocks(g2) <= ((g1.Kl <= staged::BK) == (g2.Kl <= staged::BK) ? (1 << 22) - 1 : 3072);
}

template <int PF, bool A1, bool B1, typename T1, bool ACC1, bool A2, bool B2, typename T2>
static hipError_t launch_pair_cfg(const staged::Product &x, const staged::Product &y, int smem, hipStream_t s)
{
    const unsigned grid = (unsigned)((x.total + 7) / 8 * 8 + (y.total + 7) / 8 * 8);
    hipLaunchKernelGGL((staged::gemm_pair_kernel<PF, A1, B1, T1, ACC1, A2, B2, T2>), dim3(grid), dim3(256), smem, s, x, y);
    return hipGetLastError();
}

hipError_t launch_staged_pair(const GemmDesc &g1, const void *A1, const void *B1, void *Out1, const GemmDesc &g2, const void *A2, const void *B2, void *Out2,
                              hipStream_t s)
{
    if (!staged_pair_eligible(g1, g2)) return hipErrorInvalidValue;
    staged::Product x[2];
    const GemmDesc *g[2] = {&g1, &g2};
    const void *ops[2][3] = {{A1, B1, Out1}, {A2, B2, Out2}};
    for (int i = 0; i < 2; ++i) {
        GemmLays l;
        if (!l.set(*g[i])) return hipErrorInvalidValue;
        const int tm = (g[i]->Mi + 63) / 64, tn = (g[i]->Nj + 63) / 64;
        x[i] = {(const bf16_t *)ops[i][0], (const bf16_t *)ops[i][1], const_cast<void *>(ops[i][2]), g[i]->Mi, g[i]->Nj, g[i]->Kl, tm, tn,
                tm * tn * g[i]->batch * g[i]->nb, g[i]->batch, Div::by(tm * tn), Div::by(tn), Div::by(g[i]->batch), l.a, l.b, l.o};
    }
    const bool one = g1.Kl <= staged::BK && g2.Kl <= staged::BK;
    const int stage = 128 * staged::BK * 2, smem = one ? stage : 2 * stage;
    auto launch = [&](auto pf_c) -> hipError_t {
        constexpr int PF = decltype(pf_c)::value;
        // the products of a layer: the weight gradient first, then the input gradient; of a pair of activations: the first operand's, which
        // reads the second's planes as they were encoded ([l][j] if that was stored transposed), then the second's
        if (g1.out_f32) {
            if (!(g1.a_kmajor && g1.b_kmajor) || g2.a_kmajor || g2.b_kmajor || g2.out_f32) return hipErrorInvalidValue;
            return g1.accumulate ? launch_pair_cfg<PF, true, true, float, true, false, false, bf16_t>(x[0], x[1], smem, s)
                                 : launch_pair_cfg<PF, true, true, float, false, false, false, bf16_t>(x[0], x[1], smem, s);
        }
        if (g1.a_kmajor || !(g2.a_kmajor && g2.b_kmajor) || g2.out_f32 || g1.accumulate || g2.accumulate) return hipErrorInvalidValue;
        return g1.b_kmajor ? launch_pair_cfg<PF, false, true, bf16_t, false, true, true, bf16_t>(x[0], x[1], smem, s)
                           : launch_pair_cfg<PF, false, false, bf16_t, false, true, true, bf16_t>(x[0], x[1], smem, s);
    };
    return one ? launch(std::integral_constant<int, 0>{}) : launch(std::integral_constant<int, 2>{});
}

}  // namespace stl
