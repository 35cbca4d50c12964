// Building blocks of the LDS-DMA pipelined plane products: LDS-DMA source pointers, fragment addressing, swizzles,
// instruction-order fences and counted waits.  Shared by the plane-product kernel and by the kernel that runs the
// tile maps between its blocks.
#pragma once
#include "stl_kernels.h"
#include "stl_device.h"

#include <type_traits>

namespace stl {

namespace pipe {

constexpr int BKS = 32;                 // contraction elements per stage

typedef short v4i16_t __attribute__((ext_vector_type(4)));
#define STL_LDS(p) ((__attribute__((address_space(3))) char *)(p))

typedef PlaneSplit Split;

typedef float acc4_t __attribute__((ext_vector_type(4)));

// Swizzles (16-byte chunk index XOR), chosen so that one access phase touches every bank once.  ds_read_b128 is served in
// four phases of 16 lanes, {0-3, 12-15, 20-23, 24-27}, {4-11, 16-19, 28-31} and the same +32 (measured with the
// SQ_LDS_BANK_CONFLICT counter).  A 16x16x32 fragment of a [row][l] operand reads 16 rows (lane % 16) by the four chunks of
// a 64-byte row (lane / 16): the row groups 0-3, 4-7, 8-11, 12-15 XOR with 0, 2, 3, 1 put a phase on 16 different chunks.
// An [l][row] fragment reads, per transposing instruction, the l-rows 8 (lane / 16) + 0..3 (or 4..7), 32 bytes each: a
// half wavefront touches rows {0-3, 8-11} or {16-19, 24-27}, which go to eight different 32-byte slots of the 256 bytes
// the banks span.
__device__ __forceinline__ int fswz(int row)                                     // [row][l] operand, 4 chunks per row
{
    const int g = (row >> 2) & 3;
    return ((g & 1) << 1) ^ ((g >> 1) * 3);
}
template <int ROWS>
__device__ __forceinline__ int gswz(int k)                                       // [l][row] operand, ROWS / 8 chunks per row
{
    if constexpr (ROWS == 64) return (((k >> 1) & 1) << 1) | (((k >> 3) & 1) << 2);
    return ((k & 3) << 2) | (((k >> 3) & 1) << 1);
}

// LDS-DMA load, 16 bytes per lane: lane L's bytes land at lds_wave_base + 16*L (M0 carries the wave-uniform LDS
// address).  Issued as inline assembly on purpose: the main loop orders these loads against the fragment reads
// itself (vmcnt + barrier below); letting the compiler track them makes it drain every outstanding load before
// each LDS read, which removes the prefetch distance this kernel exists for.
__device__ __forceinline__ void dma16(const bf16_t *g, uint32_t lds_wave_base)
{
    const uint32_t l = __builtin_amdgcn_readfirstlane(lds_wave_base);
    // a write of M0 by the scalar unit and the LDS-DMA load that reads it must be one wait state apart (the compiler, which
    // sees to that elsewhere, does not look into the statement)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(l) : "memory", "m0");
}

__device__ __forceinline__ const bf16_t *at_bytes(const bf16_t *base, uint32_t off)
{
    return reinterpret_cast<const bf16_t *>(reinterpret_cast<const char *>(base) + off);
}

__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Global sources of the DMA instructions a wavefront issues per operand and stage: a base that is the same for the whole
// workgroup and moves from stage to stage (scalar registers), plus a byte offset per lane and instruction that stays for the
// whole block (launchers check that it fits 32 bits: offsets_fit).
// One operand stage is ROWS x 32 contraction elements = ROWS/16 KB = ROWS/16 instructions, dealt to NW wavefronts.
// KTAIL: the contraction may end inside the last stage; pieces beyond its end are then fetched from inside the operand
// instead (the fragments are masked before they are multiplied, see mask_tail).
template <bool KMAJOR, int ROWS, int NW, bool KTAIL>
struct Src {
    static constexpr int NI = ROWS / 16 / NW;          // instructions per wavefront
    static constexpr int CPR = ROWS / 8;               // 16-byte chunks per LDS row of the [l][row] form
    const bf16_t *base;
    uint32_t off[NI];
    long step;   // elements to advance per stage
    long jump;   // [l][row] form: extra elements when the next stage starts a new group of stored rows
    int kpos, pg;
    int left, rem;   // KTAIL: stages before the last one, contraction elements of the last one
    // src: the whole batched operand; plane p of `batch`; stored rows come in groups of pg (see plane_row_base), and a
    // stage's 32 stored rows of the [l][row] form never straddle two groups (pg % 32 == 0, or one group only)
    // roff: first stored row of this problem inside the stacked operand (a multiple of 32 for the [l][row] form)
    __device__ __forceinline__ void init(const bf16_t *src, long ld, int row0, int rows_total, int wave, int lane, int plane,
                                         int batch, int pg_, int roff, int Kl)
    {
        pg = pg_;
        kpos = KMAJOR ? roff % pg_ : 0;
        const int first = KMAJOR ? roff : roff + row0;
        const size_t first_off = plane_row_base(first, pg, batch, (int)ld);
        base = src + first_off + (size_t)plane * pg * ld + (KMAJOR ? row0 : 0);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int q = NI * wave + j;
            if (!KMAJOR) {
                const int row = 16 * q + (lane >> 2), c = (lane & 3) ^ fswz(row);
                int gr = row0 + row;
                gr = gr < rows_total ? gr : rows_total - 1;   // rows past the edge feed only discarded outputs
                off[j] = (uint32_t)((plane_row_base(roff + gr, pg, batch, (int)ld) - first_off + 8 * c) * 2);
            } else {
                const int k = (64 / CPR) * q + lane / CPR, nc = (lane % CPR) ^ gswz<ROWS>(k);
                int gc = row0 + 8 * nc;
                gc = gc < rows_total ? gc : rows_total - 8;
                off[j] = (uint32_t)(((size_t)k * ld + (gc - row0)) * 2);
            }
        }
        step = KMAJOR ? (long)BKS * ld : BKS;
        jump = KMAJOR ? (long)(batch - 1) * pg * ld : 0;
        if constexpr (KTAIL) {
            left = (Kl - 1) / BKS;
            rem = Kl - left * BKS;
            if (left == 0) clamp_tail(ld, wave, lane);
        }
    }
    // last stage: move the pieces that begin beyond the contraction's end to its first chunk / its last row
    __device__ __forceinline__ void clamp_tail(long ld, int wave, int lane)
    {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int q = NI * wave + j;
            if (!KMAJOR) {
                const int row = 16 * q + (lane >> 2), c = (lane & 3) ^ fswz(row);
                if (8 * c >= rem) off[j] -= 16 * c;
            } else {
                const int k = (64 / CPR) * q + lane / CPR;
                if (k >= rem) off[j] -= (uint32_t)((k - (rem - 1)) * ld * 2);
            }
        }
    }
    // instruction j of this wavefront's share (the main loop spreads them between MFMAs)
    __device__ __forceinline__ void issue_one(uint32_t oper_stage, int wave, int j)
    {
        dma16(at_bytes(base, off[j]), oper_stage + (NI * wave + j) * 1024);
    }
    // after the last instruction of a stage: point at the next stage
    __device__ __forceinline__ void next_stage(int wave, int lane)
    {
        long adv = step;
        if (KMAJOR) {
            kpos += BKS;
            if (kpos == pg) {
                kpos = 0;
                adv += jump;
            }
        }
        base += adv;
        if constexpr (KTAIL)
            if (--left == 0) clamp_tail(KMAJOR ? step / BKS : 0, wave, lane);
    }
    __device__ __forceinline__ void issue(uint32_t oper_stage, int wave, int lane)   // LDS byte address of the operand stage
    {
#pragma unroll
        for (int j = 0; j < NI; ++j) issue_one(oper_stage, wave, j);
        next_stage(wave, lane);
    }
};


// ---- whole-line form of a [row][l] operand ------------------------------------------------------------------------------
// A [row][l] operand fetched 32 contraction elements at a time asks L2 for half a 128-byte line per row and stage, and
// for the other half one stage later: twice the requests for the same bytes (counted: TCC_REQ).  In the whole-line
// form an LDS slot holds 64 contraction elements of every row (128 bytes = one line per row, ROWS * 128 bytes per slot)
// and serves two stages; it is filled in two halves of ROWS / 2 rows, one half per stage, so that every stage still
// issues the same number of instructions.  Three slots: while pair j is multiplied, pair j+1 has landed and pair j+2
// is in flight.
// LDS: row stride 128 bytes; 16-byte chunk c of row `row` lies at chunk position c ^ ((row >> 1) & 7): the sixteen
// rows of one ds_read_b128 access phase ({0-3, 12-15, 20-23, 24-27} or {4-11, 16-19, 28-31}, see above) then fall
// on sixteen different (row parity, chunk position) pairs, i.e. on all 64 banks once.
__device__ __forceinline__ int wswz(int row) { return (row >> 1) & 7; }

template <int ROWS, int NW>
struct SrcWide {
    static constexpr int HALF = ROWS / 2;                   // rows per half slot
    static constexpr int NI = HALF / 8 / NW;                // instructions per wavefront and half (8 rows x 128 bytes each)
    static constexpr int SLOT_BYTES = ROWS * 128, HALF_BYTES = HALF * 128;
    const bf16_t *base[2];                                  // of the next piece of either half
    uint32_t off[2][NI];
    __device__ __forceinline__ void init(const bf16_t *src, long ld, int row0, int rows_total, int wave, int lane, int plane,
                                         int batch, int pg, int roff)
    {
        const size_t first_off = plane_row_base(roff + row0, pg, batch, (int)ld);
        base[0] = base[1] = src + first_off + (size_t)plane * pg * ld;
#pragma unroll
        for (int hp = 0; hp < 2; ++hp)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int q = NI * wave + j;
                const int row = HALF * hp + 8 * q + (lane >> 3), c = (lane & 7) ^ wswz(row);
                int gr = row0 + row;
                gr = gr < rows_total ? gr : rows_total - 1;   // rows past the edge feed only discarded outputs
                off[hp][j] = (uint32_t)((plane_row_base(roff + gr, pg, batch, (int)ld) - first_off + 8 * c) * 2);
            }
    }
    // instruction j of half HP into the slot at LDS byte address `slot`
    template <int HP>
    __device__ __forceinline__ void issue_one(uint32_t slot, int wave, int j)
    {
        dma16(at_bytes(base[HP], off[HP][j]), slot + HP * HALF_BYTES + (NI * wave + j) * 1024);
    }
    template <int HP>
    __device__ __forceinline__ void next_pair()               // after the last instruction of half HP: 64 elements on
    {
        base[HP] += 64;
    }
    template <int HP>
    __device__ __forceinline__ void issue_half(uint32_t slot, int wave)
    {
#pragma unroll
        for (int j = 0; j < NI; ++j) issue_one<HP>(slot, wave, j);
        next_pair<HP>();
    }
};

// Fragments of v_mfma_f32_16x16x32_bf16: lane (row or column = lane % 16, kq = lane / 16) holds the contraction elements
// 8 kq .. 8 kq + 7 of its row.  The 16x16x32 form takes the same operand bytes per product as 32x32x16 but moves half the
// accumulator bytes per flop, and the chip is power-limited under these products: a loop of nothing else on normally
// distributed operands runs at 2.0 PFLOP/s against 1.8 (2.35 both on zeros).
template <int ROWS>
struct FragWide {
    int off;        // first stage of a pair; the second stage's chunks are 4 further: off ^ 64
    __device__ __forceinline__ void init(int tile_row0, int lane)
    {
        const int row = tile_row0 + (lane & 15);
        off = row * 128 + (((lane >> 4) ^ wswz(row)) << 4);
    }
    // fragment f (16 rows further per f: the swizzle repeats after 16 rows) of stage parity sp, from the slot of its pair
    __device__ __forceinline__ bf16x8_t read(const char *slot, int f, int sp) const
    {
        return *reinterpret_cast<const bf16x8_t *>(slot + (off ^ (sp << 6)) + f * 16 * 128);
    }
};

// LDS address with some of its low bits flipped
__device__ __forceinline__ __attribute__((address_space(3))) v4i16_t *lds_xor(const char *p, uint32_t bits)
{
    const uint32_t a = (uint32_t)(uintptr_t)STL_LDS(p) ^ bits;
    return (__attribute__((address_space(3))) v4i16_t *)(uintptr_t)a;
}

// Fragment addressing: byte offset inside one operand stage for the 16 rows (columns) from frag_row0 on.
template <bool KMAJOR, int ROWS>
struct Frag {
    int off[2];      // [kk]; only the transposing form uses the second
    __device__ __forceinline__ void init(int tile_row0, int lane)
    {
        const int kq = lane >> 4;
        if (!KMAJOR) {
            const int row = tile_row0 + (lane & 15);
            off[0] = row * 64 + ((kq ^ fswz(row)) << 4);
            off[1] = 0;
        } else {
            const int i = lane & 15;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int k = 8 * kq + 4 * kk + (i >> 2);
                const int col = tile_row0 + 4 * (i & 3);
                off[kk] = k * (ROWS * 2) + (((col >> 3) ^ gswz<ROWS>(k)) << 4) + ((col & 7) << 1);
            }
        }
    }
    // fragment f (16 rows or columns further per f)
    __device__ __forceinline__ bf16x8_t read(const char *oper_stage, int f) const
    {
        if (!KMAJOR) {
            return *reinterpret_cast<const bf16x8_t *>(oper_stage + off[0] + f * 16 * 64);
        } else {
            // Fragment f starts 16 columns = 2 chunks further.  The wavefront's first column is a multiple of its number of
            // columns, so the chunk bits of f are free and "+2f" is "^ (f << 1)", which commutes with the swizzle XOR (and with
            // the stage's base, a multiple of 8 KB: applied last, the XOR of each f needs no register of its own across stages).
            const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_xor(oper_stage + off[0], f << 5));
            const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_xor(oper_stage + off[1], f << 5));
            struct { v4i16_t a, b; } both = {lo, hi};
            return __builtin_bit_cast(bf16x8_t, both);
        }
    }
};

// Fragment of the last stage of a contraction with `rem` elements in it: the elements beyond are zeroed (in both operands,
// so that whatever lies there -- infinities and NaN included -- takes no part).
__device__ __forceinline__ void mask_tail(bf16x8_t &v, int rem, int lane)
{
    u32x4_t w = __builtin_bit_cast(u32x4_t, v);
    const int k0 = 8 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] &= (k0 + 2 * i < rem ? 0xffffu : 0u) | (k0 + 2 * i + 1 < rem ? 0xffff0000u : 0u);
    v = __builtin_bit_cast(bf16x8_t, w);
}

// CUs of the device (of the first one a process uses: all are of one kind), the workgroups of a persistent launch
inline int cu_count()
{
    static const int n = []() {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
        return cus;
    }();
    return n;
}

// Block list of a persistent launch.  Hardware deals workgroup ids round-robin over the 8 XCDs; each XCD takes a contiguous
// eighth of the list (its workgroups side by side in it), so that the blocks an L2 serves at one time are neighbours of
// one or two planes.  The grid is a multiple of 8.
__device__ __forceinline__ int first_block(int total) { return (int)((long)(blockIdx.x & 7) * total / 8) + (int)(blockIdx.x >> 3); }
__device__ __forceinline__ int end_block(int total) { return (int)((long)((blockIdx.x & 7) + 1) * total / 8); }
__device__ __forceinline__ int block_step() { return (int)(gridDim.x >> 3); }
// the end of the whole rounds of this XCD's share
__device__ __forceinline__ int whole_end(int total)
{
    const int begin = (int)((long)(blockIdx.x & 7) * total / 8);
    return begin + (end_block(total) - begin) / block_step() * block_step();
}
inline unsigned list_grid(long total, int workgroups)
{
    const long wanted = total < workgroups ? (total + 7) / 8 * 8 : workgroups / 8 * 8;
    return (unsigned)(wanted < 8 ? 8 : wanted);
}

// The lane offsets of a block's DMA sources fit 32 bits: 32 rows of an [l][row] operand, 256 of a [row][l] one.  Those lie
// side by side in a plane-major operand; in a grouped one every group border among them adds the group's other planes.
inline bool offsets_fit(const GemmDesc &g)
{
    auto span = [&](bool kmajor, int pg, int ld) {
        const double rows = kmajor ? 32 : pg <= 0 ? 256 : 256 + (256.0 / pg + 1) * (g.batch - 1) * pg;
        return (rows + 1) * ld * 2;
    };
    return span(g.a_kmajor, g.a_pg, g.a_kmajor ? g.Mi : g.Kl) < 4294967296.0 &&
           span(g.b_kmajor, g.b_pg, g.b_kmajor ? g.Nj : g.Kl) < 4294967296.0;
}

// compile-time loop: the body sees its index as a constant, so register arrays are never indexed dynamically
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// wait until at most `stages` stages of D instructions each are outstanding, stages <= MAX
template <int D, int MAX>
__device__ __forceinline__ void wait_stages(int stages)
{
    if constexpr (MAX == 0) wait_vmcnt<0>();
    else if (stages >= MAX) wait_vmcnt<D * MAX>();
    else wait_stages<D, MAX - 1>(stages);
}

// fragment rows (16 output rows each) a wavefront stages per epilogue pass, in at most 4 KB of LDS
template <int FM, int FN, typename TO>
constexpr int slab_frags()
{
    constexpr int fit = 4096 / (16 * FN * 16 * (int)sizeof(TO));
    return fit < FM ? fit : FM;
}
template <int FM, int FN, typename TO>
constexpr int slab_bytes() { return slab_frags<FM, FN, TO>() * 16 * FN * 16 * (int)sizeof(TO); }

// Accumulators and operand fragments of a wavefront: FM x FN products of 16 x 16.  The first operand's fragments are kept
// once -- the next stage's replaces each as soon as its FN products are issued -- the second operand's twice.
template <int FM, int FN>
struct WaveTile {
    static_assert(FM >= FN, "one fragment of the second operand is fetched per fragment of the first");
    acc4_t acc[FM][FN];
    bf16x8_t va[FM], vb[2][FN];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) acc[a][b] = acc4_t{0.f, 0.f, 0.f, 0.f};
    }
    // One stage of 32 contraction elements, on the fragments fetched during the previous one (second operand: parity PAR).
    // read_a(f) / read_b(f) fetch the next stage's fragments, one or two LDS instructions after each of the first products so
    // that the wavefronts' reads do not arrive at the LDS in one burst; dma(j), j < FM, issues this wavefront's refill
    // loads, at most one per FN products; the fences pin the order.
    template <int PAR, class RA, class RB, class DMA>
    __device__ __forceinline__ void stage(RA &&read_a, RB &&read_b, DMA &&dma)
    {
        static_for<0, FM>([&](auto a_c) {
            constexpr int a = decltype(a_c)::value;
            static_for<0, FN>([&](auto b_c) {
                constexpr int b = decltype(b_c)::value;
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb[PAR][b], va[a], acc[a][b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (b == 0) {
                    if constexpr (a < FN) vb[PAR ^ 1][a] = read_b(a);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (b == FN / 2) {
                    dma(a_c);
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            va[a] = read_a(a);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    __device__ __forceinline__ void mask(int par, int rem, int lane)
    {
#pragma unroll
        for (int a = 0; a < FM; ++a) mask_tail(va[a], rem, lane);
        if (par) {
#pragma unroll
            for (int b = 0; b < FN; ++b) mask_tail(vb[1][b], rem, lane);
        } else {
#pragma unroll
            for (int b = 0; b < FN; ++b) mask_tail(vb[0][b], rem, lane);
        }
    }
    // Epilogue.  Operands are passed to the products as (second, first), which leaves a lane with the four consecutive output
    // columns 16 b + 4 (lane / 16) .. + 3 of output row 16 a + lane % 16: one 8- or 16-byte write into a 4 KB slab (at most)
    // that belongs to the wavefront alone, from which the rows leave in whole 16-byte pieces.  There is no workgroup barrier: a
    // wavefront's LDS operations execute in order, so the next pass's writes are issued right behind this pass's reads and
    // the read latency is spent on them.  (One pass after the other, with a padded slab of 16 rows and the group of each pass's
    // rows found by a division, took 11 of the 131 us of the forward products at 2048 x 1024 x 1024, r = 32, and 15 of 52 at
    // 3200 x 192 x 768.)
    // row0, col0: the wavefront's corner of the output; roff: stored rows before this problem; outp points at the plane; a pass's
    // rows in steps of 16 stay inside one group of the output layout.
    // PA: fragment rows per pass.
    template <typename TO, bool ACC, bool THROUGH, int PA = slab_frags<FM, FN, TO>()>
    __device__ __forceinline__ void store(char *slab, TO *outp, int row0, int col0, int Mi, int Nj, int roff, int o_pg, int batch,
                                          int lane) const
    {
        constexpr int ES = sizeof(TO), RB = FN * 16 * ES, CH = RB / 16;          // bytes and 16-byte chunks per row
        constexpr int LD = PA * 16 * CH / 64;                                    // pieces per lane and pass
        // chunk swizzle: the 16 rows one write touches, and the rows one read touches, spread over all banks
        auto swz = [](int row) { return CH == 16 ? row & 15 : CH == 8 ? (row >> 1) & 7 : (row >> 2) & 3; };
        const int wr = lane & 15, rr = lane / CH, rc = lane % CH;
        const bool col_ok = col0 + rc * (16 / ES) < Nj;
        // group and position of the pass's rows, stepped 16 rows at a time
        int gpos = (roff + row0) % o_pg;
        TO *orow = outp + plane_row_base(roff + row0, o_pg, batch, Nj) + (size_t)rr * Nj + col0 + rc * (16 / ES);
        const size_t step = (size_t)16 * Nj, jump = (size_t)(batch - 1) * o_pg * Nj;
        u32x4_t piece[LD];
        auto put = [&](auto a0_c) {
            constexpr int a0 = decltype(a0_c)::value;
            static_for<0, PA>([&](auto a_c) {
                constexpr int a = decltype(a_c)::value;
                char *rowp = slab + (16 * a + wr) * RB;
#pragma unroll
                for (int b = 0; b < FN; ++b) {
                    const acc4_t v = acc[a0 + a][b];
                    if constexpr (ES == 2)
                        *reinterpret_cast<u32x2_t *>(rowp + (((2 * b + (lane >> 5)) ^ swz(wr)) << 4) + ((lane >> 4) & 1) * 8) =
                            u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                    else
                        *reinterpret_cast<f32x4_t *>(rowp + (((4 * b + (lane >> 4)) ^ swz(wr)) << 4)) = v;
                }
            });
        };
        put(std::integral_constant<int, 0>{});
        static_for<0, FM / PA>([&](auto pass_c) {
            constexpr int a0 = decltype(pass_c)::value * PA;
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < LD; ++i) {
                const int row = i * (64 / CH) + rr;
                piece[i] = *reinterpret_cast<const u32x4_t *>(slab + row * RB + ((rc ^ swz(row)) << 4));
            }
            asm volatile("" ::: "memory");
            if constexpr (a0 + PA < FM) put(std::integral_constant<int, (a0 + PA < FM ? a0 + PA : 0)>{});
            asm volatile("" ::: "memory");
            static_for<0, PA>([&](auto a_c) {
                constexpr int a = decltype(a_c)::value;
                const int gi = row0 + (a0 + a) * 16 + rr;
#pragma unroll
                for (int i = 0; i < LD / PA; ++i) {
                    if (col_ok && gi + i * (64 / CH) < Mi) {
                        TO *o = orow + (size_t)(i * (64 / CH)) * Nj;
                        const u32x4_t w = piece[a * (LD / PA) + i];
                        if constexpr (ACC) {
                            const f32x4_t old = *reinterpret_cast<const f32x4_t *>(o);
                            f32x4_t nw = __builtin_bit_cast(f32x4_t, w);
                            nw += old;
                            *reinterpret_cast<f32x4_t *>(o) = nw;
                        } else {
                            store16<THROUGH>(o, w);
                        }
                    }
                }
                orow += step;
                gpos += 16;
                if (gpos == o_pg) {
                    gpos = 0;
                    orow += jump;
                }
            });
        });
    }
};

// Operands and output of a launch's plane products.
template <typename TO>
struct Products {
    const bf16_t *A, *B;
    TO *Out;
    int Mi, Nj, Kl, a_pg, b_pg, o_pg, batch;
};

// One block of one plane at a time on a ring of NS LDS stages of 32 contraction elements, issued NS - 1 stages ahead of their use.
// The ring's first LOW stages lie at the start of the workgroup's LDS, the others from byte HIGH on (LOW = NS: all of them side by side).
template <int BM, int BN, int WAVES_M, int WAVES_N, int NS, bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL, int LOW = NS, int HIGH = 0>
struct BlockRing {
    static constexpr int STAGES = NS;
    static constexpr int NW = WAVES_M * WAVES_N, WM = BM / WAVES_M, WN = BN / WAVES_N, FM = WM / 16, FN = WN / 16;
    static constexpr int OPER_BYTES = BM * BKS * 2, STAGE_BYTES = (BM + BN) * BKS * 2;
    static constexpr int D = (BM + BN) / 16 / NW;          // DMA instructions per wavefront and stage
    static constexpr int SLAB = slab_bytes<FM, FN, TO>();
    static_assert(NS >= 3, "ring depth");
    Frag<A_T, BM> fa;
    Frag<B_T, BN> fb;
    Src<A_T, BM, NW, KTAIL> sa;
    Src<B_T, BN, NW, KTAIL> sb;
    static __device__ __forceinline__ int at(int s)        // LDS offset of stage s
    {
        if constexpr (LOW == NS) return s % NS * STAGE_BYTES;
        const int i = s % NS;
        return i < LOW ? i * STAGE_BYTES : HIGH + (i - LOW) * STAGE_BYTES;
    }
    __device__ __forceinline__ void init(int wave, int lane)
    {
        fa.init(wave / WAVES_N * WM, lane);
        fb.init(wave % WAVES_N * WN, lane);
    }
    // point the DMA sources at block (i0, j0) of plane p of problem pb and put its first NS-1 stages in flight
    __device__ __forceinline__ void start(const Products<TO> &g, int nks, int pb, int p, int i0, int j0, uint32_t smem_lds, int wave, int lane)
    {
        // the lane id as an opaque value: what the sources derive from it is computed per block and occupies no registers while
        // the products run (spilled values would be reloaded between the loads issued here, and waited for with them)
        int sl = lane;
        asm volatile("" : "+v"(sl));
        sa.init(g.A, A_T ? g.Mi : g.Kl, i0, g.Mi, wave, sl, p, g.batch, g.a_pg, pb * (A_T ? g.Kl : g.Mi), g.Kl);
        sb.init(g.B, B_T ? g.Nj : g.Kl, j0, g.Nj, wave, sl, p, g.batch, g.b_pg, pb * (B_T ? g.Kl : g.Nj), g.Kl);
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) {
            if (s < nks) {
                sa.issue(smem_lds + at(s), wave, sl);
                sb.issue(smem_lds + at(s) + OPER_BYTES, wave, sl);
            }
        }
    }
    // Block (i0, j0) of plane p of problem pb, whose first loads are in flight: all its stages (as in gemm_pipe_kernel), next() (the loads of what
    // follows) and its stores.  One function with its accumulators: in two, the compiler moves them from register to register in every stage (64 x 64
    // blocks up to 10 % slower).
    template <class F>
    __device__ __forceinline__ void block(const Products<TO> &g, int nks, const char *smem, uint32_t smem_lds, char *slab, int pb, int p, int i0, int j0,
                                          int wave, int lane, F &&next)
    {
        const int Kl = g.Kl;
        WaveTile<FM, FN> w;
        w.clear();

        // Stage s+NS-1 is issued in iteration s; stage s+1 must have landed at the top of iteration s (its fragments are
        // fetched during stage s).  Stores of the previous epilogue may still be in flight: "at most N operations
        // outstanding" then over-waits but never under-waits.
        wait_stages<D, NS - 2>(nks - 1);
        block_barrier();
#pragma unroll
        for (int a = 0; a < FM; ++a) w.va[a] = fa.read(smem + at(0), a);
#pragma unroll
        for (int b = 0; b < FN; ++b) w.vb[0][b] = fb.read(smem + at(0) + OPER_BYTES, b);

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
            const uint32_t dst = smem_lds + at(s + NS - 1);
            const char *nxt = smem + at(s + 1);
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
        next();
        int el = lane;                                   // opaque, as above
        asm volatile("" : "+v"(el));
        w.template store<TO, ACC, false>(slab, g.Out + (size_t)p * g.o_pg * g.Nj, i0 + wave / WAVES_N * WM, j0 + wave % WAVES_N * WN, g.Mi, g.Nj,
                                         pb * g.Mi, g.o_pg, g.batch, el);
    }
};

// Parts of the blocks of a last round (Split in stl_kernels.h).
template <Split S>
struct Part {
    static constexpr int N = S == Split::b128 ? 128 : 256;       // 128 rows by so many columns of a 256 x 256 block
};

// The parts of the blocks from `first` on of an XCD's share of the list (up to end_block), numbered block by block without those beyond
// the output's edge, and dealt to its workgroups in turn.  A plane has PM x PN of them; two rows of parts lie in a row of blocks (one in the last
// row, if the other does not exist), SN columns in a column of blocks.
template <Split S>
struct PartList {
    static constexpr int N = Part<S>::N, SN = 256 / N;
    int u, end, step, PM, PN;
    __device__ __forceinline__ void init(int first, int total, int tiles_m, int tiles_n, int Mi, int Nj)
    {
        step = block_step();
        PM = (Mi + 127) / 128;
        PN = (Nj + N - 1) / N;
        auto before = [&](int v) {                       // parts of the blocks before block v
            const int q = v / (tiles_m * tiles_n), rem = v - q * (tiles_m * tiles_n), bi = rem / tiles_n, bj = rem - bi * tiles_n;
            return q * (PM * PN) + 2 * bi * PN + rows(bi) * SN * bj;
        };
        u = before(first) + (int)(blockIdx.x >> 3);
        end = before(end_block(total));
    }
    __device__ __forceinline__ int rows(int bi) const { return PM - 2 * bi < 2 ? PM - 2 * bi : 2; }
    // this workgroup's next part: false if there is none
    __device__ __forceinline__ bool next(int batch, int &pb, int &p, int &i0, int &j0)
    {
        if (u >= end) return false;
        const int q = u / (PM * PN);
        int w = u - q * (PM * PN);
        const int bi = w / (2 * PN);
        w -= bi * (2 * PN);
        const int bj = w / (rows(bi) * SN);
        w -= bj * (rows(bi) * SN);
        const int cols = PN - SN * bj < SN ? PN - SN * bj : SN, row = w / cols;
        pb = q / batch;
        p = q - pb * batch;
        i0 = (2 * bi + row) * 128;
        j0 = (SN * bj + w - row * cols) * N;
        u += step;
        return true;
    }
};

// Parts of the last blocks, one after the other, on a ring of their own: begin() puts the first one's loads in flight, run() does the rest.
template <Split S, int NS, bool A_T, bool B_T, typename TO, bool ACC, bool KTAIL, int LOW = NS, int HIGH = 0>
struct PartWalk {
    BlockRing<128, Part<S>::N, 2, 4, NS, A_T, B_T, TO, ACC, KTAIL, LOW, HIGH> ring;
    PartList<S> list;
    bool more;
    int pb, p, i0, j0;
    __device__ __forceinline__ void begin(const Products<TO> &g, int nks, int first, int total, int tiles_m, int tiles_n, uint32_t smem_lds, int wave, int lane)
    {
        list.init(first, total, tiles_m, tiles_n, g.Mi, g.Nj);
        more = list.next(g.batch, pb, p, i0, j0);
        if (more) ring.start(g, nks, pb, p, i0, j0, smem_lds, wave, lane);
    }
    __device__ __forceinline__ void run(const Products<TO> &g, int nks, const char *smem, uint32_t smem_lds, char *slab, int wave, int lane)
    {
        int fl = lane;                                   // opaque, as above
        asm volatile("" : "+v"(fl));
        ring.init(wave, fl);
        while (more) {
            const int cpb = pb, cp = p, ci0 = i0, cj0 = j0;
            ring.block(g, nks, smem, smem_lds, slab, cpb, cp, ci0, cj0, wave, lane, [&]() {
                more = list.next(g.batch, pb, p, i0, j0);
                if (more) ring.start(g, nks, pb, p, i0, j0, smem_lds, wave, lane);
            });
        }
    }
};

}  // namespace pipe

}  // namespace stl
