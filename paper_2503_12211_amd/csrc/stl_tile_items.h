// Per-wavefront item loops of the bf16 tile maps on the matrix cores (encode: step (i) of Algorithm 1, decode: step (iii),
// each optionally with the basis-gradient sum of the backward pass).  Shared by the stand-alone kernels and by the
// kernel that runs them between plane-product blocks.
#pragma once
#include "stl_kernels.h"
#include "stl_device.h"

namespace stl {

typedef short v4i16_t __attribute__((ext_vector_type(4)));

// Items of 64 tiles that follow each other in a group of 64 tile rows (FLAT below): tile t of an item, for Cc >= 32 ...
struct FlatTile {
    int I, J;
    template <class P>
    __device__ __forceinline__ P as() const { return P{I, J}; }
};
__device__ __forceinline__ FlatTile flat_tile(long item, int t, int Cc)
{
    const int g = (int)(item / Cc), o = (int)(item - (long)g * Cc) * 64, row = o / Cc, x = o - row * Cc + t;     // x < Cc + 63
    const int more = (x >= Cc ? 1 : 0) + (x >= 2 * Cc ? 1 : 0);
    return {g * 64 + row + more, x - more * Cc};
}
// ... and where its tiles from t on lie in plane 0, and how many of the group's follow there
struct FlatRun {
    size_t off;
    int left;
};
__device__ __forceinline__ FlatRun flat_run(long item, int t, int R, int Cc, int r)
{
    const int g = (int)(item / Cc), o = (int)(item - (long)g * Cc) * 64 + t, rows = R - g * 64;
    // the last group's place is as long as the others'
    return {(size_t)g * r * 64 * Cc + o, (rows < 64 ? rows : 64) * Cc - o};
}

// The item loop of one wavefront: items `first`, `first + stride`, ... below `end`, an item being (tile row index of the
// launch, 64-tile chunk) = item / chunks, item % chunks.  sT and slab are LDS areas private to the wavefront
// (sT: 64 x 32 bytes, used with OUTER only; slab: KC * 32 * 128 bytes); dacc accumulates the basis gradient (OUTER).
// `lane` is the caller's lane id (threadIdx.x % 64).  No workgroup barrier inside: wavefronts of a workgroup may run
// different numbers of items.
// THROUGH: the plane stores are written through to memory (see store16).  DEPTH: items whose operands are in flight
// at once (in registers) -- 1 where dozens of wavefronts per CU hide the latency, more where only eight run.
// ANY: any column count of at least 8 (see load8); otherwise a multiple of 8.  Bound by HBM and, for small matrices, by the
// launch; one pass over a row's planes whatever the width: with one thread per tile and a separate scalar sum, dYhat + dD of
// 512 x 250 tiles, r = 32, took 10 + 285 us, now 8; dYhat + dD of 4800 x 50 tiles 13 + 577 us, now 14.
// SHIFT (with ANY, without OUTER): an item's 64 tile columns begin where the plane rows' cache lines do, up to 63 columns to the
// left of its multiple of 64; `chunks` then counts (Cc + 126) / 64 items per row (see line_starts).
// turned: the basis is meant for the transposes of the tiles (entry 4a + b is applied to entry 4b + a); the basis gradient is that
// of the tiles as they lie.
// NARROW (no row map): an item is 64 >> lw tile rows of 1 << lw columns each, lw >= 3, and lay the planes' layout; `chunks` items to a row
// group.  Items of a single row left a matrix of 16 tile columns with a quarter of each lane's work: two
// encodes of 4800 x 16 tiles, r = 32, 12.3 -> 6.9 us, their two decodes with a basis gradient each 12.7 -> 7.6.
// FLAT (with NARROW; more than 32 columns, groups of 64 tile rows): an item is 64 tiles that follow each other in the planes' groups, whatever the
// rows; a group of Cc items.  No item but the last is incomplete, and every plane access is a whole line: dYhat + dD of 4800 x 50 tiles, r = 32,
// with their final sum 17.7 -> 13.7 us, of 8192 x 100 45.6 -> 28.7, of 2048 x 1000 84 -> 71, of 512 x 250 11.6 -> 10.7.
template <int KC, bool OUTER, bool THROUGH = false, int DEPTH = 1, bool ANY = false, bool SHIFT = false, bool NARROW = false, bool FLAT = false>
__device__ __forceinline__ void encode_items(const bf16_t *__restrict__ A, const bf16_t *__restrict__ E, bf16_t *__restrict__ P,
                                             const bf16_t *__restrict__ Qp, int R, int Cc, int r, int chunks, int pg, const RowMap &rm,
                                             long first, long stride, long end, char *sT, char *slab, f32x4_t (&dacc)[4], int lane,
                                             bool turned = false, int lw = 6, Lay lay = Lay{})
{
    constexpr int ROWB = 128;                               // bytes per plane row of the slab (64 tiles)
    // 16-byte chunk swizzle of a plane row: a fragment read takes chunk 4sx + kq of 16 rows; odd/even rows already
    // alternate the bank half, bit 1 of the row moves the chunk to the other four positions
    auto swz = [](int row) { return ((row >> 1) & 1) << 2; };
    const int pr = lane >> 3, ch = lane & 7;                // loader role: plane within a group of 8, 8-tile chunk
    const int j = lane & 15, kq = lane >> 4;
    const int ng = (r + 15) >> 4;
    const size_t ld = (size_t)Cc * 4, plane = (size_t)pg * Cc;

    // encoder fragments: lane (plane 16g + j, kq) holds E[plane][4kq + e] in K slots 8kq + e, e < 4; zeros above
    bf16x8_t eb[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int pl = 16 * g + j;
        u32x2_t ev = {0u, 0u};
        if (pl < r) {
            const bf16_t *e = E + pl * 16;
            if (turned)
                ev = u32x2_t{e[kq] | ((uint32_t)e[4 + kq] << 16), e[8 + kq] | ((uint32_t)e[12 + kq] << 16)};
            else
                ev = *reinterpret_cast<const u32x2_t *>(e + 4 * kq);
        }
        eb[g] = __builtin_bit_cast(bf16x8_t, u32x4_t{ev[0], ev[1], 0u, 0u});
    }
    // tile (relative to J0) of this lane in product u, and its row in the LDS slab: rows t and t^4 are swapped where
    // bit 3 of t is set, so that the four 4-tile groups of one write (and the four 8-tile groups of one transposing
    // read) fall into both halves of the banks
    int trel[4], srow[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        trel[u] = 8 * (j >> 2) + 4 * (u & 1) + 32 * (u >> 1) + (j & 3);
        srow[u] = trel[u] ^ (((trel[u] >> 3) & 1) << 2);
    }

    // Row I of a plane begins (I % pg) Cc elements behind the group's beginning, and the planes of a group lie pg Cc apart: a
    // multiple of a line in the grouped layout, so that one shift serves all planes.
    auto shift = [&](int I) { return SHIFT ? (int)(((size_t)(I % pg) * Cc) & 63) : 0; };

    u32x2_t xa[DEPTH][4];                   // this lane's tile rows, one per product
    u32x4_t qa[DEPTH][OUTER ? KC * 4 : 1];  // plane segments, loader role: plane 8*g8 + pr, tiles 8ch .. 8ch+7
    // NARROW: tile row and column of tile t of an item, offset of the plane row that holds chunk ch (8 tiles) of it, elements left there
    struct Pos { int I, J; };
    auto locate = [&](long item, int t) {
        if constexpr (FLAT) return flat_tile(item, t, Cc).template as<Pos>();
        const int rb = (int)(item / chunks), ck = (int)(item - (long)rb * chunks);
        return Pos{(rb << (6 - lw)) + (t >> lw), (ck << lw) + (t & ((1 << lw) - 1))};
    };
    // where chunk ch (8 tiles) of an item lies in plane 0, and how many elements from there on are the item's or follow it
    struct Run { size_t off; int left; };
    auto run = [&](long item) {
        if constexpr (FLAT) {
            const FlatRun f = flat_run(item, 8 * ch, R, Cc, r);
            return Run{f.off, f.left};
        }
        const Pos at = locate(item, 8 * ch);
        return Run{(size_t)lay.row(at.I) + at.J, at.I < R ? Cc - at.J : 0};
    };
    auto fetch_narrow = [&](int d, long item) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const Pos at = locate(item, trel[u]);
            u32x2_t v = {0u, 0u};
            if (at.I < R && at.J < Cc) v = *reinterpret_cast<const u32x2_t *>(A + ((size_t)at.I * 4 + kq) * ld + (size_t)at.J * 4);
            xa[d][u] = v;
        }
        if (OUTER) {
            const Run at = run(item);
#pragma unroll
            for (int g8 = 0; g8 < KC * 4; ++g8) {
                const int pl = 8 * g8 + pr;
                qa[d][g8] = load8<ANY>(Qp + at.off + (size_t)pl * plane, pl < r ? at.left : 0);
            }
        }
    };
    auto fetch = [&](int d, long item) {
        if constexpr (NARROW) return fetch_narrow(d, item);
        const int Ii = (int)(item / chunks), cki = (int)(item - (long)Ii * chunks);
        const int Ia = Ii < R ? rm.tile_row(Ii) : 0;        // Ii counts the tile rows of this launch, Ia is the tile row itself
        const int J0 = cki * 64 - shift(Ia);
        const size_t rowb = plane_row_base(Ia, pg, r, Cc);
        const bool row_ok = Ii < R && kq < rm.valid(Ia);    // a null row reads as zero
        const size_t r0 = rm.row0(Ia);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            u32x2_t v = {0u, 0u};
            if (row_ok && J0 + trel[u] < Cc && (!SHIFT || J0 + trel[u] >= 0)) v = *reinterpret_cast<const u32x2_t *>(A + (r0 + kq) * ld + (size_t)(J0 + trel[u]) * 4);
            xa[d][u] = v;
        }
        if (OUTER) {
#pragma unroll
            for (int g8 = 0; g8 < KC * 4; ++g8) {
                const int pl = 8 * g8 + pr, tk = J0 + 8 * ch;
                qa[d][g8] = load8<ANY>(Qp + rowb + (size_t)pl * plane + tk, Ii < R && pl < r ? Cc - tk : 0);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (first + d * stride < end) fetch(d, first + d * stride);

    for (long base = first; base < end; base += DEPTH * stride)
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        const long item0 = base + d * stride;
        if (item0 >= end) break;
        const int Iidx = (int)(item0 / chunks), cki = (int)(item0 - (long)Iidx * chunks);
        u32x2_t x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = xa[d][u];
        // plane segments -> slab (private to the wavefront, whose LDS operations execute in order: no barrier)
        if (OUTER) {
#pragma unroll
            for (int g8 = 0; g8 < KC * 4; ++g8) {
                const int pl = 8 * g8 + pr;
                *reinterpret_cast<u32x4_t *>(slab + pl * ROWB + ((ch ^ swz(pl)) << 4)) = qa[d][g8];
            }
        }
        if (item0 + DEPTH * stride < end) fetch(d, item0 + DEPTH * stride);
        if (!NARROW && Iidx >= R) continue;
        const int I = NARROW ? 0 : rm.tile_row(Iidx), J0 = NARROW ? 0 : cki * 64 - shift(I);

        // tile rows -> second slab
        if (OUTER) {
#pragma unroll
            for (int u = 0; u < 4; ++u) *reinterpret_cast<u32x2_t *>(sT + srow[u] * 32 + 8 * kq) = x[u];
        }

        // basis gradient: K = 32 tiles per product; B fragment of lane (entry j, kq) = tiles 32sx + 8kq .. +7 of entry j
#pragma unroll
        for (int sx = 0; sx < (OUTER ? 2 : 0); ++sx) {
            v4i16_t t[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // source address of this lane inside its 16-lane group: tile row (32sx + 8kq + 4h) + j/4, entries 4*(j%4)..
                const int t0 = 32 * sx + 8 * kq + 4 * h;
                const int row = (t0 ^ (((t0 >> 3) & 1) << 2)) + (j >> 2);
                t[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16_t *)(
                    (__attribute__((address_space(3))) char *)(sT + row * 32 + 8 * (j & 3))));
            }
            struct { v4i16_t a, b; } both = {t[0], t[1]};
            const bf16x8_t fb = __builtin_bit_cast(bf16x8_t, both);
#pragma unroll
            for (int g = 0; g < 2 * KC; ++g)
                if (g < ng) {
                    const int pl = 16 * g + j;
                    const bf16x8_t fp = *reinterpret_cast<const bf16x8_t *>(slab + pl * ROWB + (((4 * sx + kq) ^ swz(pl)) << 4));
                    dacc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fp, fb, dacc[g], 0, 0, 0);
                }
        }

        // encode: rows = tiles, columns = planes.  The results go through the plane slab (its fragments have been read
        // above; LDS operations of a wavefront execute in order) so that they leave as whole 128-byte lines, 8 planes
        // per store instruction, like the loads.
#pragma unroll
        for (int g = 0; g < 2 * KC; ++g) {
            if (g < ng) {
                f32x4_t o[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
                    const bf16x8_t hf = __builtin_bit_cast(bf16x8_t, u32x4_t{x[u][0], x[u][1], 0u, 0u});
                    o[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hf, eb[g], zero, 0, 0, 0);
                }
                const int pl = 16 * g + j;                  // products 2h, 2h+1: tiles 32h + 8kq .. +7 = chunk 4h + kq
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const f32x4_t a = o[2 * half], b = o[2 * half + 1];
                    const u32x4_t w = {pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]),
                                       pack_bf16x2(b[2], b[3])};
                    *reinterpret_cast<u32x4_t *>(slab + pl * ROWB + (((4 * half + kq) ^ swz(pl)) << 4)) = w;
                }
            }
        }
        if constexpr (NARROW) {
            const Run at = run(item0);
            bf16_t *o = P + at.off;
#pragma unroll
            for (int g8 = 0; g8 < KC * 4; ++g8) {
                const int pl = 8 * g8 + pr;
                if (pl < r && at.left > 0)
                    store8<ANY>(o + (size_t)pl * plane, at.left, *reinterpret_cast<const u32x4_t *>(slab + pl * ROWB + ((ch ^ swz(pl)) << 4)));
            }
            continue;
        }
        const size_t rowb_out = plane_row_base(I, pg, r, Cc);
#pragma unroll
        for (int g8 = 0; g8 < KC * 4; ++g8) {
            const int pl = 8 * g8 + pr;
            if (pl < r && J0 + 8 * ch < Cc) {
                const u32x4_t w = *reinterpret_cast<const u32x4_t *>(slab + pl * ROWB + ((ch ^ swz(pl)) << 4));
                bf16_t *o = P + rowb_out + (size_t)pl * plane + J0 + 8 * ch;
                if constexpr (SHIFT) store8_between(o, J0 + 8 * ch < 0 ? -(J0 + 8 * ch) : 0, Cc - J0 - 8 * ch, w);
                else if constexpr (ANY) store8<true>(o, Cc - J0 - 8 * ch, w);
                else store16<THROUGH>(o, w);
            }
        }
    }

}

// The item loop of one wavefront, items as in encode_items.  slab: KC * 32 * 128 bytes of LDS private to the
// wavefront; sT: 64 x 32 bytes (OUTER only); oacc accumulates the basis gradient (OUTER).  No workgroup barrier inside.
// DECODE = false: the basis gradient alone (Dm and Cmat unused).  TP: storage type of the planes; fp32 planes (the gradient of
// an encoded weight) are rounded to bf16 on their way into LDS.
template <bool GELU, int KC, bool OUTER, int DEPTH = 1, bool ANY = false, bool DECODE = true, typename TP = bf16_t, bool NARROW = false, bool FLAT = false>   // DEPTH, ANY, NARROW, FLAT as in encode_items
__device__ __forceinline__ void decode_items(const TP *__restrict__ P, const bf16_t *__restrict__ Dm, bf16_t *__restrict__ Cmat,
                                             int R, int Cc, int r, int chunks, const bf16_t *__restrict__ V, int pg, const RowMap &rm,
                                             long first, long stride, long end, char *sT, char *slab, f32x4_t (&oacc)[4], int lane,
                                             bool turned = false, int lw = 6, Lay lay = Lay{})                          // as in encode_items
{
    constexpr int ROWB = 128;                               // bytes per LDS row (64 tiles)
    const int ngroups = (r + 15) >> 4;
    const int j = lane & 15, kq = lane >> 4;
    // row of tile `lane` in sT: rows t and t^4 are swapped where bit 3 of t is set, so that the four 4-tile groups one
    // transposing read touches fall into both halves of the banks
    const int strow = lane ^ (((lane >> 3) & 1) << 2);

    // A fragments: lane (entry q = j, kq) holds D[32g + 8kq + e][q], e = 0..7
    bf16x8_t fa[KC];
#pragma unroll
    for (int g = 0; g < (DECODE ? KC : 0); ++g) {
        uint32_t w[4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            const int p0 = 32 * g + 8 * kq + 2 * e2;
            const int q = turned ? 4 * (j & 3) + (j >> 2) : j;
            const uint32_t lo = p0 < r ? Dm[p0 * 16 + q] : 0u, hi = p0 + 1 < r ? Dm[(p0 + 1) * 16 + q] : 0u;
            w[e2] = lo | (hi << 16);
        }
        fa[g] = __builtin_bit_cast(bf16x8_t, u32x4_t{w[0], w[1], w[2], w[3]});
    }
    // swizzle of the 16-byte chunk index inside a row, so that the 8 plane rows one transposing read touches
    // (planes 0-3 and 8-11, or 4-7 and 12-15, of a 16-tile column group) fall into different bank windows
    auto swz = [](int row) { return ((((row >> 1) & 1) | (((row >> 3) & 1) << 1)) << 1); };

    const size_t plane = (size_t)pg * Cc;
    const size_t ld = (size_t)Cc * 4;

    // Loader role of a lane: plane 8*g8 + pr, 16-byte chunk ch (8 tiles) -- whole 128-byte lines, 8 planes per
    // instruction; with OUTER also tile J0 + lane of V (4 rows x 8 bytes).  The NEXT item's operands are fetched into
    // registers while the current item is computed and stored.
    const int pr = lane >> 3, ch = lane & 7;
    Raw8<TP, ANY> pre[DEPTH][KC * 4];
    u32x2_t xpre[DEPTH][OUTER ? 4 : 1];
    struct Pos { int I, J; };
    auto locate = [&](long item, int t) {
        if constexpr (FLAT) return flat_tile(item, t, Cc).template as<Pos>();
        const int rb = (int)(item / chunks), ck = (int)(item - (long)rb * chunks);
        return Pos{(rb << (6 - lw)) + (t >> lw), (ck << lw) + (t & ((1 << lw) - 1))};
    };
    auto fetch_narrow = [&](int d, long item) {
        size_t off;
        int left;                                           // elements from there on that are the item's or follow it
        if constexpr (FLAT) {
            const FlatRun f = flat_run(item, 8 * ch, R, Cc, r);
            off = f.off;
            left = f.left;
        } else {
            const Pos at = locate(item, 8 * ch);
            off = (size_t)lay.row(at.I) + at.J;
            left = at.I < R ? Cc - at.J : 0;
        }
#pragma unroll
        for (int g8 = 0; g8 < KC * 4; ++g8) {
            const int pl = 8 * g8 + pr;
            pre[d][g8].load(P + off + (size_t)pl * plane, pl < r ? left : 0);
        }
        if (OUTER) {
            const Pos v = locate(item, lane);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                u32x2_t xv = {0u, 0u};
                if (v.I < R && v.J < Cc) xv = *reinterpret_cast<const u32x2_t *>(V + ((size_t)v.I * 4 + a) * ld + (size_t)v.J * 4);
                xpre[d][a] = xv;
            }
        }
    };
    auto fetch = [&](int d, long item) {
        if constexpr (NARROW) return fetch_narrow(d, item);
        const int Ii = (int)(item / chunks), cki = (int)(item - (long)Ii * chunks);
        const int Jl = cki * 64 + 8 * ch;
        const int Ia = Ii < R ? rm.tile_row(Ii) : 0;        // Ii counts the tile rows of this launch, Ia is the tile row itself
        const size_t rowb = plane_row_base(Ia, pg, r, Cc);
#pragma unroll
        for (int g8 = 0; g8 < KC * 4; ++g8) {
            const int pl = 8 * g8 + pr;
            // planes >= r stay zero (they meet zero D entries, but must be finite)
            pre[d][g8].load(P + rowb + (size_t)pl * plane + Jl, Ii < R && pl < r ? Cc - Jl : 0);
        }
        if (OUTER) {
            const int Jt = cki * 64 + lane, nv = rm.valid(Ia);
            const size_t r0 = rm.row0(Ia);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                u32x2_t xv = {0u, 0u};
                if (Ii < R && Jt < Cc && a < nv) xv = *reinterpret_cast<const u32x2_t *>(V + (r0 + a) * ld + (size_t)Jt * 4);
                xpre[d][a] = xv;
            }
        }
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (first + d * stride < end) fetch(d, first + d * stride);

    for (long base = first; base < end; base += DEPTH * stride)
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        const long item0 = base + d * stride;
        if (item0 >= end) break;
        const int In = (int)(item0 / chunks), J0 = (int)(item0 - (long)In * chunks) * 64;
        const bool live = NARROW || In < R;
        const int I = live && !NARROW ? rm.tile_row(In) : 0;
        // slab and sV belong to this wavefront alone and its LDS operations execute in order: the writes below land
        // after the previous round's fragment reads without a workgroup barrier (which would also make the wavefront
        // wait for the loads it is about to put in flight)
#pragma unroll
        for (int g8 = 0; g8 < KC * 4; ++g8) {
            const int pl = 8 * g8 + pr;
            *reinterpret_cast<u32x4_t *>(slab + pl * ROWB + ((ch ^ swz(pl)) << 4)) = pre[d][g8].take();
        }
        if (OUTER) {
            // lane = tile J0 + lane: its 16 entries (4 rows x 8 bytes) as two 16-byte writes, tile-major; they come back
            // as "entry x 4 consecutive tiles" through the transposing read below
            *reinterpret_cast<u32x4_t *>(sT + strow * 32) = u32x4_t{xpre[d][0][0], xpre[d][0][1], xpre[d][1][0], xpre[d][1][1]};
            *reinterpret_cast<u32x4_t *>(sT + strow * 32 + 16) = u32x4_t{xpre[d][2][0], xpre[d][2][1], xpre[d][3][0], xpre[d][3][1]};
        }
        if (item0 + DEPTH * stride < end) fetch(d, item0 + DEPTH * stride);
        if (live && OUTER) {
            // K = 32 tiles per MFMA: A = planes x tiles from the slab (lane: plane 16g + j, tiles 32s + 8kq ..),
            // B = tiles x entries from sT (lane: entry j, same tiles)
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                v4i16_t tb[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    // source address of this lane inside its 16-lane group: tile row (32sx + 8kq + 4h) + j/4, entries 4*(j%4)..
                    const int t0 = 32 * sx + 8 * kq + 4 * h;
                    const int row = (t0 ^ (((t0 >> 3) & 1) << 2)) + (j >> 2);
                    tb[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16_t *)(
                        (__attribute__((address_space(3))) char *)(sT + row * 32 + 8 * (j & 3))));
                }
                struct { v4i16_t a, b; } both_b = {tb[0], tb[1]};
                const bf16x8_t fb = __builtin_bit_cast(bf16x8_t, both_b);
#pragma unroll
                for (int g = 0; g < 2 * KC; ++g) {
                    if (g < ngroups) {
                        const int pl = 16 * g + j;
                        const bf16x8_t fp = *reinterpret_cast<const bf16x8_t *>(slab + pl * ROWB + (((4 * sx + kq) ^ swz(pl)) << 4));
                        oacc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fp, fb, oacc[g], 0, 0, 0);
                    }
                }
            }
        }
        if (live && DECODE) {
            const int nv_out = rm.valid(I);
            const size_t r0_out = rm.row0(I);
#pragma unroll
            for (int u = 0; u < 4; ++u) {                   // 16 tiles per MFMA
                f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int g = 0; g < KC; ++g) {
                    v4i16_t t[2];
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk) {
                        // source row for this lane of the 16-lane group: plane 32g + 8kq + 4kk + j/4, tiles 16u + 4(j%4)
                        const int row = 32 * g + 8 * kq + 4 * kk + (j >> 2);
                        const int col = 16 * u + 4 * (j & 3);
                        const char *src = slab + row * ROWB + ((((col >> 3)) ^ swz(row)) << 4) + ((col & 7) << 1);
                        t[kk] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16_t *)(
                            (__attribute__((address_space(3))) char *)src));
                    }
                    struct { v4i16_t a, b; } both = {t[0], t[1]};
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[g], __builtin_bit_cast(bf16x8_t, both), acc, 0, 0, 0);
                }
                // lane holds row a = kq of tile 16u + j of the item: entries acc[0..3]
                int J = J0 + 16 * u + j;
                size_t row = r0_out + kq;
                bool in = J < Cc && kq < nv_out;
                if constexpr (NARROW) {
                    const Pos at = locate(item0, 16 * u + j);
                    J = at.J;
                    row = (size_t)at.I * 4 + kq;
                    in = at.I < R && at.J < Cc;
                }
                if (in) {
                    float c0 = acc[0], c1 = acc[1], c2 = acc[2], c3 = acc[3];
                    if (GELU) { c0 = gelu_erf(c0); c1 = gelu_erf(c1); c2 = gelu_erf(c2); c3 = gelu_erf(c3); }
                    const u32x2_t w = {pack_bf16x2(c0, c1), pack_bf16x2(c2, c3)};
                    *reinterpret_cast<u32x2_t *>(Cmat + row * ld + (size_t)J * 4) = w;
                }
            }
        }
    }
}

// A block's partial of a basis gradient: accumulator e of group g of a wavefront is plane 16g + 4 (lane / 16) + e, tile entry lane % 16;
// fixed-order sum over the four wavefronts in `red`, 4 x (32 KC x 16) floats of LDS that they are done with otherwise.
template <int KC>
__device__ __forceinline__ void write_partial(const f32x4_t (&acc)[4], float *red, float *__restrict__ part, int r, int wave, int lane)
{
    __syncthreads();
#pragma unroll
    for (int g = 0; g < 2 * KC; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[wave * (KC * 512) + (16 * g + 4 * (lane >> 4) + e) * 16 + (lane & 15)] = acc[g][e];
    __syncthreads();
    for (int i = threadIdx.x; i < r * 16; i += 256)
        part[(size_t)blockIdx.x * r * 16 + i] = ((red[i] + red[KC * 512 + i]) + red[2 * KC * 512 + i]) + red[3 * KC * 512 + i];
}

}  // namespace stl
