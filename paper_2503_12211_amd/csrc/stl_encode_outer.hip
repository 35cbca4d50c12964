// Encode of a matrix and a basis gradient against other planes in one pass over the matrix (bf16):
//     P[p][I][J]  = sum_q E[p][q] * a[I][J][q]                  (a = 4x4 tile view of A)
//     G[p][q]    += sum_{I,J} Qp[p][I][J] * a[I][J][q]
// In the backward pass A = dC, E = D, P = dYhat, Qp = Yhat, G = dD: dC is read from HBM once for both results.
//
// Both contractions run on v_mfma_f32_16x16x32_bf16.
//  * Encode: rows = tiles, columns = planes, K = tile entries.  A lane (tile, kq) loads row kq of its tile (8 bytes,
//    entries 4kq..4kq+3) straight from HBM; padded with four zeros this is its operand fragment (K slot 8kq+e <->
//    entry 4kq+e for e < 4, zero weight on the other slots).  The tile of lane j in product u is
//    J0 + 8*(j/4) + 4*(u%2) + 32*(u/2) + j%4, which leaves a lane of the result (plane, kq) with 8 consecutive tiles
//    per product pair: 16-byte stores, 64 contiguous bytes per plane and instruction.
//  * Basis gradient: rows = planes, columns = tile entries, K = 32 tiles.  The plane segments of the item (128 bytes per
//    plane) are loaded as whole cache lines, 8 planes per instruction, into a wavefront-private LDS slab [plane][tile]
//    and read back as fragments (8 consecutive tiles of a plane = 16 bytes; fetching those 64-byte half lines
//    straight from HBM, 16 planes per instruction, ran a quarter slower).  The tile rows already in registers are
//    written tile-major into a second private slab (one 8-byte write each) and come back as "entry x 4 consecutive
//    tiles" through the transposing ds_read_b64_tr_b16.
// The next item's operands are fetched while the current one is processed; every block writes one partial of G to
// `part`, added up in block order by a second kernel (no floating-point atomics: bitwise reproducible).
#include "stl_kernels.h"
#include "stl_device.h"
#include "stl_tile_items.h"
#include <type_traits>

namespace stl {

// OUTER = false: the encode alone (Qp, part unused) -- the same whole-line stores through the slab, used for plain encodes
// ANY: column counts that are no multiple of 8 (see load8); SHIFT: with items that begin on cache lines (see encode_items)
template <int KC, bool OUTER, bool ANY, bool SHIFT = false>   // KC = number of 32-plane groups (1: r <= 32, 2: r <= 64)
__global__ __launch_bounds__(256) void encode_outer16_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ E,
                                                             bf16_t *__restrict__ P, const bf16_t *__restrict__ Qp,
                                                             float *__restrict__ part, int R, int Cc, int r, int chunks, int pg,
                                                             RowMap rm)
{
    constexpr int ROWB = 128;                               // bytes per plane row of the slab (64 tiles)
    __shared__ __align__(16) char sT_all[OUTER ? 4 : 1][OUTER ? 64 * 32 : 16];   // per wavefront: [tile][16 entries] bf16
    __shared__ __align__(16) char slab_all[4][KC * 32 * ROWB];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32x4_t dacc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) dacc[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // wavefront w of block b takes items 4b + w, 4b + w + 4 * gridDim.x, ...
    encode_items<KC, OUTER, false, 1, ANY, SHIFT>(A, E, P, Qp, R, Cc, r, chunks, pg, rm, (long)blockIdx.x * 4 + wave, (long)gridDim.x * 4,
                            (long)R * chunks, sT_all[OUTER ? wave : 0], slab_all[wave], dacc, lane);

    if (!OUTER) return;
    write_partial<KC>(dacc, reinterpret_cast<float *>(&slab_all[0][0]), part, r, wave, lane);
}

int encode_outer_blocks(int R, int Cc)
{
    const long items = (long)R * ((Cc + 63) / 64);
    const long blocks = (items + 3) / 4;
    return (int)(blocks > 1024 ? 1024 : blocks);
}

// A plane row of a width that is no multiple of 8 begins anywhere in a cache line, so that items of 64 columns counted from its
// beginning write two incomplete lines per plane.  Items that follow the planes (flat_pays) write whole ones in the grouped layout; a weight's
// plane-major planes and rows behind a row map get items that begin where the lines do, once the planes no longer fit the caches beside the
// matrix.  us, weights in items of a row / from a cache line on: 8192 x 508 tiles, r = 32 144 / 96, 4096 x 508, r = 16 32 / 25, r = 49 74 / 59; where the planes
// are that large only just 4096 x 1004, r = 8 34 both ways, 4096 x 252, r = 49 25 / 24; below, 1024 x 1004, r = 16 12.6 both ways.  Ragged forward of 64
// images of 197 rows, 508 columns, r = 32 73 / 66, of 256, 252 columns, r = 16 72 / 76.  Narrower rows pay for an item more per row (16384 x 132, r = 49,
// grouped 78 / 95).
static bool line_starts(int R, int Cc, int r) { return Cc % 8 && Cc > 192 && (double)r * R * Cc >= 3.2e7; }

// Several rows to an item: up to 1024 tile rows every CU has at most one block of four items of a single row, and fuller items only make the longest one longer:
// 512 x 15 tiles, r = 64, 4.3 us in items of a row, 5.3 in items of four; 1024 x 15, r = 49, 8 % behind, 1152 x 15 7 % ahead, 1152 x 23,
// r = 64, 14 %, 4096 x 15, r = 64, 10.1 / 7.2; at r <= 16 all the same up to 2048.
EncodeItems encode_items_of(int R, int Cc, int r, int pg, bool plain_rows)
{
    if (R > 1024 && narrow_log2(1, Cc, plain_rows)) return EncodeItems::several_rows;
    if (plain_rows && flat_pays(R, Cc, pg, row_items(R, Cc))) return EncodeItems::flat;
    return line_starts(R, Cc, r) ? EncodeItems::line_starts : EncodeItems::row;
}

// Two encodes in one launch, blockIdx.y picks the matrix: for matrices of a few microseconds, where half of each launch is its beginning
// and its end.  The pair of 96 x (50 x 16) tiles, r = 32: 6.3 + 5.6 us and 1.2 for a transposed basis of the second -> 12.3, 6.9 in items of several tile rows.
struct EncodeSide {
    const bf16_t *A, *E;
    bf16_t *P;
    int R, Cc, chunks, lw;
    long items;
    Lay lay;
    bool turned;
    // false: a layout that Lay does not describe
    bool set(const TileSide &t, int r, int pg, bool narrow, bool flat)
    {
        A = (const bf16_t *)t.matrix;
        E = (const bf16_t *)t.basis;
        P = (bf16_t *)t.planes;
        R = t.R;
        Cc = t.Cc;
        turned = t.turned;
        const int l = narrow_log2(1, Cc, true);
        lw = narrow && l ? l : 6;
        chunks = (Cc + (1 << lw) - 1) >> lw;
        items = flat ? flat_items(R, Cc) : (long)((R + (64 >> lw) - 1) / (64 >> lw)) * chunks;
        return lay.set(pg, R, Cc, r);
    }
};

template <int KC, bool ANY, bool NARROW, bool FLAT>
__global__ __launch_bounds__(256) void encode_pair_kernel(EncodeSide s0, EncodeSide s1, int r, int pg)
{
    __shared__ __align__(16) char slab_all[4][KC * 32 * 128];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const EncodeSide s = blockIdx.y ? s1 : s0;
    f32x4_t none[4];
    encode_items<KC, false, false, 1, ANY, false, NARROW, FLAT>(s.A, s.E, s.P, nullptr, s.R, s.Cc, r, s.chunks, pg, RowMap(), (long)blockIdx.x * 4 + wave,
                                                                (long)gridDim.x * 4, s.items, nullptr, slab_all[wave], none, lane, s.turned,
                                                                s.lw, s.lay);
}

// n = 2: as the name says; n = 1: one matrix of 8 to 32 tile columns or in items that follow the planes
static hipError_t launch_encode_sides(const TileSide *t, int n, int r, int pg, hipStream_t st)
{
    EncodeSide s[2] = {};
    bool any = false, narrow = false, flat = true;
    long items = 0;
    for (int i = 0; i < n; ++i) items += row_items(t[i].R, t[i].Cc);
    for (int i = 0; i < n; ++i) {
        any = any || t[i].Cc % 8;
        narrow = narrow || narrow_log2(1, t[i].Cc, true);
        flat = flat && flat_pays(t[i].R, t[i].Cc, pg, items);
    }
    long blocks = 1;
    for (int i = 0; i < n; ++i) {
        if (!s[i].set(t[i], r, pg, narrow, flat)) return hipErrorInvalidValue;
        const long b = (s[i].items + 3) / 4;
        blocks = b > blocks ? b : blocks;
    }
    auto pick = [&](auto kc) {
        constexpr int KC = decltype(kc)::value;
        if (flat) return any ? encode_pair_kernel<KC, true, true, true> : encode_pair_kernel<KC, false, true, true>;
        return narrow ? (any ? encode_pair_kernel<KC, true, true, false> : encode_pair_kernel<KC, false, true, false>)
                      : (any ? encode_pair_kernel<KC, true, false, false> : encode_pair_kernel<KC, false, false, false>);
    };
    auto kern = r <= 32 ? pick(std::integral_constant<int, 1>{}) : pick(std::integral_constant<int, 2>{});
    hipLaunchKernelGGL(kern, dim3((unsigned)(blocks > 8192 ? 8192 : blocks), n), dim3(256), 0, st, s[0], s[1], r, pg);
    return hipGetLastError();
}

// One form of items serves both matrices: one this large, which takes 1.3 to 1.6 times as long in items of a row as in items that follow the planes
// (flat_pays), stays apart from any other.
bool encode_pair_eligible(int dtype, const TileSide *s, int r)
{
    return dtype == 1 && s[0].Cc >= 8 && s[1].Cc >= 8 && !line_starts(s[0].R, s[0].Cc, r) && !line_starts(s[1].R, s[1].Cc, r);
}

hipError_t launch_encode_pair(const TileSide *t, int r, int pg, hipStream_t st) { return launch_encode_sides(t, 2, r, pg, st); }

// encode and basis gradient of a matrix of 8 to 32 tile columns, or in items that follow the planes (FLAT), nb blocks that leave one partial each
template <int KC, bool ANY, bool FLAT>
__global__ __launch_bounds__(256) void encode_outer_narrow_kernel(EncodeSide s, const bf16_t *__restrict__ Qp, float *__restrict__ part, int r, int pg)
{
    __shared__ __align__(16) char sT_all[4][64 * 32];
    __shared__ __align__(16) char slab_all[4][KC * 32 * 128];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32x4_t dacc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) dacc[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    encode_items<KC, true, false, 1, ANY, false, true, FLAT>(s.A, s.E, s.P, Qp, s.R, s.Cc, r, s.chunks, pg, RowMap(), (long)blockIdx.x * 4 + wave,
                                                             (long)gridDim.x * 4, s.items, sT_all[wave], slab_all[wave], dacc, lane, false, s.lw,
                                                             s.lay);
    write_partial<KC>(dacc, reinterpret_cast<float *>(&slab_all[0][0]), part, r, wave, lane);
}

static hipError_t launch_encode_outer_narrow(const TileSide &t, const void *Qp, float *part, int r, int pg, int nb, hipStream_t st)
{
    const bool any = t.Cc % 8, flat = flat_form(t.R, t.Cc, pg);
    EncodeSide s;
    if (!s.set(t, r, pg, true, flat)) return hipErrorInvalidValue;
    auto pick = [&](auto any_c, auto flat_c) {
        constexpr bool ANY = decltype(any_c)::value, FLAT = decltype(flat_c)::value;
        return r <= 32 ? encode_outer_narrow_kernel<1, ANY, FLAT> : encode_outer_narrow_kernel<2, ANY, FLAT>;
    };
    using T = std::true_type;
    using F = std::false_type;
    auto kern = any ? (flat ? pick(T{}, T{}) : pick(T{}, F{})) : (flat ? pick(F{}, T{}) : pick(F{}, F{}));
    hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, st, s, (const bf16_t *)Qp, part, r, pg);
    return hipGetLastError();
}

// both maps on the matrix cores (bf16, Cc >= 8), nb blocks that leave one partial each; R counts the rows of this launch
hipError_t launch_encode_outer_lines(const void *A, const void *E, void *P, const void *Qp, float *part, int R, int Cc, int r, int pg,
                                     int nb, hipStream_t s, RowMap rm)
{
    if (rm.Mt == 0 && (narrow_log2(1, Cc, true) || flat_form(R, Cc, pg)))
        return launch_encode_outer_narrow({P, E, A, R, Cc, false, nullptr, nullptr}, Qp, part, r, pg, nb, s);
    const bool any = Cc % 8 != 0;
    auto kern = r <= 32 ? (any ? encode_outer16_kernel<1, true, true> : encode_outer16_kernel<1, true, false>)
                        : (any ? encode_outer16_kernel<2, true, true> : encode_outer16_kernel<2, true, false>);
    hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, s, (const bf16_t *)A, (const bf16_t *)E, (bf16_t *)P, (const bf16_t *)Qp, part, R,
                       Cc, r, (Cc + 63) / 64, pg, rm);
    return hipGetLastError();
}

// the encode alone through the same kernel (bf16, Cc >= 8): grid-stride over (tile row, 64-tile chunk) items
hipError_t launch_encode_lines(const void *A, const void *E, void *P, int R, int Cc, int r, int pg, hipStream_t s, RowMap rm)
{
    if (pg <= 0) pg = R;
    R = rm.count(R);
    if (R <= 0) return hipSuccess;
    const EncodeItems form = encode_items_of(R, Cc, r, pg, rm.Mt == 0);
    if (form == EncodeItems::several_rows || form == EncodeItems::flat) {
        const TileSide one{P, E, A, R, Cc, false, nullptr, nullptr};
        return launch_encode_sides(&one, 1, r, pg, s);
    }
    const bool any = Cc % 8 != 0, starts = form == EncodeItems::line_starts;
    const int chunks = starts ? (Cc + 126) / 64 : (Cc + 63) / 64;
    const long items = (long)R * chunks;
    long blocks = (items + 3) / 4;
    if (blocks > 8192) blocks = 8192;
    auto kern = starts  ? (r <= 32 ? encode_outer16_kernel<1, false, true, true> : encode_outer16_kernel<2, false, true, true>)
                : r <= 32 ? (any ? encode_outer16_kernel<1, false, true> : encode_outer16_kernel<1, false, false>)
                        : (any ? encode_outer16_kernel<2, false, true> : encode_outer16_kernel<2, false, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, (const bf16_t *)A, (const bf16_t *)E, (bf16_t *)P,
                       (const bf16_t *)nullptr, (float *)nullptr, R, Cc, r, chunks, pg, rm);
    return hipGetLastError();
}

}  // namespace stl
