// Tile-level linear maps of the STL operator: encode (step (i) of Algorithm 1), decode
// (step (iii)) and the two basis-gradient reductions.  All of these stream a matrix once
// through HBM; sums are fp32.
#include "stl_kernels.h"
#include "stl_device.h"
#include "stl_tile_items.h"
#include <type_traits>


namespace stl {

// Entry i = (p, rho, c) of the decoder of an image's last tile row: its real row rho is the fold of the four decoded ones.  Composed by
// each workgroup that needs it: as a launch of its own it took 4.6 us, each way.
template <typename T>
__device__ __forceinline__ float fold_entry(const T *__restrict__ Dm, const Fold &fold, int i)
{
    const int p = i >> 4, rho = (i >> 2) & 3, c = i & 3;
    float s = 0.f;
    if (rho < fold.nrho)
#pragma unroll
        for (int a = 0; a < 4; ++a) s = fmaf(fold.coef[rho * 4 + a], Elem<T>::ld(Dm + p * 16 + 4 * a + c), s);
    return s;
}

// ---------------------------------------------------------------------------------------
// The tile maps in fp32 arithmetic on the vector ALUs, for fp32 storage (plain encodes and decodes of large matrices: one tile
// per thread, below; basis gradients of small ones: tile_grad_kernel), for bf16 rows of fewer than 8 tiles and for the folded decoder:
//   ENC    Pout[p][I][J]  = sum_q B[p][q] V[4I + q/4][4J + q%4]                  (planes of encoded tiles)
//   DEC    Cmat[4I + q/4][4J + q%4] = sum_p B[p][q] Pin[p][I][J]                 (+ optional GELU)
//   OUTER  G[p][q] = sum_{I,J} Pin[p][I][J] V[4I + q/4][4J + q%4]                (basis gradient; with ENC or DEC or alone)
// A group of 256 threads takes items of 64 tiles: 64 tile columns of one tile row, or 64 >> lw tile rows of at most
// 1 << lw columns where the matrix is narrow.  The item's planes (float4 per thread, 256 bytes per plane) and tiles are
// staged through LDS, the next item's loads in flight meanwhile, and every thread then plays a role per map: ENC (tile, every
// fourth plane), DEC (tile, tile row), OUTER (entry q, every 16th plane; the 64 tiles of an item are summed on their own
// before they join the running sum).  Bound by HBM on large matrices and by latency on small ones, which is what the
// grouping is for: with one thread per tile, planes one after the other, 64 x 64 tiles at r = 49 took 9 us to encode,
// 19 to decode and 332 for a basis gradient (16 workgroups); now 5 and 5, and the gradient, which tile_grad_kernel takes at this size, 6.
// OUTER blocks leave one partial each, added up in block order by outer_final_kernel: no floating-point atomics, so the
// results are bitwise reproducible.
// ---------------------------------------------------------------------------------------
// T: storage type; FOLD: the basis is B composed with the fold of an image's last tile row (see fold_entry).
// R counts the tile rows this launch walks over (see RowMap).
constexpr int kTilePitch = 64 + 4;          // floats per LDS row of 64 tiles

template <typename T, bool FOLD, bool ENC, bool DEC, bool OUTER, bool GELU, int GROUPS>
__global__ __launch_bounds__(GROUPS * 256) void tile_map_kernel(const T *__restrict__ V, const T *__restrict__ Pin,
                                                                const T *__restrict__ B, T *__restrict__ Pout,
                                                                T *__restrict__ Cmat, float *__restrict__ part, int R, int Cc, int r,
                                                                int lw, int pg, RowMap rm, Fold fold)
{
    constexpr bool PLANES = DEC || OUTER, TILES = ENC || OUTER;
    constexpr int TP = kTilePitch;
    extern __shared__ __align__(16) char smem[];
    const int ng = (r + 15) >> 4;                            // plane rows are staged in whole groups of 16, zeros beyond r
    float *sB = reinterpret_cast<float *>(smem);             // [r][16]
    const int gt = threadIdx.x & 255, grp = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 8));
    float *sP = sB + r * 16 + grp * ((PLANES ? ng * 16 * TP : 0) + (TILES ? 16 * TP : 0));     // [p][tile]
    float *sX = sP + (PLANES ? ng * 16 * TP : 0);            // [q][tile]
    if (ENC || DEC)
        for (int i = threadIdx.x; i < r * 16; i += GROUPS * 256) sB[i] = FOLD ? fold_entry(B, fold, i) : Elem<T>::ld(B + i);

    const int W = 1 << lw, rows = 64 >> lw, chunks = (Cc + W - 1) >> lw;
    const long items = (long)((R + rows - 1) / rows) * chunks;
    const size_t ld = (size_t)Cc * 4, plane = (size_t)pg * Cc;

    // tile t of an item: index of its tile row among the rows of this launch, its tile column
    struct Pos { int idx, J; };
    auto locate = [&](long item, int t) {
        const int rb = (int)(item / chunks), ck = (int)(item - (long)rb * chunks);
        return Pos{rb * rows + (t >> lw), (ck << lw) + (t & (W - 1))};
    };
    const int t = gt & 63, a = gt >> 6;                      // roles: tile, tile row (ENC: planes a, a + 4, ...)
    const int c4 = gt & 15, p16 = gt >> 4;                   // loader of planes: tiles 4 c4 ..; planes p16, p16 + 16, ...

    f32x4_t pre[PLANES ? 4 : 1], xpre = {0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](long item) {
        if (PLANES) {
            const Pos at = locate(item, 4 * c4);
            const bool in = item < items && at.idx < R;
            const size_t off = in ? plane_row_base(rm.tile_row(at.idx), pg, r, Cc) + at.J : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = p16 + 16 * i;
                pre[i] = i < ng ? load4<T>(Pin + off + (size_t)p * plane, in && p < r ? Cc - at.J : 0) : f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
        }
        if (TILES) {
            const Pos at = locate(item, t);
            const int I = item < items && at.idx < R && at.J < Cc ? rm.tile_row(at.idx) : -1;
            xpre = I >= 0 && a < rm.valid(I) ? load4<T>(V + (rm.row0(I) + a) * ld + (size_t)at.J * 4, 4) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    };

    float acc[4] = {0.f, 0.f, 0.f, 0.f};                     // OUTER: entry q = c4, planes p16 + 16 i
    const long stride = (long)gridDim.x * GROUPS;
    fetch((long)blockIdx.x * GROUPS + grp);
    for (long base = (long)blockIdx.x * GROUPS; base < items; base += stride) {      // same trip count for all groups
        const long item = base + grp;
        __syncthreads();                                     // previous item's readers are done (first: nothing to wait for)
        if (PLANES)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < ng) *reinterpret_cast<f32x4_t *>(sP + (p16 + 16 * i) * TP + 4 * c4) = pre[i];
        if (TILES)
#pragma unroll
            for (int b = 0; b < 4; ++b) sX[(4 * a + b) * TP + t] = xpre[b];
        __syncthreads();
        fetch(item + stride);

        const Pos at = locate(item, t);
        const bool in = item < items && at.idx < R && at.J < Cc;
        const int I = in ? rm.tile_row(at.idx) : 0;
        if (OUTER) {
            f32x4_t s[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int u = 0; u < 16; ++u) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t *>(sX + c4 * TP + 4 * u);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (i < ng) {
                        const f32x4_t y = *reinterpret_cast<const f32x4_t *>(sP + (p16 + 16 * i) * TP + 4 * u);
#pragma unroll
                        for (int e = 0; e < 4; ++e) s[i][e] = fmaf(y[e], v[e], s[i][e]);
                    }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += (s[i][0] + s[i][1]) + (s[i][2] + s[i][3]);
        }
        if (ENC) {
            float x[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) x[q] = sX[q * TP + t];
            T *out = Pout + (in ? plane_row_base(I, pg, r, Cc) + at.J : 0);
#pragma unroll 4
            for (int p = a; p < r; p += 4) {
                float s = 0.f;
#pragma unroll
                for (int q = 0; q < 16; ++q) s = fmaf(sB[p * 16 + q], x[q], s);
                if (in) Elem<T>::st(out + (size_t)p * plane, s);
            }
        }
        if (DEC) {
            f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
            for (int p = 0; p < r; ++p) {
                const float y = sP[p * TP + t];
                const f32x4_t d = *reinterpret_cast<const f32x4_t *>(sB + p * 16 + 4 * a);
#pragma unroll
                for (int e = 0; e < 4; ++e) c[e] = fmaf(d[e], y, c[e]);
            }
            if (GELU)
#pragma unroll
                for (int e = 0; e < 4; ++e) c[e] = gelu_erf(c[e]);
            if (in && a < rm.valid(I)) store4(Cmat + (rm.row0(I) + a) * ld + (size_t)at.J * 4, c);
        }
    }
    if (OUTER) {
        // fixed-order sum over the groups, then this block's partial
        __syncthreads();
        float *red = sB + r * 16;                            // [group][p][16] over the staging areas, all read by now
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < ng) red[(grp * ng * 16 + p16 + 16 * i) * 16 + c4] = acc[i];
        __syncthreads();
        for (int i = threadIdx.x; i < r * 16; i += GROUPS * 256) {
            float tot = red[i];
#pragma unroll
            for (int g = 1; g < GROUPS; ++g) tot += red[g * ng * 256 + i];
            part[(size_t)blockIdx.x * r * 16 + i] = tot;
        }
    }
}

// ---------------------------------------------------------------------------------------
// The basis gradient of a small fp32 matrix, with the encode or the decode it is fused with.  One partial sum covers 256 tiles (four
// items of 64, see above), which leaves a matrix of 64 x 64 tiles with 16 partials: as many workgroups of 1024 threads were bound by what one CU
// issues (11.5 us at r = 49, 8 of them with every sum taken out).  Here four workgroups of 256 threads share a partial: workgroup y
// sums planes 16 y .. 16 y + 15 over all its tiles (v_mfma_f32_32x32x2_f32, 64 tiles per wavefront on their own) and encodes those
// planes, or decodes item y.  All loads are in flight at once.  64 x 64 tiles, r = 49: 11.3 -> 6.1 with the encode,
// 12 -> 6.0 with the decode.
// ---------------------------------------------------------------------------------------
template <bool ENC, bool DEC>
__global__ __launch_bounds__(256) void tile_grad_kernel(const float *__restrict__ V, const float *__restrict__ Pin, const float *__restrict__ B,
                                                        float *__restrict__ Pout, float *__restrict__ Cmat, float *__restrict__ part, int R,
                                                        int Cc, int r, int lw, int chunks, Div by_chunk, Lay lp, RowMap rm)
{
    constexpr int PT = 256 + 4, PD = kTilePitch;
    __shared__ __align__(16) float sP[16][PT], sX[16][PT];   // [plane][tile], [entry][tile]; then the wavefronts' sums
    __shared__ __align__(16) float sD[DEC ? 64 : 1][PD];     // DEC: all planes of item y
    __shared__ __align__(16) float sB[ENC || DEC ? 64 * 16 : 4];
    const int tid = threadIdx.x, y = blockIdx.y, p0 = 16 * y, item0 = 4 * blockIdx.x;
    const int W = 1 << lw, rows = 64 >> lw;
    const bool sums = p0 < r;
    // tile t of the 256: its tile row among those of this launch, -1 beyond them, and its tile column
    struct Pos { int I, J; };
    auto locate = [&](int t) {
        const int item = item0 + (t >> 6), rb = by_chunk.of(item), idx = rb * rows + ((t & 63) >> lw), J = ((item - rb * chunks) << lw) + (t & (W - 1));
        return Pos{idx < R && J < Cc ? rm.tile_row(idx) : -1, J};
    };
    auto planes4 = [&](Pos at, int p) {                      // four neighbouring tiles of plane p
        return at.I >= 0 && p < r ? load4<float>(Pin + (size_t)p * lp.plane + lp.row(at.I) + at.J, Cc - at.J) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    };

    const Pos own = locate(tid);                             // ENC and the tiles' entries: a tile per thread
    const size_t ld = (size_t)Cc * 4;
    f32x4_t x[4], pv[4], dv[DEC ? 4 : 1];
    if (sums) {
        const int nv = own.I >= 0 ? rm.valid(own.I) : 0;
        const float *v = V + (own.I >= 0 ? rm.row0(own.I) * ld + (size_t)own.J * 4 : 0);
#pragma unroll
        for (int a = 0; a < 4; ++a) x[a] = a < nv ? load4<float>(v + a * ld, 4) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        const Pos at = locate(4 * (tid & 63));
#pragma unroll
        for (int i = 0; i < 4; ++i) pv[i] = planes4(at, p0 + (tid >> 6) + 4 * i);
    }
    if (DEC) {
        const Pos at = locate(64 * y + 4 * (tid & 15));
#pragma unroll
        for (int i = 0; i < 4; ++i) dv[i] = planes4(at, (tid >> 4) + 16 * i);
    }
    if (ENC || DEC)
        for (int i = tid; i < r * 16; i += 256) sB[i] = B[i];
    if (sums) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4_t *>(&sP[(tid >> 6) + 4 * i][4 * (tid & 63)]) = pv[i];
#pragma unroll
        for (int q = 0; q < 16; ++q) sX[q][tid] = x[q >> 2][q & 3];
    }
    if (DEC)
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4_t *>(&sD[(tid >> 4) + 16 * i][4 * (tid & 15)]) = dv[i];
    __syncthreads();

    const int wave = tid >> 6, fj = tid & 31, fh = (tid >> 5) & 1;
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    if (sums) {
        // rows = planes (16 of 32), columns = entries (16 of 32); a lane's four neighbouring tiles are the contraction index fh of
        // four products
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int t0 = 64 * wave + 8 * u + 4 * fh;
            const f32x4_t xv = *reinterpret_cast<const f32x4_t *>(&sX[fj & 15][t0]);
            const f32x4_t yv = *reinterpret_cast<const f32x4_t *>(&sP[fj & 15][t0]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(yv[e], xv[e], acc, 0, 0, 0);
        }
    }
    if (ENC && sums && own.I >= 0) {
        float *out = Pout + lp.row(own.I) + own.J;
        const int n = r - p0 < 16 ? r - p0 : 16;
#pragma unroll 4
        for (int p = 0; p < n; ++p) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) s = fmaf(sB[(p0 + p) * 16 + q], x[q >> 2][q & 3], s);
            out[(size_t)(p0 + p) * lp.plane] = s;
        }
    }
    if (DEC) {
        const int t = tid & 63, a = tid >> 6;
        const Pos at = locate(64 * y + t);
        f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int p = 0; p < r; ++p) {
            const f32x4_t d = *reinterpret_cast<const f32x4_t *>(sB + p * 16 + 4 * a);
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = fmaf(d[e], sD[p][t], c[e]);
        }
        if (at.I >= 0 && a < rm.valid(at.I)) store4(Cmat + (rm.row0(at.I) + a) * ld + (size_t)at.J * 4, c);
    }
    if (!sums) return;
    __syncthreads();
    float *red = &sP[0][0];                                  // [wavefront][plane][entry]
#pragma unroll
    for (int e = 0; e < 8; ++e)                              // element e: plane 8 (e / 4) + 4 fh + e % 4
        if (fj < 16) red[(wave * 16 + 8 * (e >> 2) + 4 * fh + (e & 3)) * 16 + fj] = acc[e];
    __syncthreads();
    if (p0 * 16 + tid < r * 16)
        part[(size_t)blockIdx.x * r * 16 + p0 * 16 + tid] = (red[tid] + red[256 + tid]) + (red[512 + tid] + red[768 + tid]);
}

// ---------------------------------------------------------------------------------------
// Encode and decode of large fp32 matrices, one tile per thread: the tile stays in registers, nothing but the basis goes through
// LDS, and a wavefront reads and writes whole cache lines of 64 neighbouring tiles.  The decode has eight planes' loads in
// flight.  Bound by HBM; the items of tile_map_kernel pay two barriers and an LDS round trip per 64 tiles, which only their
// fusions are worth, and help where one tile per thread leaves CUs idle.  us as items / one tile per thread:
//   encode 1024 x 1024 tiles, r = 4 / 16 / 49: 20 / 27 / 55 -> 13 / 22 / 46;  4096 x 1000, r = 16: 133 -> 104 (3.6 TB/s of 5.4 copied)
//   decode 1024 x 1024 tiles, r = 4 / 16 / 49: 27 / 31 / 62 -> 14 / 22 / 47;  4096 x 1000, r = 16: 131 -> 97;  16384 x 9, r = 16: 11.7 -> 7.6
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void encode_tiles_kernel(const float *__restrict__ A, const float *__restrict__ E, float *__restrict__ P,
                                                           int R, int Cc, int r, int pg, RowMap rm)
{
    __shared__ __align__(16) float sE[64 * 16];
    for (int i = threadIdx.y * blockDim.x + threadIdx.x; i < r * 16; i += 256) sE[i] = E[i];
    __syncthreads();
    const int J = blockIdx.x * blockDim.x + threadIdx.x;
    if (J >= Cc) return;
    const size_t ld = (size_t)Cc * 4, plane = (size_t)pg * Cc;
    for (int idx = blockIdx.y * blockDim.y + threadIdx.y; idx < R; idx += gridDim.y * blockDim.y) {
        const int I = rm.tile_row(idx), nv = rm.valid(I);
        const size_t r0 = rm.row0(I);
        f32x4_t x[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) x[a] = a < nv ? load4<float>(A + (r0 + a) * ld + (size_t)J * 4, 4) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        float *out = P + plane_row_base(I, pg, r, Cc) + J;
        for (int p = 0; p < r; ++p) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) s = fmaf(sE[p * 16 + q], x[q >> 2][q & 3], s);
            out[(size_t)p * plane] = s;
        }
    }
}

template <typename T, bool GELU>
__global__ __launch_bounds__(256) void decode_tiles_kernel(const T *__restrict__ P, const T *__restrict__ Dm, T *__restrict__ Cmat, int R,
                                                           int Cc, int r, int pg, RowMap rm)
{
    __shared__ __align__(16) float sD[64 * 16];
    for (int i = threadIdx.y * blockDim.x + threadIdx.x; i < r * 16; i += 256) sD[i] = Elem<T>::ld(Dm + i);
    __syncthreads();
    const int J = blockIdx.x * blockDim.x + threadIdx.x;
    if (J >= Cc) return;
    const size_t ld = (size_t)Cc * 4, plane = (size_t)pg * Cc;
    for (int idx = blockIdx.y * blockDim.y + threadIdx.y; idx < R; idx += gridDim.y * blockDim.y) {
        const int I = rm.tile_row(idx), nv = rm.valid(I);
        const size_t r0 = rm.row0(I);
        const T *in = P + plane_row_base(I, pg, r, Cc) + J;
        float c[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) c[q] = 0.f;
        for (int p0 = 0; p0 < r; p0 += 8) {
            float y[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) y[u] = p0 + u < r ? Elem<T>::ld(in + (size_t)(p0 + u) * plane) : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p0 + u < r)
#pragma unroll
                    for (int q = 0; q < 16; ++q) c[q] = fmaf(sD[(p0 + u) * 16 + q], y[u], c[q]);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            f32x4_t v;
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] = GELU ? gelu_erf(c[4 * a + b]) : c[4 * a + b];
            if (a < nv) store4(Cmat + (r0 + a) * ld + (size_t)J * 4, v);
        }
    }
}

// From 2^17 tiles on one tile per thread fills the chip (two wavefronts per SIMD; at 2^16 tiles and r = 64 the items are still ahead, 8.4
// against 10.7 us).  Rows of fewer than 8 tiles stay with the items at any rank (100000 x 3, r = 49: 20 against 25 us to
// encode), and so does the encode of bf16.  bf16 decodes of 9 to 15 columns: one tile per thread is ahead of items of several rows
// (decode_narrow_kernel) at the smallest ranks and behind them at 8, where the line lies since items were of a single row (10.3 us
// for 16384 x 9, r = 8).  us, one tile per thread / items of several rows: 16384 x 9 tiles, r = 1 / 3 / 8 3.9 / 4.5, 4.3 / 4.5, 5.0 / 4.5;
// 65536 x 12 9.3 / 11.0, 10.2 / 11.1, 14.6 / 11.9; 8800 x 15 3.5 / 3.9, 3.7 / 4.0, 4.6 / 4.2.
bool tile_per_thread(int dtype, bool decode, int R, int Cc, int r)
{
    if ((int64_t)R * Cc < 131072) return false;
    return dtype == 0 ? Cc >= 8 : decode && Cc % 8 && Cc >= 8 && Cc < 16 && r <= 8;
}

struct TileGrid {
    dim3 grid, block;
    // 64 tile columns where rows are whole lines of 64, otherwise as many as a row takes, up to 256: a line that two blocks
    // share costs (4096 x 1000 tiles, r = 32, encode: 176 us at 256 columns, 232 at 64), and so do planes 4 MB apart whose rows
    // all blocks walk in step (16 x 16384, r = 32: 14.0 us at 256, 8.6 at 64)
    TileGrid(int R, int Cc)
    {
        int bx = Cc % 64 == 0 ? 64 : 256;
        while (bx > 8 && bx / 2 >= Cc) bx /= 2;
        const int by = 256 / bx, rows = (R + by - 1) / by;
        grid = dim3((Cc + bx - 1) / bx, rows > 32768 ? 32768 : rows);      // the kernels stride over the rows
        block = dim3(bx, by);
    }
};

// second stage of the basis-gradient sums: the blocks' partials in block order; blockIdx.y picks the sum
struct OuterSums {
    OuterSum s[3];
};

__global__ __launch_bounds__(1024) void outer_final_kernel(OuterSums sums, int n_out)
{
    const OuterSum m = blockIdx.y == 0 ? sums.s[0] : blockIdx.y == 1 ? sums.s[1] : sums.s[2];
    const float *part = m.part;
    float *G = m.G;
    const int nblocks = m.nb;
    // 16 outputs per block of 1024 threads; 64 slices of the block range per output (up to 1024 partials: 16 loads per
    // thread, all in flight together), then a fixed-order sum over the slices.
    __shared__ float red[64][17];
    const int o = threadIdx.x & 15, sl = threadIdx.x >> 4;
    const int i = blockIdx.x * 16 + o;
    float s = 0.f;
    if (i < n_out)
#pragma unroll 16
        for (int b = sl; b < nblocks; b += 64) s += part[(size_t)b * n_out + i];
    red[sl][o] = s;
    __syncthreads();
    if (sl == 0 && i < n_out) {
        float tot = 0.f;
#pragma unroll
        for (int u = 0; u < 64; ++u) tot += red[u][o];
        const int to = m.turned ? (i & ~15) + 4 * (i & 3) + ((i >> 2) & 3) : i;
        G[to] = m.accumulate ? G[to] + tot : tot;
    }
}

// ---------------------------------------------------------------------------------------
// bf16 decode on the matrix cores:  tile entries (16) x tiles = D^T (16 x r) . Yhat (r x tiles),
// v_mfma_f32_16x16x32_bf16 with rows = tile entries, columns = 16 tiles, K = planes.
// A wavefront takes 64 consecutive tiles of one tile row: the r plane segments (128 bytes each) are
// read coalesced into a private LDS slab [plane][tile]; the transposing ds_read_b64_tr_b16 hands
// every lane 4 consecutive planes of its tile (the MFMA B fragment).  The accumulator leaves each
// lane with one row of one output tile (4 entries = 8 bytes), so 16 lanes store 128 contiguous bytes.
// ---------------------------------------------------------------------------------------
// OUTER: the same pass also accumulates the basis gradient G (r x 16) += P (r x tiles) . tileview(V) (tiles x 16)
// (dE_X with P = dXhat, V = X while dX is decoded), so that the planes are read from HBM once for both results;
// every block writes one partial to `part`, added up in block order by outer_final_kernel.  DECODE = false: G alone.
// ANY: column counts that are no multiple of 8 (see load8).  TP: storage type of the planes.
template <bool GELU, int KC, bool OUTER, bool ANY = false, bool DECODE = true, typename TP = bf16_t>   // KC = number of 32-plane groups (1: r <= 32, 2: r <= 64)
__global__ __launch_bounds__(256) void decode_mfma_kernel(const TP *__restrict__ P, const bf16_t *__restrict__ Dm,
                                                          bf16_t *__restrict__ Cmat, int R, int Cc, int r, int chunks,
                                                          const bf16_t *__restrict__ V, float *__restrict__ part, int pg,
                                                          RowMap rm)
{
    constexpr int ROWB = 128;                               // bytes per LDS row (64 tiles)
    __shared__ __align__(16) char slab_all[4][KC * 32 * ROWB];
    // OUTER: per wavefront the 64 tiles of V, tile-major [tile][16 entries] (32 bytes per tile)
    __shared__ __align__(16) char sT_all[OUTER ? 4 : 1][OUTER ? 64 * 32 : 16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32x4_t oacc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) oacc[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // wavefront w of block b takes items 4b + w, 4b + w + 4 * gridDim.x, ...
    decode_items<GELU, KC, OUTER, 1, ANY, DECODE, TP>(P, Dm, Cmat, R, Cc, r, chunks, V, pg, rm, (long)blockIdx.x * 4 + wave, (long)gridDim.x * 4,
                                  (long)R * chunks, sT_all[OUTER ? wave : 0], slab_all[wave], oacc, lane);
    if (OUTER) write_partial<KC>(oacc, reinterpret_cast<float *>(&slab_all[0][0]), part, r, wave, lane);
}

// Two decodes with a basis gradient each in one launch, blockIdx.y picks the matrix (see encode_pair_kernel).  96 x (50 x 16) tiles
// twice, r = 32: 7.7 + 8.0 -> 12.7 us, 7.6 in items of several tile rows.
struct DecodeSide {
    const bf16_t *P, *Dm, *V;
    bf16_t *Cmat;
    float *part;
    int R, Cc, chunks, nb, lw;
    long items;
    Lay lay;
    bool turned;
    bool set(const TileSide &t, int r, int pg, bool narrow, bool flat)
    {
        P = (const bf16_t *)t.planes;
        Dm = (const bf16_t *)t.basis;
        V = (const bf16_t *)t.V;
        Cmat = (bf16_t *)t.matrix;
        part = t.part;
        R = t.R;
        Cc = t.Cc;
        turned = t.turned;
        const int l = narrow_log2(1, Cc, true);
        lw = narrow && l ? l : 6;
        chunks = (Cc + (1 << lw) - 1) >> lw;
        items = flat ? flat_items(R, Cc) : (long)((R + (64 >> lw) - 1) / (64 >> lw)) * chunks;
        nb = gradient_blocks(1, R, Cc, true);
        return lay.set(pg, R, Cc, r);
    }
};

template <int KC, bool ANY, bool NARROW, bool DECODE, bool FLAT>
__global__ __launch_bounds__(256) void decode_outer_pair_kernel(DecodeSide s0, DecodeSide s1, int r, int pg)
{
    constexpr int ROWB = 128;
    __shared__ __align__(16) char slab_all[4][KC * 32 * ROWB];
    __shared__ __align__(16) char sT_all[4][64 * 32];
    const DecodeSide s = blockIdx.y ? s1 : s0;
    if ((int)blockIdx.x >= s.nb) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32x4_t oacc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) oacc[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    decode_items<false, KC, true, 1, ANY, DECODE, bf16_t, NARROW, FLAT>(s.P, s.Dm, s.Cmat, s.R, s.Cc, r, s.chunks, s.V, pg, RowMap(),
                                                                        (long)blockIdx.x * 4 + wave, (long)s.nb * 4, s.items, sT_all[wave],
                                                                        slab_all[wave], oacc, lane, s.turned, s.lw, s.lay);
    write_partial<KC>(oacc, reinterpret_cast<float *>(&slab_all[0][0]), s.part, r, wave, lane);
}

// decode of a matrix of 8 to 32 tile columns, or in items that follow the planes
template <bool GELU, int KC, bool ANY, bool FLAT>
__global__ __launch_bounds__(256) void decode_narrow_kernel(DecodeSide s, int r, int pg)
{
    __shared__ __align__(16) char slab_all[4][KC * 32 * 128];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32x4_t none[4];
    decode_items<GELU, KC, false, 1, ANY, true, bf16_t, true, FLAT>(s.P, s.Dm, s.Cmat, s.R, s.Cc, r, s.chunks, nullptr, pg, RowMap(), (long)blockIdx.x * 4 + wave,
                                                                    (long)gridDim.x * 4, s.items, nullptr, slab_all[wave], none, lane, false,
                                                                    s.lw, s.lay);
}

// ---------------------------------------------------------------------------------------
// Images whose row count the tile size does not divide (Class-1 appendix, "More Details on STL Replacement in
// T2T-ViT", item 1): the nrho = rows mod 4 real rows of an image's last tile row are linear combinations of the 4
// padded output rows, out[rho] = sum_a fold[rho][a] y[a].  Since y[a][c] = sum_p Dm[p][4a+c] yhat[p], the fold is a
// decode with the composed decoder
//     Dp[p][4 rho + c] = sum_a fold[rho][a] Dm[p][4a + c]      (zero for rho >= nrho),
// and its adjoint an encode with the same Dp.  Dp is kept in fp32.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fold_decoder_kernel(const float *__restrict__ Dm, Fold fold, float *__restrict__ Dp, int r)
{
    for (int i = threadIdx.x; i < r * 16; i += 256) Dp[i] = fold_entry(Dm, fold, i);
}

// Gt[p][4 rho + c] = sum over the images' last tile rows of Yhat[p] * dC[rho][c] (rows rho >= nrho are zero) gives both
//     dD[p][4a + c]  += sum_rho fold[rho][a] Gt[p][4 rho + c]        (added to the part from the complete tile rows)
//     dfold[rho][a] (+)= sum_{p,c} Dm[p][4a + c] Gt[p][4 rho + c]    (fixed summation order)
// A thread has one entry of dD; for dfold a thread has a plane's share of one entry, added up in plane order.  (One thread to an entry of
// dfold walked over all planes, a load at a time: 8.0 us at r = 32; 64 images of 197 tokens, 768 -> 3072, forward and backward 353.6 -> 348.8.)
template <typename T>
__global__ __launch_bounds__(1024) void fold_grads_kernel(const float *__restrict__ Gt, const T *__restrict__ Dm,
                                                          const float *__restrict__ fold, float *__restrict__ dD,
                                                          float *__restrict__ dfold, int r, int nrho, int accumulate)
{
    __shared__ float red[64][13];
    const int i = threadIdx.x, p = i >> 4, e = i & 15;               // r <= 64
    if (p < r) {
        const int a = e & 3, rho = e >> 2;                           // of dfold
        f32x4_t g = {0.f, 0.f, 0.f, 0.f};
        float d[4];
        if (rho < nrho) g = *reinterpret_cast<const f32x4_t *>(Gt + p * 16 + 4 * rho);
#pragma unroll
        for (int c = 0; c < 4; ++c) d[c] = Elem<T>::ld(Dm + p * 16 + 4 * a + c);
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) s = fmaf(d[c], g[c], s);
        if (rho < nrho) red[p][e] = s;
        if (dD) {
            const float old = dD[i];
            float t = 0.f;
#pragma unroll
            for (int q = 0; q < 3; ++q)
                if (q < nrho) t = fmaf(fold[q * 4 + rho], Gt[p * 16 + 4 * q + a], t);
            dD[i] = old + t;
        }
    }
    __syncthreads();
    if (dfold && i < nrho * 4) {
        float s = 0.f;
        for (int q = 0; q < r; ++q) s += red[q][i];
        dfold[i] = accumulate ? dfold[i] + s : s;
    }
}

hipError_t launch_fold_decoder(const void *Dm, Fold fold, float *Dp, int r, hipStream_t s)
{
    hipLaunchKernelGGL(fold_decoder_kernel, dim3(1), dim3(256), 0, s, (const float *)Dm, fold, Dp, r);
    return hipGetLastError();
}

hipError_t launch_fold_grads(int dtype, const float *Gt, const void *Dm, const float *fold, float *dD, float *dfold, int r,
                             int nrho, int accumulate, hipStream_t s)
{
    if (dtype == 0)
        hipLaunchKernelGGL(fold_grads_kernel<float>, dim3(1), dim3(1024), 0, s, Gt, (const float *)Dm, fold, dD, dfold, r, nrho,
                           accumulate);
    else
        hipLaunchKernelGGL(fold_grads_kernel<bf16_t>, dim3(1), dim3(1024), 0, s, Gt, (const bf16_t *)Dm, fold, dD, dfold, r, nrho,
                           accumulate);
    return hipGetLastError();
}

// out[p][4a + b] (+)= in[p][4b + a]: vec of a transposed tile.  An encoder for B^T given as tiles of B, and the way back
// for its gradient (the map is its own inverse).
template <typename TI, typename TO>
__global__ __launch_bounds__(256) void transpose_basis_kernel(const TI *__restrict__ in, TO *__restrict__ out, int r, int accumulate)
{
    for (int i = threadIdx.x; i < r * 16; i += 256) {
        const int p = i >> 4, a = (i >> 2) & 3, b = i & 3;
        const float v = Elem<TI>::ld(in + p * 16 + 4 * b + a);
        Elem<TO>::st(out + i, accumulate ? Elem<TO>::ld(out + i) + v : v);
    }
}

hipError_t launch_transpose_basis(int dtype, const void *E, void *Et, int r, hipStream_t s)
{
    if (dtype == 0) hipLaunchKernelGGL((transpose_basis_kernel<float, float>), dim3(1), dim3(256), 0, s, (const float *)E, (float *)Et, r, 0);
    else hipLaunchKernelGGL((transpose_basis_kernel<bf16_t, bf16_t>), dim3(1), dim3(256), 0, s, (const bf16_t *)E, (bf16_t *)Et, r, 0);
    return hipGetLastError();
}

hipError_t launch_transpose_basis_grad(const float *Gt, float *G, int r, int accumulate, hipStream_t s)
{
    hipLaunchKernelGGL((transpose_basis_kernel<float, float>), dim3(1), dim3(256), 0, s, Gt, G, r, accumulate);
    return hipGetLastError();
}

// fp32 -> bf16 (round to nearest even), 8 elements per thread; n8 = number of 8-element groups, tail handled per element
__global__ __launch_bounds__(256) void cast_bf16_kernel(const float *__restrict__ in, bf16_t *__restrict__ out, size_t n)
{
    const size_t n8 = n / 8;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (size_t)gridDim.x * 256) {
        const f32x4_t a = reinterpret_cast<const f32x4_t *>(in)[2 * i], b = reinterpret_cast<const f32x4_t *>(in)[2 * i + 1];
        reinterpret_cast<u32x4_t *>(out)[i] = u32x4_t{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]),
                                                      pack_bf16x2(b[2], b[3])};
    }
    if (blockIdx.x == 0 && threadIdx.x < (n & 7)) out[n8 * 8 + threadIdx.x] = f32_to_bf16(in[n8 * 8 + threadIdx.x]);
}

// ---------------------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------------------
hipError_t launch_cast_bf16(const float *in, void *out, size_t n, hipStream_t s)
{
    size_t blocks = (n / 8 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(cast_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, in, (bf16_t *)out, n);
    return hipGetLastError();
}

// lw: log2 of the tile columns an item takes per tile row (see tile_map_kernel), for rows of Cc tiles
static int tile_item_log2(int Cc)
{
    int lw = 2;                                             // at least the 4 tiles of a float4
    while (lw < 6 && (1 << lw) < Cc) ++lw;
    return lw;
}

// blocks > 0: exactly that many (one partial each); 0: as many as there are items, up to 8192
template <typename T, bool FOLD, bool ENC, bool DEC, bool OUTER, bool GELU>
static hipError_t launch_tile_map(const void *V, const void *Pin, const void *B, void *Pout, void *Cmat, float *part, int R, int Cc,
                                  int r, int pg, const RowMap &rm, int blocks, hipStream_t s, Fold fold = Fold())
{
    constexpr int GROUPS = OUTER ? 4 : 1;                   // a partial per four groups, as many blocks as the workspace has room for
    auto kern = tile_map_kernel<T, FOLD, ENC, DEC, OUTER, GELU, GROUPS>;
    constexpr int most = 64 * 16 * 4 + GROUPS * (64 + 16) * kTilePitch * 4;
    static_assert(most <= 160 * 1024, "LDS budget");
    const int ng = (r + 15) / 16, lw = tile_item_log2(Cc), rows = 64 >> lw;
    const int smem = r * 64 + GROUPS * ((DEC || OUTER ? ng * 16 : 0) + (ENC || OUTER ? 16 : 0)) * kTilePitch * 4;
    static std::atomic<uint64_t> granted{0};               // of this instantiation
    if (const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), smem, most, granted); e != hipSuccess) return e;
    const long items = (long)((R + rows - 1) / rows) * ((Cc + (1 << lw) - 1) >> lw);
    if (blocks <= 0) blocks = (int)(items > 8192 ? 8192 : items);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(GROUPS * 256), smem, s, (const T *)V, (const T *)Pin, (const T *)B, (T *)Pout,
                       (T *)Cmat, part, R, Cc, r, lw, pg, rm, fold);
    return hipGetLastError();
}

// the same with a basis gradient in nb partials, see tile_grad_kernel: where one partial per 256 tiles leaves CUs without one
template <bool ENC, bool DEC>
static hipError_t launch_tile_grad(const void *V, const void *Pin, const void *B, void *Pout, void *Cmat, float *part, int R, int R_all, int Cc,
                                   int r, int pg, const RowMap &rm, int nb, hipStream_t s)
{
    const int lw = tile_item_log2(Cc), chunks = (Cc + (1 << lw) - 1) >> lw;
    Lay lp;
    if (!lp.set(pg, R_all, Cc, r)) return hipErrorInvalidValue;
    const dim3 grid(nb, DEC ? 4 : (r + 15) / 16);
    hipLaunchKernelGGL((tile_grad_kernel<ENC, DEC>), grid, dim3(256), 0, s, (const float *)V, (const float *)Pin, (const float *)B, (float *)Pout,
                       (float *)Cmat, part, R, Cc, r, lw, chunks, Div::by(chunks), lp, rm);
    return hipGetLastError();
}

hipError_t launch_encode(int dtype, const void *A, const void *E, void *P, int R, int Cc, int r, int pg, hipStream_t s,
                         RowMap rm, Fold fold)
{
    if (pg <= 0) pg = R;
    const int Rs = rm.count(R);                             // tile rows this launch walks over
    if (Rs <= 0) return hipSuccess;
    if (dtype == 1 && Cc >= 8 && !fold.coef) return launch_encode_lines(A, E, P, R, Cc, r, pg, s, rm);
    if (tile_per_thread(dtype, false, Rs, Cc, r)) {
        const TileGrid t(Rs, Cc);
        hipLaunchKernelGGL(encode_tiles_kernel, t.grid, t.block, 0, s, (const float *)A, (const float *)E, (float *)P, Rs, Cc, r, pg, rm);
        return hipGetLastError();
    }
    auto run = dtype == 0     ? launch_tile_map<float, false, true, false, false, false>
               : fold.coef ? launch_tile_map<bf16_t, true, true, false, false, false>
                           : launch_tile_map<bf16_t, false, true, false, false, false>;
    return run(A, nullptr, E, P, nullptr, nullptr, Rs, Cc, r, pg, rm, 0, s, fold);
}

template <typename T>
static hipError_t launch_decode_tiles(const void *P, const void *Dm, void *Cmat, int R, int Cc, int r, bool gelu, int pg, hipStream_t s,
                                      const RowMap &rm)
{
    const TileGrid t(R, Cc);
    auto kern = gelu ? decode_tiles_kernel<T, true> : decode_tiles_kernel<T, false>;
    hipLaunchKernelGGL(kern, t.grid, t.block, 0, s, (const T *)P, (const T *)Dm, (T *)Cmat, R, Cc, r, pg, rm);
    return hipGetLastError();
}

template <bool ANY>
static auto pick_decode(int r, bool gelu)
{
    if (r <= 32) return gelu ? decode_mfma_kernel<true, 1, false, ANY> : decode_mfma_kernel<false, 1, false, ANY>;
    return gelu ? decode_mfma_kernel<true, 2, false, ANY> : decode_mfma_kernel<false, 2, false, ANY>;
}

hipError_t launch_decode(int dtype, const void *P, const void *Dm, void *Cmat, int R_all, int Cc, int r, bool gelu, int pg,
                         hipStream_t s, RowMap rm, Fold fold)
{
    if (pg <= 0) pg = R_all;
    if (fold.coef && gelu) return hipErrorInvalidValue;
    const int R = rm.count(R_all);                          // tile rows this launch walks over
    if (R <= 0) return hipSuccess;
    if ((dtype == 0 || !fold.coef) && tile_per_thread(dtype, true, R, Cc, r))
        return dtype == 0 ? launch_decode_tiles<float>(P, Dm, Cmat, R, Cc, r, gelu, pg, s, rm)
                          : launch_decode_tiles<bf16_t>(P, Dm, Cmat, R, Cc, r, gelu, pg, s, rm);
    const bool flat = dtype == 1 && rm.Mt == 0 && flat_pays(R, Cc, pg, row_items(R, Cc));
    if (dtype == 1 && !fold.coef && (flat || narrow_log2(dtype, Cc, rm.Mt == 0))) {
        DecodeSide d;
        if (!d.set({P, Dm, Cmat, R, Cc, false, nullptr, nullptr}, r, pg, true, flat)) return hipErrorInvalidValue;
        const long blocks = (d.items + 3) / 4;
        auto pick = [&](auto kc, auto flat_c) {
            constexpr int KC = decltype(kc)::value;
            constexpr bool FLAT = decltype(flat_c)::value;
            return Cc % 8 ? (gelu ? decode_narrow_kernel<true, KC, true, FLAT> : decode_narrow_kernel<false, KC, true, FLAT>)
                          : (gelu ? decode_narrow_kernel<true, KC, false, FLAT> : decode_narrow_kernel<false, KC, false, FLAT>);
        };
        using One = std::integral_constant<int, 1>;
        using Two = std::integral_constant<int, 2>;
        auto kern = flat ? (r <= 32 ? pick(One{}, std::true_type{}) : pick(Two{}, std::true_type{}))
                         : (r <= 32 ? pick(One{}, std::false_type{}) : pick(Two{}, std::false_type{}));
        hipLaunchKernelGGL(kern, dim3((unsigned)(blocks > 8192 ? 8192 : blocks)), dim3(256), 0, s, d, r, pg);
        return hipGetLastError();
    }
    if (dtype == 1 && Cc >= 8 && !fold.coef) {
        const int chunks = (Cc + 63) / 64;
        const long items = (long)R * chunks;
        long blocks = (items + 3) / 4;
        if (blocks > 8192) blocks = 8192;                   // grid-stride over (tile row, 64-tile chunk) items
        auto kern = Cc % 8 ? pick_decode<true>(r, gelu) : pick_decode<false>(r, gelu);
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, (const bf16_t *)P, (const bf16_t *)Dm, (bf16_t *)Cmat, R, Cc,
                           r, chunks, (const bf16_t *)nullptr, (float *)nullptr, pg, rm);
        return hipGetLastError();
    }
    auto run = dtype == 0     ? (gelu ? launch_tile_map<float, false, false, true, false, true> : launch_tile_map<float, false, false, true, false, false>)
               : fold.coef ? launch_tile_map<bf16_t, true, false, true, false, false>
                           : (gelu ? launch_tile_map<bf16_t, false, false, true, false, true> : launch_tile_map<bf16_t, false, false, true, false, false>);
    return run(nullptr, P, Dm, nullptr, Cmat, nullptr, R, Cc, r, pg, rm, 0, s, fold);
}

hipError_t launch_outer_finals(const OuterSum *sums, int n, int n_out, hipStream_t s)
{
    OuterSums all{};
    for (int i = 0; i < n && i < 3; ++i) all.s[i] = sums[i];
    hipLaunchKernelGGL(outer_final_kernel, dim3((n_out + 15) / 16, n), dim3(1024), 0, s, all, n_out);
    return hipGetLastError();
}

hipError_t launch_outer_final(const float *part, float *G, int nb, int n_out, int accumulate, hipStream_t s)
{
    const OuterSum one{part, G, nb, false, accumulate};
    return launch_outer_finals(&one, 1, n_out, s);
}

int decode_outer_blocks(int R, int Cc)
{
    const long items = (long)R * ((Cc + 63) / 64);
    const long blocks = (items + 3) / 4;
    return (int)(blocks > 1024 ? 1024 : blocks);
}

template <bool ANY>
static auto pick_decode_outer(int r, const void *Cmat)
{
    if (r <= 32) return Cmat ? decode_mfma_kernel<false, 1, true, ANY, true> : decode_mfma_kernel<false, 1, true, ANY, false>;
    return Cmat ? decode_mfma_kernel<false, 2, true, ANY, true> : decode_mfma_kernel<false, 2, true, ANY, false>;
}

// bf16 matrix from fp32 planes (plane-major): W <- decode(P, E) and, unless G is NULL, G (+)= P . tileview(V), the planes rounded to
// bf16 once.  Reading them as they are saves the pass that stored a rounded copy: 4096 x 4096, r = 32 (134 MB of planes), 40 + 28 us
// as rounding pass + decode, now 43 (4.7 TB/s).
hipError_t launch_decode_outer_f32(const float *P, const void *E, void *W, const void *V, float *G, float *part, int R, int Cc, int r,
                                   int accumulate, hipStream_t s)
{
    if (R <= 0 || Cc < 8) return hipErrorInvalidValue;
    const RowMap rm;
    const int chunks = (Cc + 63) / 64;
    const bf16_t *e = (const bf16_t *)E, *v = (const bf16_t *)V;
    bf16_t *w = (bf16_t *)W;
    if (!G) {
        const long items = (long)R * chunks, blocks = (items + 3) / 4;
        auto kern = r <= 32 ? (Cc % 8 ? decode_mfma_kernel<false, 1, false, true, true, float> : decode_mfma_kernel<false, 1, false, false, true, float>)
                            : (Cc % 8 ? decode_mfma_kernel<false, 2, false, true, true, float> : decode_mfma_kernel<false, 2, false, false, true, float>);
        hipLaunchKernelGGL(kern, dim3((unsigned)(blocks > 8192 ? 8192 : blocks)), dim3(256), 0, s, P, e, w, R, Cc, r, chunks, v, part, R, rm);
        return hipGetLastError();
    }
    const int nb = decode_outer_blocks(R, Cc);
    auto kern = W ? (r <= 32 ? (Cc % 8 ? decode_mfma_kernel<false, 1, true, true, true, float> : decode_mfma_kernel<false, 1, true, false, true, float>)
                             : (Cc % 8 ? decode_mfma_kernel<false, 2, true, true, true, float> : decode_mfma_kernel<false, 2, true, false, true, float>))
                  : (r <= 32 ? (Cc % 8 ? decode_mfma_kernel<false, 1, true, true, false, float> : decode_mfma_kernel<false, 1, true, false, false, float>)
                             : (Cc % 8 ? decode_mfma_kernel<false, 2, true, true, false, float> : decode_mfma_kernel<false, 2, true, false, false, float>));
    hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, s, P, e, w, R, Cc, r, chunks, v, part, R, rm);
    const hipError_t err = hipGetLastError();
    return err != hipSuccess ? err : launch_outer_final(part, G, nb, r * 16, accumulate, s);
}

// tile_grad_kernel has no loop over items and reads the matrix once per 16 planes (from L2 while it is small).  us of a step, items of
// tile_map_kernel / this: forward + backward of 128 x 256 x 256 tiles, r = 16 (128 partials) 71 / 46, 800 x 256 x 256, r = 16 (800) 177 / 162,
// 900 x 200 x 200, r = 32 (900) 262 / 258, but 250 x 256 x 256, r = 64 (250) 178 / 184.
static bool small_gradient(int nb, int r) { return nb < 1024 && (r <= 32 || nb <= 192); }

// n = 2: as the name says; n = 1: one matrix of 8 to 32 tile columns or in items that follow the planes (its matrix may be NULL: the basis gradient alone)
static hipError_t launch_decode_outer_sides(const TileSide *t, int n, int r, int pg, hipStream_t st)
{
    DecodeSide s[2] = {};
    bool any = false, narrow = false, flat = true;
    long items = 0;
    for (int i = 0; i < n; ++i) items += row_items(t[i].R, t[i].Cc);
    int nb = 1;
    for (int i = 0; i < n; ++i) {
        any = any || t[i].Cc % 8;
        narrow = narrow || narrow_log2(1, t[i].Cc, true);
        flat = flat && flat_pays(t[i].R, t[i].Cc, pg, items);
    }
    for (int i = 0; i < n; ++i) {
        if (!s[i].set(t[i], r, pg, narrow, flat)) return hipErrorInvalidValue;
        nb = s[i].nb > nb ? s[i].nb : nb;
    }
    auto pick = [&](auto kc) {
        constexpr int KC = decltype(kc)::value;
        if (flat)
            return t[0].matrix ? (any ? decode_outer_pair_kernel<KC, true, true, true, true> : decode_outer_pair_kernel<KC, false, true, true, true>)
                               : (any ? decode_outer_pair_kernel<KC, true, true, false, true> : decode_outer_pair_kernel<KC, false, true, false, true>);
        if (!t[0].matrix) return any ? decode_outer_pair_kernel<KC, true, true, false, false> : decode_outer_pair_kernel<KC, false, true, false, false>;
        return narrow ? (any ? decode_outer_pair_kernel<KC, true, true, true, false> : decode_outer_pair_kernel<KC, false, true, true, false>)
                      : (any ? decode_outer_pair_kernel<KC, true, false, true, false> : decode_outer_pair_kernel<KC, false, false, true, false>);
    };
    auto kern = r <= 32 ? pick(std::integral_constant<int, 1>{}) : pick(std::integral_constant<int, 2>{});
    hipLaunchKernelGGL(kern, dim3(nb, n), dim3(256), 0, st, s[0], s[1], r, pg);
    return hipGetLastError();
}

hipError_t launch_decode_outer_pair(const TileSide *t, int r, int pg, hipStream_t st) { return launch_decode_outer_sides(t, 2, r, pg, st); }

int narrow_log2(int dtype, int Cc, bool plain_rows)
{
    if (dtype != 1 || !plain_rows || Cc < 8 || Cc > 32) return 0;
    return Cc <= 8 ? 3 : Cc <= 16 ? 4 : 5;
}

int gradient_blocks(int dtype, int R, int Cc, bool plain_rows)
{
    const int lw = narrow_log2(dtype, Cc, plain_rows);
    if (!lw) return decode_outer_blocks(R, Cc);
    const int rows = 64 >> lw, blocks = ((R + rows - 1) / rows + 3) / 4;
    return blocks > 1024 ? 1024 : blocks;
}

// Cmat == nullptr: the basis gradient alone
hipError_t launch_decode_outer(int dtype, const void *P, const void *Dm, void *Cmat, const void *V, float *G, float *part, int R_all,
                               int Cc, int r, int accumulate, int pg, hipStream_t s, RowMap rm, bool final_sum)
{
    if (pg <= 0) pg = R_all;
    const int R = rm.count(R_all);
    if (R <= 0) return hipErrorInvalidValue;
    const int nb = gradient_blocks(dtype, R, Cc, rm.Mt == 0);
    hipError_t e;
    if (dtype == 1 && rm.Mt == 0 && (narrow_log2(dtype, Cc, true) || flat_pays(R, Cc, pg, row_items(R, Cc)))) {
        const TileSide one{P, Dm, Cmat, R, Cc, false, V, part};
        e = launch_decode_outer_sides(&one, 1, r, pg, s);
    } else if (dtype == 1 && Cc >= 8) {
        auto kern = Cc % 8 ? pick_decode_outer<true>(r, Cmat) : pick_decode_outer<false>(r, Cmat);
        hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, s, (const bf16_t *)P, (const bf16_t *)Dm, (bf16_t *)Cmat, R, Cc, r, (Cc + 63) / 64,
                           (const bf16_t *)V, part, pg, rm);
        e = hipGetLastError();
    } else {
        if (dtype == 0 && small_gradient(nb, r)) {
            e = Cmat ? launch_tile_grad<false, true>(V, P, Dm, nullptr, Cmat, part, R, R_all, Cc, r, pg, rm, nb, s)
                     : launch_tile_grad<false, false>(V, P, Dm, nullptr, nullptr, part, R, R_all, Cc, r, pg, rm, nb, s);
            return e != hipSuccess || !final_sum ? e : launch_outer_final(part, G, nb, r * 16, accumulate, s);
        }
        auto run = dtype == 0 ? (Cmat ? launch_tile_map<float, false, false, true, true, false> : launch_tile_map<float, false, false, false, true, false>)
                              : (Cmat ? launch_tile_map<bf16_t, false, false, true, true, false> : launch_tile_map<bf16_t, false, false, false, true, false>);
        e = run(V, P, Dm, nullptr, Cmat, part, R, Cc, r, pg, rm, nb, s, Fold());
    }
    if (e != hipSuccess || !final_sum) return e;
    return launch_outer_final(part, G, nb, r * 16, accumulate, s);
}

// The last tile rows of a stack of ragged images (bf16) in one pass over dC: planes of the folded rows and the partials of Yhat (x) dC.
// 64 images, 768 tile columns, r = 32: 11.2 us; 5.8 the planes and 4.9 the sums as launches of their own, and a gap between them.
hipError_t launch_fold_encode_outer(const void *A, const void *Dm, Fold fold, void *P, const void *Qp, float *part, int R_all, int Cc, int r,
                                    int pg, hipStream_t s, RowMap rm)
{
    const int R = rm.count(R_all);
    if (R <= 0) return hipErrorInvalidValue;
    return launch_tile_map<bf16_t, true, true, false, true, false>(A, Qp, Dm, P, nullptr, part, R, Cc, r, pg, rm,
                                                                   gradient_blocks(1, R, Cc, false), s, fold);
}

hipError_t launch_encode_outer(int dtype, const void *A, const void *E, void *P, const void *Qp, float *G, float *part, int R_all, int Cc,
                               int r, int accumulate, int pg, hipStream_t s, RowMap rm, bool final_sum)
{
    if (pg <= 0) pg = R_all;
    const int R = rm.count(R_all);
    if (R <= 0) return hipErrorInvalidValue;
    const int nb = gradient_blocks(dtype, R, Cc, rm.Mt == 0);
    hipError_t e;
    if (dtype == 1 && Cc >= 8) {
        e = launch_encode_outer_lines(A, E, P, Qp, part, R, Cc, r, pg, nb, s, rm);
    } else {
        if (dtype == 0 && small_gradient(nb, r)) {
            e = launch_tile_grad<true, false>(A, Qp, E, P, nullptr, part, R, R_all, Cc, r, pg, rm, nb, s);
            return e != hipSuccess || !final_sum ? e : launch_outer_final(part, G, nb, r * 16, accumulate, s);
        }
        auto run = dtype == 0 ? launch_tile_map<float, false, true, false, true, false> : launch_tile_map<bf16_t, false, true, false, true, false>;
        e = run(A, Qp, E, P, nullptr, part, R, Cc, r, pg, rm, nb, s, Fold());
    }
    if (e != hipSuccess || !final_sum) return e;
    return launch_outer_final(part, G, nb, r * 16, accumulate, s);
}

// Partials the workspaces have room for, besides decode_outer_blocks and encode_outer_blocks: their declared sizes stand.
int outer_reduce_blocks(int64_t tiles)
{
    int64_t tpb = (tiles + 511) / 512;
    tpb = (tpb + 255) / 256 * 256;
    if (tpb < 256) tpb = 256;
    return (int)((tiles + tpb - 1) / tpb);
}

}  // namespace stl
