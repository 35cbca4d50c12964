// Internal launcher interface between the C ABI (stl_api.hip) and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

namespace stl {

// Lets `kern` be launched with `bytes` of dynamic LDS, at most `most`, on the current device: more than 64 KB has to be asked for.
// `done` belongs to that kernel alone and holds the devices it has been granted on, a bit each; devices beyond 64 are asked
// every time.
inline hipError_t allow_lds(const void *kern, int bytes, int most, std::atomic<uint64_t> &done)
{
    if (bytes <= 64 * 1024) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
    if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
    return e;
}

// dtype: 0 = fp32 storage, 1 = bf16 storage (matches stl_dtype_t)
// pg: rows per group of the plane tensor's layout (see plane_row_base); 0 = plane-major (one group of all rows)
constexpr int kPlaneGroup = 64;   // group size of the activation-side plane tensors

// Which matrix rows lie behind a tile row of the plane tensors.
//   plain  (Mt == 0): tile row I covers matrix rows 4I .. 4I+3.
//   ragged (Mt > 0):  the matrix is a stack of images with `rows` real rows each (197 tokens in the Class-1 appendix),
//     thought of as padded with null rows to Mt = ceil(rows / 4) tile rows per image.  Tile row I = img * Mt + l covers
//     matrix rows img * rows + 4l + a for the a with 4l + a < rows; the other entry rows are null rows: they read as
//     zero and are never written.  Only the last tile row of an image can be incomplete.
// A launch walks over a selection of the tile rows: all of them, only the complete-by-position ones (every tile row
// but the last of each image), or only the last of each image.
struct RowMap {
    int Mt = 0, rows = 0;
    int sel = 0;                       // 0: all tile rows, 1: all but each image's last, 2: each image's last
    __host__ __device__ __forceinline__ int tile_row(int idx) const
    {
        if (Mt == 0 || sel == 0) return idx;
        if (sel == 1) return idx + idx / (Mt - 1);
        return idx * Mt + Mt - 1;
    }
    __host__ __device__ __forceinline__ size_t row0(int I) const
    {
        if (Mt == 0) return (size_t)I * 4;
        const int img = I / Mt;
        return (size_t)img * rows + (size_t)(I - img * Mt) * 4;
    }
    __host__ __device__ __forceinline__ int valid(int I) const       // real entry rows of tile row I (1..4)
    {
        if (Mt == 0) return 4;
        const int left = rows - (I % Mt) * 4;
        return left < 4 ? left : 4;
    }
    // number of tile rows a launch with this selection walks over, R = all tile rows
    __host__ __device__ __forceinline__ int count(int R) const
    {
        if (Mt == 0 || sel == 0) return R;
        return sel == 1 ? R / Mt * (Mt - 1) : R / Mt;
    }
};

// Fold of an image's last tile row (row counts not divisible by 4): nrho real rows, each a combination (nrho x 4 coefficients) of the
// four rows that its planes decode to; coef == NULL: none
struct Fold {
    const float *coef = nullptr;
    int nrho = 0;
};

// planes P[p][R][Cc] <- encoder E (r x 16) applied to every 4x4 tile of A (4R x 4Cc)
// rm: which matrix rows lie behind the tile rows, and which tile rows the launch walks over (R always counts ALL tile
// rows of the plane tensor); fold (bf16): E (or Dm) is composed with it
hipError_t launch_encode(int dtype, const void *A, const void *E, void *P, int R, int Cc, int r, int pg, hipStream_t s,
                         RowMap rm = RowMap(), Fold fold = Fold());
// matrix Cmat (4R x 4Cc) <- decoder Dm^T (r x 16 stored) applied to planes P[p][R][Cc]; gelu not with a fold
hipError_t launch_decode(int dtype, const void *P, const void *Dm, void *Cmat, int R, int Cc, int r, bool gelu, int pg,
                         hipStream_t s, RowMap rm = RowMap(), Fold fold = Fold());

// whether a plain encode or decode of R x Cc tiles goes one tile per thread (fp32 arithmetic)
bool tile_per_thread(int dtype, bool decode, int R, int Cc, int r);

// Basis gradient G[p][q] (+)= sum_tiles P[p][tile] * tileview(V)[tile][q], in one pass with the decode of the same planes
// (Cmat <- decode(P, Dm)), or alone when Cmat is NULL (Dm is not read then); `part` holds decode_outer_blocks(R, Cc) * r * 16 floats
int decode_outer_blocks(int R, int Cc);       // for the workspace; as many or fewer are used:
int gradient_blocks(int dtype, int R, int Cc, bool plain_rows);
// bf16 matrices of 8 to 32 tile columns (no row map) run in items of several tile rows, 1 << narrow_log2 columns each; 0: they do not
// (of more columns an item, 64 tiles of a power of two of columns, is a single row)
int narrow_log2(int dtype, int Cc, bool plain_rows);
// Items of a bf16 matrix without a row map: 64 tile columns of one row, or 64 tiles in a row of the planes (FLAT in stl_tile_items.h), which is
// possible where rows are no whole items and planes lie in groups of 64 tile rows.
inline long row_items(int R, int Cc) { return (long)R * ((Cc + 63) / 64); }
inline long flat_items(int R, int Cc) { return (long)(R / 64) * Cc + ((long)(R % 64) * Cc + 63) / 64; }
inline bool flat_form(int R, int Cc, int pg) { return pg == 64 && Cc > 32 && Cc % 64 && R < 1 << 24; }   // (R: Lay::set takes it)
// Whether that pays in a launch that has `items` of the first kind in all, other than the encode with a basis gradient.  An item that follows the
// planes costs two divisions more before its first load, and a launch of half a round of items or less takes the 5 us of its start either
// way.  Beyond that the planes' rows of 64 elements are whole cache lines if Cc is no multiple of 8 (2997 x 133 tiles, r = 64: encode
// 15.7 -> 12.7 us, decode 23.1 -> 15.3, with its basis gradient 31.5 -> 23.6; two such decodes 44.9 -> 32.3; large encodes, in items of a row / from a
// cache line on / this: 8192 x 508, r = 32 118 / 84 / 78, 16384 x 196, r = 32 94 / 85 / 65, 4096 x 252, r = 64 in the second and third 28.2 / 27.3, 4096 x 508,
// r = 64 71.6 / 71.5, 65536 x 201, r = 8 155 / 145 / 115; over 18 shapes of that size 1.00 to 1.30 times as fast as the second), and if it is there
// only are fewer items, which has to be felt: 3200 x 200, r = 32, 7/9 of them, decode 13.8 -> 11.5, but 2048 x 1000, 1/50 less, encode 35.6 -> 37.6.
inline bool flat_pays(int R, int Cc, int pg, long items)
{
    return flat_form(R, Cc, pg) && (Cc % 8 ? items > 2048 : items > 4096 && 8 * flat_items(R, Cc) <= 7 * row_items(R, Cc));
}
hipError_t launch_decode_outer(int dtype, const void *P, const void *Dm, void *Cmat, const void *V, float *G, float *part, int R,
                               int Cc, int r, int accumulate, int pg, hipStream_t s, RowMap rm = RowMap(), bool final_sum = true);
// the same from fp32 planes into a bf16 matrix (plane-major, Cc >= 8); W or G may be NULL
hipError_t launch_decode_outer_f32(const float *P, const void *E, void *W, const void *V, float *G, float *part, int R, int Cc, int r,
                                   int accumulate, hipStream_t s);
int outer_reduce_blocks(int64_t tiles);     // a further bound on the partials, for the declared workspace sizes

// G[i] (+)= sum over nb partials part[b][i], i < n_out, in block order (second stage of the basis-gradient sums)
hipError_t launch_outer_final(const float *part, float *G, int nb, int n_out, int accumulate, hipStream_t s);
// up to three such sums in one launch (final_sum = false in the fused passes leaves their partials for this); turned: the partials
// are of the basis for the tiles' transposes, G[p][4a + b] gets entry 4b + a
struct OuterSum {
    const float *part;
    float *G;
    int nb;
    bool turned;
    int accumulate;
};
hipError_t launch_outer_finals(const OuterSum *sums, int n, int n_out, hipStream_t s);

// encode and basis gradient in one pass over the matrix: P <- encode(A, E), G (+)= Qp . tileview(A);
// `part` holds encode_outer_blocks(R, Cc) * r * 16 floats (gradient_blocks of them are used)
int encode_outer_blocks(int R, int Cc);
hipError_t launch_encode_outer(int dtype, const void *A, const void *E, void *P, const void *Qp, float *G, float *part, int R, int Cc,
                               int r, int accumulate, int pg, hipStream_t s, RowMap rm = RowMap(), bool final_sum = true);
// its bf16 kernel (Cc >= 8); launch_encode_outer picks it
hipError_t launch_encode_outer_lines(const void *A, const void *E, void *P, const void *Qp, float *part, int R, int Cc, int r, int pg,
                                     int nb, hipStream_t s, RowMap rm);

// Two matrices of one dtype (bf16) and rank in one launch: their encodes, or their decodes with a basis gradient each (partials only;
// Cmat and V of R x Cc tiles, `part` holds decode_outer_blocks(R, Cc) * r * 16 floats).  turned: see encode_items.
struct TileSide {
    const void *planes, *basis, *matrix;          // of planes and matrix one is written
    int R, Cc;
    bool turned;
    const void *V;
    float *part;
};
bool encode_pair_eligible(int dtype, const TileSide *s, int r);
hipError_t launch_encode_pair(const TileSide *s, int r, int pg, hipStream_t st);
hipError_t launch_decode_outer_pair(const TileSide *s, int r, int pg, hipStream_t st);

// fold of an image's last tile row (row counts not divisible by 4): composed decoder Dp (r x 16 fp32) from Dm and the
// nrho x 4 fold coefficients; and the gradients that come from those tile rows, given Gt = Yhat (x) dC over them
hipError_t launch_fold_decoder(const void *Dm, Fold fold, float *Dp, int r, hipStream_t s);        // fp32 storage; bf16 maps compose it themselves
hipError_t launch_fold_encode_outer(const void *A, const void *Dm, Fold fold, void *P, const void *Qp, float *part, int R_all, int Cc, int r,
                                    int pg, hipStream_t s, RowMap rm);
hipError_t launch_fold_grads(int dtype, const float *Gt, const void *Dm, const float *fold, float *dD, float *dfold, int r,
                             int nrho, int accumulate, hipStream_t s);

// Et[p][4a+b] = E[p][4b+a] (storage type): the basis that encodes B^T when applied to the tiles of B; and the same map
// on a gradient, G[p][4a+b] (+)= Gt[p][4b+a] (fp32)
hipError_t launch_transpose_basis(int dtype, const void *E, void *Et, int r, hipStream_t s);
hipError_t launch_transpose_basis_grad(const float *Gt, float *G, int r, int accumulate, hipStream_t s);

// bf16 encode with whole-line plane stores (Cc >= 8); launch_encode picks it
// Its items: 64 columns of a row, of several rows, 64 tiles that follow each other in the planes, 64 columns from a cache line on
enum class EncodeItems { row, several_rows, flat, line_starts };
EncodeItems encode_items_of(int R, int Cc, int r, int pg, bool plain_rows);
hipError_t launch_encode_lines(const void *A, const void *E, void *P, int R, int Cc, int r, int pg, hipStream_t s, RowMap rm);

// out[i] = bf16(in[i]), round to nearest even
hipError_t launch_cast_bf16(const float *in, void *out, size_t n, hipStream_t s);

// inter-layer step of two stacked layers in one pass (bf16): Q[s] <- encode_{E2}( act( decode_{Dm}(P) ) ), planes P
// r1 x R x Cc -> planes Q r2 x R x Cc, the hidden activation never stored
bool recode_eligible(int dtype, int Cc);
hipError_t launch_recode(const void *P, const void *Dm, const void *E2, void *Q, int R, int Cc, int r1, int r2, bool gelu,
                         int pg, hipStream_t s);

// Batched plane products  Out[b][p][i][j] (+)= sum_l A[b][p](i,l) * B[b][p](l,j),  p < batch, b < nb, dense planes.
struct GemmDesc {
    int Mi, Nj, Kl;   // output rows, output columns, contraction length (all in tiles of the STL problem)
    int batch;        // number of planes r
    bool a_kmajor;    // false: A[p] stored [i][l] (l contiguous);  true: stored [l][i] (i contiguous)
    bool b_kmajor;    // true:  B[p] stored [l][j] (j contiguous);  false: stored [j][l] (l contiguous)
    bool out_f32;     // output stored as fp32 regardless of dtype (weight gradient)
    bool accumulate;  // Out += result (only with out_f32)
    // layout of each operand: rows per group (see plane_row_base), counted in the operand's stored rows -- i for A
    // stored [i][l], l for A stored [l][i], and so on; 0 = plane-major
    int a_pg = 0, b_pg = 0, o_pg = 0;
    // nb independent problems of this shape stacked along the stored rows of every operand: problem b owns stored rows
    // [b * rows, (b + 1) * rows) of A, B and Out (rows = the operand's stored row count for one problem)
    int nb = 1;
    int a_rows() const { return a_kmajor ? Kl : Mi; }
    int b_rows() const { return b_kmajor ? Kl : Nj; }
    int a_rows_per_group() const { return a_pg > 0 ? a_pg : nb * a_rows(); }
    int b_rows_per_group() const { return b_pg > 0 ? b_pg : nb * b_rows(); }
    int o_rows_per_group() const { return o_pg > 0 ? o_pg : nb * Mi; }
};

// Where the stored rows of one operand lie (see plane_row_base): row I of plane p begins at (I + (I >> shift) * skip) * ld + p * plane
// elements.  Groups have a power of two of rows, or there is one group (shift 31).
struct Lay {
    int ld, shift, skip;
    long plane;
    __device__ __forceinline__ long row(int I) const { return (long)(I + (I >> shift) * skip) * ld; }
    // an operand of `rows` stored rows per plane and `cols` columns in groups of pg rows (0: plane-major); false if it has more
    // than one group and they are no power of two
    bool set(int pg, long rows, int cols, int batch)
    {
        ld = cols;
        plane = (pg > 0 ? pg : rows) * cols;
        shift = 31;
        skip = 0;
        if (pg <= 0 || rows <= pg) return true;
        skip = (batch - 1) * pg;
        for (shift = 0; (1 << shift) < pg; ++shift) {}
        return (1 << shift) == pg && (double)rows * batch < 2147483648.0;
    }
};
struct GemmLays {
    Lay a, b, o;
    bool set(const GemmDesc &g)
    {
        return a.set(g.a_pg, (long)g.nb * g.a_rows(), g.a_kmajor ? g.Mi : g.Kl, g.batch) &&
               b.set(g.b_pg, (long)g.nb * g.b_rows(), g.b_kmajor ? g.Nj : g.Kl, g.batch) && o.set(g.o_pg, (long)g.nb * g.Mi, g.Nj, g.batch);
    }
};

// n / d for 0 <= n < 2^31, as one multiplication: mul = ceil(2^(31 + s) / d) with 2^s >= d, so that the error n (mul d - 2^(31 + s)) / d
// stays below 2^(31 + s) / d
struct Div {
    uint32_t mul, shift;
    __device__ __forceinline__ int of(int n) const { return (int)(((uint64_t)(uint32_t)n * mul) >> shift); }
    static Div by(int d)
    {
        uint32_t s = 0;
        while (((int64_t)1 << s) < d) ++s;
        return {(uint32_t)((((uint64_t)1 << (31 + s)) + d - 1) / d), 31 + s};
    }
};

hipError_t launch_plane_gemm(int dtype, const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s);
// two products that do not depend on each other, in one launch where there is a kernel for that (plane_gemm_paired), else one after the other
bool plane_gemm_paired(int dtype, const GemmDesc &g1, const GemmDesc &g2);
hipError_t launch_plane_gemm_pair(int dtype, const GemmDesc &g1, const void *A1, const void *B1, void *Out1, const GemmDesc &g2, const void *A2,
                                  const void *B2, void *Out2, hipStream_t s);
// the kernel that launch_plane_gemm takes: stl_gemm_rows.hip, stl_gemm_wide.hip, stl_gemm_pipe.hip, stl_gemm_mfma.hip, stl_gemm_generic.hip
enum class GemmPath { rows, wide, pipe, staged, generic };
GemmPath plane_gemm_path(int dtype, const GemmDesc &g);
// the any-shape path (fp32 MFMA), also used directly for fp32 storage
int generic_block(const GemmDesc &g);         // edge of the block of a plane that it takes
hipError_t launch_plane_gemm_generic(int dtype, const GemmDesc &g, const void *A, const void *B, void *Out,
                                     hipStream_t s);
// bf16 MFMA path, operands staged through registers (any width of at least 8)
bool plane_gemm_mfma_eligible(const GemmDesc &g);
int staged_block(const GemmDesc &g);          // edge of the block of a plane that it takes
int staged_groups(const GemmDesc &g);         // and, of 64 x 64 blocks, the groups of wavefronts that share the contraction (0: it is one stage)
hipError_t launch_plane_gemm_mfma(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s);
bool staged_pair_eligible(const GemmDesc &g1, const GemmDesc &g2);
hipError_t launch_staged_pair(const GemmDesc &g1, const void *A1, const void *B1, void *Out1, const GemmDesc &g2, const void *A2, const void *B2, void *Out2,
                              hipStream_t s);
// bf16 products of up to 32 rows
bool plane_gemm_rows_eligible(const GemmDesc &g);
int rows_columns(const GemmDesc &g);          // columns of the block of a plane that it takes
hipError_t launch_plane_gemm_rows(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s);
// bf16 MFMA path with LDS-DMA loads and a multi-stage LDS ring (contiguous dimensions a multiple of 8)
enum class PipeBlock { b256, b128x256, b128, b64 };
PipeBlock pipe_block(const GemmDesc &g);      // block of a plane that it takes
// What a persistent launch of 256 x 256 blocks does with those of its last round when they are fewer than its workgroups: whole
// (one each, the other workgroups idle), or in parts that are dealt to all of them
enum class PlaneSplit { none, b128x256, b128 };
PlaneSplit pipe_split(const GemmDesc &g);
bool plane_gemm_pipe_eligible(const GemmDesc &g);
bool pipe_pair_eligible(const GemmDesc &g1, const GemmDesc &g2);
hipError_t launch_pipe_pair(const GemmDesc &g1, const void *A1, const void *B1, void *Out1, const GemmDesc &g2, const void *A2, const void *B2, void *Out2,
                            hipStream_t s);
hipError_t launch_plane_gemm_pipe(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s);

// The whole forward pass as one persistent launch: encode and decode items run on some CUs while the plane products
// run on the others (bf16, r <= 32; see stl_pipeline.hip).  `counters` is forward_pipeline_counter_bytes(M) bytes of
// scratch (cleared by the launch itself).  Results are bit-identical to encode -> plane products -> decode.
bool forward_pipeline_eligible(int dtype, int M, int K, int N, int r);
size_t forward_pipeline_counter_bytes(int M);
hipError_t launch_forward_pipeline(const void *X, const void *E, const void *What, const void *Dm, void *Xhat, void *Yhat,
                                   void *C, void *counters, int M, int K, int N, int r, bool gelu, hipStream_t s);

// the same with the first ([row][l]) operand fetched as whole 128-byte lines (contraction a multiple of 64, one problem)
bool plane_gemm_wide_eligible(const GemmDesc &g);
hipError_t launch_plane_gemm_wide(const GemmDesc &g, const void *A, const void *B, void *Out, hipStream_t s);

// Forward on one output block with all planes resident (decode in the epilogue).  encode_in_kernel: Xin is X
// (single-launch fused form); otherwise Xin is Xhat.  Ysave may be NULL.  bf16 storage only.
bool block_forward_eligible(int dtype, int M, int K, int N, int r);
int block_forward_ring(bool encode, int M, int N, int r);      // LDS stages that its kernel takes
hipError_t launch_block_forward(bool encode_in_kernel, const void *Xin, const void *What, const void *E, const void *Dm,
                                void *C, void *Ysave, int M, int K, int N, int r, bool gelu, int pg, hipStream_t s);

// The single-launch form for few blocks, on 16 x 16 tiles each: whether it takes M x N output tiles (launch_block_forward picks it
// then).  round: the sums are rounded to the storage type before they are decoded, as three launches do.
bool small_forward(int M, int N, int r);
hipError_t launch_small_forward(const void *X, const void *What, const void *E, const void *Dm, void *C, void *Ysave, int M, int K, int N,
                                int r, bool gelu, bool round, int pg, hipStream_t s);

}  // namespace stl
