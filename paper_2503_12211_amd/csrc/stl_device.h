// Device-side helpers shared by the STL kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace stl {

typedef uint16_t bf16_t;  // raw bfloat16 bits in memory

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// fp32 -> bf16, round-to-nearest-even (NaN stays NaN): gfx950 has a packed hardware conversion
// (v_cvt_pk_bf16_f32), which the compiler selects for this vector conversion.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    const f32x2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack_bf16x2(f, 0.f) & 0xffffu); }

// 16-byte store that is written through the XCD's L2 to memory (cache-coherence bits sc0 sc1: system scope), for data that
// workgroups on another XCD read later in the same launch: when the store has completed (vmcnt) the data is where every
// L2 fetches from, with no write-back of the whole cache.  THROUGH = false is the ordinary store.
template <bool THROUGH>
__device__ __forceinline__ void store16(void *p, u32x4_t v)
{
    if constexpr (THROUGH) {
        // a wide store's data registers may be overwritten one wait state after it at the earliest (the compiler does
        // not look into the statement)
        asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 0" ::"v"(p), "v"(v) : "memory");
    } else {
        *reinterpret_cast<u32x4_t *>(p) = v;
    }
}

// Eight bf16 of a plane row, n of them left in the row from p on (n <= 0: none).  ANY = false: rows are whole 16-byte chunks
// (column count a multiple of 8, n then too).  ANY = true: any column count of at least 8, so that a row starts at any
// even address and its last chunk may be incomplete; gfx950 loads and stores 16 bytes at any address, and such a chunk is
// read as the eight elements that end with the row, shifted down (zeros move in), and written in pieces of 4, 2 and 1.
typedef u32x4_t u32x4_any_t __attribute__((aligned(2)));
typedef u32x2_t u32x2_any_t __attribute__((aligned(2)));
typedef uint32_t u32_any_t __attribute__((aligned(2)));

// eight elements moved h places towards the first, 0 < h < 8, zeros behind them
__device__ __forceinline__ u32x4_t shift_down(u32x4_t v, int h)
{
    uint64_t lo = v[0] | ((uint64_t)v[1] << 32), hi = v[2] | ((uint64_t)v[3] << 32);
    const int sh = 16 * h;                                   // 16 ... 112
    lo = sh < 64 ? (lo >> (sh & 63)) | (hi << ((64 - sh) & 63)) : hi >> (sh & 63);
    hi = sh < 64 ? hi >> (sh & 63) : 0;
    return u32x4_t{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

template <bool ANY>
__device__ __forceinline__ u32x4_t load8(const bf16_t *p, int n)
{
    u32x4_t v = {0u, 0u, 0u, 0u};
    if constexpr (!ANY) {
        if (n > 0) v = *reinterpret_cast<const u32x4_t *>(p);
    } else {
        const int miss = n < 8 ? 8 - n : 0;                  // elements of the chunk beyond the row's end
        if (n > 0) v = *reinterpret_cast<const u32x4_any_t *>(p - miss);
        if (n > 0 && miss) v = shift_down(v, miss);
    }
    return v;
}

template <bool ANY>
__device__ __forceinline__ void store8(bf16_t *p, int n, u32x4_t v)
{
    if constexpr (!ANY) {
        if (n > 0) *reinterpret_cast<u32x4_t *>(p) = v;
    } else if (n >= 8) {
        *reinterpret_cast<u32x4_any_t *>(p) = v;
    } else if (n > 0) {
        if (n & 4) {
            *reinterpret_cast<u32x2_any_t *>(p) = u32x2_t{v[0], v[1]};
            p += 4;
            v[0] = v[2];
            v[1] = v[3];
        }
        if (n & 2) {
            *reinterpret_cast<u32_any_t *>(p) = v[0];
            p += 2;
            v[0] = v[1];
        }
        if (n & 1) *p = (bf16_t)(v[0] & 0xffffu);
    }
}

// elements h .. min(n, 8) - 1 of the chunk at p, which may begin before its row (h > 0)
__device__ __forceinline__ void store8_between(bf16_t *p, int h, int n, u32x4_t v)
{
    if (h >= 8) return;
    if (h > 0) v = shift_down(v, h);
    store8<true>(p + h, (h > 0 && n > 8 ? 8 : n) - h, v);
}

// storage-type traits: load as fp32, store from fp32
template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float ld(const float *p) { return *p; }
    static __device__ __forceinline__ void st(float *p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
    static __device__ __forceinline__ float ld(const bf16_t *p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void st(bf16_t *p, float v) { *p = f32_to_bf16(v); }
};

// Four consecutive elements as fp32, n of them left in the row from p on (zeros for the others); p at any element.
typedef f32x4_t f32x4_any_t __attribute__((aligned(4)));

template <typename T>
__device__ __forceinline__ f32x4_t load4(const T *p, int n)
{
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    if (n >= 4) {
        if constexpr (sizeof(T) == 4) {
            v = *reinterpret_cast<const f32x4_any_t *>(p);
        } else {
            const u32x2_t w = *reinterpret_cast<const u32x2_any_t *>(p);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = bf16_to_f32((bf16_t)(w[e >> 1] >> (16 * (e & 1))));
        }
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < n) v[e] = Elem<T>::ld(p + e);
    }
    return v;
}

// Eight consecutive plane elements on their way from memory to LDS as bf16: held as loaded, so that a prefetch does not wait
// for its data, and rounded (fp32 planes) when they are taken.
template <typename T, bool ANY>
struct Raw8 {
    u32x4_t v;
    __device__ __forceinline__ void load(const T *p, int n) { v = load8<ANY>(p, n); }
    __device__ __forceinline__ u32x4_t take() const { return v; }
};
template <bool ANY>
struct Raw8<float, ANY> {
    f32x4_t a, b;
    __device__ __forceinline__ void load(const float *p, int n)
    {
        if constexpr (ANY) {
            a = load4<float>(p, n);
            b = load4<float>(p + 4, n - 4);
        } else {
            a = b = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (n > 0) {
                a = *reinterpret_cast<const f32x4_t *>(p);
                b = *reinterpret_cast<const f32x4_t *>(p + 4);
            }
        }
    }
    __device__ __forceinline__ u32x4_t take() const
    {
        return u32x4_t{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3])};
    }
};

// one row of a tile (4 elements, aligned to their size)
__device__ __forceinline__ void store4(float *p, f32x4_t v) { *reinterpret_cast<f32x4_t *>(p) = v; }
__device__ __forceinline__ void store4(bf16_t *p, f32x4_t v)
{
    *reinterpret_cast<u32x2_t *>(p) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}

// Plane tensors [p][tile row][tile column] are stored in groups of `pg` tile rows: element (p, I, J) of an
// r x R x Cc tensor lives at ((I / pg) * r + p) * pg * Cc + (I % pg) * Cc + J.  pg = R is the plain plane-major
// layout (weights and their gradients); the activation-side tensors use groups of 64 tile rows, which keeps the r
// segments belonging to one tile row within r * 64 * Cc elements of each other instead of a whole plane apart
// (the kernels that walk over all planes of a tile row run a fifth faster on it) and still leaves 64 consecutive
// rows of a plane contiguous for the plane products.  Inside a group the distance between planes is pg * Cc.
__host__ __device__ __forceinline__ size_t plane_row_base(int I, int pg, int r, int Cc)
{
    const int g = I / pg;
    return ((size_t)g * r * pg + (size_t)(I - g * pg)) * Cc;
}

// erf-form GELU in fp32, h * Phi(h), branch-free.  Phi(h) = erfc(-h / sqrt 2) / 2 with the rational-exponential
// approximation of Abramowitz & Stegun 7.1.26,  erfc(x) ~ (a1 s + ... + a5 s^5) exp(-x^2),  s = 1 / (1 + p x),  x >= 0,
// whose absolute error is below 1.5e-7 (the library erff costs about three times the instructions and diverges on
// |x| < 1, which made the GELU the bottleneck of the HBM-bound decode kernels).  |gelu error| <= 7.5e-8 |h|.
__device__ __forceinline__ float gelu_erf(float h)
{
    const float x = fabsf(h) * 0.70710678118654752440f;
    const float s = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
    float poly = fmaf(s, 1.061405429f, -1.453152027f);
    poly = fmaf(poly, s, 1.421413741f);
    poly = fmaf(poly, s, -0.284496736f);
    poly = fmaf(poly, s, 0.254829592f);
    const float half_erfc = 0.5f * poly * s * __builtin_amdgcn_exp2f(-1.44269504088896340736f * x * x);
    return h * (h < 0.f ? half_erfc : 1.0f - half_erfc);
}

}  // namespace stl
