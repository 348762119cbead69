// vkt_mfma_common.h -- pieces shared by the matrix-core ApplyFilter kernels
// (vkt_filter_mfma.hip, vkt_filter_mfma_rp.hip): operand splitting into
// 16-bit pieces, address modes, buffer loads and the output store.
//
// Split precision (16-bit operands, exact FP32 products, FP32 sums):
//   uint8   voxels: exact in fp16 (1 piece) x weights in 2 fp16 pieces;
//   uint16  voxels: hi byte * 256 and lo byte, both exact in fp16 (2 pieces)
//                   x 2 fp16 weight pieces (4 products);
//   float32 voxels: 2 (or 3) bf16 pieces x 2 (or 3) bf16 weight pieces, the
//                   products whose piece orders sum to <= 1 (3 products) or
//                   <= 2 (6 products).
// fp16 weight pieces are taken of w * 2^s, 2^s chosen on the host so that the
// largest |w| lands in [2^14, 2^15); the result is scaled back by 2^-s.
#pragma once

#include "vkt_stage.h"

#include <type_traits>

namespace vkt {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kNT = 256;                     // threads per workgroup (4 waves)

// Operand pieces and the products kept.
enum PieceMode { kU8 = 0, kU16 = 1, kF32x3 = 2, kF32x6 = 3 };
template <int PM> struct Pieces;
template <> struct Pieces<kU8> {
    static constexpr bool F16 = true;
    static constexpr int PS = 1, NBI = 2, NPROD = 2;
    static constexpr int prod[NPROD][2] = {{0, 0}, {0, 1}};
};
template <> struct Pieces<kU16> {
    static constexpr bool F16 = true;
    static constexpr int PS = 2, NBI = 2, NPROD = 4;
    static constexpr int prod[NPROD][2] = {{0, 0}, {0, 1}, {1, 0}, {1, 1}};
};
template <> struct Pieces<kF32x3> {
    static constexpr bool F16 = false;
    static constexpr int PS = 2, NBI = 2, NPROD = 3;
    static constexpr int prod[NPROD][2] = {{0, 0}, {0, 1}, {1, 0}};
};
template <> struct Pieces<kF32x6> {
    static constexpr bool F16 = false;
    static constexpr int PS = 3, NBI = 3, NPROD = 6;
    static constexpr int prod[NPROD][2] = {{0, 0}, {0, 1}, {1, 0}, {0, 2}, {1, 1}, {2, 0}};
};

__device__ inline uint32_t xcd_remap(uint32_t b, uint32_t n)
{
    const uint32_t q = n / 8, rem = n % 8, xcd = b % 8, idx = b / 8;
    return xcd < rem ? xcd * (q + 1) + idx : rem * (q + 1) + (xcd - rem) * q + idx;
}

__device__ inline uint16_t f16_bits(float x) { return __builtin_bit_cast(uint16_t, (_Float16)x); }
__device__ inline float f16_val(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
__device__ inline uint16_t bf16_bits(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
__device__ inline float bf16_val(uint16_t h) { return (float)__builtin_bit_cast(__bf16, h); }

// Split one voxel into its 16-bit pieces (bit patterns).
template <int PM, typename T>
__device__ inline void split_voxel(T s, uint16_t* p)
{
    if constexpr (PM == kU8) {
        p[0] = f16_bits((float)s);
    } else if constexpr (PM == kU16) {
        const uint32_t v = s;
        p[0] = f16_bits((float)((v >> 8) << 8));  // multiple of 256 below 2^16: exact
        p[1] = f16_bits((float)(v & 255u));
    } else {
        const float x = (float)s;
        p[0] = bf16_bits(x);
        const float r1 = x - bf16_val(p[0]);
        p[1] = bf16_bits(r1);
        if constexpr (PM == kF32x6) p[2] = bf16_bits(r1 - bf16_val(p[1]));
    }
}

// Pieces of two adjacent cells, packed as the dword pairs they are staged as
// (cell 0 in the low half): the pieces of split_voxel, converted two at a
// time (one v_cvt_pk per pair; cells and their uint16 halves are exact in
// fp16, so that the round-toward-zero packing changes nothing).
template <int PM, typename T>
__device__ inline void split_pair(T s0, T s1, uint32_t* pk)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    if constexpr (PM == kF32x3 || PM == kF32x6) {
        const float x0 = (float)s0, x1 = (float)s1;
        const uint32_t hu =
            __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x0, x1}), bf16x2));
        const float r0 = x0 - __uint_as_float(hu << 16), r1 = x1 - __uint_as_float(hu & 0xffff0000u);
        const uint32_t lu =
            __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{r0, r1}), bf16x2));
        pk[0] = hu;
        pk[1] = lu;
        if constexpr (PM == kF32x6) {
            const float t0 = r0 - __uint_as_float(lu << 16), t1 = r1 - __uint_as_float(lu & 0xffff0000u);
            pk[2] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{t0, t1}), bf16x2));
        }
    } else if constexpr (PM == kU16) {
        const uint32_t v0 = s0, v1 = s1;
        pk[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz((float)(v0 & 0xff00u),
                                                                        (float)(v1 & 0xff00u)));
        pk[1] = __builtin_bit_cast(uint32_t,
                                   __builtin_amdgcn_cvt_pkrtz((float)(v0 & 255u), (float)(v1 & 255u)));
    } else {
        pk[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz((float)s0, (float)s1));
    }
}

// Stages four cells' pieces at plane[piece][e], one 8-byte write a piece
// (none if !on).
template <int PM, typename T, int PLANE>
__device__ __attribute__((always_inline)) inline void stage_quad(uint16_t (*plane)[PLANE], const T (&v)[4],
                                                                 int e, bool on)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    uint32_t p01[3], p23[3];
    split_pair<PM>(v[0], v[1], p01);
    split_pair<PM>(v[2], v[3], p23);
    if (on) {
#pragma unroll
        for (int ps = 0; ps < Pieces<PM>::PS; ++ps)
            *reinterpret_cast<u32x2*>(&plane[ps][e]) = u32x2{p01[ps], p23[ps]};
    }
}

// Split one weight into NBI pieces.
template <int PM>
__device__ inline void split_weight(float w, float scale, uint16_t* p)
{
    if constexpr (Pieces<PM>::F16) {
        const float x = w * scale;  // exact (power of two)
        p[0] = f16_bits(x);
        p[1] = f16_bits(x - f16_val(p[0]));
    } else {
        p[0] = bf16_bits(w);
        const float r1 = w - bf16_val(p[0]);
        p[1] = bf16_bits(r1);
        if constexpr (PM == kF32x6) p[2] = bf16_bits(r1 - bf16_val(p[1]));
    }
}

// W consecutive dwords at byte offset off, in as few stores as there are.
template <int W>
__device__ inline void store_dwords(__amdgpu_buffer_rsrc_t r, uint32_t off, const uint32_t (&u)[W])
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
    constexpr int Q = W / 4;
#pragma unroll
    for (int h = 0; h < Q; ++h)
        __builtin_amdgcn_raw_buffer_store_b128(
            u32x4{u[4 * h], u[4 * h + 1], u[4 * h + 2], u[4 * h + 3]}, r, (int)off + 16 * h, 0, 0);
    if constexpr (W % 4 == 3)
        __builtin_amdgcn_raw_buffer_store_b96(u32x3{u[4 * Q], u[4 * Q + 1], u[4 * Q + 2]}, r,
                                              (int)off + 16 * Q, 0, 0);
    else if constexpr (W % 4 == 2)
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{u[4 * Q], u[4 * Q + 1]}, r, (int)off + 16 * Q, 0,
                                              0);
    else if constexpr (W % 4 == 1)
        __builtin_amdgcn_raw_buffer_store_b32(u[4 * Q], r, (int)off + 16 * Q, 0, 0);
}

// The first nx (any number) of N stored cells at byte offset off, four at a
// time where they are whole.
template <typename T, int N>
__device__ inline void store_part(__amdgpu_buffer_rsrc_t r, uint32_t off, const uint32_t (&u)[N],
                                  int nx)
{
    asm volatile("" : "+v"(off));  // (the cells' offsets are not kept over the z loop)
    constexpr int CPD = 4 / sizeof(T);
#pragma unroll
    for (int g = 0; g < N; g += 4) {
        if (g + 4 <= N && g + 4 <= nx) {
            uint32_t d[4 / CPD];
#pragma unroll
            for (int i = 0; i < 4 / CPD; ++i) {
                d[i] = u[g + CPD * i];
#pragma unroll
                for (int c = 1; c < CPD; ++c) d[i] |= u[g + CPD * i + c] << (8 * sizeof(T) * c);
            }
            store_dwords<4 / CPD>(r, off + (uint32_t)sizeof(T) * g, d);
        } else if (g < nx) {
#pragma unroll
            for (int i = g; i < g + 4 && i < N; ++i) {
                const int o = i < nx ? (int)(off + sizeof(T) * i) : (int)kOutside;
                if constexpr (sizeof(T) == 4)
                    __builtin_amdgcn_raw_buffer_store_b32(u[i], r, o, 0, 0);
                else if constexpr (sizeof(T) == 2)
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)u[i], r, o, 0, 0);
                else
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)u[i], r, o, 0, 0);
            }
        }
    }
}

// Round (integer cells) and store one lane's row of N finished outputs at
// byte offset off: vector stores when the row lies inside the volume (buffer
// stores take any cell alignment), else cell stores for the first nx cells.
// Dropped rows carry an out-of-range offset.
template <typename T, int N>
__device__ inline void store_row(__amdgpu_buffer_rsrc_t r, uint32_t off, const float (&v)[N],
                                 bool vec, int nx, float unscale)
{
    uint32_t u[N];
    if constexpr (std::is_same<T, float>::value) {
#pragma unroll
        for (int i = 0; i < N; ++i) u[i] = __float_as_uint(v[i] * unscale);
    } else {
        constexpr float kMax = std::is_same<T, uint8_t>::value ? 255.f : 65535.f;
#pragma unroll
        for (int i = 0; i < N; ++i)
            // floor(q + 1/2) saturated: truncation of a value clamped to [0, max]
            u[i] = (uint32_t)__builtin_amdgcn_fmed3f(fmaf(v[i], unscale, 0.5f), 0.f, kMax);
    }
    if (vec) {
        constexpr int CPD = 4 / sizeof(T);  // cells per dword
        constexpr int W = N / CPD, REST = N % CPD;
        if constexpr (W > 0) {
            uint32_t d[W];
#pragma unroll
            for (int i = 0; i < W; ++i) {
                d[i] = u[CPD * i];
#pragma unroll
                for (int c = 1; c < CPD; ++c) d[i] |= u[CPD * i + c] << (8 * sizeof(T) * c);
            }
            store_dwords<W>(r, off, d);
        }
        const int o = (int)off + 4 * W;
        if constexpr (sizeof(T) == 2 && REST == 1)
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)u[CPD * W], r, o, 0, 0);
        if constexpr (sizeof(T) == 1 && REST >= 2)
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(u[CPD * W] | (u[CPD * W + 1] << 8)), r, o,
                                                  0, 0);
        if constexpr (sizeof(T) == 1 && REST % 2 == 1)
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)u[N - 1], r, o + (REST & 2), 0, 0);
    } else {
        store_part<T>(r, off, u, nx);
    }
}

}  // namespace
}  // namespace vkt
