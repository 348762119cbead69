// vkt_stage.h -- staging of input planes, shared by the ApplyFilter kernels:
// each thread's 4-cell loads of a tile's rows with their halo, through the
// address mode.
#pragma once

#include "vkt_internal.h"

#include <type_traits>

namespace vkt {
namespace {

constexpr uint32_t kRsrcWord3 = 0x00020000u;  // gfx9-family raw buffer
constexpr uint32_t kOutside = 0x80000000u;    // byte offset that is dropped / reads 0

// Raw buffer loads: SGPR resource (base, size) + 32-bit VGPR byte offset.  An
// offset at or beyond the resource size reads 0 (used for border cells).
template <typename T>
__device__ inline T buf_load(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    if constexpr (sizeof(T) == 1) {
        return (T)__builtin_amdgcn_raw_buffer_load_b8(r, (int)off, 0, 0);
    } else if constexpr (sizeof(T) == 2) {
        return (T)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0);
    } else {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
    }
}

// Four consecutive cells at byte offset off (any cell alignment): one 4-, 8-
// or 16-byte load.
template <typename T>
__device__ inline void buf_load4(__amdgpu_buffer_rsrc_t r, uint32_t off, T (&v)[4])
{
    if constexpr (sizeof(T) == 1) {
        const uint32_t d = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = (T)(d >> (8 * j));
    } else if constexpr (sizeof(T) == 2) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 d = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
        v[0] = (T)d[0];
        v[1] = (T)(d[0] >> 16);
        v[2] = (T)d[1];
        v[3] = (T)(d[1] >> 16);
    } else {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 d = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = __uint_as_float(d[j]);
    }
}

// Four cells of a row at byte offset off of a plane (any cell alignment), or
// the first nx of them; offsets past the plane are dropped.
template <typename T>
__device__ inline void store4(__amdgpu_buffer_rsrc_t d, uint32_t off, const T (&r)[4], bool whole,
                              int nx)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    if (whole) {
        if constexpr (sizeof(T) == 1)
            __builtin_amdgcn_raw_buffer_store_b32((uint32_t)r[0] | (uint32_t)r[1] << 8 |
                                                      (uint32_t)r[2] << 16 | (uint32_t)r[3] << 24,
                                                  d, (int)off, 0, 0);
        else if constexpr (sizeof(T) == 2)
            __builtin_amdgcn_raw_buffer_store_b64(
                u32x2{(uint32_t)r[0] | (uint32_t)r[1] << 16, (uint32_t)r[2] | (uint32_t)r[3] << 16}, d,
                (int)off, 0, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b128(
                u32x4{__float_as_uint(r[0]), __float_as_uint(r[1]), __float_as_uint(r[2]),
                      __float_as_uint(r[3])},
                d, (int)off, 0, 0);
        return;
    }
    asm volatile("" : "+v"(off));  // (the cells' offsets are not kept over the z loop)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int o = i < nx ? (int)(off + sizeof(T) * i) : (int)kOutside;
        if constexpr (sizeof(T) == 1) __builtin_amdgcn_raw_buffer_store_b8(r[i], d, o, 0, 0);
        else if constexpr (sizeof(T) == 2) __builtin_amdgcn_raw_buffer_store_b16(r[i], d, o, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r[i]), d, o, 0, 0);
    }
}

// The planes of a volume, COLS x HY cells of each from
// (x0 - R, y0 - R), staged by NT threads four adjacent cells (a quad) at a
// time: one 4-cell load per quad and no branch around it.  Quads that reach
// past an x face of the volume are staged apart, NF of them per thread, by
// four cell loads through the address mode; only tiles at a face have any (a
// workgroup-uniform branch).  Quads that lie past X + R are not staged.  With
// the loads of a step fixed in number the compiler waits for exactly the plane
// it stages: with the face quads' cell loads in a divergent branch beside the
// others it put a memory latency into every plane step of a uint8 tile (302^3
// 5^3: 7000 cycles a step against 1536 of matrix products), and with single
// cell loads for all a tile pays four times the load and LDS instructions.
//
// Pos::at(row, column) is the place of a staged cell.
template <typename T, int R, int HY, int COLS, int NT, typename Pos>
struct PlaneStage {
    static_assert(COLS % 4 == 0, "quads inside rows");
    static constexpr int QR = COLS / 4, NQ = HY * QR;
    static constexpr int NE = (NQ + NT - 1) / NT;                // quads per thread
    static constexpr int MAXF = (R + 3) / 4 + (R + 2) / 4 + 1;   // face quads per row
    static constexpr int NF = (MAXF * HY + NT - 1) / NT;         // and per thread
    // face cells in whole registers, so that no load has to be waited for to
    // pack them
    using Tf = typename std::conditional<std::is_same<T, float>::value, float, uint32_t>::type;

    bool face;               // the tile reaches past an x face
    uint32_t goff[NE];       // byte offset of the quad's 4 cells in a plane
    // its place: where staged rows follow each other without a gap the places
    // are thread offsets and constants, apart from the last quad's
    static constexpr bool LINEAR = Pos::at(1, 0) == COLS && Pos::at(2, 0) == 2 * COLS;
    int qpos[LINEAR ? 2 : NE];
    __device__ inline int place(int i) const
    {
        if constexpr (LINEAR) return i + 1 < NE ? qpos[0] + 4 * NT * i : qpos[1];
        else return qpos[i];
    }
    uint32_t inner;          // bit i: quad i lies inside its row
    uint32_t foff[NF][4];    // byte offsets of the face quads' cells
    int fpos[NF];            // their places, -1: none
    T raw[NE][4];            // cells in flight
    Tf fraw[NF][4];

    __device__ __attribute__((always_inline)) inline void init(const VolDesc& a, int x0, int y0, int t)
    {
        const int xl = x0 - R;
        const int32_t plane_cells = a.X * a.Y;
        // staged columns up to the volume's right face, at most one quad past the
        // tile (X may be as large as 2^31 - 1: no sum of it and a width)
        const int cols = (int)min((uint32_t)a.X - (uint32_t)xl, (uint32_t)(COLS + 4));
        face = xl < 0 || cols < COLS;
        inner = 0;
        if constexpr (LINEAR) {
            qpos[0] = 4 * t;
            qpos[1] = 4 * min(t + (NE - 1) * NT, NQ - 1);
        }
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int e = min(t + i * NT, NQ - 1);  // repeats the last quad (same values)
            const int hy = e / QR, hx = 4 * (e % QR);
            if constexpr (!LINEAR) qpos[i] = Pos::at(hy, hx);
            const int gy = addr_map((int64_t)y0 - R + hy, a.Y, a.mode);
            // (a face quad's load stays inside the plane; it is not staged; a
            // row outside the volume under border mode reads 0; in planes of
            // fewer than 4 cells every quad is a face quad; columns past 2^31 - 1
            // wrap to negative ones: face quads as well)
            const int xs = (int)((uint32_t)xl + (uint32_t)hx);
            const int32_t cell = min((int32_t)((uint32_t)max(gy, 0) * (uint32_t)a.X +
                                               (uint32_t)max(xs, 0)),
                                     plane_cells - 4);
            goff[i] = gy < 0 || cell < 0 ? kOutside : (uint32_t)cell * (uint32_t)sizeof(T);
            if (xs >= 0 && xs < a.X - 3) inner |= 1u << i;
        }
#pragma unroll
        for (int i = 0; i < NF; ++i) fpos[i] = -1;
        if (face) {
            // quads with columns before cell 0, then those from the one that
            // holds column X to the one that holds column X + R - 1
            const int nl = xl < 0 ? min(QR, (-xl + 3) / 4) : 0;
            const int q1 = cols / 4, qr0 = max(nl, q1);
            const int ql = min(QR - 1, max(q1, (cols + R - 1) / 4));
            const int nf = nl + max(0, ql - qr0 + 1);
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const int j = t + i * NT;
                if (j >= nf * HY) continue;
                const int hy = j / nf, f = j - hy * nf;
                const int qx = f < nl ? f : qr0 + f - nl;
                const int gy = addr_map((int64_t)y0 - R + hy, a.Y, a.mode);
                fpos[i] = Pos::at(hy, 4 * qx);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int gx = addr_map((int64_t)xl + 4 * qx + c, a.X, a.mode);
                    foff[i][c] = (gx < 0 || gy < 0) ? kOutside
                                                    : ((uint32_t)gy * (uint32_t)a.X + (uint32_t)gx) *
                                                          (uint32_t)sizeof(T);
                }
            }
        }
    }

    // Issues the loads of input plane zi.
    __device__ __attribute__((always_inline)) inline void gather(const VolDesc& a, int zi)
    {
        const int32_t plane_bytes = (int32_t)((int64_t)a.X * a.Y * (int64_t)sizeof(T));  // < 2^31
        const int gz = addr_map(zi, a.Z, a.mode);  // -1 only for border: a zero plane
        const char* base = static_cast<const char*>(a.src) +
                           (gz < 0 ? 0 : (int64_t)gz * plane_bytes);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(base), (short)0, gz < 0 ? 0 : plane_bytes, (int)kRsrcWord3);
#pragma unroll
        for (int i = 0; i < NE; ++i) buf_load4<T>(rs, goff[i], raw[i]);
        if (face) {
#pragma unroll
            for (int i = 0; i < NF; ++i)
                if (fpos[i] >= 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) fraw[i][c] = (Tf)buf_load<T>(rs, foff[i][c]);
                }
        }
    }

    // emit(cells, place, on) for every quad of the plane in flight; a quad
    // with on = false is not staged.
    template <typename F>
    __device__ __attribute__((always_inline)) inline void put(F&& emit)
    {
        if (!face) {
#pragma unroll
            for (int i = 0; i < NE; ++i) emit(raw[i], place(i), true);
            return;
        }
#pragma unroll
        for (int i = 0; i < NE; ++i) emit(raw[i], place(i), ((inner >> i) & 1u) != 0);
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const T v[4] = {(T)fraw[i][0], (T)fraw[i][1], (T)fraw[i][2], (T)fraw[i][3]};
            emit(v, fpos[i], fpos[i] >= 0);
        }
    }
};

}  // namespace
}  // namespace vkt
