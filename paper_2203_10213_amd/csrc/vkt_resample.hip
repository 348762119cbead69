// vkt_resample.hip -- Resample (trilinear, cell-centred) and Flip of
// structured volumes.
//
// Paper Sec. 3.2: Resample is a core algorithm that changes the size of a
// volume; Flip is a transform algorithm that mirrors it.  Sec. 4 benchmarks
// both on the structured volumes: a downscale by two on every axis, and a
// flip along the axis of the longest extent.
//
// Resample: destination cell i on an axis of n source and m destination
// cells samples the source at u = (i + 1/2) n / m - 1/2 (cell centres),
// trilinear between the two neighbouring cells, neighbours clamped to the
// volume; integer formats round half-up and saturate.  The position is
// split exactly in integer arithmetic into its cell and its fraction, which
// is rounded once to FP32; the interpolation runs in FP32.  An exact factor of two
// on every axis takes a dedicated path: the mean of each 2 x 2 x 2 block
// (integer formats: (sum + 4) >> 3, exact).
// Flip: dst(x) = src(n - 1 - x) along one axis; in place (dst == src) the
// first half along the axis swaps with the mirrored half.
//
// All are HBM-bound streams at best.  The halving and flip kernels move 16
// bytes per thread at any cell alignment (rows that are not whole 16-byte
// chunks end in a chunk moved back to the row's end); items are numbered
// through rows and planes and taken apart with multiplications.
#include "vkt_internal.h"

#include <algorithm>
#include <type_traits>

namespace vkt {
namespace {

constexpr int kNT = 256;

// Items of the rows [y0, y0 + ny) x [z0, z0 + nz) of a volume, `items` per
// row, numbered through; one thread each.
struct RowBox {
    int32_t y0, z0, ny;
    uint32_t total;          // items in the box (below 2^31)
    int32_t items;
    UDiv per_row, per_plane;  // by items, by ny
};

__device__ inline uint32_t udiv(uint32_t n, UDiv d)
{
    const uint32_t t = __umulhi(d.m, n);
    return (t + ((n - t) >> d.sh1)) >> d.sh2;
}

// This thread's item: false past the last one.
__device__ inline bool row_item(const RowBox& b, int& c, int& y, int& z)
{
    const uint32_t i = blockIdx.x * (uint32_t)kNT + threadIdx.x;
    if (i >= b.total) return false;
    const uint32_t row = udiv(i, b.per_row), zr = udiv(row, b.per_plane);
    c = (int)(i - row * (uint32_t)b.items);
    y = b.y0 + (int)(row - zr * (uint32_t)b.ny);
    z = b.z0 + (int)zr;
    return true;
}

// launch(box, blocks) for boxes that cover Ys x Zs rows.
template <typename F>
hipError_t for_row_boxes(int Ys, int Zs, int items, F&& launch)
{
    RowBox b{};
    b.items = items;
    b.per_row = make_udiv((uint32_t)items);
    const int64_t most = (((int64_t)1 << 31) - 1) / items;
    const int ny = (int)std::min<int64_t>(Ys, std::max<int64_t>(1, most));
    const int nz = ny < Ys ? 1 : (int)std::min<int64_t>(Zs, std::max<int64_t>(1, most / Ys));
    for (int z0 = 0; z0 < Zs; z0 += std::min(nz, Zs - z0))
        for (int y0 = 0; y0 < Ys; y0 += std::min(ny, Ys - y0)) {
            b.y0 = y0;
            b.z0 = z0;
            b.ny = std::min(ny, Ys - y0);
            b.per_plane = make_udiv((uint32_t)b.ny);
            b.total = (uint32_t)((int64_t)items * b.ny * std::min(nz, Zs - z0));
            launch(b, dim3((b.total + kNT - 1) / kNT));
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

struct RowGrid {
    dim3 grid, block;
};

// Blocks of 256 threads: x covers `per_row` items (power of two, <= 256),
// y covers rows; the grid covers the rows once (capped; kernels loop).
RowGrid row_grid(int64_t per_row, int64_t nrows)
{
    int bx = 1;
    while (bx < per_row && bx < kNT) bx *= 2;
    const int by = kNT / bx;
    const int64_t gx = (per_row + bx - 1) / bx;
    int64_t gy = (nrows + by - 1) / by;
    if (gy > 65535) gy = 65535;
    if (gy < 1) gy = 1;
    return {dim3((unsigned)gx, (unsigned)gy), dim3((unsigned)bx, (unsigned)by)};
}

template <typename T>
__device__ inline T from_f(float v)
{
    if constexpr (std::is_same<T, float>::value) {
        return v;
    } else {
        constexpr float kMax = std::is_same<T, uint8_t>::value ? 255.f : 65535.f;
        // floor(v + 1/2) saturated: truncation of v + 1/2 clamped to [0, max]
        return (T)(uint32_t)__builtin_amdgcn_fmed3f(v + 0.5f, 0.f, kMax);
    }
}

// Lower and upper neighbour (clamped) and the weight of the upper one for
// destination cell i of m on an axis of n source cells.  The sample position
// u = (i + 1/2) n / m - 1/2 = ((2i + 1) n - m) / (2m) is split exactly in
// integers: with N = (2i + 1) n + m >= 0 (the numerator plus one
// denominator) and D = 2m, floor(u) = N / D - 1 and the fraction is
// (N mod D) / D, rounded once to FP32.  (32-bit division whenever N fits.)
__device__ inline void lin_axis(int i, int n, int m, int& i0, int& i1, float& f)
{
    const uint64_t N = (uint64_t)(2 * (int64_t)i + 1) * (uint64_t)n + (uint64_t)m;
    const uint64_t D = 2 * (uint64_t)m;
    uint64_t q, rem;
    if (N <= 0xffffffffull && D <= 0xffffffffull) {
        const uint32_t n32 = (uint32_t)N, d32 = (uint32_t)D;
        q = n32 / d32;
        rem = n32 - (uint32_t)q * d32;
    } else {
        q = N / D;
        rem = N - q * D;
    }
    f = (float)rem / (float)D;
    const int64_t a = (int64_t)q - 1;
    i0 = (int)min(max(a, (int64_t)0), (int64_t)n - 1);
    i1 = (int)min(max(a + 1, (int64_t)0), (int64_t)n - 1);
}

__device__ inline float lerp(float a, float b, float t) { return a + t * (b - a); }

// 16 bytes at any cell alignment; loads are read once (streamed past the
// caches' reuse sets).
typedef uint32_t chunk16 __attribute__((ext_vector_type(4), aligned(1)));
__device__ inline uint4 load_stream(const void* p)
{
    const chunk16 v = __builtin_nontemporal_load(static_cast<const chunk16*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ inline void store16(void* p, uint4 v)
{
    *static_cast<chunk16*>(p) = chunk16{v.x, v.y, v.z, v.w};
}

// ---- general trilinear resampling ------------------------------------------
// A thread takes 4 adjacent destination cells of a row (the groups of all rows
// numbered through, so that no lane idles) and marches through up to kZC
// destination planes, fewer where the volume would not fill the device.  Per source plane it needs, a lane
// loads the cell pairs (x0, x0 + 1) of its two source rows -- in the plane at
// one uniform address and a 32-bit offset kept over the march -- interpolates
// them along x and y, and keeps the result while further destination planes
// lie between the same source planes.  The sums are those of one cell at a
// time (x, then y, then z).  What bounded the one-cell-per-thread form (302^3
// uint8 to 403^3: 401 us, 93 MB) were some 300 instructions a cell, most of
// them the integer divisions of its three positions; here x and y positions
// are worked out once per march and z positions once per workgroup (LDS), and
// the same call takes 52 us at some 22 vector instructions a cell, which bound it
// (the vector ALUs 63 % busy).
constexpr int kZC = 32;   // destination planes per march at most
constexpr int kXV = 4;    // adjacent destination cells per thread

struct ZPos {
    int z0, z1;
    float f;
    int pad;
};

// Two adjacent cells at byte offset off of a plane (any cell alignment).
template <typename T>
__device__ inline void load_pair(__amdgpu_buffer_rsrc_t r, uint32_t off, float& lo, float& hi)
{
    if constexpr (std::is_same<T, float>::value) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
        lo = __uint_as_float(v[0]);
        hi = __uint_as_float(v[1]);
    } else if constexpr (std::is_same<T, uint16_t>::value) {
        const uint32_t v = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
        lo = (float)(v & 0xffffu);
        hi = (float)(v >> 16);
    } else {
        const uint32_t v = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0);
        lo = (float)(v & 0xffu);
        hi = (float)(v >> 8);
    }
}

// WIDE (uint8 cells, source at most twice the destination along x, planes of at
// least 8 cells): a thread's four pairs lie in 8 adjacent cells, which one
// load brings; v_perm picks the pairs (302^3 to 403^3: 52 us instead of 70).
template <typename T, bool WIDE>
__global__ __launch_bounds__(kNT) void resample_kernel(const T* __restrict__ src,
                                                       T* __restrict__ dst, int X, int Y, int Z,
                                                       int Xo, int Yo, int Zo, int zc,
                                                       uint32_t groups, UDiv per_row)
{
    __shared__ ZPos zpos[kZC];
    const int t = threadIdx.x;
    const int zb = (int)blockIdx.y * zc, nz = min(zc, Zo - zb);
    if (t < nz) {
        ZPos p{};
        lin_axis(zb + t, Z, Zo, p.z0, p.z1, p.f);
        zpos[t] = p;
    }
    __syncthreads();
    const uint32_t item = blockIdx.x * (uint32_t)kNT + (uint32_t)t;
    const uint32_t row = udiv(item, per_row);
    const int y = (int)row, x = (int)(item - row * groups) * kXV;
    if (y >= Yo) return;
    int y0, y1;
    float fy;
    lin_axis(y, Y, Yo, y0, y1, fy);
    // pairs start at xb <= X - 2; a clamped position (x0 == x1) takes one of
    // the pair's cells: float32 both times, integer cells, which cannot
    // overflow, at the fraction 0 or 1 (the same value exactly)
    uint32_t off[2][kXV];
    float fx[kXV];
    uint32_t low2 = 0, high2 = 0;  // bit j: both cells are the pair's first / second
#pragma unroll
    for (int j = 0; j < kXV; ++j) {
        int x0, x1;
        lin_axis(min(x + j, Xo - 1), X, Xo, x0, x1, fx[j]);
        const int xb = min(x0, X - 2);
        if constexpr (std::is_same<T, float>::value) {
            if (x1 == xb) low2 |= 1u << j;
            if (x0 != xb) high2 |= 1u << j;
        } else {
            if (x1 == xb) fx[j] = 0.f;
            if (x0 != xb) fx[j] = 1.f;
        }
        off[0][j] = ((uint32_t)y0 * (uint32_t)X + (uint32_t)xb) * (uint32_t)sizeof(T);
        off[1][j] = ((uint32_t)y1 * (uint32_t)X + (uint32_t)xb) * (uint32_t)sizeof(T);
    }
    uint32_t wide[2] = {};  // WIDE: the 8 cells' offset; off[][] then holds byte selectors
    if constexpr (WIDE) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            wide[r] = min(off[r][0], (uint32_t)X * (uint32_t)Y - 8u);  // inside the plane
#pragma unroll
            for (int j = 0; j < kXV; ++j) {
                const uint32_t d = off[r][j] - wide[r];
                off[r][j] = d | (d + 1u) << 8 | 0x0c0c0000u;
            }
        }
    }
    const int64_t plane = (int64_t)X * Y, oplane = (int64_t)Xo * Yo;
    // rows of one source plane interpolated along x, then y
    auto at_plane = [&](int z, float (&v)[kXV]) {
        const __amdgpu_buffer_rsrc_t p = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(src + z * plane), (short)0, (int)(uint32_t)(plane * (int64_t)sizeof(T)),
            0x00020000);
        float lo[2][kXV], hi[2][kXV];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int j = 0; j < kXV; ++j)
                if constexpr (!WIDE) load_pair<T>(p, off[r][j], lo[r][j], hi[r][j]);
        if constexpr (WIDE) {
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            u32x2 w[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) w[r] = __builtin_amdgcn_raw_buffer_load_b64(p, (int)wide[r], 0, 0);
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int j = 0; j < kXV; ++j) {
                    const uint32_t v = __builtin_amdgcn_perm(w[r][1], w[r][0], off[r][j]);
                    lo[r][j] = (float)(v & 0xffu);
                    hi[r][j] = (float)((v >> 8) & 0xffu);
                }
        }
#pragma unroll
        for (int j = 0; j < kXV; ++j) {
            float a[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float c0 = (high2 >> j) & 1u ? hi[r][j] : lo[r][j];
                const float c1 = (low2 >> j) & 1u ? lo[r][j] : hi[r][j];
                a[r] = lerp(c0, c1, fx[j]);
            }
            v[j] = lerp(a[0], a[1], fy);
        }
    };
    T* out = dst + zb * oplane + (int64_t)y * Xo + x;
    const bool whole = x <= Xo - kXV;  // (x + kXV may be 2^31)
    int have0 = -1, have1 = -1;  // source planes whose values are at hand
    float v0[kXV] = {}, v1[kXV] = {};
    for (int i = 0; i < nz; ++i, out += oplane) {
        const int z0 = __builtin_amdgcn_readfirstlane(zpos[i].z0);
        const int z1 = __builtin_amdgcn_readfirstlane(zpos[i].z1);
        const float fz = zpos[i].f;
        if (z0 != have0) {
            if (z0 == have1) {
#pragma unroll
                for (int j = 0; j < kXV; ++j) v0[j] = v1[j];
            } else {
                at_plane(z0, v0);
            }
            have0 = z0;
        }
        if (z1 != have1) {
            if (z1 == z0) {
#pragma unroll
                for (int j = 0; j < kXV; ++j) v1[j] = v0[j];
            } else {
                at_plane(z1, v1);
            }
            have1 = z1;
        }
        T r[kXV];
#pragma unroll
        for (int j = 0; j < kXV; ++j) r[j] = from_f<T>(lerp(v0[j], v1[j], fz));
        if (whole) {
            typedef T vec __attribute__((ext_vector_type(kXV), aligned(sizeof(T))));
            *reinterpret_cast<vec*>(out) = vec{r[0], r[1], r[2], r[3]};
        } else {
#pragma unroll
            for (int j = 0; j < kXV; ++j)
                if (x + j < Xo) out[j] = r[j];
        }
    }
}

// One destination cell per thread: sources one cell wide, planes of 4 GiB and
// more, and grids beyond the launch limits of the kernel above.
template <typename T>
__global__ __launch_bounds__(kNT) void resample_cell_kernel(const T* __restrict__ src,
                                                            T* __restrict__ dst, int X, int Y,
                                                            int Z, int Xo, int Yo, int Zo,
                                                            int64_t nrows)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= Xo) return;
    int x0, x1;
    float fx;
    lin_axis(x, X, Xo, x0, x1, fx);
    const int64_t plane = (int64_t)X * Y;
    for (int64_t r = (int64_t)blockIdx.y * blockDim.y + threadIdx.y; r < nrows;
         r += (int64_t)gridDim.y * blockDim.y) {
        const int y = (int)(r % Yo), z = (int)(r / Yo);
        int y0, y1, z0, z1;
        float fy, fz;
        lin_axis(y, Y, Yo, y0, y1, fy);
        lin_axis(z, Z, Zo, z0, z1, fz);
        const T* p0 = src + z0 * plane;
        const T* p1 = src + z1 * plane;
        const int64_t o0 = (int64_t)y0 * X, o1 = (int64_t)y1 * X;
        const float a0 = lerp((float)p0[o0 + x0], (float)p0[o0 + x1], fx);
        const float a1 = lerp((float)p0[o1 + x0], (float)p0[o1 + x1], fx);
        const float b0 = lerp((float)p1[o0 + x0], (float)p1[o0 + x1], fx);
        const float b1 = lerp((float)p1[o1 + x0], (float)p1[o1 + x1], fx);
        dst[r * Xo + x] = from_f<T>(lerp(lerp(a0, a1, fy), lerp(b0, b1, fy), fz));
    }
}

// ---- exact downscale by two: one destination cell per thread (rows shorter
// than 16 bytes) ---------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kNT) void halve_kernel(const T* __restrict__ src,
                                                    T* __restrict__ dst, int X, int Y, int Xo,
                                                    int Yo, int64_t nrows)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= Xo) return;
    const int64_t plane = (int64_t)X * Y;
    for (int64_t r = (int64_t)blockIdx.y * blockDim.y + threadIdx.y; r < nrows;
         r += (int64_t)gridDim.y * blockDim.y) {
        const int y = (int)(r % Yo), z = (int)(r / Yo);
        const T* s0 = src + (2 * z) * plane + (int64_t)(2 * y) * X + 2 * x;
        const T* rows[4] = {s0, s0 + X, s0 + plane, s0 + plane + X};
        if constexpr (std::is_same<T, float>::value) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) s += rows[i][0] + rows[i][1];
            dst[r * Xo + x] = s * 0.125f;
        } else {
            uint32_t s = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) s += (uint32_t)rows[i][0] + (uint32_t)rows[i][1];
            dst[r * Xo + x] = (T)((s + 4u) >> 3);  // floor(mean + 1/2), exact
        }
    }
}

// ---- exact downscale by two, 16 destination bytes per thread -------------
// Destination row (y, z) averages source rows 2y, 2y + 1 of planes 2z,
// 2z + 1; a thread reads 32 bytes (a, b) of each of those 4 rows.  Integer
// cells are summed in SIMD-within-a-register lanes (u8: two 16-bit lanes
// per dword, at most 8 * 255 each; u16: one 32-bit sum per cell pair).
template <typename T>
__device__ inline void halve_chunk(const uint4 (&a)[4], const uint4 (&b)[4], uint4& out)
{
    if constexpr (std::is_same<T, float>::value) {
        float o[4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float s0 = 0.f, s1 = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4 v = h ? b[i] : a[i];
                s0 += __uint_as_float(v.x) + __uint_as_float(v.y);
                s1 += __uint_as_float(v.z) + __uint_as_float(v.w);
            }
            o[2 * h] = s0 * 0.125f;
            o[2 * h + 1] = s1 * 0.125f;
        }
        out = make_uint4(__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]),
                         __float_as_uint(o[3]));
    } else if constexpr (std::is_same<T, uint16_t>::value) {
        uint32_t s[8] = {};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w[8] = {a[i].x, a[i].y, a[i].z, a[i].w, b[i].x, b[i].y, b[i].z, b[i].w};
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] += (w[j] & 0xFFFFu) + (w[j] >> 16);
        }
        uint32_t o[4];
#pragma unroll
        for (int m = 0; m < 4; ++m)
            o[m] = ((s[2 * m] + 4u) >> 3) | (((s[2 * m + 1] + 4u) >> 3) << 16);
        out = make_uint4(o[0], o[1], o[2], o[3]);
    } else {
        // dword j of the 32 source bytes holds x = 4j..4j+3: its two 16-bit
        // lanes collect destination cells 2j and 2j+1
        uint32_t s[8] = {};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w[8] = {a[i].x, a[i].y, a[i].z, a[i].w, b[i].x, b[i].y, b[i].z, b[i].w};
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] += (w[j] & 0x00FF00FFu) + ((w[j] >> 8) & 0x00FF00FFu);
        }
        uint32_t o[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            // (lane + 4) >> 3 in both lanes; the low lane's upper bits take
            // spill from the high lane, masked off
            const uint32_t p = ((s[2 * m] + 0x00040004u) >> 3) & 0x00FF00FFu;
            const uint32_t q = ((s[2 * m + 1] + 0x00040004u) >> 3) & 0x00FF00FFu;
            o[m] = (p & 0xFFu) | ((p >> 8) & 0xFF00u) | ((q & 0xFFu) << 16) | ((q << 8) & 0xFF000000u);
        }
        out = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

template <typename T>
__global__ __launch_bounds__(kNT) void halve_vec_kernel(const T* __restrict__ src,
                                                        T* __restrict__ dst, int Xo, int Yo,
                                                        RowBox box)
{
    constexpr int CPC = 16 / sizeof(T);
    int c, y, z;
    if (!row_item(box, c, y, z)) return;
    const int x = min(c * CPC, Xo - CPC);  // the last chunk ends the row
    const int64_t X = 2 * (int64_t)Xo, plane = X * 2 * Yo;
    const T* s0 = src + (2 * (int64_t)z) * plane + (2 * (int64_t)y) * X + 2 * (int64_t)x;
    const T* rows[4] = {s0, s0 + X, s0 + plane, s0 + plane + X};
    uint4 a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a[i] = load_stream(rows[i]);
        b[i] = load_stream(rows[i] + CPC);
    }
    uint4 o;
    halve_chunk<T>(a, b, o);
    store16(dst + ((int64_t)z * Yo + y) * Xo + x, o);
}

// ---- Flip ----------------------------------------------------------------
// The cells of a 16-byte chunk in reverse order.
template <typename T>
__device__ inline uint4 reverse_chunk(uint4 v)
{
    if constexpr (std::is_same<T, float>::value) {
        return make_uint4(v.w, v.z, v.y, v.x);
    } else if constexpr (std::is_same<T, uint16_t>::value) {
        auto sw = [](uint32_t u) { return (u >> 16) | (u << 16); };
        return make_uint4(sw(v.w), sw(v.z), sw(v.y), sw(v.x));
    } else {
        return make_uint4(__builtin_bswap32(v.w), __builtin_bswap32(v.z),
                          __builtin_bswap32(v.y), __builtin_bswap32(v.x));
    }
}

// Rows of the box [y0, y0 + ny) x [z0, z0 + nz), `items` per row: nvec 16-byte
// chunks, then single cells.  Out of place: every byte of a row; rows that are
// no whole chunks end in a chunk moved back to the row's end (rewriting some of
// its neighbour with the same values), rows shorter than a chunk go by cells.
// In place, item i swaps with its mirror: along x the chunks and cells of the
// first half (nvec chunks from either end, the cells between them), along y or
// z the first half of the rows, whole chunks and the cells behind them.  At any
// cell alignment: the one-cell-per-thread form that ragged rows took needed 76
// us for 302^3 uint8 along x (55 MB), two 64-bit divisions a cell.
struct FlipArgs {
    int32_t X, Y, Z;
    int32_t nvec;
    int32_t axis;
    int32_t inplace;
};

template <typename T>
__global__ __launch_bounds__(kNT) void flip_kernel(const T* src, T* dst, FlipArgs a, RowBox box)
{
    constexpr int CPC = 16 / sizeof(T);  // cells per chunk
    int c, y, z;
    if (!row_item(box, c, y, z)) return;
    const int my = a.axis == 1 ? a.Y - 1 - y : y;
    const int mz = a.axis == 2 ? a.Z - 1 - z : z;
    const int64_t o = ((int64_t)z * a.Y + y) * a.X, m = ((int64_t)mz * a.Y + my) * a.X;
    if (c < a.nvec) {
        const int x = a.inplace ? c * CPC : min(c * CPC, a.X - CPC);
        const int mx = a.axis == 0 ? a.X - CPC - x : x;
        const uint4 b = load_stream(src + m + mx);
        const uint4 w = a.inplace ? load_stream(src + o + x) : b;
        store16(dst + o + x, a.axis == 0 ? reverse_chunk<T>(b) : b);
        if (a.inplace) store16(dst + m + mx, a.axis == 0 ? reverse_chunk<T>(w) : w);
    } else {
        const int x = (a.inplace ? a.nvec * CPC : 0) + c - a.nvec;
        const int mx = a.axis == 0 ? a.X - 1 - x : x;
        const T b = src[m + mx], w = a.inplace ? src[o + x] : b;
        dst[o + x] = b;
        if (a.inplace) dst[m + mx] = w;
    }
}

template <typename T>
hipError_t resample_t(const void* src, void* dst, const int32_t in[3], const int32_t out[3],
                      hipStream_t s)
{
    const int64_t nrows = (int64_t)out[1] * out[2];
    const bool halve = in[0] == 2 * out[0] && in[1] == 2 * out[1] && in[2] == 2 * out[2];
    constexpr int CPC = 16 / sizeof(T);
    if (halve && out[0] >= CPC) {
        return for_row_boxes(out[1], out[2], (int)(((int64_t)out[0] + CPC - 1) / CPC),
                             [&](const RowBox& b, dim3 blocks) {
                                 hipLaunchKernelGGL((halve_vec_kernel<T>), blocks, dim3(kNT), 0, s,
                                                    static_cast<const T*>(src),
                                                    static_cast<T*>(dst), out[0], out[1], b);
                             });
    } else if (halve) {
        const RowGrid g = row_grid(out[0], nrows);
        hipLaunchKernelGGL((halve_kernel<T>), g.grid, g.block, 0, s, static_cast<const T*>(src),
                           static_cast<T*>(dst), in[0], in[1], out[0], out[1], nrows);
    } else {
        const int64_t groups = ((int64_t)out[0] + kXV - 1) / kXV;
        const int64_t gx = (groups * out[1] + kNT - 1) / kNT;
        // marches as long as the device still gets 8 workgroups per CU
        const int64_t zc =
            std::min<int64_t>(kZC, std::max<int64_t>(1, gx * out[2] / (8 * device_cus())));
        const int64_t gz = ((int64_t)out[2] + zc - 1) / zc;
        if (in[0] >= 2 && (int64_t)in[0] * in[1] * (int64_t)sizeof(T) < ((int64_t)1 << 32) &&
            gx * kNT <= INT32_MAX && gz <= 65535) {
            auto* kernel = &resample_kernel<T, false>;
            if constexpr (std::is_same<T, uint8_t>::value) {
                if (in[0] <= 2 * (int64_t)out[0] && (int64_t)in[0] * in[1] >= 8)
                    kernel = &resample_kernel<T, true>;
            }
            hipLaunchKernelGGL(kernel, dim3((unsigned)gx, (unsigned)gz), dim3(kNT), 0, s,
                               static_cast<const T*>(src), static_cast<T*>(dst), in[0], in[1],
                               in[2], out[0], out[1], out[2], (int)zc, (uint32_t)groups,
                               make_udiv((uint32_t)groups));
        } else {
            const RowGrid g = row_grid(out[0], nrows);
            hipLaunchKernelGGL((resample_cell_kernel<T>), g.grid, g.block, 0, s,
                               static_cast<const T*>(src), static_cast<T*>(dst), in[0], in[1],
                               in[2], out[0], out[1], out[2], nrows);
        }
    }
    return hipGetLastError();
}

template <typename T>
hipError_t flip_t(const void* src, void* dst, const int32_t d[3], int axis, hipStream_t s)
{
    constexpr int CPC = 16 / sizeof(T);
    FlipArgs a{};
    a.X = d[0];
    a.Y = d[1];
    a.Z = d[2];
    a.axis = axis;
    a.inplace = src == dst ? 1 : 0;
    // rows per plane and planes visited (in place along y / z: the first half)
    const int Ys = a.inplace && axis == 1 ? d[1] / 2 : d[1];
    const int Zs = a.inplace && axis == 2 ? d[2] / 2 : d[2];
    int items;
    if (!a.inplace) {
        a.nvec = d[0] >= CPC ? (int)(((int64_t)d[0] + CPC - 1) / CPC) : 0;
        items = a.nvec ? a.nvec : d[0];
    } else if (axis == 0) {
        a.nvec = d[0] / (2 * CPC);
        items = a.nvec + (d[0] - 2 * CPC * a.nvec) / 2;
    } else {
        a.nvec = d[0] / CPC;
        items = a.nvec + d[0] % CPC;
    }
    if (Ys == 0 || Zs == 0 || items == 0) return hipSuccess;  // in place along one cell
    return for_row_boxes(Ys, Zs, items, [&](const RowBox& b, dim3 blocks) {
        hipLaunchKernelGGL((flip_kernel<T>), blocks, dim3(kNT), 0, s, static_cast<const T*>(src),
                           static_cast<T*>(dst), a, b);
    });
}

}  // namespace

hipError_t launch_resample(const void* src, void* dst, vktDataFormat f, const int32_t in[3],
                           const int32_t out[3], hipStream_t s)
{
    switch (f) {
    case vktDataFormatUInt8: return resample_t<uint8_t>(src, dst, in, out, s);
    case vktDataFormatUInt16: return resample_t<uint16_t>(src, dst, in, out, s);
    case vktDataFormatFloat32: return resample_t<float>(src, dst, in, out, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_flip(const void* src, void* dst, vktDataFormat f, const int32_t dims[3],
                       int axis, hipStream_t s)
{
    switch (f) {
    case vktDataFormatUInt8: return flip_t<uint8_t>(src, dst, dims, axis, s);
    case vktDataFormatUInt16: return flip_t<uint16_t>(src, dst, dims, axis, s);
    case vktDataFormatFloat32: return flip_t<float>(src, dst, dims, axis, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace vkt
