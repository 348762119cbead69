// vkt_filter_sep.hip -- ApplyFilter for rank-1 (separable) filters,
// w[c][b][a] = t[c] v[b] u[a], as three one-dimensional passes: 3k
// multiply-adds per output instead of k^3.
//
// Operation (paper Sec. 3.2 "Volume Manipulation": a faster implementation
// of a filter must keep its behaviour; the benchmarked Gaussian blur of
// Sec. 4.3 is separable):
//   T(x,y,z) = sum_c t[c] sum_b v[b] sum_a u[a] s(A(x+a-r), A(y+b-r), A(z+c-r)),
// stored like ApplyFilter.  Integer filters are factored exactly into
// integer factors; on integer cells the host admits them only when every
// partial sum stays an exact integer -- in FP32, or in 24-bit multiply-adds
// with int32 sums (IACC) -- so the stored quotient is the dense one, and such
// filters of 5 and more (3 and more where no other path is as fast) come here
// unasked: uint16 400x380x360 7^3 box 969 -> 129 us, uint8 9^3 box 1535 -> 120 us.
//
// Mapping to gfx950 (same tiling as the vector kernel: 256 threads, 64 x 32
// output tile, 4 x 2 outputs per thread, z-slab marching):
//  * each input plane's halo tile is staged in LDS as FP32, double buffered,
//    with the loads of the plane after next in flight;
//  * x pass: the 64-wide rows of the (32 + 2r)-row halo are filtered with u
//    into a second LDS buffer, also double buffered (4 outputs per thread
//    and row, 16-byte reads); one barrier per plane separates the passes;
//  * y pass: each thread filters its 4 x 2 outputs' columns with v;
//  * z pass: the plane's result enters an input-stationary ring of k partial
//    sums with weights t (slots outside the slab are skipped); the oldest is
//    a finished output.  The z loop is unrolled by k so the ring entries
//    stay in fixed registers.
// The three factor vectors (16 floats each, zero padded) are brought into
// SGPRs by explicit scalar loads: once per tile-slab for k <= 7, else one
// per pass.
#include "vkt_stage.h"

#include <type_traits>
#include <utility>

namespace vkt {
namespace {

constexpr int kBX = 16, kBY = 16, kNT = kBX * kBY;
constexpr int kVX = 4, kVY = 2;
constexpr int kTX = kBX * kVX, kTY = kBY * kVY;  // 64 x 32 tile

template <int K>
struct GeoS {
    static constexpr int R = (K - 1) / 2;
    static constexpr int HX = kTX + 2 * R;                // staged row width
    static constexpr int HY = kTY + 2 * R;                // staged rows
    static constexpr int P = (HX + 3) & ~3;               // staged row pitch (floats)
    static constexpr int XW = kVX + K - 1;                // x-pass window
    static constexpr int XR = (XW + 3) / 4;               // 16-byte reads per window
    static constexpr int A_CELLS = HY * P;                // one staged plane
    static __device__ constexpr int at(int row, int col) { return row * P + col; }
    static constexpr int B_CELLS = HY * kTX;              // x-pass result
    static constexpr int NXR = (HY + kBY - 1) / kBY;      // x-pass rows per thread
    static_assert(4 * (kBX - 1) + 4 * XR <= P, "x window exceeds the pitch");
};

__device__ inline uint32_t xcd_remap(uint32_t b, uint32_t n)
{
    const uint32_t q = n / 8, rem = n % 8, xcd = b % 8, idx = b / 8;
    return xcd < rem ? xcd * (q + 1) + idx : rem * (q + 1) + (xcd - rem) * q + idx;
}

template <bool IACC> struct AccT { using type = float; };
template <> struct AccT<true> { using type = int32_t; };
__device__ inline float mul(float w, float v) { return w * v; }
__device__ inline int32_t mul(int32_t w, int32_t v) { return __mul24(w, v); }
__device__ inline float mac(float w, float v, float acc) { return fmaf(w, v, acc); }
__device__ inline int32_t mac(int32_t w, int32_t v, int32_t acc)
{
    return __mul24(w, v) + acc;  // |w|, |v| < 2^23 (host check): exact
}

// 16 factor weights into SGPRs; one explicit scalar load that waits for its
// data (keeps exactly one factor vector live, see the vector kernel).
template <typename Acc>
__device__ inline void load_factor(const Acc* p, Acc (&f)[16])
{
    typedef uint32_t v16 __attribute__((ext_vector_type(16)));
    // the address is uniform; readfirstlane keeps it in SGPRs even where
    // register pressure would otherwise leave a copy in VGPRs
    // (readfirstlane returns int: widen through uint32_t, not by sign)
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    const uint64_t sa = (uint64_t)lo | ((uint64_t)hi << 32);
    v16 r;
    asm volatile("s_load_dwordx16 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=&s"(r) : "s"(sa));
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const uint32_t u = r[q];
        if constexpr (std::is_same<Acc, float>::value) f[q] = __uint_as_float(u);
        else f[q] = (Acc)u;
    }
}

template <typename F, int... I>
__device__ __attribute__((always_inline)) inline void static_for_impl(
    F& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __attribute__((always_inline)) inline void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ inline uint32_t udiv(uint32_t n, UDiv d)
{
    const uint32_t t = __umulhi(d.m, n);
    return (t + ((n - t) >> d.sh1)) >> d.sh2;
}

// Stored value of one finished output (T exact integer for integer filters).
template <typename T, typename Acc>
__device__ __attribute__((always_inline)) inline T finish(Acc acc, const VolDesc& a)
{
    if constexpr (std::is_same<T, float>::value) {
        return a.epi == kEpiFloatDiv ? acc * a.inv_D : acc;
    } else {
        constexpr int kMax = std::is_same<T, uint8_t>::value ? 255 : 65535;
        if (a.epi == kEpiIntDiv) {
            const int32_t t = (int32_t)acc;
            if (t < 0) return (T)0;
            const uint32_t q = udiv(2u * (uint32_t)t + (uint32_t)a.D, a.div2D);
            return (T)(q > (uint32_t)kMax ? (uint32_t)kMax : q);
        }
        const float q = floorf((float)acc + 0.5f);
        return (T)fminf(fmaxf(q, 0.f), (float)kMax);
    }
}

// One tile-slab; f holds the factors u | v | t at offsets 0, 16, 32.
template <typename T, int K, bool IACC>
__device__ __attribute__((always_inline)) inline void sep_tile(
    const VolDesc& a, const typename AccT<IACC>::type* __restrict__ f, int tile, int slab,
    typename AccT<IACC>::type* lds)
{
    using G = GeoS<K>;
    using Acc = typename AccT<IACC>::type;
    using V4 = typename std::conditional<IACC, int4, float4>::type;
    constexpr int R = G::R;

    const int t = threadIdx.x, tx = t % kBX, ty = t / kBX;
    const int x0 = a.rx0 + (tile % a.tiles_x) * kTX, y0 = a.ry0 + (tile / a.tiles_x) * kTY;
    const int zb = a.rz0 + slab * a.tz, ze = min(zb + a.tz, a.rz1);
    // x-pass results, double buffered by plane parity like the staged
    // planes: with both double buffered, one barrier per plane suffices (the
    // x pass of plane p + 1 writes the other buffer while slower waves still
    // read plane p's; plane p + 2 reuses it only after the barrier of p + 1)
    Acc* const bx0 = lds + 2 * G::A_CELLS;

    PlaneStage<T, R, G::HY, G::P, kNT, G> in;
    in.init(a, x0, y0, t);
    auto put = [&](Acc* buf) __attribute__((always_inline)) {
        in.put([&](const T (&v)[4], int e, bool on) __attribute__((always_inline)) {
            if (on) *reinterpret_cast<V4*>(buf + e) = V4{(Acc)v[0], (Acc)v[1], (Acc)v[2], (Acc)v[3]};
        });
    };

    // z ring in fixed registers: the z loop is unrolled by K, and at plane
    // p = zi - zi_beg the ring entry of age c (output plane zi - c + r) sits
    // in slot (c - p) mod K, so no entry moves between planes
    Acc acc[K][kVY][kVX];

    // k <= 7: the three factor vectors stay in SGPRs for the whole
    // tile-slab; larger k loads each one before its pass (48 live weights
    // would spill SGPRs)
    constexpr bool kHoist = K <= 7;
    Acc u[16], v[16], tw[16];
    if constexpr (kHoist) {
        load_factor(f, u);
        load_factor(f + 16, v);
        load_factor(f + 32, tw);
    }

    const int zi_beg = zb - R, zi_end = ze + R;
    in.gather(a, zi_beg);
    put(lds);
    if (zi_beg + 1 < zi_end) in.gather(a, zi_beg + 1);
    __syncthreads();

    // (columns past 2^31 - 1 wrap to negative ones, whose offsets lie past the plane)
    const int ox = (int)((uint32_t)x0 + (uint32_t)(kVX * tx)), oy = y0 + kVY * ty;
    const bool vec = ox <= a.rx1 - kVX;
    uint32_t ooff[kVY];  // this thread's output rows (past the region: dropped)
#pragma unroll
    for (int vy = 0; vy < kVY; ++vy)
        ooff[vy] = oy + vy < a.ry1
                       ? ((uint32_t)(oy + vy) * (uint32_t)a.X + (uint32_t)ox) * (uint32_t)sizeof(T)
                       : kOutside;

    auto step = [&](int zi, auto U) __attribute__((always_inline)) {
        constexpr int P = decltype(U)::value;  // plane index mod K
        const int cur = (zi - zi_beg) & 1;
        const Acc* A = lds + cur * G::A_CELLS;
        Acc* const bx = bx0 + cur * G::B_CELLS;

        // ---- x pass over all staged rows: bx[row][x] = sum_a u[a] A[row][x + a]
        if constexpr (!kHoist) load_factor(f, u);
#pragma unroll
        for (int i = 0; i < G::NXR; ++i) {
            const int row = ty + kBY * i;
            if (row < G::HY) {
                Acc wdw[4 * G::XR];
#pragma unroll
                for (int q = 0; q < G::XR; ++q) {
                    const V4 v4 =
                        *reinterpret_cast<const V4*>(A + row * G::P + kVX * tx + 4 * q);
                    wdw[4 * q + 0] = v4.x;
                    wdw[4 * q + 1] = v4.y;
                    wdw[4 * q + 2] = v4.z;
                    wdw[4 * q + 3] = v4.w;
                }
                Acc h[kVX];
#pragma unroll
                for (int vx = 0; vx < kVX; ++vx) {
                    h[vx] = mul(u[0], wdw[vx]);
#pragma unroll
                    for (int aa = 1; aa < K; ++aa) h[vx] = mac(u[aa], wdw[vx + aa], h[vx]);
                }
                *reinterpret_cast<V4*>(bx + row * kTX + kVX * tx) = V4{h[0], h[1], h[2], h[3]};
            }
        }
        // next plane into the other staging buffer (read two barriers later)
        if (zi + 1 < zi_end) put(lds + (cur ^ 1) * G::A_CELLS);
        if (zi + 2 < zi_end) in.gather(a, zi + 2);
        __syncthreads();

        // ---- y pass: p[vy][vx] = sum_b v[b] bx[2 ty + vy + b][4 tx + vx],
        // streaming the k + 1 rows (row j feeds output row vy through v[j - vy])
        Acc pv[kVY][kVX];
        if constexpr (!kHoist) load_factor(f + 16, v);
#pragma unroll
        for (int j = 0; j < kVY + K - 1; ++j) {
            const V4 v4 = *reinterpret_cast<const V4*>(bx + (kVY * ty + j) * kTX + kVX * tx);
            const Acc row[kVX] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
            for (int vy = 0; vy < kVY; ++vy) {
                const int b = j - vy;
                if (b < 0 || b >= K) continue;
#pragma unroll
                for (int vx = 0; vx < kVX; ++vx)
                    pv[vy][vx] = b == 0 ? mul(v[0], row[vx]) : mac(v[b], row[vx], pv[vy][vx]);
            }
        }
        // ---- z pass: age c feeds output plane zi - c + r; age 0 starts its
        // sum (a slot it reuses was stored or is never stored)
        const int c_lo = max(0, zi + R - ze + 1), c_hi = min(K - 1, zi + R - zb);
        if constexpr (!kHoist) load_factor(f + 32, tw);
#pragma unroll
        for (int c = 0; c < K; ++c) {
            if (c < c_lo || c > c_hi) continue;
            const int slot = ((c - P) % K + K) % K;
#pragma unroll
            for (int vy = 0; vy < kVY; ++vy)
#pragma unroll
                for (int vx = 0; vx < kVX; ++vx)
                    acc[slot][vy][vx] = c == 0 ? mul(tw[0], pv[vy][vx])
                                               : mac(tw[c], pv[vy][vx], acc[slot][vy][vx]);
        }

        // ---- the oldest entry (age K - 1) is output plane zo = zi - r
        const int zo = zi - R;
        if (zo >= zb) {
            constexpr int old = ((K - 1 - P) % K + K) % K;
            const int32_t plane_bytes = (int32_t)((int64_t)a.X * a.Y * (int64_t)sizeof(T));
            const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(
                static_cast<char*>(a.dst) + (int64_t)zo * plane_bytes, (short)0, plane_bytes,
                (int)kRsrcWord3);
#pragma unroll
            for (int vy = 0; vy < kVY; ++vy) {
                T r4[kVX];
#pragma unroll
                for (int vx = 0; vx < kVX; ++vx) r4[vx] = finish<T>(acc[old][vy][vx], a);
                store4<T>(d, ooff[vy], r4, vec, a.rx1 - ox);
            }
        }
    };

    for (int zi = zi_beg; zi < zi_end; zi += K) {
        static_for<K>([&](auto U) {
            if (zi + decltype(U)::value < zi_end) step(zi + decltype(U)::value, U);
        });
    }
}

template <typename T, int K, bool IACC>
__global__ __launch_bounds__(kNT) void filter_sep_kernel(
    VolDesc a, const typename AccT<IACC>::type* __restrict__ f, uint32_t nblocks)
{
    using Acc = typename AccT<IACC>::type;
    __shared__ __align__(16) Acc lds[2 * GeoS<K>::A_CELLS + 2 * GeoS<K>::B_CELLS];
    const uint32_t lid = xcd_remap(blockIdx.x, nblocks);
    const uint32_t ntiles = (uint32_t)a.tiles_x * (uint32_t)a.tiles_y;
    sep_tile<T, K, IACC>(a, f, (int)(lid % ntiles), (int)(lid / ntiles), lds);
}

template <typename T, int K, bool IACC>
hipError_t launch_k(const FilterJob& j, hipStream_t s)
{
    const ClassGeom g{kTX, kTY, 4 > 2 * K ? 4 : 2 * K};
    const int RX = j.roi[3] - j.roi[0], RY = j.roi[4] - j.roi[1], RZ = j.roi[5] - j.roi[2];
    const int64_t ntiles = (int64_t)tiles_along(RX, g.tx) * tiles_along(RY, g.ty);
    const void* fn = (const void*)&filter_sep_kernel<T, K, IACC>;
    const int tz = plan_tz(ntiles, RZ, K, 1, 128, resident_wgs(fn), 1);
    const VolDesc a = make_desc(j, tz, g);
    const int64_t nb = ntiles * ((RZ + tz - 1) / tz);
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    // (the integer copies of the factors follow the float ones)
    using Acc = typename AccT<IACC>::type;
    const Acc* f = reinterpret_cast<const Acc*>(j.wsep + (IACC ? kSepInt : 0));
    hipLaunchKernelGGL((filter_sep_kernel<T, K, IACC>), dim3((unsigned)nb), dim3(kNT), 0, s, a, f,
                       (uint32_t)nb);
    return hipGetLastError();
}

template <typename T, bool IACC>
hipError_t dispatch_k(const FilterJob& j, hipStream_t s)
{
    switch (j.k) {
    case 1: return launch_k<T, 1, IACC>(j, s);
    case 3: return launch_k<T, 3, IACC>(j, s);
    case 5: return launch_k<T, 5, IACC>(j, s);
    case 7: return launch_k<T, 7, IACC>(j, s);
    case 9: return launch_k<T, 9, IACC>(j, s);
    case 11: return launch_k<T, 11, IACC>(j, s);
    case 13: return launch_k<T, 13, IACC>(j, s);
    case 15: return launch_k<T, 15, IACC>(j, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_filter_sep(const FilterJob& j, hipStream_t s)
{
    switch (j.fmt) {
    case vktDataFormatUInt8:
        return j.sep_int ? dispatch_k<uint8_t, true>(j, s) : dispatch_k<uint8_t, false>(j, s);
    case vktDataFormatUInt16:
        return j.sep_int ? dispatch_k<uint16_t, true>(j, s) : dispatch_k<uint16_t, false>(j, s);
    case vktDataFormatFloat32: return dispatch_k<float, false>(j, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace vkt
