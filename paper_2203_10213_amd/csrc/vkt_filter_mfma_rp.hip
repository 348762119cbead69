// vkt_filter_mfma_rp.hip -- ApplyFilter for filters of size 5 and 7 on the
// matrix cores: an implicit GEMM on 32x32x16 MFMA tiles over pairs of output
// rows, with split 16-bit operands and FP32 accumulation.
//
// Operation (paper Sec. 3.2 "Volume Manipulation"; benchmarked as a Gaussian
// blur, Sec. 4.3):
//   T(x,y,z) = sum_{a,b,c} w[a + k(b + k c)] * s(A(x+a-r), A(y+b-r), A(z+c-r)).
//
// GEMM embedding, per input plane zi (D += A * B on 32x32x16 tiles):
//   N (columns n) : row pairs of one x-strip: output rows y0 + 2n + dy,
//                   dy in {0, 1}, of NX output columns (3 for k = 5, 2 for 7);
//   K (reduction) : (row offset b' in 0..k, input column ax in 0..7) pairs,
//                   two rows per 16-deep chunk; the B operand is the input
//                   window s(x_s - r + ax, y0 + 2n + b' - r, zi), read
//                   straight from the LDS-staged plane;
//   M (rows)      : (filter plane c, dy, output x-offset xo), with
//                   A[(c, dy, xo)][(b', ax)] = w[c][b' - dy][ax - xo]
//                   (zero outside the filter).
// Pairing output rows lets one 16-deep chunk carry two filter rows for both
// rows of a pair.  k = 7: 28 of the 32 M rows and 49 of 64 reduction slots are
// filter taps (67 % of the products); k = 5 with three columns a strip: 30 of
// 32 and 25 of 48 (49 %; with two columns 33 %, and half as many products
// again for the same outputs).  The sum of one row's 8 slots does not depend
// on their order (checked on the GPU with permuted slots), so a strip's width
// changes no result.
//
// z ring in registers: lane l holds D rows 8 (r / 4) + 4 (l / 32) + r % 4
// in its registers r = 0..15.  M row (c, dy, xo) is placed in lane half dy at
// register NX s + xo of ring slot s; slot s accumulates output plane s mod k
// of the slab, so the filter plane that it meets moves on with each input
// plane, not the accumulators: a lane reads its 16-byte weight row of the next
// filter plane from a table in LDS (8 reads of 1 KB a plane and wave for k = 7
// instead of some 110 register moves; vector instructions without the products
// 327 -> 143 a plane and wave).  Lane l then holds output row
// y0 + 2 (l % 32) + l / 32 of its wave's strips.
//
// A workgroup is 4 waves x 4 strips: a tile of 48 (k = 5) or 32 (k = 7)
// columns and 64 rows; a wave's 4 strips are adjacent, and one segment read
// per (K chunk, operand piece) holds all their windows.
//
// What bounds it: the matrix cores (busy 78 % at 7^3, 60 % at 5^3 with 6
// products, 37 % for uint8) at the clock that the card holds under them (cycles
// counted over the time: 1.3 GHz at 7^3, 1.9 at 5^3, 2.4 for uint8).  Measured before and after the face quads of their
// own, the strips of three columns, the turning weights and the rising
// priorities: 302^3 uint8 5^3 106 -> 46 us, 512^3 float32 5^3 with 6 products
// 455 -> 409 us, 1024^3 7^3 with 3 products 2.97 -> 2.75 ms, all with the same
// bits as before.
#include "vkt_mfma_common.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace vkt {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
template <typename T, int K, int PM>
struct RpCfg {
    using Tin = T;
    using PC = Pieces<PM>;
    static constexpr int R = (K - 1) / 2;
    static_assert(K == 5 || K == 7, "filters of 5 or 7");
    static constexpr int NX = K == 5 ? 3 : 2;       // output columns per strip
    static_assert(NX + K - 1 <= 8 && K * NX <= 16, "8 input columns, 16 registers");
    static constexpr int WS = 4;                    // strips per wave
    static constexpr int WX = WS * NX;              // columns per wave
    static constexpr int NCH = (K + 2) / 2;         // 16-deep chunks: rows b' = 0..k
    static constexpr int TX = 4 * WX;               // columns per workgroup
    static constexpr int TY = 64;                   // 32 row pairs
    static constexpr int HY = TY + K - 1;           // staged rows
    static constexpr int PITCH = K == 5 ? 56 : 40;  // staged columns (x0 - r ...)
    // staged rows lie in pairs of PAIR cells: the lanes of a segment read are
    // one pair apart, and 58 dwords put the 8-byte reads of 16 lanes into
    // different banks (56: 74 cycles for 40 bytes a lane instead of 24)
    static constexpr int PAIR = K == 5 ? 116 : 80;
    static __device__ constexpr int at(int row, int col) { return (row >> 1) * PAIR + (row & 1) * PITCH + col; }
    // dwords of a lane's segment: the windows of the wave's strips, read 8
    // bytes (24-byte wave offsets, k = 5) or 16 bytes at a time
    static constexpr int RD = WX % 8 == 0 ? 4 : 2;
    static constexpr int SEGD = ((NX * (WS - 1) + 8 + 1) / 2 + RD - 1) / RD * RD;
    static_assert(TX + K - 1 <= PITCH && 3 * WX + 2 * SEGD <= PITCH && PITCH % 8 == 0, "columns");
    static_assert(2 * 31 + 2 * (NCH - 1) + 1 < HY, "staged rows");
    static constexpr int PLANE = (HY / 2 * PAIR + 7) / 8 * 8;
    static_assert(HY % 2 == 0, "row pairs");
    // output rows in LDS (floats), read and written EV floats at a time
    static constexpr int EV = K == 5 ? 2 : 4;
    static constexpr int EPITCH = TX + EV;
    // weight table in LDS: per (chunk, piece, lane half) the 16-byte rows of
    // (c, dy, xo), then a zero row for the unused M rows
    static constexpr int AROWS = 2 * NX * K + 1;
    static constexpr int TABLE = NCH * PC::NBI * 2 * AROWS * 8;  // 16-bit elements
    static constexpr int LDS_BYTES = (2 * PC::PS * PLANE + TABLE) * 2 + 2 * TY * EPITCH * 4;
    static_assert(2 * LDS_BYTES <= 160 * 1024, "two workgroups per CU");
};

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

template <bool F16>
__device__ inline f32x16 mfma32(u16x8 a, u32x4 b, f32x16 c)
{
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

template <class C>
__device__ void rp_tile(const VolDesc& a, const float* __restrict__ w, int tile, int slab,
                        uint16_t* lds_base, float (*epi)[C::TY][C::EPITCH], uint16_t* tab)
{
    using T = typename C::Tin;
    using PC = typename C::PC;
    constexpr int K = 2 * C::R + 1;
    constexpr int R = C::R;
    constexpr int PM = std::is_same<T, uint8_t>::value ? kU8
                       : std::is_same<T, uint16_t>::value ? kU16
                       : (PC::NPROD == 6 ? kF32x6 : kF32x3);
    constexpr int PLANE = C::PLANE;
    // lds[buffer][piece][C::at(row, column)]
    auto lds = reinterpret_cast<uint16_t(*)[PC::PS][PLANE]>(lds_base);

    const int t = threadIdx.x, lane = t % 64, wave = t / 64;
    const int x0 = a.rx0 + (tile % a.tiles_x) * C::TX, y0 = a.ry0 + (tile / a.tiles_x) * C::TY;
    const int zb = a.rz0 + slab * a.tz, ze = min(zb + a.tz, a.rz1);
    const int64_t plane = (int64_t)a.X * a.Y;
    const int32_t plane_bytes = (int32_t)(plane * (int64_t)sizeof(T));  // < 2^31 (host check)

    // ---- A operand (weights): row (c, dy, xo) of the table holds, per chunk
    // q, piece and lane half kg, the 8 reduction slots (b' = 2q + kg,
    // ax = 0..7); a thread builds one (q, kg, row)
    for (int i = t; i < C::NCH * 2 * C::AROWS; i += kNT) {
        const int row = i % C::AROWS, kg = (i / C::AROWS) % 2, q = i / (2 * C::AROWS);
        const int c = row / (2 * C::NX), dy = (row / C::NX) % 2, xo = row % C::NX;
        u16x8 v[PC::NBI];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int b = 2 * q + kg - dy, aa = e - xo;
            float wv = 0.f;
            if (c < K && b >= 0 && b < K && aa >= 0 && aa < K) wv = w[(c * K + b) * K + aa];
            uint16_t p[3];
            split_weight<PM>(wv, a.wscale, p);
#pragma unroll
            for (int bi = 0; bi < PC::NBI; ++bi) v[bi][e] = p[bi];
        }
#pragma unroll
        for (int bi = 0; bi < PC::NBI; ++bi)
            *reinterpret_cast<u16x8*>(&tab[(((q * PC::NBI + bi) * 2 + kg) * C::AROWS + row) * 8]) = v[bi];
    }
    // Lane l's M row is register r of lane half dy: ring slot r / NX, column
    // xo.  Slot s holds output plane s mod k of the slab, so at input plane p
    // it takes filter plane c = (p - s) mod k: the lane reads the table one
    // filter plane (ASTEP elements) further each plane.
    constexpr int ASTEP = 2 * C::NX * 8;
    int aoff, alast, afirst;
    {
        const int rho = lane % 32, kg = lane / 32;
        const int r = 4 * (rho / 8) + rho % 4, dy = (rho / 4) % 2;
        const int sl = r / C::NX, xo = r % C::NX;
        afirst = (kg * C::AROWS + (sl < K ? dy * C::NX + xo : C::AROWS - 1)) * 8;
        alast = afirst + (sl < K ? (K - 1) * ASTEP : 0);
        aoff = afirst + (sl < K ? (K - sl) % K * ASTEP : 0);
    }

    // ---- staging of the input plane: PITCH x HY cells from (x0 - r, y0 - r);
    // staged columns past X + r meet zero weights: they hold zeros
    PlaneStage<T, R, C::HY, C::PITCH, kNT, C> in;
    in.init(a, x0, y0, t);
    if (in.face) {
        for (int e = t; e < 2 * PC::PS * PLANE / 8; e += kNT)
            reinterpret_cast<u32x4*>(lds_base)[e] = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
    }
    auto put = [&](int buf) __attribute__((always_inline)) {
        in.put([&](const T (&v)[4], int e, bool on) __attribute__((always_inline)) {
            stage_quad<PM>(lds[buf], v, e, on);
        });
    };

    // ---- output: lane l holds row 2 (l % 32) + l / 32 of the tile at the
    // wave's WX columns; the workgroup's block goes through LDS (epi[P],
    // double buffered) so that each row is stored by 4 consecutive lanes, CP
    // cells each (whole rows of the tile per 4 lanes)
    constexpr int CP = C::TX / 4;
    typedef float evec __attribute__((ext_vector_type(C::EV)));
    const int srow = t / 4, scol = CP * (t % 4);
    // (columns past 2^31 - 1 wrap to negative ones, whose offsets lie past the plane)
    const int ys = y0 + srow, xst = (int)((uint32_t)x0 + (uint32_t)scol);
    // rows past the region's last row fall beyond the plane: dropped
    const uint32_t ooff =
        ys < a.ry1 ? ((uint32_t)ys * (uint32_t)a.X + (uint32_t)xst) * (uint32_t)sizeof(T) : kOutside;
    const bool vec_row = xst <= a.rx1 - CP;  // (buffer stores take any cell alignment)

    f32x16 acc[C::WS];
#pragma unroll
    for (int s = 0; s < C::WS; ++s)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[s][r] = 0.f;

    // lane's B-operand row and first column inside the staged plane
    const int brow = 2 * (lane % 32) + lane / 32;
    const int bcol = C::WX * wave, boff = C::at(brow, bcol);

    const int zi_beg = zb - R, zi_end = ze + R;
    in.gather(a, zi_beg);
    put(0);
    in.gather(a, min(zi_beg + 1, zi_end - 1));
    __syncthreads();

    // One input plane zi = zi_beg + p, U = p mod k; LDS buffer cur holds it,
    // the loads of plane zi + 1 are in flight.  That plane is staged after the
    // products and the loads of plane zi + 2 take its registers at once, so
    // that they have a whole step to arrive.  The loop is unrolled by k, which
    // fixes the ring slot that a plane finishes: with a slot index in a
    // register the compiler copied the accumulators for every indexed move.
    int cur = 0;
    auto step = [&](auto uc, int zi) __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value;

        // chunk q: lane (n, g) = (l % 32, l / 32) reads its weights and the
        // cells from the wave's first column of staged row 2n + g + 2q on; the
        // reads of chunk q + 1 go out before the products of chunk q
        u16x8 W[2][PC::NBI];
        uint32_t seg[2][PC::PS][C::SEGD];
        auto load_chunk = [&](int q, u16x8 (&wq)[PC::NBI], uint32_t (&sg)[PC::PS][C::SEGD]) {
#pragma unroll
            for (int bi = 0; bi < PC::NBI; ++bi)
                wq[bi] = *reinterpret_cast<const u16x8*>(
                    &tab[aoff + (q * PC::NBI + bi) * 2 * C::AROWS * 8]);
            const int off = boff + q * C::PAIR;
            typedef uint32_t vrd __attribute__((ext_vector_type(C::RD)));
#pragma unroll
            for (int ps = 0; ps < PC::PS; ++ps)
#pragma unroll
                for (int h = 0; h < C::SEGD / C::RD; ++h) {
                    const vrd v = *reinterpret_cast<const vrd*>(&lds[cur][ps][off + 2 * C::RD * h]);
#pragma unroll
                    for (int d = 0; d < C::RD; ++d) sg[ps][C::RD * h + d] = v[d];
                }
        };
        // Raised wave priority, higher with each chunk: the wave that is ahead
        // in its products takes the matrix cores and ends first, so that its
        // staging and output run under the other wave's products.  At one
        // priority the two waves of a SIMD share the matrix cores evenly, end
        // together and then both leave them idle.
        __builtin_amdgcn_s_setprio(1);
        load_chunk(0, W[0], seg[0]);
#pragma unroll
        for (int q = 0; q < C::NCH; ++q) {
            if (q == 1) __builtin_amdgcn_s_setprio(2);
            if (q == C::NCH - 1) __builtin_amdgcn_s_setprio(3);
            if (q + 1 < C::NCH) load_chunk(q + 1, W[(q + 1) & 1], seg[(q + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            // two strips at a time (their windows' registers), products outer:
            // consecutive products are independent
#pragma unroll
            for (int s0 = 0; s0 < C::WS; s0 += 2) {
                u32x4 B[2][PC::PS];  // the 8 cells from column NX st of the segment on
#pragma unroll
                for (int s1 = 0; s1 < 2; ++s1)
#pragma unroll
                    for (int ps = 0; ps < PC::PS; ++ps)
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const uint32_t(&sg)[C::SEGD] = seg[q & 1][ps];
                            const int st = s0 + s1, d0 = C::NX * st / 2 + d;
                            B[s1][ps][d] = C::NX * st % 2
                                               ? __builtin_amdgcn_alignbit(sg[d0 + 1], sg[d0], 16)
                                               : sg[d0];
                        }
#pragma unroll
                for (int pr = 0; pr < PC::NPROD; ++pr)
#pragma unroll
                    for (int s1 = 0; s1 < 2; ++s1)
                        acc[s0 + s1] = mfma32<PC::F16>(W[q & 1][PC::prod[pr][1]],
                                                       B[s1][PC::prod[pr][0]], acc[s0 + s1]);
                if (C::NX == 3) __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        aoff = aoff == alast ? afirst : aoff + ASTEP;
        // the next plane's cells are split and staged after the products
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        put(cur ^ 1);
        in.gather(a, min(zi + 2, zi_end - 1));

        // ---- ring slot U + 1 holds output plane zi - r; it restarts at zero
        constexpr int done = (U + 1) % K;
        const int zo = zi - R;
        const bool out = zo >= zb;
        float fin[C::WX];
#pragma unroll
        for (int st = 0; st < C::WS; ++st)
#pragma unroll
            for (int xo = 0; xo < C::NX; ++xo) {
                fin[C::NX * st + xo] = acc[st][C::NX * done + xo];
                acc[st][C::NX * done + xo] = 0.f;
            }
        if (out) {
#pragma unroll
            for (int h = 0; h < C::WX / C::EV; ++h) {
                evec v;
#pragma unroll
                for (int d = 0; d < C::EV; ++d) v[d] = fin[C::EV * h + d];
                *reinterpret_cast<evec*>(&epi[cur][brow][bcol + C::EV * h]) = v;
            }
        }
        // the next plane (staged above) and this plane's outputs are complete
        __syncthreads();
        if (out) {
            float v[CP];
#pragma unroll
            for (int h = 0; h < CP / C::EV; ++h) {
                const evec u = *reinterpret_cast<const evec*>(&epi[cur][srow][scol + C::EV * h]);
#pragma unroll
                for (int d = 0; d < C::EV; ++d) v[C::EV * h + d] = u[d];
            }
            const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
                static_cast<char*>(a.dst) + (int64_t)zo * plane_bytes, (short)0, plane_bytes,
                (int)kRsrcWord3);
            store_row<T, CP>(rd, ooff, v, vec_row, a.rx1 - xst, a.unscale);
        }
        cur ^= 1;
    };
    for (int zi = zi_beg; zi < zi_end; zi += K)
        static_for<K>([&](auto uc) __attribute__((always_inline)) {
            if (zi + decltype(uc)::value < zi_end) step(uc, zi + decltype(uc)::value);
        });
}

template <class C>
constexpr int rp_lds_elems()
{
    return 2 * C::PC::PS * C::PLANE;
}

template <class C>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(2)))
void filter_mfma_rp_kernel(VolDesc a, const float* __restrict__ w, uint32_t nblocks)
{
    __shared__ __align__(16) uint16_t lds[rp_lds_elems<C>()];
    __shared__ __align__(16) float epi[2][C::TY][C::EPITCH];
    __shared__ __align__(16) uint16_t tab[C::TABLE];
    const uint32_t lid = xcd_remap(blockIdx.x, nblocks);
    const uint32_t ntiles = (uint32_t)a.tiles_x * (uint32_t)a.tiles_y;
    rp_tile<C>(a, w, (int)(lid % ntiles), (int)(lid / ntiles), lds, epi, tab);
}

// Persistent workgroups over a queue of (volume, tile-slab) items; the last
// workgroup to finish resets the queue counters.
template <class C>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(2)))
void filter_mfma_rp_batched_kernel(BatchArgs b)
{
    __shared__ __align__(16) uint16_t lds[rp_lds_elems<C>()];
    __shared__ __align__(16) float epi[2][C::TY][C::EPITCH];
    __shared__ __align__(16) uint16_t tab[C::TABLE];
    __shared__ uint32_t s_item;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(&b.counters[0], 1u);
        __syncthreads();
        // the item index is the same in every lane: keep it (and the work item
        // and volume descriptor it selects) in scalar registers
        const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_item);
        __syncthreads();
        if (it >= b.nitems) break;
        const WorkItem wi = uniform_load(&b.items[it]);
        const VolDesc a = uniform_load(&b.vols[wi.vol]);
        const uint32_t ntiles = (uint32_t)a.tiles_x * (uint32_t)a.tiles_y;
        rp_tile<C>(a, b.wpool + a.woff, (int)(wi.lid % ntiles), (int)(wi.lid / ntiles), lds, epi, tab);
        // the next item's staging reuses the LDS buffers
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&b.counters[1], 1u) == gridDim.x - 1) {
            atomicExch(&b.counters[0], 0u);
            atomicExch(&b.counters[1], 0u);
        }
    }
}

template <class C>
ClassGeom rp_geom()
{
    ClassGeom g;
    g.tx = C::TX;
    g.ty = C::TY;
    g.tz_min = 4 * (2 * C::R + 1);
    return g;
}

template <class C>
hipError_t rp_launch(const FilterJob& j, hipStream_t s)
{
    ClassGeom g;
    g.tx = C::TX;
    g.ty = C::TY;
    g.tz_min = 1;
    const int RX = j.roi[3] - j.roi[0], RY = j.roi[4] - j.roi[1], RZ = j.roi[5] - j.roi[2];
    const int64_t ntiles = (int64_t)tiles_along(RX, g.tx) * tiles_along(RY, g.ty);
    const void* fn = (const void*)&filter_mfma_rp_kernel<C>;
    // Slots of the plan: two workgroups per CU keep the matrix cores busy except
    // for uint8 (2 products); planned for the third that fits, 1024^3 float32
    // 7^3 gets three slabs instead of one and takes 2.94 ms instead of 2.75
    int slots = resident_wgs(fn);
    if (!std::is_same<typename C::Tin, uint8_t>::value) slots = std::min(slots, 2 * device_cus());
    // (slabs as deep as one round of resident workgroups allows: 1024^3 7^3
    // 3.24 ms with slabs capped at 128 planes, 3.09 ms uncapped)
    const int tz = plan_tz(ntiles, RZ, j.k, 1, 1 << 20, slots, 1);
    const VolDesc a = make_desc(j, tz, g);
    const int64_t nb = ntiles * ((RZ + tz - 1) / tz);
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((filter_mfma_rp_kernel<C>), dim3((unsigned)nb), dim3(kNT), 0, s, a, j.wf,
                       (uint32_t)nb);
    return hipGetLastError();
}

template <typename T, int PM>
hipError_t rp_dispatch(const FilterJob& j, hipStream_t s)
{
    if (j.k == 5) return rp_launch<RpCfg<T, 5, PM>>(j, s);
    if constexpr (PM == kF32x3) {
        if (j.k == 7) return rp_launch<RpCfg<T, 7, PM>>(j, s);
    }
    return hipErrorInvalidValue;
}

template <typename T, int PM>
const void* rp_batched(int k)
{
    if (k == 5) return (const void*)&filter_mfma_rp_batched_kernel<RpCfg<T, 5, PM>>;
    if constexpr (PM == kF32x3) {
        if (k == 7) return (const void*)&filter_mfma_rp_batched_kernel<RpCfg<T, 7, PM>>;
    }
    return nullptr;
}

template <typename T, int PM>
ClassGeom rp_geom_k(int k)
{
    if (k == 5) return rp_geom<RpCfg<T, 5, PM>>();
    if constexpr (PM == kF32x3) {
        if (k == 7) return rp_geom<RpCfg<T, 7, PM>>();
    }
    return ClassGeom{};
}

}  // namespace

const void* mfma_batched_kernel_rp(vktDataFormat f, int k, bool six_products)
{
    switch (f) {
    case vktDataFormatUInt8: return rp_batched<uint8_t, kU8>(k);
    case vktDataFormatUInt16: return rp_batched<uint16_t, kU16>(k);
    case vktDataFormatFloat32:
        return six_products ? rp_batched<float, kF32x6>(k) : rp_batched<float, kF32x3>(k);
    }
    return nullptr;
}

ClassGeom mfma_geom_rp(vktDataFormat f, int k, bool six_products)
{
    switch (f) {
    case vktDataFormatUInt8: return rp_geom_k<uint8_t, kU8>(k);
    case vktDataFormatUInt16: return rp_geom_k<uint16_t, kU16>(k);
    case vktDataFormatFloat32:
        return six_products ? rp_geom_k<float, kF32x6>(k) : rp_geom_k<float, kF32x3>(k);
    }
    return ClassGeom{};
}

hipError_t launch_filter_mfma_rp(const FilterJob& j, bool six_products, hipStream_t s)
{
    switch (j.fmt) {
    case vktDataFormatUInt8: return rp_dispatch<uint8_t, kU8>(j, s);
    case vktDataFormatUInt16: return rp_dispatch<uint16_t, kU16>(j, s);
    case vktDataFormatFloat32:
        return six_products ? rp_dispatch<float, kF32x6>(j, s) : rp_dispatch<float, kF32x3>(j, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace vkt
