// vkt_filter_mfma.hip -- ApplyFilter for filters of size k >= 5 on the
// matrix cores: an implicit GEMM with split 16-bit operands and FP32
// accumulation.  This file is compiled twice: with VKT_MFMA_SHAPE=16 for
// k <= 7 (16x16x32 tiles, accumulators in VGPRs) and with VKT_MFMA_SHAPE=32
// for k >= 9 (32x32x16 tiles).
//
// Operation (paper Sec. 3.2 "Volume Manipulation"; benchmarked as a Gaussian
// blur, Sec. 4.3):
//   T(x,y,z) = sum_{a,b,c} w[a + k(b + k c)] * s(A(x+a-r), A(y+b-r), A(z+c-r)).
//
// GEMM embedding, per input plane zi (D += A * B on MFMA tiles):
//   M (rows i)    : consecutive output rows y_i of one x-strip of NX output
//                   columns (3 for k = 5 and float32 k = 9, else 2; 2 for k = 5
//                   on the short tile of small volumes),
//   K (reduction) : (filter row b, input column ax) pairs; the A operand is
//                   the input window s(x_s - r + ax, y_i + b - r, zi), read
//                   straight from the LDS-staged plane (no im2col copy),
//   N (columns j) : (filter plane c, output x-offset xo), j = c * NX + xo;
//                   B[(b, ax)][(c, xo)] = w[c][b][ax - xo] (an x-Toeplitz band
//                   of each filter row, zero outside 0 <= ax - xo < k).
// Column group c of D therefore accumulates the contribution of input plane
// zi to output plane zi - c + r: the k output planes an input plane feeds
// live side by side in D (a z ring).  On 16x16 tiles the finished group
// c = k-1 is stored after each plane and the columns shift by NX lanes.  On
// 32x32 tiles the accumulators stay (group s holds output plane s mod k of the
// slab) and the weights turn: a lane reads the weights of the next filter
// plane from a table in LDS.  Moving them instead took 64 ds_bpermute a plane
// and wave behind the last product and kept the weights in registers (11^3
// uint16 224 registers, now 152; 1024^3 15.25 -> 14.85 ms, 400x380x360 13^3
// 1.15 -> 1.06 ms, 200x190x181 float32 15^3 with 6 products 484 -> 429 us).
//
// The four x-strips a wave owns are adjacent, so one segment read per (row
// block, K chunk, operand piece) holds all their 16-byte windows.  With three
// columns a strip the k = 5 tiles fill 15 of 16 columns instead of 10: a third
// fewer products.  (The sum of 8 adjacent reduction slots does not depend on
// their order -- checked on the GPU with permuted slots -- so that this changes
// no result where a filter row lies in one such group, k <= 7; float32 k = 9
// rounds differently.)  The finished column group of all of a wave's tiles is
// transposed through LDS so that each lane rounds and stores adjacent cells of
// one row.
//
// Operand splitting: see vkt_mfma_common.h.
#include "vkt_mfma_common.h"

#include <algorithm>

#ifndef VKT_MFMA_SHAPE
#error "compile with -DVKT_MFMA_SHAPE=16 or 32"
#endif

namespace vkt {
namespace {

// MFMA tile shapes.  AXW = input columns per filter row in the K dimension,
// NACC = accumulator registers per lane.
template <int SHAPE> struct Mf;
template <> struct Mf<16> {
    static constexpr int MT = 16, NT = 16, AXW = 8, NACC = 4;
    using acc_t = f32x4;
};
template <> struct Mf<32> {
    static constexpr int MT = 32, NT = 32, AXW = 16, NACC = 16;
    using acc_t = f32x16;
};

// SYV: row blocks per workgroup (tile height variant of the batched form);
// 0 keeps the measured default below.
template <typename T, int K, int PM, int SYV = 0>
struct Cfg {
    using Tin = T;
    // the same kernel on one row block, for small volumes (16x16 tiles)
    using Short = Cfg<T, K, PM, SYV == 0 && K <= 7 ? 1 : SYV>;
    using PC = Pieces<PM>;
    static constexpr int SHAPE = K <= 7 ? 16 : 32;
    using M = Mf<SHAPE>;
    static constexpr int R = (K - 1) / 2;
    // output columns per strip (two on the short 16x16 tile: 32 columns, not 48,
    // for small volumes)
    static constexpr int NX =
        (K == 5 && SYV != 1) || (K == 9 && std::is_same<T, float>::value) ? 3 : 2;
    static_assert(K * NX <= M::NT, "column groups exceed the tile");
    static_assert(NX + K - 1 <= M::AXW, "x window exceeds the K slots");
    static constexpr int NCH = SHAPE == 16 ? (K + 3) / 4 : K;      // K chunks
    static constexpr int SX = 16;                                   // strips per workgroup
    static constexpr int WS = 4;                                    // strips per wave
    static_assert(SX == 4 * WS, "four waves");
    // row blocks per workgroup: two 16-row blocks (one for small volumes: Short;
    // with four the kernels needed a third more registers, two waves per SIMD
    // instead of three or four, and measured 5-8 % slower), one 32-row block.
    // PIPE: segment reads of the next (row block, K chunk) group issued before the
    // current group's products: on 16x16 tiles, for uint16 and for 3-product
    // float32 9^3 (no spills; with two-column strips 1024^3 12.45 -> 11.77 ms,
    // 512^3 1.66 -> 1.58 ms, bit-identical).  The other 32x32 kernels read each
    // group's segments just before its products: uint8 9^3 / 11^3 measured 1 %
    // slower pipelined, float32 11^3 the same, and 6-product float32 spilled (all
    // three measured with the weights in registers).
    static constexpr bool PIPE = SHAPE == 16 || std::is_same<T, uint16_t>::value ||
                                 (std::is_same<T, float>::value && PM != kF32x6 && K <= 9);
    static constexpr int SY_DEFAULT = SHAPE == 16 ? 2 : 1;
    static constexpr int SY = SYV ? SYV : SY_DEFAULT;
    static constexpr int TX = SX * NX, TY = SY * M::MT;
    static constexpr int WX = WS * NX;                              // columns per wave
    // dwords of a lane's segment: the 8-column windows of the wave's strips,
    // read 8 bytes (24-byte wave offsets) or 16 bytes at a time
    static constexpr int RD = WX % 8 == 0 ? 4 : 2;
    static constexpr int SEGD = ((NX * (WS - 1) + 8 + 1) / 2 + RD - 1) / RD * RD;
    // staged columns, and the row pitch: for 8-byte reads and for k = 7 an odd
    // number of reads, which spreads the segment reads of consecutive rows over the
    // LDS banks.  The other kernels with 16-byte reads keep 48 columns, 6 reads (11^3
    // uint16: bank conflicts add 66 % to the LDS cycles, under products that keep the
    // matrix cores 81 % busy)
    static constexpr int COLS = (3 * WX + (SHAPE == 16 ? 0 : 8) + 2 * SEGD + 7) / 8 * 8;
    static constexpr int PITCH = RD == 2 ? (COLS % 8 == 0 ? COLS + 4 : COLS) : COLS;
    static_assert(TX + K - 1 <= COLS && PITCH * 2 % (4 * RD) == 0, "staged columns");
    static constexpr int HY = TY + K - 1;                           // staged rows
    static constexpr int PLANE = (HY * PITCH + 7) / 8 * 8;
    static __device__ constexpr int at(int row, int col) { return row * PITCH + col; }
    // 32x32 tiles: weight table in LDS, per (chunk, piece, lane half) the
    // 16-byte rows of (c, xo), then a zero row for the unused columns
    static constexpr int BROWS = K * NX + 1;
    static constexpr int TABLE = SHAPE == 16 ? 8 : NCH * PC::NBI * 2 * BROWS * 8;
    // output block of a wave: WX x BY cells, CPL of a row per lane
    static constexpr int BY = SY * M::MT, CPL = WX * BY / 64;
    static constexpr int MTW = WS * SY;                             // M tiles per wave
    // waves per SIMD that the single-volume kernel has to reach: four for 16x16
    // tiles with uint8 or 3-product float32 operands (82 to 128 registers; uint16
    // gets there by itself with 102 to 128), three for 6-product float32 (132 to
    // 166), two for 32x32 tiles (116 to 176 registers: two to four waves).  None of
    // them spills.
    static constexpr int WAVES =
        SHAPE == 16 ? (PM == kU8 || PM == kF32x3 ? 4 : 3) : 2;
    // the persistent batched kernels need some 30 registers more: three waves for
    // the 16-bit operand classes (134 to 158 on the default tile), the float32
    // classes as they come (two or three waves); no spills there either
    static constexpr int BWAVES = SHAPE == 16 && (PM == kU8 || PM == kU16) ? 3 : 1;
};

template <int SHAPE, bool F16>
__device__ inline typename Mf<SHAPE>::acc_t mfma(u32x4 a, u16x8 b, typename Mf<SHAPE>::acc_t c)
{
    if constexpr (SHAPE == 16) {
        if constexpr (F16)
            return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                          __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                           __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    } else {
        if constexpr (F16)
            return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                          __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                           __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
}

// Shift the accumulator columns of a 16x16 tile right by NX lanes; the first
// NX columns become zero (DPP row_shr:NX inside each row of 16 lanes;
// bound_ctrl writes 0).
template <int NX>
__device__ inline float shift_cols(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x110 + NX, 0xf, 0xf, true));
}

template <class C>
__device__ void mfma_tile(const VolDesc& a, const float* __restrict__ w, int tile, int slab,
                          uint16_t* lds_base, float* epi, uint16_t* tab)
{
    using T = typename C::Tin;
    using PC = typename C::PC;
    using M = typename C::M;
    using acc_t = typename M::acc_t;
    constexpr int K = (C::R * 2) + 1;
    constexpr int R = C::R;
    constexpr int NX = C::NX;
    constexpr int PM = std::is_same<T, uint8_t>::value ? kU8
                       : std::is_same<T, uint16_t>::value ? kU16
                       : (PC::NPROD == 6 ? kF32x6 : kF32x3);
    constexpr bool TURN = C::SHAPE == 32;  // the weights turn, the accumulators stay
    // lds[buffer][piece][C::at(row, column)]
    auto lds = reinterpret_cast<uint16_t(*)[PC::PS][C::PLANE]>(lds_base);

    const int t = threadIdx.x, lane = t % 64, wave = t / 64;
    const int x0 = a.rx0 + (tile % a.tiles_x) * C::TX, y0 = a.ry0 + (tile / a.tiles_x) * C::TY;
    const int zb = a.rz0 + slab * a.tz, ze = min(zb + a.tz, a.rz1);
    const int64_t plane = (int64_t)a.X * a.Y;
    const int32_t plane_bytes = (int32_t)(plane * (int64_t)sizeof(T));  // < 2^31 (host check)
    const int jcol = lane % M::NT, gq = lane / M::NT;

    // ---- staging of the input plane: COLS x HY cells from (x0 - r, y0 - r).  The
    // first plane's loads go out before the weights are read and split, one
    // memory latency less in front of a small volume's few planes
    // (94x91x97 float32 5^3 19.05 -> 17.6 us).
    const int zi_beg = zb - R, zi_end = ze + R;
    PlaneStage<T, R, C::HY, C::COLS, kNT, C> in;
    in.init(a, x0, y0, t);
    in.gather(a, zi_beg);

    // ---- B operand: x-Toeplitz band of each filter row, split into pieces;
    // b: filter row, ax0: the first of its 8 input columns
    auto weights = [&](int c, int xo, int b, int ax0, u16x8 (&v)[PC::NBI]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int aa = ax0 + e - xo;
            float wv = 0.f;
            if (c < K && b < K && aa >= 0 && aa < K) wv = w[(c * K + b) * K + aa];
            uint16_t p[3];
            split_weight<PM>(wv, a.wscale, p);
#pragma unroll
            for (int bi = 0; bi < PC::NBI; ++bi) v[bi][e] = p[bi];
        }
    };
    u16x8 B[TURN ? 1 : C::NCH][PC::NBI];  // 16x16 tiles: all of it, in registers
    // 32x32 tiles: this lane's row of the table, moved on by a filter plane
    // (NX rows) with each input plane: group s takes filter plane
    // c = (p - s) mod k at input plane p of the slab
    int boff = 0, blast = 0, bfirst = 0;
    if constexpr (TURN) {
        for (int i = t; i < C::NCH * 2 * C::BROWS; i += kNT) {
            const int row = i % C::BROWS, g = (i / C::BROWS) % 2, q = i / (2 * C::BROWS);
            u16x8 v[PC::NBI];
            weights(row / NX, row % NX, q, 8 * g, v);
#pragma unroll
            for (int bi = 0; bi < PC::NBI; ++bi)
                *reinterpret_cast<u16x8*>(&tab[(((q * PC::NBI + bi) * 2 + g) * C::BROWS + row) * 8]) =
                    v[bi];
        }
        const int s = jcol / NX, xo = jcol % NX;
        bfirst = (gq * C::BROWS + (s < K ? xo : C::BROWS - 1)) * 8;
        blast = bfirst + (s < K ? (K - 1) * NX * 8 : 0);
        boff = bfirst + (s < K ? (K - s) % K * NX * 8 : 0);
    } else {
#pragma unroll
        for (int q = 0; q < C::NCH; ++q) weights(jcol / NX, jcol % NX, q * 4 + gq, 0, B[q]);
    }

    // staged columns past X + r meet zero weights: they hold zeros
    if (in.face) {
        for (int e = t; e < 2 * PC::PS * C::PLANE / 8; e += kNT)
            reinterpret_cast<u32x4*>(lds_base)[e] = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
    }
    auto put = [&](int buf) __attribute__((always_inline)) {
        in.put([&](const T (&v)[4], int e, bool on) __attribute__((always_inline)) {
            stage_quad<PM>(lds[buf], v, e, on);
        });
    };

    // ---- output block of the wave: its finished columns form a WX (x) by BY
    // (y) block; lanes holding a finished column write it to the wave's LDS
    // block (y fastest), then each lane reads CPL cells of one row and stores
    // them
    constexpr int BY = C::BY, CPL = C::CPL;
    float* const blk = epi + wave * C::WX * BY;
    const int lrow = lane % BY, lpart = lane / BY;
    // (columns past 2^31 - 1 wrap to negative ones, whose offsets lie past the plane)
    const int xw = (int)((uint32_t)x0 + (uint32_t)(C::WX * wave + CPL * lpart)), yl = y0 + lrow;
    // rows past the volume's last row fall beyond the plane: dropped
    const uint32_t ooff =
        yl < a.ry1 ? ((uint32_t)yl * (uint32_t)a.X + (uint32_t)xw) * (uint32_t)sizeof(T) : kOutside;
    const bool vec_row = xw <= a.rx1 - CPL;  // (buffer stores take any cell alignment)

    acc_t acc[C::MTW];
#pragma unroll
    for (int m = 0; m < C::MTW; ++m)
#pragma unroll
        for (int r = 0; r < M::NACC; ++r) acc[m][r] = 0.f;

    // lane's A-operand coordinates inside an M tile
    const int ai = lane % M::MT, ag = lane / M::MT;
    const int acol = C::WX * wave + (C::SHAPE == 16 ? 0 : 8 * ag);

    // Before plane zi's products plane zi is in LDS and the loads of plane
    // zi + 1 are in flight; it is staged after the products, and the loads of
    // plane zi + 2 take its registers at once (a whole step to arrive).
    put(0);
    in.gather(a, min(zi_beg + 1, zi_end - 1));
    __syncthreads();

    int done = TURN ? 1 : K - 1;  // column group that the next plane finishes
    for (int zi = zi_beg; zi < zi_end; ++zi) {
        const int cur = (zi - zi_beg) & 1;

        // (row block, K chunk) groups, software pipelined where C::PIPE: the
        // LDS segments (and weights) of group g + 1 are read while group g's
        // products issue
        constexpr int NG = C::SY * C::NCH;
        uint32_t seg[2][PC::PS][C::SEGD];
        u16x8 Bt[2][PC::NBI];
        auto load_seg = [&](int g, int h2) {
            const int yb = g / C::NCH, q = g % C::NCH;
            int b = C::SHAPE == 16 ? q * 4 + ag : q;
            if (b > K - 1) b = K - 1;  // zero weights there; keep A finite
            const int off = C::at(yb * M::MT + ai + b, acol);
            typedef uint32_t vrd __attribute__((ext_vector_type(C::RD)));
            // one segment per piece holds the windows of the wave's strips
#pragma unroll
            for (int ps = 0; ps < PC::PS; ++ps)
#pragma unroll
                for (int h = 0; h < C::SEGD / C::RD; ++h) {
                    const vrd v = *reinterpret_cast<const vrd*>(&lds[cur][ps][off + 2 * C::RD * h]);
#pragma unroll
                    for (int d = 0; d < C::RD; ++d) seg[h2][ps][C::RD * h + d] = v[d];
                }
            if constexpr (TURN) {
#pragma unroll
                for (int bi = 0; bi < PC::NBI; ++bi)
                    Bt[h2][bi] = *reinterpret_cast<const u16x8*>(
                        &tab[boff + (q * PC::NBI + bi) * 2 * C::BROWS * 8]);
            }
        };
        constexpr bool PIPE = C::PIPE;
        // the products at raised wave priority, higher with each third of
        // them: the wave that is ahead takes the matrix cores and ends first,
        // so that its staging and output run under another wave's products
        // (at one priority the waves of a SIMD share the matrix cores evenly
        // and end together: 1024^3 uint16 11^3 16.4 ms, rising 15.25 ms, the
        // matrix cores 70 -> 80 % busy)
        __builtin_amdgcn_s_setprio(1);
        load_seg(0, 0);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g == (NG + 2) / 3) __builtin_amdgcn_s_setprio(2);
            if (g == (2 * NG + 2) / 3) __builtin_amdgcn_s_setprio(3);
            if constexpr (PIPE) {
                if (g + 1 < NG) load_seg(g + 1, (g + 1) & 1);
                // keep those reads ahead of this group's products
                __builtin_amdgcn_sched_barrier(0);
            } else {
                if (g > 0) load_seg(g, g & 1);
            }
            const int yb = g / C::NCH, q = g % C::NCH;
            // strip s's window: the 8 cells from column NX s of the segment on
            u32x4 A[C::WS][PC::PS];
#pragma unroll
            for (int st = 0; st < C::WS; ++st)
#pragma unroll
                for (int ps = 0; ps < PC::PS; ++ps)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint32_t(&sg)[C::SEGD] = seg[g & 1][ps];
                        const int d0 = NX * st / 2 + d;
                        A[st][ps][d] = NX * st % 2
                                           ? __builtin_amdgcn_alignbit(sg[d0 + 1], sg[d0], 16)
                                           : sg[d0];
                    }
            const u16x8(&Bq)[PC::NBI] = TURN ? Bt[g & 1] : B[TURN ? 0 : q];
            // products outer, strips inner: consecutive MFMAs are independent
#pragma unroll
            for (int pr = 0; pr < PC::NPROD; ++pr)
#pragma unroll
                for (int st = 0; st < C::WS; ++st)
                    acc[yb * C::WS + st] = mfma<C::SHAPE, PC::F16>(
                        A[st][PC::prod[pr][0]], Bq[PC::prod[pr][1]], acc[yb * C::WS + st]);
        }
        if constexpr (TURN) boff = boff == blast ? bfirst : boff + NX * 8;
        // the next plane's cells are split and staged after the products
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        put(cur ^ 1);
        in.gather(a, min(zi + 2, zi_end - 1));

        // ---- column group `done` holds output plane zi - r
        const int zo = zi - R;
        const int xo = jcol - done * NX;
        const bool fin = xo >= 0 && xo < NX;
        if (zo >= zb) {
            if (fin) {
#pragma unroll
                for (int m = 0; m < C::MTW; ++m) {
                    const int yb = m / C::WS, st = m % C::WS;
                    float* col = blk + (st * NX + xo) * BY + yb * M::MT + 4 * gq;
#pragma unroll
                    for (int qd = 0; qd < M::NACC / 4; ++qd)
                        *reinterpret_cast<f32x4*>(col + 8 * qd) =
                            f32x4{acc[m][4 * qd], acc[m][4 * qd + 1], acc[m][4 * qd + 2],
                                  acc[m][4 * qd + 3]};
                }
            }
            // the wave's own LDS writes complete before its lanes read them
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            float v[CPL];
#pragma unroll
            for (int x = 0; x < CPL; ++x) v[x] = blk[(CPL * lpart + x) * BY + lrow];
            const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
                static_cast<char*>(a.dst) + (int64_t)zo * plane_bytes, (short)0, plane_bytes,
                (int)kRsrcWord3);
            store_row<T, CPL>(rd, ooff, v, vec_row, a.rx1 - xw, a.unscale);
            asm volatile("" ::: "memory");
        }
        // ---- advance the ring
        if constexpr (TURN) {
#pragma unroll
            for (int m = 0; m < C::MTW; ++m)
#pragma unroll
                for (int r = 0; r < M::NACC; ++r) acc[m][r] = fin ? 0.f : acc[m][r];
            done = done + 1 == K ? 0 : done + 1;
        } else {
#pragma unroll
            for (int m = 0; m < C::MTW; ++m)
#pragma unroll
                for (int r = 0; r < M::NACC; ++r) acc[m][r] = shift_cols<NX>(acc[m][r]);
        }
        __syncthreads();
    }
}

template <class C>
constexpr int lds_elems()
{
    return 2 * C::PC::PS * C::PLANE;
}
// output transposition blocks of the 4 waves
template <class C>
constexpr int epi_floats()
{
    return 4 * C::WX * C::BY;
}

template <class C>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(C::WAVES)))
void filter_mfma_kernel(VolDesc a,
                                                             const float* __restrict__ w,
                                                             uint32_t nblocks)
{
    __shared__ __align__(16) uint16_t lds[lds_elems<C>()];
    __shared__ __align__(16) float epi[epi_floats<C>()];
    __shared__ __align__(16) uint16_t tab[C::TABLE];
    const uint32_t lid = xcd_remap(blockIdx.x, nblocks);
    const uint32_t ntiles = (uint32_t)a.tiles_x * (uint32_t)a.tiles_y;
    mfma_tile<C>(a, w, (int)(lid % ntiles), (int)(lid / ntiles), lds, epi, tab);
}

// Persistent workgroups over a queue of (volume, tile-slab) items; the last
// workgroup to finish resets the queue counters.
template <class C>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(C::BWAVES)))
void filter_mfma_batched_kernel(BatchArgs b)
{
    __shared__ __align__(16) uint16_t lds[lds_elems<C>()];
    __shared__ __align__(16) float epi[epi_floats<C>()];
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
        mfma_tile<C>(a, b.wpool + a.woff, (int)(wi.lid % ntiles), (int)(wi.lid / ntiles), lds,
                     epi, tab);
    }
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&b.counters[1], 1u) == gridDim.x - 1) {
            atomicExch(&b.counters[0], 0u);
            atomicExch(&b.counters[1], 0u);
        }
    }
}

#if VKT_MFMA_SHAPE == 16
#define VKT_MFMA_KS(X) X(5) X(7)
#define VKT_MFMA_FN(name) name##_s16
#else
#define VKT_MFMA_KS(X) X(9) X(11) X(13) X(15)
#define VKT_MFMA_FN(name) name##_s32
#endif

template <class C>
ClassGeom geom_of()
{
    ClassGeom g;
    g.tx = C::TX;
    g.ty = C::TY;
    g.tz_min = 4 * (2 * C::R + 1);
    return g;
}

template <class C>
hipError_t launch_cfg(const FilterJob& j, hipStream_t s)
{
    const ClassGeom g = geom_of<C>();
    // the output region's tiles and z extent (the whole volume unless a range)
    const int RX = j.roi[3] - j.roi[0], RY = j.roi[4] - j.roi[1], RZ = j.roi[5] - j.roi[2];
    const int64_t ntiles = (int64_t)tiles_along(RX, g.tx) * tiles_along(RY, g.ty);
    // Volumes that do not make two workgroups per CU even with one-plane slabs
    // take the 16x16 tile of one row block: twice the workgroups, half the step
    // of each, two-column strips for k = 5 (64^3 uint8, uint16, float32 5^3 8.4,
    // 10.5 and 12.5 -> 6.9, 8.1 and 9.6 us; 40^3 7^3 9.3, 12.5 and 15 -> 7.4, 8.9
    // and 9.9 us).
    using Short = typename C::Short;
    if constexpr (!std::is_same<Short, C>::value)
        if (ntiles * RZ < 2 * (int64_t)device_cus()) return launch_cfg<Short>(j, s);
    const void* fn = (const void*)&filter_mfma_kernel<C>;
    // Slots of the plan: the workgroups that fill the device once, at most two
    // per CU, which keep the matrix cores busy; planned for the three or four
    // that fit, a small volume gets thinner slabs with more halo planes for
    // nothing (150x141x133 uint16 11^3: 157 us, for two 136 us; 144x131x127 uint8,
    // uint16 and float32 5^3 15.5, 22.3 and 34 us, for two 13.1, 18.4 and 24.6;
    // 7^3 21.8, 33.6 and 41 us, for two 17.6, 24.2 and 31.8).
    const int slots = std::min(resident_wgs(fn), 2 * device_cus());
    // (deeper slabs measured slower for the 16x16 tiles, faster for 32x32)
    const int tz = plan_tz(ntiles, RZ, j.k, 1, C::SHAPE == 16 ? 128 : 512, slots, 1);
    const VolDesc a = make_desc(j, tz, g);
    const int64_t nb = ntiles * ((RZ + tz - 1) / tz);
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((filter_mfma_kernel<C>), dim3((unsigned)nb), dim3(kNT), 0, s, a, j.wf,
                       (uint32_t)nb);
    return hipGetLastError();
}

template <typename T, int PM>
hipError_t dispatch_k(const FilterJob& j, hipStream_t s)
{
#define VKT_CASE(KK) \
    case KK: return launch_cfg<Cfg<T, KK, PM>>(j, s);
    switch (j.k) { VKT_MFMA_KS(VKT_CASE) }
#undef VKT_CASE
    return hipErrorInvalidValue;
}

// Tile-height variants of the batched kernels: 0 = the default row blocks,
// 1 = the other choice (16x16 tiles: one row block instead of two; 32x32
// tiles: two instead of one, or one instead of two).
template <typename T, int K, int PM>
constexpr int alt_sy()
{
    return Cfg<T, K, PM>::SY_DEFAULT == 2 ? 1 : 2;
}

template <typename T, int PM>
ClassGeom geom_k(int k, int variant = 0)
{
#define VKT_CASE(KK)                                                       \
    case KK:                                                               \
        return variant ? geom_of<Cfg<T, KK, PM, alt_sy<T, KK, PM>()>>()    \
                       : geom_of<Cfg<T, KK, PM>>();
    switch (k) { VKT_MFMA_KS(VKT_CASE) }
#undef VKT_CASE
    return ClassGeom{};
}

template <typename T, int PM>
const void* batched_k(int k, int variant)
{
#define VKT_CASE(KK)                                                                      \
    case KK:                                                                              \
        return variant                                                                    \
                   ? (const void*)&filter_mfma_batched_kernel<Cfg<T, KK, PM, alt_sy<T, KK, PM>()>> \
                   : (const void*)&filter_mfma_batched_kernel<Cfg<T, KK, PM>>;
    switch (k) { VKT_MFMA_KS(VKT_CASE) }
#undef VKT_CASE
    return nullptr;
}

}  // namespace

ClassGeom VKT_MFMA_FN(mfma_geom)(vktDataFormat f, int k, bool six_products, int variant)
{
    switch (f) {
    case vktDataFormatUInt8: return geom_k<uint8_t, kU8>(k, variant);
    case vktDataFormatUInt16: return geom_k<uint16_t, kU16>(k, variant);
    case vktDataFormatFloat32:
        return six_products ? geom_k<float, kF32x6>(k, variant)
                            : geom_k<float, kF32x3>(k, variant);
    }
    return ClassGeom{};
}

hipError_t VKT_MFMA_FN(launch_filter_mfma)(const FilterJob& j, bool six_products, hipStream_t s)
{
    switch (j.fmt) {
    case vktDataFormatUInt8: return dispatch_k<uint8_t, kU8>(j, s);
    case vktDataFormatUInt16: return dispatch_k<uint16_t, kU16>(j, s);
    case vktDataFormatFloat32:
        return six_products ? dispatch_k<float, kF32x6>(j, s) : dispatch_k<float, kF32x3>(j, s);
    }
    return hipErrorInvalidValue;
}

const void* VKT_MFMA_FN(mfma_batched_kernel)(vktDataFormat f, int k, bool six_products,
                                             int variant)
{
    switch (f) {
    case vktDataFormatUInt8: return batched_k<uint8_t, kU8>(k, variant);
    case vktDataFormatUInt16: return batched_k<uint16_t, kU16>(k, variant);
    case vktDataFormatFloat32:
        return six_products ? batched_k<float, kF32x6>(k, variant)
                            : batched_k<float, kF32x3>(k, variant);
    }
    return nullptr;
}

}  // namespace vkt
