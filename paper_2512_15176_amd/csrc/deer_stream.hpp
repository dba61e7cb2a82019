// GEMMs with columns enough that K need not be shared among waves: the expert projections of a mixture and the LM heads of up
// to two row tiles.
//
// A wave owns C 32-column blocks over the whole of K.  Its weights, which no other wave needs, go straight to registers, eight
// k-steps ahead; the activations, which all waves of a workgroup need, go through the LDS in stages of four k-steps, with one
// barrier per stage.  The products are taken as W^T X^T: a lane then holds 16 columns of a block for one row, and the
// epilogues run from registers.  Against the streaming kernel of deer_kernels.hpp (K in eighths over eight waves) there is no sum
// of waves through the LDS, several workgroups fit a compute unit, and one's first loads and epilogue run under the others'
// streams.
#pragma once
#include "deer_block.hpp"

namespace deer {

constexpr int SK = 4;   // k-steps per stage: every contraction here is a multiple (d_model of 128, expert widths of 64)
template <int MT> struct StreamRing { uint4 x[3][SK][2 * MT][64]; };   // [stage][k-step][row tiles hi, then lo][lane]

// acc[mt][c] += (columns of block c)^T x (row tile mt)^T over nq stages; NW waves, this is wave w; lo: lane * 16.
// wp[c]: the blocks; xb[i] + lane offset: this wave's fragments of stage 0 (fragment f = w * XP + i: k-step f / (2 MT), plane f
// % (2 MT)); lane_offset: called behind the first weights' requests, with 4 C + `extra` loads in flight at most.
// The sums are folded as in block_loop (see BK_SHORT).  Ends with every LDS read of this wave done and no loads in flight.
template <int NW, int MT, int C, bool SHORT, bool ONCE, typename F>
__device__ __forceinline__ void stream_loop(f32x16 (&acc)[MT][C], const uint4 *(&wp)[C], const char *(&xb)[SK * 2 * MT / NW], StreamRing<MT> &ring,
                                            int nq, int fold, int w, uint32_t lo, F lane_offset) {
    constexpr int P = 2 * MT, XP = SK * P / NW, LPS = XP + SK * C;   // planes; fragments of X, loads per wave and stage
    static_assert(SK * P % NW == 0 && 2 * LPS <= 63, "the counter of loads in flight has six bits");
    // (a path around the loop would leave the first requests unused, their registers in other hands while the data is on its way)
    __builtin_assume(nq >= 1);
    u32x4 wb[2][SK][C];
    auto request_w = [&](auto set_c, auto j_c) {
        constexpr int set = decltype(set_c)::value, j = decltype(j_c)::value;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            load16_async<j * 1024, ONCE>(wb[set][j][c], wp[c], lo);
            if (j == SK - 1) wp[c] += SK * 64;
        }
    };
    auto request_w4 = [&](auto set_c) {
        request_w(set_c, std::integral_constant<int, 0>{}); request_w(set_c, std::integral_constant<int, 1>{});
        request_w(set_c, std::integral_constant<int, 2>{}); request_w(set_c, std::integral_constant<int, 3>{});
    };
    request_w4(std::integral_constant<int, 0>{});
    const uint32_t vo = lane_offset();
    auto request_x = [&](int slot, int q) {
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            const char *p = xb[i] + (size_t)q * (SK * 1024);
            asm volatile("" : "+s"(p));   // a scalar address
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)(p + vo),
                                             (void __attribute__((address_space(3))) *)(&ring.x[slot][0][0][0] + (w * XP + i) * 64), 16, 0, 0);
        }
    };
    request_x(0, 0);
    if (nq > 1) {
        request_x(1, 1);
        request_w4(std::integral_constant<int, 1>{});
    }
    f32x16 sum[MT][C];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) { acc[mt][c][r] = 0.f; sum[mt][c][r] = 0.f; }
    int slot = 0;
    auto stage = [&](auto set_c, int q) {
        constexpr int set = decltype(set_c)::value;
        if (q > 0 && q % fold == 0) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float s = sum[mt][c][r], v = acc[mt][c][r], t = s + v;
                        sum[mt][c][r] = t;
                        acc[mt][c][r] = SHORT ? __builtin_amdgcn_fmed3f(v - (t - s), -3.4028234e38f, 3.4028234e38f) : 0.f;
                        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (registers)
                    }
        }
        if (q + 1 < nq) wait_loads<LPS>(); else wait_loads<0>();   // stage q has landed
#pragma unroll
        for (int j = 0; j < SK; ++j)
#pragma unroll
            for (int c = 0; c < C; ++c) tie(wb[set][j][c]);
        barrier_keep_loads();   // everybody's share of it has, and everybody has read stage q - 1
        const bool more = q + 2 < nq;
        if (more) request_x(slot == 0 ? 2 : slot - 1, q + 2);
        const uint32_t xa = lds_addr32(&ring) + slot * (SK * P * 1024) + lo;
        u32x4 x[2][P];
        lds_frags<0>(x[0], xa, std::make_integer_sequence<int, P>{});
        auto step = [&](auto j_c) {
            constexpr int j = decltype(j_c)::value;
            if constexpr (j + 1 < SK) lds_frags<(j + 1) * P * 1024>(x[(j + 1) & 1], xa, std::make_integer_sequence<int, P>{});
            wait_lds<j + 1 < SK ? P : 0>();
#pragma unroll
            for (int p = 0; p < P; ++p) tie(x[j & 1][p]);
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int c = 0; c < C; ++c) acc[p % MT][c] = mfma32(wb[set][j][c], x[j & 1][p], acc[p % MT][c]);
            if (more) request_w(set_c, j_c);
        };
        step(std::integral_constant<int, 0>{}); step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 3>{});
        slot = slot == 2 ? 0 : slot + 1;
    };
    for (int q = 0; q < nq; q += 2) {
        stage(std::integral_constant<int, 0>{}, q);
        if (q + 1 < nq) stage(std::integral_constant<int, 1>{}, q + 1);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mt][c][r] += sum[mt][c][r];
}

// SiLU(gate) * up of 32 channels of one row tile, from the accumulators of their two blocks (lane (row, half) holds columns 8 q + 4 half
// .. + 3 of a block in registers 4 q ..), into activation tile `tile` of F channels: channels 32 unit ..
__device__ __forceinline__ void stream_swiglu(uint4 *ahi, uint4 *alo, int F, const f32x16 &gate, const f32x16 &up, float rs, int tile, int unit, int row, int half) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float ge = gate[4 * q + e] * rs;
            v[e] = ge / (1.f + expf(-ge)) * (up[4 * q + e] * rs);
        }
        const uint32_t h0 = f2bf2(v[0], v[1]), h1 = f2bf2(v[2], v[3]);
        const uint32_t l0 = f2bf2(v[0] - __uint_as_float(h0 << 16), v[1] - __uint_as_float(h0 & 0xffff0000u));
        const uint32_t l1 = f2bf2(v[2] - __uint_as_float(h1 << 16), v[3] - __uint_as_float(h1 & 0xffff0000u));
        const size_t vec = (size_t)tile * (F / 16) * 64 + frag_vec(row, unit * 4 + q);
        ((uint2 *)(ahi + vec))[half] = make_uint2(h0, h1);
        ((uint2 *)(alo + vec))[half] = make_uint2(l0, l1);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Grouped expert GEMMs of passes with few rows per expert, where the expert weights' stream is all there is.  A workgroup owns
// 256 columns of one item of k_moe_group and multiplies up to 32 of its pairs at a time (items have 32 unless the blocked kernel
// takes the down projection: all rows to the same 8 of 128 experts, layer of 2048 x 768, gate/up and down of 2, 4, 6, 8 row tiles in items of 64
// 61 + 26, 66 + 45, 93 + 49, 125 + 52 us, of 32 36 + 17, 63 + 28, 71 + 38, 77 + 42); a wave has 64 of the columns, of
// gate/up the gate and the up block of 32 channels.  Gate/up gathers its rows out of the pass's fragments (lanes past the last
// pair repeat it).
// Bound: HBM.  Layer of 128 experts, top 8, d = 2048, expert width 768, means in a trace of whole decoding passes (in a sweep of three
// layers, see MOE_GATEUP_PAIRS, 3 to 5 % less), microseconds before -> now: gate/up (the streaming
// kernel, two column groups per workgroup) at 1 row tile, 111 experts or 698 MB, 125 -> 116 (6.0 TB/s), at 4 row tiles, 805 MB,
// 160 -> 139; down (k_moe_block: two row tiles of products and LDS for one to eight pairs, 36 KB of
// weights on their way per compute unit against 96 to 192 here) 72 -> 60 and 80 -> 70.  Three workgroups per compute unit; with
// two 2 % slower.
template <int MODE, bool SHORT>
__global__ __launch_bounds__(256, 3) void k_gemm_moe(const MoeArgs a, int ncb) {
    __shared__ __attribute__((aligned(16))) StreamRing<1> ring;
    const int total = a.items[0].x * ncb, per8 = (total + 7) >> 3;
    const int lin = blockIdx.x, i = (lin & 7) * per8 + (lin >> 3);
    if ((lin >> 3) >= per8 || i >= total) return;
    const int item = __builtin_amdgcn_readfirstlane(i / opaque_s(ncb)), cb = i - item * ncb;
    const int4 it = a.items[1 + item];
    const int ex = it.x, n_all = it.z;
    const int w = __builtin_amdgcn_readfirstlane(opaque_tid() >> 6);
    const int KS = a.KS;
    const int unit = cb * 4 + w, units = a.N / 64;   // this wave's 64 columns; past the matrix: the last ones again, not stored
    const int uu = min(unit, units - 1);
    const int b0 = MODE == MOE_GATEUP ? (uu >> 1) * 4 + (uu & 1) : 2 * uu, b1 = MODE == MOE_GATEUP ? b0 + 2 : b0 + 1;
    const uint4 *we = a.W + (size_t)ex * a.wexp_stride;
#pragma unroll 1
    for (int first = 0; first < n_all; first += 32) {   // row tiles of an item of 64 (the second one finds the weights in the L2)
        const int n = min(32, n_all - first), at = it.w + (first >> 5);
        const int *pairs = a.pairs + (size_t)ex * a.cap + it.y + first;
        const uint32_t lo = (opaque_tid() & 63) * 16;
        float pr_f;
        if (MODE == MOE_GATEUP) load4_async(pr_f, pairs + min((int)(lo >> 4) & 31, n - 1));
        const uint4 *wp[2] = {we + (size_t)b0 * KS * 64, we + (size_t)b1 * KS * 64};
        const size_t xo = ((MODE == MOE_GATEUP ? 0 : (size_t)at * KS) + w) * 1024;
        const char *xb[2] = {(const char *)a.Xhi + xo, (const char *)a.Xlo + xo};
        f32x16 acc[1][2];
        stream_loop<4, 1, 2, SHORT, true>(acc, wp, xb, ring, KS / SK, (a.eighths ? KS / 8 : block_fold(KS)) / SK, w, lo, [&]() -> uint32_t {
            if (MODE == MOE_DOWN) return lo;
            wait_loads<2 * SK>();
            tie(pr_f);
            const int pr = __float_as_int(pr_f) >> 3;   // this lane's row
            return (uint32_t)(pr >> 5) * (uint32_t)KS * 1024u + (pr & 31) * 16 + (lo & 512);
        });
        const int lane = opaque_tid() & 63, half = lane >> 5, row = lane & 31;
        if (MODE == MOE_GATEUP) {
            const int r = pairs[min(row, n - 1)] >> 3;
            float rs;
            if (a.eighths) {   // (in order, as that kernel did)
                const float *p = a.ssq_in + (size_t)r * a.ncg_in;
                float ss = 0.f;
#pragma unroll 4
                for (int g = 0; g < a.ncg_in; ++g) ss += p[g];
                rs = rsqrtf(ss / (float)a.d_in + a.eps);
            } else rs = wave_rstd(a.ssq_in, r, half, a.ncg_in, a.d_in, a.eps);
            if (unit < units) stream_swiglu(a.ahi, a.alo, a.Fe, acc[0][0], acc[0][1], rs, at, unit, row, half);
        } else if (row < n && unit < units) {
            const int pr = pairs[row];
            const float g = a.route_w[pr];
            float *o = a.moe_out + (size_t)pr * a.d + (size_t)unit * 64 + 4 * half;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *(float4 *)(o + 32 * b + 8 * q) = make_float4(acc[0][b][4 * q] * g, acc[0][b][4 * q + 1] * g, acc[0][b][4 * q + 2] * g, acc[0][b][4 * q + 3] * g);
        }
        if (first + 32 < n_all) barrier_keep_loads();   // everybody has read the last stages before the next row tile's arrive
    }
}

// Grouped expert GEMMs of passes with several rows per expert: a workgroup owns up to 64 (row, expert) pairs of one expert, whose
// input rows lie gathered in its activation tiles, and 256 columns.  64 rows rather than 128: the pairs of an expert are few and
// uneven, and rows past them are multiplied for nothing.  Consecutive workgroups of an XCD take the column blocks of one item,
// then the expert's next item, whose weights are then in that L2.
// Bound: the path from the L2 (12 KB per k-step; a compute unit's loads come back in order, so that weights from HBM hold up
// activations from the L2).  Layer of 128 experts, top 8, d = 2048, expert width 768, microseconds with both operands through the
// LDS and a barrier per k-step -> here, at 16, 32, 64 row tiles: gate/up 202 -> 188, 233 -> 226, 292 -> 281; down 88 -> 89, 111 -> 108,
// 159 -> 151.
template <int MODE>
union MoeBlockSmem {
    StreamRing<2> ring;
    float4 y[4][8 * 66];   // MOE_DOWN: a wave's results of one row tile, 64 columns per row (see k_lm_head)
};

template <int MODE, bool SHORT>
__global__ __launch_bounds__(256, 2) void k_moe_block(const MoeArgs a, int ncb) {
    __shared__ __attribute__((aligned(16))) MoeBlockSmem<MODE> sm;
    const int total = a.items[0].x * ncb, per8 = (total + 7) >> 3;
    const int lin = blockIdx.x, i = (lin & 7) * per8 + (lin >> 3);
    if ((lin >> 3) >= per8 || i >= total) return;
    const int item = __builtin_amdgcn_readfirstlane(i / opaque_s(ncb)), cb = i - item * ncb;
    const int4 it = a.items[1 + item];
    const int ex = it.x, n = it.z, at = it.w;
    const int w = __builtin_amdgcn_readfirstlane(opaque_tid() >> 6);
    const int KS = a.KS;
    const int unit = cb * 4 + w, units = a.N / 64, uu = min(unit, units - 1);   // as in k_gemm_moe
    const int b0 = MODE == MOE_GATEUP ? (uu >> 1) * 4 + (uu & 1) : 2 * uu, b1 = MODE == MOE_GATEUP ? b0 + 2 : b0 + 1;
    const uint4 *we = a.W + (size_t)ex * a.wexp_stride;
    const uint4 *wp[2] = {we + (size_t)b0 * KS * 64, we + (size_t)b1 * KS * 64};
    const char *xb[4];
#pragma unroll
    for (int p = 0; p < 4; ++p)   // (a row tile without pairs repeats the first one)
        xb[p] = (const char *)(p < 2 ? a.Xhi : a.Xlo) + ((size_t)(at + min(p & 1, (n - 1) >> 5)) * KS + w) * 1024;
    const uint32_t lo = (opaque_tid() & 63) * 16;
    f32x16 acc[2][2];
    stream_loop<4, 2, 2, SHORT, false>(acc, wp, xb, sm.ring, KS / SK, block_fold(KS) / SK, w, lo, [&]() { return lo; });
    const int lane = opaque_tid() & 63, half = lane >> 5, row = lane & 31;
    const int *pairs = a.pairs + (size_t)ex * a.cap + it.y;
    if (MODE == MOE_DOWN) barrier_keep_loads();   // everybody has read the last stage: the results take the ring's place
    if (unit >= units) return;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        if (mt * 32 >= n) break;
        const int pr = pairs[min(mt * 32 + row, n - 1)];
        if (MODE == MOE_GATEUP) stream_swiglu(a.ahi, a.alo, a.Fe, acc[mt][0], acc[mt][1], wave_rstd(a.ssq_in, pr >> 3, half, a.ncg_in, a.d_in, a.eps), at + mt, unit, row, half);
        else {
            // float4 g = 8 b + 2 q + half of a row's 64 columns, stored as whole rows: 16 lanes per row, 4 rows at a time
            auto yi = [](int g, int r) { return (g >> 1) * 66 + (g & 1) * 33 + r; };
            const float g = a.route_w[pr];
            float4 *y = sm.y[w];
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    y[yi(8 * b + 2 * q + half, row)] = make_float4(acc[mt][b][4 * q] * g, acc[mt][b][4 * q + 1] * g, acc[mt][b][4 * q + 2] * g, acc[mt][b][4 * q + 3] * g);
            wave_lds_sync();
#pragma unroll 4
            for (int j = 0; j < 8; ++j) {
                const int r = 4 * j + (lane >> 4), p = __builtin_amdgcn_ds_bpermute(r << 2, pr);
                const float4 v = y[yi(lane & 15, r)];
                if (mt * 32 + r < n) *(float4 *)(a.moe_out + (size_t)p * a.d + (size_t)unit * 64 + 4 * (lane & 15)) = v;
            }
            wave_lds_sync();
        }
    }
}

// RMSNorm factors of the rows of nrt <= MT row tiles, by the whole workgroup
template <int NW, int MT>
__device__ __forceinline__ void stream_rstd(const GemmArgs &a, int nrt, float *rstd) {
    constexpr int TPR = 2 * NW / MT;   // threads per row
    const int tid = opaque_tid(), row = tid / TPR, j = tid % TPR;
    const float *p = a.ssq_in + (size_t)min(row, nrt * 32 - 1) * a.ncg_in;
    float s = 0.f;
    for (int g = j; g < a.ncg_in; g += TPR) s += p[g];
#pragma unroll
    for (int off = 1; off < TPR; off <<= 1) s += shx(s, off);
    if (j == 0) rstd[row] = rsqrtf(s / (float)a.d_in + a.eps);
}

// Gate/up of a dense pass of two row tiles: a workgroup has 256 columns (128 channels) and one of S shares of K.
// Bound: HBM and what a compute unit draws (12 KB per k-step); against k_gemm<2>, which draws 8 KB per k-step for half the
// columns and sums eight waves twice: 24576 x 4096 51.5 -> 49.1 us, 19456 x 2560 32.2 -> 29.3.
constexpr size_t GU_PART = 4 * 16 * 256;   // floats of a workgroup's sums: [wave][(row tile, block, quad)][lane][4]
struct GateupSmem {
    StreamRing<2> ring;
    float rstd[64];
    int last;
};
__global__ __launch_bounds__(256, 2) void k_gemm_gateup(const GemmArgs a, int ncb, int per) {   // per: stages of a share
    __shared__ __attribute__((aligned(16))) GateupSmem sm;
    const int S = a.S, s = blockIdx.x / opaque_s(ncb), cb = blockIdx.x - s * ncb;
    gemm_stamp(a, blockIdx.x, 0);
    const int w = __builtin_amdgcn_readfirstlane(opaque_tid() >> 6);
    const int KS = a.KS, q0 = s * per, n = min(per, KS / SK - q0);   // the host keeps every share non-empty
    const int unit = cb * 4 + w, units = a.N / 64, uu = min(unit, units - 1);   // as in k_gemm_moe
    const int b0 = (uu >> 1) * 4 + (uu & 1);
    const uint4 *wp[2] = {a.W + ((size_t)b0 * KS + q0 * SK) * 64, a.W + ((size_t)(b0 + 2) * KS + q0 * SK) * 64};
    const char *xb[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) xb[p] = (const char *)(p < 2 ? a.Xhi : a.Xlo) + ((size_t)(p & 1) * KS + q0 * SK + w) * 1024;
    const uint32_t lo = (opaque_tid() & 63) * 16;
    f32x16 acc[2][2];
    stream_loop<4, 2, 2, false, true>(acc, wp, xb, sm.ring, n, block_fold(KS) / SK, w, lo, [&]() -> uint32_t { stream_rstd<4, 2>(a, 2, sm.rstd); return lo; });
    gemm_stamp(a, blockIdx.x, 1);
    const int lane = opaque_tid() & 63, half = lane >> 5, row = lane & 31;
    if (S > 1) {
        float *p0 = a.part + (size_t)w * (16 * 256) + lane * 4, *pw = p0 + ((size_t)s * ncb + cb) * GU_PART;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const f32x16 &v = acc[i >> 3][(i >> 2) & 1];
            store16_agent(pw + i * 256, v[4 * (i & 3)], v[4 * (i & 3) + 1], v[4 * (i & 3) + 2], v[4 * (i & 3) + 3]);
        }
        gemm_stamp(a, blockIdx.x, 2);
        const bool last = arrive_last(a.counters + cb, S, &sm.last);
        gemm_stamp(a, blockIdx.x, 3);
        if (!last) return;
        f32x16 sum[2][2] = {};   // the shares in their order, whoever sums them
        for (int u = 0; u < S; ++u) {
            u32x4 v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) load16_agent_async(v[i], p0 + ((size_t)u * ncb + cb) * GU_PART + i * 256);
            wait_loads<0>();
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                tie(v[i]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = __uint_as_float(v[i][e]);
                    sum[i >> 3][(i >> 2) & 1][4 * (i & 3) + e] = u == 0 ? x : sum[i >> 3][(i >> 2) & 1][4 * (i & 3) + e] + x;
                }
            }
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int c = 0; c < 2; ++c) acc[mt][c] = sum[mt][c];
    } else barrier_keep_loads();   // the RMSNorm factors are there (with shares: behind arrive_last)
    if (unit >= units) return;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) stream_swiglu(a.ahi, a.alo, a.F, acc[mt][0], acc[mt][1], sm.rstd[mt * 32 + row], mt, unit, row, half);
    gemm_stamp(a, blockIdx.x, S > 1 ? 4 : 2);
}

// LM head of a pass of nrt <= MT row tiles with logits: a workgroup has 256 columns, i.e. two of the column groups whose
// (row, group) results k_rowstat_final merges.
// Bound: HBM, and behind it the epilogues of the last workgroups.  151936 columns, microseconds in the streaming kernel (one
// workgroup of eight waves at a time on a compute unit) -> here, one row tile: d = 896 66 -> 56 (greedy), 85 -> 65 (drawing), 2048
// 129 -> 121, 2560 155 -> 146, 4096 237 -> 229; two row tiles: 92 -> 70, 127 -> 97, 158 -> 132, 192 -> 158, 283 -> 237.  Four row tiles
// in workgroups of eight waves with 32 columns each: 118 (drawing 180), 200, 240, 371 against 113 (160), 197, 240, 363 in k_gemm_block,
// which therefore keeps passes of more than two.  (Up to 32768 columns the streaming kernel is faster: see launch_gemm.)
template <int NW, int MT, int C>
struct LmHeadSmem {
    union {
        StreamRing<MT> ring;
        float4 z[NW][4 * C * 66];                    // a wave's scaled logits of one row tile: see zi
    };
    float rstd[MT * 32];
    struct { float m; int idx; float gm; int gidx; } best[MT][NW][32];
    float se[MT][NW][32];
};

template <int NW, int MT, int C, bool SHORT, int WPE>
__global__ __launch_bounds__(NW * 64, WPE) void k_lm_head(const GemmArgs a, int nrt) {
    __shared__ __attribute__((aligned(16))) LmHeadSmem<NW, MT, C> sm;
    static_assert(NW * C % 4 == 0, "whole column groups");
    constexpr int XP = SK * 2 * MT / NW, G = 4 / C;   // G: waves of a column group
    const int w = __builtin_amdgcn_readfirstlane(opaque_tid() >> 6);
    const int KS = a.KS, V = a.N;
    gemm_stamp(a, blockIdx.x, 0);
    const int unit = blockIdx.x * NW + w, units = V / (32 * C);   // this wave's columns; past the matrix: the last ones again, not stored
    const uint32_t lo = (opaque_tid() & 63) * 16;
    const uint4 *wp[C];
#pragma unroll
    for (int c = 0; c < C; ++c) wp[c] = a.W + (size_t)(min(unit, units - 1) * C + c) * KS * 64;
    const char *xb[XP];
#pragma unroll
    for (int i = 0; i < XP; ++i) {
        const int f = w * XP + i, ks = f / (2 * MT), p = f % (2 * MT), t = min(p % MT, nrt - 1);   // (a row tile that is not there: the last one again)
        xb[i] = (const char *)(p < MT ? a.Xhi : a.Xlo) + ((size_t)t * KS + ks) * 1024;
    }
    f32x16 acc[MT][C];
    stream_loop<NW, MT, C, SHORT, true>(acc, wp, xb, sm.ring, KS / SK, block_fold(KS) / SK, w, lo, [&]() -> uint32_t {
        stream_rstd<NW, MT>(a, nrt, sm.rstd);   // behind the requests of the first weights
        return lo;
    });
    gemm_stamp(a, blockIdx.x, 1);
    barrier_keep_loads();   // everybody has read the last stage: the logits take the ring's place
    const int lane = opaque_tid() & 63, half = lane >> 5, row = lane & 31;
    const float T = a.T, invT = T > 0.f ? 1.f / T : 1.f;
    const int col0 = unit * 32 * C + 4 * half;   // float4 i of the lane: columns col0 + 32 (i / 4) + 8 (i % 4) .. + 3
    // float4 g = 8 c + 2 q + half of a row's 32 C columns; padded so that 16 neighbours of one row lie in different banks
    auto zi = [](int g, int r) { return (g >> 1) * 66 + (g & 1) * 33 + r; };
    float4 *zs = sm.z[w];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (mt >= nrt) break;
        const int lm = mt * 32 + row;
        const bool live = lm < a.n_lm && lm % opaque_s(a.k) >= a.k_lo && unit < units;
        const float rs = sm.rstd[lm];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                zs[zi(8 * c + 2 * q + half, row)] = make_float4(acc[mt][c][4 * q] * rs, acc[mt][c][4 * q + 1] * rs, acc[mt][c][4 * q + 2] * rs, acc[mt][c][4 * q + 3] * rs);
        wave_lds_sync();
        if (a.logits) {   // whole lines: 8 C lanes store a row's 32 C columns (16 bytes here and there of 128 of them cost 8 to 15 us more)
            constexpr int LR = 8 * C, RI = 64 / LR;   // lanes per row, rows per store
            const uint32_t rows = (uint32_t)__ballot(live);   // (lanes 0 .. 31: the rows)
            float *o = a.logits + (size_t)(mt * 32 + lane / LR) * V + (size_t)unit * (32 * C) + 4 * (lane % LR);
#pragma unroll 2
            for (int i = 0; i < 32 / RI; ++i) {
                const int r = RI * i + lane / LR;
                const float4 z = zs[zi(lane % LR, r)];
                if (rows >> r & 1) *(float4 *)(o + (size_t)(RI * i) * V) = z;
            }
        }
        float m = -INFINITY, gm = -INFINITY;
        int idx = 0x7fffffff, gidx = 0x7fffffff;
        if (live) {
#pragma unroll 2
            for (int i = 0; i < 4 * C; ++i) {   // (short loops: a launch reads its code anew)
                const float4 z = zs[zi(2 * i + half, row)];
                const int v = col0 + 32 * (i >> 2) + 8 * (i & 3);
                argmax_merge(m, idx, z.x, v); argmax_merge(m, idx, z.y, v + 1); argmax_merge(m, idx, z.z, v + 2); argmax_merge(m, idx, z.w, v + 3);
            }
            if (T > 0.f && a.draw) {
                const uint64_t key = row_key(a.seed, TAG_DRAFT, (uint64_t)a.rm.seq[lm], (uint64_t)a.rm.pos[lm]);
#pragma unroll 2
                for (int e = 0; e < 16 * C; ++e) {
                    const int v = col0 + 32 * (e >> 4) + 8 * ((e >> 2) & 3) + (e & 3);
                    argmax_merge(gm, gidx, ((const float *)(zs + zi(2 * (e >> 2) + half, row)))[e & 3] * invT + gumbel(key, (uint64_t)v), v);
                }
            }
        }
        {
            const float m2 = shx(m, 32); const int i2 = shx(idx, 32);
            argmax_merge(m, idx, m2, i2);
            const float g2 = shx(gm, 32); const int gi2 = shx(gidx, 32);
            argmax_merge(gm, gidx, g2, gi2);
        }
        if (half == 0) sm.best[mt][w][row] = {m, idx, gm, gidx};
        barrier_keep_loads();
#pragma unroll
        for (int j = 0; j < G; ++j) {   // the group's
            const auto b = sm.best[mt][w / G * G + j][row];
            argmax_merge(m, idx, b.m, b.idx);
            argmax_merge(gm, gidx, b.gm, b.gidx);
        }
        float se = 0.f;
        if (T > 0.f) {
            if (live) {
#pragma unroll 2
                for (int i = 0; i < 4 * C; ++i) {
                    const float4 z = zs[zi(2 * i + half, row)];
                    se += expf((z.x - m) * invT); se += expf((z.y - m) * invT); se += expf((z.z - m) * invT); se += expf((z.w - m) * invT);
                }
            }
            se += shx(se, 32);
            if (half == 0) sm.se[mt][w][row] = se;
            barrier_keep_loads();
            se = 0.f;
#pragma unroll
            for (int j = 0; j < G; ++j) se += sm.se[mt][w / G * G + j][row];
        }
        if (live && half == 0 && w % G == 0) a.stat[(size_t)lm * a.ncg_v + unit / G] = RowStat{m, idx, se, gm, gidx};
    }
    gemm_stamp(a, blockIdx.x, 2);
}

}  // namespace deer
