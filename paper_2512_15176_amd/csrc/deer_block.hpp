// LDS-blocked GEMMs for passes of several row tiles (batches, prompts), two workgroups per compute unit.
//
// A workgroup of four waves owns 128 rows x 64 NB columns; wave (wr, wc) multiplies rows 64 wr .. + 63 and columns
// 32 NB wc .. of them (two row tiles x NB column tiles).  Both operands travel to LDS with direct-to-LDS loads, one
// k-step of 16 per stage in a ring of NST stages (a fragment is a plain 1 KB copy: operands are stored in MFMA
// register order).  Two workgroups share a compute unit, so that the barrier, the first loads and the epilogue of one run
// under the products of the other.  With S > 1 the workgroups of a tile take shares of K; their accumulators meet
// through memory as they lie in the registers, and the last to arrive sums the shares in order and runs the epilogue.
//
// Bound: the matrix cores for many row tiles (128 of them, 8B gate/up: 1.31 PFLOP/s issued, what the largest plain bf16
// product reaches on this card is 1.36), the L2 -> LDS path for few (a k-step of NB = 4 brings
// 16 KB; a compute unit gets 27 to 34 bytes per clock, 512 cycles of products need 32).  A 64 x 128 wave tile reads 8 KB of
// LDS per 16 products, which leaves the LDS half idle; 128 x 256 per workgroup needs 16 KB from L2 per 64 products
// against 32 KB in the streaming kernel's pairs of row tiles.  Measured against the kernels that did this work before
// (one 256 x 256 tile per 512 threads in lockstep; the streaming kernel), microseconds per launch, 8B widths: gate/up at
// 4 / 7 / 16 / 32 / 128 row tiles 85 / 146 / 224 / 439 / 1345 -> 71 / 117 / 192 / 326 / 1255, QKV at 16 / 64 / 128
// 83 / 247 / 503 -> 69 / 189 / 327, down at 24 / 64 196 / 621 -> 167 / 320, LM heads of 151936 columns at 16 (mean of
// d = 4096 and 896) 1348 -> 865.
#pragma once
#include "deer_kernels.hpp"

namespace deer {

constexpr int BK_RT = 4;     // row tiles per workgroup of k_gemm_block
// With 64 columns per wave the accumulators are added to a second set every few k-steps.  A matrix instruction adds its
// products to the running sum with a rounding of its own, and the relative error of a chain of n k-steps (2 n additions: hi
// and lo) grows like the square root of n.  The streaming kernel's eight waves hold an eighth of K each, and the folded sums
// must not be further off than theirs: every 16 k-steps do for contractions of 160 k-steps on, every 8 down to BK_SHORT.  Below that the additions of the folds themselves weigh as much as the chains: there
// (template parameter SHORT) what an addition rounds off starts the next chain (two-sum, as in Kahan's summation).
// LM heads whose input is exact, relative error of the logits against 64 bits, streaming / one chain / folded as here:
// d = 896 8.9e-8 / 1.76e-7 / 7.2e-8, 2048 1.09e-7 / 2.73e-7 / 1.0e-7, 4096 1.42e-7 / 3.96e-7 / 1.3e-7.  The drafter's QKV
// (56 k-steps, 105 row tiles): K,V values that round the other way 1.30 times the streaming kernel's with a plain fold
// every 16, 1.07 every 8 or 4, 0.98 so.  128 columns per wave leave no registers for a second set.
constexpr int BK_SHORT = 104;    // k-steps of the whole contraction
__host__ __device__ constexpr int block_fold(int KS) { return KS < 40 ? 4 : KS < 160 ? 8 : 16; }
constexpr int BT_STRIDE = 132;   // padded LDS row stride (floats) of a wave's 32 x 128 epilogue tile

template <int NB>
struct BlockFrags { u32x4 w[NB], xh[2], xl[2]; };   // one k-step of a wave

template <int NB, int RT>   // RT: row tiles of the workgroup; their lo planes follow the hi planes
__device__ __forceinline__ void block_read(BlockFrags<NB> &f, uint32_t sbw, uint32_t sbx) {
    lds_frag<0>(f.xh[0], sbx); lds_frag<1024>(f.xh[1], sbx);
    lds_frag<0>(f.w[0], sbw); lds_frag<1024>(f.w[1], sbw);
    if constexpr (NB == 4) { lds_frag<2048>(f.w[2], sbw); lds_frag<3072>(f.w[3], sbw); }
    lds_frag<RT * 1024>(f.xl[0], sbx); lds_frag<RT * 1024 + 1024>(f.xl[1], sbx);
}
// the fragments are valid after this point (they pass through the wait as operands)
template <int NB>
__device__ __forceinline__ void block_wait(BlockFrags<NB> &f) {
    if constexpr (NB == 4)
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(f.w[0]), "+v"(f.w[1]), "+v"(f.w[2]), "+v"(f.w[3]), "+v"(f.xh[0]), "+v"(f.xh[1]), "+v"(f.xl[0]), "+v"(f.xl[1])
                     :: "memory");
    else
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(f.w[0]), "+v"(f.w[1]), "+v"(f.xh[0]), "+v"(f.xh[1]), "+v"(f.xl[0]), "+v"(f.xl[1]) :: "memory");
}

template <int NB, int NST>
struct BlockSmem {
    static constexpr int RT = BK_RT, CT = 2 * NB, FRAGS = CT + 2 * RT;   // per stage: weight column tiles, row tiles hi, row tiles lo
    union {
        uint4 st[NST][FRAGS * 64];
        float tile[4][32 * BT_STRIDE];                 // epilogue: one 32 x 128 tile per wave
    };
    int last;
};

// The K loop.  base[i] + vo[i]: where a lane's 16 bytes of this wave's i-th fragment of k-step 0 lie (k-steps are 1 KB
// apart); n k-steps.  Ends with this wave's LDS reads done and none of its loads in flight.
// Schedule of k-step it (its fragments are in registers): wait until k-step it + 1 has landed | barrier: everybody's share
// of it has, and everybody has read k-step it | read the fragments of it + 1 | multiply it, and between the products
// request k-step it + NST into the buffer of k-step it.  fold: see BK_SHORT.
// What is not a product has to be short or stand between products: a matrix instruction occupies its pipe for 32 cycles
// and the wave's other instructions issue meanwhile.  The steady state therefore runs without any condition (NST k-steps
// per trip, buffers at constant offsets); the last up to 2 NST - 1 k-steps take the general form.
template <int NB, int NST, int LPW, bool SHORT>
__device__ __forceinline__ void block_loop(f32x16 (&acc)[2][NB], const char *(&base)[LPW], const uint32_t (&vo)[LPW],
                                           BlockSmem<NB, NST> &sm, int n, int fold, int w, int lane) {
    using SM = BlockSmem<NB, NST>;
    constexpr int SB = SM::FRAGS * 1024;
    static_assert((NST == 4 || NST == 8) && (NST - 1) * LPW <= 63, "the loops below are written for these; the counter of loads in flight has six bits");
    const uint32_t s0 = lds_addr32(sm.st[0]) + lane * 16;
    const uint32_t ow = s0 + (w & 1) * NB * 1024, ox = s0 + (SM::CT + (w >> 1) * 2) * 1024;
    // this wave's i-th fragment of the next k-step to be requested
    auto request1 = [&](int buf, int i) {
        asm volatile("" : "+s"(base[i]));   // stays a scalar address
        __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)(base[i] + vo[i]),
                                         (void __attribute__((address_space(3))) *)(sm.st[buf] + (w * LPW + i) * 64), 16, 0, 0);
        base[i] += 1024;
    };
    f32x16 sum[2][NB];   // NB == 2 only
    auto mul = [&](const BlockFrags<NB> &f, int j) {   // product j of 4 NB: all row and column tiles with hi, then with lo
        const int mt = (j / NB) & 1, nb = j % NB;
        acc[mt][nb] = mfma32(j < 2 * NB ? f.xh[mt] : f.xl[mt], f.w[nb], acc[mt][nb]);
    };
    BlockFrags<NB> fa, fb;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[mt][nb][r] = 0.f;
#pragma unroll
    for (int k = 0; k < NST; ++k)
        if (k < n) {
#pragma unroll
            for (int i = 0; i < LPW; ++i) request1(k, i);
        }
    if (n >= NST) wait_loads<(NST - 1) * LPW>(); else wait_loads<0>();
    barrier_keep_loads();
    block_read<NB, SM::RT>(fa, ow, ox);
    block_wait<NB>(fa);
    auto step = [&](BlockFrags<NB> &cur, BlockFrags<NB> &next, auto buf_c) {   // steady state
        constexpr int buf = decltype(buf_c)::value, nbuf = (buf + 1) % NST;
        wait_loads<(NST - 2) * LPW>();
        barrier_keep_loads();
        block_read<NB, SM::RT>(next, ow + nbuf * SB, ox + nbuf * SB);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4 * NB; ++j) {
            mul(cur, j);
            if (j % NB == NB - 1 && j / NB < 3) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = j / NB; i < LPW; i += 3) request1(buf, i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        block_wait<NB>(next);
    };
    auto fold_in = [&] {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float s = sum[mt][nb][r], a = acc[mt][nb][r], t = s + a;
                    sum[mt][nb][r] = t;
                    // (the clamp keeps an infinite sum infinite: inf - inf would make it a NaN)
                    acc[mt][nb][r] = SHORT ? __builtin_amdgcn_fmed3f(a - (t - s), -3.4028234e38f, 3.4028234e38f) : 0.f;
                }
    };
    int it = 0, next_fold = fold;
    for (; it < n - 2 * NST + 1; it += NST) {
        if constexpr (NB == 2)
            if (it >= next_fold) { next_fold = it + fold; fold_in(); }
        step(fa, fb, std::integral_constant<int, 0>{}); step(fb, fa, std::integral_constant<int, 1>{});
        step(fa, fb, std::integral_constant<int, 2>{}); step(fb, fa, std::integral_constant<int, 3>{});
        if constexpr (NST == 8) {
            step(fa, fb, std::integral_constant<int, 4>{}); step(fb, fa, std::integral_constant<int, 5>{});
            step(fa, fb, std::integral_constant<int, 6>{}); step(fb, fa, std::integral_constant<int, 7>{});
        }
    }
    auto last_steps = [&](BlockFrags<NB> &cur, BlockFrags<NB> &next) {
        const bool more = it + 1 < n;
        if (more) {
            if (n - 2 - it >= NST - 2) wait_loads<(NST - 2) * LPW>(); else wait_loads<0>();
            barrier_keep_loads();
            const int buf = it & (NST - 1), nbuf = (it + 1) & (NST - 1);
            if (it + NST < n) {
#pragma unroll
                for (int i = 0; i < LPW; ++i) request1(buf, i);
            }
            block_read<NB, SM::RT>(next, ow + nbuf * SB, ox + nbuf * SB);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4 * NB; ++j) mul(cur, j);
        __builtin_amdgcn_sched_barrier(0);
        if (more) block_wait<NB>(next);
        ++it;
    };
    if constexpr (NB == 2)
        if (it >= next_fold) fold_in();
    while (it < n) {
        last_steps(fa, fb);
        if (it < n) last_steps(fb, fa);
    }
    if constexpr (NB == 2) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mt][nb][r] += sum[mt][nb][r];
    }
}

// rstd of row (lane & 31) of the 32 rows that start at grow0, in both halves of the wave
__device__ __forceinline__ float wave_rstd(const float *ssq, size_t row, int half, int ncg, int d, float eps) {
    const float *p = ssq + row * ncg;
    float s = 0.f;
    int g = half;
    for (; g + 6 < ncg; g += 8) {
        const float v0 = p[g], v1 = p[g + 2], v2 = p[g + 4], v3 = p[g + 6];
        s += v0; s += v1; s += v2; s += v3;
    }
    for (; g < ncg; g += 2) s += p[g];
    s += shx(s, 32);
    return rsqrtf(s / (float)d + eps);
}

// LDS writes of this wave are readable by its other lanes behind this point
__device__ __forceinline__ void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Accumulators of one row tile into a 32 x 128 tile (columns col0 ..), MFMA register layout -> row-major
template <int NB>
__device__ __forceinline__ void wave_park(const f32x16 (&acc)[NB], float *tile, int col0, int lane) {
    const int half = lane >> 5, cl = lane & 31;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) tile[mfma_row(r, half) * BT_STRIDE + col0 + nb * 32 + cl] = acc[nb][r];
}

// The epilogues of deer_kernels.hpp for one wave and one 32 x 128 tile: row tile t, column group cg.  No barriers: every wave runs its own.
template <int EPI>
__device__ __forceinline__ void wave_epilogue(const GemmArgs &a, float *tile, int cg, int t) {
    const int lane = opaque_tid() & 63, half = lane >> 5, row = lane & 31;
    const size_t grow = (size_t)t * 32 + row;
    float rs = 0.f;
    if (EPI != EPI_RESID) rs = wave_rstd(a.ssq_in, grow, half, a.ncg_in, a.d_in, a.eps);
    if (EPI == EPI_SWIGLU) {
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {   // octets of 8 channels
            const int oct = 2 * i + half;
            const float *g = tile + row * BT_STRIDE + oct * 8, *u = g + 64;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float ge = g[e] * rs;
                v[e] = ge / (1.f + expf(-ge)) * (u[e] * rs);
            }
            uint4 hi, lo;
            pack8_split(v, hi, lo);
            const size_t vec = (size_t)t * (a.F / 16) * 64 + frag_vec(row, cg * 8 + oct);
            a.ahi[vec] = hi;
            a.alo[vec] = lo;
        }
    } else if (EPI == EPI_RESID) {
        const int N = a.N, c4 = row * 4;
        float *hp = a.h + ((size_t)t * 32 + half) * N + (size_t)cg * CG + c4;
        float4 hv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) hv[i] = *(const float4 *)(hp + (size_t)(2 * i) * N);
#pragma unroll
        for (int i = 0; i < 16; ++i) {   // rows 2 i + half
            float4 *tp = (float4 *)(tile + (2 * i + half) * BT_STRIDE + c4);
            const float4 y = *tp;
            const float4 v = make_float4(hv[i].x + y.x, hv[i].y + y.y, hv[i].z + y.z, hv[i].w + y.w);
            *(float4 *)(hp + (size_t)(2 * i) * N) = v;
            *tp = v;
        }
        wave_lds_sync();
        float ss[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {   // 32-column blocks: octets 4 b .. 4 b + 3, two per half
            ss[b] = 0.f;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int oct = 4 * b + 2 * j + half;
                const float *tp = tile + row * BT_STRIDE + oct * 8;
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) { v[e] = tp[e]; ss[b] += v[e] * v[e]; }
                uint4 hi, lo;
                pack8_split(v, hi, lo);
                const size_t vec = (size_t)t * (N / 16) * 64 + frag_vec(row, cg * 16 + oct);
                a.xhi_out[vec] = hi;
                a.xlo_out[vec] = lo;
            }
            ss[b] += shx(ss[b], 32);
        }
        if (half == 0) {
            if (a.ssq_sub == 4) *(float4 *)(a.ssq_out + grow * (N / 32) + cg * 4) = make_float4(ss[0], ss[1], ss[2], ss[3]);
            else if (a.ssq_sub == 2) *(float2 *)(a.ssq_out + grow * (N / 64) + cg * 2) = make_float2(ss[0] + ss[1], ss[2] + ss[3]);
            else a.ssq_out[grow * (N / CG) + cg] = (ss[0] + ss[1]) + (ss[2] + ss[3]);
        }
    } else if (EPI == EPI_QKV) {
        const int hd = a.hd, Hq = a.Hq, Hkv = a.Hkv, half_hd = hd >> 1;
        const int b = a.rm.seq[grow], slot = a.rm.slot[grow], qr = a.rm.qrow[grow];
#pragma unroll 1
        for (int i = 0; i < 8; ++i) {
            const int oct = 2 * i + half, col0 = cg * CG + oct * 8;   // first of 8 columns, all in one head
            const int kind = col0 < Hq * hd ? 0 : (col0 < (Hq + Hkv) * hd ? 1 : 2);
            const int hc = col0 - (kind == 0 ? 0 : (kind == 1 ? Hq * hd : (Hq + Hkv) * hd));
            const int head = hc / hd, i0 = hc % hd;
            const float *x = tile + row * BT_STRIDE + oct * 8;
            float v[8];
            if (kind < 2) {
                const float *xp = x + ((i0 < half_hd) ? half_hd : -half_hd);
                const float2 *cs = a.cs + grow * half_hd + (i0 < half_hd ? i0 : i0 - half_hd);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float2 c = cs[e];
                    v[e] = (i0 < half_hd) ? x[e] * rs * c.x - xp[e] * rs * c.y : x[e] * rs * c.x + xp[e] * rs * c.y;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = x[e] * rs;
            }
            if (kind == 0) {
                uint4 hi, lo;
                pack8_split(v, hi, lo);
                if (qr >= 0) {
                    const size_t vec = ((size_t)((qr >> 5) * Hq + head) * (hd / 16)) * 64 + frag_vec(qr & 31, i0 >> 3);
                    a.qhi[vec] = hi;
                    a.qlo[vec] = lo;
                }
            } else if (slot >= 0) {
                const size_t kvb = (size_t)b * a.kv.seq_stride + (size_t)head * a.kv.head_stride;
                if (kind == 1) {
                    *(uint4 *)(a.kv.k + kvb + k_cache_off(slot, i0 >> 3, hd)) = pack8(v);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) a.kv.vt[kvb + v_cache_off(slot, i0 + e, hd)] = (uint16_t)f2bf(v[e]);
                }
            }
        }
    } else if (EPI == EPI_LMHEAD) {
        const int V = a.N, sub = lane & 7;   // 8 lanes per row, 16 columns each (4 of every 32: a store fills whole lines); 8 rows at a time
        const float T = a.T, invT = T > 0.f ? 1.f / T : 1.f;
#pragma unroll 1
        for (int r0 = 0; r0 < 32; r0 += 8) {
            const int lr = r0 + (lane >> 3);
            const float sc = __int_as_float(__builtin_amdgcn_ds_bpermute(lr << 2, __float_as_int(rs)));
            const size_t lm = (size_t)t * 32 + lr;
            const bool live = (int)lm < a.n_lm && (int)lm % opaque_s(a.k) >= a.k_lo;
            float m = -INFINITY, gm = -INFINITY, se = 0.f;
            int idx = 0x7fffffff, gidx = 0x7fffffff;
            const float4 *tp = (const float4 *)(tile + lr * BT_STRIDE) + sub;   // (short loops over the tile: see epi_lmhead)
            if (live) {
                float4 *q = a.logits ? (float4 *)(a.logits + lm * V + (size_t)cg * CG) + sub : nullptr;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float4 z = make_float4(tp[8 * e].x * sc, tp[8 * e].y * sc, tp[8 * e].z * sc, tp[8 * e].w * sc);
                    if (q) q[8 * e] = z;
                    const int v = cg * CG + 4 * (8 * e + sub);
                    argmax_merge(m, idx, z.x, v); argmax_merge(m, idx, z.y, v + 1); argmax_merge(m, idx, z.z, v + 2); argmax_merge(m, idx, z.w, v + 3);
                }
                if (T > 0.f && a.draw) {
                    const uint64_t key = row_key(a.seed, TAG_DRAFT, (uint64_t)a.rm.seq[lm], (uint64_t)a.rm.pos[lm]);
                    int v = cg * CG + 4 * sub;
#pragma unroll 1
                    for (int e = 0; e < 4; ++e, v += 32) {
                        const float4 z = make_float4(tp[8 * e].x * sc, tp[8 * e].y * sc, tp[8 * e].z * sc, tp[8 * e].w * sc);
                        argmax_merge(gm, gidx, z.x * invT + gumbel(key, (uint64_t)v), v);
                        argmax_merge(gm, gidx, z.y * invT + gumbel(key, (uint64_t)(v + 1)), v + 1);
                        argmax_merge(gm, gidx, z.z * invT + gumbel(key, (uint64_t)(v + 2)), v + 2);
                        argmax_merge(gm, gidx, z.w * invT + gumbel(key, (uint64_t)(v + 3)), v + 3);
                    }
                }
            }
#pragma unroll
            for (int off = 1; off < 8; off <<= 1) {
                const float m2 = shx(m, off); const int i2 = shx(idx, off);
                argmax_merge(m, idx, m2, i2);
                const float g2 = shx(gm, off); const int gi2 = shx(gidx, off);
                argmax_merge(gm, gidx, g2, gi2);
            }
            if (live && T > 0.f) {
#pragma unroll 1
                for (int e = 0; e < 4; ++e) {
                    const float4 z = tp[8 * e];
                    se += expf((z.x * sc - m) * invT); se += expf((z.y * sc - m) * invT); se += expf((z.z * sc - m) * invT); se += expf((z.w * sc - m) * invT);
                }
            }
#pragma unroll
            for (int off = 1; off < 8; off <<= 1) se += shx(se, off);
            if (live && sub == 0) a.stat[lm * a.ncg_v + cg] = RowStat{m, idx, se, gm, gidx};
        }
    }
}

// Workgroup id -> (column block and K share p, row block).  Ids 8 apart share an XCD; every XCD gets one contiguous run
// of the order (band of up to 8 row blocks, p, row block in the band), so that the workgroups it runs together read few
// weight columns and few rows.  The order has no gaps: with a last band counted as high as the others (workgroups without a
// block) the runs would begin at the same column in every band, but the 4B's gate/up of 104 row tiles took 573 us so and takes 528
// (9728 x 896 124 and 109; QKV 202 and 203).
struct BlockItem { int p, rb; };
__device__ __forceinline__ BlockItem block_at(int i, int P, int nrb, int band) {
    int b0 = 0, rows = nrb;   // one band: no division
    if (band < nrb) {
        const int bd = min(i / opaque_s(band * P), (nrb - 1) / opaque_s(band));
        b0 = bd * band;
        rows = min(band, nrb - b0);   // the last band may be lower
        i -= b0 * P;
    }
    BlockItem it;
    it.p = i / opaque_s(rows);
    it.rb = b0 + (i - it.p * rows);
    return it;
}
inline int block_band(int nrb) { const int bands = (nrb + 7) / 8; return (nrb + bands - 1) / bands; }

// How the blocks of a launch are dealt to workgroups.  full == blocks: one workgroup per block (and K share, GemmArgs::S).
// full < blocks (S == 1): the last `blocks - full` blocks of the order, more than a compute unit's equal share of blocks, lie
// end to end as one row of k-steps that G workgroups cut into pieces of `piece` k-steps; a piece is part of one block or of two
// neighbours.  Those workgroups have the lowest ids: they start first, beside the whole blocks, and the pieces' sums meet
// while those still run.
struct BlockDeal { int blocks, full, G, piece, per; };   // per: k-steps of a uniform share
inline int block_grid(const BlockDeal &d) { return d.G + 8 * ((d.full + 7) / 8); }

// acc = the shares of a block in their order, the loads of U of them in flight together.
template <int U, int NB, typename F>
__device__ __forceinline__ void block_sum(f32x16 (&acc)[2][NB], int nmt, int nsh, F at) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
        if (mt < nmt)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mt][nb][r] = 0.f;
                for (int u0 = 0; u0 < nsh; u0 += U) {
                    u32x4 v[U][4];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const float *pu = at(min(u0 + u, nsh - 1)) + (mt * NB + nb) * 4 * 256;
#pragma unroll
                        for (int q = 0; q < 4; ++q) load16_agent_async(v[u][q], pu + q * 256);
                    }
                    wait_loads<0>();
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            tie(v[u][q]);
                            if (u0 + u < nsh)
#pragma unroll
                                for (int e = 0; e < 4; ++e) acc[mt][nb][4 * q + e] += __uint_as_float(v[u][q][e]);
                        }
                }
            }
}

// acc += the other share, its first MT row tiles' loads in flight together.
template <int MT>
__device__ __forceinline__ void block_add(f32x16 (&acc)[2][2], const float *po) {
    u32x4 v[MT * 8];
#pragma unroll
    for (int q = 0; q < MT * 8; ++q) load16_agent_async(v[q], po + q * 256);
    wait_loads<0>();
#pragma unroll
    for (int q = 0; q < MT * 8; ++q) {
        tie(v[q]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[q >> 3][(q >> 2) & 1][4 * (q & 3) + e] += __uint_as_float(v[q][e]);
    }
}

// ncb: column blocks of 64 NB columns; nrt: row tiles; SHORT: a contraction of less than BK_SHORT k-steps; PIECES: deal.G > 0
// (a form of its own: its loop keeps the arguments in scalar registers across the k-loop, which runs out of them: with one
// form for both, launches without pieces took 2 to 7 % longer)
template <int NB, int NST, int EPI, bool SHORT, bool PIECES>
__global__ __launch_bounds__(256, sizeof(BlockSmem<NB, NST>) <= 80 * 1024 ? 2 : 1) void k_gemm_block(const GemmArgs a, int ncb, int nrt, int band, const BlockDeal deal) {
    constexpr int LPW = BlockSmem<NB, NST>::FRAGS / 4;
    constexpr size_t PART = 4 * (2 * NB * 4 * 256);   // floats of a block's partial sums: [wave][(mt, nb, quad)][lane][4]
    __shared__ __attribute__((aligned(16))) BlockSmem<NB, NST> sm;
    const int w = __builtin_amdgcn_readfirstlane(opaque_tid() >> 6);
    const int wr = w >> 1, wc = w & 1;
    const int nrb = (nrt + BK_RT - 1) / BK_RT, KS = a.KS;
    const int lin = blockIdx.x;
    const bool pieces = PIECES && lin < deal.G;
    int at, end;                 // this workgroup's k-steps [at, end): of one block (share), or of the row of blocks cut into pieces
    int cb, rb, s = 0, b = 0;    // column block, row block, uniform share; pieces: the block in the row
    if (pieces) {
        const int g = (lin & 7) * (deal.G >> 3) + (lin >> 3);
        at = g * deal.piece; end = min((deal.blocks - deal.full) * KS, at + deal.piece);
        b = at / opaque_s(KS);
    } else {
        const int l = PIECES ? lin - deal.G : lin, per8 = (deal.full + 7) >> 3, i = (l & 7) * per8 + (l >> 3);
        if ((l >> 3) >= per8 || i >= deal.full) return;
        const BlockItem bi = block_at(i, ncb * a.S, nrb, band);   // the order runs over (share, column block) pairs
        if (a.S > 1) s = bi.p / opaque_s(ncb);
        cb = bi.p - s * ncb; rb = bi.rb;
        at = s * deal.per; end = min(KS, at + deal.per);          // the host keeps every share non-empty
    }
    bool first = true;
    if (PIECES && at >= end) return;
#pragma unroll 1
    do {
        // this workgroup's k-steps of the block, and where the block's shares lie
        int ks0 = at, n = end - at, nsh = a.S, mine = s, g0 = 0, odd0 = 0;
        if (pieces) {
            const BlockItem bi = block_at(deal.full + b, ncb, nrb, band);
            cb = bi.p; rb = bi.rb;
            ks0 = at - b * KS; n = min(KS - ks0, end - at);
            g0 = b * KS / opaque_s(deal.piece);                   // the first workgroup with a piece of this block
            nsh = ((b + 1) * KS - 1) / opaque_s(deal.piece) - g0 + 1;
            odd0 = g0 * deal.piece < b * KS ? 1 : 0;              // that workgroup began in the block before: its second piece
            mine = at / opaque_s(deal.piece) - g0;
        }
        // slot of share u: uniform (share, block), pieces (workgroup, first or second piece)
        auto slot = [&](int u) -> size_t { return pieces ? (size_t)2 * (g0 + u) + (u == 0 ? odd0 : 0) : (size_t)u * nrb * ncb + (size_t)rb * ncb + cb; };
        const int counter = pieces ? b : rb * ncb + cb;
        at += n; ++b;
        if (PIECES && !first) __syncthreads();   // the epilogue's tiles have been read: the ring reuses them
        first = false;
        const int nmt = max(0, min(2, nrt - (rb * BK_RT + wr * 2)));
        const int ln = opaque_tid() & 63;   // (derived again behind the loop: registers)
        const char *base[LPW];
        uint32_t vo[LPW];
#pragma unroll
        for (int i = 0; i < LPW; ++i) {   // fragments past the matrix repeat the last ones (their products are not used)
            const int f = w * LPW + i;
            const uint4 *p;
            if (f < 2 * NB) p = a.W + ((size_t)min(cb * 2 * NB + f, a.N / 32 - 1) * KS + ks0) * 64;
            else {
                const int x = f - 2 * NB, ct = min(rb * BK_RT + (x & (BK_RT - 1)), nrt - 1);
                p = (x < BK_RT ? a.Xhi : a.Xlo) + ((size_t)ct * KS + ks0) * 64;
            }
            base[i] = (const char *)p;
            vo[i] = ln * 16;
        }
        f32x16 acc[2][NB];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mt][nb][r] = 0.f;
        block_loop<NB, NST, LPW, SHORT>(acc, base, vo, sm, n, block_fold(KS), w, ln);

        const int lane = opaque_tid() & 63;
        if (nsh > 1) {
            float *p0 = a.part + (size_t)w * (2 * NB * 4 * 256) + lane * 4;
            float *pw = p0 + slot(mine) * PART;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                if (mt < nmt)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            store16_agent(pw + ((mt * NB + nb) * 4 + q) * 256, acc[mt][nb][4 * q], acc[mt][nb][4 * q + 1], acc[mt][nb][4 * q + 2], acc[mt][nb][4 * q + 3]);
            if (!arrive_last(a.counters + counter, nsh, &sm.last)) continue;
            // What the last workgroup draws bounds this part (about 60 KB per microsecond): no share is read twice but the last of
            // an odd number.  Of two, only the other one is read (both orders of a sum of two are the same; with 128 columns per
            // wave there are no registers for it), more are summed in their order.  Against four at a time, a share repeated to
            // fill them: a prompt of 7 row tiles through the 4B pair 7119 -> 6889 us, passes of 16 sequences within 0.5 %.
            auto at_share = [&](int u) { return p0 + slot(u) * PART; };
            if constexpr (NB == 4) block_sum<2>(acc, nmt, nsh, at_share);
            else if (nsh == 2 && nmt == 2) block_add<2>(acc, at_share(1 - mine));
            else if (nsh == 2) { if (nmt) block_add<1>(acc, at_share(1 - mine)); }
            else if (nsh % 4 == 0 || nsh == 7) block_sum<4>(acc, nmt, nsh, at_share);
            else block_sum<3>(acc, nmt, nsh, at_share);
        } else {
            __syncthreads();   // every wave has read the ring: the epilogue tiles reuse it
        }
        if constexpr (NB == 4) {
            const int cg = cb * 2 + wc;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                const int ct = rb * BK_RT + wr * 2 + mt;
                if (mt >= nmt || cg * CG >= a.N) continue;
                wave_park<NB>(acc[mt], sm.tile[w], 0, lane);
                wave_lds_sync();
                wave_epilogue<EPI>(a, sm.tile[w], cg, ct);
                wave_lds_sync();
            }
        } else {   // a column group is made by the two waves of a row pair: wave wc finishes row tile wc
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) wave_park<NB>(acc[mt], sm.tile[wr * 2 + mt], wc * 64, lane);
            __syncthreads();
            const int ct = rb * BK_RT + wr * 2 + wc;
            if (wc < nmt) wave_epilogue<EPI>(a, sm.tile[wr * 2 + wc], cb, ct);
        }
    } while (PIECES && at < end);
}

// The rows of the pairs, gathered into tiles of their expert for the blocked gate/up GEMM: (item, 128-column group) per
// workgroup, from the fp32 residual stream (row-major: 512 contiguous bytes per row; the same hi and lo planes as in the
// pass's own fragments, where a pair's row is 16 bytes of every 128-byte line: read from there, the GEMM moved eight
// times the bytes, 590 us for 2048 rows of the 128-expert layer).  Rows past the last pair of a tile repeat it.
__global__ __launch_bounds__(256) void k_moe_gather(const float *__restrict__ h, const MoeArgs a, uint4 *__restrict__ xhi, uint4 *__restrict__ xlo) {
    const int item = blockIdx.y, cg = blockIdx.x;
    if (item >= a.items[0].x) return;
    const int4 it = a.items[1 + item];
    const int n = it.z, at = it.w, rows = ((n + 31) >> 5) << 5;
    const int *pairs = a.pairs + (size_t)it.x * a.cap + it.y;
    for (int e = threadIdx.x; e < rows * 16; e += 256) {   // (octet pair, tile, octet, row): a wave reads 64 and writes 1024 bytes per row / fragment
        const int row = e & 31, tile = rows == 64 ? (e >> 6) & 1 : 0, oct = 2 * (rows == 64 ? e >> 7 : e >> 6) + ((e >> 5) & 1);
        const int r = pairs[min(tile * 32 + row, n - 1)] >> 3;
        const float4 *p = (const float4 *)(h + (size_t)r * a.d_in + cg * CG + oct * 8);
        const float4 v0 = p[0], v1 = p[1];
        const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        uint4 hi, lo;
        pack8_split(v, hi, lo);
        const size_t vec = (size_t)(at + tile) * (a.d_in / 16) * 64 + frag_vec(row, cg * 16 + oct);
        xhi[vec] = hi;
        xlo[vec] = lo;
    }
}

}  // namespace deer
