// Device code of libdeer: every step of the draft-verify iteration as HIP kernels for gfx950.
//
// Data layouts (all chosen for 64-lane wavefronts and the 32x32x16 bf16 MFMA):
//   * "fragment" layout of a [32 rows x K] operand tile: 16-byte vectors ordered [K/16][64 lanes],
//     lane l holding row (l % 32), k-indices 16*ks + 8*(l / 32) .. +8.  One wave-wide 16-byte load
//     is one MFMA operand.  Weights use it per 32-column block ([N/32][K/16][64][8], so a block's
//     whole K extent is one contiguous stream); activations use it per 32-row tile, as two planes
//     (hi, lo) with x ~= hi + lo in bf16, so that products against bf16 weights are exact to
//     ~2^-17 and accumulate in fp32.
//   * residual stream h: fp32 row-major [rows][d_model].
//   * K and V caches [layer][seq][kv_head] in blocks of 32 slots, each block in the fragment order of the
//     attention contractions (see k_cache_off / v_cache_off), bf16.
//   * a pass works on row tiles of 32; every tile belongs to one sequence; unused rows have
//     limit 0 and slot -1.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include <utility>
#include <stdint.h>

namespace deer {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;   // a 16-byte operand fragment held in registers

constexpr int CG = 128;          // columns per column group (4 MFMA column blocks)
constexpr int RED_STRIDE = 136;  // padded LDS row stride (floats) of a 32x128 tile

// ------------------------------------------------------------------------------------------
// small helpers
// ------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// fp32 -> bf16, round to nearest even (the hardware conversion)
__device__ __forceinline__ uint32_t f2bf(float f) {
    return (uint32_t)__builtin_bit_cast(unsigned short, (__bf16)f);
}
__device__ __forceinline__ float bf2f(uint32_t b) { return __uint_as_float(b << 16); }
// two floats -> packed bf16 pair (a in the low half)
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
    f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ uint4 pack8(const float *v) {
    return make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
}

__device__ __forceinline__ void pack8_split(const float *v, uint4 &hi, uint4 &lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        h[e] = f2bf2(v[2 * e], v[2 * e + 1]);
        l[e] = f2bf2(v[2 * e] - __uint_as_float(h[e] << 16), v[2 * e + 1] - __uint_as_float(h[e] & 0xffff0000u));
    }
    hi = make_uint4(h[0], h[1], h[2], h[3]);
    lo = make_uint4(l[0], l[1], l[2], l[3]);
}

__device__ __forceinline__ f32x16 mfma32(uint4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 mfma32(u32x4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Hand-scheduled loads (used where the compiler's wait-count insertion would drain every outstanding
// load at a loop header): the load is issued here and its result may only be read after wait_loads<N>()
// (at most N younger loads still outstanding; loads return in order) followed by tie() on the register.
__device__ __forceinline__ void load16_async(u32x4 &dst, const void *p) {
    asm volatile("global_load_dwordx4 %0, %1, off" : "=&v"(dst) : "v"(p) : "memory");
}
// the same, marked non-temporal: data read exactly once per pass (weights), which should not push activations, partial sums
// and the kernel's own instructions out of L2
__device__ __forceinline__ void load16_stream_async(u32x4 &dst, const void *p) {
    asm volatile("global_load_dwordx4 %0, %1, off nt" : "=&v"(dst) : "v"(p) : "memory");
}
// a scalar base, a lane's offset and a constant one; NT: non-temporal
template <int OFF, bool NT>
__device__ __forceinline__ void load16_async(u32x4 &dst, const void *base, uint32_t lane_off) {
    if constexpr (NT) asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3 nt" : "=&v"(dst) : "v"(lane_off), "s"(base), "n"(OFF) : "memory");
    else asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=&v"(dst) : "v"(lane_off), "s"(base), "n"(OFF) : "memory");
}
__device__ __forceinline__ void load4_async(float &dst, const void *p) {
    asm volatile("global_load_dword %0, %1, off" : "=&v"(dst) : "v"(p) : "memory");
}
__device__ __forceinline__ void tie(float &r) { asm volatile("" : "+v"(r)); }
// at most `steps` x PER loads may still be outstanding (steps <= MAX <= 5)
template <int PER, int MAX = 4>
__device__ __forceinline__ void wait_steps(int steps);
// The same with agent scope: the load is served by memory, not by an L2 that may hold an older copy of a line
// another XCD has written since.
__device__ __forceinline__ void load16_agent_async(u32x4 &dst, const void *p) {
    asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(dst) : "v"(p) : "memory");
}
// A 16-byte agent-scope (write-through) store.  The wait states behind it keep the next instruction from
// overwriting the data registers while the store still reads them (a hazard the compiler covers for its own
// stores of more than 8 bytes, but cannot see inside an asm statement).
__device__ __forceinline__ void store16_agent(void *p, float a, float b, float c, float d) {
    u32x4 v = {__float_as_uint(a), __float_as_uint(b), __float_as_uint(c), __float_as_uint(d)};
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 2" ::"v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store16_agent(uint4 *p, uint4 x) {
    store16_agent(p, __uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
template <int PER, int MAX>
__device__ __forceinline__ void wait_steps(int steps) {
    static_assert(MAX >= 3 && MAX <= 5 && MAX * PER <= 63, "the counter has six bits");
    if (steps <= 0) wait_loads<0>();
    else if (steps == 1) wait_loads<PER>();
    else if (steps == 2) wait_loads<2 * PER>();
    else if (MAX == 3 || steps == 3) wait_loads<3 * PER>();
    else if (MAX == 4 || steps == 4) wait_loads<4 * PER>();
    else wait_loads<5 * PER>();
}
__device__ __forceinline__ void tie(u32x4 &r) { asm volatile("" : "+v"(r)); }

// Fragments that direct-to-LDS loads have put into LDS are read with instructions the compiler does not see as LDS reads:
// before one of those, of memory that such loads may write, it waits for ALL loads in flight, the ones requested ahead
// included.  The caller's counted waits and barriers order the reads after their own loads, and a fragment is valid after
// wait_lds<N>() (at most N younger LDS reads outstanding) and tie().
// LDS byte address of a __shared__ object
__device__ __forceinline__ uint32_t lds_addr32(const void *p) {
    return (uint32_t)(size_t)(const void __attribute__((address_space(3))) *)p;
}
template <int OFF>
__device__ __forceinline__ void lds_frag(u32x4 &v, uint32_t addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(v) : "v"(addr), "n"(OFF));
}
template <int N>
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory"); }
template <int OFF, int... I>
__device__ __forceinline__ void lds_frags(u32x4 *v, uint32_t addr, std::integer_sequence<int, I...>) { (lds_frag<OFF + 1024 * I>(v[I], addr), ...); }

// Workgroup barrier for loops that keep direct-to-LDS loads in flight across it: __syncthreads() waits for every
// outstanding vector memory operation of the wave (its fence covers the LDS writes of those loads), which would
// empty the ring of staged buffers at every barrier.  This one waits only for the wave's LDS reads; the caller
// counts down the loads that must have landed with wait_loads<N>() first.
__device__ __forceinline__ void barrier_keep_loads() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The thread index as a value the optimiser cannot trace back to the hardware register.  Lane-dependent
// indices and addresses derived from it are recomputed where they are used instead of being hoisted to the
// top of a long kernel and kept in registers (or spilled) across all of its phases.
__device__ __forceinline__ int opaque_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Butterfly exchange with lane (lane ^ off).  The lane index is derived where it is used (see opaque_tid),
// never from a value computed once at the top of the kernel; blocks are whole wavefronts, so the low six
// bits of the thread index are the lane.
__device__ __forceinline__ int shx(int v, int off) {
    return __builtin_amdgcn_ds_bpermute(((opaque_tid() & 63) ^ off) << 2, v);
}
__device__ __forceinline__ float shx(float v, int off) { return __int_as_float(shx(__float_as_int(v), off)); }

// A uniform value the optimiser cannot trace: divisions by it are expanded where they stand.  (The reciprocal
// of a loop-invariant divisor is otherwise computed once at the top of the kernel, in a vector register that
// lives through the whole kernel, is spilled, and is reloaded from scratch memory at every use.)
__device__ __forceinline__ int opaque_s(int v) {
    asm volatile("" : "+s"(v));
    return v;
}

// Value of the lane that differs in the lane index by the pattern of one data-parallel-primitive control: 0xB1 xor 1,
// 0x4E xor 2, 0x141 mirrored in its 8 lanes, 0x140 mirrored in its 16.  A reduction that takes these four steps in order has
// the same result in all 16 lanes of a row; a step costs two instructions, an exchange through LDS over a hundred cycles.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true); }
template <int CTRL>
__device__ __forceinline__ float dppf(float v) { return __uint_as_float(dpp<CTRL>(__float_as_uint(v))); }
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64_max(uint64_t v) {
    const uint64_t o = ((uint64_t)dpp<CTRL>((uint32_t)(v >> 32)) << 32) | dpp<CTRL>((uint32_t)v);
    return o > v ? o : v;
}

// Row of the 32x32 MFMA result held in register r of a lane in half `half` (= lane / 32).
__device__ __forceinline__ int mfma_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// Index (in 16-byte vectors) of (row, k-octet) inside a fragment-layout tile with KS k-steps.
__device__ __forceinline__ size_t frag_vec(int row, int oct) { return (size_t)(oct >> 1) * 64 + row + 32 * (oct & 1); }

__device__ __forceinline__ uint64_t mix64(uint64_t z) {  // splitmix64 finaliser
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}
constexpr uint64_t GOLDEN = 0x9E3779B97F4A7C15ULL;
enum { TAG_DRAFT = 1, TAG_ACCEPT = 2, TAG_RESID = 3 };
__device__ __forceinline__ uint64_t row_key(uint64_t seed, uint64_t tag, uint64_t seq, uint64_t pos) {
    return mix64(mix64(seed + GOLDEN * tag) ^ ((seq << 40) + pos));
}
__device__ __forceinline__ float uniform01(uint64_t key, uint64_t idx) {  // (r + 0.5) / 2^23, r < 2^23
    uint64_t bits = mix64(key + GOLDEN * (idx + 1));
    return ((float)(uint32_t)(bits >> 41) + 0.5f) * (1.0f / 8388608.0f);
}
__device__ __forceinline__ float gumbel(uint64_t key, uint64_t idx) { return -logf(-logf(uniform01(key, idx))); }

// Split-K / split-KV partials cross workgroups that may sit on different XCDs (separate L2s).  They
// are written and read with agent-scope accesses, which are coherent without cache-wide
// write-backs or invalidates; the arrival counter is an agent-scope atomic.
__device__ __forceinline__ void st_agent2(float *p, float a, float b) {   // p 8-byte aligned
    unsigned long long u = ((unsigned long long)__float_as_uint(b) << 32) | (unsigned long long)__float_as_uint(a);
    __hip_atomic_store((unsigned long long *)p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_agent2(const float *p) {
    unsigned long long u = __hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((unsigned)(u & 0xffffffffu)), __uint_as_float((unsigned)(u >> 32)));
}
// Called by every thread after its partial stores: waits for them, then one thread counts the block
// in.  Returns true in every thread of the block that arrived last (counter reset for the next use).
__device__ __forceinline__ bool arrive_last(int *cnt, int expected, int *s_flag) {
    // The thread's agent-scope stores must have been performed before the block is counted in.  A
    // workgroup-scope fence does not wait for vector memory, so the wait is explicit.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        int old = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int last = (old == expected - 1);
        if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_flag = last;
    }
    __syncthreads();
    return *s_flag != 0;
}

// (value, index) max with lowest index on ties
__device__ __forceinline__ void argmax_merge(float &v, int &i, float v2, int i2) {
    if (v2 > v || (v2 == v && i2 < i)) { v = v2; i = i2; }
}

// ------------------------------------------------------------------------------------------
// weight repack: canonical [K][N_src] (fp32 or bf16) -> fragment layout, bf16
//   dest column n_dst = col_map(n_src):  plain offset (QKV concatenation) or gate/up interleave
//   (group of 128 columns = 64 gate channels followed by the same 64 up channels).
// ------------------------------------------------------------------------------------------
template <typename SrcT>
__device__ __forceinline__ uint32_t load_as_bf16(const SrcT *p);
template <>
__device__ __forceinline__ uint32_t load_as_bf16<float>(const float *p) { return f2bf(*p); }
template <>
__device__ __forceinline__ uint32_t load_as_bf16<uint16_t>(const uint16_t *p) { return *p; }

// mode 0: n_dst = n_src + col_off.  mode 1 (gate) / 2 (up): n_dst = (n_src/64)*128 + (mode-1)*64 + n_src%64
template <typename SrcT>
__global__ void k_repack(const SrcT *__restrict__ src, uint4 *__restrict__ dst, int K, int N_src, int KS_dst,
                         int mode, int col_off) {
    // one thread per (src column n, k-octet): reads 8 strided values, writes one 16-byte vector
    size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    int n = (int)(gid % N_src);
    size_t oct = gid / N_src;
    if (oct >= (size_t)K / 8) return;
    int n_dst = (mode == 0) ? n + col_off : (n / 64) * 128 + (mode - 1) * 64 + (n % 64);
    uint32_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = load_as_bf16<SrcT>(src + ((size_t)oct * 8 + e) * N_src + n);
    int nb = n_dst >> 5;
    size_t vec = ((size_t)nb * KS_dst) * 64 + frag_vec(n_dst & 31, (int)oct);
    dst[vec] = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
}

template <typename SrcT>
__global__ void k_convert_rows(const SrcT *__restrict__ src, uint16_t *__restrict__ dst, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (uint16_t)load_as_bf16<SrcT>(src + i);
}

// Measurement aid: a plain read of n 16-byte vectors (grid-stride, four loads in flight per thread and trip), the rate
// of which is what "streaming at memory speed" means for a buffer of that size on this chip.  Nothing is written
// unless the data has one particular checksum (so that the loads cannot be dropped).
template <bool NT>
__global__ __launch_bounds__(512) void k_stream_read(const u32x4 *__restrict__ p, size_t n, uint32_t *out) {
    size_t i = (size_t)blockIdx.x * 512 + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * 512;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (; i + 3 * stride < n; i += 4 * stride) {
        u32x4 v0, v1, v2, v3;
        if (NT) {
            v0 = __builtin_nontemporal_load(p + i); v1 = __builtin_nontemporal_load(p + i + stride);
            v2 = __builtin_nontemporal_load(p + i + 2 * stride); v3 = __builtin_nontemporal_load(p + i + 3 * stride);
        } else {
            v0 = p[i]; v1 = p[i + stride]; v2 = p[i + 2 * stride]; v3 = p[i + 3 * stride];
        }
        acc ^= v0 ^ v1 ^ v2 ^ v3;
    }
    for (; i < n; i += stride) acc ^= p[i];
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) out[0] = 1u;
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------------------------------------
// per-sequence state and row metadata
// ------------------------------------------------------------------------------------------
struct SeqState {       // device arrays, one entry per sequence
    int *len;           // j: committed tokens
    int *dr_len;        // tokens in the drafter cache
    int *pending;       // x_j
    int *ing_n;         // committed tokens the drafter has not cached yet
    int *ing_tok;       // [B][32]
    int *finished;      // EOS seen
};

// The rows of a pass have two numberings.  GEMM rows are packed: the rows of all sequences follow each other without gaps,
// so that no row tile is multiplied for padding but the end of the last one.  Attention works on tiles of 32 query rows
// of one sequence; attention row = 32 * attention tile + r.  The QKV epilogue writes a row's Q fragments at its attention
// row, the attention kernels write their result at the GEMM row.
struct RowMeta {
    int *pos, *slot, *seq, *qrow;         // [GEMM rows]; slot < 0: do not write K,V; qrow: the attention row, < 0: none (padding)
    int *limit, *grow;                    // [attention rows]: visible keys (0: no such row), GEMM row (< 0: none)
    int *tile_seq;                        // [attention tiles]
};

// token ids that reach the embedding gather are forced into [0, vocab): drafts come from caller memory
__device__ __forceinline__ int safe_tok(int t, int vocab) { return (t < 0 || t >= vocab) ? 0 : t; }

// Rows of a verify or draft pass (Alg. 1: one pass per model and iteration).
//   verify: sequence b has nrows GEMM rows [x_j, y^_1 .. y^_{nrows-1}] from b * nrows on and attention tile b; row i at
//   position j - 1 + i, causal over the cache.  nrows = k, or k + 1 when the bonus token is on (the last draft is a row too).
//   draft: first the k MASK rows of every sequence (GEMM rows b * k ..; positions j..j+k-1; they see the cache, the ingested
//   rows and every MASK row; their K,V land in slots past the cached length and are never kept), then the not-yet-cached
//   committed tokens of all sequences, causal.  Attention tile b holds the MASK rows; the committed tokens of b follow them
//   there if they fit for every sequence (share), else they have the tile B + b.  The first n_fixed block rows hold the
//   tokens fixed[b][0 .. n_fixed) instead of the MASK id (a partially filled block: a later pass of a multi-pass draft).
//   prefill: attention tile t holds desc[t].z & 63 rows of sequence desc[t].x, causal, at positions desc[t].y + r, whose token
//   ids start at ids[desc[t].w]; they are the GEMM rows from desc[t].z >> 6 on (packed over all sequences of the pass).
enum { ROWS_VERIFY = 0, ROWS_DRAFT = 1, ROWS_PREFILL = 2 };
struct PassRows {
    int kind;
    SeqState st;
    const int *tokens;               // verify: the draft tokens [B][k]; draft: the fixed tokens [B][k] (n_fixed > 0)
    int k, nrows, vocab;             // nrows: verify rows per sequence
    int mask_id, n_fixed;
    int B, share, n_ingest;          // sequences; draft: committed tokens in all that the drafter has not cached
    const int4 *desc; const int *ids; int n_desc;   // prefill
};
struct RowDesc { int tok, pos, slot, seq, qrow; };

// running sums of the sequences' counts of not-yet-cached tokens: pref[b] = those before b, pref[B] = all; 256 threads
__device__ __forceinline__ void ingest_prefix(const PassRows &p, int *pref) {
    for (int b = threadIdx.x; b < p.B; b += 256) pref[b + 1] = p.st.ing_n[b];
    __syncthreads();
    if (threadIdx.x < 64) {
        const int per = (p.B + 63) >> 6, b0 = min(p.B, (int)threadIdx.x * per), b1 = min(p.B, b0 + per);
        int sum = 0;
        for (int b = b0; b < b1; ++b) { sum += pref[b + 1]; pref[b + 1] = sum; }
        int run = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __builtin_amdgcn_ds_bpermute(((int)threadIdx.x - off) << 2, run);
            if ((int)threadIdx.x >= off) run += v;
        }
        for (int b = b0; b < b1; ++b) pref[b + 1] += run - sum;
        if (threadIdx.x == 0) pref[0] = 0;
    }
    __syncthreads();
}

// GEMM row g
__device__ __forceinline__ RowDesc pass_row(const PassRows &p, const int *pref, int g) {
    RowDesc d{0, 0, -1, 0, -1};
    if (p.kind == ROWS_PREFILL) {
        // tiles hold at most 32 rows, so row g lies in tile g / 32 (every tile before it is full) or a later one
        int lo = min(g >> 5, p.n_desc - 1), hi = p.n_desc - 1;
        int4 c = p.desc[lo];
        if (g - (c.z >> 6) >= (c.z & 63)) {
            while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if ((p.desc[mid].z >> 6) <= g) lo = mid; else hi = mid - 1; }
            c = p.desc[lo];
        }
        const int r = g - (c.z >> 6);
        if (r < (c.z & 63)) d = RowDesc{p.ids[c.w + r], c.y + r, c.y + r, c.x, lo * 32 + r};
        return d;
    }
    if (p.kind == ROWS_VERIFY) {
        const int b = g / p.nrows, r = g - b * p.nrows;
        if (b < p.B) {
            const int pos = p.st.len[b] - 1 + r;
            d = RowDesc{safe_tok(r == 0 ? p.st.pending[b] : p.tokens[b * p.k + r - 1], p.vocab), pos, pos, b, b * 32 + r};
        }
        return d;
    }
    const int b = g / p.k, r = g - b * p.k;
    if (b < p.B) {
        const int j = p.st.len[b];
        d = RowDesc{r < p.n_fixed ? safe_tok(p.tokens[b * p.k + r], p.vocab) : p.mask_id, j + r, j + r, b, b * 32 + r};
    } else if (p.n_ingest > 0) {
        const int q = g - p.B * p.k;
        if (q < pref[p.B]) {
            int lo = 0, hi = p.B - 1;   // the sequence with pref[lo] <= q < pref[lo + 1]
            while (lo < hi) { const int mid = (lo + hi) >> 1; if (q < pref[mid + 1]) hi = mid; else lo = mid + 1; }
            const int i = q - pref[lo], pos = p.st.dr_len[lo] + i;
            d = RowDesc{safe_tok(p.st.ing_tok[lo * 32 + i], p.vocab), pos, pos, lo, p.share ? lo * 32 + p.k + i : (p.B + lo) * 32 + i};
        }
    }
    return d;
}

// attention row r of tile t: its key limit and GEMM row; b: the tile's sequence
__device__ __forceinline__ void pass_attn_row(const PassRows &p, const int *pref, int t, int r, int &b, int &limit, int &grow) {
    limit = 0; grow = -1;
    if (p.kind == ROWS_PREFILL) {
        const int4 c = p.desc[t];
        b = c.x;
        if (r < (c.z & 63)) { limit = c.y + r + 1; grow = (c.z >> 6) + r; }
        return;
    }
    b = t < p.B ? t : t - p.B;
    if (p.kind == ROWS_VERIFY) {
        if (r < p.nrows) { limit = p.st.len[b] + r; grow = b * p.nrows + r; }
        return;
    }
    if (t < p.B && r < p.k) { limit = p.st.len[b] + p.k; grow = b * p.k + r; return; }
    if (p.n_ingest == 0) return;
    const int i = t < p.B ? (p.share ? r - p.k : 32) : r;
    if (i < pref[b + 1] - pref[b]) { limit = p.st.dr_len[b] + i + 1; grow = p.B * p.k + pref[b] + i; }
}

// ------------------------------------------------------------------------------------------
// write a 32 x 128 fp32 tile (LDS, stride RED_STRIDE) into fragment layout (hi/lo) at k-columns
// k0 .. k0+127 of a tile with KS k-steps; 512 (row, octet) items over 256 threads
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void tile_to_frag(const float *tile, uint4 *xhi, uint4 *xlo, size_t tile_base_vec, int k0) {
    for (int item = threadIdx.x; item < 512; item += 256) {
        int row = item & 31, oct = item >> 5;
        uint4 hi, lo;
        pack8_split(tile + row * RED_STRIDE + oct * 8, hi, lo);
        size_t v = tile_base_vec + frag_vec(row, (k0 >> 3) + oct);
        xhi[v] = hi;
        xlo[v] = lo;
    }
}

// embedding gather of one (column group, tile): h[row] = E[tok[row]] (bf16 table), plus fragment planes (the value itself and
// zero: the table is bf16) and sums of squares per row and 128 / ssq_sub columns;
// tok: the tile's 32 token ids (global memory or LDS); 256 threads.  16 threads per row, 8 columns each, all in registers:
// the launch is a chain of latencies (token, table row, stores), and a tile in LDS with one thread per row for the sums made
// it 17 us for a prompt of 7 row tiles, 8 us for the smallest.
__device__ __forceinline__ void embed_tile(const uint16_t *__restrict__ E, const int *tok, float *__restrict__ h,
                                           uint4 *__restrict__ xhi, uint4 *__restrict__ xlo, float *__restrict__ ssq, int d,
                                           int ncg, int ssq_sub, int cg, int t) {
    uint4 v[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int item = threadIdx.x + 256 * i, row = item >> 4, oct = item & 15;
        v[i] = *(const uint4 *)(E + (size_t)tok[row] * d + cg * CG + oct * 8);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int item = threadIdx.x + 256 * i, row = item >> 4, oct = item & 15;
        const size_t grow = (size_t)t * 32 + row;
        const float4 lo4 = make_float4(bf2f(v[i].x & 0xffffu), __uint_as_float(v[i].x & 0xffff0000u), bf2f(v[i].y & 0xffffu), __uint_as_float(v[i].y & 0xffff0000u));
        const float4 hi4 = make_float4(bf2f(v[i].z & 0xffffu), __uint_as_float(v[i].z & 0xffff0000u), bf2f(v[i].w & 0xffffu), __uint_as_float(v[i].w & 0xffff0000u));
        float4 *hp = (float4 *)(h + grow * d + cg * CG + oct * 8);
        hp[0] = lo4;
        hp[1] = hi4;
        const size_t vec = (size_t)t * (d / 16) * 64 + frag_vec(row, cg * 16 + oct);
        xhi[vec] = v[i];
        xlo[vec] = make_uint4(0u, 0u, 0u, 0u);
        // the squares in column order: the running sum moves from a row's lane to the next (row_shr:1), so that after as many
        // steps as a block has lanes its last lane has the whole sum
        const float x[8] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
        const int lanes = 16 / ssq_sub, at = oct & (lanes - 1);
        float s = 0.f;
        for (int step = 0; step < lanes; ++step) {
            const float before = dppf<0x111>(s);
            s = at == 0 ? 0.f : before;
#pragma unroll
            for (int e = 0; e < 8; ++e) s = fmaf(x[e], x[e], s);
        }
        if (at == lanes - 1) ssq[grow * (ncg * ssq_sub) + cg * ssq_sub + oct / lanes] = s;
    }
}

// The start of a pass in one launch: every block works out its tile's rows (pass_row), then blocks
// x < ncg gather the embeddings of column group x, block x == ncg writes the row metadata and the tile's RoPE table; block
// x == ncg + 1 writes the metadata of attention tile y.  (Three launches of a few microseconds each left the GPU waiting
// for the host at the start of every pass.)
__global__ __launch_bounds__(256) void k_pass_begin(PassRows p, RowMeta rm, const uint16_t *__restrict__ E, float *__restrict__ h,
                                                    uint4 *__restrict__ xhi, uint4 *__restrict__ xlo, float *__restrict__ ssq,
                                                    int d, int ncg, int ssq_sub, const double *__restrict__ theta,
                                                    float2 *__restrict__ cs, int half, int ntiles, int n_attn) {
    __shared__ int s_tok[32], s_pos[32], s_pref[1025];
    const int t = blockIdx.y;
    if (t >= ((int)blockIdx.x == ncg + 1 ? n_attn : ntiles)) return;
    if (p.kind == ROWS_DRAFT && p.n_ingest > 0) ingest_prefix(p, s_pref);
    if ((int)blockIdx.x == ncg + 1) {
        if (threadIdx.x < 32) {
            int b, limit, grow;
            pass_attn_row(p, s_pref, t, threadIdx.x, b, limit, grow);
            rm.limit[t * 32 + threadIdx.x] = limit; rm.grow[t * 32 + threadIdx.x] = grow;
            if (threadIdx.x == 0) rm.tile_seq[t] = b;
        }
        return;
    }
    if (threadIdx.x < 32) {
        const int row = t * 32 + threadIdx.x;
        const RowDesc r = pass_row(p, s_pref, row);
        s_tok[threadIdx.x] = r.tok; s_pos[threadIdx.x] = r.pos;
        if ((int)blockIdx.x == ncg) { rm.pos[row] = r.pos; rm.slot[row] = r.slot; rm.seq[row] = r.seq; rm.qrow[row] = r.qrow; }
    }
    __syncthreads();
    if ((int)blockIdx.x < ncg) {
        embed_tile(E, s_tok, h, xhi, xlo, ssq, d, ncg, ssq_sub, blockIdx.x, t);
    } else {
        for (int idx = threadIdx.x; idx < 32 * half; idx += 256) {
            const int row = idx / half, i = idx - row * half;
            double sn, c;
            sincos((double)s_pos[row] * theta[i], &sn, &c);
            cs[(size_t)(t * 32 + row) * half + i] = make_float2((float)c, (float)sn);
        }
    }
}

// ------------------------------------------------------------------------------------------
// weight-streaming GEMM for short row counts with the layer's elementwise work fused behind it
//   y[i][n] = sum_k x[i][k] W[k][n]  for MT row tiles of 32 and one group of 128 columns per block.
//   grid: x = column group, y = split s of the K range, z = group of MT row tiles.
//   block: 8 waves; wave w streams k-slice (s*8 + w) of 8*S for all 4 column blocks of the group
//   (one activation fragment pair feeds 4 weight fragments); the 8 waves are summed through LDS in a
//   fixed tree.  S == 1: the epilogue runs on the tile in LDS.  S > 1: the tile goes to a partial
//   buffer and the block that arrives last at the group's counter sums the S partials in order
//   s = 0..S-1 and runs the epilogue, so results do not depend on arrival order.
//   Row tiles of the launch: z*MT + mt.
// ------------------------------------------------------------------------------------------
enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LMHEAD = 3, EPI_ROUTER = 4 };

struct KvView {
    uint16_t *k, *vt;                                  // layer base already applied
    size_t seq_stride, head_stride;                    // elements
    int max_seq;
};

// Both caches are stored per (sequence, kv head) in blocks of 32 slots (one key tile), and inside a block in the
// order the attention kernels' MFMA operands want them: head_dim / 16 fragments of 64 lanes x 8 elements, so that
// a wave reads a fragment as one contiguous 1 KB and every cache line it touches is used whole.
//   K block, fragment s (k-step: elements 16 s .. 16 s + 15): lane (operand row r, half) holds elements
//   16 s + 8 half .. + 7 of the key whose operand row is r.  Operand rows are a permutation of the keys that gives
//   each lane of the S^T result 16 consecutive keys: key = 16 * bit2(r) + 4 * (r >> 3) + (r & 3).
//   V^T block, fragment (O^T tile tt, s2): lane (channel c = 32 tt + (lane & 31), half) holds keys
//   16 half + 8 s2 .. + 7 of channel c.
__device__ __forceinline__ int key_operand_row(int key) { return (key & 3) | (((key >> 4) & 1) << 2) | (((key >> 2) & 3) << 3); }
// element offset of octet `oct` (8 elements of head_dim) of slot `slot` inside a (sequence, kv head) K region
__device__ __forceinline__ size_t k_cache_off(int slot, int oct, int hd) {
    return ((size_t)(slot >> 5) * (hd >> 4) + (oct >> 1)) * 512 + ((oct & 1) * 32 + key_operand_row(slot & 31)) * 8;
}
// element offset of channel c of slot `slot` inside a (sequence, kv head) V^T region
__device__ __forceinline__ size_t v_cache_off(int slot, int c, int hd) {
    const int kk = slot & 31;
    return ((size_t)(slot >> 5) * (hd >> 4) + (c >> 5) * 2 + ((kk >> 3) & 1)) * 512 + ((kk >> 4) * 32 + (c & 31)) * 8 + (kk & 7);
}

struct RowStat {   // per (row, column group) partial over 128 vocabulary entries
    float m; int idx;        // max logit, its index (lowest on ties)
    float sumexp;            // sum exp(z/T - m/T)  (T > 0)
    float gm; int gidx;      // max of z/T + Gumbel, its index (T > 0)
};

// A load whose data nobody wants: it pulls a line into the L2.  The data goes to LDS (lane l's 16 bytes land at
// sink + 16 l: 1 KB per wave that the workgroup no longer needs), not to registers: a register that waits for a load
// has to be kept away from the compiler's allocator until the data is back, and nothing in the language does that
// across branches and loops.  The caller ends with wait_loads<0>(): the LDS must still be the workgroup's when the data
// arrives.
__device__ __forceinline__ void load16_discard(void *sink, const void *p) {
    asm volatile("; fetch ahead");
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)p,
                                     (void __attribute__((address_space(3))) *)sink, 16, 0, 0);
}

// What the NEXT launch of the stream will read first, for workgroups of this launch that have nothing left to do:
// they pull it into their XCD's L2 while the launch's last workgroups finish (memory is idle then), so that the next
// launch's first k-steps hit there.  Workgroup ids 8 apart share an XCD in both launches; workgroup j of this launch
// fetches for workgroup j of the next.
//   narrow_nb == 0 (the order of k_gemm and k_gemm_slim): next-launch workgroup j works on column group j % ncg and K split
//     j / ncg; fetched: the first `span` bytes of the split's K range in each of the group's nblk 32-column blocks, which
//     are adjacent or (pairs) the blocks of slim_block.
//   narrow_nb = NB > 0 (k_gemm_narrow's order): j = 8 * ((p / 8) * Z + z) + p % 8 is row tile z of the group p of NB
//     blocks, all of K; the Z workgroups of a group read the same (contiguous) NB * block_bytes: part z of Z is fetched.
struct NextWeights {
    const char *base;          // the next launch's weight matrix, fragment layout; null: nothing to fetch
    int nwg, ncg;              // its workgroups and column groups (narrow: groups of NB blocks)
    int span;                  // bytes fetched per 32-column block, from the start of the split's K range
    long long block_bytes;     // one 32-column block: KS * 1024
    long long split_bytes;     // a split's K range within a block
    int narrow_nb, Z;
    int nblk, pairs;           // 32-column blocks of a column group (k_gemm: 4)
};

// First 32-column block of column group p of k_gemm_slim and the distance to its second.  pairs: blocks two apart inside a
// group of four — a gate block and its up block, or the two halves of a 128-wide head (a rotation pair lies in both).
__device__ __forceinline__ int slim_block(int p, int C, bool pairs, int j) {
    return pairs ? ((p >> 1) << 2) + (p & 1) + 2 * j : p * C + j;
}

// lds: 8 KB of LDS the workgroup is done with
__device__ __forceinline__ void prefetch_next(const NextWeights &nx, void *lds) {
    if (!nx.base) return;
    // one next-launch workgroup per workgroup and no more: what is fetched must be back before this launch can end
    const int lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const int tid = opaque_tid();
    char *sink = (char *)lds + (__builtin_amdgcn_readfirstlane(tid >> 6) << 10);
    if (lin < nx.nwg && nx.narrow_nb > 0) {
        const int q8 = lin >> 3, z = q8 % nx.Z, grp = 8 * (q8 / nx.Z) + (lin & 7);
        if (grp < nx.ncg) {
            const int total = nx.narrow_nb * (int)nx.block_bytes;             // the group's blocks are adjacent
            const int part = ((total / 16 + nx.Z - 1) / nx.Z) * 16;
            const int end = min(total, (z + 1) * part);
            const char *p0 = nx.base + (long long)grp * total;
            for (int o = z * part + tid * 16; o < end; o += 512 * 16) load16_discard(sink, p0 + o);
        }
    } else if (lin < nx.nwg) {
        const int j = lin;
        const int cg = j % nx.ncg, sp = j / nx.ncg;
        const long long s_off = sp * nx.split_bytes;
        const int len = (int)min((long long)nx.span, nx.block_bytes - s_off);   // stays inside the block
        for (int nb = 0; nb < nx.nblk; ++nb) {
            const char *p0 = nx.base + (long long)slim_block(cg, nx.nblk, nx.pairs, nb) * nx.block_bytes + s_off;
            for (int o = tid * 16; o < len; o += 512 * 16) load16_discard(sink, p0 + o);
        }
    }
    wait_loads<0>();
}

// The same for the per-head attention launch that follows a QKV projection: its workgroups on XCD x work on kv head
// x % Hkv (Hkv divides 8; one sequence), so this launch's idle workgroups on XCD x pull that head's old K and V^T blocks
// — whole key tiles that this launch does not write — into its L2.
__device__ __forceinline__ void prefetch_kv(const uint16_t *k, const uint16_t *vt, size_t head_stride, int Hkv, int bytes, void *lds) {
    if (bytes <= 0) return;
    const int lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const int nlin = gridDim.x * gridDim.y * gridDim.z;
    const int per_x = (nlin - (lin & 7) + 7) >> 3;
    const int tid = opaque_tid();
    const size_t head = (size_t)((lin & 7) % Hkv) * head_stride;
    const char *kb = (const char *)(k + head), *vb = (const char *)(vt + head);
    char *sink = (char *)lds + (__builtin_amdgcn_readfirstlane(tid >> 6) << 10);
    for (int o = ((lin >> 3) * 512 + tid) * 16; o < bytes; o += per_x * 8192) {   // the host bounds `bytes`: a few trips
        load16_discard(sink, kb + o);
        load16_discard(sink, vb + o);
    }
    wait_loads<0>();
}

struct GemmArgs {
    NextWeights nx;
    int kv_fetch_bytes;   // QKV launch before a per-head attention launch over one sequence: bytes of each kv head's K (and V^T) blocks to pull in, or 0
    const uint4 *W, *Xhi, *Xlo;
    float *part; int *counters;
    int N, KS, S, rows_total;
    // RMSNorm of the GEMM input rows: rstd from per-group sums of squares (QKV, SWIGLU, LMHEAD)
    const float *ssq_in; int ncg_in, d_in; float eps;
    // QKV: RoPE, Q fragments, cache writes
    const float2 *cs; RowMeta rm; uint4 *qhi, *qlo; KvView kv; int Hq, Hkv, hd;
    // RESID: h += y, new fragments and sums of squares of h
    float *h; uint4 *xhi_out, *xlo_out; float *ssq_out;
    int ssq_sub;   // sums of squares per row and 128-column group: 1, 2 (passes with slim launches) or 4 (narrow launches of a small model)
    int slim;      // the pass may use k_gemm_slim
    // SWIGLU: activation fragments over F channels
    uint4 *ahi, *alo; int F;
    // LMHEAD: logits, per-group row statistics
    int k, n_lm; float *logits; float T; uint64_t seed; RowStat *stat; int ncg_v;   // n_lm: rows with logits, k of each sequence, the first GEMM rows of the pass
    int draw;   // T > 0: also the Gumbel-max of the perturbed logits (a pass that samples its rows' tokens)
    unsigned long long *stamps;   // debugging: [workgroup][8] device-clock stamps of this launch, or null
    int k_lo;   // rows below k_lo keep the logits and statistics of an earlier pass (multi-pass draft)
    // ROUTER: top-k of softmax over n_experts (<= 128), renormalised
    int n_experts, top_k; int *route_e; float *route_w;
    int route_spread;   // 0: the model's routing; layer + 1: synthetic uniform routing (benchmarks of random-init mixtures)
};

// rstd[row] = rsqrt(sum_g ssq[row][g] / d + eps) for the 32 rows of a tile, into LDS.  512 threads: 16 per
// row, each sums the groups g = j, j + 16, .. in order, then a fixed butterfly over the 16 partial sums.
__device__ __forceinline__ void tile_rstd(const float *ssq, float *rstd, int grow0, int ncg, int d, float eps) {
    const int tidx = opaque_tid();
    const int row = tidx >> 4, j = tidx & 15;
    const float *p = ssq + (size_t)(grow0 + row) * ncg;
    float s = 0.f;
    for (int g = j; g < ncg; g += 16) s += p[g];
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) s += shx(s, off);
    if (j == 0) rstd[row] = rsqrtf(s / (float)d + eps);
}

// QKV epilogue: RMSNorm scale, RoPE, Q -> fragment planes per head, K -> cache, V -> transposed cache
// The tile holds columns cg * WIDTH .. + WIDTH - 1 with row stride STRIDE.  WIDTH is a multiple of head_dim, so that
// a head, and with it every rotation pair, lies inside one tile.
// pre (optional): what qkv_prefetch loaded for this thread's item while the tile was still being summed.
constexpr int QKV_PRE = 19;   // 8 (cos, sin) pairs, the row's cache slot, its sequence, its attention row
template <int WIDTH = CG, int STRIDE = RED_STRIDE, bool PRE = false>
__device__ __forceinline__ void epi_qkv(const GemmArgs &a, const float *tile, const float *rstd, int cg, int t,
                                        const float (&pre)[QKV_PRE]) {
    const int tidx = opaque_tid();
    const int hd = a.hd, Hq = a.Hq, Hkv = a.Hkv;
    const int half_hd = hd >> 1;
    constexpr int RED_STRIDE = STRIDE;   // the row stride of this tile
    for (int item = tidx; item < 4 * WIDTH; item += 512) {   // GEMM workgroups have 512 threads
        const int row = item & 31, oct = item >> 5;
        const int grow = t * 32 + row;
        const int col0 = cg * WIDTH + oct * 8;     // first of 8 columns, all in one head
        const int kind = col0 < Hq * hd ? 0 : (col0 < (Hq + Hkv) * hd ? 1 : 2);
        const int hc = col0 - (kind == 0 ? 0 : (kind == 1 ? Hq * hd : (Hq + Hkv) * hd));
        const int head = hc / hd, i0 = hc % hd;
        const float sc = rstd[row];
        float v[8];
        if (kind < 2) {
            const int poff = (i0 < half_hd) ? half_hd : -half_hd;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float x = tile[row * RED_STRIDE + oct * 8 + e] * sc;
                float xp = tile[row * RED_STRIDE + oct * 8 + e + poff] * sc;
                const float2 c = PRE ? make_float2(pre[2 * e], pre[2 * e + 1]) : a.cs[(size_t)grow * half_hd + ((i0 + e) % half_hd)];
                v[e] = (i0 < half_hd) ? x * c.x - xp * c.y : x * c.x + xp * c.y;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = tile[row * RED_STRIDE + oct * 8 + e] * sc;
        }
        if (kind == 0) {
            uint4 hi, lo;
            pack8_split(v, hi, lo);
            const int qr = PRE ? __float_as_int(pre[18]) : a.rm.qrow[grow];
            if (qr >= 0) {
                size_t vec = ((size_t)((qr >> 5) * Hq + head) * (hd / 16)) * 64 + frag_vec(qr & 31, i0 >> 3);
                a.qhi[vec] = hi;
                a.qlo[vec] = lo;
            }
        } else {
            const int slot = PRE ? __float_as_int(pre[16]) : a.rm.slot[grow];
            if (slot >= 0) {
                const int b = PRE ? __float_as_int(pre[17]) : a.rm.seq[grow];
                size_t base = (size_t)b * a.kv.seq_stride + (size_t)head * a.kv.head_stride;
                if (kind == 1) {
                    *(uint4 *)(a.kv.k + base + k_cache_off(slot, i0 >> 3, hd)) = pack8(v);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        a.kv.vt[base + v_cache_off(slot, i0 + e, hd)] = (uint16_t)f2bf(v[e]);
                }
            }
        }
    }
}

// The QKV epilogue's own inputs (RoPE factors, cache slot, sequence) of this thread's item, requested before the
// tile is ready so that they are not one more round trip behind it.  One item per thread: WIDTH <= 128.
template <int WIDTH = CG>
__device__ __forceinline__ void qkv_prefetch(const GemmArgs &a, float (&pre)[QKV_PRE], int cg, int t) {
    const int item = opaque_tid();
#pragma unroll
    for (int i = 0; i < QKV_PRE; ++i) pre[i] = 0.f;
    if (item >= 4 * WIDTH) return;
    const int hd = a.hd, Hq = a.Hq, Hkv = a.Hkv, half_hd = hd >> 1;
    const int row = item & 31, oct = item >> 5, grow = t * 32 + row;
    const int col0 = cg * WIDTH + oct * 8;
    const int kind = col0 < Hq * hd ? 0 : (col0 < (Hq + Hkv) * hd ? 1 : 2);
    const int hc = col0 - (kind == 0 ? 0 : (kind == 1 ? Hq * hd : (Hq + Hkv) * hd));
    const int i0 = hc % hd;
    if (kind < 2) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float2 c = a.cs[(size_t)grow * half_hd + ((i0 + e) % half_hd)];
            pre[2 * e] = c.x; pre[2 * e + 1] = c.y;
        }
    }
    if (kind >= 1) { pre[16] = __int_as_float(a.rm.slot[grow]); pre[17] = __int_as_float(a.rm.seq[grow]); }
    else pre[18] = __int_as_float(a.rm.qrow[grow]);
}

// O-proj / down-proj epilogue: h += y; new fragment planes of h; per-group sum of squares.
// `hreg` holds the old h values of this thread's elements e = threadIdx.x + 512*i (row e>>7, column e&127),
// loaded by resid_prefetch() before the tile was ready.  `tile` is overwritten with the new h values.
__device__ __forceinline__ void resid_prefetch(const GemmArgs &a, float (&hreg)[8], int cg, int t) {
    const int tidx = opaque_tid();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int e = tidx + 512 * i;
        const float *hp = a.h + (size_t)(t * 32 + (e >> 7)) * a.N + cg * CG + (e & 127);
        hreg[i] = *hp;
    }
}

__device__ __forceinline__ void epi_resid(const GemmArgs &a, float *tile, float *scratch, const float (&hreg)[8], int cg, int t) {
    const int tidx = opaque_tid();
    const int N = a.N;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int e = tidx + 512 * i;
        const int row = e >> 7, col = e & 127;
        const float v = hreg[i] + tile[row * RED_STRIDE + col];
        float *hp = a.h + (size_t)(t * 32 + row) * N + cg * CG + col;
        *hp = v;
        tile[row * RED_STRIDE + col] = v;
    }
    __syncthreads();
    {   // 512 (row, octet) items, one per thread; lanes l and l^32 of a wave hold two octets of the same row
        const int row = tidx & 31, oct = tidx >> 5;
        const float *tp = tile + row * RED_STRIDE + oct * 8;
        uint4 hi, lo;
        pack8_split(tp, hi, lo);
        size_t v = (size_t)t * (N / 16) * 64 + frag_vec(row, cg * 16 + oct);
        a.xhi_out[v] = hi;
        a.xlo_out[v] = lo;
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += tp[e] * tp[e];
        ss += shx(ss, 32);
        if ((tidx & 63) < 32) scratch[(tidx >> 6) * 32 + row] = ss;   // [8 waves][32 rows]
    }
    __syncthreads();
    if (a.ssq_sub == 4) {   // wave w holds the octets 2w, 2w + 1: waves 2b, 2b + 1 make 32-column block b
        if (tidx < 128) {
            const int row = tidx & 31, blk = tidx >> 5;
            a.ssq_out[(size_t)(t * 32 + row) * (N / 32) + cg * 4 + blk] = scratch[(2 * blk) * 32 + row] + scratch[(2 * blk + 1) * 32 + row];
        }
    } else if (a.ssq_sub == 2) {   // waves 4b .. 4b + 3 make 64-column block b
        if (tidx < 64) {
            const int row = tidx & 31, blk = tidx >> 5;
            float s2 = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) s2 += scratch[(4 * blk + w) * 32 + row];
            a.ssq_out[(size_t)(t * 32 + row) * (N / 64) + cg * 2 + blk] = s2;
        }
    } else if (tidx < 32) {
        float s2 = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) s2 += scratch[w * 32 + tidx];   // fixed order
        a.ssq_out[(size_t)(t * 32 + tidx) * (N / CG) + cg] = s2;
    }
}

// gate/up epilogue: group = 64 gate + 64 up channels -> SiLU(g) * u, fragment planes over F.  Four channels per thread, so that
// all eight waves work and the code, which every launch reads anew, is half as long.
__device__ __forceinline__ void epi_swiglu(const GemmArgs &a, const float *tile, const float *rstd, int cg, int t) {
    const int tidx = opaque_tid();
    const int row = tidx & 31, c4 = (tidx >> 5) * 4;   // 16 groups of 4 channels
    const float sc = rstd[row];
    const float *tp = tile + row * RED_STRIDE + c4;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float g = tp[e] * sc, u = tp[64 + e] * sc;
        v[e] = g / (1.f + expf(-g)) * u;
    }
    const uint32_t h0 = f2bf2(v[0], v[1]), h1 = f2bf2(v[2], v[3]);
    const uint32_t l0 = f2bf2(v[0] - __uint_as_float(h0 << 16), v[1] - __uint_as_float(h0 & 0xffff0000u));
    const uint32_t l1 = f2bf2(v[2] - __uint_as_float(h1 << 16), v[3] - __uint_as_float(h1 & 0xffff0000u));
    const size_t at = ((size_t)t * (a.F / 16) * 64 + frag_vec(row, cg * 8 + (c4 >> 3))) * 2 + ((c4 >> 2) & 1);   // half a vector
    ((uint2 *)a.ahi)[at] = make_uint2(h0, h1);
    ((uint2 *)a.alo)[at] = make_uint2(l0, l1);
}

// LM-head epilogue: RMSNorm scale, optional logits store, per-(row, group) argmax / sumexp / Gumbel-max.
// LM rows are the first n_lm GEMM rows of the pass, k of each sequence.
__device__ __forceinline__ void epi_lmhead(const GemmArgs &a, const float *tile, const float *rstd, int cg, int t) {
    const int tidx = opaque_tid();
    if (tidx >= 256) return;
    const int V = a.N;
    const float T = a.T;
    const int row = tidx >> 3, sub = tidx & 7;   // 8 threads per row, 16 columns each
    const size_t lm = (size_t)t * 32 + row;
    const bool live = (int)lm < a.n_lm && (int)lm % opaque_s(a.k) >= a.k_lo;
    // The logits are taken from the tile wherever they are needed, in loops of four: unrolled, with the Gumbel draws between
    // the comparisons, the epilogue was 30 KB of code, and every launch reads its code anew (one row tile,
    // mean of the heads of d = 4096 and 896 154.4 -> 150.3 us, of 2560 and 896 118.1 -> 115.9).
    float m = -INFINITY, gm = -INFINITY, se = 0.f;
    int idx = 0x7fffffff, gidx = 0x7fffffff;
    const float invT = T > 0.f ? 1.f / T : 1.f;
    const float sc = rstd[row];
    const float4 *tp = (const float4 *)(tile + row * RED_STRIDE + sub * 16);
    if (live) {
        float4 *q = a.logits ? (float4 *)(a.logits + lm * V + (size_t)cg * CG + sub * 16) : nullptr;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float4 z = make_float4(tp[e].x * sc, tp[e].y * sc, tp[e].z * sc, tp[e].w * sc);
            if (q) q[e] = z;
            const int v = cg * CG + sub * 16 + 4 * e;
            argmax_merge(m, idx, z.x, v); argmax_merge(m, idx, z.y, v + 1); argmax_merge(m, idx, z.z, v + 2); argmax_merge(m, idx, z.w, v + 3);
        }
        if (T > 0.f && a.draw) {
            const uint64_t key = row_key(a.seed, TAG_DRAFT, (uint64_t)a.rm.seq[lm], (uint64_t)a.rm.pos[lm]);
#pragma unroll 2
            for (int e = 0; e < 16; ++e) {
                const int v = cg * CG + sub * 16 + e;
                argmax_merge(gm, gidx, ((const float *)tp)[e] * sc * invT + gumbel(key, (uint64_t)v), v);
            }
        }
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) {
        float m2 = shx(m, off); int i2 = shx(idx, off);
        argmax_merge(m, idx, m2, i2);
        float g2 = shx(gm, off); int gi2 = shx(gidx, off);
        argmax_merge(gm, gidx, g2, gi2);
    }
    if (live && T > 0.f) {
#pragma unroll 4
        for (int e = 0; e < 16; ++e) se += expf((((const float *)tp)[e] * sc - m) * invT);
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) se += shx(se, off);
    if (live && sub == 0) {
        RowStat *sp = a.stat + lm * a.ncg_v + cg;
        sp->m = m; sp->idx = idx; sp->sumexp = se; sp->gm = gm; sp->gidx = gidx;
    }
}

// router epilogue: logits over the experts -> softmax -> top_k (lowest index on ties) -> weights renormalised to sum 1.
// 16 threads per row, 8 experts each.  A candidate is one 64-bit key, the bits of its (non-negative) weight above
// 128 - index, so that a comparison decides value and tie at once.  (With two values per candidate and exchanges
// through LDS the launch took 20 us, now 12.5.)
__device__ __forceinline__ void epi_router(const GemmArgs &a, const float *tile, const float *rstd, int t) {
    const int tidx = opaque_tid();
    const int row = tidx >> 4, sub = tidx & 15;
    const int grow = t * 32 + row;
    float z[8];
    float m = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int ex = sub * 8 + e;
        z[e] = ex < a.n_experts ? tile[row * RED_STRIDE + ex] * rstd[row] : -INFINITY;
        m = fmaxf(m, z[e]);
    }
    m = fmaxf(m, dppf<0xB1>(m)); m = fmaxf(m, dppf<0x4E>(m)); m = fmaxf(m, dppf<0x141>(m)); m = fmaxf(m, dppf<0x140>(m));
    float se = 0.f;
    uint64_t key[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float w = expf(z[e] - m);   // exp(-inf) = 0 for padding, which loses every tie
        se += w;
        key[e] = ((uint64_t)__float_as_uint(w) << 32) | (uint32_t)(128 - (sub * 8 + e));
    }
    se += dppf<0xB1>(se); se += dppf<0x4E>(se); se += dppf<0x141>(se); se += dppf<0x140>(se);
    float my_w = 0.f, wsum = 0.f;
    int my_e = 0;
    for (int j = 0; j < a.top_k; ++j) {
        uint64_t best = key[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) best = key[e] > best ? key[e] : best;
        best = dpp64_max<0xB1>(best); best = dpp64_max<0x4E>(best); best = dpp64_max<0x141>(best); best = dpp64_max<0x140>(best);
#pragma unroll
        for (int e = 0; e < 8; ++e) key[e] = key[e] == best ? 0 : key[e];   // taken (keys are distinct and at least 1)
        const float w = __uint_as_float((uint32_t)(best >> 32)) / se;
        wsum += w;
        if (sub == j) { my_w = w; my_e = 128 - (int)(uint32_t)best; }
    }
    if (sub >= a.top_k) return;
    if (a.route_spread) {
        // benchmarking stand-in for a trained router (a.route_spread - 1 = layer): every row gets top_k distinct
        // pseudo-random experts with equal weights, so a block touches about n (1 - (1 - top_k / n)^rows) experts
        const uint32_t base = (uint32_t)mix64(((uint64_t)a.route_spread << 32) | (uint32_t)grow);
        const uint32_t stride = ((uint32_t)(mix64(base) >> 7) | 1u);   // odd: distinct picks when n is a power of two
        a.route_e[grow * 8 + sub] = (int)((base + (uint32_t)sub * stride) % (uint32_t)a.n_experts);
        a.route_w[grow * 8 + sub] = 1.f / (float)a.top_k;
    } else {
        a.route_e[grow * 8 + sub] = my_e;
        a.route_w[grow * 8 + sub] = my_w / wsum;
    }
}

// RSTD_READY: `rstd` already holds the tile's factors (tile_rstd ran before a barrier the caller has passed).
template <int EPI, bool RSTD_READY = false>
__device__ __forceinline__ void run_epilogue(const GemmArgs &a, float *tile, float *rstd, float *scratch,
                                             const float (&hreg)[8], int cg, int t) {
    // caller has synchronised after filling `tile`
    if (EPI != EPI_RESID && !RSTD_READY) {
        tile_rstd(a.ssq_in, rstd, t * 32, a.ncg_in, a.d_in, a.eps);
        __syncthreads();
    }
    if (EPI == EPI_QKV) {
        // the wide workgroups load the epilogue's inputs here: requesting them ahead of the tile measured slower
        const float none[QKV_PRE] = {};
        epi_qkv<>(a, tile, rstd, cg, t, none);
    }
    else if (EPI == EPI_RESID) epi_resid(a, tile, scratch, hreg, cg, t);
    else if (EPI == EPI_SWIGLU) epi_swiglu(a, tile, rstd, cg, t);
    else if (EPI == EPI_ROUTER) epi_router(a, tile, rstd, t);
    else epi_lmhead(a, tile, rstd, cg, t);
}

// Sum of the 8 waves' accumulators (one 32 x 128 tile each, MFMA register layout) in the fixed order
// w = 0..7, result as a row-major tile (stride RED_STRIDE) in `tile`.
// Every wave parks its 16 register quads in LDS as 16-byte vectors [wave][quad][lane] (conflict-free);
// after one barrier wave w sums quads w and w + 8 over the eight copies (16 independent reads in
// flight per lane) and writes its 8 rows x 64 columns of the tile.  `red` holds 8 * 4096 floats.
// Ends with a barrier.
__device__ __forceinline__ void reduce_waves_to_tile(f32x16 (&acc)[4], float *red, float *tile, int w, int lane) {
    float4 *red4 = (float4 *)red;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            red4[(w * 16 + nb * 4 + q) * 64 + lane] = make_float4(acc[nb][4 * q], acc[nb][4 * q + 1], acc[nb][4 * q + 2], acc[nb][4 * q + 3]);
    barrier_keep_loads();   // LDS traffic only: loads requested earlier (next item, old h) stay in flight
    const int half = lane >> 5, cl = lane & 31;
    float4 v[2][8];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int ww = 0; ww < 8; ++ww) v[j][ww] = red4[(ww * 16 + w + 8 * j) * 64 + lane];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        float4 sum = v[j][0];
#pragma unroll
        for (int ww = 1; ww < 8; ++ww) { sum.x += v[j][ww].x; sum.y += v[j][ww].y; sum.z += v[j][ww].z; sum.w += v[j][ww].w; }
        const int slot = w + 8 * j, nb = slot >> 2, q = slot & 3;
        float *tp = tile + (8 * q + 4 * half) * RED_STRIDE + nb * 32 + cl;   // rows 8q + 4*half + 0..3
        tp[0] = sum.x; tp[RED_STRIDE] = sum.y; tp[2 * RED_STRIDE] = sum.z; tp[3 * RED_STRIDE] = sum.w;
    }
    barrier_keep_loads();   // LDS traffic only: loads requested earlier (next item, old h) stay in flight
}

struct GemmSmem {
    float red[8 * 32 * 128];          // wave-reduction scratch (128 KB)
    float tile[32 * RED_STRIDE];      // the finished 32 x 128 tile, row-major
    float rstd[64];                   // RMSNorm factors of up to two row tiles
    int last;
};

// Sums the S partial tiles of column group cg (row-tile group z) in order s = 0..S-1 and runs the epilogue.
// RSTD_EARLY: sm.rstd already holds the RMSNorm factors of the group's MT row tiles (gemm_block computed them
// while its first weights were on their way).
template <int MT, int EPI, bool RSTD_EARLY = false>
__device__ __forceinline__ void gemm_finish(const GemmArgs &a, GemmSmem &sm, int cg, int z) {
    const int tidx = opaque_tid();
    float *tile = sm.tile;
    const int N = a.N, S = a.S;
    float hreg[MT][8];
    float4 v[MT][2];
    // the sums of all MT row tiles first (their loads do not depend on each other's epilogue), then the epilogues
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int ct = z * MT + mt;
        if (EPI == EPI_RESID) resid_prefetch(a, hreg[mt], cg, ct);
        const size_t sstride = (size_t)a.rows_total * N;
        const float *p[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = tidx + 512 * i;
            p[i] = a.part + ((size_t)ct * 32 + (e >> 5)) * N + (size_t)cg * CG + (e & 31) * 4;
            v[mt][i] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        for (int s0 = 0; s0 < S; s0 += 8) {   // 8 splits x 2 x 16 bytes of loads in flight, summed in order
            u32x4 pv[8][2];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int i = 0; i < 2; ++i) load16_agent_async(pv[u][i], p[i] + (size_t)min(s0 + u, S - 1) * sstride);
            wait_loads<0>();
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s0 + u < S) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        tie(pv[u][i]);
                        v[mt][i].x += __uint_as_float(pv[u][i][0]); v[mt][i].y += __uint_as_float(pv[u][i][1]);
                        v[mt][i].z += __uint_as_float(pv[u][i][2]); v[mt][i].w += __uint_as_float(pv[u][i][3]);
                    }
                }
        }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int ct = z * MT + mt;
        if (mt > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = tidx + 512 * i;
            float *tp = tile + (e >> 5) * RED_STRIDE + (e & 31) * 4;
            tp[0] = v[mt][i].x; tp[1] = v[mt][i].y; tp[2] = v[mt][i].z; tp[3] = v[mt][i].w;
        }
        __syncthreads();
        run_epilogue<EPI, RSTD_EARLY>(a, tile, sm.rstd + 32 * mt, sm.red, hreg[mt], cg, ct);
    }
}

// Debugging aid: thread 0 of workgroup `lin` records the 100 MHz device clock at point i of the launch.
__device__ __forceinline__ void gemm_stamp(const GemmArgs &a, int lin, int i) {
    if (a.stamps && threadIdx.x == 0) a.stamps[lin * 8 + i] = wall_clock64();
}

// One work item of the weight-streaming GEMM: column group cg, K split s, row-tile group z.
// With S > 1 the block that arrives last at the group's counter finishes the group.
// WSTREAM: weights are read once by the whole grid (non-temporal loads); false: several workgroups of an XCD read
// the same weights at about the same time and should find them in its L2 (plain loads).
template <int MT, int EPI, bool WSTREAM = true>
__device__ __forceinline__ void gemm_block(const GemmArgs &a, GemmSmem &sm, int cg, int s, int z, int ncg) {
    const int tidx = opaque_tid();
    float *red = sm.red, *tile = sm.tile, *s_rstd = sm.rstd;
    const int w = __builtin_amdgcn_readfirstlane(tidx >> 6), lane = tidx & 63;   // the wave index as a scalar: scalar loop bounds
    const int N = a.N, KS = a.KS, S = a.S;
    // K range of the workgroup: split s of S equal parts; inside it wave w takes the k-steps w, w + 8, w + 16, ...: the
    // eight waves read neighbouring 1 KB fragments at about the same time and advance together (measured against one
    // contiguous eighth per wave: 8B verify pass 4.63 -> 4.60 ms)
    // Splits are whole multiples of 8 k-steps (8 KB per column block): ranges that start anywhere cost 1.4 us per launch
    // of the 8B shape's output projection (7 splits of 36.6 k-steps against 6 of 40 and one of 16).
    constexpr int KSTEP = 8;
    const int per = (KS + S * 8 - 1) / (S * 8);
    const int ks0 = s * 8 * per + w;
    const int ks1 = min(KS, (s + 1) * 8 * per);

    const int lin = (z * S + s) * ncg + cg;   // stamps: 0 start, 1 this wave's K slice multiplied, 2 tile stored
    gemm_stamp(a, lin, 0);                    // (epilogue done if S == 1), 3 arrived, 4 last workgroup's finish done
    f32x16 acc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mt][nb][r] = 0.f;

    const uint4 *wp = a.W + ((size_t)(cg * 4) * KS) * 64 + lane;
    const size_t wstride = (size_t)KS * 64;   // between column blocks
    const uint4 *xh[MT], *xl[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        size_t tl = (size_t)(z * MT + mt);
        xh[mt] = a.Xhi + tl * KS * 64 + lane;
        xl[mt] = a.Xlo + tl * KS * 64 + lane;
    }

    // Software pipeline: D k-steps of loads are in flight while older steps are multiplied.  The loads are issued and
    // waited for by hand (load16_async / wait_steps): left to the compiler, the loop waits for ALL outstanding loads once
    // per trip (its count of conditional loads across the back edge is not exact), which empties the pipeline every D
    // k-steps (8B verify pass 4.35 -> 4.26 ms).
    constexpr int D = (MT == 1) ? 4 : 3;   // bounded by the register file: no spills.  (Deeper, 5 or 6 k-steps, or the
    // loads of k-step j + D requested before the products of k-step j through one more buffer: measured, not faster.)
    constexpr int NSLOT = D;
    constexpr int LPS = 4 + 2 * MT;        // loads per k-step
    u32x4 wb[NSLOT][4], xhb[NSLOT][MT], xlb[NSLOT][MT];
    const int n = ks0 < ks1 ? (ks1 - ks0 + KSTEP - 1) / KSTEP : 0;   // this wave's k-steps: ks0, ks0 + 8, ...
    // RMSNorm factors of the input rows: their sums of squares were finished by the previous kernel, so they are
    // requested first and turned into factors once the first k-step has arrived, instead of as a dependent round
    // trip inside the epilogue.  Thread (row, j) = (tidx >> 4, tidx & 15) holds the groups j, j + 16, ...
    constexpr bool RSTD_EARLY = EPI != EPI_RESID;
    constexpr int RSQ = 4;                 // sums per thread: ncg_in <= 64 (the host sees to it)
    float sq[MT][RSQ];
    const int nsq = RSTD_EARLY ? (a.ncg_in + 15) >> 4 : 0;
    if (RSTD_EARLY) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const float *sp = a.ssq_in + (size_t)((z * MT + mt) * 32 + (tidx >> 4)) * a.ncg_in;
#pragma unroll
            for (int i = 0; i < RSQ; ++i)
                if (i < nsq) load4_async(sq[mt][i], sp + min((tidx & 15) + 16 * i, a.ncg_in - 1));
        }
    }
    auto request = [&](int sl, int ks) {   // sl is a constant once the callers' loops are unrolled
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            if (WSTREAM) load16_stream_async(wb[sl][nb], wp + nb * wstride + (size_t)ks * 64);
            else load16_async(wb[sl][nb], wp + nb * wstride + (size_t)ks * 64);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            load16_async(xhb[sl][mt], xh[mt] + (size_t)ks * 64);
            load16_async(xlb[sl][mt], xl[mt] + (size_t)ks * 64);
        }
    };
#pragma unroll
    for (int dd = 0; dd < D; ++dd)
        if (dd < n) request(dd, ks0 + KSTEP * dd);
    for (int j0 = 0; j0 < n; j0 += NSLOT) {
#pragma unroll
        for (int dd = 0; dd < NSLOT; ++dd) {
            const int j = j0 + dd;
            if (j < n) {
                // loads requested after those of k-step j: the k-steps up to j + D - 1
                wait_steps<LPS>(min(D - 1, n - 1 - j));
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) tie(wb[dd][nb]);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) { tie(xhb[dd][mt]); tie(xlb[dd][mt]); }
                if (RSTD_EARLY && j == 0) {   // the sums of squares were requested before every k-step: they are here
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        float ssum = 0.f;
#pragma unroll
                        for (int i = 0; i < RSQ; ++i)
                            if (i < nsq) { tie(sq[mt][i]); if ((tidx & 15) + 16 * i < a.ncg_in) ssum += sq[mt][i]; }
#pragma unroll
                        for (int off = 1; off < 16; off <<= 1) ssum += shx(ssum, off);
                        if ((tidx & 15) == 0) s_rstd[32 * mt + (tidx >> 4)] = rsqrtf(ssum / (float)a.d_in + a.eps);
                    }
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb) {
                        acc[mt][nb] = mfma32(xhb[dd][mt], wb[dd][nb], acc[mt][nb]);
                        acc[mt][nb] = mfma32(xlb[dd][mt], wb[dd][nb], acc[mt][nb]);
                    }
                if (j + D < n) request(dd, ks0 + KSTEP * (j + D));
            }
        }
    }
    if (RSTD_EARLY && n == 0) {   // a wave without k-steps (short K ranges) still owes its rows' factors
        wait_loads<0>();
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float ssum = 0.f;
#pragma unroll
            for (int i = 0; i < RSQ; ++i)
                if (i < nsq) { tie(sq[mt][i]); if ((tidx & 15) + 16 * i < a.ncg_in) ssum += sq[mt][i]; }
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) ssum += shx(ssum, off);
            if ((tidx & 15) == 0) s_rstd[32 * mt + (tidx >> 4)] = rsqrtf(ssum / (float)a.d_in + a.eps);
        }
    }

    gemm_stamp(a, lin, 1);
    // sum the 8 waves, then either finish (S == 1) or hand the partial tile over
    float hreg[8];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int ct = z * MT + mt;
        if (mt > 0) __syncthreads();
        if (EPI == EPI_RESID && S == 1) resid_prefetch(a, hreg, cg, ct);
        reduce_waves_to_tile(acc[mt], red, tile, w, lane);
        if (S == 1) {
            run_epilogue<EPI, RSTD_EARLY>(a, tile, s_rstd + 32 * mt, red, hreg, cg, ct);
        } else {
            float *out = a.part + ((size_t)s * a.rows_total + (size_t)ct * 32) * N + (size_t)cg * CG;
#pragma unroll
            for (int i = 0; i < 2; ++i) {   // 16 bytes per lane: a wave writes two rows of the group's 128 columns
                const int e = tidx + 512 * i;
                const int row = e >> 5, c4 = (e & 31) * 4;
                const float *tp = tile + row * RED_STRIDE + c4;
                store16_agent(out + (size_t)row * N + c4, tp[0], tp[1], tp[2], tp[3]);
            }
        }
    }
    gemm_stamp(a, lin, 2);
    if (S == 1) return;
    // the block that arrives last at this column group's counter sums all partials and finishes
    const bool last = arrive_last(a.counters + (size_t)z * ncg + cg, S, &sm.last);
    gemm_stamp(a, lin, 3);
    if (!last) {
        // (sm.red is free: every wave has passed the barrier behind the wave sum)
        if (EPI == EPI_QKV) prefetch_kv(a.kv.k, a.kv.vt, a.kv.head_stride, a.Hkv, a.kv_fetch_bytes, sm.red);
        else prefetch_next(a.nx, sm.red);
        return;
    }
    gemm_finish<MT, EPI, RSTD_EARLY>(a, sm, cg, z);
    gemm_stamp(a, lin, 4);
}

template <int MT, int EPI>
__global__ __launch_bounds__(512) void k_gemm(const GemmArgs a) {
    __shared__ GemmSmem sm;
    gemm_block<MT, EPI>(a, sm, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.x);
}

// The same GEMM over Z > 1 row-tile groups (batched passes, prefill chunks): every group needs the same weights.
// 1-D grid; workgroup ids 8 apart run on the same XCD at about the same time, so the Z workgroups of one
// (column group, K split) pair p get the ids 8 * ((p / 8) * Z + z) + p % 8: the first of them to ask for a
// weight line fetches it from memory, the others find it in that XCD's L2.
template <int MT, int EPI>
__global__ __launch_bounds__(512) void k_gemm_rows(const GemmArgs a, int ncg, int Z) {
    __shared__ GemmSmem sm;
    const int lin = blockIdx.x, x = lin & 7, q = lin >> 3;
    const int z = q % Z, p = 8 * (q / Z) + x;
    if (p < ncg * a.S) gemm_block<MT, EPI, false>(a, sm, p % ncg, p / ncg, z, ncg);
}

// ------------------------------------------------------------------------------------------
// mixture-of-experts FFN: (row, expert) pairs are grouped per expert, every touched expert's weights
// are streamed once, and the 8 weighted expert outputs of a row are summed in routing order.
// ------------------------------------------------------------------------------------------
// Unsplit GEMMs of a small model in narrow workgroups: NB = 1 (32 columns) for the residual GEMM (O projection),
// NB = 2 (64 columns: whole heads of up to 64 channels) for the QKV projection.
// A 128-column workgroup pulls all of K for four weight blocks and both activation planes through one compute
// unit's L1 (343 KB at K = 896, 64 bytes per clock), and a matrix of 896 columns gives only 7 of them per row
// tile: the launch is bound by those few L1s, then by one SIMD's 112 products and a 128 KB sum through LDS.  Here a
// workgroup owns NB 32-column weight blocks (171 KB through its L1 for one block, 28 products per SIMD, a 32 KB
// sum), and four (two) times as many compute units take part.  Same operand layouts, same order of summation over
// the waves (w = 0..7) and over a wave's k-steps (w, w + 8, ...) as in the wide kernel.
// grid: 1-D, ids 8 apart on one XCD: the Z row tiles of column group p get the ids 8 * ((p / 8) * Z + z) + p % 8.
// Sums of squares are written per 32-column block (GemmArgs::ssq_sub == 4 for every kernel of that model).
// ------------------------------------------------------------------------------------------
template <int NB>
struct GemmNarrowSmem {
    float red[8 * NB * 4 * 64 * 4];   // [wave][register quad][lane][4]
    float tile[32 * (32 * NB + 1)];
    float ssp[2 * 32];
    float rstd[32];
};

template <int NB, int EPI>
__global__ __launch_bounds__(512) void k_gemm_narrow(const GemmArgs a, int ngrp, int Z) {
    static_assert((EPI == EPI_RESID && NB == 1) || (EPI == EPI_QKV && NB == 2), "epilogues exist for these two forms");
    constexpr int TS = 32 * NB + 1;   // row stride of the tile in LDS
    __shared__ GemmNarrowSmem<NB> sm;
    const int lin = blockIdx.x, x8 = lin & 7, q8 = lin >> 3;
    const int z = q8 % Z, p = 8 * (q8 / Z) + x8;
    if (p >= ngrp) return;
    const int tidx = opaque_tid();
    const int w = __builtin_amdgcn_readfirstlane(tidx >> 6), lane = tidx & 63;
    const int N = a.N, KS = a.KS;
    const int t = z;
    const int slin = z * ngrp + p;   // stamps: 0 start, 1 this wave's k-steps multiplied, 2 epilogue done
    gemm_stamp(a, slin, 0);
    const uint4 *wp = a.W + (size_t)(p * NB) * KS * 64 + lane;
    const size_t wstride = (size_t)KS * 64;   // between column blocks
    const uint4 *xh = a.Xhi + (size_t)t * KS * 64 + lane, *xl = a.Xlo + (size_t)t * KS * 64 + lane;
    constexpr int D = NB == 1 ? 8 : 7;   // k-steps of loads in flight per wave (K = 896: all seven of a wave at once)
    uint4 wb[D][NB], xhb[D], xlb[D];
#pragma unroll
    for (int dd = 0; dd < D; ++dd) {
        const int ks = w + 8 * dd;
        if (ks < KS) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) wb[dd][nb] = wp[nb * wstride + (size_t)ks * 64];
            xhb[dd] = xh[(size_t)ks * 64]; xlb[dd] = xl[(size_t)ks * 64];
        }
    }
    float hreg[2];   // RESID: old h of this thread's elements e = tidx + 512 i: row e >> 5, column e & 31
    if (EPI == EPI_RESID) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = tidx + 512 * i;
            hreg[i] = a.h[(size_t)(t * 32 + (e >> 5)) * N + p * 32 + (e & 31)];
        }
    } else {   // RMSNorm factors of the input rows, requested behind the first operands
        tile_rstd(a.ssq_in, sm.rstd, t * 32, a.ncg_in, a.d_in, a.eps);
    }
    f32x16 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nb][r] = 0.f;
    for (int kb = w; kb < KS; kb += 8 * D) {
#pragma unroll
        for (int dd = 0; dd < D; ++dd) {
            const int ks = kb + 8 * dd;
            if (ks < KS) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    acc[nb] = mfma32(xhb[dd], wb[dd][nb], acc[nb]);
                    acc[nb] = mfma32(xlb[dd], wb[dd][nb], acc[nb]);
                }
                const int kn = ks + 8 * D;
                if (kn < KS) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) wb[dd][nb] = wp[nb * wstride + (size_t)kn * 64];
                    xhb[dd] = xh[(size_t)kn * 64]; xlb[dd] = xl[(size_t)kn * 64];
                }
            }
        }
    }
    float qpre[QKV_PRE];
    if (EPI == EPI_QKV) qkv_prefetch<32 * NB>(a, qpre, p, t);
    gemm_stamp(a, slin, 1);
    // sum of the 8 waves in the order w = 0..7: wave s < 4 NB sums register quad s & 3 of block s >> 2 and writes
    // its rows 8 q + 4 half + 0..3
    float4 *red4 = (float4 *)sm.red;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            red4[(w * 4 * NB + nb * 4 + q) * 64 + lane] = make_float4(acc[nb][4 * q], acc[nb][4 * q + 1], acc[nb][4 * q + 2], acc[nb][4 * q + 3]);
    __syncthreads();
    if (w < 4 * NB) {
        float4 sum = red4[w * 64 + lane];
#pragma unroll
        for (int ww = 1; ww < 8; ++ww) {
            const float4 v = red4[(ww * 4 * NB + w) * 64 + lane];
            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        float *tp = sm.tile + (8 * (w & 3) + 4 * (lane >> 5)) * TS + (w >> 2) * 32 + (lane & 31);
        tp[0] = sum.x; tp[TS] = sum.y; tp[2 * TS] = sum.z; tp[3 * TS] = sum.w;
    }
    __syncthreads();
    if (EPI == EPI_QKV) {
        epi_qkv<32 * NB, TS, true>(a, sm.tile, sm.rstd, p, t, qpre);
    } else {
        // h += y; new fragment planes of h; sums of squares of the block's 32 columns
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = tidx + 512 * i;
            const int row = e >> 5, col = e & 31;
            const float v = hreg[i] + sm.tile[row * TS + col];
            a.h[(size_t)(t * 32 + row) * N + p * 32 + col] = v;
            sm.tile[row * TS + col] = v;
        }
        __syncthreads();
        if (tidx < 128) {   // (row, octet) items: wave 0 has octets 0 and 1, wave 1 octets 2 and 3
            const int row = tidx & 31, oct = tidx >> 5;
            const float *tp = sm.tile + row * TS + oct * 8;
            uint4 hi, lo;
            pack8_split(tp, hi, lo);
            const size_t v = (size_t)t * (N / 16) * 64 + frag_vec(row, p * 4 + oct);
            a.xhi_out[v] = hi;
            a.xlo_out[v] = lo;
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) ss += tp[e] * tp[e];
            ss += shx(ss, 32);
            if ((tidx & 63) < 32) sm.ssp[(tidx >> 6) * 32 + row] = ss;
        }
        __syncthreads();
        if (tidx < 32) a.ssq_out[(size_t)(t * 32 + tidx) * (N / 32) + p] = sm.ssp[tidx] + sm.ssp[32 + tidx];
    }
    gemm_stamp(a, slin, 2);
}

// ------------------------------------------------------------------------------------------
// Streaming GEMM in small workgroups, for passes of few row tiles: one row tile, C = 1 or 2 column blocks of 32, one of S
// shares of K.  Same loop as gemm_block (eight waves take the k-steps w, w + 8, ... of the share; sums over the waves in the
// order w = 0..7, over the shares s = 0..S-1), but what follows the stream is a quarter or half as long: the wave sum moves
// 32 KB per block through LDS instead of 128 KB, a share's partial tile is 4 KB per block, kept in the register layout so
// that it needs no LDS tile on its way, and the residual epilogue works on registers.
// What bounds a launch: about 6 us of start, exchange and epilogue (4.7 without shares), and behind that HBM (6.5 TB/s) or
// what one compute unit draws, 60 to 75 KB per microsecond of weights and activations together as long as the weights come
// from HBM (the estimate takes 62).  So: as many workgroups as compute units, each with few bytes; the host picks C and S
// (plan_slim).  One row tile, microseconds against k_gemm.  Launched alone, back to back with rotating weights: O 4096 x 4096
// 13.2 -> 11.0, 4096 x 2560 12.4 -> 9.4, 4096 x 2048 11.9 -> 8.6; down 9728 x 2560 18.1 -> 14.0, 4864 x 896 11.7 -> 7.4
// (12288 x 4096: 22.3 and 21.6); QKV 2048 x 5120 11.9 -> 9.3, gate/up 896 x 9728 10.4 -> 7.9.  In a pass at full depth: 8B O
// 12.5 -> 11.3, down 24.5 -> 23.5 (QKV 17.4 and 17.7: nothing gained there), 4B O 11.7 -> 9.9, down 19.8 -> 16.1, QKV one
// microsecond, drafter gate/up 11.5 -> 9.1, down 12.4 -> 9.0.
// grid: 1-D; with P = s * ngrp + p, the Z row tiles of (column group p, share s) get the ids 8 * ((P / 8) * Z + z) + P % 8
// (one XCD).  Sums of squares are written per 32 C columns (GemmArgs::ssq_sub == 4 / C).
// ------------------------------------------------------------------------------------------
template <int C>
struct GemmSlimSmem {
    float4 red[8][C * 4][64];          // [wave][block, register quad][lane]
    float tile[32 * (32 * C + 4)];     // QKV, SWIGLU: the finished tile, row-major
    float rstd[32];
    int last;
};

template <int C, int EPI>
__global__ __launch_bounds__(512) void k_gemm_slim(const GemmArgs a, int ngrp, int Z, int pairs) {
    static_assert(EPI == EPI_RESID || C == 2, "QKV and gate/up need both blocks of a pair");
    constexpr int TS = 32 * C + 4;     // row stride of the tile in LDS
    constexpr int D = C == 1 ? 6 : 4, LPS = C + 2;   // k-steps in flight per wave, loads per k-step
    __shared__ GemmSlimSmem<C> sm;
    const int lin = blockIdx.x, q8 = lin >> 3;
    const int S = a.S, z = q8 % Z, P = 8 * (q8 / Z) + (lin & 7);
    if (P >= ngrp * S) return;
    const int s = P / ngrp, p = P - s * ngrp;
    const int tidx = opaque_tid();
    const int w = __builtin_amdgcn_readfirstlane(tidx >> 6), lane = tidx & 63, half = lane >> 5, cl = lane & 31;
    const int N = a.N, KS = a.KS;
    const int slin = P * Z + z;        // stamps as in gemm_block
    gemm_stamp(a, slin, 0);
    const int per = (KS + S * 8 - 1) / (S * 8);
    const int ks0 = s * 8 * per + w, ks1 = min(KS, (s + 1) * 8 * per);
    const int n = ks0 < ks1 ? (ks1 - ks0 + 7) >> 3 : 0;   // this wave's k-steps: ks0, ks0 + 8, ...
    const uint4 *wp[C];
#pragma unroll
    for (int j = 0; j < C; ++j) wp[j] = a.W + (size_t)slim_block(p, C, pairs, j) * KS * 64 + lane;
    const uint4 *xh = a.Xhi + (size_t)z * KS * 64 + lane, *xl = a.Xlo + (size_t)z * KS * 64 + lane;
    // RMSNorm factors of the input rows, requested first (see gemm_block): thread (row, j) = (tidx >> 4, tidx & 15)
    constexpr bool RSTD = EPI != EPI_RESID;
    constexpr int RSQ = 4;
    float sq[RSQ];
    const int nsq = RSTD ? (a.ncg_in + 15) >> 4 : 0;
    if (RSTD) {
        const float *sp = a.ssq_in + (size_t)(z * 32 + (tidx >> 4)) * a.ncg_in;
#pragma unroll
        for (int i = 0; i < RSQ; ++i)
            if (i < nsq) load4_async(sq[i], sp + min((tidx & 15) + 16 * i, a.ncg_in - 1));
    }
    auto store_rstd = [&] {   // the sums of squares have arrived
        float ssum = 0.f;
#pragma unroll
        for (int i = 0; i < RSQ; ++i)
            if (i < nsq) { tie(sq[i]); if ((tidx & 15) + 16 * i < a.ncg_in) ssum += sq[i]; }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) ssum += shx(ssum, off);
        if ((tidx & 15) == 0) sm.rstd[tidx >> 4] = rsqrtf(ssum / (float)a.d_in + a.eps);
    };
    u32x4 wb[D][C], xhb[D], xlb[D];
    auto request = [&](int sl, int ks) {   // sl is a constant once the callers' loops are unrolled
#pragma unroll
        for (int j = 0; j < C; ++j) load16_stream_async(wb[sl][j], wp[j] + (size_t)ks * 64);
        load16_async(xhb[sl], xh + (size_t)ks * 64);
        load16_async(xlb[sl], xl + (size_t)ks * 64);
    };
    // A wave sums D k-steps in a chain of their own and adds them to acc.  It has up to three times the k-steps that a wave of
    // the wide kernel has (whose workgroups are fewer and whose shares more), and what a chain of additions rounds off grows
    // with the square root of its length.  Error of the rows against 64 bits, wide kernel / one chain / this: 12288 x 4096 over
    // one row tile 1.10e-7 / 1.29e-7 / 0.98e-7, 4096 x 4096 over two 0.99e-7 / 1.09e-7 / 0.89e-7, 4864 x 896 0.97e-7 each (5
    // k-steps per wave).
    f32x16 acc[C], zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
    for (int j = 0; j < C; ++j) acc[j] = zero;
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < n) request(d, ks0 + 8 * d);
    for (int j0 = 0; j0 < n; j0 += D) {
        f32x16 sum[C];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int j = j0 + d;
            if (j < n) {
                wait_steps<LPS, D - 1>(min(D - 1, n - 1 - j));   // loads requested after those of k-step j
#pragma unroll
                for (int q = 0; q < C; ++q) tie(wb[d][q]);
                tie(xhb[d]); tie(xlb[d]);
                if (RSTD && j == 0) store_rstd();
#pragma unroll
                for (int q = 0; q < C; ++q) sum[q] = mfma32(xhb[d], wb[d][q], d == 0 ? zero : sum[q]);
#pragma unroll
                for (int q = 0; q < C; ++q) sum[q] = mfma32(xlb[d], wb[d][q], sum[q]);
                if (j + D < n) request(d, ks0 + 8 * (j + D));
            }
        }
#pragma unroll
        for (int q = 0; q < C; ++q) acc[q] += sum[q];
    }
    if (RSTD && n == 0) { wait_loads<0>(); store_rstd(); }   // a wave without k-steps still owes its rows' factors
    gemm_stamp(a, slin, 1);
    // Wave w < 4 C finishes register quad w & 3 of block w >> 2: column cl of the block, rows 8 quad + 4 half .. + 3
    const bool mine = w < 4 * C;
    const int blk = slim_block(p, C, pairs, min(w >> 2, C - 1)), quad = w & 3, row0 = 8 * quad + 4 * half;
    float *hp = a.h + (size_t)(z * 32 + row0) * N + blk * 32 + cl;   // RESID
    float hv[4] = {0.f, 0.f, 0.f, 0.f};
    if (EPI == EPI_RESID && mine)
#pragma unroll
        for (int e = 0; e < 4; ++e) hv[e] = hp[(size_t)e * N];
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) sm.red[w][j * 4 + q][lane] = make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
    barrier_keep_loads();
    float y[4] = {0.f, 0.f, 0.f, 0.f};
    if (mine) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = sm.red[u][w][lane];
        y[0] = v[0].x; y[1] = v[0].y; y[2] = v[0].z; y[3] = v[0].w;
#pragma unroll
        for (int u = 1; u < 8; ++u) { y[0] += v[u].x; y[1] += v[u].y; y[2] += v[u].z; y[3] += v[u].w; }
    }
    if (S > 1) {
        float *pt = a.part + (size_t)(p * Z + z) * S * (1024 * C) + (w * 64 + lane) * 4;   // [share][wave][lane][4]
        if (mine) store16_agent(pt + (size_t)s * (1024 * C), y[0], y[1], y[2], y[3]);
        const bool last = arrive_last(a.counters + p * Z + z, S, &sm.last);
        gemm_stamp(a, slin, 3);
        if (!last) {   // (sm.red has been read: every wave has passed arrive_last's barriers)
            if (EPI == EPI_QKV) prefetch_kv(a.kv.k, a.kv.vt, a.kv.head_stride, a.Hkv, a.kv_fetch_bytes, sm.red);
            else prefetch_next(a.nx, sm.red);
            return;
        }
        if (mine) {
            u32x4 v[8];   // at most eight shares, all requested together
#pragma unroll
            for (int u = 0; u < 8; ++u) load16_agent_async(v[u], pt + (size_t)min(u, S - 1) * (1024 * C));
            wait_loads<0>();
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                tie(v[u]);
                if (u < S)
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] += __uint_as_float(v[u][e]);
            }
        }
    }
    if (EPI == EPI_RESID) {
        if (C == 1 && !mine) return;   // (C == 2: every wave has a quad)
        // h += y; new fragment planes of h (two bytes per lane: eight lanes make an octet); sums of squares of the block
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v = hv[e] + y[e];
            hp[(size_t)e * N] = v;
            const uint32_t hi = f2bf(v), lo = f2bf(v - bf2f(hi));
            const size_t at = ((size_t)z * (N / 16) * 64 + frag_vec(row0 + e, blk * 4 + (cl >> 3))) * 8 + (cl & 7);
            ((uint16_t *)a.xhi_out)[at] = (uint16_t)hi;
            ((uint16_t *)a.xlo_out)[at] = (uint16_t)lo;
            float ss = v * v;
            ss += dppf<0xB1>(ss); ss += dppf<0x4E>(ss); ss += dppf<0x141>(ss); ss += dppf<0x140>(ss);
            ss += shx(ss, 16);
            if (cl == 0) {
                if (C == 1) a.ssq_out[(size_t)(z * 32 + row0 + e) * (N / 32) + p] = ss;
                else sm.tile[(w >> 2) * 32 + row0 + e] = ss;
            }
        }
        if (C == 2) {   // both blocks' sums in one
            barrier_keep_loads();
            if (tidx < 32) a.ssq_out[(size_t)(z * 32 + tidx) * (N / 64) + p] = sm.tile[tidx] + sm.tile[32 + tidx];
        }
    } else {
        if (mine)
#pragma unroll
            for (int e = 0; e < 4; ++e) sm.tile[(row0 + e) * TS + (w >> 2) * 32 + cl] = y[e];
        __syncthreads();
        if (tidx >= (EPI == EPI_QKV ? 256 : 128)) return;
        const int row = tidx & 31, oct = tidx >> 5;
        const float sc = sm.rstd[row];
        const float *x = sm.tile + row * TS + oct * 8;
        float v[8];
        uint4 hi, lo;
        if (EPI == EPI_SWIGLU) {   // block 0: 32 gate channels, block 1: their up channels; the group's other 32 are its neighbour's
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float g = x[e] * sc, u = x[32 + e] * sc;
                v[e] = g / (1.f + expf(-g)) * u;
            }
            pack8_split(v, hi, lo);
            const size_t vec = (size_t)z * (a.F / 16) * 64 + frag_vec(row, p * 4 + oct);
            a.ahi[vec] = hi;
            a.alo[vec] = lo;
        } else {
            const int hd = a.hd, Hq = a.Hq, Hkv = a.Hkv, half_hd = hd >> 1, grow = z * 32 + row;
            const int col0 = slim_block(p, C, pairs, oct >> 2) * 32 + (oct & 3) * 8;   // first of 8 columns, all in one head
            const int kind = col0 < Hq * hd ? 0 : (col0 < (Hq + Hkv) * hd ? 1 : 2);
            const int hc = col0 - (kind == 0 ? 0 : (kind == 1 ? Hq * hd : (Hq + Hkv) * hd));
            const int head = hc / hd, i0 = hc % hd;
            if (kind < 2) {
                const int po = hd == 32 ? 16 : 32;   // the rotation partner's distance in the tile: half a head, or the other block of a 128-wide head
                const float *xp = x + (i0 < half_hd ? po : -po);
                const float2 *cs = a.cs + (size_t)grow * half_hd + (i0 < half_hd ? i0 : i0 - half_hd);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float2 c = cs[e];
                    const float xe = x[e] * sc, xq = xp[e] * sc;
                    v[e] = (i0 < half_hd) ? xe * c.x - xq * c.y : xe * c.x + xq * c.y;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = x[e] * sc;
            }
            if (kind == 0) {
                pack8_split(v, hi, lo);
                const int qr = a.rm.qrow[grow];
                if (qr >= 0) {
                    const size_t vec = ((size_t)((qr >> 5) * Hq + head) * (hd / 16)) * 64 + frag_vec(qr & 31, i0 >> 3);
                    a.qhi[vec] = hi;
                    a.qlo[vec] = lo;
                }
            } else {
                const int slot = a.rm.slot[grow];
                if (slot >= 0) {
                    const size_t base = (size_t)a.rm.seq[grow] * a.kv.seq_stride + (size_t)head * a.kv.head_stride;
                    if (kind == 1) *(uint4 *)(a.kv.k + base + k_cache_off(slot, i0 >> 3, hd)) = pack8(v);
                    else
#pragma unroll
                        for (int e = 0; e < 8; ++e) a.kv.vt[base + v_cache_off(slot, i0 + e, hd)] = (uint16_t)f2bf(v[e]);
                }
            }
        }
    }
    gemm_stamp(a, slin, S > 1 ? 4 : 2);
}

// ------------------------------------------------------------------------------------------
// One block: pairs: pair i of expert e is 8 * (pass row) + (its routing slot); items: [0].x the number of work items of up to
// item_pairs (32 or 64) pairs, from [1] on (expert, first pair, pairs, first 32-pair activation tile) of each.
// One row per thread and trip: a pass of 2048 rows takes two trips of eight LDS atomics per thread.
__global__ __launch_bounds__(1024) void k_moe_group(const int *__restrict__ route_e, const int *__restrict__ row_slot,
                                                    int rows, int top_k, int cap, int item_pairs, int *__restrict__ pairs,
                                                    int4 *__restrict__ items, unsigned long long *__restrict__ touched_total) {
    __shared__ int s_cnt[128];   // experts beyond the model's: 0
    const int tid = threadIdx.x;
    if (tid < 128) s_cnt[tid] = 0;
    __syncthreads();
    for (int row = tid; row < rows; row += 1024) {
        if (row_slot[row] < 0) continue;                 // unused rows of a tile route nowhere
        const int4 e0 = *(const int4 *)(route_e + row * 8), e1 = *(const int4 *)(route_e + row * 8 + 4);
        const int ev[8] = {e0.x, e0.y, e0.z, e0.w, e1.x, e1.y, e1.z, e1.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j >= top_k) break;
            const int e = ev[j];
            const int i = atomicAdd(&s_cnt[e], 1);       // order inside an expert does not affect results
            pairs[e * cap + i] = row * 8 + j;
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    // lane l: experts 2 l and 2 l + 1; running sums of their tiles (low half) and items (high half) over the lanes
    const int n[2] = {s_cnt[2 * tid], s_cnt[2 * tid + 1]};
    const int sh = item_pairs == 32 ? 5 : 6;
    auto load = [&](int v) { return ((v + 31) >> 5) + (((v + item_pairs - 1) >> sh) << 16); };
    int at = load(n[0]) + load(n[1]);
    const int own = at;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(at, off);
        if (tid >= off) at += v;
    }
    if (tid == 63) items[0].x = at >> 16;
    at -= own;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        for (int j = 0; j << sh < n[i]; ++j)
            items[1 + (at >> 16) + j] = make_int4(2 * tid + i, j << sh, min(item_pairs, n[i] - (j << sh)), (at & 0xffff) + (j << sh >> 5));
        at += load(n[i]);
    }
    // running count of (layer, expert) pairs whose weights a pass has to stream (for byte accounting)
    const int touched = __popcll(__ballot(n[0] > 0)) + __popcll(__ballot(n[1] > 0));
    if (tid == 0) atomicAdd(touched_total, (unsigned long long)touched);
}

enum { MOE_GATEUP = 0, MOE_DOWN = 1 };

struct MoeArgs {
    const uint4 *W; size_t wexp_stride;      // expert e's matrix at W + e * wexp_stride (16-byte units)
    const uint4 *Xhi, *Xlo;                  // GATEUP: the pass's fragments of h; DOWN: activation tiles
    int N, KS, cap;
    const int *pairs; const int4 *items;     // see k_moe_group
    int eighths;                             // k_gemm_moe: sums in eighths of K instead of folded as in block_loop
    const float *ssq_in; int ncg_in, d_in; float eps;   // GATEUP: RMSNorm scale of each pair's row
    uint4 *ahi, *alo; int Fe;                // GATEUP out: the item's activation tiles, Fe/16 k-steps
    const float *route_w; float *moe_out; int d;        // DOWN out: moe_out[row][slot][d] = w * y
};

// h += sum over the row's experts in routing order; new fragment planes and sums of squares of h
__global__ __launch_bounds__(256) void k_moe_combine(const float *__restrict__ moe_out, const int *__restrict__ row_slot,
                                                     int top_k, float *__restrict__ h, uint4 *__restrict__ xhi,
                                                     uint4 *__restrict__ xlo, float *__restrict__ ssq, int d) {
    __shared__ float tile[32 * RED_STRIDE];
    const int cg = blockIdx.x, t = blockIdx.y, ncg = gridDim.x;
    // 1024 float4 elements of the 32 x 128 tile, four per thread; all loads of a thread are requested before
    // the first is used (the expert outputs of a row are summed in routing order, then added to h)
    float4 hv[4], mv[4][8];
    bool live[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e4 = threadIdx.x + 256 * i, row = e4 >> 5, c4 = (e4 & 31) * 4;
        const int grow = t * 32 + row;
        live[i] = row_slot[grow] >= 0;
        hv[i] = *(const float4 *)(h + (size_t)grow * d + cg * CG + c4);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            mv[i][j] = (live[i] && j < top_k) ? *(const float4 *)(moe_out + ((size_t)grow * 8 + j) * d + cg * CG + c4)
                                              : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e4 = threadIdx.x + 256 * i, row = e4 >> 5, c4 = (e4 & 31) * 4;
        float4 add = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int j = 0; j < 8; ++j) { add.x += mv[i][j].x; add.y += mv[i][j].y; add.z += mv[i][j].z; add.w += mv[i][j].w; }
        float4 v = hv[i];
        if (live[i]) { v.x += add.x; v.y += add.y; v.z += add.z; v.w += add.w; }
        *(float4 *)(h + (size_t)(t * 32 + row) * d + cg * CG + c4) = v;
        float *tp = tile + row * RED_STRIDE + c4;
        tp[0] = v.x; tp[1] = v.y; tp[2] = v.z; tp[3] = v.w;
    }
    __syncthreads();
    tile_to_frag(tile, xhi, xlo, (size_t)t * (d / 16) * 64, cg * CG);
    {   // sum of squares of a row's 128 columns: 8 threads per row, 16 columns each, then a fixed butterfly
        const int row = threadIdx.x >> 3, sub = threadIdx.x & 7;
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < 16; ++c) { const float v = tile[row * RED_STRIDE + sub * 16 + c]; s += v * v; }
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) s += shx(s, off);
        if (sub == 0) ssq[(size_t)(t * 32 + row) * ncg + cg] = s;
    }
}

struct RowResult {   // per LM row
    int argmax;      // lowest index of the max logit
    int sample;      // Gumbel-max sample of softmax(z/T) (T > 0), else = argmax
    float lse;       // log sum exp(z/T) (T > 0), else 0
    float zmax;
};

// one block per LM row: merge the per-group partials
// draft != null (the drafter's pass): the row's token goes there, and the last row of a sequence counts the tokens that the pass
// took in.
// Latency: one workgroup per row, one round trip for its column groups' results (up to RS_HELD of them per thread stay in
// registers for the sum of exponentials), waves merged by shuffles.
constexpr int RS_HELD = 8;
__global__ __launch_bounds__(256) void k_rowstat_final(const RowStat *__restrict__ stat, int ncg_v, float T,
                                                       RowResult *__restrict__ res, int k, int k_lo, SeqState st, int *__restrict__ draft) {
    __shared__ float sm[4], sg[4], ss[4]; __shared__ int si[4], sgi[4];
    const int row = blockIdx.x, tid = threadIdx.x, w = tid >> 6;
    if (draft && tid == 64 && row % k == k - 1) { const int b = row / k; st.dr_len[b] += st.ing_n[b]; st.ing_n[b] = 0; }
    if (row % k < k_lo) return;   // kept from an earlier pass
    const RowStat *p = stat + (size_t)row * ncg_v;
    float m = -INFINITY, gm = -INFINITY; int idx = 0x7fffffff, gidx = 0x7fffffff;
    RowStat v[RS_HELD];
#pragma unroll
    for (int i = 0; i < RS_HELD; ++i) {
        const int g = tid + 256 * i;
        if (g < ncg_v) v[i] = p[g];
        else v[i] = RowStat{-INFINITY, 0x7fffffff, 0.f, -INFINITY, 0x7fffffff};
    }
#pragma unroll
    for (int i = 0; i < RS_HELD; ++i) { argmax_merge(m, idx, v[i].m, v[i].idx); argmax_merge(gm, gidx, v[i].gm, v[i].gidx); }
    for (int g = tid + 256 * RS_HELD; g < ncg_v; g += 256) {
        argmax_merge(m, idx, p[g].m, p[g].idx);
        argmax_merge(gm, gidx, p[g].gm, p[g].gidx);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float m2 = shx(m, off), g2 = shx(gm, off); const int i2 = shx(idx, off), gi2 = shx(gidx, off);
        argmax_merge(m, idx, m2, i2);
        argmax_merge(gm, gidx, g2, gi2);
    }
    if ((tid & 63) == 0) { sm[w] = m; si[w] = idx; sg[w] = gm; sgi[w] = gidx; }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) { argmax_merge(m, idx, sm[j], si[j]); argmax_merge(gm, gidx, sg[j], sgi[j]); }
    float se = 0.f;
    if (T > 0.f) {
        const float invT = 1.f / T;
#pragma unroll
        for (int i = 0; i < RS_HELD; ++i)
            if (tid + 256 * i < ncg_v) se += v[i].sumexp * expf((v[i].m - m) * invT);
        for (int g = tid + 256 * RS_HELD; g < ncg_v; g += 256) se += p[g].sumexp * expf((p[g].m - m) * invT);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) se += shx(se, off);
        if ((tid & 63) == 0) ss[w] = se;
        __syncthreads();
        se = (ss[0] + ss[1]) + (ss[2] + ss[3]);
    }
    if (tid == 0) {
        RowResult r;
        const int V = ncg_v * CG;
        r.argmax = (idx >= 0 && idx < V) ? idx : 0;   // a row of NaNs never updates the index
        r.zmax = m;
        if (T > 0.f) { r.sample = (gidx >= 0 && gidx < V) ? gidx : 0; r.lse = m / T + logf(se); }
        else { r.sample = r.argmax; r.lse = 0.f; }
        res[row] = r;
        if (draft) draft[row] = r.sample;
    }
}

// ------------------------------------------------------------------------------------------
// block attention for short query blocks over a long GQA cache.
//   Online softmax in fp32.  S^T = K Q^T and O^T = V^T P^T: every MFMA operand is a contraction-contiguous
//   16-byte vector and the softmax row of a lane is its own column.  Key order inside a 32-key tile is
//   permuted (operand row rho holds key 16*((rho/4)%2) + 4*(rho/8) + rho%4) so that a lane's 16 scores are
//   16 consecutive keys.  Q and P enter as (hi, lo) bf16 pairs.
//   With one key range (NS == 1) the result goes straight to the O-projection's input fragments; otherwise
//   each (tile, head, split) leaves an un-normalised partial (M, L, O) in the MFMA register layout and a
//   separate merge combines them (a merge by the last split to finish would serialise NS dependent round
//   trips to memory on one workgroup).
// ------------------------------------------------------------------------------------------
template <int HD>
struct AttnPartial {   // per (tile, head, split): O in register layout [HD/32][4 register quads][64 lanes][4], then (M, L)[32]
    static constexpr int FLOATS = 32 * HD + 64;
};

// o: O^T of one head, scaled by inv, into the output projection's input; grow: the GEMM row of this lane's query row, < 0: none
template <int HD>
__device__ __forceinline__ void attn_write_frag(const f32x16 *o, float inv, int grow, int head, int Hq, int lane,
                                                uint4 *__restrict__ xhi, uint4 *__restrict__ xlo) {
    // lane (qrow, half) holds dims 32*tt + 8*q + 4*half + 0..3 in regs 4q..4q+3; the partner lane (other
    // half) holds the other 4 dims of the octet.  Half 0 writes octets with even q, half 1 odd q.
    const int half = lane >> 5;
    const int KS = Hq * HD / 16;
#pragma unroll
    for (int tt = 0; tt < HD / 32; ++tt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float mine[4], other[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                mine[e] = o[tt][4 * q + e] * inv;
                other[e] = shx(mine[e], 32);
            }
            // octet (tt, q): dims 32*tt + 8*q + 0..7 = half-0 lane's 4 values then half-1 lane's 4 values
            if ((q & 1) == half && grow >= 0) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[e] = half ? other[e] : mine[e]; v[4 + e] = half ? mine[e] : other[e]; }
                uint4 hi, lo;
                pack8_split(v, hi, lo);
                const size_t vec = (size_t)(grow >> 5) * KS * 64 + frag_vec(grow & 31, head * (HD / 8) + tt * 4 + q);
                xhi[vec] = hi;
                xlo[vec] = lo;
            }
        }
}

// ------------------------------------------------------------------------------------------
// Block attention of passes of many row tiles or long key ranges: one (row tile, up to four query heads of a kv head, key
// range) item per workgroup of four waves, two workgroups per compute unit.
//  - wave = query head: every key tile of the range goes through all four waves, so that a tile's K and V fragments are
//    fetched once per workgroup.  They land in LDS in fragment order (direct-to-LDS loads, no registers held while they
//    travel), two tiles at a time: one pair is on its way while the other is multiplied, with one barrier per pair;
//  - a pair shares one softmax step (one maximum over 64 keys, one rescale of O), and the products of its two tiles, and of
//    the O^T tiles, are interleaved chains;
//  - Q fragments stay in registers;
//  - the two workgroups of a compute unit share nothing and drift apart, so that the products of one run under the softmax
//    of the other;
//  - the result goes to the output projection's input (NS == 1) or to an un-normalised partial (M, L, O) for the merge.
// Bound: the chain products -> softmax -> products of two waves per SIMD, at the clock that is left when matrix cores and
// HBM are both busy (counted: 1.84 GHz and the matrix pipe busy 58 % of a long-context launch).  Microseconds per launch
// against one workgroup of eight waves, two per head, behind one barrier: 8B heads, 16 sequences x 32768 keys 560 -> 531
// (4.0 TB/s of K and V), prompt of 4096 341 -> 268, batch of prompts (104 tiles) 73 -> 53; drafter, prompt of 4096
// 138 -> 96.  A ring of four single tiles took 544 and 290 (drafter 114).  Tiles of fewer than 32 rows skip the mask and the
// rescale like full ones (16 sequences x 8192 keys, 31 / 16 / 4 rows: 162 / 158 / 139 -> 153 / 153 / 132; 32 rows: 154).
// ------------------------------------------------------------------------------------------
#ifndef DEER_ATT_P_LO
#define DEER_ATT_P_LO 1
#endif
constexpr bool ATT_P_LO = DEER_ATT_P_LO != 0;   // the low-order bf16 plane of the softmax weights enters P V
constexpr int ATT_HEADS = 4;                    // query heads per workgroup
template <int HD>
struct AttnSmem {
    static constexpr int FPT = HD / 8;   // fragments of 1 KB per key tile (K k-steps, then V (tile, half) pairs)
    uint4 buf[2][2][FPT * 64];           // two pairs of key tiles
};

// grid: x = kv_head + Hkv * (group of four heads + HG * split), y = pass tile counted from the last (prompts: the longest
// key ranges start first); 256 threads
template <int HD>
__global__ __launch_bounds__(256, 2) void k_attn(const uint4 *__restrict__ Qhi, const uint4 *__restrict__ Qlo,
                                                 const uint16_t *__restrict__ Kc, const uint16_t *__restrict__ Vt,
                                                 size_t seq_stride, size_t head_stride,
                                                 const int *__restrict__ tile_seq, const int *__restrict__ row_limit,
                                                 const int *__restrict__ row_grow, float *__restrict__ part, int Hq, int Hkv, int HG, int NS, float scale_log2e,
                                                 uint4 *__restrict__ xhi, uint4 *__restrict__ xlo) {
    using SM = AttnSmem<HD>;
    constexpr int KSQ = HD / 16, HT = HD / 32, FPT = SM::FPT, LPW = FPT / 4;
    constexpr int PF = AttnPartial<HD>::FLOATS;
    __shared__ __attribute__((aligned(16))) SM as;
    const int tidx = opaque_tid();
    const int w = __builtin_amdgcn_readfirstlane(tidx >> 6), lane = tidx & 63;   // the wave index as a scalar
    const int half = lane >> 5, qrow = lane & 31;
    const int t = gridDim.y - 1 - blockIdx.y;
    const int kvh = blockIdx.x % opaque_s(Hkv), xr = blockIdx.x / opaque_s(Hkv), hg = xr % opaque_s(HG), split = xr / opaque_s(HG);
    const int G = Hq / opaque_s(Hkv), g = hg * ATT_HEADS + w;
    const bool active = g < G;
    const int head = kvh * G + min(g, G - 1);
    const int b = tile_seq[t], lim = row_limit[t * 32 + qrow];   // lim: the key limit of this lane's query row
    int maxlim = lim, minlim = lim > 0 ? lim : 0x7fffffff;   // rows that do not exist set no limit: their results, whatever they are, go nowhere
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
        maxlim = max(maxlim, shx(maxlim, off));
        minlim = min(minlim, shx(minlim, off));
    }
    maxlim = __builtin_amdgcn_readfirstlane(maxlim);
    minlim = __builtin_amdgcn_readfirstlane(minlim);
    const int nkt = (maxlim + 31) >> 5;
    const int per = (nkt + NS - 1) / opaque_s(NS);
    const int kt0 = split * per, n = max(0, min(nkt, kt0 + per) - kt0);
    const char *Kp = (const char *)(Kc + (size_t)b * seq_stride + (size_t)kvh * head_stride) + (size_t)kt0 * (64 * HD);
    const char *Vp = (const char *)(Vt + (size_t)b * seq_stride + (size_t)kvh * head_stride) + (size_t)kt0 * (64 * HD);
    // this wave's share of a key tile: fragments w LPW .. + LPW - 1, straight into LDS (lane l's 16 bytes land at base + 16 l).
    // Half of the waves fetch K, half V.  A pair's second tile past the range repeats the last one (finite values, weight 0).
    const char *src = (w < 2 ? Kp : Vp) + (w & 1) * LPW * 1024 + lane * 16;
    auto stage = [&](int buf, int pair) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const char *p = src + (size_t)min(2 * pair + j, n - 1) * (64 * HD);
#pragma unroll
            for (int f = 0; f < LPW; ++f)
                __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)(p + f * 1024),
                                                 (void __attribute__((address_space(3))) *)(as.buf[buf][j] + (w * LPW + f) * 64), 16, 0, 0);
        }
    };
    const uint32_t ring = lds_addr32(as.buf[0][0]) + lane * 16;
    f32x16 oacc[HT];
#pragma unroll
    for (int tt = 0; tt < HT; ++tt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[tt][r] = 0.f;
    // The lowest finite number, not -inf: a row that has seen no key yet keeps it as its maximum, with every weight exp2(-inf) = 0
    // and the factor of O exp2(0) = 1, so that it needs no case of its own and no rescale.
    float m_run = -3.4028234e38f, l_run = 0.f;
    if (n > 0) {
        const int np = (n + 1) >> 1;
        uint4 qh[KSQ], ql[KSQ];
        {   // this wave's Q fragments (requested first: every later wait covers them)
            const size_t qb = ((size_t)(t * Hq + head) * KSQ) * 64 + lane;
#pragma unroll
            for (int s = 0; s < KSQ; ++s) { qh[s] = Qhi[qb + (size_t)s * 64]; ql[s] = Qlo[qb + (size_t)s * 64]; }
        }
        stage(0, 0);
        for (int i = 0; i < np; ++i) {
            wait_loads<0>();
            barrier_keep_loads();   // every wave's share of pair i is in LDS, and pair i - 1 has been read by all
            if (i + 1 < np) stage((i + 1) & 1, i + 1);
            if (!active) continue;
            const uint32_t fr = ring + (i & 1) * (2 * FPT * 1024);
            // S^T of both tiles: one chain of products per tile, interleaved
            f32x16 sacc[2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) sacc[j][r] = 0.f;
            u32x4 kf[2][2][KSQ / 2];   // [half of the k-steps][tile]
            lds_frags<0>(kf[0][0], fr, std::make_integer_sequence<int, KSQ / 2>{});
            lds_frags<FPT * 1024>(kf[0][1], fr, std::make_integer_sequence<int, KSQ / 2>{});
            lds_frags<KSQ / 2 * 1024>(kf[1][0], fr, std::make_integer_sequence<int, KSQ / 2>{});
            lds_frags<FPT * 1024 + KSQ / 2 * 1024>(kf[1][1], fr, std::make_integer_sequence<int, KSQ / 2>{});
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                if (h2 == 0) wait_lds<KSQ>(); else wait_lds<0>();
#pragma unroll
                for (int s = 0; s < KSQ / 2; ++s) {
                    const int ss = h2 * (KSQ / 2) + s;
                    tie(kf[h2][0][s]); tie(kf[h2][1][s]);
                    sacc[0] = mfma32(kf[h2][0][s], qh[ss], sacc[0]);
                    sacc[1] = mfma32(kf[h2][1][s], qh[ss], sacc[1]);
                    sacc[0] = mfma32(kf[h2][0][s], ql[ss], sacc[0]);
                    sacc[1] = mfma32(kf[h2][1][s], ql[ss], sacc[1]);
                }
            }
            u32x4 vf[2 * HT];   // the first tile's V, on its way during the softmax
            lds_frags<KSQ * 1024>(vf, fr, std::make_integer_sequence<int, 2 * HT>{});
            // a lane holds keys kt*32 + 16*half + r, r = 0..15, of both tiles for query row qrow
            const int kt = kt0 + 2 * i, key0 = kt * 32 + 16 * half;
            const int lim1 = 2 * i + 1 < n ? lim : 0;   // the second tile of the last pair may lie past the range
            if (kt * 32 + 64 > minlim || 2 * i + 1 >= n) {   // only tiles that reach some row's limit need the mask
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    if (key0 + r >= lim) sacc[0][r] = -INFINITY;
                    if (key0 + 32 + r >= lim1) sacc[1][r] = -INFINITY;
                }
            }
            float mx = fmaxf(sacc[0][0], sacc[1][0]);
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(sacc[0][r], sacc[1][r]));
            mx = fmaxf(mx, shx(mx, 32));
            const float m_new = fmaxf(m_run, mx);
            const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2e);
            const float mb = m_new * scale_log2e;
            float ls0 = 0.f, ls1 = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sacc[0][r] = __builtin_amdgcn_exp2f(sacc[0][r] * scale_log2e - mb); ls0 += sacc[0][r];
                sacc[1][r] = __builtin_amdgcn_exp2f(sacc[1][r] * scale_log2e - mb); ls1 += sacc[1][r];
            }
            l_run = l_run * alpha + (ls0 + ls1);
            m_run = m_new;
            if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {   // the running max moved for some row
#pragma unroll
                for (int tt = 0; tt < HT; ++tt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[tt][r] *= alpha;
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float pr[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) pr[r] = sacc[j][r];
                uint4 ph[2], pl[2];
                pack8_split(pr, ph[0], pl[0]);
                pack8_split(pr + 8, ph[1], pl[1]);
                wait_lds<0>();
#pragma unroll
                for (int v = 0; v < 2 * HT; ++v) tie(vf[v]);
                // the O^T tiles' chains interleaved
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
#pragma unroll
                    for (int tt = 0; tt < HT; ++tt) oacc[tt] = mfma32(vf[tt * 2 + s2], ph[s2], oacc[tt]);
                    if (ATT_P_LO)
#pragma unroll
                        for (int tt = 0; tt < HT; ++tt) oacc[tt] = mfma32(vf[tt * 2 + s2], pl[s2], oacc[tt]);
                }
                if (j == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    lds_frags<(FPT + KSQ) * 1024>(vf, fr, std::make_integer_sequence<int, 2 * HT>{});
                }
            }
        }
    }
    if (!active) return;
    const float l_tot = l_run + shx(l_run, 32);
    if (NS == 1) {
        attn_write_frag<HD>(oacc, l_tot > 0.f ? 1.f / l_tot : 0.f, row_grow[t * 32 + qrow], head, Hq, lane, xhi, xlo);
    } else {
        float *pp = part + ((size_t)(t * Hq + head) * NS + split) * PF;
#pragma unroll
        for (int tt = 0; tt < HT; ++tt)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(float4 *)(pp + ((tt * 4 + q) * 64 + lane) * 4) = make_float4(oacc[tt][4 * q], oacc[tt][4 * q + 1], oacc[tt][4 * q + 2], oacc[tt][4 * q + 3]);
        if (half == 0) *(float2 *)(pp + 32 * HD + 2 * qrow) = make_float2(m_run, l_tot);
    }
}

// Writes registers 8*hh .. 8*hh+7 of O^T tile tt (held in o[0..7], scaled by inv) into the output projection's
// input fragments: octets q = 2*hh and 2*hh + 1 (see attn_write_frag for the lane pairing).
template <int HD>
__device__ __forceinline__ void attn_store_slice(const float (&o)[8], float inv, int Hq, int head, int grow, int tt, int hh,
                                                 int lane, uint4 *xhi, uint4 *xlo) {
    const int half = lane >> 5;
    const int KS = Hq * HD / 16;
#pragma unroll
    for (int qq = 0; qq < 2; ++qq) {
        const int q = 2 * hh + qq;
        float mine[4], other[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) { mine[e] = o[4 * qq + e] * inv; other[e] = shx(mine[e], 32); }
        if ((q & 1) == half && grow >= 0) {
            float v8[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) { v8[e] = half ? other[e] : mine[e]; v8[4 + e] = half ? mine[e] : other[e]; }
            uint4 hi, lo;
            pack8_split(v8, hi, lo);
            const size_t vec = (size_t)(grow >> 5) * KS * 64 + frag_vec(grow & 31, head * (HD / 8) + tt * 4 + q);
            store16_agent(xhi + vec, hi);
            store16_agent(xlo + vec, lo);
        }
    }
}

// Merge of the NS key-range partials that k_attn left: one wave per (tile, head, O^T tile tt, register half hh).  The (M, L)
// pairs and the first 16 partial outputs (two register quads of 1 KB per wave each) are requested together; ranges are
// combined in order s = 0..NS-1.  NS <= 32.  Producer and consumer are separated by a kernel boundary: plain 16-byte
// accesses (8-byte ones that bypass the L2, as between workgroups of one launch, took 20 us for 16 tiles x 32 heads x 4
// ranges).  grid: 256 threads = 4 wave items per block
template <int HD>
__global__ __launch_bounds__(256) void k_attn_merge(const float *__restrict__ part, const int *__restrict__ row_grow, int NS, int Hq, int n_items,
                                                    float scale_log2e, uint4 *__restrict__ xhi, uint4 *__restrict__ xlo) {
    constexpr int HT = HD / 32, PF = AttnPartial<HD>::FLOATS, CH = 16;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, qrow = lane & 31;
    if (j >= n_items) return;
    const int hh = j & 1, tt = (j >> 1) % HT, head = (j / (2 * HT)) % Hq, t = j / (2 * HT * Hq);
    const float *p0 = part + (size_t)(t * Hq + head) * NS * PF;
    const float4 *po = (const float4 *)(p0 + ((tt * 2 + hh) * 2 * 64 + lane) * 4);
    const int grow = row_grow[t * 32 + qrow];
    float4 v[CH][2];
    auto request = [&](int s0) {
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (s0 + u < NS) { v[u][0] = po[(size_t)(s0 + u) * (PF / 4)]; v[u][1] = po[(size_t)(s0 + u) * (PF / 4) + 64]; }
    };
    request(0);
    float f[32], M = -INFINITY, L = 0.f;
    {
        float2 ml[32];
#pragma unroll
        for (int s = 0; s < 32; ++s) ml[s] = s < NS ? *(const float2 *)(p0 + (size_t)s * PF + 32 * HD + 2 * qrow) : make_float2(-INFINITY, 0.f);
#pragma unroll
        for (int s = 0; s < 32; ++s) M = fmaxf(M, ml[s].x);
#pragma unroll
        for (int s = 0; s < 32; ++s) {
            f[s] = ml[s].x == -INFINITY ? 0.f : exp2f((ml[s].x - M) * scale_log2e);
            L += f[s] * ml[s].y;
        }
    }
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll
    for (int s0 = 0; s0 < 32; s0 += CH) {
        if (s0 >= NS) break;
        if (s0 > 0) request(s0);
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (s0 + u < NS) {
                o[0] += f[s0 + u] * v[u][0].x; o[1] += f[s0 + u] * v[u][0].y; o[2] += f[s0 + u] * v[u][0].z; o[3] += f[s0 + u] * v[u][0].w;
                o[4] += f[s0 + u] * v[u][1].x; o[5] += f[s0 + u] * v[u][1].y; o[6] += f[s0 + u] * v[u][1].z; o[7] += f[s0 + u] * v[u][1].w;
            }
    }
    attn_store_slice<HD>(o, L > 0.f ? 1.f / L : 0.f, Hq, head, grow, tt, hh, lane, xhi, xlo);
}

// Merge of the NS key-range partials of one (tile, head) written by attn_head_item: wave item (tt, hh) owns registers
// 8*hh .. 8*hh+7 of O^T tile tt, which a partial holds as two register quads of 1 KB per wave.  All (M, L) pairs and the
// outputs of the first 8 ranges (16 with head_dim <= 64) are requested together; ranges are combined in order s = 0..NS-1.
// NS <= MAX.  The merge is the tail of the launch and runs on one compute unit per head, so nothing is loaded or computed for
// ranges that do not exist (loads and factors for 32 ranges, whatever their number, made it 5.5 us behind the last arrival of
// 8), and up to 8 ranges have a short code of their own: its instructions come from the L2, as nothing on the compute unit has
// run them in this launch (3.9 us with the code for 32 ranges, 3.0 with this one; 8B heads, 129 key tiles: 17.2 -> 13.8 us
// from the launch's first workgroup to its last store).  (The factors come from the bare exp2 instruction, as in the key loop:
// one below 2^-126 is zero, beside the factor 1 of the range that holds the maximum.)
constexpr int ATT_HEAD_MAX_NS = 32, ATT_HEAD_NS = 16;   // key ranges per head; up to so many have all their (M, L) pairs in registers
template <int HD, int MAX>
__device__ __forceinline__ void attn_head_merge(const float *part, const int *row_grow, int NS, int Hq, float scale_log2e, uint4 *xhi, uint4 *xlo,
                                                int head, int t, int tt, int hh, int lane) {
    constexpr int PF = AttnPartial<HD>::FLOATS;
    const int qrow = lane & 31;
    const float *p0 = part + (size_t)(t * Hq + head) * NS * PF;
    const float *po = p0 + ((tt * 2 + hh) * 2 * 64 + lane) * 4;
    const int grow = row_grow[t * 32 + qrow];
    constexpr int CH = MAX > 8 && HD <= 64 ? 16 : 8;   // ranges whose outputs are requested together (registers: 8 per range)
    u32x4 v[CH][2];
    auto request = [&](int s0) {
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (s0 + u < NS) {
                load16_agent_async(v[u][0], po + (size_t)(s0 + u) * PF);
                load16_agent_async(v[u][1], po + (size_t)(s0 + u) * PF + 256);
            }
    };
    float f[MAX];
    float M = -INFINITY, L = 0.f;
    {
        float2 ml[MAX];
#pragma unroll
        for (int s = 0; s < MAX; ++s)
            if (s < NS) ml[s] = ld_agent2(p0 + (size_t)s * PF + 32 * HD + 2 * qrow);
        request(0);
#pragma unroll
        for (int s = 0; s < MAX; ++s)
            if (s < NS) M = fmaxf(M, ml[s].x);
#pragma unroll
        for (int s = 0; s < MAX; ++s)
            if (s < NS) {
                f[s] = ml[s].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((ml[s].x - M) * scale_log2e);
                L += f[s] * ml[s].y;
            }
    }
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll
    for (int s0 = 0; s0 < MAX; s0 += CH) {
        if (s0 < NS) {
            if (s0 > 0) request(s0);
            wait_loads<0>();
#pragma unroll
            for (int u = 0; u < CH; ++u)
                if (s0 + u < NS) {
                    tie(v[u][0]); tie(v[u][1]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        o[e] += f[s0 + u] * __uint_as_float(v[u][0][e]);
                        o[4 + e] += f[s0 + u] * __uint_as_float(v[u][1][e]);
                    }
                }
        }
    }
    attn_store_slice<HD>(o, L > 0.f ? 1.f / L : 0.f, Hq, head, grow, tt, hh, lane, xhi, xlo);
}

// The same for any number of ranges (few heads over long contexts), 8 at a time, with the sums so far rescaled in between: the
// code above for 32 ranges does not fit the registers.
template <int HD>
__device__ __forceinline__ void attn_head_merge_many(const float *part, const int *row_grow, int NS, int Hq, float scale_log2e, uint4 *xhi, uint4 *xlo,
                                                     int head, int t, int tt, int hh, int lane) {
    constexpr int PF = AttnPartial<HD>::FLOATS;
    const int qrow = lane & 31;
    const float *pm = part + (size_t)(t * Hq + head) * NS * PF + 32 * HD + 2 * qrow;
    const float *po = part + (size_t)(t * Hq + head) * NS * PF + ((tt * 2 + hh) * 2 * 64 + lane) * 4;
    float M = -INFINITY, L = 0.f, o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll 1
    for (int s0 = 0; s0 < NS; s0 += 8) {
        float2 ml[8];
        u32x4 v[8][2];
#pragma unroll
        for (int u = 0; u < 8; ++u) ml[u] = s0 + u < NS ? ld_agent2(pm + (size_t)(s0 + u) * PF) : make_float2(-INFINITY, 0.f);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < NS) {
                load16_agent_async(v[u][0], po + (size_t)(s0 + u) * PF);
                load16_agent_async(v[u][1], po + (size_t)(s0 + u) * PF + 256);
            }
        const float before = M;
#pragma unroll
        for (int u = 0; u < 8; ++u) M = fmaxf(M, ml[u].x);
        const float alpha = before == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((before - M) * scale_log2e);
        L *= alpha;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] *= alpha;
        wait_loads<0>();
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < NS) {
                const float f = ml[u].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((ml[u].x - M) * scale_log2e);
                L += f * ml[u].y;
                tie(v[u][0]); tie(v[u][1]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[e] += f * __uint_as_float(v[u][0][e]);
                    o[4 + e] += f * __uint_as_float(v[u][1][e]);
                }
            }
    }
    attn_store_slice<HD>(o, L > 0.f ? 1.f / L : 0.f, Hq, head, row_grow[t * 32 + qrow], tt, hh, lane, xhi, xlo);
}

// ------------------------------------------------------------------------------------------
// Block attention for passes of few row tiles (decoding: draft and verify passes of small batches), one
// (row tile, query head, key range) item per workgroup.  Against k_attn + k_attn_merge this spreads a pass of
// one tile over every compute unit with 8 key ranges instead of 32, so the partial results are a quarter as
// large, and needs no second kernel: the last workgroup of a head to arrive merges the ranges itself.
//  - All eight waves serve the same head; wave w takes the key tiles w, w + 8, ... of the range and keeps
//    its own running (m, l, O).  No barrier inside the key loop: a wave's tiles are its own.
//  - A wave has two key tiles on their way at any time: one lands in its private LDS slot (direct-to-LDS
//    loads, no registers while they travel), the next one in registers; tiles alternate between the two.
//  - Q (hi and lo planes of the head) is staged once in LDS and shared by the waves.
//  - The eight running states are combined through LDS (every wave parks its O in its own slot, then wave
//    (tt, hh) sums register group hh of O^T tile tt over the eight copies in wave order); with one key range
//    the result is final, otherwise it is this range's partial and the ranges meet at an arrival counter.
// The kv heads of the K/V cache are shared by the G query heads of a group through the L2 of their XCD:
// workgroup ids cycle through the kv heads first, so with 8 kv heads every XCD serves one of them.
// ------------------------------------------------------------------------------------------
template <int HD>
struct AttnHeadSmem {
    uint4 slot[8][(HD / 8) * 64];   // per wave: one key tile (K k-step fragments, then V^T fragments); later its parked O
    uint4 q[(HD / 8) * 64];         // Q fragments of the head: hi plane, then lo plane
    float2 ml[8 * 64];              // parked (m, l) per wave and lane
    int last;
};

template <int HD>
__device__ __forceinline__ void attn_head_item(const uint4 *Qhi, const uint4 *Qlo, const uint16_t *__restrict__ Kc,
                                               const uint16_t *__restrict__ Vt, size_t seq_stride, size_t head_stride,
                                               int b, int lim, const int *row_grow, float *part, int *counters, int Hq, int Hkv, int NS,
                                               float scale_log2e, uint4 *xhi, uint4 *xlo, AttnHeadSmem<HD> &as, int head,
                                               int split, int t, const NextWeights &nx) {
    constexpr int HT = HD / 32, KSQ = HD / 16, FPT = KSQ + 2 * HT;   // fragments (1 KB each) per key tile
    constexpr int PF = AttnPartial<HD>::FLOATS;
    const int tidx = opaque_tid();
    const int w = __builtin_amdgcn_readfirstlane(tidx >> 6), lane = tidx & 63;
    const int half = lane >> 5, qrow = lane & 31;
    int maxlim = lim, minlim = lim;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
        maxlim = max(maxlim, shx(maxlim, off));
        minlim = min(minlim, shx(minlim, off));
    }
    maxlim = __builtin_amdgcn_readfirstlane(maxlim);
    minlim = __builtin_amdgcn_readfirstlane(minlim);
    const int nkt = (maxlim + 31) >> 5;
    const int per = (nkt + NS - 1) / opaque_s(NS);
    const int kt0 = split * per, kt1 = min(nkt, kt0 + per);
    const int first = kt0 + w;                                  // this wave's tiles: first, first + 8, ...
    const int n = first < kt1 ? (kt1 - first + 7) >> 3 : 0;
    const int kvh = head / (Hq / opaque_s(Hkv));
    const uint16_t *Kp = Kc + (size_t)b * seq_stride + (size_t)kvh * head_stride;
    const uint16_t *Vp = Vt + (size_t)b * seq_stride + (size_t)kvh * head_stride;
    uint4 *myslot = as.slot[w];

    // fragment f of key tile kt as this lane reads it: K k-step f, or V^T (O^T tile, key half) pair f - KSQ
    auto frag_src = [&](int kt, int f) -> const uint16_t * {   // both caches hold a key tile as HD / 16 fragments of 1 KB
        int lo8 = lane * 8;
        asm volatile("" : "+v"(lo8));
        if (f < KSQ) return Kp + (lo8 + kt * (32 * HD) + f * 512);
        return Vp + (lo8 + kt * (32 * HD) + (f - KSQ) * 512);
    };
    auto issue_lds = [&](int kt) {
#pragma unroll
        for (int f = 0; f < FPT; ++f)
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)frag_src(kt, f),
                                             (void __attribute__((address_space(3))) *)(myslot + f * 64), 16, 0, 0);
    };
    u32x4 rf[FPT];   // the key tile that travels in registers
    auto issue_reg = [&](int kt) {
#pragma unroll
        for (int f = 0; f < FPT; ++f) load16_async(rf[f], frag_src(kt, f));
    };

    // Q first (every later wait covers it), then this wave's first two key tiles, the second behind the barrier
    {
        const size_t qb = ((size_t)(t * Hq + head) * KSQ) * 64 + lane;
        for (int f = w; f < 2 * KSQ; f += 8) {
            const uint4 *src = f < KSQ ? Qhi + qb + (size_t)f * 64 : Qlo + qb + (size_t)(f - KSQ) * 64;
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src,
                                             (void __attribute__((address_space(3))) *)(as.q + f * 64), 16, 0, 0);
        }
    }
    // (the second tile behind the barrier: a compute unit's loads return in the order of their requests, and the waves' second
    // tiles, 128 KB, would stand in front of the last waves' shares of Q)
    if (n > 0) issue_lds(first);
    if (n > 0) wait_loads<FPT>(); else wait_loads<0>();
    barrier_keep_loads();   // Q of every wave's share is in LDS
    if (n > 1) issue_reg(first + 8);

    f32x16 oacc[HT];
#pragma unroll
    for (int tt = 0; tt < HT; ++tt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[tt][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const uint4 *qf = as.q + lane;

    // one key tile: S^T = K Q^T, running softmax, O^T += V^T P^T; FROM_LDS: fragments from the slot, else from rf
    auto tile = [&](auto from_lds, int kt) {
        constexpr bool FROM_LDS = decltype(from_lds)::value;
        const uint4 *fr = myslot + lane;
        f32x16 sacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[r] = 0.f;
#pragma unroll
        for (int s = 0; s < KSQ; ++s) {
            const uint4 qh = qf[s * 64], ql = qf[(KSQ + s) * 64];
            if (FROM_LDS) {
                const uint4 kf = fr[s * 64];
                sacc = mfma32(kf, qh, sacc);
                sacc = mfma32(kf, ql, sacc);
            } else {
                sacc = mfma32(rf[s], qh, sacc);
                sacc = mfma32(rf[s], ql, sacc);
            }
        }
        const int key0 = kt * 32 + 16 * half;   // lane holds keys key0 + r, r = 0..15, for query row qrow
        if (kt * 32 + 32 > minlim) {            // only tiles that reach some row's limit need the mask
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (key0 + r >= lim) sacc[r] = -INFINITY;
        }
        float mx = sacc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sacc[r]);
        mx = fmaxf(mx, shx(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        float pr[16];
        if (m_new == -INFINITY) {
#pragma unroll
            for (int r = 0; r < 16; ++r) pr[r] = 0.f;
        } else {
            const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2e);   // m_run = -inf -> 0
            const float mb = m_new * scale_log2e;
            float ls = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) { pr[r] = __builtin_amdgcn_exp2f(sacc[r] * scale_log2e - mb); ls += pr[r]; }
            l_run = l_run * alpha + ls;
            m_run = m_new;
            if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {   // the running max moved for some row
#pragma unroll
                for (int tt = 0; tt < HT; ++tt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[tt][r] *= alpha;
            }
        }
        uint4 ph[2], pl[2];
        pack8_split(pr, ph[0], pl[0]);
        pack8_split(pr + 8, ph[1], pl[1]);
#pragma unroll
        for (int tt = 0; tt < HT; ++tt)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                if (FROM_LDS) {
                    const uint4 vf = fr[(KSQ + tt * 2 + s2) * 64];
                    oacc[tt] = mfma32(vf, ph[s2], oacc[tt]);
                    if (ATT_P_LO) oacc[tt] = mfma32(vf, pl[s2], oacc[tt]);
                } else {
                    oacc[tt] = mfma32(rf[KSQ + tt * 2 + s2], ph[s2], oacc[tt]);
                    if (ATT_P_LO) oacc[tt] = mfma32(rf[KSQ + tt * 2 + s2], pl[s2], oacc[tt]);
                }
            }
    };

    // loads return in order: Q, tile 0 (LDS), tile 1 (registers), tile 2 (LDS, requested after tile 0 was used), ...
    for (int i = 0; i < n; i += 2) {
        if (i + 1 < n) wait_loads<FPT>(); else wait_loads<0>();
        tile(std::true_type{}, first + 8 * i);
        if (i + 2 < n) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read
            issue_lds(first + 8 * (i + 2));
        }
        if (i + 1 < n) {
            if (i + 2 < n) wait_loads<FPT>(); else wait_loads<0>();
#pragma unroll
            for (int f = 0; f < FPT; ++f) tie(rf[f]);
            tile(std::false_type{}, first + 8 * (i + 1));
            if (i + 3 < n) issue_reg(first + 8 * (i + 3));
        }
    }

    // park (m, l) and O; the slot is this wave's own, its loads have landed and its reads are done
    const float l_tot = l_run + shx(l_run, 32);
    as.ml[w * 64 + lane] = make_float2(m_run, l_tot);
    {
        float4 *ox = (float4 *)myslot;
#pragma unroll
        for (int tt = 0; tt < HT; ++tt)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ox[(tt * 4 + q) * 64 + lane] = make_float4(oacc[tt][4 * q], oacc[tt][4 * q + 1], oacc[tt][4 * q + 2], oacc[tt][4 * q + 3]);
    }
    __syncthreads();
    if (w < 2 * HT) {   // wave (tt, hh): registers 8*hh .. 8*hh+7 of O^T tile tt, summed over the waves in order
        const int tt = w >> 1, hh = w & 1;
        float2 ml[8];
        float M = -INFINITY, L = 0.f, f[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) { ml[u] = as.ml[u * 64 + lane]; M = fmaxf(M, ml[u].x); }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            f[u] = (ml[u].x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((ml[u].x - M) * scale_log2e);
            L += f[u] * ml[u].y;
        }
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float4 *ox = (const float4 *)as.slot[u];
            const float4 a0 = ox[(tt * 4 + 2 * hh) * 64 + lane], a1 = ox[(tt * 4 + 2 * hh + 1) * 64 + lane];
            o[0] += f[u] * a0.x; o[1] += f[u] * a0.y; o[2] += f[u] * a0.z; o[3] += f[u] * a0.w;
            o[4] += f[u] * a1.x; o[5] += f[u] * a1.y; o[6] += f[u] * a1.z; o[7] += f[u] * a1.w;
        }
        if (NS == 1) {
            attn_store_slice<HD>(o, L > 0.f ? 1.f / L : 0.f, Hq, head, row_grow[t * 32 + qrow], tt, hh, lane, xhi, xlo);
        } else {
            // this range's partial: O as [(tt, hh)][register quad j][lane][4] (a wave writes 1 KB at a time), then
            // (M, L)[32 rows]
            float *pp = part + ((size_t)(t * Hq + head) * NS + split) * PF;
            store16_agent(pp + (((tt * 2 + hh) * 2 + 0) * 64 + lane) * 4, o[0], o[1], o[2], o[3]);
            store16_agent(pp + (((tt * 2 + hh) * 2 + 1) * 64 + lane) * 4, o[4], o[5], o[6], o[7]);
            if (w == 0 && half == 0) st_agent2(pp + 32 * HD + 2 * qrow, M, L);
        }
    }
    if (NS == 1) return;
    // the key range that arrives last at the head's counter merges all of them
    if (!arrive_last(counters + t * Hq + head, NS, &as.last)) { prefetch_next(nx, as.slot); return; }
    if (w >= 2 * HT) return;
    if (NS <= 8) attn_head_merge<HD, 8>(part, row_grow, NS, Hq, scale_log2e, xhi, xlo, head, t, w >> 1, w & 1, lane);
    else if (NS <= ATT_HEAD_NS) attn_head_merge<HD, ATT_HEAD_NS>(part, row_grow, NS, Hq, scale_log2e, xhi, xlo, head, t, w >> 1, w & 1, lane);
    else attn_head_merge_many<HD>(part, row_grow, NS, Hq, scale_log2e, xhi, xlo, head, t, w >> 1, w & 1, lane);
}

// grid: x = kv_head + Hkv * (head in group + G * split), y = pass tile; 512 threads
template <int HD>
__global__ __launch_bounds__(512) void k_attn_head(const uint4 *__restrict__ Qhi, const uint4 *__restrict__ Qlo,
                                                   const uint16_t *__restrict__ Kc, const uint16_t *__restrict__ Vt,
                                                   size_t seq_stride, size_t head_stride,
                                                   const int *__restrict__ tile_seq, const int *__restrict__ row_limit,
                                                   const int *__restrict__ row_grow, float *__restrict__ part, int *__restrict__ counters, int Hq, int Hkv,
                                                   int NS, float scale_log2e, uint4 *__restrict__ xhi,
                                                   uint4 *__restrict__ xlo, const NextWeights nx) {
    __shared__ __attribute__((aligned(16))) AttnHeadSmem<HD> as;
    const int t = blockIdx.y;
    const int G = Hq / Hkv, kvh = blockIdx.x % Hkv, r = blockIdx.x / Hkv;
    attn_head_item<HD>(Qhi, Qlo, Kc, Vt, seq_stride, head_stride, tile_seq[t], row_limit[t * 32 + (threadIdx.x & 31)], row_grow, part,
                       counters, Hq, Hkv, NS, scale_log2e, xhi, xlo, as, kvh * G + r % G, r / G, t, nx);
}

// ------------------------------------------------------------------------------------------
// acceptance and commit, one block per sequence
// ------------------------------------------------------------------------------------------
struct AcceptOut { int *accept_len, *n_committed, *committed; };   // [B], [B], [B][k + bonus]: written, never read (page-locked host memory, or the workspace where there is none)

// bonus = 1: the target pass had k + 1 rows and `corr` is also the extra token after k accepted drafts
__device__ __forceinline__ void commit_tokens(SeqState st, AcceptOut out, int b, int k, int a, int corr, const int *d,
                                              int eos, int bonus) {
    // thread 0 only
    const int cs = k + bonus;
    int n = (a < k) ? a + 1 : cs;
    int fin = 0, tok = corr;
    for (int i = 0; i < n; ++i) {
        tok = (i < a) ? d[i] : corr;
        out.committed[b * cs + i] = tok;
        st.ing_tok[b * 32 + i] = tok;
        if (eos >= 0 && tok == eos) { n = i + 1; fin = 1; break; }
    }
    out.accept_len[b] = a;
    out.n_committed[b] = n;
    st.ing_n[b] = n;
    st.len[b] += n;
    st.pending[b] = tok;
    if (fin) st.finished[b] = 1;
}

// T = 0: accept while the draft equals the target's argmax; the first mismatch is replaced by it; with the
// bonus token on, k matches are followed by the argmax of row k
__global__ void k_accept_greedy(SeqState st, AcceptOut out, const int *__restrict__ draft,
                                const RowResult *__restrict__ tres, int k, int eos, int bonus) {
    const int b = blockIdx.x;
    if (threadIdx.x != 0) return;
    if (st.finished[b]) { out.accept_len[b] = 0; out.n_committed[b] = 0; return; }
    const int *d = draft + b * k;
    const int kt = k + bonus;
    int a = k, corr = bonus ? tres[b * kt + k].argmax : -1;
    for (int i = 0; i < k; ++i) {
        int tgt = tres[b * kt + i].argmax;
        if (d[i] != tgt) { a = i; corr = tgt; break; }
    }
    commit_tokens(st, out, b, k, a, corr, d, eos, bonus);
}

// T > 0: u_i <= min(1, p_i(y^_i) / q_i(y^_i)) in log space, stop at the first rejection and draw the
// replacement from max(0, p_i - q_i) by Gumbel-max (falls back to p_i when the residual is empty).
// With the bonus token on, k acceptances are followed by a draw from p_{k+1} (a residual without a draft:
// the same generator stream at position j + k, weights p).
// Grid (sequence, ACC_NB): every workgroup repeats the k tests (cheap), then scans its share of the vocabulary
// row; the candidates of the ACC_NB shares meet through memory and the workgroup that arrives last picks the
// winner (largest perturbed weight, lowest index on ties: the same token whatever the split) and commits.
// The kernel reads nothing that it writes before all shares have arrived: the committed length j comes from
// the verify pass's row metadata (the sequence's first row sits at position j - 1), every share arrives
// on every path (finished sequence, all k drafts accepted, a draw), and only the last arrival touches the
// per-sequence state and resets the counter.
constexpr int ACC_NB = 32;
struct AccPart { float best; int bi; float bestp; int bpi; int any; int pad[3]; };

__global__ __launch_bounds__(1024) void k_accept_sample(SeqState st, AcceptOut out, const int *__restrict__ draft,
                                                        const RowResult *__restrict__ tres,
                                                        const RowResult *__restrict__ dres,
                                                        const float *__restrict__ tlogits,
                                                        const float *__restrict__ dlogits, int k, int V, float T,
                                                        uint64_t seed, int eos, int bonus, AccPart *parts, int *arrivals,
                                                        const int *__restrict__ verify_pos) {
    __shared__ int s_a, s_last;
    __shared__ float sv[1024]; __shared__ int sx[1024];
    __shared__ float sv2[1024]; __shared__ int sx2[1024]; __shared__ int s_any[1024];
    const int b = blockIdx.x, nb = gridDim.y, part = blockIdx.y;
    const bool finished = st.finished[b] != 0;   // written only by the last arrival, after this read
    const int *d = draft + b * k;
    const int kt = k + bonus;           // target rows per sequence
    const int j = verify_pos[b * kt] + 1;
    const float invT = 1.f / T;
    if (threadIdx.x < 64) {   // the k tests at once (each has its own uniform and rows), then the first rejection
        const int i = threadIdx.x;
        int rej = k;
        if (i < k && !finished) {
            const size_t rt = (size_t)b * kt + i, rd = (size_t)b * k + i;
            const int y = d[i];
            const float logp = tlogits[rt * V + y] * invT - tres[rt].lse;
            const float logq = dlogits[rd * V + y] * invT - dres[rd].lse;
            const float u = uniform01(row_key(seed, TAG_ACCEPT, (uint64_t)b, (uint64_t)(j + i)), 0);
            if (!(logf(u) <= fminf(0.f, logp - logq))) rej = i;
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) rej = min(rej, shx(rej, off));
        if (i == 0) s_a = rej;
    }
    __syncthreads();
    const int a = s_a;
    const bool draw = !finished && (a < k || bonus);   // a token has to be drawn (k accepted drafts without the extra token: nothing to draw)
    if (draw) {
        const bool has_q = a < k;       // a drafted token stands at this position
        const size_t rt = (size_t)b * kt + a, rd = (size_t)b * k + (has_q ? a : 0);
        const float lt = tres[rt].lse, ld = has_q ? dres[rd].lse : 0.f;
        const uint64_t key = row_key(seed, TAG_RESID, (uint64_t)b, (uint64_t)(j + a));
        float best = -INFINITY, bestp = -INFINITY; int bi = 0x7fffffff, bpi = 0x7fffffff, any = 0;
        const int share = (V + nb - 1) / nb, v0 = part * share, v1 = min(V, v0 + share);
        for (int v = v0 + threadIdx.x; v < v1; v += 1024) {
            const float logp = tlogits[rt * V + v] * invT - lt;
            const float gn = gumbel(key, (uint64_t)v);
            if (has_q) {
                const float logq = dlogits[rd * V + v] * invT - ld;
                const float diff = expf(logp) - expf(logq);
                if (diff > 0.f) { any = 1; argmax_merge(best, bi, logf(diff) + gn, v); }
            }
            argmax_merge(bestp, bpi, logp + gn, v);
        }
        s_any[threadIdx.x] = any; sv[threadIdx.x] = best; sx[threadIdx.x] = bi; sv2[threadIdx.x] = bestp; sx2[threadIdx.x] = bpi;
        __syncthreads();
        for (int off = 512; off > 0; off >>= 1) {
            if (threadIdx.x < off) {
                s_any[threadIdx.x] |= s_any[threadIdx.x + off];
                argmax_merge(sv[threadIdx.x], sx[threadIdx.x], sv[threadIdx.x + off], sx[threadIdx.x + off]);
                argmax_merge(sv2[threadIdx.x], sx2[threadIdx.x], sv2[threadIdx.x + off], sx2[threadIdx.x + off]);
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            AccPart *pp = parts + (size_t)b * nb + part;
            __hip_atomic_store(&pp->best, sv[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&pp->bi, sx[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&pp->bestp, sv2[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&pp->bpi, sx2[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&pp->any, s_any[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (!arrive_last(arrivals + b, nb, &s_last)) return;
    if (threadIdx.x != 0) return;
    if (finished) { out.accept_len[b] = 0; out.n_committed[b] = 0; return; }
    int corr = -1;
    if (draw) {
        int any_all = 0;
        for (int p = 0; p < nb; ++p) any_all |= __hip_atomic_load(&parts[(size_t)b * nb + p].any, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        float wv = -INFINITY; int wi = 0x7fffffff;
        for (int p = 0; p < nb; ++p) {
            const AccPart *pp = parts + (size_t)b * nb + p;
            const float cv = __hip_atomic_load(any_all ? &pp->best : &pp->bestp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int ci = __hip_atomic_load(any_all ? &pp->bi : &pp->bpi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            argmax_merge(wv, wi, cv, ci);
        }
        corr = (wi >= 0 && wi < V) ? wi : 0;   // all-NaN rows never update the index
    }
    commit_tokens(st, out, b, k, a, corr, d, eos, bonus);
}

// Test aid: the caller's tokens are committed in place of the acceptance rule's choice.  One thread per sequence;
// n[b] tokens tok[b * stride ..] (n[b] = 0: nothing).  Same state updates as commit_tokens.
__global__ void k_force_commit(SeqState st, const int *__restrict__ tok, const int *__restrict__ n, int stride, int eos, int B) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int nb = n[b];
    if (nb <= 0) { st.ing_n[b] = 0; return; }
    int fin = 0;
    for (int i = 0; i < nb; ++i) {
        const int t = tok[b * stride + i];
        st.ing_tok[b * 32 + i] = t;
        if (eos >= 0 && t == eos) fin = 1;
    }
    st.ing_n[b] = nb;
    st.len[b] += nb;
    st.pending[b] = tok[b * stride + nb - 1];
    if (fin) st.finished[b] = 1;
}

// Test aid: canonical K and V rows [n][kv_head][head_dim] (bf16) into cache slots first .. first + n - 1 of one
// sequence and layer.  One thread per (slot, head, channel octet).
__global__ void k_load_kv(const uint16_t *__restrict__ krows, const uint16_t *__restrict__ vrows, KvView kv, int b, int first,
                          int n, int Hkv, int hd) {
    const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int octs = hd >> 3;
    if (gid >= (size_t)n * Hkv * octs) return;
    const int oct = (int)(gid % octs), head = (int)((gid / octs) % Hkv), r = (int)(gid / ((size_t)octs * Hkv));
    const int slot = first + r;
    const size_t src = ((size_t)r * Hkv + head) * hd + oct * 8;
    const size_t base = (size_t)b * kv.seq_stride + (size_t)head * kv.head_stride;
    *(uint4 *)(kv.k + base + k_cache_off(slot, oct, hd)) = *(const uint4 *)(krows + src);
#pragma unroll
    for (int e = 0; e < 8; ++e) kv.vt[base + v_cache_off(slot, oct * 8 + e, hd)] = vrows[src + e];
}

}  // namespace deer
